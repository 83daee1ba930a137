// C ABI of the cmlbm library: handle management, host-side validation, buffer
// alternation and error reporting. Device work lives in kernels.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>

#include "../../include/cmlbm.h"
#include "kernels.hpp"
#include "rules.hpp"

struct cmlbm_lattice {
    cm::LaunchArgs a;
    void* buf[2];
    int cur;             // index of the buffer holding the current state
    size_t bytes_each;
    double* scratch;     // reduction partials
    double* result;      // host memory that the device writes the 8 reduced values to (ResultSlots)
    void* stress[2];     // sub-grid stress buffers (caller-owned); stress[k] pairs with buf[k]
    size_t stress_bytes;
    int device;          // device current at creation (the handle's work runs there)
};

namespace {

thread_local std::string g_err = "no error";

cmlbm_status fail(cmlbm_status s, const std::string& msg) {
    g_err = msg;
    return s;
}

cmlbm_status hip_fail(hipError_t e, const char* where) {
    g_err = std::string(where) + ": " + hipGetErrorString(e);
    return CMLBM_EHIP;
}

size_t elem_size(int storage) {
    switch (storage) {
        case CMLBM_F64: return 8;
        case CMLBM_F32: return 4;
        case CMLBM_F32_SHIFTED: return 4;
        case CMLBM_F16_SHIFTED: return 2;
        default: return 0;
    }
}

// Bytes of the compute type (force field, sub-grid stress, adjoint arrays).
size_t compute_size(int storage) { return storage == CMLBM_F64 ? 8 : 4; }

// Largest per-lane byte offset, plus one element, that the kernels form within
// one grid row. Every kernel addresses an element as a workgroup-uniform row
// pointer plus a per-lane 32-bit byte offset: up to three consecutive
// population rows of the internal layout (the three e_x of a gather or an odd
// in-place push, 3 nx elements of the storage type), or one row of a
// compute-type array (force field, sub-grid stress, adjoint arrays). Offsets
// must not wrap, so this span must stay below 2^32.
uint64_t lane_span(int32_t nx, int storage) {
    const uint64_t n = (uint64_t)(nx > 0 ? nx : 0);
    const uint64_t pop = 3 * n * (uint64_t)elem_size(storage), cmp = n * (uint64_t)compute_size(storage);
    return pop > cmp ? pop : cmp;
}

// Populations per cell of the lattice model.
int lattice_q(int lattice) { return lattice == CMLBM_D2Q9 ? 9 : 27; }

bool rate_ok(double w) { return std::isfinite(w) && w > 0.0 && w < 2.0; }

// Host memory that devices write reduced values to: 64 slots of 8 doubles in one
// page, allocated with the first handle and held until the process ends (an
// allocation for each handle made its creation 0.1 ms longer); handles beyond
// the 64th get memory of their own.
class ResultSlots {
public:
    hipError_t take(double** out) {
        std::lock_guard<std::mutex> lock(mu_);
        if (!page_) {
            const hipError_t e = hipHostMalloc((void**)&page_, 64 * kBytes, hipHostMallocPortable);
            if (e != hipSuccess) return e;
        }
        for (int k = 0; k < 64; ++k)
            if (!(used_ >> k & 1u)) {
                used_ |= (uint64_t)1 << k;
                *out = page_ + 8 * k;
                return hipSuccess;
            }
        return hipHostMalloc((void**)out, kBytes, hipHostMallocPortable);
    }
    hipError_t give_back(double* p) {
        std::lock_guard<std::mutex> lock(mu_);
        if (page_ && p >= page_ && p < page_ + 8 * 64) {
            used_ &= ~((uint64_t)1 << ((p - page_) / 8));
            return hipSuccess;
        }
        return hipHostFree(p);
    }

private:
    static constexpr size_t kBytes = 8 * sizeof(double);
    std::mutex mu_;
    double* page_ = nullptr;
    uint64_t used_ = 0;
};
ResultSlots g_results;

cmlbm_status check_handle(cmlbm_handle h) {
    if (!h) return fail(CMLBM_EINVAL, "null handle");
    return CMLBM_OK;
}

cmlbm_status check_dtype(cmlbm_dtype dt) {
    if (dt != CMLBM_DT_F64 && dt != CMLBM_DT_F32) return fail(CMLBM_EINVAL, "dtype must be CMLBM_DT_F64 or CMLBM_DT_F32");
    return CMLBM_OK;
}

// Point the launch arguments at the stress buffers paired with the current
// state (read) and the next one (written); null when the sub-grid force is off.
void bind_stress(cmlbm_lattice* h) {
    const bool on = (h->a.flags & CMLBM_SGS_FORCE) != 0;
    h->a.stress_prev = on ? h->stress[h->cur] : nullptr;
    h->a.stress_next = on ? h->stress[h->cur ^ 1] : nullptr;
}

cmlbm_status check_sgs_ready(cmlbm_lattice* h) {
    if ((h->a.flags & CMLBM_SGS_FORCE) && !h->stress[0])
        return fail(CMLBM_ESTATE, "the sub-grid force needs stress buffers (cmlbm_set_sgs_buffers)");
    return CMLBM_OK;
}

// A new state starts with zero sub-grid stress (no force from the previous step).
hipError_t reset_stress(cmlbm_lattice* h) {
    if (!h->stress[0]) return hipSuccess;
    hipError_t e = cm::launch_zero(h->stress[0], h->stress_bytes, h->a.stream);
    if (e == hipSuccess) e = cm::launch_zero(h->stress[1], h->stress_bytes, h->a.stream);
    return e;
}

}  // namespace

extern "C" {

int32_t cmlbm_version(void) { return 10000; }

const char* cmlbm_last_error(void) { return g_err.c_str(); }

cmlbm_status cmlbm_create(const cmlbm_desc* d, void* buf_a, void* buf_b, size_t bytes_each, void* hip_stream,
                          cmlbm_handle* out) {
    if (!d || !out) return fail(CMLBM_EINVAL, "desc and out must be non-null");
    *out = nullptr;
    if (d->nx < 1 || d->ny < 1 || d->nz < 1) return fail(CMLBM_EINVAL, "nx, ny, nz must be >= 1");
    if (d->lattice != CMLBM_D3Q27 && d->lattice != CMLBM_D2Q9) return fail(CMLBM_EINVAL, "unknown lattice");
    if (d->lattice == CMLBM_D2Q9 && d->nz != 1) return fail(CMLBM_EINVAL, "D2Q9 requires nz == 1");
    if (d->streaming != CMLBM_STREAM_TWO_BUFFERS && d->streaming != CMLBM_STREAM_IN_PLACE)
        return fail(CMLBM_EINVAL, "desc.streaming must be CMLBM_STREAM_TWO_BUFFERS or CMLBM_STREAM_IN_PLACE");
    const bool inplace = d->streaming == CMLBM_STREAM_IN_PLACE;
    if (inplace && d->lattice != CMLBM_D3Q27) return fail(CMLBM_EINVAL, "in-place streaming is implemented for D3Q27");
    const int64_t N = (int64_t)d->nx * d->ny * d->nz;
    if (N >= ((int64_t)1 << 31)) return fail(CMLBM_EINVAL, "nx*ny*nz must be < 2^31");
    if (d->ny >= 65536 || d->nz >= 65536) return fail(CMLBM_EINVAL, "ny and nz must be < 65536");
    const size_t es = elem_size(d->storage);
    if (!es) return fail(CMLBM_EINVAL, "unknown storage mode");
    if (lane_span(d->nx, d->storage) > 0xffffffffull) {
        char msg[200];
        std::snprintf(msg, sizeof msg,
                      "nx = %d too large for this storage: the kernels address a row with 32-bit byte offsets "
                      "(3*nx*%zu and nx*%zu bytes must stay below 2^32)",
                      d->nx, es, compute_size(d->storage));
        return fail(CMLBM_EINVAL, msg);
    }
    if (d->walls & ~1u) return fail(CMLBM_EINVAL, "walls: only bit 0 is defined");
    if (d->tuning & ~252u) return fail(CMLBM_EINVAL, "tuning: only bits 2-7 are defined");
    if (!(std::isfinite(d->rho0) && d->rho0 > 0)) return fail(CMLBM_EINVAL, "rho0 must be finite and > 0");
    for (int k = 0; k < 3; ++k)
        if (!std::isfinite(d->wall_u_lo[k]) || !std::isfinite(d->wall_u_hi[k]))
            return fail(CMLBM_EINVAL, "wall velocities must be finite");
    if (inplace) {
        if (!buf_a || buf_b) return fail(CMLBM_EINVAL, "in-place streaming takes one buffer (buf_b must be null)");
    } else if (!buf_a || !buf_b || buf_a == buf_b) {
        return fail(CMLBM_EINVAL, "two distinct non-null buffers are required");
    }
    const size_t need = (size_t)lattice_q(d->lattice) * (size_t)N * es;
    if (bytes_each < need) {
        char msg[160];
        std::snprintf(msg, sizeof msg, "buffers too small: %zu bytes given, %zu needed", bytes_each, need);
        return fail(CMLBM_EINVAL, msg);
    }
    int device = 0;
    if (hipError_t e = hipGetDevice(&device); e != hipSuccess) return hip_fail(e, "hipGetDevice");
    cmlbm_lattice* h = new (std::nothrow) cmlbm_lattice();
    if (!h) return fail(CMLBM_ENOMEM, "host allocation failed");
    h->device = device;
    cm::LaunchArgs& a = h->a;
    a.g.nx = d->nx;
    a.g.ny = d->ny;
    a.g.nz = d->nz;
    a.g.N = N;
    {
        a.g.rowloop = (d->tuning & 4u) ? 1 : 0;
        a.g.lanegather = (d->tuning & 32u) ? 1 : 0;
        a.g.pairs_off = (d->tuning & 64u) ? 1 : 0;
        a.g.one_launch = (d->tuning & 128u) ? 1 : 0;
        const unsigned order = (d->tuning >> 3) & 3u;
        a.g.xcd = order == 1u ? 0 : (order == 2u ? 1 : cm::kXcdRun);
        if (order == 0u)
            a.g.xcd = cm::default_order(d->lattice, d->storage, d->nx, a.g.rowloop != 0, (d->walls & 1u) != 0, inplace,
                                        a.g.lanegather != 0);
        if (a.g.xcd == 1 && need < cm::kSmallState) a.g.xcd = -1;
        a.xcd_default = order == 0u ? 1 : 0;
        a.g.aa = inplace ? 1 : 0;
        a.g.ybase = 0;
        a.g.ystride = 1;
        a.g.yrows = d->ny;
        a.g.zbase = 0;
        a.g.pack = 0;
        a.g.packm = 0;
    }
    a.lattice = d->lattice;
    a.storage = d->storage;
    a.walls = (int)(d->walls & 1u);
    a.rho0 = d->rho0;
    a.omega_shear = a.omega_bulk = 1.0;
    for (int k = 0; k < 3; ++k) a.omega3[k] = 1.0;
    a.omega4[0] = a.omega4[1] = 1.0;
    a.omega5 = a.omega6 = 1.0;
    a.cs_smag = 0.0;
    a.flags = 0;
    for (int k = 0; k < 3; ++k) {
        a.force[k] = 0.0;
        a.wall_u_lo[k] = d->wall_u_lo[k];
        a.wall_u_hi[k] = d->wall_u_hi[k];
    }
    a.force_field = nullptr;
    a.stream = hip_stream;
    a.stress_prev = nullptr;
    a.stress_next = nullptr;
    h->stress[0] = h->stress[1] = nullptr;
    h->stress_bytes = 0;
    h->buf[0] = buf_a;
    h->buf[1] = buf_b;
    h->cur = 0;
    h->bytes_each = bytes_each;
    hipError_t e = hipMalloc((void**)&h->scratch, sizeof(double) * 8 * cm::kReduceBlocks);
    if (e == hipSuccess) {
        e = g_results.take(&h->result);
        if (e != hipSuccess) (void)hipFree(h->scratch);
    }
    if (e != hipSuccess) {
        delete h;
        return hip_fail(e, "allocation of the reduction scratch");
    }
    *out = h;
    return CMLBM_OK;
}

cmlbm_status cmlbm_destroy(cmlbm_handle h) {
    if (!h) return CMLBM_OK;
    hipError_t e = hipSuccess;
    if (h->scratch) {
        // the scratch may still be in use by work queued on the stream
        e = hipStreamSynchronize((hipStream_t)h->a.stream);
        hipError_t e2 = hipFree(h->scratch);
        if (e == hipSuccess) e = e2;
        e2 = g_results.give_back(h->result);   // no queued work writes to it any more
        if (e == hipSuccess) e = e2;
    }
    delete h;
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "cmlbm_destroy");
}

cmlbm_status cmlbm_set_stream(cmlbm_handle h, void* hip_stream) {
    if (cmlbm_status s = check_handle(h)) return s;
    h->a.stream = hip_stream;
    return CMLBM_OK;
}

cmlbm_status cmlbm_set_relaxation(cmlbm_handle h, const cmlbm_relax* r) {
    // the arguments are validated before the handle so that the checks can be
    // exercised without a device
    if (!r) return fail(CMLBM_EINVAL, "relax must be non-null");
    const double rates[] = {r->omega_shear, r->omega_bulk, r->omega3[0], r->omega3[1], r->omega3[2],
                            r->omega4[0],   r->omega4[1],  r->omega5,    r->omega6};
    for (double w : rates)
        if (!rate_ok(w)) return fail(CMLBM_EINVAL, "relaxation rates must lie in (0, 2)");
    if (!(std::isfinite(r->cs_smag) && r->cs_smag >= 0.0)) return fail(CMLBM_EINVAL, "cs_smag must be finite and >= 0");
    if ((r->flags & ~7u) || r->reserved) return fail(CMLBM_EINVAL, "flags: only bits 0-2 are defined; reserved must be 0");
    if (cmlbm_status s = check_handle(h)) return s;
    if (r->flags & CMLBM_SGS_FORCE) {
        if (h->a.walls) return fail(CMLBM_EINVAL, "the sub-grid force needs a periodic lattice");
        if (h->a.g.aa) return fail(CMLBM_EINVAL, "the sub-grid force needs two-buffer streaming");
    }
    cm::LaunchArgs& a = h->a;
    a.omega_shear = r->omega_shear;
    a.omega_bulk = r->omega_bulk;
    for (int k = 0; k < 3; ++k) a.omega3[k] = r->omega3[k];
    a.omega4[0] = r->omega4[0];
    a.omega4[1] = r->omega4[1];
    a.omega5 = r->omega5;
    a.omega6 = r->omega6;
    a.cs_smag = r->cs_smag;
    a.flags = r->flags;
    return CMLBM_OK;
}

cmlbm_status cmlbm_set_force(cmlbm_handle h, const double uniform[3], const void* field) {
    if (cmlbm_status s = check_handle(h)) return s;
    for (int k = 0; k < 3; ++k) {
        const double v = uniform ? uniform[k] : 0.0;
        if (!std::isfinite(v)) return fail(CMLBM_EINVAL, "uniform force must be finite");
        h->a.force[k] = v;
    }
    h->a.force_field = field;
    return CMLBM_OK;
}

cmlbm_status cmlbm_init_equilibrium(cmlbm_handle h, const void* rho, const void* u, cmlbm_dtype dt) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (cmlbm_status s = check_dtype(dt)) return s;
    if (!u) return fail(CMLBM_EINVAL, "u must be non-null");
    h->cur = 0;
    if (h->a.g.aa) h->a.g.aa = 1;   // in place: a new state is in the even arrangement
    hipError_t e = reset_stress(h);
    if (e == hipSuccess)
        e = h->a.lattice ? cm2::launch_init_equilibrium(h->a, h->buf[0], rho, u, (int)dt)
                         : cm::launch_init_equilibrium(h->a, h->buf[0], rho, u, (int)dt);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "init_equilibrium");
}

cmlbm_status cmlbm_step(cmlbm_handle h, int64_t nsteps) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (nsteps < 0) return fail(CMLBM_EINVAL, "nsteps must be >= 0");
    if (cmlbm_status s = check_sgs_ready(h)) return s;
    if (h->a.g.aa) {
        for (int64_t n = 0; n < nsteps; ++n) {
            hipError_t e = cm::launch_step_inplace(h->a, h->buf[0]);
            if (e != hipSuccess) return hip_fail(e, "step");
            h->a.g.aa = 3 - h->a.g.aa;
        }
        return CMLBM_OK;
    }
    for (int64_t n = 0; n < nsteps; ++n) {
        bind_stress(h);
        hipError_t e = h->a.lattice ? cm2::launch_step(h->a, h->buf[h->cur], h->buf[h->cur ^ 1])
                                    : cm::launch_step(h->a, h->buf[h->cur], h->buf[h->cur ^ 1]);
        if (e != hipSuccess) return hip_fail(e, "step");
        h->cur ^= 1;
    }
    return CMLBM_OK;
}

cmlbm_status cmlbm_step_from(cmlbm_handle h, const void* src, void* dst) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (!src || !dst || src == dst) return fail(CMLBM_EINVAL, "src and dst must be distinct non-null buffers");
    if (h->a.flags & CMLBM_SGS_FORCE)
        return fail(CMLBM_EINVAL, "step_from does not carry the sub-grid stress; use cmlbm_step");
    if (h->a.g.aa) return fail(CMLBM_EINVAL, "step_from needs two-buffer streaming");
    hipError_t e = h->a.lattice ? cm2::launch_step(h->a, src, dst) : cm::launch_step(h->a, src, dst);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "step_from");
}

// Bytes of one population state.
static size_t state_bytes(cmlbm_handle h) {
    return (size_t)lattice_q(h->a.lattice) * (size_t)h->a.g.N * elem_size(h->a.storage);
}

cmlbm_status cmlbm_steps_between(cmlbm_handle h, const void* src, void* dst, int64_t nsteps) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (nsteps < 1) return fail(CMLBM_EINVAL, "nsteps must be >= 1");
    for (const void* b : h->buf)
        if (src == b || dst == b) return fail(CMLBM_EINVAL, "src and dst must not be the handle's buffers");
    for (int64_t n = 0; n < nsteps; ++n) {
        void* to = n == nsteps - 1 ? dst : h->buf[n & 1];
        if (cmlbm_status s = cmlbm_step_from(h, src, to)) return s;
        src = to;
    }
    return CMLBM_OK;
}

cmlbm_status cmlbm_steps_record(cmlbm_handle h, const void* first, void* rest, size_t stride, int64_t nsteps) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (nsteps < 0) return fail(CMLBM_EINVAL, "nsteps must be >= 0");
    if (nsteps && !rest) return fail(CMLBM_EINVAL, "rest must be non-null");
    if (stride < state_bytes(h)) return fail(CMLBM_EINVAL, "stride is smaller than a population buffer");
    for (int64_t n = 0; n < nsteps; ++n) {
        void* to = (char*)rest + (size_t)n * stride;
        if (cmlbm_status s = cmlbm_step_from(h, first, to)) return s;
        first = to;
    }
    return CMLBM_OK;
}

cmlbm_status cmlbm_state_buffer(cmlbm_handle h, void** buf, size_t* bytes) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (!buf) return fail(CMLBM_EINVAL, "buf must be non-null");
    *buf = h->buf[h->cur];
    if (bytes) *bytes = state_bytes(h);
    return CMLBM_OK;
}

cmlbm_status cmlbm_read_moments(cmlbm_handle h, void* rho, void* u, cmlbm_dtype dt) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (cmlbm_status s = check_dtype(dt)) return s;
    if (!rho || !u) return fail(CMLBM_EINVAL, "rho and u must be non-null");
    if (cmlbm_status s = check_sgs_ready(h)) return s;
    bind_stress(h);
    hipError_t e = h->a.lattice ? cm2::launch_read(h->a, h->buf[h->cur], rho, u, (int)dt, 1)
                                : cm::launch_read(h->a, h->buf[h->cur], rho, u, (int)dt, 1);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "read_moments");
}

cmlbm_status cmlbm_get_populations(cmlbm_handle h, void* f, cmlbm_dtype dt) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (cmlbm_status s = check_dtype(dt)) return s;
    if (!f) return fail(CMLBM_EINVAL, "f must be non-null");
    hipError_t e = h->a.lattice ? cm2::launch_read(h->a, h->buf[h->cur], f, nullptr, (int)dt, 0)
                                : cm::launch_read(h->a, h->buf[h->cur], f, nullptr, (int)dt, 0);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "get_populations");
}

cmlbm_status cmlbm_set_populations(cmlbm_handle h, const void* f, cmlbm_dtype dt) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (cmlbm_status s = check_dtype(dt)) return s;
    if (!f) return fail(CMLBM_EINVAL, "f must be non-null");
    if (h->a.g.aa) h->a.g.aa = 1;   // in place: set in the even arrangement
    hipError_t e = reset_stress(h);
    if (e == hipSuccess)
        e = h->a.lattice ? cm2::launch_set_populations(h->a, h->buf[h->cur], f, (int)dt)
                         : cm::launch_set_populations(h->a, h->buf[h->cur], f, (int)dt);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "set_populations");
}

cmlbm_status cmlbm_reduce(cmlbm_handle h, double out[8]) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (!out) return fail(CMLBM_EINVAL, "out must be non-null");
    if (cmlbm_status s = check_sgs_ready(h)) return s;
    bind_stress(h);
    // the last kernel writes the values to host memory: no copy to wait for
    hipError_t e = h->a.lattice ? cm2::launch_reduce(h->a, h->buf[h->cur], h->scratch, h->result)
                                : cm::launch_reduce(h->a, h->buf[h->cur], h->scratch, h->result);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)h->a.stream);
    if (e != hipSuccess) return hip_fail(e, "reduce");
    std::memcpy(out, h->result, 8 * sizeof(double));
    if (out[5] > 0) {
        char msg[96];
        std::snprintf(msg, sizeof msg, "%.0f cells with non-finite rho or u", out[5]);
        return fail(CMLBM_ENONFINITE, msg);
    }
    return CMLBM_OK;
}

cmlbm_status cmlbm_reduce_noalloc(cmlbm_handle h, double* out) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (!out) return fail(CMLBM_EINVAL, "out must be a non-null device array of 8 doubles");
    if (cmlbm_status s = check_sgs_ready(h)) return s;
    double* scratch = nullptr;
    hipError_t e = cm::static_reduce_scratch(h->device, &scratch);
    if (e != hipSuccess) return hip_fail(e, "reduce_noalloc: address of the static scratch");
    bind_stress(h);
    // partials in the static scratch, the final combination straight into out
    e = h->a.lattice ? cm2::launch_reduce(h->a, h->buf[h->cur], scratch, out)
                     : cm::launch_reduce(h->a, h->buf[h->cur], scratch, out);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "reduce_noalloc");
}

static cmlbm_status adjoint_ok(cmlbm_handle h) {
    if (h->a.lattice != CMLBM_D3Q27) return fail(CMLBM_EINVAL, "adjoint supports the D3Q27 lattice only");
    if (h->a.g.aa) return fail(CMLBM_EINVAL, "adjoint needs two-buffer streaming");
    if (h->a.flags & CMLBM_SGS_FORCE) return fail(CMLBM_EINVAL, "adjoint does not support the sub-grid stress as a force");
    return CMLBM_OK;
}

cmlbm_status cmlbm_adjoint_step(cmlbm_handle h, const void* state, const void* lam_in, void* lam_out, void* grad_F) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (cmlbm_status s = adjoint_ok(h)) return s;
    if (!state || !lam_in || !lam_out || !grad_F || lam_in == lam_out)
        return fail(CMLBM_EINVAL, "state, lam_in, lam_out, grad_F must be non-null and lam_in != lam_out");
    hipError_t e = cm::launch_adjoint(h->a, state, lam_in, lam_out, grad_F);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "adjoint_step");
}

cmlbm_status cmlbm_adjoint_steps(cmlbm_handle h, const void* first, const void* rest, size_t stride, int64_t nsteps,
                                 void* lam, void* lam_tmp, void* grad_F) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (nsteps < 0) return fail(CMLBM_EINVAL, "nsteps must be >= 0");
    if (nsteps > 1 && !rest) return fail(CMLBM_EINVAL, "rest must be non-null");
    if (stride < state_bytes(h)) return fail(CMLBM_EINVAL, "stride is smaller than a population buffer");
    for (int64_t n = nsteps - 1; n >= 0; --n) {
        const void* state = n ? (const char*)rest + (size_t)(n - 1) * stride : first;
        if (cmlbm_status s = cmlbm_adjoint_step(h, state, lam, lam_tmp, grad_F)) return s;
        void* t = lam;
        lam = lam_tmp;
        lam_tmp = t;
    }
    return CMLBM_OK;
}

cmlbm_status cmlbm_energy_seed(cmlbm_handle h, const void* state, void* lam_out, void* grad_F) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (cmlbm_status s = adjoint_ok(h)) return s;
    if (!state || !lam_out || !grad_F) return fail(CMLBM_EINVAL, "state, lam_out, grad_F must be non-null");
    hipError_t e = cm::launch_energy_seed(h->a, state, lam_out, grad_F);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "energy_seed");
}

cmlbm_status cmlbm_set_sgs_buffers(cmlbm_handle h, void* stress_a, void* stress_b, size_t bytes_each) {
    if (cmlbm_status s = check_handle(h)) return s;
    if (h->a.g.aa) return fail(CMLBM_EINVAL, "the sub-grid force needs two-buffer streaming");
    if (!stress_a || !stress_b || stress_a == stress_b)
        return fail(CMLBM_EINVAL, "two distinct non-null stress buffers are required");
    const size_t es = h->a.storage == CMLBM_F64 ? 8 : 4;
    const size_t planes = h->a.lattice == CMLBM_D2Q9 ? 3 : 6;
    const size_t need = planes * (size_t)h->a.g.N * es;
    if (bytes_each < need) {
        char msg[160];
        std::snprintf(msg, sizeof msg, "stress buffers too small: %zu bytes given, %zu needed", bytes_each, need);
        return fail(CMLBM_EINVAL, msg);
    }
    h->stress[0] = stress_a;
    h->stress[1] = stress_b;
    h->stress_bytes = need;
    hipError_t e = reset_stress(h);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "set_sgs_buffers");
}

cmlbm_status cmlbm_copy(const void* src, void* dst, size_t bytes, void* hip_stream) {
    if (!src || !dst || src == dst) return fail(CMLBM_EINVAL, "src and dst must be distinct non-null buffers");
    if (bytes % 16 || ((uintptr_t)src % 16) || ((uintptr_t)dst % 16))
        return fail(CMLBM_EINVAL, "bytes and both addresses must be multiples of 16");
    hipError_t e = cm::launch_copy(src, dst, bytes, hip_stream);
    return e == hipSuccess ? CMLBM_OK : hip_fail(e, "copy");
}

}  // extern "C"
