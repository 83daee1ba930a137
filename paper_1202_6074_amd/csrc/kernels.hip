// Device kernels of the D3Q27 cascaded central-moment LBM (gfx950).
//
// Internal memory layout (row-interleaved structure of arrays): the nx values
// of population i on grid row (y, z) are contiguous, and the 27 population
// rows of one grid row follow each other:
//     element (i, x, y, z) at ((z * ny + y) * 27 + i) * nx + x.
// A cell's 27 writes therefore land in one contiguous 27-row region and its
// gathers in nine contiguous 3-row regions (the three populations with the
// same (ey, ez) are adjacent), which keeps DRAM accesses local; arrays
// exchanged with callers (populations, moments, force, adjoint) use the plain
// structure of arrays, plane i = population i, cell c = x + nx (y + ny z).
//
// The step kernel is a pull scheme: the buffer between steps holds the
// post-collision, not yet streamed values fbar~(n-1); each thread gathers the
// 27 values arriving at its cell (standard streaming, Eq. cascadedstreaming1),
// collides (Eq. cascadedcollision1) and writes the 27 post-collision values
// back at its own cell into the other buffer. Reads come from the rows of the
// neighbour cells at x +- 1 offsets; writes are aligned and coalesced.
//
// Walls (project addition): halfway bounce-back planes at y = -1/2 and
// y = ny - 1/2 with wall velocities U_lo, U_hi. A population whose upstream
// cell lies in a wall is the opposite population of the same cell plus
// 2 w_i rho0 (e_i . U) / cs^2.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "cm_math.hpp"
#include "kernels.hpp"
#include "store.hpp"

namespace cm {

// Offset (in elements) of the row of population i at grid row (y, z) in the
// row-interleaved internal layout. (A plain-plane layout, i N + c, measured
// slower in every storage mode, and a run-time choice between the two cost
// the step kernel a third of its scalar and a sixth of its vector
// instructions, so the layout is fixed.)
__device__ __forceinline__ size_t row_base(const Geom& g, int i, int y, int z) {
    const size_t r = (size_t)z * g.ny + y;
    return (r * 27 + i) * g.nx;
}

// Plane i of grid row (y, z) for rows of at most 512 cells: 32-bit factors (27 rows
// are fewer than 2^32 bytes), where row_base multiplies in 64 bits. The scalar
// unit that forms these addresses serves all four SIMDs of a CU: with 64-bit
// products and a loop around each copy the step by rows spent 650 scalar
// instructions a wave beside 720 vector ones, now 405 (us per step, before / after:
// 301 x 200 x 200 FP16 270 / 262, 200^3 FP16 176 / 172, 300 x 181 x 90 FP32-shifted
// channel 195 / 192, 500 x 300 x 100 FP32 616 / 609; the LDS-exchange, two-cell and
// in-place kernels measured the same or up to 2 % slower with it).
template <typename T>
__device__ __forceinline__ T* short_row(T* base, const Geom& g, int i, int y, int z) {
    const uint32_t rb = (uint32_t)g.nx * (uint32_t)sizeof(T), r = (uint32_t)z * (uint32_t)g.ny + (uint32_t)y;
    using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return (T*)((C*)base + (uint64_t)r * (27u * rb) + (uint32_t)i * rb);
}

// Address of an element: a row pointer that is the same for every lane of the
// workgroup, plus the lane's 32-bit byte offset. Every kernel here takes y and
// z from the block index, so its row pointers are workgroup-uniform; read
// through readfirstlane and typed as global memory, each access then takes the
// scalar-base form of the global load and store instructions (base in scalar
// registers, 32-bit lane offset), where the compiler otherwise forms every
// address with 64-bit vector arithmetic, one instruction per access. Only for
// pointers that are uniform across the workgroup.
template <typename T>
using global_ptr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ global_ptr<T> at_row(T* row, uint32_t lane_bytes) {
    // readfirstlane returns a signed 32-bit value: each half goes through
    // uint32_t, so that the low half is zero-extended, not sign-extended.
    const uint64_t v = (uint64_t)row;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    const uint64_t u = ((uint64_t)hi << 32) | (uint64_t)lo;
    return (global_ptr<T>)((global_ptr<char>)u + lane_bytes);
}
// SB: the scalar-base form above, for kernels without a loop around the access
// (inside a loop the uniform read cannot be hoisted and costs more than it
// saves); otherwise the plain pointer.
template <bool SB, typename T>
__device__ __forceinline__ auto row_at(T* row, uint32_t lane_bytes) {
    if constexpr (SB) {
        return at_row(row, lane_bytes);
    } else {
        using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
        return (T*)((C*)row + lane_bytes);
    }
}

template <typename R>
struct Launch {
    Rates<R> P;
    R F[3];        // uniform force (used when no field is given)
    R wt_lo[27], wt_hi[27];   // wall terms per direction, lower and upper wall
    const R* rs_prev;   // sub-grid stress of the previous step, or null (read-out kernels)
};

// Acceleration a' = -div R of the sub-grid stress of the previous step at
// (x, y, z) (Sec. 14 coupling): second-order central differences on the
// periodic grid. Stress planes xx, yy, zz, xy, xz, yz, plain structure of
// arrays; y and z are block-uniform, so the row offsets are uniform.
// sgs_load reads the 18 stress values the differences need, sgs_combine forms
// the acceleration from them (two steps, so that a caller can keep the loads
// in flight together with others).
template <typename R, bool SB = false>
__device__ __forceinline__ void sgs_load(const R* __restrict__ rs, const Geom g, int x, int y, int z, R (&v)[18]) {
    const size_t N = (size_t)g.N, nx = (size_t)g.nx;
    const size_t r0 = nx * ((size_t)y + (size_t)g.ny * z);
    const size_t ryp = nx * ((size_t)(y == g.ny - 1 ? 0 : y + 1) + (size_t)g.ny * z);
    const size_t rym = nx * ((size_t)(y == 0 ? g.ny - 1 : y - 1) + (size_t)g.ny * z);
    const size_t rzp = nx * ((size_t)y + (size_t)g.ny * (z == g.nz - 1 ? 0 : z + 1));
    const size_t rzm = nx * ((size_t)y + (size_t)g.ny * (z == 0 ? g.nz - 1 : z - 1));
    // uniform row pointers, per-lane 32-bit byte offsets (x, x + 1, x - 1 with wrap)
    const uint32_t ox = (uint32_t)x * (uint32_t)sizeof(R);
    const uint32_t oxp = (uint32_t)(x == g.nx - 1 ? 0 : x + 1) * (uint32_t)sizeof(R);
    const uint32_t oxm = (uint32_t)(x == 0 ? g.nx - 1 : x - 1) * (uint32_t)sizeof(R);
    auto at = [&](int k, size_t r, uint32_t o) { return *row_at<SB>(rs + k * N + r, o); };
    // x differences of xx, xy, xz; y differences of xy, yy, yz; z differences of xz, yz, zz
    const int kx[3] = {0, 3, 4}, ky[3] = {3, 1, 5}, kz[3] = {4, 5, 2};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v[2 * c] = at(kx[c], r0, oxp);
        v[2 * c + 1] = at(kx[c], r0, oxm);
        v[6 + 2 * c] = at(ky[c], ryp, ox);
        v[6 + 2 * c + 1] = at(ky[c], rym, ox);
        v[12 + 2 * c] = at(kz[c], rzp, ox);
        v[12 + 2 * c + 1] = at(kz[c], rzm, ox);
    }
}
template <typename R>
__device__ __forceinline__ void sgs_combine(const R (&v)[18], R (&a)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
        a[c] = R(-0.5) * ((v[2 * c] - v[2 * c + 1]) + (v[6 + 2 * c] - v[6 + 2 * c + 1]) + (v[12 + 2 * c] - v[12 + 2 * c + 1]));
}
template <typename R, bool SB = false>
__device__ __forceinline__ void sgs_accel(const R* __restrict__ rs, const Geom g, int x, int y, int z, R (&a)[3]) {
    R v[18];
    sgs_load<R, SB>(rs, g, x, y, z, v);
    sgs_combine(v, a);
}

// Correction added to a bounced population arriving in direction i from a wall
// moving with velocity U, 2 w_i rho0 (e_i . U) / cs^2, precomputed on the host
// (Launch::wt_lo, wt_hi). It is added and removed with explicitly rounded
// operations, so that no code path fuses it differently into neighbouring
// arithmetic: the two-buffer and in-place schemes then agree bit for bit.
__device__ __forceinline__ float add_rn(float a, float b) { return __fadd_rn(a, b); }
__device__ __forceinline__ double add_rn(double a, double b) { return __dadd_rn(a, b); }
__device__ __forceinline__ float sub_rn(float a, float b) { return __fsub_rn(a, b); }
__device__ __forceinline__ double sub_rn(double a, double b) { return __dsub_rn(a, b); }

// Population loads. Every stored population is read exactly once per step, so
// the loads are non-temporal (measured 7 % faster for FP32 at 256^3, neutral
// for FP64; for FP16 1.5 % faster in the LDS kernel at 256^3 and 3.8 % in the
// even in-place step, since the shorter FP16 collision). Rows that lanes
// read shifted by x -+ 1 share cache lines with the neighbouring wave and keep
// ordinary loads where a wave reads them per lane (the odd in-place step: all
// non-temporal measured 13 % slower, the rows at x alone 1 % faster). In the
// LDS kernel every row is read aligned and once: all non-temporal (ordinary
// loads for the 18 rows exchanged through LDS measured 7 % slower).
template <int S, bool NT = true, typename P = const typename Store<S>::T*>
__device__ __forceinline__ typename Store<S>::T load_raw(P p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// Stored value of population i -> deviation from the rest state (compute type),
// and back. The rest-state shift of unshifted storage is rounded explicitly, so
// that no kernel fuses it with neighbouring arithmetic differently from another
// (the step kernels of the different streaming schemes agree bit for bit).
template <int S, typename R = typename Store<S>::R>
__device__ __forceinline__ R from_store(typename Store<S>::T t, int i, R rho0) {
    R v = static_cast<R>(t);
    if constexpr (!Store<S>::shifted) v = sub_rn(v, rho0 * w27<R>(i));
    return v;
}

template <int S, bool NT = true, typename R = typename Store<S>::R, typename P = const typename Store<S>::T*>
__device__ __forceinline__ R load_dev(P p, int i, R rho0) {
    return from_store<S>(load_raw<S, NT>(p), i, rho0);
}

template <int S, typename R = typename Store<S>::R>
__device__ __forceinline__ typename Store<S>::T to_store(R v, int i, R rho0) {
    if constexpr (!Store<S>::shifted) v = add_rn(v, rho0 * w27<R>(i));
    // FP16: the FP32 value is rounded to binary16 on its own (round to nearest
    // even). Without this register constraint the compiler folds the
    // conversion into the last arithmetic operation of some values (one
    // rounding instead of two), differently in different kernels; the FP16
    // kernels then would not agree bit for bit.
    if constexpr (S == 3) asm volatile("" : "+v"(v));
    return static_cast<typename Store<S>::T>(v);
}

// Two FP16 values in one 32-bit word (x, x + 1 of a row; lower address in the
// low half) and back.
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// Sums of FP16 values held in 32-bit registers (H = 0: the low halves, 1: the
// high halves) with an FP32 result: v_fma_mix_f32 widens its FP16 operands
// exactly and rounds a*1 + c once, which is the FP32 sum of the converted
// values, without the conversion instructions.
template <int H>
__device__ __forceinline__ float mix_add(uint32_t a, uint32_t c) {   // a + c
    float r;
    if constexpr (H == 0) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a), "v"(c));
    else asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a), "v"(c));
    return r;
}
template <int H>
__device__ __forceinline__ float mix_sub(uint32_t c, uint32_t a) {   // c - a
    float r;
    if constexpr (H == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(c), "v"(a));
    else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(c), "v"(a));
    return r;
}
template <int H>
__device__ __forceinline__ float mix_addf(uint32_t b, float s) {   // b + s, s in FP32
    float r;
    if constexpr (H == 0) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(b), "v"(s));
    else asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(b), "v"(s));
    return r;
}
// The velocity-independent z-line sums of collide (ls = a + c, ld = c - a,
// k0 = ls + b) of line l from FP16 values a, b, c in the halves H.
template <int H>
__device__ __forceinline__ void mix_line(uint32_t a, uint32_t b, uint32_t c, float& ls, float& ld, float& k0) {
    ls = mix_add<H>(a, c);
    ld = mix_sub<H>(c, a);
    k0 = mix_addf<H>(b, ls);
}
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
    // each value rounded to binary16 on its own, as to_store<3> does
    asm volatile("" : "+v"(a), "+v"(b));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t){a, b}, half2_t));
}


// The wall terms of the populations that arrived from a wall, on a row next to
// one (y uniform).
template <typename R>
__device__ __forceinline__ void add_wall_terms(const Geom& g, int y, const Launch<R>& L, R (&h)[27]) {
    if (y == 0) {
#pragma unroll
        for (int i = 0; i < 27; ++i)
            if ((i / 3) % 3 == 2) h[i] = add_rn(h[i], L.wt_lo[i]);
    }
    if (y == g.ny - 1) {
#pragma unroll
        for (int i = 0; i < 27; ++i)
            if ((i / 3) % 3 == 0) h[i] = add_rn(h[i], L.wt_hi[i]);
    }
}

// Gather of fbar(n) at cell (x, y, z).
// MODE 0 (two-buffer pull scheme): the buffer holds fbar~(n-1), population i
//   of the upstream cell x - e_i in plane i, or, when that is a wall, plane
//   26 - i of the cell itself plus the wall term.
// MODE 1 (in-place streaming, even parity): fbar_i(x) sits in plane i of x;
//   a population that arrived from a wall is kept without its wall term,
//   which is added here (the same arithmetic as MODE 0).
// MODE 2 (in-place streaming, odd parity): the previous (even) step stored
//   fbar~_i(x) in plane 26 - i of x, so fbar_i(x) is plane 26 - i of x - e_i,
//   or, from a wall, plane i of x plus the wall term.
// y and z are uniform across a block, so the 27 source rows are uniform
// pointers (scalar registers); only the x offset (x - 1, x, x + 1 with wrap)
// varies across lanes, as a 32-bit byte offset.
// The rows read at x, once, take non-temporal loads; the x-shifted rows ordinary ones,
// since the neighbouring wave, and at the split of a row between workgroups another
// workgroup, reads their cache lines too (non-temporal +4 % for FP32 at 512^3; reductions of
// 512 x 512 x 128 FP16 531 us non-temporal, 458 ordinary; the aligned rows of the odd in-place gather
// non-temporal: 1024 x 512 x 512 FP32 10,930 -> 10,832 us, FP16 shifted 6,038 -> 5,957 us per pair).
// gather_xlds, where one workgroup covers a row, reads every line once.
// WALLS: a group from a wall reads other rows and is not shifted; y is uniform, so
// these are scalar selects, and the wall terms are added at the end (a branch
// for each population kept the loads from being in flight together: the adjoint
// of 128^3 FP32 with the eddy viscosity between walls 175 us, now 119, periodic
// 118).
template <int S, bool WALLS, int MODE = 0, bool SB = false, typename R = typename Store<S>::R>
__device__ __forceinline__ void gather(const typename Store<S>::T* src, const Geom g, int x, int y, int z,
                                       const Launch<R>& L, R (&h)[27]) {
    using T = typename Store<S>::T;
    if constexpr (MODE == 1) {
        const uint32_t xt = (uint32_t)x * (uint32_t)sizeof(T);
#pragma unroll
        for (int i = 0; i < 27; ++i) h[i] = load_dev<S>(row_at<SB>(src + row_base(g, i, y, z), xt), i, L.P.rho0);
        if constexpr (WALLS) add_wall_terms(g, y, L, h);
        return;
    }
    const uint32_t xo[3] = {(uint32_t)(x == g.nx - 1 ? 0 : x + 1) * (uint32_t)sizeof(T), (uint32_t)x * (uint32_t)sizeof(T),
                            (uint32_t)(x == 0 ? g.nx - 1 : x - 1) * (uint32_t)sizeof(T)};   // x - ex, ex = -1, 0, +1
    const int ys[3] = {y == g.ny - 1 ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
    const int zs[3] = {z == g.nz - 1 ? 0 : z + 1, z, z == 0 ? g.nz - 1 : z - 1};
    // The three populations of a source row that differ only in ex sit in
    // consecutive rows of the interleaved layout, so each of the nine source
    // rows (ey, ez) needs one uniform pointer, and the row-in-group offset is
    // folded into the three per-lane offsets (scalar-register pressure).
    const uint32_t rb = (uint32_t)g.nx * (uint32_t)sizeof(T);
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ix = i % 3, iy = (i / 3) % 3, iz = i / 9, q = i / 3;
        const bool wall = WALLS && ((iy == 2 && y == 0) || (iy == 0 && y == g.ny - 1));
        // plane 26 - i (group 8 - q in reverse order) or i: the other one from a wall
        const bool rev = (MODE == 2) != wall;
        const T* grp = src + row_base(g, rev ? 24 - 3 * q : 3 * q, wall ? y : ys[iy], wall ? z : zs[iz]);
        const auto p = row_at<SB>(grp, xo[wall ? 1 : ix] + (uint32_t)(rev ? 2 - ix : ix) * rb);
        h[i] = ix == 1 ? load_dev<S, true>(p, i, L.P.rho0) : load_dev<S, false>(p, i, L.P.rho0);   // w_i = w_{26-i}
    }
    if constexpr (WALLS) add_wall_terms(g, y, L, h);
}

// Gather in the mode the geometry's streaming state asks for (read-out kernels).
template <int S, bool WALLS, typename R = typename Store<S>::R>
__device__ __forceinline__ void gather_any(const typename Store<S>::T* src, const Geom g, int x, int y, int z,
                                           const Launch<R>& L, R (&h)[27]) {
    if (g.aa == 0) gather<S, WALLS, 0>(src, g, x, y, z, L, h);
    else if (g.aa == 1) gather<S, WALLS, 1>(src, g, x, y, z, L, h);
    else gather<S, WALLS, 2>(src, g, x, y, z, L, h);
}

// Gather of the two-buffer pull scheme when one workgroup covers a whole grid
// row (nx <= blockDim.x = XW, lanes x >= nx idle): every population row is read
// aligned at x, so each wave reads whole cache lines and nothing twice, and the
// values that cross to x + 1 or x - 1 (the 18 rows with e_x != 0) are exchanged
// through LDS. Against per-lane shifted loads, the access pattern alone
// (trivial arithmetic, 256^3 FP32) runs 7 % faster. XW, the LDS row length, is
// the workgroup's width: with 256 for all, the 18 KB of an FP32 workgroup left
// room for eight 64-lane workgroups, eight waves, on a CU (64 x 64 x 128 FP32
// channel: 22.7 us a step, with the wall rows' own launch 33.0; now 21.0).
// WALLS: the populations that arrive from a wall are the opposite ones of the
// cell itself, row 26 - i at x, so the rows next to a wall read other rows and
// take their values without the shift; y is the same for the whole workgroup, so
// these are scalar selects and need no launch of their own. (The wall term
// itself is added by the caller.)
// Every lane of the workgroup must call this (it contains a barrier); idle
// lanes load a valid address and fill LDS columns nobody reads. pin() is
// called after all population loads are issued and before the barrier.
template <int S, bool SB, bool WALLS, int XW, typename Pin>
__device__ __forceinline__ void gather_xlds(const typename Store<S>::T* __restrict__ src, const Geom g, int x, bool act, int y,
                                            int z, typename Store<S>::T (&out)[27], Pin&& pin) {
    using T = typename Store<S>::T;
    __shared__ T sm[18][XW];
    const int ys[3] = {y == g.ny - 1 ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
    const int zs[3] = {z == g.nz - 1 ? 0 : z + 1, z, z == 0 ? g.nz - 1 : z - 1};
    // from a wall: e_y = +1 on the lowest row, e_y = -1 on the highest
    auto bounce = [&](int i) {
        const int iy = (i / 3) % 3;
        return WALLS && ((iy == 2 && y == 0) || (iy == 0 && y == g.ny - 1));
    };
    const uint32_t rb = (uint32_t)g.nx * (uint32_t)sizeof(T);
    const uint32_t xt = (uint32_t)(act ? x : 0) * (uint32_t)sizeof(T);   // idle lanes read x = 0
    T raw[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ix = i % 3, iy = (i / 3) % 3, iz = i / 9;
        const bool w = bounce(i);
        const T* grp = src + row_base(g, w ? 24 - (i - ix) : i - ix, w ? y : ys[iy], w ? z : zs[iz]);
        // (without SB the offsets are added to the pointer one after the other: with
        // their sum the compiler formed all scalar bases before the first load, us per
        // step 128^3 FP64 152 / 155, 64 x 200 x 200 FP32 95.5 / 96.7, 192^3 FP32 with the
        // sub-grid force 322 / 324)
        const uint32_t ro = (uint32_t)(w ? 2 - ix : ix) * rb;
        if constexpr (SB) raw[i] = load_raw<S>(at_row(grp, xt + ro));
        else raw[i] = load_raw<S>((const T*)((const char*)grp + xt + ro));
    }
#pragma unroll
    for (int i = 0; i < 27; ++i)
        if (i % 3 != 1) sm[(i / 3) * 2 + (i % 3) / 2][x] = raw[i];
    // The e_x = 0 values (and the caller's other loads, pin()) are used only
    // after the barrier; without these register constraints the compiler issues
    // their loads after it, a second memory round trip.
#pragma unroll
    for (int i = 1; i < 27; i += 3) asm volatile("" : "+v"(raw[i]));
    pin();
    __syncthreads();
    const int xp = x >= g.nx - 1 ? 0 : x + 1, xm = x == 0 ? g.nx - 1 : x - 1;
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ix = i % 3;   // e_x = ix - 1: the value comes from x - e_x
        out[i] = ix == 1 ? raw[i] : sm[(i / 3) * 2 + ix / 2][bounce(i) ? x : (ix == 0 ? xp : xm)];
    }
}

// The deviations h of the stored values t gathered at a cell of row y.
template <int S, bool WALLS, typename R = typename Store<S>::R>
__device__ __forceinline__ void stored_devs(const typename Store<S>::T (&t)[27], const Geom& g, int y, const Launch<R>& L,
                                            R (&h)[27]) {
#pragma unroll
    for (int i = 0; i < 27; ++i) h[i] = from_store<S>(t[i], i, L.P.rho0);
    if constexpr (WALLS) add_wall_terms(g, y, L, h);
}

// The z-line sums that collide_lines starts from, of the stored values t
// gathered at a cell of row y.
template <int S, bool WALLS, typename R = typename Store<S>::R>
__device__ __forceinline__ void stored_line_sums(const typename Store<S>::T (&t)[27], const Geom& g, int y,
                                                 const Launch<R>& L, R (&h)[27], R (&ls)[9], R (&ld)[9]) {
    if constexpr (S == 3) {
        // straight from the FP16 values (no conversions), but on the rows that
        // take wall terms; the sums round the same
        if (!(WALLS && (y == 0 || y == g.ny - 1))) {
#pragma unroll
            for (int l = 0; l < 9; ++l)
                mix_line<0>(__builtin_bit_cast(uint16_t, t[l]), __builtin_bit_cast(uint16_t, t[l + 9]),
                            __builtin_bit_cast(uint16_t, t[l + 18]), ls[l], ld[l], h[l]);
            return;
        }
    }
    stored_devs<S, WALLS>(t, g, y, L, h);
    zline_sums(h, ls, ld);
}

// ---------------------------------------------------------------- whole rows through LDS
// Direct copy of 16 bytes a lane from global memory to LDS: lane l of a wave
// writes at `lds` + 16 l (lds the same for the whole wave), without a vector
// register in between. Complete after wait_lds_copies, for the wave's own
// copies; a barrier after it makes them visible to the workgroup.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <typename P>
__device__ __forceinline__ void copy16_to_lds(P src, void* lds) {
    constexpr int kNonTemporal = 2;   // cache policy bit of the instruction
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)lds, 16, 0, kNonTemporal);
}
__device__ __forceinline__ void wait_lds_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// LDS element at a byte offset: where offsets are formed in bytes, one addition
// of a scalar makes an address, in elements the shift is a second instruction
// (54 of them in the step of 187 x 151 x 133 FP16, bound by instruction issue).
template <typename T>
__device__ __forceinline__ T& lds_at(T* sm, uint32_t bytes) { return *(T*)((unsigned char*)sm + bytes); }

// The copies of n vectors from `from` into LDS at `to` by the workgroup's lanes, at
// most PASSES vectors a lane.
template <int PASSES>
__device__ __forceinline__ void copy_vectors(const u32x4* from, unsigned char* to, uint32_t n, uint32_t tid, uint32_t wave0,
                                             uint32_t bd) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const uint32_t k = (uint32_t)p * bd;
        if (tid + k < n) copy16_to_lds(at_row(from, (tid + k) * 16u), to + 16u * (k + wave0));
    }
}

// Elements of LDS that hold a group of three adjacent rows of nx values with up
// to one 16-byte vector of misalignment, in whole vectors.
template <typename T>
__host__ __device__ constexpr uint32_t group_stride(uint32_t nx) {
    constexpr uint32_t V = 16 / sizeof(T);
    return (3u * nx + 2u * V - 1u) / V * V;
}

// Stores a block of n values at D, held in LDS from element o on (o the
// misalignment of D, so that LDS and memory vectors coincide): whole vectors
// non-temporal, the values of the vectors at the ends one by one (a block
// shorter than a vector has only those).
template <typename T>
__device__ __forceinline__ void store_block(T* D, uint32_t o, uint32_t n, const T* sm, uint32_t tid, uint32_t bd) {
    constexpr uint32_t V = 16 / sizeof(T);
    T* const D0 = D - o;   // the block's first vector
    const uint32_t end = o + n, c1 = end / V;
    for (uint32_t c = tid + (o ? 1u : 0u); c < c1; c += bd)
        __builtin_nontemporal_store(((const u32x4*)sm)[c], at_row((u32x4*)D0, c * 16u));
    if (o && tid >= o && tid < V && tid < end) D0[tid] = sm[tid];
    const uint32_t tail = c1 * V + tid;
    if (tail < end && (c1 || !o)) D0[tail] = sm[tail];
}

// Gather of the two-buffer pull scheme for a workgroup that holds a whole grid
// row, lane = cell, at any alignment: in memory the three populations of a source
// row that differ only in e_x are one contiguous block of 3 nx values; the nine
// blocks are copied straight into LDS (`sm`, 9 group_stride values) as 16-byte
// vectors of 16-byte-aligned addresses, and each lane reads its 27 values there,
// shifted by e_x. other() is called between the copies and the wait for them. A
// vector at either end of a block can hold values outside it, which are not
// used: an aligned vector with one valid byte lies in a mapped page.
// t: the stored values as the step kernels' other gathers give them. Idle lanes
// (x = 0) take part; every lane of the workgroup must call this.
template <int S, bool WALLS, typename Other>
__device__ __forceinline__ void gather_rows(const typename Store<S>::T* __restrict__ src, const Geom& g, uint32_t x, int y,
                                            int z, typename Store<S>::T* sm, typename Store<S>::T (&t)[27], Other&& other) {
    using T = typename Store<S>::T;
    const uint32_t tid = threadIdx.x, bd = blockDim.x, nx = (uint32_t)g.nx;
    const uint32_t wave0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid & ~63u));
    const int ys[3] = {y == g.ny - 1 ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
    const int zs[3] = {z == g.nz - 1 ? 0 : z + 1, z, z == 0 ? g.nz - 1 : z - 1};
    // group q = (e_x = -1, 0, 1) of (e_y, e_z); from a wall the opposite group of
    // the own row, its three populations in reverse order and not shifted
    auto bounce = [&](int q) { return WALLS && ((q % 3 == 2 && y == 0) || (q % 3 == 0 && y == g.ny - 1)); };
    const uint32_t gs = group_stride<T>(nx);
    constexpr uint32_t es = (uint32_t)sizeof(T);
    uint32_t off[9];   // misalignment of each group, in bytes
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const bool w = bounce(q);
        const T* A = short_row(src, g, w ? 24 - 3 * q : 3 * q, w ? y : ys[q % 3], w ? z : zs[q / 3]);
        off[q] = (uint32_t)((uintptr_t)A & 15u);
        const u32x4* base = (const u32x4*)((uintptr_t)A & ~(uintptr_t)15);
        const uint32_t n = (off[q] + 3u * nx * es + 15u) / 16u;
        // 3 nx values and a vector: within bd vectors of 4- or 2-byte values, 2 bd of FP64
        copy_vectors<es == 8 ? 2 : 1>(base, (unsigned char*)sm + es * q * gs, n, tid, wave0, bd);
    }
    other();
    wait_lds_copies();
    __syncthreads();
    // x - e_x, in bytes
    const uint32_t xs[3] = {es * (x + 1u >= nx ? 0u : x + 1u), es * (nx + x), es * (2u * nx + (x == 0u ? nx - 1u : x - 1u))};
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ix = i % 3, q = i / 3;
        t[i] = lds_at(sm, (es * q * gs + off[q]) + (bounce(q) ? es * (x + (uint32_t)(2 - ix) * nx) : xs[ix]));
    }
}

// ---------------------------------------------------------------- several rows per workgroup
// Short rows: the lanes of a workgroup take g.pack rows y, y + 1, ... of one z in
// turn, so that the row, unlike everywhere else, is the lane's own. Returns
// whether the lane has a cell (else x, y are some cell's). Grid: x over groups
// of g.pack rows, y over z.
__device__ __forceinline__ bool packed_cell(const Geom& g, int& x, int& y, int& z) {
    const uint32_t tid = threadIdx.x;
    const uint32_t r = (tid * g.packm) >> 16;   // tid / nx: exact for tid < 256 and nx <= 256
    x = (int)(tid - r * (uint32_t)g.nx);
    y = (int)(blockIdx.x * (uint32_t)g.pack + r);
    z = (int)blockIdx.y + g.zbase;
    const bool act = r < (uint32_t)g.pack && y < g.ny;
    if (!act) {
        x = 0;
        y = g.ny - 1;
    }
    return act;
}

// Plane i of an array in the populations' row layout at (x, y, z) + SGN e_i for
// all i, x and y the lane's own, z uniform: a row pointer per (plane, z) that
// is the same for the whole workgroup and 32-bit lane offsets, nine of them for
// the nine (e_x, e_y) (a z-plane of such rows is shorter than 2^32 bytes). The
// lanes of a row read it in one instruction, so the shifted reads touch no more
// lines than the others. WALLS: where y + SGN e_y lies beyond a wall, plane 26 - i of the
// cell itself.
template <int SGN, bool WALLS, bool NT, typename T>
__device__ __forceinline__ void gather_packed(const T* src, const Geom& g, int x, int y, int z, T (&t)[27]) {
    const uint32_t es = (uint32_t)sizeof(T), rl = 27u * (uint32_t)g.nx * es;
    const uint32_t xm = (uint32_t)(x == 0 ? g.nx - 1 : x - 1) * es, xp = (uint32_t)(x == g.nx - 1 ? 0 : x + 1) * es;
    const uint32_t ym = (uint32_t)(y == 0 ? g.ny - 1 : y - 1) * rl, yp = (uint32_t)(y == g.ny - 1 ? 0 : y + 1) * rl;
    const int zm = z == 0 ? g.nz - 1 : z - 1, zp = z == g.nz - 1 ? 0 : z + 1;
    const uint32_t xo[3] = {SGN < 0 ? xp : xm, (uint32_t)x * es, SGN < 0 ? xm : xp};
    const uint32_t yo[3] = {SGN < 0 ? yp : ym, (uint32_t)y * rl, SGN < 0 ? ym : yp};
    const int zo[3] = {SGN < 0 ? zp : zm, z, SGN < 0 ? zm : zp};
    auto at = [&](int i, int zz, uint32_t o) {
        const auto p = at_row(src + ((size_t)zz * g.ny * 27 + i) * g.nx, o);
        if constexpr (NT) return __builtin_nontemporal_load(p);
        else return *p;
    };
#pragma unroll
    for (int i = 0; i < 27; ++i) t[i] = at(i, zo[i / 9], yo[(i / 3) % 3] + xo[i % 3]);
    if constexpr (WALLS) {
        if (y == 0) {
#pragma unroll
            for (int i = 0; i < 27; ++i)
                if ((i / 3) % 3 == (SGN < 0 ? 2 : 0)) t[i] = at(26 - i, z, yo[1] + xo[1]);
        }
        if (y == g.ny - 1) {
#pragma unroll
            for (int i = 0; i < 27; ++i)
                if ((i / 3) % 3 == (SGN < 0 ? 0 : 2)) t[i] = at(26 - i, z, yo[1] + xo[1]);
        }
    }
}

template <typename R, bool FFIELD>
__device__ __forceinline__ void cell_force(const R* __restrict__ force, const Geom g, int c, const Launch<R>& L, R& Fx,
                                           R& Fy, R& Fz) {
    if constexpr (FFIELD) {
        Fx = force[c];
        Fy = force[(size_t)g.N + c];
        Fz = force[2 * (size_t)g.N + c];
    } else {
        (void)force; (void)g; (void)c;
        Fx = L.F[0];
        Fy = L.F[1];
        Fz = L.F[2];
    }
}

// ---------------------------------------------------------------- step
// The collision of one cell after its gather, and the store of its 27
// post-collision values (and, with SGS, of its sub-grid stress).
template <typename R, bool FFIELD, bool SB = false>
__device__ __forceinline__ void row_force(const R* __restrict__ force, const Geom g, const Launch<R>& L, int x, int y,
                                          int z, R (&F)[3]) {
    if constexpr (FFIELD) {
        const size_t row = (size_t)g.nx * ((size_t)y + (size_t)g.ny * z);   // uniform
        const uint32_t xb = (uint32_t)x * (uint32_t)sizeof(R);
#pragma unroll
        for (int d = 0; d < 3; ++d) F[d] = *row_at<SB>(force + (size_t)d * g.N + row, xb);
    } else {
        (void)force; (void)g; (void)x; (void)y; (void)z;
#pragma unroll
        for (int d = 0; d < 3; ++d) F[d] = L.F[d];
    }
}

// h[0..8], ls, ld: the z-line sums of the gathered populations (zline_sums).
// The collision, and the store of the sub-grid stress (SGS).
template <int S, bool LES, bool VAR, bool SGS, bool SB = false>
__device__ __forceinline__ void collide_cell(const Geom g, const Launch<typename Store<S>::R>& L, int x, int y, int z,
                                             typename Store<S>::R (&h)[27], const typename Store<S>::R (&ls)[9],
                                             const typename Store<S>::R (&ld)[9], const typename Store<S>::R (&F)[3],
                                             const typename Store<S>::R (&acc)[3],
                                             typename Store<S>::R* __restrict__ rs_next) {
    using R = typename Store<S>::R;
    R rho, ux, uy, uz;
    if constexpr (SGS) {
        R st[6];
        collide_lines<R, false, VAR, true, S == 3>(h, ls, ld, F[0], F[1], F[2], L.P, rho, ux, uy, uz, acc, st);
        const size_t row = (size_t)g.nx * ((size_t)y + (size_t)g.ny * z);   // uniform
        const uint32_t xb = (uint32_t)x * (uint32_t)sizeof(R);
#pragma unroll
        for (int k = 0; k < 6; ++k)
            __builtin_nontemporal_store(st[k], row_at<SB>(rs_next + (size_t)k * g.N + row, xb));
    } else {
        (void)acc; (void)rs_next; (void)x; (void)y; (void)z;
        collide_lines<R, LES, VAR, false, S == 3>(h, ls, ld, F[0], F[1], F[2], L.P, rho, ux, uy, uz);
    }
}
template <int S, bool LES, bool VAR, bool SGS, bool SB = false>
__device__ __forceinline__ void finish_cell(typename Store<S>::T* __restrict__ dst, const Geom g,
                                            const Launch<typename Store<S>::R>& L, int x, int y, int z,
                                            typename Store<S>::R (&h)[27], const typename Store<S>::R (&ls)[9],
                                            const typename Store<S>::R (&ld)[9], const typename Store<S>::R (&F)[3],
                                            const typename Store<S>::R (&acc)[3],
                                            typename Store<S>::R* __restrict__ rs_next) {
    using T = typename Store<S>::T;
    collide_cell<S, LES, VAR, SGS, SB>(g, L, x, y, z, h, ls, ld, F, acc, rs_next);
    const uint32_t xt = (uint32_t)x * (uint32_t)sizeof(T);
#pragma unroll
    for (int i = 0; i < 27; ++i)
        __builtin_nontemporal_store(to_store<S>(h[i], i, L.P.rho0), row_at<SB>(dst + row_base(g, i, y, z), xt));
}

// SGS: the sub-grid stress acts as a force (rs_prev read, rs_next written).
// XL: the width of the workgroup that covers each grid row (nx <= blockDim.x =
// XL), so that the x-shifted values go through LDS (gather_xlds); 0: each lane
// loads its shifted values itself (gather), looping over x when the grid has
// one workgroup per row (g.rowloop).
// FP16 storage is bound by instruction issue: five waves per SIMD (at most 96
// vector registers, which it fits without spilling) measured 3 % faster; the
// other modes gained nothing or spilled.
template <int S, bool WALLS, bool LES, bool FFIELD, bool VAR, bool SGS = false, int XL = 256>
__global__ void __launch_bounds__(256, (S == 3 && !SGS) ? 5 : 1) k_step(const typename Store<S>::T* __restrict__ src,
                                              typename Store<S>::T* __restrict__ dst,
                                              const typename Store<S>::R* __restrict__ force, const Geom g,
                                              const Launch<typename Store<S>::R> L,
                                              const typename Store<S>::R* __restrict__ rs_prev = nullptr,
                                              typename Store<S>::R* __restrict__ rs_next = nullptr) {
    using R = typename Store<S>::R;
    // Scalar-base addressing (at_row) for FP16 storage, which is bound by
    // instruction issue: 63 fewer vector instructions per wave, 4.8 % faster at
    // 512^3. The memory-bound modes measured 0.4-2 % slower with it (the extra
    // scalar work) and keep the vector addresses.
    constexpr bool SB = S == 3;
    int bx, y, z;
    block_coords(g.xcd, bx, y, z);
    y = g.ybase + y * g.ystride;
    z += g.zbase;
    if constexpr (XL != 0) {
        const int x = threadIdx.x;
        const bool act = x < g.nx;
        // the stress and force loads go out with the population loads, in the
        // same memory round trip
        R sv[SGS ? 18 : 1], F[3];
        if constexpr (SGS) sgs_load<R, SB>(rs_prev, g, act ? x : 0, y, z, sv);
        row_force<R, FFIELD, SB>(force, g, L, act ? x : 0, y, z, F);
        typename Store<S>::T t[27];
        gather_xlds<S, SB, WALLS, XL>(src, g, x, act, y, z, t, [&]() {
            if constexpr (FFIELD) {
#pragma unroll
                for (int d = 0; d < 3; ++d) asm volatile("" : "+v"(F[d]));
            }
            if constexpr (SGS) {
#pragma unroll
                for (int k = 0; k < 18; ++k) asm volatile("" : "+v"(sv[k]));
            }
        });
        R h[27], ls[9], ld[9];
        stored_line_sums<S, WALLS>(t, g, y, L, h, ls, ld);
        R acc[3];
        if constexpr (SGS) sgs_combine(sv, acc);
        if (act) finish_cell<S, LES, VAR, SGS, SB>(dst, g, L, x, y, z, h, ls, ld, F, acc, rs_next);
    } else {
        if constexpr (SB) {
            if (!g.rowloop) {   // one cell per lane, no loop around the accesses
                const int x = bx * blockDim.x + threadIdx.x;
                if (x < g.nx) {
                    R acc[3], F[3];
                    if constexpr (SGS) sgs_accel<R, true>(rs_prev, g, x, y, z, acc);
                    R h[27], ls[9], ld[9];
                    gather<S, WALLS, 0, true>(src, g, x, y, z, L, h);
                    row_force<R, FFIELD, true>(force, g, L, x, y, z, F);
                    zline_sums(h, ls, ld);
                    finish_cell<S, LES, VAR, SGS, true>(dst, g, L, x, y, z, h, ls, ld, F, acc, rs_next);
                }
                return;
            }
        }
        for (int x = bx * blockDim.x + threadIdx.x; x < g.nx; x += gridDim.x * blockDim.x) {
            R acc[3], F[3];
            if constexpr (SGS) sgs_accel(rs_prev, g, x, y, z, acc);
            R h[27], ls[9], ld[9];
            gather<S, WALLS, 0>(src, g, x, y, z, L, h);
            row_force<R, FFIELD>(force, g, L, x, y, z, F);
            zline_sums(h, ls, ld);
            finish_cell<S, LES, VAR, SGS>(dst, g, L, x, y, z, h, ls, ld, F, acc, rs_next);
        }
    }
}

// ---------------------------------------------------------------- step, whole rows through LDS
// The step on rows that do not start on cache lines (or are wider than 256
// cells): one workgroup per grid row, and the row's populations go through LDS
// in both directions, in (gather_rows) as nine blocks of 3 nx values, out as
// the one block of 27 nx values that the 27 rows of a cell row are.
// Bound by HBM; per-lane accesses to such rows touch three lines instead of two
// per wave in most rows and write partial lines, which non-temporal stores send
// to memory one by one. Vectors through registers instead of straight into LDS:
// 383 us per step at 250 x 200 x 200 FP32, against 367-374.
// DIRECT: rows that do start on cache lines: each lane stores its own values (no
// partial lines to avoid, and one barrier less).
template <int S, bool WALLS, bool LES, bool FFIELD, bool VAR, bool SGS, bool DIRECT>
__global__ void __launch_bounds__(512) k_step_row(const typename Store<S>::T* __restrict__ src,
                                                  typename Store<S>::T* __restrict__ dst,
                                                  const typename Store<S>::R* __restrict__ force, const Geom g,
                                                  const Launch<typename Store<S>::R> L,
                                                  const typename Store<S>::R* __restrict__ rs_prev = nullptr,
                                                  typename Store<S>::R* __restrict__ rs_next = nullptr) {
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    extern __shared__ __align__(16) unsigned char lds_bytes[];
    T* const sm = (T*)lds_bytes;
    int bx, y, z;
    block_coords(g.xcd, bx, y, z);
    z += g.zbase;
    const uint32_t tid = threadIdx.x, nx = (uint32_t)g.nx;
    const bool act = tid < nx;
    const uint32_t x = act ? tid : 0u;
    R sv[SGS ? 18 : 1], F[3];
    T t[27];
    gather_rows<S, WALLS>(src, g, x, y, z, sm, t, [&]() {
        if constexpr (SGS) sgs_load<R, false>(rs_prev, g, (int)x, y, z, sv);
        row_force<R, FFIELD, false>(force, g, L, (int)x, y, z, F);
    });
    R h[27], ls[9], ld[9];
    stored_line_sums<S, WALLS>(t, g, y, L, h, ls, ld);
    R acc[3];
    if constexpr (SGS) sgs_combine(sv, acc);
    if constexpr (DIRECT) {
        if (act) finish_cell<S, LES, VAR, SGS, S == 3>(dst, g, L, (int)x, y, z, h, ls, ld, F, acc, rs_next);
    } else {
        // (unguarded, the collision of the idle lanes cost 15 vector registers)
        if (act) collide_cell<S, LES, VAR, SGS>(g, L, (int)x, y, z, h, ls, ld, F, acc, rs_next);
        __syncthreads();   // every lane has read its values: the LDS takes the results
        T* const D = short_row(dst, g, 0, y, z);
        const uint32_t o = (uint32_t)((uintptr_t)D & 15u) / (uint32_t)sizeof(T);
        if (act) {
            uint32_t at = (o + x) * (uint32_t)sizeof(T);   // stepped row by row: 27 addresses held at once spilled
#pragma unroll
            for (int i = 0; i < 27; ++i) {
                lds_at(sm, at) = to_store<S>(h[i], i, L.P.rho0);
                at += nx * (uint32_t)sizeof(T);
                asm volatile("" : "+v"(at));
            }
        }
        __syncthreads();
        store_block<T>(D, o, 27u * nx, sm, tid, blockDim.x);
    }
}

// ---------------------------------------------------------------- step, several rows per workgroup
// The step on short rows, which leave lanes of a row's own workgroup idle: bound
// by instruction issue and latency there, by HBM when the lanes are full (20 x
// 200 x 200 FP32 48.7 us a step by row, 34.4 packed, 5.3 TB/s; 32 x 200 x 200 FP16
// 42.0 and 28.1). No exchange of shifted values: gather_packed.
// DIRECT: rows of whole cache lines: each lane stores its own values; else the
// workgroup's rows, one block of 27 nx values each and one after the other, go
// through LDS and are stored in whole vectors.
template <int S, bool WALLS, bool LES, bool FFIELD, bool VAR, bool SGS, bool DIRECT>
__global__ void __launch_bounds__(256) k_step_packed(const typename Store<S>::T* __restrict__ src,
                                                     typename Store<S>::T* __restrict__ dst,
                                                     const typename Store<S>::R* __restrict__ force, const Geom g,
                                                     const Launch<typename Store<S>::R> L,
                                                     const typename Store<S>::R* __restrict__ rs_prev = nullptr,
                                                     typename Store<S>::R* __restrict__ rs_next = nullptr) {
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    int x, y, z;
    const bool act = packed_cell(g, x, y, z);
    T t[27];
    R sv[SGS ? 18 : 1], F[3], acc[3];
    gather_packed<-1, WALLS, DIRECT>(src, g, x, y, z, t);
    if constexpr (SGS) sgs_load<R, false>(rs_prev, g, x, y, z, sv);
    row_force<R, FFIELD, false>(force, g, L, x, y, z, F);
    if constexpr (DIRECT) {
        if (!act) return;
    }
    const uint32_t nx = (uint32_t)g.nx;
    extern __shared__ __align__(16) unsigned char lds_bytes[];
    T* const sm = (T*)lds_bytes;
    const int y0 = (int)(blockIdx.x * (uint32_t)g.pack);
    T* const D = short_row(dst, g, 0, y0, z);   // the workgroup's block
    const uint32_t o = (uint32_t)((uintptr_t)D & 15u) / (uint32_t)sizeof(T);
    if (act) {
        R h[27], ls[9], ld[9];
        stored_line_sums<S, WALLS>(t, g, y, L, h, ls, ld);
        if constexpr (SGS) sgs_combine(sv, acc);
        collide_cell<S, LES, VAR, SGS>(g, L, x, y, z, h, ls, ld, F, acc, rs_next);
        uint32_t at = (uint32_t)(y - y0) * 27u * nx + (uint32_t)x;
        if constexpr (DIRECT) {
            at *= (uint32_t)sizeof(T);
#pragma unroll
            for (int i = 0; i < 27; ++i)
                __builtin_nontemporal_store(to_store<S>(h[i], i, L.P.rho0), at_row(D + (size_t)i * nx, at));
        } else {
            at = (at + o) * (uint32_t)sizeof(T);
#pragma unroll
            for (int i = 0; i < 27; ++i) {
                lds_at(sm, at) = to_store<S>(h[i], i, L.P.rho0);
                at += nx * (uint32_t)sizeof(T);
                asm volatile("" : "+v"(at));
            }
        }
    }
    if constexpr (!DIRECT) {
        __syncthreads();
        const uint32_t rows = (uint32_t)(g.ny - y0 < g.pack ? g.ny - y0 : g.pack);
        store_block<T>(D, o, rows * 27u * nx, sm, threadIdx.x, blockDim.x);
    }
}

// ---------------------------------------------------------------- FP16 step, two cells per lane
// Non-temporal store of a 32-bit pair at a workgroup-uniform row pointer plus a
// lane offset. (Written out as an inline-assembly store with a scalar base it
// measured 0.7 % faster, but the compiler's hazard handling does not see the
// scalar base register of an assembly statement: the five wait states a
// memory instruction needs after v_readfirstlane writes its base register are
// then missing, and a store may use a stale address. Kept as compiler code.)
__device__ __forceinline__ void store_pair(uint32_t* row, uint32_t lane_bytes, uint32_t v) {
    __builtin_nontemporal_store(v, at_row(row, lane_bytes));
}

// FP16-shifted storage is bound by instruction issue rather than by HBM: the
// loads, stores, conversions and addresses are a large part of its work. Here
// each lane takes the two adjacent cells x = 2t and 2t + 1 of a periodic row
// (nx even, nx <= 2 blockDim.x, one workgroup per row): every population row is
// read and written as aligned 32-bit pairs, half the memory instructions of one
// cell per lane. Of the 18 rows with e_x != 0 each pair needs one value from
// the neighbouring pair (x - 1 for e_x = +1, x + 2 for e_x = -1), exchanged
// through LDS as in gather_xlds. The two cells then collide one after the
// other with the same arithmetic as k_step, so the results are bitwise those of
// the one-cell kernels.
template <bool LES, bool FFIELD, bool VAR>
__global__ void __launch_bounds__(256) k_step_f16pair(const _Float16* __restrict__ src, _Float16* __restrict__ dst,
                                                      const float* __restrict__ force, const Geom g,
                                                      const Launch<float> L) {
    using T = _Float16;
    __shared__ uint16_t sm[18][256];
    int bx, y, z;
    block_coords(g.xcd, bx, y, z);
    y = g.ybase + y * g.ystride;
    z += g.zbase;
    const int t = threadIdx.x;
    const int np = g.nx >> 1;   // pairs in the row
    const bool act = t < np;
    const int tp = act ? t : 0;   // idle lanes read pair 0 and fill LDS columns nobody reads
    const int ys[3] = {y == g.ny - 1 ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
    const int zs[3] = {z == g.nz - 1 ? 0 : z + 1, z, z == 0 ? g.nz - 1 : z - 1};
    const uint32_t rb = (uint32_t)g.nx * (uint32_t)sizeof(T);
    const uint32_t xt = (uint32_t)tp * 4u;
    uint32_t raw[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ix = i % 3, iy = (i / 3) % 3, iz = i / 9;
        const T* grp = src + row_base(g, i - ix, ys[iy], zs[iz]);
        // non-temporal: every pair is read once per step (measured 3.5 % faster at 512^3)
        raw[i] = __builtin_nontemporal_load(at_row((const uint32_t*)grp, xt + (uint32_t)ix * rb));
    }
    float F[2][3];
    if constexpr (FFIELD) {
        const size_t row = (size_t)g.nx * ((size_t)y + (size_t)g.ny * z);   // uniform
        const uint32_t xb = (uint32_t)tp * 8u;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float2_t v = *at_row((const float2_t*)(force + (size_t)d * g.N + row), xb);
            F[0][d] = v.x;
            F[1][d] = v.y;
        }
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) F[0][d] = F[1][d] = L.F[d];
    }
    // e_x = -1 (ix = 0, source x + 1): the pair to the left needs this pair's
    // low value; e_x = +1 (ix = 2, source x - 1): the pair to the right needs
    // the high value
#pragma unroll
    for (int i = 0; i < 27; ++i)
        if (i % 3 != 1) sm[(i / 3) * 2 + (i % 3) / 2][t] = (uint16_t)(i % 3 == 0 ? raw[i] & 0xffffu : raw[i] >> 16);
#pragma unroll
    for (int i = 1; i < 27; i += 3) asm volatile("" : "+v"(raw[i]));
    if constexpr (FFIELD) {
#pragma unroll
        for (int d = 0; d < 3; ++d) asm volatile("" : "+v"(F[0][d]), "+v"(F[1][d]));
    }
    __syncthreads();
    const int tn = tp + 1 == np ? 0 : tp + 1, tv = tp == 0 ? np - 1 : tp - 1;
    float rho, ux, uy, uz;
    // cell x = 2t: e_x = 0 from the low halves, e_x = -1 from the high halves,
    // e_x = +1 the left pair's high values (LDS)
    float h[27], ls[9], ld[9];
#pragma unroll
    for (int l = 0; l < 9; ++l) {
        const int ix = l % 3;
        if (ix == 1) mix_line<0>(raw[l], raw[l + 9], raw[l + 18], ls[l], ld[l], h[l]);
        else if (ix == 0) mix_line<1>(raw[l], raw[l + 9], raw[l + 18], ls[l], ld[l], h[l]);
        else {
            const int k = (l / 3) * 2 + 1;   // LDS row of population i = l + 9 iz: (i / 3) * 2 + 1
            mix_line<0>(sm[k][tv], sm[k + 6][tv], sm[k + 12][tv], ls[l], ld[l], h[l]);
        }
    }
    collide_lines<float, LES, VAR, false, true>(h, ls, ld, F[0][0], F[0][1], F[0][2], L.P, rho, ux, uy, uz);
    // cell x = 2t + 1: e_x = 0 from the high halves, e_x = +1 from the low
    // halves, e_x = -1 the right pair's low values (LDS)
    float h2[27];
#pragma unroll
    for (int l = 0; l < 9; ++l) {
        const int ix = l % 3;
        if (ix == 1) mix_line<1>(raw[l], raw[l + 9], raw[l + 18], ls[l], ld[l], h2[l]);
        else if (ix == 2) mix_line<0>(raw[l], raw[l + 9], raw[l + 18], ls[l], ld[l], h2[l]);
        else {
            const int k = (l / 3) * 2;
            mix_line<0>(sm[k][tn], sm[k + 6][tn], sm[k + 12][tn], ls[l], ld[l], h2[l]);
        }
    }
    collide_lines<float, LES, VAR, false, true>(h2, ls, ld, F[1][0], F[1][1], F[1][2], L.P, rho, ux, uy, uz);
    if (act) {
#pragma unroll
        for (int i = 0; i < 27; ++i) store_pair((uint32_t*)(dst + row_base(g, i, y, z)), xt, pack_f16(h[i], h2[i]));
    }
}

// ---------------------------------------------------------------- in-place streaming
// One buffer, two kinds of step (the AA pattern of Bailey et al. 2009):
//   even: read fbar_i(x) from plane i of x, collide, write fbar~_i(x) to plane
//         26 - i of x (every access is to the thread's own cell);
//   odd:  read fbar_i(x) from plane 26 - i of x - e_i (gather MODE 2), collide,
//         write fbar~_i(x) to plane i of x + e_i, or, towards a wall, to plane
//         26 - i of x itself (the next even read adds the wall term);
// after an odd step the buffer is back in the natural arrangement. Each
// location is read and written by the same thread within a step, so the
// update is race-free in place. The collision and its arithmetic are those of
// the two-buffer step, so results are bitwise identical.
template <int S, bool WALLS, bool LES, bool FFIELD, bool VAR, bool ODD>
__global__ void __launch_bounds__(256) k_step_inplace(typename Store<S>::T* buf,
                                                      const typename Store<S>::R* __restrict__ force, const Geom g,
                                                      const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    int bx, y, z;
    block_coords(g.xcd, bx, y, z);
    y = g.ybase + y * g.ystride;
    z += g.zbase;
    for (int x = bx * blockDim.x + threadIdx.x; x < g.nx; x += gridDim.x * blockDim.x) {
        R h[27];
        if constexpr (ODD) gather<S, WALLS, 2>(buf, g, x, y, z, L, h);
        else gather<S, WALLS, 1>(buf, g, x, y, z, L, h);
        const size_t row = (size_t)g.nx * ((size_t)y + (size_t)g.ny * z);
        R Fx, Fy, Fz;
        if constexpr (FFIELD) {
            Fx = force[row + x];
            Fy = force[(size_t)g.N + row + x];
            Fz = force[2 * (size_t)g.N + row + x];
        } else {
            Fx = L.F[0];
            Fy = L.F[1];
            Fz = L.F[2];
        }
        R rho, ux, uy, uz;
        collide<R, LES, VAR, false, S == 3>(h, Fx, Fy, Fz, L.P, rho, ux, uy, uz);
        if constexpr (!ODD) {
            const uint32_t xt = (uint32_t)x * (uint32_t)sizeof(T);
#pragma unroll
            for (int i = 0; i < 27; ++i)
                __builtin_nontemporal_store(to_store<S>(h[i], 26 - i, L.P.rho0),
                                            (T*)((char*)(buf + row_base(g, 26 - i, y, z)) + xt));
        } else {
            const int xs[3] = {x == 0 ? g.nx - 1 : x - 1, x, x == g.nx - 1 ? 0 : x + 1};   // x + ex
            const int ys[3] = {y == 0 ? g.ny - 1 : y - 1, y, y == g.ny - 1 ? 0 : y + 1};
            const int zs[3] = {z == 0 ? g.nz - 1 : z - 1, z, z == g.nz - 1 ? 0 : z + 1};
            // one uniform pointer per target row (ey, ez), the row-in-group offset
            // folded into the per-lane offsets (as in the gather)
            uint32_t vo[3];
#pragma unroll
            for (int ix = 0; ix < 3; ++ix) vo[ix] = ((uint32_t)xs[ix] + (uint32_t)ix * (uint32_t)g.nx) * (uint32_t)sizeof(T);
#pragma unroll
            for (int i = 0; i < 27; ++i) {
                const int ix = i % 3, iy = (i / 3) % 3, iz = i / 9;
                const bool wall = WALLS && ((iy == 0 && y == 0) || (iy == 2 && y == g.ny - 1));
                T* const grp = buf + row_base(g, wall ? 24 - (i - ix) : i - ix, wall ? y : ys[iy], wall ? z : zs[iz]);
                const uint32_t o = wall ? ((uint32_t)x + (uint32_t)(2 - ix) * (uint32_t)g.nx) * (uint32_t)sizeof(T) : vo[ix];
                __builtin_nontemporal_store(to_store<S>(h[i], i, L.P.rho0), (T*)((char*)grp + o));   // w_i = w_{26-i}
            }
        }
    }
}

// The same with several rows per workgroup (packed_cell), for short rows. On odd
// steps plane i of x + e_i holds fbar_{26-i} and takes fbar~_i (towards a wall,
// plane 26 - i of the cell itself): the lanes of a row write all of it in one
// instruction, shifted or not.
template <int S, bool WALLS, bool LES, bool FFIELD, bool VAR, bool ODD>
__global__ void __launch_bounds__(256) k_step_inplace_packed(typename Store<S>::T* buf,
                                                             const typename Store<S>::R* __restrict__ force,
                                                             const Geom g, const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    int x, y, z;
    if (!packed_cell(g, x, y, z)) return;
    const uint32_t es = (uint32_t)sizeof(T), rl = 27u * (uint32_t)g.nx * es, own = (uint32_t)y * rl + (uint32_t)x * es;
    T* const plane = buf + (size_t)z * g.ny * 27 * g.nx;   // plane 0 of this z, y = 0
    T t[27];
    if constexpr (ODD) {
        T s[27];
        gather_packed<1, WALLS, false>(buf, g, x, y, z, s);
#pragma unroll
        for (int i = 0; i < 27; ++i) t[i] = s[26 - i];
    } else {
#pragma unroll
        for (int i = 0; i < 27; ++i) t[i] = *at_row(plane + (size_t)i * g.nx, own);
    }
    R F[3], h[27], ls[9], ld[9], acc[3];
    row_force<R, FFIELD, false>(force, g, L, x, y, z, F);
    stored_line_sums<S, WALLS>(t, g, y, L, h, ls, ld);
    collide_cell<S, LES, VAR, false>(g, L, x, y, z, h, ls, ld, F, acc, nullptr);
    if constexpr (!ODD) {
#pragma unroll
        for (int i = 0; i < 27; ++i) *at_row(plane + (size_t)(26 - i) * g.nx, own) = to_store<S>(h[i], i, L.P.rho0);
    } else {
        const uint32_t xo[3] = {(uint32_t)(x == 0 ? g.nx - 1 : x - 1) * es, (uint32_t)x * es,
                                (uint32_t)(x == g.nx - 1 ? 0 : x + 1) * es};
        const uint32_t yo[3] = {(uint32_t)(y == 0 ? g.ny - 1 : y - 1) * rl, (uint32_t)y * rl,
                                (uint32_t)(y == g.ny - 1 ? 0 : y + 1) * rl};
        const int zo[3] = {z == 0 ? g.nz - 1 : z - 1, z, z == g.nz - 1 ? 0 : z + 1};
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int iy = (i / 3) % 3;
            const T v = to_store<S>(h[i], i, L.P.rho0);   // w_i = w_{26-i}
            if (WALLS && ((iy == 0 && y == 0) || (iy == 2 && y == g.ny - 1)))
                *at_row(plane + (size_t)(26 - i) * g.nx, own) = v;
            else
                *at_row(buf + ((size_t)zo[i / 9] * g.ny * 27 + i) * g.nx, yo[iy] + xo[i % 3]) = v;
        }
    }
}

// The same on whole rows through LDS (one workgroup per row, lane = cell). The
// locations of a row's cells are, on even steps, the row's own block of 27 nx
// values, on odd ones nine blocks of 3 nx values (the three planes that differ
// only in e_x of a row (y + e_y, z + e_z)); each is copied into LDS, updated
// there and stored back as 16-byte vectors, at any alignment. A lane reads
// and writes the same 27 places, shifted by e_x on odd steps: plane i of
// x + e_i holds fbar_{26-i} and takes fbar~_i. Towards a wall the place is plane
// 26 - i of the cell itself (the group opposite, in reverse order, not
// shifted). So walls need no launch of their own, and the odd step no partial
// lines: by lanes it wrote 109 to 115 bytes a cell of 108 (FP32).
template <int S, bool WALLS, bool LES, bool FFIELD, bool VAR, bool ODD>
__global__ void __launch_bounds__(512) k_step_inplace_row(typename Store<S>::T* buf,
                                                          const typename Store<S>::R* __restrict__ force, const Geom g,
                                                          const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    using T = typename Store<S>::T;
    constexpr uint32_t V = 16 / sizeof(T);
    extern __shared__ __align__(16) unsigned char lds_bytes[];
    T* const sm = (T*)lds_bytes;
    int bx, y, z;
    block_coords(g.xcd, bx, y, z);
    const uint32_t tid = threadIdx.x, bd = blockDim.x, nx = (uint32_t)g.nx;
    const uint32_t wave0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid & ~63u));
    const bool act = tid < nx;
    const uint32_t x = act ? tid : 0u;
    constexpr int NB = ODD ? 9 : 1;
    const uint32_t len = (ODD ? 3u : 27u) * nx, gs = group_stride<T>(nx);
    const int ys[3] = {y == 0 ? g.ny - 1 : y - 1, y, y == g.ny - 1 ? 0 : y + 1};   // y + e_y
    const int zs[3] = {z == 0 ? g.nz - 1 : z - 1, z, z == g.nz - 1 ? 0 : z + 1};
    auto bounce = [&](int q) { return ODD && WALLS && ((q % 3 == 0 && y == 0) || (q % 3 == 2 && y == g.ny - 1)); };
    T* A[NB];
    uint32_t off[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const bool w = bounce(q);
        A[q] = ODD ? buf + row_base(g, w ? 24 - 3 * q : 3 * q, w ? y : ys[q % 3], w ? z : zs[q / 3])
                   : buf + row_base(g, 0, y, z);
        off[q] = (uint32_t)((uintptr_t)A[q] & 15u) / (uint32_t)sizeof(T);
        const u32x4* base = (const u32x4*)((uintptr_t)A[q] & ~(uintptr_t)15);
        const uint32_t n = (off[q] + len + V - 1u) / V;
        for (uint32_t k = 0; k < n; k += bd)
            if (tid + k < n) copy16_to_lds(at_row(base, (tid + k) * 16u), lds_bytes + 16u * (q * (gs / V) + k + wave0));
    }
    R F[3];
    row_force<R, FFIELD, false>(force, g, L, (int)x, y, z, F);
    wait_lds_copies();
    __syncthreads();
    // where plane i's place is (c the lane's cell)
    auto place = [&](int i, uint32_t c) {
        const int ix = i % 3, q = i / 3;
        if constexpr (!ODD) return off[0] + (uint32_t)i * nx + c;
        const uint32_t xs[3] = {c == 0u ? nx - 1u : c - 1u, nx + c, 2u * nx + (c + 1u >= nx ? 0u : c + 1u)};
        return q * gs + off[q] + (bounce(q) ? c + (uint32_t)(2 - ix) * nx : xs[ix]);
    };
    if (act) {
        T t[27];
#pragma unroll
        for (int i = 0; i < 27; ++i) t[i] = sm[place(ODD ? 26 - i : i, x)];
        R h[27], ls[9], ld[9], acc[3];
        stored_line_sums<S, WALLS>(t, g, y, L, h, ls, ld);
        collide_cell<S, LES, VAR, false>(g, L, (int)x, y, z, h, ls, ld, F, acc, nullptr);
        uint32_t c = x;   // the places are formed again: held over the collision they cost 27 registers
        asm volatile("" : "+v"(c));
#pragma unroll
        for (int i = 0; i < 27; ++i) sm[place(ODD ? i : 26 - i, c)] = to_store<S>(h[i], i, L.P.rho0);   // w_i = w_{26-i}
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NB; ++q) store_block<T>(A[q], off[q], len, sm + q * gs, tid, bd);
}

// ---------------------------------------------------------------- scatter of canonical populations
// Writes canonical fbar(n) at cell (x,y,z) into the internal (pull) layout:
// population i goes to the upstream cell x - e_i, or, when that is a wall, to
// the opposite plane of the same cell minus the wall term.
template <int S, bool WALLS, typename R = typename Store<S>::R>
__device__ __forceinline__ void scatter(typename Store<S>::T* __restrict__ dst, const Geom g, int x, int y, int z,
                                        const Launch<R>& L, const R (&h)[27]) {
    if (g.aa) {   // in-place streaming: a state is set in the natural (even) arrangement,
                  // populations from a wall without their wall term
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            R v = h[i];
            if constexpr (WALLS) {
                const int iy = (i / 3) % 3;
                const bool from_lo = (iy == 2) && (y == 0);
                const bool from_hi = (iy == 0) && (y == g.ny - 1);
                if (from_lo || from_hi) v = sub_rn(v, from_lo ? L.wt_lo[i] : L.wt_hi[i]);
            }
            dst[row_base(g, i, y, z) + x] = to_store<S>(v, i, L.P.rho0);
        }
        return;
    }
    const int xs[3] = {x == g.nx - 1 ? 0 : x + 1, x, x == 0 ? g.nx - 1 : x - 1};
    const int ys[3] = {y == g.ny - 1 ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
    const int zs[3] = {z == g.nz - 1 ? 0 : z + 1, z, z == 0 ? g.nz - 1 : z - 1};
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ix = i % 3, iy = (i / 3) % 3, iz = i / 9;
        if constexpr (WALLS) {
            const bool from_lo = (iy == 2) && (y == 0);
            const bool from_hi = (iy == 0) && (y == g.ny - 1);
            if (from_lo || from_hi) {
                const int o = 26 - i;
                const R v = sub_rn(h[i], from_lo ? L.wt_lo[i] : L.wt_hi[i]);
                dst[row_base(g, o, y, z) + x] = to_store<S>(v, o, L.P.rho0);
                continue;
            }
        }
        dst[row_base(g, i, ys[iy], zs[iz]) + xs[ix]] = to_store<S>(h[i], i, L.P.rho0);
    }
}

// The same for a workgroup that holds a whole grid row (lane = cell, h of lanes
// with `act`), through LDS: scattered by the lanes, the populations with e_x != 0
// write rows shifted by one value, partial lines at every wave's ends and, where
// rows do not start on cache lines, everywhere. Here the three populations that
// go to one target row, a contiguous block, are put together in LDS (`sm`, 3
// group_stride values) and stored in whole vectors, the targets of one e_z at
// a time. Before / after, us: start of 256^3 FP32 449 / 411, of
// 300 x 181 x 90 FP32-shifted 274 / 124, of 187 x 151 x 133 FP16 134 / 69;
// set_populations (FP64 values) of 300 x 181 x 90 443 / 301.
template <int S, bool WALLS, typename R = typename Store<S>::R>
__device__ __forceinline__ void push_rows(typename Store<S>::T* __restrict__ dst, const Geom g, uint32_t x, bool act,
                                          int y, int z, const Launch<R>& L, const R (&h)[27],
                                          typename Store<S>::T* sm) {
    using T = typename Store<S>::T;
    const uint32_t nx = (uint32_t)g.nx, gs = group_stride<T>(nx);
    const int ys[3] = {y == g.ny - 1 ? 0 : y + 1, y, y == 0 ? g.ny - 1 : y - 1};
    const int zs[3] = {z == g.nz - 1 ? 0 : z + 1, z, z == 0 ? g.nz - 1 : z - 1};
    const bool own = g.aa != 0;   // in place: every population stays in the cell's own rows
    const uint32_t xs[3] = {own ? x : (x + 1u >= nx ? 0u : x + 1u), nx + x,
                            2u * nx + (own ? x : (x == 0u ? nx - 1u : x - 1u))};
#pragma unroll
    for (int iz = 0; iz < 3; ++iz) {
        T* D[3];
        uint32_t o[3];
#pragma unroll
        for (int iy = 0; iy < 3; ++iy) {
            const int q = 3 * iz + iy;
            const bool lo = WALLS && iy == 2 && y == 0, hi = WALLS && iy == 0 && y == g.ny - 1;
            const bool bounce = (lo || hi) && !own;
            D[iy] = dst + row_base(g, bounce ? 24 - 3 * q : 3 * q, own || bounce ? y : ys[iy], own || bounce ? z : zs[iz]);
            o[iy] = (uint32_t)((uintptr_t)D[iy] & 15u) / (uint32_t)sizeof(T);
            if (act) {
#pragma unroll
                for (int ix = 0; ix < 3; ++ix) {
                    const int i = 3 * q + ix;
                    R v = h[i];
                    if (lo || hi) v = sub_rn(v, lo ? L.wt_lo[i] : L.wt_hi[i]);
                    // w_i = w_{26-i}: the shift of the stored value is the same
                    sm[iy * gs + o[iy] + (bounce ? (uint32_t)(2 - ix) * nx + x : xs[ix])] = to_store<S>(v, i, L.P.rho0);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int iy = 0; iy < 3; ++iy) store_block<T>(D[iy], o[iy], 3u * nx, sm + iy * gs, threadIdx.x, blockDim.x);
        if (iz < 2) __syncthreads();
    }
}

// Writes h of cell (x, y, z): ROWS, through LDS by the workgroup that covers the
// row, else by each lane for itself.
template <int S, bool WALLS, bool ROWS, typename R = typename Store<S>::R>
__device__ __forceinline__ void put_state(typename Store<S>::T* __restrict__ dst, const Geom g, int x, bool act, int y, int z,
                                          const Launch<R>& L, const R (&h)[27]) {
    if constexpr (ROWS) {
        extern __shared__ __align__(16) unsigned char lds_bytes[];
        push_rows<S, WALLS>(dst, g, (uint32_t)x, act, y, z, L, h, (typename Store<S>::T*)lds_bytes);
    } else {
        if (act) scatter<S, WALLS>(dst, g, x, y, z, L, h);
    }
}

template <int S, bool WALLS, bool FFIELD, bool ROWS>
__global__ void __launch_bounds__(ROWS ? 512 : 256) k_init_equilibrium(typename Store<S>::T* __restrict__ dst,
                                                          const typename Store<S>::R* __restrict__ force,
                                                          const void* __restrict__ rho_in, const void* __restrict__ u_in,
                                                          int dt, const Geom g, const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y, z = blockIdx.z;
    const bool act = x < g.nx;
    R h[27];
    if (act) {
        const int c = x + g.nx * (y + g.ny * z);
        const R rho = rho_in ? static_cast<R>(as_double(rho_in, dt, c)) : L.P.rho0;
        const R ux = static_cast<R>(as_double(u_in, dt, c));
        const R uy = static_cast<R>(as_double(u_in, dt, (size_t)g.N + c));
        const R uz = static_cast<R>(as_double(u_in, dt, 2 * (size_t)g.N + c));
        R Fx, Fy, Fz;
        cell_force<R, FFIELD>(force, g, c, L, Fx, Fy, Fz);
        equilibrium(h, rho, ux, uy, uz, Fx, Fy, Fz, L.P.rho0, L.P.rc != 0);
    }
    put_state<S, WALLS, ROWS>(dst, g, x, act, y, z, L, h);
}

template <int S, bool WALLS, bool ROWS>
__global__ void __launch_bounds__(ROWS ? 512 : 256) k_set_populations(typename Store<S>::T* __restrict__ dst,
                                                         const void* __restrict__ f, int dt, const Geom g,
                                                         const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y, z = blockIdx.z;
    const bool act = x < g.nx;
    R h[27];
    if (act) {
        const int c = x + g.nx * (y + g.ny * z);
#pragma unroll
        for (int i = 0; i < 27; ++i)
            h[i] = static_cast<R>(as_double(f, dt, (size_t)i * g.N + c) - (double)L.P.rho0 * (double)w27<double>(i));
    }
    put_state<S, WALLS, ROWS>(dst, g, x, act, y, z, L, h);
}

// ---------------------------------------------------------------- read-out
// Canonical populations into out0 (27 planes), or, with MOMENTS, rho into out0
// (1 plane) and u into out1 (3 planes), as OUT values. ROWS: the workgroup
// covers the row and gathers through LDS. NT: non-temporal stores (read_non_temporal).
template <int S, bool WALLS, bool FFIELD, bool MOMENTS, bool ROWS, bool NT, typename OUT>
__global__ void __launch_bounds__(ROWS ? 512 : 256) k_read(const typename Store<S>::T* __restrict__ src,
                                              const typename Store<S>::R* __restrict__ force, OUT* __restrict__ out0,
                                              OUT* __restrict__ out1, const Geom g,
                                              const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y, z = blockIdx.z;
    R h[27];
    if constexpr (ROWS) {
        extern __shared__ __align__(16) unsigned char lds_bytes[];
        typename Store<S>::T t[27];
        gather_rows<S, WALLS>(src, g, x < g.nx ? (uint32_t)x : 0u, y, z, (typename Store<S>::T*)lds_bytes, t, []() {});
        if (x >= g.nx) return;
        stored_devs<S, WALLS>(t, g, y, L, h);
    } else {
        if (x >= g.nx) return;
        gather_any<S, WALLS>(src, g, x, y, z, L, h);
    }
    const int c = x + g.nx * (y + g.ny * z);
    auto put = [&](OUT* out, size_t k, double v) {
        if constexpr (NT) __builtin_nontemporal_store(static_cast<OUT>(v), out + k);
        else out[k] = static_cast<OUT>(v);
    };
    if constexpr (!MOMENTS) {
#pragma unroll
        for (int i = 0; i < 27; ++i)
            put(out0, (size_t)i * g.N + c, (double)h[i] + (double)L.P.rho0 * w27<double>(i));
        return;
    }
    R Fx, Fy, Fz;
    cell_force<R, FFIELD>(force, g, c, L, Fx, Fy, Fz);
    R drho, jx, jy, jz;
    mass_momentum(h, drho, jx, jy, jz);
    const R rho = L.P.rho0 + drho;
    if (L.rs_prev) {   // sub-grid stress as a force: F + rho a'
        R a[3];
        sgs_accel(L.rs_prev, g, x, y, z, a);
        Fx += rho * a[0];
        Fy += rho * a[1];
        Fz += rho * a[2];
    }
    const R rho_u = L.P.rc ? L.P.rho0 : rho;   // reduced compressibility: rho0 u = j + F/2
    put(out0, c, (double)rho);
    put(out1, c, (double)((jx + R(0.5) * Fx) / rho_u));
    put(out1, (size_t)g.N + c, (double)((jy + R(0.5) * Fy) / rho_u));
    put(out1, 2 * (size_t)g.N + c, (double)((jz + R(0.5) * Fz) / rho_u));
}

// ---------------------------------------------------------------- adjoint
// Discrete adjoint of one step. The forward step maps fbar(n) -> fbar(n+1)
// by collision C (per cell) and streaming P: fbar_i(x, n+1) = fbar~_i(x - e_i, n).
// Its transpose gathers lam~_i(x) = lam_i(x + e_i, n+1); then
// lam(x, n) = J_C(x)^T lam~(x) and grad_F(x) += (dC/dF)^T lam~(x). lambda is
// held in the populations' row layout, element (i, x, y, z) at
// ((z ny + y) 27 + i) nx + x, so that its gather reads three adjacent rows in
// each of nine row groups, as the state's does (measured against 27 separate
// planes: 133.7 -> 123.0 us at 128^3, 1034 -> 1026 us at 256^3). WALLS: a
// post-collision population that leaves towards a wall comes back as the
// opposite population of its own cell (plus a constant), so there
// lam~_i(x) = lam_{26-i}(x, n+1). LES: the collision with the eddy rate;
// VAR: with the Sec. 12-13 operators (L.P.rc, L.P.fact).
// PACKED: several rows per workgroup (packed_cell), for short rows.
template <int S, bool FFIELD, bool WALLS, bool LES, bool VAR, bool PACKED>
__global__ void __launch_bounds__(256) k_adjoint(const typename Store<S>::T* __restrict__ state,
                                                 const typename Store<S>::R* __restrict__ lam_in,
                                                 typename Store<S>::R* __restrict__ lam_out,
                                                 typename Store<S>::R* __restrict__ grad_F,
                                                 const typename Store<S>::R* __restrict__ force, const Geom g,
                                                 const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    int x, y, z;
    if constexpr (PACKED) {
        if (!packed_cell(g, x, y, z)) return;
    } else {
        x = (int)(blockIdx.x * blockDim.x + threadIdx.x);
        y = (int)blockIdx.y;
        z = (int)blockIdx.z + g.zbase;
        if (x >= g.nx) return;
    }
    // fbar(n): ordinary loads also for the x-shifted rows, so that the cache
    // lines a wave shares with its neighbour stay in L2 for the second reader
    // (with non-temporal loads they were fetched from HBM again: 256 against
    // 240 B/cell of reads, 3 % slower at 256^3)
    R h[27];
    if constexpr (PACKED) {
        typename Store<S>::T t[27];
        gather_packed<-1, WALLS, false>(state, g, x, y, z, t);
        stored_devs<S, WALLS>(t, g, y, L, h);
    } else {
        gather<S, WALLS, 0>(state, g, x, y, z, L, h);
    }
    // lambda at x + e_i: the rows (y + ey, z + ez) are block-uniform (scalar
    // registers); only the x offset (x - 1, x, x + 1 with wrap) is per lane.
    // (An LDS exchange of the x-shifted values, as in the step kernel, was
    // measured slower here: it costs this kernel its occupancy.)
    const size_t N = (size_t)g.N, nx = (size_t)g.nx;
    const uint32_t xo[3] = {(uint32_t)(x == 0 ? g.nx - 1 : x - 1) * (uint32_t)sizeof(R), (uint32_t)x * (uint32_t)sizeof(R),
                            (uint32_t)(x == g.nx - 1 ? 0 : x + 1) * (uint32_t)sizeof(R)};
    const int yd[3] = {y == 0 ? g.ny - 1 : y - 1, y, y == g.ny - 1 ? 0 : y + 1};
    const int zd[3] = {z == 0 ? g.nz - 1 : z - 1, z, z == g.nz - 1 ? 0 : z + 1};
    R lam[27];
    if constexpr (PACKED) gather_packed<1, WALLS, false>(lam_in, g, x, y, z, lam);
#pragma unroll
    for (int i = 0; i < (PACKED ? 0 : 27); ++i) {
        const int ix = i % 3, iy = (i / 3) % 3, iz = i / 9;
        const bool wall = WALLS && ((iy == 0 && y == 0) || (iy == 2 && y == g.ny - 1));
        // as for the state: the rows read at x are read once (non-temporal),
        // the x-shifted ones keep ordinary loads so that the lines a wave
        // shares with its neighbour stay in L2 (non-temporal loads of the
        // aligned rows: 1,015 -> 1,000 us at 256^3, 124.7 -> 115.8 us at 128^3)
        const size_t r = (size_t)(wall ? y : yd[iy]) + (size_t)g.ny * (wall ? z : zd[iz]);
        const R* rowp = lam_in + nx * (r * 27 + (size_t)(wall ? 26 - i : i));
        if (ix == 1) lam[i] = __builtin_nontemporal_load((const R*)((const char*)rowp + xo[1]));
        else lam[i] = *(const R*)((const char*)rowp + xo[wall ? 1 : ix]);
    }
    const size_t row = nx * ((size_t)y + (size_t)g.ny * z);
    R F[3], g0[3];
    row_force<R, FFIELD>(force, g, L, x, y, z, F);
    // the force gradient so far, read with the other inputs rather than at the end
#pragma unroll
    for (int d = 0; d < 3; ++d) g0[d] = grad_F[(size_t)d * N + row + x];
    R gF[3] = {R(0), R(0), R(0)};
    collide_adjoint<R, LES, VAR>(h, lam, F[0], F[1], F[2], L.P, gF);
    if constexpr (PACKED) {
        const uint32_t o = ((uint32_t)y * 27u * (uint32_t)g.nx + (uint32_t)x) * (uint32_t)sizeof(R);
#pragma unroll
        for (int i = 0; i < 27; ++i) *at_row(lam_out + ((size_t)z * g.ny * 27 + i) * nx, o) = lam[i];
    }
#pragma unroll
    for (int i = 0; i < (PACKED ? 0 : 27); ++i) __builtin_nontemporal_store(lam[i], lam_out + (row * 27 + (size_t)i * nx) + x);
#pragma unroll
    for (int d = 0; d < 3; ++d) grad_F[(size_t)d * N + row + x] = g0[d] + gF[d];
}

// Seeds of E = sum rho |u|^2 / 2: dE/dfbar_i = u.e_i - |u|^2/2 (in the row
// layout of lambda), dE/dF = u/2. With reduced compressibility (rho0 u =
// sum fbar e + F/2, Sec. 12): dE/dfbar_i = (rho/rho0) u.e_i + |u|^2/2,
// dE/dF = (rho/rho0) u/2.
template <int S, bool FFIELD, bool WALLS = false>
__global__ void __launch_bounds__(256) k_energy_seed(const typename Store<S>::T* __restrict__ state,
                                                     typename Store<S>::R* __restrict__ lam_out,
                                                     typename Store<S>::R* __restrict__ grad_F,
                                                     const typename Store<S>::R* __restrict__ force, const Geom g,
                                                     const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y, z = blockIdx.z;
    if (x >= g.nx) return;
    const int c = x + g.nx * (y + g.ny * z);
    R h[27];
    gather<S, WALLS, 0>(state, g, x, y, z, L, h);
    R Fx, Fy, Fz;
    cell_force<R, FFIELD>(force, g, c, L, Fx, Fy, Fz);
    R drho, jx, jy, jz;
    mass_momentum(h, drho, jx, jy, jz);
    const bool rc = L.P.rc != 0;
    const R rho = L.P.rho0 + drho;
    const R inv_rho_u = rc ? R(1) / L.P.rho0 : R(1) / rho;
    const R ux = (jx + R(0.5) * Fx) * inv_rho_u, uy = (jy + R(0.5) * Fy) * inv_rho_u, uz = (jz + R(0.5) * Fz) * inv_rho_u;
    const R hu2 = R(0.5) * (ux * ux + uy * uy + uz * uz);
    const R s = rc ? rho * inv_rho_u : R(1);   // rho / rho0, or 1
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int ex = i % 3 - 1, ey = (i / 3) % 3 - 1, ez = i / 9 - 1;
        lam_out[((size_t)(y + g.ny * z) * 27 + (size_t)i) * (size_t)g.nx + x] =
            s * (R(ex) * ux + R(ey) * uy + R(ez) * uz) + (rc ? hu2 : -hu2);
    }
    grad_F[c] = R(0.5) * s * ux;
    grad_F[(size_t)g.N + c] = R(0.5) * s * uy;
    grad_F[2 * (size_t)g.N + c] = R(0.5) * s * uz;
}

// ---------------------------------------------------------------- FP64 reductions
// Partial sums per workgroup. The lattice is cut into tiles of blockDim.x cells
// along a grid row, numbered x chunk fastest, then y, then z; the lanes of row
// threadIdx.y of workgroup b combine the cells of tiles k, k + n, k + 2n, ...
// (k = blockDim.y b + threadIdx.y, n = blockDim.y times the workgroups) in that
// order, and the workgroup then reduces over its lanes in a fixed tree. At most
// kReduceBlocks workgroups, each with 8 doubles of partials: with one
// workgroup per tile the tree and its eight barriers ran per 256 cells, and the
// one workgroup that combines the partials read 4 MB of them (256^3 FP32: 451 us
// and 107 us; now 330 and 5).
// (Rows gathered through LDS lose here, where a workgroup waits for each row in
// turn: reductions of 512 x 512 x 128 FP16 435 us by lane, 547 by row.)
template <int S, bool WALLS, bool FFIELD>
__global__ void __launch_bounds__(256) k_reduce_partial(const typename Store<S>::T* __restrict__ src,
                                                        const typename Store<S>::R* __restrict__ force,
                                                        double* __restrict__ partial, const Geom g,
                                                        const Launch<typename Store<S>::R> L) {
    using R = typename Store<S>::R;
    const uint32_t gx = (uint32_t)((g.nx + (int)blockDim.x - 1) / (int)blockDim.x);
    const uint32_t ntiles = gx * (uint32_t)g.ny * (uint32_t)g.nz;   // at most N < 2^31
    // blockDim.x is a multiple of the wave: the tile is uniform within a wave
    const uint32_t ty = (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const uint32_t step = gridDim.x * blockDim.y;
    double v[8] = {0, 0, 0, 0, 0, 0, 1.0e300, 0};
    for (uint32_t t = blockIdx.x * blockDim.y + ty; t < ntiles; t += step) {
        const int x = (int)(t % gx) * (int)blockDim.x + (int)threadIdx.x;
        const uint32_t r = t / gx;
        const int y = (int)(r % (uint32_t)g.ny), z = (int)(r / (uint32_t)g.ny);
        R h[27];
        if (x >= g.nx) continue;
        gather_any<S, WALLS>(src, g, x, y, z, L, h);
        const int c = x + g.nx * (y + g.ny * z);
        double hd[27];
#pragma unroll
        for (int i = 0; i < 27; ++i) hd[i] = (double)h[i];
        double drho, jx, jy, jz;
        mass_momentum(hd, drho, jx, jy, jz);
        R Fx, Fy, Fz;
        cell_force<R, FFIELD>(force, g, c, L, Fx, Fy, Fz);
        if (L.rs_prev) {   // sub-grid stress as a force: F + rho a' (rho in the compute type)
            R a[3];
            sgs_accel(L.rs_prev, g, x, y, z, a);
            const R rho_r = L.P.rho0 + (R)drho;
            Fx += rho_r * a[0];
            Fy += rho_r * a[1];
            Fz += rho_r * a[2];
        }
        const double rho = (double)L.P.rho0 + drho;
        const double rho_u = L.P.rc ? (double)L.P.rho0 : rho;
        const double ux = (jx + 0.5 * (double)Fx) / rho_u, uy = (jy + 0.5 * (double)Fy) / rho_u,
                     uz = (jz + 0.5 * (double)Fz) / rho_u;
        const double px = rho * ux, py = rho * uy, pz = rho * uz;
        const double u2 = ux * ux + uy * uy + uz * uz;
        const bool bad = !isfinite(rho) || !isfinite(u2);
        double w[8];
        w[0] = rho;
        w[1] = px;
        w[2] = py;
        w[3] = pz;
        w[4] = 0.5 * rho * u2;
        w[5] = bad ? 1.0 : 0.0;
        w[6] = bad ? 1.0e300 : rho;
        w[7] = bad ? 0.0 : sqrt(u2);
        if (bad) { w[0] = w[1] = w[2] = w[3] = w[4] = 0.0; }
        combine(v, w);
    }
    block_reduce(v, partial + 8 * (size_t)blockIdx.x);
}

// ---------------------------------------------------------------- launch helpers
// Rows of up to 256 cells get one workgroup of the next multiple of 64 lanes
// (so that the LDS gather applies); wider rows the fewest workgroups of at most
// 256 lanes, of even width (300 cells: two of 192 lanes, not 256 and 44 of 256).
static dim3 grid_for_step(const Geom& g, int& bx) {
    const int n = (g.nx + 255) / 256;
    bx = ((g.nx + n - 1) / n + 63) / 64 * 64;
    return dim3(g.rowloop ? 1 : (g.nx + bx - 1) / bx, g.yrows, g.nz);
}

// With walls, only the rows y = 0 and y = ny - 1 need the bounce-back code.
// Where lanes gather for themselves (wide rows, odd in-place steps) the interior
// rows run the periodic kernel (its y +- 1 never wraps there) and the two wall
// rows a kernel of their own, so that the wall terms and extra row pointers do
// not burden the registers of every workgroup. The LDS-exchange kernel takes all
// rows in one launch (gather_xlds): the second launch cost 11 us of a 33 us step
// at 64 x 64 x 128 and 12 of 89 us at 128^3 FP32.
template <typename F>
static hipError_t split_wall_rows(const LaunchArgs& a, F&& launch) {
    if (!a.walls) return launch(a, false);
    const int ny = a.g.ny;
    if (ny > 2) {
        LaunchArgs in = a;
        in.g.ybase = 1;
        in.g.ystride = 1;
        in.g.yrows = ny - 2;
        hipError_t e = launch(in, false);
        if (e != hipSuccess) return e;
    }
    LaunchArgs wl = a;
    wl.g.ybase = 0;
    wl.g.ystride = ny > 1 ? ny - 1 : 1;
    wl.g.yrows = ny > 1 ? 2 : 1;
    return launch(wl, true);
}

// The kernels without a row loop: the same widths.
static dim3 grid_for(const Geom& g, int& bx) {
    const int n = (g.nx + 255) / 256;
    bx = ((g.nx + n - 1) / n + 63) / 64 * 64;
    return dim3((g.nx + bx - 1) / bx, g.ny, g.nz);
}

template <typename R>
static Launch<R> make_launch(const LaunchArgs& a) {
    Launch<R> L;
    L.P.rho0 = (R)a.rho0;
    L.P.ws = (R)a.omega_shear;
    L.P.wb = (R)a.omega_bulk;
    L.P.w3a = (R)a.omega3[0];
    L.P.w3b = (R)a.omega3[1];
    L.P.w3c = (R)a.omega3[2];
    L.P.w4a = (R)a.omega4[0];
    L.P.w4b = (R)a.omega4[1];
    L.P.w5 = (R)a.omega5;
    L.P.w6 = (R)a.omega6;
    L.P.tau0 = (R)(1.0 / a.omega_shear);
    L.P.smag = (R)(18.0 * a.cs_smag * a.cs_smag);
    L.P.fact = (a.flags & 1u) ? 1 : 0;
    L.P.rc = (a.flags & 2u) ? 1 : 0;
    L.P.sgs = (a.flags & 4u) ? (R)(4.5 * a.cs_smag * a.cs_smag * a.omega_shear * a.omega_shear) : R(0);
    derive_coefficients(L.P);
    L.rs_prev = (a.flags & 4u) ? (const R*)a.stress_prev : nullptr;
    for (int d = 0; d < 3; ++d) L.F[d] = (R)a.force[d];
    for (int i = 0; i < 27; ++i) {
        const int e[3] = {i % 3 - 1, (i / 3) % 3 - 1, i / 9 - 1};
        const double w = (i % 3 == 1 ? 2.0 / 3.0 : 1.0 / 6.0) * ((i / 3) % 3 == 1 ? 2.0 / 3.0 : 1.0 / 6.0) *
                         (i / 9 == 1 ? 2.0 / 3.0 : 1.0 / 6.0);
        double dlo = 0.0, dhi = 0.0;
        for (int d = 0; d < 3; ++d) {
            dlo += e[d] * a.wall_u_lo[d];
            dhi += e[d] * a.wall_u_hi[d];
        }
        L.wt_lo[i] = (R)(6.0 * w * a.rho0 * dlo);
        L.wt_hi[i] = (R)(6.0 * w * a.rho0 * dhi);
    }
    return L;
}

// The LDS gather needs one workgroup per grid row (a single chunk of x); wider
// rows take the per-lane gather, and so does every row when the caller asks for
// it (g.lanegather, a tuning hint).
static bool one_block_per_row(const Geom& g) { return g.nx <= 256 && !g.lanegather; }

// Rows for the kernel that moves whole rows through LDS. Rows of up to 256
// cells that start on cache lines, of a multiple of 128 bytes, stay with the LDS-exchange kernel, whose single barrier
// costs less (us per step, LDS exchange / whole rows: 256^3 FP32 587 / 609,
// 192^3 FP16 130 / 137); so do lattices whose two buffers fit the 32 MB of the
// eight L2s, where partial lines are merged before they reach memory and the
// extra barriers show (40^3 FP32 6.2 / 7.7, 45 x 60 x 80 FP16 9.5 / 10.4; beyond
// it 70^3 FP32 22.1 / 19.4, 100^3 53.6 / 43.4, 250 x 200 x 200 454 / 374,
// 187 x 151 x 133 FP16 131 / 81, 201 x 200 x 200 FP64 660 / 618). Rows of 257
// to 512 cells: all that the two-cell FP16 kernel does not take (per-lane
// gather / whole rows: 300 x 200 x 200 FP32 747 / 467, 320 574 / 469,
// 384 x 384 x 200 1,205 / 1,142, 512 x 512 x 128 1,298 / 1,275), but not FP64,
// whose LDS would leave two workgroups on a CU, and not on small lattices (wide_rows).
// Rows shorter than 16 cells fill too few lanes and vectors to gain.
// (past_l2: one buffer of more than 16 MB.)
template <int S>
static size_t state_bytes(const Geom& g) { return 27 * (size_t)g.N * sizeof(typename Store<S>::T); }
template <int S>
static bool past_l2(const Geom& g) { return state_bytes<S>(g) >= ((size_t)16 << 20); }
template <int S>
static bool whole_rows(const LaunchArgs& a) {
    constexpr size_t es = sizeof(typename Store<S>::T);
    const Geom& g = a.g;
    if (g.lanegather || g.rowloop || g.nx < 16 || g.nx > 512) return false;
    if (g.nx > 256) return es != 8 && wide_rows((int)es, g.ny, (int64_t)g.ny * g.nz, a.walls != 0, (a.flags & 4u) != 0);
    return (size_t)g.nx * es % 128 != 0 && past_l2<S>(g);
}

// Its workgroup, one lane per cell, and LDS: the nine groups of three rows (the
// block of 27 result rows that takes their place is smaller).
static int row_lanes(const Geom& g) { return (g.nx + 63) / 64 * 64; }
template <typename T>
static unsigned row_lds(const Geom& g) { return 9u * group_stride<T>((uint32_t)g.nx) * (unsigned)sizeof(T); }

// Several rows per workgroup (packed_cell): the lanes of a workgroup, 128 or 256,
// whichever its whole rows fill better (47 cells: 94 of 128, 235 of 256); where
// they are level 256, but 128 for fewer than 1,024 workgroups (step of 32^3 FP64
// 5.3 us in 128 lanes, 6.1 in 256; of 20 x 200 x 200 FP32 35.4 and 34.4).
static int pack_lanes(const Geom& g) {
    const int r1 = 128 / g.nx, r2 = 256 / g.nx;
    if (2 * r1 < r2) return 256;
    return (int64_t)((g.ny + r2 - 1) / r2) * g.nz < 1024 && r1 ? 128 : 256;
}
// The launch geometry for `lanes` lanes (at least nx), cut to the waves that its rows fill.
static dim3 pack_rows(Geom& g, int& lanes) {
    const PackedRows p = packed_rows_of(g.nx, g.ny, lanes);
    g.pack = p.rows;
    lanes = p.lanes;
    g.packm = (uint32_t)((65536 + g.nx - 1) / g.nx);
    return dim3((g.ny + g.pack - 1) / g.pack, g.nz);
}
// Short rows whose step packs several rows into a workgroup: where that fills at
// least 1.4 times the lanes of one row in workgroups of whole waves (1.2 in
// FP16, which is bound by instruction issue). us per step, row / packed: 20 x 200
// x 200 FP32 48.7 / 34.4, FP16 42.5 / 22.1; 32 x 200 x 200 FP32 50.7 / 48.0, FP16
// 42.0 / 28.1, FP64 107 / 94; 70 x 200 x 100 FP16 43.7 / 33.3, FP32 57.9 / 56.7; with
// less to fill 45 x 60 x 80 FP32 12.2 / 13.0, 96^3 36.4 / 38.5, 128^3 75.7 / 83.1. But FP32
// rows of whole cache lines of lattices inside the L2s, where launches and
// latency count (32^3 4.7 / 4.9), and not on few rows (packing_pays).
// In place (us per step, row / packed): 20 x 200 x 200 FP32 45.6 / 32.2, FP16 46.5 / 21.8,
// FP64 77.2 / 57.3; 32 x 200 x 200 FP32 51.2 / 44.5; 70 x 200 x 100 FP32 62.5 / 53.2, FP16
// 47.6 / 31.6; 32^3 FP32 6.2 / 4.7.
template <int S>
static bool packed_fill(const Geom& g) {
    constexpr size_t es = sizeof(typename Store<S>::T);
    if (g.lanegather || g.rowloop || g.nx < 8 || g.nx > 128) return false;
    const int lanes = pack_lanes(g), fill = lanes / g.nx * g.nx;
    const int row = (g.nx + 63) / 64 * 64;
    return (double)fill * row >= (es == 2 ? 1.2 : 1.4) * g.nx * lanes;
}

template <int S>
static bool packed_rows(const LaunchArgs& a) {
    constexpr size_t es = sizeof(typename Store<S>::T);
    const Geom& g = a.g;
    if (es == 4 && g.nx % 32 == 0 && !past_l2<S>(g)) return false;
    return packing_pays((int)es, (int64_t)g.ny * g.nz, a.walls != 0) && packed_fill<S>(g);
}

// Calls f with the row width XL of the LDS-exchange kernel as a compile-time
// constant: the workgroup's width for this row length (grid_for_step).
template <typename F>
static void with_row_width(int bx, F&& f) {
    if (bx <= 64) f(std::integral_constant<int, 64>());
    else if (bx <= 128) f(std::integral_constant<int, 128>());
    else if (bx <= 192) f(std::integral_constant<int, 192>());
    else f(std::integral_constant<int, 256>());
}

// FP16 rows for the two-cells-per-lane kernel: an even number of 258 to 512
// cells (one workgroup of at most 256 lanes per row; rows of up to 256 cells
// take the one-cell LDS kernel, measured 3 % faster at 256^3), LDS exchange
// allowed, no row loop, and buffers aligned for 32-bit population pairs and
// 64-bit force pairs (every row then starts on such a boundary, as nx is even).
static bool pair_rows(const Geom& g, const void* src, const void* dst, const void* force) {
    const bool aligned = (uintptr_t)src % 4 == 0 && (uintptr_t)dst % 4 == 0 && (uintptr_t)force % 8 == 0;
    return aligned && g.nx % 2 == 0 && g.nx > 256 && g.nx <= 512 && !g.lanegather && !g.rowloop && !g.pairs_off;
}

// Occupancy caps by LDS reservation: with 60,000 bytes of the CU's 160 KB of
// LDS reserved per workgroup, at most two workgroups share a CU, with 50,000
// three; with 40,960 bytes, three for a kernel that holds 9 KB of its own and four
// for one without. The reserved LDS itself is not used. Fewer resident rows per CU make the DRAM
// traffic of these kernels more efficient. The per-lane in-place pair with 4-byte
// populations on rows of at most 512 cells: two workgroups where they are full
// 256-lane ones, three where rows leave lanes idle or take 192 (us per step, two /
// three: 256 x 256 x 128 305 / 310, 512 x 256 x 128 608 / 611; 160^3 154 / 147,
// 192^3 263 / 253, 320 x 200 x 200 529 / 476, 384^3 2,279 / 2,171, 448 x 200 x 100
// 337 / 326; FP16: slower with any; rows of 1024 cells: not faster). The
// two-cells-per-lane FP16 kernel is about 1 % faster at three; the LDS-exchange
// step kernels are fastest at their full occupancy (six to seven workgroups).
constexpr unsigned kLdsTwoPerCu = 60000, kLdsThreePerCu = 50000, kLdsPairCap = 40960;

// A step over many z-planes runs as launches of at most kZChunk planes each:
// the end of each launch brings the eight XCDs back to the same planes, where
// over one long launch they drift apart and the planes being read and written
// at a time spread out. Measured (us per step, one launch / chunks of 128
// planes): 256^3 FP32 step (one workgroup per row) 591.6 / 578.2 and
// 596.0 / 586.5 on two machines, 256 x 256 x 1024 2,679 / 2,483; chunks of 64
// and 32 planes gained less or lost. The adjoint kernel gains as well (256^3
// FP32: 1,041 / 1,020 us; chunks of 64 the same there but 4 % slower at
// 128^3, chunks of 32 slower), and the two-cells-per-lane FP16 kernel in the plain
// order on large grids (there). Not faster, so kept in one launch: the other
// FP16 steps (187 x 151 x 400 226 / 240 us, 128 x 128 x 512 149 / 163, 256^3 298 /
// 299, 401^3 1,476 / 1,476), FP64 rows of 512 cells (9,953 / 9,751 on one machine
// but 9,578 / 10,113 on another), the in-place kernels (256^3: 653 / 656 us) and
// the D2Q9 step (8192^2: 869 us in one launch, 875-927 us in chunks of 4096-512
// rows). The FP32 sub-grid-force step with one workgroup per row gains 1.1 %
// (769.4 / 761.2 us at 256^3). Only where a chunk fills the chip many times over (chunks_pay).
template <typename Launch1>
static hipError_t launch_z_chunks(const Geom& g, const dim3& grid, bool chunked, Launch1&& launch, int64_t min_chunk = kMinStepChunk) {
    const int chunk = chunked && !g.one_launch && chunks_pay(g.nz, (int64_t)grid.x * grid.y, min_chunk) ? kZChunk : g.nz;
    for (int z0 = 0; z0 < g.nz; z0 += chunk) {
        Geom gg = g;
        gg.zbase = z0;
        launch(dim3(grid.x, grid.y, (unsigned)(g.nz - z0 < chunk ? g.nz - z0 : chunk)), gg);
        // the first failed launch ends the step (and is the error returned)
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// launch(grid, lanes, LDS, geometry, whether rows are whole cache lines) of a
// step with several rows per workgroup.
template <int S, typename F>
static void launch_packed(const LaunchArgs& a, F&& launch) {
    constexpr size_t es = sizeof(typename Store<S>::T);
    Geom gp = a.g;
    int lanes = pack_lanes(a.g);
    const dim3 gq = pack_rows(gp, lanes);
    if constexpr (es != 2) {   // (FP16 rows of whole lines fill their waves and are not packed)
        if ((size_t)gp.nx * es % 128 == 0) return launch(gq, lanes, 0u, gp, std::true_type());
    }
    launch(gq, lanes, (unsigned)(((size_t)gp.pack * 27 * gp.nx * es + 47) / 16 * 16), gp, std::false_type());
}

template <int S, bool W, bool LES, bool FF>
static hipError_t step_t(const LaunchArgs& a, const void* src, void* dst) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    int bx;
    const dim3 grid = grid_for_step(a.g, bx);
    const bool var = (a.flags & 3u) != 0;
    hipStream_t st = (hipStream_t)a.stream;
    const Launch<R> L = make_launch<R>(a);
    if constexpr (!W && S == 3) {
        if (pair_rows(a.g, src, dst, a.force_field)) {
            const dim3 gp(1, a.g.yrows, a.g.nz);
            // one lane per pair; at most three workgroups per CU (with the
            // kernel's own 9 KB of LDS) for the longest rows only (us per step without / with
            // the cap: 512 x 512 x 128 688 / 663, 512 x 400 x 200 830 / 811, 510 940 / 923, 464
            // 814 / 806, 450 822 / 811, but 480 799 / 799, 496 893 / 897, 448 724 / 740, 432 757 / 766, 400 x
            // 200 x 200 335 / 343; few rows 512 x 100 x 100 96.2 / 97.3)
            const int bp = (a.g.nx / 2 + 63) / 64 * 64;
            const unsigned pcap = a.g.nx > 448 ? kLdsPairCap : 0u;
            // past 2^25 cells in chunks of planes, in the plain order (us per step, one
            // launch plain / one launch XCD-aware / chunks: 512^3 2,903 / 2,712 / 2,692,
            // 512 x 512 x 256 1,397 / 1,358 / 1,343, 384^3 1,175 / 1,175 / 1,120; 320 x
            // 200 x 512 700 / 736 / 702)
            return launch_z_chunks(a.g, gp, (int64_t)a.g.N > (int64_t)1 << 25, [&](const dim3& gq, const Geom& gg) {
                if (var) k_step_f16pair<LES, FF, true><<<gq, bp, pcap, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L);
                else k_step_f16pair<LES, FF, false><<<gq, bp, pcap, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L);
            });
        }
    }
    if (packed_rows<S>(a)) {
        launch_packed<S>(a, [&](const dim3& gq, int lanes, unsigned lds, const Geom& gp, auto d) {
            constexpr bool D = decltype(d)::value;
            if (var) k_step_packed<S, W, LES, FF, true, false, D><<<gq, lanes, lds, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gp, L);
            else k_step_packed<S, W, LES, FF, false, false, D><<<gq, lanes, lds, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gp, L);
        });
        return hipGetLastError();
    }
    if (whole_rows<S>(a) && a.g.yrows == a.g.ny) {   // (the kernel takes all rows)
        // rows that start on cache lines (wider than 256 cells: the others of
        // that kind take the LDS exchange): each lane stores its own values
        // (us per step, through LDS / directly: 384 x 384 x 200 FP32 1,158 /
        // 1,142, 512 x 512 x 128 1,377 / 1,275; 250 x 200 x 200 374 / 433)
        const bool direct = (size_t)a.g.nx * sizeof(T) % 128 == 0;
        return launch_z_chunks(a.g, dim3(1, a.g.ny, a.g.nz), sizeof(T) == 4, [&](const dim3& gq, const Geom& gg) {
            auto launch = [&](auto v, auto d) {
                k_step_row<S, W, LES, FF, decltype(v)::value, false, decltype(d)::value>
                    <<<gq, row_lanes(gg), row_lds<T>(gg), st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L);
            };
            if constexpr (S != 0) {   // (FP64 rows that start on cache lines do not come here)
                if (direct) return var ? launch(std::true_type(), std::true_type()) : launch(std::false_type(), std::true_type());
            }
            if (var) launch(std::true_type(), std::false_type());
            else launch(std::false_type(), std::false_type());
        });
    }
    if (one_block_per_row(a.g)) {
        const unsigned lds = S == 0 ? xlds_reserve_f64(bx, state_bytes<S>(a.g)) : 0u;
        return launch_z_chunks(a.g, grid, sizeof(T) == 4, [&](const dim3& gq, const Geom& gg) {
            with_row_width(bx, [&](auto xl) {
                constexpr int XL = decltype(xl)::value;
                if (var) k_step<S, W, LES, FF, true, false, XL><<<gq, bx, lds, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L);
                else k_step<S, W, LES, FF, false, false, XL><<<gq, bx, lds, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L);
            });
        });
    }
    // per-lane rows of 257 to 512 cells with 4-byte values, which the hints and small lattices take:
    // four workgroups on a CU (300 x 200 x 100 FP32 380 us per step without,
    // 341 with; with the row loop 436 and 386; 512 x 512 x 128 1,323 and 1,299)
    const unsigned cap = sizeof(T) == 4 && a.g.nx > 256 && a.g.nx <= 512 ? kLdsPairCap : 0u;
    if (var) k_step<S, W, LES, FF, true, false, 0><<<grid, bx, cap, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, a.g, L);
    else k_step<S, W, LES, FF, false, false, 0><<<grid, bx, cap, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, a.g, L);
    return hipGetLastError();
}

// In-place rows through LDS: 16 to 512 cells (FP64: 256, by its LDS), but rows that
// start on cache lines keep the per-lane kernels in FP64 and on even steps, where
// those access whole lines (us per step, pair by lanes / even by lanes and odd by
// rows / both by rows: 256^3 FP32 646 / 602 / 621, 384 x 384 x 192 1,204 / 1,087 /
// 1,140, 512 x 512 x 128 FP16 735 / 687 / 707, 256 x 100 x 100 FP64 190 / 194 /
// 196; 300 x 200 x 100 FP32 332 / 283 / 229, 187 x 151 x 133 FP16 94 / 91 / 85,
// 201 x 100 x 100 FP64 174 / 184 / 166); and with 4-byte values on rows of up to
// 128 cells, where the per-lane kernels' two workgroups on a CU are two to four
// waves, all goes by rows (64^3 FP32 22.9 / 16.7 / 10.7, 128^3 98 / 84 / 79).
template <int S>
static bool inplace_rows(const LaunchArgs& a) {
    constexpr size_t es = sizeof(typename Store<S>::T);
    const Geom& g = a.g;
    if (g.lanegather || g.rowloop || g.nx < 16 || g.nx > (S == 0 ? 256 : 512)) return false;
    if (!inplace_rows_fill((int)es, g.nx, g.ny, (int64_t)g.ny * g.nz, a.walls != 0)) return false;
    if ((size_t)g.nx * es % 128 != 0 || (es == 4 && g.nx <= 128)) return true;
    return S != 0 && g.aa == 2;
}

template <int S, bool W, bool LES, bool FF>
static hipError_t step_inplace_t(const LaunchArgs& a, void* buf) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    int bx;
    const dim3 grid = grid_for_step(a.g, bx);
    const bool odd = a.g.aa == 2, var = (a.flags & 3u) != 0;
    hipStream_t st = (hipStream_t)a.stream;
    const Launch<R> L = make_launch<R>(a);
    if (packed_fill<S>(a.g)) {
        Geom gp = a.g;
        int lanes = pack_lanes(a.g);
        const dim3 gq = pack_rows(gp, lanes);
        auto launch = [&](auto v, auto o) {
            k_step_inplace_packed<S, W, LES, FF, decltype(v)::value, decltype(o)::value>
                <<<gq, lanes, 0, st>>>((T*)buf, (const R*)a.force_field, gp, L);
        };
        if (odd && var) launch(std::true_type(), std::true_type());
        else if (odd) launch(std::false_type(), std::true_type());
        else if (var) launch(std::true_type(), std::false_type());
        else launch(std::false_type(), std::false_type());
        return hipGetLastError();
    }
    if (inplace_rows<S>(a)) {
        const dim3 rows(1, a.g.ny, a.g.nz);
        const unsigned lds = odd ? row_lds<T>(a.g) : (27u * (unsigned)a.g.nx * (unsigned)sizeof(T) + 16u + 15u) / 16u * 16u;
        auto launch = [&](auto v, auto o) {
            k_step_inplace_row<S, W, LES, FF, decltype(v)::value, decltype(o)::value>
                <<<rows, row_lanes(a.g), lds, st>>>((T*)buf, (const R*)a.force_field, a.g, L);
        };
        if (odd && var) launch(std::true_type(), std::true_type());
        else if (odd) launch(std::false_type(), std::true_type());
        else if (var) launch(std::true_type(), std::false_type());
        else launch(std::false_type(), std::false_type());
        return hipGetLastError();
    }
    const unsigned cap = sizeof(T) != 4 || a.g.nx > 512 ? 0u : (a.g.nx % 256 ? kLdsThreePerCu : kLdsTwoPerCu);
    if (odd && var) k_step_inplace<S, W, LES, FF, true, true><<<grid, bx, cap, st>>>((T*)buf, (const R*)a.force_field, a.g, L);
    else if (odd) k_step_inplace<S, W, LES, FF, false, true><<<grid, bx, cap, st>>>((T*)buf, (const R*)a.force_field, a.g, L);
    else if (var) k_step_inplace<S, W, LES, FF, true, false><<<grid, bx, cap, st>>>((T*)buf, (const R*)a.force_field, a.g, L);
    else k_step_inplace<S, W, LES, FF, false, false><<<grid, bx, cap, st>>>((T*)buf, (const R*)a.force_field, a.g, L);
    return hipGetLastError();
}
template <int S, bool W>
static hipError_t step_inplace_w(const LaunchArgs& a, void* buf) {
    if (a.cs_smag > 0.0)
        return a.force_field ? step_inplace_t<S, W, true, true>(a, buf) : step_inplace_t<S, W, true, false>(a, buf);
    return a.force_field ? step_inplace_t<S, W, false, true>(a, buf) : step_inplace_t<S, W, false, false>(a, buf);
}
template <int S>
hipError_t step_inplace_s(const LaunchArgs& a, void* buf) {
    if (a.g.aa != 1 && a.g.aa != 2) return hipErrorInvalidValue;
    // by rows, and on even steps, which only add the wall terms, walls need no launch of their own
    if (packed_fill<S>(a.g) || inplace_rows<S>(a) || a.g.aa == 1)
        return a.walls ? step_inplace_w<S, true>(a, buf) : step_inplace_w<S, false>(a, buf);
    return split_wall_rows(a, [&](const LaunchArgs& b, bool w) {
        return w ? step_inplace_w<S, true>(b, buf) : step_inplace_w<S, false>(b, buf);
    });
}

// Sub-grid stress as a force (periodic lattices, no eddy rate in the collision).
template <int S, bool FF>
static hipError_t step_sgs_t(const LaunchArgs& a, const void* src, void* dst) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    int bx;
    const dim3 grid = grid_for_step(a.g, bx);
    const bool var = (a.flags & 3u) != 0;
    const bool xl = one_block_per_row(a.g);
    hipStream_t st = (hipStream_t)a.stream;
    const Launch<R> L = make_launch<R>(a);
    const R* rp = (const R*)a.stress_prev;
    R* rn = (R*)a.stress_next;
    // the stress planes read by the y-neighbour rows favour the plain order
    // over runs of rows per XCD (measured 768 against 784 us at 256^3)
    Geom g = a.g;
    if (a.xcd_default && g.xcd == kXcdRun) g.xcd = 0;
    if (packed_rows<S>(a)) {
        launch_packed<S>(a, [&](const dim3& gq, int lanes, unsigned lds, const Geom& gp, auto d) {
            constexpr bool D = decltype(d)::value;
            if (var) k_step_packed<S, false, false, FF, true, true, D><<<gq, lanes, lds, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gp, L, rp, rn);
            else k_step_packed<S, false, false, FF, false, true, D><<<gq, lanes, lds, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gp, L, rp, rn);
        });
        return hipGetLastError();
    }
    if (whole_rows<S>(a)) {
        const bool direct = (size_t)g.nx * sizeof(T) % 128 == 0;
        return launch_z_chunks(g, dim3(1, g.ny, g.nz), sizeof(T) == 4, [&](const dim3& gq, const Geom& gg) {
            auto launch = [&](auto v, auto d) {
                k_step_row<S, false, false, FF, decltype(v)::value, true, decltype(d)::value>
                    <<<gq, row_lanes(gg), row_lds<T>(gg), st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L, rp, rn);
            };
            if constexpr (S != 0) {
                if (direct) return var ? launch(std::true_type(), std::true_type()) : launch(std::false_type(), std::true_type());
            }
            if (var) launch(std::true_type(), std::false_type());
            else launch(std::false_type(), std::false_type());
        });
    }
    // FP32 rows of one workgroup in chunks of planes, as the step without the
    // stress force (256^3: 769.4 -> 761.2 us)
    return launch_z_chunks(g, grid, sizeof(T) == 4 && xl, [&](const dim3& gq, const Geom& gg) {
        if (xl) {
            with_row_width(bx, [&](auto w) {
                constexpr int XL = decltype(w)::value;
                if (var) k_step<S, false, false, FF, true, true, XL><<<gq, bx, 0, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L, rp, rn);
                else k_step<S, false, false, FF, false, true, XL><<<gq, bx, 0, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L, rp, rn);
            });
        } else if (var) k_step<S, false, false, FF, true, true, 0><<<gq, bx, 0, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L, rp, rn);
        else k_step<S, false, false, FF, false, true, 0><<<gq, bx, 0, st>>>((const T*)src, (T*)dst, (const R*)a.force_field, gg, L, rp, rn);
    });

}

template <int S, bool W, bool LES>
static hipError_t step_ff(const LaunchArgs& a, const void* src, void* dst) {
    return a.force_field ? step_t<S, W, LES, true>(a, src, dst) : step_t<S, W, LES, false>(a, src, dst);
}
template <int S, bool W>
static hipError_t step_les(const LaunchArgs& a, const void* src, void* dst) {
    return a.cs_smag > 0.0 ? step_ff<S, W, true>(a, src, dst) : step_ff<S, W, false>(a, src, dst);
}
template <int S>
hipError_t step_w(const LaunchArgs& a, const void* src, void* dst) {
    if (a.flags & 4u) {
        if (a.walls || !a.stress_prev || !a.stress_next) return hipErrorInvalidValue;   // checked by the caller
        return a.force_field ? step_sgs_t<S, true>(a, src, dst) : step_sgs_t<S, false>(a, src, dst);
    }
    const bool pairs = S == 3 && a.walls && walled_pairs(a.g.nx, (int64_t)a.g.ny * a.g.nz) && pair_rows(a.g, src, dst, a.force_field);
    if (!pairs && (packed_rows<S>(a) || whole_rows<S>(a) || one_block_per_row(a.g)))
        return a.walls ? step_les<S, true>(a, src, dst) : step_les<S, false>(a, src, dst);
    return split_wall_rows(a, [&](const LaunchArgs& b, bool w) {
        return w ? step_les<S, true>(b, src, dst) : step_les<S, false>(b, src, dst);
    });
}

// Setting a state: one workgroup per row, through LDS (push_rows), or by lanes
// (start_by_rows, set_by_rows).
template <int S>
static unsigned push_lds(const Geom& g) {
    return 3u * group_stride<typename Store<S>::T>((uint32_t)g.nx) * (unsigned)sizeof(typename Store<S>::T);
}
template <int S, bool W, bool FF>
static hipError_t init_t(const LaunchArgs& a, void* dst, const void* rho, const void* u, int dt) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    hipStream_t st = (hipStream_t)a.stream;
    if (start_by_rows((int)sizeof(T), a.g.nx, state_bytes<S>(a.g))) {
        k_init_equilibrium<S, W, FF, true><<<dim3(1, a.g.ny, a.g.nz), row_lanes(a.g), push_lds<S>(a.g), st>>>(
            (T*)dst, (const R*)a.force_field, rho, u, dt, a.g, make_launch<R>(a));
    } else {
        int bx;
        const dim3 grid = grid_for(a.g, bx);
        k_init_equilibrium<S, W, FF, false><<<grid, bx, 0, st>>>((T*)dst, (const R*)a.force_field, rho, u, dt, a.g,
                                                                 make_launch<R>(a));
    }
    return hipGetLastError();
}

template <int S, bool W>
static hipError_t setpop_t(const LaunchArgs& a, void* dst, const void* f, int dt) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    hipStream_t st = (hipStream_t)a.stream;
    if (set_by_rows((int)sizeof(T), a.g.nx, state_bytes<S>(a.g))) {
        k_set_populations<S, W, true><<<dim3(1, a.g.ny, a.g.nz), row_lanes(a.g), push_lds<S>(a.g), st>>>((T*)dst, f, dt, a.g,
                                                                                                    make_launch<R>(a));
    } else {
        int bx;
        const dim3 grid = grid_for(a.g, bx);
        k_set_populations<S, W, false><<<grid, bx, 0, st>>>((T*)dst, f, dt, a.g, make_launch<R>(a));
    }
    return hipGetLastError();
}

// Rows that the read-outs gather through LDS (read_by_rows): of two-buffer lattices.
// us by lane / by row: rho and u of 256^3 FP32 440 / 383, of 300 x 181 x 90
// FP32-shifted 160 / 118, of 201 x 160 x 100 FP64 165 / 141; populations of
// 256^3 FP32 1,014 / 857, of 300 x 181 x 90 429 / 375.
template <int S, bool W, bool FF, bool MOMENTS, typename OUT>
static hipError_t read_o(const LaunchArgs& a, const void* src, void* out0, void* out1) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    hipStream_t st = (hipStream_t)a.stream;
    const bool nt = read_non_temporal((int)sizeof(OUT), a.g.nx, a.g.N, MOMENTS);
    auto launch = [&](auto n) {
        constexpr bool NT = decltype(n)::value;
        if (a.g.aa == 0 && read_by_rows((int)sizeof(T), a.g.nx, state_bytes<S>(a.g), MOMENTS)) {
            k_read<S, W, FF, MOMENTS, true, NT, OUT><<<dim3(1, a.g.ny, a.g.nz), row_lanes(a.g), row_lds<T>(a.g), st>>>(
                (const T*)src, (const R*)a.force_field, (OUT*)out0, (OUT*)out1, a.g, make_launch<R>(a));
        } else {
            int bx;
            const dim3 grid = grid_for(a.g, bx);
            k_read<S, W, FF, MOMENTS, false, NT, OUT><<<grid, bx, 0, st>>>((const T*)src, (const R*)a.force_field,
                                                                           (OUT*)out0, (OUT*)out1, a.g, make_launch<R>(a));
        }
    };
    if (nt) launch(std::true_type());
    else launch(std::false_type());
    return hipGetLastError();
}
template <int S, bool W, bool FF>
static hipError_t read_t(const LaunchArgs& a, const void* src, void* out0, void* out1, int dt, int mode) {
    if (mode) return dt == 0 ? read_o<S, W, FF, true, double>(a, src, out0, out1) : read_o<S, W, FF, true, float>(a, src, out0, out1);
    // the populations do not depend on the force
    return dt == 0 ? read_o<S, W, false, false, double>(a, src, out0, out1)
                   : read_o<S, W, false, false, float>(a, src, out0, out1);
}

// Rows whose adjoint step packs several into a workgroup: up to 64 cells, or where
// that fills at least 1.2 times the lanes of one row (us, row / packed: 32 x 100 x
// 100 FP32 28.2 / 21.9, 64 x 100 x 100 38.3 / 35.5, 70 x 100 x 100 56.7 / 43.8, 20 x 100 x 100 FP16
// 22.8 / 14.8; 96^3 FP32 51.0 / 52.1, 128^3 119 / 137); and, one row in a workgroup, 4-byte rows
// that are not whole 32-byte sectors, for the ordinary stores, which share
// sectors between rows (150^3 269 / 234, 250 x 100 x 100 188 / 171, 101 x 90 x 80 52.9 / 46.7; of
// whole sectors 120 x 100 x 100 74 / 82, 256 x 256 x 128 497 / 549), but not where one-wave workgroups spread better
// (adjoint_one_wave).
template <int S>
static bool packed_adjoint(const Geom& g) {
    if (g.nx < 8 || g.nx > 256) return false;
    if (g.nx <= 64) return true;
    if (g.nx <= 128) {
        const int lanes = pack_lanes(g), fill = lanes / g.nx * g.nx;
        if (fill * ((g.nx + 63) / 64 * 64) * 10 >= 12 * g.nx * lanes) return true;
    }
    return sizeof(typename Store<S>::R) == 4 && g.nx % 8 != 0 && !adjoint_one_wave(g.nx, (int64_t)g.ny * g.nz);
}

template <int S, bool FF, bool W, bool LES, bool VAR>
static hipError_t adjoint_k(const LaunchArgs& a, const void* state, const void* lam_in, void* lam_out, void* grad_F) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    int bx;
    dim3 grid = grid_for(a.g, bx);
    if (adjoint_one_wave(a.g.nx, (int64_t)a.g.ny * a.g.nz)) {
        bx = 64;
        grid.x = (a.g.nx + 63) / 64;
    }
    const auto L = make_launch<R>(a);
    if (packed_adjoint<S>(a.g)) {
        Geom gp = a.g;
        int lanes = a.g.nx > 128 ? row_lanes(a.g) : pack_lanes(a.g);
        const dim3 gq = pack_rows(gp, lanes);
        k_adjoint<S, FF, W, LES, VAR, true><<<gq, lanes, 0, (hipStream_t)a.stream>>>(
            (const T*)state, (const R*)lam_in, (R*)lam_out, (R*)grad_F, (const R*)a.force_field, gp, L);
        return hipGetLastError();
    }
    return launch_z_chunks(a.g, grid, true, [&](const dim3& gq, const Geom& gg) {
        k_adjoint<S, FF, W, LES, VAR, false><<<gq, bx, 0, (hipStream_t)a.stream>>>((const T*)state, (const R*)lam_in, (R*)lam_out,
                                                                            (R*)grad_F, (const R*)a.force_field, gg, L);
    }, kMinAdjointChunk);
}
template <int S, bool FF, bool W>
static hipError_t adjoint_w(const LaunchArgs& a, const void* state, const void* lam_in, void* lam_out, void* grad_F) {
    const bool les = a.cs_smag > 0.0, var = (a.flags & 3u) != 0;
    if (var)
        return les ? adjoint_k<S, FF, W, true, true>(a, state, lam_in, lam_out, grad_F)
                   : adjoint_k<S, FF, W, false, true>(a, state, lam_in, lam_out, grad_F);
    return les ? adjoint_k<S, FF, W, true, false>(a, state, lam_in, lam_out, grad_F)
               : adjoint_k<S, FF, W, false, false>(a, state, lam_in, lam_out, grad_F);
}
template <int S, bool FF>
static hipError_t adjoint_t(const LaunchArgs& a, const void* state, const void* lam_in, void* lam_out, void* grad_F) {
    return a.walls ? adjoint_w<S, FF, true>(a, state, lam_in, lam_out, grad_F)
                   : adjoint_w<S, FF, false>(a, state, lam_in, lam_out, grad_F);
}

template <int S, bool FF>
static hipError_t seed_t(const LaunchArgs& a, const void* state, void* lam_out, void* grad_F) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    int bx;
    const dim3 grid = grid_for(a.g, bx);
    if (a.walls)
        k_energy_seed<S, FF, true><<<grid, bx, 0, (hipStream_t)a.stream>>>((const T*)state, (R*)lam_out, (R*)grad_F,
                                                                           (const R*)a.force_field, a.g, make_launch<R>(a));
    else
        k_energy_seed<S, FF><<<grid, bx, 0, (hipStream_t)a.stream>>>((const T*)state, (R*)lam_out, (R*)grad_F,
                                                                     (const R*)a.force_field, a.g, make_launch<R>(a));
    return hipGetLastError();
}

template <int S, bool W, bool FF>
static hipError_t reduce_t(const LaunchArgs& a, const void* src, double* partial, double* out) {
    using T = typename Store<S>::T;
    using R = typename Store<S>::R;
    int bx;
    const dim3 tiles = grid_for(a.g, bx);
    const int by = 256 / bx;   // narrow rows: several tiles side by side
    const size_t blocks = ((size_t)tiles.x * tiles.y * tiles.z + by - 1) / by;
    const unsigned grid = (unsigned)(blocks < kReduceBlocks ? blocks : kReduceBlocks);
    k_reduce_partial<S, W, FF><<<grid, dim3(bx, by), 0, (hipStream_t)a.stream>>>((const T*)src, (const R*)a.force_field,
                                                                                partial, a.g, make_launch<R>(a));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce_final(partial, grid, out, a.stream);
}

template <int S>
hipError_t adjoint_s(const LaunchArgs& a, const void* state, const void* lam_in, void* lam_out, void* grad_F) {
    return a.force_field ? adjoint_t<S, true>(a, state, lam_in, lam_out, grad_F)
                         : adjoint_t<S, false>(a, state, lam_in, lam_out, grad_F);
}
template <int S>
hipError_t seed_s(const LaunchArgs& a, const void* state, void* lam_out, void* grad_F) {
    return a.force_field ? seed_t<S, true>(a, state, lam_out, grad_F) : seed_t<S, false>(a, state, lam_out, grad_F);
}
template <int S>
hipError_t init_s(const LaunchArgs& a, void* dst, const void* rho, const void* u, int dt) {
    if (a.walls) return a.force_field ? init_t<S, true, true>(a, dst, rho, u, dt) : init_t<S, true, false>(a, dst, rho, u, dt);
    return a.force_field ? init_t<S, false, true>(a, dst, rho, u, dt) : init_t<S, false, false>(a, dst, rho, u, dt);
}
template <int S>
hipError_t setpop_s(const LaunchArgs& a, void* dst, const void* f, int dt) {
    return a.walls ? setpop_t<S, true>(a, dst, f, dt) : setpop_t<S, false>(a, dst, f, dt);
}
template <int S>
hipError_t read_s(const LaunchArgs& a, const void* src, void* o0, void* o1, int dt, int mode) {
    if (a.walls) return a.force_field ? read_t<S, true, true>(a, src, o0, o1, dt, mode) : read_t<S, true, false>(a, src, o0, o1, dt, mode);
    return a.force_field ? read_t<S, false, true>(a, src, o0, o1, dt, mode) : read_t<S, false, false>(a, src, o0, o1, dt, mode);
}
template <int S>
hipError_t reduce_s(const LaunchArgs& a, const void* src, double* partial, double* out) {
    if (a.walls) return a.force_field ? reduce_t<S, true, true>(a, src, partial, out) : reduce_t<S, true, false>(a, src, partial, out);
    return a.force_field ? reduce_t<S, false, true>(a, src, partial, out) : reduce_t<S, false, false>(a, src, partial, out);
}

// The launchers of one storage mode S. This file is compiled once for each mode
// with CM_STORAGE = S, which emits the kernels of that mode (the four objects
// build in parallel), and once without it for what follows, the dispatch over
// the modes and the kernels that do not depend on them.
#define CM_STORAGE_LAUNCHERS(KIND, S)                                                                        \
    KIND template hipError_t step_w<S>(const LaunchArgs&, const void*, void*);                               \
    KIND template hipError_t step_inplace_s<S>(const LaunchArgs&, void*);                                    \
    KIND template hipError_t init_s<S>(const LaunchArgs&, void*, const void*, const void*, int);             \
    KIND template hipError_t setpop_s<S>(const LaunchArgs&, void*, const void*, int);                        \
    KIND template hipError_t read_s<S>(const LaunchArgs&, const void*, void*, void*, int, int);              \
    KIND template hipError_t adjoint_s<S>(const LaunchArgs&, const void*, const void*, void*, void*);        \
    KIND template hipError_t seed_s<S>(const LaunchArgs&, const void*, void*, void*);                        \
    KIND template hipError_t reduce_s<S>(const LaunchArgs&, const void*, double*, double*);
#define CM_DEFINE
#ifdef CM_STORAGE
CM_STORAGE_LAUNCHERS(CM_DEFINE, CM_STORAGE)
#else
CM_STORAGE_LAUNCHERS(extern, 0)
CM_STORAGE_LAUNCHERS(extern, 1)
CM_STORAGE_LAUNCHERS(extern, 2)
CM_STORAGE_LAUNCHERS(extern, 3)
#endif

}  // namespace cm

#ifndef CM_STORAGE
#define CM_DISPATCH_S(fn, ...)                                  \
    switch (a.storage) {                                         \
        case 0: return fn<0>(__VA_ARGS__);                       \
        case 1: return fn<1>(__VA_ARGS__);                       \
        case 2: return fn<2>(__VA_ARGS__);                       \
        case 3: return fn<3>(__VA_ARGS__);                       \
        default: return hipErrorInvalidValue;                    \
    }

namespace cm {
// Second pass of the FP64 reductions: one workgroup combines the partials.
__global__ void __launch_bounds__(256) k_reduce_final(const double* __restrict__ partial, size_t nparts,
                                                      double* __restrict__ out) {
    double v[8] = {0, 0, 0, 0, 0, 0, 1.0e300, 0};
    for (size_t b = threadIdx.x; b < nparts; b += blockDim.x) {
        double w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = partial[8 * b + k];
        combine(v, w);
    }
    block_reduce(v, out);
}

// ---------------------------------------------------------------- plain copy
// Reference streaming kernel used to calibrate bandwidth and hardware byte
// counters against a known size: one 16-byte vector per thread, non-temporal
// load and store, 64-thread workgroups (the fastest plain copy form measured
// on MI355X, 4 GiB each way, on two machines: 6.67 and 6.73 TB/s, against 6.52
// and 6.49 with 256-thread workgroups, 6.35 with 512, 6.18 with 1024, 6.21-6.26
// with an ordinary load; two or more vectors per thread and grid-stride loops
// were slower still, 4.1-6.1 TB/s).
// 16 bytes a thread (the stress planes of 192^3 FP32, 170 MB: 46 us with 4 bytes
// a thread, now 26), the last 0 to 3 words by one thread each.
__global__ void __launch_bounds__(256) k_zero(unsigned int* __restrict__ dst, size_t n) {
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n / 4) __builtin_nontemporal_store((u32x4){0u, 0u, 0u, 0u}, (u32x4*)dst + k);
    else if (k - n / 4 < n % 4) dst[n - n % 4 + (k - n / 4)] = 0u;
}
__global__ void __launch_bounds__(256) k_zero_words(unsigned int* __restrict__ dst, size_t n) {
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = 0u;
}
__global__ void __launch_bounds__(256) k_copy(const u32x4* __restrict__ src, u32x4* __restrict__ dst, size_t n16) {
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

// Host-callable launchers (C++ linkage, used by the C ABI layer).
hipError_t launch_step(const LaunchArgs& a, const void* src, void* dst) { CM_DISPATCH_S(step_w, a, src, dst) }
hipError_t launch_init_equilibrium(const LaunchArgs& a, void* dst, const void* rho, const void* u, int dt) {
    CM_DISPATCH_S(init_s, a, dst, rho, u, dt)
}
hipError_t launch_step_inplace(const LaunchArgs& a, void* buf) { CM_DISPATCH_S(step_inplace_s, a, buf) }
hipError_t launch_set_populations(const LaunchArgs& a, void* dst, const void* f, int dt) {
    CM_DISPATCH_S(setpop_s, a, dst, f, dt)
}
hipError_t launch_read(const LaunchArgs& a, const void* src, void* out0, void* out1, int dt, int mode) {
    CM_DISPATCH_S(read_s, a, src, out0, out1, dt, mode)
}
hipError_t launch_adjoint(const LaunchArgs& a, const void* state, const void* lam_in, void* lam_out, void* grad_F) {
    CM_DISPATCH_S(adjoint_s, a, state, lam_in, lam_out, grad_F)
}
hipError_t launch_energy_seed(const LaunchArgs& a, const void* state, void* lam_out, void* grad_F) {
    CM_DISPATCH_S(seed_s, a, state, lam_out, grad_F)
}
hipError_t launch_reduce(const LaunchArgs& a, const void* src, double* partial, double* out) {
    CM_DISPATCH_S(reduce_s, a, src, partial, out)
}
hipError_t launch_copy(const void* src, void* dst, size_t bytes, void* stream) {
    const size_t n16 = bytes / 16;
    const size_t blocks = (n16 + 63) / 64;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
    k_copy<<<(unsigned)blocks, 64, 0, (hipStream_t)stream>>>((const u32x4*)src, (u32x4*)dst, n16);
    return hipGetLastError();
}
hipError_t launch_reduce_final(const double* partial, size_t nparts, double* out, void* stream) {
    k_reduce_final<<<1, 256, 0, (hipStream_t)stream>>>(partial, nparts, out);
    return hipGetLastError();
}
hipError_t launch_zero(void* dst, size_t bytes, void* stream) {
    const size_t n = bytes / 4;
    const bool vec = (uintptr_t)dst % 16 == 0;
    const size_t blocks = ((vec ? n / 4 + n % 4 : n) + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
    if (vec) k_zero<<<(unsigned)blocks, 256, 0, (hipStream_t)stream>>>((unsigned int*)dst, n);
    else k_zero_words<<<(unsigned)blocks, 256, 0, (hipStream_t)stream>>>((unsigned int*)dst, n);
    return hipGetLastError();
}
// Scratch of the allocation-free reductions: the partials of at most
// kReduceBlocks workgroups (65,536 bytes per device, held until the
// process ends). In host code `scratch` names a
// host-side stand-in, not the device array: its device address comes from
// hipGetSymbolAddress, looked up once per device with that device current.
static __device__ __align__(256) double scratch[8 * kReduceBlocks];

hipError_t static_reduce_scratch(int device, double** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double* addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) {
            const hipError_t e2 = hipSetDevice(cur);
            if (e == hipSuccess) e = e2;
        }
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = (double*)p;
    }
    *ptr = addr[device];
    return hipSuccess;
}
}  // namespace cm
#endif   // CM_STORAGE
