// Device helpers shared by the D3Q27 and D2Q9 kernels: storage types of the
// population buffers, reading caller arrays of either dtype, and the
// fixed-order FP64 block reduction.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "rules.hpp"

namespace cm {

// Storage mode S: element type T in memory, compute type R, and whether the
// stored value is shifted by the rest state w_i rho0.
template <int S> struct Store;
template <> struct Store<0> { using T = double;   using R = double; static constexpr bool shifted = false; };
template <> struct Store<1> { using T = float;    using R = float;  static constexpr bool shifted = false; };
template <> struct Store<2> { using T = float;    using R = float;  static constexpr bool shifted = true; };
template <> struct Store<3> { using T = _Float16; using R = float;  static constexpr bool shifted = true; };

// Coordinates (x block, y, z) of this workgroup in a grid of (gx, ny, nz) blocks,
// in the order `xcd` (ordered_block).
__device__ __forceinline__ void block_coords(int xcd, int& bx, int& y, int& z) {
    if (xcd == 0) {   // without the divisions
        bx = (int)blockIdx.x;
        y = (int)blockIdx.y;
        z = (int)blockIdx.z;
        return;
    }
    const uint32_t gx = gridDim.x, gy = gridDim.y, gz = gridDim.z;
    const uint32_t lin = ordered_block(blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z), gx * gy * gz, xcd);
    bx = (int)(lin % gx);
    const uint32_t r = lin / gx;
    y = (int)(r % gy);
    z = (int)(r / gy);
}

__device__ __forceinline__ double as_double(const void* p, int dt, size_t k) {
    return dt == 0 ? static_cast<const double*>(p)[k] : static_cast<double>(static_cast<const float*>(p)[k]);
}

// Per-block partials: [mass, px, py, pz, ke, nonfinite, min rho, max |u|], in
// a fixed order so that results are bitwise reproducible.
__device__ __forceinline__ void combine(double (&a)[8], const double (&b)[8]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) a[k] += b[k];
    a[6] = fmin(a[6], b[6]);
    a[7] = fmax(a[7], b[7]);
}

// Over the lanes of a wave first (halving distances), then over the waves in
// turn: a fixed order, and 512 bytes of LDS (a tree over all lanes in LDS took
// 16 KB, on the kernels that need theirs for rows).
__device__ __forceinline__ void block_reduce(double (&v)[8], double* __restrict__ out) {
    __shared__ double sm[8][8];   // of at most eight waves
    const int t = threadIdx.x + blockDim.x * threadIdx.y;
    const int waves = (int)(blockDim.x * blockDim.y) / 64;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        double w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = __shfl_down(v[k], s);
        combine(v, w);
    }
    if ((t & 63) == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) sm[t >> 6][k] = v[k];
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < waves; ++w) {
            double b[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) b[k] = sm[w][k];
            combine(v, b);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = v[k];
    }
}

}  // namespace cm
