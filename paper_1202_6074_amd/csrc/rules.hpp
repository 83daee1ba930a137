// Rules that launches follow, in plain C++ without HIP: the kernels and their
// launchers use them, and the CPU tests call them through hostmath.cpp.
#pragma once
#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define CM_RULE __host__ __device__ __forceinline__
#else
#define CM_RULE inline
#endif

namespace cm {

// Which place of a launch's plain order (x, y, z) workgroup `lin` of `total`
// takes. Consecutive workgroups go to the 8 XCDs in turn, each with an L2 of its
// own. order 1: XCD k takes the k-th contiguous eighth of the places, so that
// workgroups that share data (x-halo cache lines of a row split between them)
// read it through one L2; order R >= 2: runs of R consecutive places go to the
// XCDs in turn (8 R a round; those after the last full round in the plain
// order). Any bijection is correct; it only changes which L2 serves a place and
// when. Counts that are no multiple of 8 have no equal eighths: order 1 takes runs of
// 32 there (us per step, plain / eighths of unequal length / runs of 32: D2Q9 3179 x
// 951 FP64 83.4 / 90.8 / 82.7, 4001^2 FP32 274 / 249 / 242, D3Q27 600 x 101 x 75 FP64
// 351 / 376 / 358, 300 x 201 x 101 FP64 641 / 593 / 554, 1000 x 101 x 51 FP16 153 / 162 /
// 145, 700 x 101 x 99 FP32 461 / 445 / 434).
CM_RULE uint32_t ordered_block(uint32_t lin, uint32_t total, int order) {
    if (order == 0) return lin;
    if (order == 1 && (total & 7u) == 0u) return (lin & 7u) * (total >> 3) + (lin >> 3);
    const uint32_t run = order == 1 ? 32u : (uint32_t)order, round = lin / (8u * run), k = lin % (8u * run);
    return (round + 1u) * 8u * run <= total ? round * 8u * run + (k & 7u) * run + (k >> 3) : lin;
}

}  // namespace cm
