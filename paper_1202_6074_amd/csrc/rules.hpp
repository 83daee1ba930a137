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
// read it through one L2; order kXcdRun: runs of 32 consecutive places go to the
// XCDs in turn (256 a round; those after the last full round in the plain
// order). Any bijection is correct; it only changes which L2 serves a place and
// when. Counts that are no multiple of 8 have no equal eighths: order 1 takes runs of
// 32 there (us per step, plain / eighths of unequal length / runs of 32: D2Q9 3179 x
// 951 FP64 83.4 / 90.8 / 82.7, 4001^2 FP32 274 / 249 / 242, D3Q27 600 x 101 x 75 FP64
// 351 / 376 / 358, 300 x 201 x 101 FP64 641 / 593 / 554, 1000 x 101 x 51 FP16 153 / 162 /
// 145, 700 x 101 x 99 FP32 461 / 445 / 434, 429 x 31 x 18 FP64 26.5 / 26.6 / 25.2). order -1: as 1, in
// unequal eighths then, for states that fit the L2s, where neighbours find each other's rows
// (kSmallState; 352 x 15 x 11 FP64 9.8 / 7.5 / 8.4, 600 x 15 x 11 FP32 8.1 / 6.7 / 7.7, D2Q9 1280 x 333 FP32
// 7.9 / 7.0 / 7.5, 1001 x 101 5.1 / 4.7 / 5.1).
constexpr size_t kSmallState = (size_t)16 << 20;
constexpr int kXcdRun = 32;   // a power of two: no division (300 x 181 x 90 channel 194.0 us per step with one, 191.9)
CM_RULE uint32_t ordered_block(uint32_t lin, uint32_t total, int order) {
    if (order == kXcdRun || (order == 1 && (total & 7u) != 0u)) {
        constexpr uint32_t round = 8u * kXcdRun;
        const uint32_t k = lin % round, r0 = lin - k;
        return r0 + round <= total ? r0 + (k & 7u) * kXcdRun + (k >> 3) : lin;
    }
    if (order == 0) return lin;
    const uint32_t k = lin & 7u, rest = total & 7u;   // the first `rest` eighths are one longer
    return k * (total >> 3) + (k < rest ? k : rest) + (lin >> 3);
}

// Workgroup order when the caller gives no hint. lattice: 0 D3Q27, 1 D2Q9; storage: 0
// FP64, 1 FP32, 2 FP32 shifted, 3 FP16 shifted. When a grid row spans
// several workgroups (nx > 256 without the row loop), the plain order sends
// neighbouring workgroups of one row to different XCDs, whose L2s then fetch
// the cache lines shared at the block boundary twice (and, in the odd
// in-place step, both write parts of the same lines). Measured on MI355X
// (MLUPS, plain / XCD-aware): FP32 512^3 26,002 / 27,664; FP32 1024^3 in place
// 21,423 / 27,103; FP64 512^3 11,539 / 13,311. With one workgroup per
// row no lines are shared. FP32 and FP32-shifted rows of 129-256 cells (periodic
// D3Q27): runs of 32 rows per XCD in turn (at 256^3 the eight runs of a round cover one
// z-plane) beat both; measured on four machines at 256^3 (us per step, plain /
// XCD-aware / runs): two-buffer step 602 / 627 / 594, 614 / - / 604,
// 603 / - / 594, 599 / 624 / 591; in place 661 / 673 / 645, 661 / - / 645,
// 660 / - / 644; FP32 shifted 605 / - / 592. Not faster, so kept plain: walls
// (plain / runs 593 / 596 us), rows of 128 cells (77.4 / 78.0 us at 128^3),
// FP16 storage (plain / XCD-aware at 256^3: 329 / 330 us, in place 362 / 373).
// FP64 rows of up to 256 cells: plain where they start on cache lines (plain /
// XCD-aware / runs: 128^3 155 / 161 / 155, 96 x 200 x 101 143 / 156 / 144, 192 x 150 x
// 101 210 / 222 / 210, 64 x 363 x 75 129 / 136 / 131), else runs (201 x 200 x 200 601 /
// 616 / 589, 130 x 200 x 200 400 / 407 / 382, 150 x 150 x 101 172 / 181 / 169).
// Two-buffer D3Q27 steps on rows of 257-512 cells run one workgroup per row as
// well: FP16 in the plain order, which needs no division by the grid's sizes
// (the kernels are bound by instruction issue; us per step, plain / runs /
// XCD-aware: 301 x 200 x 200 310 / - / 345; the two-cell kernel at 512 x 512 x
// 128 656 / 666 / 671, in chunks of planes at 512^3 2,692 / - / 2,726), 4-byte rows
// in runs (plain / runs / XCD-aware: 300 x 200 x 200 - / 467 / 481, 288 x 200 x 200 425 /
// 433 / 439, 320 x 200 x 200 474 / 473 / 484, 384 x 200 x 200 571 / 570 / 580, 384^3
// 2,302 / 2,229 / 2,213, 448 x 200 x 200 679 / 675 / 681, 480 x 200 x 200 732 / 720 / 721;
// 416 x 200 x 200 618 / 626 / 637), full rows of 512 in the plain one (512 x 200 x 200
// 728 / 756 / 761, 512 x 64 x 64 78.0 / 82.5 / 84.6, 512 x 512 x 256 2,560 / 2,589 / 2,557).
// In-place rows of one workgroup go in the plain order (us per step, plain / runs
// of 32: 300 x 200 x 100 FP32 231 / 234, 512 x 256 x 128 608 / 612, 192^3 253 /
// 253, 200 x 100 x 100 FP64 150 / 159, 256 x 256 x 128 FP32 303 / 302), but for
// 4-byte rows that start on cache lines and are split into two workgroups which
// they do not fill (384 x 384 x 192 1,152 / 1,087, 448 x 200 x 100 336 / 326, 320 x
// 200 x 200 478 / 476).
inline int default_order(int lattice, int storage, int nx, bool rowloop, bool walls, bool in_place, bool lane_gather) {
    const bool f64 = storage == 0, four_byte = storage == 1 || storage == 2;
    if (lattice != 0) return f64 || (!rowloop && nx > 256) ? 1 : 0;
    if (in_place && !rowloop && !lane_gather && nx <= (f64 ? 256 : 512))
        return four_byte && nx > 256 && nx % 32 == 0 && nx % 256 != 0 ? kXcdRun : 0;
    if (f64) return nx > 256 || lane_gather || rowloop ? 1 : (nx % 16 ? kXcdRun : 0);
    if (!rowloop && nx > 256) {
        if (lane_gather || nx > 512) return 1;
        return four_byte && nx < 512 ? kXcdRun : 0;
    }
    return four_byte && !rowloop && !walls && nx > 128 ? kXcdRun : 0;
}

// LDS that an FP64 launch of the LDS-exchange kernel reserves beside the kernel's own,
// for workgroups of `width` lanes: what a 256-lane one holds (36,864 bytes, four workgroups on a
// CU) for narrower ones of states of 88 MiB or more. With fewer rows in flight their DRAM
// accesses stay closer together (us per step, own LDS / reserved: 128 x 256 x 256 617 / 589,
// 128^3 153 / 148, 112 x 200 x 200 327 / 315, 64 x 200 x 200 188 / 182, 64 x 64 x 128 43.5 / 42.0;
// smaller states fit the caches and want the lanes: 64^3 22.6 / 24.6, 64 x 100 x 50 26.6 /
// 28.5). The line lies between 69 and 99 MB.
inline unsigned xlds_reserve_f64(int width, size_t state_bytes) {
    return width <= 128 && state_bytes >= (size_t)88 << 20 ? 18u * 8u * (256u - (width <= 64 ? 64u : 128u)) : 0u;
}

// Even FP16 rows between walls: whether the interior rows take the two-cell kernel and
// the two wall rows a launch of their own, or all rows go through LDS in one launch. The
// two-cell kernel issues half the instructions for the memory accesses; the second launch costs
// about 6 us (us per step, one launch / two-cell and walls: 352 x 200 x 200 354 / 281, 368
// 358 / 330, 390 401 / 337, 400 403 / 347, 448 x 200 x 100 184 / 184, 480 x 100 x 100 109 / 101, 512 x
// 512 x 256 1,401 / 1,331, 384^3 1,197 / 1,065; narrower rows 300 x 200 x 200 295 / 319, 320 263 /
// 262, 340 349 / 348; fewer rows 510 x 64 x 64 48.1 / 50.8, 384 x 64 x 64 36.0 / 37.0, 512 x 20 x 20
// 8.7 / 14.1, but 400 x 64 x 64 45.9 / 40.5).
inline bool walled_pairs(int nx, int64_t rows) { return nx >= 352 && rows >= 8192; }

// Rows and lanes of a workgroup that takes several rows of one z-plane, given at most
// `lanes` lanes: a plane of fewer rows gets the waves that hold them (us per step, all lanes /
// cut: 20 x 1 x 8000 FP64 40.2 / 21.1, FP32 18.3 / 11.0, 32 x 1 x 4000 FP16 10.5 / 8.1, in
// place FP64 13.8 / 12.5; adjoint 32 x 1 x 4000 FP64 75.8 / 24.9).
struct PackedRows {
    int rows, lanes;
};
inline PackedRows packed_rows_of(int nx, int ny, int lanes) {
    const int r = lanes / nx, rows = r < ny ? r : ny;
    return {rows, (rows * nx + 63) / 64 * 64};
}

// Whether two-buffer rows of 257 to 512 cells (es bytes a value) are many enough for the
// kernel that copies whole rows through LDS, one workgroup a row: with about one row
// on a CU its copies, barriers and stores follow one another and show, where the
// per-lane kernel has twice the workgroups and no barrier (us per step, rows / lanes, at 256,
// 400 and 576 rows: 300 x 16 x 16 FP32 7.2 / 6.9, 330 x 20 x 20 9.1 / 9.5, 300 x 24 x 24 9.6 /
// 12.2; FP16, at 400, 676 and 1,024: 511 x 20 x 20 9.7 / 8.2, 511 x 26 x 26 11.4 / 13.8, 345 x
// 32 x 32 11.6 / 14.7, at 576 345 x 24 x 24 9.9 / 8.6; with the sub-grid force FP32 300 x 16 x 16 8.9 / 9.3,
// at 64 7.0 / 6.1, FP16 400 x 24 x 24 12.3 / 14.0, at 256 8.1 / 7.5). Between walls the per-lane
// kernels take two launches, so rows win there at any size (300 x 8 x 8 6.7 / 11.0), but
// where there are wall rows only.
inline bool wide_rows(int es, int ny, int64_t rows, bool walls, bool sgs) {
    if (walls && ny > 2) return true;
    return rows >= (es == 2 ? (sgs ? 400 : 640) : (sgs ? 256 : 320));
}

// The same of the in-place steps by rows (16 to 512 cells), whose per-lane kernels also access
// the cell's own rows: us per step, rows / lanes, FP32 55 x 8 x 8 6.3 / 5.2, 200 x 24 x 24 8.8 / 8.3,
// 55 x 26 x 30 7.4 / 8.0, 200 x 26 x 30 9.4 / 11.6, 317 x 16 x 16 8.2 / 8.0, 317 x 24 x 24 10.5 / 12.8, 512 x
// 24 x 24 15.8 / 14.7, 512 x 32 x 32 22.3 / 22.9; FP16 55 x 100 x 100 20.0 / 17.5, 100 x 64 x 64 15.0 /
// 14.0, 200 x 48 x 48 14.8 / 14.5, 200 x 64 x 64 22.4 / 23.3, 120 x 64 x 64 13.9 / 15.3, 317 x 24 x 24 10.3 / 9.1,
// 317 x 32 x 32 11.2 / 13.7; FP64 55 x 200 x 200 179 / 168, 120 x 100 x 100 92.7 / 86.9, 120 x 200 x
// 200 361 / 390, 200 x 100 x 100 150 / 151, 200 x 200 x 200 600 / 682. Between walls the odd
// per-lane step takes two launches.
inline bool inplace_rows_fill(int es, int nx, int ny, int64_t rows, bool walls) {
    if (walls && ny > 2) return true;
    if (es == 4) return rows >= (nx > 256 && nx % 32 ? 512 : 768);
    if (nx < 96) return false;
    return rows >= (es == 8 ? 16384 : (nx > 256 ? 1024 : 4096));
}

// Two-buffer rows are packed from 1,280 rows on (FP64 512): fewer leave CUs idle, and a lane's
// own row costs the packed kernel its uniform addresses (us per step, packed / by row, periodic: 256 rows 17 wide
// FP32 5.9 / 5.5, 85 wide 6.0 / 5.4, FP64 17 wide 7.0 / 6.0, 33 wide 6.7 / 5.8; 529 rows 33 wide FP32 6.0 / 5.5, 85
// wide 6.0 / 6.4, FP64 75 wide 6.8 / 8.2, 17 wide 6.9 / 6.5; 1,024 rows 17 wide FP32 6.2 / 5.7, 75 wide 7.6 / 7.0, FP64
// 20 wide 6.7 / 7.3, 30 wide 6.3 / 7.6; 1,521 rows 12 wide FP32 6.3 / 6.3, 24 wide 6.1 / 6.4, FP16 75 wide 7.1 / 7.9;
// 2,070 rows 70 wide FP32 7.7 / 10.1, FP16 7.1 / 8.6). Between walls packed at any size: the rows' own
// kernel is the slower one there (524 rows 30 wide 5.5 / 6.2).
inline bool packing_pays(int es, int64_t rows, bool walls) { return walls || rows >= (es == 8 ? 512 : 1280); }

// Adjoint rows of 65 to 256 cells: one wave a workgroup where one workgroup a row would be
// little more than one for each of the 256 CUs, a few of which then take two (us, one workgroup
// a row / one-wave ones: 280 rows 89 wide FP32 8.5 / 7.0, 150 wide 9.4 / 8.5, FP64 14.8 / 10.4, 250 wide FP32 10.8 /
// 9.6; 480 rows 101 wide 9.9 / 8.4, FP64 10.6 / 10.2, 201 wide 11.1 / 11.4, FP64 17.2 / 19.3; 256 rows 150 wide
// 7.7 / 8.2, FP64 9.2 / 9.9; 1,024 rows 250 wide 17.9 / 19.9).
inline bool adjoint_one_wave(int nx, int64_t rows) {
    return nx > 64 && nx <= 256 && rows > 256 && rows < (nx <= 128 ? 512 : 384);
}

// Whether init_equilibrium goes by whole rows through LDS or by lanes, whose scattered
// partial lines cost little where a state stays in the 256 MB Infinity Cache: from 192 MiB on, and on
// rows of 64 cells or more or of whole 16-byte vectors (others are written with most of their
// ends value by value). us, lanes / rows: 3M cells FP16 (162 MB) 256 wide 37 / 42, 187
// wide 41 / 58; 187 x 151 x 133 (203 MB) 82 / 69; 1M cells FP32 (108 MB) 300 wide 24.5 / 29.2, 128^3
// (226 MB) 56 / 42; 3M cells FP32 33 wide 126 / 163, 43 121 / 164, 50 114 / 122, 16 145 / 153, 20 137 /
// 123, 24 x 418 x 418 204 / 144, 75 wide 135 / 117; FP64 43 wide 245 / 251, 24 x 296 x 296 186 / 104.
// 4- and 8-byte rows of whole cache lines from 16 MiB on (into buffers that no cache holds 256 x 62 x 62 FP32
// 23.4 / 20.7, 64 x 125 x 125 22.7 / 22.4, FP64 256 x 34 x 34 21.7 / 20.2; into one that the last call
// filled 21.1 / 21.8, 21.2 / 22.0).
inline bool start_by_rows(int es, int nx, size_t state_bytes) {
    if (nx < 16 || nx > 512 || state_bytes < (size_t)16 << 20) return false;
    if (es != 2 && nx >= 64 && nx * es % 128 == 0) return true;
    return state_bytes >= (size_t)192 << 20 && (nx >= 64 || (nx * es % 16 == 0 && nx * es >= 80));
}

// The same of set_populations, which reads 8 or 4 bytes a value besides: from 48 MiB on; rows under
// 48 cells of whole vectors of 64 bytes or more, and FP64 ones under 40 (us, lanes / rows of FP64
// values: 300,000 cells FP32 (32 MB) 64 wide 15.1 / 16.4, 256 wide 15.9 / 17.7, 1M cells 256 wide 55 / 47,
// FP16 (54 MB) 128 wide 41.7 / 39.9, 256 wide 38.7 / 39.5, 43 wide 53.9 / 59.7; 3M cells FP16 64 wide 151 /
// 145, 20 wide 247 / 264, 33 wide 186 / 202, 40 x 229 x 229 124 / 115; 1M cells FP32 16 wide 97 / 65, 33 wide
// 66.4 / 67.3, 43 wide 65 / 67, 50 wide 59.9 / 59.5, 300 wide 69 / 52; FP64 33 wide 99 / 81, 3M cells 43
// wide 304 / 321, 50 wide 272 / 259).
inline bool set_by_rows(int es, int nx, size_t state_bytes) {
    if (nx < 16 || nx > 512 || state_bytes < (size_t)48 << 20) return false;
    return nx >= 48 || (nx * es % 16 == 0 && nx * es >= 64) || (es == 8 && nx < 40);
}

// Whether the read-outs of a two-buffer lattice go by whole rows through LDS: past the L2s (below,
// the extra barriers show: populations of 20 x 50 x 50 FP32 8.7 us by lane, 10.6 by
// row), rows of up to 512 cells (FP64: 256, by its LDS). Populations from 5 cells on, whose many stores
// want the loads out of the caches' way (us, lanes / rows: 5 x 200 x 300 FP32 96.7 / 84.6, 15 x 129 x 129 38.0 /
// 30.6, 11 x 200 x 200 80.0 / 57.8, FP64 98.3 / 57.2; 3 x 200 x 300 76.7 / 82.5), density and
// velocity from 16 (8 x 200 x 200 21.9 / 23.2, 15 x 258 x 258 45.1 / 43.1).
inline bool read_by_rows(int es, int nx, size_t state_bytes, bool moments) {
    return nx >= (moments ? 16 : 5) && nx <= (es == 8 ? 256 : 512) && state_bytes >= (size_t)16 << 20;
}

// Non-temporal stores of the read-outs (out bytes a value): of rows of whole 32-byte sectors;
// others share sectors between waves (populations of 201 x 160 x 100 FP64 313 us ordinary, 343
// non-temporal). Populations also from 320 MiB of output and 64 cells a row on: less stays in
// the Infinity Cache and is completed there (us, ordinary / non-temporal: 100^3 FP32 (216 MB) 58 / 83, 128 x 128 x
// 64 (226 MB) 55.5 / 66.4, 128^3 (453 MB) 144 / 140, 100 x 100 x 200 (432 MB) 172 / 168, 300 x 181 x 90 484 / 428;
// 20 x 400 x 400 380 / 444).
inline bool read_non_temporal(int out, int nx, int64_t cells, bool moments) {
    return (int64_t)nx * out % 32 == 0 && (moments || (nx >= 64 && 27 * cells * out >= (int64_t)320 << 20));
}

// Launches over chunks of kZChunk z-planes: where a chunk has at least min_chunk workgroups (per
// plane of them given). Every launch ends with a partly empty chip, and thin planes made chunks
// of a few microseconds (us per step, chunks / one launch: FP32 256 x 128 x 512 588 / 597,
// 256 x 64 x 1024 606 / 595, 200 x 100 x 400 316 / 304, 256 x 32 x 1024 318 / 295, 300 x 32 x 512 213 / 195, 256 x
// 8 x 2048 187 / 147, 64 x 64 x 1000 166 / 147, 100 x 1 x 4000 162 / 13; adjoint 256 x 128 x 512 986 / 1,008, 200 x
// 100 x 400 592 / 608, 256 x 64 x 1024 1,006 / 1,008, 128 x 64 x 1024 530 / 497, 256 x 32 x 1024 532 / 493).
constexpr int kZChunk = 128;
constexpr int64_t kMinStepChunk = 16384, kMinAdjointChunk = 12288;
inline bool chunks_pay(int nz, int64_t per_plane, int64_t min_chunk) { return nz > kZChunk && per_plane * kZChunk >= min_chunk; }

// Non-temporal stores of the D2Q9 step (es bytes a population). `moved`: the two population
// buffers, the force field and one set of the sub-grid stress. Up to about 360 MiB the next step finds
// much of what this one stored in the 256 MB Infinity Cache, more of it without a field (us per
// step, ordinary / non-temporal, at moved MB: FP32 with a field 2048^2 335 49.5 / 52.1, 2176^2 379 68.7 / 60.7,
// 4096^2 1,342 229 / 210; FP64 1536 x 1400 344 52.5 / 55.7, 1536^2 377 62.7 / 59.9, 2048^2 671 119 / 99; FP16 2560^2
// 288 56.9 / 59.2, 3072^2 415 87.4 / 83.7; without FP32 2304^2 382 63.7 / 67.7, 2432^2 426 78.2 / 75.1, FP64 2301 x
// 1501 497 91.4 / 89.6, 2001 x 1301 375 67.0 / 73.3; sub-grid force 1920^2 339 71.2 / 74.3, 2048^2 385 79.6 / 73.3;
// against the line's side FP64 1600 x 1104 283 48.7 / 47.3 and 1664 x 1152 307 52.6 / 51.2). Rows that share
// cache lines write them in parts, which costs more the more of the state is in memory anyway: FP16
// and, without a field, 4-byte values keep ordinary stores (4001 x 2001 FP16 75.2 / 78.4, 4001^2 152 / 161;
// 3179 x 1951 FP32 84.7 / 86.2, 2429 x 2067 63.1 / 72.0), the others from 720 MB on (FP32 2429 x 2067 402
// 78.1 / 74.0, 3001 x 2701 648 122 / 118, 3401 x 2701 735 145.6 / 144.3, 4001^2 1,281 242 / 279; FP64 1500 x 1501 360
// 57.0 / 58.6, 2501 x 1001 401 73.9 / 67.3, 2601 x 1701 708 134 / 126, 2429 x 2067 802 156.0 / 156.2, 3179 x 1951
// 992 184 / 194). Rows of less than a wave are stored by one-wave workgroups: non-temporal, FP64 from 48 MiB
// a buffer (50 x 4000 FP32 6.64 / 6.26, FP16 6.13 / 5.64, FP64 7.1 / 8.0; 50 x 40000 FP32 32.8 / 30.5, FP64 58.8 / 53.0).
inline bool d2q9_non_temporal(int es, int nx, int64_t cells, bool field, bool sgs) {
    constexpr int64_t M = (int64_t)1 << 20;
    const int64_t pop = 9 * cells * es, real = cells * (es == 8 ? 8 : 4);
    const int64_t moved = 2 * pop + (field ? 2 * real : 0) + (sgs ? 3 * real : 0);
    if (nx < 64 && (es != 8 || pop >= 48 * M)) return true;
    if (moved < (field ? 356 : 386) * M) return false;
    if ((int64_t)nx * es % 128 == 0) return true;
    if (es == 2 || (es == 4 && !field)) return false;
    return moved < 687 * M;
}

}  // namespace cm
