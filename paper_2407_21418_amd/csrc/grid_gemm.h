// Matmuls in one grid of equal tiles (grid_gemm.hip): what host and device share about them.
#pragma once
#include <stdint.h>

#include "tile_order.h"

namespace ftk {

// X(id, WM, WN, GM, GN, GK, STAGES): GK groups of GM x GN waves, each wave WM x WN of the tile; group g takes the k-tiles of 64
// g, g + GK, ... through a ring of STAGES of its own, and the groups' sums meet in LDS.
#define FT_GRID_BODIES(X)                                                                          \
    X(0, 32, 32, 1, 1, 4, 4)                                                                       \
    X(1, 16, 64, 1, 1, 4, 4)                                                                       \
    X(2, 32, 32, 1, 2, 2, 4)                                                                       \
    X(3, 48, 32, 1, 2, 2, 4)                                                                       \
    X(4, 32, 32, 2, 2, 1, 4)                                                                       \
    X(5, 48, 32, 2, 2, 1, 4)                                                                       \
    X(6, 64, 32, 2, 2, 1, 4)                                                                       \
    X(7, 48, 64, 2, 2, 1, 3)                                                                       \
    X(8, 64, 32, 2, 4, 1, 4)                                                                       \
    X(9, 64, 48, 2, 4, 1, 3)                                                                       \
    X(10, 64, 64, 2, 4, 1, 3)                                                                      \
    X(11, 32, 32, 2, 4, 1, 4)

struct GridArgs {
    const uint16_t *A;
    const uint16_t *B;
    void *C;                             // fp32 or the inputs' 16-bit type
    const float *bias;                   // one per column, or NULL
    uint32_t M, N, K;
    uint32_t rows, cols, tiles;          // tiles = rows * cols workgroups
    uint32_t group;                      // rows of tiles walked together
    uint32_t num_xcds;
    uint32_t stream;                     // rows of an fp32 C lie on 64-byte blocks: they are stored past the caches
};

// workgroup b's tile: every XCD (workgroup b runs on XCD b % nx) takes one contiguous run of the tiles in groups of `group` rows,
// column by column
struct GridTile {
    uint32_t row, col;
};
template <uint32_t NX> FT_HD GridTile grid_tile_nx(uint32_t b, uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx_in) {
    const uint32_t nx = NX ? NX : nx_in, n = rows * cols, x = b % nx, base = n / nx, rem = n % nx;
    uint32_t bi;
    GridTile t;
    grouped_coords(x * base + (x < rem ? x : rem) + b / nx, rows, cols, group, &bi, &t.row, &t.col);
    return t;
}
FT_HD GridTile grid_tile(uint32_t b, uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx) {
    return nx == 8 ? grid_tile_nx<8>(b, rows, cols, group, nx) : grid_tile_nx<0>(b, rows, cols, group, nx);
}

// Sums a wave keeps of an output, added at the end: with fp32 results the k-steps of a k-tile have one each, and where one group
// takes the whole reduce axis those of even and odd k-tiles, as far as the registers go.  The error of a sum grows with the root of
// its terms in a row, and the waves of the tiles share the reduce axis: grid_schedule lets a body stand in for tiles only if it
// adds up as many sums.
constexpr uint32_t grid_sums(uint32_t wm, uint32_t wn, uint32_t gk, bool out16) {
    return out16 || wm * wn > 48 * 64 ? 1 : gk > 1 || wm * wn > 48 * 32 ? 2 : 4;
}

struct GridBodyInfo {
    uint32_t tm, tn, gk, waves, lds;
    uint32_t sums32;                     // partial sums of an output with fp32 results
};
constexpr GridBodyInfo grid_info(uint32_t wm, uint32_t wn, uint32_t gm, uint32_t gn, uint32_t gk, uint32_t stages) {
    const uint32_t tm = gm * wm, tn = gn * wn, ring = gk * stages * (tm + tn) * 128u, sums = gk > 1 ? gk * tm * tn * 4u : 0u;
    return GridBodyInfo{tm, tn, gk, gm * gn * gk, ring > sums ? ring : sums, gk * grid_sums(wm, wn, gk, false)};
}
#define FT_X(id, WM, WN, GM, GN, GK, S) grid_info(WM, WN, GM, GN, GK, S),
constexpr GridBodyInfo kGridBodies[] = {FT_GRID_BODIES(FT_X)};
#undef FT_X
constexpr uint32_t kNumGridBodies = sizeof(kGridBodies) / sizeof(kGridBodies[0]);

}  // namespace ftk

extern "C" int ft_launch_grid(const ftk::GridArgs *args, uint32_t body, int dt, int out16, void *stream);
