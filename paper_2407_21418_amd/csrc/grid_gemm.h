// Matmuls in one grid of equal tiles (grid_gemm.hip): what host and device share about them.
#pragma once
#include <stdint.h>

#include <algorithm>

#include "tile_order.h"          // FT_HD

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

// Which tile a workgroup takes: every XCD (workgroup b runs on XCD b % nx) has one contiguous run of the tiles, walked in bands of
// `group` rows, column by column.  Packed into six words with the reciprocals of the divisors, so that all a workgroup needs to ask
// for its first k-tiles is in registers when it starts (see ft_grid); at most kGridTilesMax tiles and 255 XCDs.
struct GridOrder {
    uint32_t share;                      // tiles of an XCD | XCDs that have one more << 16 | XCDs << 24
    uint32_t band;                       // tiles of a band | its rows << 16
    uint32_t last;                       // bands of that many rows | rows of what is left below them << 16
    uint32_t per_band, per_rows, per_last;          // ceil(2^31 / tiles of a band, rows of a band, rows of the last one)
};
struct GridTile {
    uint32_t row, col;
};
constexpr uint32_t kGridTilesMax = 32767;
inline GridOrder grid_order(uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx) {
    const uint32_t n = rows * cols, low = rows % group;
    return GridOrder{n / nx | (n % nx) << 16 | nx << 24, group * cols | group << 16, rows / group | low << 16, grid_per(group * cols), grid_per(group), grid_per(low)};
}
FT_HD GridTile grid_tile(const GridOrder &o, uint32_t b) {
    const uint32_t nx = o.share >> 24, more = o.share >> 16 & 255u;
    uint32_t x, q;
    if (nx == 8) { x = b & 7u; q = b >> 3; }
    else { x = b % nx; q = b / nx; }
    const uint32_t u = x * (o.share & 0xffffu) + (x < more ? x : more) + q;
    const uint32_t i = grid_div(u, o.per_band), w = u - i * (o.band & 0xffffu);
    const bool low = i >= (o.last & 0xffffu);
    const uint32_t col = grid_div(w, low ? o.per_last : o.per_rows);
    return GridTile{i * (o.band >> 16) + w - col * (low ? o.last >> 16 : o.band >> 16), col};
}
FT_HD GridTile grid_tile(uint32_t b, uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx) { return grid_tile(grid_order(rows, cols, group, nx), b); }

// Rows of A and columns of B that the XCD with the most of them reads in that walk.  A run begins in the middle of one band and ends
// in another: rows of different bands are different ones, columns meet again.
inline uint32_t grid_reads(uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx, uint32_t tm, uint32_t tn) {
    const uint32_t n = rows * cols, band = group * cols, share = n / nx, more = n % nx;
    uint32_t most = 0;
    for (uint32_t x = 0, s = 0; x < nx && s < n; ++x) {
        const uint32_t e = s + share + (x < more ? 1 : 0), i = s / band, j = (e - 1) / band;          // its first tile, the one after its last, their bands
        const uint32_t hi = std::min(group, rows - i * group), hj = std::min(group, rows - j * group);
        const uint32_t si = s - i * band, ej = e - j * band;
        const uint32_t r = i == j ? std::min(hi, e - s) : std::min(hi, hi * cols - si) + (j - i - 1) * group + std::min(hj, ej);
        const uint32_t c = i == j ? (ej - 1) / hi - si / hi + 1 : j - i > 1 ? cols : std::min(cols, cols - si / hi + (ej - 1) / hj + 1);
        most = std::max(most, r * tm + c * tn);
        s = e;
    }
    return most;
}

// Rows of tiles walked together: those with which a run of an XCD's length that begins at the top of a band touches the fewest rows of
// A and columns of B, unless the XCD that reads the most reads a sixth less in higher bands, of equal ones the highest: a run that
// goes from one band into the next has the columns of both, and one in a low last band most columns there are.  us, the first choice /
// this: 7 rows of 16 tiles 220 x 512 x 2048 6.5 / 4.95, 9 of 24 272 x 768 x 3072 8.8 / 8.3, 18 of 12 560 x 768 x 3072 10.6 / 8.9, 8 of 24 688 x 3072 x
// 768 7.7 / 7.6 and with fp32 results 8.6 / 8.5 (in the caches 8.5 / 8.4), 10 of 24 454 x 1536 x 2048 9.0 / 8.7, 20 of 12 2518 x 2304 x 768 14.3 / 14.05.
// Lower bands are no choice, whatever they would save: each reads B again, and fewer rows of tiles fetch a window of it for one another (8 rows
// of 24 in bands of 4 for 6, a third less to read, 688 x 3072 x 768 7.9, with fp32 results 8.8; bands of 2 for 6, 2976 x 768 x 768 8.7 / 9.0; the
// exception seen is bands of 2 for 5, 29 rows of 8, 2691 x 512 x 3072 16.1 / 15.2).  On differences below a sixth the two are as often wrong
// as right (11 rows of 16, 384 rows and columns for 448, 330 x 512 x 4096 9.35 / 10.9).
inline uint32_t grid_band(uint32_t rows, uint32_t cols, uint32_t nx, uint32_t tm, uint32_t tn) {
    const uint64_t run = ((uint64_t)rows * cols + nx - 1) / nx;
    uint64_t least = ~0ull;
    uint32_t first = 1;
    for (uint32_t g = 1; g <= rows; ++g) {
        const uint64_t columns = (run + g - 1) / g, passes = (columns + cols - 1) / cols;
        const uint64_t touched = g * passes * tm + std::min<uint64_t>(columns, cols) * tn;
        if (touched < least) { least = touched; first = g; }
    }
    uint32_t fewest = ~0u, height = 0;
    for (uint32_t g = first + 1; g <= rows; ++g)
        if (const uint32_t most = grid_reads(rows, cols, g, nx, tm, tn); most <= fewest) { fewest = most; height = g; }
    return height && fewest * 6 < grid_reads(rows, cols, first, nx, tm, tn) * 5 ? height : first;
}

struct GridArgs {
    const uint16_t *A;
    const uint16_t *B;
    void *C;                             // fp32 or the inputs' 16-bit type
    const float *bias;                   // one per column, or NULL
    uint32_t M, N, K;
    uint32_t tiles;                      // workgroups
    GridOrder order;
    uint32_t through;                    // rows of C lie on 64-byte blocks: they are written through the L2
};

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
