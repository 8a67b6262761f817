// Large products in 256 x 256 blocks (big_gemm.hip): what host and device share about them.
#pragma once
#include <stdint.h>

#include "tile_order.h"

namespace ftk {

struct BigArgs {
    const uint16_t *A;
    const uint16_t *B;
    void *C;
    const float *bias;
    uint32_t out16;                      // C in the inputs' 16-bit type
    uint32_t through;                    // rows of an fp32 C lie on 64-byte blocks: they are streamed and written through the L2
    uint32_t M, N, K;
    uint32_t rows, cols;                 // grid of 256-row blocks; the strip of at most 128 rows below it is not counted
    uint32_t group;                      // rows of blocks walked together
    uint32_t n_full;                     // workgroups with a whole block; the grid's blocks beyond them come as two halves each
    uint32_t n_half;                     // workgroups with 128 rows: those halves, then the strip's blocks
    uint32_t num_xcds;
};

// Workgroup b of the range [s, e) of a launch: its position when every XCD (workgroup b runs on XCD b % nx) takes one
// contiguous run of positions
FT_HD uint32_t big_position(uint32_t b, uint32_t s, uint32_t e, uint32_t nx) {
    const uint32_t i = (b - s) % nx, base = (e - s) / nx, rem = (e - s) % nx;
    return i * base + (i < rem ? i : rem) + (b - s) / nx;
}

struct BigBlock {
    uint32_t m0, n0, half;
};
FT_HD BigBlock big_block(uint32_t b, uint32_t rows, uint32_t cols, uint32_t group, uint32_t n_full, uint32_t n_half, uint32_t nx) {
    BigBlock t;
    uint32_t u, row, col, bi, lower = 0;
    const uint32_t blocks = rows * cols, halves = 2u * (blocks - n_full);
    if (b < n_full) {
        t.half = 0;
        u = big_position(b, 0u, n_full, nx);
    } else {
        t.half = 1;
        const uint32_t h = big_position(b, n_full, n_full + n_half, nx);
        if (h >= halves) {                                            // the strip below the grid
            t.m0 = rows * 256u;
            t.n0 = (h - halves) * 256u;
            return t;
        }
        u = n_full + h / 2u;
        lower = h & 1u;
    }
    grouped_coords(u, rows, cols, group, &bi, &row, &col);
    t.m0 = row * 256u + lower * 128u;
    t.n0 = col * 256u;
    return t;
}

}  // namespace ftk

extern "C" int ft_launch_big(const ftk::BigArgs *args, int dt, void *stream);
