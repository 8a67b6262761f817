// Row runs (row_runs.hip): what host and device share about them.
#pragma once
#include <stdint.h>

#include "tile_order.h"

#if defined(__HIP__)
#define FT_RUN_HD __attribute__((host)) __attribute__((device)) inline
#else
#define FT_RUN_HD inline
#endif

namespace ftk {

constexpr uint32_t kRunMaxN = 320;     // columns of C (see row_runs.hip)

struct RunArgs {
    const uint16_t *A;
    const uint16_t *B;
    void *C;
    const float *bias;
    uint32_t out16;                      // C in the inputs' 16-bit type
    uint32_t M, N, K;
    uint32_t runs, rb_log2;              // shares per batch entry; rows of a share = 32 << rb_log2
    uint32_t n_runs;                     // shares of the launch
    uint32_t per_pitch;                  // ceil(2^20 / run_kn_pitch(N)): see small_div
    uint32_t num_xcds;
};

// What these launches take: one k-tile of whole 16-byte chunks, rows of 8 .. kRunMaxN elements.  From 193 to 256 columns a
// single tile of the tile bodies spans the row and is as fast (255: 32.0 against 33.7 us, 200: 39.9 against 40.7).
FT_RUN_HD bool run_shape_ok(uint32_t N, uint32_t K) {
    return K >= 8u && K <= 64u && K % 8u == 0 && N >= 8u && N <= kRunMaxN && (N <= 192u || N > 256u);
}

// LDS row of a [64 k][N] B tile, in 16-byte chunks: whole 32-column blocks, and twice an odd number (the rows of a
// transposing read then start in different banks)
FT_RUN_HD uint32_t run_kn_pitch(uint32_t N) { return 2u * (2u * ((N + 31u) / 32u) + 1u); }

// LDS bytes of a share: the A and B tiles, or the image of its outputs (up to 127 bytes in front, up to a whole
// chunk behind), whichever is larger
FT_RUN_HD uint32_t run_lds(uint32_t N, uint32_t rb_log2, uint32_t elem_bytes, bool bnk) {
    const uint32_t tiles = (4096u << rb_log2) + (bnk ? (N + 31u) / 32u * 4096u : 64u * 16u * run_kn_pitch(N));
    const uint32_t image = 128u + (32u << rb_log2) * N * elem_bytes + 16u;
    return ((tiles > image ? tiles : image) + 15u) & ~15u;
}

// Row blocks of a share (log2).  A wave holds at most four accumulator blocks, so shares of 128, 64 and 32 rows
// take up to 128, 256 and kRunMaxN columns.  Tall shares read B fewer times and pay a share's latencies less often: they
// are taken from three per CU on if one round of the CUs holds them all, else from four (measured with every height forced,
// 32 against 64 rows: 3 per CU 768 x 33 x 33 6.3 / 4.8 us, 2 per CU equal, 1.5 per CU 384 x 131 x 131 4.9 / 5.2; a second
// round that is nearly empty, 288 x 190 x 190 fp32: 15.3 / 16.8).
FT_RUN_HD uint32_t run_rb_log2(uint32_t M, uint32_t N, uint64_t batch, uint32_t elem_bytes, bool bnk, uint32_t num_cus) {
    uint32_t rb = N <= 128u ? 2u : N <= 256u ? 1u : 0u;
    for (; rb > 0; --rb) {
        const uint64_t shares = batch * ((M + (32u << rb) - 1) / (32u << rb));
        const uint32_t fit = 163840u / run_lds(N, rb, elem_bytes, bnk), held = fit < 5u ? fit : 5u;     // (registers: five)
        if (M > (16u << rb) && (shares >= 4ull * num_cus || (shares >= 3ull * num_cus && shares <= (uint64_t)held * num_cus))) break;
    }
    return rb;
}

}  // namespace ftk

extern "C" int ft_launch_runs(const ftk::RunArgs *args, int dt, int bnk, uint32_t lds_bytes, void *stream);
