// Convolutions from image patches in LDS (conv_patch.hip): what host and device share about them.
#pragma once
#include <stdint.h>

#include "tile_order.h"

#if defined(__HIP__)
#define FT_CONV_HD __attribute__((host)) __attribute__((device)) inline
#else
#define FT_CONV_HD inline
#endif

namespace ftk {

struct ConvArgs {
    const uint16_t *X;                   // [n, H, W, 64]
    const uint16_t *Wt;                  // [3, 3, 64, N]
    void *Y;                             // [n, P, Q, N]
    const float *bias;
    uint32_t H, W, P, Q, pad, N;
    uint32_t th, tw;                     // output pixels of a tile: th rows of tw
    uint32_t tiles_y, tiles_x, tiles;    // tiles of an image, tiles of all images
    uint32_t cols;                       // 64-channel blocks of N
    uint32_t walkers, num_xcds;          // workgroups = walkers * cols; walker i takes tiles i, i + walkers, ...
    uint32_t per_pw, per_tw;             // ceil(2^20 / (tw + 2)), ceil(2^20 / tw): see small_div
    uint32_t per_cols, per_x, per_y;     // ceil(2^31 / cols, tiles_x, tiles_y): see grid_div; per_x is 0 for more tiles than that divides
};

// pixels of the patch a th x tw tile of outputs needs
FT_CONV_HD uint32_t conv_patch_rows(uint32_t th, uint32_t tw) { return (th + 2u) * (tw + 2u); }
// LDS: the nine filter taps of 64 output channels (8 KB each), then two patches in whole kilobytes (8 pixels of 64 channels)
constexpr uint32_t kConvLds = 163840, kConvTap = 8192, kConvPatchRoom = (kConvLds - 9 * kConvTap) / 2;
constexpr uint32_t kConvCopies = 6;               // copies of a patch per wave: 8 waves of 1 KB
static_assert(kConvPatchRoom <= kConvCopies * 8192, "a patch is copied in kConvCopies instructions per wave");
FT_CONV_HD uint32_t conv_patch_bytes(uint32_t rows) { return (rows + 7u) / 8u * 1024u; }

}  // namespace ftk

// bm: 16-pixel blocks per wave, 1..4 (tiles of up to 64 * bm pixels); keep: results stay in the L2 (2), in the last-level cache (1) or in
// neither (0)
extern "C" int ft_launch_conv(const ftk::ConvArgs *args, int dt, int out16, int bm, int keep, uint32_t lds_bytes, void *stream);
