// The LDS rings of the tile bodies in one launch: the depth each body's loop is told and the LDS the launch asks for.
#pragma once
#include <stdint.h>

namespace ftk {

struct RingSlot {
    bool splitk;                         // four waves with a ring each, a quarter of the k-tiles each
    uint32_t planned;                    // stages of the plan's ring
    uint32_t stage_bytes;
    uint32_t depth;                      // result: stages as the loop sees them; depth - 1 tiles are requested before the first wait
};

// k-tiles that pass through one ring (split-k: the busiest wave's)
inline uint32_t ring_tiles(const RingSlot &s, uint32_t k_tiles) { return s.splitk ? (k_tiles + 3u) / 4u : k_tiles; }
// LDS bytes that the loop touches at this depth: a ring deeper than its tiles never touches the other stages (split-k: the
// waves' partial tiles cross two stages at least, and the rings lie this far apart)
inline uint32_t ring_bytes(const RingSlot &s, uint32_t k_tiles) {
    const uint32_t tiles = ring_tiles(s, k_tiles), touched = s.depth < tiles ? s.depth : tiles;
    return (s.splitk ? 4u * (touched < 2u ? 2u : touched) : touched) * s.stage_bytes;
}

// A reduce axis of fewer k-tiles than the plan's rings have stages uses only some of them.  The launch asks for those, so
// that more workgroups fit a CU (Q K^T and P V of 96 heads of 131 rows, one and three k-tiles: 11.6 -> 10.6 us).  A loop told
// a depth of its tiles requests the last one when the first has landed; told one stage more, it requests all of them at
// once, in the same LDS.  Which is faster was measured over 850 shapes (K of 66 to 1536, 16 to 9216 workgroups; batch x M x N x K, us, told
// `tiles` / told one more):
//   - split-k, two tiles a wave: all at once (150 x 768 x 512: 3.95 / 3.77); three and more: one at a time, whose many
//     copies per wave hold up the first tile's (272 x 768 x 768: 4.81 / 5.10)
//   - other bodies, where the launch has more than two workgroups per CU and the smaller rings let more of them in: one at a
//     time, the workgroups' copies cover for each other (768 x 128 x 64 x 128: 11.9 / 13.6); else
//   - one or two tiles: all at once (192 x 64 x 64 x 128: 4.26 / 4.11)
//   - three and more: one at a time (96 x 180 x 64 x 180: 5.53 / 5.71), but all at once in a body that is not the one whose
//     ring sets the launch's LDS (384 x 176 x 64 x 176, 16-row tiles behind 128-row ones: 15.7 / 15.2)
// Returns the LDS bytes of the launch.
inline uint32_t ring_plan(RingSlot *s, int n, uint32_t k_tiles, uint64_t workgroups, uint32_t num_cus, uint32_t planned_lds) {
    constexpr uint32_t kCuLds = 163840;
    uint32_t lds = 0;
    for (int i = 0; i < n; ++i) {
        const uint32_t tiles = ring_tiles(s[i], k_tiles);
        s[i].depth = s[i].planned < tiles ? s[i].planned : tiles;
        if (s[i].depth < 2u) s[i].depth = 2u;
        const uint32_t b = ring_bytes(s[i], k_tiles);
        if (b > lds) lds = b;
    }
    const bool crowded = workgroups > 2ull * num_cus && lds > 0 && kCuLds / lds > kCuLds / planned_lds;
    for (int i = 0; i < n; ++i) {
        const uint32_t tiles = ring_tiles(s[i], k_tiles);
        const bool at_once = s[i].splitk ? tiles <= 2u : !crowded && (tiles <= 2u || ring_bytes(s[i], k_tiles) < lds);
        if (at_once && tiles + 1u <= s[i].planned && tiles + 1u > s[i].depth) s[i].depth = tiles + 1u;
    }
    return lds;
}

}  // namespace ftk
