// 3 x 3 Conv2d over 64 input channels, stride 1, from image patches in LDS.
//
// As an implicit GEMM with a gather (gemm_fast.h) a convolution fetches every pixel once per filter tap: a 3 x 3 layer
// pulls nine times its image through the CUs' vector memory path, and the k loop runs at the rate of that path.  Here a
// workgroup keeps the filter taps of 64 output channels in LDS (72 KB) and walks over tiles of up to 256 output pixels: a
// tile's patch of the image is fetched once, halo and zero padding included, and every tap reads its rows of A from the
// patch, shifted.  8 x 224 x 224 x 64 -> 128: 89 us with the gather, 64 to 67 here with fp32 results, 87 and 60 with 16-bit ones; 8 x 56 x 56:
// 10.5 and 7.6; 8 x 28 x 28: 6.2 and 4.5.  On 224 x 224, thirteen rounds of tiles of 256 pixels, a round takes 4.9 us: 4.1 without the stores, of
// which the MFMAs are 3.0, LDS reads 0.5 and copies, waits and barrier 0.5, and 0.8 of stores that nothing hides (counters: matrix cores
// busy for 53 % of the cycles at 2.1 GHz); the smallest launches are bound by their latencies: taps and patch 1.5 us, nine taps 1.3 (27 % on 56 x 56).
//   - One workgroup of eight waves per CU, the patch of the next tile arriving while this one is computed: no wait and no
//     barrier inside a tile.  (A form that streamed the taps through a ring, two workgroups per CU, spent 0.57 us per tap
//     on 0.21 us of MFMAs: its barrier per tap and the taps' latency.  Starting a single tile before all taps have landed
//     needs the same barriers and lost 0.5 us; copies spread over the taps, as the stores are, changed nothing.)
//   - The results of a tile leave while the next one is computed, a store or two per tap: a CU's vector memory path is in
//     order, and a burst of stores would hold up the waves and the next patch behind it.
//     Where a pixel's channels lie on 64-byte blocks they are written through the L2: as dirty lines they would be written back
//     when the launch ends and while other tiles are read.  Those of more than a quarter of the last-level cache are streamed past it
//     too (KEEP).  fp32 results, kept / written through / streamed as well, us: 8 x 56 x 56 9.8 / 8.2 / 8.2, 8 x 75 x 75 12.5 / 10.5 /
//     10.9, 8 x 112 x 112 23.5 / 21.3 / 21.8, 8 x 145 x 145 38.7 / 41.6 / 32.4, 8 x 224 x 224 78.0 / 80.1 / 65.4; 16-bit results 8.1 / 7.5 /
//     7.5, 11.0 / 9.7 / 9.7, 21.2 / 20.0 / 20.3, 30.3 / 29.4 / 29.3, 64.0 / 66.3 / 61.7.
//   - A pixel's 64 channels are one 128-byte row of LDS, its 16-byte chunks at chunk ^ (x & 7), x the column in the patch: 16
//     neighbouring pixels are read without a bank conflict whatever column a tap makes them start at (counted: none on
//     224 x 224, tiles 16 wide; 23 % of the LDS cycles on 56 x 56, where 16 pixels of a tile 28 wide lie in two of its rows), and
//     a tap's rows differ from those of the tap above by a constant.
//   - Operands are handed to the MFMAs the other way round, so that a lane holds four neighbouring channels of one pixel.
//   - Before its first copies a lane finds six pixels' rows and columns in the patch, and four of its outputs': divisions by reciprocals from
//     the host (small_div), as two waves to a SIMD need half a microsecond for the general ones: 8 x 28 x 28 4.9 -> 4.5 us, 8 x 37 x 37 6.0
//     -> 5.4, 8 x 56 x 56 8.2 -> 7.6, larger ones 0.3 less.
// The host picks the tile, and the layers that are left to the gather (see conv_schedule).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "conv_patch.h"
#include "gemm_body.h"
#include "lds_limit.h"

namespace ftk {

typedef uint32_t conv_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t conv_u32x2 __attribute__((ext_vector_type(2)));
typedef float conv_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 conv_bf16x2 __attribute__((ext_vector_type(2)));

__device__ __attribute__((aligned(256))) static uint32_t conv_zero_page[64];

template <int N> __device__ __forceinline__ void conv_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void conv_dma16(const void *gptr, unsigned char *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)gptr,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 16, 0, 0);
}

// Eight waves, 4 of BM x 16 pixels by 2 of 32 channels.
// KEEP: where results stay, 2 in the L2, 1 in the last-level cache, 0 in neither.
template <int DT, bool OUT16, int BM, int KEEP>
struct ConvBody {
    static constexpr int GN = 2, WM = BM * 16, WN = 32, BN = 2, TN = 64;
    static constexpr int NR = BM + 2 * BN, NM = BM * BN;
    static constexpr int NS = OUT16 ? BM : NM;                         // stores of a tile per lane
    static constexpr int ES = OUT16 ? 2 : 4;

    template <int V> struct Int { static constexpr int value = V; };
    struct Frag { conv_u32x4 a[BM]; conv_u32x2 b[BN][2]; };
    struct Tile { uint32_t img, p0, q0; };

    // Fragment reads of filter tap T.  The taps are unrolled, so that B's addresses are immediates; A's are kept for the
    // three columns of the filter and move by a row of the patch, with one XOR for a tap's second k-step.
    struct Addr { uint32_t a[3][BM], b[2][BN]; };
    template <int T, int KS, int R> __device__ static __forceinline__ void read_b(const Addr &ad, Frag &f) {
        constexpr int off = T * (int)kConvTap + (KS * 32 + (R % 2) * 4) * TN * 2;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.b[R / 2][R % 2]) : "v"(ad.b[off / 65536][R / 2]), "n"(off % 65536));
    }
    template <int T, int KS, int I> __device__ static __forceinline__ void read_a(const Addr &ad, Frag &f) {
        asm volatile("ds_read_b128 %0, %1" : "=v"(f.a[I]) : "v"(ad.a[T % 3][I] ^ (uint32_t)(KS * 64)));
    }
    template <int T, int KS, int R = 0> __device__ static __forceinline__ void read_bs(const Addr &ad, Frag &f) {
        read_b<T, KS, R>(ad, f);
        if constexpr (R + 1 < 2 * BN) read_bs<T, KS, R + 1>(ad, f);
    }
    template <int T, int KS, int I = 0> __device__ static __forceinline__ void read_as(const Addr &ad, Frag &f) {
        read_a<T, KS, I>(ad, f);
        if constexpr (I + 1 < BM) read_as<T, KS, I + 1>(ad, f);
    }
    // waits until at most AFTER younger LDS reads are under way: those of this fragment have landed
    template <int AFTER> __device__ static __forceinline__ void arrived(Frag &f) {
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(AFTER) : "memory");
#pragma unroll
        for (int i = 0; i < BM; ++i) asm volatile("" : "+v"(f.a[i]));
#pragma unroll
        for (int i = 0; i < BN; ++i) asm volatile("" : "+v"(f.b[i][0]), "+v"(f.b[i][1]));
        __builtin_amdgcn_sched_barrier(0);
    }
    // the MFMAs of one k-step of 32 of tap T; the registers that they are done with are filled for the same k-step of the
    // next tap, so that every read has a k-step and a half to arrive
    template <int T, int KS, int I = 0>
    __device__ static __forceinline__ void phase(const Addr &ad, Frag &f, f32x4 (&acc)[BM][BN]) {
#pragma unroll
        for (int j = 0; j < BN; ++j) {
            const uint4 b = make_uint4(f.b[j][0][0], f.b[j][0][1], f.b[j][1][0], f.b[j][1][1]);
            acc[I][j] = mfma16<DT>(b, __builtin_bit_cast(uint4, f.a[I]), acc[I][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (T < 8) read_a<T + 1, KS, I>(ad, f);
        if constexpr (T < 8 && I + 1 == BM) read_bs<T + 1, KS>(ad, f);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (I + 1 < BM) phase<T, KS, I + 1>(ad, f, acc);
    }
    template <int T, typename F>
    __device__ static __forceinline__ void taps_from(Addr &ad, uint32_t row_bytes, Frag &f0, Frag &f1, f32x4 (&acc)[BM][BN], F between) {
        arrived<NR>(f0);
        phase<T, 0>(ad, f0, acc);
        between(Int<T>());
        arrived<(T < 8 ? NR : 0)>(f1);
        phase<T, 1>(ad, f1, acc);
        if constexpr (T < 8) {
            if constexpr (T + 1 < 6) {                                // the next tap's column moves on to the filter's next row
#pragma unroll
                for (int i = 0; i < BM; ++i) ad.a[(T + 1) % 3][i] += row_bytes;
            }
            taps_from<T + 1>(ad, row_bytes, f0, f1, acc, between);
        }
    }
    __device__ static __forceinline__ Tile tile_at(const ConvArgs &g, uint32_t t) {
        const uint32_t u = g.per_x ? grid_div(t, g.per_x) : t / g.tiles_x, img = g.per_x ? grid_div(u, g.per_y) : u / g.tiles_y;
        return Tile{(uint32_t)__builtin_amdgcn_readfirstlane(img), (uint32_t)__builtin_amdgcn_readfirstlane((u - img * g.tiles_y) * g.th),
                    (uint32_t)__builtin_amdgcn_readfirstlane((t - u * g.tiles_x) * g.tw)};
    }

    __device__ static __forceinline__ void run(const ConvArgs &g, uint32_t first, uint32_t n0, unsigned char *smem) {
        const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const uint32_t wm = wave / GN, wn = wave % GN, lq = lane >> 4, j16 = lane & 15u;
        const uint32_t pw = g.tw + 2u, patch_rows = conv_patch_rows(g.th, g.tw), patch_bytes = conv_patch_bytes(patch_rows);
        unsigned char *const patches = smem + 9u * kConvTap;
        // the patch: 8 pixels per wave instruction; what copy i of this lane fetches, relative to the tile's corner
        uint32_t px_yx[kConvCopies], px_off[kConvCopies];             // (LDS chunk of a pixel's channels: chunk ^ (x & 7))
#pragma unroll
        for (uint32_t i = 0; i < kConvCopies; ++i) {
            const uint32_t row = (i * 8u + wave) * 8u + lane / 8u, y = small_div(row, g.per_pw), x = row - y * pw;
            px_yx[i] = (row < patch_rows ? y : 0xffffu) << 16 | x;  // (past the patch: outside every image)
            px_off[i] = (y * g.W + x) * 128u + ((lane ^ x) & 7u) * 16u;
        }
        uint64_t zero_page = (uint64_t)(uintptr_t)conv_zero_page;
        asm volatile("" : "+s"(zero_page));                           // kept, not loaded again for every copy
        struct Corner { uint32_t h, w; uint64_t at, to_zero; };           // of a patch: image row and column, address
        auto corner_of = [&](const Tile &t) {
            const int h = (int)t.p0 - (int)g.pad, w = (int)t.q0 - (int)g.pad;
            uint64_t at = (uint64_t)(uintptr_t)g.X + (uint64_t)(((int64_t)(t.img * g.H) + h) * (int64_t)g.W + w) * 128u;
            asm volatile("" : "+s"(at));                              // computed here, not again for every copy
            return Corner{(uint32_t)h, (uint32_t)w, at, zero_page - at};
        };
        auto copy_px = [&](const Corner &c, uint32_t buf, uint32_t i) {
            const uint32_t r8 = i * 8u + wave;
            if (r8 * 1024u >= patch_bytes) return;
            const bool ok = (c.h + (px_yx[i] >> 16) < g.H) & (c.w + (px_yx[i] & 0xffffu) < g.W);     // (negative ones wrap round)
            const uint32_t lo = ok ? px_off[i] : (uint32_t)c.to_zero, hi = ok ? 0u : (uint32_t)(c.to_zero >> 32);
            conv_dma16(reinterpret_cast<const void *>(c.at + (((uint64_t)hi << 32) | lo)), patches + buf + r8 * 1024u);
        };
        Tile cur = tile_at(g, first);
        const Corner first_corner = corner_of(cur);
#pragma unroll
        for (uint32_t i = 0; i < kConvCopies; ++i) copy_px(first_corner, 0u, i);
        // filter taps: one wave instruction per tap and wave, 8 rows of [64 channels][64 outputs], swizzled on the source side
        {
            const uint32_t kr = wave * 8u + lane / 8u, col = n0 + ((lane & 7u) ^ swzB<TN>(kr)) * 8u;
            const char *src = reinterpret_cast<const char *>(g.Wt) + (kr * g.N + (col < g.N ? col : n0)) * 2u;   // clamp: garbage columns are never stored
            for (uint32_t t = 0; t < 9u; ++t, src += (uint64_t)g.N * 128u) conv_dma16(src, smem + t * kConvTap + wave * 1024u);
        }
        // fragment addresses: output pixel i of the tile (row i / tw, column i % tw) reads the patch from its own corner on
        const uint32_t sbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
        uint32_t a0[3][BM], out_yx[BM], out_off[BM];
#pragma unroll
        for (int i = 0; i < BM; ++i) {
            const uint32_t px = wm * WM + i * 16u + j16, yy = small_div(px, g.per_tw), x = px - yy * g.tw, y = yy < g.th ? yy : 0u;
#pragma unroll
            for (uint32_t s = 0; s < 3u; ++s) {
                const uint32_t col = x + s, row = y * pw + col;
                a0[s][i] = sbase + 9u * kConvTap + row * 128u + ((lq ^ (col & 7u)) << 4);
            }
            out_yx[i] = (yy < g.th ? yy : 0xffffu) << 16 | x;         // (rows beyond the tile are never stored)
            out_off[i] = ((y * g.Q + x) * g.N) * ES;
        }
        const uint32_t rb = lq * 8u + (j16 >> 2), colb = wn * WN + (j16 & 3u) * 4u;
        Addr ad;
        ad.b[0][0] = sbase + rb * (TN * 2) + (((colb >> 3) ^ swzB<TN>(rb)) << 4) + (colb & 7u) * 2u;
        ad.b[0][1] = ad.b[0][0] ^ 32u;
#pragma unroll
        for (int j = 0; j < BN; ++j) ad.b[1][j] = ad.b[0][j] + 65536u;

        // stores: lane l holds pixel l % 16, channels 4 * (l / 16) .. + 3 of every 16 x 16 block; for 16-bit results two
        // neighbouring blocks swap their odd and even 16-lane rows, which leaves 8 channels of one of them
        const uint32_t c0 = n0 + wn * WN;
        f32x4 bv[BN];
#pragma unroll
        for (int j = 0; j < BN; ++j) {
            const uint32_t c = c0 + j * 16u + lq * 4u;
            bv[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (g.bias != nullptr && c < g.N) {
#pragma unroll
                for (int e = 0; e < 4; ++e) bv[j][e] = g.bias[c + e];
            }
        }
        const uint32_t image_bytes = g.P * g.Q * g.N * ES;
        Tile out = cur;
        bool stored = false;                                          // nothing to store during the first tile
        f32x4 acc[BM][BN], old[BM][BN];
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j) old[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // of tile `out`; offsets out of range are dropped
        const uint32_t cs = OUT16 ? c0 + (lq & 1u) * 16u + (lq >> 1) * 8u : c0 + lq * 4u;
        auto store = [&](int s) {
            const uint32_t origin = ((out.p0 * g.Q + out.q0) * g.N) * ES;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<char *>(g.Y) + (uint64_t)out.img * image_bytes + origin, 0, (int)(stored ? image_bytes - origin : 0u), 0x00020000);
            const int i = OUT16 ? s : s / BN, j = OUT16 ? 0 : s % BN;
            const bool on = (out_yx[i] >> 16 < g.P - out.p0) & ((out_yx[i] & 0xffffu) < g.Q - out.q0) & (cs + j * 16u < g.N);
            const uint32_t o = on ? out_off[i] + (cs + j * 16u) * ES : 0x80000000u;
            conv_u32x4 v;
            if constexpr (OUT16) {
                auto pack = [](float a, float b) -> uint32_t {        // both rounded to nearest even
                    if constexpr (DT == DT_F16) return (uint32_t)out_cvt<OUT_F16>(a) | ((uint32_t)out_cvt<OUT_F16>(b) << 16);
                    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(conv_f32x2{a, b}, conv_bf16x2));
                };
                const auto lo = __builtin_amdgcn_permlane16_swap(pack(old[i][0][0], old[i][0][1]), pack(old[i][1][0], old[i][1][1]), false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap(pack(old[i][0][2], old[i][0][3]), pack(old[i][1][2], old[i][1][3]), false, false);
                v = conv_u32x4{lo[0], hi[0], lo[1], hi[1]};
            } else v = __builtin_bit_cast(conv_u32x4, old[i][j]);
            __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)o, 0, KEEP == 2 ? 0 : KEEP == 1 ? 16 : 18);        // sc1, sc1 | nt
        };

        conv_wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        uint32_t buf = 0;
        for (uint32_t t = first;;) {
            // the patch of tile t has landed; every wave is done with the other one
            const uint32_t next = t + g.walkers;
            const bool more = next < g.tiles;
            const Tile nt = more ? tile_at(g, next) : cur;
            if (more) {
                const Corner nc = corner_of(nt);
#pragma unroll
                for (uint32_t i = 0; i < kConvCopies; ++i) copy_px(nc, patch_bytes - buf, i);
            }
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < BM; ++j) ad.a[i][j] = a0[i][j] + buf;
            Frag f0, f1;
            read_as<0, 0>(ad, f0);
            read_bs<0, 0>(ad, f0);
            read_as<0, 1>(ad, f1);
            read_bs<0, 1>(ad, f1);
#pragma unroll
            for (int i = 0; i < BM; ++i) ad.a[0][i] += pw * 128u;
            taps_from<0>(ad, pw * 128u, f0, f1, acc, [&](auto T) {    // the stores of the tile before go with the taps
                constexpr int t = decltype(T)::value;
#pragma unroll
                for (int q = t * NS / 8; q < (t + 1) * NS / 8; ++q)
                    if (q < NS) store(q);
            });
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j) old[i][j] = g.bias != nullptr ? acc[i][j] + bv[j] : acc[i][j];
            out = cur;
            stored = true;
            if (!more) break;
            conv_wait_vm<NS>();                                       // memory operations end in order: all but the stores, issued after the patch
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            buf = patch_bytes - buf;
            cur = nt;
            t = next;
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) store(q);
    }
};

template <int DT, bool OUT16, int BM, int KEEP>
__global__ __launch_bounds__(512, 1) void ft_conv_patch(ConvArgs g) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    // workgroup b runs on XCD b % num_xcds: an XCD takes one contiguous run of the walkers, and with it neighbouring tiles
    // (whose patches overlap) at a time
    const uint32_t nx = g.num_xcds, b = blockIdx.x, n = g.walkers * g.cols;
    uint32_t x, u;
    if (nx == 8) { x = b & 7u; u = x * (n >> 3) + (x < (n & 7u) ? x : n & 7u) + (b >> 3); }
    else { x = b % nx; u = x * (n / nx) + (x < n % nx ? x : n % nx) + b / nx; }
    const uint32_t walker = grid_div(u, g.per_cols);
    ConvBody<DT, OUT16, BM, KEEP>::run(g, __builtin_amdgcn_readfirstlane(walker), __builtin_amdgcn_readfirstlane((u - walker * g.cols) * 64u), smem);
}

}  // namespace ftk

template <int DT, bool OUT16, int BM, int KEEP>
static int launch(const ftk::ConvArgs *g, uint32_t lds_bytes, void *stream) {
    constexpr auto kernel = &ftk::ft_conv_patch<DT, OUT16, BM, KEEP>;
    const hipError_t e = ftk::raise_lds_limit<kernel>();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(kernel, dim3(g->walkers * g->cols), dim3(512), lds_bytes, static_cast<hipStream_t>(stream), *g);
    return (int)hipGetLastError();
}
template <int DT, bool OUT16, int BM>
static int launch_keep(const ftk::ConvArgs *g, int keep, uint32_t lds_bytes, void *stream) {
    switch (keep) {
        case 0: return launch<DT, OUT16, BM, 0>(g, lds_bytes, stream);
        case 1: return launch<DT, OUT16, BM, 1>(g, lds_bytes, stream);
        default: return launch<DT, OUT16, BM, 2>(g, lds_bytes, stream);
    }
}
template <int DT, bool OUT16>
static int launch_bm(const ftk::ConvArgs *g, int bm, int keep, uint32_t lds_bytes, void *stream) {
    switch (bm) {
        case 1: return launch_keep<DT, OUT16, 1>(g, keep, lds_bytes, stream);
        case 2: return launch_keep<DT, OUT16, 2>(g, keep, lds_bytes, stream);
        case 3: return launch_keep<DT, OUT16, 3>(g, keep, lds_bytes, stream);
        default: return launch_keep<DT, OUT16, 4>(g, keep, lds_bytes, stream);
    }
}

extern "C" int ft_launch_conv(const ftk::ConvArgs *g, int dt, int out16, int bm, int keep, uint32_t lds_bytes, void *stream) {
    if (dt) return out16 ? launch_bm<1, true>(g, bm, keep, lds_bytes, stream) : launch_bm<1, false>(g, bm, keep, lds_bytes, stream);
    return out16 ? launch_bm<0, true>(g, bm, keep, lds_bytes, stream) : launch_bm<0, false>(g, bm, keep, lds_bytes, stream);
}
