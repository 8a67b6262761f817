// Large products in 256 x 256 blocks of C, eight waves and the whole LDS of a CU each.
//
// What bounds a large product on this device is power: the MFMAs alone run at 2.4 PFLOP/s on zeros and at 1.7-1.8
// (32x32x16) or 2.07 (16x16x32) on N(0,1) operands, the loop below at 1.65 on zeros and 1.4-1.5 on N(0,1).  (Counters of 8192 x
// 11008 x 4096 bf16, six launches in a row: the clock falls from 1.84 to 1.49 GHz, the matrix cores are busy for 80 % of the
// cycles; LDS is active for 51 % of them, four tenths of that bank conflicts.)  Against
// the tile bodies (gemm_fast.h, 1.1-1.2 PFLOP/s on the same 256 x 256 tile) it
//   - uses v_mfma_f32_16x16x32, which does the same products for less power than 32x32x16;
//   - keeps the fragments of one k-step in registers while the MFMAs of the other run, so that no MFMA waits for
//     LDS: the second k-step of tile t is read during the first one's MFMAs, the first k-step of tile t + 1 during the
//     second one's.  A tile's LDS is free half-way through its MFMAs: there stands the one barrier per k-tile;
//   - uses all 160 KB: A and B tiles take turns in five slots of 32 KB, so A is fetched two and a half tiles ahead
//     and B one and a half, with the copies spread between the MFMAs;
//   - hands the operands to the MFMA the other way round, so that a lane's four accumulator registers are four
//     neighbouring columns of C: stores are 16 bytes per lane (16-bit outputs: after a swap between two blocks'
//     lanes), where they were 4 or 2;
//   - copies with buffer loads and without a branch in the steady loop, the last three k-tiles run a copy of it (1500 x 11008 x
//     4096 145.7 -> 139.5 us, 8192 x 11008 x 4096 544 -> 533).  A swizzle of A free of bank conflicts for these reads changed
//     nothing: the LDS is not what the MFMAs wait for.
// 8192 x 11008 x 4096 bf16, the tile bodies against the first form of this: 650 -> 562 us; 4096^3: 113 -> 97; 8192^3: 883 -> 744.
//
// A block is a CU's work for 60-90 us, so a last round of few blocks is expensive: the host deals the blocks that
// would make it as halves of 128 rows (see big_schedule in host.cpp), a shorter body of the same design.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "big_gemm.h"
#include "gemm_body.h"
#include "lds_limit.h"

namespace ftk {

typedef uint32_t big_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t big_u32x2 __attribute__((ext_vector_type(2)));
typedef float big_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 big_bf16x2 __attribute__((ext_vector_type(2)));

template <int OFF> __device__ __forceinline__ big_u32x4 big_read_b128(uint32_t addr) {
    big_u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF> __device__ __forceinline__ big_u32x2 big_read_tr16(uint32_t addr) {
    big_u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int N> __device__ __forceinline__ void big_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
template <int IMM> __device__ __forceinline__ void big_copy16(__amdgpu_buffer_rsrc_t r, unsigned char *lds_wave_base, uint32_t lane_off, uint32_t tile_off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds_wave_base, 16, (int)lane_off, (int)tile_off, IMM, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t big_rsrc(const uint16_t *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p), 0, (int)bytes, 0x00020000);
}
template <int Q, int E, typename F> __device__ __forceinline__ void big_each(F f) {
    if constexpr (Q < E) { f(std::integral_constant<int, Q>{}); big_each<Q + 1, E>(f); }
}

// One block of GM * WM rows by GN * WN columns.  SLOTS = 5: A and B tiles are equally large and take turns in five
// slots (tile t: A in slot 2t mod 5, B in slot (2t + 1) mod 5).  Otherwise a ring of STAGES stages of A and B.
template <int DT, int WM, int WN, int GM, int GN, int STAGES, bool SLOTS>
struct BigBody {
    static constexpr int TM = GM * WM, TN = GN * WN, NW = GM * GN, BM = WM / 16, BN = WN / 16;
    static constexpr int A_BYTES = TM * 128, B_BYTES = TN * 128;      // 64 k
    static constexpr int LA = A_BYTES / NW / 1024, LB = B_BYTES / NW / 1024;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int NR = BM + 2 * BN, NM = BM * BN;
    static_assert(!SLOTS || A_BYTES == B_BYTES, "five equal slots");
    static_assert(NW == 8 && TN >= 128 && (SLOTS ? 5 * A_BYTES : STAGES * STAGE) <= 163840, "eight waves, one CU's LDS");
    static_assert(SLOTS || STAGES == 3, "the furthest copy is of tile t + 3");
    static constexpr int AHEAD = SLOTS ? LA : (STAGES - 2) * (LA + LB);   // copies in flight beyond the next tile, steady state

    struct Frag { big_u32x4 a[BM]; big_u32x2 b[BN][2]; };

    // r-th LDS read of k-step KS's fragments: B first (its blocks are all used by the first row of blocks)
    template <int KS, int R> __device__ static __forceinline__ void read_one(uint32_t aa, const uint32_t (&ba)[BN], Frag &f) {
        if constexpr (R < 2 * BN) f.b[R / 2][R % 2] = big_read_tr16<(KS * 32 + (R % 2) * 4) * TN * 2>(ba[R / 2]);
        else f.a[R - 2 * BN] = big_read_b128<(R - 2 * BN) * 16 * 128>(aa);
    }
    template <int KS, int R, int E> __device__ static __forceinline__ void read_range(uint32_t aa, const uint32_t (&ba)[BN], Frag &f) {
        if constexpr (R < E && R < NR) {
            read_one<KS, R>(aa, ba, f);
            read_range<KS, R + 1, E>(aa, ba, f);
        }
    }
    // every read of the set has arrived; its registers are produced here
    __device__ static __forceinline__ void arrived(Frag &f) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < BM; ++i) asm volatile("" : "+v"(f.a[i]));
#pragma unroll
        for (int i = 0; i < BN; ++i) asm volatile("" : "+v"(f.b[i][0]), "+v"(f.b[i][1]));
    }
    // m-th MFMA of a k-step: rows of blocks in turn, columns back and forth, so that one operand stays
    __device__ static __forceinline__ void mfma_one(const Frag &f, f32x4 (&acc)[BM][BN], int m) {
        const int bi = m / BN, bj = (bi & 1) ? BN - 1 - m % BN : m % BN;
        const uint4 b = make_uint4(f.b[bj][0][0], f.b[bj][0][1], f.b[bj][1][0], f.b[bj][1][1]);
        acc[bi][bj] = mfma16<DT>(b, __builtin_bit_cast(uint4, f.a[bi]), acc[bi][bj]);
    }
    // The MFMAs of `use`, with the reads of `fill` (k-step KS of some tile) in the first three quarters and, where COPY,
    // LA + LB copies spread over all of them.  Pinned: left alone, the compiler gathers the reads in front.
    template <int KS, bool COPY, int M = 0, typename F>
    __device__ static __forceinline__ void phase(uint32_t aa, const uint32_t (&ba)[BN], Frag &fill, const Frag &use, f32x4 (&acc)[BM][BN], F copy) {
        read_range<KS, M * NR * 4 / (NM * 3), (M + 1) * NR * 4 / (NM * 3)>(aa, ba, fill);
        if constexpr (COPY) {
            constexpr int L = LA + LB;
            big_each<M * L / NM, (M + 1) * L / NM>(copy);
        }
        mfma_one(use, acc, M);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (M + 1 < NM) phase<KS, COPY, M + 1>(aa, ba, fill, use, acc, copy);
    }

    __device__ static __forceinline__ void run(const BigArgs &g, uint32_t m0, uint32_t n0, unsigned char *smem) {
        const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const uint32_t wm = wave / GN, wn = wave % GN;
        const uint32_t nk = g.K / 64u;
        // copy assignments, as in gemm_fast.h: wave instruction i fills 1 KB of the tile.  Buffer loads: a lane's offset stays, A's
        // k-tile is the scalar offset, B's moves the descriptor (an operand of 4 GB is in reach); A's neighbouring kilobytes
        // share one M0 through the immediate, which moves the source too; rows below A's end read as zeros by the bound
        const __amdgpu_buffer_rsrc_t ar = big_rsrc(g.A + (uint64_t)m0 * g.K, (g.M - m0 < (uint32_t)TM ? g.M - m0 : (uint32_t)TM) * g.K * 2u);
        uint32_t off_a[LA], off_b[LB];
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const uint32_t row = wave * (LA * 8) + i * 8 + lane / 8u, kc = (lane & 7u) ^ swzA(row);
            off_a[i] = (row * g.K + kc * 8u) * 2u - (i & 3) * 1024u;  // (K >= 64: not below zero)
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const uint32_t o = wave * (LB * 1024) + i * 1024 + lane * 16u, kr = o / (TN * 2), p = o % (TN * 2) / 16u;
            const uint32_t col = n0 + (p ^ swzB<TN>(kr)) * 8u;
            off_b[i] = (kr * g.N + (col < g.N ? col : n0)) * 2u;      // clamp: garbage columns are never stored
        }
        auto copy_a = [&](uint32_t t, uint32_t slot, auto ic) {
            constexpr int i = decltype(ic)::value;
            big_copy16<(i & 3) * 1024>(ar, smem + slot + wave * (LA * 1024) + (i / 4) * 4096, off_a[i], t * 128u);
        };
        auto copy_b = [&](uint32_t t, uint32_t slot, auto ic) {
            constexpr int i = decltype(ic)::value;
            big_copy16<0>(big_rsrc(g.B + (uint64_t)t * (g.N * 64u), g.N * 128u), smem + slot + wave * (LB * 1024) + i * 1024, off_b[i], 0u);
        };
        // fragment addresses (see gemm_fast.h)
        const uint32_t sbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
        const uint32_t ra = wm * WM + (lane & 15u);
        const uint32_t fa = sbase + ra * 128u + (((lane >> 4) ^ swzA(ra)) << 4);
        const uint32_t j16 = lane & 15u, rb = (lane >> 4) * 8u + (j16 >> 2);
        uint32_t fb[BN];
#pragma unroll
        for (int j = 0; j < BN; ++j) {
            const uint32_t col = wn * WN + j * 16 + (j16 & 3u) * 4u;
            fb[j] = sbase + rb * (TN * 2) + (((col >> 3) ^ swzB<TN>(rb)) << 4) + (col & 7u) * 2u;
        }
        f32x4 acc[BM][BN];
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

        // slots of the tile being consumed
        uint32_t sa = 0, sb = A_BYTES;
        auto next = [](uint32_t s) -> uint32_t {
            constexpr uint32_t STEP = SLOTS ? 2 * A_BYTES : STAGE, RING = SLOTS ? 5 * A_BYTES : STAGES * STAGE;
            return s + STEP >= RING ? s + STEP - RING : s + STEP;
        };
        // prologue: the ring full
        {
            constexpr int TILES = SLOTS ? 3 : STAGES;
            uint32_t pa = sa, pb = sb;
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                if ((uint32_t)t < nk) {
                    big_each<0, LA>([&](auto i) { copy_a(t, pa, i); });
                    if (!SLOTS || t < 2) big_each<0, LB>([&](auto i) { copy_b(t, pb, i); });
                }
                pa = next(pa); pb = next(pb);
            }
            constexpr int BEHIND = SLOTS ? 2 * LA + LB : (STAGES - 1) * (LA + LB);     // copies behind tile 0
            if (nk >= (uint32_t)TILES) big_wait_vm<BEHIND>();
            else big_wait_vm<0>();
        }
        __builtin_amdgcn_s_barrier();
        Frag f0, f1;
        uint32_t ba[BN];
#pragma unroll
        for (int j = 0; j < BN; ++j) ba[j] = fb[j] + sb;
        read_range<0, 0, NR>(fa + sa, ba, f0);
        auto step = [&](uint32_t t, auto steady_c) {
            constexpr bool STEADY = decltype(steady_c)::value;        // every copy of the steady state is due
            arrived(f0);
            __builtin_amdgcn_sched_barrier(0);
            phase<1, false>((fa ^ 64u) + sa, ba, f1, f0, acc, [](auto) {});
            arrived(f1);
            __builtin_amdgcn_sched_barrier(0);
            // Tile t's LDS has been read by this wave; tile t + 1 must have landed.  In flight beyond it: A of t + 2 (slots), or
            // the stages up to t + STAGES - 1.
            const uint32_t behind = nk - 1u - t;                      // tiles after t
            if (STEADY || (SLOTS ? behind >= 2u : behind >= (uint32_t)STAGES - 1u)) big_wait_vm<AHEAD>();
            else big_wait_vm<0>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t na = next(sa), nb = next(sb);
#pragma unroll
            for (int j = 0; j < BN; ++j) ba[j] = fb[j] + nb;
            // (past the last tile the reads fetch what happens to be there, for nobody)
            if constexpr (SLOTS) {
                const bool more_b = STEADY || t + 2u < nk;
                phase<0, true>(fa + na, ba, f0, f1, acc, [&](auto q) {
                    constexpr int Q = decltype(q)::value;
                    if constexpr (Q < LB) { if (more_b) copy_b(t + 2u, sa, q); }
                    else if constexpr (STEADY) copy_a(t + 3u, sb, std::integral_constant<int, Q - LB>{});
                });
            } else {
                phase<0, STEADY>(fa + na, ba, f0, f1, acc, [&](auto q) {
                    constexpr int Q = decltype(q)::value;
                    if constexpr (Q < LA) copy_a(t + STAGES, sa, q);
                    else copy_b(t + STAGES, sb, std::integral_constant<int, Q - LA>{});
                });
            }
            sa = na; sb = nb;
        };
        uint32_t t = 0;
        for (; t + 3u < nk; ++t) step(t, std::true_type{});           // (A of t + 3, the furthest copy)
        for (; t < nk; ++t) step(t, std::false_type{});
        arrived(f0);                                                  // nothing of the last reads outlives the loop

        // ---- epilogue: lane l holds row l % 16, columns 4 * (l / 16) .. + 3 of every 16 x 16 block -------------
        const uint32_t row0 = m0 + wm * WM + (lane & 15u), col0 = n0 + wn * WN, q4 = lane >> 4;
        if (g.bias != nullptr) {
#pragma unroll
            for (int j = 0; j < BN; ++j) {
                const uint32_t c = col0 + j * 16u + q4 * 4u;
                f32x4 bv = {0.f, 0.f, 0.f, 0.f};
                if (c < g.N) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) bv[e] = g.bias[c + e];
                }
#pragma unroll
                for (int i = 0; i < BM; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][e] += bv[e];
            }
        }
        if (!g.out16) {
            // Rows on 64-byte blocks (an instruction fills 16 of them) are streamed and written through the L2 (sc1 nt): nothing is
            // left to write back when the launch ends, or beside the next block's copies.  Kept / this, bf16, us: 4096^3 103.5 /
            // 99.9, 2500 x 4096 x 4096 76.2 / 72.9, 600 x 11008 x 4096 62.0 / 55.8, 3000 x 11008 x 4096 236.6 / 231.8; streamed but not written
            // through 105.4, 75.7, 57.8, 241.  (16-bit results are kept: 8192 x 11008 x 4096 517 / 519, written through alone 529.)
            const uint32_t row_bytes = g.N * 4u, lane_row = (lane & 15u) * row_bytes, r0 = m0 + wm * WM;
            if (r0 < g.M && col0 < g.N) {
                const uint32_t rows = g.M - r0 < (uint32_t)WM ? g.M - r0 : (uint32_t)WM, columns = g.N - col0;
                const __amdgpu_buffer_rsrc_t rc =
                    __builtin_amdgcn_make_buffer_rsrc(static_cast<float *>(g.C) + ((uint64_t)r0 * g.N + col0), 0, (int)((rows - 1u) * row_bytes + columns * 4u), 0x00020000);
                auto store = [&](auto policy) {
#pragma unroll
                    for (int i = 0; i < BM; ++i)
#pragma unroll
                        for (int j = 0; j < BN; ++j) {
                            const uint32_t c = j * 16u + q4 * 4u;     // (rows go into the lane's offset, see grid_gemm.hip)
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(big_u32x4, acc[i][j]), rc, (int)(c < columns ? lane_row + i * 16u * row_bytes + c * 4u : 0x80000000u),
                                                                   0, decltype(policy)::value);
                        }
                };
                if (g.through) store(std::integral_constant<int, 18>{});
                else store(std::integral_constant<int, 0>{});
            }
        } else {
            // two neighbouring blocks: after the swap of odd and even 16-lane rows a lane holds 8 columns of one of them
            uint16_t *const C = static_cast<uint16_t *>(g.C);
            auto pack = [](float x, float y) -> uint32_t {            // both rounded to nearest even
                if constexpr (DT == DT_F16) return (uint32_t)out_cvt<OUT_F16>(x) | ((uint32_t)out_cvt<OUT_F16>(y) << 16);
                else return __builtin_bit_cast(uint32_t, __builtin_convertvector(big_f32x2{x, y}, big_bf16x2));
            };
            const uint32_t cc = col0 + (q4 & 1u) * 16u + (q4 >> 1) * 8u;
#pragma unroll
            for (int i = 0; i < BM; ++i) {
                const uint32_t r = row0 + i * 16u;
#pragma unroll
                for (int j = 0; j < BN; j += 2) {
                    const auto lo = __builtin_amdgcn_permlane16_swap(pack(acc[i][j][0], acc[i][j][1]), pack(acc[i][j + 1][0], acc[i][j + 1][1]), false, false);
                    const auto hi = __builtin_amdgcn_permlane16_swap(pack(acc[i][j][2], acc[i][j][3]), pack(acc[i][j + 1][2], acc[i][j + 1][3]), false, false);
                    const big_u32x4 v = {lo[0], hi[0], lo[1], hi[1]};
                    const uint32_t c = cc + j * 16u;
                    if (r < g.M && c < g.N) *reinterpret_cast<big_u32x4 *>(C + (uint64_t)r * g.N + c) = v;
                }
            }
        }
    }
};

template <int DT>
__global__ __launch_bounds__(512, 2) void ft_big(BigArgs g) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const BigBlock t = big_block(blockIdx.x, g.rows, g.cols, g.group, g.n_full, g.n_half, g.num_xcds);
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(t.m0), n0 = __builtin_amdgcn_readfirstlane(t.n0);
    if (!t.half) BigBody<DT, 128, 64, 2, 4, 2, true>::run(g, m0, n0, smem);
    else BigBody<DT, 64, 64, 2, 4, 3, false>::run(g, m0, n0, smem);
}

}  // namespace ftk

template <int DT>
static int launch(const ftk::BigArgs *g, void *stream) {
    const hipError_t e = ftk::raise_lds_limit<&ftk::ft_big<DT>>();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(ftk::ft_big<DT>, dim3(g->n_full + g->n_half), dim3(512), 163840, static_cast<hipStream_t>(stream), *g);
    return (int)hipGetLastError();
}

extern "C" int ft_launch_big(const ftk::BigArgs *g, int dt, void *stream) { return dt ? launch<1>(g, stream) : launch<0>(g, stream); }
