// Matmuls of the middle range: one grid of equal tiles, at most three per CU.
//
// What bounds these launches (a few hundred tiles, 12 to 64 k-tiles of 64) is neither memory nor the matrix cores but the
// instructions a wave issues: a SIMD with one or two waves issues one instruction of a wave every four cycles, and a k-tile of
// a small wave tile holds few MFMAs to issue them beside (128 x 64 on four waves: 16 MFMAs of 16 cycles).  Measured with the
// stores left out, a k-tile of 128 x 64 took 0.28 us whether its copies ran or not and however far ahead the fragments were
// read; with the loop below, half the instructions, 0.20 us.  So
//   - the copies are buffer loads into LDS: the lane's offset never changes, the k-tile is the instruction's scalar offset,
//     neighbouring kilobytes share one M0 through the instruction's immediate (which moves the source too: the lane's offset
//     takes it back), rows below the operand's end read as zeros by the descriptor's bound, so nothing is clamped or predicated;
//   - the steady loop has one form of every wait and no branch; the last tiles, STAGES + 1 at most, run a copy of it in which a copy, if
//     one is still due, stands in front of the MFMAs;
//   - both k-steps of a tile are in registers before its first MFMA; the next tile's are read beside them, so there is one
//     barrier and one wait for LDS per k-tile;
//   - MFMAs are 16x16x32, operands handed over the other way round (a lane's four registers are four neighbouring columns).
// Beyond that a CU pulls its operand panels through one path at 33 to 40 bytes a cycle (a k-tile's bytes over the steps of kGridCost in
// host.cpp), the tile's bytes set the time; the matrix cores are busy for 13 to 44 % of it and the LDS for a third at most.
// f16, everything in the caches, us, the program's tiles against this: 688 x 2304 x 768 8.0 / 6.2, x 768 x 768 6.9 / 4.6, x 3072 x 768
// 8.1 / 7.3, x 768 x 3072 12.9 / 10.9, 1600 x 768 x 3072 16.9 / 14.2; with fp32 results 688 x 768 x 768 6.8 / 4.9, 429 x 3072 x 768
// 7.9 / 6.1, 131 x 3072 x 768 5.9 / 4.4 (16 bytes per lane straight from the accumulators).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gemm_body.h"
#include "grid_gemm.h"
#include "lds_limit.h"

namespace ftk {

constexpr uint32_t kGridWindow = 4;                                   // k-tiles whose order differs from row to row of the tiles

typedef uint32_t grid_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t grid_u32x2 __attribute__((ext_vector_type(2)));
typedef float grid_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 grid_bf16x2 __attribute__((ext_vector_type(2)));

template <int OFF> __device__ __forceinline__ grid_u32x4 grid_read_b128(uint32_t addr) {
    grid_u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF> __device__ __forceinline__ grid_u32x2 grid_read_tr16(uint32_t addr) {
    grid_u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int N> __device__ __forceinline__ void grid_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
template <int IMM> __device__ __forceinline__ void grid_copy16(__amdgpu_buffer_rsrc_t r, unsigned char *lds_wave_base, uint32_t lane_off, uint32_t tile_off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds_wave_base, 16, (int)lane_off, (int)tile_off, IMM, 0);
}
// Swizzle of A's 16-byte chunks: a wave reads 16 rows at four neighbouring chunks, for which row & 7 lets the LDS serve 252 bytes a
// cycle (eight waves reading; swzA, made for 32 rows at two chunks, 128); the counters show no bank conflicts.
__device__ __forceinline__ uint32_t grid_swzA(uint32_t row) { return row & 7u; }
// Swizzle of B's 16-byte chunks: as swzB, and closed within rows of 24 chunks (groups of eight, neighbouring rows 32 banks apart).
template <int TN> __device__ __forceinline__ uint32_t grid_swzB(uint32_t row) {
    static_assert(TN == 32 || TN == 64 || TN == 128 || TN == 192 || TN == 256, "rows of B that the transposing reads find free of conflicts");
    if constexpr (TN == 192) return swzB<64>(row);
    else return swzB<TN>(row);
}

template <int DT, bool OUT16, int WM, int WN, int GM, int GN, int GK, int S>
struct GridBody {
    static constexpr int TM = GM * WM, TN = GN * WN, NWG = GM * GN, BM = WM / 16, BN = WN / 16, NB = BM * BN;
    static constexpr int A_BYTES = TM * 128, B_BYTES = TN * 128, STAGE = A_BYTES + B_BYTES, RING = S * STAGE;
    static constexpr int LA = A_BYTES / NWG / 1024, LB = B_BYTES / NWG / 1024, L = LA + LB;      // copies of a wave per k-tile
    static constexpr int NR1 = BM + 2 * BN, NR = 2 * NR1, NM = 2 * NB;                            // LDS reads, MFMAs per k-tile
    static_assert(LA * NWG * 1024 == A_BYTES && LB * NWG * 1024 == B_BYTES, "whole kilobytes per wave");
    static_assert(S >= 3 && (S - 1) * L <= 63, "vmcnt is 6 bits");
    static constexpr int NS = (int)grid_sums(WM, WN, GK, OUT16);                                      // sums kept of an output
    static_assert(GK == 1 || NB % GK == 0, "the groups share out the blocks");
    struct Frag { grid_u32x4 a[2][BM]; grid_u32x2 b[2][BN][2]; };

    // r-th LDS read of a k-tile's fragments: k-step by k-step, B first (its blocks are all used by the first row of blocks)
    template <int R> __device__ static __forceinline__ void read_one(uint32_t aa, const uint32_t (&ba)[BN], Frag &f) {
        constexpr int KS = R / NR1, Q = R % NR1;
        if constexpr (Q < 2 * BN) f.b[KS][Q / 2][Q % 2] = grid_read_tr16<(KS * 32 + (Q % 2) * 4) * TN * 2>(ba[Q / 2]);
        else f.a[KS][Q - 2 * BN] = grid_read_b128<(Q - 2 * BN) * 16 * 128>(KS ? aa ^ 64u : aa);
    }
    template <int R, int E> __device__ static __forceinline__ void read_range(uint32_t aa, const uint32_t (&ba)[BN], Frag &f) {
        if constexpr (R < E && R < NR) {
            read_one<R>(aa, ba, f);
            read_range<R + 1, E>(aa, ba, f);
        }
    }
    // every read of the set has arrived; its registers are produced here
    __device__ static __forceinline__ void arrived(Frag &f) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int i = 0; i < BM; ++i) asm volatile("" : "+v"(f.a[k][i]));
#pragma unroll
            for (int i = 0; i < BN; ++i) asm volatile("" : "+v"(f.b[k][i][0]), "+v"(f.b[k][i][1]));
        }
    }
    // q-th MFMA of a k-tile: rows of blocks in turn, columns back and forth, so that one operand stays
    template <int ODD> __device__ static __forceinline__ void mfma_one(const Frag &f, f32x4 (&acc)[NS][BM][BN], int q) {
        const int ks = q / NB, m = q % NB, bi = m / BN, bj = (bi & 1) ? BN - 1 - m % BN : m % BN;
        const uint4 b = make_uint4(f.b[ks][bj][0][0], f.b[ks][bj][0][1], f.b[ks][bj][1][0], f.b[ks][bj][1][1]);
        f32x4 &sum = acc[(ODD * 2 + ks) % NS][bi][bj];
        sum = mfma16<DT>(b, __builtin_bit_cast(uint4, f.a[ks][bi]), sum);
    }
    struct Copies {
        __amdgpu_buffer_rsrc_t ra, rb;
        uint32_t off_a[LA], off_b[LB];                                // the lane's source, less the instruction's immediate
        uint32_t at_a, at_b, next_a, next_b;                          // the k-tile of this wave's group that is asked for next, and the one after it
        uint32_t step_a, step_b, asked, whole, turn;
        // The t-th k-tile in this tile's order: whole windows of kGridWindow k-tiles begin at the turn-th of theirs (see run).
        __device__ __forceinline__ void after(uint32_t t) {
            const uint32_t kt = (t & ~(kGridWindow - 1u)) + ((t + (t < whole ? turn : 0u)) & (kGridWindow - 1u));
            next_a = kt * step_a; next_b = kt * step_b;
        }
        __device__ __forceinline__ void advance() { at_a = next_a; at_b = next_b; }
    };
    template <int Q, int E> __device__ static __forceinline__ void copy(const Copies &c, unsigned char *la, unsigned char *lb) {
        if constexpr (Q < E) {
            if constexpr (Q < LA) grid_copy16<(Q & 3) * 1024>(c.ra, la + (Q / 4) * 4096, c.off_a[Q], c.at_a);
            else grid_copy16<((Q - LA) & 3) * 1024>(c.rb, lb + ((Q - LA) / 4) * 4096, c.off_b[Q - LA], c.at_b);
            copy<Q + 1, E>(c, la, lb);
        }
    }
    // The MFMAs of `use`, with the reads of `fill` in the first half and, where COPY, the copies spread over all of them.
    // Pinned: left alone, the compiler gathers the reads in front.
    template <bool COPY, int ODD, int M = 0>
    __device__ static __forceinline__ void phase(uint32_t aa, const uint32_t (&ba)[BN], Frag &fill, const Frag &use, f32x4 (&acc)[NS][BM][BN], Copies &c,
                                                 unsigned char *la, unsigned char *lb) {
        read_range<M * NR * 2 / NM, (M + 1) * NR * 2 / NM>(aa, ba, fill);
        if constexpr (COPY) copy<M * L / NM, (M + 1) * L / NM>(c, la, lb);
        if constexpr (COPY && M == 1) c.after(++c.asked);             // (scalar work beside the MFMAs)
        mfma_one<ODD>(use, acc, M);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (M + 1 < NM) phase<COPY, ODD, M + 1>(aa, ba, fill, use, acc, c, la, lb);
    }
    // all but the newest min(c, C) k-tiles of this wave's copies have landed
    template <int C> __device__ static __forceinline__ void wait_tiles(uint32_t c) {
        if constexpr (C == 0) grid_wait_vm<0>();
        else {
            if (c >= (uint32_t)C) grid_wait_vm<C * L>();
            else wait_tiles<C - 1>(c);
        }
    }
    __device__ static __forceinline__ uint32_t pack(float x, float y) {                           // both rounded to nearest even
        if constexpr (DT == DT_F16) return (uint32_t)out_cvt<OUT_F16>(x) | ((uint32_t)out_cvt<OUT_F16>(y) << 16);
        else return __builtin_bit_cast(uint32_t, __builtin_convertvector(grid_f32x2{x, y}, grid_bf16x2));
    }
    // Where the rows of C lie on 64-byte blocks and an instruction fills whole ones, results are written through the L2 (sc1): as dirty
    // lines they would be written back when the launch ends, and the next one waits for that.  16-bit results stay in the
    // last-level cache, where the next Matmul finds them: 1500 x 2304 x 768 9.5 -> 8.8 us, 688 x 3072 x 768 7.9 -> 7.6, operands and C from
    // HBM 10.3 -> 9.5 and 8.8 -> 8.4; an encoder's twelve layers on 688 rows 404 -> 394 with weights from HBM, 378 -> 368 without (streamed
    // 444, 429).  fp32 results are streamed as well (sc1 nt): 800 x 4096 x 1984 18.7 -> 18.0, 688 x 768 x 768 5.0 -> 4.9, from HBM 18.8 -> 17.8
    // and 5.2 -> 5.1; without the hint 19.6 from HBM.  Parts of blocks are kept, to meet in L2 (1500 x 3080 x 768, 16-bit, from HBM 13.1 kept,
    // 15.0 written through; 1432 x 3072 x 768, whose waves are 48 columns wide, 12.5 and 14.3; groups, which store 32 bytes of a row,
    // up to 4 % slower).
    static constexpr bool WHOLE = !OUT16 || (GK == 1 && WN % 32 == 0);
    static constexpr int POLICY = OUT16 ? 16 : 18;                     // cache-policy bits: sc1, sc1 | nt
    static constexpr uint32_t ES = OUT16 ? 2 : 4;
    struct Out {                                                      // a wave's part of C
        __amdgpu_buffer_rsrc_t r;                                     // ends with the last row there is
        uint32_t row_bytes, first, columns;                           // first: this lane's row; columns of C from the wave's first one on
    };
    // 16 or 8 bytes at column c of the wave's part, 16 * i rows below the lane's first.  The row goes into the lane's offset: a 16-byte
    // buffer store with its offset in a scalar register still reads its last register when the next instruction may write it
    // already, and the compiler, which keeps the two apart otherwise, takes that form for safe (gfx950: rows 12 to 15 of a block
    // got another block's last column).
    template <bool THROUGH, typename V> __device__ static __forceinline__ void store(const Out &o, uint32_t i, uint32_t c, V v) {
        const uint32_t at = c < o.columns ? o.first + i * 16u * o.row_bytes + c * ES : 0x80000000u;  // (past the end: dropped)
        if constexpr (sizeof(V) == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(grid_u32x4, v), o.r, (int)at, 0, THROUGH ? POLICY : 0);
        else __builtin_amdgcn_raw_buffer_store_b64(v, o.r, (int)at, 0, THROUGH ? POLICY : 0);
    }
    // four neighbouring columns from c on
    template <bool THROUGH> __device__ static __forceinline__ void store4(const Out &o, uint32_t i, uint32_t c, f32x4 v) {
        if constexpr (OUT16) store<THROUGH>(o, i, c, grid_u32x2{pack(v[0], v[1]), pack(v[2], v[3])});
        else store<THROUGH>(o, i, c, v);
    }
    __device__ static __forceinline__ f32x4 bias_of(const GridArgs &g, uint32_t c) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (g.bias != nullptr && c < g.N) __builtin_memcpy(&v, g.bias + c, 16);
        return v;
    }

    // lane l holds row l % 16, columns 4 * (l / 16) .. + 3 of every 16 x 16 block
    template <bool THROUGH>
    __device__ static __forceinline__ void finish(const GridArgs &g, f32x4 (&acc)[BM][BN], const f32x4 *bias, const unsigned char *smem, uint32_t row0, uint32_t col0,
                                                  uint32_t grp, uint32_t wave, uint32_t lane) {
        if (row0 >= g.M || col0 >= g.N) return;
        const uint32_t q4 = lane >> 4, row_bytes = g.N * ES, rows = g.M - row0 < (uint32_t)WM ? g.M - row0 : (uint32_t)WM;
        const Out o = {__builtin_amdgcn_make_buffer_rsrc(static_cast<char *>(g.C) + ((uint64_t)row0 * g.N + col0) * ES, 0, (int)((rows - 1u) * row_bytes + (g.N - col0) * ES), 0x00020000),
                       row_bytes, (lane & 15u) * row_bytes, g.N - col0};
        if constexpr (GK > 1) {
            // added in group order; group g finishes blocks g * PB ..
            constexpr int PB = NB / GK;
            const f32x4 *const x = reinterpret_cast<const f32x4 *>(smem);
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const uint32_t b = grp * PB + p;
                f32x4 s = x[(wave * NB + b) * 64u + lane];
#pragma unroll
                for (int q = 1; q < GK; ++q) s += x[((q * NWG + wave) * NB + b) * 64u + lane];
                s += bias[p];
                store4<THROUGH>(o, b / BN, (b % BN) * 16u + q4 * 4u, s);
            }
        } else {
            // 16-bit results, two neighbouring blocks: after the swap of odd and even 16-lane rows a lane holds 8 columns of one of them
            const uint32_t cc = (q4 & 1u) * 16u + (q4 >> 1) * 8u;
#pragma unroll
            for (int i = 0; i < BM; ++i) {
#pragma unroll
                for (int j = 0; j < BN; ++j) acc[i][j] += bias[j];
                if constexpr (OUT16) {
#pragma unroll
                    for (int j = 0; j + 1 < BN; j += 2) {
                        const auto lo = __builtin_amdgcn_permlane16_swap(pack(acc[i][j][0], acc[i][j][1]), pack(acc[i][j + 1][0], acc[i][j + 1][1]), false, false);
                        const auto hi = __builtin_amdgcn_permlane16_swap(pack(acc[i][j][2], acc[i][j][3]), pack(acc[i][j + 1][2], acc[i][j + 1][3]), false, false);
                        store<THROUGH>(o, i, j * 16u + cc, grid_u32x4{lo[0], hi[0], lo[1], hi[1]});
                    }
                }
#pragma unroll
                for (int j = OUT16 ? BN / 2 * 2 : 0; j < BN; ++j) store4<THROUGH>(o, i, j * 16u + q4 * 4u, acc[i][j]);
            }
        }
    }

    __device__ static __forceinline__ void run(const GridArgs &g, uint32_t tile_row, uint32_t tile_col, unsigned char *smem) {
        const uint32_t m0 = tile_row * TM, n0 = tile_col * TN;
        const uint32_t tid = threadIdx.x, lane = tid & 63u, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
        const uint32_t grp = wave_all / NWG, wave = wave_all % NWG, wm = wave / GN, wn = wave % GN;
        const uint32_t n = g.K / (64u * GK);                          // k-tiles of each group
        unsigned char *const ring = smem + grp * RING;
        unsigned char *const la = ring + wave * (LA * 1024), *const lb = ring + A_BYTES + wave * (LB * 1024);
        // copy assignments, as in gemm_fast.h: wave instruction i fills 1 KB of the tile
        Copies c;
        c.ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.A), 0, (int)(g.M * g.K * 2u), 0x00020000);
        c.rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.B), 0, (int)(g.K * g.N * 2u), 0x00020000);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const uint32_t row = wave * (LA * 8) + i * 8 + lane / 8u, kc = (lane & 7u) ^ grid_swzA(row);
            c.off_a[i] = ((m0 + row) * g.K + grp * 64u + kc * 8u) * 2u - (i & 3) * 1024u;
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const uint32_t o = wave * (LB * 1024) + i * 1024 + lane * 16u, kr = o / (TN * 2), p = o % (TN * 2) / 16u;
            const uint32_t cb = n0 + (p ^ grid_swzB<TN>(kr)) * 8u;
            c.off_b[i] = ((grp * 64u + kr) * g.N + (cb < g.N ? cb : n0)) * 2u - (i & 3) * 1024u;     // (columns beyond N are never stored)
        }
        // Tiles below one another in the grid read the same columns of B, on one XCD and at the same time: whoever asks for a
        // line first waits for memory and the others wait along, so that the XCD has no more lines of B on their way than one
        // tile asks for.  Each row of tiles therefore takes a window's k-tiles in an order of its own, and fetches from memory
        // what the others then find in L2.  f16, encoder layers on 688 rows, weights from HBM: 37.4 -> 33.6 us a layer (16-bit
        // results; everything in the last-level cache 30.4 / 31.1); bf16, from HBM / in the cache 200 x 4096 x 4096 20.1 -> 17.6 /
        // 13.7 -> 13.6, 1000 x 4096 x 4096 39.5 -> 34.8 / 32.1 -> 32.5.  Windows of eight are no better and from K = 4096 on 1-4 %
        // slower, turns through the whole reduce axis lose the L2 (403 x 4096 x 4096, in the cache, 20.9 -> 33.1), and turns
        // by column, so that the readers of A part, change nothing.
        c.step_a = 128u * GK; c.step_b = g.N * (128u * GK);
        c.asked = 0; c.whole = n & ~(kGridWindow - 1u); c.turn = tile_row & (kGridWindow - 1u);
        c.after(0);
        c.advance();
        // fragment addresses (see gemm_fast.h)
        const uint32_t sbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
        const uint32_t ra = wm * WM + (lane & 15u);
        const uint32_t fa = sbase + ra * 128u + (((lane >> 4) ^ grid_swzA(ra)) << 4);
        const uint32_t j16 = lane & 15u, rb = (lane >> 4) * 8u + (j16 >> 2);
        uint32_t fb[BN];
#pragma unroll
        for (int j = 0; j < BN; ++j) {
            const uint32_t cf = wn * WN + j * 16 + (j16 & 3u) * 4u;
            fb[j] = sbase + A_BYTES + rb * (TN * 2) + (((cf >> 3) ^ grid_swzB<TN>(rb)) << 4) + (cf & 7u) * 2u;
        }
        // what the epilogue adds, asked for before the copies: it is there when they are
        constexpr int PB = NB / GK, NBIAS = GK > 1 ? PB : BN;
        const uint32_t q4 = lane >> 4, col0 = n0 + wn * WN;
        f32x4 bias[NBIAS];
#pragma unroll
        for (int p = 0; p < NBIAS; ++p) bias[p] = bias_of(g, col0 + (GK > 1 ? (grp * PB + p) % BN : (uint32_t)p) * 16u + q4 * 4u);

        auto next_tile = [&] { c.after(++c.asked); c.advance(); };
#pragma unroll
        for (int t = 0; t < S; ++t)
            if ((uint32_t)t < n) { copy<0, L>(c, la + t * STAGE, lb + t * STAGE); next_tile(); }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 sums[NS][BM][BN];                                       // (set to zero while the first copies travel)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j) sums[s][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_barrier(0);
        wait_tiles<S - 1>(n - 1u);
        if constexpr (NWG > 1) __builtin_amdgcn_s_barrier();
        Frag f0, f1;
        uint32_t slot = 0, ba[BN];                                    // the tile being consumed
#pragma unroll
        for (int j = 0; j < BN; ++j) ba[j] = fb[j];
        read_range<0, NR>(fa, ba, f0);
        // tile t from `use`, tile t + 1 into `fill` (past the last tile the reads fetch what happens to be there, for nobody)
        auto step = [&](uint32_t t, Frag &use, Frag &fill, auto steady_c, auto odd_c) {
            constexpr bool STEADY = decltype(steady_c)::value;        // tile t + S exists
            arrived(use);
            __builtin_amdgcn_sched_barrier(0);
            // tile t's LDS has been read by this wave; tile t + 1 must have landed
            if constexpr (STEADY) grid_wait_vm<(S - 2) * L>();
            else if (t + 1u < n) wait_tiles<S - 2>(n - 2u - t);
            if constexpr (NWG > 1) __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t next = slot + STAGE >= RING ? 0u : slot + STAGE;
#pragma unroll
            for (int j = 0; j < BN; ++j) ba[j] = fb[j] + next;
            if constexpr (!STEADY) {
                if (t + S < n) { copy<0, L>(c, la + slot, lb + slot); next_tile(); }
            }
            phase<STEADY, decltype(odd_c)::value>(fa + next, ba, fill, use, sums, c, la + slot, lb + slot);
            if constexpr (STEADY) c.advance();
            slot = next;
        };
        constexpr std::integral_constant<int, 0> even;
        constexpr std::integral_constant<int, 1> odd;
        uint32_t t = 0;
        for (; t + 1u + S < n; t += 2) {
            step(t, f0, f1, std::true_type{}, even);
            step(t + 1u, f1, f0, std::true_type{}, odd);
        }
        for (; t + 1u < n; t += 2) {
            step(t, f0, f1, std::false_type{}, even);
            step(t + 1u, f1, f0, std::false_type{}, odd);
        }
        if (t < n) step(t, f0, f1, std::false_type{}, even);
        arrived(f0);                                                  // nothing of the last reads outlives the loop
        arrived(f1);
        f32x4 (&acc)[BM][BN] = sums[0];
#pragma unroll
        for (int s = 1; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j) acc[i][j] += sums[s][i][j];

        if constexpr (GK > 1) {                                       // the groups' sums through LDS
            __syncthreads();
            f32x4 *const x = reinterpret_cast<f32x4 *>(smem);
#pragma unroll
            for (int b = 0; b < NB; ++b) x[((grp * NWG + wave) * NB + b) * 64u + lane] = acc[b / BN][b % BN];
            __syncthreads();
        }
        if (WHOLE && g.through) finish<WHOLE>(g, acc, bias, smem, m0 + wm * WM, col0, grp, wave, lane);
        else finish<false>(g, acc, bias, smem, m0 + wm * WM, col0, grp, wave, lane);
    }
};

// What a workgroup needs before its first copies comes first and not in a structure: the build asks for the first six arguments in
// registers (amdgpu-kernarg-preload-count), which the command processor fills before the first wave starts.  They are fourteen words, as
// many as there is room for: a longer list would leave its last ones in memory without a word.  With one structure
// read from memory and the divisions of its general form a workgroup knew its tile 0.45 us after it began; now, with everything in
// the last-level cache, 688 x 2304 x 768 6.26 -> 6.09 us, x 768 x 768 4.70 -> 4.52, x 3072 x 768 7.65 -> 7.41 (16-bit results).  The
// same arguments read from memory: 6.33, 4.79, 7.68.  (In fours: the host spends 10 ns on every argument of a launch.)
template <int DT, bool OUT16, int WM, int WN, int GM, int GN, int GK, int S>
__global__ __launch_bounds__(GM * GN * GK * 64, 2) void ft_grid(const uint16_t *A, const uint16_t *B, grid_u32x4 knm_share, grid_u32x4 band_last_per, uint32_t per_last,
                                                                uint32_t through, void *C, const float *bias) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const GridTile t = grid_tile(GridOrder{knm_share[3], band_last_per[0], band_last_per[1], band_last_per[2], band_last_per[3], per_last}, blockIdx.x);
    GridArgs g;
    g.A = A; g.B = B; g.C = C; g.bias = bias; g.K = knm_share[0]; g.N = knm_share[1]; g.M = knm_share[2]; g.through = through;
    GridBody<DT, OUT16, WM, WN, GM, GN, GK, S>::run(g, t.row, t.col, smem);
}

}  // namespace ftk

template <int DT, bool OUT16, int WM, int WN, int GM, int GN, int GK, int S>
static int launch(const ftk::GridArgs *g, void *stream) {
    constexpr auto kernel = &ftk::ft_grid<DT, OUT16, WM, WN, GM, GN, GK, S>;
    constexpr ftk::GridBodyInfo info = ftk::grid_info(WM, WN, GM, GN, GK, S);
    static_assert(info.lds <= 163840, "one CU's LDS");
    const hipError_t e = ftk::raise_lds_limit<kernel>();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(kernel, dim3(g->tiles), dim3(info.waves * 64), info.lds, static_cast<hipStream_t>(stream), g->A, g->B,
                       ftk::grid_u32x4{g->K, g->N, g->M, g->order.share}, ftk::grid_u32x4{g->order.band, g->order.last, g->order.per_band, g->order.per_rows},
                       g->order.per_last, g->through, g->C, g->bias);
    return (int)hipGetLastError();
}

template <int DT, bool OUT16>
static int launch_body(const ftk::GridArgs *g, uint32_t body, void *stream) {
    switch (body) {
#define FT_X(id, WM, WN, GM, GN, GK, S) \
    case id: return launch<DT, OUT16, WM, WN, GM, GN, GK, S>(g, stream);
        FT_GRID_BODIES(FT_X)
#undef FT_X
    default: return (int)hipErrorInvalidValue;
    }
}

extern "C" int ft_launch_grid(const ftk::GridArgs *g, uint32_t body, int dt, int out16, void *stream) {
    if (dt) return out16 ? launch_body<1, true>(g, body, stream) : launch_body<1, false>(g, body, stream);
    return out16 ? launch_body<0, true>(g, body, stream) : launch_body<0, false>(g, body, stream);
}
