// Row runs: batched products with a reduce axis of one k-tile and rows of C of at most kRunMaxN elements
// (attention scores Q K^T of short and middling lengths).
//
// Such a launch is one long stream of stores: per element of C it does 128 flops and reads almost nothing.
// What bounds it is how the stores reach memory.  The tile bodies store 128-byte segments of rows; where the
// row pitch of C is no multiple of 64 bytes (an odd sequence length) neighbouring segments share blocks and
// half-written blocks travel to memory twice (measured with a store-only kernel on 768 matrices of
// 131 x 131 fp32: 17.5 us; the same bytes written in address order: 9.6 us; 511 x 511: 179 against 139 us).
// A workgroup here takes whole rows instead: the outputs of consecutive rows are ONE contiguous run of memory
// whatever the row length is.  The accumulators go through an image of that run in LDS (same byte order, same
// alignment modulo 128) and leave as aligned 16-byte stores in address order.  Plain stores, not streamed ones: in
// address order nothing is half written, and plain ones measured 5-9 % faster.
//
// Measured with timestamps (768 matrices of 300 x 300): a workgroup of 32 rows spends 3.0 us on its loads, which
// queue behind the stores of the CU's other workgroups, 1.4 us on MFMAs and image, 1.9 us on stores.  What
// overlaps them is several workgroups per CU; from about 350 columns on the tile bodies, which hold more of them,
// are faster (300 columns: 84 against 101 us, 380: 115 against 102, 131: 18.1 against 22.1, 100: 10.7 against 17.8).  Which
// launches of up to 320 columns are left to the tiles: rows_beat_tiles in host.cpp.
// Keeping B in registers over several steps of rows, or computing and storing waves of their own, left
// fewer workgroups, or fewer of them ready, and measured 5-30 % slower.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_body.h"
#include "lds_limit.h"
#include "row_runs.h"

namespace ftk {

typedef uint32_t u32x4_run __attribute__((ext_vector_type(4)));

__device__ __attribute__((aligned(256))) static uint32_t run_zero_page[64];

__device__ __forceinline__ void run_dma16(const void *gptr, unsigned char *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)gptr,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 16, 0, 0);
}

// every LDS access of this wave done, then the workgroup's barrier; global stores stay in flight
__device__ __forceinline__ void run_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The image's `bytes` bytes (from `phase` on) to cdst = the same phase of a 128-byte line: aligned 16-byte chunks, eight
// lanes to a line, then the run's two ends element by element.  Four LDS reads are in flight per lane, and the
// stores go through a descriptor that ends with the last whole chunk, so no lane branches around one of them.
// They are streamed: a run's lines are whole but for its ends, and left in the L2 they would push out the operands and be written
// back when the launch ends.  fp32, K as [L, 64], both products of an attention, kept / streamed: 768 x 131 x 131 41.5 / 34.6 us,
// 190 64.0 / 55.6, 301 150.9 / 139.8, 77 17.9 / 17.0, 96 matrices of 190 12.7 / 11.4; 16-bit results, K as [64, L], 34.8 / 30.0, 51.6 /
// 46.0, 132.9 / 127.7, 17.0 / 16.4, 12.3 / 11.8.
template <typename T>
__device__ __forceinline__ void run_copy_out(const unsigned char *img, unsigned char *cdst, uint32_t phase, uint32_t bytes, uint32_t tid) {
    constexpr uint32_t ES = sizeof(T);
    unsigned char *const gbase = cdst - phase;                         // 128-byte aligned
    const uint32_t end = phase + bytes, c0 = (phase + 15u) / 16u, c1 = end / 16u;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(gbase, 0, (int)(c1 * 16u), 0x00020000);
    for (uint32_t base = c0 & ~7u; base < c1; base += 1024u) {         // uniform
        u32x4_run v[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t c = base + i * 256u + tid;
            v[i] = *reinterpret_cast<const u32x4_run *>(img + (c < c1 ? c : c1) * 16u);
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t c = base + i * 256u + tid;
            __builtin_amdgcn_raw_buffer_store_b128(v[i], rsrc, (int)(c < c0 ? 0x80000000u : c * 16u), 0, 2);         // nt
        }
    }
    const uint32_t head_end = c0 * 16u < end ? c0 * 16u : end, tail0 = c0 < c1 ? c1 * 16u : head_end;
    const uint32_t hb = phase + tid * ES, tb = tail0 + tid * ES;
    if (hb < head_end) *reinterpret_cast<T *>(gbase + hb) = *reinterpret_cast<const T *>(img + hb);
    if (tb < end) *reinterpret_cast<T *>(gbase + tb) = *reinterpret_cast<const T *>(img + tb);
}

// One share: rows m0 .. m0 + 32 * RB - 1 of one batch entry.  Wave w owns the column blocks w, w + 4, ... of 32
// columns (at most CB of them) in all RB row blocks.
// LDS: A [32 RB rows][64 k] with the A swizzle, then B: [N][64 k] like A (BNK) or [64 k][pitch].  The image of the
// output overlays both once every wave has its accumulators.
template <int DT, bool BNK, bool OUT16, int RB, int CB>
__device__ __forceinline__ void run_body(const RunArgs &g, const uint16_t *__restrict__ Ab, const uint16_t *__restrict__ Bb, uint64_t c_off,
                                         uint32_t M, uint32_t N, uint32_t K, uint32_t m0, unsigned char *smem) {
    constexpr int OUT = OUT16 ? (DT == DT_F16 ? OUT_F16 : OUT_BF16) : OUT_F32;
    using T = typename OutElem<OUT>::type;
    constexpr uint32_t ES = sizeof(T);
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t l32 = lane & 31u, h = lane >> 5, ncb = (N + 31u) / 32u;
    const uint32_t rows = M - m0 < 32u * RB ? M - m0 : 32u * RB, nrb = (rows + 31u) / 32u;

    // ---- copies: 1 KB per wave instruction -----------------------------------------------------------
    {
        const char *ab = reinterpret_cast<const char *>(Ab);
        for (uint32_t r8 = wave; r8 < nrb * 4u; r8 += 4u) {            // 8 rows of 128 bytes each
            const uint32_t row = r8 * 8u + lane / 8u, kc = (lane & 7u) ^ swzA(row);
            const uint32_t m = m0 + row < M ? m0 + row : M - 1u;      // clamp: garbage rows are never stored
            const void *p = kc * 8u < K ? static_cast<const void *>(ab + (m * K + kc * 8u) * 2u) : static_cast<const void *>(run_zero_page);
            run_dma16(p, smem + r8 * 1024u);
        }
    }
    unsigned char *const sb = smem + RB * 4096;
    const char *bb = reinterpret_cast<const char *>(Bb);
    const uint32_t pitch = run_kn_pitch(N);                           // (B [K][N]) 16-byte chunks per LDS row
    if constexpr (BNK) {
        for (uint32_t r8 = wave; r8 < ncb * 4u; r8 += 4u) {
            const uint32_t row = r8 * 8u + lane / 8u, kc = (lane & 7u) ^ swzA(row);
            const uint32_t n = row < N ? row : N - 1u;
            const void *p = kc * 8u < K ? static_cast<const void *>(bb + (n * K + kc * 8u) * 2u) : static_cast<const void *>(run_zero_page);
            run_dma16(p, sb + r8 * 1024u);
        }
    } else {
        const uint32_t total = 64u * pitch;                           // a multiple of 64
        for (uint32_t q0 = wave * 64u; q0 < total; q0 += 256u) {
            // (q < 64 * 42.  The general division, once a copy, took 1-3 % of a launch: 768 x 131 x 131, 16-bit, 30.0 -> 29.5 us, 96
            // matrices of 300 17.8 -> 17.2)
            const uint32_t q = q0 + lane, k = small_div(q, g.per_pitch), c = q - k * pitch;
            // Columns beyond N only reach outputs that are never stored: such chunks repeat the row's first one.  A chunk
            // that straddles N reads into the next row, except in the operand's last row, where it is fetched as the
            // row's last 8 elements and moved down below.
            const uint32_t col = c * 8u < N ? c * 8u : 0u;
            const void *p = bb + (k * N + (k + 1u == K && col + 8u > N ? N - 8u : col)) * 2u;
            if (k >= K) p = run_zero_page;
            run_dma16(p, sb + q0 * 16u);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    run_barrier();
    if constexpr (!BNK) {
        if (N % 8u) {                                                  // uniform
            if (tid == 0) {
                uint4 *q = reinterpret_cast<uint4 *>(sb + ((K - 1u) * pitch + (N - 1u) / 8u) * 16u);
                *q = shift_down_elems(*q, 8u - N % 8u);
            }
            run_barrier();
        }
    }

    // ---- fragments and MFMAs --------------------------------------------------------------------------
    f32x16 acc[RB][CB];
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const uint32_t cb = wave + 4u * j;
        if (cb < ncb) {                                                // uniform
            uint4 fb[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if constexpr (BNK) {
                    const uint32_t row = cb * 32u + l32;
                    fb[ks] = *reinterpret_cast<const uint4 *>(sb + row * 128u + (((ks * 2u + h) ^ swzA(row)) << 4));
                } else {
                    const uint32_t j16 = lane & 15u, krow = ks * 16u + h * 8u + (j16 >> 2);
                    const uint32_t off = krow * pitch * 16u + (cb * 32u + ((lane >> 4) & 1u) * 16u + (j16 & 3u) * 4u) * 2u;
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(sb + off));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(sb + off + 4u * pitch * 16u));
                    const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
                    fb[ks] = make_uint4(a.x, a.y, b.x, b.y);
                }
            }
#pragma unroll
            for (int i = 0; i < RB; ++i) {
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
                if ((uint32_t)i < nrb) {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        const uint32_t row = i * 32u + l32;
                        const uint4 fa = *reinterpret_cast<const uint4 *>(smem + row * 128u + (((ks * 2u + h) ^ swzA(row)) << 4));
                        acc[i][j] = mfma32<DT>(fa, fb[ks], acc[i][j]);
                    }
                }
            }
        }
    }
    run_barrier();                                                     // A and B are done with: the image takes their place

    // ---- image, and out ---------------------------------------------------------------------------------
    unsigned char *const cdst = static_cast<unsigned char *>(g.C) + (c_off + (uint64_t)m0 * N) * ES;
    const uint32_t phase = (uint32_t)reinterpret_cast<uintptr_t>(cdst) & 127u;
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const uint32_t col = (wave + 4u * j) * 32u + l32;
        if (col < N) {
            const float bv = g.bias != nullptr ? g.bias[col] : 0.f;
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                T *const q = reinterpret_cast<T *>(smem + phase) + ((i * 32u + 4u * h) * N + col);
                if (i * 32u + 32u <= rows) {                           // uniform: the whole block of rows exists
#pragma unroll
                    for (int e = 0; e < 16; ++e) q[(8u * (e / 4) + (e % 4)) * N] = out_cvt<OUT>(acc[i][j][e] + bv);
                } else if (i * 32u < rows) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const uint32_t r = 8u * (e / 4) + (e % 4);
                        if (i * 32u + 4u * h + r < rows) q[r * N] = out_cvt<OUT>(acc[i][j][e] + bv);
                    }
                }
            }
        }
    }
    run_barrier();
    run_copy_out<T>(smem, cdst, phase, rows * N * ES, tid);
}

template <int DT, bool BNK, bool OUT16>
__global__ __launch_bounds__(256, 4) void ft_row_runs(RunArgs g) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    // workgroup b runs on XCD b % num_xcds: every XCD takes one contiguous run of shares, so that those of a batch
    // entry find its B in one L2
    const uint32_t nx = g.num_xcds, b = blockIdx.x, x = b % nx, j = b / nx, q = g.n_runs / nx, r = g.n_runs % nx;
    const uint32_t u = x * q + (x < r ? x : r) + j;
    const uint32_t be = u / g.runs, m0 = (u - be * g.runs) * (32u << g.rb_log2);
    const uint16_t *A = g.A + (uint64_t)be * g.M * g.K, *B = g.B + (uint64_t)be * g.K * g.N;
    const uint64_t c_off = (uint64_t)be * g.M * g.N;
    if (g.rb_log2 == 0) run_body<DT, BNK, OUT16, 1, 3>(g, A, B, c_off, g.M, g.N, g.K, m0, smem);
    else if (g.rb_log2 == 1) run_body<DT, BNK, OUT16, 2, 2>(g, A, B, c_off, g.M, g.N, g.K, m0, smem);
    else run_body<DT, BNK, OUT16, 4, 1>(g, A, B, c_off, g.M, g.N, g.K, m0, smem);
}

}  // namespace ftk

template <int DT, bool BNK, bool OUT16>
static int launch(const ftk::RunArgs *g, uint32_t lds_bytes, void *stream) {
    const hipError_t e = ftk::raise_lds_limit<&ftk::ft_row_runs<DT, BNK, OUT16>>();    // (up to 65 680 bytes: run_lds)
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL((ftk::ft_row_runs<DT, BNK, OUT16>), dim3(g->n_runs), dim3(256), lds_bytes, static_cast<hipStream_t>(stream), *g);
    return (int)hipGetLastError();
}

template <int DT, bool BNK>
static int launch_any(const ftk::RunArgs *g, uint32_t lds_bytes, void *stream) {
    return g->out16 ? launch<DT, BNK, true>(g, lds_bytes, stream) : launch<DT, BNK, false>(g, lds_bytes, stream);
}

extern "C" int ft_launch_runs(const ftk::RunArgs *g, int dt, int bnk, uint32_t lds_bytes, void *stream) {
    if (dt) return bnk ? launch_any<1, true>(g, lds_bytes, stream) : launch_any<1, false>(g, lds_bytes, stream);
    return bnk ? launch_any<0, true>(g, lds_bytes, stream) : launch_any<0, false>(g, lds_bytes, stream);
}
