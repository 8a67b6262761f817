"""Large products executed in 256 x 256 blocks and halves of 128 rows: edges of blocks and of the strip below them, columns
that end inside a block, the shortest reduce axis taken and longer ones with every remainder of the rings, both output
types, fused bias; sampled rows against the CPU oracle (all rows next to a block edge among them)."""
import numpy as np
import pytest
import torch

import paper_2407_21418_amd as ft
import synth_inputs as si
from oracle import contraction as oc
from oracle import epilogue as oe
from gpu_util import GUARD, check_epilogue, dev_bits, run_at, stream

pytestmark = pytest.mark.gpu

# (M, N, K): each has enough blocks for the 256 CUs it is planned for
SHAPES = [(4096, 4096, 768), (3073, 4104, 832), (3200, 4088, 896), (3201, 5000, 960), (2049, 8192, 1024), (8191, 2056, 768),
          (1400, 11008, 768), (600, 11008, 2048), (130, 70000, 768)]
# of these, with fp32 results and a reduce axis too short for blocks: launched in tiles, at the edges that blocks would have
IN_TILES = [(3200, 4088, 896), (2049, 8192, 1024), (8191, 2056, 768), (1400, 11008, 768), (130, 70000, 768)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_blocks(M, N, K):
    dtype = (M + N // 8) % 2
    out16 = dtype if K % 128 else None
    bias = np.random.default_rng(N).standard_normal(N).astype(np.float32) if M % 2 else None
    g = np.random.default_rng([M, N, K])
    A = si.normal_bits(g, (M, K), 1.0, dtype)
    B = si.normal_bits(g, (K, N), 0.02, dtype)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_MATMUL, dtype=dtype, n=N, k=K, m_lo=1, m_hi=8192,
                                         out_dtype=ft.FT_OUT_F32 if out16 is None else ft.FT_OUT_SAME,
                                         epilogue=ft.FT_EPI_NONE if bias is None else ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(m=M))
    dA, dB = dev_bits(A), dev_bits(B)
    db = torch.from_numpy(bias).cuda() if bias is not None else None
    tdt = torch.float32 if out16 is None else torch.float16 if out16 == ft.FT_F16 else torch.bfloat16
    C = torch.full((M * N + 2 * GUARD,), float("nan"), dtype=tdt, device="cuda")
    C[:GUARD] = 7.0
    C[-GUARD:] = 7.0
    want = ft.FT_FORM_TILES if (M, N, K) in IN_TILES else ft.FT_FORM_BLOCKS
    assert ft.ft_plan_launch_form(plan, dA.data_ptr(), dB.data_ptr(), C.data_ptr() + GUARD * C.element_size()).form == want, "another form than the test is about"
    ft.ft_launch_epilogue(plan, dA.data_ptr(), dB.data_ptr(), C.data_ptr() + GUARD * C.element_size(), db.data_ptr() if db is not None else 0, stream())
    torch.cuda.synchronize()
    assert bool((C[:GUARD] == 7.0).all()) and bool((C[-GUARD:] == 7.0).all()), "write outside C"
    body = C[GUARD:-GUARD].view(M, N)
    assert bool(torch.isfinite(body).all()), "uncovered outputs"
    edges = {r for e in range(0, M + 1, 128) for r in (e - 1, e) if 0 <= r < M}
    rows = np.array(sorted(set(list(edges)[:40]) | {0, M - 1} | {int(x) for x in g.integers(0, M, 24)}))
    ref, refabs = oc.matmul(A, B, dtype, rows=rows, want_abs=True)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    got = body[torch.from_numpy(rows).cuda()].float().cpu().numpy().astype(np.float64)
    check_epilogue(got, ref, refabs, bias, out16, f"{M}x{N}x{K}")


# (M, N, K): rows and columns that end inside a block, the strip below the grid, halves alone, one tile column; the shortest reduce
# axis and every remainder of the two rings (five slots, three stages)
ANYWHERE = [(3073, 4104, 832), (3200, 4088, 896), (2049, 8192, 1024), (8191, 2056, 768), (1400, 11008, 960), (600, 11008, 2048), (130, 70000, 2112)]


@pytest.mark.parametrize("out", [ft.FT_OUT_F32, ft.FT_OUT_SAME], ids=["f32", "same"])
@pytest.mark.parametrize("M,N,K", ANYWHERE)
def test_blocks_anywhere_in_memory(M, N, K, out):
    """A and B at odd element offsets among NaNs, the launch is in blocks; with C off 16 bytes it is in tiles, within the same bounds.
    (fp32 results with a short reduce axis are launched in tiles: those take a longer one here.)"""
    K = K + 768 if out == ft.FT_OUT_F32 and K < 1536 else K
    dtype = (M + N // 8) % 2
    out16 = dtype if out == ft.FT_OUT_SAME else None
    g = np.random.default_rng([M, N, K, 1])
    bias = g.standard_normal(N).astype(np.float32) if M % 2 else None
    A = si.normal_bits(g, (M, K), 1.0, dtype)
    B = si.normal_bits(g, (K, N), 0.02, dtype)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_MATMUL, dtype=dtype, n=N, k=K, m_lo=1, m_hi=8192, out_dtype=out,
                                         epilogue=ft.FT_EPI_NONE if bias is None else ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(m=M))
    edges = {r for e in range(0, M + 1, 128) for r in (e - 1, e) if 0 <= r < M}
    rows = np.array(sorted(set(sorted(edges)[-24:]) | {0, 127, 128, M - 1} & set(range(M)) | {int(x) for x in g.integers(0, M, 12)}))
    ref, refabs = oc.matmul(A, B, dtype, rows=rows, want_abs=True)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    for off_c, form in ((4 if out16 is None else 8, ft.FT_FORM_BLOCKS), (2, ft.FT_FORM_TILES)):
        got = run_at(plan, A, B, M * N, dtype, form, bias, out16, off_c=off_c).reshape(M, N)
        assert np.isfinite(got).all(), "uncovered outputs"
        check_epilogue(got[rows], ref, refabs, bias, out16, f"{M}x{N}x{K} form {form}")


# fp32 results with rows on 64-byte blocks that end inside a block of 256 and a wave's 64 columns: odd rows, a strip of 1 to 127 rows below the
# grid, halves alone, the shortest reduce axis taken
@pytest.mark.parametrize("M,N,K", [(3073, 4112, 1536), (601, 11024, 2048), (3199, 4080, 1664), (129, 70000, 2112), (3329, 4368, 1600), (6001, 8208, 768)])
def test_fp32_results_past_the_caches_leave_the_same_bits(M, N, K):
    """C on a 64-byte block is streamed and written through the L2, 16 bytes behind one it is kept: the same bits, with bias, within the oracle's
    bounds, and nothing beside C."""
    dtype = (M + N // 16) % 2
    assert N % 16 == 0 and N % 64
    g = np.random.default_rng([M, N, K, 2])
    bias = g.standard_normal(N).astype(np.float32)
    A = si.normal_bits(g, (M, K), 1.0, dtype)
    B = si.normal_bits(g, (K, N), 0.02, dtype)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_MATMUL, dtype=dtype, n=N, k=K, m_lo=1, m_hi=8192, epilogue=ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(m=M))
    edges = sorted({r for e in range(0, M + 1, 128) for r in (e - 1, e) if 0 <= r < M})
    rows = np.array(sorted(set(edges[-16:]) | {0, 63, 64, 127, 128, M - 1} | {int(x) for x in g.integers(0, M, 8)}))
    ref, refabs = oc.matmul(A, B, dtype, rows=rows, want_abs=True)
    got = [run_at(plan, A, B, M * N, dtype, ft.FT_FORM_BLOCKS, bias, None, off_a=8, off_b=8, off_c=c).reshape(M, N) for c in (0, 4)]
    assert np.isfinite(got[0]).all(), "uncovered outputs"
    check_epilogue(got[0][rows], oe.add_bias(ref, bias), refabs, bias, None, f"{M}x{N}x{K}")
    assert np.array_equal(got[0], got[1])
