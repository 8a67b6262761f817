"""Batched products of one k-tile executed in whole rows of C (odd row lengths, enough rows for every CU):
edges of the 32-row and 32-column blocks, the limits of the row length, short reduce axes, both layouts of B, both
output types, fused bias; against the CPU oracle.  Every launch here has at least 256 workgroups' worth of rows
(the batch sees to it), which is what sends it down this path."""
import numpy as np
import pytest

import paper_2407_21418_amd as ft
import synth_inputs as si
from oracle import contraction as oc
from oracle import epilogue as oe
from gpu_util import check_epilogue, run_at, run_epilogue

pytestmark = pytest.mark.gpu

#       M,   N,  K, batch
SHAPES = [(1, 9, 64, 260), (31, 33, 64, 256), (33, 31, 8, 256), (64, 65, 64, 257), (65, 127, 56, 256), (129, 129, 64, 256),
          (100, 100, 64, 1100), (33, 191, 64, 256), (70, 257, 24, 256), (40, 319, 64, 256), (131, 8, 64, 256)]


@pytest.mark.parametrize("layout", [ft.FT_B_KN, ft.FT_B_NK], ids=["kn", "nk"])
@pytest.mark.parametrize("M,N,K,batch", SHAPES)
def test_whole_rows(M, N, K, batch, layout):
    dtype = (M + N) % 2
    out16 = None if (N + K) % 3 else dtype
    g = np.random.default_rng([M, N, K, layout])
    A = si.normal_bits(g, (batch, M, K), 1.0, dtype)
    B = si.normal_bits(g, (batch, K, N) if layout == ft.FT_B_KN else (batch, N, K), 0.2, dtype)
    bias = g.standard_normal(N).astype(np.float32) if M % 2 else None
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_BMM, dtype=dtype, k=K, m_lo=0, m_hi=512, n_lo=0, n_hi=512, batch_hi=1200, b_layout=layout,
                                         out_dtype=ft.FT_OUT_F32 if out16 is None else ft.FT_OUT_SAME,
                                         epilogue=ft.FT_EPI_NONE if bias is None else ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(batch=batch, m=M, n=N))
    ref, refabs = (oc.bmm if layout == ft.FT_B_KN else oc.bmm_nk)(A, B, dtype, want_abs=True)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    got = run_epilogue(plan, A, B, batch * M * N, bias, out16)
    check_epilogue(got, ref, refabs, bias, out16, f"{batch}x{M}x{N}x{K}")


@pytest.mark.parametrize("M,layout", [(65, ft.FT_B_NK), (128, ft.FT_B_KN), (200, ft.FT_B_NK)])
def test_the_largest_image(M, layout):
    """128 columns of fp32 off a 64-byte block in shares of 128 rows: the image of the outputs, 65 680 bytes, is the most
    LDS a share asks for, and more than a kernel gets without asking for it beforehand."""
    N, K, batch = 128, 64, 1030
    g = np.random.default_rng([M, layout])
    A = si.normal_bits(g, (batch, M, K), 1.0, ft.FT_F16)
    B = si.normal_bits(g, (batch, K, N) if layout == ft.FT_B_KN else (batch, N, K), 0.2, ft.FT_F16)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_BMM, k=K, m_lo=0, m_hi=512, n_lo=0, n_hi=512, batch_hi=1200, b_layout=layout))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(batch=batch, m=M, n=N))
    assert ft.ft_plan_launch_form(plan, 0, 0, 16).lds_bytes == 65680
    got = run_at(plan, A, B, batch * M * N, ft.FT_F16, ft.FT_FORM_ROWS, off_c=4)
    ref, refabs = (oc.bmm if layout == ft.FT_B_KN else oc.bmm_nk)(A, B, ft.FT_F16, want_abs=True)
    check_epilogue(got, ref, refabs, None, None, f"{batch}x{M}x{N}x{K}")


# (M, N, K, batch): every share height (32, 64 and 128 rows), one to ten column blocks, short reduce axes
ANYWHERE = [(1, 9, 64, 600), (33, 33, 64, 768), (64, 65, 8, 700), (65, 127, 56, 800), (129, 100, 64, 520), (100, 131, 64, 768), (33, 191, 64, 700),
            (70, 257, 24, 300), (40, 319, 64, 700), (31, 8, 16, 512)]


@pytest.mark.parametrize("layout", [ft.FT_B_KN, ft.FT_B_NK], ids=["kn", "nk"])
@pytest.mark.parametrize("M,N,K,batch", ANYWHERE)
def test_whole_rows_anywhere_in_memory(M, N, K, batch, layout):
    """Operands at odd element offsets among NaNs, C off every alignment but its element's; the launch is in whole rows."""
    dtype = (M + N + layout) % 2
    out16 = None if (N + K + layout) % 3 else dtype
    g = np.random.default_rng([M, N, K, layout, 1])
    A = si.normal_bits(g, (batch, M, K), 1.0, dtype)
    B = si.normal_bits(g, (batch, K, N) if layout == ft.FT_B_KN else (batch, N, K), 0.2, dtype)
    bias = g.standard_normal(N).astype(np.float32) if M % 2 else None
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_BMM, dtype=dtype, k=K, m_lo=0, m_hi=512, n_lo=0, n_hi=512, batch_hi=1200, b_layout=layout,
                                         out_dtype=ft.FT_OUT_F32 if out16 is None else ft.FT_OUT_SAME,
                                         epilogue=ft.FT_EPI_NONE if bias is None else ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(batch=batch, m=M, n=N))
    ref, refabs = (oc.bmm if layout == ft.FT_B_KN else oc.bmm_nk)(A, B, dtype, want_abs=True)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    got = run_at(plan, A, B, batch * M * N, dtype, ft.FT_FORM_ROWS, bias, out16, off_c=1 + M % 7)
    check_epilogue(got, ref, refabs, bias, out16, f"{batch}x{M}x{N}x{K}")
