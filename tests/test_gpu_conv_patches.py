"""3 x 3 convolutions over 64 channels, executed from image patches in LDS: images smaller than a tile and many tiles per
workgroup, tiles that overhang on either side, one-pixel and one-row images, padding 0 to 3, output channels that end inside a
block of 64, both output types, fused bias; every pixel (large images: sampled ones) against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2407_21418_amd as ft
import synth_inputs as si
from oracle import contraction as oc
from oracle import epilogue as oe
from gpu_util import GUARD, check_epilogue, dev_bits, run_at, stream

pytestmark = pytest.mark.gpu

# (images, height, width, output channels, padding)
SHAPES = [(1, 1, 1, 8, 1), (1, 3, 3, 64, 0), (3, 1, 40, 72, 1), (2, 67, 2, 136, 1), (2, 9, 31, 264, 2), (1, 16, 16, 64, 1),
          (5, 17, 33, 128, 0), (1, 64, 300, 192, 3), (8, 75, 75, 128, 1), (3, 131, 257, 200, 1), (2, 40, 40, 8200, 1)]


@pytest.mark.parametrize("n,h,w,co,pad", SHAPES)
def test_patches(n, h, w, co, pad):
    dtype = (h + co // 8) % 2
    out16 = dtype if w % 2 == 0 else None
    g = np.random.default_rng([n, h, w, co])
    bias = g.standard_normal(co).astype(np.float32) if n % 2 else None
    X = si.normal_bits(g, (n, h, w, 64), 1.0, dtype)
    Wt = si.normal_bits(g, (3, 3, 64, co), 0.04, dtype)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_CONV2D, dtype=dtype, c_in=64, c_out=co, r=3, s=3, stride=1, pad=pad, m_lo=1, m_hi=1 << 22,
                                         out_dtype=ft.FT_OUT_F32 if out16 is None else ft.FT_OUT_SAME,
                                         epilogue=ft.FT_EPI_NONE if bias is None else ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(img_n=n, img_h=h, img_w=w))
    M = n * (h + 2 * pad - 2) * (w + 2 * pad - 2)
    dX, dW = dev_bits(X), dev_bits(Wt)
    db = torch.from_numpy(bias).cuda() if bias is not None else None
    tdt = torch.float32 if out16 is None else torch.float16 if out16 == ft.FT_F16 else torch.bfloat16
    Y = torch.full((M * co + 2 * GUARD,), float("nan"), dtype=tdt, device="cuda")
    Y[:GUARD] = 7.0
    Y[-GUARD:] = 7.0
    ft.ft_launch_epilogue(plan, dX.data_ptr(), dW.data_ptr(), Y.data_ptr() + GUARD * Y.element_size(), db.data_ptr() if db is not None else 0, stream())
    torch.cuda.synchronize()
    assert bool((Y[:GUARD] == 7.0).all()) and bool((Y[-GUARD:] == 7.0).all()), "write outside Y"
    body = Y[GUARD:-GUARD].view(M, co)
    assert bool(torch.isfinite(body).all()), "uncovered outputs"
    pix = np.arange(M) if M * co < 1 << 20 else np.array(sorted({0, M - 1} | {int(x) for x in g.integers(0, M, 400 if co < 1024 else 40)}))
    ref, refabs = oc.conv2d_nhwc(X, Wt, dtype, pad=pad, pixels=pix, want_abs=True)
    ref, refabs = ref.reshape(len(pix), co), refabs.reshape(len(pix), co)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    got = body[torch.from_numpy(pix).cuda()].float().cpu().numpy().astype(np.float64)
    check_epilogue(got, ref, refabs, bias, out16, f"{n}x{h}x{w} -> {co}, padding {pad}")


# (images, height, width, output channels, padding): one tile and several per workgroup, each tile height (1 to 4 blocks of 16
# pixels per wave), channels that end inside a block
ANYWHERE = [(1, 5, 3, 8, 1), (5, 17, 33, 128, 0), (2, 40, 40, 72, 1), (8, 50, 50, 128, 1), (8, 92, 92, 128, 1), (1, 64, 300, 200, 3), (3, 131, 57, 16, 2)]


@pytest.mark.parametrize("out", [ft.FT_OUT_F32, ft.FT_OUT_SAME], ids=["f32", "same"])
@pytest.mark.parametrize("n,h,w,co,pad", ANYWHERE)
def test_patches_anywhere_in_memory(n, h, w, co, pad, out):
    """Image and filter at odd element offsets among NaNs (the gather's bodies want 16 bytes), the launch is in patches; with an
    output off 16 bytes it is in tiles, with the same results."""
    dtype = (h + n) % 2
    out16 = dtype if out == ft.FT_OUT_SAME else None
    g = np.random.default_rng([n, h, w, co, pad])
    bias = g.standard_normal(co).astype(np.float32) if h % 2 else None
    X = si.normal_bits(g, (n, h, w, 64), 1.0, dtype)
    Wt = si.normal_bits(g, (3, 3, 64, co), 0.04, dtype)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_CONV2D, dtype=dtype, c_in=64, c_out=co, r=3, s=3, stride=1, pad=pad, m_lo=1, m_hi=1 << 22,
                                         out_dtype=out, epilogue=ft.FT_EPI_NONE if bias is None else ft.FT_EPI_BIAS))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(img_n=n, img_h=h, img_w=w))
    M = n * (h + 2 * pad - 2) * (w + 2 * pad - 2)
    pix = np.arange(M) if M * co < 1 << 19 else np.array(sorted({0, M - 1} | {int(x) for x in g.integers(0, M, 400)}))
    ref, refabs = oc.conv2d_nhwc(X, Wt, dtype, pad=pad, pixels=pix, want_abs=True)
    ref, refabs = ref.reshape(len(pix), co), refabs.reshape(len(pix), co)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    per16 = 4 if out16 is None else 8                                  # elements of 16 bytes
    for off_c, form in ((per16, ft.FT_FORM_PATCHES), (1, ft.FT_FORM_TILES)):
        got = run_at(plan, X, Wt, M * co, dtype, form, bias, out16, off_c=off_c).reshape(M, co)
        assert np.isfinite(got).all(), "uncovered outputs"
        check_epilogue(got[pix], ref, refabs, bias, out16, f"{n}x{h}x{w} -> {co}, padding {pad}, form {form}")


@pytest.mark.parametrize("n,size,co,out", [(8, 41, 128, ft.FT_OUT_F32), (8, 41, 32, ft.FT_OUT_SAME), (8, 145, 128, ft.FT_OUT_F32), (8, 183, 128, ft.FT_OUT_SAME)])
def test_stores_past_the_caches_leave_the_same_bits(n, size, co, out):
    """Pixels on 64-byte blocks are written through the L2, up to 64 MB of them, and streamed beyond; 16 bytes behind a block
    they are kept.  Sampled pixels against the oracle, all of them against each other."""
    dtype = ft.FT_F16
    g = np.random.default_rng([n, size, co])
    X = si.normal_bits(g, (n, size, size, 64), 1.0, dtype)
    Wt = si.normal_bits(g, (3, 3, 64, co), 0.04, dtype)
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_CONV2D, dtype=dtype, c_in=64, c_out=co, r=3, s=3, stride=1, pad=1, m_lo=1, m_hi=1 << 22, out_dtype=out))
    plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op), ft.ft_shape(img_n=n, img_h=size, img_w=size))
    M, per16 = n * size * size, 4 if out == ft.FT_OUT_F32 else 8
    assert (M * co * 16 // per16 > 64 << 20) == (size > 100) and co * 16 // per16 % 64 == 0, "another side of the line than the test is about"
    dX, dW = dev_bits(X), dev_bits(Wt)
    got = []
    for off in (0, per16):
        Y = torch.full((M * co + 2 * GUARD,), 7.0, dtype=torch.float32 if out == ft.FT_OUT_F32 else torch.float16, device="cuda")
        body = Y[GUARD + off:GUARD + off + M * co]
        body.fill_(float("nan"))
        assert body.data_ptr() % 64 == (16 if off else 0) and ft.ft_plan_launch_form(plan, dX.data_ptr(), dW.data_ptr(), body.data_ptr()).form == ft.FT_FORM_PATCHES
        ft.ft_launch(plan, dX.data_ptr(), dW.data_ptr(), body.data_ptr(), stream())
        torch.cuda.synchronize()
        assert bool((Y[:GUARD + off] == 7.0).all()) and bool((Y[GUARD + off + M * co:] == 7.0).all()), "write outside Y"
        got.append(body.view(M, co))
    assert torch.equal(got[0], got[1])
    pix = np.array(sorted({0, M - 1} | {int(x) for x in g.integers(0, M, 100)}))
    ref, refabs = oc.conv2d_nhwc(X, Wt, dtype, pad=1, pixels=pix, want_abs=True)
    check_epilogue(got[0][torch.from_numpy(pix).cuda()].double().cpu().numpy(), ref.reshape(len(pix), co), refabs.reshape(len(pix), co), None,
                   None if out == ft.FT_OUT_F32 else dtype, f"{n}x{size}x{size} -> {co}")
