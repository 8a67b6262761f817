"""Matmuls executed in one grid of equal tiles: every body at rows and columns that end inside a tile, the shortest reduce axis
taken, even and odd numbers of k-tiles around the rings' depth, both types, with and without bias; against the CPU oracle.
The index functions that kernel and host share are walked on the CPU."""
import random

import numpy as np
import pytest
import torch

import host_shim
import paper_2407_21418_amd as ft
import synth_inputs as si
from oracle import contraction as oc
from oracle import epilogue as oe

S16, F32 = ft.FT_OUT_SAME, ft.FT_OUT_F32
# (M, N, K, tm, tn, groups along the reduce axis, result type): every body with both result types, one tile row short of full among them
CASES = [(17, 1096, 1024, 32, 32, 4, S16), (17, 1456, 1536, 32, 32, 4, S16), (33, 2144, 768, 32, 32, 4, F32),
         (66, 2952, 768, 16, 64, 4, S16), (74, 2808, 1536, 16, 64, 4, S16), (97, 2112, 1024, 16, 64, 4, F32),
         (17, 584, 896, 32, 64, 2, S16), (81, 3328, 768, 32, 64, 2, S16), (65, 2232, 896, 32, 64, 2, F32),
         (351, 1792, 1536, 48, 64, 2, S16), (449, 1224, 2048, 48, 64, 2, S16), (689, 816, 896, 48, 64, 2, F32),
         (17, 3432, 832, 64, 64, 1, S16), (129, 3304, 768, 64, 64, 1, S16), (127, 3496, 1088, 64, 64, 1, F32),
         (577, 1736, 896, 96, 64, 1, S16), (479, 2960, 1088, 96, 64, 1, S16), (497, 2456, 832, 96, 64, 1, F32),
         (655, 2680, 1024, 128, 64, 1, S16), (2065, 736, 2176, 128, 64, 1, S16), (2704, 528, 1920, 128, 64, 1, F32),
         (577, 3912, 896, 96, 128, 1, S16), (767, 2744, 1024, 96, 128, 1, S16), (1343, 2152, 1280, 96, 128, 1, F32),
         (783, 3832, 1024, 128, 128, 1, S16), (1553, 2128, 1088, 128, 128, 1, S16), (2192, 1760, 1920, 128, 128, 1, F32),
         (1425, 2712, 768, 128, 192, 1, S16), (2177, 1880, 1088, 128, 192, 1, S16), (1537, 2688, 1920, 128, 192, 1, F32),
         (2832, 2488, 1536, 128, 256, 1, S16), (1809, 3808, 2048, 128, 256, 1, S16), (2576, 2848, 1536, 128, 256, 1, F32),
         (655, 2792, 896, 64, 128, 1, S16), (1023, 1632, 1088, 64, 128, 1, S16), (1153, 1616, 768, 64, 128, 1, F32)]


def plan_of(M, N, K, dtype=ft.FT_F16, bias=False, flags=0, out=ft.FT_OUT_SAME):
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_MATMUL, dtype=dtype, n=N, k=K, m_lo=1, m_hi=8192, out_dtype=out,
                                         epilogue=ft.FT_EPI_BIAS if bias else ft.FT_EPI_NONE))
    uks = ft.ft_ukernels_derive(op)
    return op, uks, ft.ft_plan_create(op, uks, ft.ft_shape(m=M), flags)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [ft.FT_F16, ft.FT_BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("M,N,K,tm,tn,gk,out", CASES)
def test_every_body(M, N, K, tm, tn, gk, out, dtype):
    from gpu_util import check_epilogue, run_at
    g = np.random.default_rng([M, N, K, dtype])
    bias = g.standard_normal(N).astype(np.float32) if (M + dtype) % 2 else None
    _, _, plan = plan_of(M, N, K, dtype, bias is not None, out=out)
    out16 = dtype if out == S16 else None
    f = ft.ft_plan_launch_form(plan)
    body = [b for b in host_shim.grid_bodies() if b[:3] == (tm, tn, gk)]
    assert f.form == ft.FT_FORM_GRID and body and (f.workgroups, f.lds_bytes) == (-(-M // tm) * -(-N // tn), body[0][4]), "another body than the test is about"
    A = si.normal_bits(g, (M, K), 1.0, dtype)
    B = si.normal_bits(g, (K, N), 0.02, dtype)
    rows = np.array(sorted({0, M - 1} | {r for e in range(0, M, tm) for r in (e - 1, e, e + 15, e + 16) if 0 <= r < M and (e < 3 * tm or e > M - 2 * tm)}))
    ref, refabs = oc.matmul(A, B, dtype, rows=rows, want_abs=True)
    if bias is not None:
        ref = oe.add_bias(ref, bias)
    # (A and B on 16 bytes among NaNs: nothing beyond an operand may reach a result)
    got = run_at(plan, A, B, M * N, dtype, ft.FT_FORM_GRID, bias, out16, off_a=8, off_b=24, off_c=8).reshape(M, N)
    assert np.isfinite(got).all(), "uncovered outputs"
    check_epilogue(got[rows], ref, refabs, bias, out16, f"{M}x{N}x{K}")
    again = run_at(plan, A, B, M * N, dtype, ft.FT_FORM_GRID, bias, out16, off_a=8, off_b=24, off_c=8).reshape(M, N)
    assert np.array_equal(got, again)
    # off 16 bytes the same plan launches its tiles, within the same bounds
    other = run_at(plan, A, B, M * N, dtype, ft.FT_FORM_TILES, bias, out16, off_a=3, off_b=8, off_c=1).reshape(M, N)
    check_epilogue(other[rows], ref, refabs, bias, out16, f"{M}x{N}x{K} tiles")


# with 16-bit results: every group's ring many times round, on reduce axes a program has (32 to 64 k-tiles), and one to sixteen rows
LONG = [(95, 1136, 2048, 32, 32, 4), (33, 4688, 3072, 16, 64, 4), (65, 3392, 2048, 32, 64, 2), (257, 2032, 2560, 48, 64, 2),
        (671, 1592, 2304, 96, 64, 1), (513, 2952, 3072, 128, 64, 1), (863, 2552, 2048, 96, 128, 1), (1793, 2104, 3328, 128, 128, 1),
        (1, 11008, 4096, 16, 64, 4), (7, 11008, 4096, 16, 64, 4), (16, 11008, 4096, 16, 64, 4), (1, 512, 2048, 32, 32, 4),
        (5, 1280, 2048, 32, 32, 4), (688, 768, 3072, 48, 64, 2), (403, 4096, 4096, 128, 64, 1), (750, 11008, 4096, 128, 192, 1),
        (2328, 4096, 4096, 128, 192, 1), (1949, 3896, 3520, 128, 256, 1), (511, 2040, 3712, 64, 64, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [ft.FT_F16, ft.FT_BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("M,N,K,tm,tn,gk", LONG)
def test_long_reduce_axes_and_few_rows(M, N, K, tm, tn, gk, dtype):
    test_every_body(M, N, K, tm, tn, gk, S16, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,tm,tn,out", [(103, 2304, 768, 16, 64, F32), (17, 4096, 768, 32, 32, F32), (183, 3088, 768, 48, 64, F32), (690, 768, 768, 48, 64, F32), (1195, 784, 768, 64, 64, F32),
                                             (660, 3072, 768, 96, 128, F32), (1141, 3072, 768, 128, 128, F32), (1329, 3072, 768, 128, 192, F32),
                                             (441, 2304, 768, 64, 64, S16), (689, 2336, 768, 128, 64, S16), (927, 2304, 768, 96, 128, S16), (1279, 3072, 768, 128, 128, S16),
                                             (1558, 3072, 768, 128, 192, S16), (689, 768, 3072, 48, 64, S16)])
def test_rows_of_c_on_64_byte_blocks(M, N, K, tm, tn, out):
    """C on a 64-byte block with rows of whole blocks (fp32 is stored past the caches there) and 16 bytes behind
    one: the same bits, and nothing beside C."""
    from gpu_util import check_epilogue, run_at
    dtype = M % 2
    g = np.random.default_rng([M, N, K, 3])
    bias = g.standard_normal(N).astype(np.float32)
    _, _, plan = plan_of(M, N, K, dtype, True, out=out)
    out16 = dtype if out == S16 else None
    assert N * (2 if out == S16 else 4) % 64 == 0 and ft.ft_plan_launch_form(plan).workgroups == -(-M // tm) * -(-N // tn), "another body than the test is about"
    A = si.normal_bits(g, (M, K), 1.0, dtype)
    B = si.normal_bits(g, (K, N), 0.02, dtype)
    rows = np.array(sorted({0, M - 1} | {r for e in range(0, M, tm) for r in (e - 1, e) if 0 <= r < M and (e < 3 * tm or e > M - 2 * tm)}))
    ref, refabs = oc.matmul(A, B, dtype, rows=rows, want_abs=True)
    got = [run_at(plan, A, B, M * N, dtype, ft.FT_FORM_GRID, bias, out16, off_a=8, off_b=24, off_c=c).reshape(M, N) for c in (0, 4 if out == F32 else 8)]
    assert np.isfinite(got[0]).all(), "uncovered outputs"
    check_epilogue(got[0][rows], oe.add_bias(ref, bias), refabs, bias, out16, f"{M}x{N}x{K}")
    assert np.array_equal(got[0], got[1])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [ft.FT_F16, ft.FT_BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("M,N,K", [(1009, 2304, 768), (1850, 768, 768), (1524, 2304, 768), (282, 3072, 768), (688, 768, 768), (1194, 768, 768), (440, 2304, 768),
                                   (105, 3072, 768), (143, 2304, 768), (326, 1496, 1344)])
def test_fp32_results_are_no_further_from_exact_than_the_tiles(M, N, K, dtype):
    """Programs whose tiles share the reduce axis between two teams or four waves: an output in the grid is added up in as many sums.
    Of M N = 2e5 and more independent errors the root of the mean square is known to 0.2 %; half a fiftieth is the rule's own."""
    from gpu_util import run_at
    _, _, plan = plan_of(M, N, K, dtype, out=F32)
    _, _, tiles = plan_of(M, N, K, dtype, out=F32, flags=ft.FT_PLAN_TABLE_ORDER)
    g = np.random.default_rng([M, N, K, dtype, 2])
    A = si.normal_bits(g, (M, K), 1.0, dtype)
    B = si.normal_bits(g, (K, N), 0.02, dtype)
    ref = oc.matmul(A, B, dtype)
    off = [np.linalg.norm(run_at(p, A, B, M * N, dtype, f, off_a=8, off_b=8).reshape(M, N) - ref) for p, f in ((plan, ft.FT_FORM_GRID), (tiles, ft.FT_FORM_TILES))]
    assert off[0] <= 1.012 * off[1], f"{off[0] / off[1]:.3f} times as far from the exact product as the tiles"


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [ft.FT_F16, ft.FT_BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("M,N,K", [(500, 768, 3072), (1100, 768, 3072), (250, 1032, 2048), (700, 1024, 2112), (98, 2048, 4096), (177, 3000, 2048)])
def test_fp32_results_with_a_long_reduce_axis(M, N, K, dtype):
    """From 32 k-tiles on, programs that do not split them over workgroups are launched in the grid: split-k tiles, two teams and
    single grids, every output within the bounds of the tiles and the whole no further from exact than theirs."""
    from gpu_util import check_epilogue, run_at
    test_fp32_results_are_no_further_from_exact_than_the_tiles(M, N, K, dtype)
    g = np.random.default_rng([M, N, K, dtype, 4])
    bias = g.standard_normal(N).astype(np.float32)
    _, _, plan = plan_of(M, N, K, dtype, True, out=F32)
    A, B = si.normal_bits(g, (M, K), 1.0, dtype), si.normal_bits(g, (K, N), 0.02, dtype)
    rows = np.array(sorted({0, 15, 16, M // 2, M - 1}))
    ref, refabs = oc.matmul(A, B, dtype, rows=rows, want_abs=True)
    for off_c in (0, 4):
        got = run_at(plan, A, B, M * N, dtype, ft.FT_FORM_GRID, bias, None, off_a=8, off_b=24, off_c=off_c).reshape(M, N)
        assert np.isfinite(got).all(), "uncovered outputs"
        check_epilogue(got[rows], oe.add_bias(ref, bias), refabs, bias, None, f"{M}x{N}x{K}")


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,tm,out", [(201, 768, 3072, 32, S16), (688, 768, 3072, 48, S16), (688, 3072, 768, 96, S16), (700, 4096, 4096, 96, S16), (272, 768, 3072, 32, F32),
                                          (1009, 2304, 768, 96, F32)])
def test_what_of_the_last_bits_depends_on(M, N, K, tm, out):
    """Equal rows of A: launches on other streams, addresses and buffers repeat the bits of every place; within a row of tiles all rows are
    equal; between rows of tiles, which add up the k-tiles in orders of their own, each sum of K terms is within K ulp of sum |a||b| of
    the exact one (2^-24 a rounding; half an ulp of the result more where it is rounded to 16 bits)."""
    from gpu_util import run_at
    dtype = M % 2
    g = np.random.default_rng([M, N, K, 5])
    _, _, plan = plan_of(M, N, K, dtype, out=out)
    out16 = dtype if out == S16 else None
    f = ft.ft_plan_launch_form(plan)
    assert f.form == ft.FT_FORM_GRID and f.workgroups % -(-M // tm) == 0, "another body than the test is about"
    row = si.normal_bits(g, (1, K), 1.0, dtype)
    A, B = np.repeat(row, M, 0), si.normal_bits(g, (K, N), 0.02, dtype)
    got = run_at(plan, A, B, M * N, dtype, ft.FT_FORM_GRID, None, out16, off_a=8, off_b=8, off_c=8).reshape(M, N)
    with torch.cuda.stream(torch.cuda.Stream()):
        again = run_at(plan, A, B, M * N, dtype, ft.FT_FORM_GRID, None, out16, off_a=24, off_b=64, off_c=32 if out == S16 else 16).reshape(M, N)
    assert np.array_equal(got, again)
    for r in range(0, M, tm):
        assert (got[r:r + tm] == got[r]).all(), f"rows {r} to {r + tm}"
    ref, refabs = oc.matmul(row, B, dtype, want_abs=True)
    bound = refabs * K * 2.0 ** -24
    if out16 is not None:
        bound = bound + (np.abs(ref) + bound) * (2.0 ** -11 if dtype == ft.FT_F16 else 2.0 ** -8) + 2.0 ** -25
    assert (np.abs(got - ref) <= bound).all()


@pytest.mark.gpu
def test_grid_launches_in_a_graph():
    """Captured launches on rotating operands, replayed with eager launches in between, give the eager bits."""
    from gpu_util import dev_bits, stream
    M, N, K = 329, 3784, 832
    g = np.random.default_rng(9)
    _, _, plan = plan_of(M, N, K)
    A = [dev_bits(si.normal_bits(g, (M, K), 1.0, ft.FT_F16)) for _ in range(2)]
    B = [dev_bits(si.normal_bits(g, (K, N), 0.02, ft.FT_F16)) for _ in range(2)]
    want = []
    for a, b in zip(A, B):
        c = torch.empty((M, N), dtype=torch.float16, device="cuda")
        ft.ft_launch(plan, a.data_ptr(), b.data_ptr(), c.data_ptr(), stream())
        want.append(c)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(3):
        C = [torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        ft.ft_launch_timed(plan, [t.data_ptr() for t in A], [t.data_ptr() for t in B], [t.data_ptr() for t in C], side.cuda_stream, 5, graph=True)
        torch.cuda.synchronize()
        for c, w in zip(C, want):
            assert bool((c.view(torch.int16) == w.view(torch.int16)).all())
        ft.ft_launch(plan, A[0].data_ptr(), B[0].data_ptr(), C[0].data_ptr(), stream())
        torch.cuda.synchronize()
        assert bool((C[0].view(torch.int16) == want[0].view(torch.int16)).all())


@pytest.mark.parametrize("nx", [8, 1, 3])
def test_every_tile_has_one_workgroup(nx):
    rng = random.Random(nx)
    for _ in range(200):
        rows, cols = rng.randint(1, 40), rng.randint(1, 60)
        group = rng.randint(1, rows)
        tiles = [host_shim.grid_tile(b, rows, cols, group, nx) for b in range(rows * cols)]
        assert sorted(tiles) == [(r, c) for r in range(rows) for c in range(cols)], (rows, cols, group, nx)


def test_bodies_fit_a_cu():
    for tm, tn, gk, waves, lds in host_shim.grid_bodies():
        assert lds <= 163840 and waves in (4, 8) and gk * tm * tn * 4 * (gk > 1) <= lds


def test_where_the_grid_is_taken():
    def form(M, N, K, a=1 << 20, b=1 << 20, c=1 << 20, **kw):
        plan = plan_of(M, N, K, flags=ft.FT_PLAN_HOST_ONLY | kw.pop("flags", 0), **kw)[2]
        return ft.ft_plan_launch_form(plan, a, b, c).form
    grid, tiles, blocks = ft.FT_FORM_GRID, ft.FT_FORM_TILES, ft.FT_FORM_BLOCKS
    assert form(688, 2304, 768) == form(688, 768, 3072) == form(403, 4096, 4096) == form(77, 3072, 768) == grid
    assert form(8, 768, 768) == form(48, 768, 3072) == form(16, 4096, 4096) == form(1600, 5120, 2048) == tiles
    assert form(1232, 4096, 4096) == form(403, 11008, 4096) == grid and form(2600, 4096, 4096) == form(2600, 5120, 2048) == blocks
    # what the copies and stores do not take: short, ragged or unaligned operands; plans that name their tiles
    assert form(688, 2304, 704) == form(688, 2304, 776) == form(688, 2300, 768) == form(688, 504, 768) == tiles
    for kw in (dict(a=8), dict(b=8), dict(c=8)):
        kw = {k: (1 << 20) + v for k, v in kw.items()}
        assert form(688, 2304, 768, **kw) == tiles
    assert form(403, 11008, 4096, a=(1 << 20) + 2) == blocks
    assert form(688, 2304, 768, flags=ft.FT_PLAN_TABLE_ORDER) == form(688, 2304, 768, flags=ft.FT_PLAN_PAD_BASELINE) == tiles
    # fp32 results: few tiles, larger tiles beside a program of more workgroups than CUs, and long reduce axes stay where they were
    assert form(688, 768, 768, out=F32) == form(429, 3072, 768, out=F32) == form(131, 3072, 768, out=F32) == form(800, 4096, 1984, out=F32) == grid
    assert form(64, 768, 768, out=F32) == form(688, 3072, 768, out=F32) == form(429, 3072, 2048, out=F32) == tiles


def test_launches_that_tiles_serve_faster_stay_tiles():
    """Both sides of the lines that were set with operands from HBM too (grid_schedule has the times)."""
    def form(M, N, K, out=S16):
        return ft.ft_plan_launch_form(plan_of(M, N, K, flags=ft.FT_PLAN_HOST_ONLY, out=out)[2]).form
    grid, tiles = ft.FT_FORM_GRID, ft.FT_FORM_TILES
    # split-k tiles held at once: few groups that read twice as much; four groups on a reduce axis split again over workgroups
    assert form(14, 4824, 1984) == form(3, 3816, 1728) == form(1, 3752, 1920) == form(5, 5720, 1920, F32) == tiles
    assert form(61, 3272, 1472) == form(14, 10496, 1984) == form(434, 768, 3072) == form(1, 864, 1536) == form(1009, 632, 2880) == grid
    assert form(62, 4096, 4096) == form(264, 664, 6144) == tiles and form(58, 2656, 2560) == form(125, 4096, 4096) == grid
    # two tiles per CU that read more than the program's; large tiles on few CUs
    assert form(648, 11008, 4096) == tiles and form(750, 11008, 4096) == grid
    assert form(1370, 3072, 768) == form(1800, 2304, 768) == tiles and form(1432, 3072, 768) == form(1425, 2712, 768) == grid
