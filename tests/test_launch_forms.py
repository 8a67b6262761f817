"""Which form a launch takes, as ft_plan_launch_form reports it (the launch itself asks the same function): every form is
reached by the shapes it is meant for, falls back to the tiles where an operand's alignment does not allow it, is never
taken by plans that name their tiles, and reports what it computes."""
import glob
import os

import pytest

import host_shim
import paper_2407_21418_amd as ft

CSRC = os.path.join(os.path.dirname(ft.__file__), "csrc")

C0 = 1 << 20                              # an address on every alignment asked for


def plan_of(shape, flags=ft.FT_PLAN_PATCHWORK, **desc):
    op = ft.ft_op_register(ft.ft_op_desc(**desc))
    uks = ft.ft_ukernels_derive(op)
    return op, uks, ft.ft_plan_create(op, uks, shape, flags | ft.FT_PLAN_HOST_ONLY)


def matmul(m, n, k, flags=0, **kw):
    return plan_of(ft.ft_shape(m=m), flags, kind=ft.FT_OP_MATMUL, n=n, k=k, m_lo=1, m_hi=8192, **kw)


def scores(b, m, n, k=64, flags=0, **kw):
    return plan_of(ft.ft_shape(batch=b, m=m, n=n), flags, kind=ft.FT_OP_BMM, k=k, m_lo=0, m_hi=512, n_lo=0, n_hi=512, batch_hi=1200, **kw)


def conv(n, h, w, co, flags=0, ci=64, pad=1, stride=1, **kw):
    return plan_of(ft.ft_shape(img_n=n, img_h=h, img_w=w), flags, kind=ft.FT_OP_CONV2D, c_in=ci, c_out=co, r=3, s=3, stride=stride, pad=pad,
                   m_lo=1, m_hi=1 << 22, **kw)


def form(p, a=C0, b=C0, c=C0):
    return ft.ft_plan_launch_form(p[2], a, b, c)


@pytest.mark.parametrize("make,want", [
    (lambda f: matmul(4096, 4096, 4096, f), ft.FT_FORM_BLOCKS),
    (lambda f: scores(768, 131, 131, flags=f), ft.FT_FORM_ROWS),
    (lambda f: conv(8, 224, 224, 128, f), ft.FT_FORM_PATCHES),
], ids=["blocks", "rows", "patches"])
def test_a_form_is_taken_by_planned_plans_only(make, want):
    assert form(make(0)).form == want
    assert form(make(ft.FT_PLAN_PAD_BASELINE)).form == ft.FT_FORM_TILES
    assert form(make(ft.FT_PLAN_TABLE_ORDER)).form == ft.FT_FORM_TILES
    op, uks, plan = make(0)
    st = ft.ft_plan_stats_get(plan)
    forced = ft.ft_forced_program(k1=st.ukernel_id[0], count1=st.count_tau[0], k2=st.ukernel_id[1], count2=st.count_tau[1] if st.n_ukernels > 1 else 0)
    d = op.desc
    shape = ft.ft_shape(batch=st.batch, m=0 if d.kind == ft.FT_OP_CONV2D else st.m, n=st.n if d.kind == ft.FT_OP_BMM else 0)
    if d.kind == ft.FT_OP_CONV2D:
        shape = ft.ft_shape(img_n=8, img_h=224, img_w=224)
    same = ft.ft_plan_create(op, uks, shape, ft.FT_PLAN_FORCED | ft.FT_PLAN_HOST_ONLY, forced)
    assert form((op, uks, same)).form == ft.FT_FORM_TILES
    # operands at 2-byte alignment are taken, at an odd address they are not
    assert form(make(0), C0 + 2, C0 + 6).form == want
    assert form(make(0), C0 + 1).form == ft.FT_FORM_TILES
    assert form(make(0), b=C0 + 3).form == ft.FT_FORM_TILES


def test_alignment_of_c():
    for p in (matmul(4096, 4096, 4096), conv(8, 224, 224, 128)):
        assert form(p, c=C0 + 16).form != ft.FT_FORM_TILES
        assert form(p, c=C0 + 8).form == ft.FT_FORM_TILES
        assert form(p, c=C0 + 4).form == ft.FT_FORM_TILES
    # whole rows take any C; rows on 64-byte blocks are left to the tiles as long as C is on one
    assert form(scores(768, 131, 131), c=C0 + 4).form == ft.FT_FORM_ROWS
    assert form(scores(768, 160, 160)).form == ft.FT_FORM_TILES
    assert form(scores(768, 160, 160), c=C0 + 4).form == ft.FT_FORM_ROWS


def test_what_a_form_computes():
    """Padding is counted on what runs, not on the program that does not."""
    p = matmul(3073, 4104, 832, out_dtype=ft.FT_OUT_SAME)
    f, st = form(p), ft.ft_plan_stats_get(p[2])
    assert f.form == ft.FT_FORM_BLOCKS and st.useful_elems == 3073 * 4104
    # 12 x 17 blocks of 256 x 256 and the strip of 17 halves for the row below them, whatever the blocks of the last round become
    assert f.computed_elems == 12 * 17 * 65536 + 17 * 32768 and f.workgroups >= 12 * 17 + 17 and f.lds_bytes == 163840
    assert f.computed_elems > 1.09 * st.useful_elems > 1.09 * st.covered_elems * 0.99
    f = form(scores(768, 131, 131))
    assert f.form == ft.FT_FORM_ROWS and f.computed_elems == 768 * 160 * 160 and f.workgroups == 768 * 3
    f = form(conv(8, 224, 224, 128))
    st = ft.ft_plan_stats_get(conv(8, 224, 224, 128)[2])
    assert f.form == ft.FT_FORM_PATCHES and f.workgroups == 256 and st.useful_elems <= f.computed_elems < 1.2 * st.useful_elems
    assert 9 * 8192 < f.lds_bytes <= 163840
    p = matmul(77, 768, 768)
    f, st = form(p), ft.ft_plan_stats_get(p[2])
    assert f.form == ft.FT_FORM_TILES and f.computed_elems == st.covered_elems and f.workgroups == st.n_tiles * st.k_parts and f.lds_bytes == st.lds_bytes


def test_empty_grouped_and_bad_arguments():
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_BMM, k=64, m_lo=0, m_hi=512, n_lo=0, n_hi=512, batch_hi=768))
    uks = ft.ft_ukernels_derive(op)
    empty = ft.ft_plan_create(op, uks, ft.ft_shape(batch=0, m=5, n=5), ft.FT_PLAN_HOST_ONLY)
    f = ft.ft_plan_launch_form(empty)
    assert (f.form, f.workgroups, f.computed_elems) == (ft.FT_FORM_TILES, 0, 0)
    g = ft.ft_plan_create_grouped(op, uks, [ft.ft_shape(batch=384, m=131, n=131), ft.ft_shape(batch=12, m=33, n=33)], ft.FT_PLAN_HOST_ONLY)
    f, st = ft.ft_plan_launch_form(g, C0, C0, C0), ft.ft_plan_stats_get(g)
    assert f.form == ft.FT_FORM_TILES and f.workgroups == st.n_tiles and f.computed_elems == st.covered_elems
    out = ft.ft_launch_form()
    out.struct_size = 4
    assert ft.lib().ft_plan_launch_form(empty.ptr, None, None, None, out) == ft.FT_ERR_INVALID_ARG
    assert ft.lib().ft_plan_launch_form(None, None, None, None, ft.ft_launch_form()) == ft.FT_ERR_INVALID_ARG


def test_every_form_has_a_name_where_it_is_printed():
    import run_shape
    forms = {v for k, v in vars(ft).items() if k.startswith("FT_FORM_")}
    assert len({run_shape.form_name(ft, f) for f in forms}) == len(forms) >= 5 and form(matmul(272, 768, 768)).form in forms
    assert run_shape.form_name(ft, max(forms) + 1)


def test_the_benchmark_reports_what_a_launch_runs():
    """Kernel and computed outputs are the launch form's, not those of the program that is not run."""
    import bench
    op, uks, plan = matmul(528, 3072, 768)
    st = ft.ft_plan_stats_get(plan)
    tiles, kernel, computed = bench.launch_of(ft, uks, plan, C0, C0, C0 + 4)
    assert (tiles, kernel, computed) == (ft.FT_FORM_TILES, "ft_dispatch_dt0_%sc%d" % ("pp_" if ft.ft_ukset_get(uks, st.ukernel_id[0]).gk == 2 else "", st.kernel_class), st.covered_elems)
    grid, kernel, computed = bench.launch_of(ft, uks, plan, C0, C0, C0)
    assert (grid, kernel, computed) == (ft.FT_FORM_GRID, "ft_grid", form((op, uks, plan)).computed_elems) and computed > st.covered_elems


def test_launchers_raise_the_limit_before_they_ask_for_lds():
    """Whole rows of 128 fp32 columns off a 64-byte block ask for more than the 64 KB a kernel gets by itself; so do blocks,
    patches and the tiles.  Every file that launches with dynamic LDS raises the limit."""
    p = scores(1030, 128, 128)
    assert form(p, c=C0 + 16).lds_bytes > 65536
    asking = [f for f in glob.glob(os.path.join(CSRC, "*.hip")) if "extern __shared__" in open(f).read()]
    assert len(asking) >= 4
    for f in asking:
        text = open(f).read()
        assert "raise_lds_limit<" in text or "hipFuncAttributeMaxDynamicSharedMemorySize" in text, f


def test_whole_rows_are_taken_where_they_measured_faster():
    rows, tiles = ft.FT_FORM_ROWS, ft.FT_FORM_TILES
    for b, m, n, layout, out, want in [
            (768, 131, 131, ft.FT_B_NK, ft.FT_OUT_F32, rows), (768, 300, 300, ft.FT_B_KN, ft.FT_OUT_F32, rows), (96, 100, 100, ft.FT_B_NK, ft.FT_OUT_F32, rows),
            (12, 300, 300, ft.FT_B_NK, ft.FT_OUT_F32, tiles),          # fewer workgroups than CUs
            (96, 131, 131, ft.FT_B_NK, ft.FT_OUT_F32, tiles), (48, 190, 190, ft.FT_B_NK, ft.FT_OUT_F32, tiles), (384, 1, 131, ft.FT_B_NK, ft.FT_OUT_F32, tiles),
            (192, 128, 190, ft.FT_B_NK, ft.FT_OUT_F32, rows), (768, 1, 131, ft.FT_B_NK, ft.FT_OUT_F32, rows),
            (768, 512, 300, ft.FT_B_NK, ft.FT_OUT_F32, tiles), (768, 512, 300, ft.FT_B_NK, ft.FT_OUT_SAME, rows),
            (768, 319, 319, ft.FT_B_KN, ft.FT_OUT_F32, tiles), (768, 319, 319, ft.FT_B_NK, ft.FT_OUT_F32, rows)]:
        p = scores(b, m, n, b_layout=layout, out_dtype=out)
        assert form(p).form == want, (b, m, n, layout, out, ft.ft_plan_stats_get(p[2]).n_tiles)


def test_height_and_lds_of_a_share():
    lib = host_shim.load()
    for n in list(range(8, 193)) + list(range(257, 321)):
        for es in (2, 4):
            for bnk in (0, 1):
                for rb in range(3):
                    lds = lib.shim_run_lds(n, rb, es, bnk)
                    blocks = (n + 31) // 32
                    a, b = 32 * 128 << rb, blocks * 32 * 128 if bnk else 64 * 16 * lib.shim_run_pitch(n)
                    image = 127 + (32 << rb) * n * es          # furthest byte of the run's image, from any phase of a 128-byte line,
                    assert lds >= a + b and lds >= (image + 15) // 16 * 16 + 16 and lds % 16 == 0    # and the chunk behind it that is read along
                    assert lib.shim_run_pitch(n) * 8 >= blocks * 32
                for m in (1, 31, 33, 65, 129, 300, 512):
                    for batch in (1, 100, 256, 768, 5000):
                        rb = lib.shim_run_rb_log2(m, n, batch, es, bnk, 256)
                        assert rb <= (2 if n <= 128 else 1 if n <= 256 else 0)      # four accumulator blocks per wave
                        if rb:
                            assert batch * -(-m // (32 << rb)) >= 3 * 256
    # (rows, columns, matrices) -> height: three shares per CU that are all held at once; not if a second round has few
    assert lib.shim_run_rb_log2(33, 33, 768, 4, 1, 256) == 1 and lib.shim_run_rb_log2(33, 33, 384, 4, 1, 256) == 0
    assert lib.shim_run_rb_log2(190, 190, 288, 4, 1, 256) == 0 and lib.shim_run_rb_log2(190, 190, 288, 2, 1, 256) == 1


def test_patches_are_taken_where_they_measured_faster():
    patches, tiles = ft.FT_FORM_PATCHES, ft.FT_FORM_TILES
    for n, size, co, out, want in [
            (8, 28, 128, ft.FT_OUT_F32, patches), (8, 56, 128, ft.FT_OUT_F32, patches), (8, 224, 128, ft.FT_OUT_F32, patches), (1, 7, 8, ft.FT_OUT_F32, patches),
            (8, 80, 128, ft.FT_OUT_F32, tiles), (8, 80, 128, ft.FT_OUT_SAME, patches), (8, 92, 128, ft.FT_OUT_F32, patches),
            (8, 56, 256, ft.FT_OUT_F32, tiles), (1, 28, 8200, ft.FT_OUT_F32, patches),
            (256, 3, 256, ft.FT_OUT_F32, tiles), (1000, 5, 384, ft.FT_OUT_SAME, tiles), (1000, 2, 512, ft.FT_OUT_F32, tiles), (64, 14, 64, ft.FT_OUT_F32, patches),
            (8, 112, 16, ft.FT_OUT_F32, patches)]:
        p = conv(n, size, size, co, out_dtype=out)
        assert form(p).form == want, (n, size, co, out)
    assert form(conv(8, 56, 56, 128, ci=128)).form == tiles and form(conv(8, 56, 56, 128, stride=2)).form == tiles
    assert form(conv(8, 56, 56, 132)).form == tiles


def test_blocks_are_taken_where_they_measured_faster():
    blocks, tiles = ft.FT_FORM_BLOCKS, ft.FT_FORM_TILES
    for m, n, k, out, want in [
            (8192, 11008, 4096, ft.FT_OUT_SAME, blocks), (4096, 4096, 4096, ft.FT_OUT_F32, blocks), (403, 11008, 4096, ft.FT_OUT_F32, blocks),
            (403, 4096, 4096, ft.FT_OUT_F32, tiles), (2048, 3072, 768, ft.FT_OUT_F32, tiles), (2048, 3072, 2048, ft.FT_OUT_F32, blocks),
            (5000, 4096, 768, ft.FT_OUT_F32, tiles), (5000, 4096, 768, ft.FT_OUT_SAME, blocks), (6000, 8192, 768, ft.FT_OUT_F32, blocks),
            (8192, 8192, 1024, ft.FT_OUT_F32, tiles), (8192, 8192, 1024, ft.FT_OUT_SAME, blocks), (8192, 8192, 1536, ft.FT_OUT_F32, blocks),
            (4096, 4096, 768, ft.FT_OUT_F32, blocks), (4096, 4096, 704, ft.FT_OUT_SAME, tiles), (4096, 4096, 4104, ft.FT_OUT_SAME, tiles)]:
        p = matmul(m, n, k, out_dtype=out)
        assert form(p).form == want, (m, n, k, out)
    assert form(matmul(4096, 4096, 4096, b_layout=ft.FT_B_NK)).form == tiles and form(matmul(4096, 4092, 4096)).form == tiles


@pytest.mark.parametrize("cus,xcds", [(256, 8), (80, 8), (256, 1), (7, 3)])
def test_blocks_cover_c_once(cus, xcds):
    """Every element of C lies in exactly one block, half or strip of the launch the plan describes, for whatever device it is
    planned."""
    import numpy as np
    hw = ft.ft_hw_default_gfx950()
    hw.num_cus, hw.num_xcds = cus, xcds
    taken = 0
    for m, n, k in [(4096, 4096, 1024), (3073, 4104, 832), (3200, 4088, 896), (2049, 8192, 1024), (600, 11008, 2048), (130, 8200, 2048), (8191, 2056, 1536),
                    (4000, 3000, 768), (1, 8, 768), (257, 264, 2048)]:
        op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_MATMUL, n=n, k=k, m_lo=1, m_hi=8192, out_dtype=ft.FT_OUT_SAME))
        plan = ft.ft_plan_create(op, ft.ft_ukernels_derive(op, hw), ft.ft_shape(m=m), ft.FT_PLAN_HOST_ONLY)
        f = ft.ft_plan_launch_form(plan)
        if f.form != ft.FT_FORM_BLOCKS:
            continue
        taken += 1
        rows, cols = m // 256 + (m % 256 > 128), -(-n // 256)
        half = 2 * f.workgroups - f.computed_elems // (128 * 256)           # full * 2 + half = computed, full + half = workgroups
        full = f.workgroups - half
        seen = np.zeros((-(-m // 128), cols), int)
        for b in range(f.workgroups):
            m0, n0, is_half = host_shim.block(b, rows, cols, 4, full, half, xcds)
            assert m0 % 128 == 0 and n0 % 256 == 0 and is_half == (b >= full)
            seen[m0 // 128, n0 // 256] += 1
            if not is_half and m0 // 128 + 1 < seen.shape[0]:
                seen[m0 // 128 + 1, n0 // 256] += 1
        assert (seen == 1).all(), (m, n, k)
    assert taken >= 3


def test_patch_tiles_fit_and_cover():
    """Whatever the image, a patch launch fits a CU's LDS, has at most a workgroup per CU and computes every output."""
    import random
    rng = random.Random(5)
    taken = 0
    for _ in range(300):
        size = lambda hi: int(round(2 ** rng.uniform(0, hi)))
        n, h, w, co, pad = size(6), size(8), size(10), 8 * size(6), rng.randint(0, 4)
        if n * (h + 2 * pad) * (w + 2 * pad) * co >= 1 << 29 or h + 2 * pad < 3 or w + 2 * pad < 3:
            continue
        p = conv(n, h, w, co, pad=pad)
        f, st = form(p), ft.ft_plan_stats_get(p[2])
        if f.form == ft.FT_FORM_PATCHES:
            taken += 1
            assert 9 * 8192 + 1024 <= f.lds_bytes <= 163840 and f.workgroups <= 256 and f.computed_elems >= st.useful_elems, (n, h, w, co, pad)
    assert taken > 100
