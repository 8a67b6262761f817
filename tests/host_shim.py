"""The index functions and limits that the kernels share with the host, compiled for the CPU (g++) behind plain C calls."""
import ctypes as C
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "big_gemm.h"
#include "conv_patch.h"
#include "family.h"
#include "grid_gemm.h"
#include "ring.h"
#include "row_runs.h"
extern "C" {
uint32_t shim_ring(int n, const uint32_t *splitk, const uint32_t *planned, const uint32_t *stage_bytes, uint32_t k_tiles, uint64_t workgroups,
                   uint32_t cus, uint32_t planned_lds, uint32_t *depth) {
    ftk::RingSlot s[4];
    for (int i = 0; i < n; ++i) s[i] = ftk::RingSlot{splitk[i] != 0, planned[i], stage_bytes[i], 0u};
    const uint32_t lds = ftk::ring_plan(s, n, k_tiles, workgroups, cus, planned_lds);
    for (int i = 0; i < n; ++i) depth[i] = s[i].depth;
    return lds;
}
void shim_block(uint32_t b, uint32_t rows, uint32_t cols, uint32_t group, uint32_t n_full, uint32_t n_half, uint32_t nx, uint32_t *out) {
    const ftk::BigBlock t = ftk::big_block(b, rows, cols, group, n_full, n_half, nx);
    out[0] = t.m0; out[1] = t.n0; out[2] = t.half;
}
void shim_grid_tile(uint32_t b, uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx, uint32_t *out) {
    const ftk::GridTile t = ftk::grid_tile(b, rows, cols, group, nx);
    out[0] = t.row; out[1] = t.col;
}
uint32_t shim_grid_bodies() { return ftk::kNumGridBodies; }
void shim_grid_body(uint32_t i, uint32_t *out) {
    const ftk::GridBodyInfo &b = ftk::kGridBodies[i];
    out[0] = b.tm; out[1] = b.tn; out[2] = b.gk; out[3] = b.waves; out[4] = b.lds;
}
uint32_t shim_run_lds(uint32_t n, uint32_t rb_log2, uint32_t es, int bnk) { return ftk::run_lds(n, rb_log2, es, bnk != 0); }
uint32_t shim_run_rb_log2(uint32_t m, uint32_t n, uint64_t batch, uint32_t es, int bnk, uint32_t cus) {
    return ftk::run_rb_log2(m, n, batch, es, bnk != 0, cus);
}
uint32_t shim_run_pitch(uint32_t n) { return ftk::run_kn_pitch(n); }
uint32_t shim_small_div(uint32_t x, uint32_t d) { return ftk::small_div(x, ftk::small_per(d)); }
uint32_t shim_grid_reads(uint32_t rows, uint32_t cols, uint32_t group, uint32_t nx, uint32_t tm, uint32_t tn) {
    return ftk::grid_reads(rows, cols, group, nx, tm, tn);
}
uint32_t shim_grid_band(uint32_t rows, uint32_t cols, uint32_t nx, uint32_t tm, uint32_t tn) { return ftk::grid_band(rows, cols, nx, tm, tn); }
uint32_t shim_grid_div(uint32_t x, uint32_t d) { return ftk::grid_div(x, ftk::grid_per(d)); }
uint32_t shim_patch_bytes(uint32_t th, uint32_t tw) { return ftk::conv_patch_bytes(ftk::conv_patch_rows(th, tw)); }
}
"""


@functools.lru_cache(None)
def load():
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2407_21418_amd", "csrc"), src, "-o", so], check=True)
        lib = C.CDLL(so)
    u32, u64, p = C.c_uint32, C.c_uint64, C.POINTER(C.c_uint32)
    lib.shim_ring.argtypes, lib.shim_ring.restype = [C.c_int, p, p, p, u32, u64, u32, u32, p], u32
    lib.shim_block.argtypes, lib.shim_block.restype = [u32] * 7 + [p], None
    lib.shim_grid_tile.argtypes, lib.shim_grid_tile.restype = [u32] * 5 + [p], None
    lib.shim_grid_bodies.argtypes, lib.shim_grid_bodies.restype = [], u32
    lib.shim_grid_body.argtypes, lib.shim_grid_body.restype = [u32, p], None
    for name, args in (("run_lds", [u32, u32, u32, C.c_int]), ("run_rb_log2", [u32, u32, u64, u32, C.c_int, u32]), ("run_pitch", [u32]), ("patch_bytes", [u32, u32]),
                       ("small_div", [u32, u32]), ("grid_div", [u32, u32]), ("grid_reads", [u32] * 6), ("grid_band", [u32] * 5)):
        fn = getattr(lib, "shim_" + name)
        fn.argtypes, fn.restype = args, u32
    return lib


def ring_plan(slots, k_tiles, workgroups, cus, planned_lds):
    """slots: (splitk, planned stages, stage bytes) of each body; returns (LDS bytes of the launch, depth of each)."""
    n = len(slots)
    col = lambda i: (C.c_uint32 * n)(*(int(s[i]) for s in slots))
    depth = (C.c_uint32 * n)()
    lds = load().shim_ring(n, col(0), col(1), col(2), k_tiles, workgroups, cus, planned_lds, depth)
    return lds, list(depth)


def block(b, rows, cols, group, n_full, n_half, nx):
    out = (C.c_uint32 * 3)()
    load().shim_block(b, rows, cols, group, n_full, n_half, nx, out)
    return tuple(out)


def grid_tile(b, rows, cols, group, nx):
    out = (C.c_uint32 * 2)()
    load().shim_grid_tile(b, rows, cols, group, nx, out)
    return tuple(out)


def grid_bodies():
    """(tm, tn, groups along the reduce axis, waves, LDS bytes) of every body."""
    out = (C.c_uint32 * 5)()
    bodies = []
    for i in range(load().shim_grid_bodies()):
        load().shim_grid_body(i, out)
        bodies.append(tuple(out))
    return bodies
