"""The build refuses kernels that touch scratch memory, in every object that has kernels of the main path and in every
kernel of an object.  Objects made by another command are made again, and the native calls are built where that can be done
and for one interpreter."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2407_21418_amd import build

REMARK = "x.hip:1:0: remark:     ScratchSize [bytes/lane]: %d [-Rpass-analysis=kernel-resource-usage]\n"


def write(tmp_path, name, sizes):
    obj = tmp_path / name
    (tmp_path / (name + ".log")).write_text("hipcc ...\n" + "".join(REMARK % s for s in sizes))
    return str(obj)


@pytest.mark.parametrize("name", ["dispatch_dt0_c1.o", "row_runs_hip.o", "big_gemm_hip.o", "conv_patch_hip.o"])
def test_scratch_in_any_kernel_is_refused(tmp_path, name):
    assert build.check_scratch(write(tmp_path, name, [0, 0]))["ScratchSize [bytes/lane]"] == 0
    with pytest.raises(RuntimeError, match="scratch"):
        build.check_scratch(write(tmp_path, name, [16, 0]))           # not the last kernel of the object
    with pytest.raises(RuntimeError, match="no resource remarks"):
        build.check_scratch(write(tmp_path, name, []))


def test_what_may_spill(tmp_path):
    build.check_scratch(write(tmp_path, "dispatch_dt0_gen_c2.o", [32]))
    build.check_scratch(write(tmp_path, "dispatch_dt1_nk_c2.o", [8]))
    with pytest.raises(RuntimeError):
        build.check_scratch(write(tmp_path, "dispatch_dt0_nk_c2.o", [8]))
    assert build.check_scratch(write(tmp_path, "host_cpp.o", [64])) == {}


def test_objects_of_other_flags_are_stale(tmp_path):
    obj, src, log = (str(tmp_path / n) for n in ("x.o", "x.hip", "x.o.log"))
    for path in (src, obj):
        open(path, "w").close()
    cmd = ["hipcc", "-mllvm", "-amdgpu-kernarg-preload-count=6", "-c", src]
    assert build._stale(obj, [src], cmd, log)                         # (nobody knows how it was made)
    open(log, "w").write(" ".join(cmd) + "\nremarks\n")
    assert not build._stale(obj, [src], cmd, log)
    assert build._stale(obj, [src], cmd[:2] + ["-amdgpu-kernarg-preload-count=14"] + cmd[3:], log)
    os.utime(src, (2e9, 2e9))
    assert build._stale(obj, [src], cmd, log)


@pytest.fixture
def own_folder(tmp_path, monkeypatch):
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.basename(build.PYCALLS) == "_pycalls" + suffix and suffix != ".so"
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "OUT", str(tmp_path))
    monkeypatch.setattr(build, "PYCALLS", str(tmp_path / ("_pycalls" + suffix)))
    (tmp_path / "_pycalls.so").write_text("of any interpreter")
    return tmp_path


def test_native_calls_are_built_for_one_interpreter(own_folder):
    assert build.build_pycalls(verbose=False)
    assert os.path.exists(build.PYCALLS) and not (own_folder / "_pycalls.so").exists()
    t = os.path.getmtime(build.PYCALLS)
    assert build.build_pycalls(incremental=True, verbose=False) and os.path.getmtime(build.PYCALLS) == t


@pytest.mark.parametrize("lacks", ["g++", "Python.h"])
def test_the_build_goes_on_without_native_calls(own_folder, monkeypatch, capsys, lacks):
    if lacks == "g++":
        monkeypatch.setattr(build.shutil, "which", lambda name: None)
    else:
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(own_folder)})
    open(build.PYCALLS, "w").close()
    assert not build.build_pycalls()
    assert not os.path.exists(build.PYCALLS) and not (own_folder / "_pycalls.so").exists()
    assert lacks in capsys.readouterr().out


IMPORT = """
import importlib.abc, sys
class Finder(importlib.abc.MetaPathFinder):
    def find_spec(self, name, path, target=None):
        if name == "paper_2407_21418_amd._pycalls":
            raise %s
sys.meta_path.insert(0, Finder())
import paper_2407_21418_amd as ft
print(type(ft.ft_launch).__name__)
"""


@pytest.mark.parametrize("error,want", [("ModuleNotFoundError(name=name)", "function"), ("ImportError('undefined symbol', name=name)", None),
                                        ("ModuleNotFoundError(name='another')", None)])
def test_only_missing_native_calls_are_done_without(error, want):
    p = subprocess.run([sys.executable, "-c", IMPORT % error], capture_output=True, text=True, cwd=os.path.dirname(build.INC))
    assert (p.returncode == 0 and p.stdout.strip() == want) if want else (p.returncode != 0 and "Error" in p.stderr), p.stderr
