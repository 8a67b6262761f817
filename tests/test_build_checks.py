"""The build refuses kernels that touch scratch memory, in every object that has kernels of the main path and in every
kernel of an object."""
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
