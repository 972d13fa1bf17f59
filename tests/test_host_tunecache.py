"""The kernels' id in the autotuner's saved file, on the CPU."""
from paper_2608_06466_amd import build
from test_host_logic import _build_and_run


def test_tuning_file_of_other_kernels_does_not_apply(tmp_path):
    assert "tunecache kernels ok" in _build_and_run("tunecache_kernels_test.cpp", tmp_path)


def test_kernels_id_follows_the_sources_and_flags(monkeypatch, tmp_path):
    """The id changes with a kernel source and with a scheduling flag, not with host code or the
    tree's place."""
    import os
    import shutil
    first = build.kernels_id()
    copy = tmp_path / "csrc"
    shutil.copytree(build.CSRC, copy)
    monkeypatch.setattr(build, "CSRC", str(copy))
    assert build.kernels_id() == first
    with open(copy / "zb_host.hip", "a") as f:
        f.write("// host\n")
    assert build.kernels_id() == first
    with open(copy / "zb_burn_kernel.h", "a") as f:
        f.write("// kernel\n")
    assert build.kernels_id() != first
    shutil.copy(os.path.join(os.path.dirname(build.OBJ), "csrc", "zb_burn_kernel.h"), copy)
    assert build.kernels_id() == first
    monkeypatch.setitem(build.SCHED, "zb_k14.hip", "max-ilp")
    assert build.kernels_id() != first
