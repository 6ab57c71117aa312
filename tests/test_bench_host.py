"""bench.py's host-side contract that needs no GPU: more than one GPU is refused
with a message before anything is imported or measured, and the hash that ties
profiled traffic to a kernel build covers every source the kernels are made of."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_exits_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout == ""


@pytest.mark.parametrize("name,counts", [("gemm_bf16.hip", True), ("kernels.h", True), ("common.h", True),
                                         ("gemm_small.h", True), ("lds_load.h", True),
                                         ("api.cpp", False), ("plans.h", False)])
def test_source_hash_covers_what_the_kernels_include(name, counts, tmp_path, monkeypatch):
    sys.path.insert(0, ROOT)
    import bench
    before = bench.kernel_source_hash()
    csrc = tmp_path / "paper_2609_10018_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_2609_10018_amd", "csrc"), csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_source_hash() == before
    with open(csrc / name, "a") as f:
        f.write("// changed\n")
    assert (bench.kernel_source_hash() != before) == counts
