"""Host-side parts that need no GPU, built by g++ and run on the CPU:
- tests/host/block_check.cpp: the device blocks that a pool keeps (csrc/block_cache.h) on a
  model of a device runtime: who may be given which block, when, and what happens when a call
  of the runtime fails;
- tests/host/grid_check.cpp: launches over more row tiles than a grid takes (csrc/grid.h);
- tests/host/id_set_check.cpp: the pool's set of free page ids (csrc/id_set.h);
- tests/host/work_list_check.cpp: the planner's work lists for the kernels of any head count
  against those of the MFMA kernels."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WITH = {"work_list_check": ["planner.cpp"]}  # library sources that a check links


@pytest.mark.parametrize("name", ["block_check", "grid_check", "id_set_check", "work_list_check"])
def test_host_part(name, tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = os.path.join(str(tmp_path), name)
    csrc = os.path.join(ROOT, "paper_2511_02749_amd", "csrc")
    sources = [os.path.join(ROOT, "tests", "host", name + ".cpp")] + [os.path.join(csrc, f) for f in WITH.get(name, [])]
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-I", csrc, "-I",
                        os.path.join(ROOT, "include"), *sources, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout, end="")
    assert r.returncode == 0, r.stderr[-4000:]
    assert "all checks passed" in r.stdout
