"""The device blocks that a pool keeps (csrc/block_cache.h) on a model of a device runtime,
built by g++ from tests/host/block_check.cpp: who may be given which block, when, and what
happens when a call of the runtime fails (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kept_blocks(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = os.path.join(str(tmp_path), "block_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                        os.path.join(ROOT, "paper_2511_02749_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "block_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "all checks passed" in r.stdout
