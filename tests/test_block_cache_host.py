"""The cache of device blocks on the host: which device a block belongs to, which
requests it serves, how much it keeps."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2512_03452_amd", "csrc")


def test_block_cache(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "block_cache_check"
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", CSRC,
                    os.path.join(HERE, "helpers", "block_cache_check.cpp"), "-o", str(exe), "-pthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
