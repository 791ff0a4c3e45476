"""The block table of mma_kv_fetch_noalloc on its way to the launch, on the CPU (tests/cpp/noalloc_table.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_noalloc_table(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "noalloc_table")
    src = [os.path.join(ROOT, "tests", "cpp", "noalloc_table.cpp"),
           os.path.join(ROOT, "paper_2512_16056_amd", "csrc", "mma_plan.cpp")]
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-Wall", f"-I{os.path.join(ROOT, 'paper_2512_16056_amd', 'csrc')}",
                        *src, "-o", exe, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout + r.stderr
