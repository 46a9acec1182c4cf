"""Compiles a C++ file of this folder against the library's host code, without
its kernels (CPU only)."""
import os
import subprocess

import pytest

TESTS = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(TESTS)


def run_host(source, tmp_path):
    """Build tests/<source> and run it: the finished process."""
    from paper_2506_22713_amd import build
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    exe = str(tmp_path / "host")
    cmd = [cc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-w",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2506_22713_amd", "csrc"),
           os.path.join(TESTS, source), "-Wl,--unresolved-symbols=ignore-all", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(run.stdout)
    return run
