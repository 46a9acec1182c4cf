"""The partial sums of every Gram fit the buffer they are given (CPU only).

tests/host_gram_room.cpp is the library's host code compiled without its
kernels: each launch of a block's or a closing QR's Gram is recorded instead of
made, over block widths 1..128, real and complex, both data types and heights
up to 2^20, and the last double written is compared with the end of the buffer
that the workspace carve holds for it.  Blocks of 65 to 128 columns write up to
63 partials of their full square and the sum behind them, which from about a
thousand rows on is more than the partials of the narrower blocks take.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_gram_partials_fit_their_buffers(tmp_path):
    from paper_2506_22713_amd import build
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    exe = str(tmp_path / "gram_room")
    cmd = [cc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-w",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2506_22713_amd", "csrc"),
           os.path.join(ROOT, "tests", "host_gram_room.cpp"), "-Wl,--unresolved-symbols=ignore-all", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(run.stdout)
    assert run.returncode == 0, run.stdout[-2000:]
    assert " 0 overrun" in run.stdout
