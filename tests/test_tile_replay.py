"""Addresses of the batched kernel's products, from the source that ships (CPU only).

tests/host_tile_replay.cpp compiles the kernel's own header for the host (with
tests/host_shim in place of the HIP runtime header) and runs the row and column
products, X^T Y, the updates and the applies lane by lane under the address and
alignment sanitizers, on buffers of exactly the sizes they have in the kernel:
the tile with rows as tight as they come, the shared test matrix, the regions of
the scratch slot and of the LDS arena, the outputs.  Shapes as in the parity and
benchmark sets and at the edges of the panels; every basis width the rank loop
reaches and ranks at the edges of the 16-column tiles and of the two closings.
Mistakes planted in a copy of the header have to be reported.
"""
import os
import re
import shutil
import subprocess

import pytest

import workloads as W

TESTS = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(TESTS), "paper_2506_22713_amd", "csrc")
RANKS = [1, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 100, 127, 128]
EDGES = [(64, 64), (65, 63), (129, 127), (130, 260), (260, 132), (257, 255), (255, 258), (320, 321), (1024, 200),
         (201, 1023), (350, 301), (33, 17), (17, 33), (16, 16), (15, 20), (1, 1), (1, 7), (7, 1), (63, 1024), (3, 1000)]


def _clang():
    for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")):
        if c and os.path.exists(c):
            return c
    pytest.skip("needs clang++")


def _compile(out, csrc=CSRC):
    # without optimisation: no load is dropped
    res = subprocess.run([_clang(), "-std=c++17", "-O0", "-w", "-fsanitize=address,alignment", "-fno-sanitize-recover=all",
                          "-I", os.path.join(TESTS, "host_shim"), "-I", str(csrc),
                          os.path.join(TESTS, "host_tile_replay.cpp"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    return out


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return _compile(str(tmp_path_factory.mktemp("tiles") / "replay"))


def _run(exe, tiles):
    args = []
    for h, w, b, unaligned, ranks in tiles:
        args += [str(x) for x in (h, w, b, int(unaligned), *ranks)] + ["/"]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    return subprocess.run([exe] + args, capture_output=True, text=True, timeout=300, env=env)


def _check(exe, tiles):
    run = _run(exe, tiles)
    assert run.returncode == 0, run.stderr[-3000:]
    assert run.stdout == f"{len(tiles)} tiles\n"


@pytest.mark.parametrize("b", [1, 16, 31, 40, 64])
@pytest.mark.parametrize("unaligned", [False, True], ids=["aligned", "unaligned"])
def test_edge_shapes(exe, b, unaligned):
    _check(exe, [(h, w, b, unaligned, RANKS if h * w < 40000 else RANKS[::4]) for h, w in EDGES
                 if b > 1 or min(h, w) <= 20])


@pytest.mark.parametrize("b", [16, 32, 64])
def test_parity_and_benchmark_shapes(exe, b):
    shapes = W.tile_shapes(5, count=22, lo=64, hi=1024, rank_lo=5, rank_hi=80)[::4] + W.tile_shapes(0, count=1024)[b::200]
    _check(exe, [(h, w, b, i % 3 == 0, [rho, 128]) for i, (h, w, rho) in enumerate(shapes)])


PLANTED = [
    ("a column ring without its prologue clamp", r"load\(q\[p\], a\[p\], min\(p, nfull - 1\)\)", "load(q[p], a[p], p)"),
    ("a row ring without its prologue clamp", r"loadf\(q, min\(\(int64_t\)q, nfull - 1\)\)", "loadf(q, q)"),
    ("columns past the tile", r"co\[u\] = min\(cl \+ u, n - 1\)", "co[u] = cl + u"),
    ("rows past the tile", r"lda4\(min\(kr \+ v, m - 1\)\)", "lda4(kr + v)"),
    ("an output's last rows", r"if \(row \+ v < m\) zc\[row \+ v\]", "zc[row + v]"),
    ("a fold round too large", r"S = TX \* TY <= 4 \? 4", "S = TX * TY <= 16 ? 4"),
]


@pytest.mark.parametrize("what,pattern,wrong", PLANTED, ids=[p[0] for p in PLANTED])
def test_planted_mistakes_are_reported(tmp_path, what, pattern, wrong):
    csrc = tmp_path / "csrc"
    csrc.mkdir()
    for name in ("eodabe_kernels.hpp", "eodabe_tiles.hpp"):
        src = open(os.path.join(CSRC, name)).read()
        if name == "eodabe_tiles.hpp":
            src, n = re.subn(pattern, wrong.replace("\\", "\\\\"), src)
            assert n >= 1, what
        (csrc / name).write_text(src)
    exe = _compile(str(tmp_path / "planted"), csrc)
    run = _run(exe, [(20, 18, 16, True, [1, 16]), (18, 20, 16, False, [16]), (130, 130, 64, False, [64]),
                     (1023, 70, 64, True, [64]), (1024, 68, 64, False, [64])])
    assert run.returncode != 0 and "AddressSanitizer" in run.stderr, what


def test_short_buffers_are_reported(exe):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    run = subprocess.run([exe, "plant", "200", "130", "32", "0", "1"], capture_output=True, text=True, env=env)
    assert run.returncode != 0 and "AddressSanitizer" in run.stderr
