"""The rule that drops the second CholeskyQR pass of FP32 data (CPU only).

What a first pass leaves is the Gram's rounding seen through R^-1: a sum of K
products carries about sqrt(K) u64 of its columns' norms, so an entry of
V^T V - I at most sqrt(K) u64 s, s = |D R^-1|_F^2.  Whatever the rule in the
kernel header lets pass has to stay well below what rounding V to FP32 leaves
there, at few columns as at many; and real first passes are held to the bound.
"""
import os
import re

import numpy as np
import pytest

HDR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_22713_amd", "csrc",
                   "eodabe_kernels.hpp")
U32, U64 = 2.0 ** -24, 2.0 ** -53


def _rule():
    """(s, f) -> bool, read from the return statement that compares with powers of two."""
    src = open(HDR).read()
    expr = re.search(r"return ([^;]*0x1p-27[^;]*);", src).group(1)
    expr = re.sub(r"0x1p(-?\d+)", r"2.0 ** \1", expr).replace("&&", "and")
    return lambda s, f: eval(expr, {"U64": U64, "s": s, "f": f})


@pytest.mark.parametrize("f", [1, 2, 3, 5, 16, 64, 128, 300, 1500, 4096])
def test_what_passes_is_below_the_rounding(f):
    rule = _rule()
    s = f * 2.0 ** np.arange(0, 40, 0.25)                 # s >= f: D R^-1 has unit columns' inverse
    passed = [x for x in s if rule(x, f)]
    if passed:
        assert U64 * max(passed) <= U32 / 1000 and f * U64 * max(passed) <= U32 / 8
    assert f > 256 or passed, "well-conditioned blocks take one pass"
    assert not rule(float("nan"), f) and not rule(float("inf"), f)


@pytest.mark.parametrize("f,angle", [(2, 1e-2), (2, 1e-4), (5, 1e-3), (16, 1e-3), (40, 1e-2), (100, 1e-1)])
def test_first_passes_within_the_bound(f, angle):
    rng = np.random.default_rng(f)
    X = rng.standard_normal((600, 1)) + angle * rng.standard_normal((600, f))     # columns at small angles
    X = (X * 10.0 ** -rng.uniform(0, 3, f)).astype(np.float32).astype(np.float64)
    G = X.T @ X
    R = np.linalg.cholesky(G).T
    Ri = np.linalg.inv(R)
    s = float(np.sum((np.sqrt(np.diag(G))[:, None] * Ri) ** 2))
    V = X @ Ri
    assert np.abs(V.T @ V - np.eye(f)).max() <= np.sqrt(X.shape[0]) * U64 * s
