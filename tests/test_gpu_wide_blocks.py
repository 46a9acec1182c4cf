"""GPU parity of basis blocks of 65 to 128 columns on tall matrices.

From about a thousand rows on their Gram is the sum of many full partials, the
largest buffer of the basis loop; several blocks each, so that a write past it
would reach the factors of the stop test and the stored basis.  Bars as in the
oracle parity tests, set there.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle.complex_oracle as C  # noqa: E402
import oracle.eodabe_oracle as O  # noqa: E402
import workloads as W  # noqa: E402
from test_gpu_complex import check as check_complex  # noqa: E402
from test_gpu_parity import check_factor, say  # noqa: E402


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,m,n,r", [(80, 2000, 500, 210), (80, 4096, 500, 210), (96, 2000, 500, 250),
                                     (96, 4096, 500, 250), (127, 4096, 500, 300), (128, 2000, 500, 300),
                                     (128, 4096, 500, 300)])
def test_wide_blocks_on_tall_matrices(b, m, n, r, dtype):
    say(f"block {b} {m}x{n} rank {r} {dtype}")
    f64 = dtype == torch.float64
    A = W.lowrank_haar(700 + b, m=m, n=n, r=r, noise_std=0.0, decades=3.0 if f64 else 1.0)
    tol = 1e-9 if f64 else 1e-4
    stable = True if f64 else O.precision_stable(A, tol, b, 9)[0]
    f, ref = check_factor(A, dtype, tol, b=b, seed=9, stable=stable, rounding_only=True)
    assert f.blocks >= 3 and (f.rank == r or not stable)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128], ids=["c64", "c128"])
@pytest.mark.parametrize("k,m,n,r", [(64, 800, 300, 150), (64, 1500, 300, 150), (48, 1300, 300, 110)])
def test_wide_complex_blocks_on_tall_matrices(k, m, n, r, dtype):
    c128 = dtype == torch.complex128
    A = W.lowrank_complex(40 + k, m=m, n=n, r=r, decades=2.0 if c128 else 1.0)
    tol = 1e-10 if c128 else 1e-4
    stable = True if c128 else C.precision_stable_c(A, tol, k, 9)[0]
    f, ref = check_complex(A, dtype, tol, k, 9, stable=stable, rounding_only=True)
    assert f.rank == r or not stable
