"""Features at the edges of their launch: strips of 64 and of 256 pixels, chunks
of 16 features alone, spread over workgroups and several to a workgroup.

Reference: the FP64 product.  Bar: a sum of at most r products in FP32, each
step rounded, (r + 1) u32 |U||D| per entry.  What lies below D's diagonal and
between the rows of F is the caller's and is neither read nor written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2506_22713_amd as E  # noqa: E402

U32 = 2.0 ** -24


@pytest.mark.parametrize("m,r", [(1, 1), (63, 16), (64, 17), (65, 33), (255, 48), (300, 64), (1030, 100), (1024, 500),
                                 (4096, 200), (4097, 271), (16385, 17), (16384, 64), (16400, 90), (65535, 16),
                                 (65537, 17), (65536, 33), (262145, 15), (262143, 18)])
def test_features_at_launch_edges(m, r):
    print(f"[case] features {m} x {r}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1000 * r + m % 997)
    rc = r + 3
    Ut = torch.randn(r, m, generator=g, device="cuda")
    D = torch.full((rc, rc), float("nan"), device="cuda")
    D[:r, :r] = torch.randn(r, r, generator=g, device="cuda")
    low = torch.tril(torch.ones(r, r, dtype=torch.bool, device="cuda"), -1)
    D[:r, :r][low] = float("nan")
    F = torch.full((m, r + 2), 7.0, device="cuda")
    ctx = E.Context()
    st = E._lib.eodabe_features(ctx.h, Ut.data_ptr(), D.data_ptr(), m, r, rc, F.data_ptr(), F.stride(0))
    torch.cuda.synchronize()
    assert st == 0
    Dz = torch.where(low, torch.zeros((), device="cuda"), D[:r, :r])
    U64, D64 = Ut.T.double(), Dz.double()
    ref, bar = U64 @ D64, (r + 1) * U32 * (U64.abs() @ D64.abs())
    assert bool(((F[:, :r].double() - ref).abs() <= bar + 1e-30).all())
    assert bool((F[:, r:] == 7.0).all())
    assert np.isfinite(float(ref.abs().max()))
