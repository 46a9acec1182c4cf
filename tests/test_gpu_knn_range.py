"""KNN on features whose squares and products leave the FP32 range.

The FP32 filter may only drop a pair that cannot be among the k nearest; where
a product -2 x.y overflows, to either side, the pair's FP64 distance is finite
and has to be looked at.  Predictions are integers: equality with the oracle.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle.apps_oracle as P  # noqa: E402
import paper_2506_22713_amd as E  # noqa: E402


def compare(F, lab, fold, k, nclass):
    F = F.astype(np.float32)
    pred, conf, oa = E.knn_cv(torch.from_numpy(F).cuda(), torch.from_numpy(lab).cuda(), torch.from_numpy(fold).cuda(),
                              k, nclass)
    p_ref, c_ref, oa_ref = P.knn_cv(F, lab, fold, k, nclass)
    assert np.array_equal(pred.cpu().numpy(), p_ref) and np.array_equal(conf, c_ref) and oa == oa_ref


@pytest.mark.parametrize("far,near", [(1e20, -2e18), (-1e25, 1e15), (-1e20, 2e18), (3e38, -3e18), (1e19, -1e19)])
@pytest.mark.parametrize("d", [1, 5])
def test_lone_far_queries(far, near, d):
    # two queries on one side, every candidate on the other: the products
    # overflow upwards while the candidates' own norms stay in range
    print("[case] far", far, "near", near, "d", d, flush=True)
    rng = np.random.default_rng(d)
    m = 90
    F = np.empty((m, d))
    F[:] = near * (1.0 + 0.3 * rng.random((m, d)))
    F[7], F[8] = far, 0.9 * far
    lab = rng.integers(1, 4, m).astype(np.int32)
    fold = rng.integers(0, 10, m).astype(np.int32)
    compare(F, lab, fold, 5, 4)


@pytest.mark.parametrize("d,lo,hi", [(1, 17, 20), (3, 17, 20), (6, 17, 20), (17, 17, 19), (32, 16, 21), (2, -3, 38),
                                     (32, -19, -18), (32, -20, -18), (9, -19, -17), (2, -20, -18)])
def test_both_signs_across_the_range(d, lo, hi):
    print("[case] d", d, "magnitudes 10^", lo, hi, flush=True)
    rng = np.random.default_rng(100 * d + hi)
    m = 300
    F = 10.0 ** rng.uniform(lo, hi, (m, d)) * rng.choice([-1.0, 1.0], (m, d))
    lab = rng.integers(0, 5, m).astype(np.int32)
    fold = rng.integers(0, 10, m).astype(np.int32)
    compare(F, lab, fold, 4, 5)
