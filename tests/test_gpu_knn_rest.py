"""KNN where more pairs tie within the filter's bound than a query's list holds:
duplicated and quantised points.  The queries that the filter leaves are
answered by the definition, few or many of a workgroup's 32, for every width of
a row, with ties by index, empty folds and values that are no numbers.
Predictions are integers: equality with the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle.apps_oracle as P  # noqa: E402
import paper_2506_22713_amd as E  # noqa: E402


def compare(F, lab, fold, k, nclass):
    m, d = F.shape
    buf = np.full((m, d + 2), 3.0, np.float32)            # rows of a wider buffer
    buf[:, :d] = F
    pred, conf, oa = E.knn_cv(torch.from_numpy(buf).cuda()[:, :d], torch.from_numpy(lab).cuda(),
                              torch.from_numpy(fold).cuda(), k, nclass)
    p_ref, c_ref, oa_ref = P.knn_cv(buf[:, :d], lab, fold, k, nclass)
    assert np.array_equal(pred.cpu().numpy(), p_ref) and np.array_equal(conf, c_ref) and oa == oa_ref


@pytest.mark.parametrize("d", [1, 4, 5, 8, 12, 13, 16, 20, 24, 28, 29, 32])
@pytest.mark.parametrize("k", [1, 2, 7, 15, 16])
def test_quantised_features(d, k):
    print("[case] quantised d", d, "k", k, flush=True)
    rng = np.random.default_rng(17 * d + k)
    m = 700
    F = np.round(rng.standard_normal((m, d)) * (0.7 if d < 6 else 0.35))
    F[rng.random(m) < 0.4] = 0.0
    compare(F, rng.integers(0, 6, m).astype(np.int32), rng.integers(0, 10, m).astype(np.int32), k, 6)


@pytest.mark.parametrize("left", [1, 7, 8, 9, 16, 31, 32])
def test_left_queries_of_a_workgroup(left):
    # the first `left` of every 32 points are one point (more of them than a
    # list holds), the others lie apart
    print("[case] left", left, flush=True)
    rng = np.random.default_rng(left)
    m = 32 * 130 if left < 8 else 32 * 40 + 5
    F = rng.standard_normal((m, 6)) * 50.0
    F[np.arange(m) % 32 < left] = 0.5
    if left == 1:
        F[::32] = 0.5
    compare(F, rng.integers(0, 4, m).astype(np.int32), rng.integers(0, 10, m).astype(np.int32), 5, 4)


@pytest.mark.parametrize("m", [255, 256, 257, 513, 1025])
@pytest.mark.parametrize("kind", ["all", "two folds", "one fold", "few candidates", "nan", "inf"])
def test_duplicates_at_tile_edges(m, kind):
    print("[case]", kind, m, flush=True)
    rng = np.random.default_rng(m + len(kind))
    F = np.full((m, 5), 0.25)
    lab = rng.integers(0, 5, m).astype(np.int32)
    fold = rng.integers(0, 10, m).astype(np.int32)
    if kind == "two folds":
        fold = (np.arange(m) % 2).astype(np.int32)
    elif kind == "one fold":
        fold[:] = 3
    elif kind == "few candidates":                        # fewer than k for most queries
        fold[:] = 3
        fold[m // 2], fold[m - 1] = 1, 2
    elif kind == "nan":
        F[rng.random(m) < 0.2, 2] = np.nan
    elif kind == "inf":
        F[rng.random(m) < 0.2, 0] = np.inf
    if kind in ("nan", "inf"):
        # no distance to such a point compares as nearer: the definition without it
        m_ok = np.isfinite(F).all(1)
        pred, conf, oa = E.knn_cv(torch.from_numpy(F.astype(np.float32)).cuda(), torch.from_numpy(lab).cuda(),
                                  torch.from_numpy(fold).cuda(), 6, 5)
        ref = np.zeros(m, np.int32)
        idx = np.where(m_ok)[0]
        for i in idx:                                     # all distances are 0: the first six by index
            nn = idx[fold[idx] != fold[i]][:6]
            ref[i] = int(np.argmax(np.bincount(lab[nn], minlength=5)))
        assert np.array_equal(pred.cpu().numpy(), ref)
        return
    compare(F, lab, fold, 6, 5)
