"""GPU parity at the edges of the kernels' tiles and dispatch rules.

Ranks on both sides of the 16-column blocks of the Cholesky and of the 64-
and 128-column limits between its kernels; spectra on both sides of the rule
that drops the second CholeskyQR pass; capacities below the block width;
feature rows past one register slice; tiles at every width of the batched
kernel's products.  The bars are the ones of the oracle parity tests (the
oracle's relative error plus 1e-10 in FP64, plus the FP32 rounding floor of a
rank-r factorization in FP32, orthonormality per column), set before the
first run.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle.eodabe_oracle as O  # noqa: E402
import paper_2506_22713_amd as E  # noqa: E402
import workloads as W  # noqa: E402
from test_gpu_parity import ORTH_TOL, U32, U64, check_factor, fp32_floor, say  # noqa: E402


def check_factors(A, U, D, Vt, r, b, seed, tol):
    """Noise-free content of exact rank: the FP32 bars of check_factor."""
    ref = O.eod_abe(A, tol, k=b, q=0, seed=seed)
    e_ref = O.rel_err(A, ref.U, ref.D, ref.V)
    assert ref.rank == r and e_ref < 1e-9
    U, D, Vt = (x.double().cpu().numpy() for x in (U, D, Vt))
    bar = max(1e-5, fp32_floor(r, *A.shape), 4.0 * (U32 / U64) * e_ref)
    assert np.linalg.norm(A - U @ D @ Vt) / np.linalg.norm(A) <= bar + e_ref
    for Z in (U, Vt.T):
        assert np.linalg.norm(Z.T @ Z - np.eye(r)) <= ORTH_TOL[torch.float32] * math.sqrt(r)
    assert np.all(np.tril(D, -1) == 0) and np.all(np.diag(D) >= 0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("r", [1, 15, 16, 17, 31, 33, 48, 49, 63, 64, 65, 100, 127, 128, 129, 193, 257])
def test_ranks_at_cholesky_blocks(r, dtype):
    m, n, b = r + 301, r + 187, 64 if r % 2 else 32
    say(f"rank {r} {m}x{n} b {b} {dtype}")
    f64 = dtype == torch.float64
    A = W.lowrank_haar(900 + r, m=m, n=n, r=r, noise_std=0.0, decades=3.0 if f64 else 1.5)
    tol = 1e-9 if f64 else 1e-4
    stable = True if f64 else O.precision_stable(A, tol, b, 31)[0]
    f, _ = check_factor(A, dtype, tol, b=b, seed=31, stable=stable, rounding_only=True)
    assert f.rank == r or not stable


@pytest.mark.parametrize("decades", [0.0, 1.0, 2.0, 3.0])
@pytest.mark.parametrize("r,b", [(60, 64), (100, 32), (200, 64)])
def test_second_pass_rule(r, b, decades):
    # flat spectra take one CholeskyQR pass, steep ones two: orthonormality
    # and error have to hold on both sides
    say(f"rank {r} b {b} decades {decades}")
    A = W.lowrank_haar(50 + r, m=640, n=400, r=r, noise_std=0.0, decades=decades)
    tol = 1e-4 if decades < 3 else 3e-5
    stable = O.precision_stable(A, tol, b, 5)[0]
    check_factor(A, torch.float32, tol, b=b, seed=5, stable=stable, rounding_only=True)


@pytest.mark.parametrize("cap", [12, 13, 16, 20, 31])
@pytest.mark.parametrize("m,n", [(300, 200), (90, 400)])
def test_capacity_below_block(m, n, cap):
    say(f"{m}x{n} rank 12 r_cap {cap}, block 32")
    A = W.lowrank_haar(77, m=m, n=n, r=12, noise_std=0.0, decades=1.0)
    a = torch.from_numpy(A).float().cuda()
    f = E.factor(a, 1e-4, ctx=E.Context(seed=2, block=32), r_cap=cap)
    torch.cuda.synchronize()
    assert f.rank == 12
    check_factors(A, f.U, f.D, f.Vt, 12, 32, 2, 1e-4)


@pytest.mark.parametrize("m", [255, 257, 1030])
@pytest.mark.parametrize("r", [1, 15, 16, 17, 33])
def test_feature_rows(m, r):
    say(f"features {m} rows of rank {r}")
    A = W.lowrank_haar(60 + r, m=m, n=90, r=r, noise_std=0.0, decades=1.0)
    f = E.factor(torch.from_numpy(A).float().cuda(), 1e-4, ctx=E.Context(seed=4, block=64))
    F = E.features(f)
    torch.cuda.synchronize()
    assert F.shape == (m, r)
    U, D = f.U.double().cpu().numpy(), f.D.double().cpu().numpy()
    # a sum of r products in FP32, each rounded: r u32 |U||D| per entry, and one rounding of the result
    bar = (r + 1) * U32 * (np.abs(U) @ np.abs(D))
    assert np.all(np.abs(F.double().cpu().numpy() - U @ D) <= bar + 1e-30)


# sides at and around the 64-row panels, ranks at the 16-column blocks, one
# and two chunks of the rank-128 closing; tall, wide, and unaligned rows
TILE_EDGES = [(64, 64, 16), (65, 63, 17), (129, 127, 31), (130, 260, 33), (260, 132, 48), (257, 255, 64),
              (255, 258, 65), (320, 321, 100), (1024, 200, 49), (201, 1023, 63), (350, 301, 128), (33, 17, 1)]


@pytest.mark.parametrize("b", [16, 31, 40, 64])
def test_tile_widths(b):
    tiles = [W.lowrank_haar(300 + i, m=h, n=w, r=r, noise_std=0.0, decades=1.0)
             for i, (h, w, r) in enumerate(TILE_EDGES)]
    bt = E.Batch(E.Context(seed=8, block=b), [torch.from_numpy(T).float().cuda() for T in tiles])
    bt.run(1e-4)
    torch.cuda.synchronize()
    assert set(bt.status.tolist()) <= {0}, bt.status
    for t, (h, w, r) in enumerate(TILE_EDGES):
        say(f"tile {h}x{w} rank {r} b {b}")
        U, D, Vt, rk, _ = bt.result(t)
        assert rk == r, (h, w, r, rk)
        check_factors(tiles[t], U, D, Vt, r, b, 8, 1e-4)


@pytest.mark.parametrize("channels,h,w,tol", [(2, 300, 200, 1e-3), (3, 200, 300, 1e-3), (4, 333, 257, 1e-4),
                                              (3, 90, 400, 1e-4)])
def test_image_channels_overlap(channels, h, w, tol):
    # a context's first 32 images go channel by channel, later ones overlap the
    # channels: the same factors bit for bit, also where a channel's rank needs
    # several chunks of blocks, differs between channels or is zero
    say(f"image {channels}x{h}x{w} tol {tol}")
    rng = np.random.default_rng(h)
    img = np.stack([W.lowrank_haar(c, m=h, n=w, r=(70, 5, 33, 1)[c], noise_std=0.0, decades=1.0) * 40 + c
                    for c in range(channels)]).astype(np.float32)
    imgs = [img, img + rng.standard_normal(img.shape).astype(np.float32) * 1e-3, np.zeros_like(img)]
    imgs[1][channels - 1] = 0.0
    ctx = E.Context(block=16, seed=3)
    first = E.compress_image(torch.from_numpy(img).cuda(), tol, ctx)
    small = torch.from_numpy(img[:, :8, :8].copy()).cuda()
    for _ in range(31):
        E.compress_image(small, tol, ctx)
    for k, x in enumerate(imgs):
        d = torch.from_numpy(x).cuda()
        out = E.compress_image(d, tol, ctx)
        ref = first if k == 0 else E.compress_image(d, tol, E.Context(block=16, seed=3))
        assert list(out.info.rank[:channels]) == list(ref.info.rank[:channels])
        for a, b in zip(out.factors, ref.factors):
            for u, v in zip(a, b):
                assert torch.equal(u, v)
        assert torch.equal(out.recon, ref.recon)
