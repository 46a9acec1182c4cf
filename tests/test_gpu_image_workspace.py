"""compress_image with the workspace of one channel, whatever the context's
history: accepted, with the bits of the larger one."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2506_22713_amd as E  # noqa: E402
import workloads as W  # noqa: E402


def compress(ctx, img, tol, ws, nbytes):
    c, h, w = img.shape
    rc = min(h, w)
    pool = torch.zeros(c * rc * (h + rc + w), dtype=torch.float32, device="cuda")
    recon = torch.empty_like(img)
    info = E.ImageInfo()
    st = E._lib.eodabe_compress_image(ctx.h, img.data_ptr(), c, h, w, tol, ws.data_ptr(), nbytes, pool.data_ptr(),
                                      pool.numel(), recon.data_ptr(), ctypes.byref(info))
    return st, recon, [int(info.rank[i]) for i in range(c)], info


@pytest.mark.parametrize("channels,h,w", [(3, 256, 200), (4, 90, 333)])
def test_small_workspace_is_accepted_at_any_time(channels, h, w):
    print(f"[case] image {channels}x{h}x{w}", flush=True)
    img = torch.from_numpy(np.stack([W.rgb_image(5, h, w, noise_std=0.1)[c % 3] + c for c in range(channels)])
                           .astype(np.float32)).cuda()
    ctx = E.Context(block=16, seed=4)
    size = lambda: E._lib.eodabe_image_workspace_size(ctx.h, channels, h, w)
    small = size()
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    st, recon0, ranks0, info0 = compress(ctx, img, 1e-3, ws, small)
    assert st == 0
    for _ in range(35):
        E.compress_image(img[:, :8, :8].contiguous(), 1e-3, ctx)
    large = size()
    assert large > small                              # one per channel by now
    wl = torch.empty(large, dtype=torch.uint8, device="cuda")
    for buf, nbytes in ((wl, large), (ws, small), (wl, large - 1), (wl, large), (ws, small)):
        st, recon, ranks, info = compress(ctx, img, 1e-3, buf, nbytes)
        assert st == 0 and ranks == ranks0 and torch.equal(recon, recon0)
        assert (info.relerr, info.psnr, info.ssim, info.stored) == (info0.relerr, info0.psnr, info0.ssim, info0.stored)
    assert compress(ctx, img, 1e-3, ws, small - 1)[0] == E.EODABE_EWORKSPACE
