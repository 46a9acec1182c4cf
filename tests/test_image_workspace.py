"""Image workspace on the host (no GPU needed): a context that has compressed
no image asks for one channel's factorization, whatever the number of channels,
and for what the reconstruction of all of them takes."""
import pytest


@pytest.mark.parametrize("h,w", [(220, 220), (768, 1024), (1024, 768), (333, 517), (4096, 4096)])
@pytest.mark.parametrize("channels", [1, 2, 3, 4])
def test_new_context_asks_for_one_channel(h, w, channels):
    import paper_2506_22713_amd as E
    c = E.Context(host_only=True)
    one = c.workspace_size(h, w)
    got = E._lib.eodabe_image_workspace_size(c.h, channels, h, w)
    # beside it: D V^T per channel (r x w FP32), the sums of every 64 x 64 block, the criteria
    blocks = channels * ((h + 63) // 64) * ((w + 63) // 64)
    rest = 4 * channels * min(h, w) * w + 128 * blocks + 4096
    assert one < got <= one + rest
