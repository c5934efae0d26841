"""GPU parity at the sizes where the kernels' work split changes: edges of
strips and groups, remainders, the smallest sizes, misaligned buffers."""
import numpy as np
import pytest
import torch

from oracle import pyramid as pyr_ref
from test_gpu_visibility_pyramid import check_visibility

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2501_04782_amd import raster


@pytest.mark.parametrize("H,W,offset", [(1, 1, 0), (2, 2, 0), (3, 3, 0), (2, 4, 0), (5, 8, 0), (16, 12, 0),
                                        (17, 20, 1), (18, 6, 0), (33, 9, 3), (15, 16, 2)])
def test_pyramid_strip_edges(H, W, offset):
    """Strips of eight output rows and pairs of outputs: whole, cut and
    smaller than a strip; widths and base addresses that take the 16-byte loads
    and ones that do not.  Each output is a mean of values below 1 with 10
    roundings of 2^-24 per level."""
    rng = np.random.default_rng(100 * H + W)
    img = rng.random((5, H, W)).astype(np.float32)
    buf = torch.zeros(5 * H * W + offset, device="cuda")
    view = buf[offset:].view(5, H, W)
    view.copy_(torch.from_numpy(img))
    got = raster.gaussian_pyramid(view, 4)
    for lvl, (a, b) in enumerate(zip(got, pyr_ref.pyramid(img.astype(np.float64), 4))):
        assert tuple(a.shape) == b.shape
        np.testing.assert_allclose(a.cpu().numpy(), b, rtol=0, atol=(lvl + 1) * 10 * 2.0 ** -24)


@pytest.mark.parametrize("batch", [64, 128])
@pytest.mark.parametrize("kind", ["clip", "dense"])
def test_visibility_of_the_one_wave_forward(kind, batch):
    """The one-wave forward's flags (set after each batch of staged entries)
    against the oracle's contributors, as for the other kernels."""
    old = raster.get_tuning()
    raster.set_tuning(batch, old["sort_cap"], 52, 128)
    try:
        check_visibility(kind)
    finally:
        raster.set_tuning(old["batch"], old["sort_cap"], old["compact"], old["bwd_batch"])
