"""The 8x8 chunked backward keeps a non-finite pixel gradient, or colour, to the entries that blend
it: an entry just below the alpha threshold at that pixel is listed with it and adds nothing.  The
whole-list backward of the same records gives the rows that stay finite; sums differ in order only
(1e-5 of the largest)."""
import numpy as np
import pytest

from paper_2509_12138_amd import scene
from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

W, H = 16, 8


def _records():
    # A: alpha 2^-0.01 / 255 at the centre (6.5, 3.5) of pixel (6, 3); B and C: small ones there,
    # behind and in front of A; D: elsewhere in the tile
    far = float(np.sqrt(2 * (np.log(0.5 * 255) + 0.01 * np.log(2))))
    rec = np.zeros((4, 12), np.float32)
    for i, (x, y, a, o, depth) in enumerate([(6.5 - far, 3.5, 1.0, 0.5, 1.5), (6.5, 3.5, 9.0, 0.6, 2.0),
                                             (6.5, 3.5, 9.0, 0.4, 1.0), (2.5, 6.0, 2.0, 0.5, 1.2)]):
        rec[i, 0:6] = x, y, a, 0.0, a, o
        rec[i, 6:9] = 0.2 + 0.1 * i, 0.5, 0.7 - 0.1 * i
        rec[i, 9] = depth
    return rec


@pytest.mark.parametrize("chunk", [64, 128])
@pytest.mark.parametrize("what", ["gradient", "colour"])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_nonfinite_stays_with_its_pixel(gpu, what, value, chunk):
    from paper_2509_12138_amd import ops
    say("nonfinite", what, value, chunk)
    rec = _records()
    dI = np.random.default_rng(3).normal(size=(1, 3, H, W)).astype(np.float32)
    if what == "gradient":
        dI[0, 1, 3, 6] = value
    else:
        rec[0, 6] = value
    got = []
    for plan in (dict(mode="lpt", chunk=chunk), dict(mode="default")):
        n = len(rec)
        bufs = ops.RasterBuffers(ops.Views.single(n, scene.orbit_cameras(1, W, H)), W, H, (8, 8))
        bufs.set_schedule(**plan)
        bufs.rec.copy_(torch.as_tensor(rec))
        bufs.tile_bbox.copy_(torch.as_tensor(np.tile(np.array([0, 0, 1, 0], np.int16), (n, 1))))
        bufs.n_tiles.fill_(2)
        bufs.bin_sort()
        assert bufs.check()[0] == 0
        bufs.order_tiles()
        bufs.raster_fwd()
        bufs.zero_d_rec()
        bufs.raster_bwd(torch.as_tensor(dI).cuda())
        got.append(bufs.d_rec.cpu().numpy())
    g, ref = got
    fine = np.isfinite(ref)
    # with the gradient, B and C are hit; with the colour, A and what blends in front of it
    assert fine.any(axis=1).sum() >= 2 and not fine.all()
    np.testing.assert_array_equal(np.isfinite(g), fine)
    scale = np.abs(ref[fine]).max()
    assert np.abs(g[fine] - ref[fine]).max() <= 1e-5 * scale
