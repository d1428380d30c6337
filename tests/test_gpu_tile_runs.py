"""The default tile order over several images, whose runs per XCD depend on their number: every tile
is taken once, so images, per-pixel state and stored gradient sums are bit-identical to those of the
longest-first order."""
import numpy as np
import pytest

from paper_2509_12138_amd import scene
from _gpu_helpers import oracle_records, perturbed, raster_records, say, surface_scene

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,tile", [((40, 24), (16, 16)), ((70, 33), (8, 8)), ((16, 8), (16, 8))])
@pytest.mark.parametrize("slots", [1, 3, 7, 8, 9, 16, 24])
def test_default_order_takes_every_tile(gpu, slots, size, tile):
    from paper_2509_12138_amd import ops
    say("tile runs", slots, size, tile)
    W, H = size
    n = 300
    params = perturbed(surface_scene(n, 5), 5, amount=0.2)
    cams = scene.orbit_cameras(slots, W, H)
    rec, tb, nt, _ = oracle_records(params, cams, W, H, tile)
    dI = torch.as_tensor(np.random.default_rng(1).normal(size=(slots, 3, H, W)).astype(np.float32)).cuda()
    got = []
    for mode in ("default", "lpt"):
        bufs = ops.RasterBuffers(ops.Views.single(n, cams), W, H, tile)
        for t in (bufs.image, bufs.T_final):
            t.fill_(float("nan"))
        bufs.n_contrib.fill_(-1)
        bufs.set_schedule(mode, deterministic=True)
        raster_records(bufs, rec, tb, nt, (0.1, 0.2, 0.3), torch)
        bufs.zero_d_rec()
        bufs.raster_bwd(dI, bg=(0.1, 0.2, 0.3))
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in (bufs.image, bufs.T_final, bufs.n_contrib, bufs.d_rec)])
    assert np.isfinite(got[0][0]).all() and (got[0][2] >= 0).all()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
