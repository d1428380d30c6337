"""The whole-list backward of a queue's plan on both sides of its line (12 tiles a wave): a wave per
8x8 block of a tile, or per tile; against the plan without a queue, whose oracle tests stand
elsewhere (FP32 sums in another order)."""
import numpy as np
import pytest

from paper_2509_12138_amd import scene
from _gpu_helpers import (masked_image_gradient, oracle_records, perturbed, raster_records, say,
                          surface_scene)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stored", [True, False])
@pytest.mark.parametrize("waves", [1, 6, 7, 64])
@pytest.mark.parametrize("tile", [(16, 16), (8, 16), (32, 16), (8, 8)])
def test_queue_backward(gpu, tile, waves, stored):
    from paper_2509_12138_amd import ops
    say("queue backward", tile, waves, stored)
    W, H = 150, 110
    params = perturbed(surface_scene(6000, 17), 17, amount=0.2)
    cams = scene.orbit_cameras(1, W, H)
    rec, tb, nt, _ = oracle_records(params, cams, W, H, tile)
    dI = torch.as_tensor(masked_image_gradient(np.random.default_rng(4), H, W, S=1)).cuda()
    got = []
    for plan in (dict(mode="persistent", persistent_waves=waves), dict(mode="lpt")):
        bufs = ops.RasterBuffers(ops.Views.single(6000, cams), W, H, tile, store_state=stored)
        bufs.set_schedule(**plan)
        raster_records(bufs, rec, tb, nt, (0.1, 0.2, 0.3), torch)
        bufs.zero_d_rec()
        bufs.raster_bwd(dI, bg=(0.1, 0.2, 0.3))
        torch.cuda.synchronize()
        got.append(bufs.d_rec.cpu().numpy())
    assert np.linalg.norm(got[0] - got[1]) <= 1e-5 * np.linalg.norm(got[1])
