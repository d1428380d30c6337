"""The whole-list backward of many tiles with short lists (a wave per tile) against the chunked one
of the same call, and of a few tiles (a wave per 8x8 block); FP32 sums in another order."""
import numpy as np
import pytest

from paper_2509_12138_amd import scene
from _gpu_helpers import perturbed, say, surface_scene, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["default", "lpt"])
@pytest.mark.parametrize("tile,slots", [((16, 16), 9), ((16, 16), 1), ((8, 8), 3), ((32, 16), 17)])
def test_many_tiles(gpu, tile, slots, mode):
    from paper_2509_12138_amd import ops
    say("many tiles", tile, slots, mode)
    W, H, n = 1000, 530, 3000
    params = to_dev(perturbed(surface_scene(n, 23), 23, amount=0.2), torch)
    views = ops.Views.single(n, scene.orbit_cameras(slots, W, H))
    dI = torch.randn((slots, 3, H, W), generator=torch.Generator(device="cuda").manual_seed(2),
                     device="cuda")
    got = []
    for chunk in (0, 64):
        bufs = ops.RasterBuffers(views, W, H, tile)
        bufs.set_schedule(mode, chunk=chunk)
        bufs.render_checked(ops.gaussians_struct(params))
        for m in (0, 1) if chunk == 0 else (0,):      # stored, and replayed
            bufs.zero_d_rec()
            bufs.raster_bwd(dI, mode=m)
            got.append(bufs.d_rec.cpu().numpy().astype(np.float64))
        many = bufs.S * bufs.tiles_per_slot >= 64 * torch.cuda.get_device_properties(0).multi_processor_count
        blocks = ops.backward_blocks(tile, mode, size=(W, H), n_slots=slots, pairs=bufs.m)
        assert blocks == (tile[0] * tile[1] // 64 if many else 1) and many == (slots > 1)
    assert np.linalg.norm(got[2]) > 0
    for g in got[:2]:
        assert np.linalg.norm(g - got[2]) <= 1e-5 * np.linalg.norm(got[2])
