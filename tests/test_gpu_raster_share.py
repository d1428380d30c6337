"""The whole-list backward with one to eight waves sharing the entries of a
block: image sizes on each side of the rule's lines, with atomic and with
stored sums, against the oracle under the bound the other raster tests use."""
import numpy as np
import pytest

import oracle
from paper_2509_12138_amd import scene
from _gpu_helpers import (grad_tolerance_check, masked_image_gradient, oracle_records, perturbed,
                          raster_records, say, surface_scene)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, TILE, BG = 1500, (16, 16), (0.2, 0.1, 0.05)
SAME_RECORD_BITS = 1 | 2 | 4 | 8


@pytest.mark.parametrize("W,H", [(128, 128), (304, 256), (400, 400), (528, 512)])
def test_shared_entries_match_oracle(gpu, W, H):
    from paper_2509_12138_amd import ops
    say("shared backward", W, H)
    params = perturbed(surface_scene(N, 93), 93)
    cams = scene.orbit_cameras(1, W, H)
    dI = masked_image_gradient(np.random.default_rng(W), H, W, S=1)
    rec, tb, nt, views = oracle_records(params, cams, W, H, TILE)
    o = oracle.render_bwd(views[0], W, H, dI[0], tile=TILE, bg=BG, amb_bits=SAME_RECORD_BITS)
    ref = np.concatenate([o["d_mean2d"], o["d_conic"], o["d_opacity"][None], o["d_rgb"]]).T
    for det in (False, True):
        runs = []
        for _ in range(2 if det else 1):
            bufs = ops.RasterBuffers(ops.Views.single(N, cams), W, H, TILE)
            bufs.set_schedule("default", deterministic=det)
            raster_records(bufs, rec, tb, nt, BG, torch)
            bufs.zero_d_rec()
            bufs.raster_bwd(torch.as_tensor(dI).cuda(), bg=BG)
            torch.cuda.synchronize()
            runs.append(bufs.d_rec.cpu().numpy())
        ok, worst = grad_tolerance_check(runs[0].astype(np.float64), ref, o["term_mass"].T,
                                         o["amb_mass"].T)
        assert ok, (det, worst)
        if det:
            np.testing.assert_array_equal(runs[0], runs[1])
