"""The 8x8 chunked backward on both sides of its pair limit: batches of few
small footprints, of many, and of entries over the whole tile, lists that end
inside a batch, and pixels that the loss masks; against the oracle under the
bound the other raster tests use."""
import numpy as np
import pytest

import oracle
from paper_2509_12138_amd import scene
from _gpu_helpers import (grad_tolerance_check, masked_image_gradient, oracle_lists, raster_records,
                          rec_to_oracle, say)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

W, H, TILE, BG = 20, 13, (8, 8), (0.3, 0.2, 0.1)
SAME_RECORD_BITS = 1 | 2 | 4 | 8


@pytest.mark.parametrize("chunk", [64, 128])
@pytest.mark.parametrize("sigma", [0.56, 1.0, 2.0, 12.0])
@pytest.mark.parametrize("n", [1, 63, 65, 200])
def test_pairs_match_oracle(gpu, n, sigma, chunk):
    from paper_2509_12138_amd import ops
    say("pairs", n, sigma, chunk)
    rng = np.random.default_rng(int(n * 100 * sigma))
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0] = rng.uniform(-1, W + 1, n)
    rec[:, 1] = rng.uniform(-1, H + 1, n)
    th = rng.uniform(0, np.pi, n)                    # rotated, up to 1:2
    a, b = 1 / sigma ** 2, 1 / (sigma * rng.uniform(1, 2, n)) ** 2
    rec[:, 2] = a * np.cos(th) ** 2 + b * np.sin(th) ** 2
    rec[:, 3] = (a - b) * np.sin(th) * np.cos(th)
    rec[:, 4] = a * np.sin(th) ** 2 + b * np.cos(th) ** 2
    rec[:, 5] = rng.uniform(0.005, 0.9, n) * (0.05 if sigma > 5 else 1.0)
    rec[:, 6:9] = rng.uniform(0, 1, (n, 3))
    rec[:, 9] = np.linspace(1, 2, n)
    tx, ty = 3, 2
    tb = np.tile(np.array([0, 0, tx - 1, ty - 1], np.int16), (n, 1))
    nt = np.full(n, tx * ty, np.int32)
    nt, *_ = oracle_lists(rec, tb, nt, np.zeros(n, np.int64), TILE, W, H, 1)
    dI = masked_image_gradient(rng, H, W, S=1)
    views = ops.Views.single(n, scene.orbit_cameras(1, W, H))
    bufs = ops.RasterBuffers(views, W, H, TILE)
    bufs.set_schedule("lpt", chunk=chunk)
    raster_records(bufs, rec, tb, nt, BG, torch)
    bufs.zero_d_rec()
    bufs.raster_bwd(torch.as_tensor(dI).cuda(), bg=BG)
    torch.cuda.synchronize()
    o = oracle.render_bwd(rec_to_oracle(rec, tb, nt), W, H, dI[0], tile=TILE, bg=BG,
                          amb_bits=SAME_RECORD_BITS)
    ref = np.concatenate([o["d_mean2d"], o["d_conic"], o["d_opacity"][None], o["d_rgb"]]).T
    ok, worst = grad_tolerance_check(bufs.d_rec.cpu().numpy().astype(np.float64), ref,
                                     o["term_mass"].T, o["amb_mass"].T)
    assert ok, worst
