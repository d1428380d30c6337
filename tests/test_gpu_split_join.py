"""The split forward's join by all lanes and pixel by pixel: few large splats whose pixels stop inside
chunks, on both sides of the rule's line, against the oracle (1e-5: FP32 products and sums of at most
a few hundred entries) and, n_contrib, exactly outside the oracle's decision bands."""
import numpy as np
import pytest

import oracle
from paper_2509_12138_amd import scene
from _gpu_helpers import raster_records, rec_to_oracle, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SAME_RECORD_BITS = 1 | 2 | 4 | 8


@pytest.mark.parametrize("chunk", [64, 128])
@pytest.mark.parametrize("tile", [(16, 16), (16, 8), (32, 16), (8, 8)])
@pytest.mark.parametrize("n", [90, 190, 400])
def test_join_forms_match_oracle(gpu, n, tile, chunk):
    from paper_2509_12138_amd import ops
    W, H, bg = 61, 47, (0.3, 0.2, 0.1)
    many = ops.join_many(tile, (W, H), 1, n)
    say("split join", n, tile, chunk, "all lanes" if many else "pixel by pixel")
    assert many == (tile != (8, 8) and n < 192 + 12)
    rng = np.random.default_rng(n + chunk)
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0], rec[:, 1] = rng.uniform(0, W, n), rng.uniform(0, H, n)
    s = rng.uniform(8, 30, n)
    rec[:, 2] = rec[:, 4] = 1 / s ** 2
    rec[:, 5] = rng.uniform(0.05, 0.6, n)            # most pixels stop
    rec[:, 6:9] = rng.uniform(0, 1, (n, 3))
    rec[:, 9] = np.linspace(1, 2, n)
    tx, ty = -(-W // tile[0]), -(-H // tile[1])
    tb = np.tile(np.array([0, 0, tx - 1, ty - 1], np.int16), (n, 1))
    nt = np.full(n, tx * ty, np.int32)
    bufs = ops.RasterBuffers(ops.Views.single(n, scene.orbit_cameras(1, W, H)), W, H, tile)
    bufs.set_schedule("lpt+split", chunk=chunk)
    raster_records(bufs, rec, tb, nt, bg, torch)
    o = oracle.render(rec_to_oracle(rec, tb, nt), W, H, tile=tile, bg=bg)
    keep = (o["ambiguity"] & SAME_RECORD_BITS) == 0
    T = bufs.T_final[0].cpu().numpy()
    assert keep.mean() > 0.5 and (T[keep] < 3e-4).mean() > 0.2
    assert np.abs(bufs.image[0].cpu().numpy() - o["image"])[:, keep].max() <= 1e-5
    assert np.abs(T - o["T_final"])[keep].max() <= 1e-5
    keep &= (o["ambiguity"] & 32) == 0                 # list positions
    np.testing.assert_array_equal(bufs.n_contrib[0].cpu().numpy()[keep], o["n_contrib"][keep])
