"""The forward's packed 64-entry batches at their edges: lists of 1 to 193
entries that all reach every pixel, so that a batch holds an even, an odd and
the full number of entries, with and without pixels that stop inside it; and
with every other entry out of the box's reach.  The same FP32 records go to the
oracle; an FP32 composite of n entries is within 2^-23 n of it (each entry
rounds once at alpha, T and C), twice that is the bound."""
import numpy as np
import pytest

import oracle
from paper_2509_12138_amd import scene
from _gpu_helpers import raster_records, rec_to_oracle, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BG = (0.3, 0.2, 0.1)


def _records(n, opacity, sparse, rng):
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0:2] = rng.uniform(2, 6, (n, 2))
    s = rng.uniform(12, 20, n)
    rec[:, 2] = rec[:, 4] = 1 / s ** 2
    if sparse:                       # narrow, beyond the first 8x8 block
        rec[::2, 0:2] = 13.0
        rec[::2, 2] = rec[::2, 4] = 4.0
    rec[:, 5] = opacity
    rec[:, 6:9] = rng.uniform(0, 1, (n, 3))
    rec[:, 9] = np.linspace(1, 2, n)
    return rec


@pytest.mark.parametrize("plan", [("default", 0, 0), ("default", 0, 1), ("lpt", 64, 4),
                                  ("lpt+split", 64, 1)], ids=lambda p: "%s-%d-%d" % p)
@pytest.mark.parametrize("opacity,sparse", [(0.02, False), (0.5, False), (0.1, True)])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 193])
def test_forward_batches(gpu, n, opacity, sparse, plan):
    from paper_2509_12138_amd import ops
    say("forward batches", n, opacity, sparse, plan)
    W = H = 16
    rec = _records(n, opacity, sparse, np.random.default_rng(n))
    tb = np.zeros((n, 4), np.int16)
    nt = np.ones(n, np.int32)
    views = ops.Views.single(n, scene.orbit_cameras(1, W, H))
    bufs = ops.RasterBuffers(views, W, H, (16, 16))
    bufs.set_schedule(plan[0], chunk=plan[1], fwd_waves=plan[2])
    raster_records(bufs, rec, tb, nt, BG, torch)
    ref = oracle.render(rec_to_oracle(rec, tb, nt), W, H, bg=BG)
    keep = ~np.asarray(ref["ambiguous"]).astype(bool)
    assert keep.mean() > 0.9
    tol = 2 * 2.0 ** -23 * max(n, 8)
    d = np.abs(bufs.image[0].cpu().numpy() - ref["image"])[:, keep]
    assert d.max() <= tol
    assert np.abs(bufs.T_final[0].cpu().numpy() - ref["T_final"])[keep].max() <= tol
    np.testing.assert_array_equal(bufs.n_contrib[0].cpu().numpy()[keep], ref["n_contrib"][keep])
