"""The depth order of few pairs, sorted by one work-group, around its powers of
two and its limit: stable by depth, ties by pair index."""
import numpy as np
import pytest

from paper_2509_12138_amd import scene
from _gpu_helpers import raster_records, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 1000, 2047, 2049, 4095, 4096, 4097, 5000])
def test_depth_order(gpu, n, ties):
    from paper_2509_12138_amd import ops
    say("small sort", n, ties)
    rng = np.random.default_rng(n)
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0:2] = 8.0
    rec[:, 2] = rec[:, 4] = 0.01
    rec[:, 5] = 0.01
    rec[:, 9] = rng.integers(1, 9, n) * 0.5 if ties else rng.uniform(0.1, 1e4, n)
    tb = np.zeros((n, 4), np.int16)
    nt = np.ones(n, np.int32)
    nt[rng.uniform(size=n) < 0.1] = 0                       # culled pairs list nothing
    bufs = ops.RasterBuffers(ops.Views.single(n, scene.orbit_cameras(1, 16, 16)), 16, 16, (16, 16))
    raster_records(bufs, rec, tb, nt, (0.0, 0.0, 0.0), torch)
    order = np.argsort(rec[:, 9], kind="stable")
    order = order[nt[order] > 0]
    np.testing.assert_array_equal(bufs.ids[:len(order)].cpu().numpy(), order)
