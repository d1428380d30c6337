"""gs_knn over the point sets that its grid has to fit: points that fill a
volume, surfaces, lines, a flat and a degenerate extent, clusters with
outliers, fewer points than neighbours, points that are not finite; k on both
sides of every compiled list length.  Distances must be those of an FP64 brute
force to 1e-5 relative; an index may differ only where the oracle's own
distances are that close."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def points(kind, n, rng):
    if kind == "volume":
        return rng.uniform(-1, 1, (3, n))
    if kind == "sphere":
        d = rng.normal(size=(3, n))
        return d / np.linalg.norm(d, axis=0)
    if kind == "plane":
        p = rng.uniform(-1, 1, (3, n))
        p[1] = 0.25
        return p
    if kind == "line":
        t = rng.uniform(-3, 3, n)
        return np.stack([t, 0.5 * t, -t])
    if kind == "same":
        return np.tile(np.array([[0.5], [1.0], [-2.0]]), (1, n))
    # a dense surface patch and a few far points
    p = rng.uniform(-0.01, 0.01, (3, n))
    p[2] *= 1e-3
    p[:, : n // 100] = rng.uniform(-1, 1, (3, n // 100))
    return p


@pytest.mark.parametrize("k", [1, 3, 4, 5, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("kind,n", [("volume", 5000), ("sphere", 7001), ("plane", 4000),
                                    ("line", 2500), ("same", 70), ("clusters", 5000),
                                    ("volume", 7), ("sphere", 1)])
def test_knn_grids_match_oracle(gpu, kind, n, k):
    from paper_2509_12138_amd import ops
    say("knn", kind, n, k)
    P = np.ascontiguousarray(points(kind, n, np.random.default_rng(3 * n + k)), np.float32)
    idx, dist, mean = ops.knn(torch.as_tensor(P).cuda(), k, with_mean=True)
    torch.cuda.synchronize()
    idx, dist, mean = idx.cpu().numpy(), dist.cpu().numpy().astype(np.float64), mean.cpu().numpy()
    have = min(k, n - 1)
    assert np.all(idx[:, have:] == -1) and np.all(np.isinf(dist[:, have:]))
    if have == 0:
        assert np.all(mean == 0)
        return
    ridx, rdist = oracle.knn(P.astype(np.float64), min(have + 1, n - 1))
    np.testing.assert_allclose(dist[:, :have], rdist[:, :have], rtol=1e-5, atol=1e-7)
    gaps = np.diff(rdist, axis=1, append=np.inf) <= 1e-5 * np.maximum(rdist, 1e-30) + 1e-7
    near = gaps[:, :have].copy()
    near[:, 1:] |= gaps[:, :have - 1]
    np.testing.assert_array_equal(idx[:, :have][~near], ridx[:, :have][~near])
    # no point is listed twice or lists itself; zero distances, whose squares
    # are equal too (other squares may round to one root), keep index order
    rows = np.arange(n)[:, None]
    assert not np.any(idx[:, :have] == rows)
    assert all(len(set(r)) == have for r in idx[:, :have])
    tie = dist[:, 1:have] == 0
    assert np.all(idx[:, 1:have][tie] > idx[:, :have - 1][tie])
    np.testing.assert_allclose(mean, dist[:, :have].mean(1), rtol=1e-5, atol=1e-7)


def test_knn_with_points_that_are_not_finite(gpu):
    """A NaN point is nobody's neighbour and has none; the others are unaffected."""
    from paper_2509_12138_amd import ops
    say("knn with NaN points")
    rng = np.random.default_rng(8)
    P = points("sphere", 3000, rng).astype(np.float32)
    bad = np.array([0, 17, 2999])
    P[:, bad] = np.nan
    idx, dist = (t.cpu().numpy() for t in ops.knn(torch.as_tensor(P).cuda(), 4))
    good = np.setdiff1d(np.arange(3000), bad)
    assert np.all(idx[bad] == -1)
    ridx, rdist = oracle.knn(P[:, good].astype(np.float64), 4)
    np.testing.assert_allclose(dist[good], rdist, rtol=1e-5, atol=1e-7)
    np.testing.assert_array_equal(np.isin(idx[good], good), True)
