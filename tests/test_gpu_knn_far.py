"""gs_knn where many points lie far from their neighbours in cells (long tails, outliers of a line
and a plane, few points in a large box): the shells of blocks against an FP64 brute force, for k on
both sides of the compiled list lengths.  Distances to 1e-5 relative; an index may differ only where
the oracle's own distances are that close."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def points(kind, n, rng):
    p = rng.normal(size=(3, n))
    if kind == "normal":
        return p
    if kind == "tail":
        return p * np.exp(2 * rng.normal(size=n))
    if kind == "line":
        p[1:] = 0
        p[0] *= np.exp(rng.normal(size=n))
        return p
    if kind == "plane":
        p[2] = -1
        return p * np.exp(rng.normal(size=n))
    if kind == "far pair":                       # two points 1000 spans away, a shell of 6 more
        p[0, :2] += 1000
        p[1, 2:8] += 30 * np.array([1, -1, 2, -2, 3, -3])
        return p
    i = np.arange(n)                             # a lattice: every distance ties
    q = round(n ** (1 / 3))
    return np.stack([i % q, i // q % q, i // (q * q)]) * 1.0


@pytest.mark.parametrize("k", [1, 3, 8, 17, 32])
@pytest.mark.parametrize("kind,n", [("normal", 6000), ("tail", 4000), ("line", 3000), ("plane", 4000),
                                    ("far pair", 3000), ("lattice", 3375), ("normal", 40), ("tail", 5)])
def test_knn_far_points(gpu, kind, n, k):
    from paper_2509_12138_amd import ops
    say("knn far", kind, n, k)
    P = np.ascontiguousarray(points(kind, n, np.random.default_rng(n + k)), np.float32)
    idx, dist, mean = ops.knn(torch.as_tensor(P).cuda(), k, with_mean=True)
    torch.cuda.synchronize()
    idx, dist, mean = idx.cpu().numpy(), dist.cpu().numpy().astype(np.float64), mean.cpu().numpy()
    have = min(k, n - 1)
    assert np.all(idx[:, have:] == -1) and np.all(np.isinf(dist[:, have:]))
    ridx, rdist = oracle.knn(P.astype(np.float64), min(have + 1, n - 1))
    np.testing.assert_allclose(dist[:, :have], rdist[:, :have], rtol=1e-5, atol=1e-7)
    gaps = np.diff(rdist, axis=1, append=np.inf) <= 1e-5 * np.maximum(rdist, 1e-30) + 1e-7
    near = gaps[:, :have].copy()
    near[:, 1:] |= gaps[:, :have - 1]
    np.testing.assert_array_equal(idx[:, :have][~near], ridx[:, :have][~near])
    assert not np.any(idx[:, :have] == np.arange(n)[:, None])
    assert all(len(set(r)) == have for r in idx[:, :have])
    np.testing.assert_allclose(mean, dist[:, :have].mean(1), rtol=1e-5, atol=1e-7)
