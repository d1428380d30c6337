"""The network's kernels at the edges of their 16-point tiles and neighbour
lists: point counts around a tile, a wave's and a work-group's share; features
of sets with fewer than 16 other points.  Tolerances as in the other network
tests (normwise 1e-3; features within one bf16 step)."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import say
from test_gpu_mlp import (NAMES, ORACLE_NAMES, _frame_ambiguous, _surface, bf16_bits, dev32,
                          normwise, oracle_net, weights)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 16, 33, 64, 65, 16385])
def test_network_at_tile_edges(gpu, n):
    from paper_2509_12138_amd import learned_init as li
    say("network edges", n)
    rng = np.random.default_rng(n)
    w = weights(n)
    xq = oracle.bf16_round(rng.normal(size=(n, 96)))
    dy = rng.normal(size=(n, 8)) / n
    mlp = li.InitMLP({k: dev32(v) for k, v in w.items()})
    x = torch.as_tensor(bf16_bits(xq)).cuda()
    y = torch.full((n + 1, 8), 7.0, device="cuda")
    mlp.forward(x, y[:n])
    ref, cache = oracle.mlp_forward(xq, *oracle_net(w), quantize=True)
    assert normwise(y[:n].cpu().numpy(), ref) <= 1e-3
    assert torch.all(y[n] == 7.0)                        # nothing past the last point
    grads = {k: torch.zeros_like(v) for k, v in mlp.w.items()}
    mlp.backward(x, dev32(dy), grads)
    back = oracle.mlp_backward(cache, dy, quantize=True)
    for k in NAMES:
        assert normwise(grads[k].cpu().numpy(), back[ORACLE_NAMES[k]]) <= 1e-3, k


@pytest.mark.parametrize("n", [2, 5, 16, 17, 300])
def test_features_of_small_sets(gpu, n):
    from paper_2509_12138_amd import learned_init as li
    say("features of", n)
    pts, nrm = _surface(n, 40 + n)
    have = min(16, n - 1)
    ri, rd = oracle.knn(pts, have)
    idx = np.full((n, 16), -1, np.int32)
    dist = np.full((n, 16), np.inf)
    idx[:, :have], dist[:, :have] = ri, rd
    x, dbar = li.features_from_knn(dev32(pts), dev32(nrm), torch.as_tensor(idx).cuda(),
                                   dev32(dist))
    xg = (x.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    xr, dr = oracle.mlp_features(pts.astype(np.float32), nrm.astype(np.float32), idx,
                                 dist.astype(np.float32), quantize=True)
    np.testing.assert_allclose(dbar.cpu().numpy(), dr, rtol=2e-6)
    assert np.all(xg[:, 6 * have:] == 0)
    ok = ~_frame_ambiguous(nrm.astype(np.float32))
    d = np.abs(xg.astype(np.float64) - xr)[ok]
    assert np.all(d <= 2.0 ** -7 * np.abs(xr[ok]) + 1e-6)
