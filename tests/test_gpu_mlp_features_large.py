"""gs_mlp_features on more points than its grid holds at once: rows of the whole call against calls
on a few of the points (bit for bit; a row depends on its own neighbours only)."""
import pytest

from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_features_past_the_grid(gpu):
    from paper_2509_12138_amd import learned_init
    n = 2 * 2 ** 22 + 37                       # 16 lanes a point: two walks of 2^18 blocks and a bit
    say("mlp features", n)
    g = torch.Generator(device="cuda").manual_seed(1)
    P = torch.rand((3, n), generator=g, device="cuda")
    N = torch.nn.functional.normalize(torch.randn((3, n), generator=g, device="cuda"), dim=0)
    i = torch.arange(n, device="cuda", dtype=torch.int32)[:, None]
    idx = i + torch.arange(1, 17, device="cuda", dtype=torch.int32)[None]
    idx[idx >= n] = -1                         # the last points miss neighbours
    dist = torch.rand((n, 16), generator=g, device="cuda").sort(dim=1).values
    x, dbar = learned_init.features_from_knn(P, N, idx, dist)
    for a in (0, 2 ** 22 - 50, 2 ** 23 - 50, n - 100):
        b = min(a + 100, n)
        e = min(b + 16, n)                     # the rows' neighbours
        sub = idx[a:e] - a
        sub[(idx[a:e] < 0) | (sub >= e - a)] = -1
        xs, ds = learned_init.features_from_knn(P[:, a:e].contiguous(), N[:, a:e].contiguous(),
                                                sub.contiguous(), dist[a:e].contiguous())
        assert torch.equal(xs[:b - a], x[a:b]) and torch.equal(ds[:b - a], dbar[a:b])
