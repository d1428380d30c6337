"""The density control where its block counts take more than one round of the
scan (over 4096 blocks of 256 Gaussians) and where the rows of the state end
inside a work-group's share: exact copies in order."""
import math

import numpy as np
import pytest

from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,color_rows", [(4096 * 256, 3), (4096 * 256 + 1, 3), (1_100_003, 12)])
def test_counts_over_one_scan_round(gpu, n, color_rows):
    from paper_2509_12138_amd import ops
    say("density large", n, color_rows)
    rows = {"mean": 3, "log_scale": 3, "quat": 4, "opacity_logit": 0, "color": color_rows}
    base = torch.arange(n, device="cuda", dtype=torch.float32)
    P = {k: (base.clone() if r == 0 else base + 0.25 * torch.arange(r, device="cuda")[:, None])
         .contiguous() for k, r in rows.items()}
    M = {k: v + 1 for k, v in P.items()}
    V = {k: v + 2 for k, v in P.items()}
    # every 3rd is pruned (faint), of the others every 5th is cloned
    i = torch.arange(n, device="cuda")
    P["opacity_logit"] = torch.where(i % 3 == 0, -1.0, 1.0)
    P["log_scale"] = torch.zeros_like(P["log_scale"])
    den = ops.Densifier(n)
    den.denom.fill_(1.0)
    den.accum.copy_((i % 5 == 0).float())
    count = torch.where(i % 3 == 0, 0, torch.where(i % 5 == 0, 2, 1))
    n_out = den.select(P, M, V, 0.5, 1.0, 0.0, math.inf, math.log(1.6))
    assert n_out == int(count.sum())
    z = torch.zeros((n, 2, 3), device="cuda")
    P2, M2, V2 = den.apply(P, M, V, n_out, z, math.log(1.6))
    src = torch.repeat_interleave(i, count)
    first = torch.ones_like(src, dtype=torch.bool)
    first[1:] = src[1:] != src[:-1]
    for k in rows:
        assert torch.equal(P2[k], P[k][..., src]), k
        assert torch.equal(M2[k], M[k][..., src] * first), k
        assert torch.equal(V2[k], V[k][..., src] * first), k
