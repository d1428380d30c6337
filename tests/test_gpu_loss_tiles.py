"""The loss at the line between its two tile forms: a 32x32 tile whose 52x52
inputs are all foreground blurs no mask; one pixel of background, or of the
image's outside, among them takes the general form.  Tolerance as in the other
loss tests (1e-5 of the largest gradient)."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# the inputs of tile (1, 1) are rows and columns 22..73
@pytest.mark.parametrize("H,W,hole", [(74, 74, None), (73, 74, None), (74, 73, None),
                                      (84, 90, (22, 22)), (84, 90, (73, 73)), (84, 90, (22, 73)),
                                      (84, 90, (21, 40)), (84, 90, (74, 40)), (84, 90, (48, 48))])
def test_all_foreground_tiles(gpu, H, W, hole):
    from paper_2509_12138_amd import ops
    say("loss tiles", H, W, hole)
    rng = np.random.default_rng(H * W + (0 if hole is None else 7 * hole[0] + hole[1]))
    yy, xx = np.mgrid[0:H, 0:W]
    tgt = np.stack([0.5 + 0.4 * np.sin(0.11 * (c + 1) * xx) * np.cos(0.07 * yy) for c in range(3)])
    tgt = tgt[None].astype(np.float32)
    img = np.clip(tgt + rng.normal(0, 0.05, tgt.shape), 0, 1).astype(np.float32)
    mask = np.ones((1, H, W), np.uint8)
    if hole is not None:
        mask[0, hole[0], hole[1]] = 0
    L = ops.LossBuffers(1, H, W)
    loss, dI = L(torch.as_tensor(img).cuda(), torch.as_tensor(tgt).cuda(),
                 torch.as_tensor(mask).cuda(), lam=0.2, grad_scale=1.0)
    o = oracle.loss(img[0], tgt[0], mask[0], lam=0.2)
    assert abs(float(loss[0]) - o["loss"]) <= 1e-5 * abs(o["loss"])
    r = o["d_image"]
    assert np.abs(dI[0].cpu().numpy() - r).max() <= 1e-5 * np.abs(r).max()
    if hole is None:        # no mask is a mask of ones
        loss2, dI2 = L(torch.as_tensor(img).cuda(), torch.as_tensor(tgt).cuda(), None, lam=0.2,
                       grad_scale=1.0)
        assert torch.equal(loss2, loss) and torch.equal(dI2, dI)
