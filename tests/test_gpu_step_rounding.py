"""Training-step gradients to the rounding: the loss's FP32 sums against stored outputs of the
kernel that first computed them (tests/golden/README.md).  A step decides on thresholds (the sign
of the L1 term, alpha = 1/255, the stop), so gradients that move by a few roundings move a later
step's by whole terms."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


def loss_gradient(masked):
    """d loss / d image of a smooth 96x96 image: tiles inside the foreground, at its edge and at
    the image's; the rows and columns 20..75 of it."""
    from paper_2509_12138_amd import ops
    H = W = 96
    rng = np.random.default_rng(5)
    yy, xx = np.mgrid[0:H, 0:W]
    tgt = np.stack([0.5 + 0.4 * np.sin(0.09 * (c + 1) * xx) * np.cos(0.05 * yy) for c in range(3)])
    img = tgt + rng.normal(0, 0.03, tgt.shape)
    mask = ((xx - 70) ** 2 + (yy - 20) ** 2 > 14 ** 2).astype(np.uint8) if masked else None
    dev = [torch.as_tensor(np.ascontiguousarray(a[None], t)).cuda() if a is not None else None
           for a, t in ((img, np.float32), (tgt, np.float32), (mask, np.uint8))]
    _, d = ops.LossBuffers(1, H, W)(*dev, lam=0.2, grad_scale=1.0)
    return d[0, :, 20:76, 20:76].cpu().numpy()


@pytest.mark.parametrize("masked", [False, True])
def test_loss_gradient_rounding(gpu, masked):
    # the same FP32 operations on every value: one rounding (2^-24) of each is allowed
    ref = np.load(os.path.join(GOLDEN, "loss_rounding.npz"))["masked" if masked else "whole"].astype(np.float64)
    d = np.linalg.norm(loss_gradient(masked) - ref) / np.linalg.norm(ref)
    print("[gpu-test] loss gradient rounding", masked, d, flush=True)
    assert d <= 2.0 ** -24
