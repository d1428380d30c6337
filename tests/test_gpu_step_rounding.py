"""Training-step gradients to the rounding: the loss's and the chunked 8x8 backward's FP32 sums
against stored outputs of the kernels that first computed them (tests/golden/README.md).  A step decides on thresholds (the sign
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


def _unit(seed, n):
    """n values in [0, 1) by a 32-bit LCG (independent of any library's generator)."""
    x, out = np.uint64(seed * 2654435761 % 2 ** 32), np.empty(n)
    for i in range(n):
        x = (x * np.uint64(1664525) + np.uint64(1013904223)) % np.uint64(2 ** 32)
        out[i] = float(x) / 2 ** 32
    return out


def raster_gradient(chunk, split):
    """d_rec of 900 small faint splats of nearly the background's colour on 24x16 pixels: long lists
    of few pairs a batch, whose gradients are small differences."""
    from paper_2509_12138_amd import ops, scene
    W, H, n, bg = 24, 16, 900, (0.3, 0.2, 0.1)
    u = _unit(7, 10 * n).reshape(10, n)
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0], rec[:, 1] = W * u[0], H * u[1]
    th, s = np.pi * u[2], 0.5 + 0.4 * u[3]
    a, b = 1 / s ** 2, 1 / (s * (1 + u[4])) ** 2
    rec[:, 2] = a * np.cos(th) ** 2 + b * np.sin(th) ** 2
    rec[:, 3] = (a - b) * np.sin(th) * np.cos(th)
    rec[:, 4] = a * np.sin(th) ** 2 + b * np.cos(th) ** 2
    rec[:, 5] = 0.02 + 0.25 * u[5]
    rec[:, 6:9] = np.asarray(bg) + 0.05 * u[6:9].T
    rec[:, 9] = np.linspace(1, 2, n)
    tb = np.tile(np.array([0, 0, W // 8 - 1, H // 8 - 1], np.int16), (n, 1))
    dI = (_unit(11, 3 * H * W).reshape(1, 3, H, W) - 0.5).astype(np.float32)
    bufs = ops.RasterBuffers(ops.Views.single(n, scene.orbit_cameras(1, W, H)), W, H, (8, 8))
    bufs.set_schedule("lpt+split" if split else "lpt", chunk=chunk)
    bufs.rec.copy_(torch.as_tensor(rec))
    bufs.tile_bbox.copy_(torch.as_tensor(tb))
    bufs.n_tiles.fill_((W // 8) * (H // 8))
    bufs.ensure_capacity(8 * n)
    bufs.bin_sort()
    assert bufs.check()[0] == 0
    bufs.order_tiles()
    bufs.raster_fwd(bg)
    bufs.zero_d_rec()
    bufs.raster_bwd(torch.as_tensor(dI).cuda(), bg=bg)
    return bufs.d_rec.cpu().numpy()


@pytest.mark.parametrize("masked", [False, True])
def test_loss_gradient_rounding(gpu, masked):
    # the same FP32 operations on every value: one rounding (2^-24) of each is allowed
    ref = np.load(os.path.join(GOLDEN, "loss_rounding.npz"))["masked" if masked else "whole"]
    ref = ref.astype(np.float64)
    d = np.linalg.norm(loss_gradient(masked) - ref) / np.linalg.norm(ref)
    print("[gpu-test] loss gradient rounding", masked, d, flush=True)
    assert d <= 2.0 ** -24


@pytest.mark.parametrize("chunk,split", [(64, False), (128, True)])
def test_raster_gradient_rounding(gpu, chunk, split):
    # the same FP32 terms; only the order of a row's sum over its pixels (about ten, of both signs)
    # is free: four roundings of the column's norm
    ref = np.load(os.path.join(GOLDEN, "raster_rounding.npz"))["chunk%d" % chunk]
    ref = ref.astype(np.float64)
    got = raster_gradient(chunk, split)
    d = np.linalg.norm(got - ref, axis=0) / np.linalg.norm(ref, axis=0)
    print("[gpu-test] raster gradient rounding", chunk, split, d.tolist(), flush=True)
    assert d.max() <= 4 * 2.0 ** -24
