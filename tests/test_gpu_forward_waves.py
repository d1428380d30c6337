"""One forward wave per tile against several: a queue's plan runs one, and its images, per-pixel
state and the chunk checkpoints that the backward reads are bit-identical to those of the plans that
split a tile's pixels; the chunked gradients then differ in the order of the atomic sums only."""
import numpy as np
import pytest

from paper_2509_12138_amd import scene
from _gpu_helpers import oracle_records, perturbed, raster_records, say, surface_scene

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _read_checkpoints(bufs):
    """The checkpoints [S, H, W, boundaries, 4] at the boundaries behind which the pixel still
    blends (the others are never read): a list of (pixel's flat index, boundary) and the values."""
    tw, th = bufs.tile
    off = bufs.chunk_offset.cpu().numpy().view(np.uint32).astype(np.int64)
    ck = bufs.checkpoints.cpu().numpy()
    nc = bufs.n_contrib.cpu().numpy()
    S, H, W = nc.shape
    s, y, x = np.meshgrid(np.arange(S), np.arange(H), np.arange(W), indexing="ij")
    tile = s * bufs.tiles_per_slot + (y // th) * bufs.tiles_x + x // tw
    place = (y % th) * tw + x % tw
    where, vals = [], []
    for c in range(int(nc.max()) // bufs.chunk + 1):
        sel = nc > (c + 1) * bufs.chunk
        where.append(np.flatnonzero(sel))
        vals.append(ck[off[tile[sel]] + c, place[sel]])
    return where, vals


@pytest.mark.parametrize("tile,fwd_waves", [((16, 16), 2), ((16, 16), 4), ((16, 16), 1), ((8, 16), 2),
                                            ((8, 16), 1), ((16, 8), 2), ((32, 8), 4), ((32, 16), 4),
                                            ((32, 16), 1), ((16, 32), 2), ((8, 8), 1)])
def test_one_wave_and_several(gpu, tile, fwd_waves):
    from paper_2509_12138_amd import ops
    say("forward waves", tile, fwd_waves)
    W, H, chunk, bg = 150, 110, 64, (0.1, 0.2, 0.3)
    params = perturbed(surface_scene(8000, 91), 91, amount=0.2)
    cams = scene.orbit_cameras(2, W, H)
    rec, tb, nt, _ = oracle_records(params, cams, W, H, tile)
    dI = torch.as_tensor(np.random.default_rng(4).normal(size=(2, 3, H, W)).astype(np.float32)).cuda()
    got = []
    for mode, nw in (("persistent", 1), ("lpt", fwd_waves)):
        bufs = ops.RasterBuffers(ops.Views.single(8000, cams), W, H, tile)
        bufs.set_schedule(mode, chunk=chunk, fwd_waves=nw)
        raster_records(bufs, rec, tb, nt, bg, torch)
        bufs.zero_d_rec()
        bufs.raster_bwd(dI, bg=bg)
        torch.cuda.synchronize()
        got.append((bufs.image.cpu().numpy(), bufs.T_final.cpu().numpy(), bufs.n_contrib.cpu().numpy(),
                    *_read_checkpoints(bufs), bufs.d_rec.cpu().numpy()))
    assert ops.forward_waves(tile, "persistent", chunk, 1) == 1
    a, b = got
    for i in range(3):
        np.testing.assert_array_equal(a[i], b[i])
    assert sum(len(w) for w in a[3]) > 1000            # boundaries that are read
    for w0, w1, v0, v1 in zip(a[3], b[3], a[4], b[4]):
        np.testing.assert_array_equal(w0, w1)
        np.testing.assert_array_equal(v0, v1)
    # sums of a few dozen FP32 terms in another order
    assert np.linalg.norm(a[5] - b[5]) <= 1e-5 * np.linalg.norm(a[5])
