"""The rasterisers' 8x8 blocks at ragged image sizes: every tile shape, where
the last tiles hold blocks that are partly or wholly outside the image, in
every launch form of the backward (whole lists by block, whole lists by tile
with stored sums, chunks, recomputed transmittance; default, longest-first and
queue order), against the oracle under the bound the other raster tests use;
and the forward's own choice of waves per tile against one wave per tile."""
import numpy as np
import pytest

import oracle
from paper_2509_12138_amd import scene
from _gpu_helpers import (grad_tolerance_check, masked_image_gradient, oracle_records, perturbed,
                          raster_records, say, surface_scene)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

W, H, N = 77, 53, 1500
BG = (0.2, 0.1, 0.05)
SAME_RECORD_BITS = 1 | 2 | 4 | 8
TILES = [(16, 16), (8, 8), (16, 8), (8, 16), (32, 8), (32, 16), (16, 32)]
FORMS = [("default", 0, False, True), ("lpt", 0, False, True), ("persistent", 0, False, True),
         ("lpt", 0, True, True), ("lpt", 64, False, True), ("lpt", 128, True, True),
         ("default", 0, False, False), ("persistent", 0, True, False)]


@pytest.fixture(scope="module")
def inputs(gpu):
    params = perturbed(surface_scene(N, 91), 91)
    cams = scene.orbit_cameras(2, W, H)
    dI = masked_image_gradient(np.random.default_rng(17), H, W)
    refs = {}
    for tile in TILES:
        rec, tb, nt, views = oracle_records(params, cams, W, H, tile)
        grads = [oracle.render_bwd(views[v], W, H, dI[v], tile=tile, bg=BG,
                                   amb_bits=SAME_RECORD_BITS) for v in range(2)]
        refs[tile] = (rec, tb, nt, grads)
    return cams, dI, refs


@pytest.mark.parametrize("form", FORMS, ids=lambda f: "%s-%d-%s-%s" % (
    f[0], f[1], "fixed" if f[2] else "atomic", "stored" if f[3] else "recompute"))
@pytest.mark.parametrize("tile", TILES, ids=lambda t: "%dx%d" % t)
def test_backward_by_blocks_matches_oracle(inputs, tile, form):
    from paper_2509_12138_amd import ops
    sched, chunk, det, stored = form
    say("backward by blocks", tile, form)
    cams, dI, refs = inputs
    rec, tb, nt, grads = refs[tile]
    views = ops.Views.single(N, cams)
    bufs = ops.RasterBuffers(views, W, H, tile, store_state=stored)
    bufs.set_schedule(sched, chunk=chunk, deterministic=det)
    raster_records(bufs, rec, tb, nt, BG, torch)
    bufs.zero_d_rec()
    bufs.raster_bwd(torch.as_tensor(dI).cuda(), bg=BG)
    torch.cuda.synchronize()
    drec = bufs.d_rec.cpu().numpy().astype(np.float64)
    for v in range(2):
        o = grads[v]
        got = drec[v * N:(v + 1) * N]
        ref = np.concatenate([o["d_mean2d"], o["d_conic"], o["d_opacity"][None], o["d_rgb"]]).T
        ok, worst = grad_tolerance_check(got, ref, o["term_mass"].T, o["amb_mass"].T)
        assert ok, worst


@pytest.mark.parametrize("tile", TILES, ids=lambda t: "%dx%d" % t)
def test_forward_choice_of_waves_gives_identical_results(inputs, tile):
    from paper_2509_12138_amd import ops
    say("forward waves", tile)
    cams, _, refs = inputs
    rec, tb, nt, _ = refs[tile]
    views = ops.Views.single(N, cams)
    out = []
    for sched in ("default", "persistent"):                 # a queue runs one wave per tile
        bufs = ops.RasterBuffers(views, W, H, tile)
        bufs.set_schedule(sched)
        raster_records(bufs, rec, tb, nt, BG, torch)
        out.append([t.cpu().numpy() for t in (bufs.image, bufs.T_final, bufs.n_contrib)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
