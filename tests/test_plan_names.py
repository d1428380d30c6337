"""Raster plans say what runs (no GPU): forward waves of 0 or 1 leave the number to the library, so
the tuner never times one launch under two names, its plans carry the launched number, and the
kernel names that bench.py prints are instances the library holds."""
import importlib.util
import os
import random
import shutil
import subprocess

import pytest

from paper_2509_12138_amd import _lib, autotune, ops

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2509_12138_amd import build
        build.build()
    return _lib.load()


@pytest.mark.parametrize("stored", [True, False])
@pytest.mark.parametrize("seed", range(4))
def test_search_times_a_launch_once(seed, stored):
    rng = random.Random(seed)
    timed = {}

    def measure(plan):
        plan = autotune.normalize(plan)
        if not stored and plan[2]:
            return None
        assert autotune.valid(plan), plan
        return timed.setdefault(plan, rng.uniform(1, 2))

    autotune.staged_search(measure, stored)
    launches = [(t, s, c, ops.forward_waves(t, s, c, w), d) for t, s, c, w, d in timed]
    assert len(set(launches)) == len(launches)
    assert launches == list(timed)                     # the plans name what they launch


@pytest.mark.parametrize("tile,most", [((16, 16), 4), ((8, 8), 1), ((16, 8), 2), ((8, 16), 2),
                                       ((32, 8), 4), ((32, 16), 4), ((16, 32), 4)])
def test_launched_waves(tile, most):
    assert ops.forward_waves(tile, "lpt", 64, 1) == ops.forward_waves(tile) == most
    assert ops.forward_waves(tile, "lpt", 64, most) == most
    assert ops.forward_waves(tile, "persistent", 64, 1) == 1
    assert ops.forward_waves(tile, "lpt+split", 64, 1) == 1
    assert ops.forward_waves(tile, "lpt+split", 0, 1) == most      # no chunks, no split
    # a plan of an older cache, and one stored with the library's choice
    assert autotune.normalize((list(tile), "lpt", 64))[3] == most
    assert autotune.normalize((tile, "persistent", 0, 1, False))[3] == 1
    if most > 1:
        assert ops.forward_waves(tile, "lpt", 64, 2) == 2
        assert autotune.normalize((tile, "lpt", 64, 2, False))[3] == 2


def test_bench_names_are_instances():
    nm = shutil.which("nm")
    if nm is None:
        pytest.skip("no nm")
    out = subprocess.run([nm, "-C", "--defined-only", _lib.LIB_PATH], check=True,
                         capture_output=True, text=True).stdout
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    names = set()
    for tile in autotune.TILES:
        for waves in (1, 2, 4):
            if tile[0] * tile[1] // 64 % waves == 0:
                for sched, chunk in (("lpt", 64), ("default", 0), ("persistent", 0), ("lpt+split", 64)):
                    for pairs in (0, 10 ** 9):
                        names.update(bench.fwd_kernel_name(tile, 1 if sched == "persistent" else waves,
                                                           sched, chunk, pairs=pairs).split("+"))
        for chunk in (0, 64):
            for recompute in (False, True):
                for det in (False, True):
                    names.add(bench.bwd_kernel_name(tile, chunk, recompute, det))
    missing = [n for n in sorted(names) if "gsmi::__device_stub__" + n not in out
               and "gsmi::" + n + "(" not in out]
    assert not missing, missing
    assert bench.fwd_kernel_name((16, 16), 1, "lpt", 64) == "k_raster_fwd<16, 16, 4>"
    assert bench.bwd_kernel_name((16, 16), 0, False, False) == "k_raster_bwd<16, 16, 1, false>"


@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (32, 16)])
@pytest.mark.parametrize("waves", [1, 64, 4096])
def test_queue_of_few_waves_takes_tiles(tile, waves):
    # 12 tiles a wave is the line between a wave per 8x8 block and one per tile
    nb = tile[0] * tile[1] // 64
    for tiles, blocks in ((12 * waves, 1), (12 * waves + 1, nb)):
        args = dict(size=(tile[0] * tiles, tile[1]), pairs=10 ** 9)
        assert ops.backward_blocks(tile, "persistent", persistent_waves=waves, **args) == blocks
        assert ops.backward_blocks(tile, "lpt", persistent_waves=waves, **args) == 1
        assert ops.backward_blocks(tile, "lpt", True, **args) == nb


@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (32, 16)])
def test_many_tiles_of_short_lists_take_tiles(tile):
    # the rule's lines on a device of 256 CUs (the number a host without one assumes)
    from paper_2509_12138_amd.ops import backward_blocks
    if pytest.importorskip("torch").cuda.is_available():
        pytest.skip("the CU count is the device's")
    nb = tile[0] * tile[1] // 64
    for per_cu, slots in ((63, 1), (64, 1), (64, 4), (512, 32)):
        tiles = 256 * per_cu
        size = (tile[0] * tiles // slots, tile[1])
        for mode, div in (("lpt", 2), ("default", 16)):
            line = per_cu // div
            args = dict(size=size, n_slots=slots)
            few = nb if per_cu >= 64 else 1
            assert backward_blocks(tile, mode, pairs=tiles * line, **args) == few
            assert backward_blocks(tile, mode, pairs=tiles * (line + 1), **args) == 1


def test_launches_hold_their_threads():
    # a launch takes at most 2^32 - 1 threads, 64 a wave: 16x16 tiles of one 65536x65536 image are
    # 2^24, of which four waves each are one thread too many
    big, n = (65536, 65536), 10 ** 12
    below = (65536, 65520 - 16)
    assert ops.forward_waves((16, 16), size=big) == 2 and ops.forward_waves((16, 16), size=below) == 4
    assert ops.forward_waves((16, 16), size=big, n_slots=2) == 1
    assert ops.backward_blocks((16, 16), size=big, pairs=n) == 4
    assert ops.backward_blocks((16, 16), size=below, pairs=n) == 1
    assert ops.forward_waves((32, 16), size=big) == 4
    assert ops.backward_blocks((32, 16), size=big, pairs=n) == 8      # 2^23 tiles of 8 blocks
    assert ops.backward_blocks((8, 8), size=big, pairs=n) == 1


@pytest.mark.parametrize("tile", [(16, 16), (16, 8), (32, 16), (8, 8)])
def test_join_of_few_large_splats(tile):
    # a pair per 16 pixels of the tiles is the line; 8x8 tiles always go pixel by pixel
    size = (tile[0] * 10, tile[1] * 7)
    line = 3 * size[0] * size[1] // 16
    assert ops.join_many(tile, size, 3, line) == (tile != (8, 8))
    assert not ops.join_many(tile, size, 3, line + 1)
