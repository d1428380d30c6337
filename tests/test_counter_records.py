"""The committed counter records (no GPU): they name the command they were taken on, hold dispatches
of their plan only, and the tools that write them leave out what ran before the steps."""
import csv
import json
import math
import os

import pytest

from paper_2509_12138_amd import kcounters, ops, traffic

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2509_12138_amd")


@pytest.mark.parametrize("name", ["kernel_counters.json", "hbm_traffic.json"])
def test_records_name_their_command(name):
    with open(os.path.join(PKG, name)) as f:
        table = json.load(f)
    assert table
    for key, e in table.items():
        assert "bench.py" in e["command"], key
        assert key == f"{e['kernel']}|{e['plan']}"
        tile, sched, chunk, waves, _ = e["plan"].split(",")
        tile = tuple(int(x) for x in tile.split("x"))
        assert int(waves) == ops.forward_waves(tile, sched, int(chunk), int(waves)), key


def test_forward_record_is_of_one_launch():
    # 1920x1080: every dispatch has the plan's waves for each tile, none of another order's rounding
    with open(os.path.join(PKG, "kernel_counters.json")) as f:
        e = json.load(f)["k_raster_fwd<16, 16, 4>|16x16,lpt,64,4,0"]
    assert e["SQ_WAVES"] == math.ceil(1920 / 16) * math.ceil(1080 / 16) * 4


def _write(path, head, rows):
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(head)
        w.writerows(rows)


def test_dispatches_before_the_steps_are_left_out(tmp_path):
    names = ["gsmi::k_raster_fwd<16, 16, 4>(gsmi::RasterDev)", "void gsmi::k_ssim<true>(float*)",
             "gsmi::k_raster_fwd<16, 16, 4>(gsmi::RasterDev)"]
    _write(tmp_path / "a_kernel_trace.csv", ["Dispatch_Id", "Start_Timestamp", "End_Timestamp"],
           [[i + 1, 0, 1000 * (i + 1)] for i in range(3)])
    _write(tmp_path / "a_counter_collection.csv",
           ["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"],
           [[i + 1, n, "SQ_WAVES", 10.0 * (i + 1)] for i, n in enumerate(names)])
    k = "k_raster_fwd<16, 16, 4>"
    every = kcounters.summarise([kcounters.load_run(tmp_path)], [k])[k]
    steps = kcounters.summarise([kcounters.load_run(tmp_path, "k_ssim")], [k])[k]
    assert every["dispatches"] == 2 and every["SQ_WAVES"] == 20.0
    assert steps["dispatches"] == 1 and steps["SQ_WAVES"] == 30.0 and steps["mean_us"] == 3.0
    path = tmp_path / "a_counter_collection.csv"
    assert traffic.counter_kib(path, k, "SQ_WAVES") == (20.0, 2)
    assert traffic.counter_kib(path, k, "SQ_WAVES", "k_ssim") == (30.0, 1)
    with pytest.raises(SystemExit):
        kcounters.load_run(tmp_path, "k_missing")
