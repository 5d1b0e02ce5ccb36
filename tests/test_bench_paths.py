"""bench.py on a batch whose layers take both product paths: every stage keeps
its work, counted over its own layers, its rate is over the step's launches
together, and the longest stage is the one the roofline names.  No GPU needed."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2311_04406_amd.workloads import LayerSpec  # noqa: E402

BIG = LayerSpec("big", 512, 640, 512, 1, 1)        # products by residues
WIDE = LayerSpec("wide", 70, 100, 130, 2, 2)       # by digits
SKINNY = LayerSpec("skinny", 33, 70, 1, 3, 3)      # in the row pass
BATCH = [WIDE, BIG, SKINNY]
PATHS = [False, True, False]


def work(stage, mode="compact", **kw):
    return bench.batch_work(stage, BATCH, PATHS, mode, **kw)


def test_each_stage_counts_its_own_layers():
    for mode in ("compact", "spdz2k"):
        one = lambda stage, specs, **kw: bench.stage_work(stage, specs, mode, **kw)[1]
        assert work("ring_gemm", mode) == ("mfma", one("ring_gemm", [WIDE]))
        assert work("rns_gemm", mode) == ("mfma", one("rns_gemm", [BIG], rns=True))
        for stage in ("rns_open", "rns_fold"):
            assert work(stage, mode) == ("hbm", one(stage, [BIG], rns=True)) and work(stage, mode)[1] > 0
        assert work("rns_pack", mode)[1] == 0
        for stage in ("open_pack", "pack"):
            assert work(stage, mode) == ("hbm", one(stage, [WIDE, SKINNY]))
        for stage in ("row_pass", "open_u", "post"):
            assert work(stage, mode) == ("hbm", one(stage, [WIDE, SKINNY]) + one(stage, [BIG], rns=True))
    # E of a layer whose opening writes the planes is read back, the others' is opened in the pass
    assert work("row_pass")[1] == 80 * 512 * 640 + 160 * 70 * 100 + 144 * 33 * 70
    assert work("copy_base") is None and work("no_such_stage") is None


def test_one_path_only_is_the_batch_itself():
    for stage in ("ring_gemm", "open_pack", "pack", "row_pass", "post", "open_u"):
        assert bench.batch_work(stage, BATCH, [False] * 3, "compact") == bench.stage_work(stage, BATCH, "compact")
    for stage in ("rns_gemm", "rns_open", "rns_fold", "row_pass", "post"):
        assert bench.batch_work(stage, [BIG], [True], "compact") == bench.stage_work(stage, [BIG], "compact", rns=True)
    assert bench.batch_work("ring_gemm", [BIG], [True], "compact") is None
    assert bench.batch_work("rns_gemm", [WIDE], [False], "compact") is None


def test_rates_are_per_step_and_the_longest_stage_has_one():
    # 20 steps of 10 ms; the pass over M x K launched twice a step, the residue products by three groups
    stages = {"row_pass": (20 * 0.5, 40), "ring_gemm": (20 * 3.0, 20), "rns_gemm": (20 * 2.0, 60),
              "rns_open": (20 * 1.5, 60), "post": (20 * 1.0, 20), "zero_acc": (20 * 0.01, 20)}
    rows = bench.stage_figures(stages, work, 20, 10.0)
    assert rows["row_pass"]["launches"] == 40 and rows["row_pass"]["ms_per_launch"] == 0.25
    assert abs(rows["row_pass"]["achieved_GBps"] - work("row_pass")[1] / 0.5e-3 / 1e9) < 0.1
    assert abs(rows["rns_gemm"]["achieved_TOPS"] - work("rns_gemm")[1] / 2.0e-3 / 1e12) < 0.1
    assert rows["ring_gemm"]["share_of_step"] == 0.3
    timed = [k for k, v in rows.items() if "bound" in v]
    assert max(rows, key=lambda k: rows[k]["ms_per_launch"] * rows[k]["launches"]) == "ring_gemm" in timed
    assert "bound" not in rows["zero_acc"]
