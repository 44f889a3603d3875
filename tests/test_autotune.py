"""The autotuner's cache logic (host only) and, on the GPU, that every update plan it
chooses among gives the oracle's counters and that a tuned plan round-trips."""
import json

import numpy as np
import pytest

import oracle
import paper_1711_00975_amd as csk
from paper_1711_00975_amd import autotune


def test_cache_round_trip_and_classes(tmp_path):
    path = str(tmp_path / "tune.json")
    t = autotune.Tuner(path, device="dev-A")
    assert autotune.size_class(1 << 16, 70_000) == "w16_n16"
    assert autotune.size_class(1 << 20, 1) == "w20_n0"
    t.record("w16_n16", {"mode": csk.CSK_UPDATE_DIRECT, "max_wg": 0, "ms": 0.1})
    t.save()
    t2 = autotune.Tuner(path, device="dev-A")
    assert t2.lookup("w16_n16")["mode"] == csk.CSK_UPDATE_DIRECT
    assert autotune.Tuner(path, device="dev-B").lookup("w16_n16") is None   # keyed by device
    assert json.load(open(path))["dev-A"]["w16_n16"]["max_wg"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("plan", autotune.UPDATE_CANDIDATES + [autotune._plan(csk.CSK_UPDATE_AUTO)],
                         ids=autotune.plan_key)
def test_every_update_plan_matches_oracle(plan):
    # the plans differ only in speed: the counters are the same +-1 sums (Sec. 2.2 Add)
    from test_gpu_parity import clustered, dev
    for w in (1 << 16, 1 << 20):
        pos = clustered(120_000, 100.0, 5)
        s = csk.Sketch(5, w, 3)
        autotune.set_plan(s, plan)
        s.update(dev(pos), 0.1, 100.0)
        Mo, _ = oracle.sketch(pos, 5, w, 3, 0.1, 100.0, threads=8)
        assert np.array_equal(s.counters().cpu().numpy(), Mo), w
        s.close()


def test_old_cache_entries_still_apply(tmp_path):
    # a plan cached before the tiling axes (mode and max_wg only) keys and applies as before
    t = autotune.Tuner(str(tmp_path / "tune.json"), device="dev-A")
    t.record("w14_n16", {"mode": csk.CSK_UPDATE_BINNED, "max_wg": 64, "ms": 0.2})
    assert autotune.plan_key(autotune._plan(csk.CSK_UPDATE_BINNED, 64)) == "1:64:0:0:0:0"
    assert t.lookup("w14_n16")["max_wg"] == 64


@pytest.mark.gpu
def test_tuner_end_to_end(tmp_path):
    t = autotune.Tuner(str(tmp_path / "tune.json"))
    plan = t.tune_update(5, 1 << 20, 300_000, reps=2)
    keys = [autotune.plan_key(p) for p in autotune.UPDATE_CANDIDATES]
    assert autotune.plan_key(plan) in keys
    assert set(plan["all_ms"]) <= set(keys) and len(plan["all_ms"]) >= 5
    t.save()
    s = csk.Sketch(5, 1 << 20, 9)
    assert autotune.Tuner(str(tmp_path / "tune.json")).apply(s, 300_000)
    s.close()


class _Plans:
    """Stands in for a sketch: the plan set on it."""
    def __init__(self, d, w):
        self.d, self.w, self.plan = d, w, None

    def set_update_plan(self, mode, max_wg):
        self.plan = (mode, max_wg)

    def set_update_tiling(self, *tiling):
        self.plan += tiling


def test_plans_chosen_among_other_kernels_are_not_used(tmp_path):
    # a cache written before entries said what they were chosen among, and one of other candidates
    path = str(tmp_path / "tune.json")
    stale = dict(autotune._plan(csk.CSK_UPDATE_BINNED, 256, csk.CSK_BIN_GENERAL), ms=0.1)
    cls = autotune.size_class(1 << 20, 1 << 24, 5)
    with open(path, "w") as f:
        json.dump({"dev-A": {cls: stale, "w20_n24": stale, "batch_d5_m2_n20": dict(stale, wg_budget=256),
                             "w16_n16_d5": dict(stale, plans="0-other")}}, f)
    t = autotune.Tuner(path, device="dev-A")
    for c in (cls, "w20_n24", "batch_d5_m2_n20", "w16_n16_d5"):
        assert t.lookup(c) is None
    s = _Plans(5, 1 << 20)
    assert not t.apply(s, 1 << 24) and s.plan is None
    assert t.batch_budget([s, s], [1 << 19, 1 << 19]) == 0 and s.plan is None


def test_plans_are_kept_by_their_rows(tmp_path):
    path = str(tmp_path / "tune.json")
    t = autotune.Tuner(path, device="dev-A")
    t.record(autotune.size_class(1 << 16, 70_000, 5), autotune._plan(csk.CSK_UPDATE_DIRECT))
    t.save()
    t = autotune.Tuner(path, device="dev-A")
    five, eight = _Plans(5, 1 << 16), _Plans(8, 1 << 16)
    assert t.apply(five, 70_000) and five.plan[0] == csk.CSK_UPDATE_DIRECT
    assert not t.apply(eight, 70_000) and eight.plan is None
