"""Autotuner selection and persistence (CPU only: the measurement is injected)."""
import numpy as np

from paper_1704_05132_amd import autotune
from paper_1704_05132_amd.instances import draw_instance


def test_pick_returns_fastest_and_all_timings():
    times = {2: 5.0, 4: 3.0, 8: 3.0}
    best, timings = autotune.pick([dict(waves=w) for w in (2, 4, 8)], lambda c: times[c["waves"]])
    assert best == {"waves": 4}               # ties keep the earlier candidate
    assert [ms for _, ms in timings] == [5.0, 3.0, 3.0]


def test_signature_distinguishes_workloads():
    rng = np.random.default_rng(1)
    a = [draw_instance(rng, 10, 12), draw_instance(rng, 30, 52)]
    b = [draw_instance(rng, 10, 12), draw_instance(rng, 30, 24)]
    assert autotune.signature(a, 8) == "n2_K10-30_T12-52_c8"
    assert autotune.signature(a, 8) != autotune.signature(b, 8)
    assert autotune.signature(a, 8) != autotune.signature(a, 16)


def test_table_round_trip(tmp_path):
    t = autotune.TuneTable(tmp_path / "tune.json")
    assert t.get("k") is None
    t.put("k", {"waves": 4, "lds": 0}, [({"waves": 4, "lds": 0}, 1.5)])
    t2 = autotune.TuneTable(tmp_path / "tune.json")
    assert t2.get("k")["choice"] == {"waves": 4, "lds": 0}
    assert t2.get("k")["timings_ms"] == [[{"waves": 4, "lds": 0}, 1.5]]


def test_search_options_map_every_key():
    from paper_1704_05132_amd import vns
    assert autotune.search_options(dict(waves=4, lds=0, spec=0)) == {vns.OPT_RUN_WAVES: 4, vns.OPT_RUN_LDS: 0,
                                                                      vns.OPT_SPECULATE: 0}
    assert autotune.search_options(dict(spec=1, spec_waves=9, lds=65536)) == {vns.OPT_SPECULATE: 1,
                                                                               vns.OPT_SPEC_WAVES: 9,
                                                                               vns.OPT_RUN_LDS: 65536}
    assert autotune.search_options({"group": 8}) == {}
    assert autotune.search_options(dict(waves=2, state=1)) == {vns.OPT_RUN_WAVES: 2, vns.OPT_STATE_LDS: 1}
    assert autotune.search_options(dict(waves=4, iters=6)) == {vns.OPT_RUN_WAVES: 4, vns.OPT_SPEC_ITERS: 6}


def test_eval_options_map_group_and_spread():
    from paper_1704_05132_amd import vns
    assert autotune.eval_options({"group": 5}) == {vns.OPT_EVAL_SPREAD: 0, vns.OPT_EVAL_GROUP: 5}
    assert autotune.eval_options({"spread": 8}) == {vns.OPT_EVAL_SPREAD: 8}
    assert autotune.eval_options(dict(waves=4, iters=12)) == {vns.OPT_EVAL_SPREAD: 0}
    assert {c.get("spread") for c in autotune.EVAL_CANDIDATES} >= {4, 8, 12, 16}


def test_candidates_cover_both_search_kernels():
    kinds = {c.get("spec", 0) for c in autotune.SEARCH_CANDIDATES}
    assert kinds == {0, 1}
    for c in autotune.SEARCH_CANDIDATES:
        if c.get("spec"):
            assert c["spec_waves"] % 3 == 0 and 3 <= c["spec_waves"] <= 16   # whole groups of three waves
            assert "iters" not in c   # speculative iterations run the one-wavefront-per-product VND
        assert 1 <= c.get("iters", 1) <= 16
    assert any(c.get("iters", 1) > 1 for c in autotune.SEARCH_CANDIDATES)


class PricingContext:
    """What tune_eval uses of a context."""

    def __init__(self, vns, interval, options={}):
        self.ms = iter([0.9, 0.5] * 1000)   # whatever is set, the times differ
        self.options = {vns.OPT_INTERVAL: interval, vns.OPT_EVAL_SPREAD: 0, vns.OPT_EVAL_GROUP: 4, **options}

    def get_option(self, key):
        return self.options[key]

    def set_option(self, key, value):
        self.options[key] = value

    def eval_neighbourhood(self, nb_mask, chain, slot_prices):
        pass

    def stats(self):
        return {"last_eval_ms": next(self.ms)}


def test_tune_eval_keeps_the_choice_of_interval_pricing():
    from paper_1704_05132_amd import vns
    for options, choice in (({}, {"group": 4}), ({vns.OPT_EVAL_SPREAD: 8}, {"spread": 8})):
        ctx = PricingContext(vns, 1, options)
        best, timings = autotune.tune_eval(ctx, reps=1)
        assert best == choice and [c for c, _ in timings] == [choice]
        assert ctx.get_option(vns.OPT_EVAL_SPREAD) == choice.get("spread", 0)
        assert ctx.get_option(vns.OPT_EVAL_GROUP) == 4


def test_tune_eval_times_every_shape_of_the_full_decode():
    from paper_1704_05132_amd import vns
    best, timings = autotune.tune_eval(PricingContext(vns, 0), reps=1)
    assert [c for c, _ in timings] == autotune.EVAL_CANDIDATES
    assert best == autotune.EVAL_CANDIDATES[1]   # the first of the fastest
