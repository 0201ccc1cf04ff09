"""GPU: interval pricing (vns_interval.hpp) against the oracle, at the sizes where its lane groups change (16, 31
and 63 periods), at the ends of the horizon's range, with (chain, product) counts that leave lane groups without a
pair, under both carry-back readings, with the first manufacturing setup late, and on both sides of the bounds that
make a product compact.  All results are whole numbers and must be equal.
"""
import numpy as np
import pytest

import oracle
from paper_1704_05132_amd.instances import draw_instance, edge_instance

pytestmark = pytest.mark.gpu

HORIZONS = (1, 2, 3, 12, 15, 16, 17, 24, 31, 32, 33, 52, 63, 64, 65, 104, 127, 128)


@pytest.fixture(scope="module")
def vns():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1704_05132_amd import vns as v
    return v


def solution(inst, rng, p_m, p_r):
    """A feasible random solution: setups of products that it leaves infeasible become every period manufacturing."""
    zM = (rng.random((inst.K, inst.T)) < p_m).astype(np.uint8)
    zR = (rng.random((inst.K, inst.T)) < p_r).astype(np.uint8)
    _, cost = oracle.objective(inst, zM, zR)
    bad = cost == oracle.INF
    zM[bad], zR[bad] = 1, 0
    return zM, zR


def check(vns, inst, rng, mask=7, options=None, chains=3):
    sols = []
    with vns.Context(inst, seed=1, chains=chains, options=options or {}) as ctx:
        for g, (pm, pr) in enumerate([(0.3, 0.3), (0.1, 0.6), (0.6, 0.15)][:chains]):
            sols.append(solution(inst, rng, pm, pr))
            ctx.set_solution(g, *sols[-1])
        got = ctx.eval_neighbourhood(mask)
        evals = ctx.stats()["last_eval_evals"]
    n, total = 4 * inst.K * inst.T, 0
    for g, (zM, zR) in enumerate(sols):
        ref, cnt = oracle.price_all(inst, zM, zR, mask)
        total += cnt
        mine = got["slot_price"][g * n:(g + 1) * n]
        assert (mine == ref).all(), (g, np.flatnonzero(mine != ref)[:8])
        per = ref.reshape(inst.K, -1)
        assert (got["prod_best"][g * inst.K:(g + 1) * inst.K] == per.min(1)).all()
        assert (got["prod_best_slot"][g * inst.K:(g + 1) * inst.K] ==
                np.where(per.min(1) == oracle.INF, -1, per.argmin(1))).all()
        assert (int(got["best"][g]), int(got["best_slot"][g])) == oracle.argmin(ref)
    assert evals == total


@pytest.mark.parametrize("strict", [False, True])
@pytest.mark.parametrize("T", HORIZONS)
def test_horizons(vns, T, strict):
    rng = np.random.default_rng([T, strict])
    for kind in ("uniform", "sparse", "big_returns", "no_returns", "zero_demand", "returns_eq_demand"):
        inst = edge_instance(kind, 7, T, seed=T)
        inst.strict = strict
        inst.pM, inst.pR = rng.integers(0, 30, 7).astype(np.int32), rng.integers(0, 30, 7).astype(np.int32)
        check(vns, inst, rng)


@pytest.mark.parametrize("mask", [1, 2, 4, 3, 5, 6])
@pytest.mark.parametrize("T", [12, 24, 52, 104])
def test_masks(vns, T, mask):
    rng = np.random.default_rng([T, mask])
    check(vns, draw_instance(rng, 5, T), rng, mask)


@pytest.mark.parametrize("strict", [False, True])
@pytest.mark.parametrize("T", [14, 30, 60, 100])
def test_first_setup_late(vns, T, strict):
    """No demand in the first third: setups there may be missing or remanufacture only."""
    rng = np.random.default_rng([T, 9, strict])
    inst = edge_instance("big_returns", 9, T, seed=3)
    inst.strict = strict
    inst.D[:, :T // 3] = 0
    check(vns, inst, rng)


@pytest.mark.parametrize("scale", [1.0, 1.001])
@pytest.mark.parametrize("T", [12, 40, 90])
def test_compact_bounds(vns, T, scale):
    """Demand and returns that sum to just under 2^23 (interval pricing) and just over it (the full decode)."""
    rng = np.random.default_rng([T, int(scale * 1000)])
    inst = draw_instance(rng, 5, T)
    for a in (inst.D, inst.R):
        w = rng.random((5, T)) + 1e-3
        a[:] = np.floor(w / w.sum(1, keepdims=True) * (2**23 - 1) * scale).astype(np.int32)
    inst.hM[:] = rng.integers(1, 3, 5) if T < 50 else 1
    inst.hR[:] = rng.integers(0, 2, 5)
    check(vns, inst, rng)


SEARCHES = [dict(), dict(run_waves=1), dict(run_waves=2, memo=1), dict(run_waves=4, spec=4), dict(run_waves=2, state=0, lds=0)]


def options_of(vns, form):
    keys = dict(memo=vns.OPT_VND_MEMO, spec=vns.OPT_SPEC_ITERS, state=vns.OPT_STATE_LDS, lds=vns.OPT_RUN_LDS,
                run_waves=vns.OPT_RUN_WAVES)
    return {keys[k]: v for k, v in form.items()}


@pytest.mark.parametrize("form", range(len(SEARCHES)))
@pytest.mark.parametrize("T", [1, 2, 16, 33, 63, 64, 65, 128])
def test_search_horizons(vns, T, form):
    """Records and solutions of the interval search at the edges of its lane forms, against the oracle; its counts against
    the full-decode search (the one that keeps a move log)."""
    inst = draw_instance(np.random.default_rng([T, 5]), 6, T)
    for nb, strict in (((1, 2, 4), False), ((4, 1), True), ((2, 2, 4, 1), False)):
        inst.strict = strict
        memo = SEARCHES[form].get("memo", 0)
        with vns.Context(inst, seed=7, chains=2, nb_list=nb, options=options_of(vns, SEARCHES[form])) as ctx, \
                vns.Context(inst, seed=7, chains=2, nb_list=nb, options={vns.OPT_LOG: 16, vns.OPT_VND_MEMO: memo}) as full:
            chains = [oracle.Chain(inst, 7, g, nb) for g in range(2)]
            for n in (5, 20):   # the second run starts from known local optima
                ctx.run(n)
                full.run(n)
                for g, c in enumerate(chains):
                    assert (ctx.trajectory(g) == c.run(n)).all(), (nb, g)
                    zM, zR = ctx.solution(g)
                    assert (zM == c.zM).all() and (zR == c.zR).all()
                assert ctx.stats()["last_run_evals"] == full.stats()["last_run_evals"]


@pytest.mark.parametrize("T", [12, 52, 104])
def test_search_after_a_change_of_the_list(vns, T):
    """Solutions found under one list need not be local optima of another: nothing known of them may be used.  (Both
    searches go on with the shaken products only, so the full-decode one is the reference, not the oracle.)"""
    inst = draw_instance(np.random.default_rng([T, 6]), 8, T)
    with vns.Context(inst, seed=3, chains=3, nb_list=(1,)) as ctx, \
            vns.Context(inst, seed=3, chains=3, nb_list=(1,), options={vns.OPT_LOG: 16}) as full:
        for nb in ((1,), (1, 2, 4), (4, 2)):
            value = 0
            for i, b in enumerate(nb):
                value |= b << (4 * i)
            for c in (ctx, full):
                c.set_option(vns.OPT_NB_LIST, value)
                c.run(30)
            for g in range(3):
                assert (ctx.trajectory(g) == full.trajectory(g)).all(), (nb, g)
                assert all((x == y).all() for x, y in zip(ctx.solution(g), full.solution(g)))
            assert ctx.stats()["last_run_evals"] == full.stats()["last_run_evals"]


def test_searches_past_the_compact_bounds(vns):
    """Products past the 24-bit bounds search by full decodes; the records are the oracle's on both sides."""
    for scale in (0.999, 1.01):
        rng = np.random.default_rng(12)
        inst = draw_instance(rng, 4, 20)
        for a in (inst.D, inst.R):
            w = rng.random((4, 20)) + 1e-3
            a[:] = np.floor(w / w.sum(1, keepdims=True) * 2**23 * scale).astype(np.int32)
        inst.hM[:], inst.hR[:] = 2, 1
        with vns.Context(inst, seed=1, chains=2) as ctx:
            ctx.run(12)
            for g in range(2):
                assert (ctx.trajectory(g) == oracle.Chain(inst, 1, g).run(12)).all()


@pytest.mark.parametrize("strict", [False, True])
@pytest.mark.parametrize("K,T,k_max", [(1, 6, 8), (2, 12, 64), (3, 40, 5), (4, 128, 12)])
def test_shakes_that_meet_a_product_again(vns, K, T, k_max, strict):
    """More draws than products, and flips that leave a product infeasible (no demand early: setups may come late)."""
    inst = edge_instance("big_returns", K, T, seed=2)
    inst.strict = strict
    inst.D[:, :T // 3] = 0
    with vns.Context(inst, seed=5, chains=2, k_max=k_max, nb_list=(1, 2)) as ctx:
        chains = [oracle.Chain(inst, 5, g, (1, 2), k_max) for g in range(2)]
        for n in (3, 40):
            ctx.run(n)
            for g, c in enumerate(chains):
                assert (ctx.trajectory(g) == c.run(n)).all(), g
                zM, zR = ctx.solution(g)
                assert (zM == c.zM).all() and (zR == c.zR).all()


@pytest.mark.parametrize("n", [2048, 2049, 2080])
def test_best_of_many_chains(vns, n):
    """The best moves of more chains than a workgroup each takes, against one chain's call: the last sixteen of a launch
    and what is left over."""
    rng = np.random.default_rng(n)
    inst = draw_instance(rng, 3, 5)
    with vns.Context(inst, seed=1, chains=n) as ctx:
        for g in range(n):
            if g < 4 or g > n - 40:
                ctx.set_solution(g, *solution(inst, rng, 0.4, 0.4))
        got = ctx.eval_neighbourhood(7)
        for g in [0, 1, 2, 3, 15, 16, 17, 1000] + list(range(n - 39, n)):
            one = ctx.eval_neighbourhood(7, chain=g)
            assert (got["best"][g], got["best_slot"][g]) == (one["best"][0], one["best_slot"][0])
            assert (got["prod_best"][3 * g:3 * g + 3] == one["prod_best"]).all()
