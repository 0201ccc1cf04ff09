"""GPU: options changed between the runs of one context, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1704_05132_amd.instances import draw_instance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vns():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1704_05132_amd import vns as v
    return v


@pytest.mark.parametrize("form", ["plain", "one wavefront", "spec_iters", "full decode", "speculative vnd"])
@pytest.mark.parametrize("K,T,low", [(10, 12, 3), (3, 40, 1), (6, 70, 5)])
def test_k_max_lowered_below_a_chains_k(vns, K, T, low, form):
    """The next shake still takes the chain's k flips, though it is above the new k_max."""
    opts = {"plain": {}, "one wavefront": {vns.OPT_RUN_WAVES: 1}, "spec_iters": {vns.OPT_SPEC_ITERS: 4, vns.OPT_RUN_WAVES: 4},
            "full decode": {vns.OPT_LOG: 16}, "speculative vnd": {vns.OPT_SPECULATE: 1}}[form]
    inst = draw_instance(np.random.default_rng([K, T, 21]), K, T)
    with vns.Context(inst, seed=1, chains=4, k_max=64, options=opts) as ctx:
        chains = [oracle.Chain(inst, 1, g, k_max=64) for g in range(4)]
        for n, k_max in ((45, 64), (20, low)):
            ctx.set_option(vns.OPT_KMAX, k_max)
            for c in chains:
                c.k_max = k_max
            assert n == 45 or any(c.k > k_max for c in chains)
            ctx.run(n)
            for g, c in enumerate(chains):
                assert (ctx.trajectory(g) == c.run(n)).all(), g
                zM, zR = ctx.solution(g)
                assert (zM == c.zM).all() and (zR == c.zR).all(), g


@pytest.mark.parametrize("form", ["intervals", "full decode"])
def test_k_max_lowered_below_the_kept_k(vns, form):
    """Best of G as printed keeps k: every later shake takes as many flips, whatever k_max has become."""
    inst = draw_instance(np.random.default_rng([10, 12, 22]), 10, 12)
    inst.dispose = form == "full decode"
    with vns.Context(inst, seed=1, chains=4, k_max=64) as ctx:
        ref = [oracle.Chain(inst, 1, g, k_max=64) for g in range(4)]
        ctx.run(45)
        for c in ref:
            c.run(45)
        assert any(c.k > 5 for c in ref)
        ctx.set_option(vns.OPT_KMAX, 2)
        ctx.set_option(vns.OPT_BEST_OF, 3)
        ctx.set_option(vns.OPT_BEST_OF_LITERAL, 1)
        ctx.run(12)
        for g, c in enumerate(ref):
            b = oracle.BestOfChain(inst, 1, g, k_max=2, G=3, literal=True)
            b.zM, b.zR, b.k, b.it, b.F, b.F_best = c.zM, c.zR, c.k, c.it, c.F, c.F_best
            assert (ctx.trajectory(g) == b.run(12)).all(), g
            zM, zR = ctx.solution(g)
            assert (zM == b.zM).all() and (zR == b.zR).all(), g


def test_whether_interval_pricing_applies(vns):
    inst = draw_instance(np.random.default_rng(3), 4, 20)
    with vns.Context(inst, seed=1) as ctx:
        assert ctx.get_option(vns.OPT_INTERVAL) == 1
        for value in (0, 1):
            with pytest.raises(vns.VNSError) as e:
                ctx.set_option(vns.OPT_INTERVAL, value)
            assert e.value.status == vns.VNS_EINVAL
        for reading, applies in ((vns.DECODE_DISPOSE, 0), (vns.DECODE_STRICT, 1), (3, 0), (0, 1)):
            ctx.set_option(vns.OPT_DECODE, reading)
            assert ctx.get_option(vns.OPT_INTERVAL) == applies
        ctx.set_unit_costs(np.full(4, 60000), np.zeros(4))   # some 2000 units at 60000: still below 2^31
        assert ctx.get_option(vns.OPT_INTERVAL) == 1
    inst.kM[2] = 200_000_000   # twenty setups: 4e9
    with vns.Context([inst, draw_instance(np.random.default_rng(4), 3, 12)], seed=1) as ctx:
        assert ctx.get_option(vns.OPT_INTERVAL) == 0
