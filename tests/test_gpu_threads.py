"""GPU: threads that read one context side by side, while another prices its solutions."""
import threading

import numpy as np
import pytest

from paper_1704_05132_amd.instances import draw_instance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vns():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1704_05132_amd import vns as v
    return v


def test_readers_beside_a_pricing_thread(vns):
    chains, reps = 6, 60
    with vns.Context(draw_instance(np.random.default_rng(8), 40, 52), seed=2, chains=chains) as ctx:
        ctx.run(40)
        sols = [ctx.solution(g) for g in range(chains)]
        recs = [ctx.trajectory(g) for g in range(chains)]
        F = ctx.costs()
        priced = [ctx.eval_neighbourhood(7, g) for g in range(chains)]
        wrong, start = [], threading.Barrier(4)

        def reading(what):
            start.wait()
            for i in range(reps):
                g = i % chains
                if what == "solution":
                    ok = all((a == b).all() for a, b in zip(ctx.solution(g), sols[g]))
                elif what == "trajectory":
                    ok = (ctx.trajectory(g) == recs[g]).all()
                elif what == "costs":
                    ok = all((a == b).all() for a, b in zip(ctx.costs(), F))
                else:
                    got = ctx.eval_neighbourhood(7, g)
                    ok = all((got[k] == priced[g][k]).all() for k in got)
                if not ok:
                    wrong.append((what, i))

        threads = [threading.Thread(target=reading, args=(w,)) for w in ("solution", "trajectory", "costs", "prices")]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong, wrong[:4]
