"""GPU: the paths that price by full decodes, against the oracle: products past the compact bounds (interval pricing takes
every other context without disposal) and the disposal reading.
"""
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


def test_best_of_at_the_edge_of_the_lds(vns):
    """Six workgroups of two wavefronts to a compute unit, each with the 15808 bytes of a 38 x 52 instance's rows."""
    inst = draw_instance(np.random.default_rng(1), 38, 52)
    inst.dispose = True
    with vns.Context(inst, seed=1, chains=96, options={vns.OPT_BEST_OF: 16, vns.OPT_RUN_WAVES: 2}) as ctx:
        ctx.run(3)
        for g in (0, 95):
            ref = oracle.BestOfChain(inst, 1, g, G=16)
            assert (ctx.trajectory(g) == ref.run(3)).all(), g
            zM, zR = ctx.solution(g)
            assert (zM == ref.zM).all() and (zR == ref.zR).all(), g
