"""GPU: scorer training in one call of several steps (weights packed once, kept by each step) and in calls of one step
(weights gathered from the parameters): the same bits."""
import numpy as np
import pytest

from paper_1704_05132_amd.instances import workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vns():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1704_05132_amd import vns as v
    return v


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1100])
def test_steps_together_and_apart(vns, n):
    """Copies of one row: every order of a minibatch's rows is the same, whatever an epoch draws."""
    rng = np.random.default_rng(n)
    X, y = np.repeat(rng.random((1, 16)), n, 0).astype(np.float32), np.full(n, 0.7, np.float32)
    with vns.Context(workload("plain_10x12"), seed=3) as a, vns.Context(workload("plain_10x12"), seed=3) as b:
        last = a.mlp_train(X, y, 4, batch=n)
        apart = [b.mlp_train(X, y, 1, batch=n) for _ in range(4)]
        assert last == apart[-1] and len(set(apart)) == 4
        assert (a.mlp_get() == b.mlp_get()).all()
        (la, ga), (lb, gb) = a.mlp_grad(X, y), b.mlp_grad(X, y)
        assert la == lb and (ga == gb).all()
