"""pba_apply_step without a step given applies the last solved one: the poses equal those of the step handed back."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pba():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2303_16878_amd as pba
    pba.load_library()
    return pba


def _applied(pba, prob, between=None, **kw):
    """(poses of the solved step as kept, poses of the step as handed back)"""
    X = []
    for explicit in (False, True):
        with pba.context_for_problem(prob, precision=pba.PBA_F64, **kw) as ctx:
            dx = ctx.solve_step(1e-3)
            assert np.abs(dx).max() > 0
            if between:
                between(ctx)
            ctx.apply_step(dx if explicit else None)
            X.append(ctx.get_poses())
    return X


def test_a_loss_evaluated_in_between(rgbd_small, pba):
    """A line search: solve, look at the loss elsewhere, then take the step."""
    delta = np.full((rgbd_small.n, 6), 1e-3, np.float32)
    kept, given = _applied(pba, rgbd_small, between=lambda ctx: ctx.loss_forward(delta))
    assert np.array_equal(kept, given)
