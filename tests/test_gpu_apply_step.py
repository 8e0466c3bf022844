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


def _lidar(n_kf):
    import synth
    return synth.make("lidar128", kfs=range(n_kf), H=16, W=256).subset(range(n_kf))


@pytest.mark.parametrize("order", ["AUTO", "ND", "NATURAL"])
@pytest.mark.parametrize("n_kf", [3, 40, 120])
def test_every_solve_order(pba, order, n_kf):
    """A nested-dissection solve keeps its step in its own padded order (240 and 720 rows: several blocks)."""
    kept, given = _applied(pba, _lidar(n_kf), solve_order=getattr(pba, "PBA_ORDER_" + order))
    assert np.array_equal(kept, given)


@pytest.mark.parametrize("order", ["ND", "NATURAL"])
@pytest.mark.parametrize("graph", [False, True])
def test_after_steps_of_the_other_kinds(pba, order, graph):
    """An applied step, then iterations (a replayed graph included), then a solve: always the last one."""
    prob = _lidar(40)
    rng = np.random.default_rng(2)

    def between(ctx):
        ctx.iterate(1)
        ctx.apply_step(1e-5 * rng.standard_normal(6 * ctx.n_poses))
        ctx.iterate(1)

    for last in ("solve", "iterate"):
        X = []
        for explicit in (False, True):
            rng = np.random.default_rng(2)
            with pba.context_for_problem(prob, precision=pba.PBA_F64, solve_order=getattr(pba, "PBA_ORDER_" + order),
                                         use_graph=graph) as ctx:
                between(ctx)
                if last == "solve":
                    dx = ctx.solve_step(1e-3)
                else:   # the step of one Gauss-Newton iteration, solved ahead where the system is the same
                    dx = ctx.solve_step(0.0)
                    ctx.apply_step(np.zeros(6 * ctx.n_poses))
                    ctx.iterate(1)
                ctx.apply_step(dx if explicit else None)
                X.append(ctx.get_poses())
        assert np.abs(X[0] - X[1]).max() <= 1e-12, last


def test_no_step_solved(pba, rgbd_small):
    """Nothing to apply before a solve, nor once the plan it was laid out for is gone."""
    with pba.context_for_problem(rgbd_small, solve_order=pba.PBA_ORDER_ND) as ctx:
        for prepare in (lambda: None, lambda: (ctx.solve_step(1e-3), ctx.set_pairs(rgbd_small.pairs[:8]))):
            prepare()
            with pytest.raises(pba.PbaError) as e:
                ctx.apply_step()
            assert e.value.status == pba.PBA_ESTATE
