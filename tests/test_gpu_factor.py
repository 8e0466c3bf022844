"""The blocked factorisation and the triangular solves at the sizes where their tiles end: systems of one block up to
exactly 60 and 64-row padding, the first with a second, nearly empty block (66 rows), several blocks with a
ragged last one, chains and densely coupled windows, in both elimination orders."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pba():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2303_16878_amd as pba
    pba.load_library()
    return pba


def _problem(n_kf, reach):
    prob = synth.make("rgbd_small", H=24, W=32, n_kf=n_kf)
    prob.pairs = np.array([(i, j) for i in range(n_kf) for j in range(n_kf) if i != j and abs(i - j) <= reach], np.int32)
    return prob


# 12, 60, 66, 126, 132, 192, 198 and 390 rows
@pytest.mark.parametrize("n_kf,reach", [(2, 1), (10, 9), (11, 10), (21, 2), (22, 21), (32, 1), (33, 4), (65, 3)])
@pytest.mark.parametrize("order", ["NATURAL", "ND", "AUTO"])
def test_step_equals_dense_solve(pba, n_kf, reach, order):
    """(H + lambda diag H) dx = -b with the anchor fixed: the residual is rounding-sized (1e-10 of |b|, far above
    n eps cond-free backward error n * 2e-16) and the step equals numpy's dense solve to 1e-8."""
    prob = _problem(n_kf, reach)
    with pba.context_for_problem(prob, precision=pba.PBA_F64, solve_order=getattr(pba, "PBA_ORDER_" + order)) as ctx:
        ev = ctx.evaluate(want_system=True)
        for lam in (1e-3, 1e-1):
            dx = ctx.solve_step(lam)
            H, b = oracle.gauge_fix(ev["H"], ev["b"], 0)
            A = H + lam * np.diag(np.diag(H))
            ref = np.linalg.solve(A, -b)
            assert np.all(dx[:6] == 0.0)
            assert np.abs(A @ dx + b).max() <= 1e-10 * np.abs(b).max(), lam
            assert np.linalg.norm(dx - ref) <= 1e-8 * np.linalg.norm(ref), lam


@pytest.mark.parametrize("n_kf", [5, 11, 33])
def test_not_positive_definite_is_reported_and_recovered(pba, n_kf):
    """A keyframe without any correspondence leaves zero rows: the undamped system is refused, in one block and in
    several, and the context solves again once the pairs are back."""
    prob = _problem(n_kf, 2)
    with pba.context_for_problem(prob, precision=pba.PBA_F64) as ctx:
        ctx.set_pairs([p for p in prob.pairs if n_kf - 1 not in p])
        with pytest.raises(pba.PbaError) as e:
            ctx.solve_step(0.0)
        assert e.value.status == pba.PBA_ENOTPD
        with pytest.raises(pba.PbaError):
            ctx.iterate(1, use_lm=False)
        ctx.set_pairs(prob.pairs)
        ev = ctx.evaluate(want_system=True)
        dx = ctx.solve_step(1e-3)
        H, b = oracle.gauge_fix(ev["H"], ev["b"], 0)
        A = H + 1e-3 * np.diag(np.diag(H))
        assert np.abs(A @ dx + b).max() <= 1e-10 * np.abs(b).max()
