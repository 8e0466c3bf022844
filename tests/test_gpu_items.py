"""Work items of the evaluation launch: the default item size and the distribution of items over waves (by
position for the workgroups the chip holds at once, the rest through the queues) at queue lengths from one
item to several per wave, ragged images included, against the oracle; the per-pair reduction over 1 to
many items."""
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


# (keyframes, height, width, copies of every ordered pair): 2 pairs of 4x4 (one item each), a ragged window,
# 8 items per queue and one more, about one item per wave, and several per wave
CASES = [(2, 4, 4, 1), (3, 7, 65, 1), (5, 37, 53, 1), (4, 60, 80, 40), (4, 24, 33, 700), (3, 121, 167, 500)]


@pytest.mark.parametrize("prec", ["F32", "F64"])
@pytest.mark.parametrize("n,H,W,copies", CASES)
def test_every_item_is_evaluated_once(pba, n, H, W, copies, prec):
    """Each pair record equals the oracle's: all source pixels counted, valid counts equal up to the points
    within 1e-4 px of a cell boundary (counted), F and b to 1e-5 of their scale (FP32 path; FP64 1e-9; both
    only where no such point exists); copies of a pair give the same bits wherever their items ran."""
    prob = synth.make("rgbd_small", H=H, W=W, n_kf=n)
    base = np.asarray(prob.pairs)
    pairs = np.tile(base, (copies, 1))
    ref = oracle.eval_pairs(prob, prob.init_poses)
    tol = 1e-9 if prec == "F64" else 1e-5
    with pba.context_for_problem(prob, precision=pba.PBA_F64 if prec == "F64" else pba.PBA_F32) as ctx:
        ctx.set_pairs(pairs)
        ev = ctx.evaluate(want_pairs=True)
        t = ctx.timings()
        again = ctx.evaluate(want_pairs=True)
    rec = ev["pairs"]
    assert np.array_equal(again["pairs"], rec)
    assert t["items_px"] % 64 == 0 and 64 <= t["items_px"] <= 4096
    assert t["n_items"] == len(pairs) * -(-H * W // t["items_px"])
    for c in range(copies):
        assert np.array_equal(rec[c * len(base):(c + 1) * len(base)], rec[:len(base)]), c
    for k in range(len(base)):
        assert int(rec[k, 157]) == ref["n_eval"][k]
        assert abs(int(rec[k, 158]) - ref["n_valid"][k]) <= rec[k, 159], k
        if rec[k, 159] == 0 and ref["n_valid"][k]:
            assert abs(rec[k, 156] - ref["F"][k]) <= tol * ref["F"][k]
            scale = np.abs(ref["H12"][k]).max()
            assert np.abs(rec[k, :144].reshape(12, 12) - ref["H12"][k]).max() <= tol * scale
