"""Where launches switch from the grid (four workgroups per compute unit) to every workgroup that fits of their kernel:
1024 source pixels per wave, seen in the grid and the item size that the timings report, on both sides of the line;
the pair records agree across it up to the regrouping of their sums."""
import numpy as np
import pytest

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


def _pinhole():
    prob = synth.make("rgbd_small", H=64, W=96, n_kf=3)
    return prob, np.asarray(prob.pairs), 64 * 96, 6


def _spherical_to_pinhole():
    kfs = [0, 1, 2, 200, 201, 202, 203, 204]
    prob = synth.make("joint", H_l=32, W_l=256, H_c=60, W_c=80, kfs=kfs).subset(kfs)
    return prob, np.array([(s, t) for s in range(3) for t in range(3, 8)]), 32 * 256, 5


@pytest.mark.parametrize("scene", [_pinhole, _spherical_to_pinhole])
def test_the_switch(pba, scene):
    """FP32, two cues: the kernels that fit six and five workgroups per compute unit."""
    import torch
    prob, base, npx, per_cu = scene()
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    waves = {"grid": 4 * cu * 4, "full": per_cu * cu * 4}
    line = -(-1024 * waves["full"] // (len(base) * npx))   # copies of the pairs from which it is in full
    rec = {}
    with pba.context_for_problem(prob, channels=2, grad_mode=0) as ctx:
        for copies, launch in ((line - 1, "grid"), (line, "full")):
            ctx.set_pairs(np.tile(base, (copies, 1)))
            t = ctx.timings()
            assert t["grid"] == waves[launch] // 4, (copies, t)
            assert t["items_px"] == -(-(-(-copies * len(base) * npx // waves[launch])) // 64) * 64
            r = ctx.evaluate(want_pairs=True)["pairs"].reshape(copies, len(base), -1)
            assert np.array_equal(r, np.broadcast_to(r[:1], r.shape))
            rec[launch] = r[0]
    a, b = rec["grid"], rec["full"]
    assert np.array_equal(a[:, 157:], b[:, 157:]) and a[:, 158].sum() > 0
    # FP32 sums of 64 pixels in a tree: six roundings of 6e-8 on a path, so below 1e-6 of the largest entry
    for sl in (slice(0, 144), slice(144, 156), slice(156, 157)):
        assert (np.abs(a[:, sl] - b[:, sl]).max(1) <= 1e-6 * np.abs(a[:, sl]).max(1)).all()
