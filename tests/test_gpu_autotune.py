"""pba_autotune against the default work items and grid: the default is one of the points it measures, so what it keeps is
no slower a point than that, and what it kept ends with the pairs it was measured for."""
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


def _point(ctx):
    t = ctx.timings()
    return t["items_px"], t["grid"]


# copies of the 6 pairs of 64x96: default sizes of 64, 320 (not in the tuner's list) and 1536 source pixels, and
# the full grid
@pytest.mark.parametrize("copies", [1, 30, 170, 171])
def test_the_default_is_a_point(pba, copies):
    prob = synth.make("rgbd_small", H=64, W=96, n_kf=3)
    pairs = np.tile(np.asarray(prob.pairs), (copies, 1))
    with pba.context_for_problem(prob) as ctx:
        ctx.set_pairs(pairs)
        a = ctx.evaluate()
        default = _point(ctx)
        pts = {(p, g): ms for p, g, ms in ctx.autotune()}
        kept = _point(ctx)
        print("copies", copies, "default", default, pts.get(default), "kept", kept, pts.get(kept), flush=True)
        assert len(pts) == 18 and default in pts
        assert pts[kept] == min(pts.values())
        b = ctx.evaluate()
        assert b["n_valid"] == a["n_valid"] and abs(b["F"] - a["F"]) <= 1e-12 * a["F"]
        ctx.set_pairs(pairs)
        assert _point(ctx) == default


def test_a_tuned_size_is_kept_for_its_level(pba):
    prob = synth.make("rgbd_small", H=64, W=96, n_kf=3)
    with pba.context_for_problem(prob) as ctx:
        ctx.build_pyramid(2)
        ctx.set_level(1)
        level1 = _point(ctx)
        ctx.set_level(0)
        ctx.autotune()
        kept = _point(ctx)
        ctx.set_level(1)
        assert _point(ctx) == level1
        ctx.set_level(0)
        assert _point(ctx) == kept
        ctx.load_keyframes(prob.kf_sensor, prob.intensity, prob.depth)
        assert _point(ctx) == kept
