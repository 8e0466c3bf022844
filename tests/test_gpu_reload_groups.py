"""New images of a loaded keyframe set keep its pose groups, in the context and in the binding's array sizes."""
import numpy as np
import pytest

import synth
from test_gpu_failed_alloc import LARGE, _images, _loaded, _out_of_memory, _poses, pba  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def test_same_set_keeps_the_groups(pba):  # noqa: F811
    import torch
    rig = synth.make("rig_pair")
    with pba.context_for_problem(rig) as ctx:
        n_poses = ctx.n_poses
        assert n_poses < rig.n
        a = ctx.evaluate(want_system=True)
        ctx.load_keyframes(rig.kf_sensor, rig.intensity, rig.depth, rig.normals)
        assert ctx.n_poses == n_poses and ctx.get_poses().shape == (n_poses, 12)
        b = ctx.evaluate(want_system=True)
        assert b["H"].shape == (6 * n_poses, 6 * n_poses) and np.array_equal(a["H"], b["H"])
        # the loss reads the images anew on every call
        images = [torch.tensor(x, device="cuda") for l in (rig.intensity, rig.depth, rig.normals) for x in l]
        delta = torch.zeros((n_poses, 6), device="cuda", requires_grad=True)
        pba.photometric_loss(ctx, delta, images).backward()
        assert delta.grad.shape == (n_poses, 6) and bool(torch.isfinite(delta.grad).all())


def test_another_set_and_a_failed_load_end_them(pba):  # noqa: F811
    for retry in (False, True):
        with _loaded(pba, LARGE, 3, [0, 0, 1]) as ctx:
            assert ctx.n_poses == 2
            load = lambda n: ctx.load_keyframes([LARGE] * n, *_images(LARGE, n), None)
            if retry:   # the same set, but the first attempt gives the loaded one up
                assert _out_of_memory(pba, lambda: load(3), 0)
                load(3)
            else:
                load(4)
            assert ctx.n_poses == ctx.n
            ctx.set_poses(_poses(ctx.n))
