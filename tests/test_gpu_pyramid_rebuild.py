"""A pyramid built again while one of its levels is active: iterations captured on the released planes are not replayed."""
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


@pytest.mark.parametrize("levels", [2, 3])
def test_iterations_after_a_rebuilt_pyramid(rgbd_small, pba, levels):
    rows = lambda log: [dict(r, ms=0) for r in log]
    with pba.context_for_problem(rgbd_small) as ctx:
        ctx.build_pyramid(levels)
        ctx.set_level(1)
        want = rows(ctx.iterate(2) + ctx.iterate(2))
        want_poses = ctx.get_poses()
    with pba.context_for_problem(rgbd_small) as ctx:
        ctx.build_pyramid(2)
        ctx.set_level(1)
        got = rows(ctx.iterate(2))
        keep = [pba.context_for_problem(rgbd_small)]   # other planes where the old ones were
        ctx.build_pyramid(levels)
        keep.append(pba.context_for_problem(rgbd_small))
        got += rows(ctx.iterate(2))
        assert got == want and np.array_equal(ctx.get_poses(), want_poses)
        for other in keep:
            other.close()
