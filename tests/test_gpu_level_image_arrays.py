"""The arrays of get_level_image are each one's own: keeping one keeps no other's memory (tiny, below and above 4 MB a
keyframe)."""
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


def _kept_bytes(a):
    """Bytes that stay allocated as long as `a` does."""
    while isinstance(a.base, np.ndarray):
        a = a.base
    return a.nbytes if a.base is None else memoryview(a.base).nbytes


# 20 bytes a pixel
@pytest.mark.parametrize("channels", [2, 5])
@pytest.mark.parametrize("H,W", [(8, 9), (452, 463), (459, 457)])
def test_each_array_keeps_its_own_memory(pba, H, W, channels):
    prob = synth.make("rgbd_small", H=H, W=W, n_kf=2)
    rng = np.random.default_rng(3)
    N = [rng.standard_normal((H, W, 3)).astype(np.float32) for _ in range(2)]
    images = (prob.intensity, prob.depth, N)
    with pba.context_for_problem(prob, channels=channels, images=images) as ctx:
        got = ctx.get_level_image(0, 1)
    valid = got[1] > 0
    assert valid.any()
    for a, b in zip(got[:2] if channels == 2 else got, images):
        assert np.array_equal(a[valid], b[1][valid])
    for i, a in enumerate(got):
        assert a.dtype == np.float32 and a.shape == ((H, W, 3) if i == 2 else (H, W))
        assert a.flags.writeable and a.flags.c_contiguous
        assert _kept_bytes(a) == a.nbytes
        a[...] = 0
