"""Loading keyframes again after a load that ran out of device memory: the second attempt lays the planes out anew."""
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


def _images(H, W, n):
    rng = np.random.default_rng(H * W)
    depth = [np.full((H, W), 2.0, np.float32) + 0.01 * rng.random((H, W), dtype=np.float32) for _ in range(n)]
    return [rng.random((H, W), dtype=np.float32) for _ in range(n)], depth


def _context(pba):
    ctx = pba.Context(channels=2)
    for H, W in ((24, 32), (48, 72)):
        ctx.add_sensor(0, H, W, 0.8 * W, 0.8 * W, (W - 1) / 2, (H - 1) / 2, 0.1, 10.0)
    return ctx


def _evaluate(ctx, n):
    ctx.set_poses(np.tile(np.hstack([np.eye(3).ravel(), np.zeros(3)]), (n, 1)))
    ctx.set_pairs([(0, 1), (1, 0)])
    return ctx.evaluate(want_system=True)


# the planes that the larger images need are allocated in turn: depth, interval plane, intensity
@pytest.mark.parametrize("fail_at", [0, 1, 2])
def test_load_after_a_failed_load(pba, fail_at, monkeypatch):
    import torch
    n = 2
    small, large = _images(24, 32, n), _images(48, 72, n)
    with _context(pba) as ctx:
        ctx.load_keyframes([1] * n, *large, None)
        want = _evaluate(ctx, n)
    real = torch.cuda.caching_allocator_alloc
    with _context(pba) as ctx:
        ctx.load_keyframes([0] * n, *small, None)
        _evaluate(ctx, n)
        calls = []

        def limited(*args, **kw):
            calls.append(args)
            if len(calls) == fail_at + 1:
                raise torch.cuda.OutOfMemoryError("limit of the test")
            return real(*args, **kw)

        monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", limited)
        with pytest.raises(pba.PbaError):
            ctx.load_keyframes([1] * n, *large, None)
        monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", real)
        assert len(calls) == fail_at + 1
        print("loading again after allocation %d failed" % fail_at, flush=True)
        ctx.load_keyframes([1] * n, *large, None)
        got = _evaluate(ctx, n)
    assert want["n_valid"] > 0
    assert got["F"] == want["F"] and got["n_valid"] == want["n_valid"]
    assert np.array_equal(got["H"], want["H"]) and np.array_equal(got["b"], want["b"])
