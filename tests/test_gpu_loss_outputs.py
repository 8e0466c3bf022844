"""Where the loss gradients go: memory of the context's device is written by one launch, any other memory the caller calls
device memory (another device's, or as here the host's, mapped) by copies.  The pose gradient is a sum in a fixed
order, so it agrees bit for bit; image gradients are sums of float atomics in any order: at most some 50 terms of
like size, 2^-23 each, so 1e-5 of the largest."""
import ctypes

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


def _pointers(tensors):
    return (ctypes.c_void_p * len(tensors))(*[t.data_ptr() if t is not None else None for t in tensors])


@pytest.mark.parametrize("channels", [2, 5])
@pytest.mark.parametrize("elsewhere", ["delta", "one image", "all", "none"])
def test_outputs_in_mapped_host_memory(pba, lidar_mini, channels, elsewhere):
    import torch
    prob = lidar_mini
    n = prob.n

    def outputs(host_delta, host_images):
        new = lambda shape, host: torch.full(shape, float("nan"), dtype=torch.float32,
                                             **(dict(pin_memory=True) if host else dict(device="cuda")))
        shape = lambda k, c: tuple(prob.depth[k].shape) + ((3,) if c == 2 else ())
        images = [[new(shape(k, c), (k, c) in host_images) for k in range(n)] for c in range(3 if channels == 5 else 2)]
        return new((n, 6), host_delta), images

    every = {(k, c) for k in range(n) for c in range(3)}
    where = {"delta": (True, set()), "one image": (False, {(1, 1)}), "all": (True, every), "none": (False, set())}
    results = []
    with pba.context_for_problem(prob, channels=channels) as ctx:
        ctx.loss_forward(np.full((n, 6), 1e-4, np.float32))
        host = [np.empty((n, 6), np.float32)]
        lists = [[np.empty(tuple(prob.depth[k].shape) + ((3,) if c == 2 else ()), np.float32) for k in range(n)]
                 for c in range(3 if channels == 5 else 2)]
        ctx.loss_backward(1.0, host[0], tuple(lists + [None] * (3 - len(lists))))
        results.append([host[0]] + [a for l in lists for a in l])
        delta, images = outputs(*where[elsewhere])
        torch.cuda.synchronize()
        ptrs = [_pointers(l) for l in images] + [None] * (3 - len(images))
        st = ctx.lib.pba_loss_backward(ctx.h, 1.0, delta.data_ptr(), *[ctypes.cast(p, ctypes.c_void_p) if p else None
                                                                       for p in ptrs], 1)
        assert st == pba.PBA_OK
        torch.cuda.synchronize()
        results.append([delta.cpu().numpy()] + [t.cpu().numpy() for l in images for t in l])
    want, got = results
    assert np.array_equal(want[0], got[0])
    for a, b in zip(want[1:], got[1:]):
        assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max()
