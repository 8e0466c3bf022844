"""Calls that run out of device memory: for every allocation of the call in turn, the call reports PBA_ENOMEM, nothing
works on what it left half done (PBA_ESTATE until the missing part is given again), and once it is given the
results are those of a new context."""
import contextlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SMALL, LARGE = 0, 1
SIZES = ((24, 32), (48, 72))


@pytest.fixture(scope="module")
def pba():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2303_16878_amd as pba
    pba.load_library()
    return pba


@contextlib.contextmanager
def memory_for(n_alloc):
    """Device memory for n_alloc more allocations (None: no limit)."""
    import torch
    real, calls = torch.cuda.caching_allocator_alloc, []

    def limited(*args, **kw):
        calls.append(args)
        if n_alloc is not None and len(calls) > n_alloc:
            raise torch.cuda.OutOfMemoryError("limit of the test")
        return real(*args, **kw)

    torch.cuda.caching_allocator_alloc = limited
    try:
        yield calls
    finally:
        torch.cuda.caching_allocator_alloc = real


def _images(which, n, seed=0):
    H, W = SIZES[which]
    rng = np.random.default_rng(1000 * seed + H * W)
    depth = [np.full((H, W), 2.0, np.float32) + 0.01 * rng.random((H, W), dtype=np.float32) for _ in range(n)]
    return [rng.random((H, W), dtype=np.float32) for _ in range(n)], depth


def _poses(n):
    X = np.tile(np.hstack([np.eye(3).ravel(), np.zeros(3)]), (n, 1))
    X[:, 9] = 0.01 * np.arange(n)
    return X


PAIRS = [(0, 1), (1, 0)]


def _context(pba, **kw):
    ctx = pba.Context(channels=2, **kw)
    for H, W in SIZES:
        ctx.add_sensor(0, H, W, 0.8 * W, 0.8 * W, (W - 1) / 2, (H - 1) / 2, 0.1, 10.0)
    return ctx


def _loaded(pba, which, n, groups=None, **kw):
    ctx = _context(pba, **kw)
    ctx.load_keyframes([which] * n, *_images(which, n), None)
    if groups is not None:
        ctx.set_pose_groups(groups)
    ctx.set_poses(_poses(ctx.n_poses))
    ctx.set_pairs(PAIRS)
    return ctx


def _equal(a, b):
    assert a["n_valid"] > 0 and a["F"] == b["F"] and a["n_valid"] == b["n_valid"]
    assert np.array_equal(a["H"], b["H"]) and np.array_equal(a["b"], b["b"])


def _refused(pba, call, status=None):
    with pytest.raises(pba.PbaError) as e:
        call()
    assert e.value.status == (pba.PBA_ESTATE if status is None else status), e.value
    return True


def _out_of_memory(pba, call, k):
    """True if the call fails for want of memory with k allocations left to it, False if it gets by."""
    with memory_for(k) as calls:
        try:
            call()
            return False
        except pba.PbaError as e:
            assert e.status == pba.PBA_ENOMEM and len(calls) == k + 1, e
            print("out of memory at allocation %d" % k, flush=True)
            return True


@pytest.mark.parametrize("zbuffer", [False, True])
@pytest.mark.parametrize("groups", [None, [0, 0, 1]])
def test_load(pba, groups, zbuffer):
    """Larger images, as many keyframes: the old poses, pairs and work queue do not serve the new set, neither after the
    failure nor after a second attempt that succeeds."""
    n = 3
    with _loaded(pba, LARGE, n, occlusion_zbuffer=zbuffer) as ctx:
        want = ctx.evaluate(want_system=True)
    k = 0
    while True:
        with _loaded(pba, SMALL, n, groups, occlusion_zbuffer=zbuffer) as ctx:
            ctx.evaluate()
            load = lambda: ctx.load_keyframes([LARGE] * n, *_images(LARGE, n), None)
            if not _out_of_memory(pba, load, k):
                break
            for call in (ctx.evaluate, lambda: ctx.iterate(1), lambda: ctx.loss_forward(np.zeros((n, 6), np.float32)),
                         lambda: ctx.build_pyramid(2), lambda: ctx.set_pairs(PAIRS), ctx.get_poses, ctx.autotune):
                _refused(pba, call)
            load()
            for call in (ctx.evaluate, lambda: ctx.iterate(1), ctx.get_poses):
                _refused(pba, call)
            ctx.set_poses(_poses(n))
            _refused(pba, ctx.evaluate)
            ctx.set_pairs(PAIRS)
            _equal(ctx.evaluate(want_system=True), want)
        k += 1
    assert k >= 3


def test_load_of_fewer_keyframes(pba):
    k = 0
    while True:
        with _loaded(pba, SMALL, 4) as ctx:
            if not _out_of_memory(pba, lambda: ctx.load_keyframes([LARGE] * 2, *_images(LARGE, 2), None), k):
                break
            _refused(pba, lambda: ctx.get_level_image(0, 3), pba.PBA_EINVAL)
            _refused(pba, lambda: ctx.set_pose_groups([0, 0, 1, 1]))
            _refused(pba, ctx.evaluate)
        k += 1
    assert k >= 1


def test_new_images_of_the_same_set_from_a_pyramid_level(pba):
    """Host images are staged: without memory for that, the set is given up, whatever level was active."""
    n = 2
    images = _images(LARGE, n, seed=1)
    with _loaded(pba, LARGE, n) as ctx:
        ctx.load_keyframes([LARGE] * n, *images, None)
        want = ctx.evaluate(want_system=True)
    k = 0
    while True:
        with _loaded(pba, LARGE, n) as ctx:
            ctx.build_pyramid(2)
            ctx.set_level(1)
            ctx.iterate(1)
            load = lambda: ctx.load_keyframes([LARGE] * n, *images, None)
            if not _out_of_memory(pba, load, k):
                break
            _refused(pba, ctx.evaluate)
            load()
            ctx.set_poses(_poses(n))
            ctx.set_pairs(PAIRS)
            _equal(ctx.evaluate(want_system=True), want)
        k += 1
    assert k >= 1


def test_a_refused_load_changes_nothing(pba):
    """Two keyframes where the anchor is the third: refused before anything is given up."""
    with _loaded(pba, SMALL, 3, anchor=2) as ctx:
        want = ctx.evaluate(want_system=True)
        _refused(pba, lambda: ctx.load_keyframes([LARGE] * 2, *_images(LARGE, 2), None), pba.PBA_EINVAL)
        _equal(ctx.evaluate(want_system=True), want)


@pytest.mark.parametrize("zbuffer", [False, True])
@pytest.mark.parametrize("back", ["set_level", "estimate_normals"])
def test_level_switch(pba, back, zbuffer):
    """A switch to a finer level without memory for its longer queue: the next call that needs the queue builds it,
    or reports that it cannot either."""
    n, rng = 2, np.random.default_rng(5)
    I, D = _images(LARGE, n)
    N = [rng.standard_normal(i.shape + (3,)).astype(np.float32) for i in I]

    def at_level_1():
        ctx = pba.Context(occlusion_zbuffer=zbuffer)
        H, W = SIZES[LARGE]
        ctx.add_sensor(0, H, W, 0.8 * W, 0.8 * W, (W - 1) / 2, (H - 1) / 2, 0.1, 10.0)
        ctx.load_keyframes([0] * n, I, D, N)
        ctx.set_poses(_poses(n))
        ctx.build_pyramid(2)
        ctx.set_level(1)
        ctx.set_pairs(PAIRS)
        return ctx

    switch = (lambda ctx: ctx.set_level(0)) if back == "set_level" else (lambda ctx: ctx.estimate_normals())
    with at_level_1() as ctx:
        switch(ctx)
        want = ctx.evaluate(want_system=True)
        want_log = ctx.iterate(2)
    k = 0
    while True:
        with at_level_1() as ctx:
            ctx.evaluate()
            if not _out_of_memory(pba, lambda: switch(ctx), k):
                break
            with memory_for(0):
                _refused(pba, ctx.evaluate, pba.PBA_ENOMEM)
                _refused(pba, lambda: ctx.iterate(1), pba.PBA_ENOMEM)
            with memory_for(None) as calls:   # it allocates nothing, this neither
                _refused(pba, lambda: ctx.evaluate(noalloc=True))
                assert not calls
            ctx.set_level(0)
            if back == "estimate_normals":
                ctx.estimate_normals()
            _equal(ctx.evaluate(want_system=True), want)
            assert [dict(r, ms=0) for r in ctx.iterate(2)] == [dict(r, ms=0) for r in want_log]
        k += 1
    assert k >= 1


CHAIN = [(i, j) for i in range(30) for j in (i - 1, i + 1) if 0 <= j < 30]   # 30 poses: 180 rows, several blocks


@pytest.mark.parametrize("zbuffer", [False, True])
def test_set_pairs_and_build_pairs(pba, zbuffer):
    """A longer pair list (its queue, assembly lists, factorisation plan or system do not fit): no pairs, neither the old
    nor half of the new ones."""
    n = 30
    with _loaded(pba, SMALL, n, occlusion_zbuffer=zbuffer) as ctx:
        ctx.set_pairs(CHAIN)
        want = ctx.evaluate(want_system=True)
        step = ctx.solve_step(1e-3)
    for change in (lambda ctx: ctx.set_pairs(CHAIN),
                   lambda ctx: ctx.build_pairs(max_angle=0.0, max_dist=0.0, min_ratio=0.0, sequential=True)):
        k = 0
        while True:
            with _loaded(pba, SMALL, n, occlusion_zbuffer=zbuffer) as ctx:
                ctx.evaluate()
                if not _out_of_memory(pba, lambda: change(ctx), k):
                    break
                for call in (ctx.evaluate, lambda: ctx.solve_step(1e-3), lambda: ctx.iterate(1)):
                    _refused(pba, call)
                ctx.set_pairs(CHAIN)
                _equal(ctx.evaluate(want_system=True), want)
                assert np.array_equal(ctx.solve_step(1e-3), step)
            k += 1
        assert k >= 5


def test_pose_groups(pba):
    """More pose variables than before: no pairs until their plan is built."""
    n, groups = 30, [k // 15 for k in range(30)]

    def grouped():
        ctx = _loaded(pba, SMALL, n, groups)
        ctx.set_pairs(CHAIN)
        return ctx

    with _loaded(pba, SMALL, n) as ctx:
        ctx.set_pairs(CHAIN)
        want = ctx.evaluate(want_system=True)
    k = 0
    while True:
        with grouped() as ctx:
            ctx.evaluate()
            if not _out_of_memory(pba, lambda: ctx.set_pose_groups(None), k):
                break
            ctx.n_poses = n
            _refused(pba, ctx.evaluate)
            ctx.set_poses(_poses(n))
            _refused(pba, ctx.evaluate)
            ctx.set_pairs(CHAIN)
            _equal(ctx.evaluate(want_system=True), want)
        k += 1
    assert k >= 2


@pytest.mark.parametrize("graph", [False, True])
def test_iterate_without_memory_for_its_log(pba, graph):
    with _loaded(pba, SMALL, 2, use_graph=graph) as ctx:
        ctx.iterate(3)
        want = [dict(r, ms=0) for r in ctx.iterate(3)]
    with _loaded(pba, SMALL, 2, use_graph=graph) as ctx:
        ctx.iterate(3)
        assert _out_of_memory(pba, lambda: ctx.iterate(100), 0)
        with memory_for(0):
            _refused(pba, lambda: ctx.iterate(3), pba.PBA_ENOMEM)
        assert [dict(r, ms=0) for r in ctx.iterate(3)] == want


@pytest.mark.parametrize("active", [0, 1])
def test_pyramid(pba, active):
    """A pyramid that does not fit: no level of it exists, the loaded images are active."""
    with _loaded(pba, LARGE, 2) as ctx:
        want = ctx.evaluate(want_system=True)
        ctx.build_pyramid(3)
        images = ctx.get_level_image(2, 1)
    k = 0
    while True:
        with _loaded(pba, LARGE, 2) as ctx:
            if active:
                ctx.build_pyramid(2)
                ctx.set_level(1)
                ctx.evaluate()
            if not _out_of_memory(pba, lambda: ctx.build_pyramid(3), k):
                break
            for level in (1, 2):
                _refused(pba, lambda: ctx.set_level(level), pba.PBA_EINVAL)
                _refused(pba, lambda: ctx.get_level_image(level, 0), pba.PBA_EINVAL)
            _equal(ctx.evaluate(want_system=True), want)
            assert len(ctx.optimize_pyramid([1])) == 1
            ctx.build_pyramid(3)
            assert all(np.array_equal(a, b) for a, b in zip(ctx.get_level_image(2, 1), images))
        k += 1
    assert k >= 10
