"""Host logic of the factorisation's launches in both orders (no GPU): the panel and task lists that the library's own code
builds, against a plain enumeration, and a CPU run of the launches they drive, against numpy's dense solve of the
same gauge-fixed, damped system (1e-12 of its largest entry, as for the nested-dissection plan's own check).  Ragged
last blocks, chains, stars, disconnected graphs and a filled pattern."""
import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2303_16878_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("cholplan") / "chol_plan_check")
    cmd = [hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "chol_plan_check.cpp"), os.path.join(CSRC, "ordering.hip"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def _run(exe, order, N, pairs, anchor=0, lam=1e-4, seed=1, solve=True):
    rng = np.random.default_rng(seed)
    n0 = 6 * N if solve else 0
    H = np.zeros((n0, n0))
    for s, t in pairs if solve else ():
        J = rng.standard_normal((12, 12))
        idx = np.r_[6 * s:6 * s + 6, 6 * t:6 * t + 6]
        H[np.ix_(idx, idx)] += J.T @ J
    H += 5 * np.eye(n0)
    b = rng.standard_normal(n0)
    buf = struct.pack("<ii", N, len(pairs)) + b"".join(struct.pack("<ii", s, t) for s, t in pairs)
    buf += struct.pack("<iid", n0, anchor, lam) + H.astype("<f8").tobytes() + b.astype("<f8").tobytes()
    r = subprocess.run([exe, order], input=buf, capture_output=True, timeout=300)
    assert r.returncode == 0, r.stderr.decode()
    info = r.stderr.decode().split()
    stats = {info[i]: float(info[i + 1]) for i in range(0, len(info) - 1, 2)}
    if not solve:
        return None, stats
    a0 = 6 * anchor
    A = H.copy()
    A[a0:a0 + 6, :] = 0.0
    A[:, a0:a0 + 6] = 0.0
    A[a0:a0 + 6, a0:a0 + 6] = np.eye(6)
    A[np.diag_indices(n0)] *= 1.0 + lam
    rhs = -b
    rhs[a0:a0 + 6] = 0.0
    ref = np.linalg.solve(A, rhs)
    x = np.frombuffer(r.stdout, "<f8")
    return np.abs(x - ref).max() / (np.abs(ref).max() or 1.0), stats


def _chain(n):
    return [(i, i + 1) for i in range(n - 1)]


def _filled(n, seed=0):
    rng = np.random.default_rng(seed)
    return _chain(n) + [(int(a), int(b)) for a, b in rng.integers(0, n, (n, 2))]


GRAPHS = {
    "one": (1, []),
    "pair": (2, [(0, 1)]),
    "64 rows and 2": (11, _chain(11)),
    "chain": (60, _chain(60)),
    "loop": (60, _chain(60) + [(0, 59)]),
    "star": (60, [(0, i) for i in range(1, 60)]),
    "star to the last": (60, [(59, i) for i in range(59)]),
    "apart": (70, _chain(30) + [(i, i + 1) for i in range(40, 69)]),
    "filled": (64, _filled(64)),
}


@pytest.mark.parametrize("order", ["natural", "nd"])
@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("anchor", ["first", "last"])
def test_launches_solve_the_system(checker, name, order, anchor):
    N, pairs = GRAPHS[name]
    err, st = _run(checker, order, N, pairs, anchor=0 if anchor == "first" else N - 1)
    assert err <= 1e-12, (err, st)


@pytest.mark.parametrize("order", ["natural", "nd"])
@pytest.mark.parametrize("N", [300, 1000])
def test_lists_of_large_graphs(checker, N, order):
    """A filled natural order has one column a level and a sixth of nt^3 tasks."""
    _, st = _run(checker, order, N, _filled(N), solve=False)
    nt = -(-6 * N // 64)
    if order == "natural":
        assert st["levels"] == nt == st["nt"]
        assert st["tasks"] > 0.8 * nt ** 3 / 6


def test_lists_of_a_filled_order_take_no_longer_than_writing_them(checker):
    """929770 tasks at 188 block columns: 20 bytes each against a byte written per tile of the symbolic fill, which makes
    the same visits: some 12 times its time, where a sorted map of the tasks took 180 times."""
    ratio = []
    for _ in range(3):
        _, st = _run(checker, "natural", 2000, _filled(2000), solve=False)
        ratio.append(st["lists_ms"] / st["pattern_ms"])
    assert min(ratio) < 60, ratio
