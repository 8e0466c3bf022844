"""GPU normal estimation (Sec. IV-A) against the oracle's plane fits, pixel by pixel.

Has-normal masks equal except for at most 1e-4 of the pixels (ties in the neighbour tests);
angles (both normals stored in FP32) within 1e-6 rad wherever the fit is well conditioned (smallest covariance eigenvalue
separated from the next by more than 1e-3 of it), the rest counted; every GPU normal faces the sensor
(n . q < 0), and where the surface is seen edge-on either orientation is accepted."""
import sys

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


def _log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _p5(p):
    q = synth.Problem(p.name, p.sensors, p.kf_sensor, p.gt_poses, p.init_poses, p.pairs, dict(p.params, channels=5))
    q.intensity, q.depth, q.normals = list(p.intensity), list(p.depth), list(p.normals)
    return q


@pytest.mark.parametrize("fixture", ["rgbd_small", "lidar_mini", "joint_mini"])
def test_normals_match_oracle(fixture, request, pba):
    p = _p5(request.getfixturevalue(fixture))
    with pba.context_for_problem(p) as ctx:
        ctx.estimate_normals(radius_m=0.1, min_px=2.0, max_px=5.0, min_count=5)
        for k in range(p.n):
            sen = p.sensors[p.kf_sensor[k]]
            tau = 0.5 if sen["model"] == 0 else 1.0
            No, ok_o, w, _ = oracle.estimate_normals(sen, p.depth[k], radius_m=0.1, min_px=2.0, max_px=5.0,
                                                     tau=tau, min_count=5)
            _, _, Ng = ctx.get_level_image(0, k)
            ok_g = np.linalg.norm(Ng, axis=-1) > 0
            mism = int((ok_g != ok_o).sum())
            assert mism <= 1e-4 * ok_o.size + 1, (k, mism)
            both = ok_g & ok_o
            well = both & ((w[..., 1] - w[..., 0]) > 1e-3 * w[..., 1])
            # orientation: n . q < 0 on both sides; where the plane is seen edge-on (|n . q| below
            # 1e-6 |q|) the sign is a tie that the two eigen-solvers' last bits decide, so there
            # either orientation is accepted
            q = oracle.unproject_image(sen, p.depth[k])
            qn = q / np.maximum(np.linalg.norm(q, axis=-1, keepdims=True), 1e-300)
            Ngd, Nod = Ng.astype(np.float64), No.astype(np.float64)
            assert np.all(np.sum(Ngd[ok_g] * qn[ok_g], -1) < 1e-6)
            grazing = np.abs(np.sum(Nod * qn, -1)) < 1e-6
            # angle from the chord (arccos of a dot product near 1 would turn the FP32 storage's
            # 6e-8 rounding into 3e-4 rad)
            chord = np.linalg.norm(Ngd - Nod, axis=-1)
            chord = np.where(grazing, np.minimum(chord, np.linalg.norm(Ngd + Nod, axis=-1)), chord)
            ang = 2.0 * np.arcsin(np.minimum(chord[well] / 2.0, 1.0))
            _log(fixture, k, "normals: %d, mask mismatches %d, ill-conditioned %d, grazing %d, max angle %.2e rad" % (
                int(both.sum()), mism, int((both & ~well).sum()), int((both & grazing).sum()), ang.max(initial=0.0)))
            assert ang.max(initial=0.0) < 1e-6
        # the estimated normals feed the evaluation: one evaluation runs and counts pixels
        ev = ctx.evaluate()
        assert ev["n_valid"] > 0


@pytest.mark.parametrize("radius_m,min_px,max_px", [(0.1, 2.0, 5.0), (0.5, 0.0, 16.0), (0.02, 1.5, 2.5), (0.05, 3.0, 3.0)])
@pytest.mark.parametrize("name", ["rgbd", "lidar", "joint"])
def test_tile_edges_and_radii(pba, name, radius_m, min_px, max_px):
    """Images that end inside a 32 x 8 tile, windows from one pixel to the largest, both models in one context:
    has-normal masks and angles against the oracle's fits, where the fit is well conditioned (middle eigenvalue
    above 1e-6 of the trace, the smallest below a tenth of it), to 1e-6 rad."""
    if name == "rgbd":
        prob = synth.make("rgbd_small", H=37, W=67, n_kf=2)
    elif name == "lidar":
        prob = synth.make("lidar128", H=21, W=129, n_kf=300, kfs=[0, 1]).subset([0, 1])
    else:
        prob = synth.make("joint", H_l=17, W_l=97, H_c=25, W_c=33, kfs=[0, 200]).subset([0, 200])
    with pba.context_for_problem(prob, channels=5) as ctx:
        ctx.estimate_normals(radius_m=radius_m, min_px=min_px, max_px=max_px, min_count=3)
        for k in range(prob.n):
            sen = prob.sensors[prob.kf_sensor[k]]
            tau = prob.params["occ_tau_pinhole"] if sen["model"] == 0 else prob.params["occ_tau_spherical"]
            want, ok, w, cnt = oracle.estimate_normals(sen, prob.depth[k], radius_m, min_px, max_px, tau, 3)
            got = ctx.get_level_image(0, k)[2].astype(np.float64)
            tr = np.maximum(w.sum(-1), 1e-300)
            clear = (w[..., 1] > 1e-6 * tr) & (cnt >= 3)
            assert np.array_equal((np.abs(got).sum(-1) > 0)[clear], ok[clear])
            assert not np.any(got[cnt < 3])
            fit = clear & ok & (w[..., 0] < 0.1 * w[..., 1])
            ang = np.linalg.norm(np.cross(got[fit], want[fit].astype(np.float64)), axis=-1)
            assert ang.max(initial=0.0) <= 1e-6, (k, ang.max(initial=0.0))
            # orientation n . q < 0, undecided where the plane holds the sensor (three neighbours in one image row)
            q = oracle.unproject_image(sen, prob.depth[k])
            decided = fit & (np.abs(np.sum(want * q, -1)) > 1e-6 * np.linalg.norm(q, axis=-1))
            assert np.all(np.sum(got[decided] * want[decided], -1) > 0)
