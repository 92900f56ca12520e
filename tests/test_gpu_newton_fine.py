"""The dual Newton polish on the GPU where the rounding of its dual variable
matters: large beta, wrenches that are not unit vectors, and torque arms of 20
to 1000 (a large torque_scale, or points in millimetres), at each number of
lanes per QP.  Every QP is polished, with forces as good as at beta 1."""
import numpy as np
import pytest

import oracle
from oracle import cone as oc
from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl
from gpu_common import oracle_params, run_gpu

pytestmark = pytest.mark.gpu


# 32-bit forces in [0, 1] are rounded by at most 3e-8, and the oracle's carry up
# to 1e-8 at |beta t| 1000
@pytest.mark.parametrize("m,s,grasps", [(3, 9, 30), (4, 9, 7400), (5, 9, 60), (5, 9, 2400), (5, 9, 4700), (8, 9, 30),
                                        (8, 9, 2400)])
@pytest.mark.parametrize("beta,scale", [(100.0, 1.0), (1000.0, 1.0), (1.0, 1000.0)])
def test_forces_at_large_right_hand_sides(m, s, grasps, beta, scale):
    b = wl.uniform_batch(760 + m, grasps, m, s)
    b.wrench = (b.wrench * np.float32(scale)).astype(np.float32)
    print("newton fine: m %d, %d QPs, beta %g, |t| %g" % (m, b.n_qps, beta, scale), flush=True)
    gpu = run_gpu(b, beta=beta)
    assert np.all(gpu["status"] & api.ST_POLISHED)
    step = max(1, b.n_qps // 300)
    gs = list(range(0, b.n_grasps, step))
    cols = np.concatenate([np.arange(b.woff[g], b.woff[g + 1]) for g in gs])
    sub = b.subset(gs)
    ref = oracle.solve_batch(sub.counts, sub.woff, sub.points, sub.normals, sub.mu, sub.wrench,
                             oracle_params(beta=beta, eps=float(np.float32(1e-6))))
    assert np.abs(gpu["forces"][cols] - ref["forces"][:, :3 * m]).max() <= 4e-8
    assert np.abs(gpu["qp_obj"][cols] / ref["qobj"] - 1.0).max() <= 1e-6
    E = np.add.reduceat(gpu["qp_obj"].astype(np.float64), b.woff[:-1])
    assert np.abs(gpu["energy"] / E - 1.0).max() <= 1e-6


# the oracle's forces carry the rounding of G (2^-53) times the square of its
# rows over eps: 1e-16 (3 + 2 arm^2) / eps
@pytest.mark.parametrize("m,s,grasps", [(3, 9, 30), (4, 9, 7400), (5, 9, 60), (5, 9, 2400), (5, 9, 4700), (8, 9, 30)])
@pytest.mark.parametrize("kappa,unit", [(400.0, 1.0), (1000.0, 1.0), (4000.0, 1.0), (1.0, 1000.0)])
def test_every_qp_is_polished_at_long_torque_arms(m, s, grasps, kappa, unit):
    b = wl.uniform_batch(780 + m, grasps, m, s)
    b.points = (b.points * np.float32(unit)).astype(np.float32)
    arm = kappa * np.linalg.norm(b.points, axis=-1).max()
    print("newton fine: m %d, %d QPs, arms up to %.0f" % (m, b.n_qps, arm), flush=True)
    gpu = run_gpu(b, torque_scale=kappa)
    assert np.all(gpu["status"] & api.ST_POLISHED), "%d left" % ((gpu["status"] & api.ST_POLISHED) == 0).sum()
    gs = list(range(0, b.n_grasps, max(1, b.n_qps // 300)))
    cols = np.concatenate([np.arange(b.woff[g], b.woff[g + 1]) for g in gs])
    sub = b.subset(gs)
    ref = oracle.solve_batch(sub.counts, sub.woff, sub.points, sub.normals, sub.mu, sub.wrench,
                             oracle_params(kappa=kappa, eps=float(np.float32(1e-6))))
    tol = 4e-8 + 2.0 ** -53 * (3 + 2 * arm ** 2) / 1e-6
    assert np.abs(gpu["forces"][cols] - ref["forces"][:, :3 * m]).max() <= tol


@pytest.mark.parametrize("m", [3, 5])
@pytest.mark.parametrize("kw", [dict(beta=100.0), dict(beta=1000.0), dict(torque_scale=1000.0)])
def test_cone(m, kw):
    # sampled QPs against the cone oracle (a barrier method: 1e-4 of fmax)
    import torch
    b = wl.uniform_batch(790 + m, 100, m, 9)
    print("newton fine: cone, m %d, %s" % (m, kw), flush=True)
    p = api.default_params(m_max=m, s_max=9, friction_cone=api.CONE_CIRCULAR, **kw)
    sv, db = api.Solver(p), api.DeviceBatch(b)
    r = sv.solve(db, state=api.new_state(db.n_grasps, db.n_qps, m, cone=True))
    torch.cuda.synchronize()
    st, f = r["status"].cpu().numpy(), r["forces"].cpu().numpy().astype(np.float64)
    sv.close()
    assert np.all(st & api.ST_POLISHED)
    qps = np.arange(0, b.n_qps, 40)
    ref = oc.solve_batch(b.counts, b.woff, b.points, b.normals, b.mu, b.wrench, qps=qps,
                         beta=kw.get("beta", 1.0), kappa=kw.get("torque_scale", 20.0))
    assert np.abs(f[qps] - ref["forces"][qps][:, :3 * m]).max() <= 1e-4


# no force reaches the limits: the same forces, to the rounding of 32 bits
@pytest.mark.parametrize("m,s,grasps", [(4, 9, 60), (5, 9, 4700)])
def test_force_limits_no_force_reaches(m, s, grasps):
    b = wl.uniform_batch(795 + m, grasps, m, s)
    print("newton: large force_max, m %d, %d QPs" % (m, b.n_qps), flush=True)
    want = run_gpu(b, force_max=1e4)
    top = np.abs(want["forces"]).max()
    assert top < 1e3
    for fmax in (1e8, 1e12, 1e30):
        got = run_gpu(b, force_max=fmax)
        assert np.all(got["status"] & api.ST_POLISHED)
        assert np.abs(got["forces"] - want["forces"]).max() <= 2.0 ** -23 * top + 1e-6
