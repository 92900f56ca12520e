"""What the dual Newton polish leaves and the other polish finishes: such QPs
are polished, at the oracle's minimiser, with the right state and energies, in
batches of more tiles than the finishing launch has blocks."""
import numpy as np
import pytest

import oracle
from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl
from gpu_common import check_energy, check_forward, check_state_kkt
from test_gpu_newton_caps import solve

pytestmark = pytest.mark.gpu


def _grasps_of(b, w):
    return sorted({int(g) for g in np.searchsorted(b.woff, w, side="right") - 1})


# from a single ADMM iteration and at a cap of 32, the QPs that need more steps
# are left (their flop count is not that of the uncapped run); 9,000 grasps x
# 11 wrenches are 1800 tiles
@pytest.mark.parametrize("m,s,grasps", [(8, 11, 9000), (5, 16, 8192)])
def test_pyramid(m, s, grasps):
    b = wl.uniform_batch(5, grasps, m, s)
    print("newton left: m %d, %d QPs" % (m, b.n_qps), flush=True)
    cut, full = solve(b, polish_steps=32, max_iters=1), solve(b, max_iters=1)
    left = np.nonzero(cut["polish_flops"] != full["polish_flops"])[0]
    polished = (cut["status"] & api.ST_POLISHED) != 0
    print("left %d" % len(left), flush=True)
    assert 20 <= len(left) < b.n_qps // 2 and np.all(polished)
    assert np.any(left >= 1024 * s * (64 // s))  # in tiles beyond the finishing launch's 1024 blocks, too
    rest = np.setdiff1d(np.arange(b.n_qps), left)
    np.testing.assert_array_equal(cut["forces"][rest], full["forces"][rest])
    gs = _grasps_of(b, left[:: max(1, len(left) // 100)])
    cols = np.concatenate([np.arange(b.woff[g], b.woff[g + 1]) for g in gs])
    sub = b.subset(gs)
    got = {k: cut[k][cols] for k in ("forces", "qp_obj", "status")}
    got["energy"] = cut["energy"][gs]
    got["state"] = {k: v[:, cols] if v.ndim == 2 else v for k, v in cut["state"].items()}
    ref = oracle.solve_batch(sub.counts, sub.woff, sub.points, sub.normals, sub.mu, sub.wrench, oracle.params())
    print(check_forward(sub, got, ref))
    check_energy(sub, got, ref)
    check_state_kkt(sub, got, 1e-5, range(sub.n_qps))


# torque arms of 20 to 80: cone QPs run into the step cap, and the barrier
# polish, from the same ADMM point, gives them the bits it gives alone
def test_cone():
    b = wl.uniform_batch(5, 512, 5, 16)
    print("newton left: cone", flush=True)
    got, barrier = solve(b, cone=True, torque_scale=1000.0), solve(b, cone=True, torque_scale=1000.0, polish_chunk=0)
    # the flops of both polishes, the Newton steps' 128 evaluations and factors
    left = got["polish_flops"] > barrier["polish_flops"] + 128 * (266 * 5 + 235)
    print("left %d of %d" % (left.sum(), b.n_qps), flush=True)
    assert 0 < left.sum() < b.n_qps // 2
    assert np.all(got["status"] & api.ST_POLISHED) and np.all(barrier["status"] & api.ST_POLISHED)
    for k in ("forces", "qp_obj", "kkt_rel", "status", "iters"):
        np.testing.assert_array_equal(got[k][left], barrier[k][left], err_msg=k)
    for k in ("x", "z", "y", "r"):
        np.testing.assert_array_equal(got["state"][k][:, left], barrier["state"][k][:, left], err_msg=k)
    E = np.add.reduceat(got["qp_obj"].astype(np.float64), b.woff[:-1])
    assert np.abs(got["energy"] / E - 1.0).max() <= 1e-6
