"""The dual Newton polish on the GPU: every choice of lanes per QP, ragged
tiles, what it leaves to the active-set and barrier polish, and the cases in
which it is not taken."""
import numpy as np
import pytest

import oracle
from oracle import cone as oc
from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl
from gpu_common import check_energy, check_forward, check_state_kkt, oracle_params, run_gpu

pytestmark = pytest.mark.gpu


def _ref(b, prm=None):
    return oracle.solve_batch(b.counts, b.woff, b.points, b.normals, b.mu, b.wrench, prm or oracle.params())


# contacts, wrenches, QPs on both sides of each change of the lanes per QP;
# wrench counts that leave lanes of a tile idle (64 = 7 * 9 + 1 = 3 * 21 + 1)
@pytest.mark.parametrize("m,s,qps", [(1, 9, 9), (3, 21, 2100), (4, 9, 65529), (4, 9, 65547), (5, 21, 20475),
                                     (5, 21, 20496), (5, 9, 40959), (5, 9, 40968), (6, 9, 40968), (7, 9, 20475),
                                     (8, 21, 20496), (8, 64, 64)])
def test_lanes_per_qp(m, s, qps):
    b = wl.uniform_batch(700 + m, qps // s, m, s)
    print("newton: m %d s %d, %d QPs" % (m, s, b.n_qps), flush=True)
    gpu = run_gpu(b)
    ref = _ref(b)
    print(check_forward(b, gpu, ref))
    check_energy(b, gpu, ref)
    check_state_kkt(b, gpu, 1e-5, range(0, b.n_qps, max(1, b.n_qps // 300)))


@pytest.mark.parametrize("cone", [False, True])
def test_what_it_leaves_is_finished_by_the_other_polish(cone):
    # a step cap between the shortest and the longest Newton solve: some QPs of
    # each grasp are left (the cap also bounds the other polish, which does
    # not finish all of them); whatever was polished is the minimiser
    b = wl.uniform_batch(71, 40, 5, 16)
    print("newton leaves: cone %d" % cone, flush=True)
    full = run_gpu(b) if not cone else None
    if cone:
        import torch
        def solve(**kw):
            p = api.default_params(m_max=5, s_max=16, friction_cone=api.CONE_CIRCULAR, **kw)
            sv, db = api.Solver(p), api.DeviceBatch(b)
            r = sv.solve(db, state=api.new_state(db.n_grasps, db.n_qps, 5, cone=True))
            torch.cuda.synchronize()
            out = {k: v.cpu().numpy() for k, v in r.items()}
            sv.close()
            return out
        full, cut = solve(), solve(polish_steps=6)
    else:
        cut = run_gpu(b, polish_steps=16)
    done = (cut["status"] & api.ST_POLISHED) != 0
    assert np.all(full["status"] & api.ST_POLISHED) and 0 < done.sum() < b.n_qps
    assert np.all((cut["status"][~done] & api.ST_POLISH_REJ) != 0)
    assert np.abs(cut["forces"][done] - full["forces"][done]).max() <= (5e-5 if cone else 1e-5)
    E = np.add.reduceat(cut["qp_obj"].astype(np.float64), b.woff[:-1])
    assert np.abs(cut["energy"] - E).max() <= 1e-5 * max(1.0, np.abs(E).max())


@pytest.mark.parametrize("eps", [4e-7, 1e-3])
def test_regulariser_on_both_sides_of_the_rule(eps):
    b = wl.uniform_batch(72, 60, 5, 9)
    print("newton rule: eps %g" % eps, flush=True)
    gpu = run_gpu(b, eps_reg=eps)
    prm = oracle_params(eps=float(np.float32(eps)))
    ref = _ref(b, prm)
    print(check_forward(b, gpu, ref))
    check_state_kkt(b, gpu, 1e-5, range(0, b.n_qps, 7), prm)


@pytest.mark.parametrize("m,s,qps", [(1, 7, 7), (3, 9, 900), (4, 9, 8190), (5, 9, 8190), (5, 9, 8199)])
def test_cone_on_both_sides_of_the_size_limit(m, s, qps):
    # sampled QPs against the cone oracle, with the parity tests' tolerances
    import torch
    b = wl.uniform_batch(740 + m, qps // s, m, s)
    print("newton cone: m %d, %d QPs" % (m, b.n_qps), flush=True)
    p = api.default_params(m_max=m, s_max=s, friction_cone=api.CONE_CIRCULAR)
    sv, db = api.Solver(p), api.DeviceBatch(b)
    r = sv.solve(db, state=api.new_state(db.n_grasps, db.n_qps, m, cone=True))
    torch.cuda.synchronize()
    assert np.all(r["status"].cpu().numpy() & api.ST_CONVERGED)
    f = r["forces"].cpu().numpy().astype(np.float64)
    sv.close()
    qps = np.arange(0, b.n_qps, max(1, b.n_qps // 40))
    ref = oc.solve_batch(b.counts, b.woff, b.points, b.normals, b.mu, b.wrench, qps=qps)
    Q = r["qp_obj"].cpu().numpy()[qps]
    assert np.all(np.abs(Q - ref["qobj"][qps]) <= 1e-5 * np.maximum(ref["qobj"][qps], 1e-2))
    assert np.abs(f[qps] - ref["forces"][qps][:, :3 * m]).max() <= 1e-4


def test_cone_without_room_for_the_workspace():
    # a budget that holds the descriptors and nothing else: the cone's solve is
    # accepted as ever (one-lane barrier polish)
    import torch
    b = wl.uniform_batch(73, 64, 5, 16)
    print("newton: cone, tight budget", flush=True)
    out = []
    for budget in (0, 4096):
        p = api.default_params(m_max=5, s_max=16, friction_cone=api.CONE_CIRCULAR)
        sv, db = api.Solver(p, budget=budget), api.DeviceBatch(b)
        r = sv.solve(db, state=api.new_state(db.n_grasps, db.n_qps, 5, cone=True))
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        sv.close()
    for o in out:
        assert np.all(o["status"] & api.ST_CONVERGED) and np.all(o["status"] & api.ST_POLISHED)
    assert np.abs(out[0]["forces"] - out[1]["forces"]).max() <= 5e-5
