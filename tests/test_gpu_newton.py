"""The dual Newton polish on the GPU: every choice of lanes per QP, ragged
tiles, what it leaves to the active-set polish, and the regulariser's two
sides of the rule."""
import numpy as np
import pytest

import oracle
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


def test_what_it_leaves_is_finished_by_the_other_polish():
    # a step cap between the shortest and the longest Newton solve: some QPs of
    # each grasp are left (the cap also bounds the other polish, which does
    # not finish all of them); whatever was polished is the minimiser
    b = wl.uniform_batch(71, 40, 5, 16)
    print("newton leaves: step cap 16", flush=True)
    full, cut = run_gpu(b), run_gpu(b, polish_steps=16)
    done = (cut["status"] & api.ST_POLISHED) != 0
    assert np.all(full["status"] & api.ST_POLISHED) and 0 < done.sum() < b.n_qps
    assert np.all((cut["status"][~done] & api.ST_POLISH_REJ) != 0)
    assert np.abs(cut["forces"][done] - full["forces"][done]).max() <= 1e-5
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

