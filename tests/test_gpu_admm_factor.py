"""The ADMM kernel's FP32 factorisation at the edges of its split: 64 lanes take
the rows of floor(64 / 3m) slots at a time, so tiles with one slot, with one full
pass, one slot more and the most slots a tile holds, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl
from gpu_common import check_forward, oracle_params, run_gpu
from test_gpu_admm_only import _check_admm_only

pytestmark = pytest.mark.gpu


# contacts, wrenches (a tile holds min(12, 64 // wrenches) slots), grasps
@pytest.mark.parametrize("m,s,ng", [(1, 5, 13), (4, 64, 3), (4, 12, 11), (4, 10, 13), (5, 16, 9), (5, 12, 11),
                                    (5, 5, 25), (6, 21, 7), (6, 16, 9), (7, 21, 7), (7, 16, 9), (8, 32, 5),
                                    (8, 21, 7), (8, 5, 25)])
def test_slots_per_pass(m, s, ng):
    b = wl.uniform_batch(500 + m, ng, m, s)
    print("ADMM factor: m %d s %d, %d grasps, tol 1e-5" % (m, s, ng), flush=True)
    gpu = run_gpu(b, tol_rel=1e-5, max_iters=500, flags=api.F_ADAPTIVE_RHO)
    _check_admm_only(b, gpu, 1e-5, min_converged=0.5)


# 64 wrenches fill a tile: 1024 tiles (the last batch of the one-wave kernel)
# and 1025 give the same bits at every register budget
@pytest.mark.parametrize("ng", [1024, 1025])
def test_default_waves_on_both_sides_of_the_rule(ng):
    b = wl.uniform_batch(520, ng, 4, 64)
    print("ADMM waves: %d tiles" % ng, flush=True)
    outs = [run_gpu(b, admm_waves=w) for w in (0, 1, 2)]
    for o in outs[1:]:
        for k in ("x", "z", "y"):
            assert np.array_equal(outs[0]["state"][k], o["state"][k]), k
        assert np.array_equal(outs[0]["iters"], o["iters"])


# FP64 on every grasp: as many slots per pass as fit, at tiles of 1, 2, 5 and
# 12 slots, below and above the size at which the workspace is halved
@pytest.mark.parametrize("m,s,ng", [(4, 10, 13), (5, 64, 3), (8, 32, 5), (8, 11, 11), (8, 5, 25), (8, 64, 1030)])
def test_fp64_slots_per_pass(m, s, ng):
    b = wl.uniform_batch(540 + m, ng, m, s)
    print("ADMM FP64 factor: m %d s %d, %d grasps" % (m, s, ng), flush=True)
    every = range(0, ng, max(1, ng // 25))
    sub = b.subset(list(every))
    ref = oracle.solve_batch(sub.counts, sub.woff, sub.points, sub.normals, sub.mu, sub.wrench, prm=oracle_params())
    check_forward(sub, run_gpu(sub, fp64_cond=1.0), ref)
    # ADMM alone (the polish splits its sums by batch size): the grasps give the
    # same bits in the whole batch and in the part
    full = run_gpu(b, fp64_cond=1.0, flags=api.F_ADAPTIVE_RHO)
    part = run_gpu(sub, fp64_cond=1.0, flags=api.F_ADAPTIVE_RHO)
    assert np.all(full["status"] & api.ST_FP64_CHOL) and np.all(part["status"] & api.ST_FP64_CHOL)
    cols = np.concatenate([np.arange(b.woff[g], b.woff[g + 1]) for g in every])
    for k in ("x", "z", "y"):
        assert np.array_equal(full["state"][k][:, cols], part["state"][k]), k
