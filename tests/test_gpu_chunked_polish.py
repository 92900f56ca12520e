"""The active-set polish where the dual Newton polish does not take its QPs
(eps_reg below 5e-7, or polish_chunk 0): budgets of the one-lane pass, the
contact-parallel polish of what it hands on, the automatic budget on both
sides of its size limit, and the restarts that served QPs once needed.  That
the budget changes a QP's flop count tells that the active-set polish ran: the
Newton polish's does not depend on it."""
import numpy as np
import pytest

import oracle
import test_gpu_served_hard_qps as served
from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl
from gpu_common import check_energy, check_forward, check_state_kkt, oracle_params
from test_gpu_newton_caps import solve

pytestmark = pytest.mark.gpu

EPS = float(np.float32(4e-7))


def _check(b, got, gs):
    """Whole grasps gs of the batch against the oracle."""
    cols = np.concatenate([np.arange(b.woff[g], b.woff[g + 1]) for g in gs])
    sub = b.subset(gs)
    part = {k: got[k][cols] for k in ("forces", "qp_obj", "status")}
    part["energy"] = got["energy"][gs]
    part["state"] = {k: v[:, cols] if v.ndim == 2 else v for k, v in got["state"].items()}
    prm = oracle_params(eps=EPS)
    ref = oracle.solve_batch(sub.counts, sub.woff, sub.points, sub.normals, sub.mu, sub.wrench, prm)
    print(check_forward(sub, part, ref))
    check_energy(sub, part, ref)
    check_state_kkt(sub, part, 1e-5, range(0, sub.n_qps, 7), prm)


@pytest.mark.parametrize("cfg,ng", [(1, 300), (3, 300), (0, 64)])
@pytest.mark.parametrize("chunk", [1, 3, 12, 40])
def test_budgets(chunk, cfg, ng):
    b = wl.config(cfg, ng)
    print("chunked polish: %s, %d grasps, chunk %d" % (b.name, ng, chunk), flush=True)
    got, other = solve(b, eps_reg=EPS, polish_chunk=chunk), solve(b, eps_reg=EPS, polish_chunk=40 if chunk < 40 else 1)
    assert np.any(got["polish_flops"] != other["polish_flops"])
    _check(b, got, list(range(ng)))


# the automatic budget: 1 up to 40,960 QPs, 16 above; more tiles than 1024
@pytest.mark.parametrize("m,s,ng", [(5, 16, 2560), (5, 16, 2600), (8, 11, 5200), (4, 6, 12000)])
def test_automatic_budget(m, s, ng):
    b = wl.uniform_batch(810 + m, ng, m, s)
    print("chunked polish: m %d, %d QPs, automatic" % (m, b.n_qps), flush=True)
    got, other = solve(b, eps_reg=EPS), solve(b, eps_reg=EPS, polish_chunk=40)
    assert np.any(got["polish_flops"] != other["polish_flops"])
    _check(b, got, list(range(0, ng, ng // 40)))


# The third is beyond the one-lane polish (as it was before the Newton polish
# took such QPs; the contact-parallel polish solved it): it keeps its ADMM point.
@pytest.mark.parametrize("rid,step,qp", served.CASES[:2] + [
    pytest.param(*served.CASES[2], marks=pytest.mark.xfail(strict=True, reason="beyond the one-lane polish"))])
def test_served_hard_qps_on_the_active_set_polish(monkeypatch, rid, step, qp):
    default = api.default_params
    monkeypatch.setattr(api, "default_params", lambda **kw: default(**kw, polish_chunk=0))
    served.test_served_qp_converges_at_the_oracle_minimiser(rid, step, qp)
