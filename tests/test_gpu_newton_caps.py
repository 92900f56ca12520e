"""Step caps on both sides of the rule that sends the pyramid's QPs to the dual
Newton polish: below it the chunked active-set polish runs."""
import numpy as np
import pytest

from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl

pytestmark = pytest.mark.gpu


def solve(b, cone=False, **kw):
    import torch
    p = api.default_params(m_max=b.m_max, s_max=int(np.max(np.diff(b.woff))),
                           friction_cone=api.CONE_CIRCULAR if cone else api.CONE_PYRAMID8, **kw)
    sv, db = api.Solver(p), api.DeviceBatch(b)
    st = api.new_state(db.n_grasps, db.n_qps, b.m_max, cone=cone)
    res = api.new_result(db.n_grasps, db.n_qps, b.m_max)
    res["polish_flops"] = torch.zeros(db.n_qps, device="cuda")
    sv.solve(db, state=st, result=res)
    torch.cuda.synchronize()
    out = {k: v.cpu().numpy() for k, v in res.items()}
    out["state"] = {k: v.cpu().numpy() for k, v in st.items()}
    sv.close()
    return out


@pytest.mark.parametrize("steps", [1, 8, 31, 32])
def test_step_caps_on_both_sides_of_the_rule(steps):
    # a QP's flop count tells which polish it took: the uncapped run is Newton's
    b = wl.uniform_batch(6, 40, 5, 16)
    print("newton rule: %d steps" % steps, flush=True)
    got, full = solve(b, polish_steps=steps), solve(b)
    done = (got["status"] & api.ST_POLISHED) != 0
    assert np.all(got["status"][~done] & api.ST_POLISH_REJ)
    assert np.abs(got["forces"][done] - full["forces"][done]).max(initial=0.0) <= 1e-6
    if steps >= 31:
        assert done.mean() > 0.99
    newton = got["polish_flops"] == full["polish_flops"]
    assert newton.all() if steps == 32 else newton.sum() <= b.n_qps // 100
