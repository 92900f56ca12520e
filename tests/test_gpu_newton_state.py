"""The Newton polish on a pooled state and in the batched form: the same bits as
on a plain state in grasp order, cold and warm-started, and nothing written
between the pool's columns.  Small cone batches, which keep their forces in the
state between the two kernels, some of their QPs left to the barrier
(torque_scale 1000); and pyramid QPs ended in two doubles (beta 1000)."""
import numpy as np
import pytest

from paper_2412_16490_amd import api
from paper_2412_16490_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("cone,kw", [(True, {}), (True, dict(torque_scale=1000.0)), (False, dict(beta=1000.0))])
def test_pooled_state_and_batched_form(cone, kw, batched):
    import torch
    b = wl.config(3, 300)  # 4 and 5 contacts, 6 to 32 wrenches: about 5700 QPs
    print("newton state: cone %d, %s, batched %d" % (cone, kw, batched), flush=True)
    db = api.DeviceBatch(b)
    G, W = db.n_grasps, db.n_qps
    if cone:
        kw = dict(kw, friction_cone=api.CONE_CIRCULAR)
    cold = api.default_params(m_max=5, s_max=32, **kw)
    assert api.bodex_qp_polish_kind(cold, W) == "newton"
    rng = np.random.default_rng(5)
    s_of = np.diff(b.woff)
    qoff, col = np.zeros(G, np.int32), 7
    for g in rng.permutation(G):  # in a shuffled order with gaps
        qoff[g] = col
        col += int(s_of[g]) + int(rng.integers(0, 4))
    goff = (2 * rng.permutation(G) + 1).astype(np.int32)
    plain = api.new_state(G, W, 5, cone=cone)
    pool = api.new_state(3 * G, 2 * W, 5, cone=cone)
    assert col <= 2 * W
    for k in ("x", "z", "y", "r", "rho"):
        pool[k].fill_(777.0)
    pooled = dict(pool, qp_offset=qoff, grasp_offset=goff)
    outs = []
    for st, form in ((plain, 0), (pooled, api.F_BATCHED if batched else 0)):
        got = []
        for warm in (0, api.F_WARM_START):
            p = api.Params.from_buffer_copy(bytes(cold))
            p.flags |= warm | form
            sv = api.Solver(p)
            r = sv.solve(db, state=st)
            got += [r[k].cpu().numpy().copy() for k in ("forces", "qp_obj", "energy", "kkt_rel", "iters", "status")]
            if warm:
                gp, gn = sv.backward(db, st, dL_dE=torch.ones(G, device="cuda"))
                got += [gp.cpu().numpy(), gn.cpu().numpy()]
            sv.close()
        outs.append(got)
    for x, y in zip(*outs):
        np.testing.assert_array_equal(x, y)
    assert np.all(outs[0][5] & api.ST_POLISHED)
    cols = np.concatenate([qoff[g] + np.arange(s_of[g]) for g in range(G)])
    gaps = np.setdiff1d(np.arange(2 * W), cols)
    for k in ("x", "z", "y", "r"):
        got = pool[k].cpu().numpy()
        np.testing.assert_array_equal(got[:, cols], plain[k].cpu().numpy(), err_msg=k)
        assert np.all(got[:, gaps] == 777.0), k


@pytest.mark.parametrize("cone", [False, True])
def test_a_nonfinite_grasp_leaves_the_others_alone(cone):
    import torch
    b = wl.uniform_batch(91, 120, 5, 16)
    print("newton state: NaN grasp, cone %d" % cone, flush=True)
    out = []
    for bad in (False, True):
        c = b.subset(list(range(b.n_grasps)))
        if bad:
            c.points[37, 2, 1] = np.nan
            c.mu[80, 0] = -1.0
        kw = dict(friction_cone=api.CONE_CIRCULAR) if cone else {}
        db = api.DeviceBatch(c)
        sv = api.Solver(api.default_params(m_max=5, s_max=16, **kw))
        r = sv.solve(db, state=api.new_state(db.n_grasps, db.n_qps, 5, cone=cone))
        torch.cuda.synchronize()
        out.append({k: r[k].cpu().numpy() for k in ("forces", "qp_obj", "energy", "kkt_rel", "status")})
        sv.close()
    hit = np.zeros(b.n_qps, bool)
    for g in (37, 80):
        hit[b.woff[g]:b.woff[g + 1]] = True
        assert np.isnan(out[1]["energy"][g])
    assert np.all(out[1]["status"][hit] & api.ST_NONFINITE) and np.all(np.isnan(out[1]["qp_obj"][hit]))
    assert not np.any(out[1]["status"][hit] & (api.ST_POLISHED | api.ST_CONVERGED))
    for k in ("forces", "qp_obj", "kkt_rel", "status"):
        np.testing.assert_array_equal(out[1][k][~hit], out[0][k][~hit], err_msg=k)
    others = np.setdiff1d(np.arange(b.n_grasps), (37, 80))
    np.testing.assert_array_equal(out[1]["energy"][others], out[0]["energy"][others])
