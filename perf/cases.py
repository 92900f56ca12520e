"""What this library is timed on: its calls at the sizes they are made at.

Every case is one pass of a user's program through the Python API: contact-
force QPs solved for a batch of grasps (cold, warm-started, with the gradient
of their energy), the descent of floating hands, and the fine-stage surrogate
energies.  Inputs are the repository's own synthetic contact configurations
(`paper_2412_16490_amd/workload.py`: spheres and ellipsoids, 4- and
5-fingertip grasps, friction 0.3-0.8, wrench directions on S^5), drawn anew
for every seed.

`exact` solves the same QPs in 64 bits with plain torch, by another method
than the library's: in the six-dimensional dual u of
    min 1/2 |G f - t|^2 + eps/2 |f|^2,  f in C:   f(u) = P_C(G^T u / eps),
    G f(u) + u = t,
where P_C is the closed-form projection onto the contacts' friction cones.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2412_16490_amd import api, autograd
from paper_2412_16490_amd import workload as wl

EPS, KAPPA, FMAX = 1e-6, 20.0, 1.0  # the library's default parameters


def listed():
    qp = dict(m=5, s=16, shape="ellipsoid", cone=False, gamma=0.0, beta=1.0, axes=False, graph=False)
    return [
        # the smallest benchmark workload: one object, 64 four-finger grasps
        dict(qp, name="sphere-m4-s6", kind="solve", grasps=64, m=4, s=6, shape="sphere"),
        # one step of a small served request (16-4096 grasps, 4 and 5
        # contacts mixed, 6-32 wrenches): warm-started solve and gradient
        dict(qp, name="request-37", kind="step", grasps=37, m=45, s=0),
        # ... and of the grasps a server has in flight together
        dict(qp, name="request-1800", kind="step", grasps=1800, m=45, s=0),
        # the headline batch: 131,072 QPs in one solve
        dict(qp, name="ellipsoid-m5-s16", kind="solve", grasps=8192),
        # training through torch.autograd: energy and objectives, backward
        dict(qp, name="autograd-2048", kind="autograd", grasps=2048),
        # the uneven batch in its batched form (cost-sorted, one graph launch)
        dict(qp, name="uneven-50000", kind="solve", grasps=50000, m=45, s=0, graph=True),
        # the exact circular cone, at the headline size and for one object
        dict(qp, name="cone-m5-s16", kind="solve", grasps=8192, cone=True),
        dict(qp, name="cone-m4-s6", kind="gradient", grasps=64, m=4, s=6, cone=True),
        # the paper's six force axes with its lower bound on the normal forces
        dict(qp, name="force-axes", kind="solve", grasps=8192, s=6, axes=True, gamma=0.5),
        # the most contacts the library takes, at an odd size
        dict(qp, name="gradient-m8-s11", kind="gradient", grasps=777, m=8, s=11),
        # the upper-level descent of 64 floating hands, 20 steps
        dict(name="descent-64", kind="descent", grasps=64, m=5, s=16, steps=20),
        # fine-stage surrogate energies and their gradient
        dict(name="detach-1m", kind="detach", grasps=1 << 20, m=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "step", "step", "gradient", "autograd", "cone", "axes", "uneven",
                       "descent", "detach"])
    c = dict(kind=kind, grasps=_log_int(rng, 16, 8192), m=rng.choice([4, 5, 5, 3, 6, 7, 8]),
             s=_log_int(rng, 4, 32), shape=rng.choice(["ellipsoid", "ellipsoid", "sphere"]), cone=False, gamma=0.0,
             beta=1.0, axes=False, graph=False)
    if kind in ("solve", "gradient", "autograd") and c["m"] > 5:  # more contacts, fewer of them
        c["grasps"] = min(c["grasps"], 2048)
    if kind == "step":
        c.update(grasps=_log_int(rng, 16, 4096), m=45, s=0)
    elif kind == "cone":
        c.update(kind=rng.choice(["solve", "gradient"]), cone=True, m=rng.choice([4, 5]), s=_log_int(rng, 4, 16))
    elif kind == "axes":
        c.update(kind="solve", axes=True, s=6, m=rng.choice([4, 5]), gamma=rng.choice([0.0, 0.5, 1.0]),
                 beta=rng.choice([1.0, 1.0, 0.0]))
        if c["gamma"] == 0.0:
            c["beta"] = 1.0
    elif kind == "uneven":
        c.update(kind="solve", grasps=_log_int(rng, 512, 40000), m=45, s=0, graph=True)
    elif kind == "descent":
        return dict(kind=kind, grasps=_log_int(rng, 16, 512), m=rng.choice([4, 5]), s=_log_int(rng, 4, 16),
                    steps=rng.randint(3, 12))
    elif kind == "detach":
        return dict(kind=kind, grasps=_log_int(rng, 256, 1 << 20), m=rng.choice([3, 4, 5, 5, 8]))
    return c


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------

def _uneven(case, seed):
    """4 and 5 contacts in equal parts, 6-32 wrenches per grasp: the sizes
    belong to the case, the contacts and wrenches to the seed."""
    G = case["grasps"]
    r = np.random.Generator(np.random.PCG64(G))
    counts = r.permutation(4 + (np.arange(G) & 1)).astype(np.int32)
    woff = np.concatenate([[0], np.cumsum(r.integers(6, 33, G))]).astype(np.int32)
    r = np.random.Generator(np.random.PCG64(seed))
    p, n = wl.ellipsoid_contacts(r, G, 5)
    mu = np.repeat(r.uniform(0.3, 0.8, (G, 1)), 5, axis=1).astype(np.float32)
    t = wl.wrench_dirs(r, int(woff[-1]))
    pad = np.arange(5)[None, :] >= counts[:, None]
    p[pad], n[pad], mu[pad] = 0.0, (0.0, 0.0, 1.0), 0.5
    return wl.Batch(p, n, mu, t, counts, woff)


def _batch(case, seed):
    if case["m"] == 45:
        b = _uneven(case, seed)
    else:
        b = wl.uniform_batch(seed, case["grasps"], case["m"], case["s"], geometry=case["shape"])
    return wl.force_axis_batch(b) if case["axes"] else b


def _params(case, b):
    p = api.default_params(m_max=b.m_max, s_max=int(np.max(np.diff(b.woff))))
    p.gamma, p.beta = case["gamma"], case["beta"]
    if case["cone"]:
        p.friction_cone = api.CONE_CIRCULAR
    if case["shape"] == "sphere":
        p.tol_rel = 1e-6  # the tolerance the sphere workload is run at
    return p


def _walk(b, seed):
    """The contact points of the next two upper-level steps (sigma 1 mm)."""
    r = np.random.Generator(np.random.PCG64(seed + 77))
    live = (np.arange(b.m_max)[None, :] < b.counts[:, None])[..., None]
    w = (1e-3 * r.standard_normal((2,) + b.points.shape) * live).astype(np.float32)
    p1 = b.points + w[0]
    return p1, p1 + w[1]


def _weights(b, seed):
    r = np.random.Generator(np.random.PCG64(seed + 99))
    return r.uniform(0.5, 1.5, b.n_grasps).astype(np.float32), r.uniform(0.0, 0.2, b.n_qps).astype(np.float32)


def _fine(case, seed):
    """Fine-stage contacts drawn on the GPU (the distribution of
    workload.fine_contacts: a million grasps take seconds in numpy)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    G, m = case["grasps"], case["m"]
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    u = lambda *s: torch.rand(s, generator=g, device="cuda")
    unit = lambda v: v / v.norm(dim=-1, keepdim=True)
    f = object.__new__(api.DeviceFineContacts)
    f.obj_coarse = (0.02 + 0.06 * u(G, 1, 3)) * unit(n(G, m, 3))
    f.obj_fine = f.obj_coarse + 1e-3 * n(G, m, 3)
    f.hand_fine = f.obj_fine + 2e-3 * n(G, m, 3)
    w, x, y, z = unit(n(G, m, 4)).unbind(-1)
    f.link_rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                              2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                              2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                             -1).reshape(G, m, 3, 3).contiguous()
    f.link_trans = f.hand_fine - 0.02 * unit(n(G, m, 3))
    f.counts = torch.full((G,), m, dtype=torch.int32, device="cuda")
    f.w_q, f.w_e = 0.5 + 1.5 * u(G), 0.5 + 1.5 * u(G)
    f.n_grasps, f.m = G, m
    return f


def prepare(case, seed):
    kind = case["kind"]
    if kind == "detach":
        fc = _fine(case, seed)
        sv = api.Solver(api.default_params(m_max=case["m"]))
        G, m = case["grasps"], case["m"]
        e = lambda *s: torch.empty(s, device="cuda")
        return dict(kind=kind, solver=sv, fc=fc, out={"q_surr": e(G), "e_dist": e(G), "dL_dR": e(G, m, 3, 3),
                                                      "dL_dT": e(G, m, 3)})
    if kind == "descent":
        hand = api.DeviceHand(wl.hand_batch(seed, case["grasps"], m=case["m"], s=case["s"]))
        sv = api.Solver(api.default_params(m_max=case["m"], s_max=case["s"]))
        res = api.new_result(hand.n_grasps, hand.n_qps, case["m"])
        return dict(kind=kind, solver=sv, hand=hand, rot0=hand.rot.clone(), trans0=hand.trans.clone(), res=res,
                    d=api.descent(iters=case["steps"]))
    b = _batch(case, seed)
    p = _params(case, b)
    db = api.DeviceBatch(b)
    if kind == "autograd":
        we, wq = (torch.as_tensor(w, device="cuda") for w in _weights(b, seed))
        return dict(kind=kind, batch=db, params=p, we=we, wq=wq, p=db.points.clone().requires_grad_(True),
                    n=db.normals.clone().requires_grad_(True))
    s = dict(kind=kind, batch=db, state=api.new_state(db.n_grasps, db.n_qps, db.m_max, cone=case["cone"]),
             res=api.new_result(db.n_grasps, db.n_qps, db.m_max))
    if case["graph"]:  # graphs are captured on a stream of the program's own
        p.flags |= api.F_BATCHED | api.F_GRAPH
        s["stream"] = torch.cuda.Stream()
        s["stream"].wait_stream(torch.cuda.current_stream())
        s["solver"] = api.Solver(p, stream=s["stream"].cuda_stream)
        return s
    s["ones"] = torch.ones(db.n_grasps, device="cuda")
    s["grad"] = (torch.zeros_like(db.points), torch.zeros_like(db.normals))
    if kind == "step":  # the state the request's last step left
        first = api.Solver(p)
        first.solve(db, state=s["state"], result=s["res"])
        torch.cuda.synchronize()
        first.close()
        p.flags |= api.F_WARM_START
        s["at"], s["points"] = 0, [torch.as_tensor(q, device="cuda") for q in _walk(b, seed)]
    s["solver"] = api.Solver(p)
    return s


# ---------------------------------------------------------------------------
# One pass.  kkt_rel is left out of what comes back (a residual of about 1e-7
# made of rounding alone), and so are the duals y of a warm state: a contact
# without force has eight active facets in three variables, so they are not
# unique.
# ---------------------------------------------------------------------------

def _results(r):
    return {k: r[k] for k in ("forces", "qp_obj", "energy", "iters", "status")}


def run(s):
    kind = s["kind"]
    if kind == "detach":
        return s["solver"].detach_energy(s["fc"], out=s["out"])
    if kind == "descent":
        s["hand"].rot.copy_(s["rot0"])
        s["hand"].trans.copy_(s["trans0"])
        r, trace = s["solver"].descend(s["hand"], s["d"], result=s["res"])
        return {**_results(r), "trace": trace, "rot": s["hand"].rot, "trans": s["hand"].trans}
    db = s["batch"]
    if kind == "autograd":
        E, Q, f = autograd.BodexQPEnergy.apply(s["p"], s["n"], db.mu, db.wrench, db.woff, db.counts, s["params"])
        gp, gn = torch.autograd.grad([E, Q], [s["p"], s["n"]], [s["we"], s["wq"]])
        return {"forces": f, "qp_obj": Q.detach(), "energy": E.detach(), "dP": gp, "dN": gn}
    if kind == "step":
        db.points = s["points"][s["at"]]
        s["at"] ^= 1
    r = s["solver"].solve(db, state=s["state"], result=s["res"])
    out = _results(r)
    if kind in ("step", "gradient"):
        out["dP"], out["dN"] = s["solver"].backward(db, s["state"], dL_dE=s["ones"], out=s["grad"])
    if kind == "step":
        out.update({k: s["state"][k] for k in ("x", "z", "rho", "r")})
    return out


def _sizes(case):
    if case["m"] == 45:  # the means of the mixed batch
        return 4.5, 5, 19.0 * case["grasps"]
    return case["m"], case["m"], (6 if case.get("axes") else case["s"]) * case["grasps"]


def work(case):
    """Inputs read once and outputs written once; of arithmetic, per QP one
    6 x 6 matrix of the active rows formed and factored, one solve with it
    and the objective (the gradient's G-bar and chain rule where asked for)."""
    G = case["grasps"]
    if case["kind"] == "detach":
        n = G * case["m"]
        return {"bytes": n * 132 + G * 20, "flops": n * 150}
    if case["kind"] == "descent":
        n = case["steps"]
        W = G * case["s"]
        return {"bytes": G * case["m"] * 16 + W * 24 + G * 108 + W * (12 * case["m"] + 13) + n * G * 4,
                "flops": n * W * (375.0 * case["m"] + 200)}
    m, mm, W = _sizes(case)
    b = G * mm * 28 + W * 24 + W * (12 * mm + 9) + G * 4
    f = W * (339.0 * m + 172)
    if case["kind"] in ("step", "gradient", "autograd"):
        b += G * mm * 24
        f += W * 36.0 * m + G * 150.0 * m
    if case["kind"] == "step":
        b += 2 * W * 4 * (3 * mm + 2 * (9 * mm + 1)) + W * 24
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The same in 64 bits.
# ---------------------------------------------------------------------------

_C8, _TAN = math.cos(math.pi / 8), math.tan(math.pi / 8)


def _frames(n):
    n = n / n.norm(dim=-1, keepdim=True)
    x, y, z = n.unbind(-1)
    s = torch.where(torch.signbit(z), -torch.ones_like(z), torch.ones_like(z))
    a = -1 / (s + z)
    d = torch.stack([1 + s * x * x * a, s * x * y * a, -s * x], -1)
    e = torch.stack([x * y * a, s + y * y * a, -y], -1)
    return torch.stack([n, d, e], -2)


def _grasp(p, n):
    """[G, m, 3, 6]: the rows of G^T, three per contact."""
    c = _frames(n)
    return torch.cat([c, KAPPA * torch.cross(p[:, :, None, :].expand_as(c), c, dim=-1)], -1)


def _project(y, mu, cone):
    """P_C(y) per contact and rows B with B^T B its derivative."""
    y1, y2, y3 = y.unbind(-1)
    if cone:
        r = torch.hypot(y2, y3)
        rs = torch.where(r > 0, r, torch.ones_like(r))
        c, s = torch.where(r > 0, y2 / rs, torch.ones_like(r)), torch.where(r > 0, y3 / rs, torch.zeros_like(r))
        p, q, k, kt = r, torch.zeros_like(r), mu, torch.full_like(mu, math.inf)
        sg = torch.ones_like(r)
    else:  # fold onto the facet whose normal is nearest
        ph = (2 * torch.floor(torch.atan2(y3, y2) / (math.pi / 4)) + 1) * (math.pi / 8)
        c, s = torch.cos(ph), torch.sin(ph)
        p, q = c * y2 + s * y3, c * y3 - s * y2
        sg = torch.where(q < 0, -torch.ones_like(q), torch.ones_like(q))
        q, k = q.abs(), mu * _C8
        kt = k * _TAN
    inside = p <= k * y1
    ff = (y1 + k * p) / (1 + k * k)
    edge = ~inside & (q > kt * ff) if not cone else torch.zeros_like(inside)
    fe = (y1 + k * p + kt * q) / (1 + k * k + kt * kt) if not cone else ff
    f1 = torch.where(inside, y1, torch.where(edge, fe, ff))
    apex = ~inside & (f1 <= 0)
    cap = ~apex & (f1 > FMAX)
    z = torch.zeros_like(p)
    fp = torch.where(apex, z, torch.where(cap, torch.minimum(p, k * FMAX), torch.where(inside, p, k * f1)))
    fq = torch.where(apex, z, torch.where(cap, torch.where(p > k * FMAX, torch.minimum(q, kt * FMAX), q),
                                          torch.where(edge, kt * f1, q)))
    f1 = torch.where(apex, z, torch.where(cap, torch.full_like(f1, FMAX), f1))
    f = torch.stack([f1, c * fp - s * sg * fq, s * fp + c * sg * fq], -1)
    free = inside & ~cap
    ray = ~inside & ~apex & ~cap
    n1 = torch.where(edge, (1 + k * k + kt * kt) if not cone else 1 + k * k, 1 + k * k).rsqrt()
    a1 = torch.where(free, torch.ones_like(z), torch.where(ray, n1, z))
    a2 = torch.where(ray, n1 * k, z)
    a3 = torch.where(ray & edge, n1 * kt, z) if not cone else z
    rows = [torch.stack([a1, c * a2 - s * sg * a3, s * a2 + c * sg * a3], -1)]
    flat = free | (cap & (p <= k * FMAX))
    w2 = flat.to(z.dtype)
    rows.append(torch.stack([z, w2 * c, w2 * s], -1))
    if cone:  # across the axis the radius turns: |f_t| / |y_t|
        w3 = torch.where(flat, torch.ones_like(z), torch.where(ray | cap, fp / rs, z)).sqrt()
    else:
        w3 = (flat | (ray & ~edge) | (cap & (p > k * FMAX) & (q < kt * FMAX))).to(z.dtype)
    rows.append(torch.stack([z, -w3 * s * sg, w3 * c * sg], -1))
    return f, torch.stack(rows, -2)


def _newton(u, fb, sig, G, mu, t, cone, most, tol):
    """Newton with an exact line search on G P((G^T u + sig fb) / (eps + sig))
    + u = t; returns u, f and which QPs are not done."""
    e = EPS + sig
    u = u.clone()
    f = fb.clone()
    live = torch.arange(u.shape[0], device=u.device)
    for it in range(most + 1):
        Gl, ml, tl, ul = G[live], mu[live], t[live], u[live]
        y = (torch.einsum("wmck,wk->wmc", Gl, ul) + sig * fb[live]) / e
        fl, B = _project(y, ml, cone)
        f[live] = fl
        F = torch.einsum("wmck,wmc->wk", Gl, fl) + ul - tl
        keep = F.abs().amax(1) > tol
        if it == most or not bool(keep.any()):
            return u, f, live[keep]
        live, Gl, ml, tl, ul, y, B, F = live[keep], Gl[keep], ml[keep], tl[keep], ul[keep], y[keep], B[keep], F[keep]
        A = torch.einsum("wmbc,wmck->wmbk", B, Gl).flatten(1, 2)
        M = (A[:, :, :, None] * A[:, :, None, :]).sum(1) + e * torch.eye(6, dtype=u.dtype, device=u.device)
        for j in range(6):  # Cholesky and solve, entry by entry over the batch
            M[:, j, j] = (M[:, j, j] - (M[:, j, :j] ** 2).sum(-1)).clamp_min(1e-300).sqrt()
            for i in range(j + 1, 6):
                M[:, i, j] = (M[:, i, j] - (M[:, i, :j] * M[:, j, :j]).sum(-1)) / M[:, j, j]
        d = -e * F
        for i in range(6):
            d[:, i] = (d[:, i] - (M[:, i, :i] * d[:, :i]).sum(-1)) / M[:, i, i]
        for i in range(5, -1, -1):
            d[:, i] = (d[:, i] - (M[:, i + 1:, i] * d[:, i + 1:]).sum(-1)) / M[:, i, i]
        g0 = (F * d).sum(1)
        dy = torch.einsum("wmck,wk->wmc", Gl, d) / e
        du = (d * (ul - tl)).sum(1)
        dd = (d * d).sum(1)

        def slope(a):
            return e * (dy * _project(y + a[:, None, None] * dy, ml, cone)[0]).sum((1, 2)) + du + a * dd

        lo, hi = torch.zeros_like(g0), torch.ones_like(g0)
        a, g = hi.clone(), slope(hi)
        full = g <= 0
        for k in range(60):
            ok = full | (g.abs() <= 1e-3 * g0.abs())
            if bool(ok.all()):
                break
            lo, hi = torch.where(~ok & (g < 0), a, lo), torch.where(~ok & (g > 0), a, hi)
            mid = torch.where(lo > 0.05 * hi, 0.5 * (lo + hi), torch.where(lo > 0, (lo * hi).sqrt(), 0.05 * hi))
            a = torch.where(ok, a, mid)
            g = torch.where(ok, g, slope(a))
        u[live] = ul + a[:, None] * d


def _minimise(G, mu, t, cone):
    """[W, m, 3] forces of the QPs, in 64 bits."""
    W, m = G.shape[:2]
    f = torch.zeros((W, m, 3), dtype=G.dtype, device=G.device)
    left = torch.arange(W, device=G.device)
    fb, r = f.clone(), t.clone()
    for cycle in range(30):
        Gl, ml, tl = G[left], mu[left], t[left]
        fl, u = fb[left], r[left]
        sig = 1.0 if cycle == 0 else 10.0 ** -(1 + cycle % 4)
        while sig > 3e-6:  # proximal steps of falling weight around the last point
            u, fl, _ = _newton(u, fl, sig, Gl, ml, tl, cone, 2, 1e-7)
            sig *= 0.3
        fb[left], r[left] = fl, u
        u, fl, bad = _newton(u, fl, 0.0, Gl, ml, tl, cone, 40, 2e-9)
        f[left] = fl
        left = left[bad]
        if left.numel() == 0:
            return f
    return None


def _exact_batch(case, seed):
    b = _batch(case, seed)
    if case["kind"] == "step":
        b.points = _walk(b, seed)[0]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    d = lambda a: torch.as_tensor(a, device=dev).to(torch.float64)
    P, N = d(b.points).requires_grad_(True), d(b.normals).requires_grad_(True)
    of = torch.as_tensor(np.repeat(np.arange(b.n_grasps), np.diff(b.woff)), device=dev)
    live = torch.as_tensor(np.arange(b.m_max)[None, :] < b.counts[:, None], device=dev)
    Gg = _grasp(P, N) * live[:, :, None, None]
    G, t = Gg[of], case["beta"] * d(b.wrench)
    with torch.no_grad():
        f = _minimise(G.detach(), d(b.mu)[of], t, case["cone"])
    if f is None:
        return None
    Q = (torch.einsum("wmck,wmc->wk", G, f) - t).square().sum(1) + EPS * f.square().sum((1, 2))
    E = torch.zeros(b.n_grasps, dtype=Q.dtype, device=dev).index_add(0, of, Q)
    out = {"forces": f.flatten(1), "qp_obj": Q.detach(), "energy": E.detach()}
    if case["kind"] in ("step", "gradient", "autograd"):
        we, wq = (d(w) for w in _weights(b, seed)) if case["kind"] == "autograd" else (1.0, 0.0)
        out["dP"], out["dN"] = torch.autograd.grad((we * E).sum() + (wq * Q).sum(), [P, N])
    return out


def _exact_detach(case, seed):
    f = _fine(case, seed)
    R, T, cw, pf, pc, wq, we = (v.double() for v in (f.link_rot, f.link_trans, f.hand_fine, f.obj_fine,
                                                    f.obj_coarse, f.w_q, f.w_e))
    a, b, c = R.unbind(-1)  # columns; the inverse's rows are cross products of them
    det = (a * torch.cross(b, c, dim=-1)).sum(-1, keepdim=True)
    v = cw - T
    cl = torch.stack([(torch.cross(b, c, dim=-1) * v).sum(-1), (torch.cross(c, a, dim=-1) * v).sum(-1),
                      (torch.cross(a, b, dim=-1) * v).sum(-1)], -1) / det
    cp = (R * cl[..., None, :]).sum(-1) + T
    g = 2 * wq[:, None, None] * (cp - pc) + 2 * we[:, None, None] * (cp - pf)
    return {"q_surr": (cp - pc).square().sum((1, 2)), "e_dist": (cp - pf).square().sum((1, 2)),
            "dL_dR": g[..., :, None] * cl[..., None, :], "dL_dT": g}


def exact(case, seed):
    if case["kind"] == "detach":
        return _exact_detach(case, seed)
    # many steps of a descent, and the row that couples the contacts (the
    # dual then has another, inequality-constrained variable): no closed form
    if case["kind"] == "descent" or case["gamma"] > 0:
        return None
    return _exact_batch(case, seed)
