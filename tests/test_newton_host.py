"""The dual Newton polish compiled for the host (the header the GPU kernels
use): its closed-form projection and derivative against independent ones, and
its forces against the oracles from cold and poor starting points.

Tolerances: the projection is a handful of FP64 operations on numbers of
order one (1e-12); the method stops at |F| <= 2e-9 |t|, which bounds a force
error by 2e-9 / sqrt(eps) = 2e-6 along the least determined direction; the
cone oracle (a barrier method) is itself good to about 2e-5."""
import ctypes
import os

import numpy as np
import pytest

import host_build
import oracle
from oracle import cone as oc
from paper_2412_16490_amd import workload as wl

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("newton_host") / "libnewton_host.so")
    host_build.build(os.path.join(HERE, "newton_host.cpp"), out)
    return ctypes.CDLL(out)


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _solve(host, b, g, x0, cone, fmax=1.0, max_steps=200):
    m, s = int(b.counts[g]), int(b.woff[g + 1] - b.woff[g])
    c = lambda a: np.ascontiguousarray(a, np.float64)
    P, N, mu, T = c(b.points[g, :m]), c(b.normals[g, :m]), c(b.mu[g, :m]), c(b.wrench[b.woff[g]:b.woff[g + 1]])
    x0, f, info = c(x0), np.zeros((s, 3 * m)), np.zeros((s, 2), np.int32)
    host.host_newton_grasp(int(cone), m, _p(P), _p(N), _p(mu), _p(T), s, _p(x0), ctypes.c_double(1e-6),
                           ctypes.c_double(fmax), max_steps, _p(f), _p(info))
    return f, info


def _project(host, y, mu, fmax, cone):
    y, f, d = np.ascontiguousarray(y, np.float64), np.zeros(3), np.zeros((3, 3))
    host.host_newton_project(int(cone), _p(y), ctypes.c_double(mu), ctypes.c_double(fmax), _p(f), _p(d))
    return f, d


@pytest.mark.parametrize("cone", [False, True])
def test_projection_is_the_closest_point_and_its_derivative(host, cone):
    # feasible, y - f in the normal cone (no vertex of the section, and not
    # the apex, is on the far side), and the derivative by central differences
    # (skipping points within the step of a region's edge)
    rng = np.random.default_rng(3)
    far = 0
    for _ in range(3000):
        mu, fmax = rng.uniform(0.2, 1.0), rng.uniform(0.5, 2.0)
        y = rng.standard_normal(3) * rng.choice([0.1, 1.0, 4.0])
        f, d = _project(host, y, mu, fmax, cone)
        k = np.arange(512 if cone else 8)
        ang = 2 * np.pi * k / len(k)
        V = fmax * np.stack([np.ones(len(k)), mu * np.cos(ang), mu * np.sin(ang)], 1)
        for v in [np.zeros(3), *V]:
            assert (y - f) @ (v - f) <= 1e-12 * (1 + np.abs(y).max() ** 2)
        assert -1e-12 <= f[0] <= fmax + 1e-12
        if cone:
            assert np.hypot(f[1], f[2]) <= mu * f[0] + 1e-12
        else:
            ph = (2 * np.arange(8) + 1) * np.pi / 8
            assert np.max(np.cos(ph) * f[1] + np.sin(ph) * f[2]) <= mu * np.cos(np.pi / 8) * f[0] + 1e-12
        h = 1e-6
        num = np.stack([(_project(host, y + h * e, mu, fmax, cone)[0] - _project(host, y - h * e, mu, fmax, cone)[0])
                        / (2 * h) for e in np.eye(3)], 1)
        far += np.abs(num - d).max() > 1e-3
    assert far <= 3  # 3000 points, a kink within 1e-6 of a few at most


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("start,fmax", [("cold", 1.0), ("poor", 1.0), ("poor", 0.05)])
def test_forces_are_the_oracles(host, m, start, fmax):
    b = wl.uniform_batch(40 + m, 12, m, 7)
    rng = np.random.default_rng(m)
    ref = oracle.solve_batch(b.counts, b.woff, b.points, b.normals, b.mu, b.wrench, oracle.params(fmax=fmax))
    for g in range(b.n_grasps):
        x0 = np.zeros((7, 3 * m)) if start == "cold" else rng.standard_normal((7, 3 * m)) * fmax
        f, info = _solve(host, b, g, x0, False, fmax=fmax)
        assert np.all(info[:, 0] == 1)
        assert np.abs(f - ref["forces"][b.woff[g]:b.woff[g + 1], :3 * m]).max() <= 2e-6


@pytest.mark.parametrize("m", [1, 3, 4, 5])
def test_cone_forces_are_the_oracles(host, m):
    b = wl.uniform_batch(60 + m, 6, m, 5)
    rng = np.random.default_rng(m)
    ref = oc.solve_batch(b.counts, b.woff, b.points, b.normals, b.mu, b.wrench)
    for g in range(b.n_grasps):
        f, info = _solve(host, b, g, 0.3 * rng.standard_normal((5, 3 * m)), True)
        assert np.all(info[:, 0] == 1)
        assert np.abs(f - ref["forces"][b.woff[g]:b.woff[g + 1], :3 * m]).max() <= 3e-5


def test_step_cap_is_reported(host):
    b = wl.uniform_batch(5, 2, 5, 6)
    f, info = _solve(host, b, 0, np.ones((6, 15)), False, max_steps=2)
    assert np.all(info[:, 0] == 0) and np.all(info[:, 1] <= 2)
