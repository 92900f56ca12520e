"""The dual Newton polish on the host where the rounding of its dual variable
matters: right-hand sides of 10 to 1000 instead of 1 and torque arms of 5 to
200 instead of 1.  Every QP has to be solved within the default step cap, cold,
and to the minimiser, which Newton's method in 128 bits gives with F = 0 for
its certificate.

Tolerance: 2e-8 is two thirds of what 32-bit forces are rounded by; the dual's
own rounding, were it not carried in two doubles, is 1.4e-7 at |bt| 1000."""
import ctypes
import os

import numpy as np
import pytest

import host_build
from paper_2412_16490_amd import workload as wl

HERE = os.path.dirname(os.path.abspath(__file__))
EPS = float(np.float32(1e-6))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("newton_fine") / "libnewton_fine_host.so")
    host_build.build(os.path.join(HERE, "newton_fine_host.cpp"), out)
    return ctypes.CDLL(out)


def _solve(host, b, beta, kappa, cone=False, max_steps=128, fmax=1.0):
    f, info = np.zeros((b.n_qps, 3 * b.m_max)), np.zeros((b.n_qps, 2), np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    c = lambda a: np.ascontiguousarray(a, np.float64)
    for g in range(b.n_grasps):
        m, a, e = int(b.counts[g]), int(b.woff[g]), int(b.woff[g + 1])
        P, N, mu, T = c(b.points[g, :m]), c(b.normals[g, :m]), c(b.mu[g, :m]), c(beta * b.wrench[a:e].astype(float))
        ff, ii = np.zeros((e - a, 3 * m)), np.zeros((e - a, 2), np.int32)
        host.host_newton_fine(int(cone), m, ptr(P), ptr(N), ptr(mu), ptr(T), e - a, ctypes.c_double(kappa),
                              ctypes.c_double(EPS), ctypes.c_double(fmax), max_steps, ptr(ff), ptr(ii))
        f[a:e, :3 * m], info[a:e] = ff, ii
    return f, info


def _exact(host, b, beta, kappa, f0, cone=False, fmax=1.0):
    f = np.zeros_like(f0)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    c = lambda a: np.ascontiguousarray(a, np.float64)
    host.host_newton_exact.restype = ctypes.c_double
    for w in range(b.n_qps):
        g = int(np.searchsorted(b.woff, w, side="right") - 1)
        m = int(b.counts[g])
        P, N, mu, T = c(b.points[g, :m]), c(b.normals[g, :m]), c(b.mu[g, :m]), c(beta * b.wrench[w].astype(float))
        x0, x = c(f0[w, :3 * m]), np.zeros(3 * m)
        res = host.host_newton_exact(int(cone), m, ptr(P), ptr(N), ptr(mu), ptr(T), ctypes.c_double(kappa),
                                     ctypes.c_double(EPS), ctypes.c_double(fmax), ptr(x0), ptr(x))
        assert res < 1e-20, "QP %d: |F| %.1e in 128 bits" % (w, res)
        f[w, :3 * m] = x
    return f


CASES = [(10.0, 20.0), (100.0, 20.0), (1000.0, 20.0), (1.0, 100.0), (1.0, 1000.0), (1.0, 4000.0), (100.0, 1000.0)]


@pytest.mark.parametrize("m", [3, 5, 8])
@pytest.mark.parametrize("beta,kappa", CASES)
def test_large_right_hand_sides_and_torque_arms(host, m, beta, kappa):
    b = wl.uniform_batch(30 + m, 40, m, 9)
    f, info = _solve(host, b, beta, kappa)
    assert np.all(info[:, 0] == 1), "%d of %d QPs not solved" % ((info[:, 0] != 1).sum(), len(info))
    assert np.abs(f - _exact(host, b, beta, kappa, f)).max() <= 2e-8


@pytest.mark.parametrize("m", [3, 5])
@pytest.mark.parametrize("beta,kappa", [(100.0, 20.0), (1000.0, 20.0)])
def test_cone_with_large_right_hand_sides(host, m, beta, kappa):
    b = wl.uniform_batch(30 + m, 40, m, 9)
    f, info = _solve(host, b, beta, kappa, cone=True)
    assert np.all(info[:, 0] == 1)
    assert np.abs(f - _exact(host, b, beta, kappa, f, cone=True)).max() <= 2e-8


# a force_max that stands for "no limit" (the forces stay below 200, rounded to
# 32 bits by up to 8e-6)
@pytest.mark.parametrize("cone", [False, True])
@pytest.mark.parametrize("beta", [1.0, 1e-6])
@pytest.mark.parametrize("fmax", [1e6, 1e10, 1e30])
def test_force_limits_no_force_reaches(host, cone, beta, fmax):
    b = wl.uniform_batch(36, 40, 5, 9)
    f, info = _solve(host, b, beta, 20.0, cone=cone, fmax=fmax)
    assert np.all(info[:, 0] == 1)
    assert np.abs(f - _exact(host, b, beta, 20.0, f, cone=cone, fmax=fmax)).max() <= 1e-6 * beta
