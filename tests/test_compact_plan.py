"""CPU: the compacted sum's plan (sc_compact_host.cpp) interpolates the kernel to its error.

The plan replaces K(o, n) by sum_m L_m(n) K(o, m), Chebyshev in theta on [-theta_max, theta_max] (theta < 0
is theta > 0 at phi + pi) by polynomials in y, theta = theta_max asin(alpha y) / asin(alpha), and trigonometric
in phi, where
K runs over e^{ik delta} / R and (ik - 1/R) e^{ik delta} R_vec / R^2, delta = |r_s - r'| - |r_s|.  Here
that interpolation is formed with numpy from the plan's rows and columns alone, at points r' on the
sphere and the cylinder that the plan was given, and held to the error the planner aims at (1e-7 in
the FP32 form, 1e-14 in FP64, relative to the largest kernel value, times the interpolation's own
rounding in double precision: at most 1e-15 k |r'| for the phase and a Lebesgue factor below 10).
"""
import ctypes
import math
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1609_08146_amd", "csrc")

WRAP = r'''
#include "sc_compact.h"
extern "C" int plan(double f, double r_max, int n_r, int n_phi, double k_max, int n_k, int n_obs_pad, double r2,
                    double rho2, int fp64, int *head, int *cols, double *theta_max)
{
    sc::CompactInput in{f, r_max, n_r, n_phi, k_max, k_max, n_k, n_obs_pad, r2, rho2, fp64 != 0};
    sc::CompactPlan p;
    if (!sc::compact_plan(in, p)) return 0;
    head[0] = p.rows; head[1] = p.n_c; head[2] = p.split; head[3] = p.chunk;
    for (int m = 0; m < p.rows; ++m) cols[m] = p.cols[m];
    theta_max[0] = p.theta_max;
    theta_max[1] = p.alpha;
    long long work = 8 * (sc::compact_radial_doubles(p, n_r) + sc::compact_angular_doubles(p, n_phi) +
                          sc::compact_rows_doubles(p, n_phi));
    return work <= sc::COMPACT_WORK_MAX ? 1 : -1;
}
'''


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "wrap.cpp").write_text(WRAP)
    so = d / "plan.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "wrap.cpp"),
                    os.path.join(CSRC, "sc_compact_host.cpp"), "-o", str(so)], check=True)
    fn = ctypes.CDLL(str(so)).plan

    def call(f, a, n_r, n_phi, k, n_k, pad, rp, rho, fp64):
        head, cols, th = (ctypes.c_int * 4)(), (ctypes.c_int * 192)(), (ctypes.c_double * 2)()
        D = ctypes.c_double
        got = fn(D(f), D(a), n_r, n_phi, D(k), n_k, pad, D(rp * rp), D(rho * rho), int(fp64), head, cols, th)
        assert got >= 0, "working memory over its bound"
        return (list(head), list(cols[: head[0]]), th[0], th[1]) if got else None
    return call


def kernels(theta, phi, k, f, rp):
    """g and the three components of h R on a grid of directions, each over its largest size."""
    st, ct = np.sin(theta), np.cos(theta)
    r0 = f / np.cos(theta / 2) ** 2
    rs = np.stack([r0 * st * np.cos(phi), r0 * st * np.sin(phi), -r0 * ct], -1)
    d = rs - rp
    R = np.linalg.norm(d, axis=-1)
    g = np.exp(1j * k * (rp @ rp - 2 * rs @ rp) / (R + r0)) / R
    return np.concatenate([(g * f)[..., None], ((1j * k - 1 / R) * g / R)[..., None] * d * (f / k)], -1)


def check(p, n_phi, f, k, rp, rho, eps):
    (rows, n_c, split, chunk), cols, thm, alpha = p
    assert n_c == sum(cols) and split >= 1 and chunk % 32 == 0 and chunk >= 64
    theta = lambda y: thm * np.arcsin(np.minimum(alpha * y, 1.0)) / math.asin(alpha)
    z = math.sqrt(max(rp * rp - rho * rho, 0.0))
    N = 2 * rows
    x = np.cos((2 * np.arange(N) + 1) * np.pi / (2 * N))
    w = (-1.0) ** np.arange(N) * np.sin((2 * np.arange(N) + 1) * np.pi / (2 * N))
    xs = np.linspace(-1, 1, 157)
    D = xs[:, None] - x[None]
    hit = np.abs(D) < 1e-14
    L = w / np.where(hit, 1.0, D)
    L = np.where(hit.any(1, keepdims=True), hit, L / L.sum(1, keepdims=True))
    pts = [np.array(v, float) for v in ([rho, 0, z], [rho, 0, -z], [0.6 * rho, 0.8 * rho, z], [0, 0, z], [rho, 0, 0])]
    tol = eps + 1e-14 * max(10.0, k * rp)
    for r in pts:
        for ph in (0.0, 0.9, np.pi):
            full = kernels(theta(xs), np.full_like(xs, ph), k, f, r)
            at = kernels(theta(np.abs(x)), np.where(x > 0, ph, ph + np.pi), k, f, r)
            assert np.abs(np.einsum("im,mc->ic", L, at) - full).max() < tol
        for m in range(0, rows, max(1, rows // 5)):
            P = cols[m]
            own = n_phi if n_phi % 2 == 0 else 2 * n_phi
            if P == own:
                continue   # the grid's own columns and those + pi
            assert P % 2 == 1 and P < own
            phi = np.linspace(0, 2 * np.pi, 301)[:-1] + 0.0123
            psi = 2 * np.pi * np.arange(P) / P
            u = (phi[:, None] - psi[None]) / 2
            Dk = np.sin(P * u) / (P * np.sin(u))
            th = np.full_like(phi, theta(x[m]))
            full = kernels(th, phi, k, f, r)
            # (numpy's sin(P u) / sin(u) itself rounds by about 1e-16 P / u at the nodes nearest phi)
            assert np.abs(Dk @ kernels(np.full(P, th[0]), psi, k, f, r) - full).max() < tol + 1e-15 * P * P
    return n_c


@pytest.mark.parametrize("fp64", [False, True])
def test_plan_interpolates_the_kernel(planner, fp64):
    rng = random.Random(5)
    lam = 800e-9
    taken = 0
    for _ in range(60):
        f = math.exp(rng.uniform(math.log(5.0), math.log(2e5)))            # wavelengths
        a = f * rng.uniform(0.1, 3.0)
        n_r, n_phi = rng.randint(24, 500), rng.randint(24, 500)
        rp = min(math.exp(rng.uniform(math.log(0.2), math.log(30.0))), 0.3 * f)
        rho = rp * rng.choice([0.0, 0.5, 1.0])
        s = rng.choice([1.0, lam])
        p = planner(f * s, a * s, n_r, n_phi, 2 * math.pi / s, rng.choice([1, 5, 64]), 128 * rng.randint(1, 40), rp * s,
                    rho * s, fp64)
        if p is None:
            continue
        taken += 1
        assert rp / f <= 0.25
        n_c = check(p, n_phi, f * s, 2 * math.pi / s, rp * s, rho * s, 1e-14 if fp64 else 1e-7)
        assert 2 * n_c <= (n_r + 1) * n_phi
    assert taken >= 15


def test_plan_declines(planner):
    ok = dict(f=20.0, a=30.0, n_r=200, n_phi=200, k=2 * math.pi, n_k=4, pad=1024, rp=1.0, rho=1.0, fp64=False)
    assert planner(**ok) is not None
    for change in (dict(rp=6.0, rho=6.0),           # |r'| > f / 4: near the singularity of the kernel
                   dict(n_r=12, n_phi=16),           # no finer than the interpolation
                   dict(rp=math.inf, rho=0.0), dict(rp=math.nan, rho=0.0), dict(k=1e300), dict(f=0.0)):
        assert planner(**{**ok, **change}) is None, change
