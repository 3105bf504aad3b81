"""CPU: where the compacted sum is declined because the mirror is deep or the wave long."""
import math

import numpy as np
import pytest

from test_compact_plan import CSRC, ROOT, kernels  # noqa: F401

import ctypes
import os
import subprocess

WRAP = r'''
#include "sc_compact.h"
extern "C" int plan(double f, double r_max, int n_r, int n_phi, double k_min, double k_max, int n_k, int n_obs_pad,
                    double r2, double rho2, int fp64, int *head, int *cols, double *geo)
{
    sc::CompactInput in{f, r_max, n_r, n_phi, k_max, k_min, n_k, n_obs_pad, r2, rho2, fp64 != 0};
    sc::CompactPlan p;
    if (!sc::compact_plan(in, p)) return 0;
    head[0] = p.rows; head[1] = p.n_c; head[2] = p.split; head[3] = p.chunk; head[4] = p.form; head[5] = p.fold;
    for (int m = 0; m < p.rows; ++m) cols[m] = p.cols[m];
    geo[0] = p.theta_max;
    geo[1] = p.alpha;
    return 1;
}
'''


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("limits")
    (d / "wrap.cpp").write_text(WRAP)
    so = d / "plan.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "wrap.cpp"),
                    os.path.join(CSRC, "sc_compact_host.cpp"), "-o", str(so)], check=True)
    fn = ctypes.CDLL(str(so)).plan

    def call(f, a, n_r, n_phi, k_min, k_max, n_k, pad, rp, rho, fp64):
        head, cols, geo = (ctypes.c_int * 6)(), (ctypes.c_int * 192)(), (ctypes.c_double * 2)()
        D = ctypes.c_double
        if not fn(D(f), D(a), n_r, n_phi, D(k_min), D(k_max), n_k, pad, D(rp * rp), D(rho * rho), int(fp64), head, cols,
                  geo):
            return None
        return dict(zip(("rows", "n_c", "split", "chunk", "form", "fold"), head), cols=list(cols[: head[0]]),
                    theta_max=geo[0], alpha=geo[1])
    return call


def local_error(p, f, k, rp, rho):
    """Largest error of the interpolation in theta, relative to the kernel at the same place."""
    theta = lambda y: p["theta_max"] * np.arcsin(np.minimum(p["alpha"] * y, 1.0)) / math.asin(p["alpha"])  # noqa: E731
    z, N = math.sqrt(rp * rp - rho * rho), 2 * p["rows"]
    x = np.cos((2 * np.arange(N) + 1) * np.pi / (2 * N))
    w = (-1.0) ** np.arange(N) * np.sin((2 * np.arange(N) + 1) * np.pi / (2 * N))
    xs = np.linspace(-1, 1, 401)
    D = xs[:, None] - x[None]
    hit = np.abs(D) < 1e-14
    L = w / np.where(hit, 1.0, D)
    L = np.where(hit.any(1, keepdims=True), hit, L / L.sum(1, keepdims=True))
    worst = 0.0
    for r in ([rho, 0, z], [rho, 0, -z], [0, 0, z], [0.6 * rho, 0.8 * rho, z]):
        for ph in (0.0, 0.9, np.pi):
            full = kernels(theta(xs), np.full_like(xs, ph), k, f, np.array(r, float))
            at = kernels(theta(np.abs(x)), np.where(x > 0, ph, ph + np.pi), k, f, np.array(r, float))
            size = np.stack([np.abs(full[:, 0])] + [np.linalg.norm(full[:, 1:], axis=1)] * 3, 1)
            worst = max(worst, (np.abs(L @ at - full) / size).max())
    return worst


@pytest.mark.parametrize("af", [1.0, 3.0, 5.0, 5.2, 6.0, 12.0, 40.0])
@pytest.mark.parametrize("f,rp", [(20.0, 2.0), (20.0, 4.8), (1e5, 3.0)])
def test_deep_mirrors(planner, af, f, rp):
    """To the kernel's own size everywhere (1e-7 in FP32; 1e-14 in FP64 times what the double-precision sums of this
    test round, the rim's kernel being rim/f times the smaller), or the direct sum."""
    k, rim = 2 * math.pi, 1 + af * af / 4
    for fp64 in (False, True):
        p = planner(f, af * f, 800, 800, k, k, 8, 1024, rp, 0.7 * rp, fp64)
        assert (p is None) == (rim > 8.0)
        if p:
            tol = 4e-14 + 3e-16 * rim * max(10.0, k * rp) if fp64 else 1e-7
            assert local_error(p, f, k, rp, 0.7 * rp) < tol


def test_long_waves(planner):
    """A frequency whose wave is longer than 64 pi f: the FP32 form is left to the direct sum, FP64 is not."""
    args = dict(f=10.0, a=15.0, n_r=200, n_phi=240, k_max=2 * math.pi, n_k=2, pad=512, rp=1.0, rho=0.7)
    for k_min, taken in ((1.0, True), (0.0032, True), (0.0031, False), (1e-6, False)):
        assert (planner(k_min=k_min, fp64=False, **args) is not None) == taken
        assert planner(k_min=k_min, fp64=True, **args) is not None
