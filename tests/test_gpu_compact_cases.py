"""GPU: the compacted sum against the oracle at the sizes of which its kernels' branches depend.

The planner is compiled for the test, which asserts that the problem is compacted, that the branch named is the one
taken, and that the evaluation's tiles are the compacted sum's.  Random incident tables; tolerances: relative L2 1e-12
in FP64, 2e-6 in the FP32 form, and 4 k |r'| roundings of the phase besides.
"""
import numpy as np
import pytest

import workloads
from test_compact_limits import planner  # noqa: F401

pytestmark = pytest.mark.gpu
K = 2 * np.pi
TOL = {"fp64": (1e-12, 2.0 ** -52), "fp32_split": (2e-6, 2.0 ** -24)}
GH, GH_FAR, NEAR = 0, 1, 2


def rel_l2(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


# f, aperture, n_r, n_phi, frequencies, largest |r'|, points, what the plan has to be
CASES = {
    "odd n_phi, radii in parts": (20.0, 30.0, 150, 161, 1, 0.8, 2000, lambda p: p["fold"] == 0 and p["split"] > 2),
    "even n_phi, radii in parts": (20.0, 30.0, 200, 160, 1, 0.8, 2000, lambda p: p["fold"] == 1 and p["split"] > 2),
    "radii in one part": (20.0, 12.0, 60, 256, 40, 1.5, 500, lambda p: p["split"] == 1 and p["rows"] < 32),
    "past a group of 8 frequencies": (20.0, 12.0, 97, 256, 9, 2.0, 400, lambda p: p["rows"] < 32),
    "the grid's own columns, even": (20.0, 60.0, 260, 40, 3, 1.7, 3000, lambda p: p["cols"].count(40) > 5),
    "the grid's own columns, odd": (20.0, 60.0, 400, 31, 3, 2.2, 3000, lambda p: p["cols"].count(62) > 5),
    "all rows the grid's own": (20.0, 60.0, 600, 30, 4, 1.7, 1000, lambda p: p["cols"].count(30) > 0.8 * p["rows"]),
    "near |r'| = f / 4": (20.0, 40.0, 201, 200, 2, 4.9, 600, lambda p: p["rows"] > 40),
    "one kernel value, series": (1e5, 1.5e5, 150, 180, 5, 2.0, 700, lambda p: p["form"] == NEAR),
    "one kernel value, no series": (2e5, 8e3, 150, 180, 3, 140.0, 700, lambda p: p["form"] == NEAR),
    "two kernel values, one part": (900.0, 900.0, 150, 180, 3, 0.85, 700, lambda p: p["form"] == GH),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("prec", ["fp64", "fp32_split"])
def test_branches(orc, planner, name, prec):  # noqa: F811
    from paper_1609_08146_amd import Context, Problem
    f, a, nr, nphi, nk, rp, n, check = CASES[name]
    ks = K * np.linspace(0.9, 1.1, nk) if nk > 1 else np.array([K])
    rng = np.random.default_rng(n)
    obs = rng.uniform(-1.0, 1.0, (n, 3))
    obs *= rp / np.linalg.norm(obs, axis=1).max()
    r, rho = np.linalg.norm(obs, axis=1).max(), np.linalg.norm(obs[:, :2], axis=1).max()
    pad = -(-n // 128) * 128
    plan = planner(f, a, nr, nphi, ks.min(), ks.max(), nk, pad, r, rho, prec == "fp64")
    assert plan is not None, "the planner declines"
    assert check(plan), plan
    pick = slice(None, None, max(1, n // 25))
    m = orc.mirror(f, a, nr, nphi)
    Ei, Bi = workloads.random_incident_tables(nk, m.n_tot, seed=nr)
    Eo, Bo = orc.reflected_field(m, ks, Ei, Bi, obs[pick])
    ctx = Context(0)
    p = Problem(ctx)
    p.set_mirror(f, a, nr, nphi)
    p.set_frequencies(ks)
    p.set_incident(Ei, Bi)
    p.set_observation(obs)
    E, B = p.evaluate(prec)
    chunks = -(-plan["n_c"] // plan["chunk"])
    points = pad // (128 if prec == "fp32_split" else 64)
    assert p.timing()["tiles"] in [points * chunks * -(-nk // width) for width in (1, 2, 4)]
    assert max(rel_l2(E[:, pick], Eo), rel_l2(B[:, pick], Bo)) < TOL[prec][0] + 4 * ks.max() * r * TOL[prec][1]
    p.close()
    ctx.close()


@pytest.mark.parametrize("nphi", [2, 3, 4, 5])
def test_few_phi(orc, planner, nphi):  # noqa: F811
    """A handful of phi (their own columns in every row), 3 000 radii; and every point at the focus itself."""
    from paper_1609_08146_amd import Context, Problem
    f, a, nr, n = 30.0, 40.0, 3000, 6000
    ks = K * np.array([0.9, 1.0, 1.1])
    m = orc.mirror(f, a, nr, nphi)
    Ei, Bi = workloads.random_incident_tables(3, m.n_tot, seed=nphi)
    ctx = Context(0)
    p = Problem(ctx)
    p.set_mirror(f, a, nr, nphi)
    p.set_frequencies(ks)
    p.set_incident(Ei, Bi)
    for size in (1.0, 0.0):
        obs = np.random.default_rng(nphi).uniform(-1.0, 1.0, (n, 3)) * size
        r, rho = np.linalg.norm(obs, axis=1).max(), np.linalg.norm(obs[:, :2], axis=1).max()
        Eo, Bo = orc.reflected_field(m, ks, Ei, Bi, obs[::240])
        p.set_observation(obs)
        for prec in ("fp64", "fp32_split")[: 1 if nphi < 4 else 2]:      # (FP32: the direct sum is the faster one)
            plan = planner(f, a, nr, nphi, ks.min(), ks.max(), 3, -(-n // 128) * 128, r, rho, prec == "fp64")
            assert max(plan["cols"]) == (nphi if nphi % 2 == 0 else 2 * nphi)
            E, B = p.evaluate(prec)
            assert max(rel_l2(E[:, ::240], Eo), rel_l2(B[:, ::240], Bo)) < TOL[prec][0] + 4 * ks.max() * r * TOL[prec][1]
    p.close()
    ctx.close()
