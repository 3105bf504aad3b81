"""GPU: the compacted sum (sc_compact.h) against the oracle, at the sizes where it can go wrong.

Random incident tables exercise it as a linear map of arbitrary records.  Sizes cover row counts off
the tiles of 16, an odd and an even number of phi, rows that keep the grid's own columns, one and many
frequencies (the interpolation takes 8 at a time), a sum over the radii cut in parts, all table
layouts, and points on the axis alone.  Tolerances as everywhere: relative L2 1e-12 in FP64 and
2e-6 in the FP32 split form (its direct sum is held to 1e-5).
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
K = 2 * np.pi
TOL = {"fp64": 1e-12, "fp32_split": 2e-6}


def rel_l2(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1609_08146_amd import Context
    c = Context(0)
    yield c
    c.close()


def direct_tiles(p, n_obs, n_k, prec):
    """Tiles of the direct sum in the problem's launch."""
    ns, nr = p.num_nodes()
    l = p.launch(prec)
    pad = -(-n_obs // 128) * 128
    return pad // (64 * l["obs_per_lane"]) * -(-(ns + nr) // l["chunk"]) * -(-n_k // l["freq_per_lane"])


# f, aperture, n_r, n_phi, frequencies, half width of the points, points
CASES = [
    (20.0, 30.0, 150, 161, 1, 0.5, 300),      # odd n_phi, one frequency: the radii in parts
    (20.0, 12.0, 97, 256, 9, 1.5, 200),       # one frequency past a group of 8; rows < 32
    (20.0, 60.0, 260, 40, 3, 1.0, 200),       # outer rows keep the grid's own 40 columns
    (20.0, 40.0, 201, 200, 2, 2.8, 150),      # |r'| near f / 4 (the corners of the cube)
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("prec", ["fp64", "fp32_split"])
def test_random_tables(ctx, orc, case, prec):
    from paper_1609_08146_amd import Problem
    f, a, nr, nphi, nk, half, n = case
    ks = K * np.linspace(0.9, 1.1, nk) if nk > 1 else np.array([K])
    obs = workloads.random_points(n, half, seed=7)
    m = orc.mirror(f, a, nr, nphi)
    Ei, Bi = workloads.random_incident_tables(nk, m.n_tot, seed=nr)
    Eo, Bo = orc.reflected_field(m, ks, Ei, Bi, obs[::17])
    p = Problem(ctx)
    p.set_mirror(f, a, nr, nphi)
    p.set_frequencies(ks)
    p.set_incident(Ei, Bi)
    p.set_observation(obs)
    E, B = p.evaluate(prec)
    assert p.timing()["tiles"] != direct_tiles(p, n, nk, prec), "the direct sum was taken"
    errs = rel_l2(E[:, ::17], Eo), rel_l2(B[:, ::17], Bo)
    print(case, prec, [f"{e:.1e}" for e in errs])
    assert max(errs) < TOL[prec]
    # new points (on the axis alone: few columns) and new tables on the same problem
    ax = np.stack([0 * obs[:, 0], 0 * obs[:, 0], np.linspace(-half, half, n)], -1)
    p.set_observation(ax)
    E, B = p.evaluate(prec)
    Eo, Bo = orc.reflected_field(m, ks, Ei, Bi, ax[::17])
    assert max(rel_l2(E[:, ::17], Eo), rel_l2(B[:, ::17], Bo)) < TOL[prec]
    p.set_incident(Bi, Ei)
    E, B = p.evaluate(prec)
    Eo, Bo = orc.reflected_field(m, ks, Bi, Ei, ax[::17])
    assert max(rel_l2(E[:, ::17], Eo), rel_l2(B[:, ::17], Bo)) < TOL[prec]
    p.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_split"])
def test_layouts_spectrum_and_evaluation_without_allocation(ctx, orc, prec):
    """Every table layout of one beam; after the layout, the spectrum or the points change, the
    results are those of a fresh problem bit for bit (nothing stale), and evaluate_noalloc has
    evaluate's bits, also where its scratch takes the frequencies in several slabs."""
    import torch
    from paper_1609_08146_amd import problem_from_workload
    w = workloads.broadband(n_k=20, n_nodes=180).subset(obs_idx=np.arange(0, 4160, 3))
    Eo, Bo = orc.solve(w.subset(obs_idx=np.arange(0, w.n_obs, 97)))
    p = problem_from_workload(ctx, w)
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    out = tuple(torch.empty((w.n_k, w.n_obs, 3), dtype=dt, device="cuda") for _ in range(2))
    fac = np.exp(1j * np.linspace(0, 3, w.n_k))
    res = {}
    for step in ("tied", "factored", "general", "scaled", "points"):
        if step in ("tied", "factored", "general"):
            p.set_factoring(step != "general", tie_charge=step == "tied")
        elif step == "scaled":
            p.scale_spectrum(fac)
        else:
            p.set_observation(w.obs[::-1] * 0.5)
        E, B = p.evaluate(prec)
        res[step] = E
        assert p.timing()["tiles"] != direct_tiles(p, w.n_obs, w.n_k, prec)
        if step in ("tied", "factored", "general"):
            assert max(rel_l2(E[:, ::97], Eo), rel_l2(B[:, ::97], Bo)) < TOL[prec]
        q = problem_from_workload(ctx, w)
        q.set_factoring(step in ("tied", "factored"), tie_charge=step == "tied")
        if step in ("scaled", "points"):
            q.scale_spectrum(fac)
        if step == "points":
            q.set_observation(w.obs[::-1] * 0.5)
        E1, B1 = q.evaluate(prec)
        q.close()
        assert np.array_equal(E, E1) and np.array_equal(B, B1), step
        sub = 4 if prec == "fp32_split" else 8
        small = w.subset(obs_idx=np.arange(0, w.n_obs, sub))     # the direct sum's partials must fit the scratch
        r = problem_from_workload(ctx, small)
        E2, B2 = r.evaluate(prec)
        o = tuple(t[:, : small.n_obs].contiguous() for t in out)
        r.evaluate_noalloc(o, prec)
        ctx.synchronize()
        assert np.array_equal(o[0].cpu().numpy(), E2) and np.array_equal(o[1].cpu().numpy(), B2), step
        r.close()
    assert rel_l2(res["scaled"], res["general"] * fac[:, None, None]) < 5e-7
    p.close()
