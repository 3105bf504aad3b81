"""GPU: the FP64 form where the phase k delta is 2^41 turns and more (points in the far field), against the oracle.

The phase is the rounding of k delta itself, formed from FP64 coordinates: an error of a few k |r'| 2^-53 per
term, bounded as for the split form by 16 k |r'| 2^-53 relative (0.2 at 2^44 wavelengths).  Beyond that no
phase is left, but sine and cosine are still at most 1, so no component exceeds the sum of the terms' magnitudes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
K = 2 * np.pi


def rel_l2(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


@pytest.mark.parametrize("layout", ["tied", "factored", "general"])
def test_far_field_phase(orc, layout):
    import torch
    from paper_1609_08146_amd import Context, Problem
    f, a, nr, nphi = 20.0, 40.0, 24, 16
    th = np.radians([0.0, 20.0, 40.0, 65.0])
    dirs = np.stack([np.sin(th), 0.3 * np.sin(th), np.cos(th)], axis=-1)
    m = orc.mirror(f, a, nr, nphi)
    Ei, Bi = orc.incident_tables(m, np.array([K]), orc.GAUSSIAN, 20.0)
    ctx = Context(0)
    for e in (39, 41, 43, 44, 47, 60):
        d = 2.0 ** e * 1.37
        pts = d * dirs
        for where in ("host", "device"):
            p = Problem(ctx)
            p.set_factoring(layout != "general", tie_charge=layout == "tied")
            p.set_mirror(f, a, nr, nphi)
            p.set_frequencies([K])
            p.set_incident_gaussian(20.0)
            p.set_observation(pts if where == "host" else torch.tensor(pts, device="cuda"))
            E, B = p.evaluate("fp64")
            p.close()
            if e <= 44:
                Eo, Bo = orc.reflected_field(m, np.array([K]), Ei, Bi, pts)
                assert max(rel_l2(E, Eo), rel_l2(B, Bo)) < 16 * K * d * 2.0 ** -53, (e, where)
            # every term is at most (k |J~| + k |rho~|)(1 + 1/kR) / R
            W = np.abs(m.wgt)[:, None] * (np.abs(m.nrm) + 1e-300)
            bound = 8 * K / (4 * np.pi) * 4 * np.sum(np.abs(W)) * max(np.abs(Ei).max(), np.abs(Bi).max()) / d + 1e-300
            assert np.abs(E).max() < bound and np.abs(B).max() < bound, (e, where)
    ctx.close()
