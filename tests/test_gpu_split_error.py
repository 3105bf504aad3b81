"""GPU: the compacted FP32 sum is no less accurate than the direct one.

The same points from host memory (compacted) and in device memory (direct), both against the FP64 form: the error
of the compacted sum may exceed the direct one's by a quarter, what the two scatter by (fewer nodes average the
rounding of their phases), over the distances at which the FP32 form changes (q = |r'| / f of 1e-3 and 1e-2 among
them) and for little and much rounding of the phase itself (k |r'|).
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
K = 2 * np.pi


def rel_l2(a, b):
    return float(np.linalg.norm((np.asarray(a) - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("q,f", [(2e-5, 1e5), (9e-4, 3e3), (1.1e-3, 900.0), (5e-3, 200.0), (9.9e-3, 100.0), (9.9e-3, 300.0),
                                 (1.1e-2, 100.0), (0.1, 20.0)])
@pytest.mark.parametrize("field", ["beam", "random"])
def test_error_against_the_direct_sum(q, f, field):
    import torch
    from paper_1609_08146_amd import Context, Problem
    ctx = Context(0)
    nk, nr, nphi, n = 3, 200, 240, 600
    rng = np.random.default_rng(11)
    obs = rng.normal(size=(n, 3))
    obs *= (q * f * rng.uniform(0.3, 1.0, n) / np.linalg.norm(obs, axis=1))[:, None]
    obs[0] = 0.0, 0.0, q * f
    p = Problem(ctx)
    p.set_mirror(f, 1.5 * f, nr, nphi)
    p.set_frequencies(K * np.linspace(1.0, 1.1, nk))
    if field == "random":
        p.set_incident(*workloads.random_incident_tables(nk, (nr + 1) * nphi, seed=7))
    else:
        p.set_incident_gaussian(0.9 * f, 0.3, None, False)
    p.set_observation(torch.tensor(obs, device="cuda"))
    E64, B64 = p.evaluate("fp64")
    Ed, Bd = p.evaluate("fp32_split")
    direct = p.timing()["tiles"]
    p.set_observation(obs)
    E, B = p.evaluate("fp32_split")
    assert 4 * p.timing()["tiles"] < direct        # compacted
    for a, d, ref in ((E, Ed, E64), (B, Bd, B64)):
        assert rel_l2(a, ref) < 1.25 * rel_l2(d, ref)
    p.close()
    ctx.close()
