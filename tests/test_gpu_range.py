"""GPU: the compacted FP32 sum over the range of FP32, as the direct sum has it.

The incident field times 2^e gives the result times 2^e: bit for bit where neither the records nor the results
leave FP32's normal numbers (every scale in between is a power of two), and to the split form's own error near
its ends.  Wavenumbers of 8e6 / m besides 6: sums of B' = ik B must not overflow before B.  Very long waves beside
ordinary ones are summed directly, and stay finite.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
K = 2 * np.pi
NR, NPHI, NOBS = 150, 180, 400


def rel_l2(a, b):
    a, b = (np.asarray(v, np.complex128) for v in (a, b))
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1609_08146_amd import Context
    c = Context(0)
    yield c
    c.close()


def solve(ctx, f, ks, obs, fields, prec="fp32_split"):
    from paper_1609_08146_amd import Problem
    p = Problem(ctx)
    p.set_mirror(f, 1.5 * f, NR, NPHI)
    p.set_frequencies(ks)
    fields(p)
    p.set_observation(obs)
    out = p.evaluate(prec)
    tiles = p.timing()["tiles"]
    p.close()
    return out + (tiles,)


@pytest.mark.parametrize("q", [2e-5, 7e-4, 0.1])      # the three forms of the FP32 sum: see sc_compact_host.cpp
@pytest.mark.parametrize("e", [100, 110, -90, -100])
def test_fields_of_any_size(ctx, q, e):
    f = 2.0 / q
    ks = K * np.array([1.0, 1.1])
    obs = workloads.random_points(NOBS, 1.0, seed=3)
    Ei, Bi = workloads.random_incident_tables(2, (NR + 1) * NPHI, seed=5)
    E0, B0, tiles = solve(ctx, f, ks, obs, lambda p: p.set_incident(Ei, Bi))
    assert tiles < NR * NPHI / 64        # (directly: chunks of 64 nodes)
    # the tables hold fields x area; bring them near the ends of the range
    s = 2.0 ** (e - int(np.log2(f * f / (NR * NPHI))))
    E, B, _ = solve(ctx, f, ks, obs, lambda p: p.set_incident(Ei * s, Bi * s))
    if e > 0 or q > 1e-3:
        assert np.array_equal(E, (E0.astype(np.complex128) * s).astype(np.complex64))
        assert np.array_equal(B, (B0.astype(np.complex128) * s).astype(np.complex64))
    assert rel_l2(E, E0.astype(np.complex128) * s) < 2e-6 and rel_l2(B, B0.astype(np.complex128) * s) < 2e-6


def test_large_fields_in_metres(ctx):
    """A beam whose charge is tied to its current: the direct sum forms B, not B', in FP32."""
    lam, f = 800e-9, 0.1
    ks = K / lam * np.array([1.0, 1.1])
    obs = workloads.random_points(NOBS, 2 * lam, seed=3)
    amp = np.array([1.0, 0.5j])
    E0, B0, _ = solve(ctx, f, ks, obs, lambda p: p.set_incident_gaussian(0.1, 0.3, amp, False))
    s = 2.0 ** (125 - int(np.ceil(np.log2(max(np.abs(E0).max(), np.abs(B0).max())))))
    E, B, _ = solve(ctx, f, ks, obs, lambda p: p.set_incident_gaussian(0.1, 0.3, amp * s, False))
    assert np.array_equal(E, (E0.astype(np.complex128) * s).astype(np.complex64))
    assert np.array_equal(B, (B0.astype(np.complex128) * s).astype(np.complex64))


@pytest.mark.parametrize("k0", [1e-6, 1e-3, 4e-3])
def test_long_waves(ctx, orc, k0):
    ks = np.array([k0, K])
    obs = workloads.random_points(600, 1.0, seed=3)      # (400 and more would be compacted at k0 = 1)
    m = orc.mirror(10.0, 15.0, NR, NPHI)
    Ei, Bi = workloads.random_incident_tables(2, m.n_tot, seed=5)
    Eo, Bo = orc.reflected_field(m, ks, Ei, Bi, obs[::12])
    E, B, _ = solve(ctx, 10.0, ks, obs, lambda p: p.set_incident(Ei, Bi))
    for n in range(2):
        assert max(rel_l2(E[n, ::12], Eo[n]), rel_l2(B[n, ::12], Bo[n])) < 2e-6
