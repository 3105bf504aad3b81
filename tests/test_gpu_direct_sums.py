"""GPU: the direct sum, which general surfaces, points in device memory and points far from the focus take.

Problems on the built-in paraboloid with host points are compacted where that is faster, so these hand the points
over in device memory: chunks of several blocks of 512 nodes (the FP32 forms' running sums in LDS and memory), every
table layout, every launch shape, and the cap on a batch's partials.  sc_get_timing's chunk and tiles are those of
the direct sum, which shows that it was taken.  Tolerances of the forms: relative L2 1e-12 in FP64, 1e-5 in
FP32-split.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
K = 2 * np.pi
TOL = {"fp64": 1e-12, "fp32_split": 1e-5}


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


def problem(ctx, f, a, nr, nphi, ks, obs):
    import torch
    from paper_1609_08146_amd import Problem
    p = Problem(ctx)
    p.set_mirror(f, a, nr, nphi)
    p.set_frequencies(ks)
    p.set_observation(torch.tensor(obs, device="cuda"))
    return p


def direct_tiles(p, n_obs, n_k, prec):
    ns, nr = p.num_nodes()
    l, chunk = p.launch(prec), p.timing()["chunk"]
    return -(-n_obs // 128) * 128 // (64 * l["obs_per_lane"]) * -(-(ns + nr) // chunk) * -(-n_k // l["freq_per_lane"])


@pytest.mark.parametrize("layout", ["tied", "factored", "general"])
@pytest.mark.parametrize("chunk", [576, 2048, 4096, 0])
def test_chunks_of_several_blocks(ctx, orc, layout, chunk):
    """7 760 nodes: chunks of 512 + 64, 4 x 512 and 8 x 512 with ragged last ones, and the library's."""
    f, a, nr, nphi = 20.0, 40.0, 96, 80
    ks = K * np.linspace(0.9, 1.1, 5)
    obs = workloads.random_points(200, 2.0, seed=2)
    m = orc.mirror(f, a, nr, nphi)
    pairs = [orc.incident_tables(m, np.array([k]), orc.GAUSSIAN, 20.0) for k in ks]
    Ei, Bi = (np.concatenate([p[i] for p in pairs]) for i in (0, 1))
    Eo, Bo = orc.reflected_field(m, ks, Ei, Bi, obs[::5])
    p = problem(ctx, f, a, nr, nphi, ks, obs)
    p.set_factoring(layout != "general", tie_charge=layout == "tied")
    p.set_incident_gaussian(20.0)
    if chunk:
        p.set_launch(chunk=chunk)
    for prec in ("fp32_split", "fp64"):
        assert p.layout_for(prec) == layout
        E, B = p.evaluate(prec)
        t = p.timing()
        assert t["chunk"] == chunk or (chunk == 0 and t["chunk"] < 2048)
        assert t["tiles"] == direct_tiles(p, len(obs), len(ks), prec)
        assert max(rel_l2(E[:, ::5], Eo), rel_l2(B[:, ::5], Bo)) < TOL[prec], prec
    p.close()


def test_default_chunk_of_several_blocks(ctx, orc):
    """40 200 nodes and 4160 points: the library's own chunk is more than two blocks here."""
    w = workloads.broadband(n_k=8, n_nodes=200)
    import torch
    from paper_1609_08146_amd import problem_from_workload
    Eo, Bo = orc.solve(w.subset(obs_idx=np.arange(0, w.n_obs, 131)))
    p = problem_from_workload(ctx, w)
    p.set_observation(torch.tensor(np.ascontiguousarray(w.obs), device="cuda"))
    for prec in ("fp32_split", "fp64"):
        E, B = p.evaluate(prec)
        t = p.timing()
        assert t["chunk"] > 512 and t["tiles"] == direct_tiles(p, w.n_obs, w.n_k, prec)
        assert max(rel_l2(E[:, ::131], Eo), rel_l2(B[:, ::131], Bo)) < TOL[prec], prec
    p.close()


@pytest.mark.parametrize("layout", ["tied", "general"])
def test_launch_shape_does_not_change_bits(ctx, layout):
    """5 frequencies: blocks of 2 and 4 leave a ragged last one."""
    obs = workloads.random_points(300, 2.0, seed=4)
    p = problem(ctx, 20.0, 40.0, 64, 64, K * np.linspace(0.9, 1.1, 5), obs)
    p.set_factoring(layout == "tied", tie_charge=True)
    p.set_incident_gaussian(20.0)
    ref = {}
    for opl, fpb in [(1, 1), (2, 1), (1, 2), (2, 2), (1, 4)]:
        for wpb in (1, 2, 4):
            for bpc in (0, 1):
                p.set_launch(obs_per_lane=opl, freq_per_lane=fpb, waves_per_block=wpb, chunk=1024, blocks_per_cu=bpc)
                for prec in ("fp32_split", "fp64", "fp32"):
                    E, B = p.evaluate(prec)
                    assert p.timing()["tiles"] == direct_tiles(p, len(obs), 5, prec)
                    E0, B0 = ref.setdefault(prec, (E, B))
                    assert np.array_equal(E, E0) and np.array_equal(B, B0), (prec, opl, fpb, wpb, bpc)
    p.close()


def test_batch_keeps_direct_partials_within_the_cap(ctx):
    """10.3 GB of partials at 2048 nodes, for the documented 8 GiB: 4096; a problem with its own chunk keeps it."""
    big = problem(ctx, 20.0, 40.0, 320, 320, np.linspace(2 * np.pi, 3 * np.pi, 256), workloads.random_points(16384, 2.0, seed=21))
    big.set_incident_gaussian(20.0)
    small = problem(ctx, 20.0, 40.0, 40, 32, [2 * np.pi], workloads.random_points(100, 2.0, seed=22))
    small.set_launch(chunk=1024)
    small.set_incident_gaussian(20.0)
    ctx.evaluate_batch([big, small], "fp32_split")
    assert big.timing()["chunk"] == 4096 and small.timing()["chunk"] == 1024
    assert big.timing()["tiles"] == 16384 // 64 * -(-102720 // 4096) * 64
    Eb, Bb = big.result()
    Es, Bs = small.result()
    big.set_launch(chunk=4096)
    E, B = big.evaluate("fp32_split")
    assert np.array_equal(E, Eb) and np.array_equal(B, Bb)
    E, B = small.evaluate("fp32_split")
    assert np.array_equal(E, Es) and np.array_equal(B, Bs)
    big.close()
    small.close()
