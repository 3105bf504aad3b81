"""GPU: results into device memory that the caller hands over."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32_split"])
def test_overlapping_outputs_hold_b_where_they_meet(prec):
    """E first and then B, also where both go to one tensor or to parts of it that overlap; repeated, because a race
    between the two would not always show."""
    import torch
    from paper_1609_08146_amd import Context, problem_from_workload
    ctx = Context(0)
    w = workloads.broadband(n_k=6, n_nodes=100)
    p = problem_from_workload(ctx, w)
    E, B = (a.ravel() for a in p.evaluate(prec))
    n = E.size
    for shift in (0, n // 3 // 3 * 3, n):
        for _ in range(5):
            flat = torch.zeros(n + shift, dtype=torch.complex128 if prec == "fp64" else torch.complex64, device="cuda")
            shape = (w.n_k, w.n_obs, 3)
            p.evaluate(prec, out=(flat[:n].view(shape), flat[shift:].view(shape)))
            torch.cuda.synchronize()
            got = flat.cpu().numpy()
            assert np.array_equal(got[shift:], B) and np.array_equal(got[:shift], E[:shift])
    one = torch.zeros((w.n_k, w.n_obs, 3), dtype=flat.dtype, device="cuda")
    for _ in range(5):
        p.evaluate_noalloc((one.zero_(), one), prec)
        torch.cuda.synchronize()
        assert np.array_equal(one.cpu().numpy().ravel(), B)
    p.close()
    ctx.close()
