"""GPU: a BiCGStab breakdown, (r0, v) = 0, ends its right-hand side and nothing
else: iterate and residual stay those of the start, and the batch's other member
solves as it does alone. On meshes whose scalars are formed where they are used
(one and many workgroups) and on one that has them formed in launches of their
own. The inner product is exactly zero by underflow: with a float32 V-cycle the
right-hand side 1e-100 rounds to zero; in float64, values of 3e-162 have squares
of two units of the smallest number, and one damped sweep leaves v at a tenth of
them, whose products round to zero."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,value", [("fp64", 3e-162), ("fp32", 1e-100)])
@pytest.mark.parametrize("N,nz", [(4, 3), (12, 10), (40, 20), (64, 30)])
def test_breakdown_ends_one_right_hand_side(N, nz, precision, value):
    from paper_2002_00756_amd import Operator
    print(f"breakdown N={N} nz={nz} {precision}", flush=True)
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    op = Operator(N, nz, kh, kv, delta, 1, n_coarse=1, omega=0.1, precision=precision,
                  cg="bicgstab", max_batch=2)
    b = torch.from_numpy(workloads.rhs(N, nz, 2)).cuda()
    b[0] = value
    alone = op.solve(b[1], rtol=1e-12, maxiter=3)
    for hook in (False, True):
        op.profile(hook)
        x = torch.full_like(b, float("nan"))
        got = op.solve(b, rtol=1e-12, maxiter=3, out=x)
        assert not got.converged
        assert got.iters == [1, 3] and got.relres[0] == 1.0
        assert not bool(got.x[0].any())
        assert torch.equal(got.x[1], alone.x) and got.relres[1] == alone.relres[0]
    op.profile(False)
    # a later solve on the handle starts afresh
    b[0] = b[1]
    got = op.solve(b, rtol=1e-12, maxiter=3)
    assert got.iters == [3, 3] and torch.equal(got.x[0], alone.x)
