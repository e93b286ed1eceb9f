"""GPU: the CG solves whose preconditioner's last sweep forms r . z itself. Three
iterations against the same iteration written out with the apply and V-cycle
entry points, over the level counts at the edges of the sweep's compiled sizes,
a mesh whose last column tile is cut off, one level, and a batch with a member
that never starts.

The two differ by the order of the sums and the rounding of scalars, some 1e-15
of a vector per iteration; with a float32 V-cycle a residual that differs in its
last float64 bit can round to another float32, 6e-8 of single values of z. A
wrong or missing part of r . z changes x by its share of the sum."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

CASES = [  # N, nz, L, max_batch (8 or a size that keeps the level off the patches)
    (30, 1, 2, 8), (30, 8, 2, 8), (30, 32, 2, 8), (30, 33, 1, 8), (30, 72, 2, 8),
    (30, 73, 2, 8), (30, 120, 2, 8), (96, 5, 3, 2),
]


def pcg(op, b, iters):
    x, r = torch.zeros_like(b), b.clone()
    rho = p = None
    for _ in range(iters):
        z = op.vcycle(r)
        rz = (r * z).sum(dim=(1, 2), keepdim=True)
        p = z if p is None else z + rz / rho * p
        rho = rz
        q = op.apply(p)
        alpha = rho / (p * q).sum(dim=(1, 2), keepdim=True)
        x, r = x + alpha * p, r - alpha * q
    return x, r


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-7)])
@pytest.mark.parametrize("N,nz,L,max_batch", CASES)
def test_three_iterations(N, nz, L, max_batch, precision, tol):
    from paper_2002_00756_amd import Operator
    print(f"dot sweep N={N} nz={nz} L={L} {precision}", flush=True)
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    op = Operator(N, nz, kh, kv, delta, L, precision=precision, max_batch=max_batch)
    b = torch.from_numpy(workloads.rhs(N, nz, 2)).cuda()
    x, r = pcg(op, b, 3)
    norm = lambda v: v.flatten(1).norm(dim=1)  # noqa: E731
    got = op.solve(b, rtol=0.0, maxiter=3)
    assert got.iters == [3, 3]
    assert bool((norm(got.x - x) <= tol * norm(x)).all())
    one = torch.stack([torch.zeros_like(b[0]), b[1]])
    got = op.solve(one, rtol=0.0, maxiter=3)
    assert got.iters == [0, 3] and not bool(got.x[0].any())
    assert float(norm(got.x - x)[1]) <= tol * float(norm(x)[1])


@pytest.mark.parametrize("precision,word", [("fp64", 8), ("fp32", 4)])
def test_timing_hook_sees_plain_sweeps(precision, word):
    """With the hook on the last sweep runs as a plain one, 7 words per unknown,
    and r . z follows it: the counts of the hook, and the same bits."""
    from paper_2002_00756_amd import Operator, _lib
    print(f"dot sweep, hook on, {precision}", flush=True)
    N, nz = 30, 33
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    op = Operator(N, nz, kh, kv, delta, 2, precision=precision, max_batch=8)
    b = torch.from_numpy(workloads.rhs(N, nz)[0]).cuda()
    ref = op.solve(b, rtol=1e-8)
    op.profile(True)
    got = op.solve(b, rtol=1e-8)
    _, n, by = op.profile_read(_lib.PROF_SWEEP_FINE)
    op.profile(False)
    assert got.iters == ref.iters and torch.equal(got.x, ref.x)
    assert n == 2 * got.iters[0] and by == n * 7 * word * nz * 6 * N * N
