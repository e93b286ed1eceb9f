"""GPU: V-cycle entry points whose first sweep reads b and whose last one writes x in
the caller's layout, on finest levels that run sweep by sweep: the fewest sweeps
that take this route and one less of each kind (then conversion passes run), every
compiled column depth, a cut-off last tile, and a level of few columns. max_batch
keeps the finest level off the patches, which the workspace shows: it equals that
of a handle whose sweep counts exclude them. x starts as NaN, so that a value that
no sweep writes shows. Tolerances as for the other V-cycles: 1e-10, and 6e-7 for
float32 against the float64 oracle."""
import numpy as np
import pytest
import torch

import workloads
from oracle import helmholtz, mesh, multigrid
from oracle.multigrid import MGParams

pytestmark = pytest.mark.gpu

CASES = [  # N, nz, L, max_batch, (n_pre, n_post, n_coarse); 29^2 * 6 = 157 * 32 + 22
    (29, 5, 1, 2, (2, 2, 2)), (29, 5, 1, 2, (2, 2, 1)), (29, 1, 1, 2, (2, 2, 3)),
    (29, 33, 1, 2, (2, 2, 2)), (29, 73, 1, 2, (2, 2, 2)), (29, 120, 1, 2, (2, 2, 1)),
    (30, 8, 2, 8, (2, 2, 4)), (30, 32, 2, 8, (1, 2, 4)), (30, 33, 2, 8, (1, 2, 1)),
    (30, 40, 2, 8, (2, 1, 2)), (30, 72, 2, 8, (2, 2, 4)), (30, 73, 2, 8, (0, 2, 4)),
    (30, 120, 2, 8, (1, 2, 4)), (30, 9, 2, 8, (0, 0, 2)), (28, 10, 2, 9, (2, 2, 4)),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N,nz,L,max_batch,sweeps", CASES)
def test_vcycle_sweep_by_sweep(N, nz, L, max_batch, sweeps, precision):
    from paper_2002_00756_amd import Operator, _lib
    print(f"abi sweeps N={N} nz={nz} L={L} {sweeps} {precision}", flush=True)
    n_pre, n_post, n_coarse = sweeps
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)

    def operator(pre, coarse):
        return Operator(N, nz, kh, kv, delta, L, n_pre=pre, n_post=n_post, n_coarse=coarse,
                        max_batch=max_batch, precision=precision)

    op = operator(n_pre, n_coarse)
    never = operator(n_pre, 5) if L == 1 else operator(3, n_coarse)
    assert op.workspace_bytes == never.workspace_bytes
    levels, parents, childs = mesh.hierarchy(N, L)
    hier = helmholtz.Hierarchy(levels, parents, childs, kh, kv, delta)
    b = workloads.rhs(N, nz, 2)
    ref = multigrid.vcycle(hier, b, MGParams(n_pre=n_pre, n_post=n_post, n_coarse=n_coarse))
    bd = torch.from_numpy(b).cuda()
    for name in ("helmholtz_vcycle", "helmholtz_vcycle_f32"):
        src = bd.float() if name.endswith("f32") else bd
        x = torch.full_like(src, float("nan"))
        _lib.check(getattr(op.lib, name)(op._h, src.data_ptr(), x.data_ptr(), 2,
                                         torch.cuda.current_stream().cuda_stream), name)
        err = float(np.abs(x.double().cpu().numpy() - ref).max() / np.abs(ref).max())
        tol = 1e-10 if precision == "fp64" and not name.endswith("f32") else 6e-7
        print(f"  {name} {err:.2e}", flush=True)
        assert err <= tol
        assert torch.equal(src, bd.to(src.dtype))
