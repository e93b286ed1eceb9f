"""GPU: the apply and V-cycle entry points read and write the caller's arrays in
the ABI layout inside their own kernels. Against the oracle on meshes whose
last column tile is cut off, whose last level chunk is short, with one level,
with the fewest sweeps that take this route and one less, and with batches.
Tolerances are those of the other parity tests: float64 apply 1e-12, V-cycle
1e-10, float32 V-cycle 6e-7 against the float64 oracle."""
import numpy as np
import pytest
import torch

import workloads
from oracle import helmholtz, mesh, multigrid
from oracle.multigrid import MGParams

pytestmark = pytest.mark.gpu

CASES = [
    # N, nz, L, batch, n_coarse: 29^2 * 6 = 5046 columns, 22 in the last tile
    (29, 5, 1, 1, 2), (29, 5, 1, 1, 1), (29, 1, 1, 2, 4), (30, 33, 2, 1, 4),
    (34, 73, 2, 2, 4), (64, 7, 2, 1, 4), (32, 120, 1, 1, 3), (10, 9, 2, 3, 4),
]


@pytest.mark.parametrize("N,nz,L,batch,n_coarse", CASES)
def test_entry_points_in_abi_layout(N, nz, L, batch, n_coarse):
    from paper_2002_00756_amd import Operator
    print(f"abi layout N={N} nz={nz} L={L} batch={batch} n_coarse={n_coarse}", flush=True)
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    levels, parents, childs = mesh.hierarchy(N, L)
    hier = helmholtz.Hierarchy(levels, parents, childs, kh, kv, delta)
    b = workloads.rhs(N, nz, batch)
    bd = torch.from_numpy(b).cuda()
    ref = multigrid.vcycle(hier, b, MGParams(n_coarse=n_coarse))
    rel = lambda x, r: float(np.abs(x.double().cpu().numpy() - r).max() / np.abs(r).max())  # noqa: E731
    op = Operator(N, nz, kh, kv, delta, L, n_coarse=n_coarse, max_batch=batch)
    assert rel(op.apply(bd), hier.apply(0, b)) <= 1e-12
    assert rel(op.vcycle(bd), ref) <= 1e-10
    op32 = Operator(N, nz, kh, kv, delta, L, n_coarse=n_coarse, max_batch=batch, precision="fp32")
    assert rel(op32.vcycle(bd), ref) <= 6e-7
    assert rel(op32.vcycle_f32(bd), ref) <= 6e-7
    # the caller's b is left as it was
    assert torch.equal(bd.cpu(), torch.from_numpy(b))
