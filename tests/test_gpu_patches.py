"""GPU: V-cycles whose small levels run a whole leg on patches in one launch
(patch.hpp), against the oracle, at the sizes where that can go wrong: every
compiled patch size and depth, columns that fill or just exceed a compiled
depth, patches cut off at odd panel widths, one to four coarsest sweeps, cube
corners (panels one and two columns wide), and batches. Float64 to 1e-10 like
the other V-cycle parity tests; float32 to their 6e-7 against the float64
oracle. With the timing hook on the finest level runs kernel by kernel, which
must give the same bits."""
import numpy as np
import pytest
import torch

import workloads
from oracle import helmholtz, mesh, multigrid
from oracle.multigrid import MGParams

pytestmark = pytest.mark.gpu


def _setup(N, nz, L, form="sym", precision="fp64", batch=1, n_coarse=4):
    from paper_2002_00756_amd import Operator
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    ref, kw = {}, {}
    if form == "nine":
        ref["kv2"] = kw["kv2"] = workloads.next_nearest(N, nz, 10.0, True)
    if form == "weighted":
        ref["s"] = kw["s"] = workloads.row_weights(N, nz)
        kw["cg"] = "bicgstab"
    levels, parents, childs = mesh.hierarchy(N, L)
    hier = helmholtz.Hierarchy(levels, parents, childs, kh, kv, delta, **ref)
    op = Operator(N, nz, kh, kv, delta, L, n_coarse=n_coarse, precision=precision,
                  max_batch=batch, **kw)
    return hier, op


def _rel(x, ref):
    x = x.double().cpu().numpy()
    return float(np.abs(x - ref).max() / np.abs(ref).max())


CASES = [
    # N, nz, L, form, batch, n_coarse
    (8, 16, 3, "sym", 1, 4), (8, 17, 3, "sym", 1, 4),     # 2 x 2 patches, depth full / exceeded
    (12, 32, 2, "sym", 1, 1), (12, 33, 2, "sym", 1, 2),
    (14, 48, 2, "sym", 1, 3), (26, 49, 2, "sym", 1, 4),   # 4 x 4 patches, cut off at N = 14, 26
    (28, 64, 3, "sym", 1, 4), (36, 65, 3, "sym", 1, 4),   # 8 x 4 patches (float32: both)
    (64, 10, 2, "sym", 1, 4),
    (4, 120, 3, "sym", 1, 4), (20, 120, 2, "sym", 1, 4),  # the deepest columns
    (8, 1, 3, "sym", 1, 4), (8, 2, 3, "sym", 1, 4),       # one and two levels
    (1, 7, 1, "sym", 1, 4), (2, 9, 2, "sym", 1, 4), (7, 20, 1, "sym", 1, 4),
    (24, 30, 3, "sym", 3, 4), (12, 10, 3, "sym", 4, 4),
    (12, 10, 3, "nine", 1, 4), (24, 33, 2, "nine", 2, 4), (40, 20, 3, "nine", 1, 4),
    (8, 3, 2, "nine", 1, 4),
    (12, 10, 3, "weighted", 1, 4), (24, 33, 2, "weighted", 2, 4), (40, 20, 3, "weighted", 1, 4),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N,nz,L,form,batch,n_coarse", CASES)
def test_vcycle_on_patches(N, nz, L, form, batch, n_coarse, precision):
    print(f"patches {precision} N={N} nz={nz} L={L} {form} batch={batch}", flush=True)
    hier, op = _setup(N, nz, L, form, precision, batch, n_coarse)
    b = workloads.rhs(N, nz, batch)
    bd = torch.from_numpy(b).cuda()
    x = op.vcycle(bd)
    op.profile(True)
    y = op.vcycle(bd)
    op.profile(False)
    torch.cuda.synchronize()
    assert torch.equal(x, y)
    ref = multigrid.vcycle(hier, b, MGParams(n_coarse=n_coarse))
    err = _rel(x, ref)
    print(f"  error {err:.2e}", flush=True)
    assert err <= (1e-10 if precision == "fp64" else 6e-7)
