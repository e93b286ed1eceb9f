"""GPU: a V-cycle of a right-hand side with an infinite or NaN value gives the same
values, infinities and NaN on patches as kernel by kernel: rows that only fill up
a patch's columns must not turn an infinity into NaN. The reference is a handle
for so many right-hand sides that none of its levels runs on patches."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

CASES = [  # N, nz, L, form
    (12, 10, 1, "sym"), (12, 10, 3, "sym"), (8, 3, 2, "sym"), (24, 33, 1, "sym"),
    (12, 10, 1, "nine"), (12, 10, 2, "nine"), (12, 10, 1, "weighted"), (32, 20, 2, "sym"),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N,nz,L,form", CASES)
def test_nonfinite_values_on_patches(N, nz, L, form, precision):
    from paper_2002_00756_amd import Operator
    print(f"nonfinite {precision} N={N} nz={nz} L={L} {form}", flush=True)
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    kw = {}
    if form == "nine":
        kw["kv2"] = workloads.next_nearest(N, nz, 10.0, True)
    if form == "weighted":
        kw.update(s=workloads.row_weights(N, nz), cg="bicgstab")
    ops = [Operator(N, nz, kh, kv, delta, L, precision=precision, max_batch=m, **kw)
           for m in (1, 6200 // (6 * (N >> (L - 1)) ** 2) + 40000 // (6 * N * N) + 1)]
    rhs = torch.from_numpy(workloads.rhs(N, nz)[0]).cuda()
    for value in (float("inf"), float("-inf"), float("nan")):
        for k in (0, nz // 2, nz - 1):
            b = rhs.clone()
            b[k, 7] = value
            x, ref = (op.vcycle(b) for op in ops)
            assert not bool(torch.isfinite(ref).all())
            assert torch.equal(torch.isnan(x), torch.isnan(ref)), (value, k)
            assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(ref)), (value, k)
