"""GPU: the apply and V-cycle entry points with b and x in one array, whole or one
batch member apart: the result is that of separate arrays. Finest levels on
patches (one and several levels, the three operator forms), off them, and the
applies staged through LDS and not. V-cycles run the same kernels either way and
agree bit for bit; the apply may round a fused product the other way, held to
the 1e-12 of the apply's parity tests. Values read after they were overwritten
would change the result by its own size."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

CASES = [  # N, nz, L, form
    (24, 30, 3, "sym"), (12, 10, 1, "sym"), (40, 20, 2, "nine"), (24, 33, 2, "weighted"),
    (64, 7, 2, "sym"), (64, 6, 2, "nine"), (100, 9, 2, "sym"), (70, 40, 2, "weighted"),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N,nz,L,form", CASES)
def test_overlapping_arrays(N, nz, L, form, precision):
    from paper_2002_00756_amd import Operator, _lib
    print(f"in place {precision} N={N} nz={nz} L={L} {form}", flush=True)
    kh, kv, delta = workloads.coefficients(N, nz, 1.0, 1000.0, True)
    kw = {}
    if form == "nine":
        kw["kv2"] = workloads.next_nearest(N, nz, 10.0, True)
    if form == "weighted":
        kw.update(s=workloads.row_weights(N, nz), cg="bicgstab")
    op = Operator(N, nz, kh, kv, delta, L, precision=precision, max_batch=2, **kw)
    rhs = torch.from_numpy(workloads.rhs(N, nz, 2)).cuda()
    names = ["apply", "vcycle", "vcycle_f32"]
    fits = (N, nz) != (70, 40)
    if fits:  # the static scratch does not hold two right-hand sides of C70 x 40
        names.append("vcycle_noalloc")
    if form == "weighted":
        names += ["apply_adjoint", "vcycle_adjoint"]

    def call(name, b, x):
        _lib.check(getattr(op.lib, f"helmholtz_{name}")(
            op._h, b.data_ptr(), x.data_ptr(), b.shape[0],
            torch.cuda.current_stream().cuda_stream), name)

    for name in names:
        b = rhs.float() if name == "vcycle_f32" else rhs
        want = torch.empty_like(b)
        call(name, b, want)
        for shift in (0, 1, -1):
            buf = torch.zeros((3,) + tuple(b.shape[1:]), dtype=b.dtype, device=b.device)
            at, to = (1, 0) if shift < 0 else (0, shift)
            buf[at:at + 2] = b
            call(name, buf[at:at + 2], buf[to:to + 2])
            got = buf[to:to + 2]
            if name.startswith("apply"):
                assert float((got - want).abs().max()) <= 1e-12 * float(want.abs().max()), name
            else:
                assert torch.equal(got, want), (name, shift)
    if not fits:
        return
    y = rhs.clone()
    assert op.vcycle_noalloc(y, out=y).data_ptr() == y.data_ptr()
    assert torch.equal(y, op.vcycle(rhs))
