"""The ``out`` argument of solve and vcycle_noalloc: an array of another type, size,
layout or device, which the library would write out of its range, is refused before
the library is called; shapes that view as the result's are taken. On the CPU, with
an operator that has no handle and a library that must not be called."""
import pytest
import torch

from paper_2002_00756_amd import Operator


class NoCalls:
    def __getattr__(self, name):
        raise AssertionError(f"library called: {name}")


def _operator(nz, ncol, batch):
    op = Operator.__new__(Operator)
    op.device, op.nz, op.ncol, op.max_batch = torch.device("cpu"), nz, ncol, batch
    op.lib, op._h = NoCalls(), None
    return op


BAD = {
    "type": lambda: torch.zeros(2, 3, 24, dtype=torch.float32),
    "strides": lambda: torch.zeros(2, 3, 48, dtype=torch.float64)[:, :, ::2],
    "order": lambda: torch.zeros(2, 24, 3, dtype=torch.float64).transpose(1, 2),
    "device": lambda: torch.zeros(2, 3, 24, dtype=torch.float64, device="meta"),
}


@pytest.mark.parametrize("call", ["solve", "vcycle_noalloc"])
@pytest.mark.parametrize("bad", sorted(BAD))
def test_refused(call, bad):
    op = _operator(3, 24, 2)
    with pytest.raises(ValueError):
        getattr(op, call)(torch.ones(2, 3, 24, dtype=torch.float64), out=BAD[bad]())


def test_taken():
    op = _operator(3, 24, 2)
    b = torch.ones(1, 3, 24, dtype=torch.float64)
    for shape in ((1, 3, 24), (3, 24), (72,)):
        out = torch.zeros(shape, dtype=torch.float64)
        x = op._out(out, b)
        assert x.data_ptr() == out.data_ptr() and x.shape == b.shape
    assert op._out(b, b).data_ptr() == b.data_ptr()
    new = op._out(None, b)
    assert new.shape == b.shape and new.dtype == b.dtype
    with pytest.raises(RuntimeError):
        op._out(torch.zeros(71, dtype=torch.float64), b)
