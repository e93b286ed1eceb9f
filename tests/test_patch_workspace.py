"""Workspace of levels on patches (host side): the tables and the column-by-column
coefficients are laid out only for levels that run on patches in some precision.
Options that never take patches (three presmoothing sweeps, five coarsest ones)
give the size without them."""
import ctypes

import pytest

from paper_2002_00756_amd import _lib


def _bytes(N, nz, L, n_pre, n_coarse, precision, stencil=7, batch=1):
    cfg = _lib.Config(N, nz, L, n_pre, 2, n_coarse, 0.8, precision, _lib.CG_STANDARD, batch,
                      stencil, 0)
    return _lib.load().helmholtz_workspace_bytes(ctypes.byref(cfg))


@pytest.mark.parametrize("precision", [_lib.FP64, _lib.FP32])
@pytest.mark.parametrize("N,nz,L,stencil", [(48, 70, 2, 7), (64, 47, 1, 7), (80, 100, 3, 7),
                                            (48, 50, 2, 9), (26, 70, 1, 7)])
def test_no_tables_without_patches(N, nz, L, stencil, precision):
    got = _bytes(N, nz, L, 2, 4, precision, stencil)
    assert got and got == _bytes(N, nz, L, 3, 5, precision, stencil)


@pytest.mark.parametrize("precision", [_lib.FP64, _lib.FP32])
def test_tables_with_patches(precision):
    assert _bytes(24, 30, 2, 2, 4, precision) > _bytes(24, 30, 2, 3, 5, precision)
