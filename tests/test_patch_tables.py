"""Patch tables (host side) against their definition on the oracle's mesh: own columns
row by row, then ring by ring the columns one step further, and each column's four
neighbours as places in that list. Panels of one column up to several patches, cut-off
patches, every patch size; patches next to an edge and at corners among them."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import mesh

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2002_00756_amd", "csrc")
SHAPES = [(2, 2, 2, 24), (4, 4, 2, 52), (2, 2, 3, 40), (4, 4, 3, 76), (8, 4, 2, 84)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tables")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text('#include "mesh.hpp"\nextern "C" void tables(int N, const int* nbr, int pw, '
                   "int ph, int depth, int ncp, int* col, unsigned* lnb, int* cnt) {\n"
                   "hh::build_patches(N, nbr, pw, ph, depth, ncp, col, lnb, cnt); }\n")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o",
                           str(so), str(src), os.path.join(CSRC, "mesh.cpp")])
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("pw,ph,depth,ncp", SHAPES)
@pytest.mark.parametrize("N", [1, 2, 3, 5, 8, 11, 12, 17, 26, 30, 37])
def test_tables(lib, N, pw, ph, depth, ncp):
    nbr = np.ascontiguousarray(mesh.neighbours(N), dtype=np.int32)
    npatch = 6 * (-(-N // pw)) * (-(-N // ph))
    col = np.full((npatch, ncp), -7, dtype=np.int32)
    lnb = np.full((npatch, ncp), 77, dtype=np.uint32)
    cnt = np.full((npatch, 8), -7, dtype=np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    lib.tables(N, ptr(nbr), pw, ph, depth, ncp, ptr(col), ptr(lnb), ptr(cnt))
    p = 0
    for pan in range(6):
        for j0 in range(0, N, ph):
            for i0 in range(0, N, pw):
                own = [(pan * N + j) * N + i for j in range(j0, min(j0 + ph, N))
                       for i in range(i0, min(i0 + pw, N))]
                counts, cols, ring = [len(own)], list(own), own
                for _ in range(depth):
                    ring = sorted({int(c) for q in ring for c in nbr[:, q]} - set(cols))
                    cols += ring
                    counts.append(len(cols))
                assert list(cnt[p, :depth + 1]) == counts
                assert cnt[p, 4] == min(pw, N - i0)
                got = col[p]
                assert list(got[:counts[0]]) == own
                for a, b in zip(counts, counts[1:]):
                    assert sorted(got[a:b]) == cols[a:b]
                assert (got[counts[-1]:] == own[0]).all()
                for d in range(4):
                    at = (lnb[p] >> np.uint32(8 * d)) & np.uint32(255)
                    assert (at[counts[depth - 1]:] == 0).all()
                    inner = slice(0, counts[depth - 1])
                    assert (got[at[inner]] == nbr[d, got[inner]]).all()
                p += 1
    assert p == npatch
