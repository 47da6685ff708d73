"""The residual launch of a wide pass deals its rows to the 8 dies of the chip by arithmetic on the workgroup index alone
(csrc/wide_rows.h, plain C++): compiled here as it stands and checked for every number of rows a pass can have."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_03251_amd", "csrc")
XCDS, PIECE = 8, 8


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("wide_rows")
    src, so = d / "rows.cpp", d / "rows.so"
    src.write_text('#include "wide_rows.h"\n'
                   'extern "C" int grid_of(int rows) { return (int)ssd::wide_resid_grid((unsigned)rows); }\n'
                   'extern "C" void rows_of(int grid, int* out) { for (int b = 0; b < grid; ++b) out[b] = (int)ssd::wide_resid_row((unsigned)b); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so))


def test_rows_of_a_residual_launch_are_dealt_evenly(lib):
    for M in range(1, 1025):
        grid = lib.grid_of(M)
        out = np.empty(grid, np.int32)
        lib.rows_of(grid, out.ctypes.data_as(ctypes.c_void_p))
        assert grid >= M and np.array_equal(np.sort(out), np.arange(grid)), M          # every row once
        xcd = np.empty(grid, np.int64)
        xcd[out] = np.arange(grid) % XCDS
        xcd = xcd[:M]
        # the rows whose 16-byte operand pieces make up a 128-byte line share a die
        assert all(len(set(xcd[r:r + PIECE])) == 1 for r in range(0, M, PIECE)), M
        # and no die has more than one such piece above another
        n = np.bincount(xcd, minlength=XCDS)
        assert n.max() - n.min() <= PIECE, (M, n.tolist())
