"""Where the merge's blocks go: every row is taken once, by sixteen blocks of one die, in order, and few rows use as many dies as there are."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19427_amd", "csrc")
SHIM = """
#include "mfa_merge_place.hpp"
extern "C" unsigned blocks(int rows) { return mfa::merge_blocks_by_die(rows); }
extern "C" void place(int rows, int* row) { for (unsigned i = 0; i < blocks(rows); ++i) row[i] = mfa::merge_row(i, rows); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("merge_place")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("tokens", [1, 2, 3, 4])
def test_every_row_once_and_few_rows_on_many_dies(shim, tokens):
    for B in list(range(1, 140)) + [255, 256, 257, 511, 512, 513, 1000, 4095, 4096]:
        rows = B * tokens
        n = shim.blocks(rows)
        got = np.empty(n, dtype=np.int32)
        shim.place(rows, got.ctypes.data_as(ctypes.c_void_p))
        block = np.arange(n)
        die, piece = block & 7, (block >> 3) & 15
        taken = got >= 0
        assert n < 16 * (rows + 8) and taken.sum() == 16 * rows
        assert len(set(zip(got[taken].tolist(), piece[taken].tolist()))) == 16 * rows and got.max() == rows - 1
        # ties of the middle (row + 1/2) * 8 / rows with a die's end go to the die above
        assert np.array_equal(die[taken], (2 * got[taken] + 1) * 8 // (2 * rows))
        assert len(set(die[taken].tolist())) == min(8, rows), (B, tokens)
