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
extern "C" int waves(int B, int n_here, int q_len, int pieces) { return mfa::merge_waves(B, n_here, q_len, pieces); }
extern "C" int by_die(int B, int n_here, int q_len, int n_wgs, int waves) { return mfa::merge_by_die(B, n_here, q_len, n_wgs, waves); }
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


def test_form_of_few_rows(shim):
    """Nine to sixteen rows whose batch is no multiple of eight, over 256 workgroups."""
    def form(B, n_here, q_len):
        waves = shim.waves(B, n_here, q_len, 256 // B)
        return waves, bool(shim.by_die(B, n_here, q_len, 256, waves))
    for B in (5, 6, 7):
        assert form(B, 2, 2) == (8, False)                              # two tokens
        for q_len in (3, 4):
            assert form(B, 2, q_len) == (4, True)                       # two passes: what lies on a die stays there
    for B in (9, 11, 13, 15):
        assert form(B, 1, 1) == (4, False)
    assert form(3, 3, 3) == form(3, 4, 4) == (4, False)
    # the rest: no dies left idle by up to four rows, by die from five to eight and with even batches, one wave beyond sixteen
    assert form(1, 1, 1) == form(2, 2, 2) == (8, False) and form(5, 1, 1) == form(4, 2, 2) == form(3, 2, 4) == (8, True)
    assert form(8, 2, 2) == (4, True) and form(9, 2, 2) == form(17, 1, 1) == (1, True)
