"""The choice between the two kernels of the 8-bit and 4-bit caches, which is by sizes alone."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19427_amd", "csrc")
SHIM = """
#include "mfa_kernel_choice.hpp"
extern "C" int takes_short(int four_bit, int one_token, long tiles_per_wg, long tiles_per_seq)
{ return mfa::takes_short_lowbit_kernel(four_bit, one_token, tiles_per_wg, tiles_per_seq); }
"""


@pytest.fixture(scope="module")
def takes_short(tmp_path_factory):
    d = tmp_path_factory.mktemp("kernel_choice")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    f = ctypes.CDLL(str(d / "shim.so")).takes_short

    def choose(four_bit, q_len, B, hint):
        per_seq = (hint + 63) // 64
        return bool(f(four_bit, q_len == 1, ctypes.c_long(B * per_seq // min(256, B * per_seq)), ctypes.c_long(per_seq)))
    return choose


@pytest.mark.parametrize("q_len", [1, 2, 3, 4])
@pytest.mark.parametrize("four_bit", [False, True])
def test_choice(takes_short, four_bit, q_len):
    # many short sequences: a workgroup's work is pieces of a few tiles
    for B, hint in ((512, 600), (900, 448), (1500, 200)):
        assert takes_short(four_bit, q_len, B, hint), (B, hint)
    # little work at all
    for B, hint in ((2, 256), (64, 512), (8, 6000)):
        assert takes_short(four_bit, q_len, B, hint), (B, hint)
    # 16 tiles per workgroup of long sequences: two tokens have left the short kernel, one has not
    assert takes_short(four_bit, q_len, 64, 4096) == (q_len == 1)
    # long contexts
    for B, hint in ((128, 8192), (64, 12288), (16, 32768)):
        assert not takes_short(four_bit, q_len, B, hint), (B, hint)
    # more work never leads back to the short kernel
    for hint in (64, 500, 704, 705, 5000, 32768):
        seen = [takes_short(four_bit, q_len, B, hint) for B in range(1, 4097, 7)]
        assert seen == sorted(seen, reverse=True)
