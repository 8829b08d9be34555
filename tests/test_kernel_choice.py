"""Which kernel a call takes, which is by sizes alone: the two of the 8-bit and 4-bit caches, and little work uncut or in runs."""
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


def test_short_contexts(tmp_path):
    """Which calls go uncut, and into how many parts: by rows, cache bits, query tokens and hint alone."""
    (tmp_path / "shim.cpp").write_text('#include "mfa_kernel_choice.hpp"\nextern "C" int parts(int bits, int q_len, long rows, long hint) { return mfa::brief_parts(bits, q_len, rows, hint); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.cpp")], check=True)
    f = ctypes.CDLL(str(tmp_path / "shim.so")).parts

    def parts(bits, q_len, rows, hint):
        return f(bits, q_len, ctypes.c_long(rows), ctypes.c_long(hint))
    for bits in (16, 8, 4):
        for q_len in (1, 2, 3, 4):
            for rows in list(range(1, 600)) + [4096, 65536]:
                # at most a workgroup per compute unit up to 128 rows, and what is cut at one hint is cut at every longer one
                p = parts(bits, q_len, rows, 64)
                assert p in (0, 2, 4, 8, 16) and (p > 0 or rows > 128) and (rows > 128 or p * rows <= 256)
                hints = [parts(bits, q_len, rows, hint) for hint in range(32, 8192, 96)]
                assert hints == sorted(hints, reverse=True) and set(hints) <= {0, p}
            assert parts(bits, q_len, 64, 8192) == 0 and parts(bits, q_len, 400, 64) == 0
    # where one sequence of the hint's length among short ones would wait for its fixed share of the chip
    for bits, rows, hint in ((16, 40, 1024), (16, 64, 960), (16, 66, 448), (16, 128, 448), (8, 64, 1536), (8, 66, 512), (8, 128, 512), (4, 64, 2048), (4, 128, 576)):
        assert parts(bits, 1, rows, hint) == 0 == parts(bits, 2, rows, hint), (bits, rows, hint)
    assert parts(8, 4, 128, 2048) == 0 == parts(8, 3, 66, 2048) and parts(16, 4, 68, 640) == 0
    assert parts(16, 1, 2, 256) == 16 and parts(16, 1, 64, 4096) == 0 and parts(8, 4, 64, 6144) == 4 and parts(8, 2, 64, 6144) == 0


def test_runs_of_few_rows(tmp_path):
    """Into how many runs a row of a longer context is cut: what the launch and the scratch memory rely on, over all rows, hints, cache bits and query tokens."""
    (tmp_path / "shim.cpp").write_text('#include "mfa_kernel_choice.hpp"\nextern "C" int runs(int bits, int q_len, long rows, long hint) { return mfa::brief_parts(bits, q_len, rows, hint) ? -1 : mfa::brief_runs(bits, q_len, rows, hint); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.cpp")], check=True)
    f = ctypes.CDLL(str(tmp_path / "shim.so")).runs

    def runs(bits, q_len, rows, hint):
        return f(bits, q_len, ctypes.c_long(rows), ctypes.c_long(hint))
    for bits in (16, 8, 4):
        for q_len in (1, 2, 3, 4):
            for rows in list(range(q_len, 40, q_len)) + [4096, 65536]:
                seen = [runs(bits, q_len, rows, hint) for hint in list(range(1, 4500)) + [8192, 16384, 32768, 65536, 131072, 262144, 1 << 20, (1 << 31) - 1]]
                # uncut, then runs (two at least, a workgroup per compute unit at most, never fewer for a longer hint), then the other kernels
                cut = [r for r in seen if r > 0]
                assert all(2 <= r and r * rows <= 64 for r in cut) and cut == sorted(cut)
                assert [min(r, 1) for r in seen] == [-1] * seen.count(-1) + [1] * len(cut) + [0] * seen.count(0)
                assert seen[-1] == 0 and (rows <= 32 or not cut)
    assert runs(16, 1, 1, 4096) == 64 and runs(16, 1, 5, 1500) == 11 and runs(8, 4, 16, 16384) == 4 and runs(8, 1, 22, 3000) == 0
    assert runs(8, 2, 32, 2816) == 2 and runs(8, 2, 32, 2817) == 0 and runs(16, 2, 22, 2048) == 2 and runs(16, 2, 22, 2049) == 0


def test_the_gpu_tests_of_little_work_take_the_forms_they_name(tmp_path):
    """Every size of test_short_contexts goes uncut, with all four numbers of parts and sixteen up to the longest context that has them; every size of test_runs goes in runs; the infinities
    are tested in each form."""
    import test_gpu_brief, test_gpu_brief_runs
    (tmp_path / "shim.cpp").write_text('#include "mfa_kernel_choice.hpp"\nextern "C" int parts(int bits, int q_len, long rows, long hint) { return mfa::brief_parts(bits, q_len, rows, hint); }\n'
                                       'extern "C" int runs(int bits, int q_len, long rows, long hint) { return mfa::brief_runs(bits, q_len, rows, hint); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(tmp_path / "shim.so"))
    parts = lambda bits, B, q_len, hint: lib.parts(bits, q_len, ctypes.c_long(B * q_len), ctypes.c_long(hint))
    for bits in (16, 8, 4):
        seen = {case: parts(bits, *case) for case in test_gpu_brief.CASES}
        assert set(seen.values()) == {16, 8, 4, 2}, seen
        assert max(hint for (_, q_len, hint), p in seen.items() if p == 16 and q_len == 1) == 1152
        for lens, q_len, hint, kv in test_gpu_brief_runs.RUNS:
            if {"bf16": 16, "fp8": 8, "fp4": 4}[kv] == bits:
                runs = lib.runs(bits, q_len, ctypes.c_long(len(lens) * q_len), ctypes.c_long(hint))
                assert parts(bits, len(lens), q_len, hint) == 0 and runs >= 2, (bits, lens, q_len, hint)
        assert [parts(bits, B, 1, S) for B, S in test_gpu_brief.INFINITIES] == [16, 8, 4, 2, 0]
