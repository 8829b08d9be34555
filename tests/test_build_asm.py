"""Host-side check of the compiled attention kernels and linear products (the checker is paper_2507_19427_amd/asm_check.py, which
the build itself runs on every library it produces).  Here: the same checks on a fresh compilation of
mfa_attn.hip, kernel by kernel, and of mfa_qproj.hip, and the checker against planted mistakes."""
import os
import shutil
import subprocess

import pytest

from paper_2507_19427_amd import asm_check as A

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_19427_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _assembly(tmp_path_factory, name):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / f"{name}.s"
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "--cuda-device-only", "-S", "-o", str(out), os.path.join(CSRC, f"{name}.hip")]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    return out.read_text()


@pytest.fixture(scope="module")
def asm_text(tmp_path_factory):
    return _assembly(tmp_path_factory, "mfa_attn")


@pytest.fixture(scope="module")
def products_text(tmp_path_factory):
    return _assembly(tmp_path_factory, "mfa_qproj")


LOWBIT = [(paged, q_len, bits) for bits in (8, 4) for q_len in (1, 2) for paged in (0, 1)]
MULTI = [(paged, q_len) for q_len in (3, 4) for paged in (0, 1)]


@pytest.mark.parametrize("paged,q_len,bits", LOWBIT)
def test_lowbit_pipeline_registers_stay_untouched_between_load_and_wait(asm_text, paged, q_len, bits):
    """(The kernel for little work loads to registers; the other one to LDS: next test.)"""
    lines = A.kernel_body(asm_text, A.short_lowbit_kernel_name(paged, q_len, bits))
    assert any(x.in_asm and x.op in ("global_load_dwordx4", "global_load_dword") for b in A.basic_blocks(lines)[0] for x in b)
    A.check_pipeline(lines, A.SHORT_OPS_PER_STEP[bits], 2)


@pytest.mark.parametrize("paged,q_len,bits", LOWBIT)
def test_lowbit_steady_loop_issues_and_awaits_whole_stages(asm_text, paged, q_len, bits):
    A.check_steady_loop(A.kernel_body(asm_text, A.lowbit_kernel_name(paged, q_len, bits)), 32, *A.LOWBIT_STEADY[bits, q_len])


@pytest.mark.parametrize("paged,q_len", MULTI)
def test_multi_steady_loop_issues_and_awaits_whole_stages(asm_text, paged, q_len):
    A.check_steady_loop(A.kernel_body(asm_text, A.multi_kernel_name(paged, q_len)), 64, *A.MULTI_STEADY)


@pytest.mark.parametrize("name", [A.lowbit_kernel_name(*k) for k in LOWBIT] + [A.multi_kernel_name(*k) for k in MULTI] +
                         [A.short_multi_kernel_name(p) for p in (0, 1)])
def test_matrix_results_are_there_before_they_are_named(asm_text, name):
    A.check_matrix_hazards(A.kernel_body(asm_text, name))


def test_no_attention_kernel_uses_scratch_memory(asm_text):
    scratch = {k: v for k, v in A.scratch_bytes(asm_text).items() if "decode_" in k}
    assert len(scratch) == 16        # bf16 / 8 bit / 4 bit x paged or not x one or two query tokens; bf16 x paged or not x three or four
    assert all(v == 0 for v in scratch.values()), scratch


def test_everything_the_build_checks(asm_text):
    A.check_attention_asm(asm_text)


def test_loading_waves_of_the_products(products_text):
    A.check_products_asm(products_text)


def _snippet(between):
    load = [";;#ASMSTART", "global_load_dwordx4 v[10:13], v[2:3], off", ";;#ASMEND"]
    wait = [";;#ASMSTART", "s_waitcnt vmcnt(5)", ";;#ASMEND"]
    filler = [";;#ASMSTART"] + ["global_load_lds_dwordx4 v[4:5], off"] * 5 + [";;#ASMEND"]
    return wait + load + filler + wait + load + filler + between + wait + ["v_mov_b32_e32 v20, v11"]


def test_the_checker_itself_catches_planted_mistakes():
    A.check_pipeline(_snippet([]))                                   # clean: the copy comes after the wait
    A.check_pipeline(_snippet(["v_add_f32_e32 v21, v14, v15"]))      # clean: other registers
    for bad in ("v_mov_b32_e32 v20, v11",                            # copied
                "v_add_f32_e32 v21, v10, v15",                       # read by arithmetic
                "v_mov_b32_e32 v12, v30",                            # overwritten
                "v_pk_mul_f32 v[40:41], v[12:13], v[2:3]",           # read as part of a register range
                "ds_write_b128 v7, v[10:13]"):                       # stored to LDS
        with pytest.raises(AssertionError, match="touched before its wait"):
            A.check_pipeline(_snippet([bad]))
    with pytest.raises(AssertionError, match="touched by a memory instruction"):
        A.check_pipeline(_snippet(["scratch_store_dwordx4 off, v[10:13], off offset:16"]))   # spilled
    with pytest.raises(AssertionError, match="drains the pipeline"):
        A.check_pipeline(_snippet(["s_waitcnt vmcnt(0)"]))


def _loop(body, wait="s_waitcnt vmcnt(3)", loads=3):
    """A kernel with a steady loop of two matrix instructions and three direct loads per iteration, one stage left in flight."""
    asm = lambda *t: [";;#ASMSTART", *t, ";;#ASMEND"]
    load = asm("s_mov_b32 m0, s4", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3] nt")
    matrix = asm("v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]")
    return ["s_mov_b32 s0, 0", ".LBB0_1:"] + asm(wait) + ["s_barrier"] + load * loads + matrix * 2 + body + \
           ["s_add_i32 s0, s0, 1", "s_cmp_lt_i32 s0, s1", "s_cbranch_scc1 .LBB0_1", "s_endpgm"]


def test_the_steady_loop_check_catches_planted_mistakes():
    check = lambda lines: A.check_steady_loop(lines, 2, 3, 1)
    check(_loop([]))
    check(_loop(["s_waitcnt lgkmcnt(0)", "ds_read_b128 v[12:15], v3"]))
    for bad, message in ((_loop(["s_waitcnt vmcnt(0)"]), "compiler-made"),
                         (_loop(["global_load_dword v20, v1, s[2:3]"]), "no load of the pipeline"),
                         (_loop(["global_store_dword v1, v20, s[2:3]"]), "no load of the pipeline"),
                         (_loop(["scratch_load_dword v20, off, off offset:16"]), "no load of the pipeline"),
                         (_loop([], loads=2), "operations"),
                         (_loop([], loads=4), "operations"),
                         (_loop([], wait="s_waitcnt vmcnt(4)"), "waits for all but 4"),
                         (_loop([], wait="s_waitcnt lgkmcnt(0)"), "waits"),
                         (_loop(["v_cmp_eq_u32 vcc, 0, v2", "s_and_saveexec_b64 s[8:9], vcc", "s_or_b64 exec, exec, s[8:9]"]), "lanes leave"),
                         (_loop([])[:-2] + ["s_endpgm"], "in no loop")):
        with pytest.raises(AssertionError, match=message):
            check(bad)
    # two sides of a uniform condition, each with a stage's loads: the flag keeps them apart; without it both could run
    asm_load = [";;#ASMSTART"] + ["global_load_lds_dwordx4 v1, s[2:3] nt"] * 3 + [";;#ASMEND"]
    def sides(flag):
        return [".LBB0_1:", ";;#ASMSTART", "s_waitcnt vmcnt(3)", ";;#ASMEND", "s_mov_b64 s[8:9], -1", "s_cbranch_scc1 .LBB0_2"] + asm_load + flag + \
               [".LBB0_2:", "s_andn2_b64 vcc, exec, s[8:9]", "s_cbranch_vccnz .LBB0_3"] + asm_load + \
               ["v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"] * 2 + \
               [".LBB0_3:", "s_cmp_lt_i32 s0, s1", "s_cbranch_scc1 .LBB0_1", "s_endpgm"]
    check(["s_mov_b32 s0, 0"] + sides(["s_mov_b64 s[8:9], 0"]))
    for flag in ([], ["s_mov_b64 s[8:9], 0", "s_mov_b32 s9, s10"]):
        with pytest.raises(AssertionError, match="operations"):
            check(["s_mov_b32 s0, 0"] + sides(flag))


def test_the_loading_loop_check_catches_planted_mistakes():
    asm = lambda *t: [";;#ASMSTART", *t, ";;#ASMEND"]
    load = asm("s_mov_b32 m0, s4", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3] nt")

    def loop(pairs, end_wait="s_waitcnt vmcnt(0)", barrier="s_waitcnt lgkmcnt(0)\ns_barrier", extra=()):
        end = asm(end_wait) if end_wait else []
        return load * 2 + [".LBB0_1:", "s_cbranch_scc0 .LBB0_2", *pairs, *extra, "s_branch .LBB0_3", ".LBB0_2:", *end, ".LBB0_3:", *asm(*barrier.split("\n")),
                           "s_add_i32 s0, s0, 1", "s_cmp_lt_i32 s0, s1", "s_cbranch_scc1 .LBB0_1", "s_endpgm"]

    pair = asm("s_waitcnt vmcnt(1)") + load
    A.check_loading_loop(loop(pair * 2), 2, 1)
    A.check_loading_loop(loop((asm("s_waitcnt vmcnt(3)") + load) * 2, end_wait="s_waitcnt vmcnt(2)"), 2, 2)
    for bad in (loop(pair + load), loop(pair), loop(pair * 3), loop((asm("s_waitcnt vmcnt(2)") + load) * 2),       # a wait or a load too few or too many, counted wrongly
                loop(pair * 2, end_wait=None), loop(pair * 2, end_wait="s_waitcnt vmcnt(1)"),                          # the last stages not awaited
                loop(pair * 2, barrier="s_nop 0"),
                loop(pair * 2, extra=["s_waitcnt vmcnt(0)"]), loop(pair * 2, extra=["scratch_load_dword v20, off, off offset:16"]),
                loop(pair * 2, extra=["global_store_dword v1, v20, s[2:3]"]), loop(pair * 2)[:-2] + ["s_endpgm"]):
        with pytest.raises(AssertionError):
            A.check_loading_loop(bad, 2, 1)


def test_the_compiler_wait_check_catches_planted_mistakes():
    A.check_no_compiler_wait_in_loop(_loop([]), 2)
    A.check_no_compiler_wait_in_loop(_loop([]) + [".LBB0_2:", "s_waitcnt vmcnt(0)"], 2)         # (after the loop)
    with pytest.raises(AssertionError, match="compiler-made"):
        A.check_no_compiler_wait_in_loop(_loop(["s_waitcnt vmcnt(0)"]), 2)
    with pytest.raises(AssertionError, match="no pipeline loop"):
        A.check_no_compiler_wait_in_loop(_loop([]), 3)


def test_the_matrix_hazard_check_catches_planted_mistakes():
    big, small = "v_mfma_f32_32x32x64_f8f6f4 v[0:15], v[32:39], v[40:47], 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[48:51], v[52:55], a[0:15]"
    other = "v_mfma_f32_32x32x64_f8f6f4 v[64:79], v[32:39], v[40:47], 0"
    read = "v_max_f32_e32 v20, v3, v3"
    clean = [[big, "s_nop 7", "s_nop 7", "s_nop 3", read],                           # 20 wait states
             [big, other, other, read],                                              # the pipe has taken two more
             [big, other, "s_nop 2", read],                                          # 16 passes, one issue and 3
             [big, big.replace(", 0", ", v[0:15]"), other, other, read],             # its own accumulator
             [small, "s_nop 7", "s_nop 3", "v_accvgpr_read_b32 v20, a3"],
             [big, "ds_read_b128 v[16:19], v31", "v_add_f32_e32 v21, v22, v23", "s_endpgm"],
             ["v_add_f32_e32 v48, v1, v2", "s_nop 1", small]]
    bad = [[big, "s_nop 7", "s_nop 7", "s_nop 2", read],
           [big, other, "s_nop 1", read],
           [big, "s_nop 7", "v_mov_b32_e32 v0, 0"],                                  # overwritten
           [big, "s_nop 7", "ds_write_b128 v31, v[12:15]"],
           [big, "v_mfma_f32_32x32x64_f8f6f4 v[64:79], v[8:15], v[40:47], 0"],       # an operand of the next
           [big, "v_mfma_f32_32x32x64_f8f6f4 v[64:79], v[32:39], v[40:47], v[8:23]"],   # part of another accumulator
           [small, "s_nop 7", "s_nop 2", "v_accvgpr_read_b32 v20, a3"],
           [".LBB0_1:", read, "s_nop 7", big, "s_cbranch_scc1 .LBB0_1", "s_endpgm"],    # round the loop
           [big, "s_cbranch_scc1 .LBB0_1", "s_nop 7", "s_nop 7", "s_nop 7", read, ".LBB0_1:", read],
           ["v_add_f32_e32 v48, v1, v2", "s_nop 0", small],
           ["v_accvgpr_write_b32 a3, v2", small],
           ["v_permlane32_swap_b32_e32 v1, v49", small]]
    for code in clean:
        A.check_matrix_hazards(code)
    for code in bad:
        with pytest.raises(AssertionError):
            A.check_matrix_hazards(code)
    with pytest.raises(AssertionError, match="unknown matrix instruction"):
        A.check_matrix_hazards(["v_mfma_f32_4x4x4_16b_f16 a[0:3], v[0:1], v[2:3], a[0:3]"])


def test_scratch_directive_parser():
    text = "\n".join(["\t.amdhsa_kernel _ZN3mfa18decode_x", "\t\t.amdhsa_private_segment_fixed_size 24", "\t.end_amdhsa_kernel",
                      "\t.amdhsa_kernel other", "\t\t.amdhsa_private_segment_fixed_size 0", "\t.end_amdhsa_kernel"])
    assert A.scratch_bytes(text) == {"_ZN3mfa18decode_x": 24, "other": 0}
