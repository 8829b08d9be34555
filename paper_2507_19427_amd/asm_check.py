"""Host-side checks of the compiled attention kernels and linear products (no GPU needed).

The attention kernels load cache data with inline-assembly loads (to LDS; short_lowbit_kernel also to registers) and wait for them
with inline-assembly s_waitcnt, counted where several stages are in flight (left to the compiler the wait would drain the
pipeline every stage); decode_lowbit_kernel, decode_bf16_multi_kernel and short_bf16_multi_kernel have their matrix instructions in inline
assembly too, and cover by hand the wait states before a result is read.  The compiler knows about neither.  So the
build checks the machine code it has just produced:

  * where an inline-assembly load writes registers (short_lowbit_kernel): between it and the explicit wait that covers it, no
    instruction of any kind names one of its destination registers (as a source or as a destination);
  * where loads go to LDS under a counted wait (decode_lowbit_kernel, decode_bf16_multi_kernel): on every way through the steady loop
    there are exactly the vector-memory operations of one stage, all of them inline-assembly loads to LDS, and one wait, which leaves
    exactly the younger stages outstanding;
  * no compiler-made vector-memory wait inside a pipeline loop: it would wait for the pipeline's own loads;
  * no instruction reads or writes a matrix instruction's result, and no matrix instruction reads a vector instruction's, before it is
    there (check_matrix_hazards);
  * the loading waves of gemm_loader_kernel ask for a load each time the oldest has landed (check_loading_loop): on every way through
    their loop there is one barrier and either a stage's loads, each behind a wait that leaves what is in flight but one, or, towards the
    end of the k range, one wait and no load; nothing else touches vector memory, and no wait is compiler-made;
  * the kernels use no scratch memory -- for every attention kernel and product, since scratch also costs every wave its set-up,
    and a reload inside a pipeline loop waits for everything in flight.

build.py runs check_attention_asm() and check_products_asm() on the assembly of every build and fails the build on a violation;
tests/test_build_asm.py runs the same functions, and the checkers themselves against planted mistakes.
"""
import re

# decode_lowbit_kernel, by (cache bits, query tokens): vector-memory operations of a wave per stage (direct loads of keys and values and
# one of scales: LowbitShape::kOps), and stages in flight beside the one awaited (kDepth - 1).
LOWBIT_STEADY = {(8, 1): (17, 0), (4, 1): (9, 0), (8, 2): (9, 0), (4, 2): (5, 1)}
# decode_bf16_multi_kernel: kMultiOps, kMultiDepth - 1
MULTI_STEADY = (8, 1)
# short_lowbit_kernel loads to registers in two unrolled steps, each of which waits for all but the youngest step's loads.
SHORT_OPS_PER_STEP = {8: 5, 4: 3}

# gemm_loader_kernel, by (16-row blocks of a wave, strips): loads of a loading wave per stage and stages in flight (LoaderShape::kLoads, kAhead).
LOADING = {(1, 1): (4, 1), (2, 1): (4, 1), (1, 4): (8, 1), (2, 4): (4, 2)}

_REG = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")


def lowbit_kernel_name(paged, q_len, bits):
    return f"_ZN3mfa20decode_lowbit_kernelILb{paged}ELi{q_len}ELi{bits}EEEvNS_8AttnArgsE"


def short_lowbit_kernel_name(paged, q_len, bits):
    return f"_ZN3mfa19short_lowbit_kernelILb{paged}ELi{q_len}ELi{bits}EEEvNS_8AttnArgsE"


def multi_kernel_name(paged, q_len):
    return f"_ZN3mfa24decode_bf16_multi_kernelILb{paged}ELi{q_len}EEEvNS_8AttnArgsE"


def kernel_body(text, mangled):
    start = text.index("\n" + mangled + ":")
    end = text.index(".size\t" + mangled, start)
    return text[start:end].split("\n")


def registers_named(operand_text):
    regs = set()
    for m in _REG.finditer(operand_text):
        if m.group(3) is not None:
            regs.add(int(m.group(3)))
        else:
            regs.update(range(int(m.group(1)), int(m.group(2)) + 1))
    return regs


def short_multi_kernel_name(paged):
    return f"_ZN3mfa23short_bf16_multi_kernelILb{paged}EEEvNS_8AttnArgsE"


class Instr:
    def __init__(self, text, in_asm):
        self.text, self.in_asm = text, in_asm
        self.op, _, rest = text.partition(" ")
        self.operands = [o.strip() for o in rest.split(",")] if rest else []

    @property
    def is_matrix(self):
        return self.op.startswith(("v_mfma", "v_smfmac"))

    @property
    def is_vector_memory(self):
        return self.op.startswith(("global_", "buffer_", "scratch_", "flat_"))

    @property
    def vector_memory_wait(self):
        m = re.search(r"vmcnt\((\d+)\)", self.text) if self.op == "s_waitcnt" else None
        return int(m.group(1)) if m else None


def basic_blocks(lines):
    """[[Instr]] and for each block the indexes of the blocks control can go to."""
    blocks, label_of, in_asm = [[]], {}, False
    for ln in lines:
        t = ln.strip()
        if t.startswith(";;#ASMSTART") or t.startswith(";;#ASMEND"):
            in_asm = t.startswith(";;#ASMSTART")
            continue
        if t.startswith(".LBB"):
            blocks.append([])
            label_of[t.split(":")[0]] = len(blocks) - 1
            continue
        t = " ".join(t.split(";")[0].split())
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        blocks[-1].append(Instr(t, in_asm))
        if t.startswith(("s_cbranch", "s_branch", "s_endpgm")):        # a block ends with its branch
            blocks.append([])
    successors = []
    for i, b in enumerate(blocks):
        last = b[-1].op if b else ""
        to = set()
        if last.startswith(("s_cbranch", "s_branch")):
            to.add(label_of[b[-1].operands[0]])
        if last not in ("s_branch", "s_endpgm") and i + 1 < len(blocks):
            to.add(i + 1)
        successors.append(to)
    return blocks, successors


def innermost_loop(successors, block):
    """(header, blocks) of the smallest natural loop that holds `block`, or None."""
    n = len(successors)
    reachable, todo = {0}, [0]
    while todo:
        for t in successors[todo.pop()]:
            if t not in reachable:
                reachable.add(t)
                todo.append(t)
    predecessors = [{i for i in reachable if b in successors[i]} for b in range(n)]
    dominators = {b: set(reachable) for b in reachable}
    dominators[0] = {0}
    changed = True
    while changed:
        changed = False
        for b in sorted(reachable - {0}):
            new = {b} | set.intersection(*(dominators[p] for p in predecessors[b]))
            if new != dominators[b]:
                dominators[b], changed = new, True
    best = None
    headers = {h for u in reachable for h in successors[u] if h in dominators[u]}
    for h in headers:
        body, todo = {h}, [u for u in reachable if h in successors[u] and h in dominators[u]]
        while todo:
            b = todo.pop()
            if b not in body:
                body.add(b)
                todo.extend(predecessors[b])
        if block in body and (best is None or len(body) < len(best[1])):
            best = (h, body)
    return best


def check_steady_loop(lines, mfmas, ops, stages_left):
    """Raises AssertionError unless the kernel has one steady loop -- a loop with `mfmas` matrix instructions in one block and
    direct loads beside them -- and every way through it issues `ops` vector-memory operations, all of them inline-assembly loads to
    LDS, and waits once, for all but the last stages_left * ops of them."""
    blocks, successors = basic_blocks(lines)
    steady = [i for i, b in enumerate(blocks) if sum(x.is_matrix for x in b) >= mfmas and sum(x.is_vector_memory for x in b) > 1]
    assert len(steady) == 1, f"{len(steady)} steady blocks"
    loop = innermost_loop(successors, steady[0])
    assert loop is not None, "the steady block is in no loop"
    header, body = loop
    for b in body:
        for x in blocks[b]:
            assert not any(o.startswith("exec") for o in x.operands[:1]) and "saveexec" not in x.op, f"lanes leave the loop: {x.text}"
            if x.is_vector_memory:
                assert x.in_asm and x.op.startswith("global_load_lds"), f"a vector-memory operation that is no load of the pipeline: {x.text}"
            if x.vector_memory_wait is not None:
                assert x.in_asm, f"compiler-made vector-memory wait in a pipeline loop: {x.text}"
                assert x.vector_memory_wait == stages_left * ops, f"waits for all but {x.vector_memory_wait}, not {stages_left * ops}: {x.text}"
    # every way from the header back to it: operations, waits and the flags known on the way
    closed, seen, todo = set(), set(), [(header, 0, 0, frozenset())]
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        b, n_ops, n_waits, flags = state
        n_ops += sum(x.is_vector_memory for x in blocks[b])
        n_waits += sum(x.vector_memory_wait is not None for x in blocks[b])
        assert n_ops <= ops and n_waits <= 1, f"{n_ops} operations and {n_waits} waits on a way through the loop"
        flags = flags_after(blocks[b], flags)
        for t in ways_on(blocks, successors, b, flags) & body:
            if t == header:
                closed.add((n_ops, n_waits))
            else:
                todo.append((t, n_ops, n_waits, flags))
    assert closed == {(ops, 1)}, f"(operations, waits) on the ways through the loop: {sorted(closed)}, not {(ops, 1)}"


# An if/else of a wave-uniform condition reaches the machine code as two branches: the first side sets a flag (vcc, or a pair of scalar
# registers) to 0 or -1, and a second branch skips the other side by it.  The flags known on a way are followed so that only the
# ways control can take are counted.
_SPAIR = re.compile(r"s\[(\d+):(\d+)\]")
_SREG = re.compile(r"s(\d+)")


def _scalars(operand):
    """The scalar registers an operand is; vcc as "vcc"."""
    if operand.startswith("vcc"):
        return {"vcc"}
    m = _SPAIR.fullmatch(operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = _SREG.fullmatch(operand)
    return {int(m.group(1))} if m else set()


def flags_after(block, flags):
    """{(flag, True or False)}: the flags (vcc and scalar pairs) known to be all ones or zero after a block, given those before it."""
    known = dict(flags)
    for x in block:
        value = None
        if x.op == "s_mov_b64" and x.operands[1] in ("0", "-1"):
            value = x.operands[1] == "-1"
        elif x.op in ("s_and_b64", "s_andn2_b64") and x.operands[1] == "exec" and x.operands[2] in known:
            value = known[x.operands[2]] == (x.op == "s_and_b64")
        if x.op.startswith(("s_", "v_cmp", "v_read", "v_add", "v_sub", "v_div_scale")):
            written = set().union(*(_scalars(o) for o in x.operands[:2 if x.op.startswith("v_") else 1]))
            known = {k: v for k, v in known.items() if not written & _scalars(k)}
        if value is not None:
            known[x.operands[0]] = value
    return frozenset(known.items())


def ways_on(blocks, successors, b, flags):
    """The successors of a block that control can reach with these flags (exec is not zero)."""
    last = blocks[b][-1] if blocks[b] else None
    known = dict(flags, exec=True)
    m = re.fullmatch(r"s_cbranch_(vcc|exec)(z|nz)", last.op) if last else None
    if not m or m.group(1) not in known:
        return successors[b]
    taken = known[m.group(1)] == (m.group(2) == "nz")
    target = next(t for t in successors[b] if t != b + 1) if len(successors[b]) > 1 else b + 1
    return {target if taken else b + 1}


# Passes (of four cycles) for which a matrix instruction of the kernels occupies the pipe.
MATRIX_PASSES = {"v_mfma_f32_32x32x64_f8f6f4": 16, "v_mfma_scale_f32_32x32x64_f8f6f4": 16, "v_mfma_f32_32x32x16_bf16": 8,
                 "v_mfma_f32_16x16x32_bf16": 4, "v_mfma_f32_16x16x128_f8f6f4": 8, "v_mfma_scale_f32_16x16x128_f8f6f4": 8}
RESULT_STATES = 4         # wait states from a matrix instruction's last pass to an instruction that names its result
OPERAND_STATES = 2        # wait states between a vector instruction and a matrix instruction that reads its result

_VREG = re.compile(r"\b([av])\[(\d+):(\d+)\]|\b([av])(\d+)\b")


def vector_registers(text):
    """{("v" or "a", number)} named in an operand."""
    regs = set()
    for m in _VREG.finditer(text):
        if m.group(4):
            regs.add((m.group(4), int(m.group(5))))
        else:
            regs.update((m.group(1), r) for r in range(int(m.group(2)), int(m.group(3)) + 1))
    return regs


def check_matrix_hazards(lines):
    """Raises AssertionError if, on some way through the code, an instruction names a matrix instruction's result before it is there
    (the accumulator of a following matrix instruction excepted: the pipe forwards it), or a matrix instruction reads a register that a
    vector instruction has just written.  Every instruction counts as one wait state, s_nop N as N + 1; a matrix instruction cannot
    start before the pipe has taken the ones ahead of it."""
    blocks, successors = basic_blocks(lines)
    regs = [[(x, [vector_registers(o) for o in x.operands]) for x in b] for b in blocks]
    def follow(first, index, result, need, source):
        """Walks on from instruction `index` of block `first`; elapsed counts wait states since the source issued, pipe when the pipe is free."""
        todo = [(first, index, 0, MATRIX_PASSES.get(source.op, 0))]
        while todo:
            b, i, elapsed, pipe = todo.pop()
            while i < len(regs[b]) and elapsed < need:
                x, named = regs[b][i]
                if x.is_matrix:
                    elapsed = max(elapsed, pipe)
                    if elapsed >= need:
                        break
                    if source.is_matrix:
                        accumulator = named[3] & result
                        assert not accumulator or named[3] == result == named[0], f"result read as part of an accumulator: {source.text} -> {x.text}"
                        early = set().union(*named[1:3], *named[4:]) & result
                    else:
                        early = set().union(*named[1:]) & result
                    assert not early, f"operand of a matrix instruction not there yet: {source.text} -> {x.text}"
                    pipe = max(elapsed, pipe) + MATRIX_PASSES[x.op]
                elif source.is_matrix:
                    assert not (set().union(*named) & result if named else set()), f"result named {elapsed} wait states after its matrix instruction, not {need}: {source.text} -> {x.text}"
                elapsed += int(x.operands[0]) + 1 if x.op == "s_nop" else 1
                i += 1
            if i == len(regs[b]) and elapsed < need:
                for t in successors[b]:
                    todo.append((t, 0, elapsed, pipe))

    for b, block in enumerate(regs):
        for i, (x, named) in enumerate(block):
            if x.is_matrix:
                assert x.op in MATRIX_PASSES, f"unknown matrix instruction: {x.text}"
                follow(b, i + 1, named[0], MATRIX_PASSES[x.op] + RESULT_STATES, x)
            elif x.op.startswith("v_") and named:
                written = set().union(*named[:2]) if "swap" in x.op else named[0]
                if written:
                    follow(b, i + 1, written, OPERAND_STATES, x)


def check_pipeline(lines, ops_per_step=5, steps=1):
    """Raises AssertionError when the register pipeline of a kernel body (lines of assembly) is disturbed."""
    in_asm = False
    queue = []                 # vector-memory operations in issue order: the registers each one writes
                               # (empty for direct-to-LDS loads, stores and compiler-made loads)
    partial_waits = 0

    def in_flight():
        regs = set()
        for r in queue:
            regs |= r
        return regs

    for ln in lines:
        t = ln.strip()
        if t.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if t.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not t or t.startswith(";") or t.startswith("."):
            continue
        t = t.split(";")[0].strip()                    # drop trailing comments
        op, _, rest = t.partition(" ")
        if op.startswith("global_load") or op.startswith("global_store") or op.startswith("buffer_") or \
                op.startswith("scratch_") or op.startswith("flat_"):
            operands = [o.strip() for o in rest.split(",")] if rest else []
            tracked = in_asm and op in ("global_load_dwordx4", "global_load_dword")
            touched = registers_named(rest)
            if tracked:
                dest = registers_named(operands[0])
                assert not (dest & in_flight()), f"a pipeline load overwrites a register still in flight: {t}"
                assert not ((touched - dest) & in_flight()), f"in-flight register used as an address: {t}"
                queue.append(dest)
            else:
                assert not (touched & in_flight()), f"in-flight register touched by a memory instruction before its wait: {t}"
                queue.append(set())
            continue
        if op == "s_waitcnt" and "vmcnt" in rest:
            left = int(re.search(r"vmcnt\((\d+)\)", rest).group(1))
            if in_asm and left == ops_per_step:
                partial_waits += 1
            if not in_asm and partial_waits > 0:
                # a compiler-made vector-memory wait inside the pipeline loop: it must not reach the
                # pipeline's own loads (the compiler does not count them, so its number is too small)
                assert not in_flight(), f"compiler-inserted wait drains the pipeline: {t}"
            queue = queue[max(0, len(queue) - left):] if left else []
            continue
        touched = registers_named(rest)
        assert not (touched & in_flight()), f"in-flight register touched before its wait: {t}"
    assert partial_waits >= steps, "every unrolled step waits for all but the youngest stage's loads"


def check_no_compiler_wait_in_loop(lines, mfmas=32):
    """Raises AssertionError if a basic block with at least `mfmas` matrix instructions (a pipeline loop's body) holds a
    compiler-made vector-memory wait."""
    blocks, in_asm = [[0, None]], False
    for ln in lines:
        t = ln.strip()
        if t.startswith(";;#ASMSTART") or t.startswith(";;#ASMEND"):
            in_asm = t.startswith(";;#ASMSTART")
        elif t.startswith(".LBB"):
            blocks.append([0, None])
        elif "mfma" in t and not t.startswith(";"):
            blocks[-1][0] += 1
        elif t.startswith("s_waitcnt") and "vmcnt" in t and not in_asm:
            blocks[-1][1] = t
    assert any(n >= mfmas for n, _ in blocks), "no pipeline loop found"
    for n, wait in blocks:
        assert n < mfmas or wait is None, f"compiler-made vector-memory wait in a pipeline loop: {wait}"


def scratch_bytes(text):
    """{kernel name: bytes of scratch per lane} from the .amdhsa_private_segment_fixed_size directives."""
    out = {}
    name = None
    for ln in text.split("\n"):
        t = ln.strip()
        if t.startswith(".amdhsa_kernel "):
            name = t.split()[1]
        elif t.startswith(".amdhsa_private_segment_fixed_size") and name is not None:
            out[name] = int(t.split()[1])
        elif t.startswith(".end_amdhsa_kernel"):
            name = None
    return out


def check_attention_asm(text):
    """All checks on the assembly text of mfa_attn.hip.  Raises AssertionError naming the first violation."""
    checks = []
    for paged in (0, 1):
        for q_len in (1, 2):
            for bits in (8, 4):
                ops, left = LOWBIT_STEADY[bits, q_len]
                name = lowbit_kernel_name(paged, q_len, bits)
                checks += [(name, check_steady_loop, (32, ops, left)), (name, check_no_compiler_wait_in_loop, (32,)), (name, check_matrix_hazards, ())]
                checks.append((short_lowbit_kernel_name(paged, q_len, bits), check_pipeline, (SHORT_OPS_PER_STEP[bits], 2)))
            name = multi_kernel_name(paged, q_len + 2)
            checks += [(name, check_steady_loop, (64, *MULTI_STEADY)), (name, check_no_compiler_wait_in_loop, (64,)), (name, check_matrix_hazards, ())]
        checks.append((short_multi_kernel_name(paged), check_matrix_hazards, ()))
    for name, check, args in checks:
        try:
            check(kernel_body(text, name), *args)
        except AssertionError as e:
            raise AssertionError(f"{name}: {e}") from None
    scratch = scratch_bytes(text)
    decode = {k: v for k, v in scratch.items() if "decode_" in k}
    assert len(decode) == 16, f"expected 16 attention kernels, found {sorted(decode)}"
    short = {k: v for k, v in scratch.items() if "short_" in k}
    assert len(short) == 10, f"expected 10 attention kernels for little work, found {sorted(short)}"
    brief = {k: v for k, v in scratch.items() if "brief_attn" in k}
    assert len(brief) == 30, f"expected 30 attention kernels for short contexts, found {sorted(brief)}"
    for name, nbytes in {**decode, **short, **brief}.items():
        assert nbytes == 0, f"{name} uses {nbytes} bytes of scratch per lane (register spills)"


def check_loading_loop(lines, loads, stages):
    """Raises AssertionError unless the kernel's loading waves keep `stages` stages of `loads` direct loads in flight, asking for the next
    load whenever the oldest has landed."""
    blocks, successors = basic_blocks(lines)
    loading = [i for i, b in enumerate(blocks) if any(x.op.startswith("global_load_lds") for x in b) and any(x.vector_memory_wait is not None for x in b)]
    assert len(loading) == 1, f"{len(loading)} loading blocks"
    loop = innermost_loop(successors, loading[0])
    assert loop is not None, "the loading block is in no loop"
    header, body = loop
    left = stages * loads - 1
    closed, todo = set(), [(header, (), frozenset())]
    while todo:
        b, way, flags = todo.pop()
        for x in blocks[b]:
            if x.is_vector_memory:
                assert x.in_asm and x.op.startswith("global_load_lds"), f"a vector-memory operation that is no load of the pipeline: {x.text}"
                way += ("load",)
            elif x.vector_memory_wait is not None:
                assert x.in_asm, f"compiler-made vector-memory wait in a loading loop: {x.text}"
                way += (x.vector_memory_wait,)
            elif x.op == "s_barrier":
                way += ("barrier",)
            assert len(way) <= 2 * loads + 1, f"more than a stage on a way through the loop: {way}"
        flags = flags_after(blocks[b], flags)
        for t in ways_on(blocks, successors, b, flags) & body:
            if t == header:
                closed.add(way)
            else:
                todo.append((t, way, flags))
    steady = (left, "load") * loads + ("barrier",)
    ends = {(0, "barrier")} | ({((stages - 1) * loads, "barrier")} if stages > 1 else set())
    assert steady in closed and closed <= {steady} | ends, f"ways through the loop: {sorted(map(str, closed - {steady} - ends))} beside {steady in closed}"


def check_products_asm(text):
    """All checks on the assembly text of mfa_qproj.hip.  Raises AssertionError naming the first violation."""
    names = re.findall(r"^(_ZN3mfa\w*gemm_loader_kernelI\w+):", text, re.M)
    assert len(names) == 10, f"expected 10 forms of the product, found {names}"
    scratch = scratch_bytes(text)
    for name in names:
        row_blocks, strips = (int(x) for x in re.search(r"Li(\d)ELi(\d)EEEv", name).groups())
        try:
            check_loading_loop(kernel_body(text, name), *LOADING[row_blocks, strips])
        except AssertionError as e:
            raise AssertionError(f"{name}: {e}") from None
        assert scratch[name] == 0, f"{name} uses {scratch[name]} bytes of scratch per lane (register spills)"
