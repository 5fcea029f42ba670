"""Wait states around the instructions that the fine kernels write as inline assembly: the compiler inserts none for
them, so the emitted code of every kernel instance is checked, over all paths; and, in the forward, that copies to LDS have
landed before their place is used for anything else.

  M0 written by a scalar instruction, then read by a copy to LDS            1 wait state
  scalar register written by a vector instruction, then a copy's address    5
  vector result, then an operand of a matrix instruction                    2
  matrix result, then anything but the accumulator of the next one         12
  accumulator input of a matrix instruction, then a vector write over it    8 (where it is not its result)
(the "manually inserted wait states" table of the CDNA3 ISA document; the last two for matrix instructions of 8 passes,
v_mfma_f32_32x32x16_bf16, with a pass to spare.  A matrix instruction behind another starts when
that one's 8 passes are over, which counts in the last two.  The 2 count instructions, whatever lies between.
v_mfma_f32_16x16x32_bf16 has 4 passes and needs 8 and 4 states: where the rule for 8 passes holds, counting 8 for each between, so does that.)
"""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2505_13389_amd import build

FILES = ("fine_fwd.hip", "fine_fwd_short.hip", "fine_bwd.hip", "fine_bwd_dkv.hip")


def regs(operand):
    """The registers an operand names, as (kind, number)."""
    name = operand.split()[0] if operand.split() else ""
    m = re.fullmatch(r"([vas])\[(\d+):(\d+)\]", name)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.fullmatch(r"([vas])(\d+)", name)
    if m:
        return {(m[1], int(m[2]))}
    return {(name, 0)} if name in ("m0", "vcc") else set()


class Instruction:
    def __init__(self, text):
        self.text = text
        op, _, rest = text.partition(" ")
        self.op = op
        self.operands = [x.strip() for x in rest.split(",")] if rest.strip() else []
        named = [regs(x) for x in self.operands]
        self.matrix = op.startswith("v_mfma")
        self.vector = op.startswith("v_") and not self.matrix
        self.copy = "load_lds" in op
        no_result = self.copy or op.startswith(("ds_write", "global_store", "s_cmp", "s_cbranch", "s_waitcnt", "s_barrier"))
        self.writes = set() if no_result or not named else named[0]
        self.reads = set().union(*(named if no_result else named[1:]))
        self.accumulator = named[3] if self.matrix and len(named) > 3 else set()
        self.states = int(self.operands[0], 0) + 1 if op == "s_nop" else 1


def parse(lines):
    """Instructions of one kernel with their successors."""
    code, labels = [], {}
    for line in lines:
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            labels[m[1]] = len(code)
            continue
        text = " ".join(line.split(";")[0].split())
        if text and not text.startswith(".") and not text.endswith(":"):
            code.append(Instruction(text))
    for n, i in enumerate(code):
        i.next = [n + 1] if n + 1 < len(code) else []
        if i.op.startswith("s_cbranch"):
            i.next = i.next + [labels[i.operands[0]]]
        elif i.op == "s_branch":
            i.next = [labels[i.operands[0]]]
        elif i.op == "s_endpgm":
            i.next = []
    return code


def within(code, start, states, visit, passes=1):
    """visit(instruction, wait states since `start`) along every path while fewer than `states` have passed; a path ends
    where visit returns True.  `passes`: wait states a matrix instruction counts for."""
    best, todo = {}, [(n, 0) for n in code[start].next]
    while todo:
        n, age = todo.pop()
        if age >= states or best.get(n, states) <= age:
            continue
        best[n] = age
        if not visit(code[n], age):
            todo += [(m, age + (passes if code[n].matrix else code[n].states)) for m in code[n].next]


def faults(code):
    found = []

    def note(rule, a, b, age):
        found.append(f"{rule}: '{a.text}' ... {age} ... '{b.text}'")

    for n, a in enumerate(code):
        if ("m0", 0) in a.writes:
            within(code, n, 1, lambda b, age: b.copy and note("M0 before a copy", a, b, age))
        scalars = {r for r in a.writes if r[0] in ("s", "vcc")} if a.vector else set()
        if scalars:
            def address(b, age):
                if b.copy and b.reads & scalars:
                    note("address from a vector instruction", a, b, age)
                return bool(b.writes & scalars)  # (written anew by a scalar instruction, which has waited)
            within(code, n, 5, address)
        vectors = {r for r in a.writes if r[0] in ("v", "a")} if a.vector else set()
        if vectors:
            within(code, n, 2, lambda b, age: b.matrix and b.reads & vectors and note("vector result to matrix operand", a, b, age))
        if a.matrix:
            def result(b, age):
                if b.matrix and b.accumulator == a.writes:
                    if (b.reads - b.accumulator) & a.writes:
                        note("matrix result to matrix operand", a, b, age)
                    return True
                if (b.reads | b.writes) & a.writes:
                    note("matrix result used", a, b, age)
                return False
            within(code, n, 12, result, passes=8)
            if a.accumulator - a.writes:
                within(code, n, 8, lambda b, age: b.vector and b.writes & a.accumulator and
                       note("accumulator input overwritten", a, b, age), passes=8)
    return found


def before_it_lands(code, start, hit):
    """Instructions that `hit` accepts and that some path reaches from the copy `start` before it has waited for the copy:
    vector memory accesses count down in issue order, so the wait is for no more of them than were issued behind it."""
    found, best, todo = [], {}, [(n, 0) for n in code[start].next]
    while todo:
        n, behind = todo.pop()
        if best.get(n, behind + 1) <= behind:
            continue
        best[n] = behind
        i = code[n]
        wait = re.search(r"vmcnt\((\d+)\)", i.text) if i.op == "s_waitcnt" else None
        if wait and int(wait[1]) <= behind:
            continue
        if hit(i):
            found.append(i)
            continue
        behind += i.op.startswith(("global_", "buffer_", "flat_", "scratch_"))
        todo += [(m, behind) for m in i.next]
    return found


def mask_copies(code):
    return [n for n, i in enumerate(code) if i.op == "global_load_lds_dword"]


def kernels(path):
    name, lines = None, []
    for line in open(path):
        m = re.match(r"(_Z\w+):", line)
        if m:
            name, lines = m[1], []
        elif line.startswith(".Lfunc_end"):
            if name:
                yield name, parse(lines)
            name = None
        elif name:
            lines.append(line)


@pytest.fixture(scope="module")
def emitted(tmp_path_factory):
    """Source -> path of the code the compiler emits for it."""
    if shutil.which("hipcc") is None:
        pytest.skip("no compiler")
    place = tmp_path_factory.mktemp("emitted")

    def compile_one(source):
        out = str(place / source.replace(".hip", ".s"))
        subprocess.run(["hipcc", *build.FLAGS, *build.FILE_FLAGS.get(source, []), "-S", "--offload-device-only",
                        os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
        return out
    with ThreadPoolExecutor(max_workers=8) as ex:
        return dict(zip(build.SOURCES, ex.map(compile_one, build.SOURCES)))


@pytest.mark.parametrize("source", FILES)
def test_wait_states_of_the_emitted_code(source, emitted):
    seen = 0
    for name, code in kernels(emitted[source]):
        seen += sum(i.copy for i in code)
        found = faults(code)
        assert not found, f"{name}: {len(found)}, the first: {found[0]}"
    assert seen  # (the copies are where the test looks for them)


def test_key_masks_land_before_their_place_is_used_again(emitted):
    """Forward: the key masks reach registers by way of the memory that holds the softmax statistics at the end, also in a
    wavefront that has no unit to multiply."""
    seen = 0
    for name, code in kernels(emitted["fine_fwd.hip"]):
        for n in mask_copies(code):
            seen += 1
            early = before_it_lands(code, n, lambda i: i.op.startswith("ds_write"))
            assert not early, f"{name}: '{early[0].text}' while '{code[n].text}' may be in flight"
    assert seen


def test_q_lands_before_it_is_read(emitted):
    """Forward: the copies of Q, those ahead of the first key masks, have landed in every wavefront before the barrier
    behind which all of them read Q (the coarse stage inside the kernel has barriers of its own before that) and before
    the first operand is read."""
    seen = 0
    for name, code in kernels(emitted["fine_fwd.hip"]):
        masks = mask_copies(code)
        if not masks:
            continue
        coarse = re.search(r"ELb[01]ELb1E", name)  # (template arguments ..., PAIRS, COARSE, ...)
        for n in range(masks[0]):
            if code[n].op == "global_load_lds_dwordx4":
                seen += 1
                early = before_it_lands(code, n, lambda i: i.op in ("ds_read_b128", "ds_read_b64_tr_b16") or
                                        not coarse and i.op == "s_barrier")
                assert not early, f"{name}: '{early[0].text}' while '{code[n].text}' may be in flight"
    assert seen


@pytest.mark.parametrize("source", build.SOURCES)
def test_no_kernel_needs_private_memory(source, emitted):
    """The runtime provides private memory when a kernel that needs it is launched, and the library never allocates."""
    text = open(emitted[source]).read()
    sizes = re.findall(r"\.private_segment_fixed_size: +(\d+)", text)
    assert len(sizes) == len(re.findall(r"^\s*\.amdhsa_kernel ", text, re.M)) and not any(map(int, sizes)), sizes


def transcendental_results_used_at_once(code):
    return [(a.text, code[m].text) for a in code if re.match(r"v_(exp|log|rcp|rsq|sqrt)_", a.op)
            for m in a.next if code[m].vector and code[m].reads & a.writes and not re.match(r"v_(exp|log|rcp|rsq|sqrt)_", code[m].op)]


@pytest.mark.parametrize("source", FILES)
def test_transcendental_results_have_a_wait_state(source, emitted):
    """One instruction lies between an exponential and plain vector arithmetic on its result.  The compiler sees to that, but it counts
    the empty assembly statements that hold the stages of the fine kernels in place as one."""
    for name, code in kernels(emitted[source]):
        found = transcendental_results_used_at_once(code)
        assert not found, f"{name}: {len(found)}, the first: {found[0]}"


def test_the_check_sees_a_result_used_at_once():
    of = lambda *text: transcendental_results_used_at_once(parse(text + ("s_endpgm",)))
    assert of("v_exp_f32_e32 v1, v2", "v_add_f32_e32 v3, v3, v1")
    assert not of("v_exp_f32_e32 v1, v2", "s_nop 0", "v_add_f32_e32 v3, v3, v1") and not of("v_exp_f32_e32 v1, v2", "v_add_f32_e32 v3, v3, v4")


def walks(code):
    """Instructions of the loops that walk a list: without loops in them, a matrix instruction in 16 or more."""
    loops = [range(t, n + 1) for n, i in enumerate(code) for t in i.next if t <= n]
    for loop in loops:
        matrix = sum(code[n].matrix for n in loop)
        if matrix >= 16 and 16 * matrix >= len(loop) and not any(x != loop and x[0] >= loop[0] and x[-1] <= loop[-1] for x in loops):
            yield loop


def waits_for_later_operands(code, far=8):
    """Waits for some, not all, of the LDS reads in flight that are for an operand which the next `far` matrix instructions
    do not use: the reads are counted in issue order, so such a wait leaves fewer in flight than it could."""
    found = []
    for n in {n for loop in walks(code) for n in loop if code[n].op.startswith("ds_read")}:
        read, behind, wait, matrix = code[n], 0, None, 0
        for i in code[n + 1:]:
            m = re.search(r"lgkmcnt\((\d+)\)", i.text) if i.op == "s_waitcnt" else None
            if wait is None and m and int(m[1]) <= behind:
                wait = i
            behind += i.op.startswith(("ds_", "s_load"))
            if (i.reads | i.writes) & read.writes or i.op == "s_branch":
                if i.matrix and wait is not None and matrix >= far and "lgkmcnt(0)" not in wait.text:
                    found.append(f"'{wait.text}' for '{read.text}', used {matrix} matrix instructions later")
                break
            matrix += i.matrix and wait is not None
    return found


@pytest.mark.parametrize("source", ["fine_fwd.hip", "fine_bwd.hip", "fine_bwd_dkv.hip"])
def test_counted_waits_leave_later_operands_in_flight(source, emitted):
    """A wait with the wrong number waits for too much where it is too small (too large, the compiler's own waits stand in)."""
    seen = 0
    for name, code in kernels(emitted[source]):
        seen += sum(map(len, walks(code)))
        found = waits_for_later_operands(code)
        assert not found, f"{name}: {len(found)}, the first: {found[0]}"
    assert seen


def test_the_check_sees_a_wait_for_a_later_operand():
    product = "v_mfma_f32_32x32x16_bf16 v[0:15], v[{}:{}], v[24:27], v[0:15]"
    reads = [f"ds_read_b128 v[{r}:{r + 3}], v80" for r in (32, 36, 40)]
    products = [product.format(r, r + 3) for r in [32] * 9 + [36, 40] + [32] * 7]

    def of(count):
        return waits_for_later_operands(parse([".LBB0_1:", *reads, f"s_waitcnt lgkmcnt({count})", *products, "s_cbranch_scc1 .LBB0_1", "s_endpgm"]))
    assert of(1) and not of(2)
    assert not of(0)  # (for all of them: ahead of a copy over their place)


def test_the_check_sees_a_copy_in_flight():
    def of(*text):
        code = parse(text + ("ds_write_b64 v9, v[2:3]", "s_endpgm"))
        return [before_it_lands(code, n, lambda i: i.op.startswith("ds_write")) for n in mask_copies(code)]
    copy, load = "global_load_lds_dword v1, s[4:5]", "global_load_dwordx4 v[4:7], v8, s[6:7]"
    assert of(copy)[0] and of(copy, load, load, "s_waitcnt vmcnt(3)")[0] and of(copy, "s_waitcnt lgkmcnt(0)")[0]
    assert not of(copy, "s_waitcnt vmcnt(0)")[0] and not of(copy, load, load, "s_waitcnt vmcnt(2) lgkmcnt(0)")[0]
    # on one path of two
    assert of(copy, "s_cbranch_scc1 .LBB0_1", load, "s_waitcnt vmcnt(1)", ".LBB0_1:")[0]
    assert of(copy, "s_cbranch_scc1 .LBB0_1", load, ".LBB0_1:", "s_waitcnt vmcnt(1)")[0]


def test_the_check_sees_a_missing_wait():
    """Planted mistakes, and what mends them."""
    def of(*text):
        return faults(parse(text + ("s_endpgm",)))
    assert of("s_mov_b32 m0, s3", "global_load_lds_dwordx4 v1, s[4:5] offset:0")
    assert not of("s_mov_b32 m0, s3", "s_nop 0", "global_load_lds_dwordx4 v1, s[4:5] offset:0")
    assert of("v_readlane_b32 s4, v1, s2", "s_nop 3", "global_load_lds_dwordx4 v1, s[4:5] offset:0")
    assert not of("v_readlane_b32 s4, v1, s2", "s_nop 4", "global_load_lds_dwordx4 v1, s[4:5] offset:0")
    assert not of("v_readlane_b32 s4, v1, s2", "s_add_u32 s4, s4, s6", "global_load_lds_dwordx4 v1, s[4:5] offset:0")
    product = "v_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], v[24:27], v[0:15]"
    other = "v_mfma_f32_32x32x16_bf16 v[32:47], v[50:53], v[54:57], v[32:47]"
    assert of("v_cvt_pk_bf16_f32 v27, v30, v31", other, product)
    assert not of("v_cvt_pk_bf16_f32 v27, v30, v31", "s_nop 1", product)
    assert of(product, other, "s_nop 2", "v_add_f32_e32 v60, v3, v61")
    assert not of(product, other, "s_nop 3", "v_add_f32_e32 v60, v3, v61")
    assert not of(product, product)
    assert of(product, other.replace("v[50:53]", "v[12:15]"))
    from_zero = product.replace("v[24:27], v[0:15]", "v[24:27], v[64:79]")
    assert of(from_zero, "s_nop 6", "v_mov_b32_e32 v70, 0") and not of(from_zero, "s_nop 7", "v_mov_b32_e32 v70, 0")
    # around a loop: the write at its end, the copy at its beginning
    assert of(".LBB0_1:", "global_load_lds_dwordx4 v1, s[4:5] offset:0", "v_readlane_b32 s4, v1, s2", "s_cbranch_scc1 .LBB0_1")
