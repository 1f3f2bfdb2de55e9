"""The generated code of kernels whose accumulators are pinned in AGPRs (pg_bwd_wide.hpp), and the choice of the kernel.

Their matrix products are inline asm, which the compiler schedules around without knowing what they need, so the
code is checked instead: the compiler itself uses no AGPR, no scratch memory and no M0 in these kernels (it would
overwrite accumulators, add loads to the counted copies in flight, or lose a copy's destination), and on every path
the wait states stand between an operand's write and its product, a product and the use of its result, and a copy's
descriptor and the copy. CPU only (cross-compiles the device code).
"""
import re
import subprocess

import pytest

from paper_2506_05433_amd import build as pg_build
from tests.test_gpu_wide import CASES, DQ_CASES

KERNELS = ("dkdv_wide_kernel", "dq_wide_kernel")


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "pg.asm")
    cmd = [a for a in pg_build.command(out, extra=("-S", "--cuda-device-only", "-w")) if a not in ("-shared", "-fPIC")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    with open(out) as f:
        return f.read()


def _kernels(text):
    found = []
    for m in re.finditer(r"^(_ZN2pg\w*?(\w+_kernel)I\w+):", text, re.M):
        if any(m.group(1).find(k) >= 0 for k in KERNELS):
            found.append((m.group(1), text[m.end():text.index(".Lfunc_end", m.end())].split("\n")))
    return found


def _regs(op, kind="v"):
    m = re.match(kind + r"\[(\d+):(\d+)\]|" + kind + r"(\d+)$", op)
    if not m:
        return range(0)
    return range(int(m.group(1)), int(m.group(2)) + 1) if m.group(1) else range(int(m.group(3)), int(m.group(3)) + 1)


# wait states between a vector write and a product that reads it, a product (8 passes) and any other use of its result,
# and a vector write of a scalar register and a buffer instruction that reads it: what the compiler keeps for the
# same instructions where it knows them (a builtin product is followed by s_nop 11 before its result is read)
OPERAND, RESULT, SCALAR = 2, 12, 5


def _blocks(lines):
    """Basic blocks of (op, args, in inline asm, text), each with the indices of the blocks that follow it."""
    blocks, names, in_asm = [[]], {}, False
    for line in lines:
        s = line.strip()
        if "ASMSTART" in s or "ASMEND" in s:
            in_asm = "ASMSTART" in s
            continue
        label = re.match(r"(\.LBB\w+):", s)
        if label:
            blocks.append([])
            names[label.group(1)] = len(blocks) - 1
            continue
        if not s or s[0] in ".;":
            continue
        op, _, rest = s.split(";")[0].strip().partition(" ")
        blocks[-1].append((op, [a.strip() for a in rest.split(",")], in_asm, s))
        if op.startswith(("s_branch", "s_cbranch", "s_endpgm")):
            blocks.append([])
    follow = []
    for i, block in enumerate(blocks):
        last = block[-1] if block else ("", [], False, "")
        out = [names[last[1][0]]] if last[0].startswith(("s_branch", "s_cbranch")) else []
        if not last[0].startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            out.append(i + 1)
        follow.append(out)
    return blocks, follow


def _pass(block, state, found):
    """Runs the block from a state of (registers written by vector instructions, results of products, scalar
    registers written by vector instructions), each register with the wait states since; appends what comes too
    soon to `found` and returns the state after the block."""
    writes, results, scalars = (dict(x) for x in state)
    for op, args, in_asm, text in block:
        mfma = op.startswith("v_mfma")
        use = [set(_regs(a.split(" ")[0])) for a in args]
        if mfma and in_asm:
            for r in use[1] | use[2] | (use[3] - use[0]):
                if writes.get(r, OPERAND) < OPERAND:
                    found.append((text, f"v{r} written {writes[r]} wait states before"))
                if results.get(r, RESULT) < RESULT:
                    found.append((text, f"v{r} is a product's result of {results[r]} wait states before"))
        elif not op.startswith("s_") and not mfma:
            for r in set().union(*use):
                if results.get(r, RESULT) < RESULT:
                    found.append((text, f"v{r} is a product's result of {results[r]} wait states before"))
        if in_asm and op.startswith("buffer_"):
            for r in set().union(*(set(_regs(a.split(" ")[0], "s")) for a in args)):
                if scalars.get(r, SCALAR) < SCALAR:
                    found.append((text, f"s{r} written {scalars[r]} wait states before"))
        # one wait state per instruction; a product after another one waits for its 8 passes
        slots = int(args[0]) + 1 if op == "s_nop" else 1
        for x, limit, n in ((writes, OPERAND, slots), (results, RESULT, 8 if mfma else slots), (scalars, SCALAR, slots)):
            for r in list(x):
                x[r] += n
                if x[r] >= limit:
                    del x[r]
        for r in use[0] if op.startswith("v_") else ():
            results.pop(r, None)
            writes.pop(r, None)
            if mfma:
                results[r] = 0
            elif not op.startswith(("v_cmp", "v_readfirstlane", "v_readlane")):
                writes[r] = 0
        if op.startswith("v_") and not mfma:
            for r in _regs(args[0], "s"):
                scalars[r] = 0
            if len(args) > 1:  # carry-outs
                for r in _regs(args[1], "s") if "_co_" in op else ():
                    scalars[r] = 0
    return writes, results, scalars


def hazards(lines):
    """(the compiler's own AGPR, scratch or M0 instructions, instructions that come too soon after another one), over
    every path through the code."""
    blocks, follow = _blocks(lines)
    own = [text for block in blocks for op, args, in_asm, text in block if not in_asm and (
        op.startswith(("scratch_", "v_accvgpr")) or any(re.match(r"a\[?\d|m0$", a) for a in args))]
    entry = [({}, {}, {}) for _ in blocks]
    todo, close = {0}, []
    seen = set()
    while todo:
        i = todo.pop()
        seen.add(i)
        after = _pass(blocks[i], entry[i], [])
        for j in follow[i]:
            grew = j not in seen
            for mine, new in zip(entry[j], after):
                for r, n in new.items():
                    if n < mine.get(r, 99):
                        mine[r] = n
                        grew = True
            if grew:
                todo.add(j)
    for i in sorted(seen):
        _pass(blocks[i], entry[i], close)
    return own, close


def test_pinned_accumulator_kernels(listing):
    kernels = _kernels(listing)
    assert len(kernels) >= 3, [k for k, _ in kernels]  # dK/dV for both head dims, dQ for 128
    for name, lines in kernels:
        own, close = hazards(lines)
        assert sum("v_mfma" in x for x in lines) >= 32, name
        assert not own, (name, own[:5])
        assert not close, (name, close[:5])


def test_hazard_check_sees_planted_mistakes():
    def asm(*lines):
        return ["\t;;#ASMSTART", *("\t" + x for x in lines), "\t;;#ASMEND"]

    cvt = "\tv_cvt_pk_bf16_f32 v4, v1, v2"
    acc = "v_mfma_f32_32x32x16_bf16 a[0:15], v[8:11], v[4:7], a[0:15]"
    res = "v_mfma_f32_32x32x16_bf16 v[16:31], v[8:11], a[0:3], 0"
    add = "\tv_add_f32_e32 v1, v16, v2"
    assert hazards([cvt, *asm("s_nop 1", acc)]) == ([], [])
    assert hazards([cvt, *asm("s_nop 0", acc)])[1] and hazards([cvt, *asm(acc)])[1]
    assert hazards([*asm(res), "\ts_nop 11", add]) == ([], [])
    assert hazards([*asm(res), "\ts_nop 10", add])[1]
    # two products later the result is there, one later it is not
    other = acc.replace("a[0:15]", "a[16:31]")
    assert hazards([*asm(res, other, other), add]) == ([], []) and hazards([*asm(res, other), add])[1]
    # on paths: over a label, around a loop, past a branch that skips the wait
    assert hazards([cvt, ".LBB0_1:", *asm(acc)])[1]
    assert hazards([".LBB0_1:", *asm(acc), "\ts_nop 4", cvt, "\ts_cbranch_scc1 .LBB0_1", "\ts_endpgm"])[1]
    assert hazards([".LBB0_1:", *asm("s_nop 0", acc), "\ts_nop 4", cvt, "\ts_cbranch_scc1 .LBB0_1"]) == ([], [])
    skip = [*asm(res), "\ts_cbranch_scc0 .LBB0_2", "\ts_nop 15", ".LBB0_2:", add]
    assert hazards(skip)[1] and hazards([x for x in skip if "cbranch" not in x]) == ([], [])
    # an LDS copy's descriptor from a vector instruction, and the compiler's own AGPR, scratch and M0
    copy = asm("s_mov_b32 m0, s3", "s_nop 0", "buffer_load_dwordx4 v3, s[4:7], 0 offen lds")
    assert hazards(["\tv_readfirstlane_b32 s5, v1", *copy])[1]
    assert hazards(["\tv_readfirstlane_b32 s5, v1", "\ts_nop 2", *copy]) == ([], [])
    for x in ("v_accvgpr_read_b32 v1, a0", "scratch_load_dword v1, off, off", "s_mov_b32 m0, s1"):
        assert hazards(["\t" + x])[0]


def test_cases_choose_the_wide_kernels(tmp_path_factory):
    """Read from the library's own rules (pg_layout.hpp), compiled for the host."""
    from tests.test_plan_host import DTYPES, build_planner, layouts
    exe = build_planner(tmp_path_factory)

    def tiles(dtype, case):
        (p, _, s), hq, hkv, d, _ = case
        (lay,) = layouts(exe, [(DTYPES[dtype], len(p), len(s), sum(p), sum(s), hq, hkv, d)])
        assert lay["split"] == (hq == 1)  # member-aligned tiles in the one-head case only
        return lay["bm"], lay["bkv"]

    assert all(tiles("bf16", c) == (128, 256) for c in CASES)
    assert all(tiles("bf16", c) == (256, 256) for c in DQ_CASES)
    assert all(tiles("fp32", c) == (128, 128) for c in CASES + DQ_CASES)
