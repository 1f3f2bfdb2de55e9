"""The generated code of kernels whose accumulators are pinned in AGPRs (pg_bwd_wide.hpp), and the choice of the kernel.

Their matrix products are inline asm, which the compiler schedules around without knowing what they need, so the
code is checked instead: the compiler itself uses no AGPR and no scratch memory in these kernels (it would
overwrite accumulators, or add loads to the counted copies in flight), and no vector instruction writes an operand
of such a product in the two issue slots before it. CPU only (cross-compiles the device code).
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


def _regs(op):
    m = re.match(r"v\[(\d+):(\d+)\]|v(\d+)$", op)
    if not m:
        return range(0)
    return range(int(m.group(1)), int(m.group(2)) + 1) if m.group(1) else range(int(m.group(3)), int(m.group(3)) + 1)


def hazards(lines):
    """(the compiler's own AGPR or scratch instructions, pinned products whose operand was written or whose result is
    touched too soon). A product's VGPR operand may not be written by a vector instruction in the two issue slots
    before it, and its VGPR result not be read or written by another kind of instruction for 11 slots (an 8-pass
    product; one that follows it takes 8 slots)."""
    own, close, in_asm, recent, results = [], [], False, [], []
    for line in lines:
        s = line.strip()
        if "ASMSTART" in s or "ASMEND" in s:
            in_asm = "ASMSTART" in s
            continue
        if re.match(r"\.LBB\w+:", s):
            recent = []
            continue
        if not s or s[0] in ".;":
            continue
        op, _, rest = s.partition(" ")
        args = [a.strip() for a in rest.split(";")[0].split(",")]
        if not in_asm and (op.startswith(("scratch_", "v_accvgpr")) or any(re.match(r"a\[?\d", a) for a in args)):
            own.append(s)
        mfma = op.startswith("v_mfma")
        if in_asm and mfma:
            need = set(_regs(args[1])) | set(_regs(args[2]))
            if any(need & w for w in recent[-2:]):
                close.append(s)
        if not (in_asm and mfma) and not op.startswith("s_"):
            touched = set().union(*(_regs(a.split(" ")[0]) for a in args))
            close += ["%s; %s" % (r[2], s) for r in results if r[0] < 11 and r[1] & touched]
        slots = int(args[0]) + 1 if op == "s_nop" else 8 if mfma else 1
        for r in results:
            r[0] += slots
        results = [r for r in results if r[0] < 11]
        if in_asm and mfma and set(_regs(args[0])):
            results = [r for r in results if r[1] != set(_regs(args[0]))] + [[0, set(_regs(args[0])), s]]
        if op == "s_nop":
            recent += [set()] * (int(args[0]) + 1)
        else:
            valu = op.startswith("v_") and not mfma and not op.startswith(("v_cmp", "v_readfirstlane", "v_readlane"))
            recent.append(set(_regs(args[0])) if valu else set())
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
    ok = ["\tv_cvt_pk_bf16_f32 v4, v1, v2", "\t;;#ASMSTART", "\ts_nop 1",
          "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[8:11], v[4:7], a[0:15]", "\t;;#ASMEND"]
    assert hazards(ok) == ([], [])
    assert hazards([x for x in ok if "s_nop" not in x])[1]
    assert hazards(ok + ["\tv_accvgpr_read_b32 v1, a0"])[0]
    late = ["\t;;#ASMSTART", "\tv_mfma_f32_32x32x16_bf16 v[16:31], v[8:11], a[0:3], 0", "\t;;#ASMEND"]
    assert hazards(late + ["\ts_nop 11", "\tv_add_f32_e32 v1, v16, v2"]) == ([], [])
    assert hazards(late + ["\ts_nop 7", "\tv_add_f32_e32 v1, v16, v2"])[1]
    assert hazards(ok + ["\tscratch_load_dword v1, off, off"])[0]


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
