"""Every read of an MFMA's result comes late enough, in the kernels' assembly.

The hardware does not interlock the result of a matrix instruction against
other vector instructions; the compiler places the wait states, but counts
them along one path only where paths meet again.  Each MFMA is followed along
all paths here: a vector, LDS or memory instruction that names its result (or
an MFMA that multiplies by it) needs 12 (bf16, 8 passes) or 18 (float32, 16
passes) states in between.  A later MFMA waits for the matrix pipe, so it
counts as the passes of the first."""
import os
import re
import subprocess

import pytest

from paper_2210_00038_amd import build

STATES = {"v_mfma_f32_32x32x16_bf16": (12, 8), "v_mfma_f32_32x32x2_f32": (18, 16)}


def _regs(tok):
    m = re.match(r"^([va])(?:(\d+)|\[(\d+):(\d+)\])$", tok)
    if not m:
        return set()
    lo, hi = (m[2], m[2]) if m[2] else (m[3], m[4])
    return {(m[1], i) for i in range(int(lo), int(hi) + 1)}


def _kernels(text):
    """name -> list of (label, None) or (opcode, operands)."""
    out, cur = {}, None
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if m := re.match(r"^(_Z\w+):", line):
            cur = out.setdefault(m[1], [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None and (m := re.match(r"^(\.LBB\w+):", line)):
            cur.append((m[1], None))
        elif cur is not None and line and not line.startswith("."):
            op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
            op, _, tail = op.partition("\t")
            cur.append((op, [t.split()[0] for t in (tail + " " + rest).split(",") if t.strip()]))
    return out


def _early_reads(ins):
    label = {x[0]: i for i, x in enumerate(ins) if x[1] is None}
    found, mfmas = [], 0
    for i, (op0, ops0) in enumerate(ins):
        if ops0 is None or "mfma" not in op0:
            continue
        mfmas += 1
        need, passes = STATES[op0]
        work, best = [(i + 1, 0, frozenset(_regs(ops0[0])))], {}
        while work:
            j, w, live = work.pop()
            while j < len(ins) and w < need and live:
                op, ops = ins[j]
                if ops is None:
                    if best.get((j, live), need) <= w:
                        break
                    best[(j, live)] = w
                    j += 1
                    continue
                if op == "s_endpgm":
                    break
                if "mfma" in op:
                    if live & (_regs(ops[1]) | _regs(ops[2])):
                        found.append((w, op0, ops0, op, ops))
                    live, w = live - _regs(ops[0]), max(w + 1, passes)
                else:
                    named = set().union(*map(_regs, ops)) if not op.startswith("s_") else set()
                    if named & live:
                        found.append((w, op0, ops0, op, ops))
                        live = live - named
                    w += int(ops[0], 0) + 1 if op == "s_nop" else 1
                if op == "s_branch":
                    j = label[ops[0]]
                    continue
                if op.startswith("s_cbranch"):
                    work.append((label[ops[0]], w, live))
                j += 1
    return mfmas, found


def test_checker_finds_the_short_path():
    body = ("_Zk:\n v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]\n"
            " s_cbranch_scc1 .LBB0_1\n s_nop 15\n.LBB0_1:\n{}\tv_mov_b32_e32 v30, v3\n s_endpgm\n")
    for nops, bad in (("", 1), (" s_nop 9\n", 1), (" s_nop 10\n", 0)):
        mfmas, found = _early_reads(_kernels(body.format(nops))["_Zk"])
        assert (mfmas, len(found)) == (1, bad)


@pytest.mark.parametrize("source", ["ghost_norm.hip", "agemm.hip"])
def test_results_of_mfmas_are_read_late_enough(source, tmp_path):
    asm = str(tmp_path / "k.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.hipcc(), *flags, "-x", "hip", "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", asm], check=True, capture_output=True)
    with open(asm) as f:
        kernels = _kernels(f.read())
    total = 0
    for name, ins in kernels.items():
        mfmas, found = _early_reads(ins)
        total += mfmas
        assert not found, (name, found[:3])
    assert total > 100, total
