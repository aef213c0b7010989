"""Wait states around the matrix instructions that are written in assembly (gemm_mfma_ring_kernel).

The compiler inserts the wait states that an MFMA needs for its builtins only.  For v_mfma_f32_16x16x32_bf16 as an asm
statement they have to follow from the source, so the compiled code is checked here, along every path through it:
  - an operand written by another vector instruction: 2 wait states before the MFMA reads it (CDNA3/4 ISA, "manually
    inserted wait states");
  - a result read or written by another instruction: at most 12 wait states after the MFMA (8 passes).
An instruction counts one wait state, s_nop n counts n + 1.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2405_13053_amd import build

MFMA = "v_mfma_f32_16x16x32_bf16"
BEFORE, AFTER = 2, 12


def _regs(token):
    m = re.match(r"([av])\[(\d+):(\d+)\]$", token)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([av])(\d+)$", token)
    return {(m[1], int(m[2]))} if m else set()


def _parse(text):
    """[(function, operation, operand tokens)], and the index that each label stands for."""
    code, labels, fn = [], {}, ""
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if line.endswith(":") and not line.startswith((".Lfunc", ".Ltmp")):
            labels[line[:-1]] = len(code)
            if not line.startswith("."):
                fn = line[:-1]
        elif line and not line.startswith("."):
            op, _, rest = line.replace("\t", " ").partition(" ")
            code.append((fn, op, [t.split()[0] for t in rest.split(",") if t.split()]))
    return code, labels


def _violations(text):
    code, labels = _parse(text)
    follow, lead = [[] for _ in code], [[] for _ in code]
    for i, (_, op, args) in enumerate(code):
        nxt = []
        if op not in ("s_endpgm", "s_branch") and i + 1 < len(code):
            nxt.append(i + 1)
        if op == "s_branch" or op.startswith("s_cbranch"):
            nxt.append(labels[args[0]])
        follow[i] = nxt
        for j in nxt:
            lead[j].append(i)
    regs = [[_regs(t) for t in args] for _, _, args in code]
    used = [set().union(*r) if r else set() for r in regs]
    states = [int(args[0]) + 1 if op == "s_nop" else 1 for _, op, args in code]
    bad = []
    for i, (fn, op, args) in enumerate(code):
        if op != MFMA:
            continue
        todo, seen = [(j, 0) for j in lead[i]], set()
        while todo:   # back: who wrote an operand
            j, ws = todo.pop()
            if ws >= BEFORE or (j, ws) in seen:
                continue
            seen.add((j, ws))
            o = code[j][1]
            if o.startswith("v_") and not o.startswith("v_mfma") and regs[j] and regs[j][0] & used[i]:
                bad.append((fn, "operand", o, code[j][2], args))
            todo += [(p, ws + states[j]) for p in lead[j]]
        todo, seen = [(j, 0) for j in follow[i]], set()
        while todo:   # forward: who touches the result; other MFMAs wait by themselves
            j, ws = todo.pop()
            if ws >= AFTER or (j, ws) in seen:
                continue
            seen.add((j, ws))
            o = code[j][1]
            if not o.startswith("v_mfma") and used[j] & regs[i][0]:
                bad.append((fn, "result", o, code[j][2], args))
                continue
            todo += [(p, ws + states[j]) for p in follow[j]]
    return bad


def test_the_check_sees_both_kinds_and_every_path():
    m = MFMA + " a[0:3], v[2:5], v[26:29], a[0:3]\n"
    clean = "k:\n v_accvgpr_write_b32 a3, 0\n s_nop 1\n" + m + "s_nop 10\n s_nop 0\n v_accvgpr_read_b32 v0, a3\n s_endpgm\n"
    assert not _violations(clean)
    assert [b[1] for b in _violations(clean.replace("s_nop 1\n", "s_nop 0\n"))] == ["operand"]
    assert [b[1] for b in _violations(clean.replace("a3, 0", "v27, 0").replace("s_nop 1\n", ""))] == ["operand"]
    assert [b[1] for b in _violations(clean.replace(" s_nop 0\n", ""))] == ["result"]
    loop = "k:\n.LBB0_1:\n" + m + "v_mov_b32_e32 v2, v9\n s_cbranch_scc1 .LBB0_1\n s_endpgm\n"   # over the back edge
    assert [b[1] for b in _violations(loop)] == ["operand"]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_every_ring_kernel_keeps_the_wait_states(tmp_path):
    asm = tmp_path / "gemm.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    src = os.path.join(build.HERE, "csrc", "gemm.hip")
    subprocess.run(["hipcc", *flags, "--cuda-device-only", "-S", "-o", str(asm), src], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = asm.read_text()
    kernels = set(re.findall(r"^(_Z\S*gemm_mfma_ring_kernel\S*):", text, re.M))
    assert len(kernels) >= 10
    seen = {fn for fn, op, _ in _parse(text)[0] if op == MFMA}
    assert kernels <= seen
    assert not _violations(text)
