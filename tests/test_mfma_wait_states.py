"""Wait states before the matrix products written as inline assembly (CPU).

An MFMA that reads a vector register written by a VALU instruction needs two wait states
between them.  The compiler inserts them before its own MFMA instructions but does not look
into inline assembly, so the product loops have to bring them along.  The test compiles the
sources that hold such products to gfx950 assembly and walks back from every one of them:
each instruction is one wait state, s_nop N is N + 1.
"""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "paper_2609_37924_amd", "csrc"))
import build  # noqa: E402

WAIT_STATES = 2
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def registers(operands):
    """The registers an operand list names, as (file, number)."""
    out = set()
    for file, one, lo, hi in REG.findall(operands):
        out |= {(file, n) for n in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return out


def violations(asm):
    """(function, product, writer, wait states) of every inline MFMA too close behind a VALU write."""
    found, products, fn, history, inline = [], 0, "", [], False
    for line in asm.splitlines():
        text = line.split("//")[0].strip()
        if "#ASMSTART" in text or "#ASMEND" in text:
            inline = "#ASMSTART" in text
            continue
        text = text.split(";")[0].strip()
        if not text or text.startswith("."):
            continue
        if text.endswith(":"):
            if text.startswith("_Z"):
                fn, history = text[:-1], []
            continue
        op, _, operands = text.partition(" ")
        op = op.split("\t")[0]
        operands = text[len(op):]
        if op.startswith("v_mfma") and inline:
            products += 1
            reads = registers(operands.split(",", 1)[1])
            waited = 0
            for p_op, p_operands in reversed(history):
                if waited >= WAIT_STATES:
                    break
                if p_op.startswith("v_") and not p_op.startswith("v_mfma"):
                    if registers(p_operands.split(",", 1)[0]) & reads:
                        found.append((fn, text, p_op + p_operands, waited))
                waited += int(p_operands.strip(), 0) + 1 if p_op == "s_nop" else 1
        history = (history + [(op, operands)])[-8:]
    return found, products


def test_checker():
    """The walk itself, on a few lines."""
    mfma = ";;#ASMSTART\nv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], 0\n;;#ASMEND\n"
    far = "v_mov_b32_e32 v7, 0\ns_nop 1\n"
    assert violations("_Zf:\n" + far + mfma) == ([], 1)
    assert violations("_Zf:\nv_mov_b32_e32 v12, 0\n" + mfma) == ([], 1)
    assert len(violations("_Zf:\nv_mov_b32_e32 v11, 0\ns_mov_b32 s0, 0\n" + mfma)[0]) == 1
    assert len(violations("_Zf:\nv_mov_b64_e32 v[6:7], 0\ns_nop 0\n" + mfma)[0]) == 1


@pytest.mark.parametrize("source", ["gemm.hip", "head_sample.hip"])
def test_inline_products_wait_for_their_operands(source, tmp_path):
    out = str(tmp_path / "out.s")
    cmd = [build.hipcc(), "--cuda-device-only", "-S", os.path.join(build.HERE, source), "-o", out]
    r = subprocess.run(cmd + build.flags() + build.EXTRA.get(source, []), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        found, products = violations(f.read())
    assert products > 0
    assert not found, "\n".join("%s: %s after %s, %d wait states" % (f, m, w, n) for f, m, w, n in found)
