"""What the compiler makes of the kernels (gfx950 assembly of the library's own
sources, no GPU): a vector instruction that reads a scalar register comes at
least two wait states after the vector instruction that wrote it.  The compiler
keeps that rule for what it can see; text in an asm statement it cannot."""
import os
import re
import subprocess

import pytest

from paper_2311_12281_amd import build as B

WAIT = 2  # states between a vector instruction's scalar result and a vector reader


def _scalars(operands):
    """Scalar registers named in a piece of an instruction."""
    out = set()
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", operands):
        out |= {f"s{k}" for k in range(int(a), int(b) + 1)}
    out |= set(re.findall(r"\bs\d+\b", operands))
    if re.search(r"\bvcc\b", operands):
        out |= {"vcc_lo", "vcc_hi"}
    out |= set(re.findall(r"\bvcc_(?:lo|hi)\b", operands))
    return out


def _violations(lines):
    """(writer, reader) pairs closer than WAIT in straight-line order."""
    bad, recent = [], []  # recent: (states since, text, scalars written by a vector instruction)
    for line in lines:
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        ops = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
        vector = op.startswith("v_") and not op.startswith("v_mfma")
        results = 2 if "_co_" in op else 1  # a carry comes second
        written = _scalars(",".join(ops[:results])) if vector else set()
        if vector:
            read = _scalars(",".join(ops[results:]))
            bad += [(w, text) for d, w, s in recent if d < WAIT and s & read]
        states = int(rest.strip(), 0) + 1 if op == "s_nop" else 1
        recent = [(d + states, w, s) for d, w, s in recent if d + states < WAIT]
        if written:
            recent.append((0, text, written))
    return bad


def test_the_rule_is_recognised():
    near = ["v_cmp_ne_u32_e64 s[8:9], 0, v1", "v_writelane_b32 v34, s8, 0"]
    assert _violations(near)
    assert _violations([near[0], "s_nop 0", near[1]])
    assert not _violations([near[0], "s_nop 1", near[1]])
    assert not _violations([near[0], "v_mov_b32_e32 v2, v3", "s_mov_b32 s2, s3", near[1]])
    assert not _violations([near[0], "v_writelane_b32 v34, s10, 0"])


@pytest.mark.parametrize("src", B.SOURCES)
def test_scalar_results_are_waited_for(src, tmp_path):
    out = str(tmp_path / "k.s")
    cmd = [B.hipcc(), *B.common_flags(), "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        bad = _violations(f)
    assert not bad, f"{len(bad)} in {src}: " + "; ".join(f"{w} -> {t}" for w, t in bad[:4])
