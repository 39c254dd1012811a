"""The dK/dV kernel's inline-assembly MFMAs, which the compiler does not see as
such: in the code that is built, two wait states or more lie between a vector
instruction that writes an operand and the MFMA that reads it (the compiler is
free to put a copy there), an operand that another MFMA writes is older than its
result latency, and nothing but MFMAs touches the accumulators in between. Read
from the compiler's own listing of bsattn_bwd.hip, on the CPU."""
import os
import re
import subprocess

import pytest

from paper_2609_23169_amd import _build

VALU_STATES = 2     # vector write of an operand -> MFMA
MFMA_STATES = 20    # MFMA write of an operand -> MFMA (more than its 16 or fewer passes)


def _regs(op):
    """Registers of one operand: {("v", 3), ...}; other operands: empty."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", op)
    if not m:
        return set()
    lo, hi = (m.group(2), m.group(2)) if m.group(2) else (m.group(3), m.group(4))
    return {(m.group(1), r) for r in range(int(lo), int(hi) + 1)}


def _violations(lines):
    """(count of inline-assembly MFMAs, list of problems) of one function."""
    asm, found, bad, early = False, 0, [], []
    recent = []   # (states since, kind, written, text)
    for line in lines:
        if "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
            continue
        text = line.split(";")[0].strip()
        if not text or text.endswith(":") or text.startswith("."):
            continue
        name, _, rest = text.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if asm and name.startswith("v_mfma"):
            found += 1
            srcs = _regs(ops[1]) | _regs(ops[2])
            for states, kind, written, other in recent:
                limit = {"valu": VALU_STATES, "mfma": MFMA_STATES}[kind]
                if states < limit and written & srcs:
                    bad.append(f"{other} / {text}: {states} wait states")
            bad += early
            early = []
        elif not name.startswith("v_mfma") and any(r[0] == "a" for o in ops for r in _regs(o)):
            # reads of the finished accumulators come after all of the MFMAs
            (early if name == "v_accvgpr_read_b32" else bad).append(f"accumulator touched: {text}")
        states = int(rest) + 1 if name == "s_nop" else 1
        recent = [(s + states, k, w, t) for s, k, w, t in recent if s + states < MFMA_STATES]
        if name.startswith("v_mfma"):
            recent.append((0, "mfma", _regs(ops[0]), text))
        elif name.startswith("v_"):
            w = _regs(ops[0]) | (_regs(ops[1]) if "swap" in name else set())
            recent.append((0, "valu", w, text))
    return found, bad


def test_checker_finds_a_planted_hazard():
    plain = ["v_add_f32_e32 v4, v1, v2", ";;#ASMSTART",
             "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", ";;#ASMEND"]
    assert _violations(plain)[0] == 1 and len(_violations(plain)[1]) == 1
    assert _violations([plain[0], "s_nop 1"] + plain[1:])[1] == []
    assert len(_violations([plain[0], "s_nop 0"] + plain[1:])[1]) == 1
    after = ["v_mfma_f32_16x16x32_bf16 v[8:11], v[0:3], v[0:3], 0", "s_nop 1"] + plain[1:]
    assert len(_violations(after)[1]) == 1
    assert _violations(["v_mul_f32_e32 v1, a3, v2"])[1] != []
    read = ["v_accvgpr_read_b32 v1, a3"]
    assert _violations(plain[1:] + read)[1] == [] and _violations(read + plain[1:])[1] != []


def test_built_code_keeps_the_wait_states(tmp_path):
    if not os.path.exists(_build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "bwd.s")
    cmd = [_build.HIPCC, *_build.FLAGS, "-x", "hip", "--cuda-device-only", "-S",
           os.path.join(_build.CSRC, "bsattn_bwd.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(out) as f:
        text = f.read()
    bodies = re.findall(r"^(\w*bwd_dkdv64_kernel\w*):[^\n]*\n(.*?)\n\.Lfunc_end", text, re.S | re.M)
    assert len(bodies) == 2
    for name, body in bodies:
        found, bad = _violations(body.splitlines())
        assert found >= 4 * 64 + 64, (name, found)   # four unrolled tiles and the zeros
        assert not bad, (name, bad[:5])
