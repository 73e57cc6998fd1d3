"""Wait states between a vector instruction that writes a scalar register and
one that reads it (CPU only: hipcc -S).

On gfx950 a vector instruction may read a scalar register (a comparison's mask
as a select's condition or a carry-in, a value from a read-lane) only two wait
states after the vector instruction that wrote it; sooner it may see the old
value.  The compiler keeps them between its own instructions, but does not look
into inline assembly.  Every instruction is one wait state, s_nop k is k + 1.
"""
import pathlib
import re
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_1705_02045_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
WAIT = 2

SGPR = re.compile(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]|\b(vcc)(?:_lo|_hi)?\b")
# vector instructions whose first, or second, operand is a scalar destination
FIRST = re.compile(r"v_(cmp_|readlane|readfirstlane)")
SECOND = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_u32|v_div_scale|v_mad_[ui]64_[ui]32")


def registers(text):
    out = set()
    for one, lo, hi, vcc in SGPR.findall(text):
        if vcc:
            out.add("vcc")
        elif one:
            out.add(int(one))
        else:
            out.update(range(int(lo), int(hi) + 1))
    return out


def early_reads(lines):
    """(line number, text) of every read less than WAIT wait states behind its write."""
    bad, age = [], {}  # age: wait states since a vector instruction wrote the register
    for i, line in enumerate(lines):
        text = line.split(";")[0].strip()
        m = re.match(r"([a-z]\w+)\s*(.*)", text)
        if not m or text.endswith(":") or text.startswith("."):
            continue
        op, rest = m.groups()
        written = set()
        if op.startswith("v_"):
            ops = [o.strip() for o in rest.split(",")]
            k = 0 if FIRST.match(op) else 1 if SECOND.match(op) else None
            if k is not None and k < len(ops):
                written = registers(ops[k])
            reads = set()
            for j, o in enumerate(ops):
                if j != k:
                    reads |= registers(o)
            if any(age.get(r, WAIT) < WAIT for r in reads):
                bad.append((i + 1, text))
        elif op.startswith("s_"):
            for r in registers(rest.split(",")[0]):  # a scalar instruction's own result is not meant
                age.pop(r, None)
        step = int(rest, 0) + 1 if op == "s_nop" else 1
        age = {r: a + step for r, a in age.items() if a + step < WAIT}
        for r in written:
            age[r] = 0
    return bad


def test_scanner():
    late = ["v_cmp_lt_f32_e64 s[4:5], v0, v1", "v_mov_b32_e32 v2, v3"]
    read = "v_addc_co_u32_e64 v4, s[6:7], v4, v4, s[4:5]"
    assert early_reads(late + [read]) == [(3, read)]
    assert early_reads(late + ["s_nop 0", read]) == []
    assert early_reads(["v_cmp_eq_u32_e32 vcc, v0, v1", "s_nop 1", "v_cndmask_b32_e32 v0, v1, v2, vcc"]) == []
    assert early_reads(["v_cmp_eq_u32_e32 vcc, v0, v1", "v_cndmask_b32_e32 v0, v1, v2, vcc"]) != []
    assert early_reads(["v_cmp_eq_u32_e64 s[4:5], v0, v1", "s_mov_b64 s[4:5], -1", read]) == []


@pytest.mark.parametrize("name", ["change", "distinct", "float", "int", "scan", "sort"])
def test_masks_are_read_two_wait_states_after_their_comparison(name):
    if not pathlib.Path(HIPCC).exists():
        pytest.skip("hipcc not available")
    cmd = [HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "-I", str(ROOT / "include"), "-I", str(CSRC), "--offload-device-only",
           "-S", "-o", "-", str(CSRC / f"ecc_{name}.hip")]
    lines = subprocess.run(cmd, check=True, capture_output=True, text=True).stdout.splitlines()
    assert sum(line.strip().startswith("v_") for line in lines) > 100
    bad = early_reads(lines)
    assert not bad, (len(bad), bad[:5])
