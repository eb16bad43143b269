"""The resident-workgroup MFMA GEMM issues its MFMAs as bare inline asm and
loads its weight fragments with inline-asm loads the compiler cannot see in
flight.  Checked on the compiled kernels: nothing but an MFMA touches a
register between such a load and its use (or a full vmcnt(0) wait), and no
vector instruction writes an operand of an MFMA in the two wait states before
it (the compiler puts no wait there: it does not know that it is an MFMA)."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2607_20507_amd import build as B
from tests.test_isa_register_loads import check_register_loads

PATTERN = "gemm_mfma4"


def _operands(tok):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", tok)
    if m:
        return {(m.group(1), r) for r in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"([va])(\d+)$", tok)
    return {(m.group(1), int(m.group(2)))} if m else set()


def mark_tracked_loads(lines):
    """Loads outside inline asm are the compiler's own: it waits for them."""
    out, asm = [], False
    for l in lines:
        if "#ASMSTART" in l:
            asm = True
        elif "#ASMEND" in l:
            asm = False
        out.append(l if asm else l.replace("global_load_dwordx4", "tracked_load_dwordx4"))
    return out


def unwaited_writes(lines, pattern):
    """{kernel: (bare MFMAs, MFMAs with an operand written less than two wait states before)}."""
    out, name = {}, None
    for i, l in enumerate(lines):
        m = re.match(r"^(_Z\S*" + pattern + r"\S*):", l)
        if m:
            name = m.group(1)
            out[name] = (0, [])
        elif l.startswith(".Lfunc_end"):
            name = None
        if name is None or not l.strip().startswith("v_mfma") or "#ASMSTART" not in lines[i - 1]:
            continue
        n, bad = out[name]
        read = set().union(*[_operands(t.strip()) for t in l.split(None, 1)[1].split(",")])
        states, j = 0, i - 1
        while states < 2 and j > 0 and not re.match(r"^_Z", lines[j]):
            p = lines[j].strip().split(None, 1)
            j -= 1
            if not p or p[0].startswith((";", ".")) or p[0].endswith(":"):
                continue
            if p[0] == "s_nop":
                states += int(p[1]) + 1
                continue
            if p[0].startswith("v_") and not p[0].startswith("v_mfma") and len(p) == 2:
                if _operands(p[1].split(",")[0].strip()) & read:
                    bad.append(lines[j + 1].strip() + " -> " + l.strip())
            states += 1
        out[name] = (n + 1, bad)
    return out


def test_checker_flags_a_write():
    k = ["_Zgemm_mfma4_x:", ";;#ASMSTART", "v_mfma_f32_16x16x32_bf16 a[0:3], v[2:5], v[6:9], a[0:3]", ";;#ASMEND"]
    bad = k[:1] + ["v_mov_b32_e32 v3, v0", "s_add_i32 s0, s0, 1"] + k[1:]
    good = k[:1] + ["v_mov_b32_e32 v3, v0", "s_nop 1"] + k[1:]
    assert unwaited_writes(good, PATTERN)["_Zgemm_mfma4_x"] == (1, [])
    assert len(unwaited_writes(bad, PATTERN)["_Zgemm_mfma4_x"][1]) == 1


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_mfma4_loads_and_operands(tmp_path):
    out = tmp_path / "gemm.s"
    cmd = [B.hipcc()] + B.flags() + ["--cuda-device-only", "-S", os.path.join(B.CSRC, "gemm.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = out.read_text().split("\n")
    loads = check_register_loads(mark_tracked_loads(lines), PATTERN)
    writes = unwaited_writes(lines, PATTERN)
    assert len(loads) >= 17 and loads.keys() == writes.keys()
    for name, (n, bad) in loads.items():
        assert n > 0 and not bad, (name, bad[:5])
    for name, (n, bad) in writes.items():
        assert n >= 8 * 8 and not bad, (name, n, bad[:5])
