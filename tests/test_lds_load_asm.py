"""The assembly of the kernels that load straight to LDS (lds_load.h).  Their loads
are inline asm that sets m0, which the compiler keeps reserved and cannot be told
about, and whose operands its hazard recogniser does not see.  So that has to hold
in what it emits: nothing else in these kernels uses m0, and no scalar operand of a
load is written by a vector instruction fewer than five wait states before."""
import os
import re
import subprocess

import pytest

from paper_2607_17299_amd import build

SOURCES = [f for f in build.SOURCES if '#include "lds_load.h"' in open(os.path.join(build.CSRC, f)).read()]
pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")


def _scan(lines):
    """(loads, uses of m0 outside inline asm, operands written too late)."""
    loads, stray, late, asm = 0, [], [], False
    writes = []                                   # (scalar registers a vector instruction wrote, wait states since)
    for line in lines:
        if "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
            continue
        t = line.split(";")[0].strip()
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        op, _, args = t.partition(" ")
        if re.search(r"\bm0\b", args) and not asm:
            stray.append(t)
        if asm and "_load_" in op:
            loads += 1
            regs = {r for a, b in re.findall(r"s\[(\d+):(\d+)\]", args) for r in range(int(a), int(b) + 1)}
            late += [(t, w) for w, since in writes if w & regs and since < 5]
        states = int(args, 0) + 1 if op == "s_nop" else 1
        writes = [(w, since + states) for w, since in writes if since < 5]
        dst = args.split(",")[0].strip()
        if op.startswith("v_") and re.match(r"s(\d+|\[\d+:\d+\])$", dst):
            lo, hi = (re.findall(r"\d+", dst) * 2)[:2]
            writes.append((set(range(int(lo), int(hi) + 1)), 0))
    return loads, stray, late


@pytest.mark.parametrize("src", SOURCES)
def test_lds_loads_have_m0_and_their_operands(src, tmp_path):
    out = str(tmp_path / "a.s")
    subprocess.run([build.HIPCC, "-x", "hip", *build.FLAGS, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, src), "-o", out], check=True, capture_output=True)
    loads, stray, late = _scan(open(out))
    assert loads > 0 and not stray and not late, (stray[:3], late[:3])


def test_the_scan_sees_both():
    load = [";;#ASMSTART", "s_mov_b32 m0, s1", "s_nop 0", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds", ";;#ASMEND"]
    assert _scan(load) == (1, [], [])
    assert _scan(["s_mov_b32 m0, s3"] + load)[1] == ["s_mov_b32 m0, s3"]
    assert len(_scan(["v_readlane_b32 s5, v0, 3"] + load)[2]) == 1
    assert len(_scan(["v_readlane_b32 s5, v0, 3", "s_nop 1"] + load)[2]) == 1
    assert not _scan(["v_readlane_b32 s5, v0, 3", "s_nop 2"] + load)[2]
    assert not _scan(["v_readlane_b32 s8, v0, 3"] + load)[2]
