"""The row broadcasts of blk16.hpp are inline assembly, which the compiler does
not look into for hazards: a DPP read needs two wait states after the VALU
instruction that wrote its source.  The compiled kernels are checked for a
write that came too close (a copy or a reload that the register allocator
put there would be one)."""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DPP = re.compile(r"\s+v_\w+_dpp (?:v\[\d+:\d+\]|v\d+), (v\[\d+:\d+\]|v\d+)")


def _regs(text):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", text)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else {int(text[1:])}


def hazards(asm):
    """(number of broadcasts, lines whose source was written fewer than two wait states before)."""
    lines = [ln for ln in asm.splitlines() if re.match(r"\s+[a-z]\w*", ln)]
    bad, seen = [], 0
    for i, ln in enumerate(lines):
        m = DPP.match(ln)
        if not m:
            continue
        seen += 1
        src, states = _regs(m.group(1)), 0
        for prev in reversed(lines[max(0, i - 3):i]):
            if states >= 2:
                break
            op, *rest = prev.split(None, 1)
            if op == "s_nop":
                states += 1 + int(rest[0].split()[0], 0)
                continue
            written = re.match(r"(v\[\d+:\d+\]|v\d+)", rest[0]) if rest else None
            if op.startswith("v_") and written and _regs(written.group(1)) & src:
                bad.append((prev.strip(), ln.strip()))
            states += 1
    return seen, bad


def test_the_check_sees_a_hazard():
    near = "\tv_mov_b32_e32 v4, v1\n\tv_fmac_f64_dpp v[8:9], v[4:5], v[6:7] row_newbcast:3\n"
    far = "\tv_mov_b32_e32 v4, v1\n\ts_nop 1\n\tv_fmac_f64_dpp v[8:9], v[4:5], v[6:7] row_newbcast:3\n"
    assert len(hazards(near)[1]) == 1 and hazards(far) == (1, [])


@pytest.mark.parametrize("source", ["factor.hip", "kernels.hip"])
def test_broadcast_sources_are_old_enough(source, tmp_path):
    import importlib.util

    spec = importlib.util.spec_from_file_location("_b", os.path.join(ROOT, "paper_1604_02528_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    out = str(tmp_path / "k.s")
    flags = [f for f in build.common_flags() if f not in ("-fPIC", "-pthread")]
    r = subprocess.run([build.hipcc(), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    seen, bad = hazards(open(out).read())
    assert seen > 100
    assert not bad, bad[:5]
