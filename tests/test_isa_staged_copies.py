"""Build-time guard for the copies that go straight into LDS (s_mov_b32 m0 and buffer_load ... lds in one assembly statement).

The compiler puts the wait states that this hardware asks for between its own instructions, but sees neither the write of M0 nor the load in
an assembly statement.  This test compiles the attention kernels to assembly and checks in front of every such copy, scanning the text linearly:
M0, written by a scalar instruction, is one wait state old, and no scalar operand was written by a vector instruction within five."""
import os
import re
import subprocess

import pytest

from paper_2409_16997_amd import build as hip_build

SGPR = re.compile(r"\bs(?:(\d+)|\[(\d+):(\d+)\])")


def sgprs(text):
    out = set()
    for one, lo, hi in SGPR.findall(text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def instructions(lines):
    for ln in lines:
        text = ln.split(";")[0].strip()
        if text and not text.startswith(".") and not text.endswith(":"):
            yield text


def states(text):
    """Wait states that an instruction is worth for the ones behind it."""
    return int(text.split()[1], 0) + 1 if text.startswith("s_nop") else 1


def faults(code):
    """(number of staged copies, the copies in front of which a wait state is missing)"""
    copies, bad = 0, []
    for i, text in enumerate(code):
        if not (text.startswith("buffer_load") and text.endswith(" lds")):
            continue
        copies += 1
        operands = sgprs(text)
        between, j = 0, i - 1
        m0_seen = False
        while j >= 0 and (between < 5 or not m0_seen):
            before = code[j]
            op, _, rest = before.partition(" ")
            dest = rest.split(",")[0].strip()
            if not m0_seen and dest == "m0":
                m0_seen = True
                if between < 1:
                    bad.append((i, before, text))
            if between < 5 and op.startswith("v_") and sgprs(dest) & operands:
                bad.append((i, before, text))
            between += states(before)
            j -= 1
        assert m0_seen, text
    return copies, bad


def test_the_check_itself():
    copy = "buffer_load_dwordx4 v199, s[8:11], s21 offen lds"
    assert faults(["s_mov_b32 m0, s35", copy])[1] and not faults(["s_mov_b32 m0, s35", "s_nop 0", copy])[1]
    late = ["v_readfirstlane_b32 s9, v1", "s_mov_b32 m0, s35", "s_nop 0", copy]
    assert faults(late)[1] and not faults(late[:1] + ["s_nop 2"] + late[1:])[1]


@pytest.mark.timeout(600)
@pytest.mark.parametrize("source", ["intfa_attention.hip", "intfa_attention_half.hip", "intfa_attention_fewq.hip"])
def test_every_staged_copy_has_its_wait_states(source, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    out = tmp_path / "kernels.s"
    subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", "-I", hip_build.INCLUDE, "-I", hip_build.CSRC, os.path.join(hip_build.CSRC, source), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    copies, bad = faults(list(instructions(out.read_text().splitlines())))
    assert copies >= 300, f"expected the copies of every instantiation, found {copies}"
    assert not bad, f"{len(bad)} of {copies} copies, the first: {bad[0]}"
