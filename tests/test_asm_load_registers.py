"""Loads written in inline asm put their registers in the compiler's hands while they are still on their way: it may copy, spill or reuse
them.  In the code it makes, no instruction between such a load and the next wait for loads names a register that the load writes."""
import os
import re
import subprocess

import pytest

LOAD = re.compile(r"global_load_dword(?:x[234])? v(?:\[(\d+):(\d+)\]|(\d+)), v\d+, s\[")


def named(line):
    """The vector registers that an instruction names."""
    regs = {int(x) for x in re.findall(r"\bv(\d+)\b", line)}
    for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", line):
        regs |= set(range(int(lo), int(hi) + 1))
    return regs


@pytest.mark.parametrize("source,at_least", [("attn_wave.hip", 100), ("attn_mfma.hip", 40), ("head_argmax.hip", 100)])
def test_no_register_of_a_load_in_flight_is_named(tmp_path, source, at_least):
    from paper_2509_11815_amd import build
    out = str(tmp_path / "k.s")
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S", "-o", out, os.path.join(build.CSRC, source)], check=True, capture_output=True)
    with open(out) as f:
        lines = [line.strip() for line in f]
    found = 0
    for i, line in enumerate(lines):
        if not (m := LOAD.match(line)) or not any("#ASMSTART" in x for x in lines[i - 2:i]):
            continue
        found += 1
        lo, hi = int(m.group(1) or m.group(3)), int(m.group(2) or m.group(3))
        for later in lines[i + 1:]:
            if "vmcnt(" in later or later.startswith("s_endpgm"):
                break
            if later and later[0] not in ";.":
                assert not named(later) & set(range(lo, hi + 1)), (line, later)
    assert found >= at_least
