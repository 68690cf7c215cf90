"""The row-dividing attention kernels count outstanding memory operations by hand: no register may spill, and partial results
are added up while later ones are on their way."""
import os
import re
import subprocess

import pytest

def test_row_block_kernels_spill_nothing():
    from paper_2509_11815_amd import build
    usage = {k: v for k, v in build.kernel_resource_usage("attn_wave.hip").items() if "attn_wave_kernel" in k}
    assert len(usage) == 8, sorted(usage)                      # two head sizes x two block heights x contiguous / paged
    for name, u in usage.items():
        assert u["scratch"] == 0 and u["lds"] <= 160 * 1024, (name, u)


@pytest.fixture(scope="module")
def waits(tmp_path_factory):
    """Per kernel, the memory-operation counts of its waits in program order."""
    from paper_2509_11815_amd import build
    out = str(tmp_path_factory.mktemp("asm") / "attn_wave.s")
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S", "-o", out, os.path.join(build.CSRC, "attn_wave.hip")],
                   check=True, capture_output=True)
    counts, name = {}, None
    with open(out) as f:
        for line in f:
            if m := re.match(r"(_ZN\S*attn_wave_kernel\S*):", line):
                name = m.group(1)
            if m := re.search(r"s_waitcnt vmcnt\((\d+)\)\s*$", line):
                counts.setdefault(name, []).append(int(m.group(1)))
    return counts


@pytest.mark.parametrize("D,blocks,vectors", [(64, 1, 1), (64, 2, 1), (128, 1, 1), (128, 2, 2)])
@pytest.mark.parametrize("paged", [0, 1])
def test_partials_are_added_as_they_land(waits, D, blocks, vectors, paged):
    """Eight partials of `vectors` 16-byte loads each are requested together; before partial u is added, those of the 7 - u later
    ones may be outstanding."""
    found = [c for name, c in waits.items() if f"ILi{D}ELi{blocks}ELb{paged}E" in name]
    assert len(found) == 1
    want = [(7 - u) * vectors for u in range(8)]
    assert any(found[0][i:i + 8] == want for i in range(len(found[0]))), (want, found[0])
