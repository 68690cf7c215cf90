"""Kernels whose last workgroup or wavefront reads what the others have written: the reads are relaxed, so that only what stands between the ticket
and them keeps the compiler from moving them ahead of it.  In the code of every such kernel a fence or a memory barrier of the compiler does."""
import os
import re
import subprocess

import pytest

TICKET = re.compile(r'atomicrmw add ptr.* syncscope\("agent(?:-one-as)?"\) monotonic')
ORDERS = re.compile(r"\bfence\b|~\{memory\}")
READS = re.compile(r"\bload atomic\b|@llvm\.amdgcn\.raw\.ptr\.buffer\.load")


@pytest.mark.parametrize("source,at_least", [("sample_kernels.hip", 4), ("draft_tree.hip", 4), ("head_argmax.hip", 4), ("attn_wave.hip", 8),
                                             ("attn_streams.hip", 4), ("attn_mfma.hip", 4)])
def test_what_orders_the_reads_behind_the_ticket(tmp_path, source, at_least):
    from paper_2509_11815_amd import build
    out = str(tmp_path / "k.ll")
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S", "-emit-llvm", "-o", out, os.path.join(build.CSRC, source)], check=True, capture_output=True)
    with open(out) as f:
        lines = f.read().split("\n")
    found = 0
    for i, line in enumerate(lines):
        if not TICKET.search(line):
            continue
        found += 1
        for later in lines[i + 1:]:
            if ORDERS.search(later):
                break
            assert later != "}", (i, line)
            assert not READS.search(later), (line, later)
    assert found >= at_least
