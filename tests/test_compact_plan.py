"""How many KV heads a workgroup of the compaction takes, from the same header as the library (built with g++): what the kernel
relies on, and the sides of the rule at the sizes they were measured at."""
import ctypes
import functools
import os
import random
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(None)
def _library():
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
        with open(src, "w") as f:
            f.write('#include "compact_plan.hpp"\n'
                    'extern "C" int bits(long long workgroups, int chunks) { return specvlm::compact_head_bits(workgroups, chunks); }\n')
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2509_11815_amd", "csrc"),
                        src, "-o", so], check=True)
        lib = ctypes.CDLL(so)
    lib.bits.argtypes = [ctypes.c_longlong, ctypes.c_int]
    return lib


def head_bits(workgroups, chunks):
    return _library().bits(workgroups, chunks)


@pytest.mark.parametrize("seed", range(2))
def test_bounds(seed):
    rng = random.Random(seed)
    for _ in range(3000):
        workgroups, chunks = int(2 ** rng.uniform(1, 22)), rng.choice([8, 16, 32]) * rng.randint(1, 64)
        bits = head_bits(workgroups, chunks)
        assert 0 <= bits <= 3
        assert bits == 0 or (chunks << bits <= 2048 and workgroups >> bits >= 512), (workgroups, chunks, bits)


@pytest.mark.parametrize("workgroups,chunks,heads", [
    # a path of 7 - 8 rows of 256 bytes
    (1024, 112, 2), (2048, 112, 2), (2048, 128, 2), (4096, 128, 4), (8192, 128, 8), (16384, 128, 8),
    # few workgroups, long paths: fewer heads each
    (1280, 1024, 1), (1024, 1024, 1), (2048, 256, 2), (2048, 320, 2), (2048, 640, 1), (1024, 512, 1), (4096, 320, 2), (4096, 1024, 2),
    (8192, 320, 4), (8192, 640, 2), (32768, 2048, 1), (512, 56, 1),
])
def test_measured_sizes(workgroups, chunks, heads):
    assert 1 << head_bits(workgroups, chunks) == heads
