"""Which draft levels give every row a second workgroup, from the same header as the library (built with g++): what the kernel relies on, and
the sides of the rule at the sizes they were measured at."""
import pytest

from attn_plan_util import compiled

SOURCE = r"""
#include "draft_plan.hpp"
extern "C" int sums_beside(int dtype, int B, int W, int V, int root) { return specvlm::sums_beside(dtype, B, W, V, root); }
"""
BF16, F32 = 0, 1


def beside(dtype, B, W, V, root=False):
    return bool(compiled(SOURCE).sums_beside(dtype, B, W, V, int(root)))


def test_bounds():
    for dtype in (BF16, F32):
        for V in (10, 4000, 32000, 65536, 65537, 250000):
            for W in (1, 10, 31, 32, 64):
                for B in (1, 3, 4, 12, 13, 128, 129, 2**20):
                    if beside(dtype, B, W, V):
                        # a request's log-sum-exps lie behind its counter; two workgroups of 1024 threads a row, all resident on 256 compute units
                        assert W < 32 and B * W <= 128, (dtype, B, W, V)


@pytest.mark.parametrize("dtype,B,W,V,root,expected", [
    (BF16, 1, 1, 65536, True, False), (BF16, 1, 1, 65537, True, True), (F32, 1, 1, 32000, True, False), (BF16, 1, 1, 32000, False, True),
    (BF16, 12, 10, 65000, False, True), (BF16, 128, 1, 65000, False, False), (BF16, 11, 10, 100001, False, True), (BF16, 12, 10, 100001, False, False),
    (F32, 5, 10, 152064, False, True), (F32, 6, 10, 152064, False, False), (F32, 8, 10, 65537, False, False), (F32, 8, 10, 250000, False, False),
    (F32, 4, 10, 250000, False, True), (F32, 3, 10, 65000, False, True), (F32, 8, 10, 65000, False, False), (F32, 12, 10, 16000, False, True),
])
def test_measured(dtype, B, W, V, root, expected):
    assert beside(dtype, B, W, V, root) == expected
