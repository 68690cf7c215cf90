"""Row blocks in place of key ranges or of blocks of another height: the sides of the rule at head size 128 and one round of workgroups."""
import random

import pytest

from attn_plan_util import columns_of, plan_of


@pytest.mark.parametrize("shape,options,rows,splits", [
    # (requests, query heads, KV heads, head size, nodes, slots per request): seven tiles a stream of the row blocks, and eight
    ((1, 32, 32, 128, 60, 3584), {}, 32, 4), ((1, 32, 32, 128, 60, 3600), {}, 0, 8), ((2, 16, 16, 128, 60, 3328), {"paged": True}, 32, 4),
    ((1, 32, 16, 128, 60, 3584), {}, 32, 4), ((1, 32, 16, 128, 60, 3600), {}, 0, 8),
    # ten where four query heads share a KV head
    ((1, 32, 8, 128, 64, 5120), {}, 32, 4), ((1, 32, 8, 128, 64, 5136), {}, 0, 8),
    # fewer compute units than the key ranges would take; a caller's number of ranges; a call without partial results
    ((3, 16, 16, 128, 64, 1664), {}, 0, 5), ((1, 32, 32, 128, 60, 3328), {"num_splits": 8}, 0, 8), ((1, 64, 32, 128, 64, 416), {}, 16, 1),
])
def test_sides(shape, options, rows, splits):
    p = plan_of(*shape, **options)
    assert (p.block_rows, p.splits, p.columns) == (rows, splits, 0)


@pytest.mark.parametrize("seed", range(2))
def test_bounds(seed):
    """Whatever the division, it fits the workspace of the call's key ranges, and one round of workgroups stays one."""
    rng = random.Random(seed)
    for _ in range(2000):
        hkv, group = rng.choice([1, 2, 4, 5, 8, 16, 32, 40]), rng.choice([1, 1, 2, 4, 7, 8])
        B, N, cap = rng.choice([1, 1, 2, 3, 6]), rng.randint(1, 64), 16 * rng.randint(4, 500)
        p = plan_of(B, hkv * group, hkv, 128, N, cap, paged=rng.random() < 0.3)
        if p.columns or not p.block_rows or p.splits == 1:
            continue
        units = B * hkv * -(-group * N // p.block_rows)
        what = (B, hkv * group, hkv, N, cap, p)
        assert p.splits <= p.ranges and units * p.block_rows * p.splits <= B * hkv * group * 64 * p.ranges, what
        assert B * hkv * group * p.ranges > 256 or units * p.splits <= 256, what
        assert columns_of(B, hkv * group, hkv, 128, N, cap).bytes > 0, what
