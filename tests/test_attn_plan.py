"""How bf16 attention calls are divided among workgroups: bounds that the kernels and the workspace rely on, over
random shapes, and the sides of the rules at the sizes they were measured at."""
import random

import pytest

from attn_plan_util import Plan, plan_of


@pytest.mark.parametrize("seed", range(4))
def test_bounds(seed):
    rng = random.Random(seed)
    seen = set()
    for _ in range(1500):
        hkv = rng.choice([1, 2, 3, 4, 5, 8, 16, 32, 40])
        group = rng.choice([1, 1, 2, 3, 4, 7, 8])
        D, N = rng.choice([64, 128]), rng.choice([1, 13, 16, 17, 32, 60, 64])
        B = rng.choice([1, 2, 3, 4, 8, 16, 40])
        cap = int(16 * 2 ** rng.uniform(0, 9)) // 16 * 16
        given = rng.choice([0, 0, 0, 1, 2, 5, 9, 64])
        p = plan_of(B, hkv * group, hkv, D, N, cap, given, paged=rng.random() < 0.3)
        heads = B * hkv * group
        what = (B, hkv * group, hkv, D, N, cap, given, p)
        assert 1 <= p.splits <= p.ranges <= 64, what
        if heads > 1024:
            assert p.ranges == 1, what                       # one set of ticket counters per (request, head)
        elif given:
            assert p.ranges == p.splits == given, what       # a caller's count is taken as given
        if p.block_rows == 0:
            assert p.splits == p.ranges, what
        else:
            blocks = -(-group * N // p.block_rows)
            units = B * hkv * blocks
            assert p.splits == 1 or units <= 1024, what
            # partial results of the row blocks fit where those of the key ranges do (64 rows per head)
            assert units * p.block_rows * p.splits <= heads * 64 * p.ranges, what
        seen.add((p.block_rows, p.splits > 1))
    assert seen == {(0, False), (0, True), (16, False), (16, True), (32, False), (32, True)}


@pytest.mark.parametrize("shape,plan", [
    # (requests, query heads, KV heads, head size, nodes, slots per request); the second, 3324 keys: eight key ranges 16.6 us, row blocks 16.1 (paged
    # 17.8 and 16.2; 1060 keys in the same capacity 12.1 and 9.9)
    ((1, 32, 32, 128, 60, 832), Plan(7, 32, 4)), ((1, 32, 32, 128, 60, 3328), Plan(8, 32, 4)),
    ((8, 32, 32, 128, 60, 968), Plan(1, 0, 1)), ((4, 40, 40, 128, 60, 4928), Plan(3, 0, 3, 0, 6, 1)),
    # at least four query heads per KV head: four ranges, 340 - 512 work items of two per compute unit (capacities that are a
    # multiple of 16 go to the kernel with a key stream per wavefront, below)
    ((4, 32, 8, 128, 64, 3080), Plan(4, 0, 4)), ((2, 64, 8, 128, 60, 4568), Plan(4, 0, 4)), ((3, 40, 8, 128, 60, 3080), Plan(4, 0, 4)),
    ((4, 28, 4, 128, 60, 3080), Plan(4, 0, 4)), ((3, 32, 8, 128, 60, 3080), Plan(4, 0, 4)), ((2, 48, 8, 128, 60, 4568), Plan(4, 0, 4)),
    # ... where row blocks win
    ((4, 32, 8, 128, 60, 2064), Plan(2, 32, 1)), ((2, 64, 8, 128, 60, 2560), Plan(2, 32, 1)), ((2, 64, 8, 128, 60, 3072), Plan(2, 32, 1, 0, 4, 1)),
    # ... not for one request, two query heads per KV head, head size 64 or more than two ranges to begin with
    ((1, 128, 8, 128, 60, 4560), Plan(2, 0, 2)), ((4, 32, 16, 128, 60, 3080), Plan(2, 0, 2)), ((4, 32, 8, 64, 60, 4560), Plan(2, 32, 1, 0, 8, 1)),
    ((2, 32, 8, 128, 60, 3080), Plan(4, 0, 4)), ((4, 16, 4, 128, 60, 3080), Plan(4, 0, 4)),
    # the kernel with a key stream per wavefront in their place
    ((8, 32, 32, 128, 60, 976), Plan(1, 0, 1, 1, 8, 0)), ((4, 32, 8, 128, 64, 3072), Plan(4, 0, 4, 2, 8, 1)), ((2, 64, 8, 128, 60, 4560), Plan(4, 0, 4, 2, 4, 1)),
    ((3, 40, 8, 128, 60, 3072), Plan(4, 0, 4, 2, 6, 1)), ((4, 28, 4, 128, 60, 3072), Plan(4, 0, 4, 2, 8, 1)), ((3, 32, 8, 128, 60, 3072), Plan(4, 0, 4, 2, 8, 1)),
    ((2, 48, 8, 128, 60, 4560), Plan(4, 0, 4, 2, 5, 1)), ((4, 32, 16, 128, 60, 3072), Plan(2, 0, 2, 2, 8, 1)), ((2, 32, 8, 128, 60, 3072), Plan(4, 0, 4, 4, 8, 0)),
    ((4, 16, 4, 128, 60, 3072), Plan(4, 0, 4, 4, 16, 0)),
])
def test_measured_shapes(shape, plan):
    assert plan_of(*shape) == plan


def test_far_token_strides_keep_all_rows_in_a_workgroup():
    """The row-dividing kernels hold 32-bit offsets of half a tile."""
    assert plan_of(1, 4, 4, 128, 60, 160).block_rows
    assert plan_of(1, 4, 4, 128, 60, 160, token_stride=(1 << 22) - 8).block_rows
    assert plan_of(1, 4, 4, 128, 60, 160, token_stride=1 << 22).block_rows == 0
