"""Which bf16 attention calls take the kernel with a key stream per wavefront: bounds that the kernel and the workspace rely on
over random shapes, the sides of the rule at measured sizes, and no spilled register (memory operations are counted by hand)."""
import random

import pytest

from attn_plan_util import plan_of, streams_of


@pytest.mark.parametrize("seed", range(4))
def test_bounds(seed):
    rng = random.Random(seed)
    taken = set()
    for _ in range(2000):
        hkv, group = rng.choice([1, 2, 4, 5, 8, 16, 32, 40]), rng.choice([1, 1, 2, 3, 4, 8])
        B, D, N = rng.choice([1, 2, 3, 4, 5, 6, 8, 16, 40]), rng.choice([64, 128]), rng.choice([1, 13, 17, 32, 36, 60, 64])
        paged = rng.random() < 0.3
        cap = int(16 * 2 ** rng.uniform(0, 9)) // 16 * 16 + (0 if paged else rng.choice([0, 0, 1, 8]))
        given = rng.choice([0, 0, 0, 1, 3])
        what = (B, hkv * group, hkv, D, N, cap, given)
        s, plan = streams_of(*what, paged=paged), plan_of(*what, paged=paged)
        if not s:
            continue
        units = B * hkv * -(-group * N // 64)
        assert 1 <= s <= min(4, plan.ranges) and units * s <= 256 and B > 1 and not given, what
        assert cap % 16 == 0, what
        assert (s == 1) == (plan.splits == 1), what           # no partial results where there were none
        # partial results (64 rows of every unit and range) fit where those of the key ranges do
        assert s == 1 or units * s <= B * hkv * group * plan.ranges, what
        taken.add(s)
    assert taken == {1, 2, 3, 4}


@pytest.mark.parametrize("shape,streams", [
    # (requests, query heads, KV heads, head size, nodes, slots per request)
    ((4, 32, 8, 128, 64, 3072), 2), ((8, 32, 16, 128, 60, 4848), 1), ((4, 40, 40, 128, 64, 736), 1), ((2, 40, 40, 128, 64, 3808), 3),
    ((2, 32, 32, 128, 47, 4528), 4), ((5, 16, 16, 64, 60, 3088), 3), ((8, 32, 32, 128, 60, 976), 1),
    # one request; one range where there were three; few or short streams; blocks less than 55 % full; a cache that ends inside a half tile
    ((1, 32, 32, 128, 60, 3328), 0), ((4, 40, 40, 128, 60, 4928), 0), ((4, 32, 32, 128, 60, 608), 0), ((7, 32, 32, 128, 60, 288), 0),
    ((3, 40, 40, 128, 28, 1104), 0), ((8, 32, 32, 128, 60, 977), 0), ((7, 40, 40, 128, 64, 1744), 0),
])
def test_measured_shapes(shape, streams):
    assert streams_of(*shape) == streams


@pytest.mark.parametrize("shape,contiguous,paged", [
    # row blocks in one round of workgroups, a multiple of 8: the same number of key ranges loses to them ...
    ((8, 40, 10, 128, 22, 512), 0, 0), ((6, 64, 8, 64, 18, 832), 0, 0), ((4, 40, 20, 128, 46, 3872), 0, 0), ((6, 40, 8, 128, 28, 1792), 0, 0),
    # ... half as many more mostly, twice as many do not
    ((5, 28, 4, 128, 24, 2912), 0, 0), ((3, 16, 8, 128, 36, 2752), 0, 0), ((8, 20, 5, 128, 22, 3392), 3, 3), ((3, 16, 4, 64, 60, 4304), 4, 4),
    # not a multiple of 8: short streams with few blocks a unit lose
    ((5, 50, 10, 128, 30, 464), 0, 0), ((5, 50, 10, 128, 30, 1344), 1, 1), ((9, 20, 4, 128, 40, 512), 1, 1), ((10, 40, 5, 64, 19, 4448), 1, 0),
    # more than one round
    ((8, 50, 10, 128, 30, 512), 1, 1), ((6, 50, 10, 128, 42, 1040), 1, 1),
])
def test_row_blocks_in_one_round(shape, contiguous, paged):
    assert plan_of(*shape).block_rows and (streams_of(*shape), streams_of(*shape, paged=True)) == (contiguous, paged)


@pytest.mark.parametrize("shape,contiguous,paged", [
    # 224 unsplit workgroups or more without shared K and V: from 24 tiles on, paged 18; fewer workgroups, shared ones, head size 64 from 14 on
    ((7, 32, 32, 128, 64, 448), 0, 0), ((7, 32, 32, 128, 64, 560), 0, 1), ((8, 32, 32, 128, 60, 736), 0, 1), ((8, 32, 32, 128, 60, 752), 1, 1),
    ((223, 1, 1, 128, 60, 448), 1, 1), ((7, 32, 16, 128, 64, 448), 1, 1), ((7, 32, 32, 64, 64, 448), 1, 1),
])
def test_short_streams_that_share_nothing(shape, contiguous, paged):
    assert (streams_of(*shape), streams_of(*shape, paged=True)) == (contiguous, paged)


def test_far_strides_take_another_kernel():
    """32-bit offsets of half a tile."""
    assert streams_of(8, 32, 32, 128, 60, 976, token_stride=(1 << 22) - 8) == 1
    assert streams_of(8, 32, 32, 128, 60, 976, token_stride=1 << 22) == 0


def test_spills_nothing():
    from paper_2509_11815_amd import build
    usage = {k: v for k, v in build.kernel_resource_usage("attn_streams.hip").items() if "attn_streams_kernel" in k}
    assert len(usage) == 4, sorted(usage)                      # two head sizes x contiguous / paged
    for name, u in usage.items():
        assert u["scratch"] == 0 and u["lds"] <= 160 * 1024, (name, u)
