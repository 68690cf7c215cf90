"""Which bf16 attention calls deal their workgroups out to the requests by length: bounds that the kernel and the workspace rely on over
random shapes, and the sides of the rule at measured sizes."""
import random

import pytest

from attn_plan_util import columns_of, plan_of

COUNTERS = 1024 * 4 * 128


@pytest.mark.parametrize("seed", range(4))
def test_bounds(seed):
    rng = random.Random(seed)
    seen = set()
    for _ in range(6000):
        hkv, group = rng.choice([1, 2, 4, 5, 8, 16, 32, 40]), rng.choice([1, 1, 2, 3, 4, 8])
        B, D, N = rng.choice([1, 2, 3, 4, 5, 6, 8, 16, 17, 40]), rng.choice([64, 128]), rng.choice([13, 32, 36, 48, 60, 64])
        paged = rng.random() < 0.3
        cap = int(16 * 2 ** rng.uniform(0, 9)) // 16 * 16 + (0 if paged else rng.choice([0, 0, 1, 8]))
        given = rng.choice([0, 0, 0, 0, 1, 3])
        what = (B, hkv * group, hkv, D, N, cap, given)
        c, p = columns_of(*what, paged=paged), plan_of(*what, paged=paged)
        old = 0 if p.ranges == 1 else COUNTERS + B * hkv * group * p.ranges * (64 * D * 2 + 64 * 8)
        assert not c.even_by_length and c.even_bytes == old, what                   # what was enough stays enough
        assert c.even_columns in (0, B * p.streams, B) and (not p.streams or c.even_columns == B * p.streams), what
        if not c.columns:
            assert not p.streams and c.bytes == old, what
            continue
        units = hkv * -(-group * N // 64)
        assert B <= c.columns and units * c.columns <= 256 and cap % 16 == 0 and not given and B > 1, what
        if c.by_length:
            assert c.columns > B and B <= 16, what                                  # a row of 16 lanes holds the requests
            part = units * c.columns * (64 * D * (4 if p.splits == 1 else 2) + 64 * 8)
            assert c.bytes == max(old, COUNTERS + part), what
        else:
            assert c.columns == B * max(1, p.streams) and c.bytes == old, what
            assert p.splits == 1 or p.streams > 1, what                             # one column a request: no partial results
        seen.add((bool(c.by_length), p.streams, bool(p.block_rows)))
    assert {(True, 1, False), (True, 0, True), (True, 0, False), (False, 1, False), (False, 0, False)} <= seen


@pytest.mark.parametrize("shape,paged,columns,by_length", [
    # (requests, query heads, KV heads, head size, nodes, slots per request)
    ((4, 32, 8, 128, 64, 3072), False, 8, 1), ((3, 32, 16, 128, 60, 3728), False, 8, 1), ((6, 32, 32, 128, 60, 2864), False, 8, 1),
    ((4, 40, 40, 128, 60, 4928), True, 6, 1), ((4, 35, 5, 128, 48, 2064), False, 8, 1), ((4, 28, 4, 128, 60, 3072), False, 8, 1),
    # one column a request: no room for more; short
    ((8, 32, 32, 128, 60, 976), False, 8, 0), ((8, 40, 8, 128, 48, 288), True, 8, 0), ((8, 32, 32, 128, 60, 272), False, 0, 0), ((4, 40, 40, 128, 64, 736), False, 4, 0),
    # short, heads shared: from seven tiles on, at 64 always
    ((7, 32, 4, 128, 64, 144), False, 0, 0), ((7, 32, 4, 128, 64, 192), True, 0, 0), ((7, 32, 4, 128, 64, 208), False, 7, 0), ((7, 32, 4, 64, 64, 144), False, 7, 0),
    # head size 64: longer streams
    ((5, 16, 16, 64, 60, 6144), False, 16, 1), ((5, 16, 16, 64, 60, 3088), False, 15, 0),
    # key ranges and row blocks: longer ones, as they lose more where requests are shorter than their cache; row blocks whose
    # workgroups do not share the XCDs evenly, or make more than one round, lose less
    ((3, 40, 40, 128, 60, 1744), False, 0, 0), ((4, 32, 16, 128, 64, 1952), False, 0, 0), ((8, 16, 4, 64, 64, 2544), True, 0, 0),
    ((2, 16, 4, 128, 60, 5184), False, 0, 0), ((2, 64, 8, 128, 60, 3504), True, 4, 1), ((8, 32, 16, 128, 32, 3664), False, 16, 1),
    ((6, 32, 4, 64, 60, 6544), False, 8, 1), ((5, 32, 32, 128, 60, 2272), False, 8, 1),
    # the other kernels: one request, shared heads and a third of the columns idle, short row blocks, capacities that end inside 16 slots
    ((1, 64, 8, 128, 60, 4064), False, 0, 0), ((5, 32, 16, 128, 60, 4976), False, 0, 0), ((4, 32, 8, 128, 32, 1024), False, 0, 0),
    ((4, 40, 40, 128, 60, 4921), False, 0, 0),
])
def test_measured_shapes(shape, paged, columns, by_length):
    c = columns_of(*shape, paged=paged)
    assert (c.columns, c.by_length) == (columns, by_length)


def test_spills_nothing():
    from paper_2509_11815_amd import build
    usage = {k: v for k, v in build.kernel_resource_usage("attn_streams.hip").items() if "attn_shares_kernel" in k}
    assert len(usage) == 4, sorted(usage)                      # two head sizes x contiguous / paged
    for name, u in usage.items():
        assert u["scratch"] == 0 and u["lds"] <= 160 * 1024, (name, u)
