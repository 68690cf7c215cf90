"""GPU parity of the attention calls whose wavefronts have a key stream each over 64 query rows: no tile, one to five tiles per
stream, tiles cut by the tree and by the request's end, a cache that ends inside a tile, blocks across head borders, partial
results, bad requests beside good ones.  The choice is the library's; all of these are shapes it takes."""
import numpy as np
import pytest

from attn_plan_util import division_of, plan_of
from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def make(seed, B, Hq, Hkv, D, N, P, nn, paged):
    """A contiguous cache gets the least capacity that is a multiple of 16 (one that ends inside 16 slots is another kernel's)."""
    from gpu_util import random_case
    longest = max(p + (N if nn is None else nn[b]) for b, p in enumerate(P))
    case = random_case(seed, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=-longest % 16)
    cap = case["block_table"].shape[1] * 16 if paged else case["k"].shape[2]
    return case, plan_of(B, Hq, Hkv, D, N, cap, paged=paged)


# 32 keys a tile, four streams a range
# (by_length: the lengths divide the call, otherwise every request takes as many ranges)
@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,ranges,by_length", [
    (6, 32, 32, 64, 64, [0, 1, 31, 64, 127, 400], [1, 64, 33, 64, 1, 64], 1, 0),
    (5, 32, 32, 128, 40, [0, 95, 216, 300, 440], [40, 33, 40, 7, 40], 1, 0),        # 40 of 64 rows; 2, 4, 8, 10 and 15 tiles
    (5, 40, 8, 128, 48, [3, 450, 129, 96, 33], [48, 48, 2, 32, 48], 1, 0),          # 240 rows: blocks across head borders
    (8, 48, 12, 64, 24, [470, 0, 33, 64, 96, 128, 256, 17], None, 1, 0),                # 96 rows: the second block half full
    (3, 32, 16, 128, 64, [2300, 5, 511], [64, 64, 17], 2, 1),
    (5, 16, 16, 128, 60, [1400, 0, 40, 700, 96], [60, 1, 60, 59, 60], 3, 0),
    (2, 32, 32, 128, 36, [2200, 700], None, 4, 0),
])
@pytest.mark.parametrize("paged", [False, True])
def test_streams(sv, oracle, B, Hq, Hkv, D, N, P, nn, ranges, by_length, paged):
    case, plan = make(8100 + D + N + B, B, Hq, Hkv, D, N, P, nn, paged)
    assert plan.columns and (plan.streams, plan.by_length) == (ranges, by_length)
    check(case, *run_both(sv, oracle, case), f"streams {B}x{Hq}/{Hkv}x{D} N={N} ranges={ranges} paged={paged}")


@pytest.mark.parametrize("B,H,P,ranges,by_length", [(6, 32, [440, 100, 0, 300, 64, 5], 1, 0), (3, 32, [2300, 40, 500], 2, 1)])
def test_bad_requests_beside_good_ones(sv, oracle, B, H, P, ranges, by_length):
    """A malformed tree and a length past the cache set the error word and leave their requests' rows alone."""
    import torch
    from gpu_util import assert_attn_close, i32, to_dev, to_host_f64
    case, _ = make(8200 + B, B, H, H // 2 if ranges == 2 else H, 128, 56, P, None, False)
    assert division_of(B, H, case["k"].shape[1], 128, 56, case["k"].shape[2]) == (ranges, by_length)
    parent, lengths = case["parent"].copy(), case["prefix_len"].copy()
    parent[1, 7] = 7
    lengths[2] = case["k"].shape[2]
    out = torch.full(case["q"].shape, 7.0, dtype=torch.bfloat16, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    sv.specvlm_tree_verify_attn(to_dev(case["q"]), to_dev(case["k"]), to_dev(case["v"]), i32(lengths), i32(parent), out=out, err_flag=err)
    assert int(err.item()) == 1 | 4
    got = to_host_f64(out)
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None)
    good = [b for b in range(B) if b not in (1, 2)]
    assert_attn_close(got[good], ref[good], "bf16", "good requests")
    assert np.all(got[1:3] == 7.0)


@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,ranges,by_length", [
    (5, 15, 3, 128, 64, [2050, 5, 700, 33, 0], [64, 1, 64, 17, 2], 3, 0),                        # 225 workgroups
    (9, 17, 17, 64, 64, [410, 5, 77, 31, 33, 200, 0, 64, 95], None, 1, 0),                       # 153
    (3, 19, 19, 128, 60, [3100, 40, 700], None, 4, 0),                                           # 228
    (3, 19, 19, 128, 60, [3560, 40, 700], None, 4, 1),                                           # 247
])
@pytest.mark.parametrize("paged", [False, True])
def test_workgroups_no_multiple_of_eight(sv, oracle, B, Hq, Hkv, D, N, P, nn, ranges, by_length, paged):
    """The first XCDs take an item more."""
    case, plan = make(8500 + D + N + B, B, Hq, Hkv, D, N, P, nn, paged)
    assert (plan.streams, plan.by_length) == (ranges, by_length) and plan.columns * Hkv * -(-Hq // Hkv * N // 64) % 8
    check(case, *run_both(sv, oracle, case), f"streams {B}x{Hq}/{Hkv}x{D} N={N} ranges={ranges} paged={paged}")
