"""GPU parity of batches in the launch shape with two workgroups per compute unit, whose requests are spread over the XCDs
where KV heads are a multiple of 8, and of those among them that take twice the key ranges (at least four query heads
per KV head, long streams); and of batches next to them that are divided otherwise.  Each asserts its division and its kernel."""
import pytest

from attn_plan_util import Plan, plan_of_case
from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def slots(case):
    return case["k"].shape[2] if case["block_table"] is None else 16 * case["block_table"].shape[1]


# A contiguous cache gets a capacity that is no multiple of 16: with one, and paged, most of these calls are another kernel's.
@pytest.mark.parametrize("paged,B,Hq,Hkv,D,N,P,nn,splits,plan", [
    (False, 4, 32, 8, 128, 64, [2400, 33, 900, 0], [64, 1, 17, 2], 0, Plan(4, 0, 4)),     # four ranges, a request shorter than them
    (False, 2, 64, 8, 128, 60, [3900, 700], None, 0, Plan(4, 0, 4)),                      # ... a group of eight
    (False, 3, 32, 8, 128, 60, [2500, 3, 900], [60, 60, 7], 0, Plan(4, 0, 4)),            # ... 384 items
    (False, 3, 40, 10, 128, 60, [2600, 64, 1000], None, 0, Plan(4, 0, 4)),                # ... not a multiple of 8: contiguous ranges of items
    (True, 11, 8, 2, 128, 64, [2650, 33, 900, 0, 64, 5, 700, 31, 128, 1, 1300], [64, 1, 17, 2] + [64] * 7, 0, Plan(4, 0, 4)),   # paged, 352 items
    (True, 11, 8, 1, 128, 60, [3000, 700, 3, 5, 128, 2000, 60, 95, 31, 0, 40], None, 0, Plan(4, 0, 4)),                         # ... a group of eight
])
def test_four_ranges_by_the_library(sv, oracle, paged, B, Hq, Hkv, D, N, P, nn, splits, plan):
    from gpu_util import random_case
    longest = max(p + (N if nn is None else nn[b]) for b, p in enumerate(P))
    case = random_case(7300 + Hq + N + B, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged,
                       cap_extra=(8 - longest) % 16)
    assert paged or slots(case) % 16 == 8
    assert plan_of_case(case, splits) == plan and 256 < B * Hq * plan.ranges <= 512
    check(case, *run_both(sv, oracle, case, num_splits=splits), f"batch {B}x{Hq}/{Hkv}x{D} N={N} paged={paged}")


@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,splits,plan", [
    (9, 40, 40, 64, 20, [280, 5, 77, 31, 33, 200, 0, 64, 95], None, 0, Plan(1, 0, 1)),   # five heads per XCD, unsplit
    (12, 24, 24, 128, 33, [200, 5, 77, 31, 33, 150, 0, 64, 95, 1, 32, 127], None, 0, Plan(1, 0, 1)),   # three
    (2, 40, 40, 128, 60, [900, 1500], [60, 9], 4, Plan(4, 0, 4)),                  # a caller's key ranges
    (5, 20, 20, 128, 60, [900, 100, 1500, 7, 33], None, 3, Plan(3, 0, 3)),         # ... contiguous
])
@pytest.mark.parametrize("paged", [False, True])
def test_two_workgroups_per_compute_unit(sv, oracle, B, Hq, Hkv, D, N, P, nn, splits, plan, paged):
    from gpu_util import random_case
    case = random_case(7300 + Hq + N + B, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=0)
    assert plan_of_case(case, splits) == plan and 256 < B * Hq * plan.ranges <= 512
    check(case, *run_both(sv, oracle, case, num_splits=splits), f"batch {B}x{Hq}/{Hkv}x{D} N={N} splits={splits} paged={paged}")


# Streams per wavefront, most divided by the lengths: the same shapes paged, or with a capacity that is a multiple of 16.
@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,plan", [
    (4, 32, 8, 128, 64, [2400, 33, 900, 0], [64, 1, 17, 2], Plan(4, 0, 4, 2, 8, 1)),
    (2, 64, 8, 128, 60, [3900, 700], None, Plan(4, 0, 4, 2, 4, 1)),
    (3, 32, 8, 128, 60, [2500, 3, 900], [60, 60, 7], Plan(4, 0, 4, 2, 8, 1)),
    (3, 40, 10, 128, 60, [2600, 64, 1000], None, Plan(4, 0, 4, 2, 6, 1)),
    (3, 20, 20, 128, 60, [900, 100, 2500], None, Plan(4, 0, 4, 4, 12, 0)),
])
@pytest.mark.parametrize("paged", [False, True])
def test_streams_in_their_place(sv, oracle, B, Hq, Hkv, D, N, P, nn, plan, paged):
    from gpu_util import random_case
    longest = max(p + (N if nn is None else nn[b]) for b, p in enumerate(P))
    case = random_case(7300 + Hq + N + B, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=-longest % 16)
    assert plan_of_case(case) == plan
    check(case, *run_both(sv, oracle, case), f"batch {B}x{Hq}/{Hkv}x{D} N={N} paged={paged}")


@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,splits,plan", [
    (4, 32, 8, 128, 64, [1600, 33, 900, 0], [64, 1, 17, 2], 0, Plan(2, 32, 1)),    # row blocks: streams too short for four ranges
    (2, 64, 8, 128, 60, [1530, 700], None, 0, Plan(2, 32, 1)),
    (4, 32, 8, 128, 60, [1400, 3, 900, 500], None, 0, Plan(2, 32, 1)),
    (9, 24, 24, 64, 20, [600, 5, 77, 31, 33, 200, 0, 64, 95], None, 0, Plan(1, 32, 1)),
    (2, 40, 40, 128, 60, [900, 2500], [60, 9], 3, Plan(3, 0, 3)),                  # one workgroup per compute unit
    (3, 20, 20, 128, 60, [900, 100, 2500], None, 4, Plan(4, 0, 4)),
])
@pytest.mark.parametrize("paged", [False, True])
def test_divided_otherwise(sv, oracle, B, Hq, Hkv, D, N, P, nn, splits, plan, paged):
    from gpu_util import random_case
    case = random_case(7300 + Hq + N + B, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=0)
    assert plan_of_case(case, splits) == plan and (plan.block_rows or B * Hq * plan.ranges <= 256)
    check(case, *run_both(sv, oracle, case, num_splits=splits), f"batch {B}x{Hq}/{Hkv}x{D} N={N} splits={splits} paged={paged}")
