"""GPU parity of batches whose requests are spread over the XCDs (KV heads a multiple of 8), and of those among them
that take twice the key ranges (at least four query heads per KV head, long streams)."""
import pytest

from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,splits", [
    (4, 32, 8, 128, 64, [1600, 33, 900, 0], [64, 1, 17, 2], 0),     # four key ranges, two workgroups per unit
    (2, 64, 8, 128, 60, [1530, 700], None, 0),                      # ... a group of eight
    (4, 32, 8, 128, 60, [1400, 3, 900, 500], None, 0),              # streams too short for that
    (9, 24, 24, 64, 20, [600, 5, 77, 31, 33, 200, 0, 64, 95], None, 0),   # three heads per XCD, unsplit
    (2, 40, 40, 128, 60, [900, 2500], [60, 9], 3),                  # five heads per XCD, a caller's key ranges
    (3, 20, 20, 128, 60, [900, 100, 2500], None, 0),                # not a multiple of 8: contiguous ranges as before
])
@pytest.mark.parametrize("paged", [False, True])
def test_batches(sv, oracle, B, Hq, Hkv, D, N, P, nn, splits, paged):
    from gpu_util import random_case
    case = random_case(7300 + Hq + N + B, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=0)
    check(case, *run_both(sv, oracle, case, num_splits=splits), f"batch {B}x{Hq}/{Hkv}x{D} N={N} splits={splits} paged={paged}")
