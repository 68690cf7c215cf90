"""GPU parity of the attention calls whose query rows are divided among workgroups (blocks of 16 or 32 rows
of a KV head's group): block edges, rows of a block spread over several heads, tile and capacity edges,
partial results in more than one batch.  The choice is the library's; all of these are shapes it takes."""
import pytest

from attn_plan_util import plan_of_case
from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn,splits", [
    (1, 1, 1, 128, 1, [0], None, 0),                            # one row, one key, a cache of 8 slots
    (1, 2, 2, 64, 16, [15], None, 0),                           # one full row block; 31 keys: a tile one short
    (2, 2, 2, 128, 17, [16, 112], [16, 17], 0),                 # a second block of one row; 32 and 129 keys
    (1, 3, 1, 128, 33, [95], None, 0),                          # 99 rows of a group: blocks across head borders
    (2, 8, 1, 64, 13, [300, 7], [13, 2], 0),                    # 104 rows, 13 per head
    (3, 40, 40, 64, 60, [232, 100, 5], [60, 33, 1], 0),         # blocks of 32 rows, unsplit
    (2, 32, 32, 128, 64, [803, 947], [64, 31], 0),              # ... and with key ranges
    (1, 2, 2, 128, 60, [1000], None, 9),                        # more key ranges than one batch of partials
    (1, 1, 1, 64, 20, [2100], [19], 64),                        # the most a caller can ask for
    (1, 4, 2, 128, 60, [333], None, 3),
])
@pytest.mark.parametrize("paged", [False, True])
def test_row_blocks(sv, oracle, B, Hq, Hkv, D, N, P, nn, splits, paged):
    from gpu_util import random_case
    case = random_case(7000 + D + N + splits, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged,
                       cap_extra=0)
    plan = plan_of_case(case, splits)
    assert plan.block_rows and not plan.columns
    check(case, *run_both(sv, oracle, case, num_splits=splits), f"rows {B}x{Hq}/{Hkv}x{D} N={N} splits={splits} paged={paged}")


@pytest.mark.parametrize("D,N,P,splits", [(128, 8, [0, 5], 0), (64, 17, [24, 3], 0), (128, 60, [333, 40], 3)])
def test_log_sum_exp_is_of_fp32_weights(sv, oracle, D, N, P, splits):
    """The sum of a row's weights is taken before they are packed to bf16 for the product with V.  Bound: scores are
    fp32 sums of exact products and at most ~10 here (2^-24 x D terms: under 1e-5), fp32 sums of the weights and
    exp2 / log2 add a few 2^-24 each; a sum of bf16 weights is off by up to 2^-9 over the root of the key count."""
    from gpu_util import random_case
    case = random_case(7100 + D + N, "bf16", B=2, Hq=4, Hkv=4, D=D, N_max=N, P_list=P, num_nodes=None, paged=False, cap_extra=0)
    plan = plan_of_case(case, splits)
    assert plan.block_rows and not plan.columns
    _, lse, _, ref = run_both(sv, oracle, case, num_splits=splits)
    assert abs(lse - ref).max() <= 3e-5
