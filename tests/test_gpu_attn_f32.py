"""GPU parity of the fp32 attention path at its edges: one node, a block of 16 nodes and one more, 64 nodes,
key counts around a 16-key tile and around one tile per wavefront, grouped heads, both layouts."""
import pytest

from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


@pytest.mark.parametrize("B,Hq,Hkv,D,N,P,nn", [
    (1, 1, 1, 64, 1, [0], None), (1, 2, 2, 128, 16, [0], None), (2, 2, 1, 64, 17, [14, 111], [17, 16]),
    (2, 4, 2, 128, 64, [64, 65], [64, 33]), (1, 8, 8, 64, 60, [900], None),
])
@pytest.mark.parametrize("paged", [False, True])
def test_fp32_edges(sv, oracle, B, Hq, Hkv, D, N, P, nn, paged):
    from gpu_util import random_case
    case = random_case(8100 + D + N, "f32", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=0)
    check(case, *run_both(sv, oracle, case), f"f32 {B}x{Hq}/{Hkv}x{D} N={N} paged={paged}")
