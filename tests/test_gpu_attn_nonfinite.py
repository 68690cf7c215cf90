"""fp32 attention: what a node does not see does not reach it, also where that is not a finite number."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


@pytest.mark.parametrize("D,N,P,nodes", [(64, 8, 21, [3]), (128, 40, 30, [1, 17, 39]), (64, 64, 0, [5, 63]), (128, 20, 150, [19, 2])])
@pytest.mark.parametrize("bad", [float("inf"), -float("inf"), float("nan")])
@pytest.mark.parametrize("paged", [False, True])
def test_invisible_values_do_not_leak(sv, oracle, D, N, P, nodes, bad, paged):
    from gpu_util import i32, random_case, to_dev
    case = random_case(9100 + D + N, "f32", B=1, Hq=2, Hkv=1, D=D, N_max=N, P_list=[P], paged=paged)
    ref = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None,
                           block_table=case["block_table"])[0][0]
    columns = [0, D // 2 + 3, D - 1]                                    # some dimensions of the row only
    for n in nodes:
        slot = P + n
        row = (0, 0, slot) if not paged else (case["block_table"][0, slot // 16], 0, slot % 16)
        case["v"][row][columns] = bad
    table = None if not paged else i32(case["block_table"])
    got = sv.specvlm_tree_verify_attn(to_dev(case["q"]), to_dev(case["k"]), to_dev(case["v"]), i32(case["prefix_len"]),
                                      i32(case["parent"]), block_table=table).cpu().numpy()[0]
    parent = case["parent"][0]
    for i in range(N):
        seen, t = set(), i
        while t >= 0:
            seen.add(t)
            t = parent[t]
        hit = np.zeros(D, dtype=bool)
        if seen & set(nodes):
            hit[columns] = True
        np.testing.assert_allclose(got[i][:, ~hit], ref[i][:, ~hit], rtol=0, atol=1e-5)
        if np.isnan(bad):
            assert np.all(np.isnan(got[i][:, hit]))
        else:
            assert np.all(got[i][:, hit] == bad)
