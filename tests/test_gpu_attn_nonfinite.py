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


@pytest.mark.parametrize("D", [64, 128])
def test_prefix_beside_a_node(sv, oracle, D):
    """An infinity in the prefix reaches every row, the NaN of a node in the same tile only those that see it."""
    from gpu_util import i32, random_case, to_dev
    N, P, node = 24, 37, 5
    case = random_case(9300 + D, "f32", B=1, Hq=2, Hkv=2, D=D, N_max=N, P_list=[P], paged=False)
    ref = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None)[0][0]
    case["v"][0, :, P - 1, 7] = np.inf
    case["v"][0, :, P + node, 9] = np.nan
    got = sv.specvlm_tree_verify_attn(to_dev(case["q"]), to_dev(case["k"]), to_dev(case["v"]), i32(case["prefix_len"]),
                                      i32(case["parent"])).cpu().numpy()[0]
    below = np.zeros(N, dtype=bool)
    for i in range(N):
        below[i] = i == node or (i > 0 and below[case["parent"][0][i]])
    assert np.all(got[:, :, 7] == np.inf)
    assert np.array_equal(np.isnan(got[:, :, 9]), np.repeat(below[:, None], 2, axis=1))
    rest = np.ones(D, dtype=bool)
    rest[[7, 9]] = False
    np.testing.assert_allclose(got[:, :, rest], ref[:, :, rest], rtol=0, atol=1e-5)
    np.testing.assert_allclose(got[~below][:, :, 9], ref[~below][:, :, 9], rtol=0, atol=1e-5)
