"""A NaN that a row really meets stays one: in K of a key the row sees, or in the row's query, the row is NaN; in K of a
tree node, rows that do not see the node are as without it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


@pytest.mark.parametrize("dtype,B,H,D,N,P,splits", [
    ("bf16", 1, 2, 128, 20, 70, 1),           # workgroups of 16 or 32 query rows, one key range
    ("bf16", 2, 32, 128, 60, 200, 0),
    ("bf16", 1, 4, 64, 33, 900, 3),           # ... and partial results
    ("bf16", 1, 32, 128, 60, 3300, 0),        # key ranges only
    ("bf16", 8, 16, 64, 40, 1500, 2),
    ("f32", 1, 2, 64, 20, 70, 0),
])
@pytest.mark.parametrize("where", ["prefix", "node", "query"])
@pytest.mark.parametrize("paged", [False, True])
def test_nan(sv, oracle, dtype, B, H, D, N, P, splits, where, paged):
    from gpu_util import TOL, i32, random_case, to_dev, to_host_f64
    import workloads as W
    case = random_case(9300 + H + N, dtype, B=B, Hq=H, Hkv=H, D=D, N_max=N, P_list=[P] * B, paged=paged, depth=5)
    b, h = B - 1, H - 1
    check = slice(max(0, h - 1), H)                               # the head with the NaN and one without
    kv = slice(max(0, h - 1), H)
    ref = oracle.tree_attn(case["q"][b:, :, check], case["k"][:, kv] if paged else case["k"][b:, kv], case["v"][:, kv] if paged else case["v"][b:, kv],
                           case["prefix_len"][b:], case["parent"][b:], None,
                           block_table=None if not paged else case["block_table"][b:])[0][0]
    nan = W.NAN_BITS_BF16 if dtype == "bf16" else np.float32(np.nan)
    node = N // 3
    if where == "query":
        case["q"][b, node, h, 5] = nan
    else:
        slot = P // 2 if where == "prefix" else P + node
        row = (b, h, slot) if not paged else (case["block_table"][b, slot // 16], h, slot % 16)
        case["k"][row][7] = nan
    got = sv.specvlm_tree_verify_attn(to_dev(case["q"]), to_dev(case["k"]), to_dev(case["v"]), i32(case["prefix_len"]), i32(case["parent"]),
                                      block_table=None if not paged else i32(case["block_table"]), num_splits=splits)
    got = to_host_f64(got[b, :, check])
    parent, hit = case["parent"][b], np.zeros(N, dtype=bool)
    for i in range(N):
        t = i
        while t >= 0 and t != node:
            t = parent[t]
        hit[i] = {"prefix": True, "node": t == node, "query": i == node}[where]
    assert np.all(np.isnan(got[hit, -1]))
    assert np.all(np.abs(got[~hit, -1] - ref[~hit, -1]) <= TOL[dtype][0])
    assert np.all(np.abs(got[:, 0] - ref[:, 0]) <= TOL[dtype][0])
