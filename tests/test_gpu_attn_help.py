"""GPU parity of attention calls with a column of workgroups a request, in which the shorter requests' workgroups read keys of the longest
one ahead: its last rounds short and full, more rounds than are read ahead, row blocks, node counts, a bad request as the longest and as a
helper, sixteen requests."""
import numpy as np
import pytest
import torch

from attn_plan_util import columns_of

pytestmark = pytest.mark.gpu

# requests, query heads, KV heads, nodes, slots per request
SHAPES = {"heads": (8, 32, 32, 60, 976), "five": (5, 48, 48, 60, 1264), "blocks": (7, 32, 8, 64, 912), "sixteen": (16, 16, 16, 60, 1024),
          "far": (8, 32, 32, 60, 2064)}


@pytest.mark.parametrize("name,prefix,num_nodes,bad", [
    ("heads", [170, 390, 253, 339, 350, 916, 365, 287], None, None),
    ("heads", [0, 64, 68, 69, 196, 836, 197, 0], None, None),          # rounds that end on a key, one key further, requests without a prefix
    ("heads", [100, 837, 300, 900, 120, 60, 90, 200], [60, 1, 33, 17, 60, 2, 59, 60], None),
    ("heads", [170, 390, 253, 339, 350, 300, 365, 287], None, (5, 5000)),        # a length that the cache does not hold counts as the whole cache
    ("heads", [170, 390, 253, 339, 350, 906, 365, 287], None, (0, -7)),
    ("five", [1204, 1000, 300, 400, 200], None, None),
    ("blocks", [848, 100, 200, 50, 120, 300, 90], None, None),
    ("sixteen", [964] + [40 * i for i in range(15)], None, None),
    ("far", [2004, 100, 300, 150, 120, 600, 90, 200], None, None),       # more rounds than are read ahead
])
def test_against_oracle(name, prefix, num_nodes, bad):
    import oracle
    import paper_2509_11815_amd as sv
    from gpu_util import TOL, i32, random_case, to_dev, to_host_f64
    sv.load_library()
    B, Hq, Hkv, N, cap = SHAPES[name]
    c = columns_of(B, Hq, Hkv, 128, N, cap)
    assert c.columns == B and not c.by_length
    case = random_case(7700 + len(prefix) + sum(prefix), "bf16", B=B, Hq=Hq, Hkv=Hkv, D=128, N_max=N, P_list=prefix, num_nodes=num_nodes, cap_extra=0)
    short = cap - case["k"].shape[2]
    k, v = (torch.nn.functional.pad(to_dev(case[x]), (0, 0, 0, short), value=float("nan")) for x in "kv")
    q, P = to_dev(case["q"]), np.array(case["prefix_len"])
    if bad:
        P[bad[0]] = bad[1]
    nn = None if num_nodes is None else i32(case["num_nodes"])
    out, err = torch.full_like(q, 7.0), torch.zeros(1, dtype=torch.int32, device="cuda")
    for _ in range(2):                                                   # twice on one workspace
        sv.specvlm_tree_verify_attn(q, k, v, i32(P), i32(case["parent"]), num_nodes=nn, out=out, err_flag=err)
    assert int(err.item()) == (4 if bad else 0)
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], num_nodes=case["num_nodes"])
    got = to_host_f64(out)
    for b in range(B):
        n = N if num_nodes is None else num_nodes[b]
        if bad and b == bad[0]:
            assert np.all(got[b] == 7.0)
            continue
        diff = np.abs(got[b, :n] - ref[b, :n])
        assert diff.max() <= TOL["bf16"][0] and diff.mean() <= TOL["bf16"][1], (b, diff.max(), diff.mean())
