"""Split calls with more than half as many (request, head) pairs as there are ticket counter lines: the two counters of a query
block (head size 128; 64 has one) share a line.  The counters are zero again after every call."""
import pytest

from attn_plan_util import Plan, plan_of_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,B,H", [(64, 9, 57), (128, 9, 57), (128, 16, 40), (64, 16, 32)])       # 513, 640 and (lines of their own) 512 pairs
def test_second_counters(oracle, D, B, H):
    import paper_2509_11815_amd as sv
    import torch
    import numpy as np
    from gpu_util import i32, random_case, to_dev, to_host_f64
    sv.load_library()
    case = random_case(8300 + D + H, "bf16", B=B, Hq=H, Hkv=H, D=D, N_max=60, P_list=[7 * b % 70 for b in range(B)])
    assert plan_of_case(case, 3) == Plan(3, 0, 3)
    q, k, v = (to_dev(case[x]) for x in "qkv")
    out = torch.zeros_like(q)
    desc = sv.binding.make_attn_desc(q, k, out, num_splits=3)
    ws = torch.zeros(sv.specvlm_tree_verify_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    counters = ws[:1024 * 4 * 128]
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None)
    for _ in range(2):
        out.zero_()
        sv.specvlm_tree_verify_attn(q, k, v, i32(case["prefix_len"]), i32(case["parent"]), out=out, workspace=ws, desc=desc)
        # bf16 rounds to 2^-8 relative at most: the output and the partials once each, and every weight (of values whose
        # weighted mean is under 3).  Rows of few keys have outputs up to 5, so the bound follows the output.
        err = np.abs(to_host_f64(out) - ref)
        assert np.all(err <= 2.0 ** -8 * (2 * np.abs(ref) + 3)) and err.mean() <= 2e-3
        assert not counters.any()
