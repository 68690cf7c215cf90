"""A prefix length that no cache holds, in every attention kernel: reported, the request's output left alone, the other requests' as
without it.  From 2^31 - nodes on prefix and nodes do not fit in 32 bits together."""
import numpy as np
import pytest
import torch

from attn_plan_util import columns_of, plan_of

pytestmark = pytest.mark.gpu

# requests, query heads, KV heads, head size, nodes, slots, key ranges asked for; what the plan must be
KERNELS = {
    "rows_16": ((2, 16, 16, 128, 60, 272, 0), dict(block_rows=16, splits=1)),
    "rows_32": ((2, 16, 16, 128, 60, 1024, 0), dict(block_rows=32, splits=4)),
    "rows_16_d64": ((2, 8, 4, 64, 40, 512, 0), dict(block_rows=16, splits=1)),
    "ranges": ((2, 16, 16, 128, 60, 640, 8), dict(block_rows=0, splits=8)),
    "ranges_two_workgroups": ((2, 72, 72, 128, 60, 640, 3), dict(block_rows=0, splits=3)),
    "streams": ((4, 40, 40, 128, 60, 736, 0), dict(block_rows=0, splits=1)),
    "fp32": ((2, 4, 4, 64, 20, 160, 0), None),
    "vector_alu": ((2, 4, 4, 128, 20, 160, 0), None),
}


@pytest.mark.parametrize("kernel", list(KERNELS))
@pytest.mark.parametrize("paged", [False, True])
def test_length_no_cache_holds(kernel, paged):
    import paper_2509_11815_amd as sv
    from gpu_util import i32, random_case, to_dev
    sv.load_library()
    (B, Hq, Hkv, D, N, cap, splits), plan = KERNELS[kernel]
    if plan:
        p = plan_of(B, Hq, Hkv, D, N, cap, splits, paged)
        assert (p.block_rows, p.splits) == (plan["block_rows"], plan["splits"])
        assert bool(columns_of(B, Hq, Hkv, D, N, cap, num_splits=splits, paged=paged).columns) == (kernel == "streams")
    case = random_case(17, "f32" if kernel == "fp32" else "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N,
                       P_list=[cap - N - 16 * paged] * B, paged=paged, cap_extra=0)
    q, k, v = (to_dev(case[x]) for x in "qkv")
    table = None if case["block_table"] is None else i32(case["block_table"])
    parent = i32(case["parent"])

    def call(lengths):
        out, lse, err = torch.full_like(q, 7.0), torch.full((B, Hq, N), 7.0, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        if kernel == "vector_alu":
            sv.specvlm_tree_verify_attn_vector_alu(q, k, v, i32(lengths), parent, block_table=table, out=out, lse=lse, err_flag=err)
            return out, lse, int(err.item())
        desc = sv.binding.make_attn_desc(q, k, out, block_table=table, num_splits=splits)
        workspace = torch.zeros(max(256, sv.specvlm_tree_verify_attn_workspace_bytes(desc)), dtype=torch.uint8, device="cuda")
        sv.specvlm_tree_verify_attn(q, k, v, i32(lengths), parent, block_table=table, out=out, lse=lse, workspace=workspace, err_flag=err, desc=desc)
        assert not workspace[:1024 * 4 * 128].any()
        return out, lse, int(err.item())

    good = case["prefix_len"]
    out, lse, err = call(good)
    assert err == 0
    for length in (cap - N + 1, cap, -1, -2**31, 2**31 - 1, 2**31 - N, 2**31 - N - 1):
        lengths = np.array(good)
        lengths[0] = length
        bad_out, bad_lse, err = call(lengths)
        assert err == 4, length
        assert bool((bad_out[0] == 7.0).all()) and bool((bad_lse[0] == 7.0).all()), length
        assert torch.equal(bad_out[1:], out[1:]) and torch.equal(bad_lse[1:], lse[1:]), length
