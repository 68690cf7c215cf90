"""What an ordinary batch does not show of the kernel with a key stream per wavefront: NaN, a softmax reference that keeps moving, an
explicit scale, tensors that are not dense, a reused workspace, replays of a captured call, bad requests on a paged cache."""
import numpy as np
import pytest
import torch

import test_gpu_attn_nan
from attn_plan_util import division_of
from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


# key ranges: requests, query heads, KV heads, head size, nodes, prefix lengths (longest prefix + nodes: a multiple of 16).  BY_LENGTH: ranges
# of the shape that the lengths divide.
SHAPES = {
    1: (5, 32, 32, 128, 60, [420, 33, 250, 0, 419]),
    2: (3, 32, 16, 128, 64, [2304, 5, 511]),
    3: (5, 16, 16, 64, 60, [3028, 700, 64, 1, 2000]),
    4: (3, 20, 20, 128, 60, [2500, 100, 900]),
}
BY_LENGTH = 2


def make(ranges, paged=False, num_nodes=None):
    from gpu_util import random_case
    B, Hq, Hkv, D, N, P = SHAPES[ranges]
    case = random_case(8600 + ranges, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=num_nodes, paged=paged, cap_extra=0)
    cap = case["block_table"].shape[1] * 16 if paged else case["k"].shape[2]
    assert division_of(B, Hq, Hkv, D, N, cap, paged=paged) == (ranges, ranges == BY_LENGTH)
    return case


def device_args(case):
    from gpu_util import i32, to_dev
    table = None if case["block_table"] is None else i32(case["block_table"])
    return [to_dev(case[x]) for x in "qkv"] + [i32(case["prefix_len"]), i32(case["parent"])], table


@pytest.mark.parametrize("B,H,D,P,ranges,by_length", [(5, 32, 128, 413, 1, 0), (5, 32, 64, 413, 1, 0), (3, 20, 128, 2490, 4, 0), (2, 40, 128, 3741, 3, 1)])
@pytest.mark.parametrize("where", ["prefix", "node", "query"])
@pytest.mark.parametrize("paged", [False, True])
def test_nan(sv, oracle, B, H, D, P, ranges, by_length, where, paged):
    cap = ((P + 60 + 15) // 16 + 1) * 16 if paged else (P + 60 + 7 + 7) // 8 * 8
    assert division_of(B, H, H, D, 60, cap, paged=paged) == (ranges, by_length)
    test_gpu_attn_nan.test_nan(sv, oracle, "bf16", B, H, D, 60, P, 0, where, paged)


def scaled(bits, factor):
    """bf16 bit patterns times a factor, NaN as they were."""
    x = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).float() * torch.from_numpy(factor)
    y = x.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    return np.where(np.isnan(x.numpy()), bits, y)


@pytest.mark.parametrize("ranges", [1, 2, 3, 4])
@pytest.mark.parametrize("rising", [True, False])
def test_reference_moves(sv, oracle, ranges, rising):
    """Scores up to ~40 that grow along the cache, so that the reference moves in many tiles, or fall.  V is halved: a weight, a
    partial result and the output round to 2^-9 each, of values up to 2.5 then: 1.5e-2 where a row sees little else."""
    case = make(ranges)
    slots = case["k"].shape[2]
    growth = np.linspace(0.1, 8.0, slots, dtype=np.float32)[:: 1 if rising else -1]
    case["k"] = scaled(case["k"], growth.copy()[None, None, :, None])
    case["v"] = scaled(case["v"], np.full(1, 0.5, dtype=np.float32))
    check(case, *run_both(sv, oracle, case), f"moving reference, ranges {ranges}")


@pytest.mark.parametrize("ranges", [1, 2, 3, 4])
@pytest.mark.parametrize("scale", [0.02, 0.2])
def test_explicit_scale(sv, oracle, ranges, scale):
    case = make(ranges, paged=ranges % 2 == 0)
    check(case, *run_both(sv, oracle, case, scale=scale), f"scale {scale}, ranges {ranges}")


@pytest.mark.parametrize("ranges", [1, 2, 3, 4])
@pytest.mark.parametrize("paged", [False, True])
def test_tensors_that_are_not_dense(sv, ranges, paged):
    """The same call with q, o, K and V inside larger tensors: bit for bit, and nothing around o is written."""
    case = make(ranges, paged)
    (q, k, v, P, par), table = device_args(case)
    plain = sv.specvlm_tree_verify_attn(q, k, v, P, par, block_table=table)
    fused = torch.zeros((q.shape[0], q.shape[1], 3) + tuple(q.shape[2:]), dtype=q.dtype, device="cuda")
    fused[:, :, 1] = q
    wide = torch.zeros(k.shape[:3] + (2 * k.shape[3],), dtype=k.dtype, device="cuda")
    wide[..., :k.shape[3]] = k
    wide[..., k.shape[3]:] = v
    out = torch.full_like(fused, 7.0)
    sv.specvlm_tree_verify_attn(fused[:, :, 1], wide[..., :k.shape[3]], wide[..., k.shape[3]:], P, par, block_table=table, out=out[:, :, 2])
    assert torch.equal(out[:, :, 2], plain)
    assert bool((out[:, :, :2] == 7.0).all())


@pytest.mark.parametrize("ranges", [1, 2, 3, 4])
@pytest.mark.parametrize("paged", [False, True])
def test_workspace_and_replays(sv, ranges, paged):
    """Replays of a captured call, with eager calls on the same workspace between them, give the eager result bit for bit, and
    the counters are zero after each."""
    case = make(ranges, paged)
    (q, k, v, P, par), table = device_args(case)
    out = torch.zeros_like(q)
    desc = sv.binding.make_attn_desc(q, k, out, block_table=table)
    ws = torch.zeros(max(256, sv.specvlm_tree_verify_attn_workspace_bytes(desc)), dtype=torch.uint8, device="cuda")
    counters = ws[:1024 * 4 * 128] if ranges > 1 else ws
    call = lambda o: sv.specvlm_tree_verify_attn(q, k, v, P, par, block_table=table, out=o, workspace=ws, desc=desc)
    eager = torch.zeros_like(q)
    call(eager)
    assert not counters.any()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(out)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out)
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager) and not counters.any()
        again = torch.zeros_like(q)
        call(again)
        torch.cuda.synchronize()
        assert torch.equal(again, eager) and not counters.any()


@pytest.mark.parametrize("ranges", [1, 2, 3, 4])
def test_bad_requests_paged(sv, oracle, ranges):
    """A malformed tree and a length past the table set the error word and leave their requests' rows alone."""
    from gpu_util import assert_attn_close, i32, to_host_f64
    B, _, _, _, N, _ = SHAPES[ranges]
    case = make(ranges, paged=True)
    (q, k, v, _, _), table = device_args(case)
    parent, lengths = case["parent"].copy(), case["prefix_len"].copy()
    parent[1, 7] = 7
    lengths[2] = case["block_table"].shape[1] * 16 - N + 1
    out, err = torch.full_like(q, 7.0), torch.zeros(1, dtype=torch.int32, device="cuda")
    sv.specvlm_tree_verify_attn(q, k, v, i32(lengths), i32(parent), block_table=table, out=out, err_flag=err)
    assert int(err.item()) == 1 | 4
    got = to_host_f64(out)
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None, block_table=case["block_table"])
    good = [b for b in range(B) if b not in (1, 2)]
    assert_attn_close(got[good], ref[good], "bf16", "good requests")
    assert np.all(got[1:3] == 7.0)
