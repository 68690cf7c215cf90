"""GPU parity of the attention calls whose workgroups are dealt out to the requests by their lengths: equal lengths, one request with
most of the columns, columns left over, requests without a prefix, node counts, partial results in bf16 and fp32, more than four ranges
of a request, bad requests beside good ones, replays, a workspace that does not hold the partial results."""
import numpy as np
import pytest
import torch

from attn_plan_util import columns_of, plan_of

pytestmark = pytest.mark.gpu

# requests, query heads, KV heads, head size, nodes; slots per request; the call's key ranges without (1: partial results in fp32)
SHAPES = {
    "bf16": ((3, 32, 16, 128, 60, 2416), 2),
    "fp32": ((6, 32, 32, 128, 60, 1168), 1),
    "rows": ((4, 35, 5, 128, 48, 2064), 1),
    "d64": ((6, 16, 8, 64, 64, 5200), None),
    "few": ((16, 4, 4, 128, 60, 3504), None),              # 16 requests, 64 columns
    "heads": ((4, 32, 8, 128, 64, 2416), None),
}


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def make(name, fractions, num_nodes=None, paged=False, seed=9100):
    """Prefix lengths as fractions of the longest possible."""
    from gpu_util import random_case
    (B, Hq, Hkv, D, N, cap), splits = SHAPES[name]
    c, plan = columns_of(B, Hq, Hkv, D, N, cap, paged=paged), plan_of(B, Hq, Hkv, D, N, cap, paged=paged)
    assert c.by_length and (splits is None or plan.splits == splits)
    f = (list(fractions) * B)[:B]
    room = cap - 16 * paged                                # (a paged case's table has a block more than its requests fill)
    P = [int(x * (room - N)) for x in f]
    P[int(np.argmax(f))] = room - N
    nn = None if num_nodes is None else [max(1, min(N, n)) for n in (list(num_nodes) * B)[:B]]
    if nn is not None:
        nn[int(np.argmax(f))] = N
    case = random_case(seed, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, num_nodes=nn, paged=paged, cap_extra=0)
    assert (case["block_table"].shape[1] * 16 if paged else case["k"].shape[2]) == cap
    return case


def call(sv, case, workspace=None, lse=None):
    from gpu_util import i32, to_dev
    q, k, v = (to_dev(case[x]) for x in "qkv")
    table = None if case["block_table"] is None else i32(case["block_table"])
    nn = None if case["num_nodes"] is None else i32(case["num_nodes"])
    out, err = torch.full_like(q, 7.0), torch.zeros(1, dtype=torch.int32, device="cuda")
    desc = sv.binding.make_attn_desc(q, k, out, block_table=table)
    if workspace is None:
        workspace = torch.zeros(sv.specvlm_tree_verify_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    sv.specvlm_tree_verify_attn(q, k, v, i32(case["prefix_len"]), i32(case["parent"]), num_nodes=nn, block_table=table,
                                out=out, lse=lse, workspace=workspace, err_flag=err, desc=desc)
    return out, err, workspace


def close(oracle, case, out, what):
    from gpu_util import assert_attn_close, to_host_f64, valid_rows_mask
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], case["num_nodes"], block_table=case["block_table"])
    B, N = case["q"].shape[:2]
    rows = valid_rows_mask(B, N, case["num_nodes"])
    assert_attn_close(to_host_f64(out)[rows], ref[rows], "bf16", what)


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("fractions", [
    (1, 1, 1),                             # even shares
    (1, 0, 0.01),                          # one request has up to eight ranges, the rest one; columns too many
    (0.3, 1, 0.55, 0.1),
    (0.45, 0.5, 1),
    (1, 0, 0.36, 0.01),                    # the shortest length that fits is not among the first tried
], ids=["equal", "one", "mixed", "two_long", "steps"])
@pytest.mark.parametrize("paged", [False, True])
def test_lengths(sv, oracle, name, fractions, paged):
    (B, _, _, _, N, _), _ = SHAPES[name]
    case = make(name, fractions, None if fractions[0] == 1 else [N, 1, 33, N - 1, 7], paged)
    out, err, workspace = call(sv, case)
    assert int(err.item()) == 0 and not workspace[:1024 * 4 * 128].any()
    close(oracle, case, out, f"{name} {fractions}")


@pytest.mark.parametrize("name", ["bf16", "fp32"])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("length", ["slots", -5, -2**31, 2**31 - 1, 2**31 - 60, 2**31 - 61])
def test_bad_requests_beside_good_ones(sv, oracle, name, paged, length):
    """A malformed tree and a length that no cache holds take their share of the columns and are left alone: prefix and nodes of the
    largest ones do not fit in 32 bits together."""
    from gpu_util import assert_attn_close, to_host_f64
    case = make(name, (0.4, 0.6, 1, 0.5, 0.2, 0.7), paged=paged)
    B, cap = case["q"].shape[0], SHAPES[name][0][5]
    parent, lengths = case["parent"].copy(), case["prefix_len"].copy()
    parent[1, 7] = 7
    lengths[0] = cap if length == "slots" else length
    good = list(range(2, B))
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None, block_table=case["block_table"])
    out, err, workspace = call(sv, dict(case, parent=parent, prefix_len=lengths))
    assert int(err.item()) == 1 | 4 and not workspace[:1024 * 4 * 128].any()
    got = to_host_f64(out)
    assert_attn_close(got[good], ref[good], "bf16", "good requests")
    assert np.all(got[:2] == 7.0)


@pytest.mark.parametrize("name", ["bf16", "fp32"])
@pytest.mark.parametrize("nodes", [0, -1, 61, 2**31 - 1, -2**31])
def test_bad_node_counts_beside_good_ones(sv, oracle, name, nodes):
    from gpu_util import assert_attn_close, to_host_f64
    case = make(name, (0.4, 1, 0.6, 0.5, 0.2, 0.7))
    B, N = case["q"].shape[:2]
    good = list(range(1, B))
    ref, _ = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None)
    counts = np.full(B, N, dtype=np.int32)
    counts[0] = nodes
    out, err, workspace = call(sv, dict(case, num_nodes=counts))
    assert int(err.item()) == 2 and not workspace[:1024 * 4 * 128].any()
    got = to_host_f64(out)
    assert_attn_close(got[good], ref[good], "bf16", "good requests")
    assert np.all(got[0] == 7.0)


@pytest.mark.parametrize("name", list(SHAPES))
def test_replays(sv, name):
    """Replays of a captured call whose lengths change between them, as an eager call on the same workspace."""
    from gpu_util import i32, to_dev
    case = make(name, (1, 1, 1))
    shares = np.array([1, 0.2, 0.6, 0, 0.9])
    q, k, v = (to_dev(case[x]) for x in "qkv")
    P, par, out = i32(case["prefix_len"]), i32(case["parent"]), torch.zeros_like(q)
    desc = sv.binding.make_attn_desc(q, k, out)
    ws = torch.zeros(sv.specvlm_tree_verify_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    run = lambda o: sv.specvlm_tree_verify_attn(q, k, v, P, par, out=o, workspace=ws, desc=desc)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(out)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(out)
    for turn in range(4):
        P.copy_(i32((case["prefix_len"] * shares[(np.arange(len(P)) + turn) % 5]).astype(np.int32)))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        eager = torch.zeros_like(q)
        run(eager)
        torch.cuda.synchronize()
        assert torch.equal(out, eager) and not ws[:1024 * 4 * 128].any()


@pytest.mark.parametrize("name", ["bf16", "fp32", "rows"])
def test_workspaces(sv, oracle, name):
    """Less workspace than the library asks for, where the call does without: none, and one that is short or not aligned; the static
    array gives what a whole workspace does."""
    from gpu_util import i32, to_dev
    case = make(name, (0.3, 1, 0.55, 0.1))
    B, Hq, Hkv, D, N, cap = SHAPES[name][0]
    c = columns_of(B, Hq, Hkv, D, N, cap)
    out, _, _ = call(sv, case)
    q, k, v = (to_dev(case[x]) for x in "qkv")
    static = torch.full_like(q, 7.0)
    sv.specvlm_tree_verify_attn_static(q, k, v, i32(case["prefix_len"]), i32(case["parent"]), out=static)
    assert torch.equal(static, out)
    if c.even_bytes < c.bytes:
        short, _, _ = call(sv, case, workspace=torch.zeros(max(256, c.even_bytes), dtype=torch.uint8, device="cuda"))
        close(oracle, case, short, "short workspace")
    if c.even_bytes == 0:
        without = torch.full_like(q, 7.0)
        sv.specvlm_tree_verify_attn(q, k, v, i32(case["prefix_len"]), i32(case["parent"]), out=without)
        off = torch.zeros(c.bytes + 512, dtype=torch.uint8, device="cuda")[128:]
        misaligned, _, _ = call(sv, case, workspace=off)
        assert torch.equal(without, short) and torch.equal(misaligned, short) and not off.any()
    else:
        with pytest.raises(sv.SpecvlmError, match="WORKSPACE_TOO_SMALL"):
            call(sv, case, workspace=torch.zeros(c.even_bytes - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("name,fractions", [("bf16", (1, 0, 0.01)), ("fp32", (1, 0.3, 0.1)), ("d64", (1, 0.05, 0.05))])
def test_log_sum_exp(sv, oracle, name, fractions):
    from gpu_util import to_host_f64
    case = make(name, fractions)
    B, N, H, _ = case["q"].shape
    lse = torch.full((B, H, N), 7.0, dtype=torch.float32, device="cuda")
    call(sv, case, lse=lse)
    _, ref = oracle.tree_attn(case["q"], case["k"], case["v"], case["prefix_len"], case["parent"], None)
    assert np.abs(to_host_f64(lse) - ref).max() <= 1e-4              # weights are summed in fp32: 1.2e-6 seen
