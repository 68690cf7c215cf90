"""A level with its selection, a row's log-sum-exp in a workgroup of its own: where that begins and ends (rows at any alignment,
every row division, one row, 31 and 32 rows, the most rows of a call and one more), bit for bit against the separate calls
(specvlm_draft_topk, then specvlm_draft_select over its scores), which add up and rank in one workgroup a row."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def same(a, b):
    if a is None or b is None:                                                   # (no parents given, none written)
        return a is b
    bits = lambda t: t.view(torch.int32) if t.dtype == torch.float32 else t      # a NaN equals itself
    return torch.equal(bits(a), bits(b))


def level(dtype, B, W, V, offset=0, seed=0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + V + 31 * W + B)
    flat = torch.empty(offset + B * W * V, device="cuda").normal_(0.0, 2.0, generator=gen).to(dtype)
    x = flat[offset:].view(B, W, V)
    if W > 2:
        x[:, 1] = x[:, 0]                                                        # equal scores across rows
        x[:, 2, : V // 2] = -torch.inf
    cum = -torch.rand((B, W), device="cuda", generator=gen)
    if W > 2:
        cum[:, 1] = cum[:, 0]
        cum[:, W - 1] = -torch.inf
    return x, cum, torch.randint(0, 500, (B, W), dtype=torch.int32, device="cuda", generator=gen)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,W,V,K,offset", [(1, 10, 10, 10, 0), (2, 10, 32768, 10, 0), (1, 10, 32769, 10, 1), (1, 3, 65536, 64, 0), (1, 3, 65537, 10, 3),
                                            (1, 1, 65537, 10, 0), (2, 1, 9000, 10, 5), (1, 31, 4001, 33, 0), (1, 32, 4001, 32, 0), (16, 8, 2047, 7, 1),
                                            (43, 3, 2047, 7, 1), (7, 10, 31500, 10, 0), (1, 2, 200003, 5, 7),
                                            (12, 10, 2047, 7, 1), (11, 11, 2047, 7, 1), (11, 10, 65537, 10, 0), (37, 3, 65537, 5, 0), (5, 10, 65537, 10, 3),
                                            (17, 3, 65537, 10, 1)])
def test_equals_the_separate_calls(sv, dtype, B, W, V, K, offset):
    x, cum, par = level(dtype, B, W, V, offset)
    counters = torch.zeros(B * sv.binding.COUNTER_STRIDE, dtype=torch.int32, device="cuda")
    counters_left = counters.clone()
    for c, p in ((cum, par), (None, None)):
        lse = torch.zeros((B, W), device="cuda")
        score, token, parent = sv.specvlm_draft_topk(x, K, cum=c, parent_idx=p, lse_out=lse)
        for M in (W, 2 * K + 1):
            want = (score, token, parent) + tuple(sv.specvlm_draft_select(score, M, index_base=9))
            got_lse = torch.zeros((B, W), device="cuda")
            got = sv.specvlm_draft_topk_select(x, K, M, cum=c, parent_idx=p, lse_out=got_lse, index_base=9, counters=counters)
            for g, w in zip(got, want):
                assert same(g, w), (M, c is None)
            assert same(got_lse, lse)
            assert torch.equal(counters, counters_left)


def test_in_place_and_replayed(sv):
    """A program keeps one pair of tensors for what a level expands and what it selects; the call is captured and replayed with
    eager calls in between."""
    B, W, V, K = 2, 10, 32000, 10
    x, cum, par = level(torch.bfloat16, B, W, V)
    counters = torch.zeros(B * sv.binding.COUNTER_STRIDE, dtype=torch.int32, device="cuda")
    want = sv.specvlm_draft_topk_select(x, K, W, cum=cum, parent_idx=par, counters=counters)
    sel, val = par.clone(), cum.clone()
    got = sv.specvlm_draft_topk_select(x, K, W, cum=val, parent_idx=sel, sel_out=sel, sel_score_out=val, counters=counters)
    for g, w in zip(got, want):
        assert same(g, w)
    out = [torch.zeros_like(t) for t in want]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    call = lambda: sv.specvlm_draft_topk_select(x, K, W, cum=cum, parent_idx=par, score_out=out[0], token_out=out[1], parent_out=out[2],
                                                sel_out=out[3], sel_score_out=out[4], count_out=out[5], counters=counters)
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for seed in (1, 2, 3):
        x2, cum2, par2 = level(torch.bfloat16, B, W, V, seed=seed)
        x.copy_(x2), cum.copy_(cum2), par.copy_(par2)
        graph.replay()
        torch.cuda.synchronize()
        eager = sv.specvlm_draft_topk_select(x, K, W, cum=cum, parent_idx=par, counters=counters)
        for g, w in zip(out, eager):
            assert same(g, w)
        assert not counters.any()
