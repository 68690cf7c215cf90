"""Calls on an explicit stream, with everything omitted that may be omitted: what the call allocates and zeroes is ordered
before its kernels, and is not handed to another stream's work while they run."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def attention(sv, rng, stream):
    q = rng(1, 60, 8, 128).bfloat16()
    k, v = (rng(1, 8, 3400, 128).bfloat16() for _ in range(2))
    P, parent = torch.tensor([3300], device="cuda", dtype=torch.int32), torch.arange(-1, 59, device="cuda", dtype=torch.int32)[None]
    nodes = torch.tensor([57], device="cuda", dtype=torch.int32)
    return lambda: sv.specvlm_tree_verify_attn(q, k, v, P, parent, num_nodes=nodes, num_splits=4, stream=stream)


def argmax_accept(sv, rng, stream):
    logits = rng(2, 60, 4000)
    parent = torch.arange(-1, 59, device="cuda", dtype=torch.int32)[None].repeat(2, 1)
    tok = torch.zeros(2, 60, device="cuda", dtype=torch.int32)
    return lambda: sv.specvlm_node_argmax_accept(logits, parent, tok, path_cap=8, stream=stream)


def topk_select(sv, rng, stream):
    logits = rng(2, 10, 4000)
    return lambda: sv.specvlm_draft_topk_select(logits, 10, 10, stream=stream)


def head(sv, rng, stream):
    hidden, weight = rng(2, 60, 512).bfloat16(), rng(3000, 512).bfloat16()
    return lambda: sv.specvlm_head_argmax(hidden, weight, stream=stream)


def pool(sv, rng, stream):
    x, n = rng(2, 100, 64), torch.tensor([100, 30], device="cuda", dtype=torch.int32)
    return lambda: sv.specvlm_visual_pool(x, 4, num_tokens=n, stream=stream)


@pytest.mark.parametrize("make", [attention, argmax_accept, topk_select, head, pool])
def test_explicit_stream(sv, make):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    rng = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    side = torch.cuda.Stream()
    call = make(sv, rng, side)
    items = lambda got: [t for t in (got if isinstance(got, tuple) else (got,)) if t is not None]
    gen.manual_seed(5)
    expect = [t.clone() for t in items(make(sv, rng, None)())]
    torch.cuda.synchronize()
    # cached blocks that are not zero, of both streams; then work on the current stream that takes a while
    for s in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(s):
            junk = [torch.full((n,), 0x55, device="cuda", dtype=torch.uint8) for n in (512, 4096, 1 << 20, 4 << 20, 16 << 20, 48 << 20)]
            del junk
    torch.cuda.synchronize()
    a = torch.randn(4096, 4096, device="cuda")
    b = a
    for _ in range(40):
        b = a @ a
    got = items(call())
    side.synchronize()
    with torch.cuda.stream(side):
        first = [t.clone() for t in got]
    side.synchronize()
    torch.cuda.synchronize()
    again = items(call())                              # ... and into blocks that were given back
    torch.cuda.synchronize()
    assert torch.cuda.current_stream() != side
    for e, f, g, h in zip(expect, first, got, again):
        assert torch.equal(e, f) and torch.equal(e, g) and torch.equal(e, h)


def test_default_stream_and_external_stream_handles(sv):
    x = torch.randn(1, 8, 64, device="cuda")
    want = x.view(1, 4, 2, 64).mean(2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for stream in (torch.cuda.default_stream(), torch.cuda.ExternalStream(side.cuda_stream), torch.cuda.current_stream()):
        with torch.cuda.stream(side):
            got, _ = sv.specvlm_visual_pool(x, 2, stream=stream)
            assert torch.cuda.current_stream() == side
        torch.cuda.synchronize()
        torch.testing.assert_close(got, want, rtol=1e-6, atol=1e-6)
