"""What the Python binding accepts: numbers that int() and float() take, arguments that a given `out` makes irrelevant."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def walk_inputs():
    parent = torch.tensor([[-1, 0, 1, 0]], dtype=torch.int32, device="cuda")
    tok = torch.tensor([[9, 3, 5, 4]], dtype=torch.int32, device="cuda")
    logits = torch.zeros(1, 4, 100, dtype=torch.float32, device="cuda")
    for node, best in enumerate((3, 5, 7, 8)):
        logits[0, node, best] = 30.0
    return parent, tok, logits


def walk_outputs(cap=3):
    one = lambda *shape: torch.full(shape, -7, dtype=torch.int32, device="cuda")
    return [one(1), one(1, cap), one(1), one(1, cap)]


@pytest.mark.parametrize("call", ["tree_accept", "node_argmax_accept", "tree_accept_sample"])
def test_a_given_out_decides_the_path_capacity(sv, call):
    parent, tok, logits = walk_inputs()
    args = {"tree_accept": (parent, tok, torch.tensor([[3, 5, 7, 8]], dtype=torch.int32, device="cuda")),
            "node_argmax_accept": (logits, parent, tok),
            "tree_accept_sample": (parent, tok, logits, torch.full((1, 4), 0.5, device="cuda"), torch.full((1,), 0.5, device="cuda"))}[call]
    fn, skip = getattr(sv, "specvlm_" + call), 1 if call == "node_argmax_accept" else 0
    for given in (walk_outputs(), tuple(walk_outputs()), (t for t in walk_outputs())):
        got = fn(*args, path_cap=None, out=given)[skip:]
        assert [t.tolist() for t in got] == [[2], [[0, 1, 2]], [7], [[3, 5, 7]]]
    with pytest.raises(TypeError):
        fn(*args, path_cap=None)


def test_numbers_of_the_attention_call(sv):
    torch.manual_seed(0)
    q = torch.randn(1, 4, 2, 64, device="cuda").bfloat16()
    k, v = (torch.randn(1, 2, 512, 64, device="cuda").bfloat16() for _ in range(2))
    P, parent = torch.tensor([400], dtype=torch.int32, device="cuda"), torch.tensor([[-1, 0, 1, 0]], dtype=torch.int32, device="cuda")
    want = sv.specvlm_tree_verify_attn(q, k, v, P, parent, num_splits=3, softmax_scale=0.25)
    for splits in (3.0, np.int64(3), torch.tensor(3)):
        for scale in (0.25, np.float64(0.25), torch.tensor(0.25)):
            assert torch.equal(sv.specvlm_tree_verify_attn(q, k, v, P, parent, num_splits=splits, softmax_scale=scale), want)
    with pytest.raises((TypeError, ValueError)):
        sv.specvlm_tree_verify_attn(q, k, v, P, parent, num_splits=None)


def test_ranks(sv):
    parent, tok, _ = walk_inputs()
    with pytest.raises(ValueError):
        sv.specvlm_tree_accept(parent[None], tok, tok)
    with pytest.raises(ValueError):
        sv.specvlm_draft_select(torch.zeros(1, 2, 8, device="cuda"), 2)


@pytest.mark.parametrize("given", [False, True])
def test_compaction_returns_none_for_moved_idx_left_out(sv, given):
    k, v = (torch.zeros(2, 1, 1, 32, 64, device="cuda") for _ in range(2))
    P, path = torch.tensor([5], dtype=torch.int32, device="cuda"), torch.tensor([[0, 2, -1]], dtype=torch.int32, device="cuda")
    new_P = torch.zeros(1, dtype=torch.int32, device="cuda") if given else None
    got = sv.specvlm_kv_compact(k, v, P, path, torch.tensor([1], dtype=torch.int32, device="cuda"), new_prefix_len=new_P)
    assert got[0].tolist() == [7] and got[1] is None
