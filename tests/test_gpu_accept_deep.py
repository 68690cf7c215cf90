"""GPU parity (bit-exact) of the greedy acceptance on deep trees: chains of up to 64 nodes with one mismatch at the depths where pointer doubling
takes another round, branching trees of any depth, paths that do not fit, one-node trees, node counts out of range."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BAD_NUM_NODES, PATH_TOO_LONG = 2, 8


def accept(parent, tok, amax, nodes, cap, N):
    """The oracle's acceptance where nodes deeper than cap - 1 count as mismatches, and whether one of them would have been accepted."""
    import oracle
    n = np.clip(nodes, 1, N).astype(np.int32)
    full = oracle.tree_accept(parent, tok, amax, n, path_cap=64)
    depth = np.zeros_like(parent)
    for i in range(1, N):
        depth[:, i] = depth[np.arange(len(parent)), parent[:, i]] + 1
    return oracle.tree_accept(parent, np.where(depth < cap, tok, -7), amax, n, path_cap=cap), bool((full[0] >= cap).any())


def trees(N, seed):
    """Chains that match but for one depth (0: wholly), then trees that mostly go on from their last node, mostly matching."""
    rng = np.random.default_rng(seed)
    wrong = [0] + [d for d in (1, 2, 15, 16, 17, 31, 32, 33, 62, 63) if d < N]
    B = len(wrong) + 40
    parent, amax = np.zeros((B, N), dtype=np.int32), rng.integers(0, 2, size=(B, N)).astype(np.int32)
    tok = np.zeros((B, N), dtype=np.int32)
    for b in range(B):
        parent[b, 0] = -1
        for i in range(1, N):
            parent[b, i] = i - 1 if b < len(wrong) or rng.random() < 0.9 else rng.integers(0, i)
            tok[b, i] = amax[b, parent[b, i]]
            if (b < len(wrong) and i == wrong[b]) or (b >= len(wrong) and rng.random() < 0.03):
                tok[b, i] = 1 - tok[b, i]
    return rng, parent, tok, amax


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N,cap", [(64, 64), (64, 63), (64, 33), (64, 32), (64, 1), (63, 64), (33, 64), (2, 2), (1, 1), (1, 64)])
def test_deep_trees_and_node_counts(N, cap, fused):
    import paper_2509_11815_amd as sv
    from gpu_util import i32, to_dev
    sv.load_library()
    rng, parent, tok, amax = trees(N, 100 * N + cap)
    B = len(parent)
    for nodes in (None, rng.integers(1, N + 1, size=B).astype(np.int32), rng.choice([0, -1, N + 1, 2**31 - 1, N], size=B).astype(np.int32)):
        nn, am = np.full(B, N) if nodes is None else nodes, amax.copy()
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        options = dict(num_nodes=None if nodes is None else i32(nodes), path_cap=cap, err_flag=err)
        if fused:
            am[np.arange(N)[None, :] >= nn[:, None]] = -1                # rows past the count have no result
            logits = np.zeros((B, N, 8), dtype=np.float32)
            logits[np.arange(B)[:, None], np.arange(N)[None, :], amax] = 1.0
            counters = torch.zeros(B * sv.binding.COUNTER_STRIDE, dtype=torch.int32, device="cuda")
            got_am, *got = sv.specvlm_node_argmax_accept(to_dev(logits), i32(parent), i32(tok), counters=counters, **options)
            assert np.array_equal(got_am.cpu().numpy(), am) and int(counters.abs().sum().item()) == 0
        else:
            got = sv.specvlm_tree_accept(i32(parent), i32(tok), i32(am), **options)
        ref, too_long = accept(parent, tok, am, nn, cap, N)
        for g, r, name in zip(got, ref, ["accept_len", "path", "bonus", "committed"]):
            assert np.array_equal(g.cpu().numpy(), r), (name, nodes)
        assert nodes is not None or ref[0].max() == min(N, cap) - 1
        bad = bool(((nn < 1) | (nn > N)).any())
        assert int(err.item()) == BAD_NUM_NODES * bad + PATH_TOO_LONG * too_long
