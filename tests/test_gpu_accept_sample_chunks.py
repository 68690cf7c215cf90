"""The two ways in which the sampling acceptance takes a row into registers - whole aligned vectors, and vectors at any token with
the one that the row ends in read entry by entry - at vocabulary sizes around their borders.

Both add the same values up in the same order, so a call on aligned rows and one on the same values a token further on must
give the same results exactly.  The aligned call is also compared with the oracle; TOL as in test_gpu_accept_sample.py."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


# chunks of 1 token (most threads without any), 2 and 3, whole vectors (8192, 32768, 65536: aligned rows take the
# aligned form), whole vectors with the last thread's chunk cut short inside a vector, ragged chunks, the last one of 1 token
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [3, 1024, 1025, 2500, 7169, 8184, 8192, 20003, 30724, 32768, 33000, 60001, 65529, 65536])
def test_rows_aligned_and_not(sv, oracle, dtype, V):
    from gpu_util import i32, to_dev
    rng = np.random.default_rng(3 * V + len(dtype))
    B, N, cap = 6, 30, 6
    trees = [W.eagle_tree(rng, N, 5, 6) for _ in range(B)]
    parent = np.stack([t[0] for t in trees])
    logits = W.normal(rng, (B, N, V), 2.0, dtype)
    tok = rng.integers(0, V, size=(B, N)).astype(np.int32)
    chunk = -(-V // 1024)
    tok[:, 1:5] = [0, min(chunk, V - 1), (V - 1) // chunk * chunk, V - 1]     # ends of the first and of the last chunk that has any
    u_acc = rng.random((B, N), dtype=np.float32) * np.float32(0.002)
    u_bon = np.array([0.0, 1e-6, 0.37, 0.5, 0.9, 0.9999], dtype=np.float32)
    aligned = to_dev(logits)
    room = torch.empty(B * N * V + 1, dtype=aligned.dtype, device="cuda")
    shifted = room[1:].view(B, N, V)
    shifted.copy_(aligned)
    pitch = torch.empty((B, N, V + 3), dtype=aligned.dtype, device="cuda")     # rows at every alignment
    pitch[:, :, :V] = aligned
    outs = []
    for view in (aligned, shifted, pitch[:, :, :V]):
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        got = sv.specvlm_tree_accept_sample(i32(parent), i32(tok), view, torch.from_numpy(u_acc).cuda(), torch.from_numpy(u_bon).cuda(),
                                            temperature=0.8, path_cap=cap, err_flag=err)
        outs.append([t.cpu().numpy() for t in got] + [err.cpu().numpy()])
    for other in outs[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(outs[0], other))
    m, path, bonus, _, _ = outs[0]
    r_m, r_path, r_bonus, _, info = oracle.tree_accept_sample(parent, tok, logits, u_acc, u_bon, temperature=0.8, path_cap=cap)
    clear = info["margin_accept"] > TOL
    assert clear.sum() >= B - 2
    assert np.array_equal(m[clear], r_m[clear]) and np.array_equal(path[clear], r_path[clear])
    near = (info["margin_bonus"] <= TOL) & (bonus == info["bonus_alt"])
    assert np.all((bonus == r_bonus)[clear] | near[clear])
