"""GPU parity of the sampling acceptance where a row no longer stays in registers (more than 65536 tokens) and around
the borders of the register forms: rows off a 16-byte boundary, chunks with rejected tokens at their ends, draws in
the first and last chunk."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1023, 32768, 32769, 65536, 65537, 99254])
def test_sampled_walk_row_division(sv, oracle, dtype, V):
    from gpu_util import i32, to_dev
    rng = np.random.default_rng(V + len(dtype))
    B, N, cap = 6, 30, 6
    trees = [W.eagle_tree(rng, N, 5, 6) for _ in range(B)]
    parent = np.stack([t[0] for t in trees])
    wide = W.normal(rng, (B, N, V + 1), 2.0, dtype)
    logits = np.ascontiguousarray(wide[:, :, 1:])
    tok = rng.integers(0, V, size=(B, N)).astype(np.int32)
    chunk = -(-V // 1024)
    tok[:, 1:4] = [0, chunk - 1, V - 1]                          # ends of the first and the last chunk
    u_acc = rng.random((B, N), dtype=np.float32) * np.float32(0.002)
    u_bon = np.array([0.0, 1e-6, 0.37, 0.5, 0.9, 0.999], dtype=np.float32)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = sv.specvlm_tree_accept_sample(i32(parent), i32(tok), to_dev(wide)[:, :, 1:], torch.from_numpy(u_acc).cuda(),
                                        torch.from_numpy(u_bon).cuda(), temperature=0.8, path_cap=cap, err_flag=err)
    m, path, bonus, comm = (t.cpu().numpy() for t in got)
    r_m, r_path, r_bonus, _, info = oracle.tree_accept_sample(parent, tok, logits, u_acc, u_bon, temperature=0.8, path_cap=cap)
    clear = info["margin_accept"] > 1e-5
    assert clear.sum() >= B - 2
    assert np.array_equal(m[clear], r_m[clear]) and np.array_equal(path[clear], r_path[clear])
    # a draw within 1e-5 of an edge of the cumulated distribution may fall to the neighbour across it
    near = (info["margin_bonus"] <= 1e-5) & (bonus == info["bonus_alt"])
    assert np.all((bonus == r_bonus)[clear] | near[clear])
