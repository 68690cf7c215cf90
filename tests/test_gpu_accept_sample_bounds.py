"""Sampling acceptance over more than 65536 tokens where the logits fill their buffer to its ends: the first row starts
off a 16-byte boundary, the last one ends off one.  The bonus token must not depend on what lies around the buffer."""
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
@pytest.mark.parametrize("V,lead", [(65537, 1), (65543, 3), (99254, 1), (152064, 2), (70001, 0)])
def test_edge_rows(sv, oracle, dtype, V, lead):
    from gpu_util import i32, to_dev
    rng = np.random.default_rng(V + lead)
    B, N = 5, 1                                            # the root alone: every request's bonus is drawn from its own row
    logits = W.normal(rng, (B, N, V), 2.0, dtype)
    big = np.full(lead + B * V + 8, 0x7F00 if dtype == "bf16" else 3e38, dtype=logits.dtype)
    big[lead:lead + B * V] = logits.reshape(-1)
    view = to_dev(big)[lead:lead + B * V].view(B, N, V)
    u = np.array([0.0, 1e-6, 0.5, 0.99, 0.99999], dtype=np.float32)
    parent, tok = np.full((B, 1), -1, dtype=np.int32), np.zeros((B, 1), dtype=np.int32)
    got = sv.specvlm_tree_accept_sample(i32(parent), i32(tok), view, torch.zeros(B, N, device="cuda"), torch.from_numpy(u).cuda(),
                                        temperature=0.8, path_cap=2)
    _, _, want, _, info = oracle.tree_accept_sample(parent, tok, logits, np.zeros((B, N), np.float32), u, temperature=0.8, path_cap=2)
    bonus = got[2].cpu().numpy()
    near = (info["margin_bonus"] <= 1e-5) & (bonus == info["bonus_alt"])
    assert np.all((bonus == want) | near)
