"""GPU parity of specvlm_draft_topk where the row's division into chunks changes: rows shorter than a chunk or a
wavefront, starts off a 16-byte boundary with entries before and after the chunks, one entry more than what
stays in registers, rows that stream by, and more of a row than the chunk maxima kept per thread."""
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
@pytest.mark.parametrize("V,K", [(1, 1), (9, 9), (65, 64), (8191, 10), (32768, 10), (32769, 64), (65536, 10), (65543, 10),
                                 (196608, 10), (200003, 33)])
@pytest.mark.parametrize("offset", [0, 1, 5])
def test_topk_row_division(sv, oracle, dtype, V, K, offset):
    from gpu_util import to_dev
    rng = np.random.default_rng(V + 3 * K + offset)
    wide = W.normal(rng, (1, 2, V + offset), 2.0, dtype)
    logits = np.ascontiguousarray(wide[:, :, offset:])
    lse = torch.empty((1, 2), dtype=torch.float32, device="cuda")
    score, token, _ = sv.specvlm_draft_topk(to_dev(wide)[:, :, offset:], K, lse_out=lse)
    r_score, r_token, r_lse = oracle.topk_logprob(logits.reshape(2, V), K)
    assert np.array_equal(token.cpu().numpy().reshape(2, K), r_token)
    np.testing.assert_allclose(score.cpu().numpy().reshape(2, K), r_score, rtol=0, atol=2e-5)
    np.testing.assert_allclose(lse.cpu().numpy().reshape(-1), r_lse, rtol=0, atol=2e-5)


@pytest.mark.parametrize("C,M", [(64, 64), (65, 10), (128, 1), (129, 128), (255, 64), (256, 65)])
def test_select_few_candidates(sv, oracle, C, M):
    rng = np.random.default_rng(C * 3 + M)
    score = (np.round(rng.normal(0, 1, size=(3, C)) * 4) / 4).astype(np.float32)
    sel, _, count = sv.specvlm_draft_select(torch.from_numpy(score).cuda(), M)
    r_sel, r_count, _ = oracle.tree_select(score, M)
    assert np.array_equal(sel.cpu().numpy(), r_sel) and np.array_equal(count.cpu().numpy(), r_count)
