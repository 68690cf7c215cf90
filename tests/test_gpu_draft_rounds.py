"""GPU parity of specvlm_draft_topk where too many entries reach the first threshold to be ranked as they are: rows of
equal logits, rows sorted along the vocabulary, rows with fewer finite logits than winners, and rows whose best
entries all sit in the chunks of K threads, so that the second threshold does not thin them out either; entries before
and after the 8-entry chunks."""
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
@pytest.mark.parametrize("V,K", [(1100, 10), (8200, 64), (32768, 10), (65536, 33), (65551, 10), (200003, 64)])
@pytest.mark.parametrize("offset", [0, 3])
def test_topk_round_by_round(sv, oracle, dtype, V, K, offset):
    from gpu_util import to_dev
    rng = np.random.default_rng(V + K + offset)
    R = 6
    wide = np.sort(W.normal(rng, (1, R, V + offset), 1.0, "f32"), axis=2)
    wide[0, 1] = wide[0, 1, ::-1]
    wide[0, 2] = 0.5                                                   # equal
    few = rng.choice(V, size=K - 2, replace=False) + offset            # fewer finite logits than winners
    keep = wide[0, 3, few]
    wide[0, 3] = -np.inf
    wide[0, 3, few] = keep
    wide[0, 4] = np.where(rng.random(V + offset) < 0.5, np.float32(0.0), np.float32(-0.0))     # -0 and +0 are equal
    per = 8 if dtype == "bf16" else 4                                   # entries per 16 bytes: chunks start at such a boundary
    head = -((R - 1) * (V + offset) + offset) % per
    thread = (np.arange(V) - head) // 8 % 1024
    wide[0, 5] = rng.permutation(wide[0, 5])
    wide[0, 5, offset:][(thread >= 500) & (thread < 500 + K)] += 20      # K threads hold the best entries
    if dtype == "bf16":
        wide = torch.from_numpy(wide).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    logits = np.ascontiguousarray(wide[:, :, offset:])
    score, token, _ = sv.specvlm_draft_topk(to_dev(wide)[:, :, offset:], K)
    r_score, r_token, _ = oracle.topk_logprob(logits.reshape(R, V), K)
    assert np.array_equal(token.cpu().numpy().reshape(R, K), r_token)
    np.testing.assert_allclose(score.cpu().numpy().reshape(R, K), r_score, rtol=0, atol=2e-5)
