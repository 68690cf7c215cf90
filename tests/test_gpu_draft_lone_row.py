"""The borders of the ranking's forms, and the selection of a level with one row and no scores before it (the root's): its candidates are already in order, so the
launch takes them as they come.  Exact against the separate calls (specvlm_draft_topk, then specvlm_draft_select over its
scores) and against the general selection (the same call with scores of zero)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def rows(kind, B, V, rng):
    if kind == "normal":
        return rng.normal(0.0, 2.0, (B, 1, V))
    if kind == "equal":
        return np.full((B, 1, V), 1.5)
    if kind == "steps":                              # many equal logits, sorted along the vocabulary
        return np.broadcast_to(np.arange(V) // 40 * 0.25, (B, 1, V)).copy()
    x = rng.normal(0.0, 2.0, (B, 1, V))              # fewer finite logits than candidates / none at all
    x[:, :, 3 if kind == "few" else 0:] = -np.inf
    return x


# M: one, fewer than K, K, more than K; V: every row division (registers of 4 and 8 chunks, streamed)
@pytest.mark.parametrize("kind", ["normal", "equal", "steps", "few", "none"])
@pytest.mark.parametrize("dtype,V,K", [("bf16", 10, 10), ("bf16", 32003, 10), ("f32", 40000, 17), ("bf16", 70001, 64)])
@pytest.mark.parametrize("B,M", [(1, 1), (3, 8), (2, 10), (1, 64)])
def test_root_level(sv, kind, dtype, V, K, B, M):
    rng = np.random.default_rng(V + 7 * M)
    x = torch.from_numpy(rows(kind, B, V, rng)).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    counters = torch.zeros(B * sv.binding.COUNTER_STRIDE, dtype=torch.int32, device="cuda")
    score, token, _ = sv.specvlm_draft_topk(x, K)
    want = sv.specvlm_draft_select(score, M, index_base=5)
    # a NaN (no finite logit) equals itself: compare bits
    bits = lambda t: (t.view(torch.int32) if t.dtype == torch.float32 else t).cpu().numpy()
    for cum in (None, torch.zeros((B, 1), dtype=torch.float32, device="cuda")):
        got = sv.specvlm_draft_topk_select(x, K, M, cum=cum, index_base=5, counters=counters)
        assert np.array_equal(bits(got[0]), bits(score)) and np.array_equal(bits(got[1]), bits(token))
        for g, w in zip(got[3:], want):
            assert np.array_equal(bits(g), bits(w))
    assert not counters.any()


# the borders of the ranking's forms (few candidates up to 192, then a threshold first; more than 64 chosen: everybody), full ties
@pytest.mark.parametrize("C,M", [(15, 3), (16, 16), (17, 9), (192, 64), (193, 1), (193, 64), (193, 65), (255, 65), (1023, 64), (1024, 1)])
def test_select_borders(sv, C, M):
    rng = np.random.default_rng(C + M)
    score = np.concatenate([rng.normal(size=(2, C)), np.round(rng.normal(size=(1, C))), np.full((1, C), -np.inf)]).astype(np.float32)
    sel, val, count = sv.specvlm_draft_select(torch.from_numpy(score).cuda(), M)
    want = np.sort(np.argsort(-score, axis=1, kind="stable")[:, :M], axis=1)
    assert np.array_equal(sel.cpu().numpy(), want) and np.array_equal(count.cpu().numpy(), [M] * 4)
    assert np.array_equal(val.cpu().numpy(), np.take_along_axis(score, want, 1))
