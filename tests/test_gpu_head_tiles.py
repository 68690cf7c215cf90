"""GPU parity of specvlm_head_argmax over the tiles its matrix-product form chooses from.

Which tile a call takes depends on the numbers of node rows and of tokens; each of the shapes below takes
another one (named beside it), with a last vocabulary tile and a last block of node rows that are ragged.
The contraction is one or a few steps long, so that the rings are never, just, or more than once full.
"""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_head import _check, sv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,E,V", [
    (5, 13, 128, 1),           # 128 x 128, one token, 65 rows
    (2, 47, 640, 33001),       # 256 x 96
    (3, 43, 384, 20001),       # 128 x 192
    (3, 33, 256, 33001),       # 256 x 128
    (2, 64, 128, 50177),       # 256 x 128, full node tile, one token in the last tile
    (5, 61, 128, 32000),       # 256 x 160, the second node tile reaches past the rows' 64-row padding
    (6, 64, 384, 32001),       # 256 x 192
    (7, 61, 256, 32000),       # 256 x 224
    (8, 57, 640, 31999),       # 256 x 256
])
def test_tiles_match_oracle(sv, oracle, B, N, E, V):  # noqa: F811
    rng = np.random.default_rng(B * 1000 + V)
    h = W.normal(rng, (B, N, E), 1.0, "bf16")
    w = W.normal(rng, (V, E), 2.0 / np.sqrt(E), "bf16")
    clear, real = _check(sv, oracle, h, w)
    assert real == B * N and clear > 0.9 * real


def test_counters_are_left_at_zero_between_tiles(sv):  # noqa: F811
    """One workspace for calls that take different tiles: every call leaves the arrival counters at zero."""
    g = torch.Generator(device="cuda").manual_seed(3)
    w = torch.randn((33001, 256), generator=g, device="cuda").to(torch.bfloat16)
    h = torch.randn((8, 60, 256), generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.zeros(sv.specvlm_head_argmax_workspace_bytes(8, 60, 33001), dtype=torch.uint8, device="cuda")
    want = sv.specvlm_head_argmax(h, w, workspace=ws).cpu()
    for B in (1, 2, 3, 5, 8):
        got = sv.specvlm_head_argmax(h[:B], w, workspace=ws).cpu()
        assert torch.equal(got, want[:B])


def test_rows_further_apart_than_a_tile_reaches(sv, oracle):  # noqa: F811
    """Head rows 16 MB apart: beyond the tiles' 32-bit offsets, so the 64-row form takes all blocks of rows."""
    from gpu_util import to_dev
    rng = np.random.default_rng(80)
    B, N, E, V, stride = 2, 40, 256, 130, 1 << 23
    h = W.normal(rng, (B, N, E), 1.0, "bf16")
    w = W.normal(rng, (V, E), 2.0 / np.sqrt(E), "bf16")
    big = torch.empty((V - 1) * stride + E, dtype=torch.bfloat16, device="cuda")
    wv = big.as_strided((V, E), (stride, 1))
    wv.copy_(to_dev(w))
    got = sv.specvlm_head_argmax(to_dev(h), wv).cpu().numpy()
    r_amax, _, r_gap, r_second = oracle.head_argmax(h, w)
    assert np.all((got == r_amax) | ((r_gap <= 1e-2) & (got == r_second)))
