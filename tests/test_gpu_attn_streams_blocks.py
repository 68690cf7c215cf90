"""Paged cache, a key stream per wavefront: the block ids come 32 tiles of a stream at a time.  Streams that end on both sides of
those borders, and an id outside the pool on either side of the first."""
import numpy as np
import pytest

from attn_plan_util import division_of
from test_gpu_attn import check, run_both

pytestmark = pytest.mark.gpu

# tiles of the first stream of each request; 4 streams of 32-key tiles: 128 keys a round
TILES = [1, 2, 3, 4, 5, 27, 28, 29, 30, 31, 32, 33, 34, 35, 36, 37]
SHAPES = {64: (26, 8, 1, 64, 60), 128: (26, 8, 1, 128, 60)}


@pytest.fixture(scope="module")
def sv():
    import paper_2509_11815_amd as sv
    sv.load_library()
    return sv


def make(D):
    from gpu_util import random_case
    B, Hq, Hkv, _, N = SHAPES[D]
    tiles = TILES + ([63, 64, 65, 66, 67, 70] if D == 64 else [36, 35, 34, 33, 32, 31])
    tiles += [2] * (B - len(tiles))
    P = [128 * t - N - (5 * b) % 128 if t > 1 else 7 for b, t in enumerate(tiles)]
    case = random_case(8400 + D, "bf16", B=B, Hq=Hq, Hkv=Hkv, D=D, N_max=N, P_list=P, paged=True)
    assert division_of(B, Hq, Hkv, D, N, case["block_table"].shape[1] * 16, paged=True) == (1, 0)
    return case


@pytest.mark.parametrize("D", [64, 128])
def test_long_streams(sv, oracle, D):
    case = make(D)
    check(case, *run_both(sv, oracle, case), f"paged streams x{D}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("tile", [0, 1, 2, 31, 32, 34])
def test_block_outside_the_pool(sv, oracle, D, tile):
    """It sets the error word; requests that do not name it are as they were."""
    import torch
    from gpu_util import assert_attn_close, i32, to_dev, to_host_f64
    case = make(D)
    B, bad = case["q"].shape[0], 15                           # 37 tiles in its first stream
    table = case["block_table"].copy()
    table[bad, 8 * tile + 1] = case["k"].shape[0] if tile % 2 else -3
    args = [to_dev(case[x]) for x in "qkv"] + [i32(case["prefix_len"]), i32(case["parent"])]
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    good = [b for b in range(B) if b != bad]
    ref = to_host_f64(sv.specvlm_tree_verify_attn(*args, block_table=i32(case["block_table"]), err_flag=err))
    assert int(err.item()) == 0
    got = to_host_f64(sv.specvlm_tree_verify_attn(*args, block_table=i32(table), err_flag=err))
    assert int(err.item()) == 16
    assert np.array_equal(got[good], ref[good])
