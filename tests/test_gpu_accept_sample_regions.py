"""Sampling acceptance of rows that are read once, in regions of a wavefront each: sizes around whole blocks (64 vectors) and regions,
rejected tokens and the drawn position at their ends, rows with little finite in them."""
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
@pytest.mark.parametrize("V", [5, 255, 513, 4097, 16383, 65537, 131072, 131081, 270001])
def test_ends_of_blocks_and_regions(sv, oracle, dtype, V):
    from gpu_util import i32, to_dev
    rng = np.random.default_rng(V + len(dtype))
    B, N = 5, 12
    vec = 8 if dtype == "bf16" else 4
    per = -(-(-(-V // vec)) // 16)
    per = -(-per // 64) * 64 * vec                              # tokens of a region
    ends = [t for t in (0, 64 * vec - 1, 64 * vec, per - 1, per, 15 * per - 1, V - 1) if 0 <= t < V]
    parent = np.full((B, N), -1, dtype=np.int32)
    parent[:, 1:] = 0                                           # a root and its children: all tested at one node
    logits = W.normal(rng, (B, N, V), 2.0, dtype)
    tok = rng.integers(0, V, size=(B, N)).astype(np.int32)
    tok[:, 1:1 + len(ends)] = ends
    u_acc = np.ones((B, N), dtype=np.float32)                   # every child is rejected
    for u in (0.0, 0.2501, 0.75003, 0.99):
        u_bon = np.full(B, u, dtype=np.float32)
        got = sv.specvlm_tree_accept_sample(i32(parent), i32(tok), to_dev(logits), torch.from_numpy(u_acc).cuda(), torch.from_numpy(u_bon).cuda(),
                                            temperature=0.9, path_cap=4)
        m, path, bonus, _ = (t.cpu().numpy() for t in got)
        r_m, r_path, r_bonus, _, info = oracle.tree_accept_sample(parent, tok, logits, u_acc, u_bon, temperature=0.9, path_cap=4)
        clear = info["margin_accept"] > 1e-5
        assert np.array_equal(m[clear], r_m[clear]) and np.array_equal(path[clear], r_path[clear])
        # a draw within 1e-5 of an edge of the cumulated distribution may fall to the neighbour across it
        near = (info["margin_bonus"] <= 1e-5) & (bonus == info["bonus_alt"])
        assert np.all((bonus == r_bonus)[clear] | near[clear]), u


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [512, 513, 65537, 131072])
def test_little_finite(sv, dtype, V):
    """One token above a row of -inf or of the type's lowest value, a row of nothing but the lowest value, a row of -inf."""
    low = torch.finfo(dtype).min
    x = torch.full((4, 2, V), -torch.inf, dtype=dtype, device="cuda")
    x[1:3] = low
    x[0, :, V - 1] = x[1, :, V // 2] = -3.0
    parent = torch.tensor([[-1, 0]] * 4, dtype=torch.int32, device="cuda")
    tok = torch.tensor([[0, 1]] * 4, dtype=torch.int32, device="cuda")
    for u in (0.0, 0.5, 0.99999):
        m, path, bonus, _ = sv.specvlm_tree_accept_sample(parent, tok, x, torch.ones((4, 2), device="cuda"), torch.full((4,), u, device="cuda"),
                                                          temperature=1.0, path_cap=4)
        b = bonus.tolist()
        assert m.tolist() == [0] * 4 and b[0] == V - 1 and b[1] == V // 2 and b[3] == 0
        # V equal tokens less the rejected token 1, within the rounding of sums of up to V ones
        assert b[2] != 1 and abs(b[2] - u * (V - 1)) <= 2 + 1e-5 * V
    # a position that is none: the last live token, as in the register form
    for u in (-0.5, float("nan")):
        bonus = sv.specvlm_tree_accept_sample(parent, tok, x, torch.ones((4, 2), device="cuda"), torch.full((4,), u, device="cuda"),
                                              temperature=1.0, path_cap=4)[2]
        assert bonus.tolist() == [V - 1, V // 2, V - 1, 0]


@pytest.mark.parametrize("V", [20003, 152064, 200003, 250000])
def test_row_sums_do_not_lose_precision_with_length(sv, V):
    """The threshold at which a root's only child is accepted, its probability, by bisection against 64 bits.  exp2 and the quotient leave
    about 0.8e-7 (root mean square of 400 rows, any length); a sum of one chain a lane made it 1.0e-7 to 1.1e-7 from 200003 bf16 tokens on."""
    B = 400
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    x = torch.empty((B, 2, V), device="cuda").normal_(0, 0.3, generator=gen).to(torch.bfloat16)
    p = torch.softmax(x[:, 0].double(), -1)
    exact, top = p.max(1)
    parent = torch.tensor([[-1, 0]] * B, dtype=torch.int32, device="cuda")
    tok = torch.stack([torch.zeros_like(top), top], 1).int().contiguous()
    lo, hi = exact * (1 - 1e-4), exact * (1 + 1e-4)
    u = torch.ones((B, 2), device="cuda")
    for _ in range(24):
        u[:, 1] = ((lo + hi) / 2).float()
        accepted = sv.specvlm_tree_accept_sample(parent, tok, x, u, torch.full((B,), 0.5, device="cuda"), temperature=1.0, path_cap=4)[0] > 0
        lo, hi = torch.where(accepted, u[:, 1].double(), lo), torch.where(accepted, hi, u[:, 1].double())
    error = ((lo + hi) / 2 / exact - 1).square().mean().sqrt().item()
    assert error <= 0.95e-7, error
