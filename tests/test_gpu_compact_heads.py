"""Compaction with several KV heads per workgroup: a last group that is not full, path capacities at the edge of what a
workgroup's registers hold, few and many workgroups.  Byte for byte against the oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from test_compact_plan import head_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,B,H,D,dtype,path_cap", [
    (32, 8, 5, 64, np.uint16, 8),          # 4 heads a workgroup, the last has one
    (32, 16, 9, 64, np.uint16, 8),         # 8 and one
    (40, 8, 7, 128, np.float32, 16),       # 2 heads of 512-byte rows
    (40, 8, 7, 128, np.float32, 17),       # ... one row more
    (33, 8, 2, 128, np.uint16, 64),        # one of 1024 chunks
    (1, 1, 3, 64, np.uint16, 5),           # one head each
    (40, 16, 7, 128, np.float32, 16),      # 4 heads of 512-byte rows fill the registers
    (64, 8, 4, 128, np.uint16, 64),        # 2 of 1024 chunks
])
@pytest.mark.parametrize("paged", [False, True])
def test_head_groups(oracle, L, B, H, D, dtype, path_cap, paged):
    chunks = path_cap * D * np.dtype(dtype).itemsize // 16
    expected = {(32, 5, 8): 4, (32, 9, 8): 8, (40, 7, 16): 2 if B == 8 else 4, (40, 7, 17): 2, (33, 2, 64): 1, (1, 3, 5): 1, (64, 4, 64): 2}
    assert 1 << head_bits(2 * L * B * H, chunks) == expected[L, H, path_cap]
    import paper_2509_11815_amd as sv
    sv.load_library()
    rng = np.random.default_rng(path_cap + H)
    P = rng.integers(0, 9, size=B).astype(np.int32)
    m = np.minimum(rng.integers(0, path_cap, size=B), path_cap - 1).astype(np.int32)
    m[0] = path_cap - 1
    paths = np.full((B, path_cap), -1, dtype=np.int32)
    for b in range(B):
        paths[b, 0] = 0
        if m[b]:
            paths[b, 1:m[b] + 1] = np.sort(rng.choice(np.arange(1, 64), size=m[b], replace=False))
    table = None
    if paged:
        table, nb = W.block_table(rng, B, 5, spare=0.2)
        shape = (L, nb, H, 16, D)
    else:
        shape = (L, B, H, 80, D)
    draw = (lambda: rng.integers(0, 65536, size=shape, dtype=np.uint16)) if dtype == np.uint16 else (lambda: rng.standard_normal(shape, dtype=np.float32))
    k, v = draw(), draw()
    from gpu_util import i32, to_dev, to_host_bits
    kd, vd = to_dev(k), to_dev(v)
    newp, _ = sv.specvlm_kv_compact(kd, vd, i32(P), i32(paths), i32(m), block_table=None if table is None else i32(table))
    torch.cuda.synchronize()
    ref_newp, _ = oracle.kv_compact(k, v, P, paths, m, block_table=table)
    assert np.array_equal(newp.cpu().numpy(), ref_newp)
    assert np.array_equal(to_host_bits(kd), k) and np.array_equal(to_host_bits(vd), v)


@pytest.mark.parametrize("length", [80, 79 - 63, -1, -2**31, 2**31 - 1, 2**31 - 2, 2**31 - 9, 2**31 - 64])
@pytest.mark.parametrize("paged", [False, True])
def test_moves_outside_the_cache_are_not_made(oracle, paged, length):
    """A request whose prefix no cache holds, beside one that is compacted: of its path the rows that lie outside stay where they are,
    also where prefix and node do not fit in 32 bits together."""
    import paper_2509_11815_amd as sv
    from gpu_util import i32, to_dev, to_host_bits
    sv.load_library()
    rng = np.random.default_rng(7)
    L, B, H, D, slots = 3, 2, 4, 64, 80
    P = np.array([5, length], dtype=np.int32)
    path = np.array([[0, 3, 9, 20, 63], [0, 2, 5, 8, 63]], dtype=np.int32)
    m = np.array([4, 4], dtype=np.int32)
    table = None
    if paged:
        table, nb = W.block_table(rng, B, 5, spare=0.2)
        shape = (L, nb, H, 16, D)
    else:
        shape = (L, B, H, slots, D)
    k, v = (rng.integers(0, 65536, size=shape, dtype=np.uint16) for _ in range(2))
    kd, vd = to_dev(k), to_dev(v)
    sv.specvlm_kv_compact(kd, vd, i32(P), i32(path), i32(m), block_table=None if table is None else i32(table))
    torch.cuda.synchronize()
    inside = [j for j in range(5) if length >= 0 and length + int(path[1, j]) < slots]
    ref = [x.copy() for x in (k, v)]
    moves = [(0, 5 + int(a), 5 + j) for j, a in enumerate(path[0])] + [(1, length + int(path[1, j]), length + j) for j in inside]
    row = lambda x, b, s: x[:, table[b, s >> 4], :, s & 15] if paged else x[:, b, :, s]
    for old, new in zip((k, v), ref):
        for b, src, dst in moves:
            row(new, b, dst)[:] = row(old, b, src)
    assert np.array_equal(to_host_bits(kd), ref[0]) and np.array_equal(to_host_bits(vd), ref[1])
