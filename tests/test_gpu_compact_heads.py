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
