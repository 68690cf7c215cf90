"""The edge tests of the bf16 attention call, run with the kernel whose workgroups take all query rows of a head: most of
their shapes are divided by query rows otherwise.  The rows' distance in q decides: the row-dividing kernels hold it in
32 bits, so queries 2^30 elements apart in all leave every shape to the key ranges."""
import pytest
import torch

import test_gpu_attn as T
from attn_plan_util import plan_of_desc

pytestmark = pytest.mark.gpu


class FarQueries:
    """The binding with q copied into a view whose node stride is too large for the row-dividing kernels."""

    def __init__(self, sv):
        self._sv, self._buf, self.calls = sv, None, 0

    def __getattr__(self, name):
        return getattr(self._sv, name)

    def specvlm_tree_verify_attn(self, q, k, v, *args, out=None, desc=None, num_splits=0, softmax_scale=0.0, block_table=None, **kw):
        B, N, H, D = q.shape
        stride = ((1 << 30) // N + 8) // 8 * 8
        stride += 8 if stride * N < 1 << 30 else 0
        size = (N - 1) * stride + B * H * D
        far = torch.empty(size, dtype=q.dtype, device=q.device).as_strided((B, N, H, D), (H * D, stride, D, 1))
        far.copy_(q)
        out = torch.zeros(q.shape, dtype=q.dtype, device=q.device) if out is None else out
        num_splits = desc.num_splits if desc is not None else num_splits
        desc = self._sv.binding.make_attn_desc(far, k, out, block_table=block_table, num_splits=num_splits, softmax_scale=softmax_scale)
        plan = plan_of_desc(desc)
        assert plan.block_rows == 0 and plan.columns == 0
        self.calls += 1
        return self._sv.specvlm_tree_verify_attn(far, k, v, *args, out=out, desc=desc, block_table=block_table, **kw)


@pytest.fixture
def far():
    import paper_2509_11815_amd as sv
    sv.load_library()
    far = FarQueries(sv)
    yield far
    assert far.calls


@pytest.mark.parametrize("num_splits", [1, 2, 3, 5, 8, 9, 16])
def test_split_counts(far, oracle, num_splits):
    T.test_bf16_split_counts_span_tiles_and_tail(far, oracle, num_splits)


@pytest.mark.parametrize("D", [64, 128])
def test_paged_cache(far, oracle, D):
    T.test_bf16_paged_cache(far, oracle, D)


def test_mask_leaks(far, oracle):
    T.test_bf16_mask_leak_detectors(far, oracle)


@pytest.mark.parametrize("splits", [1, 3])
def test_block_outside_the_pool(far, oracle, splits):
    T.test_block_table_entry_outside_the_pool_is_reported(far, oracle, "bf16", splits)


def test_one_workspace(far, oracle):
    T.test_one_workspace_across_head_counts(far, oracle)


@pytest.mark.parametrize("seed", range(24))
def test_random_shapes(far, oracle, seed):
    T.test_random_shapes_sweep(far, oracle, seed)


def test_long_prefix(far, oracle):
    T.test_long_video_prefix(far, oracle)


def test_requests_far_apart(far, oracle):
    T.test_requests_more_than_4_gib_apart(far, oracle, "bf16")


def test_large_paged_pool(far, oracle):
    T.test_paged_pool_larger_than_4_gib(far, oracle)


def test_two_streams(far, oracle):
    T.test_two_streams_with_their_own_workspaces(far, oracle)


@pytest.mark.parametrize("D", [64, 128])
def test_capacity_above_the_lengths(far, oracle, D):
    T.test_capacity_far_above_the_lengths(far, oracle, D)
