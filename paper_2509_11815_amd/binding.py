"""Binding of libspecvlm.so: same names as the C entry points, marshalling only.

Every step runs in the library's HIP kernels; there is no fallback.  Importing this module
does not need the library; the first call loads it and raises if it has not been built
(``python -m paper_2509_11815_amd.build``).  The functions here hold names, defaults and documentation;
arguments are checked and marshalled in C++ (csrc/native_binding.cpp), because eager callers make
calls of a few microseconds of GPU time each.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os

import torch

from . import build as _build

SPECVLM_BF16, SPECVLM_F32 = 0, 1
STATUS = {0: "OK", 1: "INVALID_ARG", 2: "UNSUPPORTED", 3: "WORKSPACE_TOO_SMALL", 4: "HIP_ERROR"}
ERR_BITS = {1: "BAD_PARENT", 2: "BAD_NUM_NODES", 4: "BAD_LENGTH", 8: "PATH_TOO_LONG", 16: "BAD_BLOCK",
            32: "BAD_TOKEN", 64: "TREE_NOT_CLOSED"}


def err_flag_names(word: int) -> list[str]:
    """Names of the SPECVLM_ERR_* bits set in a device error word (after the caller synchronised)."""
    return [name for bit, name in ERR_BITS.items() if word & bit] + (
        [hex(word & ~sum(ERR_BITS))] if word & ~sum(ERR_BITS) else [])

EXPORTS = ["specvlm_version", "specvlm_last_hip_error", "specvlm_tree_verify_attn_workspace_bytes",
           "specvlm_tree_verify_attn_num_splits",
           "specvlm_tree_verify_attn", "specvlm_tree_verify_attn_static", "specvlm_tree_verify_attn_vector_alu",
           "specvlm_node_argmax", "specvlm_tree_accept", "specvlm_tree_accept_sample",
           "specvlm_kv_compact", "specvlm_draft_topk", "specvlm_draft_topk_select", "specvlm_draft_select",
           "specvlm_draft_finalize",
           "specvlm_head_argmax", "specvlm_head_argmax_workspace_bytes",
           "specvlm_visual_pool", "specvlm_visual_prune", "specvlm_visual_pool_padded", "specvlm_visual_prune_padded",
           "specvlm_node_argmax_accept"]


class SpecvlmError(RuntimeError):
    pass


class AttnDesc(ctypes.Structure):
    """Mirror of specvlm_attn_desc."""
    _fields_ = [("dtype", ctypes.c_int32), ("B", ctypes.c_int32), ("H_q", ctypes.c_int32),
                ("H_kv", ctypes.c_int32), ("D", ctypes.c_int32), ("N_max", ctypes.c_int32),
                ("softmax_scale", ctypes.c_float), ("paged", ctypes.c_int32),
                ("block_size", ctypes.c_int32), ("max_blocks_per_req", ctypes.c_int32),
                ("num_blocks", ctypes.c_int32), ("kv_capacity", ctypes.c_int32),
                ("num_splits", ctypes.c_int32),
                ("q_stride_b", ctypes.c_int64), ("q_stride_n", ctypes.c_int64), ("q_stride_h", ctypes.c_int64),
                ("o_stride_b", ctypes.c_int64), ("o_stride_n", ctypes.c_int64), ("o_stride_h", ctypes.c_int64),
                ("kv_stride_b", ctypes.c_int64), ("kv_stride_h", ctypes.c_int64), ("kv_stride_t", ctypes.c_int64)]


class _NotLoaded:
    """Stands in for the native module until the first call, which loads the library."""

    def __getattr__(self, name):
        load_library()
        return getattr(_native, name)


_lib = None
_native = _NotLoaded()


def _load_native(L):
    """The native marshalling module, bound to the entry points of the loaded library."""
    global _native
    if isinstance(_native, _NotLoaded):
        if not os.path.exists(_build.NATIVE):
            raise SpecvlmError(f"{_build.NATIVE} is missing: build it with `python -m paper_2509_11815_amd.build` "
                               "(there is no fallback path)")
        spec = importlib.util.spec_from_file_location("_specvlm_native", _build.NATIVE)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
    else:
        module = _native
    module.bind({name: ctypes.cast(getattr(L, name), ctypes.c_void_p).value for name in EXPORTS}, SpecvlmError)
    _native = module


def load_library(path: str | None = None) -> ctypes.CDLL:
    global _lib
    if _lib is not None and path is None:
        return _lib
    path = path or os.environ.get("SPECVLM_LIB") or _build.LIB       # SPECVLM_LIB: alternative build of the library
    if not os.path.exists(path):
        raise SpecvlmError(f"{path} is missing: build it with `python -m paper_2509_11815_amd.build` "
                           "(there is no fallback path)")
    L = ctypes.CDLL(path)
    missing = [name for name in EXPORTS if not hasattr(L, name)]
    if missing:
        raise SpecvlmError(f"{path} does not export {missing}: rebuild it with `python -m paper_2509_11815_amd.build`")
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    L.specvlm_version.restype = i32
    L.specvlm_last_hip_error.restype = i32
    L.specvlm_tree_verify_attn_workspace_bytes.restype = ctypes.c_size_t
    L.specvlm_tree_verify_attn_workspace_bytes.argtypes = [ctypes.POINTER(AttnDesc)]
    L.specvlm_tree_verify_attn_num_splits.restype = i32
    L.specvlm_tree_verify_attn_num_splits.argtypes = [ctypes.POINTER(AttnDesc)]
    L.specvlm_tree_verify_attn.restype = i32
    L.specvlm_tree_verify_attn.argtypes = [ctypes.POINTER(AttnDesc)] + [vp] * 9 + [vp, ctypes.c_size_t, vp, vp]
    L.specvlm_tree_verify_attn_static.restype = i32
    L.specvlm_tree_verify_attn_static.argtypes = [ctypes.POINTER(AttnDesc)] + [vp] * 9 + [vp, vp]
    L.specvlm_node_argmax.restype = i32
    L.specvlm_node_argmax.argtypes = [i32, i32, i32, i32, vp, i64, i64, vp, vp, vp]
    L.specvlm_tree_accept.restype = i32
    L.specvlm_tree_accept.argtypes = [i32, i32, i32] + [vp] * 10
    L.specvlm_tree_accept_sample.restype = i32
    L.specvlm_tree_accept_sample.argtypes = [i32, i32, i32, i32, i32, vp, vp, vp, i64, i64, vp, ctypes.c_float] + [vp] * 8
    L.specvlm_kv_compact.restype = i32
    L.specvlm_kv_compact.argtypes = [ctypes.POINTER(AttnDesc), i32, vp, vp, i64, vp, vp, vp, vp, vp, i32, vp, vp, vp, vp, vp]
    L.specvlm_tree_verify_attn_vector_alu.restype = i32
    L.specvlm_tree_verify_attn_vector_alu.argtypes = [ctypes.POINTER(AttnDesc)] + [vp] * 9 + [vp, vp]
    L.specvlm_draft_topk.restype = i32
    L.specvlm_draft_topk.argtypes = [i32] * 5 + [vp, i64, i64, vp, i64, vp, i64, vp, vp, vp, i64, vp, vp]
    L.specvlm_draft_topk_select.restype = i32
    L.specvlm_draft_topk_select.argtypes = ([i32] * 5 + [vp, i64, i64, vp, i64, vp, i64, vp, vp, vp, i64, vp] +
                                            [i32, i32, vp, vp, vp, vp, vp])
    L.specvlm_draft_select.restype = i32
    L.specvlm_draft_select.argtypes = [i32, i32, i32, vp, i64, vp, i32, vp, vp, vp, vp]
    L.specvlm_draft_finalize.restype = i32
    L.specvlm_draft_finalize.argtypes = [i32, i32, i32, vp, vp, vp, i64] + [vp] * 8
    L.specvlm_head_argmax_workspace_bytes.restype = ctypes.c_size_t
    L.specvlm_head_argmax_workspace_bytes.argtypes = [i32, i32, i32]
    L.specvlm_head_argmax.restype = i32
    L.specvlm_head_argmax.argtypes = [i32] * 5 + [vp, i64, i64, vp, i64, vp, vp, vp, vp, ctypes.c_size_t, vp]
    L.specvlm_visual_pool.restype = i32
    L.specvlm_visual_pool.argtypes = [i32] * 5 + [vp, i64, i64, vp, vp, i64, i64, vp, vp, vp]
    L.specvlm_visual_pool_padded.restype = i32
    L.specvlm_visual_pool_padded.argtypes = L.specvlm_visual_pool.argtypes
    L.specvlm_visual_prune.restype = i32
    L.specvlm_visual_prune.argtypes = [i32] * 5 + [vp, i64, i64, vp, vp, i64, i64, vp, vp]
    L.specvlm_visual_prune_padded.restype = i32
    L.specvlm_visual_prune_padded.argtypes = L.specvlm_visual_prune.argtypes
    L.specvlm_node_argmax_accept.restype = i32
    L.specvlm_node_argmax_accept.argtypes = [i32] * 5 + [vp, i64, i64] + [vp] * 11
    _load_native(L)
    _lib = L
    return L


def lib() -> ctypes.CDLL:
    return load_library()


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.bfloat16:
        return SPECVLM_BF16
    if t.dtype == torch.float32:
        return SPECVLM_F32
    raise TypeError(f"bfloat16 or float32 expected, got {t.dtype}")


COUNTER_STRIDE = 32                 # SPECVLM_COUNTER_STRIDE: int32 words between two requests' arrival counters


def make_attn_desc(q, k_cache, out=None, *, block_table=None, softmax_scale=0.0, num_splits=0) -> AttnDesc:
    """Fill a specvlm_attn_desc from tensor shapes and strides.

    q [B,N_max,H_q,D]; contiguous cache [B,H_kv,capacity,D]; paged cache [num_blocks,H_kv,16,D]."""
    B, N_max, H_q, D = q.shape
    d = AttnDesc()
    d.dtype = _dtype_code(q)
    d.B, d.H_q, d.H_kv, d.D, d.N_max = B, H_q, k_cache.shape[1], D, N_max
    d.softmax_scale = float(softmax_scale)
    d.num_splits = int(num_splits)
    if q.stride(3) != 1 or k_cache.stride(3) != 1:
        raise ValueError("innermost dimension must be contiguous")
    d.q_stride_b, d.q_stride_n, d.q_stride_h = q.stride(0), q.stride(1), q.stride(2)
    o = q if out is None else out
    d.o_stride_b, d.o_stride_n, d.o_stride_h = o.stride(0), o.stride(1), o.stride(2)
    d.kv_stride_b, d.kv_stride_h, d.kv_stride_t = k_cache.stride(0), k_cache.stride(1), k_cache.stride(2)
    if block_table is not None:
        d.paged, d.block_size = 1, k_cache.shape[2]
        d.max_blocks_per_req = block_table.shape[1]
        d.num_blocks = k_cache.shape[0]
        d.kv_capacity = d.max_blocks_per_req * d.block_size
    else:
        d.paged, d.block_size, d.max_blocks_per_req, d.num_blocks = 0, 0, 0, 0
        d.kv_capacity = k_cache.shape[2]
    return d


def specvlm_version() -> int:
    return int(lib().specvlm_version())


def specvlm_tree_verify_attn_workspace_bytes(desc: AttnDesc) -> int:
    return int(lib().specvlm_tree_verify_attn_workspace_bytes(ctypes.byref(desc)))


def specvlm_tree_verify_attn_num_splits(desc: AttnDesc) -> int:
    return int(lib().specvlm_tree_verify_attn_num_splits(ctypes.byref(desc)))


def specvlm_tree_verify_attn(q, k_cache, v_cache, prefix_len, parent, *, num_nodes=None, block_table=None,
                             out=None, lse=None, workspace=None, err_flag=None, softmax_scale=0.0,
                             num_splits=0, desc=None, stream=None):
    """One layer of tree-masked verification attention.  Returns `out` ([B,N_max,H_q,D])."""
    return _native.tree_verify_attn(q, k_cache, v_cache, prefix_len, parent, num_nodes, block_table, out, lse, workspace,
                                    err_flag, softmax_scale, num_splits, desc, stream, 0)


def specvlm_tree_verify_attn_vector_alu(q, k_cache, v_cache, prefix_len, parent, *, out, **kw):
    """Measurement aid: the same call computed by the vector-ALU kernel (see the header)."""
    return specvlm_tree_verify_attn_static(q, k_cache, v_cache, prefix_len, parent, out=out,
                                           _entry="specvlm_tree_verify_attn_vector_alu", **kw)


def specvlm_tree_verify_attn_static(q, k_cache, v_cache, prefix_len, parent, *, out, num_nodes=None,
                                    block_table=None, lse=None, err_flag=None, softmax_scale=0.0,
                                    num_splits=0, desc=None, stream=None, _entry="specvlm_tree_verify_attn_static"):
    """specvlm_tree_verify_attn on the library's own static scratch array.  Allocates nothing: `out`
    (and `lse`) must be supplied."""
    return _native.tree_verify_attn(q, k_cache, v_cache, prefix_len, parent, num_nodes, block_table, out, lse, None, err_flag,
                                    softmax_scale, num_splits, desc, stream,
                                    2 if _entry == "specvlm_tree_verify_attn_vector_alu" else 1)


def specvlm_node_argmax(logits, *, num_nodes=None, out=None, stream=None):
    """logits [B,N_max,V] -> int32 [B,N_max] lowest index of each row's maximum."""
    return _native.node_argmax(logits, num_nodes, out, stream)


def specvlm_tree_accept(parent, draft_tok, amax, *, num_nodes=None, path_cap=8, err_flag=None, out=None,
                        stream=None):
    """Returns (accept_len [B], path [B,path_cap], bonus_tok [B], committed_tok [B,path_cap]);
    `out` may supply these four int32 device tensors."""
    return _native.tree_accept(parent, draft_tok, amax, num_nodes, path_cap, err_flag, out, stream)


def specvlm_tree_accept_sample(parent, draft_tok, logits, u_accept, u_bonus, *, temperature=1.0, num_nodes=None,
                               path_cap=8, err_flag=None, out=None, stream=None):
    """Sampling-based acceptance (temperature > 0).  logits [B,N_max,V]; u_accept [B,N_max] and u_bonus [B]
    fp32 uniform numbers in [0,1).  Returns (accept_len, path, bonus_tok, committed_tok) like
    specvlm_tree_accept."""
    return _native.tree_accept_sample(parent, draft_tok, logits, u_accept, u_bonus, temperature, num_nodes, path_cap, err_flag,
                                      out, stream)


def specvlm_kv_compact(k_caches, v_caches, prefix_len, path, accept_len, *, block_table=None,
                       new_prefix_len=None, moved_idx=None, layer_ptrs=None, err_flag=None, stream=None):
    """In-place compaction.  k_caches/v_caches: one tensor [L, <per-layer cache dims>] (layer stride taken
    from the tensor), or with `layer_ptrs=(k_ptrs, v_ptrs)` (int64 device tensors of L addresses) a single
    layer's tensor that only provides the geometry.  Returns (new_prefix_len, moved_idx)."""
    k_ptrs, v_ptrs = (None, None) if layer_ptrs is None else layer_ptrs
    return _native.kv_compact(k_caches, v_caches, prefix_len, path, accept_len, block_table, new_prefix_len, moved_idx, k_ptrs,
                              v_ptrs, err_flag, stream)


def specvlm_draft_topk(logits, K, *, cum=None, parent_idx=None, score_out=None, token_out=None, parent_out=None,
                       lse_out=None, stream=None):
    """One level of draft-tree growth.  logits [B,W,V]; cum fp32 / parent_idx int32 [B,W] (row strides are
    taken from the tensors, so they may be views).  Outputs are [B, >= W*K] fp32 / int32 tensors or views
    (row stride taken from score_out; token_out and parent_out must share it): entry (b, w*K + k).
    Returns (score_out, token_out, parent_out)."""
    return _native.draft_topk(logits, K, cum, parent_idx, score_out, token_out, parent_out, lse_out, stream)


def specvlm_draft_topk_select(logits, K, M, *, cum=None, parent_idx=None, score_out=None, token_out=None,
                              parent_out=None, lse_out=None, index_base=0, sel_out=None, sel_score_out=None,
                              count_out=None, counters=None, stream=None):
    """specvlm_draft_topk and the selection of the M best of the level's W*K new candidates in one launch.
    `counters` is an int32 [B * COUNTER_STRIDE] device tensor, zero-filled once (allocated here when
    omitted).  Returns (score_out, token_out, parent_out, sel_out, sel_score_out, count_out)."""
    return _native.draft_topk_select(logits, K, M, cum, parent_idx, score_out, token_out, parent_out, lse_out, index_base, sel_out,
                                     sel_score_out, count_out, counters, stream)


def specvlm_draft_select(score, M, *, num_cand=None, index_base=0, sel_out=None, sel_score_out=None,
                         count_out=None, stream=None):
    """score fp32 [B,C] (may be a view of a wider array).  Returns (sel [B,M] int32, sel_score [B,M] fp32,
    count [B] int32)."""
    return _native.draft_select(score, M, num_cand, index_base, sel_out, sel_score_out, count_out, stream)


def specvlm_draft_finalize(cand_score, cand_parent, cand_token, root_token, N_max, *, num_cand=None, err_flag=None,
                           out=None, stream=None):
    """Candidates [B,C] (fp32 score, int32 parent and token, one row stride) -> (parent [B,N_max],
    draft_tok [B,N_max], node_cand [B,N_max], num_nodes [B]); `out` may supply these four int32 tensors."""
    return _native.draft_finalize(cand_score, cand_parent, cand_token, root_token, N_max, num_cand, err_flag, out, stream)


def specvlm_head_argmax_workspace_bytes(B, N_max, V) -> int:
    return int(lib().specvlm_head_argmax_workspace_bytes(B, N_max, V))


def specvlm_head_argmax(hidden, weight, *, num_nodes=None, out=None, max_logit=None, workspace=None, stream=None):
    """Output head fused with the greedy choice.  hidden [B,N_max,E] bf16, weight [V,E] bf16 ->
    amax [B,N_max] int32 (and the greatest logit into `max_logit` fp32 [B,N_max] if given)."""
    return _native.head_argmax(hidden, weight, num_nodes, out, max_logit, workspace, stream)


def specvlm_visual_pool(x, ratio, *, num_tokens=None, out=None, out_tokens=None, err_flag=None, stream=None):
    """Average pooling along the token sequence (window = stride = ratio, ragged last window).
    x [B,T,E] -> (y [B,ceil(T/ratio),E], out_tokens [B] int32)."""
    return _native.visual_pool(x, ratio, num_tokens, out, out_tokens, err_flag, stream)


def specvlm_visual_prune(x, keep, *, out=None, err_flag=None, stream=None):
    """Pruning as a gather: x [B,T,E], keep [B,T_keep] int32 (-1 = padding) -> y [B,T_keep,E]."""
    return _native.visual_prune(x, keep, out, err_flag, stream)


def specvlm_node_argmax_accept(logits, parent, draft_tok, *, num_nodes=None, path_cap=8, counters=None, amax=None,
                               err_flag=None, out=None, stream=None):
    """specvlm_node_argmax + specvlm_tree_accept in one launch.  `counters` is an int32
    [B * COUNTER_STRIDE] device tensor, zero-filled once (allocated here when omitted).
    Returns (amax, accept_len, path, bonus_tok, committed_tok)."""
    return _native.node_argmax_accept(logits, parent, draft_tok, num_nodes, path_cap, counters, amax, err_flag, out, stream)
