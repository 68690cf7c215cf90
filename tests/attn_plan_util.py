"""How the library divides a bf16 attention call among workgroups, from the same header as the library (built with g++)."""
from __future__ import annotations

import atexit
import collections
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# columns: workgroups per row block of a KV head in the kernel with a key stream per wavefront, 0 where one of the others takes the call (by
# row blocks, or by key ranges where block_rows is 0); by_length: the requests' lengths deal them out; streams: key ranges of a request otherwise
Plan = collections.namedtuple("Plan", "ranges block_rows splits streams columns by_length", defaults=[0, 0, 0])

SOURCE = r"""
#include "attn_plan.hpp"
extern "C" void plan(const specvlm_attn_desc* d, int* out) {
    const specvlm::AttnPlan p = specvlm::attn_plan(*d);
    out[0] = p.ranges; out[1] = p.block_rows; out[2] = p.splits; out[3] = p.streams; out[4] = p.columns; out[5] = p.by_length;
}
extern "C" void columns(const specvlm_attn_desc* d, long long* out) {
    const specvlm::AttnPlan p = specvlm::attn_plan(*d), e = specvlm::evenly(*d, p);
    out[0] = p.columns; out[1] = p.by_length; out[2] = specvlm::attn_workspace_bytes(*d, p);
    out[3] = e.columns; out[4] = e.by_length; out[5] = specvlm::attn_workspace_bytes(*d, e);
}
"""


@functools.lru_cache(None)
def compiled(source):
    """A C++ source over the library's host headers, as a loaded shared object."""
    tmp = tempfile.mkdtemp()
    atexit.register(shutil.rmtree, tmp, ignore_errors=True)
    src, so = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2509_11815_amd", "csrc"), src, "-o", so], check=True)
    return ctypes.CDLL(so)


def _library():
    return compiled(SOURCE)


def plan_of_desc(desc) -> Plan:
    out = (ctypes.c_int * 6)()
    _library().plan(ctypes.byref(desc), out)
    return Plan(*out)


def desc_of(B, Hq, Hkv, D, N, cap, num_splits=0, paged=False, token_stride=None):
    """Dense tensors of these sizes; `cap` slots per request (a multiple of 16 when paged)."""
    import paper_2509_11815_amd.binding as b
    t = D if token_stride is None else token_stride
    return b.AttnDesc(
        dtype=b.SPECVLM_BF16, B=B, H_q=Hq, H_kv=Hkv, D=D, N_max=N, paged=int(paged), block_size=16 * paged, max_blocks_per_req=cap // 16 * paged,
        num_blocks=B * (cap // 16) * paged, kv_capacity=cap, num_splits=num_splits, q_stride_b=N * Hq * D, q_stride_n=Hq * D,
        q_stride_h=D, o_stride_b=N * Hq * D, o_stride_n=Hq * D, o_stride_h=D, kv_stride_b=Hkv * cap * t, kv_stride_h=cap * t, kv_stride_t=t)


def streams_of(*shape, **options) -> int:
    """Key ranges of a request in the kernel with a key stream per wavefront, evenly divided; 0 where the call has another division."""
    return plan_of(*shape, **options).streams


def division_of(*shape, **options) -> tuple[int, int]:
    """In the kernel with a key stream per wavefront: key ranges of a request, and whether the lengths divide them instead.  A call that the
    lengths divide is divided evenly where it has no workspace for that."""
    plan = plan_of(*shape, **options)
    assert plan.columns
    return plan.streams, plan.by_length


def plan_of(*shape, **options) -> Plan:
    return plan_of_desc(desc_of(*shape, **options))


def plan_of_case(case, num_splits=0) -> Plan:
    """The plan of a problem from gpu_util.random_case()."""
    B, N, Hq, D = case["q"].shape
    Hkv, table = case["k"].shape[1], case["block_table"]
    cap = case["k"].shape[2] if table is None else table.shape[1] * 16
    return plan_of(B, Hq, Hkv, D, N, cap, num_splits, table is not None)


Columns = collections.namedtuple("Columns", "columns by_length bytes even_columns even_by_length even_bytes")


def columns_of(*shape, **options) -> Columns:
    """Workgroups per row block of a KV head, whether the lengths deal them out, workspace bytes; the same for a call that has not that much."""
    out = (ctypes.c_longlong * 6)()
    _library().columns(ctypes.byref(desc_of(*shape, **options)), out)
    return Columns(*out)
