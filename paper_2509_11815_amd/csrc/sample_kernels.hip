// Per-node vocab argmax, greedy acceptance walk and KV compaction (the T_sample part of a
// speculative round, SpecVLM Sec. 3.1 Eq. 1, plus the cache bookkeeping that follows it).
#include <limits.h>

#include "common.hpp"
#include "compact_plan.hpp"
#include "wave_ops.hpp"

namespace specvlm {

// ---------------------------------------------------------------------------------------
// node_argmax: one 1024-thread workgroup per (request, node) row.  A row of 32000 bf16
// logits is 64 KB: 16-byte loads, (value, index) kept per thread, reduced with the
// "greater value, then lower index" order, which is associative and commutative, so the
// result does not depend on the reduction shape.  Bound by a row's bytes into one compute unit and,
// fused, by the chain from the last row to the walk: wavefronts meet once in LDS, the first one goes on
// alone in registers.  us per launch, with LDS permutes, two more barriers and a walk of dependent LDS reads
// -> now, launches back to back: 60 rows of 32000 bf16 7.3 -> 6.3, 480 11.1 -> 10.3, 256 of 152064 19.65 -> 18.7; behind a
// step's attention calls in a kernel trace 7.25 -> 6.0, 13.0 -> 11.6, 17.6 -> 15.6 (a whole step of eight requests,
// 634 us, shows no difference).  (The next four loads ahead of these: 152064 entries + 0.8; the tree behind the row's
// first loads: even.)
// ---------------------------------------------------------------------------------------
struct ValIdx {
    float v;
    int i;
};

// i is greater than every index taken so far (a thread scans its entries in increasing order), so only "greater" replaces.
// -0 == +0 under the float compare, as the definition asks.
__device__ __forceinline__ void take_later(ValIdx& a, float v, int i) {
    if (v > a.v) {
        a.v = v;
        a.i = i;
    }
}

// op over the 64 lanes, in every one of them: rows of 16 by DPP, then across rows (6 LDS permutes in a row take 0.4 us, this 0.05).
template <typename Op>
__device__ __forceinline__ int over_wave(int x, Op op) {
    x = op(x, dpp<kRor8>(x));
    x = op(x, dpp<kRor4>(x));
    x = op(x, dpp<kRor2>(x));
    x = op(x, dpp<kRor1>(x));
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = op(static_cast<int>(r[0]), static_cast<int>(r[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return op(static_cast<int>(q[0]), static_cast<int>(q[1]));
}

// The best of the 64 lanes, in every one: the greatest value, the lowest index among its equals (no lane holds NaN).
__device__ __forceinline__ ValIdx best_of_wave(ValIdx a) {
    const int bits = over_wave(__float_as_int(a.v), [](int x, int y) { return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y))); });
    const float v = __int_as_float(bits);
    return ValIdx{v, over_wave(a.v == v ? a.i : INT_MAX, [](int x, int y) { return min(x, y); })};
}

template <typename T>
struct Elem;
template <>
struct Elem<uint16_t> {
    static constexpr int kPerVec = 8;
    __device__ static float at(const uint4& w, int e) {
        uint32_t x = (&w.x)[e >> 1];
        return __uint_as_float((e & 1) ? (x & 0xFFFF0000u) : (x << 16));
    }
    __device__ static float one(const uint16_t* p) { return bf16_bits_to_float(*p); }
};
template <>
struct Elem<float> {
    static constexpr int kPerVec = 4;
    __device__ static float at(const uint4& w, int e) { return __uint_as_float((&w.x)[e]); }
    __device__ static float one(const float* p) { return *p; }
};

// (defined with the acceptance kernel below)
template <bool COHERENT>
__device__ __forceinline__ void accept_walk(int b, int n, int N_max, int path_cap, int par, int tok, const int32_t* amax,
                                            int32_t* __restrict__ accept_len, int32_t* __restrict__ path,
                                            int32_t* __restrict__ bonus_tok, int32_t* __restrict__ committed_tok,
                                            int32_t* __restrict__ err_flag);

// What the fused form needs on top of the arg-max: the acceptance walk's arguments and one
// arrival counter per request (zero between calls).
struct AcceptArgs {
    int path_cap;
    const int32_t *parent, *draft_tok;
    int32_t *accept_len, *path, *bonus_tok, *committed_tok, *err_flag;
    int32_t* counters;
};

// FUSED: the workgroup that finishes the last row of a request (ticket counter) also runs the
// greedy acceptance walk of that request, so arg-max + acceptance is one launch.
template <typename T, bool FUSED>
__global__ __launch_bounds__(1024) void node_argmax_kernel(int N_max, int V, const T* __restrict__ logits,
                                                           int64_t stride_b, int64_t stride_n,
                                                           const int32_t* __restrict__ num_nodes,
                                                           int32_t* amax, AcceptArgs acc) {
    const int row = blockIdx.x;
    const int b = row / N_max, i = row % N_max;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n = num_nodes ? num_nodes[b] : N_max;
    // what the walk will need of the tree: requested ahead of the row (the request's last row walks, and any may be the last)
    int par = -1, tok = -1;
    if (FUSED && tid < N_max) {
        par = acc.parent[b * N_max + tid];
        tok = acc.draft_tok[b * N_max + tid];
    }
    // publishes this row's result; FUSED: then draws the request's ticket, and the wavefront that
    // draws the last one walks the tree (called by wavefront 0)
    auto finish = [&](int result) {
        if constexpr (!FUSED) {
            if (lane == 0) amax[row] = result;
        } else {
            int last = 0;
            if (lane == 0) {
                __hip_atomic_store(amax + row, result, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the store has been acknowledged
                int32_t* cnt = acc.counters + b * SPECVLM_COUNTER_STRIDE;     // a cache line per request
                last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == N_max - 1;
                if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (__builtin_amdgcn_readfirstlane(last)) {
                asm volatile("" ::: "memory");                          // the other rows' results are not read before the ticket was seen
                accept_walk<true>(b, n, N_max, acc.path_cap, par, tok, amax, acc.accept_len, acc.path, acc.bonus_tok, acc.committed_tok,
                                  acc.err_flag);
            }
        }
    };
    if (i >= n) {
        if (wave == 0) finish(-1);
        return;
    }
    const T* p = logits + b * stride_b + i * stride_n;
    constexpr int VEC = Elem<T>::kPerVec;
    ValIdx best{-INFINITY, INT_MAX};

    // scalar head up to the first 16-byte boundary, vector body, scalar tail
    int head = static_cast<int>(((16u - (reinterpret_cast<uintptr_t>(p) & 15u)) & 15u) / sizeof(T));
    head = min(head, V);
    // (every thread meets its entries in increasing index order: head, vector body, tail)
    for (int v = tid; v < head; v += blockDim.x) take_later(best, Elem<T>::one(p + v), v);
    const int nvec = (V - head) / VEC;
    const uint4* pv = reinterpret_cast<const uint4*>(p + head);
    // four 16-byte loads per thread are requested before the first is looked at (a row of 32000 bf16
    // logits is four per thread: one memory round trip instead of four in a row)
    for (int c0 = tid; c0 < nvec; c0 += 4 * blockDim.x) {
        uint4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * blockDim.x;
            if (c < nvec) w[u] = pv[c];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * blockDim.x;
            if (c < nvec) {
                const int base = head + c * VEC;
#pragma unroll
                for (int e = 0; e < VEC; ++e) take_later(best, Elem<T>::at(w[u], e), base + e);
            }
        }
    }
    for (int v = head + nvec * VEC + tid; v < V; v += blockDim.x) take_later(best, Elem<T>::one(p + v), v);

    // wavefront (64 lanes) reduction, then across the 16 wavefronts through LDS
    if constexpr (FUSED) asm volatile("" : "+v"(par), "+v"(tok));       // not to be loaded where they are used
    best = best_of_wave(best);
    __shared__ ValIdx s_best[16];
    if (lane == 0) s_best[wave] = best;
    __syncthreads();
    if (wave) return;
    const ValIdx r = best_of_wave(s_best[lane & 15]);
    finish(r.i == INT_MAX ? 0 : r.i);
}

int32_t launch_node_argmax(int32_t dtype, int32_t B, int32_t N_max, int32_t V, const void* logits,
                           int64_t stride_b, int64_t stride_n, const int32_t* num_nodes,
                           int32_t* amax, hipStream_t stream) {
    dim3 grid(B * N_max), block(1024);
    const AcceptArgs none{};
    if (dtype == SPECVLM_BF16)
        hipLaunchKernelGGL((node_argmax_kernel<uint16_t, false>), grid, block, 0, stream, N_max, V,
                           static_cast<const uint16_t*>(logits), stride_b, stride_n, num_nodes, amax, none);
    else
        hipLaunchKernelGGL((node_argmax_kernel<float, false>), grid, block, 0, stream, N_max, V,
                           static_cast<const float*>(logits), stride_b, stride_n, num_nodes, amax, none);
    return check_launch();
}

int32_t launch_node_argmax_accept(int32_t dtype, int32_t B, int32_t N_max, int32_t V, int32_t path_cap,
                                  const void* logits, int64_t stride_b, int64_t stride_n, const int32_t* num_nodes,
                                  const int32_t* parent, const int32_t* draft_tok, int32_t* amax, int32_t* accept_len,
                                  int32_t* path, int32_t* bonus_tok, int32_t* committed_tok, int32_t* counters,
                                  int32_t* err_flag, hipStream_t stream) {
    dim3 grid(B * N_max), block(1024);
    const AcceptArgs acc{path_cap, parent, draft_tok, accept_len, path, bonus_tok, committed_tok, err_flag, counters};
    if (dtype == SPECVLM_BF16)
        hipLaunchKernelGGL((node_argmax_kernel<uint16_t, true>), grid, block, 0, stream, N_max, V,
                           static_cast<const uint16_t*>(logits), stride_b, stride_n, num_nodes, amax, acc);
    else
        hipLaunchKernelGGL((node_argmax_kernel<float, true>), grid, block, 0, stream, N_max, V,
                           static_cast<const float*>(logits), stride_b, stride_n, num_nodes, amax, acc);
    return check_launch();
}

// ---------------------------------------------------------------------------------------
// tree_accept: one wavefront per request, lane i owns node i.  Pointer doubling tells every lane whether its
// node's path to the root is accepted and how deep it is (parent[i] < i: at most six rounds, three for
// trees of depth 7); a wavefront max over (depth, -index) picks the node, whose path is read back lane by lane.
// Registers and permutes only: the chain of the last row of a request in the fused form.  One wavefront calls.
// par, tok: node lane's, anything where lane >= n.  COHERENT: amax was written by other workgroups of the same
// kernel (device-coherent loads); otherwise by an earlier kernel.
// ---------------------------------------------------------------------------------------
template <bool COHERENT>
__device__ __forceinline__ void accept_walk(int b, int n, int N_max, int path_cap, int par, int tok, const int32_t* amax,
                                            int32_t* __restrict__ accept_len, int32_t* __restrict__ path,
                                            int32_t* __restrict__ bonus_tok, int32_t* __restrict__ committed_tok,
                                            int32_t* __restrict__ err_flag) {
    const int lane = threadIdx.x;
    int err = 0;
    if (n < 1 || n > N_max) {
        err |= SPECVLM_ERR_BAD_NUM_NODES;
        n = min(max(n, 1), N_max);
    }
    const bool real = lane < n;
    int am = -1;
    if (real) {
        if constexpr (COHERENT)
            am = __hip_atomic_load(amax + b * N_max + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            am = amax[b * N_max + lane];
    }
    const bool bad = real && (lane == 0 ? par != -1 : (par < 0 || par >= lane));
    int best = 0, m = 0;
    if (__any(bad)) {                       // malformed tree: commit the root only
        err |= SPECVLM_ERR_BAD_PARENT;
    } else {
        int up = real ? par : -1, depth = up >= 0 ? 1 : 0;
        const int wanted = __builtin_amdgcn_ds_bpermute(max(up, 0) * 4, am);      // (every lane takes part)
        bool ok = real && (up < 0 || tok == wanted);
        while (__any(up >= 0)) {
            const int at = __builtin_amdgcn_ds_bpermute(max(up, 0) * 4, (up + 1) | depth << 8 | static_cast<int>(ok) << 16);
            if (up >= 0) {
                ok = ok && (at >> 16);
                depth += (at >> 8) & 255;
                up = (at & 255) - 1;
            }
        }
        const bool too_long = ok && depth > path_cap - 1;
        if (__any(too_long)) err |= SPECVLM_ERR_PATH_TOO_LONG;
        const int key = over_wave(ok && !too_long ? depth * 64 + (63 - lane) : -1, [](int x, int y) { return max(x, y); });   // deeper first, then lower index
        best = __builtin_amdgcn_readfirstlane(63 - (key & 63));
        m = __builtin_amdgcn_readfirstlane(key >> 6);
    }
    // lane j: the path's node j, and the token it commits
    int node = -1, t = best;
    for (int j = m; j >= 0; --j) {
        if (lane == j) node = t;
        t = __builtin_amdgcn_readlane(par, t);
    }
    const int bonus = __builtin_amdgcn_readlane(am, best);
    const int node_tok = __builtin_amdgcn_ds_bpermute(max(node, 0) * 4, tok);
    const int next_tok = __builtin_amdgcn_ds_bpermute((lane + 1) * 4, node_tok);
    int32_t* prow = path + b * path_cap;
    int32_t* crow = committed_tok + b * path_cap;
    if (lane < path_cap) {                  // (at most 64: checked on the host)
        prow[lane] = node;
        crow[lane] = lane < m ? next_tok : lane == m ? bonus : -1;
    }
    if (lane == 0) {
        accept_len[b] = m;
        bonus_tok[b] = bonus;
        if (err && err_flag) atomicOr(err_flag, err);
    }
}

__global__ __launch_bounds__(64) void tree_accept_kernel(int N_max, int path_cap,
                                                         const int32_t* __restrict__ parent,
                                                         const int32_t* __restrict__ draft_tok,
                                                         const int32_t* __restrict__ amax,
                                                         const int32_t* __restrict__ num_nodes,
                                                         int32_t* __restrict__ accept_len,
                                                         int32_t* __restrict__ path,
                                                         int32_t* __restrict__ bonus_tok,
                                                         int32_t* __restrict__ committed_tok,
                                                         int32_t* __restrict__ err_flag) {
    const int b = blockIdx.x, lane = threadIdx.x;
    int par = -1, tok = -1;
    if (lane < N_max) {
        par = parent[b * N_max + lane];
        tok = draft_tok[b * N_max + lane];
    }
    accept_walk<false>(b, num_nodes ? num_nodes[b] : N_max, N_max, path_cap, par, tok, amax, accept_len, path, bonus_tok, committed_tok,
                       err_flag);
}

int32_t launch_tree_accept(int32_t B, int32_t N_max, int32_t path_cap, const int32_t* parent,
                           const int32_t* draft_tok, const int32_t* amax, const int32_t* num_nodes,
                           int32_t* accept_len, int32_t* path, int32_t* bonus_tok,
                           int32_t* committed_tok, int32_t* err_flag, hipStream_t stream) {
    hipLaunchKernelGGL(tree_accept_kernel, dim3(B), dim3(64), 0, stream, N_max, path_cap, parent,
                       draft_tok, amax, num_nodes, accept_len, path, bonus_tok, committed_tok, err_flag);
    return check_launch();
}

// ---------------------------------------------------------------------------------------
// kv_compact: one 256-thread workgroup per (layer, K|V, request, group of up to 8 KV heads).  The rows of
// the accepted path (<= 64 rows of <= 512 bytes) of these heads are read into registers as 16-byte
// chunks, the workgroup synchronises, then the chunks are written to their destination
// rows: gather semantics even though source and destination ranges overlap.  Rows that
// do not move (path[j] == j, always true for the root) are skipped.
// A workgroup's few loads and stores are one chain of latencies, so with many of them it is their number that
// counts: 32 layers x 8 requests x 32 heads with a workgroup per head (16384) 13.8 us, 2048 of them 4.0 (compact_plan.hpp).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kCompactThreads) void kv_compact_kernel(
    KvGeom g, unsigned char* k_base, unsigned char* v_base, int64_t layer_stride_bytes,
    void* const* k_ptrs, void* const* v_ptrs, int elem_bytes, int chunk_bits, int head_bits, int H_kv,
    const int32_t* __restrict__ prefix_len, const int32_t* __restrict__ path, int path_cap,
    const int32_t* __restrict__ accept_len, int32_t* __restrict__ new_prefix_len, int32_t* __restrict__ moved_idx,
    int32_t* __restrict__ err_flag) {
    const int l = blockIdx.x >> 1, which = blockIdx.x & 1;
    const int b = blockIdx.z, tid = threadIdx.x;
    const int hk0 = blockIdx.y << head_bits;
    // chunk idx of the workgroup: row j of the path, head of the group, chunk of the row
    const int bits = chunk_bits + head_bits;
    int a[kCompactChunksPerThread];
#pragma unroll
    for (int c = 0; c < kCompactChunksPerThread; ++c) {
        if (c * kCompactThreads >> bits >= path_cap) break;         // uniform: no thread has so many
        const int j = (tid + c * kCompactThreads) >> bits;
        a[c] = path[b * path_cap + min(j, path_cap - 1)];
    }
    // new_prefix_len is given here only when it does not alias prefix_len (which every workgroup
    // of the request reads): then the request's first workgroup writes the bookkeeping outputs
    if (new_prefix_len && blockIdx.x == 0 && blockIdx.y == 0 && tid < path_cap) {
        const int P0 = prefix_len[b];
        const int m0 = min(max(accept_len[b], 0), path_cap - 1);
        if (moved_idx) {
            moved_idx[(b * path_cap + tid) * 2 + 0] = tid <= m0 ? P0 + path[b * path_cap + tid] : -1;
            moved_idx[(b * path_cap + tid) * 2 + 1] = tid <= m0 ? P0 + tid : -1;
        }
        if (tid == 0) new_prefix_len[b] = P0 + m0 + 1;
    }
    unsigned char* base;
    if (k_ptrs)
        base = static_cast<unsigned char*>(which ? v_ptrs[l] : k_ptrs[l]);
    else
        base = (which ? v_base : k_base) + l * layer_stride_bytes;
    const int P = prefix_len[b];
    const int m = min(max(accept_len[b], 0), path_cap - 1);
    uint4 regs[kCompactChunksPerThread];
    int64_t dst_off[kCompactChunksPerThread];
#pragma unroll
    for (int c = 0; c < kCompactChunksPerThread; ++c) {
        const int idx = tid + c * kCompactThreads;
        const int ch = idx & ((1 << chunk_bits) - 1), hk = hk0 + ((idx >> chunk_bits) & ((1 << head_bits) - 1));
        const int j = idx >> bits;
        dst_off[c] = -1;
        regs[c] = uint4{0u, 0u, 0u, 0u};
        if (c * kCompactThreads >> bits >= path_cap) continue;      // uniform
        // a row moves only if it is a valid, different slot inside the cache
        if (j <= m && hk < H_kv && a[c] != j && a[c] < SPECVLM_MAX_NODES && slot_inside(P, a[c], g.capacity) && slot_inside(P, j, g.capacity)) {
            bool bad_block = false;
            const int64_t src = kv_row_offset(g, b, hk, P + a[c], bad_block) * elem_bytes + ch * 16;
            const int64_t dst = kv_row_offset(g, b, hk, P + j, bad_block) * elem_bytes + ch * 16;
            if (!bad_block) {                      // a row whose block id is out of range stays where it is
                regs[c] = *reinterpret_cast<const uint4*>(base + src);
                dst_off[c] = dst;
            } else if (err_flag && ch == 0 && blockIdx.x == 0 && hk == 0) {
                atomicOr(err_flag, SPECVLM_ERR_BAD_BLOCK);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kCompactChunksPerThread; ++c)
        if (dst_off[c] >= 0) *reinterpret_cast<uint4*>(base + dst_off[c]) = regs[c];
}

__global__ void kv_compact_finish_kernel(int B, const int32_t* __restrict__ prefix_len,
                                         const int32_t* __restrict__ path, int path_cap,
                                         const int32_t* __restrict__ accept_len,
                                         int32_t* new_prefix_len, int32_t* __restrict__ moved_idx) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int P = prefix_len[b];
    const int m = min(max(accept_len[b], 0), path_cap - 1);
    if (moved_idx)
        for (int j = 0; j < path_cap; ++j) {
            moved_idx[(b * path_cap + j) * 2 + 0] = j <= m ? P + path[b * path_cap + j] : -1;
            moved_idx[(b * path_cap + j) * 2 + 1] = j <= m ? P + j : -1;
        }
    new_prefix_len[b] = P + m + 1;
}

int32_t launch_kv_compact(const specvlm_attn_desc& d, int32_t L, void* k_base, void* v_base,
                          int64_t layer_stride, void* const* k_ptrs, void* const* v_ptrs,
                          const int32_t* block_table, const int32_t* prefix_len, const int32_t* path,
                          int32_t path_cap, const int32_t* accept_len, int32_t* new_prefix_len,
                          int32_t* moved_idx, int32_t* err_flag, hipStream_t stream) {
    const int eb = d.dtype == SPECVLM_BF16 ? 2 : 4;
    KvGeom g{d.kv_stride_b, d.kv_stride_h, d.kv_stride_t, d.paged ? block_table : nullptr,
             d.max_blocks_per_req, d.num_blocks,
             d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity};
    const int chunk_bits = __builtin_ctz(d.D * eb / 16);           // (8, 16 or 32 chunks of a row)
    const int head_bits = compact_head_bits(static_cast<int64_t>(L) * 2 * d.B * d.H_kv, path_cap << chunk_bits);
    dim3 grid(L * 2, (d.H_kv + (1 << head_bits) - 1) >> head_bits, d.B);
    // One launch when new_prefix_len is a buffer of its own; when it aliases prefix_len it may only
    // be written after every workgroup has read the old lengths: a second, tiny launch.
    const bool alias = new_prefix_len == prefix_len;
    hipLaunchKernelGGL(kv_compact_kernel, grid, dim3(kCompactThreads), 0, stream, g,
                       static_cast<unsigned char*>(k_base), static_cast<unsigned char*>(v_base),
                       layer_stride * eb, k_ptrs, v_ptrs, eb, chunk_bits, head_bits, d.H_kv, prefix_len, path,
                       path_cap, accept_len, alias ? nullptr : new_prefix_len, alias ? nullptr : moved_idx, err_flag);
    int32_t rc = check_launch();
    if (rc || !alias) return rc;
    hipLaunchKernelGGL(kv_compact_finish_kernel, dim3((d.B + 63) / 64), dim3(64), 0, stream, d.B,
                       prefix_len, path, path_cap, accept_len, new_prefix_len, moved_idx);
    return check_launch();
}

}  // namespace specvlm
