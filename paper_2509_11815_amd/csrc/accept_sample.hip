// Sampling-based acceptance walk over a draft tree (temperature > 0).
//
// SpecVLM Sec. 3.1 names speculative sampling as the rule that discards drafted tokens and
// Sec. 4.1 evaluates temperature 1 with the same Top-K tree.  The children of a tree node are
// fixed candidates (top-K expansion), i.e. point-mass proposals, so a child c with token x is
// accepted when its uniform number is below the residual target probability of x at the
// parent, p(x) / (1 - mass already rejected there); a rejected token leaves the distribution;
// the bonus token is drawn from the residual distribution of the last node by inverse CDF in
// vocabulary order.  Every emitted token then follows the target's own distribution.
//
// One 1024-thread workgroup per request.  The walk is sequential (at most path_cap levels) on one compute
// unit, so it is bound by latencies and by the instructions of passes over a vocabulary row.
//   row       up to 64 consecutive tokens per thread stay in registers (CH = 32, 64); the root's row is requested
//             before the tree is looked at.  Larger vocabularies (CH = 0): one pass for the maximum (16-byte
//             loads), one for the sum of exp2((l - max) log2e / T), and one for the bonus draw's chunk sums in 16-byte loads.
//   sums      in a fixed order, so that the same input gives the same decision whatever the timing; lanes
//             meet by DPP and lane swaps in the order of an xor butterfly (32, 16, 8, 4, 2, 1), then the 16
//             wavefronts through LDS in order
//   children  wavefront 0 holds a child per lane: what the earlier ones have taken is a running sum over lanes,
//             then all acceptance thresholds are computed at once and the first accepted child is a bit scan
//   bonus     a two-level scan: every thread sums a contiguous chunk of the vocabulary, the chunk sums are
//             scanned, and the chunk that contains the drawn position is walked (CH = 0: its probabilities are
//             computed by the whole workgroup first)
// Kernel alone, 4 requests, bf16: 32000 tokens 10.9 us, 20003 13.3, 60000 22.7, 65536 17.7, 152064 34.4 (beyond 65536, passes that
// read token by token took 198 us).
#include "chunk_vectors.hpp"
#include "wave_ops.hpp"

namespace specvlm {

namespace {

constexpr int kThreadsAS = 1024;
constexpr int kWalk = 2048;              // CH == 0: longest chunk whose probabilities are laid out in LDS

template <typename T>
__device__ __forceinline__ float logit_at(const T* p, int v);
template <>
__device__ __forceinline__ float logit_at<uint16_t>(const uint16_t* p, int v) { return bf16_bits_to_float(p[v]); }
template <>
__device__ __forceinline__ float logit_at<float>(const float* p, int v) { return p[v]; }

// Sum over the wavefront in the order of an xor butterfly with offsets 32, 16, 8, 4, 2, 1 (every lane gets it).
__device__ __forceinline__ float butterfly_sum(float x) {
    const uint32_t a = __float_as_uint(x);
    const auto r32 = __builtin_amdgcn_permlane32_swap(a, a, false, false);       // lower half everywhere, upper half everywhere
    x = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
    const uint32_t c = __float_as_uint(x);
    const auto r16 = __builtin_amdgcn_permlane16_swap(c, c, false, false);       // even rows, odd rows
    x = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
    return row_sum(x);                   // all rows are equal by now: a rotation by 8, 4, 2, 1 meets the xor partner's value
}

__device__ __forceinline__ float block_max(float x, float* s_red) {
    x = wave_max(x);
    __syncthreads();                                   // s_red may still be read from a previous call
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = x;
    __syncthreads();
    return row_max(s_red[threadIdx.x & 15]);
}

__device__ __forceinline__ float block_sum(float x, float* s_red) {
    x = butterfly_sum(x);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) s_red[wave] = x;
    __syncthreads();
    float r = s_red[0];
#pragma unroll
    for (int w = 1; w < kThreadsAS / 64; ++w) r += s_red[w];
    return r;
}

// Eight (bf16) or four (fp32) consecutive logits.
template <typename T>
__device__ __forceinline__ float vec_at(const uint4& w, int e) {
    const uint32_t x = (&w.x)[sizeof(T) == 2 ? e >> 1 : e];
    if constexpr (sizeof(T) == 2) return __uint_as_float((e & 1) ? (x & 0xFFFF0000u) : (x << 16));
    else return __uint_as_float(x);
}

// CH > 0: every thread keeps its chunk of the current row (at most CH consecutive tokens) in
// registers, loaded once per level with 16-byte loads; WHOLE: the chunks of every row are whole aligned vectors.
// (CH = 64 without WHOLE does not quite fit its 128 registers: 164 bytes of scratch a lane in fp32, 8 in bf16.  Reading such fp32 rows
// again, as CH = 0 does, is faster by up to a third - 4 requests of 50001 tokens 24.6 us here, 17.2 there - but adds in another order.)
// (Two kernels: with both ways of loading in one, 4 requests of 32000 tokens took 12.5 us in place of 10.9, 65536 22.8 of 17.7.)
// CH == 0: any vocabulary size, every pass reads the row again (from L2).
template <typename T, int CH, bool WHOLE>
__global__ __launch_bounds__(kThreadsAS) void tree_accept_sample_kernel(
    int N_max, int V, int path_cap, const int32_t* __restrict__ parent, const int32_t* __restrict__ draft_tok,
    const T* __restrict__ logits, int64_t stride_b, int64_t stride_n, const int32_t* __restrict__ num_nodes,
    float temperature, const float* __restrict__ u_accept, const float* __restrict__ u_bonus,
    int32_t* __restrict__ accept_len, int32_t* __restrict__ path, int32_t* __restrict__ bonus_tok,
    int32_t* __restrict__ committed_tok, int32_t* __restrict__ err_flag) {
    __shared__ int s_par[SPECVLM_MAX_NODES], s_tok[SPECVLM_MAX_NODES], s_path[SPECVLM_MAX_NODES];
    __shared__ int s_rej[SPECVLM_MAX_NODES];           // tokens rejected at the current node
    __shared__ float s_red[kThreadsAS / 64];
    __shared__ float s_scan[kThreadsAS];
    __shared__ float s_ev[CH > 0 ? 1 : kWalk];
    __shared__ int s_next, s_nrej, s_err, s_pick, s_chunk;

    const int b = blockIdx.x, tid = threadIdx.x;
    const T* base = logits + b * stride_b;
    const int chunk = (V + kThreadsAS - 1) / kThreadsAS;          // consecutive tokens per thread
    const int v0 = min(tid * chunk, V), v1 = min(v0 + chunk, V);
    constexpr int VEC = 16 / sizeof(T);
    // this thread's logits of the current row, as loaded (entry i of the chunk: vec_at(lv[i / VEC], i % VEC); -inf, i.e.
    // probability 0, past the chunk's end); repack() between passes keeps the compiler from holding a widened copy beside them (16 wavefronts leave 128 registers)
    constexpr int NV = CH > 0 ? CH / VEC : 1;
    uint4 lv[NV];
    constexpr uint32_t kInf = sizeof(T) == 2 ? 0xFF80u : 0xFF800000u, kInfWord = sizeof(T) == 2 ? 0xFF80FF80u : 0xFF800000u;
    // entry `at` of 4 n dwords (if it lies among them) becomes -inf
    auto drop = [&](uint4* w, int n, int at) __attribute__((always_inline)) {
        const int word = sizeof(T) == 2 ? at >> 1 : at, shift = sizeof(T) == 2 ? (at & 1) * 16 : 0;
        const uint32_t keep = sizeof(T) == 2 ? ~(0xFFFFu << shift) : 0u;
#pragma unroll
        for (int d = 0; d < 4 * n; ++d) {
            uint32_t& x = (&w[d >> 2].x)[d & 3];
            x = d == word ? (x & keep) | (kInf << shift) : x;
        }
    };
    auto repack = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NV; ++j) asm volatile("" : "+v"(lv[j].x), "+v"(lv[j].y), "+v"(lv[j].z), "+v"(lv[j].w));
    };
    auto put = [](uint4& w, int e, T value) __attribute__((always_inline)) {     // (a select per dword: e may be known at run time only)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t& x = (&w.x)[d];
            if constexpr (sizeof(T) == 2) {
                const uint32_t y = e & 1 ? (x & 0xFFFFu) | static_cast<uint32_t>(value) << 16 : (x & 0xFFFF0000u) | static_cast<uint32_t>(value);
                x = d == e >> 1 ? y : x;
            } else {
                x = d == e ? __float_as_uint(value) : x;
            }
        }
    };
    auto load_row = [&](const T* row) __attribute__((always_inline)) {
        if constexpr (CH > 0) {
#pragma unroll
            for (int j = 0; j < NV; ++j) lv[j] = uint4{kInfWord, kInfWord, kInfWord, kInfWord};
            if constexpr (WHOLE) {
#pragma unroll
                for (int j = 0; j < NV; ++j)
                    if (v0 + j * VEC < v1) lv[j] = *reinterpret_cast<const uint4*>(row + v0 + j * VEC);
            } else {
                // Most vocabularies: chunks start at any token.  16 bytes a load all the same (gfx950 takes them at any alignment
                // of their type); only the vector that the row ends in is read entry by entry.  (Every entry of its own, bf16:
                // 4 requests of 60000 tokens 39.4 us, now 22.7; 20003 15.5, now 13.3.)
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    const int at = v0 + j * VEC;
                    if (at < v1) {
                        if (at + VEC <= V) {
                            __builtin_memcpy(&lv[j], row + at, 16);
                        } else {
#pragma unroll
                            for (int e = 0; e < VEC - 1; ++e)
                                if (at + e < V) put(lv[j], e, row[at + e]);
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < NV; ++j)
                    if (v0 + j * VEC < v1 && v0 + (j + 1) * VEC > v1)       // the vector that the chunk ends in: entries of the next
#pragma unroll
                        for (int e = 1; e < VEC; ++e)
                            if (v0 + j * VEC + e >= v1) put(lv[j], e, sizeof(T) == 2 ? static_cast<T>(0xFF80u) : static_cast<T>(-INFINITY));
            }
        }
    };
    load_row(base);                                     // the root's row, whatever the tree is
    int err = 0;
    int n = num_nodes ? num_nodes[b] : N_max;
    if (n < 1 || n > N_max) {
        err |= SPECVLM_ERR_BAD_NUM_NODES;
        n = min(max(n, 1), N_max);
    }
    bool bad = false;
    if (tid < SPECVLM_MAX_NODES) {
        int par = -1, tok = -1;
        if (tid < n) {
            par = parent[b * N_max + tid];
            tok = draft_tok[b * N_max + tid];
            bad = tid == 0 ? par != -1 : (par < 0 || par >= tid);
        }
        s_par[tid] = par;
        s_tok[tid] = tok;
    }
    if (tid == 0) s_err = 0;
    if (__syncthreads_or(bad)) {                       // malformed tree: the root has no usable children
        err |= SPECVLM_ERR_BAD_PARENT;
        n = 1;
    }

    int cur = 0, m = 0;
    float mx = 0.f, Z = 0.f, mass = 0.f;               // mass: this thread's share of Z
    // unnormalised probability exp((l - max) / T) as one multiply and one v_exp_f32 (the whole
    // vocabulary goes through it three times on a single compute unit); -inf gives 0
    const float c2 = 1.4426950408889634f / temperature;
    auto prob_of = [&](float l) -> float { return __builtin_amdgcn_exp2f((l - mx) * c2); };
    for (;;) {
        const T* row = base + cur * stride_n;
        // Wavefront 0, lane c: child c's logit and uniform number, requested now so that they
        // arrive while the row is reduced (a dependent load after the reductions would add a
        // memory round trip to every level of the walk).
        bool is_child = false;
        float child_logit = 0.f, child_u = 1.f;
        int child_tok = -1;
        if (tid < SPECVLM_MAX_NODES) {
            is_child = tid > cur && tid < n && s_par[tid] == cur;
            if (is_child) {
                child_tok = s_tok[tid];
                if (child_tok >= 0 && child_tok < V) child_logit = logit_at<T>(row, child_tok);
                child_u = u_accept[b * N_max + tid];
            }
        }
        // target distribution at cur, unnormalised: e(v) = exp((l_v - max) / T)
        float part = -INFINITY;
        if constexpr (CH > 0) {
            if (m > 0) load_row(row);                   // uniform
#pragma unroll
            for (int i = 0; i < CH; ++i)
                part = fmaxf(part, vec_at<T>(lv[i / VEC], i % VEC));
            repack();
        } else {
            const int head = min(static_cast<int>(((16u - (reinterpret_cast<uintptr_t>(row) & 15u)) & 15u) / sizeof(T)), V);
            const int nvec = (V - head) / VEC, tail0 = head + nvec * VEC;
            if (tid < head) part = logit_at<T>(row, tid);
            if (tid >= 64 && tid - 64 < V - tail0) part = logit_at<T>(row, tail0 + tid - 64);
            const uint4* body = reinterpret_cast<const uint4*>(row + head);
#pragma unroll 4
            for (int c = tid; c < nvec; c += kThreadsAS) {
                const uint4 w = body[c];
#pragma unroll
                for (int e = 0; e < VEC; ++e) part = fmaxf(part, vec_at<T>(w, e));
            }
        }
        mx = block_max(part, s_red);
        part = 0.f;
        if constexpr (CH > 0) {
#pragma unroll
            for (int i = 0; i < CH; ++i)
                part += prob_of(vec_at<T>(lv[i / VEC], i % VEC));          // (adding the zeros of -inf changes nothing)
            repack();
        } else {
            // (a thread's tokens are 1024 apart and added in that order; 16 loads in flight)
            int v = tid;
            for (; v + 15 * kThreadsAS < V; v += 16 * kThreadsAS) {
                float l[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) l[u] = logit_at<T>(row, v + u * kThreadsAS);
#pragma unroll
                for (int u = 0; u < 16; ++u) part += prob_of(l[u]);
            }
            for (; v < V; v += kThreadsAS) part += prob_of(logit_at<T>(row, v));
        }
        mass = part;
        Z = block_sum(part, s_red);
        // The children of cur are tried in increasing node index; wavefront 0 holds child c in lane c.
        if (tid < SPECVLM_MAX_NODES) {
            const int lane = tid;
            const bool known = is_child && child_tok >= 0 && child_tok < V;
            const float ex = known ? prob_of(child_logit) : 0.f;
            unsigned long long kids = __ballot(is_child);
            const bool has_child = kids != 0;
            if (m + 1 >= path_cap) kids = 0;           // no room for a deeper node: nothing is tested
            const unsigned long long known_kids = __ballot(known) & kids;
            bool dup = false;                          // an earlier child carries the same token: residual probability 0
            for (unsigned long long k = known_kids; k; k &= k - 1) {
                const int j = __builtin_ctzll(k);
                dup = dup || (lane > j && __builtin_amdgcn_readlane(child_tok, j) == child_tok);
            }
            const bool live = ((known_kids >> lane) & 1ull) && !dup;
            const unsigned long long live_kids = __ballot(live);
            float rejmass = 0.f, gone = 0.f;           // mass of the live children before this lane's
            for (unsigned long long k = live_kids; k; k &= k - 1) {
                const int j = __builtin_ctzll(k);
                if (lane == j) rejmass = gone;
                gone += lane_of(ex, j);
            }
            const float a = ex / fmaxf(Z - rejmass, ex);       // the residual mass holds x itself
            const unsigned long long taken = __ballot(live && child_u < a);
            const int next = taken ? __builtin_ctzll(taken) : -1;
            const unsigned long long tried = taken ? (1ull << next) - 1ull : ~0ull;      // ... and not accepted
            const unsigned long long rejected = live_kids & tried;
            if ((rejected >> lane) & 1ull) s_rej[__popcll(rejected & ((1ull << lane) - 1ull))] = child_tok;
            if (lane == 0) {
                int e = (kids & ~known_kids & tried) ? SPECVLM_ERR_BAD_TOKEN : 0;
                if (has_child && m + 1 >= path_cap) e |= SPECVLM_ERR_PATH_TOO_LONG;
                s_next = next;
                s_nrej = __popcll(rejected);
                s_err |= e;
                s_path[m] = cur;
            }
        }
        __syncthreads();
        const int next = s_next;
        if (next < 0) break;                           // uniform
        cur = next;
        ++m;
        __syncthreads();                               // s_next is rewritten in the next round
    }

    // ---- bonus token: inverse CDF over the residual distribution at cur, in vocabulary order ----
    const T* row = base + cur * stride_n;
    const int nrej = s_nrej;
    float csum = 0.f;
    unsigned long long mine = 0;                       // bit r: rejected token r lies in this thread's chunk
    for (int r = 0; r < nrej; ++r) mine |= static_cast<unsigned long long>(s_rej[r] >= v0 && s_rej[r] < v1) << r;
    if constexpr (CH > 0) {                            // lv[] still holds cur's row
        // A chunk without a rejected token has the sum that went into Z, added up in the same order; few
        // wavefronts hold any other (all of them summing again: 32000 tokens 12.1 us, now 10.9; 65536 19.6, now 17.7).
        csum = mass;
        if (mine) {
            for (unsigned long long r = mine; r; r &= r - 1) drop(lv, NV, s_rej[__builtin_ctzll(r)] - v0);
            csum = 0.f;
#pragma unroll
            for (int i = 0; i < CH; ++i) csum += prob_of(vec_at<T>(lv[i / VEC], i % VEC));
        }
        repack();
    } else {
        if (v0 < v1) {
            // 16-byte vectors; entries outside the chunk count as zero, which changes no sum.  A vector that is not
            // whole inside the row is replaced by another one of it, then patched entry by entry.
            const ChunkVectors cv(reinterpret_cast<uintptr_t>(row), v0, v1, V, VEC);
            const int lead = cv.lead, len = v1 - v0;
            const uint4* pv = reinterpret_cast<const uint4*>(row + v0 - lead);
            for (int k = 0; k < cv.count; k += 4) {
                uint4 w[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) w[u] = pv[min(max(k + u, cv.lo), cv.hi)];
                if (k < cv.lo || (cv.hi < cv.count - 1 && k + 3 > cv.hi)) {       // (the row's first and last threads only)
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (k + u < cv.lo || k + u > cv.hi)
#pragma unroll
                            for (int e = 0; e < VEC; ++e) {
                                const int at = (k + u) * VEC + e - lead;
                                if (static_cast<unsigned>(at) >= static_cast<unsigned>(len)) continue;
                                uint32_t& x = (&w[u].x)[sizeof(T) == 2 ? e >> 1 : e];
                                if constexpr (sizeof(T) == 2) x = (x & (0xFFFF0000u >> (16 * (e & 1)))) | static_cast<uint32_t>(row[v0 + at]) << (16 * (e & 1));
                                else x = __float_as_uint(row[v0 + at]);
                            }
                }
                for (unsigned long long r = mine; r; r &= r - 1) drop(w, 4, s_rej[__builtin_ctzll(r)] - v0 + lead - k * VEC);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        const int at = (k + u) * VEC + e - lead;        // position in the chunk
                        const float pe = prob_of(vec_at<T>(w[u], e));
                        csum += static_cast<unsigned>(at) < static_cast<unsigned>(len) ? pe : 0.f;
                    }
            }
        }
    }
    // inclusive scan of the chunk sums: inside each wavefront by shuffles, then the 16 wavefront
    // totals (summed in order by every thread) as offsets
    float incl = csum;
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (tid == 0) { s_pick = -1; s_chunk = -1; }
    __syncthreads();                                   // s_red is free (last use: the row sum)
    if (lane == 63) s_red[wave] = incl;
    __syncthreads();
    float offset = 0.f;
    for (int w = 0; w < wave; ++w) offset += s_red[w];
    s_scan[tid] = incl + offset;
    __syncthreads();
    const float total = s_scan[kThreadsAS - 1];
    const float t = u_bonus[b] * total;
    const float before = tid ? s_scan[tid - 1] : 0.f;
    if (s_scan[tid] > t && before <= t) s_chunk = tid; // the scan is non-decreasing: exactly one such chunk
    __syncthreads();
    if constexpr (CH > 0) {
        if (s_chunk == tid) {
            float cum = before;
            int pick = -1, last_live = -1;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const float ev = prob_of(vec_at<T>(lv[i / VEC], i % VEC));
                if (ev > 0.f) last_live = v0 + i;
                cum += ev;
                if (pick < 0 && cum > t) pick = v0 + i;
            }
            s_pick = pick >= 0 ? pick : last_live;    // rounding inside the chunk: its last live token
        }
    } else if (s_chunk >= 0) {                         // uniform
        const int c0 = min(s_chunk * chunk, V), len = min(chunk, V - c0);
        auto walk = [&](auto&& ev_of) {
            float cum = s_chunk ? s_scan[s_chunk - 1] : 0.f;
            int pick = -1, last_live = -1;
#pragma unroll 4
            for (int i = 0; i < len; ++i) {
                const float ev = ev_of(i);
                if (ev > 0.f && pick < 0) last_live = c0 + i;
                cum += ev;
                if (cum > t && pick < 0) pick = c0 + i;
            }
            s_pick = pick >= 0 ? pick : last_live;
        };
        auto residual_at = [&](int v) -> float {
            bool live = true;
            for (int r = 0; r < nrej; ++r) live = live && s_rej[r] != v;
            return live ? prob_of(logit_at<T>(row, v)) : 0.f;
        };
        if (len <= kWalk) {                            // uniform
            for (int i = tid; i < len; i += kThreadsAS) s_ev[i] = residual_at(c0 + i);
            __syncthreads();
            if (tid == 0) walk([&](int i) { return s_ev[i]; });
        } else if (tid == 0) {
            walk([&](int i) { return residual_at(c0 + i); });
        }
    }
    __syncthreads();
    if (tid == 0) {
        int pick = s_pick;
        if (pick < 0) {                                // t landed on the total by rounding: last live token
            for (int v = V - 1; v >= 0 && pick < 0; --v) {
                bool live = true;
                for (int r = 0; r < nrej; ++r) live = live && s_rej[r] != v;
                if (live && prob_of(logit_at<T>(row, v)) > 0.f) pick = v;
            }
            if (pick < 0) pick = 0;
        }
        accept_len[b] = m;
        bonus_tok[b] = pick;
        int32_t* prow = path + b * path_cap;
        int32_t* crow = committed_tok + b * path_cap;
        for (int j = 0; j < path_cap; ++j) {
            prow[j] = j <= m ? s_path[j] : -1;
            crow[j] = j < m ? s_tok[s_path[j + 1]] : (j == m ? pick : -1);
        }
        err |= s_err;
        if (err && err_flag) atomicOr(err_flag, err);
    }
}

}  // namespace

int32_t launch_tree_accept_sample(int32_t dtype, int32_t B, int32_t N_max, int32_t V, int32_t path_cap,
                                  const int32_t* parent, const int32_t* draft_tok, const void* logits,
                                  int64_t stride_b, int64_t stride_n, const int32_t* num_nodes,
                                  float temperature, const float* u_accept, const float* u_bonus,
                                  int32_t* accept_len, int32_t* path, int32_t* bonus_tok,
                                  int32_t* committed_tok, int32_t* err_flag, hipStream_t stream) {
    dim3 grid(B), block(kThreadsAS);
#define SPECVLM_LAUNCH_AS2(T, CH, WHOLE)                                                                             \
    hipLaunchKernelGGL((tree_accept_sample_kernel<T, CH, WHOLE>), grid, block, 0, stream, N_max, V, path_cap, parent, \
                       draft_tok, static_cast<const T*>(logits), stride_b, stride_n, num_nodes, temperature,         \
                       u_accept, u_bonus, accept_len, path, bonus_tok, committed_tok, err_flag)
#define SPECVLM_LAUNCH_AS(T, CH)                     \
    do {                                             \
        if (whole) SPECVLM_LAUNCH_AS2(T, CH, true);  \
        else SPECVLM_LAUNCH_AS2(T, CH, false);       \
    } while (0)
    const int chunk = (V + kThreadsAS - 1) / kThreadsAS, vec = dtype == SPECVLM_BF16 ? 8 : 4;
    const bool whole = (reinterpret_cast<uintptr_t>(logits) & 15u) == 0 && (stride_b | stride_n | chunk | V) % vec == 0;
    if (dtype == SPECVLM_BF16) {
        if (chunk <= 32) SPECVLM_LAUNCH_AS(uint16_t, 32);
        else if (chunk <= 64) SPECVLM_LAUNCH_AS(uint16_t, 64);
        else SPECVLM_LAUNCH_AS2(uint16_t, 0, false);
    } else {
        if (chunk <= 32) SPECVLM_LAUNCH_AS(float, 32);
        else if (chunk <= 64) SPECVLM_LAUNCH_AS(float, 64);
        else SPECVLM_LAUNCH_AS2(float, 0, false);
    }
#undef SPECVLM_LAUNCH_AS2
#undef SPECVLM_LAUNCH_AS
    return check_launch();
}

}  // namespace specvlm
