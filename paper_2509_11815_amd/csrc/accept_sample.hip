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
//   row       up to 32 consecutive tokens per thread stay in registers where they are whole vectors (CH = 32); the root's row is
//             requested before the tree is looked at.  Other vocabularies (CH = 0) are read once a level: wavefronts have contiguous
//             regions, every load is 1 KB of memory in one piece, and lanes sum exp2((l - m) log2e / T) against the greatest logit they
//             have met, until the workgroup's is known
//   sums      in a fixed order, so that the same input gives the same decision whatever the timing; lanes
//             meet by DPP and lane swaps in the order of an xor butterfly (32, 16, 8, 4, 2, 1), then the 16
//             wavefronts through LDS in order
//   children  wavefront 0 holds a child per lane: what the earlier ones have taken is a running sum over lanes,
//             then all acceptance thresholds are computed at once and the first accepted child is a bit scan
//   bonus     a scan of the chunk sums, and the chunk that contains the drawn position is walked.  CH = 0: the regions' sums are there
//             already (regions with a rejected token are added up again without it); the region that contains the position
//             is taken apart into blocks of a wavefront's load, the block into lanes, the lane's vector is walked
// In a graph, 4 requests, us, three passes over rows beyond 64 tokens a thread -> one: bf16 100001 tokens 27.2 -> 20.4, 152064 34.6 -> 24.7 (16
// requests 42.0 -> 29.4), 250000 50.6 -> 34.1; fp32 28.2 -> 21.3, 37.1 -> 28.1, 54.6 -> 37.5.  What bounds the long ones is the
// exponentials of a row on one compute unit.
#include "chunk_vectors.hpp"
#include "wave_ops.hpp"

namespace specvlm {

namespace {

constexpr int kThreadsAS = 1024;
constexpr float kLowestAS = -3.402823466e38f;         // reference of a lane without tokens: no finite logit is below it

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

// CH == 0: a row as aligned 16-byte vectors (the first and the last may reach past its ends), dealt out to the wavefronts in contiguous
// regions of whole blocks of 64 vectors, so that every load of a wavefront is one piece of memory.
template <typename T>
struct RowVectors {
    static constexpr int VEC = 16 / sizeof(T);
    const uint4* body = nullptr;
    int lead = 0, lo = 0, hi = 0, end = 0, per = 0, r0 = 0, r1 = 0, V = 0;
    __device__ RowVectors() {}
    __device__ RowVectors(const T* row, int V_) : V(V_) {
        const ChunkVectors cv(reinterpret_cast<uintptr_t>(row), 0, V, V, VEC);
        lead = cv.lead, lo = cv.lo, hi = cv.hi, end = cv.count;
        body = reinterpret_cast<const uint4*>(row - lead);
        per = ((end + kThreadsAS / 64 - 1) / (kThreadsAS / 64) + 63) & ~63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        r0 = min(wave * per, end);
        r1 = min(r0 + per, end);
    }
    __device__ bool whole(int k) const { return k >= lo && k <= hi; }
    __device__ uint4 load(int k) const { return body[k]; }
    __device__ int first(int k) const { return k * VEC - lead; }
    __device__ int vector_at(int v) const { return (v + lead) / VEC; }
    // take(vectors, number of the first, 64 apart) for this lane's whole vectors of its wavefront's region, eight or one at a time; one(token) for the entries of the others; eight loads in flight
    template <typename Take, typename One>
    __device__ __forceinline__ void each(Take&& take, One&& one) const {
        const int lane = threadIdx.x & 63, from = max(r0, lo), to = min(r1, hi + 1);
        int k = from + lane;
        for (; k + 64 * 7 < to; k += 64 * 8) {
            uint4 w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = body[k + 64 * u];
            take(w, k);
        }
        for (; k < to; k += 64) {
            const uint4 w[1] = {body[k]};
            take(w, k);
        }
        if (r0 < r1 && lane < VEC) {
            if (r0 < lo && first(0) + lane >= 0 && first(0) + lane < V) one(first(0) + lane);
            if (r1 - 1 > hi && end > lo && first(end - 1) + lane < V) one(first(end - 1) + lane);
        }
    }
};

// CH > 0: every thread keeps its chunk of the current row (at most CH consecutive tokens, whole aligned vectors) in
// registers, loaded once per level with 16-byte loads.
// CH == 0: any vocabulary size at any alignment, a level reads its row once.
template <typename T, int CH>
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
#pragma unroll
            for (int j = 0; j < NV; ++j)
                if (v0 + j * VEC < v1) lv[j] = *reinterpret_cast<const uint4*>(row + v0 + j * VEC);
        }
    };
    RowVectors<T> rv;                                   // CH == 0: the current row
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
    // unnormalised probability exp((l - max) / T) as one multiply and one v_exp_f32 (a row goes through it once a level,
    // on a single compute unit; the bonus draw takes only chunks or regions again); -inf gives 0
    const float c2 = 1.4426950408889634f / temperature;
    auto prob_of = [&](float l) -> float { return __builtin_amdgcn_exp2f((l - mx) * c2); };
    auto sum_of = [&](const uint4& w) __attribute__((always_inline)) -> float {
        float x = prob_of(vec_at<T>(w, 0));
#pragma unroll
        for (int e = 1; e < VEC; ++e) x += prob_of(vec_at<T>(w, e));
        return x;
    };
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
            // once through the row: every lane sums against the greatest logit it has met
            rv = RowVectors<T>(row, V);
            float sum = 0.f;
            part = kLowestAS;
            auto meet = [&](float m) __attribute__((always_inline)) {
                mx = fmaxf(part, m);                   // (prob_of is relative to it)
                sum *= prob_of(part);                  // (by exactly 1 where the reference stays)
                part = mx;
            };
            rv.each([&](const auto& w, int) __attribute__((always_inline)) {
                float m = -INFINITY;
#pragma unroll
                for (const uint4& x : w)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) m = fmaxf(m, vec_at<T>(x, e));
                meet(m);
#pragma unroll
                for (const uint4& x : w) sum += sum_of(x);
            }, [&](int v) {
                const float l = logit_at<T>(row, v);
                meet(l);
                sum += prob_of(l);
            });
            mass = sum;
        }
        const float mine = part;                       // CH == 0: what `mass` is relative to
        mx = block_max(part, s_red);
        part = 0.f;
        if constexpr (CH > 0) {
#pragma unroll
            for (int i = 0; i < CH; ++i)
                part += prob_of(vec_at<T>(lv[i / VEC], i % VEC));          // (adding the zeros of -inf changes nothing)
            repack();
        } else {
            part = mass * prob_of(mine);
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
    const int lane = tid & 63, wave = tid >> 6;
    if constexpr (CH > 0) {
        float csum = 0.f;
        unsigned long long mine = 0;                   // bit r: rejected token r lies in this thread's chunk
        for (int r = 0; r < nrej; ++r) mine |= static_cast<unsigned long long>(s_rej[r] >= v0 && s_rej[r] < v1) << r;
        // lv[] still holds cur's row
        // A chunk without a rejected token has the sum that went into Z, added up in the same order; few
        // wavefronts hold any other (all of them summing again: 32000 tokens 12.1 us, now 10.9).
        csum = mass;
        if (mine) {
            for (unsigned long long r = mine; r; r &= r - 1) drop(lv, NV, s_rej[__builtin_ctzll(r)] - v0);
            csum = 0.f;
#pragma unroll
            for (int i = 0; i < CH; ++i) csum += prob_of(vec_at<T>(lv[i / VEC], i % VEC));
        }
        repack();
        // inclusive scan of the chunk sums: inside each wavefront by shuffles, then the 16 wavefront
        // totals (summed in order by every thread) as offsets
        float incl = csum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const float up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        if (tid == 0) { s_pick = -1; s_chunk = -1; }
        __syncthreads();                               // s_red is free (last use: the row sum)
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
            s_pick = pick >= 0 ? pick : last_live;     // rounding inside the chunk: its last live token
        }
    } else {
        // s_red[w] holds the sum of wavefront w's region of the row; regions with a rejected token are added up without it
        auto rejected_in = [&](int from, int to) __attribute__((always_inline)) -> unsigned long long {     // bit r: token r
            unsigned long long some = 0;
            for (int r = 0; r < nrej; ++r) {
                const int k = rv.vector_at(s_rej[r]);
                some |= static_cast<unsigned long long>(k >= from && k < to) << r;
            }
            return some;
        };
        auto without = [&](uint4& w, int k, unsigned long long some) __attribute__((always_inline)) {
            for (; some; some &= some - 1) {           // uniform in a wavefront
                const int at = s_rej[__builtin_ctzll(some)] - rv.first(k);
                if (static_cast<unsigned>(at) < static_cast<unsigned>(VEC)) drop(&w, 1, at);
            }
        };
        auto vector_of = [&](int k, unsigned long long some) __attribute__((always_inline)) -> uint4 {
            uint4 w{kInfWord, kInfWord, kInfWord, kInfWord};
            if (rv.whole(k)) {
                w = rv.load(k);
            } else if (k < rv.end) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int v = rv.first(k) + e;
                    if (v >= 0 && v < V) put(w, e, row[v]);
                }
            }
            without(w, k, some);
            return w;
        };
        if (const unsigned long long mine = rejected_in(rv.r0, rv.r1)) {           // uniform in a wavefront
            float sum = 0.f;
            rv.each([&](auto& ws, int k) __attribute__((always_inline)) {
                for (uint4 w : ws) {
                    without(w, k, mine);
                    sum += sum_of(w);
                    k += 64;
                }
            }, [&](int v) {
                bool live = true;
                for (int r = 0; r < nrej; ++r) live = live && s_rej[r] != v;
                sum += live ? prob_of(logit_at<T>(row, v)) : 0.f;
            });
            sum = butterfly_sum(sum);
            if (lane == 0) s_red[wave] = sum;
        }
        if (tid == 0) s_pick = -1;
        __syncthreads();
        float total = 0.f;
        for (int w = 0; w < kThreadsAS / 64; ++w) total += s_red[w];
        const float t = u_bonus[b] * total;
        // the region, then the block of 64 steps of `each` vectors, then the lane that the drawn position is in.  Where rounding
        // leaves it past all parts of the one before, it is the last that holds anything.
        float before = 0.f;
        int region = 0;
        for (; region < kThreadsAS / 64 && before + s_red[region] <= t; ++region) before += s_red[region];
        if (region < kThreadsAS / 64 && t >= 0.f) {    // uniform (a position that is NaN or negative is in no region)
            const int r0 = min(region * rv.per, rv.end), r1 = min(r0 + rv.per, rv.end);
            const int each = (r1 - r0 + 64 * kThreadsAS - 1) / (64 * kThreadsAS), blocks = (r1 - r0 + 64 * each - 1) / (64 * each);
            const unsigned long long some = rejected_in(r0, r1);
            auto lane_sum = [&](int block) __attribute__((always_inline)) -> float {
                float x = 0.f;
                for (int i = 0; i < each; ++i) {
                    const int k = r0 + (block * 64 + lane) * each + i;
                    if (k < r1) x += sum_of(vector_of(k, some));
                }
                return x;
            };
            for (int block = wave; block < blocks; block += kThreadsAS / 64) {
                const float x = butterfly_sum(lane_sum(block));
                if (lane == 0) s_scan[block] = x;
            }
            __syncthreads();
            if (wave == 0) {
                int block = -1, last = 0;
                float at_last = before;
                for (int i = 0; i < blocks && block < 0; ++i) {
                    const float x = s_scan[i];
                    if (x > 0.f) { last = i; at_last = before; }
                    if (before + x > t) block = i; else before += x;
                }
                if (block < 0) { block = last; before = at_last; }
                const float x = lane_sum(block);
                float incl = x;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const float up = __shfl_up(incl, off);
                    if (lane >= off) incl += up;
                }
                const float up = __shfl_up(incl, 1);
                float cum = before + (lane ? up : 0.f);
                const unsigned long long past = __ballot(before + incl > t && x > 0.f), any = __ballot(x > 0.f);
                const int who = past ? __builtin_ctzll(past) : any ? 63 - __builtin_clzll(any) : -1;
                if (lane == who) {
                    int pick = -1, last_live = -1;
                    for (int i = 0; i < each; ++i) {
                        const int k = r0 + (block * 64 + lane) * each + i;
                        if (k >= r1) break;
                        const uint4 w = vector_of(k, some);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            const float ev = prob_of(vec_at<T>(w, e));
                            if (ev > 0.f) last_live = rv.first(k) + e;
                            cum += ev;
                            if (pick < 0 && cum > t && ev > 0.f) pick = rv.first(k) + e;
                        }
                    }
                    s_pick = pick >= 0 ? pick : last_live;
                }
            }
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
#define SPECVLM_LAUNCH_AS(T, CH)                                                                                     \
    hipLaunchKernelGGL((tree_accept_sample_kernel<T, CH>), grid, block, 0, stream, N_max, V, path_cap, parent,       \
                       draft_tok, static_cast<const T*>(logits), stride_b, stride_n, num_nodes, temperature,         \
                       u_accept, u_bonus, accept_len, path, bonus_tok, committed_tok, err_flag)
    // Registers where every chunk is whole vectors and at most 32 tokens, chunks 64 bytes apart at most: us, 4 requests in a graph, registers |
    // reading once: 32000 bf16 11.0 | 13.4, 16000 11.8 | 12.5, fp32 12.0 | 12.8 (8000: 11.5 | 11.2, 4000 fp32 11.0 | 10.7).  Chunks at
    // other places lost there: 4000 bf16 13.5 | 10.6, 20003 15.2 | 12.9, 30000 fp32 14.7 | 13.3, bf16 13.1 | 13.1; and so did 33 - 64 tokens a
    // thread: 36864 bf16 21.1 | 14.6, 65536 20.0 | 16.2, 60000 22.9 | 15.7, fp32 27.2 | 17.6.
    const int chunk = (V + kThreadsAS - 1) / kThreadsAS, vec = dtype == SPECVLM_BF16 ? 8 : 4;
    const bool held = chunk <= 32 && (reinterpret_cast<uintptr_t>(logits) & 15u) == 0 && (stride_b | stride_n | chunk | V) % vec == 0;
    if (dtype == SPECVLM_BF16) {
        if (held) SPECVLM_LAUNCH_AS(uint16_t, 32);
        else SPECVLM_LAUNCH_AS(uint16_t, 0);
    } else {
        if (held) SPECVLM_LAUNCH_AS(float, 32);
        else SPECVLM_LAUNCH_AS(float, 0);
    }
#undef SPECVLM_LAUNCH_AS
    return check_launch();
}

}  // namespace specvlm
