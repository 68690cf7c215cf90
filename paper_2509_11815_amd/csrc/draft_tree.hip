// Draft-side growth of the token tree (SpecVLM Sec. 4.1: the draft grows an EAGLE-2 style tree
// with Top-K 10, 60 tokens in total, depth 7, which the target then verifies in one pass).
//
// The paper gives the three numbers; the rule is the one of the method it follows.  A node's
// value is the sum of the draft's log-probabilities along its root path.  Every level expands
// the most valuable nodes of the previous level by their Top-K tokens (draft_topk_kernel),
// the most valuable new candidates are expanded next (draft_select_kernel), and in the end the
// most valuable candidates of all levels become the tree (draft_finalize_kernel), numbered in
// increasing candidate index, which is a topological order because a parent is created before
// its children.  "More valuable" is: greater stored fp32 score, the lower candidate index among
// equal scores; Top-K inside a row: greater logit, the lower token among equal logits.
//
// All three are latency-bound single-workgroup-per-row kernels: a row of 32000 bf16 logits is
// 64 KB, a level has at most `width` rows per request, and the candidate lists hold a few
// hundred entries.
#include <limits.h>

#include "draft_plan.hpp"
#include "wave_ops.hpp"

// Products and sums stay apart: which of them the compiler fuses differs between instantiations of one kernel, and a
// level selected in the same launch has the scores of one selected in a launch of its own.
#pragma clang fp contract(off)

namespace specvlm {

namespace {

constexpr int kThreadsDT = 1024;
constexpr int kWavesDT = kThreadsDT / 64;
constexpr int kCandCap = 1024;           // Top-K: entries at or above a threshold kept in LDS
constexpr int kRankDirect = 320;         // ... and ranked as they are.  Ten rows of that many equal best entries, one call: 320
                                         // 10.6 us, 512 15.6, 1000 37.8; with the second threshold 14.8 - 16.4 at any number, so the
                                         // two meet near 500 (the line was drawn for a ranking that one lane did per entry)

// Eight consecutive entries of a row, as loaded.
template <typename T>
struct Chunk;
template <>
struct Chunk<uint16_t> {
    uint4 w;
    __device__ __forceinline__ void load(const uint16_t* p) { w = *reinterpret_cast<const uint4*>(p); }
    __device__ __forceinline__ void fill() { w = uint4{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u}; }     // -inf
    __device__ __forceinline__ float at(int e) const {
        const uint32_t x = (&w.x)[e >> 1];
        return __uint_as_float((e & 1) ? (x & 0xFFFF0000u) : (x << 16));
    }
};
template <>
struct Chunk<float> {
    float f[8];
    __device__ __forceinline__ void load(const float* p) {
        *reinterpret_cast<float4*>(f) = *reinterpret_cast<const float4*>(p);
        *reinterpret_cast<float4*>(f + 4) = *reinterpret_cast<const float4*>(p + 4);
    }
    __device__ __forceinline__ void fill() {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = -INFINITY;
    }
    __device__ __forceinline__ float at(int e) const { return f[e]; }
};
template <typename T>
__device__ __forceinline__ float chunk_max(const Chunk<T>& c) {
    return fmaxf(fmaxf(fmaxf(c.at(0), c.at(1)), fmaxf(c.at(2), c.at(3))), fmaxf(fmaxf(c.at(4), c.at(5)), fmaxf(c.at(6), c.at(7))));
}

__device__ __forceinline__ float entry(const uint16_t* p) { return bf16_bits_to_float(*p); }
__device__ __forceinline__ float entry(const float* p) { return *p; }

// (logit, token) as one unsigned key whose order is "greater logit, then lower token".
// -0 and +0 are the same real number and must tie: adding +0 turns -0 into +0.
__device__ __forceinline__ unsigned long long order_key(float v, int idx) {
    uint32_t u = __float_as_uint(v + 0.0f);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return (static_cast<unsigned long long>(u) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(idx));
}

__device__ __forceinline__ float key_value(unsigned long long k) {     // the logit inside an order_key
    uint32_t u = static_cast<uint32_t>(k >> 32);
    u = (u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u;
    return __uint_as_float(u);
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const unsigned long long y = __shfl_xor(x, off);
        x = y > x ? y : x;
    }
    return x;
}

// ---------------------------------------------------------------------------------------
// Ranking of scored candidates: candidate i beats j when score[i] > score[j], or the scores
// are equal and i < j -- i.e. when its order_key(score, index) is the greater one.  rank(i) =
// number of candidates that beat i; the M winners are the candidates of rank < M; a winner's
// position is the number of winners of lower index.
// s_key holds the c keys (16-byte aligned).  On return the low word of s_key[i] holds candidate
// i's position among the winners, or -1 (pos_of below); the keys are gone.
// All c*c comparisons run on one compute unit, so what counts is instructions per comparison
// (two, see below) and that every wavefront has work: with few candidates several groups of
// wavefronts share the candidates, each taking a slice of the others.  s_key needs room for an
// even number of keys.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int pos_of(const unsigned long long* s_key, int i) {
    return reinterpret_cast<const int*>(s_key)[2 * i];
}

// How many of n keys are above the key of this row of 16 lanes (every lane of the row gets it): lanes take the keys in turn.
__device__ __forceinline__ int keys_above(const unsigned long long* s_key, int n, unsigned long long key) {
    int above = 0;
#pragma unroll 4
    for (int x = threadIdx.x & 15; x < n; x += 16) above += s_key[x] > key ? 1 : 0;
    return row_sum(above);
}

// Many candidates, few winners (the whole tree's 500 candidates, 59 nodes): ranking everybody
// against everybody is mostly wasted on candidates that cannot win.  The candidates are dealt
// into kGroupsDT groups (candidate i -> group i mod kGroupsDT); the M-th largest of the group
// maxima is a key that at least M candidates reach, so nobody below it wins, and at most
// M * ceil(c / kGroupsDT) candidates reach it (the members of M groups).  Only those are ranked,
// among themselves.  Same result as rank_winners' full ranking: keys are distinct, so "the M
// greatest keys" is one set whatever way it is found.  Needs kGroupsDT <= c <= kThreadsDT (every
// group has a member, one candidate per thread) and M <= kGroupsDT.  Rows of 16 lanes count as below; the survivors are
// gathered in any order, the winners meet in a bitmap: five barriers.  A select call of 510 candidates, 59 chosen, 4.8 -> 4.3 us
// (before: LDS counts of slices, survivors in index order, eight barriers).
constexpr int kGroupsDT = 128;

__device__ __forceinline__ void rank_winners_prefiltered(unsigned long long* s_key, int c, int M) {
    __shared__ __attribute__((aligned(16))) unsigned long long s_gmax[kGroupsDT];
    __shared__ unsigned long long s_surv[kThreadsDT];
    __shared__ unsigned long long s_thr;
    __shared__ int s_ns;
    __shared__ unsigned long long s_winmask[kWavesDT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long ki = tid < c ? s_key[tid] : 0ull;          // 0: below every real key
    if (tid < kGroupsDT) {
        unsigned long long m = ki;
        for (int i = tid + kGroupsDT; i < c; i += kGroupsDT) {
            const unsigned long long k = s_key[i];
            m = k > m ? k : m;
        }
        s_gmax[tid] = m;
    }
    if (tid < kWavesDT) s_winmask[tid] = 0ull;
    if (tid == 0) s_ns = 0;
    __syncthreads();
    // the M-th greatest group maximum
#pragma unroll
    for (int j = tid >> 4; j < kGroupsDT; j += kThreadsDT / 16) {
        const unsigned long long kj = s_gmax[j];
        const int above = keys_above(s_gmax, kGroupsDT, kj);
        if ((tid & 15) == 0 && above == M - 1) s_thr = kj;               // exactly one group: the ranks are a permutation
    }
    __syncthreads();
    const unsigned long long thr = s_thr;
    // the candidates that reach the threshold, in any order
    const bool surv = ki >= thr;                                         // thr is a real key: never true for tid >= c
    const unsigned long long bal = __ballot(surv);
    if (bal) {                                                           // uniform in a wavefront
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_ns, __popcll(bal));
        at = __builtin_amdgcn_readfirstlane(at);
        if (surv) s_surv[at + __popcll(bal & ((1ull << lane) - 1ull))] = ki;
    }
    __syncthreads();
    const int ns = s_ns;
    for (int a = tid >> 4; a < ns; a += kThreadsDT / 16) {
        const unsigned long long ka = s_surv[a];
        const int above = keys_above(s_surv, ns, ka);
        const uint32_t idx = 0xFFFFFFFFu - static_cast<uint32_t>(ka);   // the candidate's index sits in the key's low word
        if ((tid & 15) == 0 && above < M) atomicOr(&s_winmask[idx >> 6], 1ull << (idx & 63));
    }
    __syncthreads();
    if (tid < c) {                                                       // position = winners of lower index
        const unsigned long long mine = s_winmask[wave];
        int pos = __popcll(mine & ((1ull << lane) - 1ull));
        for (int w = 0; w < wave; ++w) pos += __popcll(s_winmask[w]);
        reinterpret_cast<int*>(s_key)[2 * tid] = (mine >> lane) & 1ull ? pos : -1;      // every key is in a register or in s_surv by now
    }
    __syncthreads();
}

// Few candidates (a level's Top-K lists): everybody against everybody, a row of 16 lanes per candidate, and a winner's
// position as a population count over the ballots of the winners -- two workgroup barriers (the general form below takes eight).
// A select call of 100 candidates 3.2 -> 3.05 us (before: counts of slices meeting in LDS atomics, five barriers).
__device__ __forceinline__ void rank_winners_few(unsigned long long* s_key, int c, int M) {
    __shared__ int s_win[2 * kGroupsDT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid >> 4; i < c; i += kThreadsDT / 16) {                // the same in a row of lanes
        const int above = keys_above(s_key, c, s_key[i]);
        if ((tid & 15) == 0) s_win[i] = above < M;
    }
    __syncthreads();
    if (wave * 64 < c) {                                                 // uniform in a wavefront
        int before = 0, pos = -1;
        for (int w = 0; w <= wave; ++w) {
            const int i = w * 64 + lane;
            const bool win = i < c && s_win[i];
            const unsigned long long bal = __ballot(win);
            if (w == wave && win) pos = before + __popcll(bal & ((1ull << lane) - 1ull));
            before += __popcll(bal);
        }
        if (tid < c) reinterpret_cast<int*>(s_key)[2 * tid] = pos;
    }
    __syncthreads();
}

__device__ __forceinline__ void rank_winners(unsigned long long* s_key, int c, int M) {
    __shared__ int s_wcount[kWavesDT];
    __shared__ int s_cnt[kThreadsDT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (below: select 192 of 10 3.6 us so and 3.8 by the few's form, of 64 3.9 and 3.8; 255 3.6 and 5.4, 4.0 and 5.4)
    if (c > 3 * kGroupsDT / 2 && c <= kThreadsDT && M >= 1 && M <= kGroupsDT / 2) {    // uniform
        rank_winners_prefiltered(s_key, c, M);
        return;
    }
    if (c < 2 * kGroupsDT) {                               // uniform
        rank_winners_few(s_key, c, M);
        return;
    }
    // `parts` groups of wavefronts share the candidates of a pass: group `part` counts, for every
    // candidate of the pass, the keys of its slice [j0, j1) of the others that beat it.
    int parts = 1, shift = 0;                              // uniform; a group is at least one wavefront
    while (parts < kWavesDT && c * (parts * 2) <= kThreadsDT) { parts *= 2; ++shift; }
    const int per_pass = kThreadsDT >> shift;              // candidates per pass (>= 64)
    const int part = tid / per_pass, slot = tid & (per_pass - 1);
    const int c_even = (c + 1) & ~1;                       // keys are read in pairs: an odd count is padded with a key nothing loses to
    if (tid == 0 && (c & 1)) s_key[c] = 0ull;
    __syncthreads();
    const int per = ((c_even / 2 + parts - 1) / parts) * 2;
    const int j0 = min(part * per, c_even), j1 = min(j0 + per, c_even);
    unsigned winbits = 0;                                  // bit p: this thread's candidate of pass p won (at most 8 passes)
    int pass = 0;
    for (int i0 = 0; i0 < c; i0 += per_pass, ++pass) {     // uniform trip count
        const int i = i0 + slot;
        const unsigned long long ki = i < c ? s_key[i] : ~0ull;
        const uint32_t hi = static_cast<uint32_t>(ki >> 32);
        // The candidates of this wavefront are iw0 .. iw0 + 63.  A key j below all of them beats
        // candidate i when its upper word is >= i's (equal scores: the lower index wins), a key
        // above all of them when it is > : one 32-bit compare and an add-with-carry per key (a
        // 64-bit compare runs at a quarter of that rate).  Only the keys among the wavefront's own
        // candidates need the whole key.  (No score is NaN, so an upper word is never 0.)
        const int iw0 = i0 + ((wave * 64) & (per_pass - 1));
        const int a_end = max(j0, min(j1, iw0 & ~1));             // pairs entirely below iw0
        const int b_end = max(a_end, min(j1, (iw0 + 65) & ~1));   // pairs that may hold one of the wavefront's candidates
        int beaten = 0;
        const uint32_t thr_below = hi - 1u;
#pragma unroll 4
        for (int j = j0; j < a_end; j += 2) {
            const ulonglong2 q = *reinterpret_cast<const ulonglong2*>(s_key + j);
            beaten += static_cast<uint32_t>(q.x >> 32) > thr_below ? 1 : 0;
            beaten += static_cast<uint32_t>(q.y >> 32) > thr_below ? 1 : 0;
        }
        for (int j = a_end; j < b_end; j += 2) {
            const ulonglong2 q = *reinterpret_cast<const ulonglong2*>(s_key + j);
            beaten += q.x > ki ? 1 : 0;
            beaten += q.y > ki ? 1 : 0;
        }
#pragma unroll 4
        for (int j = b_end; j < j1; j += 2) {
            const ulonglong2 q = *reinterpret_cast<const ulonglong2*>(s_key + j);
            beaten += static_cast<uint32_t>(q.x >> 32) > hi ? 1 : 0;
            beaten += static_cast<uint32_t>(q.y >> 32) > hi ? 1 : 0;
        }
        if (parts > 1) {                                   // uniform: add the groups' counts up
            if (part == 0) s_cnt[slot] = 0;
            __syncthreads();
            atomicAdd(&s_cnt[slot], beaten);
            __syncthreads();
            beaten = s_cnt[slot];
            __syncthreads();                               // s_cnt is cleared again by the next pass
        }
        if (i < c && part == 0 && beaten < M) winbits |= 1u << pass;
    }
    __syncthreads();                                       // the keys have been read for the last time
    // position of a winner = winners of lower index: earlier passes, earlier wavefronts, lower lanes
    int base = 0;
    pass = 0;
    for (int i0 = 0; i0 < c; i0 += per_pass, ++pass) {
        const int i = i0 + slot;
        const bool win = (winbits >> pass) & 1u;
        const unsigned long long bal = __ballot(win);
        if (lane == 0) s_wcount[wave] = __popcll(bal);
        __syncthreads();
        int before = base, total = 0;
#pragma unroll
        for (int x = 0; x < kWavesDT; ++x) {
            const int n = s_wcount[x];
            before += x < wave ? n : 0;
            total += n;
        }
        if (i < c && part == 0)
            reinterpret_cast<int*>(s_key)[2 * i] = win ? before + __popcll(bal & ((1ull << lane) - 1ull)) : -1;
        base += total;
        __syncthreads();                                   // s_wcount is rewritten by the next pass
    }
}

// ---------------------------------------------------------------------------------------
// draft_topk_kernel: one workgroup per (request, expanded node) row, so one compute unit reads the row and
// what counts is passes, instructions per entry and the latencies between the steps.
//   entries   chunks of 8 (from the row's first 16-byte boundary), thread t takes chunks t, t + 1024, ...; the up to
//             7 entries before and after are one thread's each.  NC = 4, 8: a row of up to 8192 NC entries stays in
//             registers.  NC = 0: the row streams by once, in groups of four chunks a thread with a running maximum and sum,
//             (bf16) the next group on its way while one is added up; of a chunk only its maximum is kept.
//   lse       every thread sums against its own maximum, so maximum and sum need one meeting of the workgroup
//             instead of two; lanes meet by DPP.
//   Top-K     every row of 16 lanes reduces its greatest logit; the K-th greatest of the 64 is a value that at least K
//             entries reach, and (for logits that do not follow the token order) about 2K do.  These are collected
//             in LDS and ranked against each other: an entry beaten by r others is the r-th best.  Keys are
//             distinct, so the order of collection does not matter.  More than kRankDirect of them (many equal, logits
//             sorted along the vocabulary, fewer than K groups with finite ones): the threshold becomes the K-th best
//             of the threads' best keys, with the token order among equal logits; if that does not help either
//             (the best entries sit in few threads), K rounds of one winner each.
// Per level (10 rows, kernel alone): 32000 bf16 logits 10.4 -> 6.6 us; rows of 99254 and 152064, which used to be re-read
// entry by entry in every pass, 66 and 96 us -> 12.9 and 14.4.  Ten rows of equal logits, one call: 32000 42.7 -> 18.7,
// 152064 97.9 -> 57.7; sorted along the vocabulary 44.5 -> 16.1 and 97.7 -> 41.0.
// Entries ranked by rows of 16 lanes (a lane's share instead of a lane for all others) and the log-sum-exp left to one wavefront
// beside the collection: 5.75 -> 5.3 us a call; a growth of six levels with its finalize 53.4 -> 49.2, nearly all of it at the root, the last
// level and the finalize (the levels between, ten rows with the selection, take 9.2 - 9.3 us each in a trace of the growth, as before).
// ---------------------------------------------------------------------------------------
// With the selection (kSelect, kBeside): the workgroup that finishes a request's last row also chooses the M most valuable of the
// request's W*K new candidates (what draft_select_kernel does in a launch of its own): scores
// are stored write-through, acknowledged, then a ticket per request is drawn.  kBeside: a row has two workgroups on two compute
// units, one for its log-sum-exp, which waits for no ranking, and one for its Top-K, which then leaves the exponentials (1.5 us of
// 32000) alone.  They store a log-sum-exp and K logits; the scores are put together by the one that selects, from the same operations.
// A growth of six levels, ten rows each but the root, in a graph, one workgroup a row -> two: bf16, one request 32000 tokens 48.8 -> 44.4 us,
// 65000 59.4 -> 53.8, 152064 108.2 -> 94.0; eight requests 54.0 -> 50.1, 63.0 -> 60.6, 121.7 -> 106.7; fp32, one 50.4 -> 47.3, 62.3 -> 58.5,
// 110.7 -> 98.0.  Then nothing summed where a row beyond 65536 entries has ended, chunks that reach the threshold found by a bit mask, and in bf16 the
// next group of loads requested ahead: bf16, one request 70000 69.9 -> 65.9, 100001 81.7 -> 75.4, 152064 94.5 -> 87.8, eight 106.2 -> 95.5 (four or eight
// chunks a group: 87.8 and 92.6); fp32 (and one workgroup a row for eight requests) one 83.6 -> 68.5, 99.7 -> 80.7, 112.6 -> 93.8, eight 95.1 -> 83.7, 109.0 ->
// 95.2, 123.7 -> 108.5 from what there was at first.  (Tried: the log-sum-exp of a long row shared by up to five workgroups in segments of 32768
// entries, and rows of up to 163840 bf16 entries in registers: the segments' reductions cost the other calls 1 us, the longer unrolled code 5.)
struct SelArgs {
    int M, index_base;
    int32_t* sel_out;
    float* sel_score_out;
    int32_t* count_out;
    int32_t* counters;            // [B * SPECVLM_COUNTER_STRIDE] tickets, zero between calls; kBeside: word 1 + w, row w's log-sum-exp
    int rows;                     // kBeside: rows of a request
};

enum Level { kPlain, kSelect, kBeside };                   // scores only; with the selection; with that, and the log-sum-exps in workgroups of their own

constexpr float kLowest = -3.402823466e38f;         // reference of a thread without entries: no finite logit is below it
constexpr int kStream = 24;              // NC == 0: chunks per thread whose maximum is kept (196608 entries)

// exp(x) for a difference x <= 0 of two logits.  The difference is taken first: the row's greatest entry then adds
// exactly 1, the sum is at least 1 and no log-probability is positive, so a child never outranks its parent
// (a fused multiply-add with the reference already scaled saves an instruction, but adds 2^r, r the rounding of that).
__device__ __forceinline__ float exp_of(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

template <typename T, int NC, Level LEVEL>
__global__ __launch_bounds__(kThreadsDT) void draft_topk_kernel(
    int V, int K, const T* __restrict__ logits, int64_t stride_b, int64_t stride_w,
    const float* __restrict__ cum, int64_t cum_stride_b, const int32_t* __restrict__ parent_idx,
    int64_t parent_stride_b, float* score_out, int32_t* __restrict__ token_out,
    int32_t* __restrict__ parent_out, int64_t out_stride_b, float* __restrict__ lse_out, SelArgs sel) {
    __shared__ float s_wmax[kWavesDT], s_wsum[kWavesDT];
    __shared__ __attribute__((aligned(16))) float s_grp[64];
    __shared__ unsigned long long s_key[2][kWavesDT];
    __shared__ __attribute__((aligned(16))) unsigned long long s_cand[kCandCap];
    __shared__ unsigned long long s_grp_key[64], s_thr_key;
    __shared__ int s_last, s_ncand;
    __shared__ float s_thr, s_lse;

    constexpr bool SEL = LEVEL != kPlain, BESIDE = LEVEL == kBeside;
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nrows = BESIDE ? sel.rows : gridDim.x;
    const bool summing = BESIDE && static_cast<int>(blockIdx.x) >= nrows;       // uniform: this workgroup adds up, the row's other one ranks
    const int w = summing ? blockIdx.x - nrows : blockIdx.x;
    const T* row = logits + b * stride_b + w * stride_w;
    const float c = cum ? cum[b * cum_stride_b + w] : 0.f;
    const int par = parent_idx ? parent_idx[b * parent_stride_b + w] : -1;
    const int head = min(static_cast<int>(((16u - (reinterpret_cast<uintptr_t>(row) & 15u)) & 15u) / sizeof(T)), V);
    const int nck = (V - head) / 8;                      // whole chunks
    const int tail0 = head + nck * 8;
    const T* body = row + head;
    // the single entry of this thread, if it has one
    const int vs = tid < head ? tid : (tid >= 64 && tid - 64 < V - tail0) ? tail0 + tid - 64 : -1;
    const float es = vs >= 0 ? entry(row + vs) : -INFINITY;

    // ---- maximum and sum of exponentials of this thread's entries ------------------------------
    constexpr int NM = NC > 0 ? NC : kStream;
    constexpr int U = 4;                                 // NC == 0: chunks of a thread requested together
    // ... in bf16 a group ahead of the one being taken.  A group of fp32 is twice the bytes, and 16 wavefronts' requests fill the unit's
    // queue by themselves: 40 rows, from cache, ahead | not: 65537 entries 9.98 | 8.85 us, 128256 12.95 | 12.26, 250000 25.3 | 24.8 (one row
    // 23.0 | 21.9; 80 rows from HBM 34.4 | 34.3, 152064 19.4 | 19.9)
    constexpr bool AHEAD = sizeof(T) == 2;
    Chunk<T> ch[NC > 0 ? NC : U];
    float cmax[NM];
    float tmax = es;                                     // greatest entry
    float m, sum;                                        // finite reference, sum of exp(entry - m)
    if constexpr (NC > 0) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int k = tid + kThreadsDT * j;
            if (k < nck) ch[j].load(body + 8 * k); else ch[j].fill();
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            cmax[j] = chunk_max(ch[j]);
            tmax = fmaxf(tmax, cmax[j]);
        }
        m = fmaxf(tmax, kLowest);
        sum = 0.f;
        if (!BESIDE || summing) {
            float part[4] = {exp_of(es - m), 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) part[e & 3] += exp_of(ch[j].at(e) - m);     // exp(-inf) = 0
            sum = (part[0] + part[1]) + (part[2] + part[3]);
        }
    } else {
        m = fmaxf(es, kLowest);
        sum = es > -INFINITY ? 1.f : 0.f;
        Chunk<T> next[U];                                // the group requested last
        auto request = [&](int k0) __attribute__((always_inline)) {                     // chunks k0, k0 + 1024, ...
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + kThreadsDT * u;
                if (k < nck) next[u].load(body + 8 * static_cast<int64_t>(k)); else next[u].fill();
            }
        };
        auto take = [&](int j, float (&cm)[U]) __attribute__((always_inline)) {         // group j, j + 1, ... j + U - 1 of 1024 chunks
            if constexpr (!AHEAD) request(tid + kThreadsDT * j);
#pragma unroll
            for (int u = 0; u < U; ++u) ch[u] = next[u];
            if constexpr (AHEAD)
                if ((j + U) * kThreadsDT < nck) request(tid + kThreadsDT * (j + U));    // uniform
            float gm = -INFINITY;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cm[u] = chunk_max(ch[u]);
                gm = fmaxf(gm, cm[u]);
            }
            tmax = fmaxf(tmax, gm);
            if (BESIDE && !summing) return;
            const float mn = fmaxf(m, gm);
            float part[4] = {sum * exp_of(m - mn), 0.f, 0.f, 0.f};         // (times exactly 1 where the maximum stays)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((j + u) * kThreadsDT < nck)          // uniform
#pragma unroll
                    for (int e = 0; e < 8; ++e) part[e & 3] += exp_of(ch[u].at(e) - mn);
            sum = (part[0] + part[1]) + (part[2] + part[3]);
            m = mn;
        };
        if constexpr (AHEAD) request(tid);
#pragma unroll
        for (int j = 0; j < kStream; j += U) {
            float cm[U];
#pragma unroll
            for (int u = 0; u < U; ++u) cm[u] = -INFINITY;
            if (j * kThreadsDT < nck) take(j, cm);       // uniform
#pragma unroll
            for (int u = 0; u < U; ++u) cmax[j + u] = cm[u];
        }
        for (int j = kStream; j * kThreadsDT < nck; j += U) {               // (vocabularies beyond 196608)
            float cm[U];
            take(j, cm);
        }
    }
    auto wave_sums = [&]() __attribute__((always_inline)) {
        const float wm = wave_max(m);
        const float ws = wave_sum(sum * exp_of(m - wm));
        if (lane == 0) { s_wmax[wave] = wm; s_wsum[wave] = ws; }
    };
    auto log_sum = [&]() __attribute__((always_inline)) -> float {         // of the row, in every row of 16 lanes
        const float mx = row_max(s_wmax[tid & 15]);
        return mx + logf(row_sum(s_wsum[tid & 15] * exp_of(s_wmax[tid & 15] - mx)));
    };
    // The root's only row: its candidates come in the order of their scores (rounding keeps it, equal ones go by
    // index, with a NaN all are), so the selection is the first M and nobody has to be met: 7.7 -> 5.6 us a call.
    const bool lone = LEVEL == kSelect && nrows == 1 && !cum;
    if (summing) {
        wave_sums();
        __syncthreads();
        if (wave == 0) {
            const float l = log_sum();
            if (lane == 0) {
                __hip_atomic_store(sel.counters + b * SPECVLM_COUNTER_STRIDE + 1 + w, static_cast<int32_t>(__float_as_uint(l)),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (lse_out) lse_out[b * nrows + w] = l;
            }
        }
    } else {
    {
        const float gmax = row_max(tmax);                // of the row of 16 lanes
        if constexpr (!BESIDE) wave_sums();
        if ((tid & 15) == 0) s_grp[tid >> 4] = gmax;
        if (tid == 0) s_ncand = 0;
    }
    __syncthreads();
    // ---- the K-th greatest of the 64 group maxima: 16 lanes per group, four comparisons each -----------
    {
        const int j = tid >> 4, part = tid & 15;
        const float gj = s_grp[j];
        const float4 o = *reinterpret_cast<const float4*>(s_grp + 4 * part);
        int beaten = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float x = (&o.x)[u];
            beaten += (x > gj || (x == gj && 4 * part + u < j)) ? 1 : 0;
        }
        beaten = row_sum(beaten);
        if (part == 0 && beaten == K - 1) s_thr = gj;    // exactly one group: the ranks are a permutation
    }
    __syncthreads();
    const float thr = s_thr;
    if (!BESIDE && wave == kWavesDT - 1) {               // beside the collection, in one wavefront's chain only
        const float l = log_sum();
        if (lane == 0) {
            s_lse = l;
            if (lse_out) lse_out[b * nrows + w] = l;
        }
    }

    // ---- the entries that reach it ------------------------------------------------------------------
    auto collect = [&](float x, int v) {
        if (x >= thr) {
            const int pos = atomicAdd(&s_ncand, 1);
            if (pos < kCandCap) s_cand[pos] = order_key(x, v);
        }
    };
    if (tmax >= thr) {
        if (vs >= 0) collect(es, vs);
        // Registers need a copy of this code per chunk, of which a wavefront takes one or two and fetches all: from eight chunks on
        // the few that reach the threshold are read again (eight requests of 65000 bf16 tokens 60.5 -> 59.1 us a growth; with four chunks
        // in registers reading again costs 1 us)
        if constexpr (NC > 0 && NC <= 4) {
#pragma unroll
            for (int j = 0; j < NM; ++j) {
                const int k = tid + kThreadsDT * j;
                if (cmax[j] >= thr && k < nck)
#pragma unroll
                    for (int e = 0; e < 8; ++e) collect(ch[j].at(e), head + 8 * k + e);
            }
        } else {
            uint32_t hits = 0;
#pragma unroll
            for (int j = 0; j < NM; ++j) hits |= static_cast<uint32_t>(cmax[j] >= thr && tid + kThreadsDT * j < nck) << j;
            for (; hits; hits &= hits - 1) {
                const int k = tid + kThreadsDT * __builtin_ctz(hits);
                Chunk<T> again;
                again.load(body + 8 * k);
#pragma unroll
                for (int e = 0; e < 8; ++e) collect(again.at(e), head + 8 * k + e);
            }
        }
        if constexpr (NC == 0)
            for (int k = tid + kThreadsDT * kStream; k < nck; k += kThreadsDT)
                for (int e = 0; e < 8; ++e) collect(entry(body + 8 * static_cast<int64_t>(k) + e), head + 8 * k + e);
    }
    __syncthreads();
    int nc = s_ncand;
    const float lse = BESIDE ? 0.f : s_lse;
    const int64_t out0 = b * out_stride_b + static_cast<int64_t>(w) * K;
    auto emit = [&](int k, unsigned long long key) {     // k-th best of the row
        token_out[out0 + k] = static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(key));
        const float sc = BESIDE ? key_value(key) : c + (key_value(key) - lse);       // (kBeside: the logit, for the last workgroup)
        if constexpr (SEL)                               // may be read by another workgroup in this kernel
            __hip_atomic_store(reinterpret_cast<uint32_t*>(score_out + out0 + k), __float_as_uint(sc),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            score_out[out0 + k] = sc;
        if (parent_out) parent_out[out0 + k] = par;
        if constexpr (SEL) {
            if (lone && k < sel.M) {
                sel.sel_out[b * sel.M + k] = k + sel.index_base;
                if (sel.sel_score_out) sel.sel_score_out[b * sel.M + k] = sc;
            }
        }
    };
    auto rank_them = [&]() __attribute__((always_inline)) {
        for (int i = tid >> 4; i < nc; i += kThreadsDT / 16) {           // a row of 16 lanes per entry
            const unsigned long long k = s_cand[i];
            const int beaten = keys_above(s_cand, nc, k);
            if ((tid & 15) == 0 && beaten < K) emit(beaten, k);
        }
    };
    if (nc <= kRankDirect) {                             // uniform
        rank_them();
    } else {
        // ---- too many: a threshold from the threads' best entries -----------------------------------------
        // every entry of this thread, in ascending token order
        auto each = [&](auto&& f) __attribute__((always_inline)) {
            if (vs >= 0 && vs < head) f(es, vs);
            if constexpr (NC > 0) {
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int k = tid + kThreadsDT * j;
                    if (k < nck)
#pragma unroll
                        for (int e = 0; e < 8; ++e) f(ch[j].at(e), head + 8 * k + e);
                }
            } else {
                for (int k0 = tid; k0 < nck; k0 += U * kThreadsDT) {
#pragma unroll
                    for (int u = 0; u < U; ++u) ch[u].load(body + 8 * static_cast<int64_t>(min(k0 + kThreadsDT * u, nck - 1)));
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int k = k0 + kThreadsDT * u;
                        if (k < nck)
#pragma unroll
                            for (int e = 0; e < 8; ++e) f(ch[u].at(e), head + 8 * k + e);
                    }
                }
            }
            if (vs >= tail0) f(es, vs);
        };
        // the key of the best of them that comes after (bx, bv) in the order, 0 if there is none (a real key is never 0);
        // "greater" alone keeps the lowest token among equal logits (no logit is NaN)
        auto best_after = [&](float bx, int bv) __attribute__((always_inline)) -> unsigned long long {
            float bf = 0.f;
            int bi = -1;
            each([&](float x, int v) __attribute__((always_inline)) {
                const bool take = ((x < bx) | ((x == bx) & (v > bv))) & ((x > bf) | (bi < 0));
                bf = take ? x : bf;
                bi = take ? v : bi;
            });
            return bi >= 0 ? order_key(bf, bi) : 0ull;
        };
        unsigned long long mine = best_after(INFINITY, -1);
        {
            unsigned long long grp = mine;               // best of the row of 16 lanes
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) {
                const unsigned long long y = __shfl_xor(grp, off);
                grp = y > grp ? y : grp;
            }
            if ((tid & 15) == 0) s_grp_key[tid >> 4] = grp;
            if (tid == 0) { s_thr_key = 0; s_ncand = 0; }
        }
        __syncthreads();
        // the K-th best of `n` keys, if there are so many, becomes the threshold (keys are distinct; 0: no entry)
        auto kth_of = [&](const unsigned long long* keys, int n) __attribute__((always_inline)) {
            if (tid < n) {
                const unsigned long long k = keys[tid];
                int beaten = 0;
#pragma unroll 4
                for (int x = 0; x < n; ++x) beaten += keys[x] > k ? 1 : 0;
                if (beaten == K - 1 && k != 0) s_thr_key = k;
            }
        };
        auto collect_key = [&](unsigned long long k) __attribute__((always_inline)) {
            const int pos = atomicAdd(&s_ncand, 1);
            if (pos < kCandCap) s_cand[pos] = k;
        };
        kth_of(s_grp_key, 64);
        __syncthreads();
        if (mine != 0 && mine >= s_thr_key) collect_key(mine);       // threads of K groups, or all
        __syncthreads();
        nc = s_ncand;
        __syncthreads();
        if (tid == 0) s_ncand = 0;
        kth_of(s_cand, nc);
        __syncthreads();
        const unsigned long long thr_key = s_thr_key;
        if (mine >= thr_key)                             // K threads, or all
            each([&](float x, int v) __attribute__((always_inline)) {
                const unsigned long long k = order_key(x, v);
                if (k >= thr_key) collect_key(k);
            });
        __syncthreads();
        nc = s_ncand;
        if (nc <= kCandCap) {                            // uniform
            rank_them();
        } else {
            // ---- still too many (the best entries sit in few threads): one winner per round; only its owner looks
            // for its next best --------------------------------------------------------------------------
            for (int k = 0; k < K; ++k) {
                const unsigned long long best = wave_max_u64(mine);
                if (lane == 0) s_key[k & 1][wave] = best;
                __syncthreads();                         // (the other buffer was last read two rounds ago)
                unsigned long long win = s_key[k & 1][0];
#pragma unroll
                for (int x = 1; x < kWavesDT; ++x) {
                    const unsigned long long y = s_key[k & 1][x];
                    win = y > win ? y : win;
                }
                if (mine == win) {                       // exactly one thread (K <= V: never empty)
                    emit(k, win);
                    mine = best_after(key_value(win), static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(win)));
                }
            }
        }
    }
    }
    if constexpr (SEL) {
        const int nc = nrows * K, count = min(sel.M, nc);
        auto rest = [&]() __attribute__((always_inline)) {     // what follows the selected ones
            for (int pw = count + tid; pw < sel.M; pw += kThreadsDT) {
                sel.sel_out[b * sel.M + pw] = -1;
                if (sel.sel_score_out) sel.sel_score_out[b * sel.M + pw] = -INFINITY;
            }
            if (tid == 0 && sel.count_out) sel.count_out[b] = count;
        };
        if (lone) {                                        // uniform
            rest();
            return;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's score stores have been acknowledged
        __syncthreads();
        if (tid == 0) {
            int32_t* cnt = sel.counters + b * SPECVLM_COUNTER_STRIDE;
            const int ticket = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int last = ticket == static_cast<int>(gridDim.x) - 1;
            if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = last;
        }
        __syncthreads();
        if (!s_last) return;
        // the request's W*K new candidates (at most kCandCap, checked on the host), one per thread
        float sc = 0.f;
        if (tid < nc) {
            sc = __uint_as_float(__hip_atomic_load(reinterpret_cast<uint32_t*>(score_out + b * out_stride_b + tid),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if constexpr (BESIDE) {
                const int of = tid / K;
                int32_t* const at = sel.counters + b * SPECVLM_COUNTER_STRIDE + 1 + of;
                const float l = __uint_as_float(static_cast<uint32_t>(__hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
                sc = (cum ? cum[b * cum_stride_b + of] : 0.f) + (sc - l);
                score_out[b * out_stride_b + tid] = sc;
            }
            s_cand[tid] = order_key(sc, tid);
        }
        __syncthreads();
        if constexpr (BESIDE) {
            if (tid < nrows) __hip_atomic_store(sel.counters + b * SPECVLM_COUNTER_STRIDE + 1 + tid, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        rank_winners(s_cand, nc, sel.M);
        if (tid < nc) {
            const int pw = pos_of(s_cand, tid);
            if (pw >= 0) {
                sel.sel_out[b * sel.M + pw] = tid + sel.index_base;
                if (sel.sel_score_out) sel.sel_score_out[b * sel.M + pw] = sc;
            }
        }
        rest();
    }
}

__global__ __launch_bounds__(kThreadsDT) void draft_select_kernel(
    int C, int M, const float* __restrict__ score, int64_t score_stride_b, const int32_t* __restrict__ num_cand,
    int index_base, int32_t* __restrict__ sel_out, float* __restrict__ sel_score_out,
    int32_t* __restrict__ count_out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    unsigned long long* s_key = reinterpret_cast<unsigned long long*>(s_dyn);
    const int b = blockIdx.x, tid = threadIdx.x;
    const int c = num_cand ? min(max(num_cand[b], 0), C) : C;
    for (int i = tid; i < c; i += kThreadsDT) s_key[i] = order_key(score[b * score_stride_b + i], i);
    __syncthreads();
    rank_winners(s_key, c, M);
    const int count = min(M, c);
    for (int i = tid; i < c; i += kThreadsDT) {
        const int p = pos_of(s_key, i);
        if (p >= 0) {
            sel_out[b * M + p] = i + index_base;
            if (sel_score_out) sel_score_out[b * M + p] = score[b * score_stride_b + i];
        }
    }
    for (int p = count + tid; p < M; p += kThreadsDT) {
        sel_out[b * M + p] = -1;
        if (sel_score_out) sel_score_out[b * M + p] = -INFINITY;
    }
    if (tid == 0 && count_out) count_out[b] = count;
}

__global__ __launch_bounds__(kThreadsDT) void draft_finalize_kernel(
    int C, int N_max, const float* __restrict__ cand_score, const int32_t* __restrict__ cand_parent,
    const int32_t* __restrict__ cand_token, int64_t cand_stride_b, const int32_t* __restrict__ num_cand,
    const int32_t* __restrict__ root_token, int32_t* __restrict__ parent_out, int32_t* __restrict__ draft_tok_out,
    int32_t* __restrict__ node_cand_out, int32_t* __restrict__ num_nodes_out, int32_t* __restrict__ err_flag) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    unsigned long long* s_key = reinterpret_cast<unsigned long long*>(s_dyn);
    const int b = blockIdx.x, tid = threadIdx.x;
    int err = 0;
    int c = num_cand ? num_cand[b] : C;
    if (c < 0 || c > C) {
        err |= SPECVLM_ERR_BAD_NUM_NODES;
        c = min(max(c, 0), C);
    }
    const int M = N_max - 1;
    const int64_t base = b * cand_stride_b;
    // what the chosen ones will need, for the first candidate of a thread on its way while they are ranked; after the scores,
    // which are waited for first
    float score0 = 0.f;
    int parent0 = -1, token0 = -1, root = -1;
    if (tid < c) {
        score0 = cand_score[base + tid];
        asm volatile("" ::: "memory");
        parent0 = cand_parent[base + tid];
        token0 = cand_token[base + tid];
        s_key[tid] = order_key(score0, tid);
    }
    if (tid == 0) root = root_token[b];
    for (int i = tid + kThreadsDT; i < c; i += kThreadsDT) s_key[i] = order_key(cand_score[base + i], i);
    __syncthreads();
    rank_winners(s_key, c, M);
    const int count = min(M, c);
    for (int i = tid; i < c; i += kThreadsDT) {
        const int p = pos_of(s_key, i);
        if (p < 0) continue;
        const int cp = i == tid ? parent0 : cand_parent[base + i];
        int pn = -1;
        if (cp < -1 || cp >= i) {
            err |= SPECVLM_ERR_BAD_PARENT;
        } else if (cp < 0) {
            pn = 0;
        } else if (pos_of(s_key, cp) < 0) {
            err |= SPECVLM_ERR_TREE_NOT_CLOSED;         // a chosen candidate whose parent was not chosen
        } else {
            pn = pos_of(s_key, cp) + 1;
        }
        const int node = p + 1;
        parent_out[b * N_max + node] = pn;
        draft_tok_out[b * N_max + node] = i == tid ? token0 : cand_token[base + i];
        if (node_cand_out) node_cand_out[b * N_max + node] = i;
    }
    for (int node = count + 1 + tid; node < N_max; node += kThreadsDT) {
        parent_out[b * N_max + node] = -1;
        draft_tok_out[b * N_max + node] = -1;
        if (node_cand_out) node_cand_out[b * N_max + node] = -1;
    }
    if (tid == 0) {
        parent_out[b * N_max] = -1;
        draft_tok_out[b * N_max] = root;
        if (node_cand_out) node_cand_out[b * N_max] = -1;
        num_nodes_out[b] = count + 1;
    }
    if (err && err_flag) atomicOr(err_flag, err);
}

}  // namespace

int32_t launch_draft_topk(int32_t dtype, int32_t B, int32_t W, int32_t V, int32_t K, const void* logits,
                          int64_t stride_b, int64_t stride_w, const float* cum, int64_t cum_stride_b,
                          const int32_t* parent_idx, int64_t parent_stride_b, float* score_out,
                          int32_t* token_out, int32_t* parent_out, int64_t out_stride_b, float* lse_out,
                          int32_t M, int32_t index_base, int32_t* sel_out, float* sel_score_out,
                          int32_t* count_out, int32_t* counters, hipStream_t stream) {
    const bool fused = counters != nullptr;             // with the selection of the level's candidates
    const bool beside = fused && sums_beside(dtype, B, W, V, !cum);
    const dim3 grid(beside ? 2 * W : W, B), block(kThreadsDT);
    const SelArgs sel{M, index_base, sel_out, sel_score_out, count_out, counters, W};
#define SPECVLM_LAUNCH_TK2(T, NC, LEVEL)                                                                            \
    hipLaunchKernelGGL((draft_topk_kernel<T, NC, LEVEL>), grid, block, 0, stream, V, K, static_cast<const T*>(logits), \
                       stride_b, stride_w, cum, cum_stride_b, parent_idx, parent_stride_b, score_out,               \
                       token_out, parent_out, out_stride_b, lse_out, sel)
#define SPECVLM_LAUNCH_TK(T, NC)                                      \
    do {                                                              \
        if (beside) SPECVLM_LAUNCH_TK2(T, NC, kBeside);               \
        else if (fused) SPECVLM_LAUNCH_TK2(T, NC, kSelect);           \
        else SPECVLM_LAUNCH_TK2(T, NC, kPlain);                       \
    } while (0)
    if (dtype == SPECVLM_BF16) {
        if (V <= 4 * 8 * kThreadsDT) SPECVLM_LAUNCH_TK(uint16_t, 4);
        else if (V <= 8 * 8 * kThreadsDT) SPECVLM_LAUNCH_TK(uint16_t, 8);
        else SPECVLM_LAUNCH_TK(uint16_t, 0);
    } else {
        if (V <= 4 * 8 * kThreadsDT) SPECVLM_LAUNCH_TK(float, 4);
        else if (V <= 8 * 8 * kThreadsDT) SPECVLM_LAUNCH_TK(float, 8);
        else SPECVLM_LAUNCH_TK(float, 0);
    }
#undef SPECVLM_LAUNCH_TK
#undef SPECVLM_LAUNCH_TK2
    return check_launch();
}

int32_t launch_draft_select(int32_t B, int32_t C, int32_t M, const float* score, int64_t score_stride_b,
                            const int32_t* num_cand, int32_t index_base, int32_t* sel_out,
                            float* sel_score_out, int32_t* count_out, hipStream_t stream) {
    const size_t lds = static_cast<size_t>((C + 1) & ~1) * 8;         // keys are ranked in pairs
    hipLaunchKernelGGL(draft_select_kernel, dim3(B), dim3(kThreadsDT), lds, stream, C, M, score, score_stride_b,
                       num_cand, index_base, sel_out, sel_score_out, count_out);
    return check_launch();
}

int32_t launch_draft_finalize(int32_t B, int32_t C, int32_t N_max, const float* cand_score,
                              const int32_t* cand_parent, const int32_t* cand_token, int64_t cand_stride_b,
                              const int32_t* num_cand, const int32_t* root_token, int32_t* parent_out,
                              int32_t* draft_tok_out, int32_t* node_cand_out, int32_t* num_nodes_out,
                              int32_t* err_flag, hipStream_t stream) {
    const size_t lds = static_cast<size_t>((C + 1) & ~1) * 8;         // keys are ranked in pairs
    hipLaunchKernelGGL(draft_finalize_kernel, dim3(B), dim3(kThreadsDT), lds, stream, C, N_max, cand_score,
                       cand_parent, cand_token, cand_stride_b, num_cand, root_token, parent_out, draft_tok_out,
                       node_cand_out, num_nodes_out, err_flag);
    return check_launch();
}

}  // namespace specvlm
