// Tree-masked verification attention for bf16 caches: 64 query rows per workgroup, a key stream per wavefront.
//
// For batches whose (request, head) pairs fill the chip with long streams.  What bounds such a call is the K/V stream (6.2 - 7
// TB/s over all compute units, 57 GB/s into one of them) as long as a step's own chain is shorter; attn_mfma.hip needs
// 0.43 us per 32-key tile and compute unit (two streams, a barrier per step, every tile read from LDS by four wavefronts),
// more than the stream where K and V come from L2 (grouped heads) or few long requests are left.  Here:
//
//   grid      (KV head, column, block of 64 rows of the group), 4 wavefronts each, all 64 rows in every one.  A column is a key range of
//             a request: one per request (attn_streams_kernel), or as many as its length earns, worked out by every workgroup
//             from the lengths (attn_shares_kernel; the host does not know them).  Wavefront w has the tiles of stream w ranges + split,
//             so a tile is read from LDS once, there is no barrier in the loop, and four tiles take 0.73 us without fetches.  Columns
//             inside heads, so that every XCD has its part of the longest request (with the requests outermost one XCD has all of
//             it: 8 x 32 heads, 906 - 170 keys 21.6 -> 20.0; equal lengths + 0.2)
//   product   v_mfma_f32_32x32x16_bf16: half the matrix instructions of 16 x 16 x 32, and a lane holds 2 query rows x 16 keys
//             instead of 4 x 8 (half the softmax state).  S^T = K Q^T of tile j + 1 stands beside the softmax of tile j
//             in one block, so that the compiler interleaves matrix and vector instructions; the last three tiles are
//             unrolled to keep it that way (one loop with run-time conditions costs 1 us per call)
//   fetch     as in attn_wave.hip: direct-to-LDS, two K and two V areas per wavefront, K three tiles and V two tiles ahead
//   merge     the four streams meet in LDS, every wavefront owns 32 head dims of all rows; key ranges as in attn_wave.hip
//
//   tree      ancestor masks while the first tile is on its way, two instructions a masked score; what needs no tile before the wait for
//             the first (8 x 32 heads, 170 - 906 keys 20.1 -> 19.2, eight of 443 17.0 -> 15.7, 4 x 32 / 8 heads below 20.6 -> 19.7)
//
// us per call (HIP-graph replay), attn_mfma / attn_wave -> here, before the last point; head size 128, 60 - 64 nodes unless said: 4 x 32 query / 8
// KV heads, 2048, 1311, 3000, 777 keys 27.6 -> 20.1 (23.5 with two ranges each); 8 x 32 / 16 heads, 4788 keys 82.4 -> 65.7; 3 x 32 / 16 heads,
// 3664 - 500 keys 34.8 -> 20.4 (27.2); 4 x 40 heads, 671 keys 18.5 -> 16.4; 6 x 32 heads, 2800 - 300 keys 44.7 -> 33.8 (35.6); 5 x 40 heads of
// 64, 1935 keys 26.0 -> 20.4.  Tried and slower: two wavefronts sharing a stream of 128 rows (26.3 at the first of these), wavefronts
// instead of whole workgroups dealt out by length (24.4), the row blocks of a head walking their tiles in different orders so that each finds
// in L2 what another fetched (28.1; by one to three tiles of every four 25.0), tiles touched three steps ahead by one of them (+ 1.7), loads that stay in L2 where blocks share them (a branch in
// the loop: + 1; without one 22.8 - 24.6 against 23.9 - 24.4).
#include <type_traits>

#include "attn_rows.hpp"

namespace specvlm {

namespace {

// What the two kernels here take beside WaveParams.
struct StreamsParams : WaveParams {
    int B, columns, each;       // workgroups per row block of a KV head; as many per request (attn_plan.hpp)
    int by_length;              // columns go to the requests by their lengths, not `each` to everyone
    int wide;                   // partial results in fp32
    int help;                   // short requests' workgroups bring keys of the longest one into the L2
    uint32_t magic_columns, magic_each;
    float inv_columns, least_gain;   // rounds that a division must save
};

typedef float f32x16 __attribute__((ext_vector_type(16)));

// The greatest of sixteen scores, NaN where one is.
__device__ __forceinline__ float max16(const f32x16& a) {
    auto max3 = [](float x, float y, float z) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z); };
    const float u = max3(a[0], a[1], a[2]), v = max3(a[3], a[4], a[5]), w = max3(a[6], a[7], a[8]), x = max3(a[9], a[10], a[11]);
    const float y = max3(a[12], a[13], a[14]);
    return max3(max3(u, v, w), max3(x, y, a[15]), a[15]);
}

// op over lanes 0 .. i of this lane's row of 16.
template <typename Op>
__device__ __forceinline__ int row_scan(int x, Op op) {
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true));     // row_shr:1, zero where there is none
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true));
    x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true));
    return op(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true));
}

// What the other half of the wavefront (lane ^ 32) holds.
__device__ __forceinline__ float other_half(float x) {
    const uint32_t a = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);     // lower half everywhere, upper half everywhere
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

template <int D, bool PAGED, bool SHARES>
__device__ __forceinline__ void attend(const StreamsParams& p) {
    constexpr int NC = D / 16;                 // QK^T contraction steps of 16
    constexpr int NT = D / 32;                 // output blocks of 32 head dims
    constexpr int ROWG = D / 8;                // 16-byte granules per K/V row
    constexpr int RPI = 64 / ROWG;             // rows per load instruction (4 or 8)
    constexpr int NH = 16 / RPI;               // load instructions per half tile (4 or 2)
    constexpr int KLD = 2 * NH;                // ... per K (or V) tile
    constexpr int kTileBytes = kKeys * D * 2;
    constexpr int kSlotBytes = 2 * kTileBytes;           // K tile then V tile
    constexpr int kRingBytes = 2 * kSlotBytes;           // two slots per wavefront
    constexpr int NQ = kQRows / RPI / 4;                 // query-row load instructions per wavefront
    constexpr int OWN = NT / 2;                          // (32 query rows, 32 head dims) blocks of an owner at the merge
    static_assert(kWaveWgs * kRingBytes >= 4 * 3 * OWN * 4096, "merge scratch must fit in the rings");
    static_assert(kSharesRound == kWaveWgs * kKeys, "a round is a tile of every stream");

    constexpr bool HELPS = !SHARES && !PAGED && D == 128;      // (paged 0 - 2 % faster, head size 64 up to 1 % slower)

    __shared__ __attribute__((aligned(1024))) unsigned char s_ring[kWaveWgs * kRingBytes];
    __shared__ __attribute__((aligned(1024))) unsigned char s_q[kQRows * D * 2];
    __shared__ float s_m[kWaveWgs][kQRows];
    __shared__ float s_l[kWaveWgs][kQRows];
    __shared__ int s_par[kWaveWgs][64];
    __shared__ int s_blocks[PAGED ? kWaveWgs : 1][64];

    // work item: (KV head, column, row block); every XCD gets a contiguous range of items, so that the blocks of a head
    // share an L2, the first ones an item more where their number is no multiple of 8 (dealt out to the XCDs in turn: 39.2 us for the
    // 210 of 3 x 35 query / 7 KV heads, 4060 keys, now 29.6; the 250 of 5 x 25 / 5, 5312 keys 53.3, now 37.0).
    const uint32_t xcd = blockIdx.x & 7;
    const uint32_t work = xcd * (gridDim.x >> 3) + min(xcd, gridDim.x & 7) + (blockIdx.x >> 3);
    const uint32_t group_item = divide(work, p.magic_rb);
    const int rb = work - group_item * p.row_blocks;
    const int hk = divide(group_item, p.magic_columns);
    const int column = group_item - hk * p.columns;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;

    typedef const __attribute__((address_space(4))) int32_t* const_i32;
    // (dealt out evenly, as if all requests had one length; corrected below)
    int b = SHARES ? min(static_cast<int>(divide(column, p.magic_each)), p.B - 1) : column;
    int ranges = SHARES ? p.each : 1, split = SHARES ? min(column - b * p.each, p.each - 1) : 0;
    int n_raw = p.num_nodes ? ((const_i32)p.num_nodes)[b] : p.N_max;
    int P_raw = ((const_i32)p.prefix_len)[b];

    unsigned char* ring = s_ring + wave * kRingBytes;
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    typedef __attribute__((address_space(3))) int lds_int;
    const uint32_t ring_lds = (uint32_t)(uintptr_t)(lds_byte*)ring;

    if (SHARES ? p.by_length : HELPS && p.help) {          // lane i (mod 16): request i
        const int at = min(lane & 15, p.B - 1);
        dma4(p.prefix_len + at, (uint32_t)(uintptr_t)(lds_byte*)s_m[wave]);
        if (p.num_nodes) dma4(p.num_nodes + at, (uint32_t)(uintptr_t)(lds_byte*)s_l[wave]);
    }
    // the parent array before the rest (every wavefront its own copy)
    auto request_parents = [&]() __attribute__((always_inline)) {
        dma4(p.parent + static_cast<int64_t>(b) * p.N_max + min(lane, p.N_max - 1), (uint32_t)(uintptr_t)(lds_int*)s_par[wave]);
    };
    request_parents();

    // ---- tile fetch -------------------------------------------------------------------------
    const int lrow = lane / ROWG, lpos = lane % ROWG;
    const uint32_t row_bytes = static_cast<uint32_t>(p.g.stride_t) * 2u;
    const uint32_t lrow_off = __umul24(lrow, row_bytes);   // (row_bytes < 2^24: checked on the host)
    // V granules: the 64-byte block of 32 head dims c of row r lands at block c ^ vswz(r)
    auto vswz = [](int r) { return D == 128 ? (r & 3) : ((r >> 1) & 1); };
    uint32_t voff_k[NH], voff_v[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        const int r = i * RPI + lrow;
        voff_k[i] = lrow_off + ((lpos ^ (r & (ROWG - 1))) << 4) + i * (RPI * row_bytes - 1024);   // (row_bytes >= 2 D)
        voff_v[i] = lrow_off + ((lpos ^ (vswz(r) << 2)) << 4) + i * (RPI * row_bytes - 1024);
    }
    int nstream, stream;
    int64_t head_off, tile_step;
    const uint16_t *k_next, *v_next;                       // contiguous: the next tile to request
    auto place = [&]() __attribute__((always_inline)) {
        nstream = kWaveWgs * ranges;
        stream = wave * ranges + split;
        head_off = hk * p.g.stride_h + (PAGED ? 0 : b * p.g.stride_b);                 // elements
        tile_step = static_cast<int64_t>(nstream) * kKeys * p.g.stride_t;              // from one tile of the stream to its next
        // (a first tile beyond the cache is replaced by the cache's first: never used)
        const int64_t off = head_off + (PAGED || stream * kKeys >= p.g.capacity ? 0 : static_cast<int64_t>(stream) * kKeys * p.g.stride_t);
        k_next = p.k + off;
        v_next = p.v + off;
    };
    place();
    const int64_t half_step = 16 * p.g.stride_t;
    // Tile j of this stream, K or V, into slot j % 2: two halves of 16 rows.  The capacity is a multiple of 16 (host), so a half
    // lies inside the cache or beyond it; one beyond is replaced by the tile's first half (its keys do not exist, weight zero).
    auto issue = [&](const uint16_t*& src, const uint32_t (&voff)[NH], int area, int j, const int (&phys)[2]) __attribute__((always_inline)) {
        const uint32_t dst = ring_lds + (j & 1) * kSlotBytes + area;
        if constexpr (PAGED) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
                dma_half<D>(src + min(max(phys[x], 0), p.g.num_blocks - 1) * p.g.stride_b, voff, dst + x * (kTileBytes / 2));
        } else {
            const int lo = (stream + j * nstream) * kKeys;
            dma_half<D>(src, voff, dst);
            dma_half<D>(src + (lo + 16 < p.g.capacity ? half_step : 0), voff, dst + kTileBytes / 2);
            src += tile_step;
        }
    };
    auto issue_k = [&](int j, const int (&phys)[2]) __attribute__((always_inline)) { issue(k_next, voff_k, 0, j, phys); };
    auto issue_v = [&](int j, const int (&phys)[2]) __attribute__((always_inline)) { issue(v_next, voff_v, kTileBytes, j, phys); };
    int phys[2] = {0, 0};
    // query rows of this block: row r of the block is row R = 64 rb + r of the group's (head, node) rows
    const int rows_total = p.group * p.N_max;
    const uint32_t q_lds = (uint32_t)(uintptr_t)(lds_byte*)s_q;
    const int row0 = rb * kQRows;
    const int q_row = static_cast<int>(p.q_sn) * 2, q_head = static_cast<int>(p.q_sh) * 2;     // bytes (checked on the host)
    auto request_first = [&]() __attribute__((always_inline)) {
        if constexpr (!PAGED) issue_k(0, phys);
        const uint16_t* q_base = p.q + b * p.q_sb + static_cast<int64_t>(hk * p.group) * p.q_sh;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int r = (wave * NQ + i) * RPI + lrow;
            const int R = min(row0 + r, rows_total - 1);
            const int hh = divide(R, p.magic_nmax);
            const int node = R - hh * p.N_max;
            dma16s(q_base, static_cast<uint32_t>(node * q_row + hh * q_head) + ((lpos ^ (r & (ROWG - 1))) << 4), q_lds + (wave * NQ + i) * 1024);
        }
    };
    request_first();
    // The columns of a row block, dealt out by the lengths: every request gets as many as bring its rounds of four tiles down to the
    // least `len` for which they suffice, one each if that saves too little.  Lanes 16 g + i look at request i for the g-th of four
    // lengths.  (Through the scalar cache, request by request, this took 1 us longer; with the requests above sent only afterwards
    // 0.7 us.  What was requested for another request or range lands before what replaces it: loads return in order.)
    if (SHARES && p.by_length) {
        wait_vmcnt<1 + (PAGED ? 0 : KLD) + NQ>();
        const int my_P = __float_as_int(s_m[wave][lane]);
        const int my_n = p.num_nodes ? __float_as_int(s_l[wave][lane]) : p.N_max;
        const int keys = keys_of(my_P, my_n, p.N_max, p.g.capacity);
        const int rounds = (lane & 15) < p.B ? (keys + kSharesRound - 1) / kSharesRound : 0;
        const int longest = __builtin_amdgcn_readlane(row_scan(rounds, [](int x, int y) { return max(x, y); }), 15);
        const int total = __builtin_amdgcn_readlane(row_scan(rounds, [](int x, int y) { return x + y; }), 15);
        auto columns_for = [&](float len) __attribute__((always_inline)) { return columns_of(rounds, len, __builtin_amdgcn_rcpf(len)); };
        auto upto_for = [&](float len) __attribute__((always_inline)) { return row_scan(columns_for(len), [](int x, int y) { return x + y; }); };
        float len = ceilf(fmaxf(total * p.inv_columns, longest * (1.f / kMostRanges)) - 0.01f) + (lane >> 4);
        unsigned long long fits;
        for (;; len += 4.f) {                              // ends where len >= longest: a column each
            const int upto = upto_for(len);                // (not in the condition below: every lane takes part)
            if ((fits = __ballot(((lane & 15) == 15) & (upto <= p.columns))) != 0) break;
        }
        len = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(len), __builtin_ctzll(fits)));
        if (longest - len < p.least_gain) len = longest;
        const int mine = columns_for(len), upto = upto_for(len);
        const unsigned long long here = __ballot((lane < 16) & (column < upto) & (column >= upto - mine));
        if (!here) {                                       // a column too many
            wait_vmcnt<0>();
            return;
        }
        const int to = __builtin_ctzll(here);
        const int to_ranges = __builtin_amdgcn_readlane(mine, to), to_split = column - __builtin_amdgcn_readlane(upto, to) + to_ranges;
        P_raw = __builtin_amdgcn_readlane(my_P, to);
        n_raw = __builtin_amdgcn_readlane(my_n, to);
        if (to != b || to_split != split || to_ranges != ranges) {
            b = to;
            split = to_split;
            ranges = to_ranges;
            request_parents();
            place();
            request_first();
        }
    }
    const uint32_t head_block = hk * p.row_blocks + rb;
    const uint32_t unit = b * p.H_kv * p.row_blocks + head_block;
    if constexpr (!PAGED) issue_v(0, phys);

    int err = 0;
    int n = n_raw;
    const int P = P_raw;
    if (n < 1 || n > p.N_max) err |= SPECVLM_ERR_BAD_NUM_NODES;
    n = min(max(n, 1), p.N_max);
    if (!length_fits(P, n, p.g.capacity)) err |= SPECVLM_ERR_BAD_LENGTH;
    const int S = P + n;
    const int ntile = (S + kKeys - 1) / kKeys;
    const int my_tiles = (!err && stream < ntile) ? static_cast<int>(static_cast<uint32_t>(ntile - stream + nstream - 1) / static_cast<uint32_t>(nstream)) : 0;
    // Block ids: the first three tiles' through the scalar cache (the third's again for V); from there on lane 2i + x holds that of
    // half x of tile i (mod 32), fetched for 32 tiles at once.  (A scalar load per tile shares its counter with the LDS reads, which
    // then all have to wait for it: 2 x 64 query / 8 KV heads, 4500 + 900 keys 33.4 us; 3 x 32 / 8, 3000 - 500 26.4.)
    const int last_blk = (max(S, 1) - 1) >> 4;
    const int64_t table_row = static_cast<int64_t>(b) * p.g.max_blocks;
    bool bad_block = false;
    auto fetch_blocks = [&](int j, int (&phys)[2]) __attribute__((always_inline)) {
        if constexpr (PAGED) {
#pragma unroll
            for (int x = 0; x < 2; ++x) phys[x] = ((const_i32)p.g.block_table)[table_row + min((stream + j * nstream) * 2 + x, last_blk)];
        }
    };
    auto request_ids = [&](int j) __attribute__((always_inline)) {       // of tiles j .. j + 31 (past the last: the request's last block again)
        const int blk = min((stream + (j + (lane >> 1)) * nstream) * 2 + (lane & 1), last_blk);
        dma4(p.g.block_table + table_row + blk, (uint32_t)(uintptr_t)(lds_int*)s_blocks[PAGED ? wave : 0]);
    };
    int ids = 0;
    auto read_ids = [&]() __attribute__((always_inline)) {
        ids = s_blocks[PAGED ? wave : 0][lane];
        bad_block = bad_block || static_cast<uint32_t>(ids) >= static_cast<uint32_t>(p.g.num_blocks);
    };
    auto blocks_of = [&](int j, int (&phys)[2]) __attribute__((always_inline)) {
        if constexpr (PAGED) {
#pragma unroll
            for (int x = 0; x < 2; ++x) phys[x] = __builtin_amdgcn_readlane(ids, ((2 * j) & 63) + x);
        }
    };
    if constexpr (PAGED) {
        if (my_tiles > 0) request_ids(0);
    }
    if (PAGED && my_tiles > 0) { fetch_blocks(0, phys); issue_k(0, phys); issue_v(0, phys); }
    if (my_tiles > 1) { fetch_blocks(1, phys); issue_k(1, phys); issue_v(1, phys); }
    int phys2[2] = {0, 0};
    if (my_tiles > 2) fetch_blocks(2, phys2);

    const float c2 = p.c2, tau = p.tau;
    // K fragments of a tile (A operand): lane (key l32, half hf) holds dims 16c + 8hf .. +7; the query rows likewise
    uint32_t kaddr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) kaddr[c] = l32 * (ROWG * 16) + (((2 * c + hf) ^ (l32 & (ROWG - 1))) << 4);
    bf16x8 ka[NC];
    auto read_k = [&](int slot_off) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c) ka[c] = *reinterpret_cast<const bf16x8*>(ring + slot_off + kaddr[c]);
    };
    // Ancestor-or-self masks of this lane's two query rows, while the first tile is on its way (in the tile that needs them, the last of its
    // stream, they stand in the call's chain): pointer doubling over the lanes (lane i holds node i).  Requested after the parents: K0 (an early
    // request), the query rows, then block ids, K0, V0, K1, V1.
    if (my_tiles > 1) wait_vmcnt<NQ + 4 * KLD + (PAGED ? 1 : 0)>();
    else if (my_tiles == 1) wait_vmcnt<NQ + 2 * KLD + (PAGED ? 1 : 0)>();
    else wait_vmcnt<NQ>();
    const int par = s_par[wave][lane];
    const bool bad_par = lane < n && (lane == 0 ? par != -1 : (par < 0 || par >= lane));
    if (__any(bad_par)) err |= SPECVLM_ERR_BAD_PARENT;
    uint32_t anc_lo[2], anc_hi[2];
    {
        uint32_t mlo = lane < 32 ? 1u << (lane & 31) : 0u, mhi = lane < 32 ? 0u : 1u << (lane & 31);
        int up = lane < n && !err ? par : -1;              // (a bad array may have cycles)
#pragma unroll 1
        while (__any(up >= 0)) {
            const int src = max(up, 0) * 4;
            const uint32_t alo = __builtin_amdgcn_ds_bpermute(src, mlo), ahi = __builtin_amdgcn_ds_bpermute(src, mhi);
            const int up2 = __builtin_amdgcn_ds_bpermute(src, up);
            if (up >= 0) { mlo |= alo; mhi |= ahi; up = up2; }
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            const int R = min(row0 + qb * 32 + l32, rows_total - 1);
            const int node = R - divide(R, p.magic_nmax) * p.N_max;
            anc_lo[qb] = __builtin_amdgcn_ds_bpermute(node * 4, mlo);
            anc_hi[qb] = __builtin_amdgcn_ds_bpermute(node * 4, mhi);
        }
    }
    // Softmax state of query row 32 qb + l32 (both halves agree): reference maximum, the same times c2 (0 while no key was
    // seen), the maximum that moves it, and this lane's part of the sum of the row's weights.
    // acc[qb][t][i]: O^T row 32t + 8 (i / 4) + 4 hf + i % 4.
    float m_run[2], mrc[2], thr[2], l_run[2];
    f32x16 acc[2][NT];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        m_run[qb] = -INFINITY;
        thr[qb] = -INFINITY;
        mrc[qb] = 0.f;
        l_run[qb] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[qb][t][i] = 0.f;
    }
    // V operands: va[t][x] element e is key 16x + 8 (e / 4) + 4 hf + e % 4, dim 32t + l32.  A transposing read hands lane i of a
    // 16-lane block four keys at dim i of the 16 that the block's lanes address (lane j: key j / 4, dims 4 (j % 4) ..)
    const int k0 = 4 * hf + ((lane & 15) >> 2);
    const uint32_t vaddr = kTileBytes + k0 * (ROWG * 16) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8 + (vswz(k0) << 6);
    // (all of this before the wait: the compiler would put it behind, where the first products wait for it)
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(kaddr[c]));
    asm volatile("" : : "v"(vaddr));
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int t = 0; t < NT; ++t) asm volatile("" : "+v"(acc[qb][t]));
    // requested after the query rows: V0, K1, V1 (an early request) or K0, V0, K1, V1
    if (my_tiles > 1) wait_vmcnt<3 * KLD>();
    else if (my_tiles == 1) wait_vmcnt<KLD>();
    else wait_vmcnt<0>();
    __syncthreads();
    if constexpr (PAGED) {
        if (my_tiles > 0) read_ids();
    }
    bf16x8 qf[2][NC];
    if (err) {                                             // the same in every wavefront of the request
        if (tid == 0 && p.err_flag) atomicOr(p.err_flag, err);
        wait_vmcnt<0>();
        return;
    }
    bf16x8 va[NT][2];
    auto read_v = [&](int t, int slot_off) __attribute__((always_inline)) {
        const uint32_t a = (vaddr ^ (t << 6)) + slot_off;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const s16x4 lo = lds_read_tr16(ring + a + (16 * x) * ROWG * 16);
            const s16x4 hi = lds_read_tr16(ring + a + (16 * x + 8) * ROWG * 16);
            const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            va[t][x] = __builtin_bit_cast(bf16x8, both);
        }
    };
    // S^T = K Q^T: s[qb][i] = score of key 8 (i / 4) + 4 hf + i % 4 of the tile against query row 32 qb + l32
    f32x16 s[2], s_next[2];
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto scores = [&](f32x16& d, int qb) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c], qf[qb][c], c ? d : zero, 0, 0, 0);
    };
    bf16x8 pf[2][2];
    auto weights = [&](int qb) __attribute__((always_inline)) {     // exp2(S^T) packed to bf16 is the B operand of PV
        float pr[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) pr[i] = fast_exp2(fmaf(s[qb][i], c2, -mrc[qb]));
        float sum[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = (pr[4 * i] + pr[4 * i + 1]) + (pr[4 * i + 2] + pr[4 * i + 3]);
        l_run[qb] += (sum[0] + sum[1]) + (sum[2] + sum[3]);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(pr[8 * x + 2 * e], pr[8 * x + 2 * e + 1]);
            pf[qb][x] = __builtin_bit_cast(bf16x8, w);
        }
    };
    // A column a request: where one is longer than the mean, its workgroups are still at work when the others have ended, and what bounds them
    // is what one compute unit takes in of HBM, 57 GB/s; from the L2 it is 109.  So the workgroups of a head's other requests touch every
    // 128-byte line of rounds that it has yet to come to (which ones: lengths.hpp) as soon as their own first tiles are on their way.  Touched
    // lines go to LDS that nothing reads any more.  Where the workgroups of a head are all on one XCD (KV heads a multiple of 8) they find that
    // one's L2; where a head lies across two of them (8 x 32 / 4: every one) some touch for an L2 that the longest request does not use.
    // us per call without -> with, same box (8 x 32 heads unless said): 170 - 906 keys 19.7 -> 19.4, another box 19.8 -> 19.2; 900 and seven of 200
    // 18.3 -> 18.0; 90 - 2000 31.3 -> 30.4; heads across two XCDs: 8 x 32 / 4, 170 - 906 14.8 -> 14.7, 90 - 2000 22.3 -> 22.0; 4 x 40 / 10,
    // 200 - 1000 15.7 -> 15.5; 5 x 28, 200 - 1000 17.4 -> 16.5; 7 x 36, 100 - 1800 27.5 -> 26.7; equal lengths even (443 keys 16.4 | 16.5, 503
    // 17.4 | 17.3, 700 21.2 | 21.2).  Tried: only what is beyond the mean (half the gain), after the workgroup's last tile or one before (half),
    // the last rounds where shares are more than eight (7 x 36, 100 - 1800 26.6 -> 27.1; 8 x 32 / 4, 90 - 4000 34.2 -> 34.5; else even), all of
    // this worked out before the wait for the first tile (even; 443 keys 16.5 -> 16.8), the lengths through the scalar cache (even).
    auto help = [&]() __attribute__((always_inline)) {
        const int my_P = __float_as_int(s_m[wave][lane]);
        const int my_n = p.num_nodes ? __float_as_int(s_l[wave][lane]) : p.N_max;
        const int keys = keys_of(my_P, my_n, p.N_max, p.g.capacity);
        const int rounds = (lane & 15) < p.B ? (keys + kSharesRound - 1) / kSharesRound : 0;
        const int longest = __builtin_amdgcn_readlane(row_scan(rounds, [](int x, int y) { return max(x, y); }), 15);
        const int total = __builtin_amdgcn_readlane(row_scan(rounds, [](int x, int y) { return x + y; }), 15);
        const int mean = static_cast<int>(ceilf(total * p.inv_columns - 0.01f));
        if (longest - mean < 2) return;
        const int mine = (lane & 15) < p.B ? rounds_read_ahead(rounds, longest, mean) : 0;
        const int upto = row_scan(mine, [](int x, int y) { return x + y; });
        const int to = __builtin_ctzll(__ballot(rounds == longest)), last = __builtin_amdgcn_readlane(keys, to) - 1;
        const int first = first_read_ahead(longest, __builtin_amdgcn_readlane(upto, 15)), all = min(longest - first, kMostReadAhead);
        const int64_t off = hk * p.g.stride_h + to * p.g.stride_b + (64 * (lane & 1));
        const int end = min(__builtin_amdgcn_readlane(upto, b), all);
        for (int j = __builtin_amdgcn_readlane(upto - mine, b); j < end; ++j) {
            const int key = min((first + j) * kSharesRound + wave * kKeys + (lane >> 1), last);
            dma4(p.k + off + key * p.g.stride_t, (uint32_t)(uintptr_t)(lds_int*)s_par[wave]);
            dma4(p.v + off + key * p.g.stride_t, (uint32_t)(uintptr_t)(lds_int*)s_par[wave]);
        }
    };
    float lmax[2];

    if (my_tiles > 0) {
        read_k(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the K area of slot 0 is free
        if (my_tiles > 2) issue_k(2, phys2);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) qf[qb][c] = *reinterpret_cast<const bf16x8*>(s_q + qb * 32 * ROWG * 16 + kaddr[c]);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                asm volatile("" : "+a"(qf[qb][c]));
                s[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c], qf[qb][c], c ? s[qb] : zero, 0, 0, 0);
            }
        if constexpr (HELPS) {
            if (p.help && rb == 0) help();
        }
        // V0 and K1 (the requests after them: V1, K2; touched lines come on top, their workgroup can wait)
        if (my_tiles > 2) wait_vmcnt<2 * KLD>();
        else if (my_tiles == 2) wait_vmcnt<KLD>();
        else wait_vmcnt<0>();
        if (my_tiles > 1) read_k(kSlotBytes);
#pragma unroll
        for (int t = 0; t < NT; ++t) read_v(t, 0);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) lmax[qb] = max16(s[qb]);
        // The first reference, where every key is visible: as in the step below, with nothing accumulated that it would scale
        if (stream * kKeys + kKeys <= P && __any((lmax[0] > thr[0]) | (lmax[1] > thr[1]))) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                m_run[qb] = fmaxf(m_run[qb], fmaxf(lmax[qb], other_half(lmax[qb])));
                thr[qb] = m_run[qb] + tau;
                mrc[qb] = (m_run[qb] == -INFINITY ? 0.f : m_run[qb]) * c2;
            }
        }
    }
    // One tile.  At its start s holds tile j's scores and lmax their maxima; va (being read) its V operands, ka the next tile's
    // K operands.  LEFT: tiles after this one (3: three or more).
    auto step = [&](auto after, int j) __attribute__((always_inline)) {
        constexpr int LEFT = decltype(after)::value;
        const int slot0 = (stream + j * nstream) * kKeys;
        if (slot0 + kKeys > P) {                           // reaches past the prefix: tree region or tail
            // bit k of `visible`: key slot0 + k.  Its place among this lane's scores is a constant once the lane's half is shifted out, so a
            // score takes two instructions (a sign-extended bit and a bitwise select)
            const int before = P - slot0;                  // keys of the tile in the prefix, < 32
            const uint32_t exist = S - slot0 < 32 ? (1u << (S - slot0)) - 1u : ~0u;
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                const unsigned long long anc = (static_cast<unsigned long long>(anc_hi[qb]) << 32) | anc_lo[qb];
                uint32_t visible = before > 0 ? (anc_lo[qb] << before) | ((1u << before) - 1u) : static_cast<uint32_t>(anc >> -before);
                visible = (visible & exist) >> (4 * hf);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint32_t seen = static_cast<uint32_t>(static_cast<int32_t>(visible << (31 - (8 * (i >> 2) + (i & 3)))) >> 31);
                    s[qb][i] = __uint_as_float((seen & __float_as_uint(s[qb][i])) | (~seen & 0xFF800000u));
                }
                lmax[qb] = max16(s[qb]);
            }
            if (slot0 + kKeys > S) {                       // keys that do not exist: zero weight must meet a finite value
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    uint32_t keep[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {          // dword e of an operand: keys kk, kk + 1
                        const int kk = slot0 + 16 * x + 8 * (e >> 1) + 4 * hf + 2 * (e & 1);
                        keep[e] = (kk < S ? 0xFFFFu : 0u) | (kk + 1 < S ? 0xFFFF0000u : 0u);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        u32x4 w = __builtin_bit_cast(u32x4, va[t][x]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] &= keep[e];
                        va[t][x] = __builtin_bit_cast(bf16x8, w);
                    }
                }
            }
        }
        // Online softmax with a lazily updated reference: a weight may exceed 1; the reference only moves when
        // some score would exceed it by more than 2^kTau (or on the first visible key).
        if (__builtin_expect(__any((lmax[0] > thr[0]) | (lmax[1] > thr[1])), 0)) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                const float mx = fmaxf(lmax[qb], other_half(lmax[qb]));
                const float m_new = fmaxf(m_run[qb], mx);
                const float m_safe = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = m_run[qb] == -INFINITY ? 1.f : fast_exp2((m_run[qb] - m_safe) * c2);
                m_run[qb] = m_new;
                thr[qb] = m_new + tau;
                mrc[qb] = m_safe * c2;
                l_run[qb] *= alpha;
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[qb][t] *= alpha;
            }
        }
        // weights of tile j beside the next tile's scores
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            if constexpr (LEFT > 0) scores(s_next[qb], qb);
            weights(qb);
        }
        const int next_off = ((j + 1) & 1) * kSlotBytes;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // ka and va are in registers: their areas are free
        if constexpr (LEFT >= 2) {
            blocks_of(j + 2, phys);
            int phys3[2] = {0, 0};
            if constexpr (LEFT >= 3 && PAGED) {                // (uniform branches, once in 32 tiles)
                if (((j + 3) & 31) == 0) read_ids();           // landed: the step before has waited past its requests
                blocks_of(j + 3, phys3);
                if (((j + 4) & 31) == 0) request_ids(j + 4);
            }
            issue_v(j + 2, phys);
            if constexpr (LEFT >= 3) issue_k(j + 3, phys3);
        }
        // V of tile j + 1 and K of tile j + 2 have landed (the requests after them: V of j + 2, K of j + 3)
        if constexpr (LEFT >= 3) wait_vmcnt<2 * KLD>();
        else if constexpr (LEFT == 2) wait_vmcnt<KLD>();
        else if constexpr (LEFT == 1) wait_vmcnt<0>();
        if constexpr (LEFT >= 2) read_k(next_off ^ kSlotBytes);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) acc[qb][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[t][x], pf[qb][x], acc[qb][t], 0, 0, 0);
            if constexpr (LEFT >= 1) read_v(t, next_off);
        }
        if constexpr (LEFT >= 1) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) { s[qb] = s_next[qb]; lmax[qb] = max16(s[qb]); }
        }
    };
    {
        int j = 0;
        for (; j < my_tiles - 3; ++j) step(std::integral_constant<int, 3>{}, j);
        if (my_tiles > 2) step(std::integral_constant<int, 2>{}, j++);
        if (my_tiles > 1) step(std::integral_constant<int, 1>{}, j++);
        if (my_tiles > 0) step(std::integral_constant<int, 0>{}, j);
    }

    if (__any(bad_block) && lane == 0 && p.err_flag) atomicOr(p.err_flag, SPECVLM_ERR_BAD_BLOCK);
    // ---- merge the four streams ---------------------------------------------------------------------
    // Owner w takes OWN blocks of 32 rows x 32 dims: both row blocks at dims 32w (head size 128), or rows 32 (w / 2), dims 32 (w % 2).
    auto own_qb = [](int w, int e) { return D == 128 ? e : w >> 1; };
    auto own_t = [](int w, int e) { return D == 128 ? w : w & 1; };
    bool real[OWN];
    int64_t o_off[OWN], lse_off[OWN];
    bool any_real = false;
#pragma unroll
    for (int e = 0; e < OWN; ++e) {
        const int R = row0 + own_qb(wave, e) * 32 + l32;
        const int hh = divide(R, p.magic_nmax);
        const int node = R - hh * p.N_max;
        const int h = hk * p.group + hh;
        real[e] = R < rows_total && node < n;
        any_real = any_real || real[e];
        // lanes 0-31 store dims 16u + 0..7, lanes 32-63 dims 16u + 8..15 of the block
        o_off[e] = b * p.o_sb + node * p.o_sn + static_cast<int64_t>(h) * p.o_sh + 32 * own_t(wave, e) + 8 * hf;
        lse_off[e] = (static_cast<int64_t>(b) * p.H_q + h) * p.N_max + node;
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        l_run[qb] += other_half(l_run[qb]);
        if (hf == 0) {
            s_m[wave][qb * 32 + l32] = m_run[qb];
            s_l[wave][qb * 32 + l32] = l_run[qb];
        }
    }
    __syncthreads();                                       // every stream is done with its ring
    f32x16 out[OWN];
#pragma unroll
    for (int o = 0; o < kWaveWgs; ++o) {
        if (o == wave) {                                   // uniform
#pragma unroll
            for (int e = 0; e < OWN; ++e) out[e] = acc[own_qb(o, e)][own_t(o, e)];
        } else {
            const int idx = wave < o ? wave : wave - 1;
            f32x4* dst = reinterpret_cast<f32x4*>(s_ring) + (o * 3 + idx) * (OWN * 4) * 64 + lane;
#pragma unroll
            for (int e = 0; e < OWN; ++e)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const f32x16& a = acc[own_qb(o, e)][own_t(o, e)];
                    dst[(e * 4 + u) * 64] = f32x4{a[4 * u], a[4 * u + 1], a[4 * u + 2], a[4 * u + 3]};
                }
        }
    }
    __syncthreads();
    float Mq[OWN], Lq[OWN];
#pragma unroll
    for (int e = 0; e < OWN; ++e) {
        const int qrow = own_qb(wave, e) * 32 + l32;
        float m[kWaveWgs], w[kWaveWgs];
#pragma unroll
        for (int x = 0; x < kWaveWgs; ++x) m[x] = s_m[x][qrow];
        Mq[e] = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
        const float m_safe = Mq[e] == -INFINITY ? 0.f : Mq[e];
        Lq[e] = 0.f;
#pragma unroll
        for (int x = 0; x < kWaveWgs; ++x) {               // (in this order in every owner of the rows)
            w[x] = fast_exp2((m[x] - m_safe) * c2);
            Lq[e] += s_l[x][qrow] * w[x];
        }
        out[e] *= wave == 0 ? w[0] : wave == 1 ? w[1] : wave == 2 ? w[2] : w[3];
        const f32x4* src = reinterpret_cast<const f32x4*>(s_ring) + (wave * 3 * OWN + e) * 4 * 64 + lane;
#pragma unroll
        for (int idx = 0; idx < 3; ++idx) {
            const float wx = wave <= idx ? w[idx + 1] : w[idx];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const f32x4 v = src[(idx * OWN * 4 + u) * 64];
#pragma unroll
                for (int i = 0; i < 4; ++i) out[e][4 * u + i] += v[i] * wx;
            }
        }
    }
    if (!__any(any_real)) return;                          // uniform over the splits of the unit as well
    auto store_out = [&](const float (&M)[OWN], const float (&L)[OWN]) {
#pragma unroll
        for (int e = 0; e < OWN; ++e) {
            const float inv = 1.f / L[e];
#pragma unroll
            for (int u = 0; u < 2; ++u) {                  // 16 dims: registers 8u .. 8u + 7
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(out[e][8 * u + 2 * i] * inv, out[e][8 * u + 2 * i + 1] * inv);
                // the halves of the wavefront hold dims 0-3, 8-11 and 4-7, 12-15: the lower keeps 0-7, the upper 8-15
                const auto r0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                const auto r1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                if (real[e]) *reinterpret_cast<u32x4*>(p.o + o_off[e] + 16 * u) = u32x4{r0[0], r1[0], r0[1], r1[1]};
            }
            if (real[e] && p.lse && hf == 0 && own_t(wave, e) == 0) p.lse[lse_off[e]] = M[e] * p.scale + __log2f(L[e]) * kLn2;
        }
    };
    if (!SHARES || ranges == 1) {
        store_out(Mq, Lq);
        return;
    }
    if constexpr (SHARES) {
        // ---- split partials ----------------------------------------------------------------------------
        // partial results: 16-byte vectors, OWN x 2 a lane as bf16, OWN x 4 as fp32 (calls that the library does not split by itself)
        const int64_t part0 = static_cast<int64_t>(head_block) * p.columns + column - split;
        const int vectors = p.wide ? OWN * 4 : OWN * 2;
        const int part_bytes = kWaveWgs * vectors * 1024;      // one split's partial
        {
            unsigned char* dst = p.ws_acc + (part0 + split) * part_bytes + wave * vectors * 1024 + lane * 16;
            if (p.wide) {
#pragma unroll
                for (int e = 0; e < OWN; ++e)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        u32x4 x;
#pragma unroll
                        for (int i = 0; i < 4; ++i) x[i] = __float_as_uint(out[e][4 * u + i]);
                        store16_coherent(dst + (e * 4 + u) * 1024, x);
                    }
            } else {
#pragma unroll
                for (int e = 0; e < OWN; ++e)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        u32x4 x;
#pragma unroll
                        for (int i = 0; i < 4; ++i) x[i] = pack_bf16x2(out[e][8 * u + 2 * i], out[e][8 * u + 2 * i + 1]);
                        store16_coherent(dst + (e * 2 + u) * 1024, x);
                    }
            }
            // (every owner of a row stores the same pair)
#pragma unroll
            for (int e = 0; e < OWN; ++e)
                if (hf == 0) store8_coherent(p.ws_ml + ((part0 + split) * kQRows + own_qb(wave, e) * 32 + l32) * 2, u32x2{__float_as_uint(Mq[e]), __float_as_uint(Lq[e])});
        }
        wait_vmcnt<0>();
        int is_last = 0;
        if (lane == 0) {
            int32_t* cnt = p.ws_cnt + (static_cast<int64_t>(unit) * 4 + wave) * kCounterStride;
            const int ticket = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = ticket == ranges - 1;
            if (is_last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (!__builtin_amdgcn_readfirstlane(is_last)) return;
        asm volatile("" ::: "memory");
        // device-coherent (sc1) buffer loads, which the compiler counts; not before the ticket was seen
        constexpr int kCoherent = 16;
        const auto acc_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.ws_acc + part0 * part_bytes + wave * vectors * 1024, 0, 0x7FFFFFFF, 0x00027000);
        const auto ml_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.ws_ml + part0 * kQRows * 2, 0, 0x7FFFFFFF, 0x00027000);
        const int last = ranges - 1;
        float Mall[OWN], Lall[OWN];
#pragma unroll
        for (int e = 0; e < OWN; ++e) {
            Mall[e] = -INFINITY;
            Lall[e] = 0.f;
            out[e] = zero;
        }
        auto merge = [&](auto kind) __attribute__((always_inline)) {
            constexpr bool WIDE = decltype(kind)::value;
            constexpr int PV = WIDE ? OWN * 4 : OWN * 2;
            constexpr int BATCH = 4;
            for (int first = 0; first <= last; first += BATCH) {       // four ranges' loads at once (past the last: it again, weight zero)
                u32x2 ml[BATCH][OWN];
                u32x4 part[BATCH][PV];
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
#pragma unroll
                    for (int e = 0; e < OWN; ++e)
                        ml[u][e] = __builtin_amdgcn_raw_buffer_load_b64(ml_rsrc, (own_qb(wave, e) * 32 + l32) * 8, min(first + u, last) * (kQRows * 8), kCoherent);
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
#pragma unroll
                    for (int v = 0; v < PV; ++v)
                        part[u][v] = __builtin_amdgcn_raw_buffer_load_b128(acc_rsrc, lane * 16, min(first + u, last) * part_bytes + v * 1024, kCoherent);
#pragma unroll
                for (int e = 0; e < OWN; ++e) {
                    float M = Mall[e];
#pragma unroll
                    for (int u = 0; u < BATCH; ++u) M = fmaxf(M, __uint_as_float(ml[u][e][0]));
                    const float m_safe = M == -INFINITY ? 0.f : M;
                    if (first) {
                        const float alpha = fast_exp2((Mall[e] - m_safe) * c2);
                        Lall[e] *= alpha;
                        out[e] *= alpha;
                    }
                    Mall[e] = M;
#pragma unroll
                    for (int u = 0; u < BATCH; ++u) {
                        const float w = first + u <= last ? fast_exp2((__uint_as_float(ml[u][e][0]) - m_safe) * c2) : 0.f;
                        Lall[e] += __uint_as_float(ml[u][e][1]) * w;
                        if constexpr (WIDE) {
#pragma unroll
                            for (int v = 0; v < 4; ++v)
#pragma unroll
                                for (int i = 0; i < 4; ++i) out[e][4 * v + i] = fmaf(__uint_as_float(part[u][4 * e + v][i]), w, out[e][4 * v + i]);
                        } else {
#pragma unroll
                            for (int v = 0; v < 2; ++v)
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const uint32_t x = part[u][2 * e + v][i];
                                    out[e][8 * v + 2 * i] = fmaf(__uint_as_float(x << 16), w, out[e][8 * v + 2 * i]);
                                    out[e][8 * v + 2 * i + 1] = fmaf(__uint_as_float(x & 0xFFFF0000u), w, out[e][8 * v + 2 * i + 1]);
                                }
                        }
                    }
                }
            }
        };
        if (p.wide) merge(std::true_type{});
        else merge(std::false_type{});
        store_out(Mall, Lall);
    }
}

template <int D, bool PAGED>
__global__ __launch_bounds__(kWaveWgs * 64) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_streams_kernel(StreamsParams p) {
    attend<D, PAGED, false>(p);
}

template <int D, bool PAGED>
__global__ __launch_bounds__(kWaveWgs * 64) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_shares_kernel(StreamsParams p) {
    attend<D, PAGED, true>(p);
}

template <int D, bool PAGED>
void launch_as(const StreamsParams& p, dim3 grid, hipStream_t stream) {
    if (p.columns > p.B) hipLaunchKernelGGL((attn_shares_kernel<D, PAGED>), grid, dim3(kWaveWgs * 64), 0, stream, p);
    else hipLaunchKernelGGL((attn_streams_kernel<D, PAGED>), grid, dim3(kWaveWgs * 64), 0, stream, p);
}

template <int D>
void launch_d(const StreamsParams& p, dim3 grid, hipStream_t stream) {
    if (p.g.block_table) launch_as<D, true>(p, grid, stream);
    else launch_as<D, false>(p, grid, stream);
}

}  // namespace

int32_t launch_attn_streams(const AttnArgs& a) {
    unsigned workgroups;
    StreamsParams p;
    static_cast<WaveParams&>(p) = wave_params(a, kQRows, 1, workgroups);
    p.B = a.d.B;
    p.columns = a.plan.columns;
    p.each = std::min(p.columns / p.B, kMostRanges);
    p.by_length = a.plan.by_length;
    p.wide = a.plan.splits == 1;
    p.help = p.B <= kMostByLength;
    p.magic_columns = divisor(p.columns);
    p.magic_each = divisor(p.each);
    p.inv_columns = 1.f / p.columns;
    p.least_gain = a.d.D == 128 ? 1.3f : 2.5f;             // meeting of partial results, 1.5 us, in rounds
    workgroups = static_cast<unsigned>(p.columns) * a.d.H_kv * p.row_blocks;
    p.ws_acc = static_cast<unsigned char*>(a.workspace) + kCounterBytes + static_cast<size_t>(workgroups) * kQRows * 8;
    if (a.d.D == 128) launch_d<128>(p, dim3(workgroups), a.stream);
    else launch_d<64>(p, dim3(workgroups), a.stream);
    return check_launch();
}

}  // namespace specvlm
