// Tree-masked verification attention for bf16 caches, query rows divided among workgroups.
//
// What bounds a call with few (request, head) pairs or short prefixes is not the K/V stream but a chain of
// latencies: launch, first memory round trip, a few tiles, the meeting of partial results.  attn_mfma.hip
// gives a workgroup all 64 query rows and fills the chip with key ranges, up to 64 of them per head, whose
// partial results then meet.  Here a workgroup takes 16 or 32 rows (of one KV head: with grouped query heads
// the rows of the whole group are dealt out together, so small trees do not leave a matrix tile half empty)
// and the chip is filled with row blocks first: a quarter or half of the arithmetic per workgroup, fewer or
// no partial results, each a quarter or half the size.  K and V are then fetched by 2 - 4 workgroups of a
// head, from L2 for all but the first, which is what ends its usefulness for long prefixes (attn_plan()).
//
//   grid      (request, KV head, row block, key range), 4 wavefronts each; a wavefront has a key stream of
//             its own (32-key tiles stream, stream + 4 splits, ...), so the loop has no barrier at all
//   fetch     direct-to-LDS loads into two K and two V areas per wavefront; an area is requested again as soon
//             as its operands are in registers, K three tiles and V two tiles ahead of the products
//   product   S^T = K Q^T of tile j + 1 before the softmax of tile j is needed, so that the matrix
//             pipe has work while the vector ALU does exponentials; a row's weights are summed in fp32 before
//             they are packed (one more matrix product, with ones, in place of the eight additions is 0.1 - 0.6 %
//             faster per step, but sums bf16 weights: log-sum-exp off by up to 1e-3 in place of 1e-6)
//   tree      ancestor masks by pointer doubling across lanes, built by every wavefront while the first tile is on its
//             way: the tile that needs them is the last of its stream, where nothing hides them; a masked score takes
//             two instructions of the tile's visibility word (masks on demand, eight instructions a score, and the
//             addresses, accumulators and query operands behind the wait for the first tile: 828 keys 9.46 us, so 9.03)
//   merge     as in attn_mfma.hip: streams through LDS, key ranges through the workspace and tickets; the last
//             arrival reads up to four partials at once, more in batches of eight (a caller's 9 - 64 splits too)
//
// Measured per call (HIP-graph replay), key ranges only -> here: 1 x 32 heads, 828 keys 11.1 -> 9.0 us, 3324 keys 16.3 -> 15.5;
// 4 x 8 heads, 144 keys 8.8 -> 5.8; 2 x 8 heads, 1197 keys, paged 16.6 -> 10.2; 1 x 8 heads of 64, 4200 keys 21.4 -> 8.5;
// 4 x 32 query / 16 KV heads of 64, 13 nodes 9.0 -> 6.0 (the last four before the line above).
#include "attn_rows.hpp"

namespace specvlm {

namespace {

// The greatest of eight scores, NaN where one is: v_maximum3 takes its operands as they are (fmaxf would quiet each first).
__device__ __forceinline__ float max8(f32x4 a, f32x4 b) {
    auto max3 = [](float x, float y, float z) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z); };
    return max3(max3(a[0], a[1], a[2]), max3(a[3], b[0], b[1]), __builtin_elementwise_maximum(b[2], b[3]));
}

// op over the four lanes g = 0 .. 3 of a row, in every one of them: (0 1) (2 3), or (1 0) (3 2), then across.
template <typename Op>
__device__ __forceinline__ float across_row(float x, Op op) {
    const uint32_t a = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);     // lanes 16 apart
    const uint32_t y = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
    const auto q = __builtin_amdgcn_permlane32_swap(y, y, false, false);     // lanes 32 apart
    return op(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

template <int D, int QB, bool PAGED>
__global__ __launch_bounds__(kWaveWgs * 64) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_wave_kernel(WaveParams p) {
    constexpr int NC = D / 32;                 // QK^T contraction steps of 32
    constexpr int NT = D / 16;                 // output row blocks (head dim)
    constexpr int ROWG = D / 8;                // 16-byte granules per K/V row
    constexpr int RPI = 64 / ROWG;             // rows per load instruction (4 or 8)
    constexpr int NH = 16 / RPI;               // load instructions per half tile (4 or 2)
    constexpr int KLD = 2 * NH;                // ... per K (or V) tile
    constexpr int kTileBytes = kKeys * D * 2;
    constexpr int kSlotBytes = 2 * kTileBytes;           // K tile then V tile
    constexpr int kRingBytes = 2 * kSlotBytes;           // two slots per wavefront
    constexpr int NQ = (QB * 16 / RPI + 3) / 4;          // query-row load instructions per wavefront
    constexpr int NS = 4 / QB < NT / 2 ? 4 / QB : NT / 2;    // head-dim slices of a query block at the merge
    constexpr int OT = NT / NS;                          // output blocks of an owner
    static_assert(QB * NS <= kWaveWgs, "one owner per wavefront");
    static_assert(kWaveWgs * kRingBytes >= QB * NS * 3 * OT * 1024, "merge scratch must fit in the rings");

    __shared__ __attribute__((aligned(1024))) unsigned char s_ring[kWaveWgs * kRingBytes];
    __shared__ __attribute__((aligned(1024))) unsigned char s_q[QB * 16 * D * 2];
    __shared__ float s_m[kWaveWgs][QB * 16];
    __shared__ float s_l[kWaveWgs][QB * 16];
    __shared__ int s_par[kWaveWgs][64];

    // What the first requests need of the arguments, in one trip to memory (left to itself the compiler loads them where they
    // are used: two more trips, one of them the lengths', before the first request; 2 x 16 / 4 heads, 300 keys 6.50 -> 6.37 us)
    asm volatile("" : : "s"(p.g.stride_b), "s"(p.g.stride_h), "s"(p.g.stride_t), "s"(p.g.capacity), "s"(p.N_max), "s"(p.H_kv), "s"(p.group), "s"(p.row_blocks),
                 "s"(p.num_splits), "s"(p.magic_splits), "s"(p.magic_rb), "s"(p.magic_hkv), "s"(p.magic_nmax), "s"(p.magic_nstream), "s"(p.q), "s"(p.k), "s"(p.v),
                 "s"(p.q_sb), "s"(p.q_sn), "s"(p.q_sh), "s"(p.prefix_len), "s"(p.num_nodes), "s"(p.parent));
    // work item: (request, KV head, row block, split); every XCD gets a contiguous range of items, the first ones an item more where their
    // number is no multiple of 8 (dealt out to the XCDs in turn every L2 fetches a head's K and V: 3 x 20 / 4 heads, 44 nodes, 1100 keys
    // 13.7 us, so 9.7; 3 x 7, 3000 keys 16.7, so 12.7)
    const uint32_t xcd = blockIdx.x & 7;
    const uint32_t work = xcd * (gridDim.x >> 3) + min(xcd, gridDim.x & 7) + (blockIdx.x >> 3);
    const uint32_t unit = divide(work, p.magic_splits);
    const int split = work - unit * p.num_splits;
    const uint32_t bk = divide(unit, p.magic_rb);
    const int rb = unit - bk * p.row_blocks;
    const int b = divide(bk, p.magic_hkv);
    const int hk = bk - b * p.H_kv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;

    typedef const __attribute__((address_space(4))) int32_t* const_i32;
    const int nstream = kWaveWgs * p.num_splits;
    const int stream = wave * p.num_splits + split;

    unsigned char* ring = s_ring + wave * kRingBytes;
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const uint32_t ring_lds = (uint32_t)(uintptr_t)(lds_byte*)ring;

    // the parent array, first in the queue and waited for on its own (every wavefront its own copy)
    typedef __attribute__((address_space(3))) int lds_int;
    dma4(p.parent + b * p.N_max + min(lane, p.N_max - 1), (uint32_t)(uintptr_t)(lds_int*)s_par[wave]);

    // ---- tile fetch -------------------------------------------------------------------------
    const int lrow = lane / ROWG, lpos = lane % ROWG;
    const uint32_t row_bytes = static_cast<uint32_t>(p.g.stride_t) * 2u;
    const uint32_t lrow_off = __umul24(lrow, row_bytes);   // (row_bytes < 2^24: checked on the host)
    auto vswz = [](int r) { return D == 128 ? (r & 7) : ((r >> 1) & 3); };
    uint32_t voff_k[NH], voff_v[NH];
    // row r = i RPI + lrow of a half tile; K lands with granule g of row r at position g ^ (r % ROWG), V with the
    // 32-byte chunk c of row r at chunk c ^ vswz(r)
    auto offsets_k = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NH; ++i)
            voff_k[i] = lrow_off + ((lpos ^ ((i * RPI + lrow) & (ROWG - 1))) << 4) + i * (RPI * row_bytes - 1024);   // (row_bytes >= 2 D)
    };
    auto offsets_v = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NH; ++i)
            voff_v[i] = lrow_off + ((lpos ^ (vswz(i * RPI + lrow) << 1)) << 4) + i * (RPI * row_bytes - 1024);
    };
    const int64_t head_off = hk * p.g.stride_h + (PAGED ? 0 : b * p.g.stride_b);   // elements
    // Tile j of this stream, K or V, into slot j % 2: two halves of 16 rows.  Rows past the request's last
    // key are fetched as they are (they are memory that may be read, and their weight is zero).
    const int64_t tile_step = static_cast<int64_t>(nstream) * kKeys * p.g.stride_t;         // elements from one tile of the stream to its next
    const int64_t first_off = head_off + static_cast<int64_t>(stream) * kKeys * p.g.stride_t;
    const uint16_t* k_next = p.k + (PAGED ? head_off : first_off);       // contiguous: the next tile to request
    const uint16_t* v_next = p.v + (PAGED ? head_off : first_off);
    auto issue = [&](const uint16_t*& src, const uint32_t (&voff)[NH], int area, int j, const int (&phys)[2]) __attribute__((always_inline)) {
        const uint32_t dst = ring_lds + (j & 1) * kSlotBytes + area;
        if constexpr (PAGED) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
                dma_half<D>(src + min(max(phys[x], 0), p.g.num_blocks - 1) * p.g.stride_b, voff, dst + x * (kTileBytes / 2));
        } else {
            const int lo = (stream + j * nstream) * kKeys;
            if (__builtin_expect(lo + kKeys <= p.g.capacity, 1)) {
                dma_half<D>(src, voff, dst);
                dma_half<D>(src + 16 * p.g.stride_t, voff, dst + kTileBytes / 2);
            } else {
                // the cache ends inside this tile (or before it): rows past its end re-read its last row
#pragma unroll 1
                for (int x = 0; x < 2; ++x) {
                    const int r0 = min(lo + 16 * x, p.g.capacity - 1);
                    uint32_t vo[NH];
#pragma unroll
                    for (int i = 0; i < NH; ++i)
                        vo[i] = voff[i] + (min(i * RPI + lrow, p.g.capacity - 1 - r0) - (i * RPI + lrow)) * row_bytes + 4096;
                    dma_half<D>(src + static_cast<int64_t>(r0 - lo) * p.g.stride_t - 2048, vo, dst + x * (kTileBytes / 2));
                }
            }
            src += tile_step;
        }
    };
    auto issue_k = [&](int j, const int (&phys)[2]) __attribute__((always_inline)) { issue(k_next, voff_k, 0, j, phys); };
    auto issue_v = [&](int j, const int (&phys)[2]) __attribute__((always_inline)) { issue(v_next, voff_v, kTileBytes, j, phys); };
    int phys[2] = {0, 0};                                   // block ids of the tile requested next
    // With a contiguous cache the first tile's address needs no length: requested before the lengths arrive.
    constexpr bool early = !PAGED;
    offsets_k();
    if (early) issue_k(0, phys);
    // the request's lengths through the scalar cache, not before that request
    const int32_t *lengths = p.prefix_len, *counts = p.num_nodes ? p.num_nodes : p.prefix_len;
    asm volatile("" : "+s"(lengths), "+s"(counts));
    const int P_raw = ((const_i32)lengths)[b];
    const int n_given = ((const_i32)counts)[b], n_raw = p.num_nodes ? n_given : p.N_max;

    // query rows of this block: row r of the block is row R = 16 QB rb + r of the group's (head, node) rows
    const int rows_total = p.group * p.N_max;
    typedef __attribute__((address_space(3))) unsigned char lds_u8;
    const uint32_t q_lds = (uint32_t)(uintptr_t)(lds_u8*)s_q;
    const int row0 = rb * (QB * 16);
    const int q_row = static_cast<int>(p.q_sn) * 2, q_head = static_cast<int>(p.q_sh) * 2;     // bytes (checked on the host)
    const uint16_t* q_base = p.q + b * p.q_sb + static_cast<int64_t>(hk * p.group) * p.q_sh;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int inst = (wave * NQ + i) % (QB * 16 / RPI);
        const int r = inst * RPI + lrow;
        const int R = min(row0 + r, rows_total - 1);
        const int hh = divide(R, p.magic_nmax);
        const int node = R - hh * p.N_max;
        const uint32_t voff = static_cast<uint32_t>(node * q_row + hh * q_head) + ((lpos ^ (r & (ROWG - 1))) << 4);
        dma16s(q_base, voff, q_lds + inst * 1024);
    }
    offsets_v();
    if (early) issue_v(0, phys);

    int err = 0;
    int n = n_raw;
    const int P = P_raw;
    if (n < 1 || n > p.N_max) err |= SPECVLM_ERR_BAD_NUM_NODES;
    n = min(max(n, 1), p.N_max);
    if (!length_fits(P, n, p.g.capacity)) err |= SPECVLM_ERR_BAD_LENGTH;
    const int S = P + n;
    const int ntile = (S + kKeys - 1) / kKeys;
    const int my_tiles = (!err && stream < ntile) ? static_cast<int>(divide(ntile - stream + nstream - 1, p.magic_nstream)) : 0;
    int bad_block = 0;                                     // uniform
    auto fetch_blocks = [&](int j, int (&phys)[2]) __attribute__((always_inline)) {
        if constexpr (PAGED) {
            const int blk0 = (stream + j * nstream) * (kKeys >> 4), last_blk = (S - 1) >> 4;
            const const_i32 row = (const_i32)p.g.block_table + static_cast<int64_t>(b) * p.g.max_blocks;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                phys[x] = row[min(blk0 + x, last_blk)];
                bad_block |= static_cast<uint32_t>(phys[x]) >= static_cast<uint32_t>(p.g.num_blocks) ? 1 : 0;
            }
        }
    };
    if (!early && my_tiles > 0) { fetch_blocks(0, phys); issue_k(0, phys); issue_v(0, phys); }
    if (my_tiles > 1) { fetch_blocks(1, phys); issue_k(1, phys); issue_v(1, phys); }
    int phys_k[2] = {0, 0}, phys_v[2] = {0, 0};            // block ids of the next K and V tile to request
    if (my_tiles > 2) { fetch_blocks(2, phys_k); phys_v[0] = phys_k[0]; phys_v[1] = phys_k[1]; }

    const float c2 = p.c2, tau = p.tau;
    // ---- K fragments of a tile (A operand): lane (key 16x + l16, g) holds d = 32c + 8g .. +7 ------
    uint32_t kaddr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) kaddr[c] = l16 * (ROWG * 16) + (((4 * c + g) ^ (l16 & (ROWG - 1))) << 4);
    bf16x8 ka[2][NC];
    auto read_k = [&](int slot_off) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                ka[x][c] = *reinterpret_cast<const bf16x8*>(ring + slot_off + kaddr[c] + x * 16 * ROWG * 16);
    };
    // Where this wavefront's share of the result goes (worked out while the first tile is on its way): wavefront w owns query
    // block w / NS, head-dim slice w % NS
    const int oqb = wave / NS, osl = wave % NS, qrow = oqb * 16 + l16;
    int64_t o_off, lse_off;
    unsigned long long real_rows;
    {
        const int R = row0 + qrow;
        const int hh = divide(R, p.magic_nmax);
        const int node = R - hh * p.N_max;
        const int h = hk * p.group + hh;
        real_rows = __ballot(R < rows_total && node < n);
        o_off = b * p.o_sb + node * p.o_sn + static_cast<int64_t>(h) * p.o_sh + 4 * (g & ~1) + osl * OT * 16;
        lse_off = (static_cast<int64_t>(b) * p.H_q + h) * p.N_max + node;
    }
    // Softmax state of query row 16 qb + l16 (the four lanes of a row agree): reference maximum, the same times
    // c2 (0 while no key was seen), and this lane's part of the sum of the row's weights.
    // acc[qb][t]: O^T rows 16t + 4g .. + 3.
    float m_run[QB], mrc[QB], l_run[QB];
    f32x4 acc[QB][NT];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_run[qb] = -INFINITY;
        mrc[qb] = 0.f;
        l_run[qb] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[qb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // V operands: lane supplies key 4g + l16/4 (and 16 keys further), dims 16t + 4 (l16 % 4)
    const int k0 = 4 * g + (l16 >> 2);
    const uint32_t vaddr = kTileBytes + k0 * (ROWG * 16) + (l16 & 3) * 8 + (vswz(k0) << 5);
    int row_node[QB];                                      // the node of this lane's query rows
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int R = min(row0 + qb * 16 + l16, rows_total - 1);
        row_node[qb] = R - divide(R, p.magic_nmax) * p.N_max;
    }
    // (all of this before the waits: the compiler would put it behind, where the tree and the first products wait for it)
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(kaddr[c]));
    asm volatile("" : : "v"(vaddr), "v"(row_node[0]), "v"(row_node[QB - 1]), "v"(o_off), "v"(lse_off), "s"(real_rows));
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int t = 0; t < NT; ++t) asm volatile("" : "+v"(acc[qb][t]));
    // ---- the tree: every wavefront checks it and builds the ancestor masks in registers ----------
    // requested after the parent array: K0, the query rows, V0 (an early request) or the query rows, K0, V0,
    // and the second tile
    if (my_tiles > 1) wait_vmcnt<4 * KLD + NQ>();
    else if (my_tiles == 1 || early) wait_vmcnt<2 * KLD + NQ>();
    else wait_vmcnt<NQ>();
    const int par = s_par[wave][lane];
    const bool bad_par = lane < n && (lane == 0 ? par != -1 : (par < 0 || par >= lane));
    if (__any(bad_par)) err |= SPECVLM_ERR_BAD_PARENT;
    if (err) {                                             // the same in every wavefront of the request
        if (tid == 0 && p.err_flag) atomicOr(p.err_flag, err);
        wait_vmcnt<0>();
        return;
    }
    // Ancestor-or-self masks of this lane's query rows, while the first tile is on its way (the tile that needs them is the last of its
    // stream): pointer doubling over the lanes (lane i holds node i), at most six rounds.
    uint32_t anc_lo[QB], anc_hi[QB];
    {
        uint32_t mlo = lane < 32 ? 1u << (lane & 31) : 0u, mhi = lane < 32 ? 0u : 1u << (lane & 31);
        int up = lane < n ? par : -1;
#pragma unroll 1
        while (__any(up >= 0)) {
            const int src = max(up, 0) * 4;
            const uint32_t alo = __builtin_amdgcn_ds_bpermute(src, mlo), ahi = __builtin_amdgcn_ds_bpermute(src, mhi);
            const int up2 = __builtin_amdgcn_ds_bpermute(src, up);
            if (up >= 0) { mlo |= alo; mhi |= ahi; up = up2; }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            anc_lo[qb] = __builtin_amdgcn_ds_bpermute(row_node[qb] * 4, mlo);
            anc_hi[qb] = __builtin_amdgcn_ds_bpermute(row_node[qb] * 4, mhi);
        }
    }

    // K0 and the query rows of this wavefront have landed; the barrier extends the latter to the workgroup
    if (my_tiles > 1) wait_vmcnt<3 * KLD>();
    else if (my_tiles == 1) wait_vmcnt<KLD>();
    else wait_vmcnt<0>();
    __syncthreads();
    bf16x8 qf[QB][NC];
    bf16x8 va[NT];
    auto read_v = [&](int t, int slot_off) __attribute__((always_inline)) {
        const uint32_t a = (vaddr ^ (t << 5)) + slot_off;
        const s16x4 lo = lds_read_tr16(ring + a);
        const s16x4 hi = lds_read_tr16(ring + a + 16 * ROWG * 16);
        const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        va[t] = __builtin_bit_cast(bf16x8, both);
    };
    // S^T = K Q^T: s[qb][x][i] = score of key 16x + 4g + i of the tile against query row 16qb + l16
    f32x4 s[QB][2];
    auto scores = [&](int qb) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int x = 0; x < 2; ++x)
                s[qb][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[x][c], qf[qb][c], c ? s[qb][x] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    };
    bf16x8 pf[QB];
    auto weights = [&](int qb) __attribute__((always_inline)) {     // exp2(S^T) packed to bf16 is the B operand of PV
        float pr[8];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) pr[jj] = fast_exp2(fmaf(s[qb][jj >> 2][jj & 3], c2, -mrc[qb]));
        l_run[qb] += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
        u32x4 w;
#pragma unroll
        for (int x = 0; x < 4; ++x) w[x] = pack_bf16x2(pr[2 * x], pr[2 * x + 1]);
        pf[qb] = __builtin_bit_cast(bf16x8, w);
    };
    float lmax[QB];
    auto maxima = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) lmax[qb] = max8(s[qb][0], s[qb][1]);
    };

    if (my_tiles > 0) {
        read_k(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the K area of slot 0 is free
        if (my_tiles > 2) { issue_k(2, phys_k); if (my_tiles > 3) fetch_blocks(3, phys_k); }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) qf[qb][c] = *reinterpret_cast<const bf16x8*>(s_q + qb * 16 * ROWG * 16 + kaddr[c]);
        // Query fragments live in accumulation registers (a matrix instruction takes its operands from there as well).
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                asm volatile("" : "+a"(qf[qb][c]));
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    s[qb][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[x][c], qf[qb][c], c ? s[qb][x] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            }
        // V0 and K1 (the requests after them: V1, K2)
        if (my_tiles > 2) wait_vmcnt<2 * KLD>();
        else if (my_tiles == 2) wait_vmcnt<KLD>();
        else wait_vmcnt<0>();
        if (my_tiles > 1) read_k(kSlotBytes);
#pragma unroll
        for (int t = 0; t < NT; ++t) read_v(t, 0);
        maxima();
        // The first reference, where every key is visible: as in the loop, with nothing accumulated that it would scale
        if (stream * kKeys + kKeys <= P) {
            bool any = false;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) any = any | (lmax[qb] > -INFINITY);
            if (__any(any)) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    m_run[qb] = fmaxf(-INFINITY, across_row(lmax[qb], fmaxf));
                    mrc[qb] = (m_run[qb] == -INFINITY ? 0.f : m_run[qb]) * c2;
                }
            }
        }
    }
    for (int j = 0; j < my_tiles; ++j) {
        const int left = my_tiles - 1 - j;                 // tiles after this one
        const int slot0 = (stream + j * nstream) * kKeys;
        // s holds tile j's scores, va its V operands, ka the next tile's K operands; both their areas are free
        if (slot0 + kKeys > P) {                           // reaches past the prefix: tree region or tail
            // bit k of `visible`: key slot0 + k.  Its place among this lane's scores is a constant once the lane's group is shifted out, so a
            // score takes two instructions (a sign-extended bit and a bitwise select)
            const int before = P - slot0;                  // keys of the tile in the prefix, < 32
            const uint32_t exist = S - slot0 < 32 ? (1u << (S - slot0)) - 1u : ~0u;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const unsigned long long anc = (static_cast<unsigned long long>(anc_hi[qb]) << 32) | anc_lo[qb];
                uint32_t visible = before > 0 ? (anc_lo[qb] << before) | ((1u << before) - 1u) : static_cast<uint32_t>(anc >> -before);
                visible = (visible & exist) >> (4 * g);
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t seen = static_cast<uint32_t>(static_cast<int32_t>(visible << (31 - (16 * x + i))) >> 31);
                        s[qb][x][i] = __uint_as_float((seen & __float_as_uint(s[qb][x][i])) | (~seen & 0xFF800000u));
                    }
            }
            maxima();
            if (slot0 + kKeys > S) {                       // keys that do not exist: zero weight must meet a finite value
                uint32_t keep[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {              // dword e of an operand: keys kk, kk + 1
                    const int kk = slot0 + 16 * (e >> 1) + 4 * g + 2 * (e & 1);
                    keep[e] = (kk < S ? 0xFFFFu : 0u) | (kk + 1 < S ? 0xFFFF0000u : 0u);
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    u32x4 w = __builtin_bit_cast(u32x4, va[t]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] &= keep[e];
                    va[t] = __builtin_bit_cast(bf16x8, w);
                }
            }
        }
        // Online softmax with a lazily updated reference: a weight may exceed 1; the reference only moves when
        // some score would exceed it by more than 2^kTau (or on the first visible key).
        bool trig = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) trig = trig | (lmax[qb] > m_run[qb] + tau);
        if (__builtin_expect(__any(trig), 0)) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const float m_new = fmaxf(m_run[qb], across_row(lmax[qb], fmaxf));
                const float m_safe = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = m_run[qb] == -INFINITY ? 1.f : fast_exp2((m_run[qb] - m_safe) * c2);
                m_run[qb] = m_new;
                mrc[qb] = m_safe * c2;
                l_run[qb] *= alpha;
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[qb][t] *= alpha;
            }
        }
        if (left == 0) break;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // ka and va are in registers
        if (left >= 2) {
            issue_v(j + 2, phys_v);
            if (left >= 3) {
                phys_v[0] = phys_k[0]; phys_v[1] = phys_k[1];
                issue_k(j + 3, phys_k);
                if (left >= 4) fetch_blocks(j + 4, phys_k);
            }
        }
        // weights of tile j; the next tile's scores replace them block by block
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            weights(qb);
            scores(qb);
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) asm volatile("" : "+v"(pf[qb]));      // not to be moved past the waits below
        // V of tile j + 1 and K of tile j + 2 have landed (the requests after them: V of j + 2, K of j + 3)
        if (left >= 3) wait_vmcnt<2 * KLD>();
        else if (left == 2) wait_vmcnt<KLD>();
        else wait_vmcnt<0>();
        const int next_off = ((j + 1) & 1) * kSlotBytes;
        if (left >= 2) read_k(next_off ^ kSlotBytes);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) acc[qb][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t], pf[qb], acc[qb][t], 0, 0, 0);
            read_v(t, next_off);
        }
        maxima();
    }
    if (my_tiles > 0) {                                    // the last tile's weights and products
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            weights(qb);
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[qb][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t], pf[qb], acc[qb][t], 0, 0, 0);
        }
    }

    if (bad_block && lane == 0 && p.err_flag) atomicOr(p.err_flag, SPECVLM_ERR_BAD_BLOCK);
    // ---- merge the four streams --------------------------------------------------------------------
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        l_run[qb] = across_row(l_run[qb], [](float x, float y) { return x + y; });
        if (g == 0) {
            s_m[wave][qb * 16 + l16] = m_run[qb];
            s_l[wave][qb * 16 + l16] = l_run[qb];
        }
    }
    __syncthreads();                                       // every stream is done with its ring
    f32x4 out[OT];
#pragma unroll
    for (int o = 0; o < QB * NS; ++o) {
        const int qb = o / NS, sl = o % NS;
        if (o == wave) {                                   // uniform
#pragma unroll
            for (int t = 0; t < OT; ++t) out[t] = acc[qb][sl * OT + t];
        } else {
            const int idx = wave < o ? wave : wave - 1;
            f32x4* dst = reinterpret_cast<f32x4*>(s_ring) + (o * 3 + idx) * OT * 64;
#pragma unroll
            for (int t = 0; t < OT; ++t) dst[t * 64 + lane] = acc[qb][sl * OT + t];
        }
    }
    __syncthreads();
    if (wave >= QB * NS) return;
    float Mq = s_m[0][qrow];
#pragma unroll
    for (int x = 1; x < kWaveWgs; ++x) Mq = fmaxf(Mq, s_m[x][qrow]);
    float Lq = 0.f;
    {
        const float m_safe = Mq == -INFINITY ? 0.f : Mq;
        float w[kWaveWgs];
#pragma unroll
        for (int x = 0; x < kWaveWgs; ++x) {               // (in this order in every owner of the query block)
            w[x] = fast_exp2((s_m[x][qrow] - m_safe) * c2);
            Lq += s_l[x][qrow] * w[x];
        }
        const float w0 = fast_exp2((s_m[wave][qrow] - m_safe) * c2);
#pragma unroll
        for (int t = 0; t < OT; ++t) out[t] *= w0;
        const f32x4* src = reinterpret_cast<const f32x4*>(s_ring) + wave * 3 * OT * 64;
#pragma unroll
        for (int idx = 0; idx < 3; ++idx) {
            const float wx = wave <= idx ? w[idx + 1] : w[idx];
#pragma unroll
            for (int t = 0; t < OT; ++t) out[t] += src[(idx * OT + t) * 64 + lane] * wx;
        }
    }
    if (!real_rows) return;                                // uniform over the splits of the unit as well
    const bool real = (real_rows >> lane) & 1;
    auto store_out = [&](float M, float L) {
        const float inv = 1.f / L;
        const bool odd = g & 1;
        uint16_t* orow = p.o + o_off;
#pragma unroll
        for (int u = 0; u < OT / 2; ++u) {
            const uint32_t e0 = pack_bf16x2(out[2 * u][0] * inv, out[2 * u][1] * inv);
            const uint32_t e1 = pack_bf16x2(out[2 * u][2] * inv, out[2 * u][3] * inv);
            const uint32_t o0 = pack_bf16x2(out[2 * u + 1][0] * inv, out[2 * u + 1][1] * inv);
            const uint32_t o1 = pack_bf16x2(out[2 * u + 1][2] * inv, out[2 * u + 1][3] * inv);
            // an even group's lane holds dims 0-3 of two blocks of 16, its odd neighbour 4-7: even keeps the first block, odd the second
            const auto r0 = __builtin_amdgcn_permlane16_swap(e0, o0, false, false);
            const auto r1 = __builtin_amdgcn_permlane16_swap(e1, o1, false, false);
            const u32x4 w = u32x4{r0[0], r1[0], r0[1], r1[1]};
            if (real) *reinterpret_cast<u32x4*>(orow + 16 * (2 * u + (odd ? 1 : 0))) = w;
        }
        if (real && p.lse && g == 0 && osl == 0)
            p.lse[lse_off] = M * p.scale + __log2f(L) * kLn2;
    };
    if (p.num_splits == 1) {
        store_out(Mq, Lq);
        return;
    }
    // ---- split partials ----------------------------------------------------------------------------
    constexpr int PV = OT / 2;                             // 16-byte vectors per lane per partial
    const int64_t part0 = static_cast<int64_t>(unit) * p.num_splits;
    constexpr int kPartBytes = QB * NS * PV * 1024;        // one split's partial
    {
        u32x4* dst = reinterpret_cast<u32x4*>(p.ws_acc + (part0 + split) * kPartBytes + wave * PV * 1024);
#pragma unroll
        for (int u = 0; u < PV; ++u) {
            u32x4 x;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = pack_bf16x2(out[2 * u][i], out[2 * u + 1][i]);
            store16_coherent(dst + u * 64 + lane, x);
        }
        if (g == 0) {
            float* ml = p.ws_ml + ((part0 + split) * (QB * 16) + qrow) * 2;     // (every slice's owner stores the same pair)
            store8_coherent(ml, u32x2{__float_as_uint(Mq), __float_as_uint(Lq)});
        }
    }
    wait_vmcnt<0>();
    int is_last = 0;
    if (lane == 0) {
        int32_t* cnt = p.ws_cnt + (static_cast<int64_t>(unit) * 4 + wave) * kCounterStride;
        const int ticket = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_last = ticket == p.num_splits - 1;
        if (is_last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!__builtin_amdgcn_readfirstlane(is_last)) return;
    asm volatile("" ::: "memory");                         // no partial result is read before the ticket was seen
    if (p.num_splits <= 4) {                               // uniform; what the library chooses by itself, mostly
        // (four partials in place of eight: half the instructions of the chain's last link: 1 x 32 heads, 828 keys 9.85 -> 9.25 us)
        constexpr int kFew = 4, kCoherent = 16;            // sc1; buffer loads, which the compiler counts
        const auto acc_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.ws_acc + part0 * kPartBytes + wave * PV * 1024, 0, 0x7FFFFFFF, 0x00027000);
        const auto ml_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.ws_ml + part0 * (QB * 16) * 2, 0, 0x7FFFFFFF, 0x00027000);
        const int last = p.num_splits - 1;
        u32x4 part[kFew][PV];
        u32x2 ml[kFew];
#pragma unroll
        for (int u = 0; u < kFew; ++u)
            ml[u] = __builtin_amdgcn_raw_buffer_load_b64(ml_rsrc, qrow * 8, min(u, last) * (QB * 16 * 8), kCoherent);
#pragma unroll
        for (int u = 0; u < kFew; ++u)
#pragma unroll
            for (int v = 0; v < PV; ++v)
                part[u][v] = __builtin_amdgcn_raw_buffer_load_b128(acc_rsrc, lane * 16, min(u, last) * kPartBytes + v * 1024, kCoherent);
        float Mall = -INFINITY, Lall = 0.f;
#pragma unroll
        for (int u = 0; u < kFew; ++u) Mall = fmaxf(Mall, __uint_as_float(ml[u][0]));
        const float m_safe = Mall == -INFINITY ? 0.f : Mall;
#pragma unroll
        for (int t = 0; t < OT; ++t) out[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < kFew; ++u) {
            const float w = u <= last ? fast_exp2((__uint_as_float(ml[u][0]) - m_safe) * c2) : 0.f;
            Lall += __uint_as_float(ml[u][1]) * w;
#pragma unroll
            for (int v = 0; v < PV; ++v)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t x = part[u][v][i];
                    out[2 * v][i] = fmaf(__uint_as_float(x << 16), w, out[2 * v][i]);
                    out[2 * v + 1][i] = fmaf(__uint_as_float(x & 0xFFFF0000u), w, out[2 * v + 1][i]);
                }
        }
        store_out(Mall, Lall);
        return;
    }
    constexpr int MB = 8;                                  // splits requested together
    const uint32_t voff_part = lane * 16, voff_ml = qrow * 8;
    const unsigned char* acc_base = p.ws_acc + part0 * kPartBytes + wave * PV * 1024;
    const unsigned char* ml_base = reinterpret_cast<const unsigned char*>(p.ws_ml) + part0 * (QB * 16) * 8;
    const int last = p.num_splits - 1;
    float Mall = -INFINITY, Lall = 0.f;
#pragma unroll
    for (int t = 0; t < OT; ++t) out[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 <= last; s0 += MB) {               // uniform
        u32x4 part[MB][PV];
        f32x2 ml[MB];
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const unsigned char* sb = ml_base + static_cast<int64_t>(min(s0 + u, last)) * (QB * 16 * 8);
            asm volatile("global_load_dwordx2 %0, %1, %2 sc1" : "=v"(ml[u]) : "v"(voff_ml), "s"(sb) : "memory");
        }
#pragma unroll
        for (int u = 0; u < MB; ++u)
#pragma unroll
            for (int v = 0; v < PV; ++v) {
                const unsigned char* sb = acc_base + static_cast<int64_t>(min(s0 + u, last)) * kPartBytes + v * 1024;
                asm volatile("global_load_dwordx4 %0, %1, %2 sc1" : "=v"(part[u][v]) : "v"(voff_part), "s"(sb) : "memory");
            }
        wait_vmcnt<MB * PV>();
        float M_new = Mall;
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            asm volatile("" : "+v"(ml[u]));
            M_new = fmaxf(M_new, ml[u][0]);
        }
        const float m_safe = M_new == -INFINITY ? 0.f : M_new;
        if (s0 > 0) {
            const float alpha = fast_exp2((Mall - m_safe) * c2);
            Lall *= alpha;
#pragma unroll
            for (int t = 0; t < OT; ++t) out[t] *= alpha;
        }
        Mall = M_new;
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            wait_vmcnt_unrolled((MB - 1 - u) * PV);
#pragma unroll
            for (int v = 0; v < PV; ++v) asm volatile("" : "+v"(part[u][v]));
            const float w = s0 + u <= last ? fast_exp2((ml[u][0] - m_safe) * c2) : 0.f;
            Lall += ml[u][1] * w;
#pragma unroll
            for (int v = 0; v < PV; ++v)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t x = part[u][v][i];
                    out[2 * v][i] = fmaf(__uint_as_float(x << 16), w, out[2 * v][i]);
                    out[2 * v + 1][i] = fmaf(__uint_as_float(x & 0xFFFF0000u), w, out[2 * v + 1][i]);
                }
        }
    }
    store_out(Mall, Lall);
}

template <int D, int QB>
void launch_rows(const WaveParams& p, dim3 grid, hipStream_t stream) {
    if (p.g.block_table) hipLaunchKernelGGL((attn_wave_kernel<D, QB, true>), grid, dim3(kWaveWgs * 64), 0, stream, p);
    else hipLaunchKernelGGL((attn_wave_kernel<D, QB, false>), grid, dim3(kWaveWgs * 64), 0, stream, p);
}

template <int D>
void launch_d(const WaveParams& p, int block_rows, dim3 grid, hipStream_t stream) {
    if (block_rows == 16) launch_rows<D, 1>(p, grid, stream);
    else launch_rows<D, 2>(p, grid, stream);
}

}  // namespace

int32_t launch_attn_wave(const AttnArgs& a) {
    unsigned workgroups;
    const WaveParams p = wave_params(a, a.plan.block_rows, a.plan.splits, workgroups);
    if (a.d.D == 128) launch_d<128>(p, a.plan.block_rows, dim3(workgroups), a.stream);
    else launch_d<64>(p, a.plan.block_rows, dim3(workgroups), a.stream);
    return check_launch();
}

}  // namespace specvlm
