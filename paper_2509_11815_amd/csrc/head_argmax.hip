// Output head fused with the greedy choice (SpecVLM Fig. 3: one output head, shared by target
// and draft; Sec. 4.1: temperature 0): amax[b,i] = argmax_v sum_e hidden[b,i,e] * W[v,e], lowest
// token on ties, without ever storing the [nodes, vocabulary] logits.
//
// Two kernels.  Up to 64 node rows (one request) the call is bound by streaming the head matrix from
// HBM (262 MB for 32000 x 4096 bf16): head_argmax_kernel.  With more rows it is a matrix product, and
// the tile decides: head_gemm_kernel.  Both compute logits^T[vocab x node] += W . hidden^T with
// v_mfma_f32_16x16x32_bf16 and end alike: every lane orders its logits by (greater value, lower
// token) as one 64-bit key; keys are maximised across lanes, wavefronts, and -- through a workspace
// and a ticket counter -- across the vocabulary tiles by the last workgroup to arrive.
#include <limits.h>

#include "common.hpp"

namespace specvlm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kHeadThreads = 512;
constexpr int kVT = 128;                 // vocabulary rows per workgroup
constexpr int kMB = 64;                  // node rows per block
constexpr int kKC = 128;                 // hidden units per chunk (256-byte rows in LDS)
constexpr int kRing = 3;                 // slots of the W and of the hidden-state ring
constexpr int kWBytes = kVT * kKC * 2;   // 32 KB: a chunk of W
constexpr int kHBytes = kMB * kKC * 2;   // 16 KB: the same chunk of one block of 64 hidden-state rows
constexpr int kNIW = kVT / 4 / 4;        // load instructions per wavefront for a W chunk (4 rows each, wavefronts 0-3)
constexpr int kNIHid = kMB / 4 / 4;      // ... and for a hidden-state chunk (wavefronts 4-7)

struct HeadParams {
    const uint16_t* hidden;
    const uint16_t* W;
    int64_t h_stride_row;        // elements between consecutive (request, node) rows; rows are b*N_max + i
    int64_t w_stride_v;
    int M, E, V, N_max;
    const int32_t* num_nodes;
    int32_t* amax;
    float* max_logit;
    int32_t* ws_cnt;             // [node blocks] arrival tickets, zero between calls
    unsigned long long* ws_key;  // best keys: [blocks of node rows][vocabulary tiles][rows of the block]
};

__device__ __forceinline__ void head_dma(const void* sbase, uint32_t voff, uint32_t lds_dst, bool stream_once) {
    if (stream_once)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                     : : "v"(voff), "s"(sbase), "s"(lds_dst) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     : : "v"(voff), "s"(sbase), "s"(lds_dst) : "memory");
}

template <int N>
__device__ __forceinline__ void head_wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// (logit, token) as one unsigned key ordered by "greater logit, then lower token"; -0 == +0.
__device__ __forceinline__ unsigned long long head_key(float v, int idx) {
    uint32_t u = __float_as_uint(v + 0.0f);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return (static_cast<unsigned long long>(u) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(idx));
}

__device__ __forceinline__ float head_key_value(unsigned long long k) {
    uint32_t u = static_cast<uint32_t>(k >> 32);
    u = (u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u;
    return __uint_as_float(u);
}

// The end of both kernels, for node rows row0 .. row0 + rows - 1 (rows even, <= ROWS; a request's padding rows included)
// of vocabulary tile vt: s_key[w][row] holds the tile's best keys, in PARTS parts.  They go to the workspace; the last
// workgroup of these rows to arrive takes the maximum over the tiles.
template <int PARTS, int ROWS>
__device__ __forceinline__ void head_finish(const HeadParams& p, unsigned long long (*s_key)[ROWS], int* s_flag, int vt, int nvt,
                                            int group, int row0, int rows) {
    const int tid = threadIdx.x;
    unsigned long long* const keys = p.ws_key + static_cast<int64_t>(row0) * nvt;
    if (tid < rows) {
        unsigned long long best = s_key[0][tid];
#pragma unroll
        for (int w = 1; w < PARTS; ++w) best = s_key[w][tid] > best ? s_key[w][tid] : best;
        // write-through: read by another workgroup in this kernel
        __hip_atomic_store(keys + static_cast<int64_t>(vt) * rows + tid, best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    head_wait_vmcnt<0>();                                  // the stores have been acknowledged
    __syncthreads();
    if (tid == 0) {
        int32_t* cnt = p.ws_cnt + group;
        const int last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nvt - 1;
        if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = last;
    }
    __syncthreads();
    if (!*s_flag) return;
    // A thread takes two neighbouring rows (16 bytes) of every kSlices-th tile, 16 device-coherent loads
    // requested back to back and waited for once (requested one by one, each costs a memory round
    // trip: 8.7 us for 250 tiles, against 1 us this way).  The compiler does not track these
    // loads; every register passes through an empty asm after the wait so that no use can
    // be scheduled before it.  Tiles and rows past the last are clamped: taking a key
    // twice does not change a maximum.
    constexpr int kPairs = ROWS / 2, kSlices = kHeadThreads / kPairs;
    unsigned long long best0 = 0, best1 = 0;
    const int pair = tid % kPairs, slice = tid / kPairs;
    if (slice < kSlices) {
        for (int t0 = slice; t0 < nvt; t0 += 16 * kSlices) {
            u32x4 r[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const uint32_t voff = static_cast<uint32_t>(min(t0 + kSlices * u, nvt - 1)) * (rows * 8) + min(2 * pair, rows - 2) * 8;
                asm volatile("global_load_dwordx4 %0, %1, %2 sc1" : "=v"(r[u]) : "v"(voff), "s"(keys) : "memory");
            }
            head_wait_vmcnt<0>();
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                asm volatile("" : "+v"(r[u]));
                const unsigned long long k0 = (static_cast<unsigned long long>(r[u][1]) << 32) | r[u][0];
                const unsigned long long k1 = (static_cast<unsigned long long>(r[u][3]) << 32) | r[u][2];
                best0 = k0 > best0 ? k0 : best0;
                best1 = k1 > best1 ? k1 : best1;
            }
        }
        s_key[slice][2 * pair] = best0;
        s_key[slice][2 * pair + 1] = best1;
    }
    __syncthreads();
    if (tid < rows) {
        unsigned long long best = s_key[0][tid];
#pragma unroll
        for (int w = 1; w < kSlices; ++w) best = s_key[w][tid] > best ? s_key[w][tid] : best;
        const int row = row0 + tid;
        if (row < p.M) {
            const int b = row / p.N_max, i = row % p.N_max;
            const int n = p.num_nodes ? p.num_nodes[b] : p.N_max;
            const bool real = i < n;
            p.amax[row] = real ? static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(best)) : -1;
            if (p.max_logit) p.max_logit[row] = real ? head_key_value(best) : 0.f;
        }
    }
}

// ---- one block of 64 node rows per pass over W ------------------------------------------------------
//   grid      (vocabulary tiles of 128 rows) x (blocks of 64 node rows; more than one only for row
//             strides that head_gemm_kernel's 32-bit offsets cannot reach).  A workgroup is 8
//             wavefronts: wavefront (vs, nh) owns the 32 x 32 block (vocabulary rows 32vs.., nodes
//             32nh..) of the tile's 128 x 64 logits, 16 accumulator registers
//   fetch     the contraction runs in chunks of 128 hidden units, every workgroup starting at a
//             different chunk (so that the loads in flight spread over all memory channels).  A
//             chunk is 128 rows of W and 64 rows of hidden states, 256 bytes each, brought into two
//             three-slot LDS rings (two chunks ahead) by direct-to-LDS loads (non-temporal for W,
//             which is used once; the hidden states are re-read by every workgroup and stay in L2);
//             one load instruction moves four whole rows, and lands them XOR-swizzled so that the
//             operand reads are conflict-free.  Completion is tracked by hand with s_waitcnt vmcnt;
//             one barrier per chunk publishes the landed shares and frees the consumed slot
__global__ __launch_bounds__(kHeadThreads) void head_argmax_kernel(HeadParams p) {
    __shared__ __attribute__((aligned(1024))) unsigned char s_wring[kRing * kWBytes];
    __shared__ __attribute__((aligned(1024))) unsigned char s_hring[kRing * kHBytes];
    __shared__ unsigned long long s_key[16][kMB];
    __shared__ int s_flag;

    const int vt = blockIdx.x, nvt = gridDim.x, mb = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int vs = wave & 3, nh = wave >> 2;
    const int l16 = lane & 15, g = lane >> 4;
    const int v0 = vt * kVT;
    const int nch = p.E / kKC;

    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const uint32_t wring_lds = (uint32_t)(uintptr_t)(lds_byte*)s_wring;
    const uint32_t hring_lds = (uint32_t)(uintptr_t)(lds_byte*)s_hring;

    // ---- chunk fetch: load instruction i moves rows 4i .. 4i+3 (lane -> row lane/16, granule lane%16,
    // fetched from granule position ^ (row % 16)).  Wavefronts 0-3 fetch W (instructions 8*wave + ii),
    // wavefronts 4-7 the hidden states (instructions 4*(wave-4) + ii).
    // Rows past the vocabulary / past the last node row re-read the last real row.
    const int lrow = lane >> 4, lpos = lane & 15;
    const bool w_issuer = wave < 4;                        // uniform
    const int iw = w_issuer ? wave : wave - 4;
    uint32_t voff_w[kNIW];
    const uint16_t* base_w[kNIW];
#pragma unroll
    for (int ii = 0; ii < kNIW; ++ii) {
        const int r = (kNIW * iw + ii) * 4 + lrow;                          // row of the tile
        const int r0 = min(v0 + (kNIW * iw + ii) * 4, p.V - 1);             // uniform: first row of the group, clamped
        const int rl = min(v0 + r, p.V - 1) - r0;                           // this lane's row relative to it (>= 0)
        base_w[ii] = p.W + static_cast<int64_t>(r0) * p.w_stride_v;
        voff_w[ii] = static_cast<uint32_t>(rl * p.w_stride_v * 2) + (lpos ^ (r & 15)) * 16;
    }
    // The j-th chunk a workgroup takes is chunk (j + rot) mod nch of the hidden dimension: if all
    // workgroups walked the columns of W in step, every load in flight on the chip would sit at the
    // same offset inside an 8 KB row, i.e. on a few of the memory channels (measured at 32000 x 4096:
    // 63 us without the rotation, 55 us with it -- the same as with W repacked into contiguous
    // 32 KB blocks; multipliers 1, 3, 11, 13 gave 56 us, 7 and 9 gave 58 - 62 us).
    const int rot = (5 * vt + vt / 8) % nch;
    auto chunk_of = [&](int j) { const int c = j + rot; return c >= nch ? c - nch : c; };
    auto issue_w = [&](int j) {                            // wavefronts 0-3: chunk j of W
        const uint32_t dst = wring_lds + (j % kRing) * kWBytes;
        const int c = chunk_of(j);
#pragma unroll
        for (int ii = 0; ii < kNIW; ++ii)
            head_dma(base_w[ii] + c * kKC, voff_w[ii], dst + (kNIW * iw + ii) * 1024, true);
    };
    auto issue_h = [&](int j) {                            // wavefronts 4-7: chunk j of the hidden states
        const uint32_t dst = hring_lds + (j % kRing) * kHBytes;
        const int c = chunk_of(j);
        const int m0 = mb * kMB;
#pragma unroll
        for (int ii = 0; ii < kNIHid; ++ii) {
            const int r = (kNIHid * iw + ii) * 4 + lrow;
            const int r0 = min(m0 + (kNIHid * iw + ii) * 4, p.M - 1);        // uniform
            const int rl = min(m0 + r, p.M - 1) - r0;
            const uint32_t voff = static_cast<uint32_t>(rl * p.h_stride_row * 2) + (lpos ^ (r & 15)) * 16;
            head_dma(p.hidden + static_cast<int64_t>(r0) * p.h_stride_row + c * kKC, voff,
                     dst + (kNIHid * iw + ii) * 1024, false);
        }
    };
    // waits until at most `ahead` (0 or 1) requests of this wavefront's kind are outstanding
    auto wait_ahead = [&](int ahead) {
        if (ahead < 1) head_wait_vmcnt<0>();
        else if (w_issuer) head_wait_vmcnt<kNIW>();
        else head_wait_vmcnt<kNIHid>();
    };
    auto issue = [&](int j) { if (w_issuer) issue_w(j); else issue_h(j); };
    issue(0);
    if (nch > 1) issue(1);
    wait_ahead(min(2, nch) - 1);                           // chunk 0 has landed
    __syncthreads();

    f32x4 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int j = 0; j < nch; ++j) {
        // the slot a request goes to was last read before the barrier that ended the previous step
        if (j + 2 < nch) issue(j + 2);
        const unsigned char* wt = s_wring + (j % kRing) * kWBytes;
        // A: lane (vocab row 32vs + 16x + l16, g) holds hidden units 32c + 8g .. +7 of the chunk
        bf16x8 wa[2][4];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int r = 32 * vs + 16 * x + l16;
                wa[x][c] = *reinterpret_cast<const bf16x8*>(wt + (r * 16 + ((4 * c + g) ^ (r & 15))) * 16);
            }
        // B: lane (node 32nh + 16y + l16 of the block, g) holds the same units of that node's hidden state
        const unsigned char* ht = s_hring + (j % kRing) * kHBytes;
        bf16x8 hb[2][4];
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int r = 32 * nh + 16 * y + l16;
                hb[y][c] = *reinterpret_cast<const bf16x8*>(ht + (r * 16 + ((4 * c + g) ^ (r & 15))) * 16);
            }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[x][c], hb[y][c], acc[x][y], 0, 0, 0);
        // this wavefront's reads of the slots have returned and its share of the next chunk has
        // landed; the barrier extends both to the workgroup
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_ahead(min(j + 2, nch - 1) - (j + 1));
        __syncthreads();
    }

    // ---- epilogue: acc[x][y][i] = logit of token v0 + 32vs + 16x + 4g + i at node row 64mb + 32nh + 16y + l16.
#pragma unroll
    for (int y = 0; y < 2; ++y) {
        unsigned long long best = 0;                       // 0 = no token (a real key is never 0)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int v = v0 + 32 * vs + 16 * x + 4 * g + i;
                const unsigned long long k = v < p.V ? head_key(acc[x][y][i], v) : 0ull;
                best = k > best ? k : best;
            }
        unsigned long long o = __shfl_xor(best, 16);
        best = o > best ? o : best;
        o = __shfl_xor(best, 32);
        best = o > best ? o : best;
        if (g == 0) s_key[vs][32 * nh + 16 * y + l16] = best;
    }
    __syncthreads();
    head_finish<4, kMB>(p, s_key, &s_flag, vt, nvt, mb, mb * kMB, kMB);
}

// ---- more than 64 node rows: a matrix product --------------------------------------------------------
//   tile      a workgroup of 8 wavefronts computes BV = 64 WV vocabulary rows x BM = 128/WV TN node rows;
//             wavefront (wv, wm) owns 64 x 16 TN of it.  A wavefront tile of 64 x 128 reads 12 operand
//             granules from LDS for 32 products; the 32 x 32 of head_argmax_kernel 4 for 4, which
//             holds the matrix pipe to half its rate whatever else is done
//   fetch     in steps of 64 hidden units: rows of 128 bytes, one cache line each (64-byte rows, for
//             deeper rings, halve what the vector cache delivers: 161 us in place of 146 below),
//             swizzled like above.  What bounds the larger tiles is the distance of the requests
//             from HBM: 160 KB of LDS hold three steps of W and two of hidden states of a 256 x 256
//             tile.  Without the products it takes 113 us below, without fetches and LDS reads 100
//   pipeline  operands of the half step after the one being multiplied are read from LDS meanwhile;
//             the one barrier per step stands between the two halves, so the wavefronts reach it with
//             a half step of products whose operands they hold already
//   order     workgroups that share a W tile are neighbours on one XCD: its L2 fetches W once
// 480 rows x 5120 x 32000: 146 us (1.08 PFLOP/s; 193 with eight blocks of 64 rows per pass over W);
// 360 x 3584 x 32000: 87 us (140); 240 x 5120 x 32000: 95 (115); 180 x 4096 x 50000: 95 (162);
// 120 x 4096 x 32000: 53 (60; streaming W alone 50).
constexpr int kGK = 64;

template <int WV, int TN, int SW, int SH>                  // SW, SH: slots of the W and of the hidden-state ring
struct GemmTile {
    static constexpr int WM = 8 / WV, BV = 64 * WV, BM = WM * TN * 16;
    static constexpr int kWSlot = BV * kGK * 2, kHSlot = BM * kGK * 2;
    static constexpr int kLds = SW * kWSlot + SH * kHSlot;
};

template <int WV, int TN, int SW, int SH, bool ONCE>       // ONCE: one tile of node rows, W is read by one workgroup only
__global__ __launch_bounds__(kHeadThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void head_gemm_kernel(HeadParams p, int nvt, int nmb, int per_xcd) {
    using G = GemmTile<WV, TN, SW, SH>;
    constexpr int BV = G::BV, BM = G::BM, TV = 4;
    constexpr int IW = BV / 64, IH = (BM + 63) / 64;       // load instructions (8 rows each) per wavefront and step
    constexpr int kDeep = SW > SH ? SW : SH;
    static_assert(G::kLds <= 160 * 1024 && SH >= 2 && SW >= 2, "rings");
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[G::kLds];
    unsigned char* const s_w = s_mem;
    unsigned char* const s_h = s_mem + SW * G::kWSlot;

    const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (work >= nvt * nmb) return;
    const int vt = work / nmb, mb = work - vt * nmb;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wv = wave % WV, wm = wave / WV;
    const int l16 = lane & 15, g = lane >> 4;
    const int v0 = vt * BV, m0 = mb * BM;
    const int nch = p.E / kGK;

    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const uint32_t w_lds = (uint32_t)(uintptr_t)(lds_byte*)s_w, h_lds = (uint32_t)(uintptr_t)(lds_byte*)s_h;
    // load instruction i moves rows 8i .. 8i+7 (lane -> row lane/8, fetched granule (lane % 8) ^ (row % 8)); rows past the
    // vocabulary / the last node row re-read the last real row
    const int lrow = lane >> 3, lgran = ((lane & 7) ^ lrow) << 4;
    uint32_t voff_w[IW], voff_h[IH];
    const uint32_t wrow = static_cast<uint32_t>(p.w_stride_v) * 2u, hrow = static_cast<uint32_t>(p.h_stride_row) * 2u;
#pragma unroll
    for (int i = 0; i < IW; ++i) voff_w[i] = min((wave * IW + i) * 8 + lrow, p.V - 1 - v0) * wrow + lgran;
#pragma unroll
    for (int i = 0; i < IH; ++i) {
        const int inst = min(wave * IH + i, BM / 8 - 1);   // (fewer rows than 64 per wavefront: the last ones are fetched twice)
        voff_h[i] = min(inst * 8 + lrow, p.M - 1 - m0) * hrow + lgran;
    }
    const uint16_t* wbase = p.W + static_cast<int64_t>(v0) * p.w_stride_v;
    const uint16_t* hbase = p.hidden + static_cast<int64_t>(m0) * p.h_stride_row;
    // XCDs walk the columns of W from different places (memory channels, as above); within one, where the workgroups
    // share the hidden states' columns in L2, only by up to three chunks
    const int rot = ((blockIdx.x & 7) * nch / 8 + (vt & 3)) % nch;
    auto chunk_of = [&](int j) { const int c = j + rot; return c >= nch ? c - nch : c; };
    auto issue_w = [&](int j, int slot) __attribute__((always_inline)) {
        const uint16_t* src = wbase + chunk_of(j) * kGK;
        const uint32_t dst = w_lds + slot * G::kWSlot + wave * (IW * 1024);
#pragma unroll
        for (int i = 0; i < IW; ++i) head_dma(src, voff_w[i], dst + i * 1024, ONCE);
    };
    auto issue_h = [&](int j, int slot) __attribute__((always_inline)) {
        const uint16_t* src = hbase + chunk_of(j) * kGK;
        const uint32_t dst = h_lds + slot * G::kHSlot;
#pragma unroll
        for (int i = 0; i < IH; ++i) head_dma(src, voff_h[i], dst + min(wave * IH + i, BM / 8 - 1) * 1024, false);
    };
    // Step t issues H(t + SH), then W(t + SW), where they exist; the prologue is steps -kDeep .. -1.  When step t waits for
    // the operands of t + 1, the requests after them are those of the steps since, and step t + 1 - SH's own W:
    constexpr int kLater = SW > SH ? (SH - 2) * (IH + IW) + IW : (SW - 2) * (IH + IW);
    static_assert(kLater + IH + IW <= 63, "vmcnt");
#pragma unroll
    for (int t = -kDeep; t < 0; ++t) {
        if (t + SH >= 0 && t + SH < nch) issue_h(t + SH, t + SH);
        if (t + SW >= 0 && t + SW < nch) issue_w(t + SW, t + SW);
    }
    if (kDeep <= nch) head_wait_vmcnt<kLater + IH + IW>(); else head_wait_vmcnt<0>();
    __syncthreads();

    f32x4 acc[TV][TN];
#pragma unroll
    for (int x = 0; x < TV; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int frag = l16 * 128 + ((g ^ (l16 & 7)) << 4);   // granule 4c + g of row l16: this ^ (c << 6)
    const unsigned char* const wfrag = s_w + wv * TV * 16 * 128, * const hfrag = s_h + wm * TN * 16 * 128;
    bf16x8 wa[2][TV], hb[2][TN];
    auto fetch = [&](int c, int ws, int hs) __attribute__((always_inline)) {
        const unsigned char* wt = wfrag + ws * G::kWSlot;
        const unsigned char* ht = hfrag + hs * G::kHSlot;
#pragma unroll
        for (int x = 0; x < TV; ++x) wa[c][x] = *reinterpret_cast<const bf16x8*>(wt + x * (16 * 128) + (frag ^ (c << 6)));
#pragma unroll
        for (int y = 0; y < TN; ++y) hb[c][y] = *reinterpret_cast<const bf16x8*>(ht + y * (16 * 128) + (frag ^ (c << 6)));
    };
    auto product = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
            for (int x = 0; x < TV; ++x) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[c][x], hb[c][y], acc[x][y], 0, 0, 0);
    };
    int ws = 0, hs = 0;                                    // slots of step j
    fetch(0, 0, 0);
    for (int j = 0; j < nch - 1; ++j) {
        fetch(1, ws, hs);
        product(0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // step j + 1 has landed
        if (j + kDeep - 1 < nch) head_wait_vmcnt<kLater>(); else head_wait_vmcnt<0>();
        __syncthreads();                                   // and nobody reads slot j any more
        __builtin_amdgcn_sched_barrier(0);
        const int ws1 = ws == SW - 1 ? 0 : ws + 1, hs1 = hs == SH - 1 ? 0 : hs + 1;
        fetch(0, ws1, hs1);
        if (j + SH < nch) issue_h(j + SH, hs);
        if (j + SW < nch) issue_w(j + SW, ws);
        product(1);
        ws = ws1;
        hs = hs1;
    }
    fetch(1, ws, hs);
    product(0);
    product(1);
    __syncthreads();

    // ---- epilogue: acc[x][y][i] = logit of token v0 + 64wv + 16x + 4g + i at node row m0 + wm 16 TN + 16y + l16 ------
    unsigned long long (*s_key)[BM] = reinterpret_cast<unsigned long long (*)[BM]>(s_mem);      // [WV]; the rings are done with
#pragma unroll
    for (int y = 0; y < TN; ++y) {
        unsigned long long best = 0;                       // 0 = no token (a real key is never 0)
#pragma unroll
        for (int x = 0; x < TV; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int v = v0 + 16 * TV * wv + 16 * x + 4 * g + i;
                const unsigned long long k = v < p.V ? head_key(acc[x][y][i], v) : 0ull;
                best = k > best ? k : best;
            }
        unsigned long long o = __shfl_xor(best, 16);
        best = o > best ? o : best;
        o = __shfl_xor(best, 32);
        best = o > best ? o : best;
        if (g == 0) s_key[wv][(wm * TN + y) * 16 + l16] = best;
    }
    __syncthreads();
    int* const s_flag = reinterpret_cast<int*>(s_mem + G::kLds - 16);
    head_finish<WV, BM>(p, s_key, s_flag, vt, nvt, mb, m0, min(BM, (p.M + 63) / 64 * 64 - m0));
}

template <int WV, int TN, int SW, int SH>
void launch_gemm(const HeadParams& p, hipStream_t stream) {
    using G = GemmTile<WV, TN, SW, SH>;
    const int nvt = (p.V + G::BV - 1) / G::BV, nmb = (p.M + G::BM - 1) / G::BM;
    const int per_xcd = (nvt * nmb + 7) / 8;
    const dim3 grid(per_xcd * 8), block(kHeadThreads);
    if (nmb == 1) hipLaunchKernelGGL((head_gemm_kernel<WV, TN, SW, SH, true>), grid, block, 0, stream, p, nvt, nmb, per_xcd);
    else hipLaunchKernelGGL((head_gemm_kernel<WV, TN, SW, SH, false>), grid, block, 0, stream, p, nvt, nmb, per_xcd);
}

// The tiles.  A workgroup fills a compute unit, so a call takes ceil(tiles / 256) rounds of the hidden dimension; a
// step of one takes 0.36 us + 2.15e-5 us x BV x BM (fits the measured steps of all of these within a tenth: 0.74 - 0.83 us
// for 128 x 128, 1.04 - 1.19 for 256 x 128, 1.48 - 1.56 for 256 x 192, 1.77 for 256 x 256).  The tile with the least sum
// was the fastest, or within 2 % of it, at 26 of 28 shapes from 80 x 4096 x 50000 to 480 x 4096 x 152064 (5 % off at the
// others).  Of 128 x 192 and 256 x 96, which cost the same, the former is faster (113 against 121 us at 180 x 4096 x 50000).
struct HeadTile {
    int bv, bm;
    void (*launch)(const HeadParams&, hipStream_t);
};
const HeadTile kHeadTiles[] = {
    {128, 128, launch_gemm<2, 2, 5, 4>}, {128, 192, launch_gemm<2, 3, 5, 3>}, {256, 96, launch_gemm<4, 3, 3, 4>},
    {256, 128, launch_gemm<4, 4, 3, 3>}, {256, 160, launch_gemm<4, 5, 3, 3>}, {256, 192, launch_gemm<4, 6, 3, 2>},
    {256, 224, launch_gemm<4, 7, 3, 2>}, {256, 256, launch_gemm<4, 8, 3, 2>},
};

const HeadTile& head_tile(int M, int V) {
    const HeadTile* best = nullptr;
    int64_t least = 0;
    for (const HeadTile& t : kHeadTiles) {
        const int64_t tiles = static_cast<int64_t>((V + t.bv - 1) / t.bv) * ((M + t.bm - 1) / t.bm);
        const int64_t cost = (tiles + 255) / 256 * (16744 + t.bv * t.bm);       // 16744 = 0.36 / 2.15e-5
        if (!best || cost < least) best = &t, least = cost;
    }
    return *best;
}

static size_t head_counter_bytes(int mblocks) {
    return (static_cast<size_t>(mblocks) * sizeof(int32_t) + 255) / 256 * 256;
}

}  // namespace

size_t head_argmax_workspace_bytes(int32_t B, int32_t N_max, int32_t V) {
    const int M = B * N_max;
    const int mblocks = (M + kMB - 1) / kMB, nvt = (V + kVT - 1) / kVT;
    return head_counter_bytes(mblocks) + static_cast<size_t>(mblocks) * nvt * kMB * sizeof(unsigned long long);
}

int32_t launch_head_argmax(int32_t B, int32_t N_max, int32_t E, int32_t V, const void* hidden,
                           int64_t h_stride_row, const void* W, int64_t w_stride_v, const int32_t* num_nodes,
                           int32_t* amax, float* max_logit, void* workspace, hipStream_t stream) {
    HeadParams p;
    p.hidden = static_cast<const uint16_t*>(hidden);
    p.W = static_cast<const uint16_t*>(W);
    p.h_stride_row = h_stride_row;
    p.w_stride_v = w_stride_v;
    p.M = B * N_max; p.E = E; p.V = V; p.N_max = N_max;
    p.num_nodes = num_nodes;
    p.amax = amax;
    p.max_logit = max_logit;
    const int mblocks = (p.M + kMB - 1) / kMB, nvt = (V + kVT - 1) / kVT;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    p.ws_cnt = reinterpret_cast<int32_t*>(ws);
    p.ws_key = reinterpret_cast<unsigned long long*>(ws + head_counter_bytes(mblocks));
    // head_gemm_kernel addresses the rows of a tile by 32-bit offsets from its first one
    constexpr int64_t kStrideLimit = (1ll << 32) / (2 * 256);
    if (mblocks == 1 || h_stride_row >= kStrideLimit || w_stride_v >= kStrideLimit)
        hipLaunchKernelGGL(head_argmax_kernel, dim3(nvt, mblocks), dim3(kHeadThreads), 0, stream, p);
    else
        head_tile(p.M, V).launch(p, stream);
    return check_launch();
}

}  // namespace specvlm
