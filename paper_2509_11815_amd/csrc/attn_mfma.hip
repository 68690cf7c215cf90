// Tree-masked verification attention for bf16 caches on the gfx950 matrix cores.
//
// The step is bound by streaming K and V once from HBM (SpecVLM Sec. 3.2); all (up to 64)
// tree queries of a head share that single pass.  Work decomposition:
//
//   grid      one workgroup (8 wavefronts, two per SIMD) per (request, query head, split).
//             A workgroup runs 2 independent key "streams"; stream s of the 2*splits streams
//             of a (request, head) owns the 32-key tiles s, s + 2*splits, ... (neighbouring
//             streams read neighbouring memory: measured 5 % faster than one contiguous chunk
//             per stream; a step costs the same whatever part of its tile is real, so cutting
//             the last round into equal shorter spans gained nothing).  Four wavefronts
//             share a stream: each takes 16 of the 64 query rows, so a K/V byte is fetched
//             from HBM exactly once and read from LDS four times.  Two wavefronts per SIMD
//             let one's matrix work overlap the other's softmax arithmetic and LDS latency
//   fetch     every stream keeps a private four-slot LDS ring filled by direct-to-LDS loads
//             (global_load_lds_dwordx4, non-temporal since the bytes are used once: no registers
//             are tied up by bytes in flight); one load
//             instruction moves four whole 256-byte rows, fully coalesced.  Each wavefront of
//             a stream requests 8 of a tile's 32 rows.  Two tiles per stream are in flight
//             ahead of the one consumed (64 KB per compute unit): with every compute unit
//             streaming the chip is saturated at that depth, more in flight measured
//             slower.  Completion is tracked by hand with
//             s_waitcnt vmcnt, and one workgroup barrier per tile publishes the landed
//             shares and frees the consumed slot.  With a contiguous cache a stream's first
//             tile is requested before the request's lengths have arrived
//   QK^T      S^T[32 keys x 64 q] = K . Q^T with v_mfma_f32_16x16x32_bf16; the lanes fetch
//             K granules in XOR-swizzled order so that the operand reads (16 different rows
//             per 16 lanes) are free of LDS bank conflicts; a wavefront's Q fragments stay in
//             registers for the whole kernel (staged once through the idle ring slot)
//   softmax   online (running max / sum per query) in fp32 on the S^T fragments: a lane
//             holds one query and 8 keys, so row statistics need two cross-lane steps, and
//             exp2(S^T) packed to bf16 is already the B operand of the next MFMA
//   PV        O^T[D x 64 q] += V^T . P^T; the V^T operand comes out of LDS transposed
//             (ds_read_b64_tr_b16 on V tiles swizzled in 32-byte chunks; the contraction
//             index may be permuted freely, so an operand's "8 consecutive k" are the 8
//             keys whose probabilities the lane already holds)
//   masks     prefix keys need none; only tiles touching the tree region or the request's
//             end test the per-query ancestor bit mask (select, never multiply)
//   merge     the streams of a workgroup are merged through LDS (one round, the rings are
//             free by then; every wavefront ends up owning 16 query rows x half the head
//             dims, at head size 64 and one workgroup per compute unit four of them 16 rows); the workgroup's partial goes, as bf16, to a lane-major
//             workspace with write-through stores, and for every (query block, half) the last
//             split to arrive -- found with a ticket counter -- merges the splits, adding a
//             split up while the next ones still load.  (With one owner for all head dims of a block four of the
//             eight wavefronts idled from here on: 16.87 -> 16.42 us per call at the 2880-visual-token prefix)
#include <atomic>

#include "attn_common.hpp"

namespace specvlm {

constexpr int kWaves = 8;           // wavefronts per workgroup: two per SIMD
constexpr int kShare = 4;           // wavefronts sharing one key stream, 64/kShare query rows each
constexpr int kAhead = 2;           // tiles per stream kept in flight ahead of the one being consumed
constexpr int kThreads = kWaves * 64;
static_assert(kWaves / kShare == kStreamsPerWg, "the plan's streams");

struct MfmaParams {
    KvGeom g;
    int N_max, H_q, group, num_splits;
    float scale;                // softmax scale
    const uint16_t *q, *k, *v;
    uint16_t* o;
    float* lse;
    int64_t q_sb, q_sn, q_sh, o_sb, o_sn, o_sh;
    const int32_t *prefix_len, *num_nodes, *parent;
    int32_t* err_flag;
    int32_t* ws_cnt;            // [B*H_q][4 query blocks] arrival tickets, kCounterStride words apart, zero between calls
    int second_counters;        // words from a query block's first ticket counter to its second (one per half of the head dims)
    float* ws_acc;              // [B*H_q*num_splits][4 qb][2 halves][D/64][64 lanes] 16-byte vectors of packed bf16
    float* ws_ml;               // [B*H_q*num_splits][64 q][2] (max, sum)
    int xcd_heads;              // query heads of every request an XCD takes, 0: a contiguous range of items each
};

// Writes half the head dims of 16 query rows: out[t][i] = O^T[d = 16 (half NT + t) + 4g + i][q], unnormalised.
template <int NT>
__device__ __forceinline__ void store_rows(const MfmaParams& p, const f32x4 (&out)[NT], float M, float L,
                                           int b, int h, int qi, int g, int n, int half) {
    if (qi >= n) return;
    const float inv = 1.f / L;
    // A lane holds 4 consecutive head dims per block t.  Lanes g = 2v and 2v+1 of a query row
    // trade halves so that each stores 8 consecutive dims (16 bytes): the even lane keeps the
    // even blocks, the odd lane the odd ones.
    const bool odd = g & 1;
    uint16_t* orow = p.o + b * p.o_sb + qi * p.o_sn + h * p.o_sh + 4 * (g & ~1) + half * (NT * 16);
#pragma unroll
    for (int u = 0; u < NT / 2; ++u) {
        const uint32_t e0 = pack_bf16x2(out[2 * u][0] * inv, out[2 * u][1] * inv);
        const uint32_t e1 = pack_bf16x2(out[2 * u][2] * inv, out[2 * u][3] * inv);
        const uint32_t o0 = pack_bf16x2(out[2 * u + 1][0] * inv, out[2 * u + 1][1] * inv);
        const uint32_t o1 = pack_bf16x2(out[2 * u + 1][2] * inv, out[2 * u + 1][3] * inv);
        const uint32_t r0 = __shfl_xor(odd ? e0 : o0, 16);     // the partner's share of the block this lane keeps
        const uint32_t r1 = __shfl_xor(odd ? e1 : o1, 16);
        const u32x4 w = odd ? u32x4{r0, r1, o0, o1} : u32x4{e0, e1, r0, r1};
        *reinterpret_cast<u32x4*>(orow + 16 * (2 * u + (odd ? 1 : 0))) = w;
    }
    if (p.lse && g == 0 && half == 0)
        p.lse[(static_cast<int64_t>(b) * p.H_q + h) * p.N_max + qi] = M * p.scale + __log2f(L) * kLn2;
}

// PD tiles per stream are kept in flight ahead of the one consumed.  Measured on the 2880-visual-token workload, with a merge that
// had one owner per query block: PD = 2 19.5 us per layer, 3 20.0, 1 20.8; two wavefronts of 32 query rows per stream, four streams,
// PD = 1 21.8 (a form that is gone).
// Two launch shapes of the same body (attn_mfma_body.inc).
//   attn_mfma_kernel      128 KB of rings (four slots per stream, two tiles in flight ahead), one
//                         workgroup per compute unit: few (request, head) pairs, long streams
//   attn_mfma_kernel_2wg  64 KB of rings (two slots, one tile ahead) and at most 128 registers, so
//                         that two workgroups share a compute unit: twice as many (request, head,
//                         split) items are resident at once
template <int D, int PD>
__global__ __launch_bounds__(kThreads) void attn_mfma_kernel(MfmaParams p) {
    // Two owners per query block shorten the chain at head size 128.  At 64 a half is one 16-byte vector, and twice the tickets and
    // (max, sum) pairs cost more: 7 x 40 query / 10 KV heads, 560 keys, four ranges 29.3 us with one owner, 30.6 with two.
    constexpr int SL = 4, MB = 8, OWNERS = D == 128 ? 2 : 1;
#include "attn_mfma_body.inc"
}

template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void attn_mfma_kernel_2wg(MfmaParams p) {
    constexpr int PD = 1, SL = 2, MB = 3, OWNERS = 2;
#define SPECVLM_SPREAD_REQUESTS
#include "attn_mfma_body.inc"
#undef SPECVLM_SPREAD_REQUESTS
}

// ---- library-owned scratch for callers that cannot allocate device memory -----------------------
// One array per GPU (each device holds its own copy of the code object's globals, zero when the
// object is loaded).  Host code must not use the array's name as an address: the device address
// is asked for once per device and kept.
static __device__ __align__(256) unsigned char scratch[SPECVLM_STATIC_WORKSPACE_BYTES];

int32_t attn_static_workspace(void** ptr_out) {
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> ptr_of_device[kMaxDevices];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        note_hip_error(e != hipSuccess ? e : hipErrorInvalidDevice);
        return SPECVLM_HIP_ERROR;
    }
    void* ptr = ptr_of_device[dev].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));         // this device's copy (the current device)
        if (e != hipSuccess || !ptr) {
            note_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
            return SPECVLM_HIP_ERROR;
        }
        ptr_of_device[dev].store(ptr, std::memory_order_release);   // two threads racing here store the same address
    }
    *ptr_out = ptr;
    return SPECVLM_OK;
}

int32_t launch_attn_mfma(const AttnArgs& a) {
    const specvlm_attn_desc& d = a.d;
    if (a.plan.columns) return launch_attn_streams(a);
    if (a.plan.block_rows) return launch_attn_wave(a);
    MfmaParams p;
    p.g = KvGeom{d.kv_stride_b, d.kv_stride_h, d.kv_stride_t, d.paged ? a.block_table : nullptr,
                 d.max_blocks_per_req, d.num_blocks,
                 d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity};
    p.N_max = d.N_max; p.H_q = d.H_q; p.group = d.H_q / d.H_kv;
    p.num_splits = a.plan.splits;
    p.xcd_heads = d.B > 1 && d.H_kv % 8 == 0 ? d.H_q / 8 : 0;
    p.scale = a.scale;
    p.q = static_cast<const uint16_t*>(a.q);
    p.k = static_cast<const uint16_t*>(a.k);
    p.v = static_cast<const uint16_t*>(a.v);
    p.o = static_cast<uint16_t*>(a.o);
    p.lse = a.lse;
    p.q_sb = d.q_stride_b; p.q_sn = d.q_stride_n; p.q_sh = d.q_stride_h;
    p.o_sb = d.o_stride_b; p.o_sn = d.o_stride_n; p.o_sh = d.o_stride_h;
    p.prefix_len = a.prefix_len; p.num_nodes = a.num_nodes; p.parent = a.parent;
    p.err_flag = a.err_flag;
    const size_t parts = static_cast<size_t>(d.B) * d.H_q * p.num_splits;
    unsigned char* ws = static_cast<unsigned char*>(a.workspace);
    p.ws_cnt = reinterpret_cast<int32_t*>(ws);
    // a line of its own for the second counters too, where the region has one (more than 512 pairs: the first ones' lines)
    p.second_counters = d.B * d.H_q <= kMaxSplitHeads / 2 ? kMaxSplitHeads / 2 * 4 * kCounterStride : kCounterStride / 2;
    p.ws_acc = reinterpret_cast<float*>(ws + kCounterBytes);
    p.ws_ml = p.ws_acc + parts * kQRows * d.D / 2;
    const dim3 grid(static_cast<unsigned>(parts)), block(kThreads);
    // More work items than compute units, but no more than fit two to a unit: the second shape keeps
    // all of them resident at once instead of running a second, partly filled round (13B-shaped
    // batch of 4 with 3 splits, 480 items: 70.7 against 75.8 us; with 256 items or fewer the first
    // shape's deeper rings win: 16.5 against 23.3 us at the 2880-visual-token prefix).
    if (parts > 256 && parts <= kMostTwoPerCu) {
        if (d.D == 128) hipLaunchKernelGGL((attn_mfma_kernel_2wg<128>), grid, block, 0, a.stream, p);
        else hipLaunchKernelGGL((attn_mfma_kernel_2wg<64>), grid, block, 0, a.stream, p);
    } else {
        if (d.D == 128) hipLaunchKernelGGL((attn_mfma_kernel<128, kAhead>), grid, block, 0, a.stream, p);
        else hipLaunchKernelGGL((attn_mfma_kernel<64, kAhead>), grid, block, 0, a.stream, p);
    }
    return check_launch();
}

}  // namespace specvlm
