// Tree-masked verification attention in fp32 arithmetic throughout.
//
// attn_f32_kernel is the path for SPECVLM_F32 tensors (tolerance 1e-5): the products run on the matrix
// cores' fp32 form (v_mfma_f32_16x16x4_f32, a full fp32 fused multiply-add).  One workgroup of 8 wavefronts
// per (request, query head, block of 16 tree nodes); wavefront w takes the 16-key tiles w, w + 8, ... straight
// from memory into operand registers (a tile never straddles a page).  It is bound by latency: memory round
// trips and a merge of eight streams through LDS.
// Before, fp32 ran on the kernel below, one workgroup per node, whose merge of 256 private states was
// 6 x D dependent cross-lane steps: 18.3 -> 5.4 us per call at 72 keys, 4 heads of 64, 8 nodes.
//
// attn_valu_kernel, vector ALUs only, is the measurement aid (what a kernel without matrix cores reaches):
// one 256-thread workgroup per (request, query head, tree node).  Thread t visits the
// visible keys t, t+256, ... with a private online softmax (running max, sum and a D-wide
// accumulator in registers); the 256 partial states are merged at the end.
#include <type_traits>

#include "common.hpp"

namespace specvlm {

template <typename T>
__device__ __forceinline__ void load16(const T* p, float* out);   // 16 bytes -> floats

template <>
__device__ __forceinline__ void load16<float>(const float* p, float* out) {
    float4 w = *reinterpret_cast<const float4*>(p);
    out[0] = w.x; out[1] = w.y; out[2] = w.z; out[3] = w.w;
}
template <>
__device__ __forceinline__ void load16<uint16_t>(const uint16_t* p, float* out) {
    uint4 w = *reinterpret_cast<const uint4*>(p);
    const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        out[2 * e] = __uint_as_float(x[e] << 16);
        out[2 * e + 1] = __uint_as_float(x[e] & 0xFFFF0000u);
    }
}

__device__ __forceinline__ void store_elem(float* p, float x) { *p = x; }
__device__ __forceinline__ void store_elem(uint16_t* p, float x) {
    uint32_t u = __float_as_uint(x);                     // round to nearest even
    u += 0x7FFFu + ((u >> 16) & 1u);
    *p = static_cast<uint16_t>(u >> 16);
}

struct ValuParams {
    KvGeom g;
    int N_max, H_q, group;
    float scale;
    const void *q, *k, *v;
    void* o;
    float* lse;
    int64_t q_sb, q_sn, q_sh, o_sb, o_sn, o_sh;
    const int32_t *prefix_len, *num_nodes, *parent;
    int32_t* err_flag;
};

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_valu_kernel(ValuParams p) {
    constexpr int VEC = 16 / sizeof(T);
    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int hk = h / p.group;
    __shared__ float s_q[D];
    __shared__ unsigned long long s_mask;
    __shared__ int s_err;
    __shared__ float s_red[4][D];
    __shared__ float s_m[4], s_l[4];

    int n = p.num_nodes ? p.num_nodes[b] : p.N_max;
    const int P = p.prefix_len[b];
    int err = 0;
    if (n < 1 || n > p.N_max) err |= SPECVLM_ERR_BAD_NUM_NODES;
    n = min(max(n, 1), p.N_max);
    if (!length_fits(P, n, p.g.capacity)) err |= SPECVLM_ERR_BAD_LENGTH;
    if (tid == 0) {
        // ancestor-or-self bit mask of node i; the walk is bounded by 64 steps
        unsigned long long mask = 0;
        if (i < n) {
            int t = i;
            for (int step = 0; step < SPECVLM_MAX_NODES && t != -1; ++step) {
                mask |= 1ull << t;
                const int par = p.parent[b * p.N_max + t];
                if (t == 0 ? par != -1 : (par < 0 || par >= t)) {
                    err |= SPECVLM_ERR_BAD_PARENT;
                    break;
                }
                t = par;
            }
        }
        s_mask = mask;
        s_err = err;
    }
    const T* q = static_cast<const T*>(p.q) + b * p.q_sb + i * p.q_sn + h * p.q_sh;
    if (i < n && !err && tid < D / VEC) {
        float tmp[VEC];
        load16<T>(q + tid * VEC, tmp);
#pragma unroll
        for (int e = 0; e < VEC; ++e) s_q[tid * VEC + e] = tmp[e];
    }
    __syncthreads();
    err = s_err;
    if (err) {
        if (tid == 0 && p.err_flag) atomicOr(p.err_flag, err);
        return;
    }
    if (i >= n) return;
    const unsigned long long mask = s_mask;
    const int S = P + n;
    const T* kbase = static_cast<const T*>(p.k);
    const T* vbase = static_cast<const T*>(p.v);

    float m = -INFINITY, l = 0.f;
    float acc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) acc[d] = 0.f;
    bool bad_block = false;
    for (int j = tid; j < S; j += 256) {
        const bool visible = j < P || ((mask >> (j - P)) & 1ull);
        if (!visible) continue;
        const int64_t off = kv_row_offset(p.g, b, hk, j, bad_block);
        float dot = 0.f;
#pragma unroll
        for (int c = 0; c < D / VEC; ++c) {
            float kk[VEC];
            load16<T>(kbase + off + c * VEC, kk);
#pragma unroll
            for (int e = 0; e < VEC; ++e) dot = fmaf(s_q[c * VEC + e], kk[e], dot);
        }
        const float s = dot * p.scale;
        const float m_new = fmaxf(m, s);
        const float alpha = expf(m - m_new);          // exp(-inf) = 0 on the first key
        const float w = expf(s - m_new);
        l = l * alpha + w;
#pragma unroll
        for (int c = 0; c < D / VEC; ++c) {
            float vv[VEC];
            load16<T>(vbase + off + c * VEC, vv);
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[c * VEC + e] = fmaf(w, vv[e], acc[c * VEC + e] * alpha);
        }
        m = m_new;
    }
    if (bad_block && p.err_flag) atomicOr(p.err_flag, SPECVLM_ERR_BAD_BLOCK);
    // merge the 256 private states: common max, rescale, sum
    float M = m;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    const int wave = tid >> 6, lane = tid & 63;
    if (lane == 0) s_m[wave] = M;
    __syncthreads();
    M = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));   // finite: node i always sees itself
    const float w = m == -INFINITY ? 0.f : expf(m - M);
    float lw = l * w;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lw += __shfl_xor(lw, off);
    if (lane == 0) s_l[wave] = lw;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        float x = acc[d] * w;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
        if (lane == 0) s_red[wave][d] = x;
    }
    __syncthreads();
    const float Z = (s_l[0] + s_l[1]) + (s_l[2] + s_l[3]);
    T* o = static_cast<T*>(p.o) + b * p.o_sb + i * p.o_sn + h * p.o_sh;
    if (tid < D) {
        const float x = (s_red[0][tid] + s_red[1][tid]) + (s_red[2][tid] + s_red[3][tid]);
        store_elem(o + tid, x / Z);
    }
    if (tid == 0 && p.lse) p.lse[(static_cast<int64_t>(b) * p.H_q + h) * p.N_max + i] = M + logf(Z);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Waves = 8;

template <int D>
__global__ __launch_bounds__(kF32Waves * 64) void attn_f32_kernel(ValuParams p) {
    constexpr int ND = D / 16;                 // 16-wide head-dim blocks
    constexpr int kRow = D + 4;                // floats per row of the merge buffer (padded: 16 rows hit different banks)
    __shared__ __attribute__((aligned(16))) float s_acc[kF32Waves][16 * kRow];
    __shared__ float s_m[kF32Waves][16], s_l[kF32Waves][16];
    const int h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hk = h / p.group, l16 = lane & 15, g = lane >> 4;
    const int row0 = blockIdx.x * 16;

    const int par = p.parent[b * p.N_max + min(lane, p.N_max - 1)];
    int n = p.num_nodes ? p.num_nodes[b] : p.N_max;
    const int P = p.prefix_len[b];
    int err = 0;
    if (n < 1 || n > p.N_max) err |= SPECVLM_ERR_BAD_NUM_NODES;
    n = min(max(n, 1), p.N_max);
    if (!length_fits(P, n, p.g.capacity)) err |= SPECVLM_ERR_BAD_LENGTH;
    const int node = row0 + l16;               // this lane's query (column of S^T and O^T)
    // Q operand: the contraction index of product i of a 16-wide block c is 16c + 4g + i, for K alike
    f32x4 qf[ND];
    {
        const float* q = static_cast<const float*>(p.q) + b * p.q_sb + static_cast<int64_t>(min(node, n - 1)) * p.q_sn + h * p.q_sh;
#pragma unroll
        for (int c = 0; c < ND; ++c) qf[c] = *reinterpret_cast<const f32x4*>(q + 16 * c + 4 * g);
    }
    if (__any(lane < n && (lane == 0 ? par != -1 : (par < 0 || par >= lane)))) err |= SPECVLM_ERR_BAD_PARENT;
    if (err) {                                 // the same in every workgroup of the request
        if (tid == 0 && p.err_flag) atomicOr(p.err_flag, err);
        return;
    }
    if (row0 >= n) return;
    // ancestor-or-self mask of node `lane` by pointer doubling, then of this lane's query
    unsigned long long mask = 1ull << lane;
    {
        int up = lane < n ? par : -1;
        while (__any(up >= 0)) {
            const unsigned long long m2 = __shfl(mask, max(up, 0));
            const int up2 = __shfl(up, max(up, 0));
            if (up >= 0) { mask |= m2; up = up2; }
        }
        mask = __shfl(mask, min(node, n - 1));
    }
    const int S = P + n, ntile = (S + 15) / 16;
    float m, l;
    f32x4 acc[ND];
    bool bad_block = false;
    // Not every row sees every node, and a weight of zero times a V that is not finite is NaN.  `careful` takes such entries
    // of a tile with tree nodes out of the product and adds them to the rows that see them.  It is a second pass, for the
    // wavefronts whose sums are not all finite: looking at V in the first one cost 20.3 -> 22.5 us per call at
    // 500 keys, 2 x 8 heads of 128, 60 nodes; looking at the sums costs 20.35.
    auto stream = [&](auto careful) __attribute__((always_inline)) {
        m = -INFINITY;
        l = 0.f;
#pragma unroll
        for (int t = 0; t < ND; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int tile = wave; tile < ntile; tile += kF32Waves) {
            const int last = S - 1 - 16 * tile;    // rows past the last key re-read it; their weight is zero
            const int64_t base = kv_row_offset(p.g, b, hk, 16 * tile, bad_block);
            const float* kr = static_cast<const float*>(p.k) + base + min(l16, last) * p.g.stride_t + 4 * g;
            f32x4 kf[ND];
#pragma unroll
            for (int c = 0; c < ND; ++c) kf[c] = *reinterpret_cast<const f32x4*>(kr + 16 * c);
            float vf[4][ND];                       // V^T operand: head dim 16t + l16 of key 4g + i
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float* vr = static_cast<const float*>(p.v) + base + min(4 * g + i, last) * p.g.stride_t + l16;
#pragma unroll
                for (int t = 0; t < ND; ++t) vf[i][t] = vr[16 * t];
            }
            bool special = false;
            if constexpr (careful) {
                if (16 * tile + 16 > P) {          // uniform
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int t = 0; t < ND; ++t) {
                            special |= !(fabsf(vf[i][t]) < INFINITY);
                            vf[i][t] = fabsf(vf[i][t]) < INFINITY ? vf[i][t] : 0.f;
                        }
                    special = __any(special);
                }
            }
            f32x4 s = {0.f, 0.f, 0.f, 0.f};        // s[i]: key 4g + i of the tile against this lane's query
#pragma unroll
            for (int c = 0; c < ND; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][i], qf[c][i], s, 0, 0, 0);
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int key = 16 * tile + 4 * g + i, rel = key - P;
                const bool visible = key < S && (rel < 0 || ((mask >> (rel & 63)) & 1ull));
                s[i] = visible ? s[i] * p.scale : -INFINITY;
                mx = fmaxf(mx, s[i]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx);
            const float m_safe = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = expf(m - m_safe);  // 0 while no key was seen
            float w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = expf(s[i] - m_safe);
            l = l * alpha + ((w[0] + w[1]) + (w[2] + w[3]));
            m = m_new;
#pragma unroll
            for (int t = 0; t < ND; ++t) {
                acc[t] *= alpha;
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][t], w[i], acc[t], 0, 0, 0);
            }
            if (careful && special)
                for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = 16 * tile + 4 * k4 + i, rel = key - P;
                        const float weight = __shfl(w[i], 16 * k4 + l16);      // of this key for this lane's query
                        const bool visible = key < S && (rel < 0 || ((mask >> (rel & 63)) & 1ull));
                        const float* vr = static_cast<const float*>(p.v) + base + min(4 * k4 + i, last) * p.g.stride_t + 4 * g;
#pragma unroll
                        for (int t = 0; t < ND; ++t) {
                            const f32x4 x = *reinterpret_cast<const f32x4*>(vr + 16 * t);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (visible && !(fabsf(x[e]) < INFINITY)) acc[t][e] += weight * x[e];
                        }
                    }
        }
    };
    stream(std::false_type{});
    // An entry that is not finite makes the sums of its head dim so in all rows, and they stay so when they are rescaled.
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < ND; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum = fmaf(acc[t][i], 0.f, sum);
    if (__builtin_expect(__any(sum != sum), 0)) stream(std::true_type{});
    if (bad_block && p.err_flag) atomicOr(p.err_flag, SPECVLM_ERR_BAD_BLOCK);
    // merge: acc[t][i] is O^T at head dim 16t + 4g + i, query l16
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (g == 0) {
        s_m[wave][l16] = m;
        s_l[wave][l16] = l;
    }
#pragma unroll
    for (int t = 0; t < ND; ++t) *reinterpret_cast<f32x4*>(&s_acc[wave][l16 * kRow + 16 * t + 4 * g]) = acc[t];
    __syncthreads();
    for (int x = tid; x < 16 * D / 4; x += kF32Waves * 64) {
        const int q = x / (D / 4), d = (x % (D / 4)) * 4;
        if (row0 + q >= n) continue;
        float M = s_m[0][q];
#pragma unroll
        for (int w = 1; w < kF32Waves; ++w) M = fmaxf(M, s_m[w][q]);     // finite: a node always sees itself
        float Z = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) {
            const float f = expf(s_m[w][q] - M);
            Z += s_l[w][q] * f;
            o += *reinterpret_cast<const f32x4*>(&s_acc[w][q * kRow + d]) * f;
        }
        float* orow = static_cast<float*>(p.o) + b * p.o_sb + static_cast<int64_t>(row0 + q) * p.o_sn + h * p.o_sh;
        *reinterpret_cast<f32x4*>(orow + d) = o / Z;
        if (d == 0 && p.lse) p.lse[(static_cast<int64_t>(b) * p.H_q + h) * p.N_max + row0 + q] = M + logf(Z);
    }
}

static ValuParams valu_params(const AttnArgs& a) {
    const specvlm_attn_desc& d = a.d;
    ValuParams p;
    p.g = KvGeom{d.kv_stride_b, d.kv_stride_h, d.kv_stride_t, d.paged ? a.block_table : nullptr,
                 d.max_blocks_per_req, d.num_blocks,
                 d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity};
    p.N_max = d.N_max; p.H_q = d.H_q; p.group = d.H_q / d.H_kv; p.scale = a.scale;
    p.q = a.q; p.k = a.k; p.v = a.v; p.o = a.o; p.lse = a.lse;
    p.q_sb = d.q_stride_b; p.q_sn = d.q_stride_n; p.q_sh = d.q_stride_h;
    p.o_sb = d.o_stride_b; p.o_sn = d.o_stride_n; p.o_sh = d.o_stride_h;
    p.prefix_len = a.prefix_len; p.num_nodes = a.num_nodes; p.parent = a.parent;
    p.err_flag = a.err_flag;
    return p;
}

int32_t launch_attn_f32(const AttnArgs& a) {
    const specvlm_attn_desc& d = a.d;
    const ValuParams p = valu_params(a);
    const dim3 grid((d.N_max + 15) / 16, d.H_q, d.B), block(kF32Waves * 64);
    if (d.D == 64) hipLaunchKernelGGL(attn_f32_kernel<64>, grid, block, 0, a.stream, p);
    else hipLaunchKernelGGL(attn_f32_kernel<128>, grid, block, 0, a.stream, p);
    return check_launch();
}

int32_t launch_attn_valu(const AttnArgs& a) {
    const specvlm_attn_desc& d = a.d;
    const ValuParams p = valu_params(a);
    dim3 grid(d.N_max, d.H_q, d.B), block(256);
    if (d.dtype == SPECVLM_F32) {
        if (d.D == 64) hipLaunchKernelGGL((attn_valu_kernel<float, 64>), grid, block, 0, a.stream, p);
        else hipLaunchKernelGGL((attn_valu_kernel<float, 128>), grid, block, 0, a.stream, p);
    } else {
        if (d.D == 64) hipLaunchKernelGGL((attn_valu_kernel<uint16_t, 64>), grid, block, 0, a.stream, p);
        else hipLaunchKernelGGL((attn_valu_kernel<uint16_t, 128>), grid, block, 0, a.stream, p);
    }
    return check_launch();
}

}  // namespace specvlm
