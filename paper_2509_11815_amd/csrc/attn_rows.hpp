// Shared by the bf16 attention kernels whose wavefronts have a key stream of their own (attn_wave.hip, attn_streams.hip):
// parameters, divisions by constants of the call, direct-to-LDS loads of half a tile.
#pragma once
#include <cmath>

#include "attn_common.hpp"

namespace specvlm {

constexpr int kWaveWgs = 4;               // wavefronts per workgroup, one per SIMD, a key stream each
constexpr int kKeys = 32;                 // keys per tile

struct WaveParams {
    KvGeom g;
    int N_max, H_q, H_kv, group, row_blocks, num_splits;
    uint32_t magic_splits, magic_rb, magic_hkv, magic_nmax, magic_nstream;   // divisors, see divide()
    float scale;                // softmax scale
    float c2, tau;              // scale x log2 e; how far a score may lie above the reference before that moves
    const uint16_t *q, *k, *v;
    uint16_t* o;
    float* lse;
    int64_t q_sb, q_sn, q_sh, o_sb, o_sn, o_sh;
    const int32_t *prefix_len, *num_nodes, *parent;
    int32_t* err_flag;
    int32_t* ws_cnt;            // [units][4 owners] arrival tickets, kCounterStride words apart, zero between calls
    // one part per unit and split, or per workgroup (attn_streams.hip)
    unsigned char* ws_acc;      // [parts][owners][..][64 lanes] 16-byte vectors of packed bf16, or of fp32 (attn_streams.hip, `wide`)
    float* ws_ml;               // [parts][block rows][2] (max, sum)
};

// n / d for n * d < 2^31, with m = ceil(2^31 / d) from the host.
__device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t m) { return __umulhi(2 * n, m); }
inline uint32_t divisor(uint32_t d) { return (0x80000000u + d - 1) / d; }

// The parameters of a call whose workgroups take `block_rows` rows of a KV head's group and one of `splits` key ranges
// each.  Workspace: tickets, (max, sum) pairs, partial results.
inline WaveParams wave_params(const AttnArgs& a, int block_rows, int splits, unsigned& workgroups) {
    const specvlm_attn_desc& d = a.d;
    WaveParams p;
    p.g = KvGeom{d.kv_stride_b, d.kv_stride_h, d.kv_stride_t, d.paged ? a.block_table : nullptr,
                 d.max_blocks_per_req, d.num_blocks,
                 d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity};
    p.N_max = d.N_max; p.H_q = d.H_q; p.H_kv = d.H_kv; p.group = d.H_q / d.H_kv;
    p.row_blocks = (p.group * d.N_max + block_rows - 1) / block_rows;
    p.num_splits = splits;
    p.magic_splits = divisor(p.num_splits); p.magic_rb = divisor(p.row_blocks); p.magic_hkv = divisor(p.H_kv);
    p.magic_nmax = divisor(p.N_max); p.magic_nstream = divisor(kWaveWgs * p.num_splits);
    p.scale = a.scale;
    p.c2 = a.scale * kLog2e;
    p.tau = std::fmin(kTau / p.c2, 1e30f);
    p.q = static_cast<const uint16_t*>(a.q);
    p.k = static_cast<const uint16_t*>(a.k);
    p.v = static_cast<const uint16_t*>(a.v);
    p.o = static_cast<uint16_t*>(a.o);
    p.lse = a.lse;
    p.q_sb = d.q_stride_b; p.q_sn = d.q_stride_n; p.q_sh = d.q_stride_h;
    p.o_sb = d.o_stride_b; p.o_sn = d.o_stride_n; p.o_sh = d.o_stride_h;
    p.prefix_len = a.prefix_len; p.num_nodes = a.num_nodes; p.parent = a.parent;
    p.err_flag = a.err_flag;
    workgroups = static_cast<unsigned>(d.B) * d.H_kv * p.row_blocks * p.num_splits;
    unsigned char* ws = static_cast<unsigned char*>(a.workspace);
    p.ws_cnt = reinterpret_cast<int32_t*>(ws);
    p.ws_ml = reinterpret_cast<float*>(ws + kCounterBytes);
    p.ws_acc = ws + kCounterBytes + static_cast<size_t>(workgroups) * block_rows * 8;
    return p;
}

// Four (head size 128) or two (64) consecutive direct-to-LDS loads: the 16 rows of half a tile.  The
// instruction offset advances the LDS and the global address alike, so voff[i] holds what is left.
template <int D>
__device__ __forceinline__ void dma_half(const void* sbase, const uint32_t (&voff)[D / 32], uint32_t lds_dst) {
    if constexpr (D == 128)
        asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %0, %4 nt\n\t"
                     "global_load_lds_dwordx4 %1, %4 offset:1024 nt\n\t"
                     "global_load_lds_dwordx4 %2, %4 offset:2048 nt\n\t"
                     "global_load_lds_dwordx4 %3, %4 offset:3072 nt"
                     : : "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(sbase), "s"(lds_dst) : "memory");
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %0, %2 nt\n\t"
                     "global_load_lds_dwordx4 %1, %2 offset:1024 nt"
                     : : "v"(voff[0]), "v"(voff[1]), "s"(sbase), "s"(lds_dst) : "memory");
}

}  // namespace specvlm
