// Shared by the bf16 tree-verify attention kernels: vector types, direct-to-LDS loads, hand-counted
// waits, device-coherent stores and the counter region's geometry.
#pragma once
#include "common.hpp"

namespace specvlm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// ds_read_b64_tr_b16: inside a block of 16 lanes, lane i receives element i % 4 of the four
// 8-byte rows whose addresses lanes i/4, i/4 + 4, i/4 + 8 and i/4 + 12 pass.
__device__ __forceinline__ s16x4 lds_read_tr16(const unsigned char* generic_lds_addr) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)generic_lds_addr);
}

constexpr int kQRows = 64;          // padded query rows: 4 MFMA column blocks of 16
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kTau = 8.0f;        // log2 of how far a probability may exceed 1 before the reference max moves
constexpr int kCounterStride = 32;    // int32 words from one ticket counter to the next: every counter has a 128-byte line of
                                      // its own, but two of a query block share one above 512 pairs (attn_mfma.hip) (with the counters of eight heads in one line, 256 atomics queued up on it:
                                      // 17.1 -> 16.6 us per call at the 2880-visual-token prefix, 12.4 -> 11.3 us at 576)
static_assert(kCounterBytes == static_cast<size_t>(kMaxSplitHeads) * 4 * kCounterStride * sizeof(int32_t), "counter region");

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2 f = {lo, hi};
    bf16x2 h = __builtin_convertvector(f, bf16x2);      // v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// 16 bytes per lane from global memory straight into LDS at lds_dst + 16*lane (the LDS base
// travels in M0).  The compiler does not see the LDS write: every consumer sits behind
// wait_vmcnt<>() below, which is also a compiler memory barrier.
__device__ __forceinline__ void dma16(const void* gsrc, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :
                 : "v"(gsrc), "s"(lds_dst)
                 : "memory");
}

// Same with a wavefront-uniform base address and a 32-bit lane offset in bytes.
__device__ __forceinline__ void dma16s(const void* sbase, uint32_t voff, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :
                 : "v"(voff), "s"(sbase), "s"(lds_dst)
                 : "memory");
}

// Same, 4 bytes per lane: lds_dst + 4*lane.
__device__ __forceinline__ void dma4(const void* gsrc, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :
                 : "v"(gsrc), "s"(lds_dst)
                 : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// The same for a count that is a constant only after loop unrolling (up to 30).
__device__ __forceinline__ void wait_vmcnt_unrolled(int n) {
    switch (n) {
#define SPECVLM_WAIT_CASE(N) case N: wait_vmcnt<N>(); break;
        SPECVLM_WAIT_CASE(0) SPECVLM_WAIT_CASE(1) SPECVLM_WAIT_CASE(2) SPECVLM_WAIT_CASE(3) SPECVLM_WAIT_CASE(4) SPECVLM_WAIT_CASE(5) SPECVLM_WAIT_CASE(6) SPECVLM_WAIT_CASE(7) SPECVLM_WAIT_CASE(8) SPECVLM_WAIT_CASE(9)
        SPECVLM_WAIT_CASE(10) SPECVLM_WAIT_CASE(11) SPECVLM_WAIT_CASE(12) SPECVLM_WAIT_CASE(13) SPECVLM_WAIT_CASE(14) SPECVLM_WAIT_CASE(15) SPECVLM_WAIT_CASE(16) SPECVLM_WAIT_CASE(17) SPECVLM_WAIT_CASE(18) SPECVLM_WAIT_CASE(19)
        SPECVLM_WAIT_CASE(20) SPECVLM_WAIT_CASE(21) SPECVLM_WAIT_CASE(22) SPECVLM_WAIT_CASE(23) SPECVLM_WAIT_CASE(24) SPECVLM_WAIT_CASE(25) SPECVLM_WAIT_CASE(26) SPECVLM_WAIT_CASE(27) SPECVLM_WAIT_CASE(28) SPECVLM_WAIT_CASE(29)
        SPECVLM_WAIT_CASE(30)
#undef SPECVLM_WAIT_CASE
        default: wait_vmcnt<0>(); break;
    }
}

// Write-through (device-coherent) 16-byte store for data that another workgroup, possibly
// behind another L2, reads in the same kernel.
// (A store of more than 8 bytes reads its data registers for a cycle after it has issued: a
// vector instruction that overwrites them right behind it would corrupt the data of the last
// lanes.  The compiler pads its own stores; it cannot know that this asm is one, hence the s_nop.)
__device__ __forceinline__ void store16_coherent(void* dst, u32x4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(dst), "v"(v) : "memory");
}

__device__ __forceinline__ void store8_coherent(void* dst, u32x2 v) {
    asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1" : : "v"(dst), "v"(v) : "memory");
}

}  // namespace specvlm
