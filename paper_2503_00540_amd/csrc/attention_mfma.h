// Device pieces shared by the bf16 MFMA attention kernels (attention_bf16.hip, attention_wave.hip):
// register types, the LDS layout of a K or V tile, global -> LDS loads and lane-pair reductions.
#pragma once

#include <type_traits>

#include "common.h"

namespace rekv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 tr4_t;

#define LDS_AS __attribute__((address_space(3)))
#define GLOBAL_AS __attribute__((address_space(1)))

constexpr int BN = 32;        // keys per tile (one MFMA row block of S^T)
constexpr float RESCALE_GAP = 8.0f;  // log2 units the running max may lag before O is rescaled
constexpr int MAX_INDEXED_FRAMES = 1024;   // index entries staged in LDS per workgroup

// Swizzle of the chunk index inside a key row: the two 2-bit fields of (key mod 16) swapped.
// 16 consecutive keys get 16 different values; 4 consecutive keys differ in the upper field.
template <int D>
__device__ inline int swz(int key) {
    return (((key & 3) << 2) | ((key >> 2) & 3)) & (D / 8 - 1);
}

// Blocks are dealt to the 8 XCDs round-robin by hardware; give each XCD one contiguous
// range of logical blocks so that blocks sharing K/V tiles share an L2.
__device__ inline int xcd_remap(int bid, int nb) {
    const int x = bid & 7, per = nb >> 3, rem = nb & 7;
    return x * per + (x < rem ? x : rem) + (bid >> 3);
}

__device__ inline void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// One 16-byte-per-lane load from global memory straight into LDS: lane i's 16 bytes land at
// lds_addr + 16 * i.  Written as asm so that the loads stay invisible to the compiler's
// wait-count bookkeeping: with more than a handful of such loads in a loop it would drain
// all of them before any LDS read.  Ordering is explicit instead.
// The source address is a wave-uniform base plus a 32-bit per-lane byte offset.
// NT marks the load non-temporal: for keys and values that no other workgroup will read again
// (a decode step), so they stream past the caches instead of displacing what is reused.
template <bool NT>
__device__ inline void dma16(const void* base, uint32_t lane_off, uint32_t lds_addr) {
    if (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                     ::"v"(lane_off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     ::"v"(lane_off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory", "m0");
}
__device__ inline uint32_t lds_addr_of(const void* p) {
    return (uint32_t)(uintptr_t)(LDS_AS const void*)p;
}

// Device-scope accesses to the partial results (buffer instructions with the sc1 bit).
constexpr int SC1 = 16;
typedef uint32_t buf4 __attribute__((ext_vector_type(4)));
typedef uint32_t buf2 __attribute__((ext_vector_type(2)));
__device__ inline __amdgpu_buffer_rsrc_t part_buffer(float* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}

template <int I>
using IC = std::integral_constant<int, I>;

// A query's two lanes (lane, lane ^ 32) combine a value without touching LDS:
// v_permlane32_swap hands every lane both halves' values.
__device__ inline float pair_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float pair_sum(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

}  // namespace rekv
