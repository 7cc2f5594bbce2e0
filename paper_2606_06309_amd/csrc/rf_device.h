// Device helpers shared by the attention kernels.
#pragma once

#include "rf_internal.h"

namespace rf {

// Word 3 of a raw (untyped, stride 0) buffer resource on gfx9-class GPUs.
constexpr int kBufferWord3 = 0x00020000;

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// A pointer every lane holds the same value of, rebuilt from its first lane.
__device__ __forceinline__ void *uniform_ptr(const void *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return reinterpret_cast<void *>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Combine the values of lanes l and l ^ 32 with one VALU swap of the wave
// halves: r[0] holds lanes 0..31 in both halves, r[1] lanes 32..63.
__device__ __forceinline__ float halves_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 16 bytes per lane from a buffer resource straight into LDS: lane l's bytes
// land at dst + 16 l; offsets at or past the resource's range read as zero.
// (Kept out of the kernel templates: the host pass drops the launch stub of a
// template that names this builtin.)
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, lds_void_t *dst, int voffset) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voffset, 0, 0, 0);
}

// At most kLoads of this wave's memory loads still in flight (vmcnt is six bits, split).
template <int kLoads>
__device__ __forceinline__ void wait_loads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (kLoads & 15) | ((kLoads >> 4) << 14));
    asm volatile("" ::: "memory");
}
// Every LDS read of this wave has returned.
__device__ __forceinline__ void wait_lds_reads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
}

}  // namespace rf
