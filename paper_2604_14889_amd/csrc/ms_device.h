// Device-side element helpers: storage types and conversions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ms {

// bfloat16 storage: the upper 16 bits of an IEEE-754 binary32.
struct bf16_t {
    uint16_t bits;
};

__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits) { return __uint_as_float(bits << 16); }

// Round to nearest, ties to even; NaN stays NaN.
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Sum over a workgroup of kThreads threads; every thread gets the total.  red: kThreads / 64 floats of LDS.
template <int kThreads>
__device__ __forceinline__ float block_sum(float x, float* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = x;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) t += red[i];
    return t;
}

// 64 lanes x 16 bytes from base + voff into LDS at lds .. lds + 1024, lane order.
template <bool kStream>
__device__ __forceinline__ void load_lds_1k(uint32_t lds, uint32_t voff, const void* base) {
    if (kStream) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
// An address that is the same in every lane, in scalar registers.
__device__ __forceinline__ const char* wave_uniform(const char* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char*)(((uint64_t)hi << 32) | lo);
}
template <int kN>
__device__ __forceinline__ void wait_loads() {   // at most kN of this wave's loads are still on their way; its LDS reads are done
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kN) : "memory");
}

__device__ __forceinline__ void wave_lds_fence() {   // LDS operations of a wave are carried out in order: only the compiler has to keep them so
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// The larger of x and its value 16 or 32 lanes away (lane ^ 16, lane ^ 32): a row or half swap in the vector unit, no trip through LDS.
__device__ __forceinline__ float max_across_16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_across_32(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Row kernels with a norm (one workgroup per row, the row held in registers between the two passes):
// threads per row and 8-element chunks per thread; rows of up to 8192 elements.
constexpr int kNormThreads = 512;
constexpr int kNormMaxPerThread = 2;

__device__ __forceinline__ float to_float(float x) { return x; }
__device__ __forceinline__ float to_float(bf16_t x) { return bf16_bits_to_float(x.bits); }

template <typename T>
__device__ __forceinline__ T from_float(float f);
template <>
__device__ __forceinline__ float from_float<float>(float f) {
    return f;
}
template <>
__device__ __forceinline__ bf16_t from_float<bf16_t>(float f) {
    bf16_t r;
    r.bits = float_to_bf16_bits(f);
    return r;
}

}  // namespace ms
