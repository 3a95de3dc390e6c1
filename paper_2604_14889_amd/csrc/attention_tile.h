// Pieces shared by the bf16 matrix-core attention kernels (head_dim 128, 32-token tiles): operand
// layouts, tile loads, rotation and masks.
#pragma once

#include <math.h>

#include "attention.h"
#include "ms_device.h"

namespace ms {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

constexpr int kD = 128;
constexpr int kRows = 64;               // query rows per KV head (padded)
constexpr int kVRowBytes = 320;         // LDS bytes per V row: 256 + 64.  The transposed 8-byte reads of the PV operand
                                        // take 64 bytes of 4 consecutive rows per 32 lanes: with a stride of 16 banks
                                        // (mod 64) those fall on disjoint banks (288 left 22 % of the LDS cycles as conflicts)
constexpr int kQRowBytes = 272;         // LDS bytes per rotated-Q row
constexpr int kVTileBytes = kTile * kVRowBytes;
constexpr float kRescaleThreshold = 24.0f;  // log2 units: P stays below 2^24
constexpr int kPartFloats = 2 * kRows + kRows * kD;  // m[64], l[64], O[128 regs][64 lanes]

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    f32x2_t f = {a, b};
    bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
    return __builtin_bit_cast(uint32_t, h);
}

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;

// sin and cos of an fp32 angle of any size (RoPE angles reach 1e5 rad): the reduction by pi/2 is
// done in fp64 (two-term constant), the kernels on [-pi/4, pi/4] are the single-precision minimax
// polynomials published in the Cephes mathematical library (S. Moshier, sinf / cosf).  About 1e-7 absolute error, far below the bf16 rounding of the rotated rows,
// and much cheaper than the library routine's large-argument path.
__device__ __forceinline__ void sincos_reduced(float x, float* sn, float* cs) {
    const double xd = (double)x;
    const double n = rint(xd * 0.63661977236758134308);
    double r = fma(n, -1.57079632679489655800e+00, xd);
    r = fma(n, -6.12323399573676603587e-17, r);
    const float t = (float)r, t2 = t * t;
    const float sp = t + t * t2 * (-1.6666654611e-1f + t2 * (8.3321608736e-3f + t2 * -1.9515295891e-4f));
    const float cp = 1.0f - 0.5f * t2 + t2 * t2 * (4.166664568298827e-2f + t2 * (-1.388731625493765e-3f + t2 * 2.443315711809948e-5f));
    const int q = (int)n & 3;
    const float s1 = (q & 1) ? cp : sp, c1 = (q & 1) ? sp : cp;
    *sn = (q & 2) ? -s1 : s1;
    *cs = ((q + 1) & 2) ? -c1 : c1;
}

// 16-byte non-temporal global load.
__device__ __forceinline__ uint4 load_stream(const char* p) {
    const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}

// Read-only, wave-uniform control data (the work plan, position ids) is read through the constant
// address space: scalar loads, which return out of order with respect to the vector loads and so do
// not queue behind the tile loads in flight.
template <typename T>
__device__ __forceinline__ T uniform_load(const T* p) {
    return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding
// global load, which would stall the set-up phases on the tile loads already in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Page ids of a tile's two pages.  `tile` may lie past the segment: it is clamped, so that loads
// stay unconditional (a fixed number of loads in flight lets the waits stay partial).
__device__ __forceinline__ void tile_pages(const int* __restrict__ pt, int tile, int n_tiles, int t0, int last_page,
                                           int& pa, int& pb) {
    const int tc = tile < n_tiles ? tile : n_tiles - 1;
    const int pg0 = (t0 >> 4) + 2 * tc;
    pa = __builtin_amdgcn_readfirstlane(pt[pg0 < last_page ? pg0 : last_page]);
    pb = __builtin_amdgcn_readfirstlane(pt[pg0 + 1 < last_page ? pg0 + 1 : last_page]);
}

// K operand of a tile straight from the pool.  Addresses are a uniform base plus a 32-bit byte
// offset per lane (page_bytes * page id + lane part), which keeps the per-lane address state to one
// register; layer pools of 4 GiB and more take the kBigPool build below.
template <bool kBigPool>
__device__ __forceinline__ void load_k(uint4 (&k)[8], const char* __restrict__ pool, int pa, int pb,
                                       uint32_t page_bytes, uint32_t lane_off_k, int lane) {
    if (!kBigPool) {
        const uint32_t off = (uint32_t)((lane & 16) ? pb : pa) * page_bytes + lane_off_k;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) k[kk] = *reinterpret_cast<const uint4*>(pool + off + 32 * kk);
    } else {
        // layer pools of 4 GiB and more: the page's base is a 64-bit (wave-uniform) address, the
        // half-waves pick theirs, the lane part stays a 32-bit offset
        const char* base_a = pool + (size_t)(uint32_t)pa * page_bytes;
        const char* base_b = pool + (size_t)(uint32_t)pb * page_bytes;
        const char* base = (lane & 16) ? base_b : base_a;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) k[kk] = *reinterpret_cast<const uint4*>(base + lane_off_k + 32 * kk);
    }
}

// V rows of a tile: tokens 4 rr + lane / 16 of page a (rr < 4) and of page b.  V is read exactly once
// per call: streaming (non-temporal) loads keep it out of the caches.
template <bool kBigPool>
__device__ __forceinline__ void load_v(uint4 (&v)[8], const char* __restrict__ pool, int pa, int pb,
                                       uint32_t page_bytes, uint32_t lane_off_v) {
    if (kBigPool) {
        const char* base_a = pool + (size_t)(uint32_t)pa * page_bytes;
        const char* base_b = pool + (size_t)(uint32_t)pb * page_bytes;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) v[rr] = load_stream(base_a + lane_off_v + 4 * rr * kD * 2);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) v[4 + rr] = load_stream(base_b + lane_off_v + 4 * rr * kD * 2);
        return;
    }
    const uint32_t oa = (uint32_t)pa * page_bytes + lane_off_v, ob = (uint32_t)pb * page_bytes + lane_off_v;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) v[rr] = load_stream(pool + oa + 4 * rr * kD * 2);
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) v[4 + rr] = load_stream(pool + ob + 4 * rr * kD * 2);
}

// Accumulator i of a lane holds token 8 (i / 4) + 4 (lane / 32) + i % 4 of the tile.
__device__ __forceinline__ void mask_tail(f32x16_t& s, int valid, int hf) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + 4 * hf + (i & 3) >= valid) s[i] = -INFINITY;
}

// Visibility of the in-flight tile (token j = in-flight query/key j): a row sees tokens below `lim`
// and token `self` (lim = min(ctx, n_q), self = its own query index; padding rows: lim 0, self 0).
__device__ __forceinline__ void mask_inflight(f32x16_t& s, int lim, int self, int hf) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int tok = 8 * (i >> 2) + 4 * hf + (i & 3);
        s[i] = (tok < lim || tok == self) ? s[i] : -INFINITY;
    }
}

}  // namespace ms
