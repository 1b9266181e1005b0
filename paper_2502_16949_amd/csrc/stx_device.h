// Device-side helpers shared by the kernels: one-workgroup scans and sub-wavefront reductions.
// gfx950 only (64-lane wavefronts).
//
// No kernel here passes data between workgroups of one launch: on this multi-die GPU that needs a
// device-scope release/acquire per workgroup, i.e. an L2 write-back each, which costs far more than
// the extra kernel launch that a grid-wide dependency is turned into instead.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define STX_CONST_AS __attribute__((address_space(4)))      // uniform loads from here are scalar loads

namespace stx {

// Wavefront-uniform values (kernel arguments) that are to be in scalar registers here.  Argument loads return in no order, so
// each wait is for all of them; side by side they cost one.
template <class... T>
__device__ __forceinline__ void together(const T... v) { (..., [](const T x) { asm volatile("" ::"s"(x)); }(v)); }
#define STX_TOGETHER(...) stx::together(__VA_ARGS__)

// Inclusive prefix sum of one value per lane across a wavefront, by data-parallel moves between lanes (all lanes active).
__device__ inline int32_t wave_inclusive_scan(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // from 1, 2, 4 and 8 lanes below in a row of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // the last lane of rows 0 and 2 into rows 1 and 3 ...
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // ... and lane 31 into rows 2 and 3
    return v;
}

// Exclusive prefix sum of one value per thread across a 256-thread workgroup; *total (shared or
// register, may be null) receives the sum.  All 256 threads must call it.  Two barriers; with every doubling of the
// distance a round through LDS, as it was, sixteen: 1.0 us of a scatter pass's 9.1.
__device__ inline int32_t block_exclusive_scan(int32_t v, int32_t *total)
{
    __shared__ int32_t s_wave[4];
    const int w = threadIdx.x >> 6;
    const int32_t incl = wave_inclusive_scan(v);
    __syncthreads();   // protect s_wave against a previous use
    if ((threadIdx.x & 63) == 63) s_wave[w] = incl;
    __syncthreads();
    int32_t before = 0, sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int32_t t = s_wave[u];
        before += u < w ? t : 0;
        sum += t;
    }
    if (total) *total = sum;
    return before + incl - v;
}

// The lanes of the wavefront (among those with `valid`) whose digit equals this lane's: one ballot per bit of the
// digit, and per lane an exclusive-nor of the ballot with the lane's own bit spread over a word.
__device__ inline uint64_t digit_class_mask(int dgt, bool valid, int bits)
{
    const uint64_t v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        if (bit < bits) {   // uniform
            const uint32_t x = (uint32_t)(-(int32_t)((dgt >> bit) & 1));   // all ones when the lane's bit is set
            const uint64_t bm = __ballot(x != 0u);
            lo &= ~((uint32_t)bm ^ x);
            hi &= ~((uint32_t)(bm >> 32) ^ x);
        }
    }
    return (uint64_t)hi << 32 | lo;
}

// Sum over the LPR consecutive lanes that share a row (LPR a power of two <= 64, groups aligned).
// Butterfly: every lane of the group ends with the same bits.
template <int LPR>
__device__ inline float group_sum(float v)
{
#pragma unroll
    for (int m = LPR / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, LPR);
    return v;
}

// Streaming variants: data that is read or written once and not needed in cache afterwards.
typedef float stx_f4 __attribute__((ext_vector_type(4)));
__device__ inline float4 ld4_stream(const float *p)
{
    stx_f4 t = __builtin_nontemporal_load(reinterpret_cast<const stx_f4 *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ inline void st4_stream(float *p, float4 v)
{
    stx_f4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<stx_f4 *>(p));
}
__device__ inline float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ inline void st4(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }

}  // namespace stx
