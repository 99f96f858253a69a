// FP32 values as two FP16 halves for the FP16 matrix cores (kernels_split.hip,
// kernels_dsplit.hip): v 2^s = hi + lo 2^-11, hi = f16(v 2^s), lo = f16((v 2^s -
// hi) 2^11).
#pragma once
#include "dloc_internal.h"

namespace dloc {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_h2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, (h2{(_Float16)a, (_Float16)b}));
}

// largest |v| over the wave's lanes (v >= 0), in every lane
__device__ __forceinline__ float wave_max(float v)
{
    int x = __float_as_int(v);           // non-negative floats order as integers
#define DLOC_DPP_MAX(ctrl, rmask) x = max(x, __builtin_amdgcn_update_dpp(0, x, ctrl, rmask, 0xF, false))
    DLOC_DPP_MAX(0x111, 0xF);            // row_shr:1
    DLOC_DPP_MAX(0x112, 0xF);            // row_shr:2
    DLOC_DPP_MAX(0x114, 0xF);            // row_shr:4
    DLOC_DPP_MAX(0x118, 0xF);            // row_shr:8
    DLOC_DPP_MAX(0x142, 0xA);            // row_bcast:15 into rows 1, 3
    DLOC_DPP_MAX(0x143, 0xC);            // row_bcast:31 into rows 2, 3
#undef DLOC_DPP_MAX
    return __int_as_float(__builtin_amdgcn_readlane(x, 63));
}

// four values' halves to LDS: hi at d, lo at d + lo_off
__device__ __forceinline__ void split_store(const v4f &v, int lo_off, char *d)
{
    uint2 hi{pack_h2(v[0], v[1]), pack_h2(v[2], v[3])};
    asm("" : "+v"(hi.x), "+v"(hi.y));                  // (one conversion for hi and for v - hi)
    const h2 a0 = __builtin_bit_cast(h2, hi.x), a1 = __builtin_bit_cast(h2, hi.y);
    const uint2 lo{pack_h2(fmaf((float)a0[0], -2048.f, v[0] * 2048.f), fmaf((float)a0[1], -2048.f, v[1] * 2048.f)),
                   pack_h2(fmaf((float)a1[0], -2048.f, v[2] * 2048.f), fmaf((float)a1[1], -2048.f, v[3] * 2048.f))};
    *reinterpret_cast<uint2 *>(d) = hi;
    *reinterpret_cast<uint2 *>(d + lo_off) = lo;
}

// The exponent s that brings a largest magnitude of bits mb into [2^14, 2^15), so
// that values down to 2^-28 of it keep 22 bits (below, hi is an FP16 subnormal and
// the pair is off by 2^-36 / 2^14 = 2^-50 of it at most); within +-60.
__device__ __forceinline__ int split_exp(uint32_t mb)
{
    const int e = (int)(mb >> 23) - 127;               // floor(log2), -127 for zero and subnormals
    return min(60, max(-60, 14 - e));
}
// ... and whether the halves cannot hold values of that magnitude
__device__ __forceinline__ bool split_misfit(uint32_t mb)
{
    const int e = (int)(mb >> 23) - 127;
    return (e >= 75) | ((e < -65) & (mb != 0));
}

// ---- weights as pairs (kernels_split.hip: k_pack_pairs) ----
// A convolution's weights [cout][ld][taps], its first cin inputs of them, into the
// kernels' MFMA fragments; scale [cout] takes the rows' powers of two (all 0: the
// halves cannot hold the rows' magnitudes, every tile goes through plain FP32);
// raw (or null) a copy of the weights.  K is taken in groups of 16 or 32 channels
// (group; 1x1: 16).  All pointers are device memory.
struct PairJob {
    const float *w;
    int cout, cin, ld, taps, group;
    void *dst;
    float *scale, *raw;
};
// weight steps (32 values of K) of one group
__host__ __device__ constexpr int pair_steps(int taps, int group) { return taps == 1 ? 1 : group == 32 ? 9 : 5; }
inline size_t pair_packed_bytes(int cout, int cin, int taps, int group)
{
    return (size_t)(cin / group) * pair_steps(taps, group) * (cout / 16) * 2048;
}
hipError_t launch_pack_pairs(const PairJob *jobs, int n, hipStream_t s);

}  // namespace dloc
