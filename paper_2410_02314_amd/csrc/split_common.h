// FP32 values as two FP16 halves for the FP16 matrix cores (kernels_split.hip,
// kernels_dsplit.hip): v 2^s = hi + lo 2^-11, hi = f16(v 2^s), lo = f16((v 2^s -
// hi) 2^11).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstring>

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

// an FP16 value's bits (round to nearest even; |f| < 2^15) and the value of such
// bits, both without branches: loops over them become vector code
inline uint16_t f16_bits(float f)
{
    uint32_t u, v;
    std::memcpy(&u, &f, 4);
    const uint32_t sign = (u >> 16) & 0x8000u;
    u &= 0x7FFFFFFFu;
    float t;                                   // below 2^-14: steps of 2^-24, as those of 0.5 + |f|
    std::memcpy(&t, &u, 4);
    t += 0.5f;
    std::memcpy(&v, &t, 4);
    const uint32_t n = ((u + 0xFFFu + ((u >> 13) & 1u)) >> 13) - (112u << 10);
    return (uint16_t)(sign | (u >= 0x38800000u ? n : v - 0x3F000000u));
}
inline float f16_value(uint16_t h)
{
    const uint32_t u = (uint32_t)(h & 0x7FFFu) << 13 | (uint32_t)(h & 0x8000u) << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f * 0x1p112f;                       // the exponents' biases differ by 112
}

// A row of n weights as halves of w up, up the power of two in 2^-60 .. 2^60
// that brings the largest into [2^14, 2^15).  Returns 1 / up; 0 (the row's tiles go
// through plain FP32) where the halves cannot hold it.
inline float split_row(const float *w, int n, uint16_t *hi, uint16_t *lo)
{
    int32_t mb = 0;
    for (int k = 0; k < n; ++k) {
        int32_t u;
        std::memcpy(&u, w + k, 4);
        mb = std::max(mb, u & 0x7FFFFFFF);
    }
    float mx;
    std::memcpy(&mx, &mb, 4);
    if (mb && !(mx >= 0x1p-60f && mx < 0x1p75f)) {
        std::fill(hi, hi + n, (uint16_t)0);
        std::fill(lo, lo + n, (uint16_t)0);
        return 0.f;
    }
    const int e = mb ? std::min(60, std::max(-60, 14 - std::ilogb(mx))) : 0;
    const float up = std::ldexp(1.f, e);
    for (int k = 0; k < n; ++k) {
        const float ws = w[k] * up;
        const uint16_t h = f16_bits(ws);
        hi[k] = h;
        lo[k] = f16_bits((ws - f16_value(h)) * 2048.f);
    }
    return std::ldexp(1.f, -e);
}

}  // namespace dloc
