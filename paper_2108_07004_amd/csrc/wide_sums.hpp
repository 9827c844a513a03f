// Sums of likelihoods with the exponent range of a double (gfx950), for the fix-up: exponents t in FP32
// as everywhere, split into n + f with n whole and |f| <= 1/2, and 2^n * 2^f summed as doubles (2^f from
// v_exp_f32, n added to the exponent field).  Terms are at most 2^123 and so are their sums, so the
// doubles are 2^kWideShift times the sums: they hold every term down to 2^-1900, no maxima are
// needed and one pass over the points serves all label bits.
#pragma once
#include "device_common.hpp"

namespace dm {

constexpr int kWideShift = 880;

// 2^(t + kWideShift) as a double, t clamped to at least -1900 (the result is then a normal double).
__device__ __forceinline__ double wide_exp2(float t) {
    // 1.5 * 2^23: the sum's low mantissa bits are the nearest whole number, here with the shift added
    constexpr float kMagic = 12582912.0f + (float)kWideShift;
    t = fmaxf(t, -1900.0f);
    const float z = t + kMagic;
    const double e = (double)hw_exp2(t - (z - kMagic));
    const uint64_t u = __builtin_bit_cast(uint64_t, e);
    const uint32_t hi = (uint32_t)(u >> 32) + (__float_as_uint(z) << 20);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | (uint32_t)u);
}

// log2(a) - log2(b) of two sums in range, with exact binary exponents.
__device__ __forceinline__ float wide_log2_ratio(double a, double b) {
    const int ea = __builtin_amdgcn_frexp_exp(a), eb = __builtin_amdgcn_frexp_exp(b);
    const float ma = (float)__builtin_amdgcn_frexp_mant(a), mb = (float)__builtin_amdgcn_frexp_mant(b);
    return (float)(ea - eb) + (hw_log2(ma) - hw_log2(mb));
}

// Both sums (of terms down to 2^-1900) finite and at least 2^-1860: what clamping added, at most 2^13 terms
// (half of 16384 points) of 2^-1900 each, is then below 2^-26 of them.  (With sums accepted down
// to 2^20 times the clamp, LLRs at that end were off by up to 4e-3.)
__device__ __forceinline__ bool wide_ok(double a, double b) {
    return fmin(a, b) >= 0x1p-980 && fmax(a, b) < 0x1p+1020;
}
static_assert(kWideShift - 1860 == -980, "wide_ok's bound");

// MI term of a symbol with m label bits: the sum over all points and the transmitted point's exponent.
__device__ __forceinline__ float wide_mi(int m, double all, float ttx) {
    const int e = __builtin_amdgcn_frexp_exp(all) - kWideShift;
    return finite_term(((float)(m - e) + ttx) - hw_log2((float)__builtin_amdgcn_frexp_mant(all)));
}

}  // namespace dm
