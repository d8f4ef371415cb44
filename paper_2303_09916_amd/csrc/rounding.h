// Correctly rounded square root, reciprocal and quotient without the compiler's handling
// of denormal and extreme arguments: the hardware estimate and one residual step each
// (Markstein).  Device code.  Private to the library.
//
// For arguments in kNormalLo..kNormalHi (a quotient also wants one there).  Root and
// reciprocal are correctly rounded for every float in [2^-96, 64), the quotient for all of
// 1.7e10 pairs tried; rsqrtf is the bare estimate there.  tests/rounding_check.hip goes
// over every float and 2^30 pairs.  41 to 101 cycles of one wave become 9 to 40.
#pragma once

#include <hip/hip_runtime.h>

namespace dsdp {

constexpr float kNormalLo = 0x1p-80f, kNormalHi = 64.0f;
__device__ __forceinline__ bool in_normal(float x)
{
    return __float_as_uint(x) - __float_as_uint(kNormalLo) < __float_as_uint(kNormalHi) - __float_as_uint(kNormalLo);
}
// whether any active lane's x lies outside the range
__device__ __forceinline__ bool any_odd(float x) { return __builtin_amdgcn_ballot_w64(!in_normal(x)) != 0; }
__device__ __forceinline__ float sqrt_normal(float x)
{
#pragma clang fp contract(off)
    const float y = __builtin_amdgcn_rsqf(x), g = x * y;
    return fmaf(fmaf(-g, g, x), 0.5f * y, g);
}
__device__ __forceinline__ float rcp_normal(float b)
{
#pragma clang fp contract(off)
    const float y = __builtin_amdgcn_rcpf(b);
    return fmaf(fmaf(-b, y, 1.0f), y, y);
}
__device__ __forceinline__ float div_normal(float a, float b)
{
#pragma clang fp contract(off)
    const float y = rcp_normal(b);
    const float q = a * y;
    return fmaf(fmaf(-b, q, a), y, q);
}

}  // namespace dsdp
