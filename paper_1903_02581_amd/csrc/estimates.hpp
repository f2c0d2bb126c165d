// FP64 reciprocal and reciprocal square root from the hardware estimates: two Newton
// steps bring their 2^-24 or better to within an ulp or two, in 5 and 9 instructions
// where the correctly rounded library forms take several times that.
#pragma once

#include <hip/hip_runtime.h>

namespace hom4d_impl {
namespace dev {

// 1 / sqrt(x) for normal x > 0
__device__ __forceinline__ double rsqrt_of(double x) {
    const double h = 0.5 * x;
    double r = __builtin_amdgcn_rsq(x);
    r *= fma(-h * r, r, 1.5);
    r *= fma(-h * r, r, 1.5);
    return r;
}
// 1 / x for normal x
__device__ __forceinline__ double rcp_of(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

}  // namespace dev
}  // namespace hom4d_impl
