// exp(-i theta) for the per-point potential factor (FP64).
#pragma once

#include <hip/hip_runtime.h>

namespace hom4d_impl {
namespace dev {

// theta - 2 pi * rint(theta / 2 pi), 2 pi split in three parts (Cody & Waite);
// the first part has 9 significant bits, so q * c1 is exact for |q| < 2^44.
__host__ __device__ __forceinline__ double reduce_2pi(double th) {
    const double inv2pi = 0.15915494309189535;
    const double c1 = 6.28125;
    const double c2 = 0.001935307179586477;
    const double c3 = -1.0033115225336665e-19;
    const double q = rint(th * inv2pi);
    return fma(-q, c3, fma(-q, c2, fma(-q, c1, th)));
}

// exp(-i th): the angle reduced mod 2 pi, then to |s| <= pi / 4 around the nearest
// quarter turn, where the Maclaurin series of sine and cosine to s^17 and s^16 leave less
// than 3e-18.  Within 2e-16 of the exact value of the reduced angle.  The per-point passes
// are bound by these instructions: with it and the estimate-based 1 / r in place of the
// library's sincos (which reduces any argument again), square root and division, 256x128
// complex64 x2+V went 7.62 -> 6.09 ms and y2+V 6.91 -> 5.55, the 64x64 complex128
// plane pass 214 -> 143 us, 96x24 complex128 x2+V 59 -> 52 us.  Past the range of reduce_2pi (|th| of about
// 1e14, where th itself is rounded by 0.01) the result is still a unit number.  An infinite or
// NaN angle has none: it gives NaN, which the norm then shows.
__host__ __device__ __forceinline__ double2 expmi(double th) {
    const double r = reduce_2pi(th);
    const double q = rint(r * 0.6366197723675814);  // 2 / pi
    double s = fma(-q, 6.123233995736766e-17, fma(-q, 1.5707963267948966, r));
    s = fabs(s) >= 1.0 ? 0.0 : s;
    const double z = s * s;
    double ps = 2.8114572543455206e-15;   // 1 / 17!
    ps = fma(ps, z, -7.647163731819816e-13);
    ps = fma(ps, z, 1.6059043836821613e-10);
    ps = fma(ps, z, -2.505210838544172e-08);
    ps = fma(ps, z, 2.7557319223985893e-06);
    ps = fma(ps, z, -1.984126984126984e-04);
    ps = fma(ps, z, 8.333333333333333e-03);
    ps = fma(ps, z, -0.16666666666666666);
    const double sn = fma(s * z, ps, s);
    double pc = 4.779477332387385e-14;    // 1 / 16!
    pc = fma(pc, z, -1.1470745597729725e-11);
    pc = fma(pc, z, 2.08767569878681e-09);
    pc = fma(pc, z, -2.755731922398589e-07);
    pc = fma(pc, z, 2.48015873015873e-05);
    pc = fma(pc, z, -1.388888888888889e-03);
    pc = fma(pc, z, 4.1666666666666664e-02);
    pc = fma(pc, z, -0.5);
    const double cs = fma(pc, z, 1.0);
    const int k = (int)(q == q ? q : 0.0);  // -2 .. 2 in range
    const double c = (k & 1) ? sn : cs, t = (k & 1) ? cs : sn;
    // cos(s + k pi / 2), -sin(s + k pi / 2)
    return make_double2(((k + 1) & 2) ? -c : c, (k & 2) ? t : -t);
}

}  // namespace dev
}  // namespace hom4d_impl
