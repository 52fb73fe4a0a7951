// fastmath.hpp -- the FP64 natural logarithm and two-argument arctangent used
// by the assembly and adjoint kernels.
//
// Every influence coefficient needs one logarithm and one arctangent (the
// paper's Sec. 3 names them as the cost of the assembly).  The device
// library's general-purpose versions spend ~150 instructions each on
// extended-precision internals; these spend ~25-30 and stay within 1-2 ulp
// (measured against the host libm in the tests), which is well inside what
// the 1e-10 solution tolerance needs (entry errors up to ~1e-14 relative
// leave Cp within ~1e-11 at N = 256).
//
// log(x), x > 0 normal: x = 2^e m with m in [sqrt(1/2), sqrt(2)); with
// f = m - 1 and s = f / (2 + f), log(m) = 2 atanh(s) = 2s + s R(s^2) where
// R(z) = z (2/3 + 2z/5 + 2z^2/7 + ...), |s| <= 0.172; the bracket is replaced
// by its interpolant of degree 6 at the Chebyshev nodes of [0, 0.02945], which
// leaves 1e-17 of the logarithm.  Since 2s = f - s f,
// log(m) = f - s (f - R): the leading term f is exact and the rounding of the
// small correction barely matters.  e ln2 is added in two pieces, the high
// one with few enough bits that e * LN2_HI is exact (Cody and Waite's
// argument-reduction split; the constants are ln 2 and pi themselves, cut
// into a short head and the remainder).
//
// atan2(y, x): fold to t = min(|x|,|y|) / max(|x|,|y|) in [0, 1], pick the
// nearest centre c = i/16 (i = 0..16), and use atan(t) = atan(c) + atan(u) with
// u = (t - c) / (1 + c t) = (num - c den) / (den + c num) (one division,
// |u| <= 1/32); atan(u) = u + u z P(z), z = u^2, P the interpolant of the
// Taylor series' tail at the Chebyshev nodes of [0, 0.00101] (degree 3, error
// 1e-18 of the result).  Octant and quadrant only change the constant and the
// sign of atan(u): the constants atan(c), pi/2 - atan(c), pi - atan(c) and
// pi/2 + atan(c) come from a table of 4 x 17 doubles in LDS, read by a per-lane
// index.  (With five centres, a series of nine terms, selects for the centre
// and two conditional subtractions an interior entry of the assembly took 110
// vector instructions; it takes 86.)
#pragma once

#include <hip/hip_runtime.h>

namespace panel {

// q = a / b for b of moderate size (no overflow / underflow paths): hardware
// reciprocal, one Newton step on it, and one residual correction of the
// quotient (within 1 ulp).
__device__ __forceinline__ double pdiv(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

namespace fm {
constexpr double kSqrtHalf = 0.7071067811865476;
constexpr double kLn2Hi = 0.6931471803691238;      // ln 2 to 32 significant bits
constexpr double kLn2Lo = 1.9082149292705877e-10;  // ln 2 - kLn2Hi
// Series coefficients, read from constant memory: loaded once per kernel
// into scalar registers, they enter each FMA as a scalar operand (written
// as literals, the compiler keeps them in vector registers and copies one
// into the accumulator of every Horner step).
inline __constant__ double kLogPoly[7] = {0.1461703754879165, 0.1533167403016786, 0.18182890556695602,
                                          0.2222221111514416, 0.2857142862609589, 0.3999999999989924,
                                          0.666666666666667};
inline __constant__ double kAtanPoly[4] = {0.11092769031484487, -0.14285702711480552, 0.19999999997662343,
                                           -0.3333333333333326};
// atan(i/16), pi/2 - atan(i/16), pi - atan(i/16), pi/2 + atan(i/16), i = 0..16
constexpr int kAtanTab = 68;
inline __constant__ double kAtanBase[kAtanTab] = {
    0.0, 0.06241880999595735, 0.12435499454676144, 0.18534794999569476, 0.24497866312686414, 0.3028848683749714,
    0.35877067027057225, 0.4124104415973873, 0.4636476090008061, 0.5123894603107377, 0.5585993153435624,
    0.6022873461349642, 0.6435011087932844, 0.6823165548747481, 0.7188299996216245, 0.7531512809621944,
    0.7853981633974483,
    1.5707963267948966, 1.5083775167989393, 1.446441332248135, 1.3854483767992019, 1.3258176636680326,
    1.2679114584199251, 1.2120256565243244, 1.1583858851975093, 1.1071487177940904, 1.0584068664841588,
    1.0121970114513341, 0.9685089806599324, 0.9272952180016122, 0.8884797719201485, 0.8519663271732721,
    0.8176450458327023, 0.7853981633974483,
    3.141592653589793, 3.079173843593836, 3.017237659043032, 2.9562447035940984, 2.896613990462929,
    2.838707785214822, 2.782821983319221, 2.729182211992406, 2.677945044588987, 2.6292031932790554,
    2.5829933382462307, 2.539305307454829, 2.498091544796509, 2.459276098715045, 2.4227626539681686,
    2.388441372627599, 2.356194490192345,
    1.5707963267948966, 1.633215136790854, 1.695151321341658, 1.7561442767905915, 1.8157749899217608,
    1.873681195169868, 1.9295669970654687, 1.9832067683922838, 2.0344439357957027, 2.0831857871056343,
    2.129395642138459, 2.173083672929861, 2.214297435588181, 2.2531128816696446, 2.289626326416521,
    2.323947607757091, 2.356194490192345};
}  // namespace fm

__device__ __forceinline__ double plog(double x) {
    double m = __builtin_amdgcn_frexp_mant(x);   // [0.5, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool lo = m < fm::kSqrtHalf;
    m = lo ? 2.0 * m : m;
    e = lo ? e - 1 : e;
    const double f = m - 1.0;
    const double s = pdiv(f, 2.0 + f);
    const double z = s * s;
    double R = fm::kLogPoly[0];   // 2/3 + 2z/5 + ...
#pragma unroll
    for (int k = 1; k < 7; ++k) R = fma(R, z, fm::kLogPoly[k]);
    R *= z;
    const double lm = f - s * (f - R);
    const double ef = (double)e;
    return fma(ef, fm::kLn2Hi, fma(ef, fm::kLn2Lo, lm));
}

// The kernel's copy of the arctangent table (LDS, kAtanTab doubles): every
// thread of the workgroup calls it, a barrier follows before the first patan2.
__device__ __forceinline__ void load_atan_table(double *tab) {
    for (int i = threadIdx.x; i < fm::kAtanTab; i += blockDim.x) tab[i] = fm::kAtanBase[i];
}

__device__ __forceinline__ double patan2(double y, double x, const double *tab) {
    const double ax = fabs(x), ay = fabs(y);
    const bool sw = ay > ax, neg = x < 0.0;
    const double num = sw ? ax : ay, den = sw ? ay : ax;
    // nearest centre from an approximate quotient (any centre keeps |u| small)
    const double fi = fmin(__builtin_rint(16.0 * (num * __builtin_amdgcn_rcp(den))), 16.0);
    const double c = 0.0625 * fi;
    const double u = pdiv(fma(-c, den, num), fma(c, num, den));
    const double z = u * u;
    double P = fm::kAtanPoly[0];   // -1/3 + z/5 - ...
#pragma unroll
    for (int k = 1; k < 4; ++k) P = fma(P, z, fm::kAtanPoly[k]);
    const double at = fma(u * z, P, u);
    const double base = tab[(int)fi + (sw ? 17 : 0) + (neg ? 34 : 0)];
    return copysign(base + (sw != neg ? -at : at), y);
}

}  // namespace panel
