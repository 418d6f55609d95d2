// gf_math.hpp -- double-precision sine/cosine and arctangent for the bounded
// arguments of the SU(2) over-relaxation step, written to keep the register
// footprint and the dependent chain of the sweep kernel small (one wave per
// SIMD runs the step three times a site, so its latency adds to every
// half-sweep whose field fits the caches). Usable on host and device so the
// host-side checks exercise the very code the kernels run.
//
// sincos: argument in [0, 2 pi]. Quadrant reduction x = k pi/2 + r (k =
//   rint(2x/pi), r in [-pi/4, pi/4]) with pi/2 split into a double head and
//   a tail (Cody and Waite's method), each subtracted with one fused
//   multiply-add; then minimax polynomials of sin r (to r^13, error 2^-57.6)
//   and cos r (to r^14, 2^-59.9).
// atan2: the vector (|x|, |y|) is turned by the nearest of 0, pi/4, pi/2, so
//   that the one quotient left is u in [-tan(pi/8), tan(pi/8)]; there atan u
//   is a minimax polynomial to u^23 (relative error 2^-58.5).
// The polynomials (Remez exchange in 50 digits, coefficients rounded to double;
// the errors are those with the rounded coefficients, exactly evaluated) are
// evaluated by Estrin's scheme: their pairs are independent, so the chain is
// a third of Horner's.
#pragma once

#include <hip/hip_runtime.h>

namespace gf {

#define GF_HD __host__ __device__ __forceinline__

constexpr double GF_PI = 3.141592653589793;         // pi rounded to double
constexpr double GF_PI_2 = 1.5707963267948966;      // pi/2 rounded to double
constexpr double GF_PI_2_TAIL = 6.123233995736766e-17;  // pi/2 - GF_PI_2
constexpr double GF_PI_4 = 0.7853981633974483;
constexpr double GF_2_PI = 0.6366197723675814;      // 2/pi
constexpr double GF_TAN_PI_8 = 0.41421356237309515; // sqrt(2) - 1

// Coefficients: sin r = r + r^3 S(r^2), cos r = 1 - r^2 (1/2 - r^2 C(r^2)),
// atan u = u + u^3 A(u^2).
struct TrigTable {
    double S[6], C[6], A[11], tail, two_pi;
};
#define GF_TRIG_VALUES                                                                                   \
    {{-0.16666666666666632, 0.008333333333322418, -0.00019841269829812388,  \
      2.755731369357538e-06, -2.50507583847801e-08, 1.5896811821695718e-10}, \
     {0.0416666666666666, -0.0013888888888874131, 2.4801587289486985e-05,  \
      -2.7557314353781716e-07, 2.087572347809026e-09, -1.1359658797584345e-11}, \
     {-0.333333333333332, 0.1999999999995404, -0.1428571428024414, 0.1111111078590868,  \
      -0.09090897829588034, 0.0769206151073182, -0.06663118902257834, 0.05847997833644728,  \
      -0.050397943118446295, 0.0380769901294441, -0.01792079100108122}, \
     GF_PI_2_TAIL, GF_2_PI}
constexpr TrigTable GF_TRIG_HOST = GF_TRIG_VALUES;
static __constant__ TrigTable GF_TRIG_DEV = GF_TRIG_VALUES;

// The table as the code reads it. On the device it is read through a uniform
// pointer whose origin the compiler cannot see: known constants are
// materialised as pairs of 32-bit moves into vector registers, one pair in
// front of every multiply-add (64 of the 213 vector instructions of a
// step); scalar loads bring them as scalar operands instead.
#ifdef __HIP_DEVICE_COMPILE__
typedef const __attribute__((address_space(4))) TrigTable *TrigPtr;
GF_HD TrigPtr gf_trig() {
    TrigPtr t = (TrigPtr)&GF_TRIG_DEV;
    asm("" : "+s"(t));
    return t;
}
#else
typedef const TrigTable *TrigPtr;
GF_HD TrigPtr gf_trig() { return &GF_TRIG_HOST; }
#endif

// 1/x and 1/sqrt(x) to about 1 ulp for x > 0: the hardware's estimate (2^-24
// or better; the host takes the rounded value instead) and one step of third
// order. Without the range scaling and fix-ups of the general division and
// square root, which the arguments here (quotients in [-1, 1], norms of
// staple quaternions) do not need.
GF_HD double gf_rcp(double x) {
#ifdef __HIP_DEVICE_COMPILE__
    const double r = __builtin_amdgcn_rcp(x);
#else
    const double r = 1.0 / x;
#endif
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

GF_HD double gf_rsqrt(double x) {
#ifdef __HIP_DEVICE_COMPILE__
    const double r = __builtin_amdgcn_rsq(x);
#else
    const double r = 1.0 / sqrt(x);
#endif
    const double e = fma(-(x * r), r, 1.0);
    return fma(r * e, fma(e, 0.375, 0.5), r);
}

// sqrt(x) for finite x >= 0: one correction of x / sqrt(x), rounded as the library's
// (2e6 random normal arguments, the estimate cut to 24 bits: no bit differs); a
// subnormal x to its own spacing. Only 0 needs the clamp, to the smallest positive
// number: with a larger one, smaller arguments would get the root of the clamp.
GF_HD double gf_sqrt(double x) {
    const double y = gf_rsqrt(fmax(x, 4.9406564584124654e-324));
    const double s = x * y;
    return fma(fma(-s, s, x), 0.5 * y, s);
}

GF_HD void gf_sincos(TrigPtr T, double x, double *s, double *c) {
    const double k = rint(x * T->two_pi);
    double r = fma(-k, GF_PI_2, x);
    r = fma(-k, T->tail, r);
    const double z = r * r, z2 = z * z, z4 = z2 * z2;
    const double ps = fma(fma(T->S[5], z, T->S[4]), z4, fma(fma(T->S[3], z, T->S[2]), z2, fma(T->S[1], z, T->S[0])));
    const double pc = fma(fma(T->C[5], z, T->C[4]), z4, fma(fma(T->C[3], z, T->C[2]), z2, fma(T->C[1], z, T->C[0])));
    const double sr = fma(ps * z, r, r);
    const double cr = fma(-fma(-pc, z, 0.5), z, 1.0);
    const int q = (int)k;
    const double sv = (q & 1) ? cr : sr;
    const double cv = (q & 1) ? sr : cr;
    *s = (q & 2) ? -sv : sv;
    *c = ((q + 1) & 2) ? -cv : cv;
}

// atan2(y, x) in [0, pi] for y >= 0; atan2(0, 0) = 0.
GF_HD double gf_atan2_upper(TrigPtr T, double y, double x) {
    const double ax = fabs(x);
    // (ax, y) turned by -0, -pi/4 or -pi/2 (times sqrt 2 for the middle one)
    const bool lo = y <= GF_TAN_PI_8 * ax, hi = ax < GF_TAN_PI_8 * y;
    const double num = lo ? y : (hi ? -ax : y - ax);
    const double den = lo ? ax : (hi ? y : y + ax);
    const double base = lo ? 0.0 : (hi ? GF_PI_2 : GF_PI_4);
    const double d = fmax(den, 1e-300);  // 0 / 0 -> 0
    const double r = gf_rcp(d);
    double u = num * r;
    u = fma(fma(-d, u, num), r, u);
    const double w = u * u, w2 = w * w, w4 = w2 * w2, w8 = w4 * w4;
    const double p01 = fma(T->A[1], w, T->A[0]), p23 = fma(T->A[3], w, T->A[2]);
    const double p45 = fma(T->A[5], w, T->A[4]), p67 = fma(T->A[7], w, T->A[6]);
    const double p89 = fma(T->A[9], w, T->A[8]);
    const double pl = fma(fma(p67, w2, p45), w4, fma(p23, w2, p01));
    const double p = fma(fma(T->A[10], w2, p89), w8, pl);
    const double a = base + fma(p * w, u, u);
    return x < 0.0 ? GF_PI - a : a;
}

// atan2(y, x) in (-pi, pi]; atan2(0, 0) = 0.
GF_HD double gf_atan2(double y, double x) {
    const double a = gf_atan2_upper(gf_trig(), fabs(y), x);
    return y < 0.0 ? -a : a;
}

// Local SU(2) maximiser of Re Tr[g k] for a 2x2 block whose quaternion part
// is b = (b0, b1, b2, b3), i.e. eq. (6) g = q^dagger / |q|, raised to the
// exact principal power omega. With g = (cos phi, n sin phi),
// phi = atan2(|b_vec|, b0) in [0, pi], n = -b_vec / |b_vec|:
// g^omega = (cos(omega phi), n sin(omega phi)). A zero block gives g = 1;
// g = -1 (b_vec = 0, b0 < 0) turns about the third axis.
//
// FULL (double links): |b_vec| and s / |b_vec| each by the product with the
// reciprocal root and one correction. The products alone round once more than a
// root and a quotient do (near the solution 6.5e-17 instead of 5.3e-17 rms at
// omega 1.7); that is left so for float links, where the group element is rounded
// to 6e-8 next.
template <bool FULL = true>
GF_HD void gf_su2_overrelax(const double b[4], double omega, double r[4]) {
    const TrigPtr T = gf_trig();
    const double v2 = fma(b[1], b[1], fma(b[2], b[2], b[3] * b[3]));
    const bool deg = !(v2 > 0.0);
    const double rv = deg ? 0.0 : gf_rsqrt(v2);  // 1 / |b_vec|
    double vn = v2 * rv;
    if (FULL) vn = fma(fma(-vn, vn, v2), 0.5 * rv, vn);
    const double phi = gf_atan2_upper(T, vn, b[0]);
    double s, c;
    gf_sincos(T, omega * phi, &s, &c);
    double f = s * rv;
    if (FULL) f = fma(fma(-vn, f, s), rv, f);
    f = -f;
    r[0] = c;
    r[1] = b[1] * f;
    r[2] = b[2] * f;
    r[3] = deg ? s : b[3] * f;
}

#undef GF_HD

}  // namespace gf
