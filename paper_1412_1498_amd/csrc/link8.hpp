// link8.hpp -- 8-real storage of SU(3) links (the paper's most compressed
// link format): a link is kept as U01, U02, U10 (three complex numbers) and
// the phases of U00 and U20 (coded as below). Usable on host and device,
// so host-side checks run the very code the kernels run.
//
// Reconstruction, from unitarity and det U = 1 (U^dagger = adj U, i.e. each
// element is the complex conjugate of its cofactor):
//   n2  = |U01|^2 + |U02|^2            (= 1 - |U00|^2, row 0 is a unit vector)
//   U00 = sqrt(1 - n2) e^{i phase00}
//   U20 = sqrt(n2 - |U10|^2) e^{i phase20}   (column 0 is a unit vector)
//   U11 = -(conj(U00) U01 U10 + conj(U02) conj(U20)) / n2
//   U12 =  (conj(U01) conj(U20) - conj(U00) U02 U10) / n2
//   U21 = -conj(U00 U12 - U02 U10)
//   U22 =  conj(U00 U11 - U01 U10)
// The divisor is formed as |U01|^2 + |U02|^2 rather than 1 - |U00|^2: near
// the unit matrix numerator and divisor are then products of small numbers,
// held to full relative precision. What remains near 1 is that the stored
// reals fix an exact SU(3) matrix, so a link that is SU(3) only to O(u) (u
// the unit roundoff of the storage precision) is moved to it: a link eps
// away from 1 moves by about u/eps. For float storage this stays at the
// float rounding of the link itself (measured below 3e-6 down to 1e-6 from
// 1); in double it is 2e-9 at 1e-6 from 1. Where |U00| or |U20| is tiny, the
// square roots lose digits: errors of about u/|U00|, u/|U20|.
//
// Row 0 without off-diagonal part (U01 = U02 = 0 exactly, n2 = 0; the unit
// matrix is one): then |U00| = 1, so U10 = U20 = 0, and the divisor above
// vanishes. The lower 2x2 block B is unitary with det B = conj(U00), i.e.
// B = [[a, b], [-conj(U00) conj(b), conj(U00) conj(a)]] with |a|^2 + |b|^2
// = 1. The U10 slot, free in this case, then holds a = U11, and the phase
// code of U20 is replaced by that of b = U12 (|b| = sqrt(1 - |a|^2)); the
// decoder recognises the case by n2 = 0 and the link is held exactly like
// any other.
//
// The phases are not stored as angles but as a rational code of the unit
// complex number w = z/|z| (no trigonometry either way): with
// t = Im w / (1 + |Re w|) in [-1, 1] (the tangent of half the angle
// between w and the real axis on its side), the stored value is t if
// Re w >= 0, else 2 - t (t >= 0) or -2 - t (t < 0). Decoding: the branch is
// |p| > 1, t = copysign(2 - |p|, p) there, and |Re w| = (1 - t^2)/(1 + t^2),
// Im w = 2t/(1 + t^2). z = 0 is stored as 4 and decodes to 0, so an element
// that is exactly zero comes back exactly zero whatever rounding its
// modulus, a square root of a difference, suffers.
#pragma once

#include <hip/hip_runtime.h>

#include "gf_math.hpp"

namespace gf {

#define GF_HD __host__ __device__ __forceinline__

// Reciprocal and square root. In float on the GPU these are the hardware
// instructions (about 1 ulp) rather than the correctly rounded sequences:
// the format's own rounding (a few ulp) dominates, and the exact sequences
// made the float 8-real sweep instruction-bound. In double they are gf_rcp
// and gf_sqrt, which round like the general operations but skip their range
// scaling: a site's 8 links take 40 reciprocals and 32 square roots, half of
// the double sweep's instructions in their general form. gf_sqrt takes every
// finite x >= 0, subnormal ones too (squares of elements below 1e-154). Float
// host code uses the general operations.
template <typename R> GF_HD R link8_rcp(R x) {
    if constexpr (sizeof(R) == 8) return gf_rcp(x);
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (sizeof(R) == 4) return __builtin_amdgcn_rcpf(x);
#endif
    return R(1) / x;
}
template <typename R> GF_HD R link8_sqrt(R x) {
    if constexpr (sizeof(R) == 8) return gf_sqrt(x);
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (sizeof(R) == 4) return __builtin_amdgcn_sqrtf(x);
#endif
    return sqrt(x);
}

// a b + c d: one multiply and one FMA in double; in float both products are
// rounded first (a fused form is as exact, but fields stored with it drift
// from fields stored without it, by up to 1e-3 at the links with tiny |U00|).
template <typename R>
GF_HD R link8_dot(R a, R b, R c, R d) {
    if constexpr (sizeof(R) == 8) return fma(a, b, c * d);
    else return a * b + c * d;
}

template <typename R>
GF_HD R link8_phase_code(R re, R im) {
    const R m = link8_sqrt<R>(link8_dot<R>(re, re, im, im));
    if (!(m > R(0))) return R(4);  // z = 0: a code outside [-2, 2] that decodes to 0
    const R t = im * link8_rcp<R>(m + fabs(re));
    return re >= R(0) ? t : (t >= R(0) ? R(2) - t : R(-2) - t);
}

// unit complex number (c, s) of a phase code; (0, 0) for the code of 0
template <typename R>
GF_HD void link8_phase_decode(R p, R *c, R *s) {
    const bool zero = fabs(p) > R(3);
    const bool neg = fabs(p) > R(1);
    const R t = neg ? copysign(R(2) - fabs(p), p) : p;
    const R d = link8_rcp<R>(link8_dot<R>(t, t, R(1), R(1)));
    const R ac = link8_dot<R>(-t, t, R(1), R(1)) * d;
    *s = zero ? R(0) : R(2) * t * d;
    *c = zero ? R(0) : (neg ? -ac : ac);
}

// Where the n2 = 0 case is dealt with. In double by selects in place. In float
// (link8_late) at the end, behind a branch of the whole wave (link8_any; on the
// host, of the one link): what it takes, two elements more of the rotated link,
// a phase and the selects, is a tenth of the instructions of the sweep, which
// they bound. With the same bits, a sweep and a tenth of a check in float:
// 40x40x40x24 181 -> 174 us, 48^4 560 -> 534, 32^4 127 -> 121. In double a
// one-lane site has no registers left for the branches.
template <typename R> constexpr bool link8_late = sizeof(R) == 4;

GF_HD bool link8_any(bool deg) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ballot_w64(deg) != 0;
#else
    return deg;
#endif
}

// The four stored complex values of a 3x3 link (re[9], im[9], element (r, c)
// at 3r + c): U01, U02, U10, (phase code of U00, phase code of U20).
// When U01 = U02 = 0, the third value is U11 and the second phase code is
// that of U12 instead (see above); the two are used, and by the compiler
// formed, only behind that branch.
template <typename R>
GF_HD void link8_compress(const R *re, const R *im, R *sre, R *sim) {
    const bool deg = re[1] == R(0) && im[1] == R(0) && re[2] == R(0) && im[2] == R(0);
    R vr = re[3], vi = im[3];
    if constexpr (link8_late<R>) {
        R wr = re[6], wi = im[6];
        if (link8_any(deg)) {
            vr = deg ? re[4] : vr; vi = deg ? im[4] : vi;
            wr = deg ? re[5] : wr; wi = deg ? im[5] : wi;
        }
        sre[3] = link8_phase_code<R>(re[0], im[0]);
        sim[3] = link8_phase_code<R>(wr, wi);
    } else {
        vr = deg ? re[4] : vr; vi = deg ? im[4] : vi;
        sre[3] = link8_phase_code<R>(re[0], im[0]);
        sim[3] = deg ? link8_phase_code<R>(re[5], im[5]) : link8_phase_code<R>(re[6], im[6]);
    }
    sre[0] = re[1]; sim[0] = im[1];
    sre[1] = re[2]; sim[1] = im[2];
    sre[2] = vr; sim[2] = vi;
}

// c2 = -conj(a1 b3 - a3 b1), c3 = conj(a1 b2 - a2 b1) from rows 0 and 1
template <typename R>
GF_HD void link8_row2(R *re, R *im) {
    const R a1r = re[0], a1i = im[0], a2r = re[1], a2i = im[1], a3r = re[2], a3i = im[2];
    const R b1r = re[3], b1i = im[3], b2r = re[4], b2i = im[4], b3r = re[5], b3i = im[5];
    const R x2r = link8_dot<R>(a1r, b3r, -a1i, b3i) - link8_dot<R>(a3r, b1r, -a3i, b1i);
    const R x2i = link8_dot<R>(a1r, b3i, a1i, b3r) - link8_dot<R>(a3r, b1i, a3i, b1r);
    const R x3r = link8_dot<R>(a1r, b2r, -a1i, b2i) - link8_dot<R>(a2r, b1r, -a2i, b1i);
    const R x3i = link8_dot<R>(a1r, b2i, a1i, b2r) - link8_dot<R>(a2r, b1i, a2i, b1r);
    re[7] = -x2r; im[7] = x2i;
    re[8] = x3r; im[8] = -x3i;
}

template <typename R>
GF_HD void link8_reconstruct(const R *sre, const R *sim, R *re, R *im) {
    const R a2r = sre[0], a2i = sim[0], a3r = sre[1], a3i = sim[1];
    const R n2 = link8_dot<R>(a2r, a2r, a2i, a2i) + link8_dot<R>(a3r, a3r, a3i, a3i);
    const bool deg = !(n2 > R(0));         // U01 = U02 = 0: the slot holds U11
    const bool now = !link8_late<R> && deg;
    const R sl = link8_dot<R>(sre[2], sre[2], sim[2], sim[2]);
    const R b1r = now ? R(0) : sre[2], b1i = now ? R(0) : sim[2];
    R s, c;
    link8_phase_decode<R>(sre[3], &c, &s);
    const R m1 = link8_sqrt<R>(fmax(R(1) - n2, R(0)));
    const R a1r = m1 * c, a1i = m1 * s;
    link8_phase_decode<R>(sim[3], &c, &s);
    // |U20| in general; |U12| = sqrt(1 - |U11|^2) in the n2 = 0 case
    const R m3 = link8_sqrt<R>(fmax((now ? R(1) : n2) - sl, R(0)));
    const R zr = m3 * c, zi = m3 * s;
    const R c1r = now ? R(0) : zr, c1i = now ? R(0) : zi;
    // conj(a1) a2 b1, conj(a1) a3 b1
    const R pr = link8_dot<R>(a1r, a2r, a1i, a2i), pi = link8_dot<R>(a1r, a2i, -a1i, a2r);   // conj(a1) a2
    const R qr = link8_dot<R>(a1r, a3r, a1i, a3i), qi = link8_dot<R>(a1r, a3i, -a1i, a3r);   // conj(a1) a3
    const R t1r = link8_dot<R>(pr, b1r, -pi, b1i), t1i = link8_dot<R>(pr, b1i, pi, b1r);
    const R t2r = link8_dot<R>(qr, b1r, -qi, b1i), t2i = link8_dot<R>(qr, b1i, qi, b1r);
    // conj(a3) conj(c1) = conj(a3 c1), conj(a2) conj(c1) = conj(a2 c1)
    const R u3r = link8_dot<R>(a3r, c1r, -a3i, c1i), u3i = -link8_dot<R>(a3r, c1i, a3i, c1r);
    const R u2r = link8_dot<R>(a2r, c1r, -a2i, c1i), u2i = -link8_dot<R>(a2r, c1i, a2i, c1r);
    const R inv = link8_rcp<R>(now ? R(1) : n2);
    re[0] = a1r; im[0] = a1i;
    re[1] = a2r; im[1] = a2i;
    re[2] = a3r; im[2] = a3i;
    re[3] = b1r; im[3] = b1i;
    // n2 = 0: U11 from the slot, U12 from its phase code and modulus
    re[4] = now ? sre[2] : -(t1r + u3r) * inv; im[4] = now ? sim[2] : -(t1i + u3i) * inv;
    re[5] = now ? zr : (u2r - t2r) * inv; im[5] = now ? zi : (u2i - t2i) * inv;
    re[6] = c1r; im[6] = c1i;
    if (link8_late<R> && link8_any(deg)) {
        const R m = link8_sqrt<R>(fmax(R(1) - sl, R(0)));
        re[3] = deg ? R(0) : re[3]; im[3] = deg ? R(0) : im[3];
        re[4] = deg ? sre[2] : re[4]; im[4] = deg ? sim[2] : im[4];
        re[5] = deg ? m * c : re[5]; im[5] = deg ? m * s : im[5];
        re[6] = deg ? R(0) : re[6]; im[6] = deg ? R(0) : im[6];
    }
    link8_row2<R>(re, im);
}

#undef GF_HD

}  // namespace gf
