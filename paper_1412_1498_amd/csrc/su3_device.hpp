// su3_device.hpp -- what the gfx950 kernels of libgf share: sums across the
// lanes of a site and of a wave in registers, link loads and stores in the
// even/odd element-major layout, and Gram-Schmidt reunitarisation.
#pragma once

#include <hip/hip_runtime.h>

#include "gf_internal.hpp"
#include "gf_math.hpp"
#include "link8.hpp"

namespace gf {

template <typename R> struct V2;
template <> struct V2<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct V2<double> { typedef double type __attribute__((ext_vector_type(2))); };

// x of lane l gets lane l ^ M's value (both lanes active): M < 16 by DPP
// moves within rows of 16 lanes (quad permutations, and for 4 the mirror
// image of each half row, turned back quad by quad).
template <int M>
__device__ __forceinline__ int dpp_xor(int x) {
    static_assert(M == 1 || M == 2 || M == 4 || M == 8, "within a row");
    if constexpr (M == 1) return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);       // quad_perm 1 0 3 2
    else if constexpr (M == 2) return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);  // quad_perm 2 3 0 1
    else if constexpr (M == 8) return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true); // row_ror 8
    else  // i -> 7 - i -> i ^ 4
        return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
}

// v of this lane plus v of lane ^ M, in registers: a shuffle through the LDS
// crossbar is a trip to the one unit that all waves of the CU share, 72 of
// them a site at four lanes. A sweep and a check with shuffles and without:
// double 4^4 22.2 -> 20.5 us, 12^4 28.2 -> 26.4, float 16^4 32.3 -> 30.4,
// SU(4) double 8^4 31.7 -> 28.7; nothing from 22x18x26x30 on, where memory
// bounds.
template <int M>
__device__ __forceinline__ double xor_sum(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
    auto join = [](unsigned l, unsigned h) {
        return __builtin_bit_cast(double, (unsigned long long)h << 32 | l);
    };
    if constexpr (M < 16) {
        return v + join((unsigned)dpp_xor<M>((int)lo), (unsigned)dpp_xor<M>((int)hi));
    } else {
        // both halves (or row pairs) of v side by side: the sum of the two is
        // v + v(lane ^ M) in either order
        const auto l = M == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                               : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = M == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                               : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return join(l[0], h[0]) + join(l[1], h[1]);
    }
}

// Sum over a wave by the fixed butterfly 32, 16, .., 1 (every lane gets it).
__device__ __forceinline__ double wave_sum(double v) {
    v = xor_sum<32>(v);
    v = xor_sum<16>(v);
    v = xor_sum<8>(v);
    v = xor_sum<4>(v);
    v = xor_sum<2>(v);
    return xor_sum<1>(v);
}

// Sum over the LPS neighbouring lanes of a site, by 1, 2, 4.
template <int LPS>
__device__ __forceinline__ double site_sum(double v) {
    if constexpr (LPS >= 2) v = xor_sum<1>(v);
    if constexpr (LPS >= 4) v = xor_sum<2>(v);
    if constexpr (LPS >= 8) v = xor_sum<4>(v);
    return v;
}

// Global-address-space views: a uniform (scalar) base pointer plus a 32-bit
// per-lane byte offset lets the compiler emit global_load/store with an SGPR
// base instead of 64-bit flat addresses per lane.
typedef __attribute__((address_space(1))) char gchar;

template <bool NT, typename T>
__device__ __forceinline__ T ld(const gchar *base, uint32_t byte_off) {
    const __attribute__((address_space(1))) T *p =
        reinterpret_cast<const __attribute__((address_space(1))) T *>(base + byte_off);
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT, typename T>
__device__ __forceinline__ void st(gchar *base, uint32_t byte_off, T v) {
    __attribute__((address_space(1))) T *p =
        reinterpret_cast<__attribute__((address_space(1))) T *>(base + byte_off);
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

__device__ __forceinline__ gchar *as_global(void *p) { return (gchar *)p; }
__device__ __forceinline__ const gchar *as_global(const void *p) { return (const gchar *)p; }

// A 3x3 complex matrix held in registers as separate real/imaginary parts,
// element (r, c) at index 3r + c.
template <typename R> struct Mat {
    R re[9], im[9];
};

// Rebuild row 2 of a special unitary matrix from rows 0 and 1:
// row2 = conj(row0 x row1).
template <typename R>
__device__ __forceinline__ void rebuild_row2(Mat<R> &m) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        // (row0 x row1)_c = r0[c1] r1[c2] - r0[c2] r1[c1]
        R xr = fma(m.re[c1], m.re[3 + c2], -m.im[c1] * m.im[3 + c2]);
        xr = fma(-m.re[c2], m.re[3 + c1], fma(m.im[c2], m.im[3 + c1], xr));
        R xi = fma(m.re[c1], m.im[3 + c2], m.im[c1] * m.re[3 + c2]);
        xi = fma(-m.re[c2], m.im[3 + c1], fma(-m.im[c2], m.re[3 + c1], xi));
        m.re[6 + c] = xr;
        m.im[6 + c] = -xi;
    }
}

// A link from its NE stored complex values. NE = 9: full matrix; NE = 6:
// rows 0, 1; NE = 4: the 8-real form of link8.hpp.
template <typename R, int NE>
__device__ __forceinline__ void unpack_link(const typename V2<R>::type v[NE], Mat<R> &m) {
    if constexpr (NE == 4) {
        R sre[4], sim[4];
#pragma unroll
        for (int e = 0; e < 4; e++) { sre[e] = v[e].x; sim[e] = v[e].y; }
        link8_reconstruct<R>(sre, sim, m.re, m.im);
    } else {
#pragma unroll
        for (int e = 0; e < NE; e++) { m.re[e] = v[e].x; m.im[e] = v[e].y; }
        if constexpr (NE == 6) rebuild_row2(m);
    }
}

// Link whose element 0 sits at complex offset `off` (see link_off); element
// e is BLK complex values further.
template <typename R, int NE, bool NT>
__device__ __forceinline__ void load_link(Mat<R> &m, const gchar *base, long long off) {
    typedef typename V2<R>::type v2;
    const gchar *p = base + off * (long long)sizeof(v2);
    v2 v[NE];
#pragma unroll
    for (int e = 0; e < NE; e++) v[e] = ld<NT, v2>(p, (uint32_t)(e * BLK * sizeof(v2)));
    unpack_link<R, NE>(v, m);
}

template <typename R, int NE, bool NT>
__device__ __forceinline__ void store_link(const Mat<R> &m, gchar *base, long long off) {
    typedef typename V2<R>::type v2;
    gchar *p = base + off * (long long)sizeof(v2);
    if constexpr (NE == 4) {
        R sre[4], sim[4];
        link8_compress<R>(m.re, m.im, sre, sim);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            v2 v;
            v.x = sre[e];
            v.y = sim[e];
            st<NT, v2>(p, (uint32_t)(e * BLK * sizeof(v2)), v);
        }
    } else {
#pragma unroll
        for (int e = 0; e < NE; e++) {
            R x = m.re[e], y = m.im[e];
            // keep the pair as two register values: otherwise the compiler may
            // fetch re[e] together with its neighbour re[e + 1] as one 8-byte
            // load, which keeps m in memory (LDS) instead of registers
            asm("" : "+v"(x), "+v"(y));
            v2 v;
            v.x = x;
            v.y = y;
            st<NT, v2>(p, (uint32_t)(e * BLK * sizeof(v2)), v);
        }
    }
}

// r / |r| for a row of three complex numbers. Rows of float links take one
// reciprocal square root and six products (the result is rounded to float);
// double links keep the correctly rounded quotients.
template <typename R>
__device__ __forceinline__ void normalise_row(double r[3], double i[3]) {
    const double n2 = r[0] * r[0] + i[0] * i[0] + r[1] * r[1] + i[1] * i[1] + r[2] * r[2] + i[2] * i[2];
    if constexpr (sizeof(R) == 4) {
        const double f = gf_rsqrt(n2);
#pragma unroll
        for (int c = 0; c < 3; c++) { r[c] *= f; i[c] *= f; }
    } else {
        const double n = sqrt(n2);
#pragma unroll
        for (int c = 0; c < 3; c++) { r[c] /= n; i[c] /= n; }
    }
}

// Gram-Schmidt reunitarisation in double: r0 /= |r0|; r1 -= (r0^+ r1) r0;
// r1 /= |r1|; r2 = conj(r0 x r1). Result rounded to the link precision.
template <typename R>
__device__ __forceinline__ void reunitarise(Mat<R> &m) {
    double r0r[3], r0i[3], r1r[3], r1i[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        r0r[c] = m.re[c]; r0i[c] = m.im[c];
        r1r[c] = m.re[3 + c]; r1i[c] = m.im[3 + c];
    }
    normalise_row<R>(r0r, r0i);
    double pr = 0.0, pi = 0.0;  // r0^+ r1
#pragma unroll
    for (int c = 0; c < 3; c++) {
        pr += r0r[c] * r1r[c] + r0i[c] * r1i[c];
        pi += r0r[c] * r1i[c] - r0i[c] * r1r[c];
    }
#pragma unroll
    for (int c = 0; c < 3; c++) {
        r1r[c] -= pr * r0r[c] - pi * r0i[c];
        r1i[c] -= pr * r0i[c] + pi * r0r[c];
    }
    normalise_row<R>(r1r, r1i);
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        double xr = r0r[c1] * r1r[c2] - r0i[c1] * r1i[c2] - (r0r[c2] * r1r[c1] - r0i[c2] * r1i[c1]);
        double xi = r0r[c1] * r1i[c2] + r0i[c1] * r1r[c2] - (r0r[c2] * r1i[c1] + r0i[c2] * r1r[c1]);
        m.re[6 + c] = (R)xr;
        m.im[6 + c] = (R)(-xi);
        m.re[c] = (R)r0r[c]; m.im[c] = (R)r0i[c];
        m.re[3 + c] = (R)r1r[c]; m.im[3 + c] = (R)r1i[c];
    }
}

__device__ __forceinline__ int pick4(const int v[4], int i) {
    return i == 0 ? v[0] : (i == 1 ? v[1] : (i == 2 ? v[2] : v[3]));
}

}  // namespace gf
