// fft.hpp -- the lattice Fourier transforms of Alg. 2 (fft.hip), as seen by
// the host code that plans and launches them.
#pragma once

#include "gf_internal.hpp"

namespace gf {

// Lattice Fourier transforms of Alg. 2 (fft.hip). Spectrum of the eight
// components spec[t][a][z][y][kx], kx = 0..nx/2. A workgroup transforms a tile
// of at most FFT_TILE_POINTS complex points in LDS (in place, in double, with
// the roots: <= 40 KB), so an axis may be at most FFT_MAX_N long (whose
// radices take at most FFT_MAX_PASSES passes).
constexpr int FFT_BLOCK = 256;
constexpr int FFT_TILE_POINTS = 1536;
constexpr int FFT_MAX_N = 1024;
// Along x a tile holds the eight components of whole site rows (four complex
// pencils per row), so nx is at most FFT_TILE_POINTS / 4.
constexpr int FFT_MAX_NX = FFT_TILE_POINTS / 4;

// Division by a small divisor d as a multiply-high: floor(n / d) =
// (n * ceil(2^32 / d)) >> 32 exactly for n, d < 2^16 (d = 1 kept apart).
struct FastDiv {
    unsigned d, m;
};

inline FastDiv make_fastdiv(unsigned d) {
    FastDiv f;
    f.d = d;
    f.m = d > 1 ? (unsigned)((0x100000000ULL + d - 1) / d) : 0u;
    return f;
}

__device__ __forceinline__ unsigned fdiv(unsigned n, const FastDiv &f) { return f.d == 1 ? n : __umulhi(n, f.m); }

// Division by any d of a number below 2^31: floor(n / d) = (n m) >> (31 + s) for
// s = ceil(log2 d), m = ceil(2^(31 + s) / d) (n times m's excess over
// 2^(31 + s) / d stays below 2^31 <= 2^(31 + s) / d, so the floor is exact).
struct WideDiv {
    unsigned d, m;
    int s;
};

inline WideDiv make_widediv(unsigned d) {
    WideDiv w{d, 0u, 0};
    while ((1ULL << w.s) < d) w.s++;
    if (d > 1) w.m = (unsigned)(((1ULL << (31 + w.s)) + d - 1) / d);
    return w;
}

__host__ __device__ __forceinline__ unsigned wdiv(unsigned n, const WideDiv &w) {
    return w.d == 1 ? n : (unsigned)(((unsigned long long)n * w.m) >> 32) >> (w.s - 1);
}

constexpr int FFT_MAX_PASSES = 12;
struct FftPlan {     // radices of the Stockham passes, in order
    int nf;
    int fac[FFT_MAX_PASSES];
    FastDiv ns[FFT_MAX_PASSES];  // division by Ns = product of the earlier radices
};

struct FftSite {      // Delta and the real <-> half-complex transform along x, by site rows
    int n;            // nx
    FftPlan pl;
    int nkx;          // nx / 2 + 1
    int ys;           // site rows (lines along x) per workgroup: 4 ys complex pencils
    long long srows;  // nt * nz * ny
    FastDiv dn, dnkx, dnc;  // division by nx, nkx and 4 ys
    int n1, n2;       // nx = n1 n2 for the two-butterfly form (0: nx does not split)
    FastDiv dn1;
};

struct FftAxis {     // complex, in place, along y, z or t
    int n;           // axis length
    FftPlan pl;
    int np, nkx, nchunk;  // kx per workgroup, kx count, kx chunks per row
    long long s_ax;  // spectrum stride along the axis
    int r[3];        // the other three of (t, a, z, y): extents ...
    long long s[3];  // ... and strides
    int Lx, Lax, L[3];    // lattice lengths entering p^2 (0: not a transformed direction)
    double scale, p2max;  // filter factor scale * p2max / p^2(k)
    FastDiv dnp;          // division by np
};

// The same transform by two butterflies of n1 and n2 points in registers
// (n = n1 n2, both at most FFT_LINE_RADIX), for lengths that split so. The
// pencils are numbered P = outer * Q + inner, inner running over Q contiguous
// values.
constexpr int FFT_LINE_RADIX = 13;
constexpr int FFT_SITE_RADIX = 8;  // of the x transforms, which keep Delta's or g's registers as well
struct FftLine {
    int n, n1, n2;        // n1 = 0: the length does not split
    unsigned total;       // pencils
    WideDiv dQ;           // division by Q
    long long s_ax, s_o;  // spectrum strides along the axis and of the outer index
    WideDiv dkx, dy;      // the filter's decoding of the inner index: kx, y, z
    int nz;               // extent of z in the inner index (0: not there)
    double scale, p2max;
};

FftSite make_fft_site(const Geom &g);
FftAxis make_fft_axis(const Geom &g, int axis, bool coulomb);  // axis 1 = y, 2 = z, 3 = t
FftLine make_fft_line(const Geom &g, int axis);
// W: a table of exp(2 pi i m / n), m < n, for the transform's length; p2: one
// of 4 sin^2(pi m / n) (launch_fft_roots fills both)
hipError_t launch_fft_roots(void *W, double *p2, int n, hipStream_t st);
// Delta (eq. 3) of every site -> its components' x-transformed half spectrum;
// with part, also sd_delta_groups(f) pairs of partial sums for F and theta
int sd_delta_groups(const FftSite &f);
hipError_t launch_sd_delta_fx(int prec, int nelem, int gauge, const Geom &g, const FftSite &f, const void *W,
                              const void *U, void *spec, double *part, hipStream_t st);
// half spectrum -> inverse x transform -> g = reunit(1 + X) as the g field (gfield_off)
hipError_t launch_sd_fx_gfield(int prec, const Geom &g, const FftSite &f, const void *W, const void *spec,
                               void *gfield, hipStream_t st);
// one axis, by the two-butterfly kernel where the length splits (l.n1), else in
// LDS (f); p2: the four axes' tables, FFT_MAX_N doubles each
hipError_t launch_fft_axis(int prec, const FftAxis &f, const FftLine &l, const void *W, const double *p2, void *spec,
                           int axis, int sign, int filter, hipStream_t st);

}  // namespace gf
