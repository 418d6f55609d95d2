// fft.hip -- steepest descent with Fourier acceleration (Alg. 2, eqs. 7-9) on
// gfx950: Delta of eq. (3) as its eight real su(3) components, their lattice
// Fourier transform, the p2_max / p^2(k) filter, the inverse transform, and
// the step's gauge transformation g = reunit(1 + X) as a g field for
// k_gauge_transform.
//
// The components' spectrum is held as spec[t][a][z][y][kx] with kx = 0..nx/2
// (the real transform along x keeps half the spectrum, the other half being
// its complex conjugate). One pass per axis: x (real <-> half complex), with
// Delta computed in the forward x pass and g formed in the inverse one, so
// the components never go to memory in lattice space; then y, z and t
// (complex, in place). The multiplication by p2_max / p^2(k) is fused into
// the last forward pass, between its forward and inverse transform, so that
// pass writes back the filtered field already transformed back along its own
// axis.
//
// Lengths that split into two factors of at most 13 are transformed by two
// butterflies in registers with one trip through LDS between them
// (k_fft_line; along x, where the tile sits in LDS anyway, lds_split_forward
// and lds_split_inverse for factors of at most 8). Any other length: a
// workgroup loads a tile of pencils (for y, z, t: consecutive kx of one row,
// so every global access is a contiguous run) into LDS and transforms them by
// the mixed-radix Stockham algorithm (radix 4, 2, 3, 5 butterflies in
// registers, any larger prime by a direct sum), in place: one LDS read, one
// write and one twiddle per point and pass. The arithmetic is in double for
// both link precisions (a double FMA costs the same as a float one on this
// GPU); the spectrum is stored in the context precision between passes.
#include "fft.hpp"
#include "su3_device.hpp"
#include "tile_order.hpp"

namespace gf {

namespace {

// 16-byte aligned so that a value moves to and from LDS as one 128-bit
// access: as two 64-bit halves, consecutive lanes' values fell into the same
// banks and every LDS instruction of the transforms stalled on conflicts.
struct alignas(16) Cd {
    double x, y;
};

__device__ __forceinline__ Cd cmul(Cd a, Cd b) {
    Cd r;
    r.x = fma(a.x, b.x, -a.y * b.y);
    r.y = fma(a.x, b.y, a.y * b.x);
    return r;
}

__device__ __forceinline__ void cmac(Cd &acc, Cd a, Cd b) {
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(-a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(a.y, b.x, acc.y);
}

// LDS of a transform tile: one buffer holding element j of pencil q at
// a[j * ld + q] (ld >= np pencils; the x transforms pad it so that a pencil's
// consecutive elements fall in different banks), transformed in place, and
// the n roots exp(2 pi i m / n).
struct Tile {
    Cd *a, *Wl;
    int ld;
    FastDiv dnp;  // division by the pencil count
};

__host__ __device__ inline int tile_lds_points(int n, int ld) { return n * ld + n; }

__device__ __forceinline__ Tile tile_setup(Cd *lds, const Cd *__restrict__ Wg, int n, int ld, const FastDiv &dnp) {
    Tile t;
    t.a = lds;
    t.ld = ld;
    t.dnp = dnp;
    t.Wl = lds + n * ld;
    return t;
}

// The n roots into the tile: called after the tile's own loads are issued,
// so their latency overlaps those instead of preceding them (lds_dft begins
// with a barrier).
__device__ __forceinline__ void load_roots(const Tile &t, const Cd *__restrict__ Wg, int n) {
    for (int m = threadIdx.x; m < n; m += blockDim.x) t.Wl[m] = Wg[m];
}

// w or its conjugate: the table holds exp(+2 pi i m / n); SIGN = -1 forward.
template <int SIGN>
__device__ __forceinline__ Cd root(Cd w) {
    if constexpr (SIGN < 0) w.y = -w.y;
    return w;
}

__device__ __forceinline__ Cd cadd(Cd a, Cd b) { return Cd{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ Cd csub(Cd a, Cd b) { return Cd{a.x - b.x, a.y - b.y}; }
// i s z for s = +-1
template <int S>
__device__ __forceinline__ Cd imul(Cd z) { return S > 0 ? Cd{-z.y, z.x} : Cd{z.y, -z.x}; }

// In-register R-point DFTs, X_s = sum_m v_m exp(SIGN 2 pi i m s / R).
template <int SIGN>
__device__ __forceinline__ void bfly2(Cd *v) {
    const Cd a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <int SIGN>
__device__ __forceinline__ void bfly4(Cd *v) {
    const Cd t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const Cd t2 = cadd(v[1], v[3]), t3 = imul<SIGN>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
}

template <int SIGN>
__device__ __forceinline__ void bfly3(Cd *v) {
    const double h = 0.86602540378443864676;  // sin(2 pi / 3)
    const Cd s = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const Cd t = Cd{v[0].x - 0.5 * s.x, v[0].y - 0.5 * s.y};
    const Cd u = imul<SIGN>(Cd{h * d.x, h * d.y});
    v[0] = cadd(v[0], s);
    v[1] = cadd(t, u);
    v[2] = csub(t, u);
}

template <int SIGN>
__device__ __forceinline__ void bfly5(Cd *v) {
    const double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;  // cos(2 pi/5), cos(4 pi/5)
    const double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;   // sin(2 pi/5), sin(4 pi/5)
    const Cd a1 = cadd(v[1], v[4]), b1 = csub(v[1], v[4]);
    const Cd a2 = cadd(v[2], v[3]), b2 = csub(v[2], v[3]);
    const Cd p = Cd{v[0].x + c1 * a1.x + c2 * a2.x, v[0].y + c1 * a1.y + c2 * a2.y};
    const Cd r = Cd{v[0].x + c2 * a1.x + c1 * a2.x, v[0].y + c2 * a1.y + c1 * a2.y};
    const Cd u = imul<SIGN>(Cd{s1 * b1.x + s2 * b2.x, s1 * b1.y + s2 * b2.y});
    const Cd w = imul<SIGN>(Cd{s2 * b1.x - s1 * b2.x, s2 * b1.y - s1 * b2.y});
    v[0] = cadd(v[0], cadd(a1, a2));
    v[1] = cadd(p, u);
    v[4] = csub(p, u);
    v[2] = cadd(r, w);
    v[3] = csub(r, w);
}

// 8 points as two of 4 and the twiddles exp(SIGN 2 pi i m / 8).
template <int SIGN>
__device__ __forceinline__ void bfly8(Cd *v) {
    const double h = 0.70710678118654752440;
    Cd e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    bfly4<SIGN>(e);
    bfly4<SIGN>(o);
    const Cd i1 = imul<SIGN>(o[1]), i3 = imul<SIGN>(o[3]);
    o[1] = Cd{h * (o[1].x + i1.x), h * (o[1].y + i1.y)};
    o[2] = imul<SIGN>(o[2]);
    o[3] = Cd{h * (i3.x - o[3].x), h * (i3.y - o[3].y)};
#pragma unroll
    for (int k = 0; k < 4; k++) { v[k] = cadd(e[k], o[k]); v[k + 4] = csub(e[k], o[k]); }
}

// An odd number of points R: with the sums a_j = v_j + v_(R-j) and differences
// b_j, X_k = v_0 + sum_j cos(2 pi j k / R) a_j + SIGN i sum_j sin(2 pi j k / R) b_j.
template <int R> struct OddRoots;
template <> struct OddRoots<7> {
    static constexpr double c[4] = {1.0, 0.6234898018587335, -0.2225209339563144, -0.9009688679024191};
    static constexpr double s[4] = {0.0, 0.7818314824680298, 0.9749279121818236, 0.4338837391175581};
};
template <> struct OddRoots<9> {
    static constexpr double c[5] = {1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084};
    static constexpr double s[5] = {0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386,
                                    0.3420201433256687};
};
template <> struct OddRoots<11> {
    static constexpr double c[6] = {1.0, 0.8412535328311812, 0.41541501300188644, -0.14231483827328514,
                                    -0.6548607339452851, -0.9594929736144974};
    static constexpr double s[6] = {0.0, 0.5406408174555976, 0.9096319953545183, 0.9898214418809327,
                                    0.7557495743542583, 0.28173255684142967};
};
template <> struct OddRoots<13> {
    static constexpr double c[7] = {1.0, 0.8854560256532099, 0.5680647467311558, 0.12053668025532305,
                                    -0.3546048870425356, -0.7485107481711011, -0.970941817426052};
    static constexpr double s[7] = {0.0, 0.46472317204376856, 0.8229838658936564, 0.992708874098054,
                                    0.9350162426854148, 0.6631226582407952, 0.23931566428755777};
};

template <int SIGN, int R>
__device__ __forceinline__ void bfly_odd(Cd *v) {
    constexpr int H = (R - 1) / 2;
    Cd a[H + 1], b[H + 1];
#pragma unroll
    for (int j = 1; j <= H; j++) { a[j] = cadd(v[j], v[R - j]); b[j] = csub(v[j], v[R - j]); }
    const Cd v0 = v[0];
    Cd sum = v0;
#pragma unroll
    for (int j = 1; j <= H; j++) sum = cadd(sum, a[j]);
    v[0] = sum;
#pragma unroll
    for (int k = 1; k <= H; k++) {
        Cd p = v0, q = {0.0, 0.0};
#pragma unroll
        for (int j = 1; j <= H; j++) {
            const int m = j * k % R, i = m <= H ? m : R - m;
            const double c = OddRoots<R>::c[i], s = m <= H ? OddRoots<R>::s[i] : -OddRoots<R>::s[i];
            p = Cd{fma(c, a[j].x, p.x), fma(c, a[j].y, p.y)};
            q = Cd{fma(s, b[j].x, q.x), fma(s, b[j].y, q.y)};
        }
        q = imul<SIGN>(q);
        v[k] = cadd(p, q);
        v[R - k] = csub(p, q);
    }
}

template <int SIGN, int R>
__device__ __forceinline__ void bfly(Cd *v);

// R = P Q points, P and Q without common factor, by the prime-factor map: input
// (Q i + P j) mod R, output (e_P k + e_Q l) mod R with e_P = 1 mod P, 0 mod Q
// and e_Q the other way round: no twiddles between the two.
template <int SIGN, int P, int Q, int EP, int EQ>
__device__ __forceinline__ void bfly_pfa(Cd *v) {
    constexpr int R = P * Q;
    static_assert(EP % P == 1 && EP % Q == 0 && EQ % Q == 1 && EQ % P == 0, "prime-factor map");
    Cd t[Q][P];
#pragma unroll
    for (int j = 0; j < Q; j++)
#pragma unroll
        for (int i = 0; i < P; i++) t[j][i] = v[(Q * i + P * j) % R];
#pragma unroll
    for (int j = 0; j < Q; j++) bfly<SIGN, P>(t[j]);
#pragma unroll
    for (int k = 0; k < P; k++) {
        Cd u[Q];
#pragma unroll
        for (int j = 0; j < Q; j++) u[j] = t[j][k];
        bfly<SIGN, Q>(u);
#pragma unroll
        for (int l = 0; l < Q; l++) v[(EP * k + EQ * l) % R] = u[l];
    }
}

template <int SIGN, int R>
__device__ __forceinline__ void bfly(Cd *v) {
    if constexpr (R == 2) bfly2<SIGN>(v);
    else if constexpr (R == 3) bfly3<SIGN>(v);
    else if constexpr (R == 4) bfly4<SIGN>(v);
    else if constexpr (R == 5) bfly5<SIGN>(v);
    else if constexpr (R == 6) bfly_pfa<SIGN, 2, 3, 3, 4>(v);
    else if constexpr (R == 8) bfly8<SIGN>(v);
    else if constexpr (R == 10) bfly_pfa<SIGN, 2, 5, 5, 6>(v);
    else if constexpr (R == 12) bfly_pfa<SIGN, 4, 3, 9, 4>(v);
    else bfly_odd<SIGN, R>(v);
}

// Butterflies per thread in a radix-R pass: a tile holds at most
// FFT_TILE_POINTS points, i.e. FFT_TILE_POINTS / R butterflies, over
// FFT_BLOCK threads; outputs per thread in a pass of any other radix.
constexpr int pass_b(int R) { return (FFT_TILE_POINTS / R + FFT_BLOCK - 1) / FFT_BLOCK; }
constexpr int PASS_OUT = (FFT_TILE_POINTS + FFT_BLOCK - 1) / FFT_BLOCK;
// Global loads per thread when a tile is filled (all issued before the first
// use, so a workgroup waits for one memory latency, not one per element).
constexpr int LOAD_C = (FFT_TILE_POINTS + FFT_BLOCK - 1) / FFT_BLOCK;

// One radix-R pass of the Stockham autosort algorithm over np pencils (element
// j of pencil q at [j * ld + q]), in place: Ns = product of the earlier
// radices; butterfly j reads j + r n/R, twiddles by
// exp(SIGN 2 pi i r (j mod Ns) / (Ns R)), and writes (j / Ns) Ns R + (j mod Ns) + r Ns.
// Every thread reads all its butterflies into registers before the barrier
// and writes them after it.
template <int SIGN, int R>
__device__ __forceinline__ void stockham_pass(Cd *buf, const Cd *Wl, int n, int Ns, int np, int ld,
                                              const FastDiv &dnp, const FastDiv &dns) {
    constexpr int B = pass_b(R);
    const int nb = n / R, tw = n / (Ns * R), total = nb * np;
    Cd v[B][R];
#pragma unroll
    for (int i = 0; i < B; i++) {
        const int bi = threadIdx.x + i * FFT_BLOCK;
        if (bi < total) {
            const int j = (int)fdiv((unsigned)bi, dnp), q = bi - j * np;
            const int k = j - (int)fdiv((unsigned)j, dns) * Ns;
#pragma unroll
            for (int r = 0; r < R; r++) v[i][r] = buf[(j + r * nb) * ld + q];
#pragma unroll
            for (int r = 1; r < R; r++) v[i][r] = cmul(v[i][r], root<SIGN>(Wl[r * k * tw]));
            bfly<SIGN, R>(v[i]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < B; i++) {
        const int bi = threadIdx.x + i * FFT_BLOCK;
        if (bi < total) {
            const int j = (int)fdiv((unsigned)bi, dnp), q = bi - j * np;
            const int jh = (int)fdiv((unsigned)j, dns), k = j - jh * Ns;
            const int d = jh * Ns * R + k;
#pragma unroll
            for (int r = 0; r < R; r++) buf[(d + r * Ns) * ld + q] = v[i][r];
        }
    }
}

// A pass of any radix R (the primes above 5), in place: one output per
// thread and slot, the R-point sum over the root table.
template <int SIGN>
__device__ __forceinline__ void stockham_pass_any(Cd *buf, const Cd *Wl, int n, int Ns, int R, int np, int ld) {
    const int nb = n / R, tw = n / (Ns * R), nR = n / R, total = n * np;
    Cd o[PASS_OUT];
#pragma unroll
    for (int i = 0; i < PASS_OUT; i++) {
        const int idx = threadIdx.x + i * FFT_BLOCK;
        if (idx < total) {
            const int q = idx % np, rest = idx / np, j = rest % nb, s = rest / nb, k = j % Ns;
            Cd acc = {0.0, 0.0};
            for (int r = 0; r < R; r++) {
                Cd x = buf[(j + r * nb) * ld + q];
                if (r) x = cmul(x, root<SIGN>(Wl[r * k * tw]));
                cmac(acc, x, root<SIGN>(Wl[((r * s) % R) * nR]));
            }
            o[i] = acc;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PASS_OUT; i++) {
        const int idx = threadIdx.x + i * FFT_BLOCK;
        if (idx < total) {
            const int q = idx % np, rest = idx / np, j = rest % nb, s = rest / nb, k = j % Ns;
            buf[((j / Ns) * Ns * R + k + s * Ns) * ld + q] = o[i];
        }
    }
}

// DFT of np pencils of length n held in t.a, in place. Begins and ends with
// a barrier.
template <int SIGN>
__device__ __forceinline__ void lds_dft(const Tile &t, const FftPlan &pl, int n, int np) {
    int Ns = 1;
    for (int f = 0; f < pl.nf; f++) {
        __syncthreads();
        const int R = pl.fac[f];
        if (R == 4) stockham_pass<SIGN, 4>(t.a, t.Wl, n, Ns, np, t.ld, t.dnp, pl.ns[f]);
        else if (R == 2) stockham_pass<SIGN, 2>(t.a, t.Wl, n, Ns, np, t.ld, t.dnp, pl.ns[f]);
        else if (R == 3) stockham_pass<SIGN, 3>(t.a, t.Wl, n, Ns, np, t.ld, t.dnp, pl.ns[f]);
        else if (R == 5) stockham_pass<SIGN, 5>(t.a, t.Wl, n, Ns, np, t.ld, t.dnp, pl.ns[f]);
        else stockham_pass_any<SIGN>(t.a, t.Wl, n, Ns, R, np, t.ld);
        Ns *= R;
    }
    __syncthreads();
}

// Two butterflies over np pencils held in LDS, n = n1 n2 (index n2 i + j, spectrum
// k + n1 l), where the axis length splits so: three barriers instead of two a
// radix, and no point is moved between its two reads. Forward: a lane
// transforms the n1 points i of one j in place (place k n2 + j gets k), then
// the n2 points j of one k; mode k + n1 l ends at place k n2 + l. Inverse: the
// same backwards, from those places to natural order.
#define GF_SITE_RADICES(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

// points at base + m step (m < R) of every pencil, for rows 0 .. rows - 1 whose
// base is row * rstep; times W^(row m) before (PRE) or after the butterfly
template <int SIGN, int R, bool PRE>
__device__ __forceinline__ void lds_rows(const Tile &t, int rows, int rstep, int step, bool twiddle, int np) {
    for (int idx = threadIdx.x; idx < rows * np; idx += blockDim.x) {
        const int row = (int)fdiv((unsigned)idx, t.dnp), q = idx - row * np;
        Cd *a = t.a + row * rstep * t.ld + q;
        Cd v[R];
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = a[m * step * t.ld];
        if (PRE && twiddle) {
#pragma unroll
            for (int m = 1; m < R; m++) v[m] = cmul(v[m], root<SIGN>(t.Wl[row * m]));
        }
        bfly<SIGN, R>(v);
#pragma unroll
        for (int m = 0; m < R; m++)
            a[m * step * t.ld] = (!PRE && twiddle && m) ? cmul(v[m], root<SIGN>(t.Wl[row * m])) : v[m];
    }
}

// forward transform; begins and ends with a barrier
__device__ __forceinline__ void lds_split_forward(const Tile &t, int n1, int n2, int np) {
    __syncthreads();
#define GF_S(r) case r: lds_rows<-1, r, false>(t, n2, 1, n2, true, np); break;
    switch (n1) { GF_SITE_RADICES(GF_S) default: break; }
#undef GF_S
    __syncthreads();
#define GF_S(r) case r: lds_rows<-1, r, false>(t, n1, n2, 1, false, np); break;
    switch (n2) { GF_SITE_RADICES(GF_S) default: break; }
#undef GF_S
    __syncthreads();
}

// inverse transform; begins and ends with a barrier
__device__ __forceinline__ void lds_split_inverse(const Tile &t, int n1, int n2, int np) {
    __syncthreads();
#define GF_S(r) case r: lds_rows<1, r, false>(t, n1, n2, 1, false, np); break;
    switch (n2) { GF_SITE_RADICES(GF_S) default: break; }
#undef GF_S
    __syncthreads();
#define GF_S(r) case r: lds_rows<1, r, true>(t, n2, 1, n2, true, np); break;
    switch (n1) { GF_SITE_RADICES(GF_S) default: break; }
#undef GF_S
    __syncthreads();
}

// place of mode m of a split length
__device__ __forceinline__ int split_place(const FftSite &f, int m) {
    const int l = (int)fdiv((unsigned)m, f.dn1);
    return (m - l * f.n1) * f.n2 + l;
}

__device__ __forceinline__ double lattice_p2(int k, int L) {
    if (L <= 0) return 0.0;
    const double s = sinpi((double)k / (double)L);
    return 4.0 * s * s;
}

}  // namespace

// The transform kernels ask for four waves per SIMD (at most 128 VGPRs): a
// pass's butterflies fit in that without spilling, and a CU then holds four
// workgroups to overlap one tile's memory phase with another's passes.

namespace {

// Delta(x) of eq. (3) at site (p, h) as its eight real su(3) components
// o_a = Tr[lambda_a Delta] / (2i): M = sum_mu [U_mu(x - mu) - U_mu(x)] in
// double, A = M - M^dagger, whose traceless part is Delta (the trace part
// drops out of these traces, so only Im of the diagonal and the off-diagonal
// entries of A enter).
template <typename R, int NE, bool SUMS>
__device__ __forceinline__ void delta_components(const Geom &g, int nd, const gchar *U, int p, int h, double o[8],
                                                 double &fsum, double &tsum) {
    const SiteNbr nb = site_neighbours(g, p, h);
    double mr[9], mi[9];
#pragma unroll
    for (int e = 0; e < 9; e++) { mr[e] = 0.0; mi[e] = 0.0; }
    for (int mu = 0; mu < nd; mu++) {
        Mat<R> f, b;
        load_link<R, NE, false>(f, U, link_off(g, mu, p, h));
        load_link<R, NE, false>(b, U, link_off(g, mu, 1 - p, pick4(nb.hb, mu)));
#pragma unroll
        for (int e = 0; e < 9; e++) {
            mr[e] += (double)b.re[e] - (double)f.re[e];
            mi[e] += (double)b.im[e] - (double)f.im[e];
        }
        if (SUMS) fsum += (double)f.re[0] + (double)f.re[4] + (double)f.re[8];
    }
    double ar[9], ai[9];
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int c = 0; c < 3; c++) {
            ar[3 * r + c] = mr[3 * r + c] - mr[3 * c + r];
            ai[3 * r + c] = mi[3 * r + c] + mi[3 * c + r];
        }
    const double r3 = 0.57735026918962576451;  // 1/sqrt(3)
    o[0] = 0.5 * (ai[3] + ai[1]);
    o[1] = 0.5 * (ar[1] - ar[3]);
    o[2] = 0.5 * (ai[0] - ai[4]);
    o[3] = 0.5 * (ai[6] + ai[2]);
    o[4] = 0.5 * (ar[2] - ar[6]);
    o[5] = 0.5 * (ai[7] + ai[5]);
    o[6] = 0.5 * (ar[5] - ar[7]);
    o[7] = 0.5 * r3 * (ai[0] + ai[4] - 2.0 * ai[8]);
    if (SUMS) {
        const double trr = (ar[0] + ar[4] + ar[8]) / 3.0;
        const double tri = (ai[0] + ai[4] + ai[8]) / 3.0;
#pragma unroll
        for (int r = 0; r < 3; r++) { ar[4 * r] -= trr; ai[4 * r] -= tri; }
#pragma unroll
        for (int e = 0; e < 9; e++) tsum += ar[e] * ar[e] + ai[e] * ai[e];
    }
}

// g = reunit(1 + i H), H = sum_a s_a lambda_a (the first-order exponential
// of the step, Gram-Schmidt), in double.
__device__ __forceinline__ void step_matrix(const double s[8], Mat<double> &m) {
    const double r3 = 0.57735026918962576451;
    double hr[9], hi[9];
    hr[0] = s[2] + r3 * s[7];  hi[0] = 0.0;
    hr[4] = -s[2] + r3 * s[7]; hi[4] = 0.0;
    hr[8] = -2.0 * r3 * s[7];  hi[8] = 0.0;
    hr[1] = s[0]; hi[1] = -s[1];
    hr[3] = s[0]; hi[3] = s[1];
    hr[2] = s[3]; hi[2] = -s[4];
    hr[6] = s[3]; hi[6] = s[4];
    hr[5] = s[5]; hi[5] = -s[6];
    hr[7] = s[5]; hi[7] = s[6];
#pragma unroll
    for (int e = 0; e < 9; e++) {
        m.re[e] = (e % 4 == 0 ? 1.0 : 0.0) - hi[e];
        m.im[e] = hr[e];
    }
    reunitarise(m);
}

// (t, z, y) of the site rows of a tile, and z ny + y (row index within a
// time slice), kept in LDS so each is divided out once.
struct RowInfo {
    int t, z, y, zy;
};

__device__ __forceinline__ void row_info(RowInfo *ri, const Geom &g, long long sr0, int ys, long long srows) {
    for (int yl = threadIdx.x; yl < ys; yl += blockDim.x) {
        const long long sr = sr0 + yl;
        RowInfo r = {0, 0, 0, -1};
        if (sr < srows) {
            const int q = (int)(sr / g.ny);
            r.y = (int)(sr - (long long)q * g.ny);
            r.t = q / g.nz;
            r.z = q - r.t * g.nz;
            r.zy = r.z * g.ny + r.y;
        }
        ri[yl] = r;
    }
}

// spec[t][a][z][y][kx] index of component a, kx of a site row
__device__ __forceinline__ long long spec_index(const Geom &g, int nkx, const RowInfo &r, int a, int k) {
    return (((long long)r.t * 8 + a) * g.nz * g.ny + r.zy) * nkx + k;
}

}  // namespace

// Delta and its forward real transform along x, for ys site rows (lines
// along x at fixed y, z, t; consecutive in (t, z, y)). The eight components of
// a site row travel as four complex rows, components 2c + i (2c + 1) in
// pencil 4 yl + c; after the transform A[k] = (Z[k] + conj Z[-k]) / 2 and
// B[k] = (Z[k] - conj Z[-k]) / 2i are the two components' spectra. A site
// row holds both parities, so a site's x-backward link is the other
// parity's forward link of the same tile and its y-backward link that of the
// previous row.
//
// SUMS: the workgroup's sums for F and theta as well (of site rows instead of
// F/theta's tiles), one pair per workgroup into part: a step that follows a
// check has every link in registers here, so the check needs no pass of its own.
// Steps with a check each, before and after: double 20x28x18x30 (Coulomb) 1059
// -> 915 us for five, 32^4 3670 -> 3155, float 16^4 735 -> 596 for ten; float 48^4
// with one check in five 8150 -> 7840.
template <typename R, int NE, bool SUMS>
__global__ void __launch_bounds__(FFT_BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
k_sd_delta_fx(Geom g, int nd, const typename V2<R>::type *__restrict__ Uv, FftSite f, const Cd *__restrict__ Wg,
              typename V2<R>::type *__restrict__ spec, SlabOrder so, double *__restrict__ part) {
    extern __shared__ Cd lds[];
    const int nx = g.nx, nc = 4 * f.ys;
    const Tile t = tile_setup(lds, Wg, nx, nc + 1, f.dnc);
    load_roots(t, Wg, nx);
    RowInfo *ri = (RowInfo *)(t.Wl + nx);
    // slab order over tiles of ys site rows: a time slice is ny nz rows, so
    // the rows holding the t-backward links were read ny nz / ys tiles
    // before, in the same column block
    const int tile = slab_tile(xcd_tile(blockIdx.x, gridDim.x), so);
    const long long sr0 = (long long)tile * f.ys;
    row_info(ri, g, sr0, f.ys, f.srows);
    __syncthreads();
    const gchar *U = as_global((const void *)Uv);
    double fsum = 0.0, tsum = 0.0;
    for (int idx = threadIdx.x; idx < f.ys * nx; idx += blockDim.x) {
        const int yl = (int)fdiv((unsigned)idx, f.dn), x = idx - yl * nx;
        const RowInfo r = ri[yl];
        double o[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if (r.zy >= 0) {
            const int lx = x + nx * (int)(sr0 + yl);  // x + nx (y + ny (z + nz t))
            delta_components<R, NE, SUMS>(g, nd, U, (x + r.y + r.z + r.t) & 1, lx >> 1, o, fsum, tsum);
        }
#pragma unroll
        for (int c = 0; c < 4; c++) t.a[x * t.ld + yl * 4 + c] = Cd{o[2 * c], o[2 * c + 1]};
    }
    if constexpr (SUMS) {
        __shared__ Cd sums[FFT_BLOCK / 64];
        fsum = wave_sum(fsum);
        tsum = wave_sum(tsum);
        if (threadIdx.x % 64 == 0) sums[threadIdx.x / 64] = Cd{fsum, tsum};
        __syncthreads();
        if (threadIdx.x == 0) {
            Cd v = sums[0];
#pragma unroll
            for (int w = 1; w < FFT_BLOCK / 64; w++) { v.x += sums[w].x; v.y += sums[w].y; }
            part[2 * tile] = v.x;
            part[2 * tile + 1] = v.y;
        }
    }
    if (f.n1) lds_split_forward(t, f.n1, f.n2, nc);
    else lds_dft<-1>(t, f.pl, nx, nc);
    for (int idx = threadIdx.x; idx < 8 * f.ys * f.nkx; idx += blockDim.x) {
        const int row = (int)fdiv((unsigned)idx, f.dnkx), k = idx - row * f.nkx;
        const int yl = row >> 3, a = row & 7;
        const RowInfo r = ri[yl];
        if (r.zy < 0) continue;
        const int cr = yl * 4 + (a >> 1);
        const int km = k ? nx - k : 0;
        const Cd zk = t.a[(f.n1 ? split_place(f, k) : k) * t.ld + cr];
        const Cd zm = t.a[(f.n1 ? split_place(f, km) : km) * t.ld + cr];
        typename V2<R>::type v;
        if (a & 1) {  // (zk - conj zm) / 2i
            v.x = (R)(0.5 * (zk.y + zm.y));
            v.y = (R)(-0.5 * (zk.x - zm.x));
        } else {      // (zk + conj zm) / 2
            v.x = (R)(0.5 * (zk.x + zm.x));
            v.y = (R)(0.5 * (zk.y - zm.y));
        }
        spec[spec_index(g, f.nkx, r, a, k)] = v;
    }
}

// Inverse real transform along x of ys site rows' eight component spectra
// (the rest of each by conjugate symmetry; the imaginary parts at kx = 0 and
// nx/2 are dropped, as for any real inverse transform), components 2c and
// 2c + 1 travelling as Z = A + i B; then every site's step matrix
// g = reunit(1 + i sum_a s_a lambda_a), written as the g field (gfield_off).
template <typename R>
__global__ void __launch_bounds__(FFT_BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
k_sd_fx_gfield(Geom g, FftSite f, const Cd *__restrict__ Wg, const typename V2<R>::type *__restrict__ spec,
               typename V2<R>::type *__restrict__ gf) {
    extern __shared__ Cd lds[];
    const int nx = g.nx, nc = 4 * f.ys, h = nx / 2;
    const Tile t = tile_setup(lds, Wg, nx, nc + 1, f.dnc);
    RowInfo *ri = (RowInfo *)(t.Wl + nx);
    const long long sr0 = (long long)xcd_tile(blockIdx.x, gridDim.x) * f.ys;
    row_info(ri, g, sr0, f.ys, f.srows);
    __syncthreads();
    // Every lane loads unconditionally (a pair that does not exist reads
    // element 0 and is zeroed afterwards): loads under a branch made the
    // compiler copy each result at the branch's end, which waited for it, so
    // only two loads were ever in flight.
    typename V2<R>::type va[LOAD_C], vb[LOAD_C];
    bool ok[LOAD_C];
#pragma unroll
    for (int i = 0; i < LOAD_C; i++) {  // nc nkx <= FFT_TILE_POINTS (pencil, frequency) pairs
        const int idx = threadIdx.x + i * FFT_BLOCK;
        const bool in = idx < nc * f.nkx;
        const int cr = in ? (int)fdiv((unsigned)idx, f.dnkx) : 0, k = idx - cr * f.nkx;
        const RowInfo r = ri[cr >> 2];
        ok[i] = in && r.zy >= 0;
        const int a = 2 * (cr & 3);
        const long long ia = ok[i] ? spec_index(g, f.nkx, r, a, k) : 0;
        const long long ib = ok[i] ? spec_index(g, f.nkx, r, a + 1, k) : 0;
        va[i] = spec[ia];
        vb[i] = spec[ib];
    }
    load_roots(t, Wg, nx);
#pragma unroll
    for (int i = 0; i < LOAD_C; i++) {
        const int idx = threadIdx.x + i * FFT_BLOCK;
        if (idx >= nc * f.nkx) continue;
        const int cr = (int)fdiv((unsigned)idx, f.dnkx), k = idx - cr * f.nkx;
        const double z = ok[i] ? 1.0 : 0.0;
        const Cd A = Cd{z * (double)va[i].x, z * (double)va[i].y}, B = Cd{z * (double)vb[i].x, z * (double)vb[i].y};
        const int pk = f.n1 ? split_place(f, k) : k;
        if (k == 0 || k == h) {
            t.a[pk * t.ld + cr] = Cd{A.x, B.x};
        } else {
            const int pm = f.n1 ? split_place(f, nx - k) : nx - k;
            t.a[pk * t.ld + cr] = Cd{A.x - B.y, A.y + B.x};
            t.a[pm * t.ld + cr] = Cd{A.x + B.y, B.x - A.y};
        }
    }
    if (f.n1) lds_split_inverse(t, f.n1, f.n2, nc);
    else lds_dft<1>(t, f.pl, nx, nc);
    for (int idx = threadIdx.x; idx < f.ys * nx; idx += blockDim.x) {
        const int yl = (int)fdiv((unsigned)idx, f.dn), x = idx - yl * nx;
        const RowInfo r = ri[yl];
        if (r.zy < 0) continue;
        double sv[8];
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const Cd z = t.a[x * t.ld + yl * 4 + c];
            sv[2 * c] = z.x;
            sv[2 * c + 1] = z.y;
        }
        Mat<double> m;
        step_matrix(sv, m);
        const int lx = x + nx * (int)(sr0 + yl);
        const long long o = gfield_off(g, (x + r.y + r.z + r.t) & 1, lx >> 1, 0);
#pragma unroll
        for (int e = 0; e < 9; e++) {
            typename V2<R>::type v;
            v.x = (R)m.re[e];
            v.y = (R)m.im[e];
            gf[o + (long long)e * BLK] = v;
        }
    }
}

// Complex transform along one of y, z, t, in place. A workgroup takes np
// consecutive kx of one row (outer index = the other three of t, a, z, y).
// FILTER: forward transform, multiply by scale p2max / p^2(k) (0 at p^2 = 0),
// inverse transform.
template <typename R, bool FILTER>
__global__ void __launch_bounds__(FFT_BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
k_fft_axis(FftAxis f, const Cd *__restrict__ Wg, typename V2<R>::type *__restrict__ spec, int sign) {
    extern __shared__ Cd lds[];
    const int n = f.n, np = f.np;
    const Tile t = tile_setup(lds, Wg, n, np, f.dnp);
    // XCD-contiguous tile order: neighbouring tiles (the kx chunks of a row,
    // then the next row) share cache lines and meet in one L2
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = tile % f.nchunk;
    int o = tile / f.nchunk;
    const int d0 = o % f.r[0];
    o /= f.r[0];
    const int d1 = o % f.r[1], d2 = o / f.r[1];
    const int kx0 = chunk * np;
    const long long base = d0 * f.s[0] + d1 * f.s[1] + d2 * f.s[2] + kx0;
    {
        typename V2<R>::type v[LOAD_C];
#pragma unroll
        for (int i = 0; i < LOAD_C; i++) {
            const int idx = threadIdx.x + i * FFT_BLOCK;
            v[i].x = v[i].y = (R)0;
            if (idx < n * np) {
                const int j = (int)fdiv((unsigned)idx, f.dnp), q = idx - j * np;
                if (kx0 + q < f.nkx) v[i] = spec[base + j * f.s_ax + q];
            }
        }
        load_roots(t, Wg, n);
#pragma unroll
        for (int i = 0; i < LOAD_C; i++) {
            const int idx = threadIdx.x + i * FFT_BLOCK;
            if (idx < n * np) t.a[idx] = Cd{(double)v[i].x, (double)v[i].y};
        }
    }
    if (FILTER || sign < 0) lds_dft<-1>(t, f.pl, n, np);
    else lds_dft<1>(t, f.pl, n, np);
    Cd *res = t.a;
    if constexpr (FILTER) {
        // 4 sin^2(pi k / L) of this axis and of the tile's kx, once per workgroup
        double *p2ax = (double *)(t.Wl + n), *p2x = p2ax + n;
        for (int m = threadIdx.x; m < n + np; m += blockDim.x) {
            if (m < n) p2ax[m] = lattice_p2(m, f.Lax);
            else p2x[m - n] = lattice_p2(kx0 + m - n, f.Lx);
        }
        __syncthreads();
        const double p2o = lattice_p2(d0, f.L[0]) + lattice_p2(d1, f.L[1]) + lattice_p2(d2, f.L[2]);
        const double sp = f.scale * f.p2max;
        for (int idx = threadIdx.x; idx < n * np; idx += blockDim.x) {
            const int k = (int)fdiv((unsigned)idx, f.dnp), q = idx - k * np;
            const double p2 = p2o + p2ax[k] + p2x[q];
            const double fac = p2 > 0.0 ? sp / p2 : 0.0;
            res[idx].x *= fac;
            res[idx].y *= fac;
        }
        lds_dft<1>(t, f.pl, n, np);  // back along the same axis
    }
    for (int idx = threadIdx.x; idx < n * np; idx += blockDim.x) {
        const int j = (int)fdiv((unsigned)idx, f.dnp), q = idx - j * np;
        if (kx0 + q < f.nkx) {
            typename V2<R>::type v;
            v.x = (R)res[idx].x;
            v.y = (R)res[idx].y;
            spec[base + j * f.s_ax + q] = v;
        }
    }
}

// One axis by two butterflies in registers: n = n1 n2, input index
// n2 i + j, output index k + n1 l. A lane takes the n1 points i of one (j,
// pencil) straight from memory, transforms them, multiplies by
// W^(j k) and leaves them in LDS; after the one barrier a lane takes the n2
// points j of one (k, pencil), transforms them and writes them back. With
// FILTER they are scaled instead, transformed back in place (same lane, same
// LDS places) and, after a second barrier, along i.
// What bounds it: memory. The LDS kernel below moves every point through LDS
// once a radix (4, 4, 3 at 48) and once more at either end, with a barrier
// each, and its four workgroups a CU could not hide that: 3.0 TB/s in float.
// A pass at 48^4, before -> after: float 119 -> 50-59 us (6-7 TB/s: the
// spectrum fits the last-level cache), filtered 232 -> 77 us; double
// 136 -> 119-124 us, filtered 249 -> 167 us. The LDS kernel stays for the
// lengths that do not split (a prime factor above 13, or above 13^2).
// Tiles are LINE_NP consecutive pencils, so that every access is a run of 256
// bytes, aligned wherever the inner extent is a multiple of it.
template <typename R> constexpr int LINE_NP = sizeof(R) == 4 ? 32 : 16;

template <typename R>
struct LineCtx {
    const FftLine &f;
    const Cd *W;
    Cd *lds;
    typename V2<R>::type *at;  // the lane's pencil
    int q, row;                // pencil within the tile, the lane's j or k
    bool in;                   // the pencil exists
};

// memory -> i-transform -> LDS
template <typename R, int SIGN, int N1>
__device__ __forceinline__ void line_first(const LineCtx<R> &c) {
    const int n2 = c.f.n2, j = c.row;
    if (j >= n2) return;
    typename V2<R>::type x[N1];
    Cd v[N1], w[N1];
#pragma unroll
    for (int i = 0; i < N1; i++) x[i] = c.at[(long long)(i * n2 + j) * c.f.s_ax];
#pragma unroll
    for (int k = 1; k < N1; k++) w[k] = c.W[j * k];
#pragma unroll
    for (int i = 0; i < N1; i++) v[i] = Cd{(double)x[i].x, (double)x[i].y};
    bfly<SIGN, N1>(v);
#pragma unroll
    for (int k = 0; k < N1; k++)
        c.lds[(k * n2 + j) * LINE_NP<R> + c.q] = k ? cmul(v[k], root<SIGN>(w[k])) : v[0];
}

// LDS -> j-transform -> memory, or filter and back to LDS
template <typename R, int SIGN, bool FILTER, int N2>
__device__ __forceinline__ void line_second(const LineCtx<R> &c, const double *p2ax, double p2) {
    const int n1 = c.f.n1, k = c.row;
    if (k >= n1) return;
    Cd v[N2];
    Cd *l = c.lds + k * N2 * LINE_NP<R> + c.q;
#pragma unroll
    for (int j = 0; j < N2; j++) v[j] = l[j * LINE_NP<R>];
    bfly<SIGN, N2>(v);
    if constexpr (!FILTER) {
        if (!c.in) return;
#pragma unroll
        for (int i = 0; i < N2; i++)
            c.at[(long long)(k + n1 * i) * c.f.s_ax] = typename V2<R>::type{(R)v[i].x, (R)v[i].y};
    } else {
        const double sp = c.f.scale * c.f.p2max;
#pragma unroll
        for (int i = 0; i < N2; i++) {
            const double s = p2 + p2ax[k + n1 * i];
            const double fac = s > 0.0 ? sp / s : 0.0;
            v[i].x *= fac;
            v[i].y *= fac;
        }
        bfly<1, N2>(v);
#pragma unroll
        for (int j = 0; j < N2; j++) l[j * LINE_NP<R>] = j ? cmul(v[j], c.W[j * k]) : v[0];
    }
}

// LDS -> inverse i-transform -> memory
template <typename R, int N1>
__device__ __forceinline__ void line_third(const LineCtx<R> &c) {
    const int n2 = c.f.n2, j = c.row;
    if (j >= n2) return;
    Cd v[N1];
#pragma unroll
    for (int k = 0; k < N1; k++) v[k] = c.lds[(k * n2 + j) * LINE_NP<R> + c.q];
    bfly<1, N1>(v);
    if (!c.in) return;
#pragma unroll
    for (int i = 0; i < N1; i++)
        c.at[(long long)(i * n2 + j) * c.f.s_ax] = typename V2<R>::type{(R)v[i].x, (R)v[i].y};
}

// MAXR: largest radix (8, whose registers allow twice the waves, or 13).
template <typename R, int SIGN, bool FILTER, int MAXR>
__global__ void __launch_bounds__(MAXR * LINE_NP<R> > 256 ? 448 : 256)
k_fft_line(FftLine f, const Cd *__restrict__ W, const double *__restrict__ p2, int axis,
           typename V2<R>::type *__restrict__ spec) {
    extern __shared__ Cd lds[];
    constexpr int NP = LINE_NP<R>;
    const int q = threadIdx.x % NP, row = threadIdx.x / NP;
    const unsigned P = (unsigned)xcd_tile(blockIdx.x, gridDim.x) * NP + q;
    const bool in = P < f.total;
    const unsigned Pc = in ? P : 0u;  // lanes past the last pencil read pencil 0 and write nothing
    const unsigned o = wdiv(Pc, f.dQ), inner = Pc - o * f.dQ.d;
    const LineCtx<R> c{f, W, lds, spec + (long long)o * f.s_o + inner, q, row, in};
    double p2p = 0.0;
    if constexpr (FILTER) {
        const unsigned yz = wdiv(inner, f.dkx), y0 = wdiv(yz, f.dy);
        p2p = p2[inner - yz * f.dkx.d] + p2[FFT_MAX_N + yz - y0 * f.dy.d];
        if (f.nz) p2p += p2[2 * FFT_MAX_N + (int)y0 % f.nz];
    }
#define GF_RADICES(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13)
#define GF_R1(r) case r: if constexpr (r <= MAXR) line_first<R, SIGN, r>(c); break;
    switch (f.n1) { GF_RADICES(GF_R1) default: break; }
    __syncthreads();
#define GF_R2(r) case r: if constexpr (r <= MAXR) line_second<R, SIGN, FILTER, r>(c, p2 + axis * FFT_MAX_N, p2p); break;
    switch (f.n2) { GF_RADICES(GF_R2) default: break; }
    if constexpr (FILTER) {
        __syncthreads();
#define GF_R3(r) case r: if constexpr (r <= MAXR) line_third<R, r>(c); break;
        switch (f.n1) { GF_RADICES(GF_R3) default: break; }
    }
#undef GF_R1
#undef GF_R2
#undef GF_R3
#undef GF_RADICES
}

// W[m] = exp(2 pi i m / n) and p2[m] = 4 sin^2(pi m / n), m < n.
__global__ void __launch_bounds__(256) k_fft_roots(Cd *__restrict__ W, double *__restrict__ p2, int n) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double s, c;
    sincospi(2.0 * (double)m / (double)n, &s, &c);
    W[m] = Cd{c, s};
    p2[m] = lattice_p2(m, n);
}

// Radices of a length: 4s first, then 2, 3, 5, then any other primes.
static FftPlan plan_length(int n) {
    FftPlan p{};
    int ns = 1;
    auto push = [&](int r) { p.ns[p.nf] = make_fastdiv((unsigned)ns); p.fac[p.nf++] = r; ns *= r; };
    while (n % 4 == 0) { push(4); n /= 4; }
    for (int r : {2, 3, 5})
        while (n % r == 0) { push(r); n /= r; }
    for (int r = 7; n > 1; r += 2)
        while (n % r == 0) { push(r); n /= r; }
    return p;
}

// n = n1 n2 with n1 <= n2 <= rmax as close as they come (0, 0: none).
static void split_length(int n, int rmax, int *n1, int *n2) {
    *n1 = *n2 = 0;
    for (int a = 2; a * a <= n; a++)
        if (n % a == 0 && n / a <= rmax) { *n1 = a; *n2 = n / a; }
}

FftLine make_fft_line(const Geom &g, int axis) {
    FftLine f{};
    const long long nkx = g.nx / 2 + 1, sy = nkx, sz = g.ny * sy, sa = g.nz * sz, st = 8 * sa;
    long long Q, outer;
    if (axis == 1) { f.n = g.ny; f.s_ax = Q = sy; outer = (long long)g.nt * 8 * g.nz; f.s_o = sz; }
    else if (axis == 2) { f.n = g.nz; f.s_ax = Q = sz; outer = (long long)g.nt * 8; f.s_o = sa; }
    else { f.n = g.nt; f.s_ax = Q = st; outer = 1; f.s_o = 0; }
    f.dQ = make_widediv((unsigned)Q);
    f.total = (unsigned)(outer * Q);
    f.dkx = make_widediv((unsigned)nkx);
    f.dy = make_widediv((unsigned)g.ny);
    f.nz = axis == 3 ? g.nz : 0;
    split_length(f.n, FFT_LINE_RADIX, &f.n1, &f.n2);
    return f;
}

FftSite make_fft_site(const Geom &g) {
    FftSite f;
    f.n = g.nx;
    f.nkx = g.nx / 2 + 1;
    f.pl = plan_length(f.n);
    split_length(f.n, FFT_SITE_RADIX, &f.n1, &f.n2);
    f.dn1 = make_fastdiv((unsigned)(f.n1 ? f.n1 : 1));
    f.ys = FFT_TILE_POINTS / (4 * g.nx);  // site rows per workgroup (>= 1: nx <= FFT_MAX_NX)
    f.srows = (long long)g.nt * g.nz * g.ny;
    f.dn = make_fastdiv((unsigned)f.n);
    f.dnkx = make_fastdiv((unsigned)f.nkx);
    f.dnc = make_fastdiv((unsigned)(4 * f.ys));
    return f;
}

// axis: 1 = y, 2 = z, 3 = t. spec strides: kx 1, y nkx, z ny nkx, a nz ny nkx, t 8 nz ny nkx.
FftAxis make_fft_axis(const Geom &g, int axis, bool coulomb) {
    FftAxis f{};
    const long long nkx = g.nx / 2 + 1, sy = nkx, sz = g.ny * sy, sa = g.nz * sz, st = 8 * sa;
    f.nkx = (int)nkx;
    f.Lx = g.nx;
    if (axis == 1) {
        f.n = g.ny; f.s_ax = sy;
        f.r[0] = g.nz; f.s[0] = sz; f.L[0] = g.nz;
        f.r[1] = 8;    f.s[1] = sa; f.L[1] = 0;
        f.r[2] = g.nt; f.s[2] = st; f.L[2] = coulomb ? 0 : g.nt;
    } else if (axis == 2) {
        f.n = g.nz; f.s_ax = sz;
        f.r[0] = g.ny; f.s[0] = sy; f.L[0] = g.ny;
        f.r[1] = 8;    f.s[1] = sa; f.L[1] = 0;
        f.r[2] = g.nt; f.s[2] = st; f.L[2] = coulomb ? 0 : g.nt;
    } else {
        f.n = g.nt; f.s_ax = st;
        f.r[0] = g.ny; f.s[0] = sy; f.L[0] = g.ny;
        f.r[1] = g.nz; f.s[1] = sz; f.L[1] = g.nz;
        f.r[2] = 8;    f.s[2] = sa; f.L[2] = 0;
    }
    f.Lax = f.n;
    f.pl = plan_length(f.n);
    // kx chunks of at most FFT_TILE_POINTS / n, as even as possible
    const int cap = FFT_TILE_POINTS / f.n > 0 ? FFT_TILE_POINTS / f.n : 1;
    f.nchunk = (f.nkx + cap - 1) / cap;
    f.np = (f.nkx + f.nchunk - 1) / f.nchunk;
    f.dnp = make_fastdiv((unsigned)f.np);
    return f;
}

static size_t lds_bytes(int n, int np) { return (size_t)tile_lds_points(n, np) * sizeof(Cd); }

hipError_t launch_fft_roots(void *W, double *p2, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_fft_roots, dim3((n + 255) / 256), dim3(256), 0, st, (Cd *)W, p2, n);
    return hipGetLastError();
}

static size_t site_lds_bytes(const FftSite &f) {
    return lds_bytes(f.n, 4 * f.ys + 1) + (size_t)f.ys * sizeof(RowInfo);
}

int sd_delta_groups(const FftSite &f) { return (int)((f.srows + f.ys - 1) / f.ys); }

hipError_t launch_sd_delta_fx(int prec, int nelem, int gauge, const Geom &g, const FftSite &f, const void *W,
                              const void *U, void *spec, double *part, hipStream_t st) {
    const dim3 grid((unsigned)sd_delta_groups(f));
    const size_t sh = site_lds_bytes(f);
    const int nd = gauge == 0 ? 4 : 3;
    const Cd *w = (const Cd *)W;
    const SlabOrder so = make_slab_order(g.ny * g.nz, f.ys, (int)grid.x);
#define GF_S(R, NE, SUMS)                                                                             \
    hipLaunchKernelGGL((k_sd_delta_fx<R, NE, SUMS>), grid, dim3(FFT_BLOCK), sh, st, g, nd,           \
                       (const V2<R>::type *)U, f, w, (V2<R>::type *)spec, so, part)
#define GF_L(R, NE) do { if (part) GF_S(R, NE, true); else GF_S(R, NE, false); } while (0)
    if (prec == 0) { if (nelem == 9) GF_L(double, 9); else if (nelem == 6) GF_L(double, 6); else GF_L(double, 4); }
    else { if (nelem == 9) GF_L(float, 9); else if (nelem == 6) GF_L(float, 6); else GF_L(float, 4); }
#undef GF_L
#undef GF_S
    return hipGetLastError();
}

hipError_t launch_sd_fx_gfield(int prec, const Geom &g, const FftSite &f, const void *W, const void *spec,
                               void *gfield, hipStream_t st) {
    const dim3 grid((unsigned)((f.srows + f.ys - 1) / f.ys));
    const size_t sh = site_lds_bytes(f);
    const Cd *w = (const Cd *)W;
    if (prec == 0)
        hipLaunchKernelGGL(k_sd_fx_gfield<double>, grid, dim3(FFT_BLOCK), sh, st, g, f, w,
                           (const V2<double>::type *)spec, (V2<double>::type *)gfield);
    else
        hipLaunchKernelGGL(k_sd_fx_gfield<float>, grid, dim3(FFT_BLOCK), sh, st, g, f, w,
                           (const V2<float>::type *)spec, (V2<float>::type *)gfield);
    return hipGetLastError();
}

template <typename R, int MAXR>
static hipError_t launch_line(const FftLine &l, const Cd *w, const double *p2, void *spec, int axis, int sign,
                              int filter, hipStream_t st) {
    constexpr int NP = LINE_NP<R>;
    const dim3 grid((l.total + NP - 1) / NP), block((l.n2 * NP + 63) / 64 * 64);  // n1 <= n2
    const size_t sh = (size_t)l.n * NP * sizeof(Cd);
    typename V2<R>::type *sp = (typename V2<R>::type *)spec;
    if (filter) hipLaunchKernelGGL((k_fft_line<R, -1, true, MAXR>), grid, block, sh, st, l, w, p2, axis, sp);
    else if (sign < 0) hipLaunchKernelGGL((k_fft_line<R, -1, false, MAXR>), grid, block, sh, st, l, w, p2, axis, sp);
    else hipLaunchKernelGGL((k_fft_line<R, 1, false, MAXR>), grid, block, sh, st, l, w, p2, axis, sp);
    return hipGetLastError();
}

hipError_t launch_fft_axis(int prec, const FftAxis &f, const FftLine &l, const void *W, const double *p2, void *spec,
                           int axis, int sign, int filter, hipStream_t st) {
    const Cd *w = (const Cd *)W;
    if (l.n1) {
        if (prec == 0)
            return l.n2 <= 8 ? launch_line<double, 8>(l, w, p2, spec, axis, sign, filter, st)
                             : launch_line<double, FFT_LINE_RADIX>(l, w, p2, spec, axis, sign, filter, st);
        return l.n2 <= 8 ? launch_line<float, 8>(l, w, p2, spec, axis, sign, filter, st)
                         : launch_line<float, FFT_LINE_RADIX>(l, w, p2, spec, axis, sign, filter, st);
    }
    const dim3 grid((unsigned)((long long)f.r[0] * f.r[1] * f.r[2] * f.nchunk));
    // the filter's tables of the axis and kx terms (n + np doubles) follow the roots
    const size_t sh = lds_bytes(f.n, f.np) + (filter ? (size_t)(f.n + f.np) * sizeof(double) : 0);
    const int sg = sign < 0 ? -1 : 1;
#define GF_L(R, FL) \
    hipLaunchKernelGGL((k_fft_axis<R, FL>), grid, dim3(FFT_BLOCK), sh, st, f, w, (V2<R>::type *)spec, sg)
    if (prec == 0) { if (filter) GF_L(double, true); else GF_L(double, false); }
    else { if (filter) GF_L(float, true); else GF_L(float, false); }
#undef GF_L
    return hipGetLastError();
}

}  // namespace gf
