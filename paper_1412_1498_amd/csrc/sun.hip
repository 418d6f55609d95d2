// sun.hip -- Alg. 1 for SU(N) links, N = 2 and 4 (the paper's method for a
// general number of colours: the local maximisation visits all N(N-1)/2
// SU(2) subgroups (a, b), a < b, in lexicographic order).
//
// The half-sweep has the structure of the SU(3) kernel: a site owns its
// eight links; K(x) = sum_mu [U_mu(x) + U_mu(x - mu)^dagger] (eq. 5) is
// built once in double over the link slots (fwd 0, bwd 0, ..., fwd 3,
// bwd 3) in the fixed tree ((s0 + s1) + (s2 + s3)) + ((s4 + s5) + (s6 + s7)),
// the upper levels across the LPS lanes of a site; every
// subgroup step (eq. 6 on the (a, b) block, exact principal power for the
// over-relaxation) acts on K (K <- G K) and on the running product T, and
// the eight links are rotated once by T (rounded to the link precision).
// All schedules give bitwise identical links. N = 4 needs LPS >= 2 (eight
// 4x4 links do not fit one lane's registers).
//
// Also here: pack/unpack between the canonical [site][mu][N][N] layout and
// the blocked layout, and standalone reunitarisation.
#include "pack_tile.hpp"
#include "sun_device.hpp"
#include "sun_internal.hpp"

namespace gf {

namespace {

struct Q4n { double v[4]; };

template <typename R>
__device__ __forceinline__ Q4n sun_su2_step(Q4n b, double omega) {
    Q4n r;
    gf_su2_overrelax<sizeof(R) == 8>(b.v, omega, r.v);
    return r;
}

// Rows a, b of m <- g (rows a, b of m), g = [[g0 + i g3, g2 + i g1],
// [-g2 + i g1, g0 - i g3]].
template <int N>
__device__ __forceinline__ void rot_rows_n(DMN<N> &m, int a, int b, const Q4n &g) {
    const double ar = g.v[0], ai = g.v[3], br = g.v[2], bi = g.v[1];
#pragma unroll
    for (int c = 0; c < N; c++) {
        const double xr = m.re[N * a + c], xi = m.im[N * a + c];
        const double yr = m.re[N * b + c], yi = m.im[N * b + c];
        m.re[N * a + c] = fma(ar, xr, fma(-ai, xi, fma(br, yr, -bi * yi)));
        m.im[N * a + c] = fma(ar, xi, fma(ai, xr, fma(br, yi, bi * yr)));
        m.re[N * b + c] = fma(-br, xr, fma(-bi, xi, fma(ar, yr, ai * yi)));
        m.im[N * b + c] = fma(-br, xi, fma(bi, xr, fma(ar, yi, -ai * yr)));
    }
}

// o = g u
template <typename R, int N>
__device__ __forceinline__ void apply_left_n(const MatN<R, N> &u, const MatN<R, N> &g, MatN<R, N> &o) {
#pragma unroll
    for (int r = 0; r < N; r++)
#pragma unroll
        for (int c = 0; c < N; c++) {
            R sr = g.re[N * r] * u.re[c];
            R si = g.re[N * r] * u.im[c];
            sr = fma(-g.im[N * r], u.im[c], sr);
            si = fma(g.im[N * r], u.re[c], si);
#pragma unroll
            for (int k = 1; k < N; k++) {
                sr = fma(g.re[N * r + k], u.re[N * k + c], sr);
                sr = fma(-g.im[N * r + k], u.im[N * k + c], sr);
                si = fma(g.re[N * r + k], u.im[N * k + c], si);
                si = fma(g.im[N * r + k], u.re[N * k + c], si);
            }
            o.re[N * r + c] = sr;
            o.im[N * r + c] = si;
        }
}

// o = u g^dagger: o_rc = sum_k u_rk conj(g_ck)
template <typename R, int N>
__device__ __forceinline__ void apply_right_dag_n(const MatN<R, N> &u, const MatN<R, N> &g, MatN<R, N> &o) {
#pragma unroll
    for (int r = 0; r < N; r++)
#pragma unroll
        for (int c = 0; c < N; c++) {
            R sr = u.re[N * r] * g.re[N * c];
            R si = u.im[N * r] * g.re[N * c];
            sr = fma(u.im[N * r], g.im[N * c], sr);
            si = fma(-u.re[N * r], g.im[N * c], si);
#pragma unroll
            for (int k = 1; k < N; k++) {
                sr = fma(u.re[N * r + k], g.re[N * c + k], sr);
                sr = fma(u.im[N * r + k], g.im[N * c + k], sr);
                si = fma(u.im[N * r + k], g.re[N * c + k], si);
                si = fma(-u.re[N * r + k], g.im[N * c + k], si);
            }
            o.re[N * r + c] = sr;
            o.im[N * r + c] = si;
        }
}

template <typename R, int N, int LPS, bool NT, bool RU>
__device__ __forceinline__ void or_site_n(const CfgDesc &d, int p, int h, int sub) {
    constexpr int L = 8 / LPS;  // links per lane
    constexpr int E = N * N;
    const Geom &g = d.g;
    gchar *U = as_global(d.U);
    SiteNbr nb = site_neighbours(g, p, h);
    const bool landau = d.gauge == 0;

    bool bwd[L], in[L];
#pragma unroll
    for (int k = 0; k < L; k++) {
        const int slot = sub * L + k;
        bwd[k] = (slot & 1) != 0;  // compile-time unless LPS == 8
        in[k] = landau || (slot >> 1) != 3;
    }
    auto slot_off = [&](int k) {
        const int mu = (sub * L + k) >> 1;
        return bwd[k] ? link_off(g, mu, 1 - p, pick4(nb.hb, mu)) : link_off(g, mu, p, h);
    };
    MatN<R, N> w[L];
#pragma unroll
    for (int k = 0; k < L; k++) load_link_n<R, N, NT>(w[k], U, slot_off(k));
    __builtin_amdgcn_sched_barrier(0);  // all loads before the first use, as in the SU(3) sweep

    DMN<N> K;
#pragma unroll
    for (int r = 0; r < N; r++) {
#pragma unroll
        for (int c = 0; c < N; c++) {
            const int e = N * r + c, et = N * c + r;
            double tr[L], ti[L];
#pragma unroll
            for (int k = 0; k < L; k++) {
                const double xr = bwd[k] ? (double)w[k].re[et] : (double)w[k].re[e];
                const double xi = bwd[k] ? -(double)w[k].im[et] : (double)w[k].im[e];
                tr[k] = in[k] ? xr : 0.0;
                ti[k] = in[k] ? xi : 0.0;
            }
#pragma unroll
            for (int step = 1; step < L; step *= 2)
#pragma unroll
                for (int k = 0; k < L; k += 2 * step) {
                    tr[k] = tr[k] + tr[k + step];
                    ti[k] = ti[k] + ti[k + step];
                }
            K.re[e] = site_sum<LPS>(tr[0]);
            K.im[e] = site_sum<LPS>(ti[0]);
        }
    }

    DMN<N> T;
#pragma unroll
    for (int e = 0; e < E; e++) { T.re[e] = (e % (N + 1) == 0) ? 1.0 : 0.0; T.im[e] = 0.0; }
#pragma unroll
    for (int a = 0; a < N; a++)
#pragma unroll
        for (int b = a + 1; b < N; b++) {
            const int aa = N * a + a, bb = N * b + b, ab = N * a + b, ba = N * b + a;
            Q4n q;
            q.v[0] = 0.5 * (K.re[aa] + K.re[bb]);
            q.v[1] = 0.5 * (K.im[ab] + K.im[ba]);
            q.v[2] = 0.5 * (K.re[ab] - K.re[ba]);
            q.v[3] = 0.5 * (K.im[aa] - K.im[bb]);
            const Q4n gq = sun_su2_step<R>(q, d.omega);
            rot_rows_n<N>(K, a, b, gq);
            rot_rows_n<N>(T, a, b, gq);
        }
    MatN<R, N> G;
#pragma unroll
    for (int e = 0; e < E; e++) { G.re[e] = (R)T.re[e]; G.im[e] = (R)T.im[e]; }

    // places recomputed, as in the SU(3) sweep
    asm("" : "+v"(h));
#pragma unroll
    for (int mu = 0; mu < 4; mu++) asm("" : "+v"(nb.hb[mu]));
#pragma unroll
    for (int k = 0; k < L; k++) {
        MatN<R, N> o;
        if (LPS == 8) {
            MatN<R, N> f, r;
            apply_left_n(w[k], G, f);
            apply_right_dag_n(w[k], G, r);
#pragma unroll
            for (int e = 0; e < E; e++) {
                o.re[e] = bwd[k] ? r.re[e] : f.re[e];
                o.im[e] = bwd[k] ? r.im[e] : f.im[e];
            }
        } else if (bwd[k]) {
            apply_right_dag_n(w[k], G, o);
        } else {
            apply_left_n(w[k], G, o);
        }
        if constexpr (RU) reunitarise_n(o);
        store_link_n<R, N, NT>(o, U, slot_off(k));
    }
}

template <typename R, int N, int LPS, bool NT, bool RU>
__global__ void __launch_bounds__(256)
k_sun_half_sweep(const CfgDesc *__restrict__ desc, const int *__restrict__ tile_cfg,
                 const int *__restrict__ active, int parity, int order) {
    const int b = parity ? xcd_reverse(blockIdx.x, gridDim.x) : (int)blockIdx.x;  // as in the SU(3) sweep
    const int tile = order ? xcd_tile(b, gridDim.x) : b;
    const int c = tile_cfg[tile];
    if (!active[c]) return;
    const CfgDesc d = desc[c];
    const int h = (tile - d.tile0) * (int)(blockDim.x / LPS) + (int)(threadIdx.x / LPS);
    if (h >= d.g.Vh) return;
    or_site_n<R, N, LPS, NT, RU>(d, parity, h, threadIdx.x % LPS);
}

template <typename R, int N, int LPS>
hipError_t launch_sun_t(const Schedule &s, const CfgDesc *d_desc, const int *d_tile_cfg,
                        const int *d_active, int ntiles, int parity, int reunit, hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
#define GF_S(NT, RU)                                                                                \
    hipLaunchKernelGGL((k_sun_half_sweep<R, N, LPS, NT, RU>), dim3(ntiles), dim3(s.block), s.lds, st, \
                       d_desc, d_tile_cfg, d_active, parity, s.order)
    if (reunit) { if (s.nt) GF_S(true, true); else GF_S(false, true); }
    else { if (s.nt) GF_S(true, false); else GF_S(false, false); }
#undef GF_S
    return hipGetLastError();
}

template <typename R, int N>
hipError_t launch_sun_lps(const Schedule &s, const CfgDesc *d_desc, const int *d_tile_cfg,
                          const int *d_active, int ntiles, int parity, int reunit, hipStream_t st) {
    switch (s.lps) {
        case 1:
            if constexpr (N == 2)
                return launch_sun_t<R, N, 1>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st);
            else
                return hipErrorInvalidValue;
        case 2: return launch_sun_t<R, N, 2>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st);
        case 4: return launch_sun_t<R, N, 4>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st);
        case 8: return launch_sun_t<R, N, 8>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st);
        default: return hipErrorInvalidValue;
    }
}

// Canonical AoS [site][mu][N][N] <-> blocked layout: the tiles of the SU(3) packer,
// a lane per link between LDS and the blocked layout. Packing zeroes the rest of
// a parity's last block.
template <typename R, int N, bool UNPACK>
__global__ void __launch_bounds__(PACK_BLOCK) k_sun_pack(Geom g, typename V2<R>::type *__restrict__ aos,
                                                         typename V2<R>::type *__restrict__ U) {
    typedef typename V2<R>::type v2;
    constexpr int E = N * N;
    typedef PackTile<v2, 4 * E> T;
    __shared__ v2 lds[T::SIZE];
    const int h0 = (int)blockIdx.x * T::TH;
    const int sites = 2 * max(0, min(T::TH, g.Vh - h0));
    v2 *run = aos + 8LL * E * h0;
    if (!UNPACK) T::fill(lds, run, sites);
#pragma unroll
    for (int l = threadIdx.x; l < 8 * T::TH; l += PACK_BLOCK) {
        const int q = l / T::TH, h = l % T::TH, p = q >> 2, mu = q & 3;
        const bool in = 2 * h < sites;
        v2 *at = lds + (pack_side(g, p, h0 + h) * T::TH + h) * T::STRIDE + E * mu;
        v2 *field = U + link_off(g, mu, p, h0 + h);
#pragma unroll
        for (int e = 0; e < E; e++) {
            if (!UNPACK) field[e * BLK] = in ? at[e] : v2{R(0), R(0)};
            else if (in) at[e] = field[e * BLK];
        }
    }
    if (UNPACK) T::drain(lds, run, sites);
}

// Standalone reunitarisation of every link; one thread per link.
template <typename R, int N>
__global__ void __launch_bounds__(256) k_sun_reunit(Geom g, void *Uv) {
    const long long l = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= 4LL * g.V) return;
    const int n = (int)(l >> 2), mu = (int)(l & 3);
    const int p = n >= g.Vh, h = n - p * g.Vh;
    gchar *U = as_global(Uv);
    const long long o = link_off(g, mu, p, h);
    MatN<R, N> m;
    load_link_n<R, N, false>(m, U, o);
    reunitarise_n(m);
    store_link_n<R, N, false>(m, U, o);
}

}  // namespace

hipError_t launch_sun_half_sweep(int prec, int nc, const Schedule &s, const CfgDesc *d_desc,
                                 const int *d_tile_cfg, const int *d_active, int ntiles, int parity,
                                 int reunit, hipStream_t st) {
    if (nc == 2)
        return prec == 0 ? launch_sun_lps<double, 2>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st)
                         : launch_sun_lps<float, 2>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st);
    if (nc == 4)
        return prec == 0 ? launch_sun_lps<double, 4>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st)
                         : launch_sun_lps<float, 4>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st);
    return hipErrorInvalidValue;
}

hipError_t launch_sun_pack(int prec, int nc, const Geom &g, const void *aos, void *U, int to_aos,
                           hipStream_t st) {
#define GF_U(R, N, UN)                                                                               \
    hipLaunchKernelGGL((k_sun_pack<R, N, UN>), dim3(g.nb * (BLK / PackTile<V2<R>::type, 4 * N * N>::TH)), \
                       dim3(PACK_BLOCK), 0, st, g, (V2<R>::type *)aos, (V2<R>::type *)U)
#define GF_P(R, N) do { if (to_aos) GF_U(R, N, true); else GF_U(R, N, false); } while (0)
    if (nc == 2) { if (prec == 0) GF_P(double, 2); else GF_P(float, 2); }
    else if (nc == 4) { if (prec == 0) GF_P(double, 4); else GF_P(float, 4); }
    else return hipErrorInvalidValue;
#undef GF_P
#undef GF_U
    return hipGetLastError();
}

hipError_t launch_sun_reunit(int prec, int nc, const Geom &g, void *U, hipStream_t st) {
    const long long n = 4LL * g.V;
    const int B = 256;
    const dim3 grid((unsigned)((n + B - 1) / B));
    if (nc == 2) {
        if (prec == 0) hipLaunchKernelGGL((k_sun_reunit<double, 2>), grid, dim3(B), 0, st, g, U);
        else hipLaunchKernelGGL((k_sun_reunit<float, 2>), grid, dim3(B), 0, st, g, U);
    } else if (nc == 4) {
        if (prec == 0) hipLaunchKernelGGL((k_sun_reunit<double, 4>), grid, dim3(B), 0, st, g, U);
        else hipLaunchKernelGGL((k_sun_reunit<float, 4>), grid, dim3(B), 0, st, g, U);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace gf
