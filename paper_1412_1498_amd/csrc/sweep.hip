// sweep.hip -- the overrelaxation half-sweep of Alg. 1 on gfx950.
//
// One launch updates every site of one parity of every active ensemble
// member. A site x owns the eight links that touch it: U_mu(x) (parity p
// array, "forward") and U_mu(x - mu) (parity 1 - p array, "backward");
// same-parity sites share none, so the sites are independent and each link
// is read and written exactly once per half-sweep.
//
// Per site: K(x) = sum_mu [U_mu(x) + U_mu(x - mu)^dagger] (eq. 5, the field
// already carrying every transformation so far) is built once, in double.
// Applying a subgroup element G to the site's links (U_mu(x) <- G U_mu(x),
// U_mu(x - mu) <- U_mu(x - mu) G^dagger) maps K to G K exactly, so the three
// subgroup steps of Alg. 1 -- solve eq. (6) on the (a, b) block, over-relax,
// rotate -- are carried out on K alone, in double, and the product
// G3 G2 G1 is applied to each of the eight links once at the end. The result
// is that of rotating the links after every subgroup, with two fewer
// roundings of each link.
//
// What bounds it: memory, for every form but the smallest lattices. The rate
// depends on how many waves are in flight (too few: memory idles while they
// solve; too many on a field beyond the caches: they evict each other's
// neighbours), hence the lane count, workgroup size and occupancy limit by
// lattice size in default_schedule (api.cpp). Half-sweeps at 48^4, before and
// after the solve was shortened, its registers trimmed and the tiles taken
// from alternating ends: float 18-real 546-552 -> 535 us, 12-real 373 -> 342,
// 8-real 372 -> 259, double 18-real 1146 -> 1123-1136, 8-real 684 -> 492-500;
// at 22x18x26x30 42.2 -> 30.7, 27.0 -> 22.4, 31.6 -> 21.5, 79.1 -> 54.1,
// 52.8 -> 32.2.
//
// Schedules: LPS lanes cooperate on a site (LPS = 1, 2, 4, 8), each holding
// 8/LPS links. Link slots are ordered (fwd 0, bwd 0, fwd 1, bwd 1, ...,
// fwd 3, bwd 3); a lane owns consecutive slots and K is summed over slots in
// the fixed tree ((s0 + s1) + (s2 + s3)) + ((s4 + s5) + (s6 + s7)), the
// upper levels across the site's lanes. Every lane then
// runs the (cheap, double) subgroup steps redundantly. The tree does not
// depend on LPS, so all schedules give bitwise identical links.
#include "su3_device.hpp"

namespace gf {

// 3x3 complex matrix in double.
struct DM {
    double re[9], im[9];
};

// A complex double, and products of one FMA chain per component:
// a x + b y, -conj(b) x + conj(a) y (the two rows of an SU(2) rotation),
// a x, conj(a) x.
struct Cz {
    double re, im;
};

__device__ __forceinline__ Cz rot_top(Cz a, Cz b, Cz x, Cz y) {
    return Cz{fma(a.re, x.re, fma(-a.im, x.im, fma(b.re, y.re, -b.im * y.im))),
              fma(a.re, x.im, fma(a.im, x.re, fma(b.re, y.im, b.im * y.re)))};
}

__device__ __forceinline__ Cz rot_bottom(Cz a, Cz b, Cz x, Cz y) {
    return Cz{fma(-b.re, x.re, fma(-b.im, x.im, fma(a.re, y.re, a.im * y.im))),
              fma(-b.re, x.im, fma(b.im, x.re, fma(a.re, y.im, -a.im * y.re)))};
}

__device__ __forceinline__ Cz cz_mul(Cz a, Cz x) {
    return Cz{fma(a.re, x.re, -a.im * x.im), fma(a.re, x.im, a.im * x.re)};
}

__device__ __forceinline__ Cz cz_mul_conj(Cz a, Cz x) {
    return Cz{fma(a.re, x.re, a.im * x.im), fma(a.re, x.im, -a.im * x.re)};
}

// First row (al, be) of the SU(2) element g^omega of eq. (6) for the 2x2
// block [[aa, ab], [ba, bb]] of K; the second row is (-conj be, conj al).
template <typename R>
__device__ __forceinline__ void subgroup_step(Cz aa, Cz ab, Cz ba, Cz bb, double omega, Cz &al, Cz &be) {
    const double q[4] = {0.5 * (aa.re + bb.re), 0.5 * (ab.im + ba.im), 0.5 * (ab.re - ba.re),
                         0.5 * (aa.im - bb.im)};
    double r[4];
    gf_su2_overrelax<sizeof(R) == 8>(q, omega, r);
    al = Cz{r[0], r[3]};
    be = Cz{r[2], r[1]};
}

// o = g u (forward link) or o = u g^dagger (backward link), g in the link
// precision. The result goes to a separate matrix that is stored directly:
// copying it back into u would make the compiler keep a private array.
template <typename R>
__device__ __forceinline__ void apply_left(const Mat<R> &u, const Mat<R> &g, Mat<R> &o) {
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int c = 0; c < 3; c++) {
            R sr = g.re[3 * r] * u.re[c];
            R si = g.re[3 * r] * u.im[c];
            sr = fma(-g.im[3 * r], u.im[c], sr);
            si = fma(g.im[3 * r], u.re[c], si);
#pragma unroll
            for (int k = 1; k < 3; k++) {
                sr = fma(g.re[3 * r + k], u.re[3 * k + c], sr);
                sr = fma(-g.im[3 * r + k], u.im[3 * k + c], sr);
                si = fma(g.re[3 * r + k], u.im[3 * k + c], si);
                si = fma(g.im[3 * r + k], u.re[3 * k + c], si);
            }
            o.re[3 * r + c] = sr;
            o.im[3 * r + c] = si;
        }
}

// (u g^dagger)_rc = sum_k u_rk conj(g_ck)
template <typename R>
__device__ __forceinline__ void apply_right_dag(const Mat<R> &u, const Mat<R> &g, Mat<R> &o) {
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int c = 0; c < 3; c++) {
            R sr = u.re[3 * r] * g.re[3 * c];
            R si = u.im[3 * r] * g.re[3 * c];
            sr = fma(u.im[3 * r], g.im[3 * c], sr);
            si = fma(-u.re[3 * r], g.im[3 * c], si);
#pragma unroll
            for (int k = 1; k < 3; k++) {
                sr = fma(u.re[3 * r + k], g.re[3 * c + k], sr);
                sr = fma(u.im[3 * r + k], g.im[3 * c + k], sr);
                si = fma(u.im[3 * r + k], g.re[3 * c + k], si);
                si = fma(-u.re[3 * r + k], g.im[3 * c + k], si);
            }
            o.re[3 * r + c] = sr;
            o.im[3 * r + c] = si;
        }
}

template <typename R, int NE, int LPS, bool NT, bool RU>
__device__ __forceinline__ void or_site(const CfgDesc &d, int p, int h, int sub) {
    constexpr int L = 8 / LPS;  // links per lane
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

    typedef typename V2<R>::type v2;
    const gchar *base[L];
    v2 raw[L][NE];
    Mat<R> w[L];
#pragma unroll
    for (int k = 0; k < L; k++) base[k] = U + slot_off(k) * (long long)sizeof(v2);
#pragma unroll
    for (int k = 0; k < L; k++)
#pragma unroll
        for (int e = 0; e < NE; e++) raw[k][e] = ld<NT, v2>(base[k], (uint32_t)(e * BLK * sizeof(v2)));
    // every load is issued before the first value is used: left to itself the
    // scheduler defers loads into the solves to save registers, and a wave
    // then waits for several memory latencies instead of one. Not for full float
    // links streamed by one lane, the access of fields far beyond the last-level
    // cache: there the memory is busy anyway, and fewer loads at a time disturb
    // each other less (48^3 x 96 2360 -> 2211 us a sweep, 48^4 1164 -> 1106)
    if constexpr (!(NT && LPS == 1 && NE == 9 && sizeof(R) == 4)) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < L; k++) unpack_link<R, NE>(raw[k], w[k]);

    // K = sum over slots of U (forward) or U^dagger (backward), promoted to
    // double; per element, the lane's slots are summed in place in the fixed
    // tree, then the site's lanes combine.
    DM K;
#pragma unroll
    for (int r = 0; r < 3; r++) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const int e = 3 * r + c, et = 3 * c + r;
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

    // Three subgroup steps on K: (0,1), (0,2), (1,2). Only the entries of the
    // rotated K that a later step reads are formed: K01 and K02 of the rotated
    // row 0, K11 and K12 of row 1, then K21 and K22 of row 2.
    auto k_at = [&](int e) { return Cz{K.re[e], K.im[e]}; };
    Cz a1, b1, a2, b2, a3, b3;
    subgroup_step<R>(k_at(0), k_at(1), k_at(3), k_at(4), d.omega, a1, b1);
    const Cz k00 = rot_top(a1, b1, k_at(0), k_at(3)), k01 = rot_top(a1, b1, k_at(1), k_at(4)),
             k02 = rot_top(a1, b1, k_at(2), k_at(5));
    const Cz k11 = rot_bottom(a1, b1, k_at(1), k_at(4)), k12 = rot_bottom(a1, b1, k_at(2), k_at(5));
    subgroup_step<R>(k00, k02, k_at(6), k_at(8), d.omega, a2, b2);
    subgroup_step<R>(k11, k12, rot_bottom(a2, b2, k01, k_at(7)), rot_bottom(a2, b2, k02, k_at(8)), d.omega, a3, b3);

    // G = G3 G2 G1 (double), rounded to the link precision. With every G a 2x2
    // block and a 1, the rows are
    //   row 0:  (a2 a1, a2 b1, b2)
    //   rows 1, 2: G3 on (-conj b1, conj a1, 0) and
    //              (-conj(b2) a1, -conj(b2) b1, conj a2).
    // (Three general row rotations of the identity took 150 more of the
    // wave's 2300 vector instructions, most of them on zeros.)
    Mat<R> G;
    auto set = [&](int e, Cz z) { G.re[e] = (R)z.re; G.im[e] = (R)z.im; };
    const Cz mb2 = Cz{-b2.re, -b2.im};
    const Cz t10 = Cz{-b1.re, b1.im}, t11 = Cz{a1.re, -a1.im};
    const Cz t20 = cz_mul_conj(mb2, a1), t21 = cz_mul_conj(mb2, b1), t22 = Cz{a2.re, -a2.im};
    set(0, cz_mul(a2, a1));
    set(1, cz_mul(a2, b1));
    set(2, b2);
    set(3, rot_top(a3, b3, t10, t20));
    set(4, rot_top(a3, b3, t11, t21));
    set(5, cz_mul(b3, t22));
    set(6, rot_bottom(a3, b3, t10, t20));
    set(7, rot_bottom(a3, b3, t11, t21));
    set(8, cz_mul_conj(a3, t22));

    // the links' places are worked out again from the five half indices: kept,
    // the eight 64-bit offsets hold 16 registers through the solves (float
    // 18-real: 266 registers with them, 237 without, i.e. two waves per SIMD)
    asm("" : "+v"(h));
#pragma unroll
    for (int mu = 0; mu < 4; mu++) asm("" : "+v"(nb.hb[mu]));
#pragma unroll
    for (int k = 0; k < L; k++) {
        Mat<R> o;
        if (LPS == 8) {
            // the lane's one link is forward or backward at run time
            Mat<R> f, r;
            apply_left(w[k], G, f);
            apply_right_dag(w[k], G, r);
#pragma unroll
            for (int e = 0; e < 9; e++) {
                o.re[e] = bwd[k] ? r.re[e] : f.re[e];
                o.im[e] = bwd[k] ? r.im[e] : f.im[e];
            }
        } else if (bwd[k]) {
            apply_right_dag(w[k], G, o);
        } else {
            apply_left(w[k], G, o);
        }
        if constexpr (RU) reunitarise(o);
        store_link<R, NE, NT>(o, U, slot_off(k));
    }
}

// Waves per SIMD the compiler is asked to leave room for: what each form
// reaches without spilling. Fields that fit the last-level cache run at the
// rate at which waves in their solves leave memory idle, so a second (third)
// wave pays there: float 18-real at 22x18x26x30, one lane per site, one wave
// 36.3 us, two waves 31.6 us.
template <typename R, int NE, int LPS>
constexpr int sweep_waves() {
    if (sizeof(R) == 4) return LPS == 1 ? 2 : LPS == 2 ? 3 : 4;
    return LPS == 1 ? 1 : 2;
}

// One workgroup per tile of blockDim/LPS sites of one member. (A persistent
// grid-stride form was measured to double the register footprint, since
// loop-invariant state stays live across the tile loop, so every tile gets
// its own workgroup; the dispatcher balances the tiles over the CUs.)
template <typename R, int NE, int LPS, bool NT, bool RU>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sweep_waves<R, NE, LPS>())))
k_half_sweep(const CfgDesc *__restrict__ desc, const int *__restrict__ tile_cfg,
             const int *__restrict__ active, int parity, int order) {
    // The tile order is a schedule choice: every tile is independent. The odd
    // half-sweep takes the tiles from the other end, so that it starts on the
    // links that the even one touched last, still in the last-level cache
    // (256 MB), and the next even one on those of the odd one. Half-sweep at
    // 40^4 in float (737 MB) 276 -> 248 us, at 32^4 in double (604 MB)
    // 212 -> 194 us. Counted within each XCD, so that a field that fits the
    // L2s meets every tile on the XCD that held it.
    const int b = parity ? xcd_reverse(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int tile = order ? xcd_tile(b, gridDim.x) : b;
    const int c = tile_cfg[tile];
    if (!active[c]) return;
    const CfgDesc d = desc[c];
    const int h = (tile - d.tile0) * (int)(blockDim.x / LPS) + (int)(threadIdx.x / LPS);
    if (h >= d.g.Vh) return;
    or_site<R, NE, LPS, NT, RU>(d, parity, h, threadIdx.x % LPS);
}

template <typename R, int NE, int LPS, bool NT>
static hipError_t launch_t(const Schedule &s, const CfgDesc *d_desc, const int *d_tile_cfg,
                           const int *d_active, int ntiles, int parity, int reunit, hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
    if (reunit)
        hipLaunchKernelGGL((k_half_sweep<R, NE, LPS, NT, true>), dim3(ntiles), dim3(s.block), s.lds, st,
                           d_desc, d_tile_cfg, d_active, parity, s.order);
    else
        hipLaunchKernelGGL((k_half_sweep<R, NE, LPS, NT, false>), dim3(ntiles), dim3(s.block), s.lds, st,
                           d_desc, d_tile_cfg, d_active, parity, s.order);
    return hipGetLastError();
}

template <typename R, int NE>
static hipError_t launch_lps(const Schedule &s, const CfgDesc *d_desc, const int *d_tile_cfg,
                             const int *d_active, int ntiles, int parity, int reunit, hipStream_t st) {
#define GF_CASE(L)                                                                                  \
    case L:                                                                                         \
        return s.nt ? launch_t<R, NE, L, true>(s, d_desc, d_tile_cfg, d_active, ntiles, parity,    \
                                               reunit, st)                                          \
                    : launch_t<R, NE, L, false>(s, d_desc, d_tile_cfg, d_active, ntiles, parity,   \
                                                reunit, st);
    switch (s.lps) {
        GF_CASE(1)
        GF_CASE(2)
        GF_CASE(4)
        GF_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef GF_CASE
}

hipError_t launch_half_sweep(int prec, int nelem, const Schedule &s, const CfgDesc *d_desc,
                             const int *d_tile_cfg, const int *d_active, int ntiles, int parity,
                             int reunit, hipStream_t st) {
#define GF_S3(R)                                                                                  \
    (nelem == 9   ? launch_lps<R, 9>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st)     \
     : nelem == 6 ? launch_lps<R, 6>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st)     \
                  : launch_lps<R, 4>(s, d_desc, d_tile_cfg, d_active, ntiles, parity, reunit, st))
    const hipError_t e = prec == 0 ? GF_S3(double) : GF_S3(float);
#undef GF_S3
    return e;
}

}  // namespace gf
