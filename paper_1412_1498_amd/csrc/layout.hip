// layout.hip -- conversion between the canonical [t][z][y][x][mu][r][c]
// link layout and the even/odd, element-major layout of the kernels
// (section "Implementation"), the same for algebra fields [t][z][y][x][a] <->
// [a][p][h], and standalone reunitarisation.
#include "pack_tile.hpp"
#include "su3_device.hpp"

namespace gf {

// One workgroup per tile of PackTile::TH half indices; a lane per link between
// LDS and the blocked layout. Packing zeroes the rest of a parity's last
// block.
template <typename R, int NE, bool UNPACK>
__global__ void __launch_bounds__(PACK_BLOCK) k_pack(Geom g, typename V2<R>::type *__restrict__ aos,
                                                     typename V2<R>::type *__restrict__ U) {
    typedef typename V2<R>::type v2;
    typedef PackTile<v2, 36> T;
    __shared__ v2 lds[T::SIZE];
    const int h0 = (int)blockIdx.x * T::TH;
    const int sites = 2 * max(0, min(T::TH, g.Vh - h0));
    v2 *run = aos + 72LL * h0;
    if (!UNPACK) T::fill(lds, run, sites);
#pragma unroll
    for (int l = threadIdx.x; l < 8 * T::TH; l += PACK_BLOCK) {
        const int q = l / T::TH, h = l % T::TH, p = q >> 2, mu = q & 3;
        const long long off = link_off(g, mu, p, h0 + h);
        const bool in = 2 * h < sites;
        v2 *at = lds + (pack_side(g, p, h0 + h) * T::TH + h) * T::STRIDE + 9 * mu;
        Mat<R> m;
        if (UNPACK) {
            if (!in) continue;
            load_link<R, NE, false>(m, as_global((const void *)U), off);
#pragma unroll
            for (int e = 0; e < 9; e++) at[e] = v2{m.re[e], m.im[e]};
        } else if (in) {
#pragma unroll
            for (int e = 0; e < 9; e++) {
                const v2 v = at[e];
                m.re[e] = v.x;
                m.im[e] = v.y;
            }
            store_link<R, NE, false>(m, as_global((void *)U), off);
        } else {
#pragma unroll
            for (int e = 0; e < NE; e++) U[off + e * BLK] = v2{R(0), R(0)};
        }
    }
    if (UNPACK) T::drain(lds, run, sites);
}

// One lane per (mu, site) link.
template <typename R, int NE>
__global__ void __launch_bounds__(256) k_reunit(Geom g, typename V2<R>::type *__restrict__ U) {
    const long long l = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= 4LL * g.V) return;
    const int mu = (int)(l / g.V);
    const int n = (int)(l - (long long)mu * g.V);
    const int p = n >= g.Vh, h = n - p * g.Vh;
    const long long off = link_off(g, mu, p, h);
    Mat<R> m;
    load_link<R, NE, false>(m, as_global((const void *)U), off);
    reunitarise(m);
    store_link<R, NE, false>(m, as_global((void *)U), off);
}

// Canonical s[site][a] <-> internal s[a][p][h]: the tiles of k_pack, a lane per
// site between LDS and the blocked layout. Packing zeroes the rest of a
// parity's last block.
template <typename R, bool UNPACK>
__global__ void __launch_bounds__(PACK_BLOCK) k_pack_alg(Geom g, R *__restrict__ aos, R *__restrict__ s) {
    typedef PackTile<R, 8> T;
    __shared__ R lds[T::SIZE];
    const int h0 = (int)blockIdx.x * T::TH;
    const int sites = 2 * max(0, min(T::TH, g.Vh - h0));
    R *run = aos + 16LL * h0;
    if (!UNPACK) T::fill(lds, run, sites);
#pragma unroll
    for (int l = threadIdx.x; l < 16 * T::TH; l += PACK_BLOCK) {
        const int q = l / T::TH, h = l % T::TH, p = q >> 3, a = q & 7;
        const bool in = 2 * h < sites;
        R *at = lds + (pack_side(g, p, h0 + h) * T::TH + h) * T::STRIDE + a;
        R *field = s + alg_off(g, p, h0 + h, a);
        if (!UNPACK) *field = in ? *at : R(0);
        else if (in) *at = *field;
    }
    if (UNPACK) T::drain(lds, run, sites);
}

hipError_t launch_pack(int prec, int nelem, const Geom &g, const void *aos, void *U, int unpack,
                       hipStream_t st) {
#define GF_U(R, NE, UN)                                                                          \
    hipLaunchKernelGGL((k_pack<R, NE, UN>), dim3(g.nb * (BLK / PackTile<V2<R>::type, 36>::TH)),  \
                       dim3(PACK_BLOCK), 0, st, g, (V2<R>::type *)aos, (V2<R>::type *)U)
#define GF_L(R, NE) do { if (unpack) GF_U(R, NE, true); else GF_U(R, NE, false); } while (0)
    if (prec == 0) { if (nelem == 9) GF_L(double, 9); else if (nelem == 6) GF_L(double, 6); else GF_L(double, 4); }
    else { if (nelem == 9) GF_L(float, 9); else if (nelem == 6) GF_L(float, 6); else GF_L(float, 4); }
#undef GF_L
#undef GF_U
    return hipGetLastError();
}

hipError_t launch_reunit(int prec, int nelem, const Geom &g, void *U, hipStream_t st) {
    const long long n = 4LL * g.V;
    const int B = 256;
    const dim3 grid((unsigned)((n + B - 1) / B));
#define GF_L(R, NE) \
    hipLaunchKernelGGL((k_reunit<R, NE>), grid, dim3(B), 0, st, g, (typename V2<R>::type *)U)
    if (prec == 0) { if (nelem == 9) GF_L(double, 9); else if (nelem == 6) GF_L(double, 6); else GF_L(double, 4); }
    else { if (nelem == 9) GF_L(float, 9); else if (nelem == 6) GF_L(float, 6); else GF_L(float, 4); }
#undef GF_L
    return hipGetLastError();
}

hipError_t launch_pack_alg(int prec, const Geom &g, const void *aos, void *s, int unpack,
                           hipStream_t st) {
#define GF_L(R, UN)                                                                              \
    hipLaunchKernelGGL((k_pack_alg<R, UN>), dim3(g.nb * (BLK / PackTile<R, 8>::TH)),             \
                       dim3(PACK_BLOCK), 0, st, g, (R *)aos, (R *)s)
    if (prec == 0) { if (unpack) GF_L(double, true); else GF_L(double, false); }
    else { if (unpack) GF_L(float, true); else GF_L(float, false); }
#undef GF_L
    return hipGetLastError();
}

}  // namespace gf
