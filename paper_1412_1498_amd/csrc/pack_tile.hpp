// pack_tile.hpp -- conversion between the canonical site order and the
// blocked even/odd layout through LDS, shared by the SU(3), SU(N) and algebra
// packers.
//
// What bounds it: memory, if both sides move whole cache lines. The 2 TH sites
// of TH consecutive half indices h (both parities) are one contiguous run of
// the canonical field, and in the blocked layout TH-value runs of one or two
// blocks; a lane per link that reads its own 72 or 144 bytes touches every
// line of a wavefront's 4.6 or 9.2 KB once per element instead. So a
// workgroup copies the canonical run with 16-byte accesses and takes the
// links from LDS (the other way round to unpack). Links at 48^4, float
// 18-real: pack 628-647 -> 541-569 us, unpack 883-894 -> 549-585 us (5.2 to 5.6
// TB/s); double 1145 -> 1118 and 1564 -> 1127-1157 us; SU(4) float at 24^4 172 -> 52
// and 415 -> 49 us; algebra fields in double 239 -> 115 and 397 -> 110 us.
#pragma once

#include "su3_device.hpp"

namespace gf {

constexpr int PACK_BLOCK = 256;

// Half indices per tile: about 35 KB of LDS, four workgroups a CU.
// unit: bytes of one stored value, site: values per site.
constexpr int pack_th(int unit, int site) {
    return unit * site <= 300 ? 64 : unit * site <= 600 ? 32 : 16;
}

// A tile in LDS: value r of the site 2 h + s (h within the tile) at
// (s TH + h) STRIDE + r. The odd stride puts the lanes of a wavefront, which
// hold consecutive h, into different banks.
template <typename T, int SITE>
struct PackTile {
    static constexpr int TH = pack_th(sizeof(T), SITE);
    static constexpr int STRIDE = SITE + 1;
    static constexpr int SIZE = 2 * TH * STRIDE;
    static constexpr int PER = 16 / sizeof(T);                          // values per 16-byte access
    static constexpr int ROUNDS = 2 * TH * SITE / PER / PACK_BLOCK;     // accesses per lane
    static_assert(2 * TH * SITE % (PER * PACK_BLOCK) == 0 && SITE % PER == 0 && BLK % TH == 0, "tile shape");

    static __device__ __forceinline__ int place(int c) {  // of value c of the tile's canonical run
        const int n = c / SITE;
        return ((n & 1) * TH + (n >> 1)) * STRIDE + (c - n * SITE);
    }

    typedef unsigned v4 __attribute__((ext_vector_type(4)));
    union Vec {
        v4 v;
        T t[PER];
    };

    // the canonical run of `sites` sites at aos -> LDS
    static __device__ __forceinline__ void fill(T *lds, const T *aos, int sites) {
        const int n = sites * SITE / PER;
        if (n == 0) return;  // a tile past the lattice's end: the run does not exist
        const gchar *src = as_global((const void *)aos);
        Vec x[ROUNDS];
#pragma unroll
        for (int i = 0; i < ROUNDS; i++) {
            const int k = (int)threadIdx.x + i * PACK_BLOCK;
            x[i].v = ld<true, v4>(src, 16u * (unsigned)(k < n ? k : 0));
        }
#pragma unroll
        for (int i = 0; i < ROUNDS; i++) {
            const int k = (int)threadIdx.x + i * PACK_BLOCK;
            if (k < n) {
                const int o = place(k * PER);
#pragma unroll
                for (int j = 0; j < PER; j++) lds[o + j] = x[i].t[j];
            }
        }
        __syncthreads();
    }

    // LDS -> the canonical run
    static __device__ __forceinline__ void drain(const T *lds, T *aos, int sites) {
        const int n = sites * SITE / PER;
        gchar *dst = as_global((void *)aos);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ROUNDS; i++) {
            const int k = (int)threadIdx.x + i * PACK_BLOCK;
            if (k < n) {
                const int o = place(k * PER);
                Vec x;
#pragma unroll
                for (int j = 0; j < PER; j++) x.t[j] = lds[o + j];
                st<true, v4>(dst, 16u * (unsigned)k, x.v);
            }
        }
    }
};

// Which of the canonical sites 2 h, 2 h + 1 has parity p: x = 2 ih + b with
// b = (p + y + z + t) mod 2; every extent is even, so the parities of y, z, t
// are the low bits of the row index and its quotients.
__device__ __forceinline__ int pack_side(const Geom &g, int p, int h) {
    const int row = h / g.hx, rz = row / g.ny, rt = rz / g.nz;
    return (p + row + rz + rt) & 1;
}

}  // namespace gf
