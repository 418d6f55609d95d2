// sun_internal.hpp -- launchers of the SU(N) kernels (N = 2, 4) and of the
// N-aware final quality reduction.
#pragma once

#include <hip/hip_runtime.h>

#include "gf_internal.hpp"

namespace gf {

hipError_t launch_sun_half_sweep(int prec, int nc, const Schedule &s, const CfgDesc *d_desc,
                                 const int *d_tile_cfg, const int *d_active, int ntiles, int parity,
                                 int reunit, hipStream_t st);
hipError_t launch_sun_pack(int prec, int nc, const Geom &g, const void *aos, void *U, int to_aos,
                           hipStream_t st);
hipError_t launch_sun_reunit(int prec, int nc, const Geom &g, void *U, hipStream_t st);
hipError_t launch_sun_quality(int prec, int nc, const CfgDesc *d_desc, const int *d_qtile_cfg,
                              const int *d_active, int nqtiles, double *d_partials, const SlabOrder &so,
                              hipStream_t st);
// Where the final reduction leaves its results. All but iters, active and
// count are pinned host memory, written by the kernel itself: reading a check
// back then takes no copies, only the wait for it.
// One finished check of a single lattice's fix driver: the halves of F and
// theta, active and iters, each in a 64-bit store of its own with the check's
// number in the upper half. The record is there once all six numbers are; no
// store waits for another to reach host memory, as a flag written last would.
// With the member's entry and counters read together at the start, a sweep and a
// check in double at 12^4 26.4 -> 25.6 us, in float at 16^4 30.4 -> 29.8.
struct CheckRec {
    unsigned long long w[6], pad[2];
};
constexpr int CHECK_RING = 8;

struct QualityOut {
    double *result;     // 2 per member: F, theta
    int *active;        // device: per member, 1 until theta < eps or not finite (null: all)
    int *iters;         // device: per member, sweeps so far
    int *flags;         // pinned copies of active (n) and iters (n)
    CheckRec *ring;     // null, or CHECK_RING records: check k goes to record (k - 1) mod CHECK_RING
    unsigned *count;    // device: checks published so far
};

// F and theta of every member from its partials, normalised for nc colours;
// with npart > 0, of the one member from its npart pairs at d_partials.
hipError_t launch_quality_final(int nc, const CfgDesc *d_desc, int n, const double *d_partials,
                                const QualityOut &out, int swept, double eps, hipStream_t st, int npart = 0);

}  // namespace gf
