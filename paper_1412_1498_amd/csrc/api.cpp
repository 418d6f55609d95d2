// api.cpp -- the C ABI of libgf (declared in include/gf.h): contexts,
// argument validation, the Alg. 1 drivers for one lattice and for ensembles
// (with hipGraph replay of a check period), the schedule autotuner and
// kernel timing. All device work goes to the context's stream.
#include <hip/hip_runtime.h>
#include <sched.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <map>
#include <sstream>
#include <string>
#include <tuple>
#include <vector>

#include "gf.h"
#include "gf_internal.hpp"
#include "fft.hpp"
#include "gf_math.hpp"
#include "link8.hpp"
#include "sun_internal.hpp"

using namespace gf;

// Hash of the library's sources, set by the build; keys autotuner cache
// entries so that a schedule measured on other kernels is not reused.
#ifndef GF_SOURCE_HASH
#define GF_SOURCE_HASH "unknown"
#endif

struct gf_ctx {
    int n = 0;
    int prec = 0;
    int nc = 3;                      // colours: 3, or 2 / 4 (SU(N) kernels)
    int nelem = 9;
    int device = 0;
    hipStream_t stream = nullptr;
    gf_params p{};
    std::vector<CfgDesc> desc;       // host copy of the member table
    CfgDesc *d_desc = nullptr;
    CfgDesc *h_stage = nullptr;      // pinned staging for table uploads
    hipEvent_t stage_evt = nullptr;  // last upload from h_stage
    int *d_tile_cfg = nullptr;
    int tile_cap = 0;
    int ntiles = 0;
    int *d_qtile_cfg = nullptr;
    int nqtiles = 0;
    SlabOrder qslab{0, 0, 0, 0, 0};  // quality tile order (single lattices only)
    bool qstream = false;            // F/theta by k_quality_tstream (single SU(3) lattices)
    double *d_partials = nullptr;
    int *d_active = nullptr;         // per member (fix drivers)
    int *d_ones = nullptr;           // per member, all 1 (plain calls)
    int *d_iters = nullptr;
    unsigned *d_count = nullptr;     // checks published to the ring
    double *h_result = nullptr;      // pinned, written by the kernels: 2n results
    int *h_flags = nullptr;          // pinned: n active, n iters (written by the kernels), n ones, n zeros, 1 count
    CheckRec *ring = nullptr;        // pinned, written by the kernels: last checks of a single lattice
    unsigned checks = 0;             // number of the last check taken from the ring
    Schedule sched{};
    long long sweeps_done = 0;
    std::string err;
    // timing
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_busy, ev_free;
    // graphs of check periods, keyed by (sweeps, reunit pattern, bits of eps):
    // eps is a kernel argument of the captured final reduction
    std::map<std::tuple<int, unsigned long long, unsigned long long>, std::pair<hipGraph_t, hipGraphExec_t>> graphs;
    hipStream_t cap_stream = nullptr;
    // differentiation scratch: g field (9 complex per site) and partials
    void *d_gfield = nullptr;
    double *d_fpart = nullptr;
    // Fourier-accelerated steepest descent: the half spectrum of the su(3)
    // components of Delta, and the tables of roots of unity for the x, y, z
    // and t lengths (FFT_MAX_N complex doubles each), then their 4 sin^2(pi m / L)
    void *d_spec = nullptr;
    double *d_sdpart = nullptr;      // F and theta's partials of the Delta pass
    void *d_roots = nullptr;
    // per-time-slice quality: partials and results
    double *d_slice_part = nullptr;
    double *d_slice_out = nullptr;
    // per-check JSON-lines log of the fix drivers (gf_params.log_path)
    std::string log_path;
    FILE *log = nullptr;
    long long log_calls = 0;
};

namespace {

int fail(gf_ctx *ctx, int code, const char *fmt, ...) {
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        ctx->err = buf;
    }
    return code;
}

#define HIPTRY(ctx, call)                                                                        \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return fail(ctx, GF_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_));         \
    } while (0)

#define CHECK(ctx, cond, code, ...)                                                              \
    do {                                                                                         \
        if (!(cond)) return fail(ctx, code, __VA_ARGS__);                                        \
    } while (0)

// ---- per-check log (gf_params.log_path) ----------------------------------
// One JSON object per line and per member at every F/theta evaluation of a
// fix driver: the driver ("alg1" overrelaxation, "alg2" Fourier-accelerated
// steepest descent), the driver call's number within the context, the
// member, its sweeps (steps) so far in this call, F, theta and the seconds
// since the call began. Appended to the file, flushed after every check.
using Clock = std::chrono::steady_clock;

void log_open(gf_ctx *ctx) {
    if (!ctx->log && !ctx->log_path.empty()) ctx->log = std::fopen(ctx->log_path.c_str(), "a");
}

void log_check(gf_ctx *ctx, bool sd, int member, long long iters, double F, double theta,
               Clock::time_point t0) {
    if (!ctx->log) return;
    const double el = std::chrono::duration<double>(Clock::now() - t0).count();
    std::fprintf(ctx->log,
                 "{\"driver\": \"%s\", \"call\": %lld, \"member\": %d, \"%s\": %lld, \"F\": %.17g, "
                 "\"theta\": %.17g, \"elapsed_s\": %.9f}\n",
                 sd ? "alg2" : "alg1", ctx->log_calls, member, sd ? "step" : "sweep", iters, F, theta, el);
}

void log_flush(gf_ctx *ctx) {
    if (ctx->log) std::fflush(ctx->log);
}

// Make the context's device current for the duration of a call.
struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) (void)hipSetDevice(dev);
        else prev = -1;
    }
    ~DeviceGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

size_t csize(const gf_ctx *c) { return c->prec == GF_F64 ? 16 : 8; }

int check_dims(gf_ctx *ctx, const int *d) {
    CHECK(ctx, d != nullptr, GF_EINVAL, "dims is NULL");
    long long V = 1;
    for (int i = 0; i < 4; i++) {
        CHECK(ctx, d[i] >= 2 && d[i] % 2 == 0, GF_EINVAL,
              "dims[%d] = %d: every lattice dimension must be even and >= 2", i, d[i]);
        V *= d[i];
    }
    CHECK(ctx, 4 * V < (1LL << 31), GF_EINVAL, "lattice volume %lld too large (4V must fit 31 bits)", V);
    return GF_OK;
}

int check_field(gf_ctx *ctx, const void *U, const char *what) {
    CHECK(ctx, U != nullptr, GF_EINVAL, "%s is NULL", what);
    CHECK(ctx, (reinterpret_cast<uintptr_t>(U) & 15) == 0, GF_EINVAL,
          "%s must be at least 16-byte aligned", what);
    return GF_OK;
}

int check_omega(gf_ctx *ctx, double omega) {
    CHECK(ctx, std::isfinite(omega) && omega > 0.0 && omega < 2.0, GF_EINVAL,
          "omega = %g must lie in (0, 2)", omega);
    return GF_OK;
}

// Dynamic LDS that leaves room for three 128-thread workgroups on a CU
// (160 KB): the occupancy limit of the sweep on fields beyond the
// last-level cache.
constexpr int SWEEP_LDS_3WG = 54272;

// Occupancy limit for a schedule: six waves a CU for full and 12-real SU(3)
// links in 128-thread workgroups once the fields are larger than the
// last-level cache. More waves in flight only spread the accesses over more
// DRAM pages and evict what the other half-sweep left in that cache: float
// 18-real 48^4 563 -> 534 us, 12-real 354 -> 334 us, double 32^4 195 -> 191,
// 48^4 1153 -> 1121 us. 8-real links, whose waves compute longer, lose by it
// (float 48^4 261 -> 378 us).
int sweep_lds(const Schedule &s, int nc, int nelem, double bytes) {
    return nc == 3 && nelem != 4 && s.block == 128 && bytes > 230e6 ? SWEEP_LDS_3WG : 0;
}

// Default schedule by lattice size (`sites` and `bytes` of all members), from
// sweeps over every lane count, workgroup size, access kind and tile order on
// lattices from 4^4 to 48^4 in all six forms of SU(3) links (the lines are within
// 2 % of the best schedule there in the geometric mean) and over access kinds
// and orders up to 80^4.
// `most` and `hx`: bytes of the largest member and its half extent in x.
Schedule default_schedule(int prec, int nc, int nelem, int n, double sites, double bytes, double most, int hx,
                          const gf_params &p) {
    Schedule s{};
    const bool f64 = prec == GF_F64, c8 = nc == 3 && nelem == 4;
    const double half = 0.5 * sites;
    if (nc != 3) {
        // SU(4) links need two lanes a site (registers), four while that fills
        // the chip better (8^4 in float 9.9 us with two, 8.2 us with four);
        // SU(2) one, two on few sites and in double. The rest as for SU(3)
        // below: SU(4) in float at 24^4 64 us plain in XCD shares, 75 us
        // streaming; at 16^4 (34 MB) 16.0 and 14.5 us; at 32^4 189 us plain in
        // dispatch order, 201 us streaming in shares.
        if (nc == 4) s.lps = half * 4 <= 512 * 64 ? 4 : 2;
        else s.lps = f64 || half * 2 <= 1024 * 64 ? 2 : 1;
        s.block = bytes <= 230e6 ? 64 : 128;
        // SU(4) from about 1 GB on shares again (in double 36^4 648 -> 616 us; SU(2)
        // in double 48^4 475 us in dispatch order, 499 in shares), both from 2 GB on
        // streaming (SU(4) 48^4 1964 -> 1837 us).
        s.nt = (bytes > 16e6 && bytes < (nc == 4 ? 70e6 : 48e6)) || bytes > 2.2e9;
        s.order = n == 1 && (bytes <= 230e6 || (nc == 4 && bytes > 1.2e9));
    } else if (bytes <= 230e6) {
        // Fields in the last-level cache. Few sites: more lanes a site shorten
        // a wave's work while the chip has idle SIMDs anyway (1024 of them);
        // 8-real lanes have the coding of their links to share as well. 8^4
        // in double 7.4 us with one lane, 5.5 us with four; 8-real 10.7 us with
        // one, 5.6 us with eight. From there two lanes, whose waves fit
        // two or three to a SIMD (double 20^4 32.9 -> 29.2 us), except float
        // 12-real links beyond 1.2e5 sites, where one lane fits twice as well.
        // Tiles in contiguous XCD shares: neighbouring tiles share the cache
        // lines at their seams (22x18x26x30 float 31.5 -> 29.0 us).
        if (c8) s.lps = half * 8 <= 512 * 64 ? 8 : half * 4 <= 1024 * 64 ? 4 : 2;
        else s.lps = half * 4 <= 512 * 64 ? 4 : 2;
        s.block = half * s.lps <= 4096 * 64 ? 64 : 128;
        if (!f64 && nelem == 6 && half > 60000) { s.lps = 1; s.block = 256; }
        // streaming access only just above the L2s (32 MB), which plain access
        // keeps filled with lines that are evicted before their next use:
        // double 16^4 13.7 us plain, 11.6 us streaming
        s.nt = bytes > 16e6 && bytes < 48e6;
        s.order = n == 1;  // an ensemble's members converge one by one and would empty their XCD's share
    } else if (c8) {
        s.lps = f64 ? 2 : 1;
        s.block = f64 ? 64 : 128;
        s.nt = 0;
        s.order = 0;
    } else {
        // Plain access keeps the end of one half-sweep in the last-level cache for
        // the start of the next; the larger the field, the less that is of it, and
        // streaming access moves the rest a little faster. It does so best where
        // rows begin on whole 64-byte pieces (half extent in x a multiple of 8 in
        // float), and not at all where the half extent is odd: runs of neighbouring
        // rows then begin inside a 32-byte sector, which streaming likely fetches
        // twice. A sweep with a check in ten, plain and streaming:
        //   float   18-real 48^4 (1.5 GB) 1126 and 1137 us, 48^3 x 96 (3.1 GB) 2337 and
        //           2278, 64^4 (4.8 GB) 3676 and 3474; on half pieces 56^4 (2.8 GB)
        //           2147 and 2247, 56x64x56x64 (3.7 GB) 2855 and 2927, 72^4 (7.7 GB)
        //           6513 and 6208; odd 66^4 (5.5 GB) 4590 and 4966
        //           12-real 72^4 (5.2 GB) 3777 and 4182, 80^4 (7.9 GB) 5782 and 6103
        //   double  18-real 48^4 (3.1 GB) 2371, two lanes streaming in shares 2324; odd
        //           54^4 (4.9 GB) 4643 and 4179, one lane streaming 4097
        //           12-real 60^4 (5.0 GB) 3702 and 4062, 64^4 (6.4 GB) 4788 and 4572
        // An ensemble is judged over its run, in which the small members retire
        // early and the largest works on alone: in float it takes that one's access
        // (48^3 x 96 and 64 small lattices to 1e-7, 5.4 GB: one lane streaming 5.86 s,
        // plain 5.93, two lanes plain 6.07); in double (7.8 GB, a sweep with all
        // members active and with the largest alone) one lane streaming takes 6746 and
        // 4782 us, two lanes 6788 and 4827.
        const bool full = nelem == 9, even = hx % 2 == 0;
        s.lps = f64 ? 2 : 1;
        s.block = 128;
        if (!f64) {
            s.nt = full && (hx % 8 == 0 ? most > 2.2e9 : even && n == 1 && bytes > 5e9);
        } else if (n > 1) {
            if (bytes > 2.2e9) { s.lps = 1; s.nt = 1; }
        } else if (full && bytes > 2.2e9) {
            s.lps = even ? 2 : 1;
            s.nt = 1;
            s.order = even;
        } else {
            s.nt = !full && even && bytes > 5.5e9;
        }
        // What plain access leaves in the cache to be written back, a check behind
        // every sweep pays for (48^4 in float: a check 375 us, 268 after a streaming
        // sweep), and a sweep's gain is less than that from some 600 MB on where rows
        // begin on whole sectors: with a check each, float 48^4 1458 us plain, 1404
        // streaming, 12-real 968 and 926, double 32^4 548 and 521, 40^4 1454 and 1404;
        // float 36^4 (0.5 GB) 459 and 473, 44^4 (half sectors) 1039 and 1056.
        const bool asked = p.lanes_per_site > 0 || p.block_threads > 0 || p.nontemporal >= 0 || p.tile_order >= 0;
        s.nt_check = n == 1 && hx % (f64 ? 2 : 4) == 0 && bytes > 6e8 && !asked;
    }
    if (p.lanes_per_site > 0) s.lps = p.lanes_per_site;
    if (p.block_threads > 0) s.block = p.block_threads;
    if (p.nontemporal >= 0) s.nt = p.nontemporal;
    if (p.tile_order >= 0) s.order = p.tile_order;
    s.lds = sweep_lds(s, nc, nelem, bytes);
    s.nt_check |= s.nt;
    return s;
}

// The same for n lattices of the given extents.
Schedule schedule_of(int prec, int nc, int nelem, int n, const int *dims, const gf_params &p) {
    double sites = 0.0, bytes = 0.0, most = 0.0;
    int hx = 0;
    for (int c = 0; c < n; c++) {
        const Geom g = make_geom(dims + 4 * c, nelem);
        const double b = (double)field_complex(g) * (prec == GF_F64 ? 16 : 8);
        sites += g.V;
        bytes += b;
        if (b > most) { most = b; hx = g.hx; }
    }
    return default_schedule(prec, nc, nelem, n, sites, bytes, most, hx, p);
}

int links_stored(int nc, int storage) {
    return nc != 3 ? nc * nc : storage == GF_STORE_12 ? 6 : storage == GF_STORE_8 ? 4 : 9;
}

int check_schedule(gf_ctx *ctx, const Schedule &s, int nc) {
    CHECK(ctx, s.lps == 1 || s.lps == 2 || s.lps == 4 || s.lps == 8, GF_EINVAL,
          "lanes_per_site = %d must be 1, 2, 4 or 8", s.lps);
    CHECK(ctx, nc != 4 || s.lps >= 2, GF_EINVAL, "SU(4) links need lanes_per_site >= 2");
    CHECK(ctx, s.block >= 64 && s.block <= 256 && s.block % 64 == 0, GF_EINVAL,
          "block_threads = %d must be 64, 128, 192 or 256", s.block);
    CHECK(ctx, s.order == 0 || s.order == 1, GF_EINVAL, "tile_order = %d must be 0 or 1", s.order);
    return GF_OK;
}

void destroy_graphs(gf_ctx *ctx) {
    for (auto &kv : ctx->graphs) {
        (void)hipGraphExecDestroy(kv.second.second);
        (void)hipGraphDestroy(kv.second.first);
    }
    ctx->graphs.clear();
}

// Upload the member table (after the previous upload from the staging
// buffer has been consumed).
int upload_desc(gf_ctx *ctx) {
    HIPTRY(ctx, hipEventSynchronize(ctx->stage_evt));
    std::memcpy(ctx->h_stage, ctx->desc.data(), ctx->n * sizeof(CfgDesc));
    HIPTRY(ctx, hipMemcpyAsync(ctx->d_desc, ctx->h_stage, ctx->n * sizeof(CfgDesc),
                               hipMemcpyHostToDevice, ctx->stream));
    HIPTRY(ctx, hipEventRecord(ctx->stage_evt, ctx->stream));
    return GF_OK;
}

// (Re)build the sweep tile map for the current schedule.
int build_tiles(gf_ctx *ctx) {
    const int spt = ctx->sched.block / ctx->sched.lps;
    std::vector<int> map;
    for (int c = 0; c < ctx->n; c++) {
        ctx->desc[c].tile0 = (int)map.size();
        const int nt = (ctx->desc[c].g.Vh + spt - 1) / spt;
        map.insert(map.end(), nt, c);
    }
    if ((int)map.size() > ctx->tile_cap) {
        if (ctx->d_tile_cfg) HIPTRY(ctx, hipFree(ctx->d_tile_cfg));
        ctx->d_tile_cfg = nullptr;
        if (hipMalloc(&ctx->d_tile_cfg, map.size() * sizeof(int)) != hipSuccess)
            return fail(ctx, GF_ENOMEM, "cannot allocate the tile map (%zu tiles)", map.size());
        ctx->tile_cap = (int)map.size();
    }
    ctx->ntiles = (int)map.size();
    HIPTRY(ctx, hipStreamSynchronize(ctx->stream));  // no launch may still read the old map
    HIPTRY(ctx, hipMemcpy(ctx->d_tile_cfg, map.data(), map.size() * sizeof(int), hipMemcpyHostToDevice));
    destroy_graphs(ctx);
    return upload_desc(ctx);
}

// Point the member table at the given fields / omegas, uploading only on change.
int set_fields(gf_ctx *ctx, void *const *U, const double *omega) {
    bool changed = false;
    for (int c = 0; c < ctx->n; c++) {
        if (ctx->desc[c].U != U[c]) { ctx->desc[c].U = U[c]; changed = true; }
        const double w = omega ? omega[c] : ctx->desc[c].omega;
        if (ctx->desc[c].omega != w) { ctx->desc[c].omega = w; changed = true; }
    }
    if (changed) return upload_desc(ctx);
    return GF_OK;
}

int half_sweep(gf_ctx *ctx, int parity, int reunit, const int *d_active) {
    std::pair<hipEvent_t, hipEvent_t> ev{nullptr, nullptr};
    if (ctx->p.timing) {
        if (ctx->ev_free.empty()) {
            HIPTRY(ctx, hipEventCreate(&ev.first));
            HIPTRY(ctx, hipEventCreate(&ev.second));
        } else {
            ev = ctx->ev_free.back();
            ctx->ev_free.pop_back();
        }
        HIPTRY(ctx, hipEventRecord(ev.first, ctx->stream));
    }
    if (ctx->nc == 3)
        HIPTRY(ctx, launch_half_sweep(ctx->prec, ctx->nelem, ctx->sched, ctx->d_desc, ctx->d_tile_cfg,
                                      d_active, ctx->ntiles, parity, reunit, ctx->stream));
    else
        HIPTRY(ctx, launch_sun_half_sweep(ctx->prec, ctx->nc, ctx->sched, ctx->d_desc, ctx->d_tile_cfg,
                                          d_active, ctx->ntiles, parity, reunit, ctx->stream));
    if (ctx->p.timing) {
        HIPTRY(ctx, hipEventRecord(ev.second, ctx->stream));
        ctx->ev_busy.push_back(ev);
    }
    return GF_OK;
}

bool reunit_due(const gf_ctx *ctx, long long sweep_index) {
    return ctx->p.reunit_every > 0 && sweep_index % ctx->p.reunit_every == 0;
}

// n full sweeps on `st` (the context stream, or a capture stream), with
// the reunitarisation schedule continuing from ctx->sweeps_done.
int full_sweeps(gf_ctx *ctx, int n, const int *d_active, hipStream_t st) {
    hipStream_t keep = ctx->stream;
    ctx->stream = st;
    int rc = GF_OK;
    for (int i = 0; i < n && rc == GF_OK; i++) {
        rc = half_sweep(ctx, 0, 0, d_active);
        if (rc == GF_OK) rc = half_sweep(ctx, 1, reunit_due(ctx, ctx->sweeps_done + 1) ? 1 : 0, d_active);
        if (rc == GF_OK) ctx->sweeps_done++;
    }
    ctx->stream = keep;
    return rc;
}

int quality_launch(gf_ctx *ctx, const int *d_active, int update, int swept, double eps, hipStream_t st) {
    if (ctx->qstream)
        HIPTRY(ctx, launch_quality_tstream(ctx->prec, ctx->nelem, ctx->desc[0].g, ctx->d_desc, d_active,
                                           ctx->d_partials, st));
    else if (ctx->nc == 3)
        HIPTRY(ctx, launch_quality(ctx->prec, ctx->nelem, ctx->d_desc, ctx->d_qtile_cfg, d_active,
                                   ctx->nqtiles, ctx->d_partials, ctx->qslab, st));
    else
        HIPTRY(ctx, launch_sun_quality(ctx->prec, ctx->nc, ctx->d_desc, ctx->d_qtile_cfg, d_active,
                                       ctx->nqtiles, ctx->d_partials, ctx->qslab, st));
    // pinned memory has one address on host and device
    const QualityOut out{ctx->h_result, update ? ctx->d_active : nullptr, ctx->d_iters, ctx->h_flags,
                         update && ctx->n == 1 ? ctx->ring : nullptr, ctx->d_count};
    HIPTRY(ctx, launch_quality_final(ctx->nc, ctx->d_desc, ctx->n, ctx->d_partials, out, swept, eps, st));
    return GF_OK;
}

struct Check {
    double F, theta;
    int active, iters;
};

// Check number `seq` of a single lattice, if all words of its record are there.
bool read_check(const gf_ctx *ctx, unsigned seq, Check *out) {
    const CheckRec &r = ctx->ring[(seq - 1) % CHECK_RING];
    unsigned v[6];
    for (int i = 0; i < 6; i++) {
        const unsigned long long w = __atomic_load_n(&r.w[i], __ATOMIC_RELAXED);
        if ((unsigned)(w >> 32) != seq) return false;
        v[i] = (unsigned)w;
    }
    const unsigned long long f = (unsigned long long)v[1] << 32 | v[0], t = (unsigned long long)v[3] << 32 | v[2];
    std::memcpy(&out->F, &f, sizeof f);
    std::memcpy(&out->theta, &t, sizeof t);
    out->active = (int)v[4];
    out->iters = (int)v[5];
    return true;
}

// The checks of a driver call are numbered past any record that a call before
// left behind when it failed.
int start_checks(gf_ctx *ctx) {
    int *count = ctx->h_flags + 4 * ctx->n;
    ctx->checks += CHECK_RING;
    *count = (int)ctx->checks;
    HIPTRY(ctx, hipMemcpyAsync(ctx->d_count, count, sizeof(int), hipMemcpyHostToDevice, ctx->stream));
    return GF_OK;
}

// Whether the process waits for its device by spinning (the runtime's default as
// well) or has asked for waits that leave the core to others.
bool waits_spin() {
    unsigned flags = 0;
    if (hipGetDeviceFlags(&flags) != hipSuccess) {
        (void)hipGetLastError();  // not the next launch's error
        return true;
    }
    return !(flags & (hipDeviceScheduleYield | hipDeviceScheduleBlockingSync));
}

// Wait for check number `seq`: by the runtime's own wait for the stream, or (watch)
// by watching its record, with the stream asked now and then, so that a failed
// launch ends the wait.
int wait_check(gf_ctx *ctx, unsigned seq, Check *out, bool watch) {
    if (!watch) {
        HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
        CHECK(ctx, read_check(ctx, seq, out), GF_EDEVICE, "a check's result is missing");
        return GF_OK;
    }
    for (long long spin = 0; !read_check(ctx, seq, out); spin++) {
        if (spin % 1024 != 1023) continue;
        const hipError_t e = hipStreamQuery(ctx->stream);
        if (e == hipErrorNotReady) {
            if (spin > 200000) sched_yield();  // a long period: let other threads run
            continue;
        }
        HIPTRY(ctx, e);
        CHECK(ctx, read_check(ctx, seq, out), GF_EDEVICE, "a check's result is missing");
        break;
    }
    return GF_OK;
}

int create_impl(gf_ctx **out, int n, const int *dims, const int *gauge, int prec, void *stream,
                const gf_params *pp, int nc) {
    if (!out) return GF_EINVAL;
    *out = nullptr;
    gf_ctx tmp;  // for error messages during validation
    if (n < 1) return GF_EINVAL;
    if (prec != GF_F64 && prec != GF_F32) return GF_EINVAL;
    for (int c = 0; c < n; c++) {
        if (check_dims(&tmp, dims + 4 * c) != GF_OK) return GF_EINVAL;
        if (gauge[c] != GF_LANDAU && gauge[c] != GF_COULOMB) return GF_EINVAL;
    }
    gf_params p;
    gf_params_default(&p, prec);
    if (pp) p = *pp;
    if (p.check_every < 1) p.check_every = 1;
    if (p.reunit_every < 0) return GF_EINVAL;
    if (p.storage != GF_STORE_18 && p.storage != GF_STORE_12 && p.storage != GF_STORE_8) return GF_EINVAL;
    if (nc != 3 && p.storage != GF_STORE_18) return GF_EUNSUPPORTED;  // 12-/8-real are SU(3) only
    const int nelem = links_stored(nc, p.storage);
    const Schedule s = schedule_of(prec, nc, nelem, n, dims, p);
    if (check_schedule(&tmp, s, nc) != GF_OK) return GF_EINVAL;

    gf_ctx *ctx = new gf_ctx();
    ctx->n = n;
    ctx->prec = prec;
    ctx->nc = nc;
    ctx->nelem = nelem;
    ctx->stream = (hipStream_t)stream;
    ctx->p = p;
    ctx->sched = s;
    ctx->sweeps_done = p.start_sweep;
    if (p.log_path) ctx->log_path = p.log_path;
    ctx->p.log_path = nullptr;  // the context keeps its own copy
    int rc = GF_OK;
    auto bail = [&](int code) { gf_destroy(ctx); return code; };
    if (hipGetDevice(&ctx->device) != hipSuccess) return bail(GF_EDEVICE);
    ctx->desc.resize(n);
    int nq = 0;
    for (int c = 0; c < n; c++) {
        CfgDesc &d = ctx->desc[c];
        std::memset(&d, 0, sizeof d);
        d.g = make_geom(dims + 4 * c, ctx->nelem);
        d.gauge = gauge[c];
        d.omega = 1.0;
        d.qtile0 = nq;
        d.nqtiles = (d.g.Vh + QTILE / 2 - 1) / (QTILE / 2);  // QTILE/2 half-indices, both parities
        nq += d.nqtiles;
    }
    ctx->nqtiles = nq;
    // Plain order for an ensemble, whose tiles are several lattices end to end, and
    // for fields up to 100 MB: in plain order an XCD walks the tiles that the sweep
    // before gave it, and finds in its L2 what slab blocks fetch from the last-level
    // cache. A sweep and a check, slabs -> plain order: double 16^4 (38 MB) 50.9 ->
    // 41.8 us, 20^4 (92 MB) 85.7 -> 84.7, float 20^4 (46 MB) 65 -> 58, 24^4 (96 MB)
    // 91.2 -> 91.0, SU(2) 24^4 (42 MB) 57 -> 48, SU(4) 16^4 (34 MB) 56 -> 47. Beyond,
    // nothing is left of it, and with the field out of the caches the slabs' fewer
    // reads count: 28^4 double (354 MB) 309 and 314, float 32^4 (302 MB) 259 and 278.
    const Geom &g0 = ctx->desc[0].g;
    const double bytes0 = (double)field_complex(g0) * 2 * (prec == GF_F64 ? 8 : 4);
    if (n == 1 && bytes0 > 100e6) {
        const int nd = ctx->desc[0].gauge == GF_LANDAU ? 4 : 3;
        const long long tile_bytes = (long long)QTILE * nd * ctx->nelem * 2 * (prec == GF_F64 ? 8 : 4);
        ctx->qslab = pick_slab_order(g0.st, g0.sz, g0.hx, g0.nz, QTILE / 2, nq, tile_bytes);
    }
    // in double a single lattice's F/theta walks time slices (its tiles' t neighbours
    // missed L2 in any slab order); in float the slab order is as fast
    ctx->qstream = n == 1 && ctx->nc == 3 && prec == GF_F64 && quality_tstream_ok(ctx->desc[0].g, nelem, ctx->desc[0].gauge);
    std::vector<int> qmap;
    for (int c = 0; c < n; c++) qmap.insert(qmap.end(), ctx->desc[c].nqtiles, c);
    if (hipMalloc(&ctx->d_desc, n * sizeof(CfgDesc)) != hipSuccess ||
        hipMalloc(&ctx->d_qtile_cfg, nq * sizeof(int)) != hipSuccess ||
        hipMalloc(&ctx->d_partials, 2 * (size_t)nq * sizeof(double)) != hipSuccess ||
        hipMalloc(&ctx->d_active, n * sizeof(int)) != hipSuccess ||
        hipMalloc(&ctx->d_ones, n * sizeof(int)) != hipSuccess ||
        hipMalloc(&ctx->d_iters, n * sizeof(int)) != hipSuccess ||
        hipMalloc(&ctx->d_count, sizeof(int)) != hipSuccess ||
        hipHostMalloc(&ctx->h_stage, n * sizeof(CfgDesc), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&ctx->h_result, 2 * n * sizeof(double), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&ctx->h_flags, (4 * n + 1) * sizeof(int), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&ctx->ring, CHECK_RING * sizeof(CheckRec), hipHostMallocDefault) != hipSuccess)
        return bail(GF_ENOMEM);
    if (hipEventCreateWithFlags(&ctx->stage_evt, hipEventDisableTiming) != hipSuccess ||
        hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking) != hipSuccess)
        return bail(GF_EDEVICE);
    for (int c = 0; c < n; c++) { ctx->h_flags[2 * n + c] = 1; ctx->h_flags[3 * n + c] = 0; }
    std::memset(ctx->ring, 0, CHECK_RING * sizeof(CheckRec));
    if (hipMemcpy(ctx->d_ones, ctx->h_flags + 2 * n, n * sizeof(int), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(ctx->d_active, ctx->h_flags + 2 * n, n * sizeof(int), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(ctx->d_qtile_cfg, qmap.data(), nq * sizeof(int), hipMemcpyHostToDevice) != hipSuccess)
        return bail(GF_EDEVICE);
    rc = build_tiles(ctx);
    if (rc != GF_OK) return bail(rc);
    if (hipStreamSynchronize(ctx->stream) != hipSuccess) return bail(GF_EDEVICE);
    *out = ctx;
    return GF_OK;
}

int need_single(gf_ctx *ctx) {
    CHECK(ctx, ctx->n == 1, GF_EINVAL, "this entry point needs a single-lattice context (n = %d)", ctx->n);
    return GF_OK;
}

// The su(3)-algebra entry points (differentiation, Fourier-accelerated
// steepest descent) exist for N = 3 only.
int need_su3(gf_ctx *ctx) {
    CHECK(ctx, ctx->nc == 3, GF_EUNSUPPORTED, "this entry point is implemented for SU(3) only (nc = %d)", ctx->nc);
    return GF_OK;
}

}  // namespace

extern "C" {

void gf_params_default(gf_params *p, int prec) {
    if (!p) return;
    std::memset(p, 0, sizeof *p);
    p->check_every = 1;
    p->reunit_every = prec == GF_F64 ? 20 : 10;
    p->start_sweep = 0;
    p->storage = GF_STORE_18;
    p->nontemporal = -1;
    p->tile_order = -1;
}

int gf_create(gf_ctx **out, const int dims[4], int nc, int gauge, int prec, void *stream,
              const gf_params *p) {
    if (!out) return GF_EINVAL;
    *out = nullptr;
    if (nc != 2 && nc != 3 && nc != 4) return GF_EUNSUPPORTED;
    return create_impl(out, 1, dims, &gauge, prec, stream, p, nc);
}

int gf_batch_create(gf_ctx **out, int n, const int *dims, const int *gauge, int prec, void *stream,
                    const gf_params *p) {
    if (!out) return GF_EINVAL;
    *out = nullptr;
    if (n < 1 || !dims || !gauge) return GF_EINVAL;
    return create_impl(out, n, dims, gauge, prec, stream, p, 3);
}

int gf_destroy(gf_ctx *ctx) {
    if (!ctx) return GF_OK;
    DeviceGuard dg(ctx->device);
    (void)hipStreamSynchronize(ctx->stream);
    destroy_graphs(ctx);
    for (auto &e : ctx->ev_busy) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
    for (auto &e : ctx->ev_free) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
    if (ctx->stage_evt) (void)hipEventDestroy(ctx->stage_evt);
    if (ctx->cap_stream) (void)hipStreamDestroy(ctx->cap_stream);
    (void)hipFree(ctx->d_desc);
    (void)hipFree(ctx->d_tile_cfg);
    (void)hipFree(ctx->d_qtile_cfg);
    (void)hipFree(ctx->d_partials);
    (void)hipFree(ctx->d_active);
    (void)hipFree(ctx->d_ones);
    (void)hipFree(ctx->d_iters);
    (void)hipFree(ctx->d_count);
    (void)hipFree(ctx->d_spec);
    (void)hipFree(ctx->d_sdpart);
    (void)hipFree(ctx->d_roots);
    (void)hipFree(ctx->d_gfield);
    (void)hipFree(ctx->d_fpart);
    if (ctx->h_stage) (void)hipHostFree(ctx->h_stage);
    if (ctx->h_result) (void)hipHostFree(ctx->h_result);
    if (ctx->h_flags) (void)hipHostFree(ctx->h_flags);
    if (ctx->ring) (void)hipHostFree(ctx->ring);
    (void)hipFree(ctx->d_slice_part);
    (void)hipFree(ctx->d_slice_out);
    if (ctx->log) std::fclose(ctx->log);
    delete ctx;
    return GF_OK;
}

int gf_batch_destroy(gf_ctx *ctx) { return gf_destroy(ctx); }

const char *gf_last_error(const gf_ctx *ctx) { return ctx ? ctx->err.c_str() : noalloc_last_error(); }

size_t gf_field_bytes(const gf_ctx *ctx, int member) {
    if (!ctx || member < 0 || member >= ctx->n) return 0;
    return (size_t)field_complex(ctx->desc[member].g) * csize(ctx);
}

int gf_pack(gf_ctx *ctx, const void *U_aos, void *U) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = check_field(ctx, U_aos, "U_aos")) || (rc = check_field(ctx, U, "U")))
        return rc;
    DeviceGuard dg(ctx->device);
    if (ctx->nc == 3)
        HIPTRY(ctx, launch_pack(ctx->prec, ctx->nelem, ctx->desc[0].g, U_aos, U, 0, ctx->stream));
    else
        HIPTRY(ctx, launch_sun_pack(ctx->prec, ctx->nc, ctx->desc[0].g, U_aos, U, 0, ctx->stream));
    return GF_OK;
}

int gf_unpack(gf_ctx *ctx, const void *U, void *U_aos) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = check_field(ctx, U_aos, "U_aos")) || (rc = check_field(ctx, U, "U")))
        return rc;
    DeviceGuard dg(ctx->device);
    if (ctx->nc == 3)
        HIPTRY(ctx, launch_pack(ctx->prec, ctx->nelem, ctx->desc[0].g, U_aos, const_cast<void *>(U), 1,
                                ctx->stream));
    else
        HIPTRY(ctx, launch_sun_pack(ctx->prec, ctx->nc, ctx->desc[0].g, U_aos, const_cast<void *>(U), 1,
                                    ctx->stream));
    return GF_OK;
}

int gf_sweep(gf_ctx *ctx, void *U, int parity, double omega) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = check_field(ctx, U, "U")) || (rc = check_omega(ctx, omega)))
        return rc;
    CHECK(ctx, parity == 0 || parity == 1, GF_EINVAL, "parity must be 0 or 1");
    DeviceGuard dg(ctx->device);
    if ((rc = set_fields(ctx, &U, &omega))) return rc;
    return half_sweep(ctx, parity, 0, ctx->d_ones);
}

int gf_sweeps(gf_ctx *ctx, void *U, double omega, int nsweeps) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = check_field(ctx, U, "U")) || (rc = check_omega(ctx, omega)))
        return rc;
    CHECK(ctx, nsweeps >= 0, GF_EINVAL, "nsweeps must be >= 0");
    DeviceGuard dg(ctx->device);
    if ((rc = set_fields(ctx, &U, &omega))) return rc;
    return full_sweeps(ctx, nsweeps, ctx->d_ones, ctx->stream);
}

int gf_reunit(gf_ctx *ctx, void *U) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = check_field(ctx, U, "U"))) return rc;
    DeviceGuard dg(ctx->device);
    if (ctx->nc == 3)
        HIPTRY(ctx, launch_reunit(ctx->prec, ctx->nelem, ctx->desc[0].g, U, ctx->stream));
    else
        HIPTRY(ctx, launch_sun_reunit(ctx->prec, ctx->nc, ctx->desc[0].g, U, ctx->stream));
    return GF_OK;
}

int gf_batch_quality(gf_ctx *ctx, void *const *U, double *F, double *theta) {
    if (!ctx) return GF_EINVAL;
    CHECK(ctx, U && F && theta, GF_EINVAL, "NULL argument");
    int rc;
    for (int c = 0; c < ctx->n; c++)
        if ((rc = check_field(ctx, U[c], "U[i]"))) return rc;
    DeviceGuard dg(ctx->device);
    if ((rc = set_fields(ctx, U, nullptr))) return rc;
    if ((rc = quality_launch(ctx, nullptr, 0, 0, 0.0, ctx->stream))) return rc;
    HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
    int bad = 0;
    for (int c = 0; c < ctx->n; c++) {
        F[c] = ctx->h_result[2 * c];
        theta[c] = ctx->h_result[2 * c + 1];
        if (!std::isfinite(F[c]) || !std::isfinite(theta[c])) bad = 1;
    }
    if (bad) return fail(ctx, GF_ENONFINITE, "F or theta is not finite");
    return GF_OK;
}

int gf_quality(gf_ctx *ctx, const void *U, double *F, double *theta) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx))) return rc;
    void *u = const_cast<void *>(U);
    return gf_batch_quality(ctx, &u, F, theta);
}

int gf_quality_slices(gf_ctx *ctx, const void *U, double *F_t, double *theta_t) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = need_su3(ctx)) || (rc = check_field(ctx, U, "U"))) return rc;
    CHECK(ctx, F_t && theta_t, GF_EINVAL, "NULL argument");
    DeviceGuard dg(ctx->device);
    const Geom &g = ctx->desc[0].g;
    if (!ctx->d_slice_part) {
        const size_t np = 2 * (size_t)g.nt * quality_slice_chunks(g);
        if (hipMalloc(&ctx->d_slice_part, np * sizeof(double)) != hipSuccess) {
            ctx->d_slice_part = nullptr;
            return fail(ctx, GF_ENOMEM, "cannot allocate the per-slice partials");
        }
    }
    if (!ctx->d_slice_out && hipMalloc(&ctx->d_slice_out, 2 * (size_t)g.nt * sizeof(double)) != hipSuccess) {
        ctx->d_slice_out = nullptr;
        return fail(ctx, GF_ENOMEM, "cannot allocate the per-slice results");
    }
    CfgDesc d = ctx->desc[0];
    d.U = const_cast<void *>(U);
    HIPTRY(ctx, launch_quality_slices(ctx->prec, ctx->nelem, d, ctx->d_slice_part, ctx->d_slice_out, ctx->stream));
    std::vector<double> h(2 * (size_t)g.nt);
    HIPTRY(ctx, hipMemcpyAsync(h.data(), ctx->d_slice_out, h.size() * sizeof(double), hipMemcpyDeviceToHost,
                               ctx->stream));
    HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
    bool bad = false;
    for (int t = 0; t < g.nt; t++) {
        F_t[t] = h[2 * t];
        theta_t[t] = h[2 * t + 1];
        if (!std::isfinite(F_t[t]) || !std::isfinite(theta_t[t])) bad = true;
    }
    if (bad) return fail(ctx, GF_ENONFINITE, "a slice's F or theta is not finite");
    return GF_OK;
}

int gf_fix(gf_ctx *ctx, void *U, double omega, double eps, int max_iter, int *iters, double *F,
           double *theta) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx))) return rc;
    return gf_batch_fix(ctx, &U, &omega, eps, max_iter, iters, F, theta);
}

int gf_batch_fix(gf_ctx *ctx, void *const *U, const double *omega, double eps, int max_iter,
                 int *iters, double *F, double *theta) {
    if (!ctx) return GF_EINVAL;
    CHECK(ctx, U && omega && iters && F && theta, GF_EINVAL, "NULL argument");
    CHECK(ctx, std::isfinite(eps) && eps >= 0.0, GF_EINVAL, "eps must be finite and >= 0");
    CHECK(ctx, max_iter >= 0, GF_EINVAL, "max_iter must be >= 0");
    int rc;
    for (int c = 0; c < ctx->n; c++) {
        if ((rc = check_field(ctx, U[c], "U[i]")) || (rc = check_omega(ctx, omega[c]))) return rc;
    }
    DeviceGuard dg(ctx->device);
    if ((rc = set_fields(ctx, U, omega))) return rc;
    const int n = ctx->n;
    const Clock::time_point t0 = Clock::now();
    log_open(ctx);
    ctx->log_calls++;
    // every member starts active with zero sweeps
    HIPTRY(ctx, hipMemcpyAsync(ctx->d_active, ctx->h_flags + 2 * n, n * sizeof(int), hipMemcpyHostToDevice, ctx->stream));
    HIPTRY(ctx, hipMemcpyAsync(ctx->d_iters, ctx->h_flags + 3 * n, n * sizeof(int), hipMemcpyHostToDevice, ctx->stream));
    if ((rc = start_checks(ctx))) return rc;
    if ((rc = quality_launch(ctx, ctx->d_active, 1, 0, eps, ctx->stream))) return rc;
    // members active before a check (those whose result it refreshed)
    std::vector<int> was_active(n, 1);
    auto log_members = [&]() {
        if (!ctx->log) return;
        for (int c = 0; c < n; c++)
            if (was_active[c])
                log_check(ctx, false, c, ctx->h_flags[n + c], ctx->h_result[2 * c], ctx->h_result[2 * c + 1], t0);
        log_flush(ctx);
        for (int c = 0; c < n; c++) was_active[c] = ctx->h_flags[c];
    };
    const bool graphs = ctx->p.use_graph && !ctx->p.timing && ctx->p.check_every <= 64;
    // the sweeps of a period: one alone with the access of a sweep between two checks
    auto sweeps = [&](int m, hipStream_t st) -> int {
        const int nt = ctx->sched.nt;
        if (m == 1) ctx->sched.nt = ctx->sched.nt_check;
        const int r = full_sweeps(ctx, m, ctx->d_active, st);
        ctx->sched.nt = nt;
        return r;
    };
    // one check period of m sweeps and its check, enqueued
    auto period = [&](int m) -> int {
        int r;
        if (!graphs) {
            if ((r = sweeps(m, ctx->stream))) return r;
            return quality_launch(ctx, ctx->d_active, 1, m, eps, ctx->stream);
        }
        unsigned long long pattern = 0;
        for (int k = 1; k <= m; k++)
            if (reunit_due(ctx, ctx->sweeps_done + k)) pattern |= 1ULL << (k - 1);
        unsigned long long eps_bits;
        std::memcpy(&eps_bits, &eps, sizeof eps_bits);
        auto key = std::make_tuple(m, pattern, eps_bits);
        auto f = ctx->graphs.find(key);
        if (f == ctx->graphs.end()) {
            hipGraph_t g;
            hipGraphExec_t ge;
            const long long keep = ctx->sweeps_done;
            HIPTRY(ctx, hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeThreadLocal));
            int r1 = sweeps(m, ctx->cap_stream);
            int r2 = r1 ? r1 : quality_launch(ctx, ctx->d_active, 1, m, eps, ctx->cap_stream);
            hipError_t ec = hipStreamEndCapture(ctx->cap_stream, &g);
            ctx->sweeps_done = keep;
            if (r2) return r2;
            HIPTRY(ctx, ec);
            HIPTRY(ctx, hipGraphInstantiate(&ge, g, nullptr, nullptr, 0));
            f = ctx->graphs.emplace(key, std::make_pair(g, ge)).first;
        }
        HIPTRY(ctx, hipGraphLaunch(f->second.second, ctx->stream));
        ctx->sweeps_done += m;
        return GF_OK;
    };
    auto nonfinite = [&]() {
        for (int c = 0; c < n; c++)
            if (!std::isfinite(ctx->h_result[2 * c]) || !std::isfinite(ctx->h_result[2 * c + 1])) return true;
        return false;
    };
    if (n == 1) {
        // The host stays one period ahead of the check it waits for: a check
        // that ends the run retires the lattice on the device, and the period
        // already enqueued finds it retired and does nothing. Only for short
        // periods, whose launches and read-back the GPU would wait for (4^4 in
        // double, 20 sweeps with a check each: 660 us without and 440 with); a
        // long one's launches hide behind the period itself. And not where the
        // next check will likely end the run, since launches that find the lattice
        // retired still take 3 us each: theta is taken to fall as it did in the
        // period before. With less than two checks to go by, five sweeps are the
        // most to be thrown away (a field fixed already, 4^4, check every 5, 16 and
        // 150 sweeps: 45, 45 and 45 us without, 68, 124 and 794 with; one period
        // of a run 108, 214 and 1561 without, 88, 195 and 1499 with).
        // The record is watched where the process's waits spin anyway; it is there some
        // 5 us before the runtime's own wait ends (32^4 12-real, a check every ten sweeps:
        // 2626 us for twenty, 2613 watched).
        const bool watch = waits_spin() && !ctx->p.timing;
        const bool brief = watch && (double)ctx->desc[0].g.V * ctx->p.check_every <= 4e6;
        double before = 0.0;  // theta of the check before the last
        int taken = 0;
        const long long sweeps0 = ctx->sweeps_done;
        int enqueued = 0, pending = 1;
        Check k{};
        auto ahead = [&]() {
            if (!brief || eps == 0.0) return brief;  // no theta is below 0: max_iter sweeps
            if (taken < 2) return ctx->p.check_every <= 5;
            return k.theta * (k.theta / before) >= eps;
        };
        for (;;) {
            while (pending < (ahead() ? 2 : 1) && enqueued < max_iter) {
                const int m = std::min(ctx->p.check_every, max_iter - enqueued);
                if ((rc = period(m))) return rc;
                enqueued += m;
                pending++;
            }
            if (pending == 0) break;
            before = k.theta;
            if ((rc = wait_check(ctx, ctx->checks + 1, &k, watch))) return rc;
            ctx->checks++;
            taken++;
            pending--;
            ctx->h_result[0] = k.F;
            ctx->h_result[1] = k.theta;
            ctx->h_flags[0] = k.active;
            ctx->h_flags[1] = k.iters;
            log_members();
            if (!k.active) break;
        }
        ctx->sweeps_done = sweeps0 + k.iters;
        HIPTRY(ctx, hipStreamSynchronize(ctx->stream));  // the call returns with its stream idle
    } else {
        HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
        log_members();
        int it = 0;
        auto any_active = [&]() {
            for (int c = 0; c < n; c++) if (ctx->h_flags[c]) return true;
            return false;
        };
        while (it < max_iter && any_active() && !nonfinite()) {
            const int m = std::min(ctx->p.check_every, max_iter - it);
            if ((rc = period(m))) return rc;
            it += m;
            HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
            log_members();
        }
    }
    bool all = true;
    for (int c = 0; c < n; c++) {
        F[c] = ctx->h_result[2 * c];
        theta[c] = ctx->h_result[2 * c + 1];
        iters[c] = ctx->h_flags[n + c];
        if (!(theta[c] < eps)) all = false;
    }
    if (nonfinite()) return fail(ctx, GF_ENONFINITE, "F or theta is not finite");
    return all ? GF_OK : GF_NOT_CONVERGED;
}

int gf_get_schedule(const gf_ctx *ctx, int *lps, int *block, int *nt, int *tile_order) {
    if (!ctx) return GF_EINVAL;
    if (lps) *lps = ctx->sched.lps;
    if (block) *block = ctx->sched.block;
    if (nt) *nt = ctx->sched.nt;
    if (tile_order) *tile_order = ctx->sched.order;
    return GF_OK;
}

int gf_timing(gf_ctx *ctx, double *ms, long long *launches) {
    if (!ctx) return GF_EINVAL;
    DeviceGuard dg(ctx->device);
    HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
    double tot = 0.0;
    for (auto &e : ctx->ev_busy) {
        float t = 0.f;
        HIPTRY(ctx, hipEventElapsedTime(&t, e.first, e.second));
        tot += t;
        ctx->ev_free.push_back(e);
    }
    if (ms) *ms = tot;
    if (launches) *launches = (long long)ctx->ev_busy.size();
    ctx->ev_busy.clear();
    return GF_OK;
}

int gf_set_sweep_count(gf_ctx *ctx, long long s) {
    if (!ctx) return GF_EINVAL;
    CHECK(ctx, s >= 0, GF_EINVAL, "sweep count must be >= 0");
    ctx->sweeps_done = s;
    return GF_OK;
}

long long gf_get_sweep_count(const gf_ctx *ctx) { return ctx ? ctx->sweeps_done : -1; }

// ---- autotuner ----------------------------------------------------------

int gf_autotune(gf_ctx *ctx, void *const *U, double omega, const char *cache_path) {
    if (!ctx) return GF_EINVAL;
    CHECK(ctx, U != nullptr, GF_EINVAL, "U is NULL");
    int rc;
    for (int c = 0; c < ctx->n; c++)
        if ((rc = check_field(ctx, U[c], "U[i]"))) return rc;
    if ((rc = check_omega(ctx, omega))) return rc;
    DeviceGuard dg(ctx->device);
    hipDeviceProp_t prop;
    HIPTRY(ctx, hipGetDeviceProperties(&prop, ctx->device));
    std::ostringstream key;
    key << prop.gcnArchName << "|cu" << prop.multiProcessorCount << "|src" << GF_SOURCE_HASH << "|n" << ctx->nc
        << "|p" << ctx->prec << "|e" << ctx->nelem;
    for (int c = 0; c < ctx->n; c++) {
        const Geom &g = ctx->desc[c].g;
        key << "|" << g.nx << "x" << g.ny << "x" << g.nz << "x" << g.nt << "g" << ctx->desc[c].gauge;
    }
    const std::string k = key.str();
    auto total_bytes = [&]() {
        double b = 0.0;
        for (int c = 0; c < ctx->n; c++) b += (double)gf_field_bytes(ctx, c);
        return b;
    };
    if (cache_path) {
        std::ifstream in(cache_path);
        std::string line, found;
        while (std::getline(in, line))
            if (line.compare(0, k.size() + 1, k + " ") == 0) found = line.substr(k.size() + 1);
        if (!found.empty()) {
            Schedule s{};
            std::istringstream is(found);
            if (is >> s.lps >> s.block >> s.nt >> s.order && check_schedule(ctx, s, ctx->nc) == GF_OK) {
                s.lds = sweep_lds(s, ctx->nc, ctx->nelem, total_bytes());
                s.nt_check = s.nt;
                ctx->sched = s;
                return build_tiles(ctx);
            }
        }
    }
    // scratch copy of every member's field
    std::vector<size_t> bytes(ctx->n);
    size_t total = 0;
    for (int c = 0; c < ctx->n; c++) { bytes[c] = (gf_field_bytes(ctx, c) + 255) & ~size_t(255); total += bytes[c]; }
    char *scratch = nullptr;
    if (hipMalloc(&scratch, total) != hipSuccess) return fail(ctx, GF_ENOMEM, "autotune scratch (%zu bytes)", total);
    rc = GF_OK;
    auto ok = [&](hipError_t e, const char *what) {
        if (e != hipSuccess && rc == GF_OK) rc = fail(ctx, GF_EDEVICE, "autotune: %s failed: %s", what, hipGetErrorString(e));
        return rc == GF_OK;
    };
    std::vector<void *> su(ctx->n);
    size_t o = 0;
    for (int c = 0; c < ctx->n; c++) {
        su[c] = scratch + o;
        ok(hipMemcpyAsync(su[c], U[c], gf_field_bytes(ctx, c), hipMemcpyDeviceToDevice, ctx->stream), "hipMemcpyAsync");
        o += bytes[c];
    }
    std::vector<double> om(ctx->n, omega);
    std::vector<void *> keepU(ctx->n);
    std::vector<double> keepW(ctx->n);
    for (int c = 0; c < ctx->n; c++) { keepU[c] = ctx->desc[c].U; keepW[c] = ctx->desc[c].omega; }
    const Schedule keep = ctx->sched;
    const int keep_timing = ctx->p.timing;
    ctx->p.timing = 0;
    if (rc == GF_OK) rc = set_fields(ctx, su.data(), om.data());
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ok(hipEventCreate(&e0), "hipEventCreate");
    ok(hipEventCreate(&e1), "hipEventCreate");
    // Time of `count` half-sweeps with schedule s over the members of mask.
    auto measure = [&](const Schedule &s, const int *mask, int count) -> float {
        float ms = 0.f;
        ctx->sched = s;
        if (rc != GF_OK || (rc = build_tiles(ctx))) return ms;
        for (int w = 0; w < 2 && rc == GF_OK; w++) rc = half_sweep(ctx, w & 1, 0, mask);
        ok(hipEventRecord(e0, ctx->stream), "hipEventRecord");
        for (int w = 0; w < count && rc == GF_OK; w++) rc = half_sweep(ctx, w & 1, 0, mask);
        ok(hipEventRecord(e1, ctx->stream), "hipEventRecord");
        ok(hipEventSynchronize(e1), "hipEventSynchronize");
        ok(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
        return ms / count;
    };
    // An ensemble's members converge one by one, the largest usually last: its
    // candidates are timed with every member active and with the largest alone,
    // and judged by the sum (timed with all members only, the ensemble of 48^3 x 96
    // and 64 small lattices got a schedule that ran 4 % slower to the end).
    const bool ensemble = ctx->n > 1;
    if (ensemble) {
        int big = 0;
        for (int c = 1; c < ctx->n; c++)
            if (ctx->desc[c].g.V > ctx->desc[big].g.V) big = c;
        for (int c = 0; c < ctx->n; c++) ctx->h_flags[c] = c == big;
        ok(hipMemcpyAsync(ctx->d_active, ctx->h_flags, ctx->n * sizeof(int), hipMemcpyHostToDevice, ctx->stream),
           "hipMemcpyAsync");
    }
    auto cost = [&](const Schedule &s) { return measure(s, ctx->d_ones, 4) + measure(s, ctx->d_active, 4); };
    std::vector<std::pair<float, Schedule>> tried;
    float full = 1e30f;  // an ensemble's fastest with every member active
    for (int lps : {1, 2, 4, 8})
        for (int block : {64, 128, 256})
            for (int nt = 0; nt < 2; nt++)
                // XCD-contiguous shares only for a single lattice: an ensemble's members
                // converge one by one, and a retired member empties its XCD's share while
                // others still carry the large members' tiles (measured on the uneven
                // ensemble: tuned with every member active it won, then ran 11 % slower)
                for (int order = 0; order < (ensemble ? 1 : 2) && rc == GF_OK; order++) {
                    Schedule s{lps, block, nt, order, 0, nt};
                    s.lds = sweep_lds(s, ctx->nc, ctx->nelem, total_bytes());
                    if (ctx->nc == 4 && s.lps < 2) continue;       // registers
                    float ms = measure(s, ctx->d_ones, ensemble ? 4 : 6);
                    if (ensemble) {
                        full = std::min(full, ms);
                        if (ms > 1.1f * full) continue;  // behind by more than the large member alone makes good
                        ms += measure(s, ctx->d_active, 4);
                    }
                    if (rc == GF_OK) tried.emplace_back(ms, s);
                }
    std::sort(tried.begin(), tried.end(),
              [](const std::pair<float, Schedule> &x, const std::pair<float, Schedule> &y) { return x.first < y.first; });
    Schedule best = keep;
    float best_ms = tried.empty() ? 0.f : tried[0].first;
    if (!ensemble) {
        if (!tried.empty()) best = tried[0].second;
    } else if (rc == GF_OK) {
        // An ensemble's candidates lie closer together than one timing resolves: the
        // three best and the context's own schedule are timed again in turn, and the
        // latter stays unless another is faster by more than its own runs differ.
        std::vector<Schedule> last{keep};
        for (size_t i = 0; i < tried.size() && i < 3; i++) last.push_back(tried[i].second);
        std::vector<float> lo(last.size(), 1e30f), hi(last.size(), 0.f);
        for (int round = 0; round < 3 && rc == GF_OK; round++)
            for (size_t i = 0; i < last.size() && rc == GF_OK; i++) {
                const float ms = cost(last[i]);
                lo[i] = std::min(lo[i], ms);
                hi[i] = std::max(hi[i], ms);
            }
        size_t pick = 0;
        for (size_t i = 1; i < last.size(); i++)
            if (hi[i] < lo[0] && lo[i] < lo[pick]) pick = i;
        best = last[pick];
        best_ms = lo[pick] / 2;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    ctx->p.timing = keep_timing;
    ok(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");
    (void)hipFree(scratch);
    for (int c = 0; c < ctx->n; c++) { ctx->desc[c].U = keepU[c]; ctx->desc[c].omega = keepW[c]; }
    ctx->sched = rc == GF_OK ? best : keep;
    const int rc2 = build_tiles(ctx);  // also re-uploads the restored member table
    if (rc) return rc;
    if (rc2) return rc2;
    if (cache_path) {
        std::ofstream outf(cache_path, std::ios::app);
        outf << k << " " << best.lps << " " << best.block << " " << best.nt << " " << best.order << " "
             << best_ms << "\n";
    }
    return GF_OK;
}

// ---- differentiation --------------------------------------------------------

namespace {

int ensure_diff_scratch(gf_ctx *ctx) {
    const Geom &g = ctx->desc[0].g;
    // each buffer on its own, so a call after a failed allocation retries it
    if (!ctx->d_gfield && hipMalloc(&ctx->d_gfield, (size_t)gfield_complex(g) * csize(ctx)) != hipSuccess) {
        ctx->d_gfield = nullptr;
        return fail(ctx, GF_ENOMEM, "cannot allocate the g field");
    }
    const int nb = (g.V + 255) / 256;
    if (!ctx->d_fpart && hipMalloc(&ctx->d_fpart, nb * sizeof(double)) != hipSuccess) {
        ctx->d_fpart = nullptr;
        return fail(ctx, GF_ENOMEM, "cannot allocate functional partials");
    }
    return GF_OK;
}

int diff_prologue(gf_ctx *ctx, const void *U, const void *s) {
    int rc;
    if ((rc = need_single(ctx)) || (rc = need_su3(ctx)) || (rc = check_field(ctx, U, "U")) ||
        (rc = check_field(ctx, s, "s")))
        return rc;
    if ((rc = ensure_diff_scratch(ctx))) return rc;
    HIPTRY(ctx, launch_expS(ctx->prec, ctx->desc[0].g, s, ctx->d_gfield, ctx->stream));
    return GF_OK;
}

}  // namespace

int gf_pack_alg(gf_ctx *ctx, const void *s_aos, void *s) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = need_su3(ctx)) || (rc = check_field(ctx, s_aos, "s_aos")) ||
        (rc = check_field(ctx, s, "s")))
        return rc;
    DeviceGuard dg(ctx->device);
    HIPTRY(ctx, launch_pack_alg(ctx->prec, ctx->desc[0].g, s_aos, s, 0, ctx->stream));
    return GF_OK;
}

int gf_unpack_alg(gf_ctx *ctx, const void *s, void *s_aos) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = need_su3(ctx)) || (rc = check_field(ctx, s_aos, "s_aos")) ||
        (rc = check_field(ctx, s, "s")))
        return rc;
    DeviceGuard dg(ctx->device);
    HIPTRY(ctx, launch_pack_alg(ctx->prec, ctx->desc[0].g, s_aos, const_cast<void *>(s), 1, ctx->stream));
    return GF_OK;
}

int gf_functional(gf_ctx *ctx, const void *U, const void *s, double *F) {
    if (!ctx) return GF_EINVAL;
    CHECK(ctx, F != nullptr, GF_EINVAL, "F is NULL");
    DeviceGuard dg(ctx->device);
    int rc;
    if ((rc = diff_prologue(ctx, U, s))) return rc;
    const Geom &g = ctx->desc[0].g;
    const int nb = (g.V + 255) / 256;
    HIPTRY(ctx, launch_functional(ctx->prec, ctx->nelem, ctx->desc[0].gauge, g, U, ctx->d_gfield,
                                  ctx->d_fpart, ctx->stream));
    HIPTRY(ctx, launch_sum_partials(ctx->d_fpart, nb, ctx->h_result, ctx->stream));  // pinned: no copy
    HIPTRY(ctx, hipStreamSynchronize(ctx->stream));
    const int nd = ctx->desc[0].gauge == GF_LANDAU ? 4 : 3;
    *F = ctx->h_result[0] / (nd * 3.0 * (double)g.V);
    if (!std::isfinite(*F)) return fail(ctx, GF_ENONFINITE, "F is not finite");
    return GF_OK;
}

int gf_functional_grad(gf_ctx *ctx, const void *U, const void *s, double dF, void *grad) {
    if (!ctx) return GF_EINVAL;
    CHECK(ctx, std::isfinite(dF), GF_EINVAL, "dF must be finite");
    int rc;
    if ((rc = check_field(ctx, grad, "grad"))) return rc;
    DeviceGuard dg(ctx->device);
    if ((rc = diff_prologue(ctx, U, s))) return rc;
    HIPTRY(ctx, launch_functional_grad(ctx->prec, ctx->nelem, ctx->desc[0].gauge, ctx->desc[0].g, U, s,
                                       ctx->d_gfield, dF, grad, ctx->stream));
    return GF_OK;
}

int gf_gauge_transform(gf_ctx *ctx, void *U, const void *s) {
    if (!ctx) return GF_EINVAL;
    DeviceGuard dg(ctx->device);
    int rc;
    if ((rc = diff_prologue(ctx, U, s))) return rc;
    HIPTRY(ctx, launch_gauge_transform(ctx->prec, ctx->nelem, ctx->desc[0].g, U, ctx->d_gfield, ctx->stream));
    return GF_OK;
}

// ---- steepest descent with Fourier acceleration (Alg. 2) ----------------------

namespace {

// Buffers of one step: the half spectrum spec[t][a][z][y][kx] (kx = 0..nx/2)
// of the eight su(3) components of Delta, and the root tables. Made once per
// context; a call after a failed allocation retries what is missing.
int sd_prepare(gf_ctx *ctx) {
    const Geom &g = ctx->desc[0].g;
    CHECK(ctx, g.nx <= FFT_MAX_NX && g.ny <= FFT_MAX_N && g.nz <= FFT_MAX_N && g.nt <= FFT_MAX_N,
          GF_EUNSUPPORTED, "Fourier acceleration supports nx up to %d and ny, nz, nt up to %d", FFT_MAX_NX,
          FFT_MAX_N);
    int rc;
    if ((rc = ensure_diff_scratch(ctx))) return rc;
    const size_t rs = ctx->prec == GF_F64 ? 8 : 4;
    const long long S = (long long)g.nz * g.ny * (g.nx / 2 + 1);
    if (!ctx->d_spec && hipMalloc(&ctx->d_spec, 8 * (size_t)g.nt * S * 2 * rs) != hipSuccess) {
        ctx->d_spec = nullptr;
        return fail(ctx, GF_ENOMEM, "cannot allocate the Fourier acceleration buffers");
    }
    if (!ctx->d_sdpart &&
        hipMalloc(&ctx->d_sdpart, 2 * (size_t)sd_delta_groups(make_fft_site(g)) * sizeof(double)) != hipSuccess) {
        ctx->d_sdpart = nullptr;
        return fail(ctx, GF_ENOMEM, "cannot allocate the Fourier acceleration buffers");
    }
    if (!ctx->d_roots) {
        void *w = nullptr;
        if (hipMalloc(&w, 4 * (size_t)FFT_MAX_N * (16 + 8)) != hipSuccess)
            return fail(ctx, GF_ENOMEM, "cannot allocate the Fourier acceleration buffers");
        const int len[4] = {g.nx, g.ny, g.nz, g.nt};
        for (int a = 0; a < 4; a++) {
            double *p2 = (double *)((char *)w + 4 * (size_t)FFT_MAX_N * 16) + (size_t)a * FFT_MAX_N;
            const hipError_t e = launch_fft_roots((char *)w + (size_t)a * FFT_MAX_N * 16, p2, len[a], ctx->stream);
            if (e != hipSuccess) {
                (void)hipFree(w);
                return fail(ctx, GF_EDEVICE, "root tables: %s", hipGetErrorString(e));
            }
        }
        ctx->d_roots = w;
    }
    return GF_OK;
}

const void *sd_roots(const gf_ctx *ctx, int axis) {
    return (const char *)ctx->d_roots + (size_t)axis * FFT_MAX_N * 16;
}

const double *sd_p2(const gf_ctx *ctx) { return (const double *)sd_roots(ctx, 4); }

// One step of Alg. 2: Delta -> F (x, y, z and, for Landau, t) -> times
// (alpha/2) p2max / p^2 / N -> F^-1 -> g = reunit(1 + X) -> U <- g U g^dagger.
// Delta is formed in the forward x pass and g in the inverse one; the filter
// sits in the last forward pass (t for Landau, z for Coulomb), between its
// forward and inverse transform.
// Everything of a step that only reads the links, in two parts: Delta with the
// forward x transform, and the rest up to the g field. With `check`, F and theta
// of those links come from the Delta pass and are published as the next check.
int sd_delta(gf_ctx *ctx, const void *U, bool check) {
    const Geom &g = ctx->desc[0].g;
    const FftSite fx = make_fft_site(g);
    hipStream_t st = ctx->stream;
    HIPTRY(ctx, launch_sd_delta_fx(ctx->prec, ctx->nelem, ctx->desc[0].gauge, g, fx, sd_roots(ctx, 0), U, ctx->d_spec,
                                   check ? ctx->d_sdpart : nullptr, st));
    if (check) {
        const QualityOut out{nullptr, nullptr, nullptr, nullptr, ctx->ring, ctx->d_count};
        HIPTRY(ctx, launch_quality_final(3, ctx->d_desc, 1, ctx->d_sdpart, out, 0, 0.0, st, sd_delta_groups(fx)));
    }
    return GF_OK;
}

int sd_gfield(gf_ctx *ctx, double alpha) {
    const Geom &g = ctx->desc[0].g;
    const bool landau = ctx->desc[0].gauge == GF_LANDAU;
    const FftSite fx = make_fft_site(g);
    const FftAxis fy = make_fft_axis(g, 1, !landau);
    const FftAxis fz = make_fft_axis(g, 2, !landau);
    const int last = landau ? 3 : 2;
    FftAxis flt = landau ? make_fft_axis(g, 3, false) : fz;
    const FftLine ly = make_fft_line(g, 1), lz = make_fft_line(g, 2);
    FftLine llt = make_fft_line(g, last);
    const double nfft = landau ? (double)g.V : (double)g.nx * g.ny * g.nz;
    flt.scale = llt.scale = 0.5 * alpha / nfft;
    flt.p2max = llt.p2max = landau ? 16.0 : 12.0;
    hipStream_t st = ctx->stream;
    const void *wx = sd_roots(ctx, 0), *wy = sd_roots(ctx, 1), *wz = sd_roots(ctx, 2);
    const double *p2 = sd_p2(ctx);
    void *spec = ctx->d_spec;
    HIPTRY(ctx, launch_fft_axis(ctx->prec, fy, ly, wy, p2, spec, 1, -1, 0, st));
    if (landau) HIPTRY(ctx, launch_fft_axis(ctx->prec, fz, lz, wz, p2, spec, 2, -1, 0, st));
    HIPTRY(ctx, launch_fft_axis(ctx->prec, flt, llt, sd_roots(ctx, last), p2, spec, last, -1, 1, st));
    if (landau) HIPTRY(ctx, launch_fft_axis(ctx->prec, fz, lz, wz, p2, spec, 2, 1, 0, st));
    HIPTRY(ctx, launch_fft_axis(ctx->prec, fy, ly, wy, p2, spec, 1, 1, 0, st));
    HIPTRY(ctx, launch_sd_fx_gfield(ctx->prec, g, fx, wx, ctx->d_spec, ctx->d_gfield, st));
    return GF_OK;
}

int sd_apply(gf_ctx *ctx, void *U) {
    HIPTRY(ctx, launch_gauge_transform(ctx->prec, ctx->nelem, ctx->desc[0].g, U, ctx->d_gfield, ctx->stream));
    return GF_OK;
}

int sd_step_impl(gf_ctx *ctx, void *U, double alpha) {
    int rc;
    if ((rc = sd_delta(ctx, U, false)) || (rc = sd_gfield(ctx, alpha))) return rc;
    return sd_apply(ctx, U);
}

int check_alpha(gf_ctx *ctx, double alpha) {
    CHECK(ctx, std::isfinite(alpha) && alpha > 0.0, GF_EINVAL, "alpha = %g must be finite and > 0", alpha);
    return GF_OK;
}

}  // namespace

int gf_sd_step(gf_ctx *ctx, void *U, double alpha) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = need_su3(ctx)) || (rc = check_field(ctx, U, "U")) ||
        (rc = check_alpha(ctx, alpha)))
        return rc;
    DeviceGuard dg(ctx->device);
    if ((rc = sd_prepare(ctx))) return rc;
    return sd_step_impl(ctx, U, alpha);
}

int gf_sd_fix(gf_ctx *ctx, void *U, double alpha, double eps, int max_iter, int *iters, double *F,
              double *theta) {
    if (!ctx) return GF_EINVAL;
    int rc;
    if ((rc = need_single(ctx)) || (rc = need_su3(ctx)) || (rc = check_field(ctx, U, "U")) ||
        (rc = check_alpha(ctx, alpha)))
        return rc;
    CHECK(ctx, iters && F && theta, GF_EINVAL, "NULL argument");
    CHECK(ctx, std::isfinite(eps) && eps >= 0.0, GF_EINVAL, "eps must be finite and >= 0");
    CHECK(ctx, max_iter >= 0, GF_EINVAL, "max_iter must be >= 0");
    DeviceGuard dg(ctx->device);
    if ((rc = sd_prepare(ctx))) return rc;
    const Clock::time_point t0 = Clock::now();
    log_open(ctx);
    ctx->log_calls++;
    *iters = 0;
    const bool watch = waits_spin() && !ctx->p.timing;  // the stream goes on behind the check
    if ((rc = start_checks(ctx))) return rc;
    int it = 0;
    for (;;) {
        // A check that a step can follow comes from that step's own Delta pass, with
        // the step's direction enqueued behind it (it leaves the links alone): a pass
        // over the links and the wait for the result less. F and theta as returned are
        // those of gf_quality, which the last check is. It also decides where the run
        // ends: the Delta pass adds the same terms in another order, so that its theta is
        // within 1e-12 of gf_quality's (some hundred roundings of 1.1e-16 on the largest
        // lattices); from there down gf_quality is asked.
        // A field that is fixed already takes no direction: on large lattices the first
        // check is waited for before the transforms are enqueued (48^4 in float 1242 ->
        // 763 us a call, 32^4 305 -> 176; a run that goes on loses 8 us once: 48^4, five
        // steps 7842 -> 7850). On small ones that gap is worth more (4^4 in double, five
        // steps 235 -> 275 us; a fixed field 75 -> 60).
        const bool first = it == 0 && ctx->desc[0].g.V >= 1000000;
        bool last = it >= max_iter;
        if (!last) {
            Check k{};
            if ((rc = sd_delta(ctx, U, true))) return rc;
            if (!first && (rc = sd_gfield(ctx, alpha))) return rc;
            if ((rc = wait_check(ctx, ctx->checks + 1, &k, watch))) return rc;
            ctx->checks++;
            *F = k.F;
            *theta = k.theta;
            last = k.theta < eps * (1.0 + 1e-12) || !std::isfinite(k.F) || !std::isfinite(k.theta);
        }
        if (last && (rc = gf_quality(ctx, U, F, theta))) return rc;
        log_check(ctx, true, 0, it, *F, *theta, t0);
        log_flush(ctx);
        if (it >= max_iter || *theta < eps) break;
        const int m = std::min(ctx->p.check_every, max_iter - it);
        if (first && (rc = sd_gfield(ctx, alpha))) return rc;
        if ((rc = sd_apply(ctx, U))) return rc;
        for (int k = 1; k < m; k++)
            if ((rc = sd_step_impl(ctx, U, alpha))) return rc;
        it += m;
        *iters = it;
    }
    return *theta < eps ? GF_OK : GF_NOT_CONVERGED;
}

// ---- host-only checks ------------------------------------------------------

void gf_host_su2_step(const double b[4], double omega, double r[4]) {
    if (b && r) gf_su2_overrelax(b, omega, r);
}

int gf_host_schedule(int prec, int nc, int storage, int n, const int *dims, int out[6]) {
    if (!dims || !out || n < 1 || (prec != GF_F64 && prec != GF_F32) || nc < 2 || nc > 4) return GF_EINVAL;
    if (storage != GF_STORE_18 && (nc != 3 || (storage != GF_STORE_12 && storage != GF_STORE_8))) return GF_EINVAL;
    gf_ctx tmp;
    for (int c = 0; c < n; c++)
        if (check_dims(&tmp, dims + 4 * c) != GF_OK) return GF_EINVAL;
    gf_params p;
    gf_params_default(&p, prec);
    const Schedule s = schedule_of(prec, nc, links_stored(nc, storage), n, dims, p);
    if (check_schedule(&tmp, s, nc) != GF_OK) return GF_EINVAL;
    const int v[6] = {s.lps, s.block, s.nt, s.order, s.lds, s.nt_check};
    std::copy(v, v + 6, out);
    return GF_OK;
}

void gf_host_trig(double x, double y, double out[3]) {
    if (!out) return;
    gf_sincos(gf_trig(), x, &out[0], &out[1]);
    out[2] = gf_atan2(y, x);
}

int gf_host_link8(int prec, const double in[18], double stored[8], double out[18]) {
    if (!in || !stored || !out || (prec != GF_F64 && prec != GF_F32)) return GF_EINVAL;
    if (prec == GF_F64) {
        double re[9], im[9], sre[4], sim[4];
        for (int e = 0; e < 9; e++) { re[e] = in[2 * e]; im[e] = in[2 * e + 1]; }
        link8_compress<double>(re, im, sre, sim);
        link8_reconstruct<double>(sre, sim, re, im);
        for (int e = 0; e < 4; e++) { stored[2 * e] = sre[e]; stored[2 * e + 1] = sim[e]; }
        for (int e = 0; e < 9; e++) { out[2 * e] = re[e]; out[2 * e + 1] = im[e]; }
    } else {
        float re[9], im[9], sre[4], sim[4];
        for (int e = 0; e < 9; e++) { re[e] = (float)in[2 * e]; im[e] = (float)in[2 * e + 1]; }
        link8_compress<float>(re, im, sre, sim);
        link8_reconstruct<float>(sre, sim, re, im);
        for (int e = 0; e < 4; e++) { stored[2 * e] = sre[e]; stored[2 * e + 1] = sim[e]; }
        for (int e = 0; e < 9; e++) { out[2 * e] = re[e]; out[2 * e + 1] = im[e]; }
    }
    return GF_OK;
}


int gf_site_links(const int dims[4], int parity, long long h, long long out[8]) {
    gf_ctx tmp;
    if (!out || check_dims(&tmp, dims) != GF_OK || (parity != 0 && parity != 1)) return GF_EINVAL;
    const Geom g = make_geom(dims, 9);
    if (h < 0 || h >= g.Vh) return GF_EINVAL;
    const SiteNbr nb = site_neighbours(g, parity, (int)h);
    for (int mu = 0; mu < 4; mu++) {
        out[mu] = link_off(g, mu, parity, (int)h);
        out[4 + mu] = link_off(g, mu, 1 - parity, nb.hb[mu]);
    }
    return GF_OK;
}

}  // extern "C"
