// api.hip -- the extern "C" entry points of igg.h: argument checks (all on
// the host, before any HIP call), the implicit global grid state (one rank,
// or several virtual ranks as blocks on this device), the boundary-first
// schedule of the steps, the time loop with its captured graph, and kernel
// timing.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <string>

#include "host.hpp"

namespace igg {

static thread_local std::string t_last_error;

int fail(int code, const std::string &msg)
{
    t_last_error = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    char buf[512];
    snprintf(buf, sizeof buf, "HIP error %d (%s) in %s", (int)e, hipGetErrorString(e), what);
    return fail(IGG_ERR_HIP, buf);
}

Grid &grid()
{
    static Grid g;
    return g;
}

int64_t zmarch_min_points() { return grid().zmarch_min; }

void rank_coords(int r, int c[3])
{
    const Grid &g = grid();
    c[0] = r % g.dims[0];
    c[1] = (r / g.dims[0]) % g.dims[1];
    c[2] = r / (g.dims[0] * g.dims[1]);
}

int rank_neighbor(int r, int d, int side)
{
    const Grid &g = grid();
    int c[3];
    rank_coords(r, c);
    c[d] += side ? 1 : -1;
    if (c[d] < 0 || c[d] >= g.dims[d]) {
        if (!g.periods[d]) return -1;
        c[d] = (c[d] + g.dims[d]) % g.dims[d];
    }
    return c[0] + g.dims[0] * (c[1] + g.dims[1] * c[2]);
}

int elem_bytes(int dtype) { return dtype == IGG_F64 ? 8 : dtype == IGG_F32 ? 4 : 2; }

int64_t field_elems(const igg_field &f) { return f.size[0] * f.size[1] * f.size[2]; }

bool overlaps_mem(const igg_field &a, const igg_field &b)
{
    uintptr_t a0 = (uintptr_t)a.data, a1 = a0 + (uintptr_t)(field_elems(a) * elem_bytes(a.dtype));
    uintptr_t b0 = (uintptr_t)b.data, b1 = b0 + (uintptr_t)(field_elems(b) * elem_bytes(b.dtype));
    return a0 < b1 && b0 < a1;
}

int check_field(const igg_field *f, const char *name, bool grid_sized)
{
    Grid &g = grid();
    if (!f) return fail(IGG_ERR_ARG, std::string(name) + ": null field");
    if (!f->data) return fail(IGG_ERR_ARG, std::string(name) + ": null data pointer");
    if (f->reserved != 0) return fail(IGG_ERR_ARG, std::string(name) + ": reserved must be 0");
    if (f->dtype < IGG_F64 || f->dtype > IGG_F16)
        return fail(IGG_ERR_DTYPE, std::string(name) + ": unknown dtype " + std::to_string(f->dtype));
    for (int d = 0; d < 3; ++d) {
        int64_t s = f->size[d];
        bool ok = grid_sized ? (s == g.n[d]) : (s == g.n[d] || s == g.n[d] + 1);
        if (!ok) {
            char buf[256];
            snprintf(buf, sizeof buf, "%s: size (%lld,%lld,%lld) does not fit the grid (%d,%d,%d)%s",
                     name, (long long)f->size[0], (long long)f->size[1], (long long)f->size[2],
                     g.n[0], g.n[1], g.n[2], grid_sized ? "" : " (n or n+1 per dimension)");
            return fail(IGG_ERR_SIZE, buf);
        }
    }
    return IGG_OK;
}

// A field of rank r, named name[r] where there are several ranks (names are
// only put together for a message).
static int check_rank_field(const igg_field *f, const char *name, int r, bool grid_sized = true)
{
    if (grid().nranks == 1) return check_field(f, name, grid_sized);
    return check_field(f, (std::string(name) + "[" + std::to_string(r) + "]").c_str(), grid_sized);
}

static int check_finite_pos(double v, const char *name, bool allow_zero)
{
    if (!isfinite(v) || v < 0.0 || (!allow_zero && v == 0.0))
        return fail(IGG_ERR_ARG, std::string(name) + " must be finite and " +
                                     (allow_zero ? "non-negative" : "positive"));
    return IGG_OK;
}

int plan_split(const int n[3], const int w[3], Split &s)
{
    s.nb = 0;
    int kz0 = std::min(w[2], n[2] - 1), kz1 = std::max(n[2] - w[2], kz0);
    int jy0 = std::min(w[1], n[1] - 1), jy1 = std::max(n[1] - w[1], jy0);
    int ix0 = std::min(w[0], n[0] - 1), ix1 = std::max(n[0] - w[0], ix0);
    auto add = [&](int kind, int i0, int i1, int j0, int j1, int k0, int k1) {
        if (i0 < i1 && j0 < j1 && k0 < k1) {
            s.kind[s.nb] = kind;
            s.boundary[s.nb++] = Box{i0, i1, j0, j1, k0, k1};
        }
    };
    const int X = n[0] - 1, Y = n[1] - 1, Z = n[2] - 1;
    add(1, 1, X, 1, Y, 1, kz0);        // z low slab
    add(1, 1, X, 1, Y, kz1, Z);        // z high slab
    add(1, 1, X, 1, jy0, kz0, kz1);    // y low slab
    add(1, 1, X, jy1, Y, kz0, kz1);    // y high slab
    add(0, 1, ix0, jy0, jy1, kz0, kz1);  // x low slab
    add(0, ix1, X, jy0, jy1, kz0, kz1);  // x high slab
    s.inner = Box{ix0, ix1, jy0, jy1, kz0, kz1};
    return IGG_OK;
}

BoxSet make_boxset(const Box *b, int nb)
{
    BoxSet bs{};
    bs.n = nb;
    int64_t t = 0;
    for (int q = 0; q < nb; ++q) {
        int w = b[q].i1 - b[q].i0;
        int lg = 3;
        while ((1 << lg) < w && lg < 6) ++lg;
        bs.b[q] = b[q];
        bs.lpr_log2[q] = lg;
        bs.nseg_x[q] = (w + (1 << lg) - 1) >> lg;
        bs.first[q] = t;
        t += (int64_t)bs.nseg_x[q] * (b[q].j1 - b[q].j0) * (b[q].k1 - b[q].k0) << lg;
    }
    for (int q = nb; q < 7; ++q) bs.first[q] = t;
    return bs;
}

uint32_t sr_key(uint64_t seed, uint64_t counter)
{
    uint32_t h = pcg_hash((uint32_t)(counter >> 32));
    h = pcg_hash((uint32_t)counter ^ h);
    h = pcg_hash((uint32_t)(seed >> 32) ^ h);
    return pcg_hash((uint32_t)seed ^ h);
}

int ensure_device()
{
    Grid &g = grid();
    int dev = -1;
    IGG_HIP(hipGetDevice(&dev));
    if (g.dev_ready) {
        if (dev != g.device)
            return fail(IGG_ERR_ARG, "the grid's GPU resources live on device " + std::to_string(g.device) +
                                         ", current device is " + std::to_string(dev));
        return IGG_OK;
    }
    // default priority: the helper stream is an ordinary second stream
    IGG_HIP(hipStreamCreateWithFlags(&g.side, hipStreamNonBlocking));
    // fork/join events order work between two streams of this device only:
    // no timing and no system-scope fence (a fence writes back the caches
    // at every record, tens of microseconds per step at 512^3)
    IGG_HIP(hipEventCreateWithFlags(&g.ev_fork, hipEventDisableTiming | hipEventDisableSystemFence));
    IGG_HIP(hipEventCreateWithFlags(&g.ev_join, hipEventDisableTiming | hipEventDisableSystemFence));
    // Send and receive planes of one field each (one plane of the largest
    // field, n+1 per dimension in FP64, rounded to 256 B).  One rank fills its
    // halo from its own points and needs them only where the slabs pack (512^3:
    // 67 MB).
    if (g.nranks > 1 || g.slab_pack == 1) {
        int64_t m0 = (int64_t)(g.n[1] + 1) * (g.n[2] + 1), m1 = (int64_t)(g.n[0] + 1) * (g.n[2] + 1),
                m2 = (int64_t)(g.n[0] + 1) * (g.n[1] + 1);
        int64_t cap = std::max(m0, std::max(m1, m2)) * 8;
        g.halo_cap = (size_t)((cap + 255) / 256 * 256);
        IGG_HIP(hipMalloc((void **)&g.halo_buf, g.halo_cap * 2 * 2 * IGG_MAX_FIELDS * g.nranks));
    }
    {
        RedSlots first;  // allocated here, so that a reduction allocates nothing
        int rc;
        if ((rc = first.acquire())) return rc;
    }
    g.device = dev;
    g.dev_ready = true;
    return IGG_OK;
}

// Puts the time loop's kept graph aside: nothing says that a graph may be
// destroyed while it runs, and its replays may be queued still.  Those put aside
// are destroyed together when there are 16 (or all of them, with the grid),
// after the device's work.  (An event behind every call's replays to wait for
// instead: 50 -> 53 us for a loop of 48 x 176 x 45 in one replay.)
static int retire_run_graph(bool all)
{
    Grid &g = grid();
    if (g.run_exec) g.run_old.push_back(g.run_exec);
    g.run_exec = nullptr;
    if (g.run_old.empty() || (!all && g.run_old.size() < 16)) return IGG_OK;
    IGG_HIP(hipDeviceSynchronize());
    std::vector<hipGraphExec_t> old;
    old.swap(g.run_old);
    int rc = IGG_OK;
    for (hipGraphExec_t e : old) {
        const hipError_t h = hipGraphExecDestroy(e);
        if (h != hipSuccess && rc == IGG_OK) rc = hip_fail(h, "hipGraphExecDestroy");
    }
    return rc;
}

static int release_device()
{
    Grid &g = grid();
    if (!g.dev_ready) return IGG_OK;
    int rc = IGG_OK;
    auto chk = [&](hipError_t e, const char *w) {
        if (e != hipSuccess && rc == IGG_OK) rc = hip_fail(e, w);
    };
    chk(hipStreamSynchronize(g.side), "hipStreamSynchronize(side)");
    const int rc_graph = retire_run_graph(true);
    chk(hipFree(g.halo_buf), "hipFree(halo_buf)");
    for (double *p : g.red_free) chk(hipHostFree(p), "hipHostFree(red_free)");
    g.red_free.clear();
    chk(hipEventDestroy(g.ev_fork), "hipEventDestroy");
    chk(hipEventDestroy(g.ev_join), "hipEventDestroy");
    for (hipEvent_t e : g.tev) chk(hipEventDestroy(e), "hipEventDestroy(timing)");
    chk(hipStreamDestroy(g.side), "hipStreamDestroy(side)");
    if (g.cap) chk(hipStreamDestroy(g.cap), "hipStreamDestroy(cap)");
    g.cap = nullptr;
    g.run_key.clear();
    g.tev.clear();
    g.dev_ready = false;
    return rc ? rc : rc_graph;
}

// events made when timing is switched on: 1024 timed launches
static const size_t kTimingPool = 2048;

// Bracket a launch on stream s with timing events when timing is enabled;
// kind 0 marks the inner-region kernel, kind 1 the boundary kernels.
static int timing_mark(hipStream_t s, int kind)
{
    Grid &g = grid();
    if (!g.timing) return IGG_OK;
    if (g.tev_used == g.tev.size()) {
        // timing only: no system-scope fence, which would add a cache
        // write-back to the work being timed
        hipEvent_t e;
        IGG_HIP(hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
        g.tev.push_back(e);
        g.tev_kind.push_back(0);
    }
    g.tev_kind[g.tev_used] = kind;
    IGG_HIP(hipEventRecord(g.tev[g.tev_used++], s));
    return IGG_OK;
}

static int64_t box_points(const Box &b)
{
    return (int64_t)std::max(0, b.i1 - b.i0) * std::max(0, b.j1 - b.j0) * std::max(0, b.k1 - b.k0);
}

// A fixed-length wait on one wavefront, `iters` rounds of the longest
// s_sleep: put into one stream by the IGG_TEST_DELAY setting, it lets a test
// hold back one side of the boundary-first schedule and check that the
// events between the streams, not the timing, order the work.
__global__ void k_test_delay(int iters)
{
    for (int q = 0; q < iters; ++q) __builtin_amdgcn_s_sleep(127);
}

static int test_delay(int where, hipStream_t s)
{
    Grid &g = grid();
    if (g.delay_where != where || g.delay_iters <= 0) return IGG_OK;
    hipLaunchKernelGGL(k_test_delay, dim3(1), dim3(64), 0, s, g.delay_iters);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

// inner regions of at least this many points run the boundary slabs and the
// halo update on the helper stream by default, smaller ones in one chain on
// the caller stream
static const int64_t kSideMinPoints = (int64_t)1 << 21;

static int check_split(const int *split, const int *ol)
{
    if (!split) return IGG_OK;
    for (int d = 0; d < 3; ++d)
        if (split[d] < ol[d])
            return fail(IGG_ERR_ARG, "split width " + std::to_string(split[d]) + " in dimension " +
                                         std::to_string(d) + " is below the overlap " +
                                         std::to_string(ol[d]));
    return IGG_OK;
}

static int check_spacings(double lam, double dt, double dx, double dy, double dz)
{
    int rc;
    if ((rc = check_finite_pos(lam, "lam", false))) return rc;
    if ((rc = check_finite_pos(dt, "dt", true))) return rc;
    if ((rc = check_finite_pos(dx, "dx", false))) return rc;
    if ((rc = check_finite_pos(dy, "dy", false))) return rc;
    if ((rc = check_finite_pos(dz, "dz", false))) return rc;
    return IGG_OK;
}

// One step with boundary-first split: the slabs the halo update reads, then
// the update of `out`.  Schedule 1 runs both on the helper stream while the
// inner region runs on the caller stream (as hide_communication does with
// its boundary streams); schedule 0 runs the slabs on the caller stream ahead
// of the inner region and only the update beside it; schedule 2 runs slabs,
// update and inner region in that order on the caller stream; schedule 3
// (where the caller provides fused_launch) runs the slabs and the inner
// region in one launch whose first work-groups take the slabs, and then
// whatever halo update is left.  By default a caller with fused_launch (the
// one-rank step, whose slab waves store the y and z halo themselves)
// takes schedule 3: at 512^3 it is 0.8-2.6% faster than the unsplit step
// while schedules 1 and 2 are slower, the slabs beside the inner launch
// costing more bandwidth than the update they hide.  Otherwise large inner
// regions take schedule 1; small grids are launch-bound, the cross-stream
// fork and join cost more than the update they would hide, and a captured
// graph of a single chain replays fastest, so they take schedule 2.  FP16
// fields take schedule 2 at any size, as do callers whose inner kernel is
// partly latency-bound (the adjoint passes side_ok = false): its slabs
// beside the inner region cost 5.5% at 256^3 and 2% at 512^3.  When the x
// exchange is fused into the stores (or x is not periodic) the update never
// reads the x slabs, so they join the inner launch and the boundary phase is
// the y and z slabs.
// boundary(r, slabs, stream) and inner(r, box, stream) launch rank r's
// kernels, halo(stream) the halo update of the results.
template <typename HaloLaunch, typename BoundaryLaunch, typename InnerLaunch>
static int run_split(const int *split, int dtype, HaloLaunch halo, BoundaryLaunch boundary,
                     InnerLaunch inner_launch, hipStream_t s, bool side_ok = true,
                     int (*fused_launch)(int, const Split &, const Box &, hipStream_t, void *) = nullptr,
                     void *fused_ctx = nullptr)
{
    Grid &g = grid();
    int rc;
    Split sp;
    plan_split(g.n, split, sp);
    Split bnd = sp;
    Box inner = sp.inner;
    if (g.fuse_x) {
        bnd.nb = 0;
        for (int q = 0; q < sp.nb; ++q) {
            if (sp.kind[q] == 0) continue;
            bnd.boundary[bnd.nb] = sp.boundary[q];
            bnd.kind[bnd.nb++] = sp.kind[q];
        }
        inner.i0 = 1;
        inner.i1 = g.n[0] - 1;
    }
    const bool side_pays = side_ok && box_points(inner) >= kSideMinPoints && dtype != IGG_F16;
    int sched = g.schedule >= 0 ? g.schedule : (fused_launch ? 3 : side_pays ? 1 : 2);
    if (sched == 3 && !fused_launch) sched = 2;
    if (sched == 3) {
        // one launch: the slab work-groups first, then the inner tiles; the
        // halo update (if any is left after the fused pack) follows it
        for (int r = 0; r < g.nranks; ++r) {
            if ((rc = timing_mark(s, 0))) return rc;
            if ((rc = fused_launch(r, bnd, inner, s, fused_ctx))) return rc;
            if ((rc = timing_mark(s, 0))) return rc;
            if (g.timing) {
                g.t_launches++;
                g.t_points += box_points(inner);
                for (int q = 0; q < bnd.nb; ++q) g.t_points += box_points(bnd.boundary[q]);
            }
        }
        if ((rc = test_delay(3, s))) return rc;
        return halo(s);
    }
    const bool on_side = sched == 1, serial = sched == 2;
    hipStream_t bs = on_side ? g.side : s;
    if (on_side) {
        IGG_HIP(hipEventRecord(g.ev_fork, s));
        IGG_HIP(hipStreamWaitEvent(g.side, g.ev_fork, 0));
    }
    if ((rc = test_delay(1, on_side ? g.side : s))) return rc;
    if (bnd.nb) {
        if ((rc = timing_mark(bs, 1))) return rc;
        for (int r = 0; r < g.nranks; ++r)
            if ((rc = boundary(r, bnd, bs))) return rc;
        if ((rc = timing_mark(bs, 1))) return rc;
    }
    if (serial) {
        if ((rc = test_delay(3, s))) return rc;
        if ((rc = halo(s))) return rc;
    } else {
        if (!on_side) {
            IGG_HIP(hipEventRecord(g.ev_fork, s));
            IGG_HIP(hipStreamWaitEvent(g.side, g.ev_fork, 0));
        }
        if ((rc = test_delay(3, g.side))) return rc;
        if ((rc = halo(g.side))) return rc;
        IGG_HIP(hipEventRecord(g.ev_join, g.side));
    }
    if ((rc = test_delay(2, s))) return rc;
    for (int r = 0; r < g.nranks && box_points(inner) > 0; ++r) {
        if ((rc = timing_mark(s, 0))) return rc;
        if ((rc = inner_launch(r, inner, s))) return rc;
        if ((rc = timing_mark(s, 0))) return rc;
        if (g.timing) { g.t_launches++; g.t_points += box_points(inner); }
    }
    if (!serial) IGG_HIP(hipStreamWaitEvent(s, g.ev_join, 0));
    return IGG_OK;
}

// One rank, its own neighbour in every periodic dimension, with the x
// exchange in the stores and the y/z halo filled without send buffers
// (IGG_SLAB_PACK=2).
static bool self_halo_ok()
{
    const Grid &g = grid();
    return g.nranks == 1 && g.fuse_x && g.slab_pack == 2;
}


// Whether a step takes the small-grid kernel: its inner points in three arrays
// of at most 90 MiB (200 x 180 x 100 FP64, 79 MiB: 22.2 us against 24.5; 400 x
// 100 x 100 FP64, 87 MiB: 27.1 against 25.6 on inputs that were not in the
// caches, 19.3 against 26.5 in a time loop; 256^3 FP32, 188 MiB: 61 against 41
// and 38.8 against 46.7); in FP16, whose points cost as many instructions in
// half the bytes, 25 MiB (200 x 180 x 100, 20 MiB: 14.0 against 16.6 with
// stochastic rounding, 13.0 against 12.8 without; 180 x 160 x 200, 32 MiB: 18.2
// against 19.8 and 14.7 against 14.0; 256^3: 45 against 28.7).  Planes of at
// most four inner rows leave most of a z-march tile's threads idle and have
// their rows side by side for the small-grid kernel, which takes them at any
// size (4000 x 6 x 2000 FP64 227 against 327, without periods 186 against 212;
// 4000 x 8 x 2000 322 against 354, 287 against 244).  Or the inner points that
// IGG_ZMARCH_MIN_POINTS asks for.  The split does not come into it: the kernel
// has no slabs.
static bool step_is_small(int dtype, const int n[3])
{
    const int64_t zm = zmarch_min_points(), points = (int64_t)(n[0] - 2) * (n[1] - 2) * (n[2] - 2);
    if (!rows_dispatched()) return points < zm;
    return n[1] <= 6 || points * 3 * elem_bytes(dtype) <= ((int64_t)(dtype == IGG_F16 ? 25 : 90) << 20);
}

// The same for the adjoint: five arrays of at most 96 MiB (128^3 FP64, 76 MiB:
// 23.4 us against 32.1; 160^3 FP32, 75 MiB: 19.9 against 30.3), but 84 MiB in FP64
// where the z-march's tiles leave fewer than a third of their lanes idle.  There,
// from 84 MiB on, this kernel is 2-25% faster with all five arrays in the caches,
// but 3-7% slower in a reverse sweep of single steps, whose states T_n come from
// snapshots that are not, and 9-25% on inputs of which none is; with more lanes
// idle it is 26-39% faster and 9% slower to 6% faster (136 x 104 x 184 28 against 39
// us, 49.5 against 52.6); FP32 19-40% faster, as fast and 4-8% slower.  And rows of
// up to 40 (FP64) or 64 points at any size, which leave z-march tiles' lanes idle
// (42 x 700 x 450 FP64 188 against 196, 46 x 700 x 420 189 against 188; 66 x 600 x
// 350 FP32 87 against 92, 72 x 600 x 320 89 against 86; 13 x 1500 x 600 163 against
// 456 and 79 against 291).
static bool adjoint_is_small(int dtype, const int n[3])
{
    const int64_t zm = zmarch_min_points(), points = (int64_t)(n[0] - 2) * (n[1] - 2) * (n[2] - 2);
    if (!rows_dispatched()) return points < zm;
    const RowTiles t = row_tiles(Box{1, n[0] - 1, 1, n[1] - 1, 1, n[2] - 1}, 2, 128);
    const bool full = dtype == IGG_F64 && (int64_t)3 * (n[0] - 2) > (int64_t)2 * t.n * t.w;
    return n[0] - 2 <= (dtype == IGG_F64 ? 40 : 64) || points * 5 * elem_bytes(dtype) <= ((int64_t)(full ? 84 : 96) << 20);
}

// The same for the flux form: six arrays of at most 96 MiB (160^3 FP32, 98 MB:
// 29.5 us against 40.8 with the halo update; 200 x 180 x 100 FP64, 173 MB: 52.5
// against 50.0), and rows of up to 40 (FP64) or 88 cells at any size (34 x 800 x 500
// FP64 196 against 204, on inputs that were not in the caches 197 against 220; 50 x
// 700 x 400 193 against 167; 78 x 500 x 330 FP32 104 against 112 and 94 against
// 114, 98 x 450 x 310 105 against 100 and 96 against 106).
static bool flux_is_small(int dtype, const int n[3])
{
    const int64_t zm = zmarch_min_points(), points = (int64_t)(n[0] - 2) * (n[1] - 2) * (n[2] - 2);
    if (!rows_dispatched()) return points < zm;
    return n[0] - 2 <= (dtype == IGG_F64 ? 40 : 88) || points * 6 * elem_bytes(dtype) <= ((int64_t)96 << 20);
}

// The step's launch arguments for rank r: its arrays, the fused x exchange
// into its x neighbours' arrays, and its origin in the global index space.
static int step_args(int r, const igg_field *T2, const igg_field *T, const igg_field *Ci, double lam,
                     double dt, double dx, double dy, double dz, uint32_t key, int stochastic, StepArgs &a)
{
    Grid &g = grid();
    int c[3];
    rank_coords(r, c);
    XHalo xh{0, 0, g.ol[0] - 1, g.n[0] - g.ol[0], 0, 0};
    if (g.fuse_x) {
        const int64_t esz = elem_bytes(T2[r].dtype);
        for (int side = 0; side < 2; ++side) {
            const int q = rank_neighbor(r, 0, side);
            if (q < 0) continue;
            const int64_t diff = (int64_t)((intptr_t)T2[q].data - (intptr_t)T2[r].data);
            if (diff % esz) return fail(IGG_ERR_ARG, "T2 blocks must be aligned to their element size");
            (side == 0 ? xh.on_lo : xh.on_hi) = 1;
            (side == 0 ? xh.d_lo : xh.d_hi) = diff / esz;
        }
    }
    // global indices wrap at the period of a periodic dimension (a point and
    // its copies in overlapping planes draw the same random bits)
    int per[3];
    for (int d = 0; d < 3; ++d) per[d] = g.periods[d] ? g.dims[d] * (g.n[d] - g.ol[d]) : 0;
    const int gnx = g.dims[0] * (g.n[0] - g.ol[0]) + g.ol[0];
    const SrOrigin so{c[0] * (g.n[0] - g.ol[0]), c[1] * (g.n[1] - g.ol[1]), c[2] * (g.n[2] - g.ol[2]),
                      gnx, per[0], per[1], per[2], (gnx + 1) / 2};
    a = StepArgs{T2[r].data, T[r].data, Ci[r].data, g.n[0], g.n[1], g.n[2],
                 dt * lam, 1.0 / (dx * dx), 1.0 / (dy * dy), 1.0 / (dz * dz), key, stochastic, xh, so};
    return IGG_OK;
}

// The slabs and the inner region of one step in one launch (schedule 3).
struct FusedStep {
    int dtype;
    const StepArgs *args;
    const SlabPack *pk;
};
static int fused_step(int r, const Split &slabs, const Box &inner, hipStream_t s, void *ctx)
{
    const FusedStep &f = *static_cast<const FusedStep *>(ctx);
    return launch_step_inner(f.dtype, f.args[r], inner, s, &slabs, f.pk);
}

// The argument checks of diffusion_step for the grid's nranks ranks (host
// only).
static int check_step(const igg_field *T2, const igg_field *T, const igg_field *Ci, double lam, double dt, double dx,
                      double dy, double dz, const int split[3], const igg_rounding *rnd)
{
    Grid &g = grid();
    int rc;
    const int P = g.nranks;
    for (int r = 0; r < P; ++r) {
        if ((rc = check_rank_field(&T2[r], "T2", r))) return rc;
        if ((rc = check_rank_field(&T[r], "T", r))) return rc;
        if ((rc = check_rank_field(&Ci[r], "Ci", r))) return rc;
        if (T2[r].dtype != T[0].dtype || T[r].dtype != T[0].dtype || Ci[r].dtype != T[0].dtype)
            return fail(IGG_ERR_DTYPE, "T2, T and Ci must share one dtype");
    }
    for (int r = 0; r < P; ++r)
        for (int q = 0; q < P; ++q) {
            if (overlaps_mem(T2[r], T[q]) || overlaps_mem(T2[r], Ci[q]))
                return fail(IGG_ERR_ALIAS, "T2 shares memory with T or Ci");
            if (q != r && overlaps_mem(T2[r], T2[q])) return fail(IGG_ERR_ALIAS, "two T2 blocks share memory");
        }
    if ((rc = check_spacings(lam, dt, dx, dy, dz))) return rc;
    if ((rc = check_split(split, g.ol))) return rc;
    if (rnd) {
        if (rnd->reserved != 0) return fail(IGG_ERR_ARG, "rounding.reserved must be 0");
        if (rnd->mode != IGG_ROUND_NEAREST && rnd->mode != IGG_ROUND_STOCHASTIC)
            return fail(IGG_ERR_ARG, "unknown rounding mode");
    }
    return IGG_OK;
}

// diffusion_step for the grid's nranks ranks: fields[r] is rank r's block.
static int step_ranks(const igg_field *T2, const igg_field *T, const igg_field *Ci, double lam, double dt,
                      double dx, double dy, double dz, const int split[3], const igg_rounding *rnd,
                      void *stream)
{
    Grid &g = grid();
    int rc;
    const int P = g.nranks;
    if ((rc = check_step(T2, T, Ci, lam, dt, dx, dy, dz, split, rnd))) return rc;
    const int stochastic = rnd && rnd->mode == IGG_ROUND_STOCHASTIC;
    const uint32_t key = rnd ? sr_key(rnd->seed, rnd->counter) : 0;
    std::vector<StepArgs> args(P);
    for (int r = 0; r < P; ++r)
        if ((rc = step_args(r, T2, T, Ci, lam, dt, dx, dy, dz, key, stochastic, args[r]))) return rc;
    if ((rc = ensure_device())) return rc;

    // With x periodic the step kernels also store the x halo of T2 (the
    // exchange between x neighbours on this device is a copy of the two
    // source columns, fused into the kernels that compute them); the halo
    // update then moves the y and z planes only.
    const int halo_dims = g.fuse_x ? 6 : 7;
    const int dtype = T[0].dtype;
    hipStream_t s = (hipStream_t)stream;
    // One rank, x exchange in the stores, no schedule asked for: one launch.
    // Small grids take a kernel of their own; on larger ones the slab waves
    // store the y and z halo planes as they compute the points those planes
    // copy.  Against slabs, halo update and inner region in launches of their
    // own: 256^3 FP64 without periods 83.5 -> 74.7 us, with two 84.6 -> 76.3,
    // unsplit 80.0 -> 73.5.  Whatever the split, there are slabs in periodic
    // dimensions only, of the least width: nothing waits for them, and a slab
    // wave takes longer for a point than a tile (512^3 FP64 with slabs of 100
    // planes 673 us, of 2 533; without periods and slabs 529, with slabs of 2
    // 535; 4000 x 2000 x 4 89 and 105).
    if (self_halo_ok() && (g.schedule < 0 || g.schedule == 3)) {
        args[0].ed = edge_lines();
        if (step_is_small(dtype, g.n)) {
            if ((rc = timing_mark(s, 0))) return rc;
            if ((rc = launch_step_small(dtype, args[0], s))) return rc;
            if ((rc = timing_mark(s, 0))) return rc;
            if (g.timing) {
                g.t_launches++;
                g.t_points += box_points(Box{1, g.n[0] - 1, 1, g.n[1] - 1, 1, g.n[2] - 1});
            }
            return test_delay(3, s);
        }
        SlabPack pk{};
        int widths[3];
        for (int d = 0; d < 3; ++d) {
            pk.ol[d] = g.ol[d];
            pk.per[d] = g.periods[d];
            widths[d] = g.periods[d] ? g.ol[d] : 1;
        }
        pk.direct = 1;
        FusedStep ctx{dtype, args.data(), &pk};
        return run_split(
            widths, dtype, [&](hipStream_t) { return IGG_OK; },
            [&](int r, const Split &b, hipStream_t st) { return launch_step_slabs(dtype, args[r], b, &pk, st); },
            [&](int r, const Box &b, hipStream_t st) { return launch_step_inner(dtype, args[r], b, st); }, s, true,
            fused_step, &ctx);
    }
    if (!split) {
        Box all{1, g.n[0] - 1, 1, g.n[1] - 1, 1, g.n[2] - 1};
        for (int r = 0; r < P; ++r) {
            if ((rc = timing_mark(s, 0))) return rc;
            if ((rc = launch_step_inner(dtype, args[r], all, s))) return rc;
            if ((rc = timing_mark(s, 0))) return rc;
            if (g.timing) { g.t_launches++; g.t_points += box_points(all); }
        }
        return launch_halo(T2, 1, s, halo_dims);
    }
    // One rank, periodic in every dimension, x exchange in the stores: the
    // slab kernel packs the y and z planes as it computes them, and the
    // exchange and unpack are one copy into the halo planes.
    if (P == 1 && g.fuse_x && g.slab_pack && g.periods[0] && g.periods[1] && g.periods[2]) {
        SlabPack pk{};
        pk.direct = g.slab_pack == 2;
        for (int d = 0; d < 2 && !pk.direct; ++d)
            for (int side = 0; side < 2; ++side) pk.send[d][side] = halo_send_plane(0, d, side);
        for (int d = 0; d < 3; ++d) {
            pk.ol[d] = g.ol[d];
            pk.per[d] = 1;
        }
        FusedStep ctx{dtype, args.data(), &pk};
        return run_split(
            split, dtype,
            [&](hipStream_t st) { return pk.direct ? IGG_OK : launch_unpack_self(T2[0], pk, st); },
            [&](int r, const Split &b, hipStream_t st) { return launch_step_slabs(dtype, args[r], b, &pk, st); },
            [&](int r, const Box &b, hipStream_t st) { return launch_step_inner(dtype, args[r], b, st); }, s, true,
            fused_step, &ctx);
    }
    return run_split(
        split, dtype, [&](hipStream_t st) { return launch_halo(T2, 1, st, halo_dims); },
        [&](int r, const Split &b, hipStream_t st) { return launch_step_boundary(dtype, args[r], b, st); },
        [&](int r, const Box &b, hipStream_t st) { return launch_step_inner(dtype, args[r], b, st); }, s);
}

// Whether two steps may run as one launch (launch_step_pair,
// launch_adjoint_pair): one rank, the default schedule, overlaps of 2 in the
// periodic dimensions.  Nothing here changes while the grid lives: a caller
// that planned pairs can launch them.  Timing is about single steps, so where
// it is on none are planned (pairs_planned), but those launched are timed too.
static bool pairs_allowed()
{
    const Grid &g = grid();
    for (int d = 0; d < 3; ++d)
        if (g.periods[d] && g.ol[d] != 2) return false;
    return g.nranks == 1 && g.fuse_x && g.slab_pack == 2 && (g.schedule < 0 || g.schedule == 3) && g.delay_where == 0;
}
static bool pair_ok(int dtype) { return pairs_allowed() && step_pair_pays(dtype, grid().n); }
static bool adjoint_pair_ok(int dtype) { return pairs_allowed() && adjoint_pair_pays(dtype, grid().n); }
static bool pairs_planned() { return !grid().timing; }

// A pair's launch, timed as one launch that computes every inner point twice.
template <typename Launch>
static int timed_pair(hipStream_t s, Launch launch)
{
    Grid &g = grid();
    int rc;
    if ((rc = timing_mark(s, 0))) return rc;
    if ((rc = launch())) return rc;
    if ((rc = timing_mark(s, 0))) return rc;
    if (g.timing) {
        g.t_launches++;
        g.t_points += 2 * box_points(Box{1, g.n[0] - 1, 1, g.n[1] - 1, 1, g.n[2] - 1});
    }
    return IGG_OK;
}

// Two checked steps T -> T2 in one launch, the state between them stored in
// mid when given.
static int step_pair(const igg_field *T2, const igg_field *mid, const igg_field *T, const igg_field *Ci, double lam,
                     double dt, double dx, double dy, double dz, const igg_rounding *rnd, hipStream_t s)
{
    int rc;
    StepArgs a;
    const int stochastic = rnd && rnd->mode == IGG_ROUND_STOCHASTIC;
    if ((rc = step_args(0, T2, T, Ci, lam, dt, dx, dy, dz, 0, stochastic, a))) return rc;
    if ((rc = ensure_device())) return rc;
    const Grid &g = grid();
    const StepPairArgs p{a.T2, mid ? mid->data : nullptr, a.T, a.Ci, a.nx, a.ny, a.nz,
                         {g.periods[0], g.periods[1], g.periods[2]}, a.a, a.rx, a.ry, a.rz,
                         rnd ? sr_key(rnd->seed, rnd->counter) : 0, rnd ? sr_key(rnd->seed, rnd->counter + 1) : 0,
                         stochastic, a.so};
    return timed_pair(s, [&] { return launch_step_pair(T->dtype, p, s); });
}

// update_halo over the grid's ranks: fields[r * nfields + f] is field f of
// rank r; field f has one size and dtype on every rank.
static int update_halo_ranks(const igg_field *fields, int nfields, void *stream)
{
    Grid &g = grid();
    if (!fields) return fail(IGG_ERR_ARG, "fields is null");
    if (nfields < 1 || nfields > IGG_MAX_FIELDS)
        return fail(IGG_ERR_ARG, "nfields must be in 1.." + std::to_string(IGG_MAX_FIELDS));
    int rc;
    const int total = nfields * g.nranks;
    for (int e = 0; e < total; ++e) {
        const int r = e / nfields, f = e % nfields;
        std::string nm = "field " + std::to_string(f) + (g.nranks > 1 ? " of rank " + std::to_string(r) : "");
        if ((rc = check_field(&fields[e], nm.c_str(), false))) return rc;
        const igg_field &f0 = fields[f];
        if (fields[e].dtype != f0.dtype || fields[e].size[0] != f0.size[0] || fields[e].size[1] != f0.size[1] ||
            fields[e].size[2] != f0.size[2])
            return fail(IGG_ERR_SIZE, nm + " differs in size or dtype from the same field of rank 0");
        for (int q = 0; q < e; ++q)
            if (overlaps_mem(fields[e], fields[q]))
                return fail(IGG_ERR_ALIAS, "fields " + std::to_string(q) + " and " + std::to_string(e) +
                                               " share memory");
    }
    if ((rc = ensure_device())) return rc;
    return launch_halo(fields, nfields, (hipStream_t)stream);
}

// The argument checks of an adjoint step for the grid's nranks ranks (host
// only).
static int check_adjoint(const igg_field *lam_n, const igg_field *lam_np1, const igg_field *T_n, const igg_field *Ci,
                         const igg_field *gCi, double lam, double dt, double dx, double dy, double dz,
                         const int split[3])
{
    Grid &g = grid();
    int rc;
    const int P = g.nranks;
    if (!lam_n || !lam_np1 || !T_n || !Ci || !gCi) return fail(IGG_ERR_ARG, "null field");
    const int dt_ = lam_n[0].dtype;
    for (int r = 0; r < P; ++r) {
        if ((rc = check_rank_field(&lam_n[r], "lam_n", r))) return rc;
        if ((rc = check_rank_field(&lam_np1[r], "lam_np1", r))) return rc;
        if ((rc = check_rank_field(&T_n[r], "T_n", r))) return rc;
        if ((rc = check_rank_field(&Ci[r], "Ci", r))) return rc;
        if ((rc = check_rank_field(&gCi[r], "gCi", r))) return rc;
        if (lam_n[r].dtype != dt_ || lam_np1[r].dtype != dt_ || T_n[r].dtype != dt_ || Ci[r].dtype != dt_ ||
            gCi[r].dtype != dt_)
            return fail(IGG_ERR_DTYPE, "adjoint fields must share one dtype");
    }
    if (dt_ == IGG_F16) return fail(IGG_ERR_DTYPE, "the adjoint runs in FP64 or FP32");
    for (int r = 0; r < P; ++r)
        for (int q = 0; q < P; ++q) {
            for (const igg_field *o : {&lam_n[r], &gCi[r]})
                for (const igg_field *i : {&lam_np1[q], &T_n[q], &Ci[q]})
                    if (overlaps_mem(*o, *i)) return fail(IGG_ERR_ALIAS, "an output shares memory with an input");
            if (overlaps_mem(lam_n[r], gCi[q])) return fail(IGG_ERR_ALIAS, "lam_n shares memory with gCi");
            if (q != r && (overlaps_mem(lam_n[r], lam_n[q]) || overlaps_mem(gCi[r], gCi[q])))
                return fail(IGG_ERR_ALIAS, "two ranks' outputs share memory");
        }
    if ((rc = check_spacings(lam, dt, dx, dy, dz))) return rc;
    if ((rc = check_split(split, g.ol))) return rc;
    return IGG_OK;
}

// The adjoint step of either form (0: Laplacian, 1: staggered flux form)
// for the grid's nranks ranks: each argument is an array of one field per
// rank (a single field on a one-rank grid).
static int adjoint_step(int form, const igg_field *lam_n, const igg_field *lam_np1, const igg_field *T_n,
                        const igg_field *Ci, const igg_field *gCi, double lam, double dt, double dx, double dy,
                        double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    int rc;
    const int P = g.nranks;
    if ((rc = check_adjoint(lam_n, lam_np1, T_n, Ci, gCi, lam, dt, dx, dy, dz, split))) return rc;
    const int dt_ = lam_n[0].dtype;
    // per rank: the x exchange of lam_n stored by the adjoint kernels into
    // the x neighbours' lam_n, as in the step
    std::vector<AdjArgs> args(P);
    const int64_t esz = elem_bytes(dt_);
    for (int r = 0; r < P; ++r) {
        XHalo xh{0, 0, g.ol[0] - 1, g.n[0] - g.ol[0], 0, 0};
        if (g.fuse_x)
            for (int side = 0; side < 2; ++side) {
                const int q = rank_neighbor(r, 0, side);
                if (q < 0) continue;
                const int64_t diff = (int64_t)((intptr_t)lam_n[q].data - (intptr_t)lam_n[r].data);
                if (diff % esz) return fail(IGG_ERR_ARG, "lam_n blocks must be aligned to their element size");
                (side == 0 ? xh.on_lo : xh.on_hi) = 1;
                (side == 0 ? xh.d_lo : xh.d_hi) = diff / esz;
            }
        args[r] = form == 0 ? AdjArgs{lam_n[r].data, lam_np1[r].data, T_n[r].data, Ci[r].data, gCi[r].data, g.n[0],
                                      g.n[1], g.n[2], dt * lam, 1.0 / (dx * dx), 1.0 / (dy * dy), 1.0 / (dz * dz),
                                      xh}
                            : AdjArgs{lam_n[r].data, lam_np1[r].data, T_n[r].data, Ci[r].data, gCi[r].data, g.n[0],
                                      g.n[1], g.n[2], dt, 1.0 / dx, 1.0 / dy, 1.0 / dz, xh, 1, lam};
    }
    if ((rc = ensure_device())) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int halo_dims = g.fuse_x ? 6 : 7;
    Box all{1, g.n[0] - 1, 1, g.n[1] - 1, 1, g.n[2] - 1};
    if (self_halo_ok() && (g.schedule < 0 || g.schedule == 3)) {
        // one rank: one launch over every inner point, which also stores the
        // x halo of lam_n and, for every inner point that is the image of y/z
        // halo points, those points (the adjoint runs its chain serially
        // anyway, so the boundary has nothing to overlap)
        AdjArgs a0 = args[0];
        a0.ed = edge_lines();
        a0.yz = YZImg{1, -1, -1, -1, -1, g.n[1], g.n[2]};
        if (g.periods[1]) {
            a0.yz.jl = g.ol[1] - 1;
            a0.yz.jh = g.n[1] - g.ol[1];
        }
        if (g.periods[2]) {
            a0.yz.kl = g.ol[2] - 1;
            a0.yz.kh = g.n[2] - g.ol[2];
        }
        if ((rc = timing_mark(s, 0))) return rc;
        const bool small = adjoint_is_small(dt_, g.n);
        if ((rc = small ? launch_adjoint_small(dt_, a0, s) : launch_adjoint_inner(dt_, a0, all, s))) return rc;
        if ((rc = timing_mark(s, 0))) return rc;
        if (g.timing) { g.t_launches++; g.t_points += box_points(all); }
        return IGG_OK;
    }
    if (!split) {
        for (int r = 0; r < P; ++r) {
            if ((rc = timing_mark(s, 0))) return rc;
            if ((rc = launch_adjoint_inner(dt_, args[r], all, s))) return rc;
            if ((rc = timing_mark(s, 0))) return rc;
            if (g.timing) { g.t_launches++; g.t_points += box_points(all); }
        }
        return launch_halo(lam_n, 1, s, halo_dims);
    }
    return run_split(
        split, dt_, [&](hipStream_t st) { return launch_halo(lam_n, 1, st, halo_dims); },
        [&](int r, const Split &b, hipStream_t st) { return launch_adjoint_boxes(dt_, args[r], b.boundary, b.nb, st); },
        [&](int r, const Box &b, hipStream_t st) { return launch_adjoint_inner(dt_, args[r], b, st); }, s, false);
}

static int check_face(const igg_field *q, const char *name, int dim, int r)
{
    Grid &g = grid();
    int rc;
    if ((rc = check_rank_field(q, name, r, false))) return rc;
    for (int d = 0; d < 3; ++d)
        if (q->size[d] != g.n[d] + (d == dim ? 1 : 0))
            return fail(IGG_ERR_SIZE, std::string(name) + (g.nranks > 1 ? "[" + std::to_string(r) + "]" : "") + " must have n+1 points in its own dimension "
                                                          "and n in the others");
    return IGG_OK;
}


// The fused flux-form step for the grid's nranks ranks: each argument is an
// array of one field per rank (a single field on a one-rank grid).
static int flux_step_ranks(const igg_field *T2, const igg_field *T, const igg_field *Ci, const igg_field *qx,
                           const igg_field *qy, const igg_field *qz, double lam, double dt, double dx, double dy,
                           double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    int rc;
    const int P = g.nranks;
    if (!T2 || !T || !Ci || !qx || !qy || !qz) return fail(IGG_ERR_ARG, "null field");
    const int ty = T[0].dtype;
    for (int r = 0; r < P; ++r) {
        if ((rc = check_rank_field(&T2[r], "T2", r))) return rc;
        if ((rc = check_rank_field(&T[r], "T", r))) return rc;
        if ((rc = check_rank_field(&Ci[r], "Ci", r))) return rc;
        if ((rc = check_face(&qx[r], "qx", 0, r))) return rc;
        if ((rc = check_face(&qy[r], "qy", 1, r))) return rc;
        if ((rc = check_face(&qz[r], "qz", 2, r))) return rc;
        for (const igg_field *f : {&T2[r], &T[r], &Ci[r], &qx[r], &qy[r], &qz[r]})
            if (f->dtype != ty) return fail(IGG_ERR_DTYPE, "flux-form fields must share one dtype");
    }
    if (ty == IGG_F16) return fail(IGG_ERR_DTYPE, "the flux form runs in FP64 or FP32");
    for (int r = 0; r < P; ++r) {
        const igg_field *outs[4] = {&T2[r], &qx[r], &qy[r], &qz[r]};
        for (int o = 0; o < 4; ++o)
            for (int q = 0; q < P; ++q) {
                if (overlaps_mem(*outs[o], T[q]) || overlaps_mem(*outs[o], Ci[q]))
                    return fail(IGG_ERR_ALIAS, "an output shares memory with T or Ci");
                const igg_field *others[4] = {&T2[q], &qx[q], &qy[q], &qz[q]};
                for (int p = 0; p < 4; ++p)
                    if ((q != r || p != o) && overlaps_mem(*outs[o], *others[p]))
                        return fail(IGG_ERR_ALIAS, "outputs share memory");
            }
    }
    if ((rc = check_spacings(lam, dt, dx, dy, dz))) return rc;
    // the face fields overlap their neighbours by ol+1 planes in their own
    // dimension, so each split width must cover that many planes
    const int olf[3] = {g.ol[0] + 1, g.ol[1] + 1, g.ol[2] + 1};
    if ((rc = check_split(split, olf))) return rc;
    // per rank: the x exchange of all four fields is stored by the flux pass
    // into the x neighbours' arrays; the halo update then moves y and z
    std::vector<FluxArgs> args(P);
    const int64_t esz = elem_bytes(ty);
    for (int r = 0; r < P; ++r) {
        FluxXH xh{};
        xh.ol = g.ol[0];
        if (g.fuse_x)
            for (int side = 0; side < 2; ++side) {
                const int q = rank_neighbor(r, 0, side);
                if (q < 0) continue;
                const igg_field *mine[4] = {&T2[r], &qx[r], &qy[r], &qz[r]};
                const igg_field *theirs[4] = {&T2[q], &qx[q], &qy[q], &qz[q]};
                for (int a = 0; a < 4; ++a) {
                    const int64_t diff = (int64_t)((intptr_t)theirs[a]->data - (intptr_t)mine[a]->data);
                    if (diff % esz) return fail(IGG_ERR_ARG, "flux-form blocks must be aligned to their element size");
                    (side == 0 ? xh.d_lo : xh.d_hi)[a] = diff / esz;
                }
                (side == 0 ? xh.on_lo : xh.on_hi) = 1;
            }
        args[r] = FluxArgs{qx[r].data, qy[r].data, qz[r].data, T[r].data, T2[r].data, Ci[r].data, g.n[0], g.n[1],
                           g.n[2], lam, dt, 1.0 / dx, 1.0 / dy, 1.0 / dz, ty, xh};
    }
    if ((rc = ensure_device())) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int halo_dims = g.fuse_x ? 6 : 7;
    std::vector<igg_field> hf((size_t)4 * P);
    for (int r = 0; r < P; ++r) {
        hf[4 * r] = T2[r];
        hf[4 * r + 1] = qx[r];
        hf[4 * r + 2] = qy[r];
        hf[4 * r + 3] = qz[r];
    }
    const Box all{1, g.n[0] - 1, 1, g.n[1] - 1, 1, g.n[2] - 1};
    if (self_halo_ok() && (g.schedule < 0 || g.schedule == 3)) {
        // one rank: every cell in one launch, then the halo of the four
        // fields in one; slabs beside them only read their rows again (256^3
        // FP32 116 us with slabs on the helper stream, 107 without)
        if ((rc = timing_mark(s, 0))) return rc;
        const bool small = flux_is_small(ty, g.n);
        if ((rc = small ? launch_flux_small(ty, args[0], s) : launch_flux_inner(ty, args[0], all, s))) return rc;
        if ((rc = timing_mark(s, 0))) return rc;
        if (g.timing) { g.t_launches++; g.t_points += box_points(all); }
        return launch_halo(hf.data(), 4, s, halo_dims);
    }
    if (!split) {
        for (int r = 0; r < P; ++r) {
            if ((rc = timing_mark(s, 0))) return rc;
            if ((rc = launch_flux_inner(ty, args[r], all, s))) return rc;
            if ((rc = timing_mark(s, 0))) return rc;
            if (g.timing) { g.t_launches++; g.t_points += box_points(all); }
        }
        return launch_halo(hf.data(), 4, s, halo_dims);
    }
    return run_split(
        split, ty, [&](hipStream_t st) { return launch_halo(hf.data(), 4, st, halo_dims); },
        [&](int r, const Split &b, hipStream_t st) { return launch_flux_boxes(ty, args[r], b.boundary, b.nb, st); },
        [&](int r, const Box &b, hipStream_t st) { return launch_flux_inner(ty, args[r], b, st); }, s);
}

}  // namespace igg

using namespace igg;

extern "C" {

const char *igg_last_error(void) { return t_last_error.c_str(); }

const char *igg_version(void) { return "igg-mi355x 0.1 (gfx950)"; }

int igg_init_global_grid(int nx, int ny, int nz, const int dims[3], const int periods[3],
                         const int overlaps[3], int *me)
{
    Grid &g = grid();
    if (g.init) return fail(IGG_ERR_STATE, "the global grid is already initialised");
    int n[3] = {nx, ny, nz};
    int ol[3] = {2, 2, 2}, per[3] = {0, 0, 0}, dm[3] = {1, 1, 1};
    for (int d = 0; d < 3; ++d) {
        if (overlaps) ol[d] = overlaps[d];
        if (periods) per[d] = periods[d];
        if (dims) dm[d] = dims[d] == 0 ? 1 : dims[d];
        if (ol[d] < 2) return fail(IGG_ERR_ARG, "overlaps must be >= 2");
        if (per[d] != 0 && per[d] != 1) return fail(IGG_ERR_ARG, "periods must be 0 or 1");
        if (dm[d] < 0) return fail(IGG_ERR_ARG, "dims must be >= 0");
        if (n[d] < ol[d] + 1)
            return fail(IGG_ERR_ARG, "local size " + std::to_string(n[d]) +
                                         " must exceed the overlap " + std::to_string(ol[d]));
        if (n[d] > (1 << 24)) return fail(IGG_ERR_ARG, "local size above 2^24");
    }
    const int64_t P = (int64_t)dm[0] * dm[1] * dm[2];
    if (P < 1 || P > IGG_MAX_RANKS)
        return fail(IGG_ERR_ARG, "dims must multiply to a rank count in 1.." + std::to_string(IGG_MAX_RANKS));
    if ((int64_t)(nx + 1) * (ny + 1) > 0x7fffffffLL || (int64_t)(nx + 1) * (nz + 1) > 0x7fffffffLL ||
        (int64_t)(ny + 1) * (nz + 1) > 0x7fffffffLL)
        return fail(IGG_ERR_ARG, "a plane of the grid exceeds 2^31 points");
    for (int d = 0; d < 3; ++d) {
        g.n[d] = n[d];
        g.ol[d] = ol[d];
        g.periods[d] = per[d];
        g.dims[d] = dm[d];
    }
    g.nranks = (int)P;
    g.init = true;
    g.timing = false;
    {
        const char *e = getenv("IGG_SCHEDULE");
        const int sv = (e && *e) ? atoi(e) : -1;
        g.schedule = (sv >= 0 && sv <= 3) ? sv : -1;  // anything else: chosen by size and type
        const char *x = getenv("IGG_X_EXCHANGE");
        g.fuse_x = !(x && strcmp(x, "halo") == 0);
        // IGG_TEST_DELAY=<where>:<rounds>, where = side (before the helper
        // stream's first launch), inner (before the inner launch) or halo
        // (before the halo update); rounds of about 3.4 us each, at most 4096
        g.delay_where = 0;
        g.delay_iters = 0;
        const char *td = getenv("IGG_TEST_DELAY");
        if (td && *td) {
            const char *c = strchr(td, ':');
            const size_t len = c ? (size_t)(c - td) : strlen(td);
            int where = 0;
            if (len == 4 && strncmp(td, "side", 4) == 0) where = 1;
            if (len == 5 && strncmp(td, "inner", 5) == 0) where = 2;
            if (len == 4 && strncmp(td, "halo", 4) == 0) where = 3;
            const int it = c ? atoi(c + 1) : 0;
            if (where && it > 0) {
                g.delay_where = where;
                g.delay_iters = std::min(it, 4096);
            }
        }
        const char *sp = getenv("IGG_SLAB_PACK");
        const int spv = (sp && *sp) ? atoi(sp) : -1;
        g.slab_pack = (spv >= 0 && spv <= 2) ? spv : 2;
        const char *zm = getenv("IGG_ZMARCH_MIN_POINTS");
        g.zmarch_min = (zm && *zm) ? atoll(zm) : kZmarchMinPoints;
    }
    g.tev_used = 0;
    g.t_launches = g.t_points = 0;
    if (me) *me = 0;
    return IGG_OK;
}

int igg_global_size(int64_t n_g[3])
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (!n_g) return fail(IGG_ERR_ARG, "n_g is null");
    for (int d = 0; d < 3; ++d)
        n_g[d] = (int64_t)g.dims[d] * (g.n[d] - g.ol[d]) + (int64_t)g.ol[d] * (1 - g.periods[d]);
    return IGG_OK;
}

int igg_topology(int n[3], int dims[3], int periods[3], int overlaps[3], int coords[3])
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    for (int d = 0; d < 3; ++d) {
        if (n) n[d] = g.n[d];
        if (dims) dims[d] = g.dims[d];
        if (periods) periods[d] = g.periods[d];
        if (overlaps) overlaps[d] = g.ol[d];
        if (coords) coords[d] = 0;
    }
    return IGG_OK;
}

int igg_update_halo(const igg_field *fields, int nfields, void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1) return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use igg_update_halo_ranks");
    return update_halo_ranks(fields, nfields, stream);
}

int igg_update_halo_ranks(const igg_field *fields, int nfields, void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    return update_halo_ranks(fields, nfields, stream);
}

int igg_nranks(int *nranks)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (!nranks) return fail(IGG_ERR_ARG, "nranks is null");
    *nranks = g.nranks;
    return IGG_OK;
}

int igg_rank_coords(int rank, int coords[3])
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (!coords) return fail(IGG_ERR_ARG, "coords is null");
    if (rank < 0 || rank >= g.nranks) return fail(IGG_ERR_ARG, "rank out of range");
    rank_coords(rank, coords);
    return IGG_OK;
}

int igg_neighbors(int rank, int lower[3], int upper[3])
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (!lower || !upper) return fail(IGG_ERR_ARG, "null argument");
    if (rank < 0 || rank >= g.nranks) return fail(IGG_ERR_ARG, "rank out of range");
    for (int d = 0; d < 3; ++d) {
        lower[d] = rank_neighbor(rank, d, 0);
        upper[d] = rank_neighbor(rank, d, 1);
    }
    return IGG_OK;
}


int igg_finalize_global_grid(void)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    int rc = release_device();
    g = Grid();
    return rc;
}

int igg_plan_split(const int n[3], const int split[3], int boxes[7][6], int *nboxes)
{
    if (!n || !split || !boxes || !nboxes) return fail(IGG_ERR_ARG, "null argument");
    for (int d = 0; d < 3; ++d) {
        if (n[d] < 3) return fail(IGG_ERR_ARG, "n must be >= 3");
        if (split[d] < 1) return fail(IGG_ERR_ARG, "split widths must be >= 1");
    }
    Split s;
    plan_split(n, split, s);
    for (int q = 0; q < s.nb; ++q) {
        const Box &b = s.boundary[q];
        int v[6] = {b.i0, b.i1, b.j0, b.j1, b.k0, b.k1};
        memcpy(boxes[q], v, sizeof v);
    }
    const Box &b = s.inner;
    int v[6] = {b.i0, b.i1, b.j0, b.j1, b.k0, b.k1};
    memcpy(boxes[s.nb], v, sizeof v);
    *nboxes = s.nb + 1;
    return IGG_OK;
}

int diffusion_step(const igg_field *T2, const igg_field *T, const igg_field *Ci, double lam,
                   double dt, double dx, double dy, double dz, const int split[3],
                   const igg_rounding *rnd, void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1) return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_step_ranks");
    if (!T2 || !T || !Ci) return fail(IGG_ERR_ARG, "null field");
    return step_ranks(T2, T, Ci, lam, dt, dx, dy, dz, split, rnd, stream);
}

int diffusion_step_ranks(const igg_field *T2, const igg_field *T, const igg_field *Ci, double lam,
                         double dt, double dx, double dy, double dz, const int split[3],
                         const igg_rounding *rnd, void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (!T2 || !T || !Ci) return fail(IGG_ERR_ARG, "null field array");
    return step_ranks(T2, T, Ci, lam, dt, dx, dy, dz, split, rnd, stream);
}

int diffusion_run(const igg_field *T, const igg_field *T2, const igg_field *Ci, double lam, double dt,
                  double dx, double dy, double dz, const int split[3], const igg_rounding *rnd, int nt,
                  int use_graph, int *final_buf, void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1) return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_step_ranks");
    if (!T || !T2 || !Ci || !final_buf) return fail(IGG_ERR_ARG, "null argument");
    if (nt < 0) return fail(IGG_ERR_ARG, "nt must be >= 0");
    if (use_graph && rnd && rnd->mode == IGG_ROUND_STOCHASTIC)
        return fail(IGG_ERR_ARG, "graph replays would repeat the stochastic-rounding counter: use_graph = 0");
    hipStream_t s = (hipStream_t)stream;
    int rc;
    *final_buf = 0;
    const igg_field *buf[2] = {T, T2};
    auto round_at = [&](int it, igg_rounding &r) -> const igg_rounding * {
        if (!rnd) return nullptr;
        r = *rnd;
        r.counter += (uint64_t)it;
        return &r;
    };
    // Launches: single steps, and pairs of steps in one launch where they
    // apply.  Every launch swaps the buffers, so an even number of pairs
    // leaves T_nt and T_{nt-1} where single steps would; the first step is a
    // single one, which gives the state the halo the pairs rely on, and the
    // last one too, which leaves T_{nt-1} in the other buffer.
    const int npair = nt >= 6 && pairs_planned() && pair_ok(T->dtype) ? (nt - 2) / 4 * 2 : 0;
    int cur = 0, it = 0;
    auto single = [&](hipStream_t st) {
        igg_rounding r;
        const int e = step_ranks(buf[1 - cur], buf[cur], Ci, lam, dt, dx, dy, dz, split, round_at(it, r), st);
        cur = 1 - cur;
        it += 1;
        return e;
    };
    auto pair = [&](hipStream_t st) {
        igg_rounding r;
        const int e = it == 1 ? check_step(buf[1 - cur], buf[cur], Ci, lam, dt, dx, dy, dz, split, rnd) : IGG_OK;
        if (e) return e;
        const int e2 = step_pair(buf[1 - cur], nullptr, buf[cur], Ci, lam, dt, dx, dy, dz, round_at(it, r), st);
        cur = 1 - cur;
        it += 2;
        return e2;
    };
    // the graph holds up to 16 launches of the loop's repeating part (an even
    // number, so that it ends in the buffer it began with): pairs, or single
    // steps where pairs do not apply
    const int body = npair ? npair : nt / 2 * 2, nrec = std::min(16, body);
    auto direct = [&]() -> int {
        if (npair) {
            if ((rc = single(s))) return rc;
            for (int p = 0; p < npair; ++p)
                if ((rc = pair(s))) return rc;
        }
        while (it < nt)
            if ((rc = single(s))) return rc;
        *final_buf = nt & 1;
        return IGG_OK;
    };
    if (!use_graph || nrec < 2) return direct();
    // A stream that is being captured records the launches themselves: a graph
    // launched on it would not become part of what the caller captures.
    if (s) {
        if ((rc = check_step(T2, T, Ci, lam, dt, dx, dy, dz, split, rnd))) return rc;
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        IGG_HIP(hipStreamIsCapturing(s, &st));
        if (st != hipStreamCaptureStatusNone) return direct();
    }
    std::vector<unsigned char> key;
    auto put = [&](const void *p, size_t n) {
        const unsigned char *c = (const unsigned char *)p;
        key.insert(key.end(), c, c + n);
    };
    for (const igg_field *f : {T, T2, Ci}) put(f, sizeof(igg_field));
    for (double v : {lam, dt, dx, dy, dz}) put(&v, sizeof v);
    const int nosplit[3] = {-1, -1, -1};
    put(split ? split : nosplit, 3 * sizeof(int));
    const int mode = rnd ? rnd->mode : -1;
    put(&mode, sizeof mode);
    put(&nrec, sizeof nrec);
    put(&npair, sizeof npair);
    if (key != g.run_key) {
        // a new argument set is launched directly, and captured when it comes
        // a second time in a row: the capture takes the host longer than the
        // launches it saves in one call (96 x 80 x 64, 50 steps: 226 us with a
        // capture per call, 180 without)
        if ((rc = retire_run_graph(false))) return rc;
        g.run_key = key;
        return direct();
    }
    if (npair && (rc = single(s))) return rc;
    if (!g.run_exec) {
        // both steps run their argument checks while being recorded, and a
        // failed check ends the capture without keeping anything
        if ((rc = ensure_device())) return rc;
        if (!g.cap) IGG_HIP(hipStreamCreateWithFlags(&g.cap, hipStreamNonBlocking));
        const bool timing = g.timing;
        g.timing = false;
        const int cur0 = cur, it0 = it;
        IGG_HIP(hipStreamBeginCapture(g.cap, hipStreamCaptureModeThreadLocal));
        int rc2 = IGG_OK;
        for (int p = 0; p < nrec && !rc2; ++p) rc2 = npair ? pair(g.cap) : single(g.cap);
        cur = cur0;
        it = it0;
        hipGraph_t graph = nullptr;
        hipError_t e = hipStreamEndCapture(g.cap, &graph);
        g.timing = timing;
        if (rc2) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc2;
        }
        if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
        hipGraphExec_t exec = nullptr;
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return hip_fail(e, "hipGraphInstantiate");
        g.run_exec = exec;
    }
    const int replays = body / nrec;
    for (int p = 0; p < replays; ++p) {
        IGG_HIP(hipGraphLaunch(g.run_exec, s));
        it += nrec * (npair ? 2 : 1);
    }
    for (int p = replays * nrec; p < npair; ++p)
        if ((rc = pair(s))) return rc;
    while (it < nt)
        if ((rc = single(s))) return rc;
    *final_buf = nt & 1;
    return IGG_OK;
}

int igg_steps_per_launch(int dtype)
{
    if (!grid().init || dtype < IGG_F64 || dtype > IGG_F16) return 0;
    return pairs_planned() && pair_ok(dtype) ? 2 : 1;
}

int diffusion_step_pair(const igg_field *T2, const igg_field *mid, const igg_field *T, const igg_field *Ci, double lam,
                        double dt, double dx, double dy, double dz, const int split[3], const igg_rounding *rnd,
                        void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1) return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_step_ranks");
    if (!T2 || !T || !Ci) return fail(IGG_ERR_ARG, "null field");
    int rc;
    if ((rc = check_step(T2, T, Ci, lam, dt, dx, dy, dz, split, rnd))) return rc;
    if (mid) {
        if ((rc = check_step(mid, T, Ci, lam, dt, dx, dy, dz, split, rnd))) return rc;
        if (overlaps_mem(*T2, *mid)) return fail(IGG_ERR_ALIAS, "T2 shares memory with mid");
    }
    if (!pair_ok(T->dtype)) return fail(IGG_ERR_STATE, "two steps in one launch do not apply on this grid");
    return step_pair(T2, mid, T, Ci, lam, dt, dx, dy, dz, rnd, (hipStream_t)stream);
}

int diffusion_dt(const igg_field *Ci, double lam, double dx, double dy, double dz, double *dt,
                 void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    int rc;
    if ((rc = check_field(Ci, "Ci", false))) return rc;
    if (!dt) return fail(IGG_ERR_ARG, "dt is null");
    if ((rc = check_spacings(lam, 0.0, dx, dy, dz))) return rc;
    if ((rc = ensure_device())) return rc;
    double m = 0.0;
    if ((rc = launch_reduce(IGG_RED_MAX, *Ci, nullptr, &m, (hipStream_t)stream))) return rc;
    if (!(m > 0.0) || !isfinite(m)) return fail(IGG_ERR_ARG, "maximum(Ci) must be positive and finite");
    double mn = std::min(dx * dx, std::min(dy * dy, dz * dz));
    *dt = mn / lam / m / 6.1;
    return IGG_OK;
}

int diffusion_step_adjoint(const igg_field *lam_n, const igg_field *lam_np1,
                           const igg_field *T_n, const igg_field *Ci, const igg_field *gCi,
                           double lam, double dt, double dx, double dy, double dz,
                           const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1)
        return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_step_adjoint_ranks");
    return adjoint_step(0, lam_n, lam_np1, T_n, Ci, gCi, lam, dt, dx, dy, dz, split, stream);
}

int igg_adjoints_per_launch(int dtype)
{
    if (!grid().init || dtype < IGG_F64 || dtype > IGG_F16) return 0;
    return pairs_planned() && adjoint_pair_ok(dtype) ? 2 : 1;
}

int diffusion_step_adjoint_pair(const igg_field *lam_n, const igg_field *lam_np2, const igg_field *T_n,
                                const igg_field *Ci, const igg_field *gCi, double lam, double dt, double dx, double dy,
                                double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1)
        return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_step_adjoint_ranks");
    int rc;
    if ((rc = check_adjoint(lam_n, lam_np2, T_n, Ci, gCi, lam, dt, dx, dy, dz, split))) return rc;
    if (!adjoint_pair_ok(lam_n->dtype))
        return fail(IGG_ERR_STATE, "two adjoint steps in one launch do not apply on this grid");
    if ((rc = ensure_device())) return rc;
    const AdjPairArgs a{lam_n->data, lam_np2->data, T_n->data, Ci->data, gCi->data,
                        g.n[0], g.n[1], g.n[2], {g.periods[0], g.periods[1], g.periods[2]},
                        dt * lam, 1.0 / (dx * dx), 1.0 / (dy * dy), 1.0 / (dz * dz)};
    return timed_pair((hipStream_t)stream,
                      [&] { return launch_adjoint_pair(lam_n->dtype, a, (hipStream_t)stream); });
}

int diffusion_step_adjoint_ranks(const igg_field *lam_n, const igg_field *lam_np1, const igg_field *T_n,
                                 const igg_field *Ci, const igg_field *gCi, double lam, double dt, double dx,
                                 double dy, double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    return adjoint_step(0, lam_n, lam_np1, T_n, Ci, gCi, lam, dt, dx, dy, dz, split, stream);
}


int diffusion_flux_step(const igg_field *T2, const igg_field *T, const igg_field *Ci,
                        const igg_field *qx, const igg_field *qy, const igg_field *qz, double lam,
                        double dt, double dx, double dy, double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1) return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_flux_step_ranks");
    return flux_step_ranks(T2, T, Ci, qx, qy, qz, lam, dt, dx, dy, dz, split, stream);
}

int diffusion_flux_step_ranks(const igg_field *T2, const igg_field *T, const igg_field *Ci,
                              const igg_field *qx, const igg_field *qy, const igg_field *qz, double lam,
                              double dt, double dx, double dy, double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    return flux_step_ranks(T2, T, Ci, qx, qy, qz, lam, dt, dx, dy, dz, split, stream);
}

int diffusion_flux_step_adjoint(const igg_field *lam_n, const igg_field *lam_np1, const igg_field *T_n,
                                const igg_field *Ci, const igg_field *gCi, double lam, double dt, double dx,
                                double dy, double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (g.nranks > 1)
        return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: use diffusion_flux_step_adjoint_ranks");
    return adjoint_step(1, lam_n, lam_np1, T_n, Ci, gCi, lam, dt, dx, dy, dz, split, stream);
}

int diffusion_flux_step_adjoint_ranks(const igg_field *lam_n, const igg_field *lam_np1, const igg_field *T_n,
                                      const igg_field *Ci, const igg_field *gCi, double lam, double dt, double dx,
                                      double dy, double dz, const int split[3], void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    return adjoint_step(1, lam_n, lam_np1, T_n, Ci, gCi, lam, dt, dx, dy, dz, split, stream);
}

// Argument checks of igg_reduce and igg_reduce_noalloc (host only); *two is
// set when the operation reads b.
static int check_reduce(int op, const igg_field *a, const igg_field *b, const double *out, bool *two)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    if (!out) return fail(IGG_ERR_ARG, "out is null");
    if (op < IGG_RED_MAX || op > IGG_RED_MAX_ABS) return fail(IGG_ERR_ARG, "unknown reduction");
    int rc;
    if ((rc = check_field(a, "a", false))) return rc;
    *two = op == IGG_RED_SUM_RATIO || op == IGG_RED_HALF_SQDIFF || op == IGG_RED_DOT || op == IGG_RED_MAX_ABS_DIFF;
    if (*two) {
        if ((rc = check_field(b, "b", false))) return rc;
        for (int d = 0; d < 3; ++d)
            if (a->size[d] != b->size[d]) return fail(IGG_ERR_SIZE, "a and b differ in size");
        if (a->dtype != b->dtype) return fail(IGG_ERR_DTYPE, "a and b must share one dtype");
    }
    return IGG_OK;
}

int igg_reduce(int op, const igg_field *a, const igg_field *b, double *out, void *stream)
{
    bool two = false;
    int rc;
    if ((rc = check_reduce(op, a, b, out, &two))) return rc;
    if ((rc = ensure_device())) return rc;
    return launch_reduce(op, *a, two ? b : nullptr, out, (hipStream_t)stream);
}

int igg_adjoint_seed(const igg_field *T, const igg_field *T_obs, const igg_field *lam, int halo, double *loss,
                     void *stream)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    int rc;
    if ((rc = check_field(lam, "lam", true))) return rc;
    if (T_obs && !T) return fail(IGG_ERR_ARG, "T_obs without T");
    if (loss && !T_obs) return fail(IGG_ERR_ARG, "the loss needs T and T_obs");
    if (halo != 0 && halo != 1) return fail(IGG_ERR_ARG, "halo must be 0 or 1");
    if (halo && g.nranks > 1)
        return fail(IGG_ERR_STATE, "the grid holds several virtual ranks: seed each block with halo = 0, then "
                                   "igg_update_halo_ranks");
    for (const igg_field *f : {T, T_obs}) {
        if (!f) continue;
        if ((rc = check_field(f, f == T ? "T" : "T_obs", true))) return rc;
        if (f->dtype != lam->dtype) return fail(IGG_ERR_DTYPE, "T, T_obs and lam must share one dtype");
        if (overlaps_mem(*f, *lam)) return fail(IGG_ERR_ALIAS, "lam shares memory with an input");
    }
    if ((rc = ensure_device())) return rc;
    hipStream_t s = (hipStream_t)stream;
    RedSlots slots;
    if ((rc = launch_seed(T, T_obs, *lam, loss ? &slots : nullptr, s))) return rc;
    if (halo && (rc = launch_halo(lam, 1, s))) return rc;
    return loss ? read_seed_loss(slots, loss, s) : IGG_OK;
}

int igg_reduce_noalloc(int op, const igg_field *a, const igg_field *b, double *out_dev, void *stream)
{
    bool two = false;
    int rc;
    if ((rc = check_reduce(op, a, b, out_dev, &two))) return rc;
    return launch_reduce_noalloc(op, *a, two ? b : nullptr, out_dev, (hipStream_t)stream);
}

int igg_timing_enable(int on)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    g.timing = on != 0;
    if (g.timing) {
        // make the event pool now, so that timed work does not pay for
        // creating events (it grows later if more launches are timed)
        int rc;
        if ((rc = ensure_device())) return rc;
        while (g.tev.size() < kTimingPool) {
            hipEvent_t e;
            IGG_HIP(hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
            g.tev.push_back(e);
            g.tev_kind.push_back(0);
        }
    }
    return IGG_OK;
}

int igg_timing_read(double *ms, int64_t *launches, int64_t *points, double *boundary_ms)
{
    Grid &g = grid();
    if (!g.init) return fail(IGG_ERR_STATE, "the global grid is not initialised");
    double total[2] = {0.0, 0.0};
    for (size_t q = 0; q + 1 < g.tev_used; q += 2) {
        float t = 0.f;
        IGG_HIP(hipEventSynchronize(g.tev[q + 1]));
        IGG_HIP(hipEventElapsedTime(&t, g.tev[q], g.tev[q + 1]));
        total[g.tev_kind[q] ? 1 : 0] += t;
    }
    if (ms) *ms = total[0];
    if (boundary_ms) *boundary_ms = total[1];
    if (launches) *launches = g.t_launches;
    if (points) *points = g.t_points;
    g.tev_used = 0;
    g.t_launches = g.t_points = 0;
    return IGG_OK;
}

}  // extern "C"
