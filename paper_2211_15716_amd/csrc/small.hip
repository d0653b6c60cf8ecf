// small.hip -- one step of the time loop on one rank in one launch, halo update
// included, for grids that sit in the caches: a thread per column of a few
// points, plain loads and stores.  Any periods and overlaps.
//
// Every inner point goes through igg::diffuse, so its bits are those of the
// kernels in step.hip.  The point a halo point of a periodic dimension copies
// (plane ol-1 for plane n-1, plane n-ol for plane 0) is stored there too by
// the thread that computes it.  Where some dimensions have a period and
// others none, the points in which the latter's planes meet the former's halo
// are copied by the launch's last work-groups (k_step_edges after the z-march
// kernel), as the halo update copies them: their sources are points that no
// step writes.
#include "host.hpp"

namespace igg {

namespace {

template <typename C> struct OneCoef {
    C a, rx, ry, rz;
};

struct OneGeom {
    int n[3];
    int per[3];
    int lo[3], hi[3];  // per dimension: the plane copied to plane n-1, and to plane 0
};

// ------------------------------------------------------------------- edges
// y and z halo planes of periodic y and z at the points where another
// dimension has no period: point (i, j, k) takes the value at the images of j
// and k.  Line by line, e = 0..: count in one_edges().
struct OneEdges {
    int64_t first;   // first work-group of the edges
    int line[3];     // points per dimension whose lines exist (0: none): along x, y, z
    int total;
};

template <typename S>
__device__ __forceinline__ void one_edge_point(S *A, const OneGeom &g, const OneEdges &ed, int e)
{
    // lines along x (y and z at a boundary), along y (x and z), along z (x and y)
    int c[3], d = 0;
    while (d < 2 && e >= 4 * ed.line[d]) e -= 4 * ed.line[d++];
    const int l = ed.line[d];
    const int s = e / l, a = d == 0 ? 1 : 0, b = d == 2 ? 1 : 2;
    c[d] = e - s * l;
    c[a] = s & 1 ? g.n[a] - 1 : 0;
    c[b] = s & 2 ? g.n[b] - 1 : 0;
    bool fixed = false, moved = false;
    int m[3] = {c[0], c[1], c[2]};
    for (int q = 0; q < 3; ++q) {
        const bool end = c[q] == 0 || c[q] == g.n[q] - 1;
        if (!end) continue;
        if (!g.per[q]) fixed = true;
        else if (q > 0) {
            m[q] = c[q] == 0 ? g.hi[q] : g.lo[q];
            moved = true;
        }
    }
    if (!fixed || !moved) return;
    const int64_t sy = g.n[0], sz = (int64_t)g.n[0] * g.n[1];
    A[c[0] + sy * c[1] + sz * c[2]] = A[m[0] + sy * m[1] + sz * m[2]];
}

template <typename S>
__global__ void __launch_bounds__(256) k_step_edges(S *__restrict__ T2, OneGeom g, OneEdges ed)
{
    const int e = (int)blockIdx.x * 256 + threadIdx.x;
    if (e < ed.total) one_edge_point(T2, g, ed, e);
}

// Stores v at (i, j, k) and at the halo points that copy it.
template <typename S>
__device__ __forceinline__ void one_store(const OneGeom &g, int i, int j, int k, S *A, S v)
{
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    S *P = A + (i + sy * j + sz * k);
    *P = v;
    const bool xe = g.per[0] && (i == g.lo[0] || i == g.hi[0]), ye = g.per[1] && (j == g.lo[1] || j == g.hi[1]);
    const bool ze = g.per[2] && (k == g.lo[2] || k == g.hi[2]);
    if (!xe && !ye && !ze) return;
    const int64_t dx[3] = {0, xe && i == g.lo[0] ? nx - 1 - i : 0, xe && i == g.hi[0] ? -i : 0};
    const int64_t dy[3] = {0, ye && j == g.lo[1] ? sy * (ny - 1 - j) : 0, ye && j == g.hi[1] ? -sy * j : 0};
    const int64_t dz[3] = {0, ze && k == g.lo[2] ? sz * (nz - 1 - k) : 0, ze && k == g.hi[2] ? -sz * k : 0};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (c && !dz[c]) continue;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if (b && !dy[b]) continue;
#pragma unroll
            for (int a = 0; a < 3; ++a)
                if (!a ? (b || c) : dx[a] != 0) P[dx[a] + dy[b] + dz[c]] = v;
        }
    }
}

// ------------------------------------------------------------- small grids
// 256 consecutive inner points of a plane per work-group, in NZ planes, so no
// lane idles at any row length.  Bound by the launch and the loads' latency,
// which NZ independent columns of loads cover.  Against the boundary slabs and
// the box kernel or z-march in their launches: 128^3 FP64 12.5 us a step
// against 23.7, 96 x 80 x 64 9 against 13, 160^3 FP32 12.7 against 15.7,
// 69 x 300 x 301 FP32 17.4 against 34.8.
template <typename S, int NZ, int SR>
__global__ void __launch_bounds__(256)
k_step_small(S *__restrict__ T2, const S *__restrict__ T, const S *__restrict__ Ci, OneGeom g, OneEdges ed, int nbp,
             OneCoef<compute_t<S>> cf, uint32_t key, SrOrigin so)
{
    using C = compute_t<S>;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    if (blockIdx.x >= ed.first) {
        const int e = (int)(blockIdx.x - ed.first) * 256 + threadIdx.x;
        if (e < ed.total) one_edge_point(T2, g, ed, e);
        return;
    }
    const uint32_t b = (uint32_t)xcd_remap(blockIdx.x, ed.first);
    const uint32_t bp = b % (uint32_t)nbp, bz = b / (uint32_t)nbp;
    const uint32_t q = bp * 256 + threadIdx.x, w = (uint32_t)(nx - 2);
    const int j = 1 + (int)(q / w), i = 1 + (int)(q % w), k0 = 1 + (int)bz * NZ;
    if (j > ny - 2) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    const int64_t p0 = i + sy * j + sz * k0;
    S z[NZ + 2], xm[NZ], xp[NZ], ym[NZ], yp[NZ], ci[NZ];
    // (planes past the last inner one read the last ones again)
#pragma unroll
    for (int t = 0; t < NZ + 2; ++t) z[t] = T[p0 + sz * (min(k0 - 1 + t, nz - 1) - k0)];
#pragma unroll
    for (int t = 0; t < NZ; ++t) {
        const int64_t p = p0 + sz * (min(k0 + t, nz - 2) - k0);
        xm[t] = T[p - 1];
        xp[t] = T[p + 1];
        ym[t] = T[p - sy];
        yp[t] = T[p + sy];
        ci[t] = Ci[p];
    }
#pragma unroll
    for (int t = 0; t < NZ; ++t) {
        const int k = k0 + t;
        if (k > nz - 2) break;
        const C o = diffuse<C>(widen<C>(z[t + 1]), widen<C>(xm[t]), widen<C>(xp[t]), widen<C>(ym[t]), widen<C>(yp[t]),
                               widen<C>(z[t]), widen<C>(z[t + 2]), widen<C>(ci[t]), cf.a, cf.rx, cf.ry, cf.rz);
        uint32_t r = 0;
        if (SR) r = sr_point_bits(sr_plane_key(key, k, so), i, j, so);
        one_store(g, i, j, k, T2, Store<S>::put(o, r, SR));
    }
}

OneGeom geom(const int n[3])
{
    const Grid &gr = grid();
    OneGeom g;
    for (int d = 0; d < 3; ++d) {
        g.n[d] = n[d];
        g.per[d] = gr.periods[d];
        g.lo[d] = gr.ol[d] - 1;
        g.hi[d] = n[d] - gr.ol[d];
    }
    return g;
}

// The edge lines of a grid of mixed periods (none otherwise), after `first`
// work-groups; returns the number of work-groups they add.
int64_t one_edges(const OneGeom &g, int64_t first, int threads, OneEdges &ed)
{
    ed = OneEdges{first, {0, 0, 0}, 0};
    const int np = g.per[0] + g.per[1] + g.per[2];
    if (np == 0 || np == 3 || (!g.per[1] && !g.per[2])) return 0;
    for (int d = 0; d < 3; ++d) {
        ed.line[d] = g.n[d];
        ed.total += 4 * g.n[d];
    }
    return (ed.total + threads - 1) / threads;
}

template <typename S, int NZ>
int run_small(const StepArgs &a, hipStream_t s)
{
    using C = compute_t<S>;
    const int n[3] = {a.nx, a.ny, a.nz};
    const OneGeom g = geom(n);
    const int nbp = (int)(((int64_t)(a.nx - 2) * (a.ny - 2) + 255) / 256);
    int64_t blocks = (int64_t)nbp * ((a.nz - 2 + NZ - 1) / NZ);
    OneEdges ed;
    blocks += one_edges(g, blocks, 256, ed);
    const OneCoef<C> cf{(C)a.a, (C)a.rx, (C)a.ry, (C)a.rz};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, (S *)a.T2, (const S *)a.T, (const S *)a.Ci, g,
                           ed, nbp, cf, a.key, a.so);
    };
    if constexpr (sizeof(S) == 2) {
        if (a.stochastic) {
            go(k_step_small<S, NZ, 1>);
            IGG_HIP(hipGetLastError());
            return IGG_OK;
        }
    }
    go(k_step_small<S, NZ, 0>);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

template <typename S>
int run_edges(void *A, const int n[3], hipStream_t s)
{
    OneEdges ed;
    const OneGeom g = geom(n);
    const int64_t blocks = one_edges(g, 0, 256, ed);
    if (blocks == 0) return IGG_OK;
    hipLaunchKernelGGL(k_step_edges<S>, dim3((unsigned)blocks), dim3(256), 0, s, (S *)A, g, ed);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

}  // namespace

// Columns of 4 points, 2 where that would leave fewer than 512 work-groups.
template <typename S>
static int small_typed(const StepArgs &a, hipStream_t s)
{
    const int64_t blocks = ((int64_t)(a.nx - 2) * (a.ny - 2) + 255) / 256 * ((a.nz + 1) / 4);
    return blocks < 512 ? run_small<S, 2>(a, s) : run_small<S, 4>(a, s);
}

int launch_step_small(int dtype, const StepArgs &a, hipStream_t s)
{
    if (dtype == IGG_F64) return small_typed<double>(a, s);
    if (dtype == IGG_F32) return small_typed<float>(a, s);
    return small_typed<_Float16>(a, s);
}

int launch_step_edges(int dtype, void *A, const int n[3], hipStream_t s)
{
    if (dtype == IGG_F64) return run_edges<double>(A, n, s);
    if (dtype == IGG_F32) return run_edges<float>(A, n, s);
    return run_edges<_Float16>(A, n, s);
}

}  // namespace igg
