// small.hip -- one step of the time loop on one rank in one launch, halo update
// included, for grids that sit in the caches: a thread per column of a few
// points, plain loads and stores.  Any periods and overlaps.
//
// Every inner point goes through igg::diffuse, so its bits are those of the
// kernels in step.hip.  The point a halo point of a periodic dimension copies
// (plane ol-1 for plane n-1, plane n-ol for plane 0) is stored there too by
// the thread that computes it.  Where some dimensions have a period and
// others none, the points in which the latter's planes meet the former's halo
// are copied by the launch's last work-groups (EdgeLines).
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
k_step_small(S *__restrict__ T2, const S *__restrict__ T, const S *__restrict__ Ci, OneGeom g, EdgeLines ed, int first_edge, int nbp,
             OneCoef<compute_t<S>> cf, uint32_t key, SrOrigin so)
{
    using C = compute_t<S>;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    if ((int)blockIdx.x >= first_edge) {
        const int e = ((int)blockIdx.x - first_edge) * 256 + threadIdx.x;
        if (e < ed.total) edge_point(T2, ed, e);
        return;
    }
    const uint32_t b = (uint32_t)xcd_remap(blockIdx.x, first_edge);
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

template <typename S, int NZ>
int run_small(const StepArgs &a, hipStream_t s)
{
    using C = compute_t<S>;
    const int n[3] = {a.nx, a.ny, a.nz};
    const OneGeom g = geom(n);
    const int nbp = (int)(((int64_t)(a.nx - 2) * (a.ny - 2) + 255) / 256);
    const int main = (int)((int64_t)nbp * ((a.nz - 2 + NZ - 1) / NZ));
    const int64_t blocks = (int64_t)main + (a.ed.total + 255) / 256;
    const OneCoef<C> cf{(C)a.a, (C)a.rx, (C)a.ry, (C)a.rz};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, (S *)a.T2, (const S *)a.T, (const S *)a.Ci, g,
                           a.ed, main, nbp, cf, a.key, a.so);
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

EdgeLines edge_lines()
{
    const Grid &g = grid();
    EdgeLines ed{};
    for (int d = 0; d < 3; ++d) {
        ed.n[d] = g.n[d];
        ed.per[d] = g.periods[d];
    }
    ed.ylo = g.ol[1] - 1;
    ed.yhi = g.n[1] - g.ol[1];
    ed.zlo = g.ol[2] - 1;
    ed.zhi = g.n[2] - g.ol[2];
    const bool all = g.periods[0] && g.periods[1] && g.periods[2];
    if (!all && (g.periods[1] || g.periods[2])) ed.total = 4 * (g.n[0] + g.n[1] + g.n[2]);
    return ed;
}

}  // namespace igg
