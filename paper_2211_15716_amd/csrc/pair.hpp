// pair.hpp -- what the kernels that take two steps in one launch share: the
// geometry of one rank, the stores that fill a halo, and the choice of tiles.
#pragma once

#include "host.hpp"

namespace igg {

struct PairGeom {
    int n[3];
    int per[3];
};

// Stores v at (i, j, k) and at the halo points whose image it is in periodic
// dimensions of overlap 2.
template <typename S>
__device__ __forceinline__ void pair_store(const PairGeom &g, int i, int j, int k, S *A, S v)
{
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    S *P = A + (i + sy * j + sz * k);
    *P = v;
    const bool xe = g.per[0] && (i == 1 || i == nx - 2), ye = g.per[1] && (j == 1 || j == ny - 2);
    const bool ze = g.per[2] && (k == 1 || k == nz - 2);
    if (!xe && !ye && !ze) return;
    // the distance to the image in each dimension, twice where both halo
    // planes copy the point (n = 3)
    const int64_t dx[3] = {0, xe && i == 1 ? nx - 2 : 0, xe && i == nx - 2 ? -(nx - 2) : 0};
    const int64_t dy[3] = {0, ye && j == 1 ? sy * (ny - 2) : 0, ye && j == ny - 2 ? -sy * (ny - 2) : 0};
    const int64_t dz[3] = {0, ze && k == 1 ? sz * (nz - 2) : 0, ze && k == nz - 2 ? -sz * (nz - 2) : 0};
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

// The plane, row or column read for index c in -1..n (others: clamped): in a
// periodic dimension the one the halo update copies it from.  Ci's own halo is
// never read, nor are T's edges, where a plane of a dimension without a period
// meets a halo plane (a step leaves them as they are).
__device__ __forceinline__ int wrap(int c, int n, int per)
{
    if (per) c = c <= 0 ? c + n - 2 : (c >= n - 1 ? c - (n - 2) : c);
    return c < 0 ? 0 : (c > n - 1 ? n - 1 : c);
}

// Stores a vector of VEC points from (i, j, k) on: its inner points (not all
// of them need be), and the halo points whose images they are.
template <typename S, int VEC, typename V>
__device__ __forceinline__ void pair_put(const PairGeom &g, S *A, int i, int j, int k, const V &v, int nt)
{
    constexpr uint32_t E = sizeof(S);
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int64_t sxy = (int64_t)nx * ny;
    const bool full = i >= 1 && i + VEC <= nx - 1;
    const bool xedge = g.per[0] && (i <= 1 || i + VEC >= nx - 1);
    auto row = [&](int kk, int jj) {
        const __amdgpu_buffer_rsrc_t d = buf_rsrc(A + (int64_t)kk * sxy, sxy * (int64_t)E);
        const uint32_t o = (uint32_t)(jj * nx) * E;
        if (full) {
            if (nt) buf_store<V, 2>(v, d, o + (uint32_t)i * E);
            else buf_store<V, 0>(v, d, o + (uint32_t)i * E);
        } else {
#pragma unroll
            for (int q = 0; q < VEC; ++q)
                if (i + q >= 1 && i + q <= nx - 2) buf_store<S, 0>(v[q], d, o + (uint32_t)(i + q) * E);
        }
        if (xedge) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                if (i + q == 1) buf_store<S, 0>(v[q], d, o + (uint32_t)(nx - 1) * E);
                if (i + q == nx - 2) buf_store<S, 0>(v[q], d, o);
            }
        }
    };
    row(k, j);
    if ((g.per[2] && (k == 1 || k == nz - 2)) || (g.per[1] && (j == 1 || j == ny - 2))) {
#pragma unroll 1
        for (int m = 1; m < 9; ++m) {
            const int a = m % 3, c = m / 3;
            const int jj = a == 0 ? j : (!g.per[1] ? -1 : a == 1 ? (j == 1 ? ny - 1 : -1) : (j == ny - 2 ? 0 : -1));
            const int kk = c == 0 ? k : (!g.per[2] ? -1 : c == 1 ? (k == 1 ? nz - 1 : -1) : (k == nz - 2 ? 0 : -1));
            if (kk >= 0 && jj >= 0) row(kk, jj);
        }
    }
}

// Tiles of the kernels that march z: work-groups of W vectors (the tile's and
// one on each side) by HG groups of RY rows.
struct PairTile {
    PairGeom g;
    int W, HG;       // vectors and row groups of the work-group
    int ntx, nty;    // tiles
    int zc;          // planes per work-group
    int nt;          // 1: non-temporal stores
    int deal;        // 1: tile rows dealt to the XCDs in turn, 0: in ranges
};

// The tile and the planes per work-group for which the launch ends
// soonest: rounds of 256 work-groups (one of 700 to 1024 threads per CU;
// two of half the size read more rows around their tiles), each of zc
// planes and about one more to fill the pipeline, a plane costing a fixed
// time, one for its points and a little for its width.  Tiles start at
// whole 128-byte lines of a row (512^3 FP64: 650 us a launch against 661
// with the vectors beside the tile in the same waves as the tile's).
// Over 13 grids from 160^3 to 512^3 the choice is 4% slower than the
// fastest of about 200 shapes on average and 11% at worst; a launch of
// just over 256 work-groups instead costs up to twice the time.
template <int VEC, int RY>
void pair_tiles(int nx, int ny, int nz, PairTile &z)
{
    const int nv = (nx - 2) / VEC + 1;  // vectors up to that of the last inner point
    double best = 0;
    for (int target = 128; target >= 32; target /= 2) {
        const int ntx = (nv + target - 1) / target, W = ((nv + ntx - 1) / ntx + 7) / 8 * 8 + 2;
        if (best > 0 && W < (RY == 1 ? 34 : 42)) continue;
        for (int hg = 1024 / W; hg * RY >= 6 && hg * W > 700 - W; --hg) {
            const int th = hg * RY - 4;
            const int64_t cols = (int64_t)ntx * ((ny - 2 + th - 1) / th);
            for (int zc = 6; zc <= 64; ++zc) {
                const int64_t wg = cols * ((nz - 2 + zc - 1) / zc);
                const double cost = (double)((wg + 255) / 256) * (zc + 1) * (400 + th * (W - 2) + 2 * W);
                if (best == 0 || cost < best) {
                    best = cost;
                    z.ntx = ntx;
                    z.W = W;
                    z.HG = hg;
                    z.zc = zc;
                }
            }
        }
    }
    z.nty = (ny - 2 + z.HG * RY - 5) / (z.HG * RY - 4);
}

}  // namespace igg
