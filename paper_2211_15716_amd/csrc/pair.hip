// pair.hip -- two steps of the time loop in one launch.
//
// T_{n+1} = u is computed from T_n tile by tile, kept on chip, and T_{n+2} is
// computed from it: T_n and Ci are read and T_{n+2} is written once for two
// steps instead of once for each.  Every point of u and of T_{n+2} goes
// through igg::diffuse with the operands the one-step kernels give it, so the
// bits are those of two single steps.  A work-group recomputes the u points
// its tile shares with its neighbours (one layer on every side).
//
// One rank, overlaps of 2 in the periodic dimensions.  The halo of u is
// formed as the halo update would: in a periodic dimension the point of plane
// 0 is the point of plane n-2 and that of plane n-1 the point of plane 1; in
// a dimension without a period it keeps T_n's value.  The halo of T_{n+2} is
// stored with the points it copies.
#include "pair.hpp"

namespace igg {

namespace {

template <typename C> struct PairCoef {
    C a, rx, ry, rz;
};

// ------------------------------------------------------------ small grids
// One block of BX x BY x BZ points of T_{n+2} per work-group: the u points of
// the block and one layer around it go to LDS, each from global loads of its
// seven T points (the grid sits in the caches), then the block is computed
// from LDS.  Bound by its instructions, the chain of its loads and the launch:
// 1024 threads for the fewest points in turn per thread, 32-bit byte offsets
// (arrays below 2^31 bytes).  Per step in a time loop: 32^3 FP64 1.7 us
// against 3.2 for a launch per step, 96 x 80 x 64 3.5 against 5.1, 128^3 9.8
// against 12.1, FP32 6.9 against 7.5.  Slower: 256 threads and blocks of 16 x
// 4 x 4 (96 x 80 x 64 4.4), a T tile in LDS too (its own index arithmetic),
// and the loads of three points at a time issued together.
template <typename S, int BX, int BY, int BZ, int SR, int MID>
__global__ void __launch_bounds__(1024)
k_step2_block(S *__restrict__ out, S *__restrict__ mid, const S *__restrict__ T, const S *__restrict__ Ci, PairGeom g,
              int nbx, int nby, PairCoef<compute_t<S>> cf, uint32_t key1, uint32_t key2, SrOrigin so)
{
    using C = compute_t<S>;
    constexpr int UX = BX + 2, UY = BY + 2, UZ = BZ + 2, NU = UX * UY * UZ, NO = BX * BY * BZ, NT = 1024;
    constexpr uint32_t E = sizeof(S);
    __shared__ C u[UZ][UY][UX];
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = 1 + b % nbx * BX, y0 = 1 + b / nbx % nby * BY, z0 = 1 + b / nbx / nby * BZ;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const uint32_t ey = (uint32_t)nx * E, ez = ey * (uint32_t)ny;
    auto ld = [](const S *A, uint32_t o) -> C {
        return widen<C>(*reinterpret_cast<const S *>(reinterpret_cast<const char *>(A) + o));
    };
#pragma unroll
    for (int t = 0; t < (NU + NT - 1) / NT; ++t) {
        const int q = t * NT + threadIdx.x;
        const int ux = q % UX, uy = q / UX % UY, uz = q / (UX * UY);
        const int x = x0 - 1 + ux, y = y0 - 1 + uy, z = z0 - 1 + uz;
        // edges and corners of the layer are nobody's neighbours
        const int sides = (ux == 0 || ux == UX - 1) + (uy == 0 || uy == UY - 1) + (uz == 0 || uz == UZ - 1);
        if (q >= NU || x >= nx || y >= ny || z >= nz || sides > 1) continue;
        const bool hx = x == 0 || x == nx - 1, hy = y == 0 || y == ny - 1, hz = z == 0 || z == nz - 1;
        C v;
        if ((hx && !g.per[0]) || (hy && !g.per[1]) || (hz && !g.per[2])) {
            v = ld(T, (uint32_t)x * E + ey * (uint32_t)y + ez * (uint32_t)z);
        } else {
            const int xi = hx ? wrap(x, nx, 1) : x, yi = hy ? wrap(y, ny, 1) : y, zi = hz ? wrap(z, nz, 1) : z;
            const uint32_t p = (uint32_t)xi * E + ey * (uint32_t)yi + ez * (uint32_t)zi;
            const C o = diffuse<C>(ld(T, p), ld(T, p - E), ld(T, p + E), ld(T, p - ey), ld(T, p + ey), ld(T, p - ez),
                                   ld(T, p + ez), ld(Ci, p), cf.a, cf.rx, cf.ry, cf.rz);
            uint32_t r = 0;
            if (SR) r = sr_point_bits(sr_plane_key(key1, zi, so), xi, yi, so);
            const S s = Store<S>::put(o, r, SR);
            v = widen<C>(s);
            if (MID && sides == 0 && !hx && !hy && !hz)
                pair_store(g, x, y, z, mid, s);
        }
        u[uz][uy][ux] = v;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NO / NT; ++t) {
        const int q = t * NT + threadIdx.x;
        const int ux = 1 + q % BX, uy = 1 + q / BX % BY, uz = 1 + q / (BX * BY);
        const int x = x0 - 1 + ux, y = y0 - 1 + uy, z = z0 - 1 + uz;
        if (x > nx - 2 || y > ny - 2 || z > nz - 2) continue;
        const C o = diffuse<C>(u[uz][uy][ux], u[uz][uy][ux - 1], u[uz][uy][ux + 1], u[uz][uy - 1][ux],
                               u[uz][uy + 1][ux], u[uz - 1][uy][ux], u[uz + 1][uy][ux],
                               ld(Ci, (uint32_t)x * E + ey * (uint32_t)y + ez * (uint32_t)z), cf.a, cf.rx, cf.ry,
                               cf.rz);
        uint32_t r = 0;
        if (SR) r = sr_point_bits(sr_plane_key(key2, z, so), x, y, so);
        pair_store(g, x, y, z, out, Store<S>::put(o, r, SR));
    }
}

// ------------------------------------------------------------ large grids
// z-march over tiles of TWV vectors (16 bytes) x TH rows.  The work-group's
// threads cover the tile and what the two steps read around it: W = TWV + 2
// vectors (one on each side) by H = TH + 4 rows, each thread RY rows of one
// vector: first the tile's columns, rows following each other through the
// waves, then the vectors beside it.  At plane k
// a thread holds T of planes k-1, k, k+1 (k+2 in flight) and u of planes
// k-2 and k-1 (the older of each in LDS), computes u of plane k from the T tile of plane k in LDS and
// then T_{n+2} of plane k-1 from the u tile of plane k-1: one barrier for
// two point evaluations.  Bound by HBM bytes and the rows re-read around the
// tiles; a 1024-thread work-group per CU (128 registers, 127 KB of LDS) keeps
// 64 KB of loads in flight.  Time per step in a time loop, against single
// steps: 512^3 FP64 319 us against 527, FP32 172 against 285; 256^3 FP64 44
// against 73, FP32 23 against 47; 301 x 257 x 203 FP32 25 against 48.
template <typename S, int VEC, int RY, int CROSS, int MID>
__global__ void __launch_bounds__(1024)
k_step2_zmarch(S *__restrict__ out, S *__restrict__ mid, const S *__restrict__ T, const S *__restrict__ Ci, PairTile z,
               PairCoef<S> cf)
{
    typedef S V __attribute__((ext_vector_type(VEC)));
    constexpr uint32_t E = sizeof(S);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const PairGeom &g = z.g;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int64_t sxy = (int64_t)nx * ny;
    const int W = z.W, H = z.HG * RY;
    // one vector before and after the tiles: the x neighbours beyond a
    // tile's first and last vector are read and not used
    V *lds = reinterpret_cast<V *>(lds_raw) + 1;
    const int plane = W * H;  // vectors of one tile

    uint32_t b = blockIdx.x;
    if (!z.deal) {
        b = (uint32_t)xcd_remap(b, gridDim.x);
    } else {
        const uint32_t ntx = (uint32_t)z.ntx, P8 = gridDim.x / ntx / 8 * 8;
        if (b < ntx * P8) {
            const uint32_t x = b % 8, slot = b / 8;
            b = slot % ntx + ntx * (x + 8 * (slot / ntx));
        }
    }
    const int bx = (int)(b % z.ntx), by = (int)(b / z.ntx % z.nty), bz = (int)(b / z.ntx / z.nty);
    const int t = threadIdx.x, th = t - z.HG * (W - 2);  // th >= 0: a vector beside the tile
    const bool live = th < 2 * z.HG;
    const int tg = min(th < 0 ? t / (W - 2) : th >> 1, z.HG - 1);
    const int tv = th < 0 ? 1 + t % (W - 2) : (th & 1 ? W - 1 : 0);
    const int i = (bx * (W - 2) + tv - 1) * VEC;
    const int jb = 1 + by * (H - 4);
    const int kb = 1 + bz * z.zc;
    const int ke = kb + z.zc < nz - 1 ? kb + z.zc : nz - 1;

    // where a vector is read: at its own place, a period away when it lies
    // wholly outside the row, point by point when it crosses the row's end.
    // Element hq, where it is the row's halo point, is read from the point it
    // copies: of Ci always, of T where the row may be a fixed one.
    int iv = i;
    if (i < 0) iv = g.per[0] ? i + nx - 2 : 0;
    if (i >= nx) iv = g.per[0] ? i - (nx - 2) : 0;
    const bool cross = i < nx && i + VEC > nx;
    int hq = -1, hx = 0;
    if (g.per[0] && i == 0) { hq = 0; hx = nx - 2; }
    if (g.per[0] && i < nx && i + VEC >= nx) { hq = nx - 1 - i; hx = 1; }
    const bool edges = g.per[0] && !(g.per[1] && g.per[2]);

    uint32_t off[RY];  // byte offsets of the rows in a plane
    int jr[RY];
    uint32_t fixed = 0;       // points of u that keep T's value
    uint32_t st = 0;          // rows whose results this thread stores
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int lr = tg * RY + r;
        const int j = jb - 2 + lr;
        jr[r] = j;
        off[r] = (uint32_t)(wrap(j, ny, g.per[1]) * nx) * E;
        if (live && lr >= 2 && lr < H - 2 && j <= ny - 2 && tv >= 1 && tv < W - 1) st |= 1u << r;
#pragma unroll
        for (int q = 0; q < VEC; ++q)
            if ((!g.per[0] && (i + q <= 0 || i + q >= nx - 1)) || (!g.per[1] && (j <= 0 || j >= ny - 1)))
                fixed |= 1u << (r * VEC + q);
    }
    const uint32_t vo = (uint32_t)iv * E;

    const int64_t pb = sxy * (int64_t)E;
    auto rs = [&](const S *A, int k) { return buf_rsrc(A + (int64_t)k * sxy, pb); };
    auto ldv = [&](__amdgpu_buffer_rsrc_t d, uint32_t row) -> V {
        V v;
        if (!CROSS || !cross) {
            v = buf_load<V, 0>(d, row + vo);
        } else {
#pragma unroll
            for (int q = 0; q < VEC; ++q) v[q] = buf_load<S, 0>(d, row + (uint32_t)wrap(i + q, nx, g.per[0]) * E);
        }
        return v;
    };
    auto ld1 = [&](__amdgpu_buffer_rsrc_t d, uint32_t row) -> S {
        S x = S(0);
        if (hq >= 0) x = buf_load<S, 0>(d, row + (uint32_t)hx * E);
        return x;
    };
    auto patch = [&](V v, S x) -> V {
#pragma unroll
        for (int q = 0; q < VEC; ++q)
            if (q == hq) v[q] = x;
        return v;
    };
    auto put = [&](S *A, int k, const V (&v)[RY]) {
#pragma unroll
        for (int r = 0; r < RY; ++r)
            if (st >> r & 1) pair_put<S, VEC>(g, A, i, jr[r], k, v[r], z.nt);
    };

    const int lbase = tg * RY * W + tv;
    const int up = tg > 0 ? lbase - W : lbase, dn = tg < z.HG - 1 ? lbase + RY * W : lbase + (RY - 1) * W;
    // (threads past the last row group read what the last ones do and store
    // nothing)
    auto dsc = [&](const S *A, int k) { return rs(A, wrap(k, nz, g.per[2])); };
    auto ldT = [&](int k, int r) -> V {
        const __amdgpu_buffer_rsrc_t d = dsc(T, k);
        const V v = ldv(d, off[r]);
        return edges ? patch(v, ld1(d, off[r])) : v;
    };
    V tc[RY], tp[RY], cc[RY], cp[RY], uc[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const V t = ldT(kb - 2, r);
        if (live) lds[2 * plane + lbase + r * W] = t;
        tc[r] = ldT(kb - 1, r);
        tp[r] = ldT(kb, r);
        const __amdgpu_buffer_rsrc_t d = dsc(Ci, kb - 1);
        cc[r] = patch(ldv(d, off[r]), ld1(d, off[r]));
        cp[r] = uc[r] = V{};
    }
    for (int k = kb - 1; k <= ke; ++k) {
        const int buf = (k - kb + 1) & 1;
        V *sT = lds + buf * 2 * plane, *sU = sT + plane;
        V tn[RY], cn[RY];
        S t1[RY], c1[RY];
        // (the last plane's loads are read again and not used)
        const __amdgpu_buffer_rsrc_t dT = dsc(T, k < ke ? k + 2 : k), dC = dsc(Ci, k < ke ? k + 1 : k);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            tn[r] = ldv(dT, off[r]);
            cn[r] = ldv(dC, off[r]);
            c1[r] = ld1(dC, off[r]);
            t1[r] = edges ? ld1(dT, off[r]) : S(0);
        }
        if (live) {
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                sT[lbase + r * W] = tc[r];
                sU[lbase + r * W] = uc[r];
            }
        }
        __syncthreads();
        // T of plane k-1 and u of plane k-2: this thread's own, in the other
        // tiles until the next plane is written there
        const V *oT = lds + (buf ^ 1) * 2 * plane + lbase, *oU = oT + plane;
        // one plane of either step from its LDS tile and the planes around it
        auto plane_of = [&](const V *s, const V *om, const V (&c)[RY], const V (&p)[RY], const V (&ci)[RY],
                            V (&o)[RY]) {
            const S *e = reinterpret_cast<const S *>(s);
            const V vu = s[up], vd = s[dn];
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                const int l0 = (lbase + r * W) * VEC;
                const S xl = e[l0 - 1], xr = e[l0 + VEC];
                const V m = om[r * W];
                const V ym = r == 0 ? vu : c[r > 0 ? r - 1 : 0], yp = r == RY - 1 ? vd : c[r < RY - 1 ? r + 1 : r];
#pragma unroll
                for (int q = 0; q < VEC; ++q)
                    o[r][q] = diffuse<S>(c[r][q], q == 0 ? xl : c[r][q > 0 ? q - 1 : 0],
                                         q == VEC - 1 ? xr : c[r][q < VEC - 1 ? q + 1 : q], ym[q], yp[q], m[q],
                                         p[r][q], ci[r][q], cf.a, cf.rx, cf.ry, cf.rz);
            }
        };
        V un[RY], o[RY];
        plane_of(sT, oT, tc, tp, cc, un);
        const uint32_t fx = !g.per[2] && (k <= 0 || k >= nz - 1) ? ~0u : fixed;
        if (fx) {
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int q = 0; q < VEC; ++q)
                    if (fx >> (r * VEC + q) & 1) un[r][q] = tc[r][q];
        }
        plane_of(sU, oU, uc, un, cp, o);
        // the loads are waited for here, before the stores: a wait after them
        // would wait for the stores too
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            __asm__ volatile("" : "+v"(tn[r]));
            __asm__ volatile("" : "+v"(cn[r]));
            __asm__ volatile("" : "+v"(c1[r]));
            if (edges) __asm__ volatile("" : "+v"(t1[r]));
        }
        if (MID && k >= kb && k < ke) put(mid, k, un);
        if (k > kb) put(out, k - 1, o);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            tc[r] = tp[r];
            tp[r] = edges ? patch(tn[r], t1[r]) : tn[r];
            cp[r] = cc[r];
            cc[r] = patch(cn[r], c1[r]);
            uc[r] = un[r];
        }
    }
}

template <typename S, int BX, int BY, int BZ>
int run_block(const StepPairArgs &a, hipStream_t s)
{
    using C = compute_t<S>;
    const PairGeom g{{a.nx, a.ny, a.nz}, {a.per[0], a.per[1], a.per[2]}};
    const int nbx = (a.nx - 2 + BX - 1) / BX, nby = (a.ny - 2 + BY - 1) / BY, nbz = (a.nz - 2 + BZ - 1) / BZ;
    const PairCoef<C> cf{(C)a.a, (C)a.rx, (C)a.ry, (C)a.rz};
    const dim3 grd((unsigned)((int64_t)nbx * nby * nbz));
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grd, dim3(1024), 0, s, (S *)a.T2, (S *)a.mid, (const S *)a.T, (const S *)a.Ci, g, nbx,
                           nby, cf, a.key1, a.key2, a.so);
    };
    if constexpr (sizeof(S) == 2) {
        if (a.stochastic) {
            if (a.mid) go(k_step2_block<S, BX, BY, BZ, 1, 1>);
            else go(k_step2_block<S, BX, BY, BZ, 1, 0>);
            IGG_HIP(hipGetLastError());
            return IGG_OK;
        }
    }
    if (a.mid) go(k_step2_block<S, BX, BY, BZ, 0, 1>);
    else go(k_step2_block<S, BX, BY, BZ, 0, 0>);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

template <typename S, int VEC, int RY>
int run_zmarch2(const StepPairArgs &a, hipStream_t s)
{
    PairTile z{};
    z.g = PairGeom{{a.nx, a.ny, a.nz}, {a.per[0], a.per[1], a.per[2]}};
    pair_tiles<VEC, RY>(a.nx, a.ny, a.nz, z);
    const int64_t blocks = (int64_t)z.ntx * z.nty * ((a.nz - 2 + z.zc - 1) / z.zc);
    // Stores that stay in the caches where T, T2 and Ci fit the 256 MB
    // last-level cache together (256^3 FP32 47 us a launch against 52, 320 x
    // 200 x 150 FP64 52 against 54; 320 x 300 x 170 FP64, 392 MB, 90 against
    // 86), and for launches of several rounds tile rows dealt to the XCDs in
    // turn instead of in ranges (512^3 FP64 630 against 639, FP32 322 against
    // 338; 256^3 FP64, one round, 87 against 84).
    z.nt = (int64_t)a.nx * a.ny * a.nz * 3 * (int64_t)sizeof(S) > ((int64_t)240 << 20);
    z.deal = blocks > 512;
    const size_t lds = ((size_t)4 * z.W * z.HG * RY + 2) * VEC * sizeof(S);
    const int tpb = (z.W * z.HG + 63) / 64 * 64;
    const PairCoef<S> cf{(S)a.a, (S)a.rx, (S)a.ry, (S)a.rz};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(tpb), lds, s, (S *)a.T2, (S *)a.mid, (const S *)a.T,
                           (const S *)a.Ci, z, cf);
    };
    if (a.nx % VEC == 0) {
        if (a.mid) go(k_step2_zmarch<S, VEC, RY, 0, 1>);
        else go(k_step2_zmarch<S, VEC, RY, 0, 0>);
    } else {
        if (a.mid) go(k_step2_zmarch<S, VEC, RY, 1, 1>);
        else go(k_step2_zmarch<S, VEC, RY, 1, 0>);
    }
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

}  // namespace

// Whether a pair is launched for this grid, and by which kernel.  Regions of
// zmarch_min_points() points (2^21) and more march (128^3 FP64, 2.0e6 points:
// 22.6 us a launch either way; 96 x 80 x 64: 9 us by blocks, 23 marching).
// FP16 marches in single steps: its step is bound by issue, which pairs do
// not lessen.
static bool pair_marches(int dtype, const int n[3])
{
    const int64_t pts = (int64_t)(n[0] - 2) * (n[1] - 2) * (n[2] - 2);
    return dtype != IGG_F16 && pts >= zmarch_min_points();
}

bool step_pair_pays(int dtype, const int n[3])
{
    const int64_t pts = (int64_t)(n[0] - 2) * (n[1] - 2) * (n[2] - 2);
    if (pts < zmarch_min_points()) return (int64_t)n[0] * n[1] * n[2] * elem_bytes(dtype) < ((int64_t)1 << 31);
    // the z-march kernel reads a whole vector a period away at either end of
    // a row, and addresses a plane with 32-bit offsets
    return dtype != IGG_F16 && n[0] >= 16 && (int64_t)n[0] * n[1] * elem_bytes(dtype) < ((int64_t)1 << 31);
}

// Blocks of 16 x 8 x 8 points below 2^20 points, for more work-groups (32^3
// FP64 1.7 us a step against 2.9 with 32 x 8 x 8; 300 x 70 x 50 6.1 against
// 7.2), 32 x 8 x 8 above, which recompute less of u (128^3 9.8 against 10.4,
// FP32 6.9 against 8.3).
template <typename S>
static int pair_blocks(const StepPairArgs &a, hipStream_t s)
{
    const int64_t pts = (int64_t)(a.nx - 2) * (a.ny - 2) * (a.nz - 2);
    return pts < ((int64_t)1 << 20) ? run_block<S, 16, 8, 8>(a, s) : run_block<S, 32, 8, 8>(a, s);
}

int launch_step_pair(int dtype, const StepPairArgs &a, hipStream_t s)
{
    const int n[3] = {a.nx, a.ny, a.nz};
    if (!pair_marches(dtype, n)) {
        if (dtype == IGG_F64) return pair_blocks<double>(a, s);
        if (dtype == IGG_F32) return pair_blocks<float>(a, s);
        return pair_blocks<_Float16>(a, s);
    }
    if (dtype == IGG_F64) return run_zmarch2<double, 2, 2>(a, s);
    return run_zmarch2<float, 4, 2>(a, s);
}

}  // namespace igg
