// flux.hip -- staggered-grid flux form of the diffusion step (Sec. 2 on the
// regular staggered grid): face fluxes q = -lam*grad(T) and the cell update
// T2 = T - dt*Ci*div(q), in one pass per cell.  Its adjoint runs in
// adjoint.hip (the same kernels as the Laplacian form's adjoint).
//
// Sizes: cells (nx,ny,nz); qx (nx+1,ny,nz), qy (nx,ny+1,nz), qz (nx,ny,nz+1).
// Face f of a dimension lies between cells f-1 and f; fluxes are computed on
// faces 1..n-1 of the inner rows of the other two dimensions.
#include <stdlib.h>

#include "host.hpp"

namespace igg {

// Cell grid size (the face fields add one point in their own dimension).
struct FaceGeom {
    int nx, ny, nz;
};

static unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

// ------------------------------------------------------------ fused step
// One pass per cell (i, j, k): its lower faces qx[i], qy[j], qz[k] (and the
// upper face where the cell is the last of its row, column or plane), the
// update T2 = T - dt*Ci*div(q) from the cell's six faces, and the x
// exchange of all four fields with the x neighbours (FluxXH).  The faces
// come from one expression (face_flux) and the divergence sums in a fixed
// order (flux_div), so every value equals a face pass followed by a cell
// pass.

// Stores of one cell that are not plain per-cell stores: the upper faces at
// the ends and the x-exchange copies.  p: the cell's offset in a cell-sized
// array, px and py: its lower faces' offsets in qx and qy.
template <typename C>
__device__ __forceinline__ void flux_extra_stores(C *T2, C *qx, C *qy, C *qz, int i, int j, int k,
                                                  int64_t p, int64_t px, int64_t py, const FaceGeom &g,
                                                  const FluxXH &xh, C v2, C qxl, C qxu, C qyl, C qyu,
                                                  C qzl, C qzu)
{
    const int nx = g.nx;
    const int64_t sz = (int64_t)nx * g.ny;
    const bool lastx = i == nx - 2, lasty = j == g.ny - 2, lastz = k == g.nz - 2;
    if (lastx) qx[px + 1] = qxu;
    if (lasty) qy[py + nx] = qyu;
    if (lastz) qz[p + sz] = qzu;
    // T2, qy, qz: column ol-1 -> lower neighbour's nx-1, column nx-ol ->
    // upper neighbour's 0
    for (int side = 0; side < 2; ++side) {
        if (!(side == 0 ? xh.on_lo : xh.on_hi)) continue;
        const int src = side == 0 ? xh.ol - 1 : nx - xh.ol;
        if (i != src) continue;
        const int64_t sh = side == 0 ? (int64_t)(nx - 1 - i) : -(int64_t)i;
        const int64_t *d = side == 0 ? xh.d_lo : xh.d_hi;
        T2[p + sh + d[0]] = v2;
        qy[py + sh + d[2]] = qyl;
        qz[p + sh + d[3]] = qzl;
        if (lasty) qy[py + nx + sh + d[2]] = qyu;
        if (lastz) qz[p + sz + sh + d[3]] = qzu;
    }
    // qx: face ol -> lower neighbour's nx, face nx-ol -> upper neighbour's 0
    // (faces i, and i+1 at the last cell)
    for (int f = i; f <= (lastx ? i + 1 : i); ++f) {
        const C v = f == i ? qxl : qxu;
        const int64_t pf = px + (f - i);
        if (xh.on_lo && f == xh.ol) qx[pf + (nx - f) + xh.d_lo[1]] = v;
        if (xh.on_hi && f == nx - xh.ol) qx[pf - f + xh.d_hi[1]] = v;
    }
}

template <typename C>
__global__ void __launch_bounds__(256)
k_flux_fused_boxes(C *__restrict__ T2, C *__restrict__ qx, C *__restrict__ qy, C *__restrict__ qz,
                   const C *__restrict__ T, const C *__restrict__ Ci, BoxSet bs, FaceGeom g, FluxXH xh, C lam,
                   C dt, C rdx, C rdy, C rdz)
{
    int i, j, k;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (!boxset_point(bs, t, i, j, k)) return;
    const int nx = g.nx, ny = g.ny;
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    const int64_t p = i + sy * j + sz * k;
    const C t0 = T[p];
    const C qxl = face_flux<C>(t0, T[p - 1], lam, rdx), qxu = face_flux<C>(T[p + 1], t0, lam, rdx);
    const C qyl = face_flux<C>(t0, T[p - sy], lam, rdy), qyu = face_flux<C>(T[p + sy], t0, lam, rdy);
    const C qzl = face_flux<C>(t0, T[p - sz], lam, rdz), qzu = face_flux<C>(T[p + sz], t0, lam, rdz);
    const C v2 = fma_(-dt * Ci[p], flux_div<C>(qxl, qxu, qyl, qyu, qzl, qzu, rdx, rdy, rdz), t0);
    const int64_t px = i + (int64_t)(nx + 1) * (j + (int64_t)ny * k);
    const int64_t py = i + (int64_t)nx * (j + (int64_t)(ny + 1) * k);
    T2[p] = v2;
    qx[px] = qxl;
    qy[py] = qyl;
    qz[p] = qzl;
    flux_extra_stores<C>(T2, qx, qy, qz, i, j, k, p, px, py, g, xh, v2, qxl, qxu, qyl, qyu, qzl, qzu);
}

// One thread per column of NZ inner cells, 256 consecutive cells of a plane per
// work-group (grids that sit in the caches, as k_step_small).
template <typename C, int NZ>
__global__ void __launch_bounds__(256)
k_flux_small(C *__restrict__ T2, C *__restrict__ qx, C *__restrict__ qy, C *__restrict__ qz, const C *__restrict__ T,
             const C *__restrict__ Ci, FaceGeom g, FluxXH xh, int nbp, C lam, C dt, C rdx, C rdy, C rdz)
{
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const uint32_t b = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t bp = b % (uint32_t)nbp, bz = b / (uint32_t)nbp;
    const uint32_t q = bp * 256 + threadIdx.x, w = (uint32_t)(nx - 2);
    const int j = 1 + (int)(q / w), i = 1 + (int)(q % w), k0 = 1 + (int)bz * NZ;
    if (j > ny - 2) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny, p0 = i + sy * j + sz * k0;
    C t[NZ + 2], nb[NZ][4], ci[NZ];
    // (planes past the last inner one read the last ones again)
#pragma unroll
    for (int z = 0; z < NZ + 2; ++z) t[z] = T[p0 + sz * (min(k0 - 1 + z, nz - 1) - k0)];
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        const int64_t p = p0 + sz * (min(k0 + z, nz - 2) - k0);
        nb[z][0] = T[p - 1];
        nb[z][1] = T[p + 1];
        nb[z][2] = T[p - sy];
        nb[z][3] = T[p + sy];
        ci[z] = Ci[p];
    }
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        const int k = k0 + z;
        if (k > nz - 2) break;
        const C t0 = t[z + 1];
        const C qxl = face_flux<C>(t0, nb[z][0], lam, rdx), qxu = face_flux<C>(nb[z][1], t0, lam, rdx);
        const C qyl = face_flux<C>(t0, nb[z][2], lam, rdy), qyu = face_flux<C>(nb[z][3], t0, lam, rdy);
        const C qzl = face_flux<C>(t0, t[z], lam, rdz), qzu = face_flux<C>(t[z + 2], t0, lam, rdz);
        const C v2 = fma_(-dt * ci[z], flux_div<C>(qxl, qxu, qyl, qyu, qzl, qzu, rdx, rdy, rdz), t0);
        const int64_t p = i + sy * j + sz * k;
        const int64_t px = i + (int64_t)(nx + 1) * (j + (int64_t)ny * k);
        const int64_t py = i + (int64_t)nx * (j + (int64_t)(ny + 1) * k);
        T2[p] = v2;
        qx[px] = qxl;
        qy[py] = qyl;
        qz[p] = qzl;
        if (i == nx - 2 || j == ny - 2 || k == nz - 2 ||
            ((xh.on_lo || xh.on_hi) && (i <= xh.ol || i >= nx - xh.ol)))
            flux_extra_stores<C>(T2, qx, qy, qz, i, j, k, p, px, py, g, xh, v2, qxl, qxu, qyl, qyu, qzl, qzu);
    }
}

template <typename C, int VEC> struct FVec {
    typedef C type __attribute__((ext_vector_type(VEC)));
    typedef C mem __attribute__((ext_vector_type(VEC), aligned(sizeof(C))));  // rows start at any element
};

struct FluxTile {
    Box b;
    int xa, ntx, nty, zc, remap;
    FaceGeom g;
    FluxXH xh;
};

// z-march of the fused step: BX x TY threads, a row of VEC cells each; T of
// planes k-1, k, k+1 (k+2 in flight) in registers, plane k in a
// double-buffered LDS tile for the x and y neighbours (the forward step
// kernel's scheme).  The four outputs leave as vectors where the cells of a
// vector all lie in the box.  (Its one row per thread stands in loops of one
// turn: without them the compiler copies the plane's body for a chunk's last
// plane, 768^3 FP32 2113 us against 2087.)
template <typename C, int VEC, int BX, int TY>
__global__ void __launch_bounds__(BX *TY)
k_flux_fused_zmarch(C *__restrict__ T2, C *__restrict__ qx, C *__restrict__ qy, C *__restrict__ qz,
                    const C *__restrict__ T, const C *__restrict__ Ci, FluxTile z, C lam, C dt, C rdx, C rdy,
                    C rdz)
{
    using V = typename FVec<C, VEC>::type;
    using M = typename FVec<C, VEC>::mem;
    constexpr int RY = 1, TW = BX * VEC, TH = TY * RY, LH = TH + 2, LW = TW + 2;
    __shared__ C tile[2][LH][LW];
    const int tx = threadIdx.x % BX, ty = threadIdx.x / BX;
    int64_t gidx = blockIdx.x;
    if (z.remap == 2) {  // x-rows of tiles dealt to the XCDs in turn
        const int64_t ntx0 = z.ntx, P = gridDim.x / ntx0, P8 = P / 8 * 8;
        if (gidx < ntx0 * P8) {
            const int64_t x = gidx % 8, slot = gidx / 8;
            gidx = slot % ntx0 + ntx0 * (x + 8 * (slot / ntx0));
        }
    }
    const int bx = (int)(gidx % z.ntx);
    const int64_t rest = gidx / z.ntx;
    const int by = (int)(rest % z.nty);
    const int bz = (int)(rest / z.nty);
    const int nx = z.g.nx, ny = z.g.ny;
    const int64_t sxy = (int64_t)nx * ny;
    const int x0 = z.xa + bx * TW;
    const int i = x0 + tx * VEC;
    const bool xin = i < nx;
    const int jb = z.b.j0 + by * TH;
    const int kb = z.b.k0 + bz * z.zc;
    const int ke = (kb + z.zc < z.b.k1) ? kb + z.zc : z.b.k1;
    int64_t col[RY];
    int jr[RY];
    bool crow[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        jr[r] = jb + ty * RY + r;
        col[r] = (int64_t)(jr[r] > ny - 1 ? ny - 1 : jr[r]) * nx + i;
        crow[r] = jr[r] < z.b.j1;
    }
    const bool hy = ty == 0 || ty == TY - 1;
    const int jh = (ty == 0) ? jb - 1 : (jb + TH > ny - 1 ? ny - 1 : jb + TH);
    const int64_t colhy = (int64_t)jh * nx + i;
    const int hyrow = (ty == 0) ? 0 : LH - 1;
    const bool own_h = (tx == 0 && x0 >= 1) || (tx == BX - 1 && x0 + TW < nx);
    const int xh = (tx == 0) ? x0 - 1 : x0 + TW;
    const int hcol = (tx == 0) ? 0 : LW - 1;

    auto ld = [&](const C *A, int k, int64_t c) -> V {
        V v{};
        if (xin) v = *reinterpret_cast<const M *>(A + (int64_t)k * sxy + c);
        return v;
    };
    // A vector that runs over its row's end reads the start of the next row,
    // which is not used.  The plane above the box's last one is read for the
    // rows computed only; other rows read the row before theirs there, which
    // keeps such vectors inside the array in the last plane too.
    auto above = [&](int k, int r) { return col[r] - (k >= z.b.k1 && !crow[r] ? nx : 0); };
    auto ld_nt = [&](const C *A, int k, int64_t c) -> V {
        V v{};
        if (xin) v = __builtin_nontemporal_load(reinterpret_cast<const M *>(A + (int64_t)k * sxy + c));
        return v;
    };

    V tm[RY], tc[RY], tp[RY], ci[RY];
    C hx[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        tm[r] = ld(T, kb - 1, col[r]);
        tc[r] = ld(T, kb, col[r]);
        tp[r] = ld(T, kb + 1, above(kb + 1, r));
        ci[r] = crow[r] ? ld_nt(Ci, kb, col[r]) : V{};
        hx[r] = own_h ? T[(int64_t)kb * sxy + col[r] - i + xh] : C(0);
    }
    V yh = hy ? ld(T, kb, colhy) : V{};

    for (int k = kb; k < ke; ++k) {
        const int buf = (k - kb) & 1;
        const bool more = k + 1 < ke;
        V tn[RY], cn[RY], yn{};
        C hn[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            tn[r] = more ? ld(T, k + 2, above(k + 2, r)) : V{};
            cn[r] = (more && crow[r]) ? ld_nt(Ci, k + 1, col[r]) : V{};
            hn[r] = (more && own_h) ? T[(int64_t)(k + 1) * sxy + col[r] - i + xh] : C(0);
        }
        if (more && hy) yn = ld(T, k + 1, colhy);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) tile[buf][1 + ty * RY + r][1 + tx * VEC + q] = tc[r][q];
            if (own_h) tile[buf][1 + ty * RY + r][hcol] = hx[r];
        }
        if (hy) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) tile[buf][hyrow][1 + tx * VEC + q] = yh[q];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            if (!crow[r] || !xin) continue;
            const int lr = 1 + ty * RY + r;
            V o2, oy, oz;
            C oxl[VEC], oxu[VEC], oyu[VEC], ozu[VEC];
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const int lc = 1 + tx * VEC + q;
                const C t0 = tc[r][q];
                const C txm = (q == 0) ? tile[buf][lr][lc - 1] : tc[r][q - 1];
                const C txp = (q == VEC - 1) ? tile[buf][lr][lc + 1] : tc[r][q + 1];
                const C tym = tile[buf][lr - 1][lc];
                const C typ = tile[buf][lr + 1][lc];
                const C qxl = face_flux<C>(t0, txm, lam, rdx), qxu = face_flux<C>(txp, t0, lam, rdx);
                const C qyl = face_flux<C>(t0, tym, lam, rdy), qyu = face_flux<C>(typ, t0, lam, rdy);
                const C qzl = face_flux<C>(t0, tm[r][q], lam, rdz);
                const C qzu = face_flux<C>(tp[r][q], t0, lam, rdz);
                o2[q] = fma_(-dt * ci[r][q], flux_div<C>(qxl, qxu, qyl, qyu, qzl, qzu, rdx, rdy, rdz), t0);
                oy[q] = qyl;
                oz[q] = qzl;
                oxl[q] = qxl;
                oxu[q] = qxu;
                oyu[q] = qyu;
                ozu[q] = qzu;
            }
            // the loads are waited for here: a wait after the stores would
            // wait for the stores too
            __asm__ volatile("" : "+v"(tn[0]), "+v"(cn[0]), "+v"(hn[0]), "+v"(yn));
            const int j = jr[r];
            const int64_t p = (int64_t)k * sxy + col[r];
            const int64_t px = i + (int64_t)(nx + 1) * (j + (int64_t)ny * k);
            const int64_t py = i + (int64_t)nx * (j + (int64_t)(ny + 1) * k);
            const bool full = i >= z.b.i0 && i + VEC <= z.b.i1;
            if (full) {
                __builtin_nontemporal_store(o2, reinterpret_cast<M *>(T2 + p));
                __builtin_nontemporal_store(oy, reinterpret_cast<M *>(qy + py));
                __builtin_nontemporal_store(oz, reinterpret_cast<M *>(qz + p));
                V ox;
#pragma unroll
                for (int q = 0; q < VEC; ++q) ox[q] = oxl[q];
                *reinterpret_cast<M *>(qx + px) = ox;
            }
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const int ii = i + q;
                if (ii < z.b.i0 || ii >= z.b.i1) continue;
                if (!full) {
                    T2[p + q] = o2[q];
                    qy[py + q] = oy[q];
                    qz[p + q] = oz[q];
                    qx[px + q] = oxl[q];
                }
                if (ii == nx - 2 || j == ny - 2 || k == z.g.nz - 2 ||
                    ((z.xh.on_lo || z.xh.on_hi) && (ii <= z.xh.ol || ii >= nx - z.xh.ol)))
                    flux_extra_stores<C>(T2, qx, qy, qz, ii, j, k, p + q, px + q, py + q, z.g, z.xh, o2[q], oxl[q],
                                         oxu[q], oy[q], oyu[q], oz[q], ozu[q]);
            }
        }
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            tm[r] = tc[r];
            tc[r] = tp[r];
            tp[r] = tn[r];
            ci[r] = cn[r];
            hx[r] = hn[r];
        }
        yh = yn;
    }
}

static int env_int_flux(const char *name, int dflt)
{
    const char *s = getenv(name);
    return (s && *s) ? atoi(s) : dflt;
}

template <typename C>
static int run_fused_boxes(const FluxArgs &a, const Box *b, int nb, hipStream_t s)
{
    BoxSet bs = make_boxset(b, nb);
    const int64_t threads = bs.first[nb];
    if (threads == 0) return IGG_OK;
    FaceGeom g{a.nx, a.ny, a.nz};
    hipLaunchKernelGGL(k_flux_fused_boxes<C>, dim3(blocks_for(threads)), dim3(256), 0, s, (C *)a.T2, (C *)a.qx,
                       (C *)a.qy, (C *)a.qz, (const C *)a.T, (const C *)a.Ci, bs, g, a.xh, (C)a.lam, (C)a.dt,
                       (C)a.rdx, (C)a.rdy, (C)a.rdz);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

template <typename C, int VEC, int BX, int TY>
static int run_fused_zmarch(const FluxArgs &a, const Box &b, hipStream_t s)
{
    constexpr int TW = BX * VEC, TH = TY;
    FluxTile z{};
    z.b = b;
    z.g = FaceGeom{a.nx, a.ny, a.nz};
    z.xh = a.xh;
    RowTiles t = row_tiles(b, VEC, TW);
    // (four FP64 outputs off their alignment cost more than one of several
    // tiles: 258 x 300 x 170 on inputs out of the caches 147 us, 160 from i0)
    if (sizeof(C) == 8 && t.n > 1) t = row_tiles(Box{b.i0 / VEC * VEC, b.i1, 0, 0, 0, 0}, VEC, TW);
    z.xa = t.xa;
    z.ntx = t.n;
    z.nty = (b.j1 - b.j0 + TH - 1) / TH;
    const int depth = b.k1 - b.k0;
    int zc = env_int_flux("IGG_FLUX_ZCHUNK", 0);
    // chunks of 4 planes: at 768^3 (FP32) 9% faster than 16 and 4% faster
    // than 8 (the two extra planes a chunk reads mostly hit in L2)
    if (zc < 1) zc = zchunk_for_groups((int64_t)z.ntx * z.nty, depth, 4);
    z.zc = zc;
    z.remap = env_int_flux("IGG_FLUX_REMAP", 2);
    const int64_t blocks = (int64_t)z.ntx * z.nty * ((depth + zc - 1) / zc);
    if (blocks <= 0) return IGG_OK;
    hipLaunchKernelGGL((k_flux_fused_zmarch<C, VEC, BX, TY>), dim3((unsigned)blocks), dim3(BX * TY), 0, s,
                       (C *)a.T2, (C *)a.qx, (C *)a.qy, (C *)a.qz, (const C *)a.T, (const C *)a.Ci, z, (C)a.lam,
                       (C)a.dt, (C)a.rdx, (C)a.rdy, (C)a.rdz);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

template <typename C>
static int run_small(const FluxArgs &a, hipStream_t s)
{
    constexpr int NZ = 2;
    const FaceGeom g{a.nx, a.ny, a.nz};
    const int nbp = (int)(((int64_t)(a.nx - 2) * (a.ny - 2) + 255) / 256);
    const int64_t blocks = (int64_t)nbp * ((a.nz - 2 + NZ - 1) / NZ);
    hipLaunchKernelGGL((k_flux_small<C, NZ>), dim3((unsigned)blocks), dim3(256), 0, s, (C *)a.T2, (C *)a.qx,
                       (C *)a.qy, (C *)a.qz, (const C *)a.T, (const C *)a.Ci, g, a.xh, nbp, (C)a.lam, (C)a.dt,
                       (C)a.rdx, (C)a.rdy, (C)a.rdz);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

int launch_flux_small(int dtype, const FluxArgs &a, hipStream_t s)
{
    return dtype == IGG_F64 ? run_small<double>(a, s) : run_small<float>(a, s);
}

int launch_flux_boxes(int dtype, const FluxArgs &a, const Box *b, int nb, hipStream_t s)
{
    return dtype == IGG_F64 ? run_fused_boxes<double>(a, b, nb, s) : run_fused_boxes<float>(a, b, nb, s);
}

// The inner region: z-march tiles of 1 KB rows (128 FP64 or 256 FP32 cells),
// one row per thread: two rows per thread (FP32 180 registers against 133)
// were 3-12% slower (768^3 FP32 2147 us against 2093, 452 x 360 x 440 FP64 772
// against 724; FP64 in 8 rows, 4 rows 740).  FP32 takes 128-cell rows where
// they leave a fifth fewer lanes past the rows' ends (384^3 334 -> 289 us,
// 301 x 257 x 203 122 -> 97).  Tiles of 64 cells take rows of at most 64 (50 x
// 700 x 400 FP64 257 -> 167, FP32 163 -> 118) and of 129 to 160, where they leave a
// fourth of the lanes less (131 x 400 x 260 FP64 197 -> 149, FP32 114 -> 100; 194 x
// 330 x 220 on inputs out of the caches FP64 167, 190 in tiles of 64).  Rows of
// any length are read and written in vectors (255 x 190 x 131 FP32 52 -> 44 with
// the rows per thread).  Regions below zmarch_min_points() and the shortest rows,
// which leave most of a tile's lanes idle, take the box kernel (two ranks of 13
// x 1500 x 600 FP64 792 us against 1020, FP32 374 against 532; 34 x 800 x 500 591
// against 690, FP32 410 against 351).
int launch_flux_inner(int dtype, const FluxArgs &a, const Box &b, hipStream_t s)
{
    const int row = b.i1 - b.i0;
    if (box_count(b) < zmarch_min_points() || a.nx < 4 || (rows_dispatched() && row <= (dtype == IGG_F64 ? 40 : 20)))
        return launch_flux_boxes(dtype, a, &b, 1, s);
    const bool quarter = row <= 64 || (row > 128 && row <= 160);
    if (dtype == IGG_F64)
        return quarter ? run_fused_zmarch<double, 2, 32, 8>(a, b, s) : run_fused_zmarch<double, 2, 64, 8>(a, b, s);
    if (quarter) return run_fused_zmarch<float, 2, 32, 8>(a, b, s);
    return narrow_pays(row_tiles(b, 4, 256), row_tiles(b, 2, 128)) ? run_fused_zmarch<float, 2, 64, 4>(a, b, s)
                                                                   : run_fused_zmarch<float, 4, 64, 4>(a, b, s);
}

}  // namespace igg
