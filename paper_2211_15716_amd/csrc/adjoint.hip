// adjoint.hip -- transposed diffusion step, for the Laplacian form and the
// staggered flux form.
//
// The forward step is T_{n+1} = T_n + a*Ci.*(L T_n) on the inner points
// (a = dt*lam, L = sum_d d2_d/dd^2, symmetric on the periodic grid).  Given
// lp = dLoss/dT_{n+1} with a valid halo, one adjoint step computes
//   lam_n = lp + a*L(mu),  mu = Ci.*lp        (mu formed on the fly at the
//                                               six neighbours)
//   gCi  += a*lp.*(L T_n)
// on the inner points.  k_adj_boxes is the one-thread-per-point form used
// for the boundary slabs; k_adj_zmarch marches z with the forward kernel's
// tiling, keeping lp, mu and T_n of planes k-1, k, k+1 in registers and
// staging mu and T_n of plane k in LDS for the x and y neighbours.
#include <stdlib.h>

#include "host.hpp"

namespace igg {

// One cell of the adjoint from mu = Ci.*lp and T_n at the cell and its six
// neighbours.  FORM 0, the Laplacian step (a = dt*lam, r = 1/dd^2):
//   lam_n = lp + a*L(mu),  gCi += a*lp*L(T_n).
// FORM 1, the staggered flux form (a = dt, r = 1/dd, lamf = lam), with the
// face fluxes p = -lam*grad(mu) and q = -lam*grad(T_n) formed on the fly:
//   lam_n = lp - dt*div(p),  gCi += -dt*lp*div(q).
template <typename C, int FORM>
__device__ __forceinline__ void adj_cell(C l, C m0, C mxm, C mxp, C mym, C myp, C mzm, C mzp, C t0, C txm,
                                         C txp, C tym, C typ, C tzm, C tzp, C a, C rx, C ry, C rz, C lamf,
                                         C &ln, C &g)
{
    if constexpr (FORM == 0) {
        const C lapmu = laplace<C>(m0, mxm, mxp, mym, myp, mzm, mzp, rx, ry, rz);
        const C lapT = laplace<C>(t0, txm, txp, tym, typ, tzm, tzp, rx, ry, rz);
        ln = adjoint_lam<C>(l, lapmu, a);
        g = adjoint_grad<C>(l, lapT, a, g);
    } else {
        const C divp = flux_div<C>(face_flux<C>(m0, mxm, lamf, rx), face_flux<C>(mxp, m0, lamf, rx),
                                   face_flux<C>(m0, mym, lamf, ry), face_flux<C>(myp, m0, lamf, ry),
                                   face_flux<C>(m0, mzm, lamf, rz), face_flux<C>(mzp, m0, lamf, rz), rx, ry, rz);
        const C divq = flux_div<C>(face_flux<C>(t0, txm, lamf, rx), face_flux<C>(txp, t0, lamf, rx),
                                   face_flux<C>(t0, tym, lamf, ry), face_flux<C>(typ, t0, lamf, ry),
                                   face_flux<C>(t0, tzm, lamf, rz), face_flux<C>(tzp, t0, lamf, rz), rx, ry, rz);
        ln = fma_(-a, divp, l);
        g = fma_(-a * l, divq, g);
    }
}

// The y/z halo rows of row j at plane k under YZImg: every (jj, kk) other
// than (j, k) with jj in {j, ny-1 if j = jl, 0 if j = jh} and kk in {k,
// nz-1 if k = kl, 0 if k = kh} (with n = ol+1 one row is the image of both
// halo rows).  f(jj, kk) is called for each.
template <typename F>
__device__ __forceinline__ void yz_images(const YZImg &yz, int j, int k, F &&f)
{
    if (j != yz.jl && j != yz.jh && k != yz.kl && k != yz.kh) return;
    const int js[3] = {j, j == yz.jl ? yz.ny - 1 : -1, j == yz.jh ? 0 : -1};
    const int ks[3] = {k, k == yz.kl ? yz.nz - 1 : -1, k == yz.kh ? 0 : -1};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
            if ((a | b) && js[a] >= 0 && ks[b] >= 0) f(js[a], ks[b]);
}

template <typename C, int FORM>
__global__ void __launch_bounds__(256)
k_adj_boxes(C *__restrict__ lam_n, const C *__restrict__ lp, const C *__restrict__ Tn,
            const C *__restrict__ Ci, C *__restrict__ gCi, BoxSet bs, int nx, int ny, C a, C rx, C ry,
            C rz, C lamf, XHalo xh, YZImg yz)
{
    int i, j, k;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (!boxset_point(bs, t, i, j, k)) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    const int64_t p = i + sy * j + sz * k;
    auto mu = [&](int64_t q) { return Ci[q] * lp[q]; };
    C ln, g = gCi[p];
    adj_cell<C, FORM>(lp[p], mu(p), mu(p - 1), mu(p + 1), mu(p - sy), mu(p + sy), mu(p - sz), mu(p + sz), Tn[p],
                      Tn[p - 1], Tn[p + 1], Tn[p - sy], Tn[p + sy], Tn[p - sz], Tn[p + sz], a, rx, ry, rz, lamf,
                      ln, g);
    lam_n[p] = ln;
    gCi[p] = g;
    // x exchange of lam_n fused into the store
    if (xh.on_lo && i == xh.lo) lam_n[p - i + nx - 1 + xh.d_lo] = ln;
    if (xh.on_hi && i == xh.hi) lam_n[p - i + xh.d_hi] = ln;
    // y/z halo planes whose image is this point, each with its x exchange
    if (yz.on)
        yz_images(yz, j, k, [&](int jj, int kk) {
            const int64_t q0 = sz * kk + sy * jj;
            lam_n[q0 + i] = ln;
            if (xh.on_lo && i == xh.lo) lam_n[q0 + nx - 1 + xh.d_lo] = ln;
            if (xh.on_hi && i == xh.hi) lam_n[q0 + xh.d_hi] = ln;
        });
}

// One thread per column of NZ inner points, 256 consecutive points of a plane
// per work-group (grids that sit in the caches, as k_step_small).  Bound by
// the loads' latency and the launch; two points a thread (128^3 FP64 23.4 us,
// one 26.4, four 24.7) against the box kernel's or the z-march's 33.9; 160^3
// FP32 29.0 -> 19.9, 352 x 53 x 59 FP64 24.7 -> 16.2.
struct AdjSmall {
    int nx, ny, nz;
    int nbp;  // work-groups per plane
    XHalo xh;
    YZImg yz;
    int main;  // work-groups of the points; the rest copy lam_n's edges
    EdgeLines ed;
};
template <typename C, int FORM, int NZ>
__global__ void __launch_bounds__(256)
k_adj_small(C *__restrict__ lam_n, const C *__restrict__ lp, const C *__restrict__ Tn, const C *__restrict__ Ci,
            C *__restrict__ gCi, AdjSmall g, C a, C rx, C ry, C rz, C lamf)
{
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    if ((int)blockIdx.x >= g.main) {
        const int e = ((int)blockIdx.x - g.main) * 256 + threadIdx.x;
        if (e < g.ed.total) edge_point(lam_n, g.ed, e);
        return;
    }
    const uint32_t b = (uint32_t)xcd_remap(blockIdx.x, g.main);
    const uint32_t bp = b % (uint32_t)g.nbp, bz = b / (uint32_t)g.nbp;
    const uint32_t q = bp * 256 + threadIdx.x, w = (uint32_t)(nx - 2);
    const int j = 1 + (int)(q / w), i = 1 + (int)(q % w), k0 = 1 + (int)bz * NZ;
    if (j > ny - 2) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny, p0 = i + sy * j + sz * k0;
    C l[NZ + 2], m[NZ + 2], t[NZ + 2], c[NZ + 2];
    // (planes past the last inner one read the last ones again)
#pragma unroll
    for (int z = 0; z < NZ + 2; ++z) {
        const int64_t p = p0 + sz * (min(k0 - 1 + z, nz - 1) - k0);
        l[z] = lp[p];
        c[z] = Ci[p];
        t[z] = Tn[p];
    }
#pragma unroll
    for (int z = 0; z < NZ + 2; ++z) m[z] = c[z] * l[z];
    C mn[NZ][4], tn[NZ][4], gc[NZ];
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        const int64_t p = p0 + sz * (min(k0 + z, nz - 2) - k0);
        const int64_t o[4] = {p - 1, p + 1, p - sy, p + sy};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mn[z][e] = Ci[o[e]] * lp[o[e]];
            tn[z][e] = Tn[o[e]];
        }
        gc[z] = gCi[p];
    }
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        const int k = k0 + z;
        if (k > nz - 2) break;
        C ln, gg = gc[z];
        adj_cell<C, FORM>(l[z + 1], m[z + 1], mn[z][0], mn[z][1], mn[z][2], mn[z][3], m[z], m[z + 2], t[z + 1],
                          tn[z][0], tn[z][1], tn[z][2], tn[z][3], t[z], t[z + 2], a, rx, ry, rz, lamf, ln, gg);
        const int64_t row = sz * k + sy * j;
        auto put = [&](int64_t r) {
            lam_n[r + i] = ln;
            if (g.xh.on_lo && i == g.xh.lo) lam_n[r + nx - 1 + g.xh.d_lo] = ln;
            if (g.xh.on_hi && i == g.xh.hi) lam_n[r + g.xh.d_hi] = ln;
        };
        put(row);
        gCi[row + i] = gg;
        if (g.yz.on) yz_images(g.yz, j, k, [&](int jj, int kk) { put(sz * kk + sy * jj); });
    }
}

struct AdjTile {
    Box b;
    int nx, ny, nz;
    int xa;
    int ntx, nty;
    int zc;
    int remap;
    int rblock;  // mode 2: x-rows of tiles per block dealt to one XCD
    XHalo xh;
    YZImg yz;
    int main;  // work-groups of the tiles; the rest copy lam_n's edges
    EdgeLines ed;
};

template <typename C, int VEC> struct AVec {
    typedef C type __attribute__((ext_vector_type(VEC)));
};
template <typename C, int VEC>
__device__ __forceinline__ C el(const typename AVec<C, VEC>::type &v, int q)
{
    return v[q];
}
// element q of a vector for a q known only at run time
template <typename C, int VEC>
__device__ __forceinline__ C el_dyn(const typename AVec<C, VEC>::type &v, int q)
{
    C x = el<C, VEC>(v, 0);
#pragma unroll
    for (int p = 1; p < VEC; ++p)
        if (q == p) x = el<C, VEC>(v, p);
    return x;
}
template <typename C, int VEC>
__device__ __forceinline__ void set_el(typename AVec<C, VEC>::type &v, int q, C x)
{
    v[q] = x;
}

// BX x TY threads, a row of VEC points per thread (the forward kernel's
// tiling; the row stands in loops of one turn and its elements are read and
// set through el and set_el: written out, the same arithmetic was scheduled
// 2-7% slower, 512^3 FP64 1135 -> 1205 us).  mu = Ci .* lp and T_n of plane k are staged in two
// double-buffered LDS tiles; lp, mu and T_n of planes k-1..k+1 (k+2 in
// flight) sit in registers.  gCi is read and written once per point and
// lam_n written once: non-temporal.  The products mu of the planes in
// flight are formed when the queue rotates, after the plane's arithmetic,
// so the loads are not waited for inside the plane (256^3: 3.5% faster).
template <typename C, int VEC, int BX, int TY, int FORM, int WAVES>
__global__ void __launch_bounds__(BX *TY) __attribute__((amdgpu_waves_per_eu(WAVES)))
k_adj_zmarch(C *__restrict__ lam_n, const C *__restrict__ lp, const C *__restrict__ Tn,
             const C *__restrict__ Ci, C *__restrict__ gCi, AdjTile z, C a, C rx, C ry, C rz, C lamf)
{
    using V = typename AVec<C, VEC>::type;
    static_assert(BX == 64, "a wave holds one thread row (the y/z image stores rely on it)");
    constexpr int RY = 1, TW = BX * VEC, TH = TY * RY, LH = TH + 2, LW = TW + 2;
    __shared__ C smu[2][LH][LW];
    __shared__ C sT[2][LH][LW];
    const int tx = threadIdx.x % BX, ty = threadIdx.x / BX;
    if ((int)blockIdx.x >= z.main) {
        const int e = ((int)blockIdx.x - z.main) * (BX * TY) + threadIdx.x;
        if (e < z.ed.total) edge_point(lam_n, z.ed, e);
        return;
    }
    int64_t g = blockIdx.x;
    if (z.remap == 2) {  // blocks of rblock x-rows of tiles dealt to the XCDs in turn
        const int64_t ntx0 = z.ntx, B = z.rblock, P = z.main / ntx0, P8 = P / (8 * B) * (8 * B);
        if (g < ntx0 * P8) {
            const int64_t x = g % 8, slot = g / 8, q = slot / ntx0;
            g = slot % ntx0 + ntx0 * (((q / B) * 8 + x) * B + q % B);
        }
    }
    const int bx = (int)(g % z.ntx);
    const int64_t rest = g / z.ntx;
    const int by = (int)(rest % z.nty);
    const int bz = (int)(rest / z.nty);
    const int nx = z.nx, ny = z.ny;
    const int64_t sxy = (int64_t)nx * ny;
    const int x0 = z.xa + bx * TW;
    const int i = x0 + tx * VEC;
    const bool xin = i < nx;
    const int jb = z.b.j0 + by * TH;
    const int kb = z.b.k0 + bz * z.zc;
    const int ke = (kb + z.zc < z.b.k1) ? kb + z.zc : z.b.k1;
    int64_t col[RY];
    bool crow[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int j = jb + ty * RY + r;
        col[r] = (int64_t)(j > ny - 1 ? ny - 1 : j) * nx + i;
        crow[r] = j < z.b.j1;
    }
    const bool hy = ty == 0 || ty == TY - 1;
    const int jh = (ty == 0) ? jb - 1 : (jb + TH > ny - 1 ? ny - 1 : jb + TH);
    const int64_t colhy = (int64_t)jh * nx + i;
    const int hyrow = (ty == 0) ? 0 : LH - 1;
    const bool own_h = (tx == 0 && x0 >= 1) || (tx == BX - 1 && x0 + TW < nx);
    const int xh = (tx == 0) ? x0 - 1 : x0 + TW;
    const int hcol = (tx == 0) ? 0 : LW - 1;

    // loads through a buffer descriptor per array and plane (scalar
    // registers) with 32-bit byte offsets in the plane (the launcher keeps
    // planes below 2 GiB): no 64-bit address registers per lane, which
    // leaves room under the 128-register cap for the deferred products below
    // (rows of any length: a vector that runs over its row's end reads the
    // start of the next row, which is not used; the descriptor lets it run
    // into the next plane, and past the array's end it reads zero)
    const int64_t pb = sxy * (int64_t)sizeof(C);
    auto rs = [&](const C *A, int k) { return buf_rsrc(A + (int64_t)k * sxy, pb + (k < z.nz - 1 ? 16 : 0)); };
    auto ld = [&](const C *A, int k, int64_t c) -> V {
        V v{};
        if (xin) v = buf_load<V, 0>(rs(A, k), (uint32_t)(c * (int64_t)sizeof(C)));
        return v;
    };
    auto ld_nt = [&](const C *A, int k, int64_t c) -> V {
        V v{};
        if (xin) v = buf_load<V, 2>(rs(A, k), (uint32_t)(c * (int64_t)sizeof(C)));
        return v;
    };
    auto lds1 = [&](const C *A, int k, int64_t c) -> C { return buf_load<C, 0>(rs(A, k), (uint32_t)(c * (int64_t)sizeof(C))); };
    auto mul = [](V x, V y) -> V {
        V out;
#pragma unroll
        for (int q = 0; q < VEC; ++q) set_el<C, VEC>(out, q, el<C, VEC>(x, q) * el<C, VEC>(y, q));
        return out;
    };

    V mm[RY], mc[RY], mp[RY], tm[RY], tc[RY], tp[RY], lc[RY], lq[RY], gc[RY];
    C hmu[RY], hT[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        mm[r] = mul(ld(Ci, kb - 1, col[r]), ld(lp, kb - 1, col[r]));
        lc[r] = ld(lp, kb, col[r]);
        mc[r] = mul(ld(Ci, kb, col[r]), lc[r]);
        lq[r] = ld(lp, kb + 1, col[r]);
        mp[r] = mul(ld(Ci, kb + 1, col[r]), lq[r]);
        tm[r] = ld(Tn, kb - 1, col[r]);
        tc[r] = ld(Tn, kb, col[r]);
        tp[r] = ld(Tn, kb + 1, col[r]);
        gc[r] = crow[r] ? ld_nt(gCi, kb, col[r]) : V{};
        const int64_t ph = col[r] - i + xh;
        hmu[r] = own_h ? lds1(Ci, kb, ph) * lds1(lp, kb, ph) : C(0);
        hT[r] = own_h ? lds1(Tn, kb, ph) : C(0);
    }
    V ymu = hy ? mul(ld(Ci, kb, colhy), ld(lp, kb, colhy)) : V{};
    V yT = hy ? ld(Tn, kb, colhy) : V{};

    for (int k = kb; k < ke; ++k) {
        const int buf = (k - kb) & 1;
        const bool more = k + 1 < ke;
        // loads for the next planes, consumed one iteration later (Ci and
        // lp raw: their products are formed at the rotation below)
        V cn[RY], tn[RY], ln2[RY], gn[RY], yc_n{}, yl_n{}, yT_n{};
        C hc_n[RY], hl_n[RY], hT_n[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            ln2[r] = more ? ld(lp, k + 2, col[r]) : V{};
            cn[r] = more ? ld(Ci, k + 2, col[r]) : V{};
            tn[r] = more ? ld(Tn, k + 2, col[r]) : V{};
            gn[r] = (more && crow[r]) ? ld_nt(gCi, k + 1, col[r]) : V{};
            const int64_t ph = col[r] - i + xh;
            hc_n[r] = (more && own_h) ? lds1(Ci, k + 1, ph) : C(0);
            hl_n[r] = (more && own_h) ? lds1(lp, k + 1, ph) : C(0);
            hT_n[r] = (more && own_h) ? lds1(Tn, k + 1, ph) : C(0);
        }
        if (more && hy) {
            yc_n = ld(Ci, k + 1, colhy);
            yl_n = ld(lp, k + 1, colhy);
            yT_n = ld(Tn, k + 1, colhy);
        }
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            const int lr = 1 + ty * RY + r;
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                smu[buf][lr][1 + tx * VEC + q] = el<C, VEC>(mc[r], q);
                sT[buf][lr][1 + tx * VEC + q] = el<C, VEC>(tc[r], q);
            }
            if (own_h) {
                smu[buf][lr][hcol] = hmu[r];
                sT[buf][lr][hcol] = hT[r];
            }
        }
        if (hy) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                smu[buf][hyrow][1 + tx * VEC + q] = el<C, VEC>(ymu, q);
                sT[buf][hyrow][1 + tx * VEC + q] = el<C, VEC>(yT, q);
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            if (!crow[r]) continue;
            const int lr = 1 + ty * RY + r;
            V lo, go;
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const int lc_ = 1 + tx * VEC + q;
                const C m0 = el<C, VEC>(mc[r], q), t0 = el<C, VEC>(tc[r], q);
                const C mxm = (q == 0) ? smu[buf][lr][lc_ - 1] : el<C, VEC>(mc[r], q - 1);
                const C mxp = (q == VEC - 1) ? smu[buf][lr][lc_ + 1] : el<C, VEC>(mc[r], q + 1);
                const C mym = smu[buf][lr - 1][lc_];
                const C myp = smu[buf][lr + 1][lc_];
                const C txm = (q == 0) ? sT[buf][lr][lc_ - 1] : el<C, VEC>(tc[r], q - 1);
                const C txp = (q == VEC - 1) ? sT[buf][lr][lc_ + 1] : el<C, VEC>(tc[r], q + 1);
                const C tym = sT[buf][lr - 1][lc_];
                const C typ = sT[buf][lr + 1][lc_];
                C ln, gg = el<C, VEC>(gc[r], q);
                adj_cell<C, FORM>(el<C, VEC>(lc[r], q), m0, mxm, mxp, mym, myp, el<C, VEC>(mm[r], q),
                                  el<C, VEC>(mp[r], q), t0, txm, txp, tym, typ, el<C, VEC>(tm[r], q),
                                  el<C, VEC>(tp[r], q), a, rx, ry, rz, lamf, ln, gg);
                set_el<C, VEC>(lo, q, ln);
                set_el<C, VEC>(go, q, gg);
            }
            // the loads are waited for here: a wait after the stores would
            // wait for the stores too
            __asm__ volatile("" : "+v"(cn[r]), "+v"(ln2[r]), "+v"(tn[r]), "+v"(gn[r]));
            __asm__ volatile("" : "+v"(hc_n[r]), "+v"(hl_n[r]), "+v"(hT_n[r]));
            __asm__ volatile("" : "+v"(yc_n), "+v"(yl_n), "+v"(yT_n));
            const int64_t p = (int64_t)k * sxy + col[r];
            if (xin && i >= z.b.i0 && i + VEC <= z.b.i1) {
                const uint32_t ob = (uint32_t)(col[r] * (int64_t)sizeof(C));
                buf_store<V, 2>(lo, rs(lam_n, k), ob);
                buf_store<V, 2>(go, rs(gCi, k), ob);
            } else if (xin) {
#pragma unroll
                for (int q = 0; q < VEC; ++q)
                    if (i + q >= z.b.i0 && i + q < z.b.i1) {
                        lam_n[p + q] = el<C, VEC>(lo, q);
                        gCi[p + q] = el<C, VEC>(go, q);
                    }
            }
            // x exchange of lam_n fused into the store
            if (z.xh.on_lo && xin && i <= z.xh.lo && i + VEC > z.xh.lo && z.xh.lo >= z.b.i0 && z.xh.lo < z.b.i1)
                lam_n[p - i + nx - 1 + z.xh.d_lo] = el_dyn<C, VEC>(lo, z.xh.lo - i);
            if (z.xh.on_hi && xin && i <= z.xh.hi && i + VEC > z.xh.hi && z.xh.hi >= z.b.i0 && z.xh.hi < z.b.i1)
                lam_n[p - i + z.xh.d_hi] = el_dyn<C, VEC>(lo, z.xh.hi - i);
            // y/z halo rows whose image is this row, each with its x exchange
            // (a wave holds one row, BX being 64: the row index is the same
            // in every lane, and the branch is taken by whole waves)
            if (z.yz.on && xin)
                yz_images(z.yz, __builtin_amdgcn_readfirstlane(jb + ty * RY + r), k, [&](int jj, int kk) {
                    C *row = lam_n + (int64_t)kk * sxy + (int64_t)jj * nx;
#pragma unroll
                    for (int q = 0; q < VEC; ++q)
                        if (i + q >= z.b.i0 && i + q < z.b.i1) row[i + q] = el<C, VEC>(lo, q);
                    if (z.xh.on_lo && i <= z.xh.lo && i + VEC > z.xh.lo && z.xh.lo >= z.b.i0 && z.xh.lo < z.b.i1)
                        row[nx - 1 + z.xh.d_lo] = el_dyn<C, VEC>(lo, z.xh.lo - i);
                    if (z.xh.on_hi && i <= z.xh.hi && i + VEC > z.xh.hi && z.xh.hi >= z.b.i0 && z.xh.hi < z.b.i1)
                        row[z.xh.d_hi] = el_dyn<C, VEC>(lo, z.xh.hi - i);
                });
        }
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            mm[r] = mc[r];
            mc[r] = mp[r];
            mp[r] = mul(cn[r], ln2[r]);
            lc[r] = lq[r];
            lq[r] = ln2[r];
            tm[r] = tc[r];
            tc[r] = tp[r];
            tp[r] = tn[r];
            gc[r] = gn[r];
            hmu[r] = hc_n[r] * hl_n[r];
            hT[r] = hT_n[r];
        }
        ymu = mul(yc_n, yl_n);
        yT = yT_n;
    }
}

static int env_int(const char *name, int dflt)
{
    const char *s = getenv(name);
    return (s && *s) ? atoi(s) : dflt;
}

template <typename C, int FORM>
static int run_boxes(const AdjArgs &a, const Box *b, int nb, hipStream_t s)
{
    BoxSet bs = make_boxset(b, nb);
    int64_t threads = bs.first[nb];
    if (threads == 0) return IGG_OK;
    hipLaunchKernelGGL((k_adj_boxes<C, FORM>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       (C *)a.lam_n, (const C *)a.lp, (const C *)a.Tn, (const C *)a.Ci, (C *)a.gCi, bs,
                       a.nx, a.ny, (C)a.a, (C)a.rx, (C)a.ry, (C)a.rz, (C)a.lamf, a.xh, a.yz);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

int launch_adjoint_boxes(int dtype, const AdjArgs &a, const Box *b, int nb, hipStream_t s)
{
    if (a.form == 1) return dtype == IGG_F64 ? run_boxes<double, 1>(a, b, nb, s) : run_boxes<float, 1>(a, b, nb, s);
    return dtype == IGG_F64 ? run_boxes<double, 0>(a, b, nb, s) : run_boxes<float, 0>(a, b, nb, s);
}

template <typename C, int VEC, int BX, int TY, int FORM, int WAVES = 1>
static int run_zmarch(const AdjArgs &a, const Box &b, hipStream_t s)
{
    constexpr int TW = BX * VEC, TH = TY;
    AdjTile z;
    z.b = b;
    z.nx = a.nx;
    z.ny = a.ny;
    z.nz = a.nz;
    const RowTiles t = row_tiles(b, VEC, TW);
    z.xa = t.xa;
    z.ntx = t.n;
    z.nty = (b.j1 - b.j0 + TH - 1) / TH;
    int depth = b.k1 - b.k0;
    int zc = env_int("IGG_ADJ_ZCHUNK", 0);
    // chunks of at most 8 planes: 3% faster than 16 at 512^3; FP64 in 4-row
    // tiles 6 (256^3 155.9 us against 160.5 with 8 and 158.5 with 16, 301 x
    // 257 x 203 160.5 against 164.3)
    if (zc < 1) zc = zchunk_for_groups((int64_t)z.ntx * z.nty, depth, sizeof(C) == 8 && TH == 4 ? 6 : 8);
    z.zc = zc;
    z.remap = env_int("IGG_ADJ_REMAP", 2);
    // blocks of 4 x-rows of tiles per XCD, so y-neighbour tiles share an
    // L2: the fastest block at 256^3 and 768^3 (by 2-6% over 1, 8, 16 and
    // 24); at 512^3 blocks of 16 are 4% faster
    z.rblock = std::max(1, env_int("IGG_ADJ_XCD_BLOCK", 4));
    z.xh = a.xh;
    z.yz = a.yz;
    int64_t blocks = (int64_t)z.ntx * z.nty * ((depth + zc - 1) / zc);
    if (blocks == 0) return IGG_OK;
    z.main = (int)blocks;
    z.ed = a.ed;
    blocks += (a.ed.total + BX * TY - 1) / (BX * TY);
    hipLaunchKernelGGL((k_adj_zmarch<C, VEC, BX, TY, FORM, WAVES>), dim3((unsigned)blocks), dim3(BX * TY), 0, s,
                       (C *)a.lam_n, (const C *)a.lp, (const C *)a.Tn, (const C *)a.Ci, (C *)a.gCi, z,
                       (C)a.a, (C)a.rx, (C)a.ry, (C)a.rz, (C)a.lamf);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

// 1 KB tile rows of 4 rows, 256 threads, one row per thread (the two
// staged fields need many registers), 16-byte loads: FP64 128 points per
// row (10% faster than 512-byte rows of 16 at 256^3 and 512^3 on MI355X;
// two rows per thread need 206 registers; since the products of the planes
// in flight moved to the rotation, 16-row tiles of 1024 threads pay at
// 512^3, see below),
// FP32 256 points (24% faster than 8-byte loads on 512-byte rows at 512^3
// and 768^3).  Rows of any length and alignment are read in vectors (255 x
// 190 x 131 FP64 77 -> 67 us, FP32 43 -> 36, 301 x 257 x 203 FP64 195 -> 161,
// against one point per lane).  The FP64 kernel is
// held to 128 registers, which fits without spills and lets 4 waves share
// each SIMD instead of 3: the kernel is partly latency-bound, and that made
// it 11% faster at 256^3 and 5% at 512^3 (unsplit; both forms).
template <int FORM>
static int adjoint_inner(int dtype, const AdjArgs &a, const Box &b, hipStream_t s)
{
    if (dtype == IGG_F64)
    {
        const int waves = env_int("IGG_ADJ_WAVES", 4);
        if (waves != 4) return run_zmarch<double, 2, 64, 4, FORM>(a, b, s);
        // regions of 2^26 points and more: 16-row tiles over 1024 threads
        // (512^3: 4-10% faster than 4 rows on three boxes; 384^3 and 256^3
        // keep 4 rows, equal or faster there)
        if (box_count(b) >= ((int64_t)1 << 26)) return run_zmarch<double, 2, 64, 16, FORM, 4>(a, b, s);
        return run_zmarch<double, 2, 64, 4, FORM, 4>(a, b, s);
    }
    // 128-point rows where they leave a fifth fewer lanes past the rows' ends
    // (301 x 257 x 203 117 -> 94 us, 384^3 305 -> 267; where both fit alike
    // 512^3 600 against 628, 401 x 300 x 250 180 against 193)
    return narrow_pays(row_tiles(b, 4, 256), row_tiles(b, 2, 128)) ? run_zmarch<float, 2, 64, 4, FORM>(a, b, s)
                                                                   : run_zmarch<float, 4, 64, 4, FORM>(a, b, s);
}

template <typename C, int FORM>
static int run_small(const AdjArgs &a, hipStream_t s)
{
    constexpr int NZ = 2;
    AdjSmall g{a.nx, a.ny, a.nz, (int)(((int64_t)(a.nx - 2) * (a.ny - 2) + 255) / 256), a.xh, a.yz, 0, a.ed};
    g.main = g.nbp * ((a.nz - 2 + NZ - 1) / NZ);
    const int64_t blocks = (int64_t)g.main + (a.ed.total + 255) / 256;
    hipLaunchKernelGGL((k_adj_small<C, FORM, NZ>), dim3((unsigned)blocks), dim3(256), 0, s, (C *)a.lam_n,
                       (const C *)a.lp, (const C *)a.Tn, (const C *)a.Ci, (C *)a.gCi, g, (C)a.a, (C)a.rx, (C)a.ry,
                       (C)a.rz, (C)a.lamf);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

int launch_adjoint_small(int dtype, const AdjArgs &a, hipStream_t s)
{
    if (a.form == 1) return dtype == IGG_F64 ? run_small<double, 1>(a, s) : run_small<float, 1>(a, s);
    return dtype == IGG_F64 ? run_small<double, 0>(a, s) : run_small<float, 0>(a, s);
}

// The edges alone, after launches whose kernel does not copy them.
template <typename S>
__global__ void __launch_bounds__(256) k_edges(S *A, EdgeLines g)
{
    const int e = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (e < g.total) edge_point(A, g, e);
}

static int launch_edges(int dtype, void *A, const EdgeLines &ed, hipStream_t s)
{
    const dim3 blocks((ed.total + 255) / 256);
    if (dtype == IGG_F64)
        hipLaunchKernelGGL(k_edges<double>, blocks, dim3(256), 0, s, (double *)A, ed);
    else
        hipLaunchKernelGGL(k_edges<float>, blocks, dim3(256), 0, s, (float *)A, ed);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

int launch_adjoint_inner(int dtype, const AdjArgs &a, const Box &b, hipStream_t s)
{
    // the z-march kernel addresses a plane with 32-bit offsets (2 GiB at
    // most), and leaves most of its lanes idle in rows of up to 36 points (two
    // ranks of 13 x 1500 x 600 FP64 510 us by the box kernel against 957, FP32 265
    // against 612; 34 x 800 x 500 475 against 508 and 254 against 350; 50 x 700 x
    // 400 600 against 390 and 323 against 263)
    const int64_t plane = (int64_t)a.nx * a.ny * (dtype == IGG_F64 ? 8 : 4);
    if (box_count(b) < zmarch_min_points() || plane + 16 >= ((int64_t)1 << 31) || a.nx < 4 ||
        (rows_dispatched() && b.i1 - b.i0 <= 36)) {
        const int rc = launch_adjoint_boxes(dtype, a, &b, 1, s);
        return rc || !a.ed.total ? rc : launch_edges(dtype, a.lam_n, a.ed, s);
    }
    return a.form == 1 ? adjoint_inner<1>(dtype, a, b, s) : adjoint_inner<0>(dtype, a, b, s);
}

}  // namespace igg
