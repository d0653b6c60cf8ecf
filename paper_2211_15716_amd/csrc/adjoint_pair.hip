// adjoint_pair.hip -- two adjoint steps of the Laplacian form in one launch.
//
// From lambda_{n+2} and T_n: T_{n+1} (the forward step's own arithmetic) and
// lambda_{n+1} are computed tile by tile and kept on chip, then lambda_n is
// computed from lambda_{n+1}, and gCi takes the terms of both steps, the later
// one's first.  lambda_{n+2}, T_n, Ci and gCi are read and lambda_n and gCi
// are written once for two steps, and T_{n+1} need not be stored at all.
// Every point goes through the arithmetic of the one-step kernels with the
// operands they give it, so the bits are those of two single steps.  A
// work-group recomputes the lambda_{n+1} and T_{n+1} points its tile shares
// with its neighbours (one layer on every side).
//
// One rank, overlaps of 2 in the periodic dimensions.  The halo of
// lambda_{n+1} and T_{n+1} is formed as the halo update would: a periodic
// dimension's from its images; one without a period keeps lambda_{n+2}'s
// (zero) and T_n's.  The halo of lambda_n is stored with the points it copies.
#include "pair.hpp"

namespace igg {

namespace {

template <typename C> struct AdjPairCoef {
    C a, rx, ry, rz;
};

// ------------------------------------------------------------ small grids
// One block of BX x BY x BZ points of lambda_n per work-group, as
// k_step2_block: lambda_{n+1}, mu = Ci.*lambda_{n+1} and T_{n+1} of the block
// and one layer around it go to LDS.  Bound by the loads' instructions and latency.
template <typename C, int BX, int BY, int BZ>
__global__ void __launch_bounds__(1024)
k_adj2_block(C *__restrict__ lam, const C *__restrict__ l2, const C *__restrict__ T, const C *__restrict__ Ci,
             C *__restrict__ gCi, PairGeom g, int nbx, int nby, AdjPairCoef<C> cf)
{
    constexpr int UX = BX + 2, UY = BY + 2, UZ = BZ + 2, NU = UX * UY * UZ, NO = BX * BY * BZ, NT = 1024;
    constexpr uint32_t E = sizeof(C);
    __shared__ C u[UZ][UY][UX];  // lambda_{n+1}
    __shared__ C m[UZ][UY][UX];  // Ci.*lambda_{n+1}
    __shared__ C w[UZ][UY][UX];  // T_{n+1}
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = 1 + b % nbx * BX, y0 = 1 + b / nbx % nby * BY, z0 = 1 + b / nbx / nby * BZ;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const uint32_t ey = (uint32_t)nx * E, ez = ey * (uint32_t)ny;
    auto ld = [](const C *A, uint32_t o) -> C {
        return *reinterpret_cast<const C *>(reinterpret_cast<const char *>(A) + o);
    };
    auto mu = [&](uint32_t o) -> C { return ld(Ci, o) * ld(l2, o); };
    auto lapT = [&](uint32_t p) -> C {
        return laplace<C>(ld(T, p), ld(T, p - E), ld(T, p + E), ld(T, p - ey), ld(T, p + ey), ld(T, p - ez),
                          ld(T, p + ez), cf.rx, cf.ry, cf.rz);
    };
    auto lapS = [&](const C (&s)[UZ][UY][UX], int x, int y, int z) -> C {
        return laplace<C>(s[z][y][x], s[z][y][x - 1], s[z][y][x + 1], s[z][y - 1][x], s[z][y + 1][x], s[z - 1][y][x],
                          s[z + 1][y][x], cf.rx, cf.ry, cf.rz);
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
        C v, c, tn;
        if ((hx && !g.per[0]) || (hy && !g.per[1]) || (hz && !g.per[2])) {
            const uint32_t p = (uint32_t)x * E + ey * (uint32_t)y + ez * (uint32_t)z;
            c = ld(Ci, p);
            v = ld(l2, p);
            tn = ld(T, p);
        } else {
            const int xi = hx ? wrap(x, nx, 1) : x, yi = hy ? wrap(y, ny, 1) : y, zi = hz ? wrap(z, nz, 1) : z;
            const uint32_t p = (uint32_t)xi * E + ey * (uint32_t)yi + ez * (uint32_t)zi;
            const C l = ld(l2, p);
            c = ld(Ci, p);
            const C lap = laplace<C>(c * l, mu(p - E), mu(p + E), mu(p - ey), mu(p + ey), mu(p - ez), mu(p + ez),
                                     cf.rx, cf.ry, cf.rz);
            v = adjoint_lam<C>(l, lap, cf.a);
            tn = fma_(cf.a * c, lapT(p), ld(T, p));
        }
        u[uz][uy][ux] = v;
        w[uz][uy][ux] = tn;
        m[uz][uy][ux] = c * v;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NO / NT; ++t) {
        const int q = t * NT + threadIdx.x;
        const int ux = 1 + q % BX, uy = 1 + q / BX % BY, uz = 1 + q / (BX * BY);
        const int x = x0 - 1 + ux, y = y0 - 1 + uy, z = z0 - 1 + uz;
        if (x > nx - 2 || y > ny - 2 || z > nz - 2) continue;
        const uint32_t p = (uint32_t)x * E + ey * (uint32_t)y + ez * (uint32_t)z;
        const C l1 = u[uz][uy][ux];
        const C ga = adjoint_grad<C>(ld(l2, p), lapS(w, ux, uy, uz), cf.a, ld(gCi, p));
        const C gg = adjoint_grad<C>(l1, lapT(p), cf.a, ga);
        pair_store(g, x, y, z, lam, adjoint_lam<C>(l1, lapS(m, ux, uy, uz), cf.a));
        *reinterpret_cast<C *>(reinterpret_cast<char *>(gCi) + p) = gg;
    }
}

// ------------------------------------------------------------ large grids
// Vectors of one LDS tile: a constant, so that the four tiles are at constant
// distances and share their address registers.
constexpr int kAdjPlane = 1024;

// The tiling of k_step2_zmarch with one row per thread.  At plane k a work-group
// has four LDS tiles (mu_{n+2} and T_n of plane k, mu_{n+1} and T_{n+1} of
// plane k-1) in one of two buffers, the tiles of the plane before in the other,
// and in registers Ci and lambda_{n+2} of planes k and k+1 and T_n of plane
// k+1, with the next planes in flight: one barrier a plane.  It computes
// T_{n+1} and lambda_{n+1} at plane k, then lambda_n and both terms of gCi at
// plane k-1.
// Bound by HBM bytes (6 arrays for two steps: 4.5 TB/s at 256^3 FP64, 4.6 at
// 400^3) and the rows re-read around the tiles; about 100 registers, so that
// 1024 threads fit a CU (kept through the loop: the state above only, the
// Laplacians' operands for one of the four at a time; with all four at once
// and the store addresses kept, 44 registers spilled).  Reading T_{n+1} from
// memory instead of forming it: 200 us at 256^3 FP64 against 179.  pair_tiles
// chose within 2% of the fastest of about 60 shapes at 256^3, 160^3, 200 x 180
// x 150 and 301 x 257 x 203.
template <typename S, int VEC, int GEN>
__global__ void __launch_bounds__(1024)
k_adj2_zmarch(S *__restrict__ lam, const S *__restrict__ l2, const S *__restrict__ T, const S *__restrict__ Ci,
              S *__restrict__ gCi, PairTile z, AdjPairCoef<S> cf)
{
    typedef S V __attribute__((ext_vector_type(VEC)));
    constexpr uint32_t E = sizeof(S);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const PairGeom &g = z.g;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int64_t sxy = (int64_t)nx * ny;
    const int W = z.W, H = z.HG;
    V *lds = reinterpret_cast<V *>(lds_raw) + 1;
    constexpr int plane = kAdjPlane;

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
    const int t = threadIdx.x, th = t - H * (W - 2);  // th >= 0: a vector beside the tile
    const bool live = th < 2 * H;
    const int lr = min(th < 0 ? t / (W - 2) : th >> 1, H - 1);
    const int tv = th < 0 ? 1 + t % (W - 2) : (th & 1 ? W - 1 : 0);
    const int i = (bx * (W - 2) + tv - 1) * VEC;
    const int j = 1 + by * (H - 4) - 2 + lr;
    const int kb = 1 + bz * z.zc;
    const int ke = kb + z.zc < nz - 1 ? kb + z.zc : nz - 1;

    // lambda_{n+2}, T_n and Ci: where a vector is read (as in k_step2_zmarch)
    int iv = i;
    if (i < 0) iv = g.per[0] ? i + nx - 2 : 0;
    if (i >= nx) iv = g.per[0] ? i - (nx - 2) : 0;
    const bool cross = i < nx && i + VEC > nx;
    int hq = -1, hx = 0;
    if (g.per[0] && i == 0) { hq = 0; hx = nx - 2; }
    if (g.per[0] && i < nx && i + VEC >= nx) { hq = nx - 1 - i; hx = 1; }
    const bool edges = GEN && g.per[0] && !(g.per[1] && g.per[2]);
    const uint32_t row = (uint32_t)(wrap(j, ny, g.per[1]) * nx) * E, vo = row + (uint32_t)iv * E;
    // gCi is read where it is written (elsewhere an offset past every plane:
    // the load gives zero and touches no memory)
    constexpr uint32_t none = 0xffffff00u;
    const bool st = live && lr >= 2 && lr < H - 2 && j <= ny - 2 && tv >= 1 && tv < W - 1 && i < nx;
    const uint32_t go_ = st ? (uint32_t)(j * nx + i) * E : none;
    const uint32_t h1 = edges && hq >= 0 ? row + (uint32_t)hx * E : none;
    uint32_t fixed = 0;  // points that keep lambda_{n+2}'s and T_n's values
#pragma unroll
    for (int q = 0; q < VEC; ++q)
        if ((!g.per[0] && (i + q <= 0 || i + q >= nx - 1)) || (!g.per[1] && (j <= 0 || j >= ny - 1))) fixed |= 1u << q;

    const int64_t pb = sxy * (int64_t)E;
    // (a vector that runs over its row's end may run into the next plane; past
    // the array's end it reads zero, which is not used)
    auto rs = [&](const S *A, int k) { return buf_rsrc(A + (int64_t)k * sxy, pb + (GEN && k < nz - 1 ? 16 : 0)); };
    auto ldw = [&](const S *A, int k) -> V {
        const __amdgpu_buffer_rsrc_t d = rs(A, wrap(k, nz, g.per[2]));
        V v;
        if (!GEN || !cross) {
            v = buf_load<V, 0>(d, vo);
        } else {
#pragma unroll
            for (int q = 0; q < VEC; ++q) v[q] = buf_load<S, 0>(d, row + (uint32_t)wrap(i + q, nx, g.per[0]) * E);
        }
        return v;
    };
    auto ld1 = [&](const S *A, int k) -> S {
        if constexpr (GEN) return buf_load<S, 0>(rs(A, wrap(k, nz, g.per[2])), h1);
        return S(0);
    };
    auto patch = [&](V v, S x) -> V {
        if constexpr (GEN) {
#pragma unroll
            for (int q = 0; q < VEC; ++q)
                if (h1 != none && q == hq) v[q] = x;
        }
        return v;
    };
    auto ldp = [&](const S *A, int k) -> V { return patch(ldw(A, k), ld1(A, k)); };

    // (threads beyond the work-group's vectors have places of their own)
    const int lb = live ? lr * W + tv : t, up = live && lr > 0 ? lb - W : lb, dn = live && lr < H - 1 ? lb + W : lb;
    // the Laplacian of a plane from its LDS tile, this thread's vector of the
    // plane before (which stands in the other buffer's tile until this plane
    // is done) and of the plane after
    auto lap = [&](const V *s, const V &m, const V &p) -> V {
        const S *e = reinterpret_cast<const S *>(s) + lb * VEC;
        const S xl = e[-1], xr = e[VEC];
        const V c = s[lb], vu = s[up], vd = s[dn];
        V o;
#pragma unroll
        for (int q = 0; q < VEC; ++q)
            o[q] = laplace<S>(c[q], q == 0 ? xl : c[q > 0 ? q - 1 : 0], q == VEC - 1 ? xr : c[q < VEC - 1 ? q + 1 : q],
                              vu[q], vd[q], m[q], p[q], cf.rx, cf.ry, cf.rz);
        return o;
    };

    V lc = ldp(l2, kb - 1), lp = ldp(l2, kb), cc = ldp(Ci, kb - 1), cp = ldp(Ci, kb), tp = ldp(T, kb);
    V gk{}, l1{}, l2p{}, ltp{};  // of plane k-1: gCi, lambda_{n+1}, lambda_{n+2}, the Laplacian of T_n
    {
        V *o = lds + lb;
        o[0] = cc * lc;
        o[plane] = ldp(T, kb - 1);
        o[2 * plane] = o[3 * plane] = V{};
        o += 4 * plane;
        o[0] = ldp(Ci, kb - 2) * ldp(l2, kb - 2);
        o[plane] = ldp(T, kb - 2);
        o[2 * plane] = o[3 * plane] = V{};
    }
    for (int k = kb - 1; k <= ke; ++k) {
        const int buf = (k - kb + 1) & 1;
        V *sM2 = lds + buf * 4 * plane, *sT0 = sM2 + plane, *sM1 = sT0 + plane, *sT1 = sM1 + plane;
        V *oM2 = lds + (buf ^ 1) * 4 * plane + lb, *oT0 = oM2 + plane, *oM1 = oT0 + plane, *oT1 = oM1 + plane;
        // (the last plane's loads are read again and not used)
        const int kn = k < ke ? k + 2 : k;
        V ln = ldw(l2, kn), cn = ldw(Ci, kn), tn = ldw(T, kn);
        S ln1 = ld1(l2, kn), cn1 = ld1(Ci, kn), tn1 = ld1(T, kn);
        V gn = buf_load<V, 2>(rs(gCi, min(k, nz - 2)), go_);
        __syncthreads();
        const uint32_t fx = !g.per[2] && (k <= 0 || k >= nz - 1) ? ~0u : fixed;
        // (one Laplacian's operands in registers at a time; the next plane's
        // vectors go to the other buffer as soon as this one's are used)
        V lt, un, tu, go, o;
        {
            const V c = sT0[lb];
            lt = lap(sT0, *oT0, tp);
            *oT0 = tp;
#pragma unroll
            for (int q = 0; q < VEC; ++q) tu[q] = fx >> q & 1 ? c[q] : fma_(cf.a * cc[q], lt[q], c[q]);
        }
        __asm__ volatile("" : "+v"(lt), "+v"(tu));
        __builtin_amdgcn_sched_barrier(0);
        {
            const V lu = lap(sT1, *oT1, tu);
            *oT1 = tu;
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const S ga = adjoint_grad<S>(l2p[q], lu[q], cf.a, gk[q]);
                go[q] = adjoint_grad<S>(l1[q], ltp[q], cf.a, ga);
            }
        }
        __asm__ volatile("" : "+v"(go));
        __builtin_amdgcn_sched_barrier(0);
        {
            const V mp = cp * lp, lm = lap(sM2, *oM2, mp);
            *oM2 = mp;
#pragma unroll
            for (int q = 0; q < VEC; ++q) un[q] = fx >> q & 1 ? lc[q] : adjoint_lam<S>(lc[q], lm[q], cf.a);
        }
        __asm__ volatile("" : "+v"(un));
        __builtin_amdgcn_sched_barrier(0);
        {
            const V mp = cc * un, lm = lap(sM1, *oM1, mp);
            *oM1 = mp;
#pragma unroll
            for (int q = 0; q < VEC; ++q) o[q] = adjoint_lam<S>(l1[q], lm[q], cf.a);
        }
        __asm__ volatile("" : "+v"(o));
        // the loads are waited for here, before the stores: a wait after them
        // would wait for the stores too
        __asm__ volatile("" : "+v"(ln), "+v"(cn), "+v"(tn), "+v"(gn));
        if constexpr (GEN) __asm__ volatile("" : "+v"(ln1), "+v"(cn1), "+v"(tn1));
        if (k > kb && st) {
            // (addresses formed here, not kept through the loop: registers)
            int is = i, js = j;
            __asm__ volatile("" : "+v"(is), "+v"(js));
            pair_put<S, VEC>(g, lam, is, js, k - 1, o, 1);
            const __amdgpu_buffer_rsrc_t d = buf_rsrc(gCi + (int64_t)(k - 1) * sxy, pb);
            if (is >= 1 && is + VEC <= nx - 1) {
                buf_store<V, 2>(go, d, go_);
            } else {
#pragma unroll
                for (int q = 0; q < VEC; ++q)
                    if (is + q >= 1 && is + q <= nx - 2) buf_store<S, 0>(go[q], d, (uint32_t)(js * nx + is + q) * E);
            }
        }
        l2p = lc;
        lc = lp;
        cc = cp;
        lp = patch(ln, ln1);
        cp = patch(cn, cn1);
        tp = patch(tn, tn1);
        gk = gn;
        l1 = un;
        ltp = lt;
    }
}

template <typename C, int BX, int BY, int BZ>
int run_block(const AdjPairArgs &a, hipStream_t s)
{
    const PairGeom g{{a.nx, a.ny, a.nz}, {a.per[0], a.per[1], a.per[2]}};
    const int nbx = (a.nx - 2 + BX - 1) / BX, nby = (a.ny - 2 + BY - 1) / BY, nbz = (a.nz - 2 + BZ - 1) / BZ;
    const AdjPairCoef<C> cf{(C)a.a, (C)a.rx, (C)a.ry, (C)a.rz};
    hipLaunchKernelGGL((k_adj2_block<C, BX, BY, BZ>), dim3((unsigned)((int64_t)nbx * nby * nbz)), dim3(1024), 0, s,
                       (C *)a.lam, (const C *)a.l2, (const C *)a.T, (const C *)a.Ci, (C *)a.gCi, g, nbx, nby, cf);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

template <typename S, int VEC>
int run_march(const AdjPairArgs &a, hipStream_t s)
{
    PairTile z{};
    z.g = PairGeom{{a.nx, a.ny, a.nz}, {a.per[0], a.per[1], a.per[2]}};
    pair_tiles<VEC, 1>(a.nx, a.ny, a.nz, z);
    const int64_t blocks = (int64_t)z.ntx * z.nty * ((a.nz - 2 + z.zc - 1) / z.zc);
    z.deal = blocks > 512;
    const size_t lds = ((size_t)8 * kAdjPlane + 2) * VEC * sizeof(S);
    const int tpb = (z.W * z.HG + 63) / 64 * 64;
    const AdjPairCoef<S> cf{(S)a.a, (S)a.rx, (S)a.ry, (S)a.rz};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(tpb), lds, s, (S *)a.lam, (const S *)a.l2,
                           (const S *)a.T, (const S *)a.Ci, (S *)a.gCi, z, cf);
    };
    // GEN: rows that end inside a vector, or a halo of x that meets planes of a
    // dimension without a period
    if (a.nx % VEC == 0 && !(a.per[0] && !(a.per[1] && a.per[2]))) go(k_adj2_zmarch<S, VEC, 0>);
    else go(k_adj2_zmarch<S, VEC, 1>);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

}  // namespace

// Which kernel takes a pair on this grid (0: none, two single steps are as
// fast).  A pair saves the store of T_{n+1} in the forward steps too; us for
// the adjoint pair and a forward pair without that store against two adjoint
// steps and a forward pair with it.  Marching in FP64 from 3 * 2^18 points on
// (96^3 35 against 42, 128^3 52 against 78), in FP32 from 7 * 2^18 (128^3 41
// against 47, 110^3 49 against 36); blocks below that in FP64 and below 2^19
// points in FP32 (80^3 24 against 27, FP32 19 against 19, 96^3 30 against 27,
// but one launch less to make: 48^3 FP64 11.5 against 21 for the adjoint steps
// called in turn from Python).  256^3 FP64: 179 against 323 for the adjoint
// steps, FP32 93 against 161.  Or marching from the points that
// IGG_ZMARCH_MIN_POINTS asks for on.
enum { kNoPair, kPairBlocks, kPairMarch };
static int adjoint_pair_kernel(int dtype, const int n[3])
{
    if (dtype == IGG_F16) return kNoPair;
    const int64_t pts = (int64_t)(n[0] - 2) * (n[1] - 2) * (n[2] - 2), zm = zmarch_min_points();
    const bool def = zm == kZmarchMinPoints;
    const int64_t esz = elem_bytes(dtype);
    // 32-bit offsets in a plane (marching) or an array (blocks); rows that
    // can be read a period away
    if (pts >= (def ? (dtype == IGG_F64 ? 3 << 18 : 7 << 18) : zm))
        return n[0] >= 16 && (int64_t)n[0] * n[1] * esz + 16 < ((int64_t)1 << 31) ? kPairMarch : kNoPair;
    if (def && dtype == IGG_F32 && pts >= 1 << 19) return kNoPair;
    return (int64_t)n[0] * n[1] * n[2] * esz < ((int64_t)1 << 31) ? kPairBlocks : kNoPair;
}

bool adjoint_pair_pays(int dtype, const int n[3])
{
    return adjoint_pair_kernel(dtype, n) != kNoPair;
}

int launch_adjoint_pair(int dtype, const AdjPairArgs &a, hipStream_t s)
{
    const int n[3] = {a.nx, a.ny, a.nz};
    if (adjoint_pair_kernel(dtype, n) == kPairBlocks)
        return dtype == IGG_F64 ? run_block<double, 16, 8, 8>(a, s) : run_block<float, 16, 8, 8>(a, s);
    return dtype == IGG_F64 ? run_march<double, 2>(a, s) : run_march<float, 4>(a, s);
}

}  // namespace igg
