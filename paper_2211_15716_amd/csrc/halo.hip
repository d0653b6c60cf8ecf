// halo.hip -- halo update of the implicit global grid (Fig. 1 `update_halo!`,
// Sec. 2).  Neighbouring local grids share `ol` planes: my plane ol-1 is the
// last plane of my lower neighbour and my plane n-ol is the first plane of my
// upper neighbour.  For each dimension x, y, z in turn, the two planes of
// every field are packed into send buffers, exchanged (the lower neighbour
// receives plane ol-1 into the buffer that fills its last plane, the upper
// one plane n-ol into the buffer that fills its first plane), and unpacked.
// Dimensions go in order and planes are whole, so a later dimension carries
// the halo values an earlier one wrote, and edges and corners come out as
// images in every periodic dimension.
//
// The process holds every rank of the topology (one, or several virtual
// ranks as separate blocks on this device), so the exchange is a device copy
// from a rank's send buffer into its neighbour's receive buffer.  One launch
// per dimension and rank runs all three phases: each thread packs its
// elements, exchanges them and unpacks them into the neighbour's halo.  One
// rank is its own neighbour in every periodic dimension, and one launch fills
// its halo without buffers (launch_halo_one).
#include "host.hpp"

namespace igg {

// One side of one field in one dimension.  Element (a, b) of a plane is at
// base[plane*sd + a*sa + b*sb] and at buf[a + na*b]; units are `esz` bytes
// (16 when whole rows move as 16-byte vectors).
struct HaloDesc {
    unsigned char *src_base;  // my field
    unsigned char *dst_base;  // the neighbour's field (mine on a periodic single rank)
    unsigned char *send;      // my send buffer for this side
    unsigned char *recv;      // the neighbour's receive buffer this side's data lands in
    int64_t sd, sa, sb;
    int na, nb;
    int src, dst;  // plane packed from, plane unpacked into
    int esz;
};

struct HaloSet {
    HaloDesc d[2 * IGG_MAX_FIELDS];
};

template <typename E>
__device__ __forceinline__ void halo_elem(const HaloDesc &d, int64_t e)
{
    const int a = (int)(e % d.na);
    const int b = (int)(e / d.na);
    const int64_t off = (int64_t)a * d.sa + (int64_t)b * d.sb;
    const E *A = reinterpret_cast<const E *>(d.src_base);
    E *B = reinterpret_cast<E *>(d.dst_base);
    E *send = reinterpret_cast<E *>(d.send);
    E *recv = reinterpret_cast<E *>(d.recv);
    send[e] = A[(int64_t)d.src * d.sd + off];  // pack
    recv[e] = send[e];                         // exchange (a device copy: the neighbour is on this GPU)
    B[(int64_t)d.dst * d.sd + off] = recv[e];  // unpack into the neighbour's halo
}

// blockIdx.y selects the (field, side); x-threads walk the plane.
__global__ void __launch_bounds__(256) k_halo_self(HaloSet hs)
{
    const HaloDesc &d = hs.d[blockIdx.y];
    const int64_t count = (int64_t)d.na * d.nb;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x) {
        switch (d.esz) {
        case 16: halo_elem<uint4>(d, e); break;
        case 8: halo_elem<uint64_t>(d, e); break;
        case 4: halo_elem<uint32_t>(d, e); break;
        default: halo_elem<uint16_t>(d, e); break;
        }
    }
}

// Rank r owns 4 * IGG_MAX_FIELDS planes: send buffers of (field, side), then
// receive buffers of (field, side); side 0 faces the lower neighbour.
static unsigned char *send_buf(Grid &g, int r, int f, int side)
{
    return g.halo_buf + ((size_t)r * 4 * IGG_MAX_FIELDS + f * 2 + side) * g.halo_cap;
}

static unsigned char *recv_buf(Grid &g, int r, int f, int side)
{
    return g.halo_buf + ((size_t)r * 4 * IGG_MAX_FIELDS + 2 * IGG_MAX_FIELDS + f * 2 + side) * g.halo_cap;
}

unsigned char *halo_send_plane(int r, int f, int side) { return send_buf(grid(), r, f, side); }

// Exchange and unpack of the planes the boundary-slab kernel packed, for a
// rank that is its own neighbour: the receive side of the exchange is the
// destination halo plane itself, so each element is copied once, from the
// send buffer into the field.  d[q] is plane q: element (a, b) of the
// packed plane (a fastest) goes to dst[a*sa + b*sb], units of esz bytes.
struct PlaneCopy {
    const unsigned char *src;
    unsigned char *dst;
    int64_t sa, sb;
    int na, nb;
    int esz;
};
struct PlaneCopySet {
    PlaneCopy d[4];
};

template <typename E>
__device__ __forceinline__ void copy_elem(const PlaneCopy &d, int64_t e)
{
    const int a = (int)(e % d.na);
    const int b = (int)(e / d.na);
    reinterpret_cast<E *>(d.dst)[(int64_t)a * d.sa + (int64_t)b * d.sb] = reinterpret_cast<const E *>(d.src)[e];
}

__global__ void __launch_bounds__(256) k_unpack_planes(PlaneCopySet ps)
{
    const PlaneCopy &d = ps.d[blockIdx.y];
    const int64_t count = (int64_t)d.na * d.nb;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x) {
        switch (d.esz) {
        case 16: copy_elem<uint4>(d, e); break;
        case 8: copy_elem<uint64_t>(d, e); break;
        case 4: copy_elem<uint32_t>(d, e); break;
        default: copy_elem<uint16_t>(d, e); break;
        }
    }
}

int launch_unpack_self(const igg_field &f, const SlabPack &pk, hipStream_t s)
{
    const int64_t nx = f.size[0], ny = f.size[1], nz = f.size[2];
    const int64_t e = elem_bytes(f.dtype);
    PlaneCopySet ps{};
    int64_t maxcount = 0;
    for (int d = 0; d < 2; ++d)
        for (int side = 0; side < 2; ++side) {
            PlaneCopy &c = ps.d[2 * d + side];
            c.esz = (int)e;
            c.src = (const unsigned char *)pk.send[d][side];
            c.na = (int)nx;
            c.sa = 1;
            if (d == 0) {  // y plane: a = x, b = z, into row j
                const int64_t j = side == 0 ? ny - 1 : 0;
                c.dst = (unsigned char *)f.data + j * nx * e;
                c.nb = (int)nz;
                c.sb = nx * ny;
            } else {  // z plane: a = x, b = y, into plane k
                const int64_t k = side == 0 ? nz - 1 : 0;
                c.dst = (unsigned char *)f.data + k * nx * ny * e;
                c.nb = (int)ny;
                c.sb = nx;
            }
            // whole rows as 16-byte vectors where the row length and base allow
            if ((nx * e) % 16 == 0 && ((uintptr_t)f.data % 16) == 0) {
                c.na = (int)(nx * e / 16);
                c.sb = c.sb * e / 16;
                c.esz = 16;
            }
            maxcount = std::max(maxcount, (int64_t)c.na * c.nb);
        }
    const int64_t b = (maxcount + 255) / 256;
    dim3 grd((unsigned)std::min<int64_t>(std::max<int64_t>(b, 1), 1024), 4);
    hipLaunchKernelGGL(k_unpack_planes, grd, dim3(256), 0, s, ps);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

// ------------------------------------------------------------- one rank
// The halo update of a rank that is its own neighbour in the periodic
// dimensions: the dimension-ordered exchange of whole planes leaves at a halo
// point the value at its image, the index map img(0) = n-ol, img(n-1) = ol-1,
// img(c) = c otherwise, applied in every updated dimension.  Images are not
// halo points of those dimensions, so every halo point of every field and
// dimension is filled at once, each from one read.  Bound by the launch and by
// the x planes, which are two elements of every row.
struct GatherField {
    unsigned char *base;
    int n[3];
    int lo[3], hi[3];  // images of n-1 and 0
    int esz;
};
struct GatherSet {
    GatherField f[IGG_MAX_FIELDS];
    int dims;  // bit d: dimension d is updated (and periodic)
    int rows_blocks;  // work-groups of the y and z planes; the rest take the x planes
};

__device__ __forceinline__ int halo_img(int c, int n, int lo, int hi) { return c == 0 ? hi : (c == n - 1 ? lo : c); }

template <typename E>
__device__ __forceinline__ void gather_field(const GatherField &f, int dims, int rb)
{
    constexpr int VEC = 16 / (int)sizeof(E);
    typedef E V __attribute__((ext_vector_type(VEC)));
    typedef E M __attribute__((ext_vector_type(VEC), aligned(sizeof(E))));
    E *A = reinterpret_cast<E *>(f.base);
    const int nx = f.n[0], ny = f.n[1], nz = f.n[2];
    const int64_t sxy = (int64_t)nx * ny;
    const bool dx = dims & 1, dy = dims & 2, dz = dims & 4;
    auto src_row = [&](int j, int k) -> const E * {
        const int js = dy ? halo_img(j, ny, f.lo[1], f.hi[1]) : j, ks = dz ? halo_img(k, nz, f.lo[2], f.hi[2]) : k;
        return A + ks * sxy + (int64_t)js * nx;
    };
    if ((int)blockIdx.x < rb) {
        // y and z planes: vectors of their rows (2 nz rows of the y planes,
        // then 2 ny of the z planes)
        const uint32_t nv = (uint32_t)((nx + VEC - 1) / VEC), yr = dy ? 2u * nz : 0u, zr = dz ? 2u * ny : 0u;
        const uint32_t count = nv * (yr + zr);
        for (uint32_t e = blockIdx.x * 256 + threadIdx.x; e < count; e += (uint32_t)rb * 256) {
            const uint32_t row = e / nv;
            const int i = (int)(e - row * nv) * VEC;
            int j, k;
            if (row < yr) {
                j = row & 1 ? ny - 1 : 0;
                k = (int)(row >> 1);
            } else {
                j = (int)((row - yr) >> 1);
                k = (row - yr) & 1 ? nz - 1 : 0;
            }
            E *D = A + k * sxy + (int64_t)j * nx;
            const E *P = src_row(j, k);
            if (i + VEC <= nx) {
                V v = *reinterpret_cast<const M *>(P + i);
                if (dx && i == 0) v[0] = P[f.hi[0]];
                if (dx && i + VEC == nx) v[VEC - 1] = P[f.lo[0]];
                *reinterpret_cast<M *>(D + i) = v;
            } else {
                for (int q = i; q < nx; ++q) D[q] = P[dx ? halo_img(q, nx, f.lo[0], f.hi[0]) : q];
            }
        }
    } else if (dx) {
        // x planes: both ends of every row that is in no updated y or z plane
        const uint32_t j0 = dy ? 1 : 0, k0 = dz ? 1 : 0, h = ny - 2 * j0, count = h * (nz - 2 * k0);
        const uint32_t step = (gridDim.x - rb) * 256;
        for (uint32_t e = (blockIdx.x - rb) * 256 + threadIdx.x; e < count; e += step) {
            const uint32_t k = e / h;
            E *D = A + (int64_t)(k + k0) * sxy + (int64_t)(e - k * h + j0) * nx;
            const E a = D[f.hi[0]], b = D[f.lo[0]];
            D[0] = a;
            D[nx - 1] = b;
        }
    }
}

__global__ void __launch_bounds__(256) k_halo_gather(GatherSet gs)
{
    const GatherField &f = gs.f[blockIdx.y];
    switch (f.esz) {
    case 8: gather_field<uint64_t>(f, gs.dims, gs.rows_blocks); break;
    case 4: gather_field<uint32_t>(f, gs.dims, gs.rows_blocks); break;
    default: gather_field<uint16_t>(f, gs.dims, gs.rows_blocks); break;
    }
}

static int launch_halo_one(const igg_field *fl, int nf, hipStream_t s, int dims)
{
    Grid &g = grid();
    GatherSet gs{};
    for (int d = 0; d < 3; ++d)
        if (((dims >> d) & 1) && g.periods[d]) gs.dims |= 1 << d;
    if (gs.dims == 0) return IGG_OK;
    int64_t rows = 0, cols = 0;
    for (int q = 0; q < nf; ++q) {
        GatherField &f = gs.f[q];
        f.base = (unsigned char *)fl[q].data;
        f.esz = elem_bytes(fl[q].dtype);
        for (int d = 0; d < 3; ++d) {
            f.n[d] = (int)fl[q].size[d];
            const int ol = g.ol[d] + (f.n[d] - g.n[d]);
            f.lo[d] = ol - 1;
            f.hi[d] = f.n[d] - ol;
        }
        const int64_t nv = ((int64_t)f.n[0] * f.esz + 15) / 16;
        rows = std::max(rows, nv * ((gs.dims & 2 ? 2 * f.n[2] : 0) + (gs.dims & 4 ? 2 * f.n[1] : 0)));
        cols = std::max(cols, gs.dims & 1 ? (int64_t)f.n[1] * f.n[2] : 0);
    }
    auto blocks = [](int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 2048); };
    gs.rows_blocks = blocks(rows);
    hipLaunchKernelGGL(k_halo_gather, dim3((unsigned)(gs.rows_blocks + blocks(cols)), nf), dim3(256), 0, s, gs);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

int launch_halo(const igg_field *fl, int nf, hipStream_t s, int dims)
{
    Grid &g = grid();
    if (g.nranks == 1) return launch_halo_one(fl, nf, s, dims);
    for (int d = 0; d < 3; ++d) {
        if (!((dims >> d) & 1)) continue;  // done elsewhere (fused into the step)
        for (int r = 0; r < g.nranks; ++r) {
            HaloSet hs{};
            int nd = 0;
            int64_t maxcount = 0;
            const int lo_nbr = rank_neighbor(r, d, 0), hi_nbr = rank_neighbor(r, d, 1);
            for (int f = 0; f < nf; ++f) {
                const igg_field &F = fl[(size_t)r * nf + f];
                const int64_t nx = F.size[0], ny = F.size[1], nz = F.size[2];
                const int nA = (int)F.size[d];
                const int olA = g.ol[d] + (nA - g.n[d]);
                HaloDesc base{};
                base.esz = elem_bytes(F.dtype);
                if (d == 0) {
                    base.sd = 1; base.na = (int)ny; base.sa = nx; base.nb = (int)nz; base.sb = nx * ny;
                } else if (d == 1) {
                    base.sd = nx; base.na = (int)nx; base.sa = 1; base.nb = (int)nz; base.sb = nx * ny;
                } else {
                    base.sd = nx * ny; base.na = (int)nx; base.sa = 1; base.nb = (int)ny; base.sb = nx;
                }
                // whole rows as 16-byte vectors where rows, strides and bases allow
                const int64_t e = base.esz;
                bool vec = base.sa == 1 && (base.na * e) % 16 == 0 && (base.sb * e) % 16 == 0 &&
                           (base.sd * e) % 16 == 0 && ((uintptr_t)F.data % 16) == 0;
                for (int q : {lo_nbr, hi_nbr})
                    if (q >= 0 && ((uintptr_t)fl[(size_t)q * nf + f].data % 16) != 0) vec = false;
                if (vec) {
                    base.na = (int)(base.na * e / 16);
                    base.sb = base.sb * e / 16;
                    base.sd = base.sd * e / 16;
                    base.esz = 16;
                }
                base.src_base = (unsigned char *)F.data;
                if (lo_nbr >= 0) {
                    // plane ol-1 becomes the lower neighbour's last plane
                    HaloDesc lo = base;
                    lo.dst_base = (unsigned char *)fl[(size_t)lo_nbr * nf + f].data;
                    lo.src = olA - 1;
                    lo.dst = nA - 1;
                    lo.send = send_buf(g, r, f, 0);
                    lo.recv = recv_buf(g, lo_nbr, f, 1);
                    hs.d[nd++] = lo;
                }
                if (hi_nbr >= 0) {
                    // plane n-ol becomes the upper neighbour's first plane
                    HaloDesc hi = base;
                    hi.dst_base = (unsigned char *)fl[(size_t)hi_nbr * nf + f].data;
                    hi.src = nA - olA;
                    hi.dst = 0;
                    hi.send = send_buf(g, r, f, 1);
                    hi.recv = recv_buf(g, hi_nbr, f, 0);
                    hs.d[nd++] = hi;
                }
                maxcount = std::max(maxcount, (int64_t)base.na * base.nb);
            }
            if (nd == 0) continue;  // no neighbour in this dimension
            int64_t b = (maxcount + 255) / 256;
            dim3 grd((unsigned)std::min<int64_t>(std::max<int64_t>(b, 1), 1024), nd);
            hipLaunchKernelGGL(k_halo_self, grd, dim3(256), 0, s, hs);
            IGG_HIP(hipGetLastError());
        }
    }
    return IGG_OK;
}

}  // namespace igg
