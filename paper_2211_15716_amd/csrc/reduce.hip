// reduce.hip -- FP64 reductions over a field (maximum(Ci) of Fig. 1, loss,
// conservation and dot-product sums).  Values are widened to FP64 before
// they are combined; rows are dealt to a fixed number of waves and combined
// in a fixed tree, so a call's bits do not vary between runs.
#include <string.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <string>
#include <type_traits>

#include "host.hpp"

namespace igg {

constexpr int RED_THREADS = 256;
constexpr int RED_BLOCKS = 1024;

__host__ __device__ __forceinline__ double combine(int op, double x, double y)
{
    if (op == IGG_RED_MIN) return (x < y || x != x) ? x : y;
    if (op == IGG_RED_MAX || op == IGG_RED_MAX_ABS_DIFF || op == IGG_RED_MAX_ABS)
        return (x > y || x != x) ? x : y;
    return x + y;
}

__host__ __device__ __forceinline__ double identity(int op)
{
    if (op == IGG_RED_MIN) return __builtin_inf();
    if (op == IGG_RED_MAX || op == IGG_RED_MAX_ABS_DIFF || op == IGG_RED_MAX_ABS) return -__builtin_inf();
    return 0.0;
}

template <typename S>
__device__ __forceinline__ double term(int op, S a, S b)
{
    const double x = (double)(compute_t<S>)a, y = (double)(compute_t<S>)b;
    switch (op) {
    case IGG_RED_SUM_RATIO: return x / y;
    case IGG_RED_HALF_SQDIFF: { double d = x - y; return 0.5 * (d * d); }
    case IGG_RED_DOT: return x * y;
    case IGG_RED_MAX_ABS_DIFF: return __builtin_fabs(x - y);
    case IGG_RED_MAX_ABS: return __builtin_fabs(x);
    default: return x;
    }
}

__device__ __forceinline__ double block_combine(int op, double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = RED_THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] = combine(op, sh[threadIdx.x], sh[threadIdx.x + w]);
        __syncthreads();
    }
    return sh[0];
}

// The rows (j, k) of a region of h x depth rows and nx points per row, i0 to
// i1 of each, dealt to the waves of the launch in turn (ROWS at a time, so
// that their loads are in flight together) and walked in vectors of 16 bytes:
// load(q, p, n) reads the n points at offset p into slot q, use(q, p, n, skip)
// takes them but for the first `skip`, in an order that depends on the region
// and the launch only.  n is VEC (the vector at the end of a row begins before
// it would, and skips what the one before it took), or 1 in rows shorter than
// that.  (Points read one by one at the end of a row cost a load's latency each:
// 61 x 152 x 288 FP32 sum 15.0 us against 12.1, 301 x 257 x 203 20.7 against
// 17.1.)
struct RedRegion {
    int nx, ny, i0, i1, j0, k0, h;
    int64_t rows;
    int dj, dk;  // rows and planes from one of a wave's rows to its next
};
template <int VEC, int ROWS, typename Load, typename Use>
__device__ __forceinline__ void red_walk(const RedRegion &g, Load &&load, Use &&use)
{
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (RED_THREADS / 64);
    const int first = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (RED_THREADS / 64) + (threadIdx.x >> 6)));
    int j = first % g.h, k = first / g.h;
    for (int64_t r = first; r < g.rows; r += ROWS * waves) {
        int64_t base[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
            base[q] = ((int64_t)(g.k0 + k) * g.ny + g.j0 + j) * g.nx;
            j += g.dj;
            k += g.dk;
            if (j >= g.h) {
                j -= g.h;
                ++k;
            }
        }
        // the rows past the last are read as the first again and not used: a
        // branch around each load made the compiler wait for the one before
        const int nr = r + (ROWS - 1) * waves < g.rows ? ROWS : (int)((g.rows - r + waves - 1) / waves);
#pragma unroll
        for (int q = 1; q < ROWS; ++q)
            if (q >= nr) base[q] = base[0];
        auto points = [&](int64_t i, auto n, int skip) {
#pragma unroll
            for (int q = 0; q < ROWS; ++q) load(q, base[q] + i, n);
            if (skip == 0) {
#pragma unroll
                for (int q = 0; q < ROWS; ++q)
                    if (q < nr) use(q, base[q] + i, n, 0);
            } else {
#pragma unroll
                for (int q = 0; q < ROWS; ++q)
                    if (q < nr) use(q, base[q] + i, n, skip);
            }
        };
        if (g.i1 - g.i0 >= VEC) {
            for (int i = g.i0 + lane * VEC; i < g.i1; i += 64 * VEC) {
                const int at = min(i, g.i1 - VEC);
                points(at, std::integral_constant<int, VEC>(), i - at);
            }
        } else if (lane < g.i1 - g.i0) {
            points(g.i0 + lane, std::integral_constant<int, 1>(), 0);
        }
    }
}

template <typename S> struct RedVec {
    static constexpr int N = 16 / (int)sizeof(S);
    typedef S type __attribute__((ext_vector_type(N)));
    typedef S mem __attribute__((ext_vector_type(N), aligned(sizeof(S))));  // rows start at any element
};

// Rows of one array, or of two, that a wave reads together.
constexpr int RED_ROWS1 = 8, RED_ROWS2 = 4;

// A thread's accumulators into one.
template <int N>
__device__ __forceinline__ double red_lanes(int op, const double (&acc)[N])
{
    double v = acc[0];
#pragma unroll
    for (int e = 1; e < N; ++e) v = combine(op, v, acc[e]);
    return v;
}

// Bound by the loads it has in flight (8 KB of one array or of two per wave)
// and the ramp of a launch; the operation is a template argument because a
// branch per point cost as much as the loads.  256 x 250 x 241 FP64: maximum
// 56 -> 31 us, sum 53 -> 29 (123 MB), dot product 59 -> 43 (247 MB); 512^3:
// maximum 363 -> 202 us (5.3 TB/s), dot product 423 -> 367 (5.9 TB/s), against
// one row per work-group and one point per lane.  Loads without a branch: 301 x
// 257 x 203 FP64 maximum 39 -> 31 us, 512^3 218 -> 202.
template <typename S, int OP>
__global__ void __launch_bounds__(RED_THREADS)
k_reduce(const S *__restrict__ a, const S *__restrict__ b, RedRegion g, double *__restrict__ part)
{
    using R = RedVec<S>;
    constexpr bool TWO = OP == IGG_RED_SUM_RATIO || OP == IGG_RED_HALF_SQDIFF || OP == IGG_RED_DOT ||
                         OP == IGG_RED_MAX_ABS_DIFF;
    constexpr int ROWS = TWO ? RED_ROWS2 : RED_ROWS1;
    __shared__ double sh[RED_THREADS];
    double acc[R::N];  // one per element of a vector
#pragma unroll
    for (int e = 0; e < R::N; ++e) acc[e] = identity(OP);
    typename R::type va[ROWS], vb[ROWS];
    red_walk<R::N, ROWS>(
        g,
        [&](int q, int64_t p, auto n) {
            if constexpr (n.value > 1) {
                va[q] = *reinterpret_cast<const typename R::mem *>(a + p);
                if (TWO) vb[q] = *reinterpret_cast<const typename R::mem *>(b + p);
            } else {
                va[q][0] = a[p];
                if (TWO) vb[q][0] = b[p];
            }
        },
        [&](int q, int64_t, auto n, int skip) {
#pragma unroll
            for (int e = 0; e < n.value; ++e)
                if (e >= skip) acc[e] = combine(OP, acc[e], term<S>(OP, va[q][e], TWO ? vb[q][e] : S(0)));
        });
    double v = block_combine(OP, red_lanes<R::N>(OP, acc), sh);
    // (the host may be waiting for it)
    if (threadIdx.x == 0) __hip_atomic_store(part + blockIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Combines the n partial results in `part` and writes the value to *result.
__global__ void __launch_bounds__(RED_THREADS)
k_reduce_final(int op, int n, const double *__restrict__ part, double *__restrict__ result)
{
    __shared__ double sh[RED_THREADS];
    double acc = identity(op);
    for (int q = threadIdx.x; q < n; q += RED_THREADS) acc = combine(op, acc, part[q]);
    double v = block_combine(op, acc, sh);
    if (threadIdx.x == 0) *result = v;
}

static RedRegion red_region(const igg_field &a, bool all, int &blocks)
{
    RedRegion g{};
    const int nx = (int)a.size[0], ny = (int)a.size[1], nz = (int)a.size[2], in = all ? 0 : 1;
    g.nx = nx;
    g.ny = ny;
    g.i0 = g.j0 = g.k0 = in;
    g.i1 = nx - in;
    g.h = ny - 2 * in;
    g.rows = (int64_t)g.h * (nz - 2 * in);
    const int64_t want = (g.rows + RED_THREADS / 64 - 1) / (RED_THREADS / 64);
    blocks = (int)(want < RED_BLOCKS ? (want < 1 ? 1 : want) : RED_BLOCKS);
    const int64_t waves = (int64_t)blocks * (RED_THREADS / 64);
    g.dj = (int)(waves % g.h);
    g.dk = (int)(waves / g.h);
    return g;
}

// Partial results of `blocks` work-groups (at most RED_BLOCKS) into part.
template <typename S>
static int launch_part(int op, const igg_field &a, const igg_field *b, double *part, int part_cap, int *blocks,
                       hipStream_t s)
{
    const RedRegion g = red_region(a, op == IGG_RED_MAX || op == IGG_RED_MIN, *blocks);
    if (*blocks > part_cap)
        return fail(IGG_ERR_SIZE, "reduction needs " + std::to_string(*blocks) + " partial results, the buffer holds " +
                                      std::to_string(part_cap));
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(*blocks), dim3(RED_THREADS), 0, s, (const S *)a.data,
                           b ? (const S *)b->data : (const S *)nullptr, g, part);
    };
    switch (op) {
    case IGG_RED_MAX: go(k_reduce<S, IGG_RED_MAX>); break;
    case IGG_RED_MIN: go(k_reduce<S, IGG_RED_MIN>); break;
    case IGG_RED_SUM: go(k_reduce<S, IGG_RED_SUM>); break;
    case IGG_RED_SUM_RATIO: go(k_reduce<S, IGG_RED_SUM_RATIO>); break;
    case IGG_RED_HALF_SQDIFF: go(k_reduce<S, IGG_RED_HALF_SQDIFF>); break;
    case IGG_RED_DOT: go(k_reduce<S, IGG_RED_DOT>); break;
    case IGG_RED_MAX_ABS_DIFF: go(k_reduce<S, IGG_RED_MAX_ABS_DIFF>); break;
    case IGG_RED_MAX_ABS: go(k_reduce<S, IGG_RED_MAX_ABS>); break;
    default: return fail(IGG_ERR_ARG, "unknown reduction");
    }
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

static int launch_typed(int op, const igg_field &a, const igg_field *b, double *part, int part_cap, int *blocks,
                        hipStream_t s)
{
    if (b && b->dtype != a.dtype) return fail(IGG_ERR_DTYPE, "a and b must share one dtype");
    if (a.dtype == IGG_F64) return launch_part<double>(op, a, b, part, part_cap, blocks, s);
    if (a.dtype == IGG_F32) return launch_part<float>(op, a, b, part, part_cap, blocks, s);
    return launch_part<_Float16>(op, a, b, part, part_cap, blocks, s);
}

// k_reduce_final on the host, in the same order (the same bits).
static double combine_host(int op, int n, const double *part)
{
    double acc[RED_THREADS];
    for (int t = 0; t < RED_THREADS; ++t) {
        acc[t] = identity(op);
        for (int q = t; q < n; q += RED_THREADS) acc[t] = combine(op, acc[t], part[q]);
    }
    for (int w = RED_THREADS / 2; w > 0; w >>= 1)
        for (int t = 0; t < w; ++t) acc[t] = combine(op, acc[t], acc[t + w]);
    return acc[0];
}

// Pinned memory for the partial results of one call that returns them to the
// host.  Calls that overlap in time (from several host threads) each have
// their own; those not in use wait in the grid's list, which so holds as many
// as there were such calls at once.
static std::mutex g_red_mu;

int RedSlots::acquire()
{
    Grid &g = grid();
    {
        std::lock_guard<std::mutex> lock(g_red_mu);
        if (!g.red_free.empty()) {
            part = g.red_free.back();
            g.red_free.pop_back();
            return IGG_OK;
        }
    }
    IGG_HIP(hipHostMalloc((void **)&part, RED_BLOCKS * sizeof(double), hipHostMallocDefault));
    return IGG_OK;
}
RedSlots::~RedSlots()
{
    if (!part) return;
    std::lock_guard<std::mutex> lock(g_red_mu);
    grid().red_free.push_back(part);
}

// The work-groups write their partial results straight to pinned host memory
// (8 KB) and the host combines them: no second launch and no copy.  The host
// watches for them itself for up to 2 ms: the stream's work before them has
// ended when all have arrived, and a wait for the stream takes about 10 us
// longer to return.  A slot still holding its mark by then (a long queue, an
// error, or a field that holds that very NaN) is left to a wait for the stream.
constexpr uint64_t kRedMark = 0x7ff8c0de5eed0001ull;
static int wait_parts(const double *part, int n, hipStream_t s)
{
    const volatile uint64_t *p = reinterpret_cast<const volatile uint64_t *>(part);
    const auto end = std::chrono::steady_clock::now() + std::chrono::milliseconds(2);
    for (int q = 0; q < n; ++q)
        for (int spin = 0; p[q] == kRedMark; ++spin)
            if ((spin & 63) == 63 && std::chrono::steady_clock::now() > end) {
                IGG_HIP(hipStreamSynchronize(s));
                return IGG_OK;
            }
    std::atomic_thread_fence(std::memory_order_acquire);
    return IGG_OK;
}
static void mark_parts(double *part)
{
    for (int q = 0; q < RED_BLOCKS; ++q) memcpy(part + q, &kRedMark, sizeof kRedMark);
    std::atomic_thread_fence(std::memory_order_release);
}

int launch_reduce(int op, const igg_field &a, const igg_field *b, double *out, hipStream_t s)
{
    RedSlots slots;
    int rc, blocks = 0;
    if ((rc = slots.acquire())) return rc;
    mark_parts(slots.part);
    if ((rc = launch_typed(op, a, b, slots.part, RED_BLOCKS, &blocks, s))) return rc;
    if ((rc = wait_parts(slots.part, blocks, s))) return rc;
    *out = combine_host(op, blocks, slots.part);
    return IGG_OK;
}

// ------------------------------------------------------- adjoint seed
// lam = a - b on the inner points (a alone without b, zero without a), zero
// on every halo point; with want_loss, the partial sums of 0.5*(a-b)^2.  The
// inner rows are walked exactly as k_reduce walks them for
// IGG_RED_HALF_SQDIFF, so the loss has the bits of that reduction.  The halo
// rows and columns are zeroed in a second walk.
template <typename S>
__global__ void __launch_bounds__(RED_THREADS)
k_seed(const S *__restrict__ a, const S *__restrict__ b, S *__restrict__ lam, int nz, RedRegion g,
       double *__restrict__ part)
{
    using C = compute_t<S>;
    using R = RedVec<S>;
    __shared__ double sh[RED_THREADS];
    double acc[R::N] = {};
    const int nx = g.nx, ny = g.ny;
    typename R::type va[RED_ROWS2], vb[RED_ROWS2];
    red_walk<R::N, RED_ROWS2>(
        g,
        [&](int q, int64_t p, auto n) {
            if (!a) return;
            if constexpr (n.value > 1) {
                va[q] = *reinterpret_cast<const typename R::mem *>(a + p);
                if (b) vb[q] = *reinterpret_cast<const typename R::mem *>(b + p);
            } else {
                va[q][0] = a[p];
                if (b) vb[q][0] = b[p];
            }
        },
        [&](int q, int64_t p, auto n, int skip) {
            typename R::type v{};
#pragma unroll
            for (int e = 0; e < n.value; ++e) {
                if (a && b) {
                    v[e] = (S)((C)va[q][e] - (C)vb[q][e]);
                    const double d = (double)(C)va[q][e] - (double)(C)vb[q][e];
                    if (e >= skip) acc[e] += 0.5 * (d * d);
                } else if (a) {
                    v[e] = va[q][e];
                }
            }
            if constexpr (n.value > 1) *reinterpret_cast<typename R::mem *>(lam + p) = v;
            else lam[p] = v[0];
        });
    const int64_t t = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x, nt = (int64_t)gridDim.x * RED_THREADS;
    // halo columns of the inner rows
    for (int64_t r = t; r < g.rows; r += nt) {
        const int64_t base = ((1 + r / g.h) * ny + 1 + r % g.h) * nx;
        lam[base] = S(0);
        lam[base + nx - 1] = S(0);
    }
    // halo rows: j = 0 and ny-1 of every plane, then every row of planes 0 and nz-1
    const int64_t hrows = 2 * (int64_t)nz + 2 * (int64_t)(ny - 2);
    for (int64_t r = blockIdx.x; r < hrows; r += gridDim.x) {
        int j, k;
        if (r < 2 * (int64_t)nz) {
            j = (r & 1) ? ny - 1 : 0;
            k = (int)(r >> 1);
        } else {
            const int64_t q = r - 2 * (int64_t)nz;
            j = 1 + (int)(q >> 1);
            k = (q & 1) ? nz - 1 : 0;
        }
        const int64_t base = (int64_t)k * nx * ny + (int64_t)j * nx;
        for (int i = threadIdx.x; i < nx; i += RED_THREADS) lam[base + i] = S(0);
    }
    if (part) {
        double v = block_combine(IGG_RED_HALF_SQDIFF, red_lanes<R::N>(IGG_RED_HALF_SQDIFF, acc), sh);
        if (threadIdx.x == 0) part[blockIdx.x] = v;
    }
}

template <typename S>
static int seed_typed(const igg_field *a, const igg_field *b, const igg_field &lam, double *part, int *blocks,
                      hipStream_t s)
{
    const RedRegion g = red_region(lam, false, *blocks);
    hipLaunchKernelGGL(k_seed<S>, dim3(*blocks), dim3(RED_THREADS), 0, s, a ? (const S *)a->data : nullptr,
                       b ? (const S *)b->data : nullptr, (S *)lam.data, (int)lam.size[2], g, part);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

int launch_seed(const igg_field *a, const igg_field *b, const igg_field &lam, RedSlots *loss, hipStream_t s)
{
    int rc, blocks = 0;
    if (loss && (rc = loss->acquire())) return rc;
    double *part = loss ? loss->part : nullptr;
    rc = lam.dtype == IGG_F64   ? seed_typed<double>(a, b, lam, part, &blocks, s)
                   : lam.dtype == IGG_F32 ? seed_typed<float>(a, b, lam, part, &blocks, s)
                                          : seed_typed<_Float16>(a, b, lam, part, &blocks, s);
    if (loss) loss->n = blocks;
    return rc;
}

int read_seed_loss(const RedSlots &loss, double *out, hipStream_t s)
{
    IGG_HIP(hipStreamSynchronize(s));
    *out = combine_host(IGG_RED_HALF_SQDIFF, loss.n, loss.part);
    return IGG_OK;
}

// ----------------------------------------------------- without allocation
// Partial results of igg_reduce_noalloc: one array of 1024 doubles (8 KiB)
// per device, held until the process ends.  Every call writes the partial
// results it reads before reading them (same stream), so nothing needs
// clearing; calls that overlap in time on one device share the array and
// race.  Host code never uses its name as an address (on the host it is
// only a stand-in); it takes the device address that hipGetSymbolAddress
// returns for the current device, once per device.
constexpr int kNoallocScratch = 1024;
static __device__ __align__(256) double scratch[kNoallocScratch];

static std::mutex g_scratch_mu;
static double *g_scratch_ptr[IGG_MAX_DEVICES];

// The device address of `scratch` on the current device (looked up on the
// first call on that device).
static int scratch_on_current_device(double **ptr)
{
    int dev = -1;
    IGG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= IGG_MAX_DEVICES)
        return fail(IGG_ERR_ARG, "device index " + std::to_string(dev) + " above the library's limit");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        IGG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(IGG_ERR_HIP, "hipGetSymbolAddress returned a null address for the reduction scratch");
        g_scratch_ptr[dev] = (double *)p;
    }
    *ptr = g_scratch_ptr[dev];
    return IGG_OK;
}

int launch_reduce_noalloc(int op, const igg_field &a, const igg_field *b, double *out_dev, hipStream_t s)
{
    double *part = nullptr;
    int rc, blocks = 0;
    if ((rc = scratch_on_current_device(&part))) return rc;
    if ((rc = launch_typed(op, a, b, part, kNoallocScratch, &blocks, s))) return rc;
    hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(RED_THREADS), 0, s, op, blocks, (const double *)part, out_dev);
    IGG_HIP(hipGetLastError());
    return IGG_OK;
}

}  // namespace igg
