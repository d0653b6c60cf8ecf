// reduce.hip -- FP64 reductions over a field (maximum(Ci) of Fig. 1, loss,
// conservation and dot-product sums).  Values are widened to FP64 before
// they are combined; the field's vectors are dealt to a fixed number of threads
// and combined in a fixed tree, so a call's bits do not vary between runs.
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

// A field is walked in vectors of 16 bytes from its first point to its last,
// whatever its rows: a work-group takes chunks of U * RED_THREADS vectors, each
// thread one in U turns whose loads are in flight together.  load(u, p) reads
// the vector at offset p into slot u, use(u, p, m) takes it, where bit e of m
// says that point e is one of the region's (IN: the inner points; else every
// point); vectors without such a point are not read.  point(p) takes the points
// after the last whole vector, which lie in a halo plane.  The order in which
// points meet depends on the field's size and the launch only.
//
// Whole rows for each wave instead left waves idle where rows are few, lanes
// where they are short, and stored to as many places as there were waves: 20000
// x 20 x 20 FP64 maximum 69 us against 15, 13 x 500 x 700 42 against 10, seed
// without a loss 512^3 FP64 767 against 590, 256^3 80 against 74.
struct RedRegion {
    int nx, ny, nz;
    int64_t nv;      // whole vectors
    int tail;        // points after them
    int ui, uj, uk;  // points, rows and planes from a thread's vector to its next in the turn
    int di, dj, dk;  // and from its last in a turn to the first in the next
};
// The inner points of the vector at (i, j, k), without a branch: lo of them in
// its own row, hi in the next (a vector ends no later than the row after its
// own, which is never a row of the next plane's inside).
template <int VEC>
__device__ __forceinline__ uint32_t red_inner(const RedRegion &g, int i, int j, int k)
{
    constexpr uint32_t all = (1u << VEC) - 1;
    const bool ks = k > 0 && k < g.nz - 1;
    if (g.nx < VEC) {  // several rows
        uint32_t m = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (i > 0 && i < g.nx - 1 && j > 0 && j < g.ny - 1 && k > 0 && k < g.nz - 1) m |= 1u << e;
            if (++i == g.nx) {
                i = 0;
                if (++j == g.ny) {
                    j = 0;
                    ++k;
                }
            }
        }
        return m;
    }
    const int left = min(g.nx - i, VEC + 1);  // points to the row's end
    const uint32_t lo = ((1u << (left - 1)) - 1) & ~(i == 0 ? 1u : 0u), hi = all & ~((2u << left) - 1);
    return (ks && j > 0 && j < g.ny - 1 ? lo : 0) | (ks && j < g.ny - 2 ? hi : 0);
}
template <int VEC, int U, int IN, typename Load, typename Use, typename Point>
__device__ __forceinline__ void red_walk(const RedRegion &g, Load &&load, Use &&use, Point &&point)
{
    // a work-group takes U * RED_THREADS vectors in a row, its threads one each
    // in turn
    int64_t v = (int64_t)blockIdx.x * (U * RED_THREADS) + threadIdx.x;
    int i = 0, j = 0, k = 0;
    if (IN) {
        const int64_t row = v * VEC / g.nx;
        i = (int)(v * VEC - row * g.nx);
        k = (int)(row / g.ny);
        j = (int)(row - (int64_t)k * g.ny);
    }
    auto on = [&](int di, int dj, int dk) {
        i += di;
        j += dj;
        k += dk;
        if (i >= g.nx) {
            i -= g.nx;
            ++j;
        }
        if (j >= g.ny) {
            j -= g.ny;
            ++k;
        }
    };
    for (; v < g.nv; v += (int64_t)gridDim.x * (U * RED_THREADS)) {
        uint32_t m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            m[u] = IN ? red_inner<VEC>(g, i, j, k) : (1u << VEC) - 1;
            if (v + u * RED_THREADS >= g.nv) m[u] = 0;
            if (IN) on(g.ui, g.uj, g.uk);
        }
        if (IN) on(g.di, g.dj, g.dk);
        // vectors without a point of the region are read as the first again and
        // not used: a branch around each load made the compiler wait for the
        // one before
#pragma unroll
        for (int u = 0; u < U; ++u) load(u, (m[u] ? v + u * RED_THREADS : v) * VEC);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v + u * RED_THREADS < g.nv) use(u, (v + u * RED_THREADS) * VEC, m[u]);
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < g.tail) point(g.nv * VEC + threadIdx.x);
}

template <typename S> struct RedVec {
    static constexpr int N = 16 / (int)sizeof(S);
    typedef S type __attribute__((ext_vector_type(N)));
    typedef S mem __attribute__((ext_vector_type(N), aligned(sizeof(S))));  // fields start at any element
};

// Vectors of one array, or of two, that a thread reads together.
constexpr int RED_TURNS1 = 8, RED_TURNS2 = 4;

constexpr bool red_two(int op)
{
    return op == IGG_RED_SUM_RATIO || op == IGG_RED_HALF_SQDIFF || op == IGG_RED_DOT || op == IGG_RED_MAX_ABS_DIFF;
}
constexpr int red_turns(int op) { return red_two(op) ? RED_TURNS2 : RED_TURNS1; }

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
// branch per point cost as much as the loads.  256 x 250 x 241 FP64: maximum 24
// us, sum 24 (123 MB), dot product 43 (247 MB); 512^3: maximum 187 us (5.7
// TB/s), dot product 350 (6.1 TB/s).
template <typename S, int OP>
__global__ void __launch_bounds__(RED_THREADS)
k_reduce(const S *__restrict__ a, const S *__restrict__ b, RedRegion g, double *__restrict__ part)
{
    using R = RedVec<S>;
    constexpr bool TWO = red_two(OP);
    constexpr int TURNS = red_turns(OP), IN = OP != IGG_RED_MAX && OP != IGG_RED_MIN;
    __shared__ double sh[RED_THREADS];
    double acc[R::N];  // one per element of a vector
#pragma unroll
    for (int e = 0; e < R::N; ++e) acc[e] = identity(OP);
    typename R::type va[TURNS], vb[TURNS];
    red_walk<R::N, TURNS, IN>(
        g,
        [&](int u, int64_t p) {
            va[u] = *reinterpret_cast<const typename R::mem *>(a + p);
            if (TWO) vb[u] = *reinterpret_cast<const typename R::mem *>(b + p);
        },
        [&](int u, int64_t, uint32_t m) {
#pragma unroll
            for (int e = 0; e < R::N; ++e) {
                const double v = combine(OP, acc[e], term<S>(OP, va[u][e], TWO ? vb[u][e] : S(0)));
                acc[e] = !IN || (m >> e & 1) ? v : acc[e];
            }
        },
        [&](int64_t p) {
            if (!IN) acc[0] = combine(OP, acc[0], term<S>(OP, a[p], S(0)));
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

// The walk of a field of vectors of vec points, and its launch.
static RedRegion red_region(const igg_field &a, int vec, int turns, int &blocks)
{
    RedRegion g{};
    g.nx = (int)a.size[0];
    g.ny = (int)a.size[1];
    g.nz = (int)a.size[2];
    g.nv = field_elems(a) / vec;
    g.tail = (int)(field_elems(a) % vec);
    const int64_t want = (g.nv + RED_THREADS * turns - 1) / (RED_THREADS * turns);
    blocks = (int)(want < RED_BLOCKS ? want : RED_BLOCKS);
    auto steps = [&](int64_t points, int &i, int &j, int &k) {
        i = (int)(points % g.nx);
        j = (int)(points / g.nx % g.ny);
        k = (int)(points / g.nx / g.ny);
    };
    steps((int64_t)RED_THREADS * vec, g.ui, g.uj, g.uk);
    steps((int64_t)(blocks - 1) * RED_THREADS * turns * vec, g.di, g.dj, g.dk);
    return g;
}

// Partial results of `blocks` work-groups (at most RED_BLOCKS) into part.
template <typename S>
static int launch_part(int op, const igg_field &a, const igg_field *b, double *part, int part_cap, int *blocks,
                       hipStream_t s)
{
    const RedRegion g = red_region(a, RedVec<S>::N, red_turns(op), *blocks);
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
// ended when all have arrived, and waiting for the stream too takes 9 us longer
// (halo update, time step and sum of 256 x 250 x 241 FP64: 87 us against 104;
// 136 watching with hipStreamQuery).  A slot still holding its mark by then (a long queue, an
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
// on every halo point, each vector stored whole; with part, the partial sums of
// 0.5*(a-b)^2.  The field is walked exactly as k_reduce walks it for
// IGG_RED_HALF_SQDIFF, so the loss has the bits of that reduction.
template <typename S>
__global__ void __launch_bounds__(RED_THREADS)
k_seed(const S *__restrict__ a, const S *__restrict__ b, S *__restrict__ lam, RedRegion g, double *__restrict__ part)
{
    using C = compute_t<S>;
    using R = RedVec<S>;
    __shared__ double sh[RED_THREADS];
    double acc[R::N] = {};
    typename R::type va[RED_TURNS2], vb[RED_TURNS2];
    red_walk<R::N, RED_TURNS2, 1>(
        g,
        [&](int u, int64_t p) {
            if (!a) return;
            va[u] = *reinterpret_cast<const typename R::mem *>(a + p);
            if (b) vb[u] = *reinterpret_cast<const typename R::mem *>(b + p);
        },
        [&](int u, int64_t p, uint32_t m) {
            typename R::type v{};
#pragma unroll
            for (int e = 0; e < R::N; ++e) {
                const bool in = m >> e & 1;
                if (a && b) {
                    v[e] = in ? (S)((C)va[u][e] - (C)vb[u][e]) : S(0);
                    const double d = (double)(C)va[u][e] - (double)(C)vb[u][e];
                    acc[e] = in ? acc[e] + 0.5 * (d * d) : acc[e];
                } else if (a) {
                    v[e] = in ? va[u][e] : S(0);
                }
            }
            *reinterpret_cast<typename R::mem *>(lam + p) = v;
        },
        [&](int64_t p) { lam[p] = S(0); });
    if (part) {
        double v = block_combine(IGG_RED_HALF_SQDIFF, red_lanes<R::N>(IGG_RED_HALF_SQDIFF, acc), sh);
        if (threadIdx.x == 0) part[blockIdx.x] = v;
    }
}

template <typename S>
static int seed_typed(const igg_field *a, const igg_field *b, const igg_field &lam, double *part, int *blocks,
                      hipStream_t s)
{
    const RedRegion g = red_region(lam, RedVec<S>::N, RED_TURNS2, *blocks);
    hipLaunchKernelGGL(k_seed<S>, dim3(*blocks), dim3(RED_THREADS), 0, s, a ? (const S *)a->data : nullptr,
                       b ? (const S *)b->data : nullptr, (S *)lam.data, g, part);
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
