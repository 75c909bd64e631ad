// observables.hip -- ensemble averages of per-path / per-oscillator arrays
// (the quantities of interest of Sec. 4: averages over realizations, the
// asymptotic velocity of Sec. 5, the Kuramoto order parameter).
//
// A group is reduced in slices of at most kObsThreads * kObsItems elements,
// one workgroup each, that are read once: the workgroup holds its slice in
// registers (FP64), sums it, and takes the spread about the slice's own mean
// from the registers (no cancellation from sum of squares minus squared
// sum).  A second kernel combines a group's slices in a fixed order: the
// mean from the sums, and about it
//   sum (x - mean)^2 = sum_s [ M2_s + n_s (mean_s - mean)^2 ].
// Where no group needs more than one slice, or there are groups enough to fill
// the chip, a workgroup takes a whole group instead.  All sums run
// in a fixed order (elements by thread, wavefront butterfly, waves, slices),
// so results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "sde_internal.h"

namespace sde {

constexpr int kObsThreads = 256;

template <int THREADS>
__device__ double block_sum(double x, double* lds)
{
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    x = wave_sum(x);
    if constexpr (THREADS == kWave) return x;
    if (lane == 0) lds[wid] = x;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < THREADS / kWave; ++w) t += lds[w];
    __syncthreads();
    return t;
}

// Elements per lane of a slice.  One workgroup per group and two passes over
// it (the earlier kernel) read a single group of 2^19 values with one CU:
// 580-930 us; in slices of 1024-4096 the same call takes 24 us, its launches
// and the final synchronization.
constexpr uint32_t kObsItems = 16;
// The most that a workgroup with a group of its own holds.
constexpr uint32_t kObsGroupItems = 32;
// Workgroups in a grid's x; past them y counts on (their threads would not fit
// 32 bits).
constexpr uint32_t kObsGrid = 1u << 20;

static dim3 obs_grid(uint32_t n) { return dim3(std::min(n, kObsGrid), (n + kObsGrid - 1) / kObsGrid); }
__device__ __forceinline__ uint32_t obs_block() { return blockIdx.y * kObsGrid + blockIdx.x; }

struct ObsArgs {
    const void* in;
    const uint64_t* first;         // [n_groups] first element of the group
    const uint32_t* counts;        // [n_groups]
    const uint32_t* slice_begin;   // [n_groups + 1] slices before the group
    double* part;                  // [slices][2]: (sum, M2 about the slice's mean), or (sum cos, sum sin)
    double* out;                   // [n_groups][2]
    uint32_t n_groups, n_slices;
    uint32_t slice;                // elements per slice, at most kObsThreads * kObsItems
};

// The two sums (every thread has them) of n <= ITEMS * THREADS elements:
// (sum, M2 about its mean); of any number of them for the order parameter:
// (sum cos, sum sin) in FP64.
template <int KIND, int ITEMS, int THREADS = kObsThreads>
__device__ __forceinline__ void obs_slice(const void* in, uint64_t base, uint32_t n, double* lds, double& a, double& b)
{
    using T = typename std::conditional<KIND == SDE_OBS_MEAN_F64, double, float>::type;
    const T* p = static_cast<const T*>(in) + base;
    a = 0.0;
    b = 0.0;
    if constexpr (KIND == SDE_OBS_ORDER) {
        auto add = [&](T x) {
            double sn, cs;
            sincospi(2.0 * (double)x, &sn, &cs);
            a += cs;
            b += sn;
        };
        // a thread's elements in order, four loads in flight
        uint64_t i = threadIdx.x;
        for (; i + 3 * THREADS < n; i += 4 * THREADS) {
            T raw[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) raw[k] = p[i + k * THREADS];
#pragma unroll
            for (int k = 0; k < 4; ++k) add(raw[k]);
        }
        for (; i < n; i += THREADS) add(p[i]);
        a = block_sum<THREADS>(a, lds);
        b = block_sum<THREADS>(b, lds);
    } else {
        if (n == 0) return;
        // no condition on the loads, so that all of them are in flight (past the
        // end the last element again)
        T raw[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) raw[k] = p[min((uint32_t)(k * THREADS) + threadIdx.x, n - 1)];
        double x[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            x[k] = (uint32_t)(k * THREADS) + threadIdx.x < n ? (double)raw[k] : 0.0;
            if (KIND == SDE_OBS_MEANSQ_F32) x[k] *= x[k];
            a += x[k];  // lanes past the end hold zero
        }
        a = block_sum<THREADS>(a, lds);
        const double mean = a / (double)n;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const double d = (uint32_t)(k * THREADS) + threadIdx.x < n ? x[k] - mean : 0.0;
            b += d * d;
        }
        b = block_sum<THREADS>(b, lds);
    }
}

__device__ __forceinline__ void obs_finish(int kind, uint32_t n, double a, double b, double* out)
{
    double2 r;
    if (kind == SDE_OBS_ORDER) {
        const double inv = n ? 1.0 / (double)n : 0.0;
        r.x = std::sqrt(a * a + b * b) * inv;
        r.y = n ? atan2(b, a) / (2.0 * M_PI) : 0.0;
    } else {
        r.x = n ? a / (double)n : 0.0;
        r.y = n > 1 ? std::sqrt(b / (double)(n - 1) / (double)n) : 0.0;
    }
    *reinterpret_cast<double2*>(out) = r;  // one store over the bus
}

// One workgroup per group, of one wave for groups of up to 256 elements (16384
// groups of 100: 64 us with four, 50 so).
template <int KIND, int ITEMS, int THREADS>
__global__ __launch_bounds__(THREADS) void obs_group_kernel(ObsArgs A)
{
    __shared__ double lds[THREADS / kWave];
    const uint32_t g = obs_block();
    if (g >= A.n_groups) return;
    const uint32_t n = A.counts[g];
    double a, b;
    obs_slice<KIND, ITEMS, THREADS>(A.in, A.first[g], n, lds, a, b);
    if (threadIdx.x == 0) obs_finish(KIND, n, a, b, A.out + 2 * (uint64_t)g);
}

// One workgroup per slice; a group of one slice (or none) is finished here.
template <int KIND, int ITEMS>
__global__ __launch_bounds__(kObsThreads) void obs_slice_kernel(ObsArgs A)
{
    __shared__ double lds[kObsThreads / kWave];
    const uint32_t s = obs_block();
    if (s >= A.n_slices) return;
    // the group of this slice: the last one whose slices begin at or before it
    uint32_t lo = 0, hi = A.n_groups;
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (A.slice_begin[mid] <= s)
            lo = mid;
        else
            hi = mid;
    }
    const uint32_t sl = s - A.slice_begin[lo], n = A.counts[lo];
    const uint64_t off = (uint64_t)sl * A.slice;
    const uint32_t cnt = (uint32_t)min((uint64_t)A.slice, (uint64_t)n - off);
    double a, b;
    obs_slice<KIND, ITEMS>(A.in, A.first[lo] + off, cnt, lds, a, b);
    if (threadIdx.x) return;
    if (n <= A.slice)
        obs_finish(KIND, n, a, b, A.out + 2 * (uint64_t)lo);
    else {
        A.part[2 * (uint64_t)s] = a;
        A.part[2 * (uint64_t)s + 1] = b;
    }
}

// One workgroup per group of more than one slice: its slices, in order.
__global__ __launch_bounds__(kObsThreads) void obs_combine_kernel(ObsArgs A, int kind)
{
    __shared__ double lds[kObsThreads / kWave];
    const uint32_t g = obs_block();
    if (g >= A.n_groups) return;
    const uint32_t n = A.counts[g];
    if (n <= A.slice) return;
    const uint32_t s0 = A.slice_begin[g], ns = A.slice_begin[g + 1] - s0;
    const double* p = A.part + 2 * (uint64_t)s0;
    double a = 0.0, b = 0.0;
    for (uint32_t i = threadIdx.x; i < ns; i += kObsThreads) a += p[2 * (uint64_t)i];
    a = block_sum<kObsThreads>(a, lds);
    const double mean = a / (double)n;
    for (uint32_t i = threadIdx.x; i < ns; i += kObsThreads) {
        b += p[2 * (uint64_t)i + 1];
        if (kind != SDE_OBS_ORDER) {
            const double cnt = (double)min((uint64_t)A.slice, (uint64_t)n - (uint64_t)i * A.slice);
            const double m = p[2 * (uint64_t)i] / cnt;
            const double d = m == mean ? 0.0 : m - mean;  // equal infinities: the slice's own spread stands
            b += cnt * (d * d);
        }
    }
    b = block_sum<kObsThreads>(b, lds);
    if (threadIdx.x == 0) obs_finish(kind, n, a, b, A.out + 2 * (uint64_t)g);
}

// ---- histograms ------------------------------------------------------------
// Counting rows of 4-byte values into bins.  A workgroup counts its share of
// a row in LDS (32-bit; the grid keeps a share below 2^31) and adds its bins
// to the 64-bit totals; more bins than fit in LDS go straight to global
// 64-bit atomics.  Integer sums: the result does not depend on the order.
//
// What bounds it: an ensemble sits in a few bins, and atomics of one wave on
// one LDS word are taken one after the other.  So every bin has up to 32
// copies side by side (lane l adds to copy l mod 32, another bank); values
// come 16 bytes a lane, two loads in flight.  200 rows of 2^19 windings: 227 us
// (1.85 TB/s) with one copy and 4-byte loads, 75-79 us (5.3-5.6 TB/s) with
// these.  Of short rows the clearing and adding up of the bins is the work, so
// the copies stay within a sixteenth of the values that a workgroup counts
// (20000 rows of 1000 values, 500 bins: 32 us with one copy, 165 with 32; 2000
// rows of 20000, 10 bins: 33 with one, 27 with 8), and a workgroup has as many
// waves as it has work for (20000 rows of 100, 100 bins: 16 us with one wave,
// 39 with eight; 20000 of 1000, 8000 bins: 500 with one, 278 with eight).
constexpr uint32_t kHistThreads = 512;
constexpr uint32_t kHistWords = 16384;  // LDS words for bins and their copies
// Values far fewer than bins are counted in memory at once (rows of 10 values,
// 2000 bins: 299 us against 387 by way of LDS, 500 bins: 107 against 106).
constexpr uint64_t kHistSparse = 64;
// A share of at least this many values, so that few workgroups add to the
// same totals (one row of 2^19 phases: 24 us with 1024 of them, 6 with 64).
constexpr uint64_t kHistShare = 8192;

__global__ void hist_zero_kernel(uint64_t* counts, uint64_t n)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) counts[i] = 0ull;
}

struct HistArgs {
    const void* data;  // rows of n values, row pitch `pitch`
    uint64_t n, pitch, rows;
    int64_t x0;        // positions: first bin
    uint32_t nb;       // bins asked for
    uint32_t total;    // bins counted: with those for values outside
    int32_t log_copies;
    int32_t store;     // a row has one workgroup: its counts are stored, not added
    uint64_t* counts;  // [rows][total]
};

// Windings: one bin per potential period.  With x = theta + winding and theta
// in [0, 1), the bin of x is its winding count: bin 0 below x0, bin nb + 1
// from x0 + nb on.  x0 in the range of int32 (a saturated difference keeps
// the order), or any.
struct PositionBin {
    typedef int32_t Value;
    int32_t x0, nb;
    __device__ __forceinline__ explicit PositionBin(const HistArgs& A) : x0((int32_t)A.x0), nb((int32_t)A.nb) {}
    __device__ __forceinline__ uint32_t operator()(int32_t w) const
    {
        return (uint32_t)(min(max(__builtin_elementwise_sub_sat(w, x0), -1), nb) + 1);
    }
};
struct WidePositionBin {
    typedef int32_t Value;
    int64_t x0;
    uint32_t nb;
    __device__ __forceinline__ explicit WidePositionBin(const HistArgs& A) : x0(A.x0), nb(A.nb) {}
    __device__ __forceinline__ uint32_t operator()(int32_t w) const
    {
        const int64_t d = (int64_t)w - x0;
        return d < 0 ? 0u : d >= (int64_t)nb ? nb + 1 : (uint32_t)d + 1;
    }
};

// Phases in revolutions (the density P(x; t) of Fig. 4): bin b = floor(theta
// nb) for theta in [0, 1] (theta = 1 into the last bin), anything else
// (outside [0, 1], NaN) into bin nb.  theta nb is formed in FP64, exactly for
// nb < 2^29, so the bin is the exact floor.
struct PhaseBin {
    typedef float Value;
    uint32_t nb;
    double nbd;
    __device__ __forceinline__ explicit PhaseBin(const HistArgs& A) : nb(A.nb), nbd((double)A.nb) {}
    __device__ __forceinline__ uint32_t operator()(float t) const
    {
        return t >= 0.f && t <= 1.f ? min((uint32_t)((double)t * nbd), nb - 1) : nb;
    }
};

// Row r = blockIdx.y, blockIdx.y + gridDim.y, ...; the workgroups of a row
// take turns of 16-byte pieces of it.
template <typename Bin>
__global__ __launch_bounds__(kHistThreads) void hist_kernel(HistArgs A)
{
    typedef typename Bin::Value T;
    typedef T V4 __attribute__((ext_vector_type(4)));
    extern __shared__ uint32_t h[];  // [total][copies], or nothing
    const Bin bin(A);
    const int lc = A.log_copies;
    const bool lds = lc >= 0;
    const uint32_t copy = lds ? threadIdx.x & ((1u << lc) - 1u) : 0u;
    const uint32_t threads = blockDim.x;
    if (lds)
        for (uint32_t i = threadIdx.x; i < A.total << lc; i += threads) h[i] = 0u;
    for (uint64_t r = blockIdx.y; r < A.rows; r += gridDim.y) {
        const T* row = static_cast<const T*>(A.data) + r * A.pitch;
        uint64_t* cr = A.counts + r * (uint64_t)A.total;
        __syncthreads();
        auto count = [&](T x) {
            const uint32_t b = bin(x);
            if (lds)
                atomicAdd(&h[(b << lc) + copy], 1u);
            else
                atomicAdd(reinterpret_cast<unsigned long long*>(cr + b), 1ull);
        };
        // single values up to the first 16-byte boundary and after the last
        const uint64_t head = min(A.n, (uint64_t)((16u - ((uint32_t)(uintptr_t)row & 15u)) & 15u) / 4);
        const V4* body = reinterpret_cast<const V4*>(row + head);
        const uint64_t n4 = (A.n - head) / 4, tail = head + 4 * n4;
        if (blockIdx.x == 0) {
            if (threadIdx.x < head) count(row[threadIdx.x]);
            if (tail + threadIdx.x < A.n) count(row[tail + threadIdx.x]);
        }
        const uint64_t stride = (uint64_t)gridDim.x * threads;
        uint64_t i = (uint64_t)blockIdx.x * threads + threadIdx.x;
        for (; i + stride < n4; i += 2 * stride) {
            const V4 a = body[i], b = body[i + stride];
#pragma unroll
            for (int k = 0; k < 4; ++k) count(a[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) count(b[k]);
        }
        if (i < n4) {
            const V4 a = body[i];
#pragma unroll
            for (int k = 0; k < 4; ++k) count(a[k]);
        }
        __syncthreads();
        if (lds)
            for (uint32_t b = threadIdx.x; b < A.total; b += threads) {
                uint64_t sum = 0;  // and the bin is cleared for the next row
                const uint32_t turn = b >> (5 - lc);  // of 32 neighbouring bins no two on a bank
                for (uint32_t c = 0; c < 1u << lc; ++c) {
                    uint32_t* q = &h[(b << lc) + ((c + turn) & ((1u << lc) - 1u))];
                    sum += *q;
                    *q = 0u;
                }
                if (A.store)
                    cr[b] = sum;
                else if (sum)
                    atomicAdd(reinterpret_cast<unsigned long long*>(cr + b), (unsigned long long)sum);
            }
    }
}

static int launch_hist(sde_ctx* ctx, HistArgs A, void (*kern)(HistArgs), hipStream_t stream)
{
    const uint64_t nc = (uint64_t)A.total * A.rows;
    const uint64_t zb = (nc + 255) / 256;
    if (zb > 0x7fffffffull) return fail(ctx, SDE_ERR_INVALID, "too many counts");
    // about 4 workgroups per CU in all, at least one per row (up to 65535
    // rows in flight), shares of kHistShare to 2^31 values
    const uint64_t gy = std::min<uint64_t>(A.rows, 65535);
    uint64_t gx = std::max<uint64_t>(1, (uint64_t)ctx->n_cu * 4 / gy);
    gx = std::min<uint64_t>(gx, (A.n + kHistShare - 1) / kHistShare);
    gx = std::max<uint64_t>(gx, (A.n >> 31) + 1);
    const uint64_t share = (A.n + gx - 1) / gx;
    A.log_copies = -1;
    if (A.total <= kHistWords && A.total <= kHistSparse * share) {
        const uint64_t words = std::min<uint64_t>(kHistWords, share / 16);
        A.log_copies = 0;
        while (A.log_copies < 5 && ((uint64_t)A.total << (A.log_copies + 1)) <= words) ++A.log_copies;
    }
    const size_t lds = A.log_copies < 0 ? 0 : ((size_t)A.total << A.log_copies) * sizeof(uint32_t);
    // a row of one workgroup needs no totals to add to (20000 rows of 1000
    // phases, 2000 bins: 358 us with them, 75 without)
    A.store = gx == 1 && A.log_copies >= 0;
    if (!A.store || A.n == 0) {
        hipLaunchKernelGGL(hist_zero_kernel, dim3((uint32_t)zb), dim3(256), 0, stream, A.counts, nc);
        SDE_HIP(ctx, hipGetLastError());
        if (A.n == 0) return SDE_OK;
    }
    // a wave for less than 2048 values and bins to clear and add up, two, four
    // or eight for more
    const uint64_t work = share + (A.log_copies < 0 ? 0u : 2u * A.total);
    const uint32_t threads = work < 2048 ? 64 : work < 4096 ? 128 : work < 16384 ? 256 : kHistThreads;
    hipLaunchKernelGGL(kern, dim3((uint32_t)gx, (uint32_t)gy), dim3(threads), lds, stream, A);
    SDE_HIP(ctx, hipGetLastError());
    return SDE_OK;
}

int histogram_impl(sde_ctx* ctx, const int32_t* winding, uint64_t n, uint64_t pitch, uint64_t n_rows, int64_t x0,
                   uint32_t n_bins, uint64_t* counts, hipStream_t stream)
{
    if ((!winding && n) || !counts) return fail(ctx, SDE_ERR_INVALID, "null winding or counts");
    if (n_bins == 0 || n_bins > (1u << 24)) return fail(ctx, SDE_ERR_INVALID, "n_bins must be in [1, 2^24]");
    if (n_rows == 0 || n_rows > (1ull << 32)) return fail(ctx, SDE_ERR_INVALID, "n_rows must be in [1, 2^32]");
    if (n_rows > 1 && pitch < n) return fail(ctx, SDE_ERR_INVALID, "row pitch below the row length");
    if (!aligned(winding, 4) || !aligned(counts, 8)) return fail(ctx, SDE_ERR_INVALID, "misaligned pointer");
    const HistArgs A{winding, n, n_rows > 1 ? pitch : n, n_rows, x0, n_bins, n_bins + 2, 0, 0, counts};
    return launch_hist(ctx, A, x0 == (int32_t)x0 ? hist_kernel<PositionBin> : hist_kernel<WidePositionBin>, stream);
}

int phase_histogram_impl(sde_ctx* ctx, const float* theta, uint64_t n, uint64_t pitch, uint64_t n_rows,
                         uint32_t n_bins, uint64_t* counts, hipStream_t stream)
{
    if ((!theta && n) || !counts) return fail(ctx, SDE_ERR_INVALID, "null theta or counts");
    if (n_bins == 0 || n_bins > (1u << 24)) return fail(ctx, SDE_ERR_INVALID, "n_bins must be in [1, 2^24]");
    if (n_rows == 0 || n_rows > (1ull << 32)) return fail(ctx, SDE_ERR_INVALID, "n_rows must be in [1, 2^32]");
    if (n_rows > 1 && pitch < n) return fail(ctx, SDE_ERR_INVALID, "row pitch below the row length");
    if (!aligned(theta, 4) || !aligned(counts, 8)) return fail(ctx, SDE_ERR_INVALID, "misaligned pointer");
    const HistArgs A{theta, n, n_rows > 1 ? pitch : n, n_rows, 0, n_bins, n_bins + 1, 0, 0, counts};
    return launch_hist(ctx, A, hist_kernel<PhaseBin>, stream);
}

template <int KIND>
static void launch_obs_kind(uint32_t items, bool split, const ObsArgs& A, hipStream_t stream)
{
    void (*kern)(ObsArgs);
    uint32_t threads = kObsThreads;
    if (split) {
        kern = items <= 4 ? obs_slice_kernel<KIND, 4> : items <= 8 ? obs_slice_kernel<KIND, 8> : obs_slice_kernel<KIND, 16>;
    } else if (items <= 1) {
        kern = obs_group_kernel<KIND, kObsThreads / kWave, kWave>;
        threads = kWave;
    } else {
        kern = items <= 4    ? obs_group_kernel<KIND, 4, kObsThreads>
               : items <= 16 ? obs_group_kernel<KIND, 16, kObsThreads>
                             : obs_group_kernel<KIND, kObsGroupItems, kObsThreads>;
    }
    hipLaunchKernelGGL(kern, obs_grid(split ? A.n_slices : A.n_groups), dim3(threads), 0, stream, A);
}

static void launch_obs(int kind, uint32_t items, bool split, const ObsArgs& A, hipStream_t stream)
{
    switch (kind) {
    case SDE_OBS_MEAN_F32: return launch_obs_kind<SDE_OBS_MEAN_F32>(items, split, A, stream);
    case SDE_OBS_MEAN_F64: return launch_obs_kind<SDE_OBS_MEAN_F64>(items, split, A, stream);
    case SDE_OBS_MEANSQ_F32: return launch_obs_kind<SDE_OBS_MEANSQ_F32>(items, split, A, stream);
    default: return launch_obs_kind<SDE_OBS_ORDER>(items, split, A, stream);
    }
}

int observables_impl(sde_ctx* ctx, int kind, const void* in, const uint32_t* counts, uint32_t n_groups,
                     double* host_out, hipStream_t stream)
{
    if (kind < SDE_OBS_MEAN_F32 || kind > SDE_OBS_ORDER) return fail(ctx, SDE_ERR_INVALID, "unknown kind %d", kind);
    if (!in || !counts || !host_out || n_groups == 0) return fail(ctx, SDE_ERR_INVALID, "null argument or no groups");
    if (!aligned(in, kind == SDE_OBS_MEAN_F64 ? 8 : 4)) return fail(ctx, SDE_ERR_INVALID, "misaligned input");
    uint64_t total = 0;
    uint32_t most = 0;
    for (uint32_t g = 0; g < n_groups; ++g) {
        total += counts[g];
        most = counts[g] > most ? counts[g] : most;
    }
    // Slices of 4 elements per lane until there are 4 workgroups per CU, then
    // of up to 16 (fewer partials for the same bandwidth).
    const uint64_t enough = 4ull * ctx->n_cu;
    uint32_t items = 4;
    while (items < kObsItems && total / ((uint64_t)items * kObsThreads) >= enough) items *= 2;
    ObsArgs A;
    A.slice = items * kObsThreads;
    // No group is split where one slice holds the longest, or where there are 4
    // groups per CU and a workgroup's registers hold the longest, or, for the
    // order parameter (a single pass), it is no longer than the mean of as many
    // (4000 groups of 4097 floats: their means 50 us in two slices each and a
    // launch to add them, 33 so).
    const bool split = most > A.slice && !(n_groups >= enough && most <= kObsGroupItems * kObsThreads) &&
                       !(kind == SDE_OBS_ORDER && most <= total / enough);
    if (!split) items = (uint32_t)(((uint64_t)most + kObsThreads - 1) / kObsThreads);
    // layout of the workspace: first[n_groups] (u64) | counts[n_groups] (u32) |
    // where groups are split slice_begin[n_groups + 1] (u32)
    const size_t meta_bytes = (size_t)n_groups * 12 + (split ? 4 * ((size_t)n_groups + 1) : 0);
    std::vector<uint64_t> meta((meta_bytes + 7) / 8);
    uint64_t off = 0, slices = 0;
    for (uint32_t g = 0; g < n_groups; ++g) {
        meta[g] = off;
        off += counts[g];
    }
    unsigned char* words = reinterpret_cast<unsigned char*>(meta.data() + n_groups);
    std::memcpy(words, counts, 4 * (size_t)n_groups);
    if (split) {
        words += 4 * (size_t)n_groups;
        for (uint32_t g = 0; g < n_groups; ++g) {
            const uint32_t s32 = (uint32_t)slices;
            std::memcpy(words + 4 * (size_t)g, &s32, 4);
            slices += counts[g] ? ((uint64_t)counts[g] + A.slice - 1) / A.slice : 1;  // an empty group still has a result
            if (slices > 0x7fffffffull) return fail(ctx, SDE_ERR_INVALID, "observables: too many elements in one call");
        }
        const uint32_t all = (uint32_t)slices;
        std::memcpy(words + 4 * (size_t)n_groups, &all, 4);
    }
    int st = upload(ctx, kSlotMisc, 3, meta.data(), meta_bytes, stream);
    if (st) return st;
    // The results (16 B a group) go straight to pinned host memory, which the
    // final synchronization makes visible: no copy after the kernels (a call
    // on one group of 2^19 values 33 -> 24 us; of any number of groups it is
    // no slower: 2000 groups of 100 values 29 -> 20, 262144 of 10 831 -> 775).
    const size_t out_bytes = (size_t)n_groups * 2 * sizeof(double);
    DevBuf& host = ctx->obs_host;
    if (host.bytes < out_bytes) {
        if (host.ptr) SDE_HIP(ctx, hipHostFree(host.ptr));  // every earlier call has synchronized
        host.ptr = nullptr;
        host.bytes = 0;
        const size_t cap = std::max<size_t>(4096, out_bytes + out_bytes / 4);
        if (hipHostMalloc(&host.ptr, cap, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            host.ptr = nullptr;
            return fail(ctx, SDE_ERR_NOMEM, "observables: cannot allocate %zu bytes of pinned memory", cap);
        }
        host.bytes = cap;
    }
    void* part = nullptr;
    if (split && (st = ensure_ws(ctx, kSlotObs, (size_t)slices * 2 * sizeof(double), &part))) return st;
    const unsigned char* dmeta = static_cast<const unsigned char*>(ctx->ws[kSlotMisc].ptr);
    A.in = in;
    A.first = reinterpret_cast<const uint64_t*>(dmeta);
    A.counts = reinterpret_cast<const uint32_t*>(dmeta + 8 * (size_t)n_groups);
    A.slice_begin = A.counts + n_groups;
    A.part = static_cast<double*>(part);
    A.out = static_cast<double*>(host.ptr);
    A.n_groups = n_groups;
    A.n_slices = (uint32_t)slices;
    launch_obs(kind, items, split, A, stream);
    SDE_HIP(ctx, hipGetLastError());
    if (split) {
        hipLaunchKernelGGL(obs_combine_kernel, obs_grid(n_groups), dim3(kObsThreads), 0, stream, A, kind);
        SDE_HIP(ctx, hipGetLastError());
    }
    SDE_HIP(ctx, hipStreamSynchronize(stream));
    std::memcpy(host_out, host.ptr, out_bytes);
    return SDE_OK;
}

}  // namespace sde
