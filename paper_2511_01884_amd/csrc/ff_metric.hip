// Profiling-metric selection (the paper's Sec. 2.3, Steps 2 and 3; Alg. 2).
//
// Input: n tasks, V kernels per task, J metrics per kernel, one runtime per kernel.
//   Step 2, per task: r[i][m] = Pearson correlation over the task's kernels between metric m and
//   the runtime; optionally drop metrics that duplicate an earlier kept one (|correlation| >= tau);
//   Top-k = the k kept metrics with the largest |r|.
//   Step 3: candidates = union of the Top-k lists; score S[m] = mean over all tasks of |r[i][m]|;
//   selected = candidates that are in the Top-k of at least `min_tasks` tasks, whose r has one sign
//   over those tasks, and whose score exceeds the given percentile of the candidates' scores.
// The correlations (one thread per task and metric, and one pair of metrics at a time for the duplicate
// filter) are computed on the GPU in fp64, all tasks in one launch, and so is the filter's greedy pass; the
// selection itself is a few hundred numbers and runs on the host.  An undefined correlation (constant
// column or constant runtime) is NaN: it never enters a Top-k and counts as 0 in the score.  Ties in |r|
// go to the lower metric index.  The percentile interpolates linearly between order statistics.
#include "ff_tile.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace ff {

namespace {

// One thread per task and metric, two passes over the V values of the column (mean, then centred sums),
// all in fp64: r, and for the duplicate filter (STATS) the column's mean and 1 / sqrt(sum of squares about
// it), NaN for a constant column.  Workgroups of one wavefront: a few thousand columns are all there is.
constexpr int kColumnThreads = 64;
template <bool STATS>
__global__ __launch_bounds__(kColumnThreads) void pearson_kernel(const double *values, const double *runtime, double *r,
                                                                 double *mean, double *inv, int V, int J)
{
    const int m = blockIdx.x * kColumnThreads + threadIdx.x;
    const int i = blockIdx.y;
    if (m >= J)
        return;
    const double *col = values + (size_t)i * V * J + m;
    const double *rt = runtime + (size_t)i * V;
    // a sample is constant when all its values are equal (compared as values: the mean of equal
    // values need not round back to that value, so the variance is no test)
    double mx = 0.0, my = 0.0;
    bool x_const = true, y_const = true;
    const double x0 = col[0], y0 = rt[0];
#pragma unroll 8
    for (int v = 0; v < V; ++v) {
        const double x = col[(size_t)v * J], y = rt[v];
        mx += x;
        my += y;
        x_const = x_const && x == x0;
        y_const = y_const && y == y0;
    }
    mx /= (double)V;
    my /= (double)V;
    double sxy = 0.0, sxx = 0.0, syy = 0.0;
#pragma unroll 8
    for (int v = 0; v < V; ++v) {
        const double dx = col[(size_t)v * J] - mx;
        const double dy = rt[v] - my;
        sxy += dx * dy;
        sxx += dx * dx;
        syy += dy * dy;
    }
    const size_t at = (size_t)i * J + m;
    r[at] = (!x_const && !y_const && sxx > 0.0 && syy > 0.0) ? sxy / sqrt(sxx * syy) : __builtin_nan("");
    if (STATS) {
        mean[at] = mx;
        inv[at] = (!x_const && sxx > 0.0) ? 1.0 / sqrt(sxx) : __builtin_nan("");
    }
}

// Bit b of mask[task][a][b / 64], b > a: the columns a and b, standardised, correlate at |c| >= tau (never for a
// constant column: its c is NaN).  A workgroup takes 64 x 64 pairs on or above the diagonal, a thread 4 x 4 of
// them; the sum of a pair runs over v in order, the next 16 rows are requested before these are used.  (8 x 8
// pairs per lane of a lone wavefront read the LDS half as often and took 65 instead of 45 us on twelve tasks of
// 64 x 1024: nothing covered the loads.)  Bits, not the matrix of correlations: the greedy pass needs no
// more, and they are a 64th of its bytes (eight tasks of 300 metrics: 92 KB against 5.8 MB that went to the host).
constexpr int kPairTile = 64, kPairRows = 16;
__global__ __launch_bounds__(256) void duplicate_kernel(const double *values, const double *mean, const double *inv,
                                                        unsigned long long *mask, double tau, int V, int J)
{
    if (blockIdx.x < blockIdx.y)
        return;
    __shared__ __align__(16) double za[kPairRows][kPairTile], zb[kPairRows][kPairTile];
    __shared__ unsigned long long bits[kPairTile];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int a0 = blockIdx.y * kPairTile, b0 = blockIdx.x * kPairTile;
    const size_t task = blockIdx.z;
    values += task * V * J;
    mean += task * J;
    inv += task * J;
    // a thread standardises one column of each side, every fourth row
    const int col = tid & 63, vrow = tid >> 6;
    const int ca = a0 + col < J ? a0 + col : J - 1, cb = b0 + col < J ? b0 + col : J - 1;
    const double ma = mean[ca], ia = inv[ca], mb = mean[cb], ib = inv[cb];
    double acc[4][4], ra[kPairRows / 4], rb[kPairRows / 4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = 0.0;
    if (tid < kPairTile)
        bits[tid] = 0;
    auto request = [&](int v0) {  // rows past the end read the last one; they are not summed
#pragma unroll
        for (int u = 0; u < kPairRows / 4; ++u) {
            const int v = v0 + vrow + u * 4 < V ? v0 + vrow + u * 4 : V - 1;
            ra[u] = values[(size_t)v * J + ca];
            rb[u] = values[(size_t)v * J + cb];
        }
    };
    request(0);
    for (int v0 = 0; v0 < V; v0 += kPairRows) {
        const int left = V - v0 < kPairRows ? V - v0 : kPairRows;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPairRows / 4; ++u) {
            za[vrow + u * 4][col] = (ra[u] - ma) * ia;
            zb[vrow + u * 4][col] = (rb[u] - mb) * ib;
        }
        __syncthreads();
        if (v0 + kPairRows < V)
            request(v0 + kPairRows);
        for (int v = 0; v < left; ++v) {
            typedef double double2_t __attribute__((ext_vector_type(2)));
            double x[4], y[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const double2_t xv = *reinterpret_cast<const double2_t *>(&za[v][ty * 4 + 2 * i]);
                const double2_t yv = *reinterpret_cast<const double2_t *>(&zb[v][tx * 2 + 32 * i]);
                x[2 * i] = xv[0];
                x[2 * i + 1] = xv[1];
                y[2 * i] = yv[0];
                y[2 * i + 1] = yv[1];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] += x[i] * y[j];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned long long w = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int at = tx * 2 + (j & 1) + 32 * (j >> 1);  // column inside the tile
            const int a = a0 + ty * 4 + i, b = b0 + at;
            if (b < J && b > a && fabs(acc[i][j]) >= tau)
                w |= 1ull << at;
        }
        if (w != 0)
            atomicOr(&bits[ty * 4 + i], w);
    }
    __syncthreads();
    const int words = (J + 63) / 64;
    if (tid < kPairTile && a0 + tid < J)
        mask[(task * J + a0 + tid) * words + blockIdx.x] = bits[tid];
}

// keep[task][m]: metrics in index order, a metric goes when it duplicates (bit in the mask) one already kept.
// One workgroup per task walks the metrics 64 at a time: the wavefronts have the 64 rows of the mask in
// registers (requested a block ahead: they do not depend on what is kept), the first one decides the block's 64
// metrics one after the other from the rows' diagonal word, then every kept row strikes out later metrics.
constexpr int kGreedyWaves = 16, kGreedyRows = 64 / kGreedyWaves;
constexpr int kGreedyMaxWords = 128;  // 8192 metrics
__global__ __launch_bounds__(64 * kGreedyWaves) void greedy_kernel(const unsigned long long *mask, unsigned char *keep, int J)
{
    __shared__ unsigned long long gone[kGreedyMaxWords];
    __shared__ unsigned long long kept_block;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int words = (J + 63) / 64;
    mask += (size_t)blockIdx.x * J * words;
    keep += (size_t)blockIdx.x * J;
    if (tid < kGreedyMaxWords)
        gone[tid] = 0;
    unsigned long long row[kGreedyRows][2], diag = 0;
    auto request = [&](int block) {  // in bounds for every lane; what is not wanted is dropped below
#pragma unroll
        for (int u = 0; u < kGreedyRows; ++u) {
            const int m = block * 64 + wave * kGreedyRows + u < J ? block * 64 + wave * kGreedyRows + u : J - 1;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                row[u][h] = mask[(size_t)m * words + (lane + 64 * h < words ? lane + 64 * h : words - 1)];
        }
        if (wave == 0)
            diag = mask[(size_t)(block * 64 + lane < J ? block * 64 + lane : J - 1) * words + block];
    };
    request(0);
    __syncthreads();
    for (int block = 0; block < words; ++block) {
        if (wave == 0) {
            // only rows with a duplicate inside the block can decide anything in it
            const unsigned long long here = gone[block];
            unsigned long long g = (unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(here >> 32)) << 32 |
                                   (unsigned)__builtin_amdgcn_readfirstlane((unsigned)here);
            const int count = J - block * 64 < 64 ? J - block * 64 : 64;
            unsigned long long deciders = __ballot(lane < count && diag != 0);
            while (deciders != 0) {
                const int j = __builtin_ctzll(deciders);
                deciders &= deciders - 1;
                if (!((g >> j) & 1))
                    g |= (unsigned long long)(unsigned)__builtin_amdgcn_readlane((unsigned)(diag >> 32), j) << 32 |
                         (unsigned)__builtin_amdgcn_readlane((unsigned)diag, j);
            }
            if (lane < count)
                keep[block * 64 + lane] = ((g >> lane) & 1) ? 0 : 1;
            if (lane == 0)
                kept_block = ~g & (count == 64 ? ~0ull : (1ull << count) - 1);
        }
        __syncthreads();
        const unsigned long long kept = kept_block;
        unsigned long long strike[2] = {0, 0};
#pragma unroll
        for (int u = 0; u < kGreedyRows; ++u)
            if ((kept >> (wave * kGreedyRows + u)) & 1) {
                strike[0] |= row[u][0];
                strike[1] |= row[u][1];
            }
        if (block + 1 < words)
            request(block + 1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int w = lane + 64 * h;
            if (w > block && w < words && strike[h] != 0)  // words at or below the diagonal are not written
                atomicOr(&gone[w], strike[h]);
        }
        __syncthreads();
    }
}

// Correlations, pair bits and the greedy pass in one launch, for what fits the LDS (selection_fits): a workgroup takes 64 x 64
// pairs on or above the diagonal of a task, brings their columns into LDS once, and finds their means and scales itself; those on
// the diagonal write r.  The last workgroup of a task to arrive has all its bits and decides.  Every sum runs in the
// order it has in the kernels above: the same bits.
//
// Bound by latency: a load of the columns, one store and one arrival, one load of the bits.  Three launches with a load or two
// each were 22 us of eight tasks of 10 x 300; this one is 13.5.  Pair bits lie in memory as the greedy pass reads them: the rows
// of block b, 64 of them, hold words b .. words - 1.
constexpr int kFusedThreads = 256;
__host__ __device__ constexpr size_t pair_words(int words) { return (size_t)32 * words * (words + 1); }
__device__ __forceinline__ int pair_block(int words, int b) { return 64 * (b * words - b * (b - 1) / 2); }

__global__ __launch_bounds__(kFusedThreads) void selection_kernel(const double *values, const double *runtime, double *r,
                                                                  unsigned char *keep, unsigned long long *mask,
                                                                  unsigned *arrived, double tau, int V, int J)
{
    extern __shared__ __align__(16) double z[];  // [V][128]: 64 columns of side a, 64 of side b; later the pair bits
    __shared__ double s_mean[128], s_inv[128];
    __shared__ unsigned long long bits[kPairTile];
    __shared__ int s_last;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int words = (J + 63) / 64;
    const size_t task = blockIdx.y;
    int by = 0, bx = (int)blockIdx.x;  // the bx-th of row by, row by + 1, ... of the upper triangle
    while (bx >= words - by) {
        bx -= words - by;
        ++by;
    }
    bx += by;
    const int a0 = by * kPairTile, b0 = bx * kPairTile;
    const bool diagonal = bx == by;
    values += task * V * J;
    runtime += task * V;
    mask += task * pair_words(words);

    {
        const int col = tid & 127, first = (col < 64 ? a0 : b0) + (col & 63);
        const double *src = values + (first < J ? first : J - 1);
        for (int v0 = tid >> 7; v0 < V; v0 += 32) {
            double x[16];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                x[u] = src[(size_t)(v0 + 2 * u < V ? v0 + 2 * u : V - 1) * J];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (v0 + 2 * u < V)
                    z[(v0 + 2 * u) * 128 + col] = x[u];
        }
    }
    if (tid < kPairTile)
        bits[tid] = 0;
    __syncthreads();
    if (tid < 128) {
        double mx = 0.0;
        bool x_const = true;
        const double x0 = z[tid];
#pragma unroll 8
        for (int v = 0; v < V; ++v) {
            const double x = z[v * 128 + tid];
            mx += x;
            x_const = x_const && x == x0;
        }
        mx /= (double)V;
        double sxx = 0.0;
#pragma unroll 8
        for (int v = 0; v < V; ++v) {
            const double dx = z[v * 128 + tid] - mx;
            sxx += dx * dx;
        }
        s_mean[tid] = mx;
        s_inv[tid] = (!x_const && sxx > 0.0) ? 1.0 / sqrt(sxx) : __builtin_nan("");
        if (diagonal && tid < 64 && a0 + tid < J) {
            double my = 0.0;
            bool y_const = true;
            const double y0 = runtime[0];
#pragma unroll 8
            for (int v = 0; v < V; ++v) {
                const double y = runtime[v];
                my += y;
                y_const = y_const && y == y0;
            }
            my /= (double)V;
            double sxy = 0.0, syy = 0.0;
#pragma unroll 8
            for (int v = 0; v < V; ++v) {
                const double dx = z[v * 128 + tid] - mx, dy = runtime[v] - my;
                sxy += dx * dy;
                syy += dy * dy;
            }
            r[task * J + a0 + tid] = (!x_const && !y_const && sxx > 0.0 && syy > 0.0) ? sxy / sqrt(sxx * syy) : __builtin_nan("");
        }
    }
    __syncthreads();
    for (int e = tid; e < V * 128; e += kFusedThreads)
        z[e] = (z[e] - s_mean[e & 127]) * s_inv[e & 127];
    __syncthreads();
    double acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = 0.0;
#pragma unroll 2
    for (int v = 0; v < V; ++v) {
        typedef double double2_t __attribute__((ext_vector_type(2)));
        double x[4], y[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double2_t xv = *reinterpret_cast<const double2_t *>(&z[v * 128 + ty * 4 + 2 * i]);
            const double2_t yv = *reinterpret_cast<const double2_t *>(&z[v * 128 + 64 + tx * 2 + 32 * i]);
            x[2 * i] = xv[0];
            x[2 * i + 1] = xv[1];
            y[2 * i] = yv[0];
            y[2 * i + 1] = yv[1];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] += x[i] * y[j];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned long long w = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int at = tx * 2 + (j & 1) + 32 * (j >> 1);  // column inside the tile
            const int a = a0 + ty * 4 + i, b = b0 + at;
            if (b < J && b > a && fabs(acc[i][j]) >= tau)
                w |= 1ull << at;
        }
        if (w != 0)
            atomicOr(&bits[ty * 4 + i], w);
    }
    __syncthreads();
    if (tid < kPairTile)
        __hip_atomic_store(mask + pair_block(words, by) + tid * (words - by) + bx - by, bits[tid], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    wait_published();
    __syncthreads();
    if (tid == 0)
        s_last = atomic_add_device(arrived + task * 32, 1u) == gridDim.x - 1u;
    __syncthreads();
    if (!s_last)
        return;

    // ---- the greedy pass ----
    unsigned long long *m = reinterpret_cast<unsigned long long *>(z);
    const int total = (int)pair_words(words);
    for (int e0 = tid; e0 < total; e0 += kFusedThreads * 8) {
        unsigned long long w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)  // other units' bits: past the L2 of this one
            w[u] = __hip_atomic_load(mask + (e0 + u * kFusedThreads < total ? e0 + u * kFusedThreads : total - 1), __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (e0 + u * kFusedThreads < total)
                m[e0 + u * kFusedThreads] = w[u];
    }
    if (tid == 0)
        atomic_store_device(arrived + task * 32, 0u);
    __syncthreads();
    if (tid >= 64)
        return;
    // One wavefront: lane l has word l % 16 of what is struck out; it looks at every fourth row from l / 16 on.
    const int word = tid & 15;
    unsigned long long gone = 0;
    for (int b = 0; b < words; ++b) {
        const int pitch = words - b;
        const unsigned long long *rows = m + pair_block(words, b);
        const int count = J - b * 64 < 64 ? J - b * 64 : 64;
        const unsigned long long diag = rows[tid * pitch];
        unsigned long long g = (unsigned long long)__builtin_amdgcn_readlane((unsigned)(gone >> 32), b) << 32 |
                               (unsigned)__builtin_amdgcn_readlane((unsigned)gone, b);
        // only rows with a duplicate inside the block can decide anything in it
        unsigned long long deciders = __ballot(tid < count && diag != 0);
        while (deciders != 0) {
            const int j = __builtin_ctzll(deciders);
            deciders &= deciders - 1;
            if (!((g >> j) & 1))
                g |= (unsigned long long)(unsigned)__builtin_amdgcn_readlane((unsigned)(diag >> 32), j) << 32 |
                     (unsigned)__builtin_amdgcn_readlane((unsigned)diag, j);
        }
        if (tid < count)
            keep[task * J + b * 64 + tid] = ((g >> tid) & 1) ? 0 : 1;
        const unsigned long long kept = ~g & (count == 64 ? ~0ull : (1ull << count) - 1);
        const int at = word > b && word < words ? word - b : 0;
        unsigned long long strike = 0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int row = u * 4 + (tid >> 4);
            const unsigned long long w = rows[row * pitch + at];
            strike |= ((kept >> row) & 1) ? w : 0;
        }
        strike |= __shfl_xor(strike, 16);
        strike |= __shfl_xor(strike, 32);
        gone |= at != 0 ? strike : 0;
    }
}

// LDS of the kernel above: the columns, or the pair bits.
size_t selection_lds(int V, int J)
{
    return std::max((size_t)V * 128 * sizeof(double), pair_words((J + 63) / 64) * sizeof(unsigned long long));
}

}  // namespace

// Whether that kernel takes tasks of this size: two workgroups to a unit's LDS, and a lane for every word of a row of bits.
bool selection_fits(int V, int J) { return J <= 1024 && selection_lds(V, J) <= 76u << 10; }
size_t selection_mask_bytes(int J) { return pair_words((J + 63) / 64) * sizeof(unsigned long long); }

// r and keep of n tasks; mask has room for selection_mask_bytes of each, arrived a zero word in every 128 bytes for each
hipError_t launch_selection(const double *values, const double *runtime, double *r, unsigned char *keep, unsigned long long *mask,
                            unsigned *arrived, double tau, int n, int V, int J, hipStream_t stream)
{
    const int words = (J + 63) / 64;
    hipLaunchKernelGGL(selection_kernel, dim3(words * (words + 1) / 2, n), dim3(kFusedThreads), selection_lds(V, J), stream, values,
                       runtime, r, keep, mask, arrived, tau, V, J);
    return hipGetLastError();
}

hipError_t launch_pearson(const double *values, const double *runtime, double *r, double *mean, double *inv, int n,
                          int V, int J, hipStream_t stream)
{
    const dim3 grid((J + kColumnThreads - 1) / kColumnThreads, n);
    if (mean != nullptr)
        hipLaunchKernelGGL(pearson_kernel<true>, grid, dim3(kColumnThreads), 0, stream, values, runtime, r, mean, inv, V, J);
    else
        hipLaunchKernelGGL(pearson_kernel<false>, grid, dim3(kColumnThreads), 0, stream, values, runtime, r, mean, inv, V, J);
    return hipGetLastError();
}

// keep[n][J] of n tasks; mask has room for n * J * ((J + 63) / 64) words
hipError_t launch_duplicate_filter(const double *values, const double *mean, const double *inv, double tau,
                                   unsigned long long *mask, unsigned char *keep, int n, int V, int J, hipStream_t stream)
{
    const int words = (J + 63) / 64;
    hipLaunchKernelGGL(duplicate_kernel, dim3(words, words, n), dim3(256), 0, stream, values, mean, inv, mask, tau, V, J);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(greedy_kernel, dim3(n), dim3(64 * kGreedyWaves), 0, stream, mask, keep, J);
    return hipGetLastError();
}

// Steps after the correlations, on the host.  r [n][J]; keep [n][J] or null (all kept).
// top [n][k] (-1 padded), score [J], selected [J] (0/1), *threshold; each output optional.
void metric_select_host(const double *r, const unsigned char *keep, int n, int J, int k, double q,
                        int min_tasks, int *top, double *score, unsigned char *selected, double *threshold)
{
    constexpr int kInsert = 64;  // up to this k a task's list is kept sorted as its metrics pass by
    std::vector<int> tops((size_t)n * k, -1);
    std::vector<double> S(J, 0.0);
    struct Seen { int tasks; unsigned char signs; };  // Top-k lists a metric is in, and its signs there: 1 +, 2 -, 4 zero
    std::vector<Seen> seen(J, Seen{0, 0});
    std::vector<std::pair<double, int>> cand;
    auto before = [](const std::pair<double, int> &a, const std::pair<double, int> &b) {
        return a.first > b.first || (a.first == b.first && a.second < b.second);
    };
    for (int i = 0; i < n; ++i) {
        const double *ri = r + (size_t)i * J;
        const unsigned char *ki = keep ? keep + (size_t)i * J : nullptr;
        int *list = tops.data() + (size_t)i * k;
        int filled = 0;
        if (k <= kInsert) {
            double best[kInsert] = {};
            for (int m = 0; m < J; ++m) {
                const double v = std::fabs(ri[m]);
                if (!std::isnan(v))
                    S[m] += v;
                // (a NaN compares false; an equal |r| further on stays behind)
                if ((ki && !ki[m]) || !(filled < k ? v >= 0.0 : v > best[k - 1]))
                    continue;
                int at = filled < k ? filled++ : k - 1;
                // (a new largest one moves the list as a whole: |r| that rise with m, 12 tasks of 1024 with k = 64, 580 us one by one, 230)
                if (best[0] < v) {
                    std::memmove(best + 1, best, (size_t)at * sizeof(double));
                    std::memmove(list + 1, list, (size_t)at * sizeof(int));
                    at = 0;
                }
                for (; at > 0 && best[at - 1] < v; --at) {
                    best[at] = best[at - 1];
                    list[at] = list[at - 1];
                }
                best[at] = v;
                list[at] = m;
            }
        } else {
            cand.clear();
            for (int m = 0; m < J; ++m) {
                const double v = std::fabs(ri[m]);
                if (std::isnan(v))
                    continue;
                S[m] += v;
                if (!ki || ki[m])
                    cand.emplace_back(v, m);
            }
            filled = cand.size() < (size_t)k ? (int)cand.size() : k;
            std::partial_sort(cand.begin(), cand.begin() + filled, cand.end(), before);
            for (int j = 0; j < filled; ++j)
                list[j] = cand[j].second;
        }
        for (int j = 0; j < filled; ++j) {
            const double v = ri[list[j]];
            Seen &s = seen[list[j]];
            ++s.tasks;
            s.signs |= v > 0.0 ? 1 : (v < 0.0 ? 2 : 4);
        }
    }
    for (int m = 0; m < J; ++m)
        S[m] /= (double)n;
    std::vector<double> cs;
    for (int m = 0; m < J; ++m)
        if (seen[m].tasks > 0)
            cs.push_back(S[m]);
    double cut = std::nan("");
    if (!cs.empty()) {
        std::sort(cs.begin(), cs.end());
        const double pos = (double)(cs.size() - 1) * q / 100.0;
        const size_t lo = (size_t)std::floor(pos);
        const size_t hi = lo + 1 < cs.size() ? lo + 1 : cs.size() - 1;
        cut = cs[lo] + (pos - (double)lo) * (cs[hi] - cs[lo]);
    }
    if (selected)
        for (int m = 0; m < J; ++m) {
            const unsigned char one = seen[m].signs;
            selected[m] = seen[m].tasks >= min_tasks && (one == 1 || one == 2 || one == 4) && S[m] > cut ? 1 : 0;
        }
    if (top)
        std::copy(tops.begin(), tops.end(), top);
    if (score)
        std::copy(S.begin(), S.end(), score);
    if (threshold)
        *threshold = cut;
}

}  // namespace ff
