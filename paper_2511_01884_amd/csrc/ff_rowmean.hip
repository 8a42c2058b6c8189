// Second fused chain (the paper's fused-epilogue case study, App. B.1):
//
//     Out[m][k] = X[m][k] + GELU( mean_n( X[m] . W[n] + b[n] - s[n] ) )
//
// The case study is about removing global-memory round trips from this chain
// (the GEMM output re-read, the second read of the original row).  On top of
// that, the mean over n of a linear layer is itself linear in the row:
//     mean_n( x . W[n] + b[n] - s[n] ) = x . wbar + c,
//     wbar[k] = mean_n W[n][k],  c = mean_n (b[n] - s[n]),
// so the M x N x K GEMM collapses to one read of W (column means) and one
// dot product per row: O(NK + MK) work, bound by HBM traffic
// (W + X read once, Out written once).
//
// One launch of one workgroup per compute unit, two phases separated by one
// grid-wide arrival (counters in the control region, bounded wait):
//   1  column sums of W: a work item is a 128-byte strip of columns times a chunk
//      of rows, 8 lanes per row piece and 64 rows per step, reduced by shuffles and
//      once through LDS; fp32 partials [chunks][K] are written through.  Every
//      workgroup also sums its slice of b - s.  Then every wavefront requests its
//      first rows of X, which travel while the grid meets.
//   2  each workgroup adds the few chunk partials in chunk order into LDS: wbar;
//      one wavefront per row (several, for rows of more than 512 loads): the row is read once and kept in
//      registers (the case study's "cache the original row in registers"), dotted with wbar,
//      butterfly-reduced, GELU, broadcast add, store, while the next set of rows travels.
// Bound by HBM: 16384 x 8192 x 256 bf16 moves 541 MB in 105 us, 5.2 TB/s (one row after the other, whole in the
// registers of one wavefront: 195 us); 4096 x 4096 x 4096 bf16 100.7 MB in 22.7 us (24.3), which is the three
// streams at the rate of a large copy and 4 us of launch, ramp and meeting; 4096 x 4096 x 2048 fp32 38.0 us (52).
// All sums run in fixed order: results are bitwise reproducible on a device.
#include "ff_tile.hpp"

#include <type_traits>

namespace ff {

namespace {

constexpr int kThreads = kRowMeanThreads;         // 512
constexpr int kWaves = kThreads / 64;             // phase 2: rows in flight per workgroup
constexpr int kPieces = 8;                        // 16-byte pieces of a 128-byte strip
constexpr int kRowsPerStep = kRowMeanRowsPerStep; // phase 1: rows of W one load instruction of the workgroup covers
constexpr int kInFlight = 8;                      // phase 1: load instructions a thread keeps in flight
constexpr int kMaxChunks = 8;                     // 16-byte chunks of a row of X one lane keeps in registers
static_assert(kRowsPerStep * kPieces == kThreads, "one 16-byte piece per thread per step");

// a plain value another workgroup (on another XCD, behind another L2) reads later in this launch
__device__ __forceinline__ void store_through(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T> struct Vec16 { static constexpr int n = 16 / (int)sizeof(T); };

__device__ __forceinline__ void unpack(const uintx4 &v, float (&f)[8], const __bf16 *)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(v[i] << 16);
        f[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void unpack(const uintx4 &v, float (&f)[4], const float *)
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
        f[i] = __uint_as_float(v[i]);
}

// v, or zeros (by bits: a branch around the sum would draw the load into it, one latency for each)
__device__ __forceinline__ floatx4 masked(const floatx4 &v, bool ok)
{
    return __builtin_bit_cast(floatx4, __builtin_bit_cast(uintx4, v) & (ok ? 0xffffffffu : 0u));
}

// A row is shared by WPR wavefronts; PL = 16-byte chunks of it a lane keeps in registers; R = rows of a set: in
// phase 2 one of SETS = 2 is finished while the other travels, or (SETS = 1) a wavefront has no row after its first.
template <typename T, int PL, int R, int WPR, int SETS>
__global__ __launch_bounds__(kThreads) void rowmean_kernel(const RowMeanParams p)
{
    constexpr int E = Vec16<T>::n;
    constexpr int kStripElems = kPieces * E;        // columns of a strip
    __shared__ float red[kWaves][kPieces * 8];
    __shared__ __align__(16) float s_meet[kThreads * 4];
    __shared__ float s_dot[2][R][kWaves];
    extern __shared__ __align__(16) float s_w[];    // K floats (phase 2)
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = p.K, N = p.N, M = p.M;
    const int G = gridDim.x;
    const T *W = reinterpret_cast<const T *>(p.W);
    const T *X = reinterpret_cast<const T *>(p.X);
    T *Out = reinterpret_cast<T *>(p.Out);

    // ---- phase 1: partial[chunk][k] = sum over the chunk's rows of W[n][k] ----
    {
        const int piece = tid % kPieces;
        const int r = tid / kPieces;
        for (int item = blockIdx.x; item < p.strips * p.chunks; item += G) {
            const int strip = item % p.strips;
            const int chunk = item / p.strips;
            const int k0 = strip * kStripElems + piece * E;
            const int n_begin = chunk * p.rows_per_chunk;
            const int n_end = n_begin + p.rows_per_chunk < N ? n_begin + p.rows_per_chunk : N;
            float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (k0 < K) {
                const T *w = W + (size_t)(n_begin + r) * K + k0;
                const size_t step = (size_t)kRowsPerStep * K;
                // U rows of this thread, kRowsPerStep apart; MASK: those at or beyond n_end read the last row
                // there is and count as zeros, so that the end of a chunk is one more batch and no chain of loads
                // (1024 x 2304 x 740 fp32, four rows a thread: 20 us)
                auto batch = [&](auto count, auto mask, int n) {
                    constexpr int U = decltype(count)::value;
                    constexpr bool kMask = decltype(mask)::value;
                    uintx4 v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const T *at = w + u * step;
                        if (kMask)
                            at = n + u * kRowsPerStep < n_end ? at : W + (size_t)(n_end - 1) * K + k0;
                        v[u] = __builtin_nontemporal_load(reinterpret_cast<const uintx4 *>(at));
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        float f[E];
                        unpack(kMask ? v[u] & (n + u * kRowsPerStep < n_end ? 0xffffffffu : 0u) : v[u], f, (const T *)nullptr);
#pragma unroll
                        for (int e = 0; e < E; ++e)
                            acc[e] += f[e];
                    }
                };
                constexpr int kSpan = kInFlight * kRowsPerStep;
                int n = n_begin;  // (the batch's first row: the same for the whole workgroup)
                for (; n + kSpan <= n_end; n += kSpan, w += kInFlight * step)
                    batch(std::integral_constant<int, kInFlight>(), std::false_type(), n + r);
                const int left = (n_end - n + kRowsPerStep - 1) / kRowsPerStep;
                if (left > kInFlight / 2)
                    batch(std::integral_constant<int, kInFlight>(), std::true_type(), n + r);
                else if (left > kInFlight / 4)
                    batch(std::integral_constant<int, kInFlight / 2>(), std::true_type(), n + r);
                else if (left > 1)
                    batch(std::integral_constant<int, kInFlight / 4>(), std::true_type(), n + r);
                else if (n + r < n_end)
                    batch(std::integral_constant<int, 1>(), std::false_type(), n + r);
            }
            // the 8 rows of a wavefront (lane / 8), fixed butterfly; lanes 0..7 end with the piece sums
#pragma unroll
            for (int off = 8; off <= 32; off <<= 1)
#pragma unroll
                for (int e = 0; e < E; ++e)
                    acc[e] += __shfl_xor(acc[e], off);
            __syncthreads();  // the previous item's readers are done with red
            if (lane < kPieces)
#pragma unroll
                for (int e = 0; e < E; ++e)
                    red[wave][lane * E + e] = acc[e];
            __syncthreads();
            if (tid < kStripElems) {
                float t = red[0][tid];
#pragma unroll
                for (int w8 = 1; w8 < kWaves; ++w8)
                    t += red[w8][tid];
                // the partial rows are padded to whole strips: columns at or beyond K hold zeros
                store_through(p.partial + (size_t)chunk * p.k_pad + strip * kStripElems + tid, t);
            }
        }
        // this workgroup's slice of sum(b - s): wavefront 0, lanes stride the slice, fixed butterfly
        if (wave == 0) {
            const T *b = reinterpret_cast<const T *>(p.b);
            const T *sv = reinterpret_cast<const T *>(p.s);
            const int per = (N + G - 1) / G;
            const int s_begin = blockIdx.x * per < N ? blockIdx.x * per : N;
            const int s_end = s_begin + per < N ? s_begin + per : N;
            float acc = 0.0f;
            for (int n = s_begin + lane; n < s_end; n += 64)
                acc += (b ? load_as_float(b + n) : 0.0f) - (sv ? load_as_float(sv + n) : 0.0f);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
                acc += __shfl_xor(acc, off);
            if (lane == 0)
                store_through(p.cpart + blockIdx.x, acc);
        }
    }

    // ---- arrival: every partial is written ----
    wait_published();
    __syncthreads();
    const int way = blockIdx.x % kSyncWays;
    if (tid == 0)
        atomic_add_device(p.counters + (size_t)way * kSyncStride, 1u);

    // ---- the first sets of every wavefront: requested now, they travel while the grid meets ----
    const int nchunks = K / E;                       // 16-byte chunks per row
    const int per_lane = (nchunks + 64 * WPR - 1) / (64 * WPR);  // chunks per lane, interleaved by lane
    constexpr bool kRest = WPR == kWaves && E * PL * 64 * WPR < kRowMeanMaxK;  // a row may outgrow the registers
    constexpr int kRowsAtOnce = kWaves / WPR;
    const int row_step = G * kRowsAtOnce;
    const int first = (wave % WPR) * 64 + lane;      // this lane's chunks: first, first + 64 WPR, ...
    uintx4 keep[SETS][R][PL];
    // a lane past the row's end re-reads the last chunk and masks it out later
    auto load_rows = [&](int m, uintx4 (&dst)[R][PL]) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (m + r * row_step < M) {
                const T *x = X + (size_t)(m + r * row_step) * K;
#pragma unroll
                for (int u = 0; u < PL; ++u) {
                    int ch = u * 64 * WPR + first;
                    ch = ch < nchunks ? ch : nchunks - 1;
                    dst[r][u] = __builtin_nontemporal_load(reinterpret_cast<const uintx4 *>(x + (size_t)ch * E));
                }
            }
    };
    const int m_first = blockIdx.x * kRowsAtOnce + wave / WPR;
    load_rows(m_first, keep[0]);
    if constexpr (SETS == 2)
        load_rows(m_first + R * row_step, keep[1]);

    if (wave == 0) {
        const int l = lane < kSyncWays ? lane : 0;
        const unsigned target = (unsigned)(G + kSyncWays - 1 - l) / kSyncWays + (l == 0 ? (unsigned)p.extra_arrivals : 0u);
        if (!wait_counters_wave(p.counters, target, p.wait_ticks) && lane == 0)
            atomic_store_device(p.err, 1u);
    }
    __syncthreads();
    Departure leave;
    if (tid == 0)
        leave.begin(p.counters, way);

    // ---- phase 2: wbar into LDS (chunk partials added in chunk order), c, then one wavefront per row ----
    const int quads = K / 4;
    if (quads * 2 <= kThreads && p.chunks > 16) {
        // few columns, many chunks: groups of threads take neighbouring chunks, and their sums meet in LDS in
        // group order; a batch of loads of one thread's own costs 0.3 us, so up to 16 chunks it adds them itself
        int width = 64;
        while (width < quads)
            width *= 2;
        const int parts = kThreads / width, part = tid / width, q = tid % width;
        const int each = (p.chunks + parts - 1) / parts;
        const int ch_end = (part + 1) * each < p.chunks ? (part + 1) * each : p.chunks;
        floatx4 t = {0.0f, 0.0f, 0.0f, 0.0f};
        if (q < quads)
            for (int ch = part * each; ch < ch_end; ch += 8) {
                floatx4 u[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    u[j] = *reinterpret_cast<const floatx4 *>(p.partial + (size_t)(ch + j < ch_end ? ch + j : ch_end - 1) * p.k_pad + q * 4);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    t += masked(u[j], ch + j < ch_end);
            }
        floatx4 *meet = reinterpret_cast<floatx4 *>(s_meet);
        meet[tid] = t;
        __syncthreads();
        if (tid < quads) {
            for (int w = 1; w < parts; ++w)
                t += meet[w * width + tid];
            *reinterpret_cast<floatx4 *>(s_w + tid * 4) = t / (float)N;
        }
    } else {
        // two blocks of columns per pass, so that all of a thread's loads are in flight together
        for (int k = tid * 4; k < K; k += kThreads * 8) {
            const int k2 = k + kThreads * 4;
            const bool two = k2 < K;
            const float *src0 = p.partial + k;
            const float *src1 = p.partial + (two ? k2 : k);
            floatx4 t0 = {0.0f, 0.0f, 0.0f, 0.0f};
            floatx4 t1 = {0.0f, 0.0f, 0.0f, 0.0f};
            int ch = 0;
            for (; ch + 4 <= p.chunks; ch += 4) {
                floatx4 u0[4], u1[4];
#pragma unroll
                for (int j = 0; j < 4; ++j, src0 += p.k_pad, src1 += p.k_pad) {
                    u0[j] = *reinterpret_cast<const floatx4 *>(src0);
                    u1[j] = *reinterpret_cast<const floatx4 *>(src1);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    t0 += u0[j];
                    t1 += u1[j];
                }
            }
            if (ch < p.chunks) {
                floatx4 u0[4], u1[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {  // past the end the last chunk is read again and not added
                    const size_t at = (size_t)(ch + j < p.chunks ? j : p.chunks - 1 - ch) * p.k_pad;
                    u0[j] = *reinterpret_cast<const floatx4 *>(src0 + at);
                    u1[j] = *reinterpret_cast<const floatx4 *>(src1 + at);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    t0 += masked(u0[j], ch + j < p.chunks);
                    t1 += masked(u1[j], ch + j < p.chunks);
                }
            }
            *reinterpret_cast<floatx4 *>(s_w + k) = t0 / (float)N;
            if (two)
                *reinterpret_cast<floatx4 *>(s_w + k2) = t1 / (float)N;
        }
    }
    float c = 0.0f;  // every wavefront adds the workgroups' slices in the same order
    for (int j = lane; j < G; j += 64)
        c += p.cpart[j];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        c += __shfl_xor(c, off);
    c /= (float)N;
    __syncthreads();
    int turn = 0;
    // One branch for a set: were its rows tested again before the stores, the compiler would count them as still
    // travelling there and each store would wait for the one before it (1792 x 524 x 768 fp32: 0.2 us; 10692 x
    // 992 x 1792 fp32: 21.2 us, 20.2).  Two bf16 rows of eight loads a lane spill with it and test each row twice.
    constexpr bool kOneTest = R == 1 || PL < 8 || sizeof(T) == 4;
    auto finish_rows = [&](int m0, const uintx4 (&rows)[R][PL]) {
        if (kOneTest && m0 >= M) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // nothing travels any more; known here, nothing later waits for stores instead
            if (WPR > 1) {
                lds_barrier();
                turn ^= 1;
            }
            return;
        }
        float dot[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            dot[r] = 0.0f;
            if ((r > 0 || !kOneTest) && m0 + r * row_step >= M)
                continue;
            const T *x = X + (size_t)(m0 + r * row_step) * K;
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                const int ch_raw = u * 64 * WPR + first;
                const bool live = ch_raw < nchunks;
                const int ch = live ? ch_raw : nchunks - 1;
                float f[E];
                unpack(rows[r][u], f, (const T *)nullptr);
                float part = 0.0f;
#pragma unroll
                for (int e = 0; e < E; ++e)
                    part = fmaf(f[e], s_w[ch * E + e], part);
                dot[r] += live ? part : 0.0f;
            }
            // rows longer than the register budget: the rest is read here and again below
            for (int u = PL; kRest && u < per_lane; ++u) {
                const int ch = u * 64 * WPR + first;
                if (ch < nchunks) {
                    float f[E];
                    unpack(*reinterpret_cast<const uintx4 *>(x + (size_t)ch * E), f, (const T *)nullptr);
                    float part = 0.0f;
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        part = fmaf(f[e], s_w[ch * E + e], part);
                    dot[r] += part;
                }
            }
        }
        // every lane ends with the same sum; the R rows' steps overlap
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int r = 0; r < R; ++r)
                dot[r] += __shfl_xor(dot[r], off);
        if (WPR > 1) {
            // the row's wavefronts meet in LDS (two places in turn: one barrier a set is enough)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (lane == 0)
                    s_dot[turn][r][wave] = dot[r];
            lds_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dot[r] = 0.0f;
#pragma unroll
                for (int w = 0; w < WPR; ++w)
                    dot[r] += s_dot[turn][r][wave / WPR * WPR + w];
            }
            turn ^= 1;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if ((r > 0 || !kOneTest) && m0 + r * row_step >= M)
                continue;
            const T *x = X + (size_t)(m0 + r * row_step) * K;
            T *o = Out + (size_t)(m0 + r * row_step) * K;
            const float g = gelu_erf(dot[r] + c);
            auto emit = [&](const uintx4 &v, int ch) {
                float f[E];
                unpack(v, f, (const T *)nullptr);
                uintx4 q;
                if (sizeof(T) == 2) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        q[i] = pack_bf16x2(f[2 * i] + g, f[2 * i + 1] + g);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        q[i] = __float_as_uint(f[i] + g);
                }
                __builtin_nontemporal_store(q, reinterpret_cast<uintx4 *>(o + (size_t)ch * E));
            };
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                const int ch = u * 64 * WPR + first;
                if (ch < nchunks)
                    emit(rows[r][u], ch);
            }
            for (int u = PL; kRest && u < per_lane; ++u) {
                const int ch = u * 64 * WPR + first;
                if (ch < nchunks)
                    emit(*reinterpret_cast<const uintx4 *>(x + (size_t)ch * E), ch);
            }
        }
    };
    if (tid == 0)
        leave.middle(p.counters, way, G);
    if constexpr (SETS == 1) {
        finish_rows(m_first, keep[0]);
    } else {
        // (the bound is the workgroup's first row: with a shared row its wavefronts meet at barriers)
        for (int base = blockIdx.x * kRowsAtOnce, m = m_first; base < M; base += 2 * R * row_step, m += 2 * R * row_step) {
            finish_rows(m, keep[0]);
            load_rows(m + 2 * R * row_step, keep[0]);
            if (base + R * row_step < M)
                finish_rows(m + R * row_step, keep[1]);
            load_rows(m + 3 * R * row_step, keep[1]);
        }
    }

    if (tid == 0)
        leave.end(p.counters, G);
}

template <typename T, int PL, int R, int WPR, int SETS = 2>
hipError_t launch_plr(const RowMeanParams &p, hipStream_t stream)
{
    const size_t lds_bytes = (size_t)p.K * sizeof(float);
    if (lds_bytes > 32 * 1024) {  // static + dynamic beyond the default limit
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&rowmean_kernel<T, PL, R, WPR, SETS>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL((rowmean_kernel<T, PL, R, WPR, SETS>), dim3(p.grid), dim3(kThreads), lds_bytes, stream, p);
    return hipGetLastError();
}

// rows of a set: two sets fill up to 128 registers of chunks, unless a wavefront has no more than two rows
// (14848 x 1792 x 256 bf16: 23.3 us, with 64 registers 29.9).  Registers they are only while every array around
// them is used whole: with an eight-wide array for four floats the compiler put the sets on the stack (528
// bytes a lane), and 10692 x 992 x 1792 fp32 took 39.7 us for 21.8, 16384 x 1024 x 1024 52.9 for 29.0.
template <typename T, int PL>
hipError_t launch_pl(const RowMeanParams &p, hipStream_t stream)
{
    constexpr int kMost = 16 / PL < 8 ? 16 / PL : 8;
    // One row a wavefront at the most: no second set, whose code every launch would run past (a launch that
    // short reads its instructions from memory: 92 x 1048 x 544 bf16 11.4 us, 10.9 without; 1000^3 fp32 11.7, 11.4).
    if (p.M <= p.grid * kWaves)
        return launch_plr<T, PL, 1, 1, 1>(p, stream);
    return p.M > p.grid * kWaves * 2 ? launch_plr<T, PL, kMost, 1>(p, stream) : launch_plr<T, PL, 1, 1>(p, stream);
}

template <typename T>
hipError_t launch_t(const RowMeanParams &p, hipStream_t stream)
{
    constexpr int E = Vec16<T>::n;
    const int per_lane = (p.K / E + 63) / 64;
    if (per_lane <= 1) return launch_pl<T, 1>(p, stream);
    if (per_lane <= 2) return launch_pl<T, 2>(p, stream);
    if (per_lane <= 4) return launch_pl<T, 4>(p, stream);
    if (per_lane <= 8) return launch_pl<T, 8>(p, stream);
    if (per_lane <= 16) return launch_plr<T, 8, 1, 2>(p, stream);
    if (per_lane <= 32) return launch_plr<T, 8, 1, 4>(p, stream);
    return launch_plr<T, 8, 1, 8>(p, stream);
}

}  // namespace

hipError_t launch_rowmean_chain(bool bf16, const RowMeanParams &p, hipStream_t stream)
{
    return bf16 ? launch_t<__bf16>(p, stream) : launch_t<float>(p, stream);
}

}  // namespace ff
