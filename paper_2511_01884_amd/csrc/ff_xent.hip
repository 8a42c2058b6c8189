// Row-wise cross-entropy: the row reduction of the paper's case study (Sec. 4),
//
//     loss[r] = log( sum_c exp(L[r][c]) ) - L[r][t[r]],    mean = (1/B) sum_r loss[r].
//
// The case study's kernel went from block-wide shared-memory reductions to
// shuffle reductions with a single cross-wavefront combine, and then removed the
// second global read of the logits by buffering the row on chip.  Here a row is
// read exactly once too:
//   short rows (up to 512 loads of 16 bytes)  L lanes of a wavefront hold the whole row in
//     registers: its maximum, then one exponential per element against it;
//   longer rows  a wavefront takes a row, or a segment of one where the rows alone are too few to
//     fill the chip; every lane keeps a running (maximum, sum of exp(x - maximum)) pair and rescales
//     the sum when its maximum moves.
// Loads are 16 bytes wherever a row begins: the elements before its first and after its last
// 16-byte boundary are loaded one by one, by the first lanes, together with the rest.  What is
// left over after whole batches of loads is one more batch in which excluded loads repeat the
// last one and count as -inf, so no load waits for another.
// The kernel is bound by the HBM read of L; bf16 rows of middle length by the vector ALUs.
//
// The mean over rows is part of the same launch: each workgroup adds the losses
// of its rows in a fixed order, publishes that one number, and the workgroup that
// arrives last adds the published numbers in workgroup order (with segments: it combines the
// published pairs of every row first).  All orders are fixed by the launch shape, so results are
// bitwise reproducible.
#include "ff_tile.hpp"

#include <type_traits>

namespace ff {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kBatch = 8;  // 16-byte loads a lane issues back to back
constexpr float kLog2e = 1.44269504088896341f;
constexpr float kLn2 = 0.693147180559945309f;

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

// Reference point for the exponents: the maximum, or 0 while the maximum is still -inf
// (so that -inf - (-inf) never appears).
__device__ __forceinline__ float ref_of(float m) { return m == -INFINITY ? 0.0f : m; }

// 0 in every lane, in a vector register and unknown to the compiler
__device__ __forceinline__ int zero_lane()
{
    int z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}

// Reductions over the L neighbouring lanes of a row; every lane ends with the same bits (each step
// combines the two same numbers in both lanes of a pair).
template <int ctrl> __device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true));
}
template <int L, typename F> __device__ __forceinline__ float reduce(float v, F f)
{
    static_assert(L == 4 || L == 16 || L == 64, "lanes per row");
    if (L == 4) {
        v = f(v, dpp<0xB1>(v));   // quad_perm 1,0,3,2
        return f(v, dpp<0x4E>(v));  // quad_perm 2,3,0,1
    }
    v = f(v, dpp<0x128>(v));  // row_ror:8, 4, 2, 1
    v = f(v, dpp<0x124>(v));
    v = f(v, dpp<0x122>(v));
    v = f(v, dpp<0x121>(v));
    if (L == 64) {
        v = f(v, __shfl_xor(v, 16));
        v = f(v, __shfl_xor(v, 32));
    }
    return v;
}
template <int L> __device__ __forceinline__ float reduce_max(float v)
{
    return reduce<L>(v, [](float a, float b) { return fmaxf(a, b); });
}
template <int L> __device__ __forceinline__ float reduce_sum(float v)
{
    return reduce<L>(v, [](float a, float b) { return a + b; });
}

// 16 bytes of a row, or (VEC = 1) one element
template <typename T, int VEC> struct Chunk;
template <> struct Chunk<float, 4> {
    uintx4 v;
    __device__ __forceinline__ void load(const float *p) { v = __builtin_nontemporal_load(reinterpret_cast<const uintx4 *>(p)); }
    __device__ __forceinline__ void keep(bool ok) { v = ok ? v : uintx4{0xff800000u, 0xff800000u, 0xff800000u, 0xff800000u}; }
    __device__ __forceinline__ void get(float (&f)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            f[i] = __uint_as_float(v[i]);
    }
};
template <> struct Chunk<__bf16, 8> {
    uintx4 v;
    __device__ __forceinline__ void load(const __bf16 *p) { v = __builtin_nontemporal_load(reinterpret_cast<const uintx4 *>(p)); }
    __device__ __forceinline__ void keep(bool ok) { v = ok ? v : uintx4{0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u}; }
    __device__ __forceinline__ void get(float (&f)[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(v[i] << 16);
            f[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
        }
    }
};
template <typename T> struct Chunk<T, 1> {
    float v;
    __device__ __forceinline__ void load(const T *p) { v = load_as_float(p); }
    __device__ __forceinline__ void keep(bool ok) { v = ok ? v : -INFINITY; }
    __device__ __forceinline__ void get(float (&f)[1]) const { f[0] = v; }
};

// U chunks of a lane, L chunks apart, the first at ch; MASK: those at or beyond n count as -inf
template <typename T, int VEC, int U, int L, bool MASK>
__device__ __forceinline__ void load_batch(const T *body, int ch, int n, float (&f)[U][VEC])
{
    Chunk<T, VEC> c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int at = ch + u * L;
        c[u].load(body + (size_t)(MASK && at >= n ? n - 1 : at) * VEC);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (MASK)
            c[u].keep(ch + u * L < n);
        c[u].get(f[u]);
    }
}
template <int VEC, int U> __device__ __forceinline__ float batch_max(float m, const float (&f)[U][VEC])
{
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            m = fmaxf(m, f[u][e]);
    return m;
}
// sum of exp(f - ref): sums of a chunk's elements, added in chunk order
template <int VEC, int U> __device__ __forceinline__ float batch_sum(float ref, const float (&f)[U][VEC])
{
    float add = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float part = 0.0f;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            part += exp2_hw((f[u][e] - ref) * kLog2e);
        add += part;
    }
    return add;
}
// Folds a batch into the lane's running pair with one rescale.
template <int VEC, int U> __device__ __forceinline__ void fold(float &m, float &s, const float (&f)[U][VEC])
{
    const float mn = batch_max<VEC, U>(m, f);
    const float ref = ref_of(mn);
    s = fmaf(s, exp2_hw((m - ref) * kLog2e), batch_sum<VEC, U>(ref, f));
    m = mn;
}

// A row's elements that 16-byte loads at 16-byte boundaries do not cover: head before the first, tail after
// the last.  PEEL = 0: rows are whole 16-byte pieces, there are none.
template <typename T, int VEC, int L, bool PEEL> struct Edges {
    static constexpr int kMost = 2 * VEC - 2;
    static constexpr int U = PEEL && VEC > 1 ? (kMost + L - 1) / L : 0;
    int head, n;  // elements before the first chunk, chunks
    float f[U > 0 ? U : 1];
    __device__ __forceinline__ Edges(const T *row, int C)
    {
        head = U > 0 ? (int)((0u - (unsigned)(reinterpret_cast<uintptr_t>(row) / sizeof(T))) % VEC) : 0;
        n = (C - head) / VEC;
    }
    __device__ __forceinline__ void load(const T *row, int C, int tl)
    {
        const int count = C - n * VEC;  // head and tail together
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = tl + u * L;
            f[u] = load_as_float(row + (k < head ? k : (k < count ? n * VEC + k : 0)));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            f[u] = tl + u * L < count ? f[u] : -INFINITY;
    }
    __device__ __forceinline__ float max(float m) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u)
            m = fmaxf(m, f[u]);
        return m;
    }
    __device__ __forceinline__ float sum(float ref) const
    {
        float add = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u)
            add += exp2_hw((f[u] - ref) * kLog2e);
        return add;
    }
};

// The end of a launch: the workgroup's number is published, and the workgroup that arrives last goes on.
// Arrivals on one word queue up at about 6 ns each, so a large launch arrives on kSyncWays words and the last
// of each goes on to the final one; a small launch arrives there at once.
constexpr unsigned kOneLevel = 256;
__device__ __forceinline__ bool last_to_arrive(const XentParams &p, unsigned *s_last)
{
    wait_published();
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned arrivals = gridDim.x;
        bool on = true;
        if (gridDim.x > kOneLevel) {
            const unsigned way = blockIdx.x % kSyncWays;
            unsigned *c = p.ways + (size_t)way * kSyncStride;
            on = atomic_add_device(c, 1u) + 1u == (gridDim.x + kSyncWays - 1 - way) / kSyncWays;
            if (on)
                atomic_store_device(c, 0u);  // ready for the next launch
            arrivals = kSyncWays;
        }
        *s_last = on && atomic_add_device(p.counter, 1u) + 1u == arrivals ? 1u : 0u;
    }
    __syncthreads();
    return *s_last != 0u;
}
// ... and adds `acc` of its threads: the mean of the launch.
__device__ __forceinline__ void finish_mean(const XentParams &p, float acc, float *s_red)
{
    acc = reduce_sum<64>(acc);
    if ((threadIdx.x & 63) == 0)
        s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float total = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            total += s_red[w];
        *p.mean_loss = total / (float)p.B;
        atomic_store_device(p.counter, 0u);  // ready for the next launch
    }
}
// The workgroup's sum of losses (each row's in one lane, zero elsewhere) and the mean of the launch.
__device__ __forceinline__ void sum_losses(const XentParams &p, float loss_sum)
{
    __shared__ float s_red[kWaves];
    __shared__ unsigned s_last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    loss_sum = reduce_sum<64>(loss_sum);
    if (lane == 0)
        s_red[wave] = loss_sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float total = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            total += s_red[w];
        publish_pair(p.partials + blockIdx.x, floatx2{total, 0.0f});
    }
    if (!last_to_arrive(p, &s_last))
        return;
    float acc = 0.0f;
    for (int i = threadIdx.x; i < (int)gridDim.x; i += kBatch * kThreads) {
        float u[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j)  // all under way together; past the end the last is read again
            u[j] = read_pair(p.partials + (i + j * kThreads < (int)gridDim.x ? i + j * kThreads : (int)gridDim.x - 1))[0];
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            acc += i + j * kThreads < (int)gridDim.x ? u[j] : 0.0f;
    }
    finish_mean(p, acc, s_red);
}

// Short rows: L lanes hold a row, Q chunks each; 64 / L rows per wavefront at a time.
template <typename T, int VEC, int L, int Q, bool PEEL>
__global__ __launch_bounds__(kThreads) void xent_short_kernel(XentParams p)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tl = lane % L;
    constexpr int kRows = 64 / L;
    const int stride = (int)gridDim.x * kWaves * kRows;
    const T *logits = reinterpret_cast<const T *>(p.logits);
    float loss_sum = 0.0f;
    int r = (blockIdx.x * kWaves + wave) * kRows + lane / L;
    long long t = p.targets[r < p.B ? r : p.B - 1];
    // (the loop's bound is the wavefront's first row: its lanes stay together)
    for (int r0 = r - lane / L; r0 < p.B; r0 += stride, r += stride) {
        const bool ok = r < p.B;
        const T *row = logits + (size_t)(ok ? r : p.B - 1) * (size_t)p.C;
        const bool t_ok = t >= 0 && t < (long long)p.C;
        const float xt = load_as_float(row + (t_ok ? t : 0));
        const int next = r + stride;  // its target, one row ahead: the target's logit is a second load behind it
        t = p.targets[next < p.B ? next : p.B - 1];
        Edges<T, VEC, L, PEEL> edges(row, p.C);
        float f[Q][VEC];
        edges.load(row, p.C, tl);
        load_batch<T, VEC, Q, L, true>(row + edges.head, tl, edges.n, f);
        const float m = reduce_max<L>(edges.max(batch_max<VEC, Q>(-INFINITY, f)));
        const float ref = ref_of(m);
        const float s = reduce_sum<L>(batch_sum<VEC, Q>(ref, f) + edges.sum(ref));
        float loss = (m - xt) + __builtin_amdgcn_logf(s) * kLn2;
        if (!t_ok)
            loss = __builtin_nanf("");
        if (tl == 0 && ok) {
            if (p.row_loss)
                p.row_loss[r] = loss;
            loss_sum += loss;
        }
    }
    sum_losses(p, loss_sum);
}

// Longer rows: a wavefront takes segment seg of row r (p.segs segments of p.seg_chunks chunks each).
template <typename T, int VEC, bool PEEL, bool SPLIT>
__global__ __launch_bounds__(kThreads) void xent_long_kernel(XentParams p)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T *logits = reinterpret_cast<const T *>(p.logits);
    const int segs = SPLIT ? p.segs : 1;
    const int items = p.B * segs;
    float loss_sum = 0.0f;
    int item = blockIdx.x * kWaves + wave;
    const int stride = (int)gridDim.x * kWaves;
    // (per lane, so that the load is one of the vector queue and waited for with the others)
    auto target_of = [&](int it) { return p.targets[(SPLIT ? (it < items ? it : items - 1) / segs : (it < items ? it : items - 1)) + zero_lane()]; };
    long long t = target_of(item);
    for (; item < items; item += stride) {
        const int r = SPLIT ? item / segs : item;
        const int seg = SPLIT ? item - r * segs : 0;
        const T *row = logits + (size_t)r * (size_t)p.C;
        const bool t_ok = t >= 0 && t < (long long)p.C;
        const float xt = load_as_float(row + (t_ok ? t : 0));
        t = target_of(item + stride);  // one row ahead: the target's logit is a second load behind it
        Edges<T, VEC, 64, PEEL> edges(row, p.C);
        const T *body = row + edges.head;
        float m = -INFINITY, s = 0.0f;
        int ch = 0, n = edges.n;
        if (seg == 0)
            edges.load(row, p.C, lane);
        if (SPLIT) {
            ch = seg * p.seg_chunks;
            n = ch + p.seg_chunks < n ? ch + p.seg_chunks : n;
        }
        for (; ch + kBatch * 64 <= n; ch += kBatch * 64) {
            float f[kBatch][VEC];
            load_batch<T, VEC, kBatch, 64, false>(body, ch + lane, n, f);
            fold<VEC, kBatch>(m, s, f);
        }
        const int left = n - ch;
        if (left > 4 * 64) {
            float f[kBatch][VEC];
            load_batch<T, VEC, kBatch, 64, true>(body, ch + lane, n, f);
            fold<VEC, kBatch>(m, s, f);
        } else if (left > 64) {
            float f[4][VEC];
            load_batch<T, VEC, 4, 64, true>(body, ch + lane, n, f);
            fold<VEC, 4>(m, s, f);
        } else if (left > 0) {
            float f[1][VEC];
            load_batch<T, VEC, 1, 64, true>(body, ch + lane, n, f);
            fold<VEC, 1>(m, s, f);
        }
        const float mn = reduce_max<64>(seg == 0 ? edges.max(m) : m);
        const float ref = ref_of(mn);
        s *= exp2_hw((m - ref) * kLog2e);
        if (seg == 0)
            s += edges.sum(ref);
        s = reduce_sum<64>(s);
        if (SPLIT) {
            if (lane == 0) {
                publish_pair(p.partials + item, floatx2{mn, s});
                if (seg == 0)  // a target outside the row makes its loss NaN
                    publish_pair(p.picked + r, floatx2{t_ok ? xt : __builtin_nanf(""), 0.0f});
            }
        } else if (lane == 0) {
            float loss = (mn - xt) + __builtin_amdgcn_logf(s) * kLn2;
            if (!t_ok)
                loss = __builtin_nanf("");
            if (p.row_loss)
                p.row_loss[r] = loss;
            loss_sum += loss;
        }
    }
    if (!SPLIT) {
        sum_losses(p, loss_sum);
        return;
    }
    __shared__ float s_red[kWaves];
    __shared__ unsigned s_last;
    if (!last_to_arrive(p, &s_last))
        return;
    // a thread combines the segments of every 256th row, in order; all of a row's travel together (four at a
    // time, one batch after the other, they were 0.7 of 5.9 us at 1 x 4517 fp32, 16 segments)
    float acc = 0.0f;
    auto combine = [&](auto count, int r) {
        constexpr int U = decltype(count)::value;
        const float xt = read_pair(p.picked + r)[0];
        floatx2 u[U];
#pragma unroll
        for (int g = 0; g < U; ++g)
            u[g] = read_pair(p.partials + (size_t)r * segs + (g < segs ? g : segs - 1));
        float m = -INFINITY, s = 0.0f;
#pragma unroll
        for (int g = 0; g < U; ++g)
            if (g < segs) {
                const float mn = fmaxf(m, u[g][0]);
                const float ref = ref_of(mn);
                s = s * exp2_hw((m - ref) * kLog2e) + u[g][1] * exp2_hw((u[g][0] - ref) * kLog2e);
                m = mn;
            }
        const float loss = (m - xt) + __builtin_amdgcn_logf(s) * kLn2;
        if (p.row_loss)
            p.row_loss[r] = loss;
        acc += loss;
    };
    for (int r = threadIdx.x; r < p.B; r += kThreads) {
        if (segs <= 4)
            combine(std::integral_constant<int, 4>(), r);
        else if (segs <= 8)
            combine(std::integral_constant<int, 8>(), r);
        else
            combine(std::integral_constant<int, kXentMaxSegs>(), r);
    }
    finish_mean(p, acc, s_red);
}

template <typename T, int VEC, bool PEEL>
hipError_t launch_v(const XentParams &p, hipStream_t stream)
{
#define FF_SHORT(L, Q)                                                                                               \
    case L * 16 + Q:                                                                                                 \
        hipLaunchKernelGGL((xent_short_kernel<T, VEC, L, Q, PEEL>), dim3(p.grid), dim3(kThreads), 0, stream, p);      \
        return hipGetLastError();
    switch (p.lanes * 16 + p.per_lane) {
        FF_SHORT(4, 1)
        FF_SHORT(4, 2)
        FF_SHORT(4, 4)
        FF_SHORT(16, 2)
        FF_SHORT(16, 4)
        FF_SHORT(64, 2)
        FF_SHORT(64, 4)
        FF_SHORT(64, 8)
    }
#undef FF_SHORT
    if (p.segs > 1)
        hipLaunchKernelGGL((xent_long_kernel<T, VEC, PEEL, true>), dim3(p.grid), dim3(kThreads), 0, stream, p);
    else
        hipLaunchKernelGGL((xent_long_kernel<T, VEC, PEEL, false>), dim3(p.grid), dim3(kThreads), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_xent_kernel(bool bf16, const XentParams &p, hipStream_t stream)
{
    if (p.vec == 1)
        return bf16 ? launch_v<__bf16, 1, false>(p, stream) : launch_v<float, 1, false>(p, stream);
    if (bf16)
        return p.C % 8 == 0 ? launch_v<__bf16, 8, false>(p, stream) : launch_v<__bf16, 8, true>(p, stream);
    return p.C % 4 == 0 ? launch_v<float, 4, false>(p, stream) : launch_v<float, 4, true>(p, stream);
}

}  // namespace ff
