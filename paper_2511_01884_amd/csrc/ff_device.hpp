// Device-side building blocks shared by the gfx950 kernels: bf16 <-> fp32,
// erf-form GELU, pairwise merge of (count, mean, M2) row statistics, and the
// workspace layout the kernels and the host agree on.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ff {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));

// ---- workspace layout (bytes from the workspace base) ----------------------
// [0, 4)                error word: non-zero once a wait inside a launch gave up
// [256, CTRL_BYTES)     arrival / departure counters, two uint32 per row-block (row_counter); zero between launches
// [CTRL_BYTES, ...)     per-tile row statistics (float2 mean, M2), then the
//                       two-pass variant's fp32 G; other entry points' scratch
constexpr size_t kCtrlBytes = 1u << 20;
constexpr size_t kCounterOffset = 256;
constexpr int64_t kMaxRowBlocks = (int64_t)((kCtrlBytes - kCounterOffset) / 8);

// Index of a row-block's counter pair.  The row-blocks of a round arrive at the same time, and words that share a line
// are one queue at the memory side (6 ns an access, polls included): 256 consecutive row-blocks have pairs 256 bytes
// apart.  Side by side, the last of 240 workgroups in four row-blocks of 60 tiles took 3.2 us from its arrival to seeing
// it, now 1.4, which every round of tiles waits for (6912 x 256 x 15208 bf16 222 -> 202 us, 8192 x 4096 x 16384 982 ->
// 950, 65536 x 1024 x 1024 178 -> 175); pairs 4 KiB apart are no faster.  One to one on every block of 8192; beyond the
// last whole one that fits the control region, in order.
constexpr int kRowCounterStride = 32;  // pairs
constexpr int kRowCounterBlock = 256 * kRowCounterStride;
__host__ __device__ __forceinline__ int row_counter(int rb)
{
    constexpr int kWhole = (int)(kMaxRowBlocks / kRowCounterBlock) * kRowCounterBlock;
    return rb < kWhole ? rb / kRowCounterBlock * kRowCounterBlock + (rb & 255) * kRowCounterStride +
                             ((rb >> 8) & (kRowCounterStride - 1))
                       : rb;
}
// Counter pairs that hold those of the first `row_blocks` row-blocks.
inline int row_counter_pairs(int row_blocks)
{
    constexpr int kWhole = (int)(kMaxRowBlocks / kRowCounterBlock) * kRowCounterBlock;
    if (row_blocks <= 256)
        return row_counter(row_blocks - 1) + 1;
    return row_blocks > kWhole ? row_blocks : (row_blocks + kRowCounterBlock - 1) / kRowCounterBlock * kRowCounterBlock;
}

// Workgroup barrier that carries no fence: unlike __syncthreads() it does not wait for outstanding
// global loads, so loads requested ahead (registers or direct-to-LDS) stay in flight across it;
// their completion is awaited explicitly with vmcnt where it matters.  It waits for this wave's own
// LDS reads and writes, and the barrier instruction itself is a compiler-level ordering point for
// memory operations.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) only
    __builtin_amdgcn_s_barrier();
}

// ---- bf16 <-> fp32 -----------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(unsigned short h)
{
    return __uint_as_float(((unsigned)h) << 16);
}
__device__ __forceinline__ float load_as_float(const float *p) { return *p; }
__device__ __forceinline__ float load_as_float(const __bf16 *p)
{
    return bf16_bits_to_float(*reinterpret_cast<const unsigned short *>(p));
}
// Round-to-nearest-even pack of two floats (hardware conversion on gfx950).
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi)
{
    floatx2 v = {lo, hi};
    bf16x2 h = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<unsigned *>(&h);
}

// ---- GELU, erf form -----------------------------------------------------------
// g = z * Phi(z), Phi the standard normal distribution function, Phi(z) = 0.5 * erfc(-z / sqrt 2).
// With q = Phi(-|z|) evaluated directly (no 1 + erf cancellation), g = max(z, 0) - |z| q for either
// sign of z.  q is smooth, positive and falls like exp(-z^2 / 2), so its base-2 logarithm is close to
// a low-degree polynomial: q ~ 2^P(|z|), P of degree 5, fitted (fit_gelu_tail.py beside this file) so
// that the error of |z| q, which is the error of g, is below 4.7e-7 for every z; P has a negative
// leading coefficient and no real stationary point, so 2^P decays to 0 for large |z|.  One hardware
// 2^x (1 ulp) and five multiply-adds: the epilogue's cost per element is what matters here, the
// matrix pipe is idle while it runs.
__device__ __forceinline__ float gelu_erf(float z)
{
    const float x = fabsf(z);
    float p = -0.000473293995f;
    p = fmaf(p, x, 0.00708446082f);
    p = fmaf(p, x, -0.051827167f);
    p = fmaf(p, x, -0.459992648f);
    p = fmaf(p, x, -1.15078777f);
    p = fmaf(p, x, -1.00003763f);
    const float q = __builtin_amdgcn_exp2f(p);
    return fmaf(-x, q, fmaxf(z, 0.0f));
}

// ---- (count, mean, M2) merge (Chan et al. pairwise update) ---------------------
// Folds block b into block a:  delta = mean_b - mean_a; n = n_a + n_b;
// mean = mean_a + delta * n_b / n;  M2 = M2_a + M2_b + delta^2 * n_a * n_b / n.
__device__ __forceinline__ void merge_stats(float &na, float &mean_a, float &m2a,
                                            float nb, float mean_b, float m2b)
{
    const float n = na + nb;
    if (n > 0.0f) {
        const float inv = 1.0f / n;
        const float delta = mean_b - mean_a;
        mean_a = fmaf(delta, nb * inv, mean_a);
        m2a = m2a + m2b + delta * delta * (na * nb * inv);
    }
    na = n;
}

// Cross-workgroup exchange of row statistics.  Workgroups of one launch run on
// different XCDs with separate L2 caches, so the 8-byte (mean, M2) partials are
// written and read with device-scope atomic accesses: the store writes through to
// the level all XCDs share, the load never takes a stale line of the local L2.
// A full fence (L2 write-back plus invalidate) would also be correct but costs
// tens of microseconds per launch.  Ordering: every publishing thread waits for
// its own stores to complete (vmcnt), the workgroup meets at a barrier, and only
// then one thread bumps the arrival counter; readers load the partials after they
// have seen the counter reach its target.
__device__ __forceinline__ void publish_pair(floatx2 *p, floatx2 v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p),
                       __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ floatx2 read_pair(const floatx2 *p)
{
    const unsigned long long bits = __hip_atomic_load(
        reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(floatx2, bits);
}
// This thread's published partials have reached the shared level.
__device__ __forceinline__ void wait_published()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
}

__device__ __forceinline__ unsigned atomic_add_device(unsigned *p, unsigned v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned atomic_load_device(const unsigned *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_store_device(unsigned *p, unsigned v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wait (bounded) until *counter >= target.  Returns false if the bound expired.
// One thread calls this; the rest of the workgroup waits at a barrier.  The clock
// is read only every 256 polls: reading it costs as much as a poll.
__device__ __forceinline__ bool wait_counter(const unsigned *counter, unsigned target,
                                             long long limit_ticks)
{
    if (atomic_load_device(counter) >= target)
        return true;
    const long long t0 = wall_clock64();
    for (;;) {
        for (int i = 0; i < 256; ++i) {
            __builtin_amdgcn_s_sleep(1);
            if (atomic_load_device(counter) >= target)
                return true;
        }
        if (wall_clock64() - t0 > limit_ticks)
            return false;
    }
}

// Grid-wide arrival spread over several counters.  A few hundred workgroups bumping and polling one
// word queue up behind each other at the memory side; with kSyncWays words on different
// 4 KiB pages the queues are kSyncWays times shorter.  Way w of the control region's counter
// array: arrivals at [w * kSyncStride], departures at [w * kSyncStride + 1]; word [2] counts the
// ways whose workgroups have all departed.
constexpr int kSyncWays = 32;
constexpr int kSyncStride = 1024;  // uint32 words between ways

// Departure from such a meeting: the last workgroup of the last way re-arms every counter (only then has every workgroup
// left its wait, so that no poller can see a counter go back to zero).  In three steps, one thread's, begun as soon as
// the workgroup's own wait is over: the two round trips to memory pass behind the work that follows, and do not
// stand at the end of the kernel (16 x 8192 x 8192 36.6 us, now 36.2; second chain 300 x 4096 x 1024 12.4, 11.9).
// Departures are counted in lines that nobody polls.  Beside a way's arrivals they hold up whoever still waits: the second
// chain with more than 40 KiB of X a unit took 1.01 (90 drawn shapes; at most 1.08) of its time with departures at the end of the kernel,
// in lines of their own 0.98 (at most 1.01; 4222 x 2048 x 868 fp32 16.7 us, 18.1, now 16.4).
constexpr int kSyncDeparted = 32;            // uint32 words from a way's arrivals to its departures
constexpr int kSyncWaysDeparted = 64;        // and, from the first way's arrivals, to the ways that all have left
static_assert(kSyncWaysDeparted < kSyncStride, "inside the first way's own words");
struct Departure {
    unsigned seen = 0;
    __device__ __forceinline__ void begin(unsigned *counters, unsigned way)
    {
        seen = atomic_add_device(counters + (size_t)way * kSyncStride + kSyncDeparted, 1u);
    }
    // behind the loads that the workgroup waits for next
    __device__ __forceinline__ void middle(unsigned *counters, unsigned way, unsigned grid)
    {
        const bool last = seen == (grid + kSyncWays - 1 - way) / kSyncWays - 1u;
        seen = last ? atomic_add_device(counters + kSyncWaysDeparted, 1u) + 1u : 0u;
    }
    __device__ __forceinline__ void end(unsigned *counters, unsigned grid)
    {
        if (seen == (grid < (unsigned)kSyncWays ? grid : (unsigned)kSyncWays)) {
            for (int w = 0; w < kSyncWays; ++w) {
                atomic_store_device(counters + (size_t)w * kSyncStride, 0u);
                atomic_store_device(counters + (size_t)w * kSyncStride + kSyncDeparted, 0u);
            }
            atomic_store_device(counters + kSyncWaysDeparted, 0u);
        }
    }
};

// Called by every lane of one wavefront: the lanes with `polls` set wait for their own word `mine` to
// reach their `target` (sticky: a word counts once seen).  False if the bound expired.
__device__ __forceinline__ bool wait_ways(const unsigned *mine, bool polls, unsigned target, long long limit_ticks)
{
    bool seen = !polls || atomic_load_device(mine) >= target;
    if (__all(seen))
        return true;
    const long long t0 = wall_clock64();
    for (;;) {
        for (int i = 0; i < 256; ++i) {
            __builtin_amdgcn_s_sleep(1);
            if (!seen)
                seen = atomic_load_device(mine) >= target;
            if (__all(seen))
                return true;
        }
        if (wall_clock64() - t0 > limit_ticks)
            return false;
    }
}

// Lane l < kSyncWays polls way l.
__device__ __forceinline__ bool wait_counters_wave(const unsigned *counters, unsigned target,
                                                   long long limit_ticks)
{
    const int lane = threadIdx.x & 63;
    const bool polls = lane < kSyncWays;
    return wait_ways(counters + (size_t)(polls ? lane : 0) * kSyncStride, polls, target, limit_ticks);
}

}  // namespace ff
