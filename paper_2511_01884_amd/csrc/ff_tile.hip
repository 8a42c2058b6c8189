// Tiled MFMA path of the fused linear + erf-GELU + LayerNorm operator (gfx950).
//
// One workgroup (4 or 8 wavefronts) owns a BM x BN tile of the output and walks K in
// 128-byte slabs (whole cache lines: one L2 request per line).  X and W slabs go
// HBM -> LDS with 16-byte direct-to-LDS loads into STAGES stages (two or three); the loads of the
// slab STAGES further on are issued in the shadow of the MFMAs, the single barrier per slab
// sits in its last k-step, and MFMA fragments are read one k-step ahead of
// their use, so the matrix pipe does not wait on LDS latency after the barrier.  The MFMA is issued
// "transposed" (A operand = W rows, B operand = X rows), so that a lane's
// accumulator registers run along N — the LayerNorm reduction
// axis — and the row statistics need only one or two cross-lane steps.
//
// The epilogue never leaves the registers (the fused-epilogue pattern of the
// paper's App. B.1 case, with the "cross-tile aggregation" it names as the hard
// part): bias + GELU in place, per-row (mean, M2) of the tile, exchange of those
// 8-byte partials with the other tiles of the same rows through global memory
// and an arrival counter, merge in fixed order, normalise, convert, and store Y
// through an LDS transpose in 16-byte coalesced rows.  G is never written to
// global memory (Sec. 4: removing the second global read).
//
// Modes: kFused (above), kTwoPass (writes fp32 G and the partials; a second
// kernel normalises — used when a row has more tiles than co-resident
// workgroups), kLinearOnly (test hook: fp32 Z = X W^T + b).
#include <algorithm>

#include "ff_tile.hpp"

namespace ff {

namespace {

constexpr int kRowBytes = 128;  // bytes of one tile row per K slab (8 chunks of 16 B)
constexpr int kChunksPerRow = kRowBytes / 16;
constexpr int kRowsPerDma = 1024 / kRowBytes;     // one direct-to-LDS instruction fills 1 KiB

// The matrix instruction of a type: blocks of kBlock x kBlock outputs, whose kLaneGroups lane groups hold one
// 16-byte chunk along K each, so that a k-step takes kLaneGroups chunks of a row.  A lane's results are those of
// row lane % kBlock (of X), columns 4 (kLaneGroups q + group) + (0..3), q = 0 .. kQuads - 1.
//
// bf16 multiplies in blocks of 16: the chip's power sets the rate of a long product, and a 16 x 16 x 32 instruction
// moves half the accumulators of a 32 x 32 x 16 one for each product.  Nothing but either in a loop, random operands:
// 2002 against 1774 TFLOP/s.  fp32 is bound by the issue of its matrix instructions, whatever their shape.
//
// FULL: the accumulators take one half of the register file to the last register (256 x 256 by four wavefronts).  Blocks of
// 32 there in bf16 too: with sixty-four blocks of 16 and no register to spare the compiler moved them about, 264
// copies for the 128 instructions of a slab.
template <typename T, bool FULL>
struct Mma;

template <>
struct Mma<__bf16, false> {
    using Acc = floatx4;
    static constexpr int kBlock = 16, kLaneGroups = 4, kQuads = 1;
    static __device__ __forceinline__ void step(const uintx4 &a, const uintx4 &b, Acc &c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                    __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};

template <>
struct Mma<__bf16, true> {
    using Acc = floatx16;
    static constexpr int kBlock = 32, kLaneGroups = 2, kQuads = 4;
    static __device__ __forceinline__ void step(const uintx4 &a, const uintx4 &b, Acc &c)
    {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                    __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};

template <bool FULL>
struct Mma<float, FULL> {
    using Acc = floatx16;
    static constexpr int kBlock = 32, kLaneGroups = 2, kQuads = 4;
    // One 16-byte fragment per lane holds 4 floats along K: four 32x32x2 MFMAs.
    static __device__ __forceinline__ void step(const uintx4 &a, const uintx4 &b, Acc &c)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]),
                                                     c, 0, 0, 0);
    }
};

// Compiler-level ordering of LDS traffic inside one wavefront (the LDS itself
// serves a wave's requests in issue order).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Ordering point for the instruction scheduler: the listed accumulators must have
// been produced before it, and no memory operation moves across it.  The constraint also says where
// they live.  Where a wavefront's 256 registers hold everything, the accumulators are ordinary vector
// registers, which the epilogue reads and writes as they are: as accumulation registers they cost two
// copies an element in the GELU pass and one before the stores (v_accvgpr_read, _write: 640 of 2900 vector instructions
// of an epilogue) and 46 registers more (before the loop had 16 x 16 x 32 instructions: 1018 x 256 x 10944 bf16
// 25.9 -> 25.1 us, 6912 x 256 x 15208 196 -> 186).  Only
// the four-wavefront 256 x 256 tile, whose accumulators alone are 256 registers, needs the other half of the register file.
template <bool kAcc, typename Acc> __device__ __forceinline__ void pin_order(Acc &c)
{
    if (kAcc)
        asm volatile("" : "+a"(c) : : "memory");
    else
        asm volatile("" : "+v"(c) : : "memory");
}

// s_waitcnt vmcnt(n), n < 64, nothing else
template <int n> __device__ __forceinline__ void wait_vm()
{
    __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | ((n >> 4) << 14));
}

// The lane index, computed where it is asked for: the compiler can neither move the computation out
// of a loop nor keep its result across one (values that the K loop does not use would have to be
// carried across it in scratch memory).
__device__ __forceinline__ int opaque_lane()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}
// The value of a uniform integer, hidden from the optimiser in the same way.
__device__ __forceinline__ int opaque_uniform(int v)
{
    int r;
    asm volatile("s_mov_b32 %0, %1" : "=s"(r) : "s"(v));
    return r;
}
// Another lane's value, through the LDS crossbar.
__device__ __forceinline__ float from_lane(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(lane << 2, __float_as_int(v)));
}

// LDS placement of 16-byte chunk `c` (0..7) of tile row `row`: slot c ^ swizzle, so that the rows a fragment read touches
// spread over all 64 banks (two rows to 256 bytes).  The LDS serves such a read sixteen lanes at a time, 0-3 with 12-15,
// 20-23 and 24-27 and so on: in blocks of 32 sixteen rows of one chunk, in blocks of 16 eight rows of one chunk and the
// eight between them of its neighbour.  This swizzle has no conflict in either (255 bytes a clock of a unit read by eight
// wavefronts; with row & 7 ^ row >> 3 & 1, free in blocks of 32 only, 128 in blocks of 16, and half of a bf16 product's LDS
// cycles were conflicts).  The chip's power sets the rate of a long product, so that the time gains little: 4096^3 bf16 105.9 ->
// 105.3 us, 8192 x 4096 x 16384 861 -> 856, 16384 x 512 x 4096 110.8 -> 109.6.
__device__ __forceinline__ int swizzle_of_row(int row) { return (row >> 1) & 7; }

// RAGGED_N: N is not a multiple of the tile width, so the last tile of each row
// masks the columns at or beyond N in the statistics (chosen on the host).
//
// Wave layout: kWavesN x kWavesM wavefronts, each owning WTN x WTM times 32 x 32 outputs.  The
// 256-tile runs as 2 x 4 wavefronts of 4 x 2 blocks (two wavefronts per SIMD: 128 accumulator
// registers each, and eight wavefronts keep twice as many loads in flight on the L2 -> LDS path
// as four) or as 2 x 2 wavefronts of 4 x 4 blocks; the 256 x 128 tile as 4 x 2 wavefronts of 2 x 2 blocks; the 128-
// and 64-tiles as 2 x 2 wavefronts, two workgroups per compute unit (second launch bound: two wavefronts per SIMD must fit).
//
// STAGES: slabs the LDS has room for beside the parameters, two at 256 x 256 and where two workgroups share a unit,
// three at 256 x 128 (one per unit): there two slabs travel while one is multiplied.
//
// LINES: what travels is not a tile row's 128 bytes of a slab but the 128-byte line of memory that holds its beginning, so that
// rows that do not begin on line boundaries still have one request a slab (a unit's load path takes 27 bytes a clock and a
// line at a time).  Rows begin on 16-byte boundaries, that is on a chunk: chunk c of a row's slab i is chunk (c + lead) % 8 of its
// line i, or of line i + 1 where c + lead >= 8, and lies in LDS at the slot that it would have without the shift, so that
// only the stage it is read from differs between lanes.  Slab i needs lines i and i + 1: three stages, two slabs' time less
// one.  4462 x 3848 x 952 67.9 us, now 61.8; 1024 x 4104 x 8192 72.6, 65.6; the same bits.
//
// Launch bound: 512 threads also where four wavefronts are launched, if 256 registers hold all of one's values.  Left with
// 512, the compiler keeps the accumulators in the other half and copies them out and back at every pin_order.
constexpr int launch_bound(int waves, int part) { return part >= 16 ? 64 * waves : 512; }

template <typename T, int kWavesN, int kWavesM, int WTN, int WTM, int MODE, bool RAGGED_N, int STAGES, bool LINES>
__global__ __launch_bounds__(launch_bound(kWavesN * kWavesM, WTN * WTM), (kWavesN * kWavesM * WTN * WTM <= 32) ? 2 : 1)
void tile_kernel(const TileParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)  // the body uses device-only types (buffer descriptors)
    constexpr int kWaves = kWavesN * kWavesM;
    constexpr int kThreads = 64 * kWaves;
    constexpr int BN = kWavesN * WTN * 32;
    constexpr int BM = kWavesM * WTM * 32;
    constexpr bool kAccRegs = WTN * WTM >= 16;
    using Product = Mma<T, kAccRegs>;
    using Acc = typename Product::Acc;
    constexpr int kBlock = Product::kBlock, kLaneGroups = Product::kLaneGroups;
    constexpr int kBlocksN = WTN * 32 / kBlock, kBlocksM = WTM * 32 / kBlock;  // matrix blocks of a wavefront
    constexpr int kSteps = kChunksPerRow / kLaneGroups;                        // k-steps of a slab
    constexpr int kChunkElems = 16 / (int)sizeof(T);
    constexpr int kSlabElems = kRowBytes / (int)sizeof(T);
    constexpr int kABytes = BN * kRowBytes;
    constexpr int kBBytes = BM * kRowBytes;
    // LDS placement of the slabs: slab s in stage s % STAGES, W rows first
    constexpr int kStageBytes = kABytes + kBBytes;
    constexpr int kSlabLdsBytes = STAGES * kStageBytes;
    // direct-to-LDS instructions per wave per slab
    constexpr int kDmaA = BN / kRowsPerDma / kWaves;
    constexpr int kDmaB = BM / kRowsPerDma / kWaves;
    constexpr int kDmaPerSlab = kDmaA + kDmaB;
    // epilogue LDS regions (reuse the stage buffers)
    using OutT = typename std::conditional<MODE == kFused, T, float>::type;
    constexpr int kOutRowBytes = WTN * 32 * (int)sizeof(OutT);
    constexpr int kOutPitch = kOutRowBytes + 16;
    constexpr int kOffWst = 0;                               // kWavesN * BM float2
    constexpr int kOffRst = kOffWst + kWavesN * BM * 8;      // BM float2
    constexpr int kOffOut = (kOffRst + BM * 8 + 1023) & ~1023;
    constexpr int kEpiBytes = kOffOut + kWaves * 32 * kOutPitch;
    constexpr int kSmemBytes = (kSlabLdsBytes > kEpiBytes) ? kSlabLdsBytes : kEpiBytes;

    // One LDS object for everything: with a second one the compiler can no longer tell the DMA's LDS
    // writes from the fragment reads and waits for all loads in flight before every read.
    constexpr int kPrmBytes = 3 * BN * 4;
    __shared__ __attribute__((aligned(1024))) char smem[kSmemBytes + kPrmBytes];
    // Bias, gamma and beta of the tile's columns: requested ahead of the first slab and parked in LDS of their own
    // when it has landed, so that the epilogue finds them there.
    constexpr int kPrmPerThread = (3 * BN + kThreads - 1) / kThreads;
    float *s_prm = reinterpret_cast<float *>(smem + kSmemBytes);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave % kWavesN;
    const int wm = wave / kWavesN;

    // Phase timestamps (test hook): when a timeline buffer is bound, thread 0 of every workgroup writes
    // the wall clock at the phase boundaries of each of its first `timeline_rounds` tiles into
    // timeline[(round * grid + workgroup) * kTimelineSlots + k].
    int round = 0;
    bool stamper = false;  // thread 0 of the workgroup, decided per tile
    auto stamp = [&](int k) {
        if (p.timeline != nullptr && stamper && round < p.timeline_rounds)
            p.timeline[((size_t)round * gridDim.x + blockIdx.x) * kTimelineSlots + k] =
                k < kTimelineCycleSlot ? wall_clock64() : clock64();
    };

    bool first_tile = true;
    for (; round < p.rounds; ++round) {
        // ---- tile coordinates (XCD-aware order inside a round when enabled) ----
        int rb, cb;
        if (p.swz_sc_log2 >= 0) {
            // 8 XCDs x (grid / 8) workgroups, grid and NT powers of two: all quotients are shifts.
            // XCD x takes a block of sr x sc tiles (sc = 1 << swz_sc_log2 columns, sr = grid / 8 / sc
            // rows) of the round's (grid / NT) x NT tiles; the workgroups of the second half of the
            // grid take the lower rows of their XCD's block.
            const int xcd = blockIdx.x & 7;
            const int slot = blockIdx.x >> 3;
            const int scl = p.swz_sc_log2;
            const int across_log2 = p.nt_log2 - scl;
            const int sbr = xcd >> across_log2, sbc = xcd & ((1 << across_log2) - 1);
            rb = (round << (p.grid_log2 - p.nt_log2)) + (sbr << (p.grid_log2 - 3 - scl)) + (slot >> scl);
            cb = (sbc << scl) + (slot & ((1 << scl) - 1));
        } else if (p.round_rows > 0) {
            // A round takes round_rows whole row-blocks (grid = round_rows * NT).  The workgroups of one XCD
            // get consecutive numbers, row-block fastest: a block of round_rows x a few tiles, which share
            // their X and W panels in its L2.
            const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
            const int each = (int)gridDim.x >> 3, more = (int)gridDim.x & 7;
            const int t = xcd * each + (xcd < more ? xcd : more) + slot;
            cb = t / p.round_rows;
            rb = round * p.round_rows + t - cb * p.round_rows;
        } else {
            const int t = round * (int)gridDim.x + (int)blockIdx.x;
            rb = t / p.NT;
            cb = t - rb * p.NT;
        }
        if (rb >= p.RB)
            continue;  // uniform for the workgroup
        // Everything derived from the lane index and from the shape is computed here, per tile, where
        // it is used.
        const int lane = opaque_lane();
        const int M = opaque_uniform(p.M), N = opaque_uniform(p.N), K = opaque_uniform(p.K);
        const int slabs = (K + kSlabElems - 1) / kSlabElems;
        const bool k_ragged = (K % kSlabElems) != 0;
        const size_t row_stride = (size_t)K * sizeof(T);
        stamper = wave == 0 && lane == 0;
        stamp(0);
        const int m0 = rb * BM;
        const int n0 = cb * BN;
        const int group = lane / kBlock;
        const int block_row = lane % kBlock;
        // fragment read offsets (bytes inside a stage); k-step s reads chunk (s * kLaneGroups + group) ^ swizzle
        const int frag_swz = swizzle_of_row(block_row);
        const int a_frag_base = (wn * WTN * 32 + block_row) * kRowBytes;
        const int b_frag_base = kABytes + (wm * WTM * 32 + block_row) * kRowBytes;
        // DMA lane geometry: lane -> (row within a 16-row group, stored chunk slot)
        const int dma_r = lane / kChunksPerRow;
        const int dma_cs = lane % kChunksPerRow;
        // LINES: a row's first chunk is chunk `lead` of its first line; a tile begins at a multiple of eight rows, so that the
        // lead of its row r is (phase + r * row_chunks) % 8.
        const int row_chunks = K / kChunkElems;
        const int w_phase = LINES ? (int)(reinterpret_cast<uintptr_t>(p.W) >> 4) & 7 : 0;
        const int x_phase = LINES ? (int)(reinterpret_cast<uintptr_t>(p.X) >> 4) & 7 : 0;
        auto lead = [&](int phase, int r) { return LINES ? (phase + r * row_chunks) & 7 : 0; };
        const int a_lead = lead(w_phase, block_row), b_lead = lead(x_phase, block_row);
        // where the line (LINES) or slab of row r begins, and the chunk of it that lies in `slot` of row `row` in LDS
        auto line_offset = [&](int phase, int row, int r, int slot) {
            const unsigned at = (unsigned)r * (unsigned)row_stride + phase * 16;
            return (LINES ? at & ~127u : at) + ((((slot ^ swizzle_of_row(row)) + lead(phase, r)) & 7) << 4);
        };

        // ---- per-lane byte offsets of the DMA sources, relative to the tile's first row ----
        const char *w_tile = (const char *)p.W - w_phase * 16 + (size_t)n0 * row_stride;
        const char *x_tile = (const char *)p.X - x_phase * 16 + (size_t)m0 * row_stride;
        unsigned offa[kDmaA], offb[kDmaB];
#pragma unroll
        for (int j = 0; j < kDmaA; ++j) {
            const int row = wave * (BN / kWaves) + j * kRowsPerDma + dma_r;
            const int rr = (n0 + row < N) ? row : (N - 1 - n0);  // clamp to the last valid row
            offa[j] = line_offset(w_phase, row, rr, dma_cs);
        }
#pragma unroll
        for (int j = 0; j < kDmaB; ++j) {
            const int row = wave * (BM / kWaves) + j * kRowsPerDma + dma_r;
            const int rr = (m0 + row < M) ? row : (M - 1 - m0);
            offb[j] = line_offset(x_phase, row, rr, dma_cs);
        }

        // full slab: direct-to-LDS, nothing passes through registers.  dma_one issues
        // the x-th of the wave's kDmaPerSlab instructions (W rows first, then X rows).
        // Buffer descriptors over the tile's rows: the per-lane 32-bit byte offset is
        // the loop-invariant part of a load's address, the slab offset rides in a scalar
        // register, so a DMA instruction costs no vector ALU work.  All addresses are
        // clamped in-bounds above; K is bounded so that a tile's rows span at most kRangeBytes, and an
        // offset of kRangeBytes is outside: such a lane reads zeros (dma_cut).
        constexpr unsigned kRangeBytes = 0x80000000u;
        const __amdgpu_buffer_rsrc_t w_rsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(w_tile), 0, kRangeBytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t x_rsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(x_tile), 0, kRangeBytes, 0x00020000);
        auto dma_one = [&](int slab, int stage, int x) {
            char *st = smem + stage * kStageBytes;
            if (x < kDmaA) {
                char *sa = st + wave * (BN / kWaves) * kRowBytes;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    w_rsrc, (__attribute__((address_space(3))) void *)(sa + x * 1024), 16,
                    offa[x < kDmaA ? x : 0], slab * kRowBytes, 0, 0);
            } else {
                const int y = x - kDmaA;
                char *sb = st + kABytes + wave * (BM / kWaves) * kRowBytes;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    x_rsrc, (__attribute__((address_space(3))) void *)(sb + y * 1024), 16,
                    offb[y >= 0 && y < kDmaB ? y : 0], slab * kRowBytes, 0, 0);
            }
        };
        // The last slab when K cuts it: a lane whose chunk lies at or beyond K reads outside the descriptor's range,
        // which puts zeros into its place in LDS.  (Through registers, with zeros
        // written for the missing chunks, it was a load latency in the open: 3001 x 2056 x 5000 spent 54.5 us up
        // to the end of the product, against 46.2 for K = 2048.)  In the loop's last steady step these loads stand one
        // behind the other after the barrier, each in a loop of one round over the lanes (the compiler keeps the slab's
        // offset in a vector register), not between the products as the uncut slabs' do.
        auto dma_cut = [&](int slab, int stage, int half) {
            // lane geometry re-derived through an opaque move: this rarely taken path
            // must not have its offsets precomputed (and spilled) at kernel entry
            const int lane_c = opaque_lane();
#pragma unroll
            for (int x = 0; x < (half == 0 ? kDmaA : kDmaB); ++x) {
                const int row = wave * ((half == 0 ? BN : BM) / kWaves) + x * kRowsPerDma + lane_c / kChunksPerRow;
                const int c = (lane_c % kChunksPerRow) ^ swizzle_of_row(row);
                int first = slab * kChunksPerRow;  // chunk of the matrix row that the slab or line begins with
                if (LINES) {
                    const int last = half == 0 ? N - 1 - n0 : M - 1 - m0;
                    first -= c + lead(half == 0 ? w_phase : x_phase, row < last ? row : last) >= 8 ? 8 : 0;
                }
                const bool in = (unsigned)(first + c) < (unsigned)row_chunks;
                char *dst = smem + stage * kStageBytes + (half == 0 ? 0 : kABytes) +
                            wave * ((half == 0 ? BN : BM) / kWaves) * kRowBytes + x * 1024;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    half == 0 ? w_rsrc : x_rsrc, (__attribute__((address_space(3))) void *)dst, 16,
                    in ? (half == 0 ? offa[x < kDmaA ? x : 0] : offb[x < kDmaB ? x : 0]) : kRangeBytes, slab * kRowBytes, 0, 0);
            }
            asm volatile("");  // keeps the last instruction apart from the uncut slab's: merged, every fragment read waits for both
        };

        // The accumulators start from a zero the optimiser cannot see through: given a constant it
        // parks a block of sixteen zeros in scratch memory for the path that skips the steady iterations.
        float zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        Acc acc[kBlocksN][kBlocksM];
#pragma unroll
        for (int i = 0; i < kBlocksN; ++i)
#pragma unroll
            for (int j = 0; j < kBlocksM; ++j)
#pragma unroll
                for (int r = 0; r < 4 * Product::kQuads; ++r)
                    acc[i][j][r] = zero;

        // Fragments: W's in one buffer, each read again for the next k-step as soon as its products are issued; X's,
        // which every group of products reads, in two, by k-step.
        uintx4 fa[kBlocksN], fb[2][kBlocksM];
        // byte offset of k-step s of the slab in `stage`; LINES: the line behind it where the shift carries the chunk there
        auto step_offset = [&](int stage, int s, int ld) {
            const int c = s * kLaneGroups + group;
            const int ahead = stage + 1 < STAGES ? kStageBytes : -(STAGES - 1) * kStageBytes;
            return stage * kStageBytes + ((c ^ frag_swz) << 4) + (LINES && c + ld >= 8 ? ahead : 0);
        };
        auto read_a = [&](int stage, int s, int x) {
            fa[x] = *reinterpret_cast<const uintx4 *>(smem + step_offset(stage, s, a_lead) + a_frag_base + x * kBlock * kRowBytes);
        };
        auto read_b = [&](int stage, int s, int x) {
            fb[s & 1][x] = *reinterpret_cast<const uintx4 *>(smem + step_offset(stage, s, b_lead) + b_frag_base +
                                                             x * kBlock * kRowBytes);
        };
        // The products of a k-step are issued in groups, one per fragment of W.
        auto products = [&](int g, int s) {
#pragma unroll
            for (int j = 0; j < kBlocksM; ++j)
                Product::step(fa[g], fb[s & 1][j], acc[g][j]);
        };
        auto end_group = [&](int g) {
#pragma unroll
            for (int j = 0; j < kBlocksM; ++j)
                pin_order<kAccRegs>(acc[g][j]);
            __builtin_amdgcn_sched_barrier(0);
        };
        static_assert(kBlocksM <= kBlocksN && kSteps % 2 == 0, "the X fragments of the next k-step, one per group");
        // k-step s of the slab in `stage`, not its last: the next one's fragments are read behind its products.
        // (Always in line: a call, which the compiler prefers for the 256 x 256 tile of four wavefronts in fp32, takes
        // everything that the body names through scratch memory, accumulators and all.)
        auto step_inside = [&](int stage, int s) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < kBlocksN; ++g) {
                if (g < kBlocksM)
                    read_b(stage, s + 1, g);
                products(g, s);
                read_a(stage, s + 1, g);
                end_group(g);
            }
        };
        auto steps_inside = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s + 1 < kSteps; ++s)
                step_inside(stage, s);
        };

        // ---- main loop over K slabs ----
        // Every group of products has the fragment reads of the next k-step, and in a slab's last k-step the direct-to-LDS
        // loads of the slab that takes its stage, in its shadow.  The slab's one barrier stands in its last k-step, behind
        // the first kSync groups, which cover the last fragment reads: there slab i + 1 has landed for everyone and
        // everyone has read slab i, whose stage takes slab i + STAGES.  So a load has STAGES - 1 slabs' time to arrive.
        // (Loads in a burst behind the barrier, or spread into the next slab, cost 2 to 6 %.)
        constexpr int kSync = kBlocksN >= 8 ? 2 : (kBlocksN > 1 ? 1 : 0);
        static_assert((STAGES == 2 || STAGES == 3) && kSync < kBlocksN, "the waits of the last slabs; reads behind the barrier");
        enum { kNoDma = 0, kDmaFull = 1, kDmaCut = 2 };
        auto request = [&](int slab, int stage) {
            if (!LINES && (!k_ragged || slab + 1 < slabs)) {
#pragma unroll
                for (int x = 0; x < kDmaPerSlab; ++x)
                    dma_one(slab, stage, x);
            } else {
                dma_cut(slab, stage, 0);
                dma_cut(slab, stage, 1);
            }
        };
        // The previous tile's epilogue is done with the LDS once every wave is here (its LDS reads
        // completed before its stores could issue).  No wait for those stores: they drain while the
        // first slab of this tile travels.
        // The parameter loads are the oldest loads in flight: every wait for a slab below covers them.
        // Entry c of [bias | gamma | beta] goes to thread c % kThreads; loads never branch (what has
        // no source reads the first element of W and is replaced by the default).
        float prm[kPrmPerThread];
#pragma unroll
        for (int u = 0; u < kPrmPerThread; ++u) {
            const int c = wave * 64 + lane + u * kThreads;
            const int which = c / BN;
            const int n = n0 + (c & (BN - 1));
            const T *src = reinterpret_cast<const T *>(which == 0 ? p.b : (which == 1 ? p.gamma : p.beta));
            const bool ok = which < 3 && n < N && src != nullptr;
            const float v = load_as_float(ok ? src + n : reinterpret_cast<const T *>(p.W));
            prm[u] = ok ? v : (which == 1 ? 1.0f : 0.0f);
        }
        lds_barrier();
        request(0, 0);
        constexpr int kFirst = LINES ? 2 : 1;  // slabs or lines that the first slab's products need
        const int requests = LINES ? slabs + 1 : slabs;
        if (LINES)
            request(1, 1);
        // (The slabs after the first are requested behind the first fragment reads: their instructions ahead of the wait
        // delayed the start of every tile by 1 us.  A workgroup's first tile has nothing to wait for but slab 0.)
        const bool ahead = first_tile && p.timeline == nullptr && requests >= STAGES;
        auto request_early = [&]() {
#pragma unroll
            for (int t = kFirst; t < STAGES; ++t)
                if (t < requests)
                    request(t, t);
        };
        if (ahead) {
            request_early();
            wait_vm<(STAGES - kFirst) * kDmaPerSlab>();  // slab 0 landed
        } else {
            wait_vm<0>();  // also the previous tile's stores, whose completion order relative to loads is not relied on
        }
        first_tile = false;
        // the previous tile's last readers of the parameter region passed the barrier above
#pragma unroll
        for (int u = 0; u < kPrmPerThread; ++u) {
            const int c = wave * 64 + lane + u * kThreads;
            if (c < 3 * BN)
                s_prm[c] = prm[u];
        }
        lds_barrier();
        stamp(1);
        stamp(kTimelineCycleSlot);
#pragma unroll
        for (int x = 0; x < kBlocksM; ++x)
            read_b(0, 0, x);
#pragma unroll
        for (int x = 0; x < kBlocksN; ++x)
            read_a(0, 0, x);
        if (!ahead)
            request_early();
        int i = 0, stage = 0;  // slab i lies in `stage`
        // The last k-step of slab i; `dma`: what to do about slab i + STAGES, `later`: slabs behind i + 1 that are in
        // flight at its barrier, -1 if there is no slab i + 1.
        auto step_last = [&](auto later_c, auto dma_c) __attribute__((always_inline)) {
            constexpr int later = decltype(later_c)::value, dma = decltype(dma_c)::value;
            constexpr bool more = later >= 0;
            constexpr int kRest = kBlocksN - kSync;  // groups behind the barrier
            const int next = stage + 1 < STAGES ? stage + 1 : 0;
#pragma unroll
            for (int g = 0; g < kBlocksN; ++g) {
                if (more && g >= kSync) {
                    const int q = g - kSync;
                    if (q == 0) {
                        wait_vm<(more ? later : 0) * kDmaPerSlab>();  // this wave's rows of slab i + 1 have landed
                        lds_barrier();
                        if (dma == kDmaCut) {
                            dma_cut(i + STAGES, stage, 0);
                            dma_cut(i + STAGES, stage, 1);
                        }
                    }
                    if (dma == kDmaFull) {
#pragma unroll
                        for (int x = q * kDmaPerSlab / kRest; x < (q + 1) * kDmaPerSlab / kRest; ++x)
                            dma_one(i + STAGES, stage, x);
                    }
#pragma unroll
                    for (int x = q * kBlocksM / kRest; x < (q + 1) * kBlocksM / kRest; ++x)
                        read_b(next, 0, x);
                    if (q == 0) {
#pragma unroll
                        for (int x = 0; x < kSync; ++x)
                            read_a(next, 0, x);
                    }
                }
                products(g, kSteps - 1);
                if (more && g >= kSync)
                    read_a(next, 0, g);
                end_group(g);
            }
            ++i;
            stage = next;
        };
        using std::integral_constant;
        if constexpr (LINES) {
            // Slab i + 1 needs lines i + 1 and i + 2; line i is done with.  A row's end cuts its last line or the one before.
            static_assert(!LINES || STAGES == 3, "a line more than two slabs' in LDS");
            const int whole = row_chunks / 8 - 1;
            while (i + STAGES <= whole) {
                steps_inside(stage);
                step_last(integral_constant<int, 0>(), integral_constant<int, kDmaFull>());
            }
            while (i + STAGES <= slabs) {
                steps_inside(stage);
                step_last(integral_constant<int, 0>(), integral_constant<int, kDmaCut>());
            }
            while (i + 1 < slabs) {
                steps_inside(stage);
                step_last(integral_constant<int, 0>(), integral_constant<int, kNoDma>());
            }
        } else {
            while (i < slabs - STAGES - (k_ragged ? 1 : 0)) {
                steps_inside(stage);
                step_last(integral_constant<int, STAGES - 2>(), integral_constant<int, kDmaFull>());
            }
            if (k_ragged && slabs > STAGES) {
                steps_inside(stage);
                step_last(integral_constant<int, STAGES - 2>(), integral_constant<int, kDmaCut>());
            }
            if (STAGES == 3 && slabs > 2) {
                steps_inside(stage);
                step_last(integral_constant<int, 1>(), integral_constant<int, kNoDma>());
            }
            if (slabs > 1) {
                steps_inside(stage);
                step_last(integral_constant<int, 0>(), integral_constant<int, kNoDma>());
            }
        }
        steps_inside(stage);
        step_last(integral_constant<int, -1>(), integral_constant<int, kNoDma>());
        __syncthreads();  // all fragment reads done: LDS becomes epilogue scratch
        stamp(2);
        stamp(kTimelineCycleSlot + 1);

        // ---- epilogue ----
        // The lane index and the row length are taken afresh so that the epilogue's many
        // lane-dependent addresses and its float constants are computed here, once per tile,
        // instead of being hoisted out of the tile loop and carried (spilled) across the main loop.
        {
        const int lane = opaque_lane();
        const int M = opaque_uniform(p.M), N = opaque_uniform(p.N);
        const int group = lane / kBlock;
        const int block_row = lane % kBlock;
        float *s_b = s_prm;
        float *s_g = s_b + BN;
        float *s_be = s_g + BN;
        floatx2 *s_wst = reinterpret_cast<floatx2 *>(smem + kOffWst);
        floatx2 *s_rst = reinterpret_cast<floatx2 *>(smem + kOffRst);
        char *s_out = smem + kOffOut + wave * 32 * kOutPitch;

        const int ncol_wave = wn * WTN * 32;            // wave's first column inside the tile
        const int nvalid_tile = (N - n0 < BN) ? (N - n0) : BN;

        // A lane's values of one of its rows, in quads of neighbouring columns: quad t of the wavefront's strip starts at
        // column t * kQuadStep + 4 * group.
        constexpr int kQpb = Product::kQuads, kQuadStep = 4 * kLaneGroups;
        constexpr int kQuadsRow = kBlocksN * kQpb;
        constexpr int kPass = kQuadsRow < 4 ? kQuadsRow : 4;  // quads of a row worked on at a time

        // bias + GELU in place in the accumulators, and per-row (count, mean, M2) of
        // the tile.  Sums are taken about the row's first value in the strip (a shift that keeps sum-of-squares
        // cancellation harmless), added up over the lane groups, merged across waves.
        {
            const bool cut = RAGGED_N && nvalid_tile < BN;  // only the last tile of a row is cut by N
            float shift[kBlocksM], s1[kBlocksM], s2[kBlocksM];
            {
                const floatx4 bb = *reinterpret_cast<const floatx4 *>(s_b + ncol_wave + group * 4);
#pragma unroll
                for (int j = 0; j < kBlocksM; ++j) {
                    shift[j] = from_lane(gelu_erf(acc[0][j][0] + bb[0]), block_row);
                    s1[j] = s2[j] = 0.0f;
                    if (kAccRegs)
                        pin_order<kAccRegs>(acc[0][j]);
                }
            }
#pragma unroll
            for (int t0 = 0; t0 < kQuadsRow; t0 += kPass) {
                floatx4 bb[kPass];  // bias of this lane's columns
#pragma unroll
                for (int q = 0; q < kPass; ++q)
                    bb[q] = *reinterpret_cast<const floatx4 *>(s_b + ncol_wave + (t0 + q) * kQuadStep + group * 4);
                float s1_before[kBlocksM], s2_before[kBlocksM];
#pragma unroll
                for (int j = 0; j < kBlocksM; ++j) {
                    s1_before[j] = s1[j];
                    s2_before[j] = s2[j];
                }
#pragma unroll
                for (int j = 0; j < kBlocksM; ++j) {
#pragma unroll
                    for (int q = 0; q < kPass; ++q) {
                        Acc &c = acc[(t0 + q) / kQpb][j];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int r = (t0 + q) % kQpb * 4 + e;
                            const float z = c[r] + bb[q][e];
                            if (MODE == kLinearOnly) {
                                c[r] = z;
                                continue;
                            }
                            const float g = gelu_erf(z);
                            const float d = g - shift[j];
                            c[r] = g;
                            s1[j] += d;
                            s2[j] = fmaf(d, d, s2[j]);
                        }
                    }
#pragma unroll
                    for (int i = t0 / kQpb; i < (t0 + kPass) / kQpb; ++i)
                        pin_order<kAccRegs>(acc[i][j]);  // G goes back to the accumulator registers
                    // The sums are complete here.  The compiler put them off to where the statistics are stored, which
                    // kept every G of a row in ordinary registers until then, and 24 to 76 bytes in scratch memory.
                    if (kAccRegs)
                        asm volatile("" : "+v"(s1[j]), "+v"(s2[j]));
                    __builtin_amdgcn_sched_barrier(0);
                }
                // What N cuts is summed again, with what lies beyond N left out.  (Masks in
                // the pass itself made it 10.0 instead of 6.8 us for every tile of such a problem; two passes
                // behind a branch spilled 60 registers; the columns beyond N repeat the last one, are
                // never stored, and only the sums must not see them.)
                const int limit = nvalid_tile - ncol_wave - t0 * kQuadStep;
                if (RAGGED_N && MODE != kLinearOnly && limit < kPass * kQuadStep) {
#pragma unroll
                    for (int j = 0; j < kBlocksM; ++j) {
                        s1[j] = s1_before[j];
                        s2[j] = s2_before[j];
                        if (limit > 0) {
                            int lane_limit = limit - group * 4;
                            asm volatile("" : "+v"(lane_limit));  // the masks are made anew for every row
#pragma unroll
                            for (int q = 0; q < kPass; ++q) {  // a quad lies inside or beyond N as a whole
                                const bool in = q * kQuadStep < lane_limit;
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const float d = in ? acc[(t0 + q) / kQpb][j][(t0 + q) % kQpb * 4 + e] - shift[j] : 0.0f;
                                    s1[j] += d;
                                    s2[j] = fmaf(d, d, s2[j]);
                                }
                            }
                        }
                    }
                }
            }
            if (MODE != kLinearOnly) {
                // (the lane index is taken afresh after the pass over the accumulators and again
                // before the stores: values derived from it are not carried across those passes)
                const int lane = opaque_lane();
                const int cols = cut ? nvalid_tile - ncol_wave : WTN * 32;  // of the strip, inside N
                const float inv = cols > 0 ? 1.0f / (float)(cols < WTN * 32 ? cols : WTN * 32) : 0.0f;
#pragma unroll
                for (int j = 0; j < kBlocksM; ++j) {
                    // sums of the lane groups: the same bits in each of them
#pragma unroll
                    for (int across = kBlock; across < 64; across *= 2) {
                        s1[j] += from_lane(s1[j], lane ^ across);
                        s2[j] += from_lane(s2[j], lane ^ across);
                    }
                    if (lane < kBlock) {
                        floatx2 v = {fmaf(s1[j], inv, shift[j]), fmaxf(s2[j] - s1[j] * s1[j] * inv, 0.0f)};
                        if (RAGGED_N && cols <= 0)
                            v[0] = 0.0f;
                        s_wst[wn * BM + wm * WTM * 32 + j * kBlock + lane] = v;
                    }
                }
            }
        }

        const int tid = wave * 64 + opaque_lane();  // taken afresh: not carried across the pass above
        if (MODE != kLinearOnly) {
            __syncthreads();
            if (tid < BM) {
                int c0 = nvalid_tile < WTN * 32 ? nvalid_tile : WTN * 32;
                float na = (float)c0;
                floatx2 v = s_wst[tid];
                float mean_a = v[0], m2a = v[1];
#pragma unroll
                for (int w = 1; w < kWavesN; ++w) {
                    int cw = nvalid_tile - w * WTN * 32;
                    cw = cw < 0 ? 0 : (cw > WTN * 32 ? WTN * 32 : cw);
                    const floatx2 u = s_wst[w * BM + tid];
                    merge_stats(na, mean_a, m2a, (float)cw, u[0], u[1]);
                }
                floatx2 o = {mean_a, m2a};
                if (MODE == kFused)
                    publish_pair(p.partials + ((size_t)rb * p.NT + cb) * BM + tid, o);
                else
                    p.partials[((size_t)rb * p.NT + cb) * BM + tid] = o;
            }
        }

        stamp(3);
        if (MODE == kFused) {
            // exchange with the other tiles of these rows
            wait_published();
            __syncthreads();
            if (tid == 0) {
                unsigned *arrive = p.counters + 2 * row_counter(rb);
                atomic_add_device(arrive, 1u);
                if (!wait_counter(arrive, (unsigned)(p.NT + p.extra_arrivals), p.wait_ticks))
                    atomic_store_device(p.err, 1u);
            }
            __syncthreads();
            stamp(4);
            // Plain loads: each line was written through by its single owner before the counter
            // could reach its target, and no cache of this XCD can hold an older copy within this
            // launch.  Loads are issued 16 at a time, the merge runs in tile order.  Where the
            // workgroup has two threads per row and a row more than 16 tiles, each thread takes
            // half of the row's tiles (the load latency, not the arithmetic, is what the merge
            // costs) and the halves meet in LDS.
            constexpr int kParts = (64 * kWaves >= 2 * BM) ? 2 : 1;
            const bool split = kParts == 2 && p.NT > 16;
            const int row = tid & (BM - 1);
            const int per = split ? (p.NT + 1) / 2 : p.NT;
            float na = 0.0f, mean_a = 0.0f, m2a = 0.0f;
            if (tid < BM || (split && tid < kParts * BM)) {
                // Buffer loads: a row block's partials as the resource, the tile as the scalar
                // offset and the row as the one vector offset, so that no load needs a 64-bit
                // address of its own in vector registers.
                const int part = wave / (BM / 64);  // uniform in a wavefront
                const __amdgpu_buffer_rsrc_t st_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    reinterpret_cast<char *>(p.partials + (size_t)rb * p.NT * BM), 0,
                    (unsigned)(p.NT * BM * (int)sizeof(floatx2)), 0x00020000);
                const unsigned row_off = (unsigned)row * (unsigned)sizeof(floatx2);
                const int c_begin = part * per < p.NT ? part * per : p.NT;
                const int c_end = c_begin + per < p.NT ? c_begin + per : p.NT;
                auto merge_from = [&](int c0, auto batch) {
                    constexpr int kB = decltype(batch)::value;
                    floatx2 u[kB];
#pragma unroll
                    for (int j = 0; j < kB; ++j) {
                        const int c = c0 + j < c_end ? c0 + j : c_end - 1;  // unconditional loads
                        if (kParts == 2)
                            u[j] = __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(
                                                           st_rsrc, row_off, c * BM * (int)sizeof(floatx2), 0));
                        else  // one thread per row: plain addressing takes fewer registers there
                            u[j] = p.partials[((size_t)rb * p.NT + c) * BM + row];
                    }
                    // The tiles' counts are the same in every lane: mean and M2 of the batch about its first mean in
                    // six operations a tile and one division a batch.  (A merge of its own for every tile, 20 operations,
                    // was half of the merge: 6912 x 256 x 15208 bf16, 60 tiles, 4.8 us of each round, now 3.3;
                    // 4785 x 128 x 59136, 231 tiles, 723 us in all, 652.)
                    const int last = c0 + kB < c_end ? c0 + kB : c_end;
                    const float nb = (float)((last * BN < N ? last * BN : N) - c0 * BN), inv = 1.0f / nb;
                    auto count = [&](int j) {
                        const int left = N - (c0 + j) * BN;
                        return c0 + j < c_end ? (float)(left < BN ? left : BN) : 0.0f;
                    };
                    float d = 0.0f;
#pragma unroll
                    for (int j = 1; j < kB; ++j)
                        d = fmaf(u[j][0] - u[0][0], count(j), d);
                    const float mean_b = fmaf(d, inv, u[0][0]);
                    float m2b = 0.0f;
#pragma unroll
                    for (int j = 0; j < kB; ++j) {
                        const float e = u[j][0] - mean_b;
                        m2b = fmaf(e * count(j), e, m2b);
                        m2b += c0 + j < c_end ? u[j][1] : 0.0f;
                    }
                    merge_stats(na, mean_a, m2a, nb, mean_b, m2b);
                };
                if (c_end - c_begin <= 4) {
                    if (c_begin < c_end)
                        merge_from(c_begin, std::integral_constant<int, 4>());
                } else {
                    for (int c0 = c_begin; c0 < c_end; c0 += 16)
                        merge_from(c0, std::integral_constant<int, 16>());
                }
                if (split && part == 1) {  // s_wst is free: its last readers passed the barriers above
                    floatx2 o = {mean_a, m2a};
                    s_wst[row] = o;
                }
            }
            if (split)
                __syncthreads();
            if (tid < BM) {
                if (split) {
                    const int rest = N - per * BN;  // columns of the second half's tiles
                    const floatx2 u = s_wst[row];
                    merge_stats(na, mean_a, m2a, rest > 0 ? (float)rest : 0.0f, u[0], u[1]);
                }
                const float var = m2a / (float)N;
                floatx2 o = {mean_a, 1.0f / sqrtf(var + p.eps)};
                s_rst[tid] = o;
            }
            __syncthreads();
        }

        stamp(5);
        // ---- (normalise,) convert, transpose through LDS, store 16-byte rows ----
        OutT *out_base = (MODE == kFused) ? reinterpret_cast<OutT *>(p.Y)
                                          : reinterpret_cast<OutT *>(p.F);
        const int lane_o = opaque_lane();
        {
        const int lane = lane_o;
        const int group = lane / kBlock;
        const int block_row = lane % kBlock;
        constexpr int kRowBlocks = 32 / kBlock;  // blocks of a pass of 32 rows
#pragma unroll
        for (int j = 0; j < WTM; ++j) {
            float rstd[kRowBlocks], shift[kRowBlocks];  // y = (g * rstd + shift) * gamma + beta
#pragma unroll
            for (int u = 0; u < kRowBlocks; ++u) {
                rstd[u] = 1.0f;
                shift[u] = 0.0f;
                if (MODE == kFused) {
                    const floatx2 ms = s_rst[wm * WTM * 32 + j * 32 + u * kBlock + block_row];
                    rstd[u] = ms[1];
                    shift[u] = -ms[0] * ms[1];
                }
            }
#pragma unroll
            for (int t = 0; t < kQuadsRow; ++t) {
                const int cw = t * kQuadStep + group * 4;  // column inside the wave's strip
                floatx4 ga4, be4;
                if (MODE == kFused) {
                    ga4 = *reinterpret_cast<const floatx4 *>(s_g + ncol_wave + cw);
                    be4 = *reinterpret_cast<const floatx4 *>(s_be + ncol_wave + cw);
                }
#pragma unroll
                for (int u = 0; u < kRowBlocks; ++u) {
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        y[e] = acc[t / kQpb][j * kRowBlocks + u][t % kQpb * 4 + e];
                        if (MODE == kFused)
                            y[e] = fmaf(fmaf(y[e], rstd[u], shift[u]), ga4[e], be4[e]);
                    }
                    char *dst = s_out + (u * kBlock + block_row) * kOutPitch + cw * (int)sizeof(OutT);
                    if (sizeof(OutT) == 2) {
                        uintx2 v = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                        *reinterpret_cast<uintx2 *>(dst) = v;
                    } else {
                        floatx4 v = {y[0], y[1], y[2], y[3]};
                        *reinterpret_cast<floatx4 *>(dst) = v;
                    }
                }
            }
            wave_lds_sync();
            constexpr int kCpr = kOutRowBytes / 16;  // 16-byte chunks per row
            constexpr int kIters = 32 * kCpr / 64;
            constexpr int kChunkOut = 16 / (int)sizeof(OutT);
#pragma unroll
            for (int it = 0; it < kIters; ++it) {
                const int idx = it * 64 + lane;
                const int r = idx / kCpr;
                const int c = idx % kCpr;
                const uintx4 v = *reinterpret_cast<const uintx4 *>(s_out + r * kOutPitch + c * 16);
                const int gm = m0 + wm * WTM * 32 + j * 32 + r;
                const int gn = n0 + ncol_wave + c * kChunkOut;
                if (gm < M && gn < N)  // streaming store: Y is not read again by this launch
                    __builtin_nontemporal_store(v, reinterpret_cast<uintx4 *>(out_base + (size_t)gm * N + gn));
            }
            wave_lds_sync();
        }
        }
        if (MODE == kFused && tid == 0) {
            // Departure, after the stores have been issued so that the wait for the counter's old value
            // delays nothing: the last tile of the row-block to get here re-arms its counters (every
            // tile of the row-block has read the partials by then).
            unsigned *cnt = p.counters + 2 * row_counter(rb);
            if (atomic_add_device(cnt + 1, 1u) == (unsigned)p.NT - 1u) {
                atomic_store_device(cnt, 0u);
                atomic_store_device(cnt + 1, 0u);
            }
        }
        stamp(6);
        }  // epilogue scope
    }
#else
    (void)p;
#endif
}

// Second kernel of the two-pass variant: one workgroup per row.  Merges the
// row's per-tile (mean, M2) in a fixed order, then normalises the fp32 G row.
template <typename T>
__global__ __launch_bounds__(256) void finalize_kernel(const FinalizeParams p)
{
    __shared__ float s_stat[2];
    const int m = blockIdx.x;
    const int tid = threadIdx.x;
    const int rb = m / p.BM;
    const int r = m % p.BM;
    if (tid < 64) {
        float na = 0.0f, mean_a = 0.0f, m2a = 0.0f;
        for (int c = tid; c < p.NT; c += 64) {
            const int cnt = (p.N - c * p.BN < p.BN) ? (p.N - c * p.BN) : p.BN;
            const floatx2 u = p.partials[((size_t)rb * p.NT + c) * p.BM + r];
            merge_stats(na, mean_a, m2a, (float)cnt, u[0], u[1]);
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const float nb = __shfl_down(na, off);
            const float mb = __shfl_down(mean_a, off);
            const float qb = __shfl_down(m2a, off);
            merge_stats(na, mean_a, m2a, nb, mb, qb);
        }
        if (tid == 0) {
            s_stat[0] = mean_a;
            s_stat[1] = 1.0f / sqrtf(m2a / (float)p.N + p.eps);
        }
    }
    __syncthreads();
    const float mu = s_stat[0], rstd = s_stat[1];
    const float *g = p.G + (size_t)m * p.N;
    T *y = reinterpret_cast<T *>(p.Y) + (size_t)m * p.N;
    const T *gamma = reinterpret_cast<const T *>(p.gamma);
    const T *beta = reinterpret_cast<const T *>(p.beta);
    for (int n = tid * 4; n < p.N; n += 256 * 4) {
        const floatx4 gv = *reinterpret_cast<const floatx4 *>(g + n);
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ga = gamma ? load_as_float(gamma + n + e) : 1.0f;
            const float be = beta ? load_as_float(beta + n + e) : 0.0f;
            o[e] = fmaf((gv[e] - mu) * rstd, ga, be);
        }
        if (sizeof(T) == 2) {
            uintx2 v = {pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
            *reinterpret_cast<uintx2 *>(y + n) = v;
        } else {
            floatx4 v = {o[0], o[1], o[2], o[3]};
            *reinterpret_cast<floatx4 *>(y + n) = v;
        }
    }
}

// The instances that exist by lines: fused bf16 where LDS has a third stage.
template <typename T, int MODE, int STAGES> constexpr bool has_lines() { return sizeof(T) == 2 && MODE == kFused && STAGES == 3; }
// Whether such a launch goes by lines.  13 shapes with rows at every 16 bytes: 0.94 of the time (0.90 to 1.00).  At every 32 bytes
// 0.96 of it with eight row-blocks and more, which find lines in the L2; with fewer every line comes from HBM, and one
// line less in flight costs more (275 x 4240 x 13312 87.1 us, by lines 90.8).  At every 64 bytes it always does (3840 x 5408 x
// 1280 73.5, 78.9).
bool takes_lines(const TileParams &p)
{
    const unsigned off = ((unsigned)p.K * 2u | (unsigned)(uintptr_t)p.W | (unsigned)(uintptr_t)p.X) & 127u;
    return off != 0 && (off % 32 != 0 || (off % 64 != 0 && p.RB >= 8));
}

template <typename T, int MODE, int STAGES> bool by_lines(const TileParams &p) { return has_lines<T, MODE, STAGES>() && takes_lines(p); }

template <typename T, int WN, int WM, int WTN, int WTM, int MODE, int STAGES>
hipError_t launch_tile(const TileParams &p, int grid, hipStream_t stream)
{
    constexpr int BN = WN * WTN * 32;
    constexpr int kThreads = 64 * WN * WM;
    if constexpr (has_lines<T, MODE, STAGES>())
        if (by_lines<T, MODE, STAGES>(p)) {
            if (p.N % BN != 0)
                hipLaunchKernelGGL((tile_kernel<T, WN, WM, WTN, WTM, MODE, true, STAGES, true>), dim3(grid), dim3(kThreads), 0,
                                   stream, p);
            else
                hipLaunchKernelGGL((tile_kernel<T, WN, WM, WTN, WTM, MODE, false, STAGES, true>), dim3(grid), dim3(kThreads), 0,
                                   stream, p);
            return hipGetLastError();
        }
    if (p.N % BN != 0)
        hipLaunchKernelGGL((tile_kernel<T, WN, WM, WTN, WTM, MODE, true, STAGES, false>), dim3(grid), dim3(kThreads), 0,
                           stream, p);
    else
        hipLaunchKernelGGL((tile_kernel<T, WN, WM, WTN, WTM, MODE, false, STAGES, false>), dim3(grid), dim3(kThreads), 0,
                           stream, p);
    return hipGetLastError();
}

template <typename T, int WN, int WM, int WTN, int WTM, int MODE, int STAGES>
int max_blocks_per_cu()
{
    int least = 0;
    auto ask = [&](auto kernel) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, 64 * WN * WM, 0) != hipSuccess) {
            (void)hipGetLastError();
            n = 0;
        }
        return n;
    };
    constexpr bool kLines = has_lines<T, MODE, STAGES>();
    least = ask(tile_kernel<T, WN, WM, WTN, WTM, MODE, true, STAGES, false>);
    least = std::min(least, ask(tile_kernel<T, WN, WM, WTN, WTM, MODE, false, STAGES, false>));
    if (kLines) {
        least = std::min(least, ask(tile_kernel<T, WN, WM, WTN, WTM, MODE, true, STAGES, kLines>));
        least = std::min(least, ask(tile_kernel<T, WN, WM, WTN, WTM, MODE, false, STAGES, kLines>));
    }
    return least;
}

}  // namespace

// Dispatch over (dtype, tile shape, mode): wave layout, blocks per wave and LDS stages per shape.
#define FF_TILE_DISPATCH(CALL)                                                         \
    if (bf16) {                                                                        \
        switch (shape) {                                                               \
        case kTile256x128: FF_MODES(__bf16, 4, 2, 2, 2, 3, CALL)                       \
        case kTile256W8: FF_MODES(__bf16, 2, 4, 4, 2, 2, CALL)                         \
        case kTile256: FF_MODES(__bf16, 2, 2, 4, 4, 2, CALL)                           \
        case kTile128: FF_MODES(__bf16, 2, 2, 2, 2, 2, CALL)                           \
        default: FF_MODES(__bf16, 2, 2, 1, 1, 2, CALL)                                 \
        }                                                                              \
    }                                                                                  \
    switch (shape) {                                                                   \
    case kTile256x128: FF_MODES(float, 4, 2, 2, 2, 3, CALL)                            \
    case kTile256W8: FF_MODES(float, 2, 4, 4, 2, 2, CALL)                              \
    case kTile256: FF_MODES(float, 2, 2, 4, 4, 2, CALL)                                \
    case kTile128: FF_MODES(float, 2, 2, 2, 2, 2, CALL)                                \
    default: FF_MODES(float, 2, 2, 1, 1, 2, CALL)                                      \
    }
#define FF_MODES(T, WN, WM, WTN, WTM, STAGES, CALL)                                    \
    switch (mode) {                                                                    \
    case kFused: return CALL(T, WN, WM, WTN, WTM, kFused, STAGES);                     \
    case kTwoPass: return CALL(T, WN, WM, WTN, WTM, kTwoPass, STAGES);                 \
    default: return CALL(T, WN, WM, WTN, WTM, kLinearOnly, STAGES);                    \
    }

hipError_t launch_tile_kernel(bool bf16, int shape, int mode, const TileParams &p, int grid, hipStream_t stream)
{
#define FF_CALL(T, WN, WM, WTN, WTM, MODE, STAGES) launch_tile<T, WN, WM, WTN, WTM, MODE, STAGES>(p, grid, stream)
    FF_TILE_DISPATCH(FF_CALL)
#undef FF_CALL
}

// Whether such a launch goes by lines.
bool tile_kernel_by_lines(bool bf16, int shape, int mode, const TileParams &p)
{
#define FF_CALL(T, WN, WM, WTN, WTM, MODE, STAGES) by_lines<T, MODE, STAGES>(p)
    FF_TILE_DISPATCH(FF_CALL)
#undef FF_CALL
}

// Workgroups of this kernel that fit one compute unit at once (registers, LDS), as the runtime
// reports it; 0 if the query fails.  A launch whose workgroups wait for one another inside the
// launch must not be larger than this many per compute unit.
int tile_kernel_blocks_per_cu(bool bf16, int shape, int mode)
{
#define FF_CALL(T, WN, WM, WTN, WTM, MODE, STAGES) max_blocks_per_cu<T, WN, WM, WTN, WTM, MODE, STAGES>()
    FF_TILE_DISPATCH(FF_CALL)
#undef FF_CALL
}
#undef FF_MODES
#undef FF_TILE_DISPATCH

hipError_t launch_finalize_kernel(bool bf16, const FinalizeParams &p, hipStream_t stream)
{
    if (bf16)
        hipLaunchKernelGGL(finalize_kernel<__bf16>, dim3(p.M), dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL(finalize_kernel<float>, dim3(p.M), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace ff
