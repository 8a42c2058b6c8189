// Fused linear + erf-GELU + LayerNorm for problems with too few tiles to fill the chip (gfx950):
// output tiles of 32 x 32 to 128 x 128 (columns x rows, six shapes) whose K range is cut over S workgroups.
//
// One round: grid = tiles * S workgroups, all resident.  Workgroup (tile, s) walks its share of the
// 128-byte K slabs through a ring of kRing LDS stages filled by direct-to-LDS loads, so kRing - 1
// slabs are in flight while one is multiplied: such a problem is bound by the latency and rate of
// reading W and X (the two-stage loop of the persistent tile kernel keeps one slab, 16 KB, in flight
// per workgroup and waits 0.8 us for each).  Then
//   1  S > 1: the fp32 tile goes to global memory in row slices, the tile's S workgroups meet, and each
//      adds the S partial products of its slice of BM / S rows in s order;
//   2  bias, GELU and the slice's row statistics (mean, M2) over the tile's columns; the workgroups
//      with the same rows exchange those and merge them in fixed order;
//   3  normalise, convert, store.
// Measured against the two-stage loop of the tile kernel (cold inputs, whole call): 96 x 8192 x 8192
// bf16 104.7 -> 44.5 us (W at 3.0 TB/s), 512 x 8192 x 8192 bf16 125 -> 86, 64 x 4096 x 4096 fp32 98 -> 31,
// 256 x 512 x 512 fp32 17.3 -> 9.6; over 336 drawn shapes 1.36 (bf16) and 1.50 (fp32) times
// as fast, none slower.  What is left at 96 x 8192 x 8192: 27 us of reading W at the rate of a large copy, and
// launch, two meetings and the ramp of the stream.
// A thread owns four consecutive columns of one row per pass, so everything after the product stays in
// its registers and a row's statistics are sums over 16 or 32 neighbouring lanes.
// All sums run in fixed order: results are bitwise reproducible.
#include "ff_tile.hpp"

namespace ff {

namespace {

constexpr int kRowBytes = 128;   // bytes of one tile row per K slab (8 chunks of 16 B)
// LDS stages of a tile shape: four, and eight of the small slabs of 32 x 32 tiles, so that as many bytes are in flight
constexpr int ring_of(int tile_cols, int tile_rows) { return tile_cols + tile_rows <= 64 ? 8 : 4; }

// c: a block's sum, or in fp32 the SUMS that it is kept in, its products dealt to them in turn
template <int SUMS> __device__ __forceinline__ void mma(const uintx4 &a, const uintx4 &b, floatx16 (&c)[SUMS], const __bf16 *)
{
    c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c[0], 0, 0, 0);
}
template <int SUMS> __device__ __forceinline__ void mma(const uintx4 &a, const uintx4 &b, floatx16 (&c)[SUMS], const float *)
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
        c[e % SUMS] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]), c[e % SUMS], 0, 0, 0);
}

// LDS placement of 16-byte chunk c of tile row `row`: slot c ^ swizzle, conflict-free for the fragment reads
__device__ __forceinline__ int swizzle_of_row(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// s_waitcnt vmcnt(n), n < 64, nothing else
template <int n> __device__ __forceinline__ void wait_vm()
{
    __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | ((n >> 4) << 14));
}

template <int ctrl> __device__ __forceinline__ float lane_dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true));
}
template <int ror> __device__ __forceinline__ float rotate16(float v) { return lane_dpp<0x120 + ror>(v); }
// Sum over the 8, 16 or 32 neighbouring lanes of a row; the same bits in each of them (every step adds
// the two same numbers in both lanes of a pair).
template <int LANES> __device__ __forceinline__ float row_sum(float v)
{
    if (LANES == 8) {  // neighbour, neighbouring pair, the other four of the eight (mirrored)
        v += lane_dpp<0xb1>(v);
        v += lane_dpp<0x4e>(v);
        return v + lane_dpp<0x141>(v);
    }
    v += rotate16<8>(v);
    v += rotate16<4>(v);
    v += rotate16<2>(v);
    v += rotate16<1>(v);
    if (LANES == 32)
        v += __shfl_xor(v, 16);
    return v;
}

// Four neighbouring elements of a column vector as they lie in memory
template <typename T> struct RawCols;
template <> struct RawCols<float> {
    floatx4 v;
    static __device__ __forceinline__ RawCols load(const void *p, int n)
    {
        return RawCols{*reinterpret_cast<const floatx4 *>(reinterpret_cast<const float *>(p) + n)};
    }
    __device__ __forceinline__ floatx4 get() const { return v; }
};
template <> struct RawCols<__bf16> {
    uintx2 v;
    static __device__ __forceinline__ RawCols load(const void *p, int n)
    {
        return RawCols{*reinterpret_cast<const uintx2 *>(reinterpret_cast<const __bf16 *>(p) + n)};
    }
    __device__ __forceinline__ floatx4 get() const
    {
        return floatx4{__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xffff0000u), __uint_as_float(v[1] << 16),
                       __uint_as_float(v[1] & 0xffff0000u)};
    }
};

// kWN x kWM x kWK wavefronts: kWN x kWM blocks of WTN x WTM MFMA tiles, the k-steps of a slab dealt to kWK.
//
// Tiles of 128 columns and 64 or more rows, one workgroup a unit, run eight wavefronts, two at each block with half the
// k-steps each: the loads of a slab are issued by twice as many, one wavefront of a SIMD reads fragments while the other
// multiplies, and the epilogue has twice the threads.  With four: 512 x 8192 x 8192 bf16 97.5 us, now 85.5;
// 384 x 2048 x 6000 34.9, 31.4; 200 x 16384 x 3000 50.5, 47.2; 512 x 4096 x 4096 fp32 146, 139.  (A ring of five stages
// is no faster, so it is not the time of a load; the fragments of the next slab read ahead of its barrier neither in
// bf16, 4 % faster in long fp32 products and 0.3 us slower in short ones.  Both point at the rate at which a unit's
// loads reach its LDS: 57 bytes a nanosecond.)  The plan keeps four in the 128 x 128 tile for long rows off the 64-byte
// boundaries, which by slabs are faster so (plan_split has both sides).
//
// Tiles of 32 x 32 by four wavefronts, each with a quarter of every slab's k-steps, are for calls bound by latency: so many of
// them that a tile has the whole of K, which spares its workgroups' meeting (2.4 of 11.6 us at 256 x 512 x 512 fp32), with
// eight stages, so that 56 KB are in flight a workgroup.
//
// LINES: what travels is not a tile row's 128 bytes of a slab but the 128-byte line of memory that holds its beginning.  Rows
// that do not begin on line boundaries have two lines to every slab, and a unit's load path, which takes 27 bytes a
// clock and a line at a time, is what bounds these shapes; each line is now requested once.  Rows begin on 16-byte
// boundaries, that is on a chunk: chunk c of a row's slab i is chunk (c + lead) % 8 of its line i, or of line i + 1 where
// c + lead >= 8, and lies in LDS at the slot that it would have without the shift, so that only the stage it is read from
// differs between lanes.  Slab i needs lines i and i + 1: one line less is in flight and a share has one line more, which
// short shares and W that lies in the L2 do not earn back (takes_lines).
// 512 x 4104 x 4096 33.2 us, now 30.1; 237 x 6408 x 7648 62.1, 50.8; 2089 x 2952 x 1232 40.3, 31.4; 96 x 8200 x 8192 48.2,
// 39.3; the same bits.
template <typename T, int kWN, int kWM, int kWK, int WTN, int WTM, bool LINES, int kSums>
__global__ __launch_bounds__(64 * kWN * kWM * kWK, kWN * kWM * kWK == 8 || WTN == 1 ? 2 : 1) void split_kernel(const SplitParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)  // the body uses device-only types (buffer descriptors)
    constexpr int kWaves = kWN * kWM * kWK, kThreads = 64 * kWaves;
    static_assert(kWaves == 4 || kWaves == 8, "four or eight wavefronts");
    constexpr int BN = kWN * WTN * 32, BM = kWM * WTM * 32, kRing = ring_of(BN, BM);
    constexpr int kChunkElems = 16 / (int)sizeof(T);
    constexpr int kSlabElems = kRowBytes / (int)sizeof(T);
    constexpr int kStageBytes = (BN + BM) * kRowBytes;
    constexpr int kDmaA = BN / 8 / kWaves, kDmaB = BM / 8 / kWaves;  // direct-to-LDS instructions (8 rows each) per wave and slab
    constexpr int kDma = kDmaA + kDmaB;
    constexpr int kPitch = BN + 4;                   // floats of a row of the product in LDS
    constexpr int kProdBytes = kWK * BM * kPitch * 4;
    constexpr int kSmemBytes = kRing * kStageBytes > kProdBytes ? kRing * kStageBytes : kProdBytes;
    constexpr int kLanes = BN / 4;                   // lanes that share a row after the product
    constexpr int kRowsPerPass = kThreads / kLanes;
    constexpr int kMaxPass = BM / kRowsPerPass;
    __shared__ __attribute__((aligned(1024))) char smem[kSmemBytes];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % kWN, wm = (wave / kWN) % kWM, wk = wave / (kWN * kWM);
    const int h = lane >> 5, l32 = lane & 31;
    const int M = p.M, N = p.N, K = p.K, S = p.S;

    // Workgroup -> (s, column tile, row block), row block fastest: the workgroups of one XCD (blockIdx
    // modulo 8) get consecutive numbers, so that those which read the same rows of W share an L2.
    int rb, cb, s;
    {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int each = (int)gridDim.x >> 3, more = (int)gridDim.x & 7;
        const int t = xcd * each + (xcd < more ? xcd : more) + slot;
        const int u = t / p.RB;
        rb = t - u * p.RB;
        s = u / p.NT;
        cb = u - s * p.NT;
    }
    const int m0 = rb * BM, n0 = cb * BN;

    // Phase timestamps (test hook), as in the tile kernel; slot 7 where the tile's S workgroups have met
    auto stamp = [&](int k) {
        if (p.timeline != nullptr && tid == 0)
            p.timeline[(size_t)blockIdx.x * kTimelineSlots + k] = k < kTimelineCycleSlot ? wall_clock64() : clock64();
    };
    stamp(0);

    // this thread's column vectors: the oldest loads in flight, waited for together with the first slab
    const int c4 = (tid % kLanes) * 4;
    const bool col_ok = n0 + c4 < N;  // N is a multiple of 4: four columns are in or out together
    const int n4 = col_ok ? n0 + c4 : 0;
    // (loads never branch and nothing uses them before the product is there: a use, a conversion
    // included, would wait for the load first)
    const RawCols<T> raw_b = RawCols<T>::load(p.b ? p.b : p.W, p.b ? n4 : 0);
    const RawCols<T> raw_g = RawCols<T>::load(p.gamma ? p.gamma : p.W, p.gamma ? n4 : 0);
    const RawCols<T> raw_be = RawCols<T>::load(p.beta ? p.beta : p.W, p.beta ? n4 : 0);

    // ---- this workgroup's slabs ----
    const int slabs = (K + kSlabElems - 1) / kSlabElems;
    const int per = (slabs + S - 1) / S;
    const int sl0 = s * per < slabs ? s * per : slabs;
    const int sl1 = sl0 + per < slabs ? sl0 + per : slabs;
    const int total = sl1 - sl0;
    const int full = total - (total > 0 && sl1 * kSlabElems > K ? 1 : 0);  // the rest: the slab that K cuts

    const size_t row_stride = (size_t)K * sizeof(T);
    // LINES: a row's first chunk is chunk `lead` of its first line; a tile begins at a multiple of
    // eight rows, so that the lead of its row r is (phase + r * row_chunks) % 8.
    const int row_chunks = K / kChunkElems;
    const int w_phase = LINES ? (int)(reinterpret_cast<uintptr_t>(p.W) >> 4) & 7 : 0;
    const int x_phase = LINES ? (int)(reinterpret_cast<uintptr_t>(p.X) >> 4) & 7 : 0;
    const char *w_tile = (const char *)p.W - w_phase * 16 + (size_t)n0 * row_stride + (size_t)sl0 * kRowBytes;
    const char *x_tile = (const char *)p.X - x_phase * 16 + (size_t)m0 * row_stride + (size_t)sl0 * kRowBytes;
    auto lead = [&](int phase, int r) { return LINES ? (phase + r * row_chunks) & 7 : 0; };
    // where the line (LINES) or slab of row r begins, and the chunk of it that lies in `slot` of row `row` in LDS
    auto line_offset = [&](int phase, int row, int r, int slot) {
        const unsigned at = (unsigned)r * (unsigned)row_stride + phase * 16;
        return (LINES ? at & ~127u : at) + ((((slot ^ swizzle_of_row(row)) + lead(phase, r)) & 7) << 4);
    };
    unsigned offa[kDmaA], offb[kDmaB];
    // lane -> (row of an instruction's eight, stored chunk slot); rows beyond the matrix read its last row
#pragma unroll
    for (int j = 0; j < kDmaA; ++j) {
        const int row = wave * (BN / kWaves) + j * 8 + (lane >> 3);
        const int rr = n0 + row < N ? row : N - 1 - n0;
        offa[j] = line_offset(w_phase, row, rr, lane & 7);
    }
#pragma unroll
    for (int j = 0; j < kDmaB; ++j) {
        const int row = wave * (BM / kWaves) + j * 8 + (lane >> 3);
        const int rr = m0 + row < M ? row : M - 1 - m0;
        offb[j] = line_offset(x_phase, row, rr, lane & 7);
    }
    // Addresses are in bounds by construction: a tile's rows span at most 2^30 bytes.  An offset of kRangeBytes is
    // outside, and such a lane puts zeros into its place in LDS: the chunks of the last slab that lie beyond K.
    constexpr unsigned kRangeBytes = 0x80000000u;
    const __amdgpu_buffer_rsrc_t w_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(w_tile), 0, kRangeBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t x_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(x_tile), 0, kRangeBytes, 0x00020000);
    // the x-th of the wave's loads of this workgroup's slab i, into stage i % kRing
    auto dma_one = [&](int i, int x, bool in) {
        char *st = smem + (i % kRing) * kStageBytes;
        if (x < kDmaA)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                w_rsrc, (__attribute__((address_space(3))) void *)(st + (wave * (BN / kWaves) + x * 8) * kRowBytes), 16,
                in ? offa[x < kDmaA ? x : 0] : kRangeBytes, i * kRowBytes, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                x_rsrc, (__attribute__((address_space(3))) void *)(st + (BN + wave * (BM / kWaves) + (x - kDmaA) * 8) * kRowBytes), 16,
                in ? offb[x < kDmaA ? 0 : x - kDmaA] : kRangeBytes, i * kRowBytes, 0, 0);
    };
    auto request = [&](int i) {
#pragma unroll
        for (int x = 0; x < kDma; ++x)
            dma_one(i, x, true);
    };
    auto request_cut = [&](int i) {
#pragma unroll
        for (int x = 0; x < kDma; ++x) {
            const int row = x < kDmaA ? wave * (BN / kWaves) + x * 8 : wave * (BM / kWaves) + (x - kDmaA) * 8;
            const int chunk = (lane & 7) ^ swizzle_of_row(row + (lane >> 3));
            int first = (sl0 + i) * 8;  // chunk of the matrix row that a slab or line begins with
            if (LINES) {
                const int r = row + (lane >> 3), last = x < kDmaA ? N - 1 - n0 : M - 1 - m0;
                const int ld = lead(x < kDmaA ? w_phase : x_phase, r < last ? r : last);
                first -= chunk + ld >= 8 ? 8 : 0;
            }
            dma_one(i, x, (unsigned)(first + chunk) < (unsigned)row_chunks);
        }
    };

    floatx16 acc[WTN][WTM][kSums];
#pragma unroll
    for (int i = 0; i < WTN; ++i)
#pragma unroll
        for (int j = 0; j < WTM; ++j)
#pragma unroll
            for (int k = 0; k < kSums; ++k)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[i][j][k][r] = 0.0f;
    const int swz = swizzle_of_row(l32);
    const int a_base = (wn * WTN * 32 + l32) * kRowBytes;
    const int b_base = (BN + wm * WTM * 32 + l32) * kRowBytes;
    const int a_lead = lead(w_phase, l32), b_lead = lead(x_phase, l32);
    auto multiply = [&](int stage) {
        const char *st = smem + stage * kStageBytes;
        const int ahead = stage + 1 < kRing ? kStageBytes : -(kRing - 1) * kStageBytes;  // the next line's stage
        constexpr int kSteps = 4 / kWK;
        uintx4 a[kSteps][WTN], b[kSteps][WTM];
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks) {
            const int chunk = 2 * (wk * kSteps + ks) + h, coff = (chunk ^ swz) << 4;
            const int a_off = a_base + coff + (LINES && chunk + a_lead >= 8 ? ahead : 0);
            const int b_off = b_base + coff + (LINES && chunk + b_lead >= 8 ? ahead : 0);
#pragma unroll
            for (int i = 0; i < WTN; ++i)
                a[ks][i] = *reinterpret_cast<const uintx4 *>(st + a_off + i * 32 * kRowBytes);
#pragma unroll
            for (int j = 0; j < WTM; ++j)
                b[ks][j] = *reinterpret_cast<const uintx4 *>(st + b_off + j * 32 * kRowBytes);
        }
        __builtin_amdgcn_sched_barrier(0);  // all reads are under way before the first product waits for its own
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks)
#pragma unroll
            for (int i = 0; i < WTN; ++i)
#pragma unroll
                for (int j = 0; j < WTM; ++j)
                    mma(a[ks][i], b[ks][j], acc[i][j], (const T *)nullptr);
    };

    // ---- main loop ----
    if constexpr (LINES) {
#pragma unroll
        for (int t = 0; t < kRing - 1; ++t)
            if (total > 0 && t <= total)
                request_cut(t);
    } else {
#pragma unroll
        for (int t = 0; t < kRing - 1; ++t)
            if (t < full)
                request(t);
        if (__builtin_expect(total > full && total < kRing, 0))
            request_cut(total - 1);
    }
    if (p.timeline != nullptr) {  // the first slab has landed
        if (!LINES && total >= kRing - 1)
            wait_vm<(kRing - 2) * kDma>();
        else
            wait_vm<0>();
        lds_barrier();
    }
    stamp(1);
    stamp(kTimelineCycleSlot);
    int i = 0;
    if constexpr (LINES) {
        // Slab i needs lines i and i + 1; line i - 1 is done with.  Lines that a row's end cuts, or that lie behind it: the
        // last two of the row.
        const int whole = row_chunks / 8 - 1 - sl0 < total ? row_chunks / 8 - 1 - sl0 : total;
        for (; i + kRing - 1 <= whole; ++i) {
            wait_vm<(kRing - 3) * kDma>();
            lds_barrier();
            request(i + kRing - 1);
            multiply(i % kRing);
        }
        for (; i + kRing - 1 <= total; ++i) {
            wait_vm<(kRing - 3) * kDma>();
            lds_barrier();
            request_cut(i + kRing - 1);
            multiply(i % kRing);
        }
    } else {
        for (; i + kRing - 1 < full; ++i) {
            wait_vm<(kRing - 2) * kDma>();  // this wave's rows of slab i have landed
            lds_barrier();                  // everyone's have, and everyone has read slab i - 1
            request(i + kRing - 1);  // into the stage slab i - 1 occupied
            multiply(i % kRing);
        }
        if (__builtin_expect(i + kRing - 1 < total, 0)) {  // the last slab, cut by K
            wait_vm<(kRing - 2) * kDma>();
            lds_barrier();
            request_cut(i + kRing - 1);
            multiply(i % kRing);
            ++i;
        }
    }
    auto last = [&](auto left_c) {
        constexpr int left = decltype(left_c)::value;
        if (__builtin_expect(total - i > left, 1)) {  // in line: short calls pay for every jump to code of its own
            wait_vm<left * kDma>();
            lds_barrier();
            multiply(i % kRing);
            ++i;
        }
    };
    static_assert(kRing == 4 || (kRing == 8 && !LINES), "the last slabs");
    if constexpr (kRing == 8) {
        last(std::integral_constant<int, 6>());
        last(std::integral_constant<int, 5>());
        last(std::integral_constant<int, 4>());
        last(std::integral_constant<int, 3>());
    }
    if constexpr (!LINES)
        last(std::integral_constant<int, 2>());
    last(std::integral_constant<int, 1>());
    last(std::integral_constant<int, 0>());
    stamp(2);
    stamp(kTimelineCycleSlot + 1);
    lds_barrier();  // all fragment reads done: the stages become the product's place

    static_assert(kSums == 1 || WTN * WTM == 1, "several sums of one block only");
    if constexpr (kSums > 2)
        acc[0][0][0] = (acc[0][0][0] + acc[0][0][1]) + (acc[0][0][2] + acc[0][0][3]);
    else if constexpr (kSums > 1)
        acc[0][0][0] += acc[0][0][1];

    // ---- product to LDS, [kWK][row][column] ----
    float *prod = reinterpret_cast<float *>(smem);
    {
        // a lane's registers of a 32 x 32 block: row (of the output) l32, columns 8 q + 4 h + (0..3)
        float *mine = prod + wk * BM * kPitch;
#pragma unroll
        for (int i = 0; i < WTN; ++i)
#pragma unroll
            for (int j = 0; j < WTM; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<floatx4 *>(mine + ((wm * WTM + j) * 32 + l32) * kPitch + (wn * WTN + i) * 32 + q * 8 + h * 4) =
                        floatx4{acc[i][j][0][4 * q], acc[i][j][0][4 * q + 1], acc[i][j][0][4 * q + 2], acc[i][j][0][4 * q + 3]};
    }
    lds_barrier();
    const int r_in_pass = tid / kLanes;
    auto product = [&](int row) {
        floatx4 v = *reinterpret_cast<const floatx4 *>(prod + row * kPitch + c4);
#pragma unroll
        for (int w = 1; w < kWK; ++w)
            v += *reinterpret_cast<const floatx4 *>(prod + (w * BM + row) * kPitch + c4);
        return v;
    };
    const int rows = BM / S;            // rows of this workgroup's slice
    const int row0 = s * rows;          // first of them in the tile
    const int passes = (rows + kRowsPerPass - 1) / kRowsPerPass;
    const bool mine = r_in_pass < rows; // fewer rows than a pass takes: the rest of the threads idle

    // ---- 1: sum over the tile's workgroups ----
    // Departures: begun as soon as a wait is over, looked at when the rest is done.  (At the end of the kernel their round trips
    // to memory stood one behind the other.)  All tiles of the rows meet at one word of the second, whose answer stands ahead of whatever
    // its wavefront loads next: the last wavefront begins it, which has no statistics to load where there are few tiles.
    // Of the time with both at the end: K cut, 90 drawn shapes, 0.924 (0.943 with the second by wavefront 0), whole, 70 shapes, 0.963 (0.980),
    // and 60 whole ones that lose by wavefront 0 0.986 (1.010: 512 x 256 x 512 bf16 8.3 us, by wavefront 0 8.5, now 8.0).
    constexpr int kLeaver = kThreads - 64;
    unsigned left_tile = 0, left_group = 0;
    floatx4 v[kMaxPass];
    const int tile = rb * p.NT + cb;
    if (S > 1) {
        // partial products [tile][s][BM][BN]; the writer keeps its own slice.  Written through (sc1) to
        // the level all XCDs share; each 128-byte line has one writer and is read by one other workgroup.
        float *part = p.sums + ((size_t)tile * S + s) * (BM * BN);
        const __amdgpu_buffer_rsrc_t st_rsrc = __builtin_amdgcn_make_buffer_rsrc(part, 0, BM * BN * 4, 0x00020000);
#pragma unroll
        for (int q = 0; q < kMaxPass; ++q) {
            const int row = q * kRowsPerPass + r_in_pass;
            if (row < row0 || row >= row0 + rows)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, product(row)), st_rsrc,
                                                       (row * BN + c4) * 4, 0, 16 /* sc1 */);
        }
        wait_published();
        __syncthreads();
        unsigned *c = p.counters + (size_t)tile * kSplitCounterStride;
        if (tid == 0) {
            atomic_add_device(c, 1u);
            if (!wait_counter(c, (unsigned)S, p.wait_ticks))
                atomic_store_device(p.err, 1u);
        }
        __syncthreads();
        if (tid == 0)
            left_tile = atomic_add_device(c + 1, 1u);
        const float *all = p.sums + (size_t)tile * S * (BM * BN);
        if constexpr (kWaves == 8) {
            // The parts of all of a thread's passes are requested together (S of each, kMaxPass or S in all) and added
            // in s order; one pass after the other is a load latency each (96 x 8192 x 8192 bf16 46.0 us, now 45.2;
            // 30 x 4096 x 4096 in 128 x 128 tiles cut in two 27.2, 25.7).
            auto add_parts = [&](auto s_c) {
                constexpr int kS = decltype(s_c)::value;
                constexpr int kPasses = kMaxPass / kS > 0 ? kMaxPass / kS : 1;
                floatx4 u[kPasses][kS];
#pragma unroll
                for (int q = 0; q < kPasses; ++q) {
                    const int rr = mine ? row0 + q * kRowsPerPass + r_in_pass : row0;
#pragma unroll
                    for (int t = 0; t < kS; ++t)
                        u[q][t] = *reinterpret_cast<const floatx4 *>(all + ((size_t)t * BM + rr) * BN + c4);
                }
#pragma unroll
                for (int q = 0; q < kPasses; ++q) {
                    const floatx4 own = product(mine ? row0 + q * kRowsPerPass + r_in_pass : row0);
                    floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int t = 0; t < kS; ++t)
                        sum += t == s ? own : u[q][t];
                    v[q] = sum;
                }
            };
            static_assert(kSplitMaxS == 16, "the cases below");
            if (S == 2)
                add_parts(std::integral_constant<int, 2>());
            else if (S == 4)
                add_parts(std::integral_constant<int, 4>());
            else if (S == 8)
                add_parts(std::integral_constant<int, 8>());
            else
                add_parts(std::integral_constant<int, 16>());
        } else {
            // The smaller tiles have one pass mostly.  (Requested together, calls that cut nothing lost more than the
            // others won: 256 x 512 x 512 bf16, S = 1, 10.1 instead of 9.2 us; fp32, S = 4, 11.5 instead of 11.7.)
#pragma unroll
            for (int q = 0; q < kMaxPass; ++q)
                if (q < passes) {
                    const int row = row0 + q * kRowsPerPass + r_in_pass;
                    const int rr = mine ? row : row0;
                    const floatx4 own = product(rr);
                    floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
                    for (int t0 = 0; t0 < S; t0 += 4) {
                        floatx4 u[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int o = t0 + t < S ? t0 + t : S - 1;
                            u[t] = *reinterpret_cast<const floatx4 *>(all + ((size_t)o * BM + rr) * BN + c4);
                        }
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            if (t0 + t < S)
                                sum += t0 + t == s ? own : u[t];
                    }
                    v[q] = sum;
                }
        }
    } else {
#pragma unroll
        for (int q = 0; q < kMaxPass; ++q)
            v[q] = product(q * kRowsPerPass + r_in_pass);
    }
    stamp(7);

    // ---- 2: bias, GELU, row statistics over the tile's columns, exchange ----
    floatx4 bias = {0.0f, 0.0f, 0.0f, 0.0f}, gamma = {1.0f, 1.0f, 1.0f, 1.0f}, beta = {0.0f, 0.0f, 0.0f, 0.0f};
    if (p.b)
        bias = raw_b.get();
    if (p.gamma)
        gamma = raw_g.get();
    if (p.beta)
        beta = raw_be.get();
    const int nvalid = N - n0 < BN ? N - n0 : BN;
    const float inv_valid = 1.0f / (float)nvalid;
    const int rows_pad = rows < 16 ? 16 : rows;  // a workgroup's partials fill whole 128-byte lines
    floatx2 *stats = p.partials + (size_t)(rb * S + s) * p.NT * rows_pad;
#pragma unroll
    for (int q = 0; q < kMaxPass; ++q)
        if (q < passes) {
            float sum = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[q][e] = gelu_erf(v[q][e] + bias[e]);
                sum += v[q][e];
            }
            const float mean = row_sum<kLanes>(col_ok ? sum : 0.0f) * inv_valid;
            float m2 = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d = v[q][e] - mean;
                m2 = fmaf(d, d, m2);
            }
            m2 = row_sum<kLanes>(col_ok ? m2 : 0.0f);
            if (mine && c4 == 0)
                publish_pair(stats + (size_t)cb * rows_pad + q * kRowsPerPass + r_in_pass, floatx2{mean, m2});
        }
    stamp(3);
    wait_published();
    __syncthreads();
    // the row slice's NT workgroups meet: arrivals spread over kSplitWays words in lines of their own
    unsigned *group = p.counters + ((size_t)p.RB * p.NT + (size_t)(rb * S + s) * kSplitWays) * kSplitCounterStride;
    if (tid == 0)
        atomic_add_device(group + (cb % kSplitWays) * kSplitCounterStride, 1u);
    if (wave == 0) {
        const int w = lane < kSplitWays ? lane : 0;
        const unsigned target = (unsigned)((p.NT + kSplitWays - 1 - w) / kSplitWays + (w == 0 ? p.extra_arrivals : 0));
        if (!wait_ways(group + (size_t)w * kSplitCounterStride, lane < kSplitWays, target, p.wait_ticks) && lane == 0)
            atomic_store_device(p.err, 1u);
    }
    __syncthreads();
    if (tid == kLeaver)
        left_group = atomic_add_device(group + 1, 1u);
    stamp(4);

    // ---- 3: merge, normalise, store ----
    // Thread -> (row of the slice, every chunks-th tile), so that a load instruction reads neighbouring
    // rows of one tile and up to eight are in flight; the chunks of a row meet in LDS in chunk order.
    // (A row's own lanes reading its tiles touch a line each: 40 x 512 x 15360, 240 tiles, 34 us a call.)
    float *s_n = reinterpret_cast<float *>(smem);             // [kMaxChunks][rows]: columns seen
    floatx2 *s_mm = reinterpret_cast<floatx2 *>(smem + kThreads * 4);   // [kMaxChunks][rows]: mean, M2
    floatx2 *s_row = reinterpret_cast<floatx2 *>(smem + kThreads * 12);  // [rows]: mean, 1 / standard deviation
    constexpr int kMaxChunks = 16, kBatch = 8;
    const int rows_log2 = 31 - __builtin_clz(rows);
    // (no more chunks than there are batches: 256 x 512 x 512 fp32, eight tiles a row, 13.4 us with 16 chunks
    // of at most one tile to meet in LDS, 12.2 with one)
    const int batches = (p.NT + kBatch - 1) / kBatch, places = kThreads >> rows_log2;
    const int chunks = batches < places ? (batches < kMaxChunks ? batches : kMaxChunks) : (places < kMaxChunks ? places : kMaxChunks);
    {
        const int r = tid & (rows - 1), chunk = tid >> rows_log2;
        if (chunk < chunks) {
            float na = 0.0f, mean_a = 0.0f, m2a = 0.0f;
            for (int c0 = chunk; c0 < p.NT; c0 += chunks * kBatch) {
                floatx2 u[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const int c = c0 + j * chunks < p.NT ? c0 + j * chunks : p.NT - 1;
                    u[j] = stats[(size_t)c * rows_pad + r];
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const int c = c0 + j * chunks;
                    if (c < p.NT)
                        merge_stats(na, mean_a, m2a, (float)(N - c * BN < BN ? N - c * BN : BN), u[j][0], u[j][1]);
                }
            }
            s_n[tid] = na;
            s_mm[tid] = floatx2{mean_a, m2a};
        }
        __syncthreads();
        if (tid < rows) {
            float na = s_n[tid];
            floatx2 u = s_mm[tid];
            float mean_a = u[0], m2a = u[1];
            for (int c = 1; c < chunks; ++c) {
                u = s_mm[c * rows + tid];
                merge_stats(na, mean_a, m2a, s_n[c * rows + tid], u[0], u[1]);
            }
            s_row[tid] = floatx2{mean_a, 1.0f / sqrtf(m2a / (float)N + p.eps)};
        }
        __syncthreads();
    }
    stamp(5);
    T *Y = reinterpret_cast<T *>(p.Y);
#pragma unroll
    for (int q = 0; q < kMaxPass; ++q)
        if (q < passes) {
            const int r = q * kRowsPerPass + r_in_pass;
            const int gm = m0 + row0 + r;
            if (mine && col_ok && gm < M) {
                const floatx2 ms = s_row[r];
                float y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    y[e] = fmaf((v[q][e] - ms[0]) * ms[1], gamma[e], beta[e]);
                T *dst = Y + (size_t)gm * N + n0 + c4;
                if (sizeof(T) == 2)
                    *reinterpret_cast<uintx2 *>(dst) = uintx2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                else
                    *reinterpret_cast<floatx4 *>(dst) = floatx4{y[0], y[1], y[2], y[3]};
            }
        }
    // ---- departure: the last to leave a counter re-arms it ----
    if (tid == 0 && S > 1 && left_tile == (unsigned)S - 1u) {
        unsigned *c = p.counters + (size_t)tile * kSplitCounterStride;
        atomic_store_device(c, 0u);
        atomic_store_device(c + 1, 0u);
    }
    if (tid == kLeaver && left_group == (unsigned)p.NT - 1u) {
        for (int w = 0; w < kSplitWays; ++w)
            atomic_store_device(group + (size_t)w * kSplitCounterStride, 0u);
        atomic_store_device(group + 1, 0u);
    }
    stamp(6);
#else
    (void)p;
#endif
}

}  // namespace

#define FF_SPLIT_TYPES(SHAPE, WN, WM, WK, WTN, WTM, CALL)                                                       \
    static_assert(split_shape_cols(SHAPE) == WN * WTN * 32 && split_shape_rows(SHAPE) == WM * WTM * 32 &&       \
                      split_shape_waves(SHAPE) == WN * WM * WK, "what the plan says of this shape");            \
    return bf16 ? CALL(__bf16, WN, WM, WK, WTN, WTM) : CALL(float, WN, WM, WK, WTN, WTM);
#define FF_SPLIT_DISPATCH(CALL)                                            \
    switch (shape) {                                                       \
    case kSplit64x32: FF_SPLIT_TYPES(kSplit64x32, 2, 1, 2, 1, 1, CALL)     \
    case kSplit128x32: FF_SPLIT_TYPES(kSplit128x32, 2, 1, 2, 2, 1, CALL)   \
    case kSplit64: FF_SPLIT_TYPES(kSplit64, 2, 2, 1, 1, 1, CALL)           \
    case kSplit128x64: FF_SPLIT_TYPES(kSplit128x64, 2, 2, 2, 2, 1, CALL)   \
    case kSplit32: FF_SPLIT_TYPES(kSplit32, 1, 1, 4, 1, 1, CALL)           \
    case kSplit128W4:                                                      \
        static_assert(split_shape_waves(kSplit128W4) == 4, "2 x 2 x 1");   \
        return CALL(__bf16, 2, 2, 1, 2, 2);                                \
    default: FF_SPLIT_TYPES(kSplit128, 2, 2, 2, 2, 2, CALL)                \
    }

// The instances that exist by lines: bf16, tiles of 128 columns and 64 or 128 rows.  (In fp32, bound by the matrix units, lines
// take 1 to 4 % more time, in the smaller tiles 0 to 8 %.)
template <typename T, int WN, int WM, int WTN, int WTM> static constexpr bool has_lines()
{
    return sizeof(T) == 2 && WN * WTN == 4 && WM * WTM >= 2;
}

// Sums of a block in fp32 tiles of one block a wavefront.  Four, one for each of a chunk's elements, in those that take the place of larger ones
// (32 x 32, and 64 x 32 over 64 rows): K is cut over fewer workgroups there, and this way no sum has more terms than in the larger tiles (316 x 3328 x
// 512: 208 in 64 x 64 tiles cut in eight; in 32 x 32 with the whole of K 416 with two sums, which was up to 1.11 of the error,
// 208 with four).  Two elsewhere: the others add 0.1 us.
template <typename T, int WN, int WM, int WTN, int WTM> static constexpr int sums_of()
{
    return sizeof(T) == 2 || WTN * WTM > 1 ? 1 : (WM == 1 ? 4 : 2);
}
// the same up to 64 rows, where 64 x 32 tiles replace nothing
template <typename T, int WN, int WM, int WTN, int WTM> static constexpr int few_rows_sums()
{
    return sums_of<T, WN, WM, WTN, WTM>() == 4 && WN == 2 ? 2 : sums_of<T, WN, WM, WTN, WTM>();
}

// Whether such a launch goes by lines: rows off the line boundaries, and enough slabs for each workgroup.  170 shapes, M
// 33..2048: rows on every other 64-byte boundary, or K cut over four and more workgroups (narrow W mostly, which the L2
// holds), gain from 24 slabs on (0.92 of the time; 10 to 23: 1.01), the rest from 9 (0.93; below 1.03).  The four wavefronts of the
// long rows gain 0.84 where rows come from HBM; from the caches, where other row blocks find the second half of a line, they lose 1.02.
// Timed on three sets of inputs in turn, X and W together stay in the 256 MB of the Infinity Cache up to 72 MB, with the whole of K in
// a tile and W the larger of them up to 81 MB (72 to 81 MB: 19 such shapes 1.02 by lines, 19 with K cut 0.96).
static bool takes_lines(const SplitParams &p, int waves)
{
    const unsigned off = ((unsigned)p.K * 2u | (unsigned)(uintptr_t)p.W | (unsigned)(uintptr_t)p.X) & 127u;
    if (off == 0)
        return false;
    if (waves == 4)
        return ((double)p.M + (double)p.N) * (double)p.K * 2.0 > (p.S == 1 && p.M < p.N ? 81e6 : 72e6);
    const int slabs = (p.K + 63) / 64, per = (slabs + p.S - 1) / p.S;
    return per >= (off % 64 == 0 || p.S >= 4 ? 24 : 9);
}

template <typename T, int WN, int WM, int WK, int WTN, int WTM> static bool by_lines(const SplitParams &p)
{
    return has_lines<T, WN, WM, WTN, WTM>() && takes_lines(p, WN * WM * WK);
}

template <typename T, int WN, int WM, int WK, int WTN, int WTM>
static hipError_t launch_split(const SplitParams &p, int grid, hipStream_t stream)
{
    const dim3 threads(64 * WN * WM * WK);
    constexpr int kSums = sums_of<T, WN, WM, WTN, WTM>();
    if constexpr (has_lines<T, WN, WM, WTN, WTM>())
        if (by_lines<T, WN, WM, WK, WTN, WTM>(p)) {
            hipLaunchKernelGGL((split_kernel<T, WN, WM, WK, WTN, WTM, true, 1>), dim3(grid), threads, 0, stream, p);
            return hipGetLastError();
        }
    constexpr int kFewRowsSums = few_rows_sums<T, WN, WM, WTN, WTM>();
    if constexpr (kFewRowsSums != kSums)
        if (p.M <= 64) {
            hipLaunchKernelGGL((split_kernel<T, WN, WM, WK, WTN, WTM, false, kFewRowsSums>), dim3(grid), threads, 0, stream, p);
            return hipGetLastError();
        }
    hipLaunchKernelGGL((split_kernel<T, WN, WM, WK, WTN, WTM, false, kSums>), dim3(grid), threads, 0, stream, p);
    return hipGetLastError();
}

template <typename T, int WN, int WM, int WK, int WTN, int WTM>
static int split_blocks()
{
    constexpr int kSums = sums_of<T, WN, WM, WTN, WTM>();
    int a = 0, b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, split_kernel<T, WN, WM, WK, WTN, WTM, false, kSums>, 64 * WN * WM * WK, 0) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, split_kernel<T, WN, WM, WK, WTN, WTM, has_lines<T, WN, WM, WTN, WTM>(), few_rows_sums<T, WN, WM, WTN, WTM>()>,
                                                     64 * WN * WM * WK, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return a < b ? a : b;
}

hipError_t launch_split_kernel(bool bf16, int shape, const SplitParams &p, int grid, hipStream_t stream)
{
#define FF_CALL(T, WN, WM, WK, WTN, WTM) launch_split<T, WN, WM, WK, WTN, WTM>(p, grid, stream)
    FF_SPLIT_DISPATCH(FF_CALL)
#undef FF_CALL
}

// Whether such a launch goes by lines.
bool split_kernel_by_lines(bool bf16, int shape, const SplitParams &p)
{
#define FF_CALL(T, WN, WM, WK, WTN, WTM) by_lines<T, WN, WM, WK, WTN, WTM>(p)
    FF_SPLIT_DISPATCH(FF_CALL)
#undef FF_CALL
}

// Workgroups of this kernel that fit one compute unit at once, as the runtime reports it; 0 if it does not.
int split_kernel_blocks_per_cu(bool bf16, int shape)
{
#define FF_CALL(T, WN, WM, WK, WTN, WTM) split_blocks<T, WN, WM, WK, WTN, WTM>()
    FF_SPLIT_DISPATCH(FF_CALL)
#undef FF_CALL
}
#undef FF_SPLIT_DISPATCH
#undef FF_SPLIT_TYPES

}  // namespace ff
