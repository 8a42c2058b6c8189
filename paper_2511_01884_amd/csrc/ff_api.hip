// Host side of the C ABI declared in include/ff.h: argument validation, variant
// selection by shape, workspace management and kernel launches.  Nothing here
// computes on tensors and nothing falls back to a library GEMM or LayerNorm.
#include <mutex>
#include <vector>
#include <algorithm>
#include <cstring>

#include "../../include/ff.h"
#include "ff_tile.hpp"

namespace {

using namespace ff;

constexpr int kMaxDevices = 64;

// Scratch memory of the entry point that allocates nothing: error word, arrival counters and per-tile
// row statistics of one call, laid out like a workspace.  One copy per device that loads the library,
// held until the process ends.  Host code never uses this name as an address: the per-device address
// comes from hipGetSymbolAddress (no_alloc_scratch below).
constexpr size_t kNoAllocBytes = 8u << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];
// The split kernel's partial products of such a call: at most one 64 KiB tile for each of 256 units.
constexpr size_t kNoAllocSumBytes = 16u << 20;
static __device__ __align__(256) unsigned char scratch_sums[kNoAllocSumBytes];

// Sets `words` 32-bit words at `dst` to `value` (a fill kernel, not a memset node, so that a caller
// may record it into a graph).
__global__ __launch_bounds__(256) void fill_words_kernel(unsigned *dst, size_t words, unsigned value)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256)
        dst[i] = value;
}

// The state a workspace must be in between launches: error word and counters zero.
hipError_t init_control_region(void *ws)
{
    hipError_t e = hipMemset(ws, 0, kCtrlBytes);
    if (e == hipSuccess)
        e = hipDeviceSynchronize();
    return e;
}

struct DeviceState {
    bool probed = false;
    int num_cus = 256;
    long long ticks_per_us = 100;
    void *ws = nullptr;       // bound or owned workspace; its control region is zeroed when it is bound or allocated
    size_t ws_bytes = 0;
    bool ws_owned = false;
    bool ws_recorded = false;                // owned, and a captured call holds its address
    struct Kept { void *ptr; size_t bytes; } kept[64] = {};  // recorded ones that were outgrown or unbound
    int n_kept = 0;
    void *no_alloc_ptr = nullptr;            // this device's copy of `scratch`, once asked for
    void *no_alloc_sums = nullptr;           // the same for `scratch_sums`
    bool no_alloc_used = false;
    void *pinned = nullptr;                  // host memory that the selection's kernels write their results to, with the own workspace
    size_t pinned_bytes = 0;
    unsigned long long *timeline = nullptr;  // test hook: phase timestamps of the tiled kernels
    size_t timeline_bytes = 0;
    signed char blocks_per_cu[2][kNumTileShapes][3] = {};  // cached occupancy answers [bf16][shape][mode], 0 = not asked
    signed char split_blocks[2][kNumSplitShapes] = {};     // the same for the split kernel
};

std::mutex g_mutex;
DeviceState g_dev[kMaxDevices];
int g_forced_variant = FF_VARIANT_AUTO;
long long g_wait_limit_us = 2000000;
int g_extra_arrivals = 0;
int g_forced_tile = 0;        // 0 = automatic, else 64, 128 or 256
int g_forced_wg_per_cu = 0;   // 0 = automatic (one workgroup per compute unit), else 1 or 2
int g_forced_waves = 0;       // 0 = automatic, else 4 or 8 wavefronts per workgroup of the 256 x 256 tile
thread_local int t_last_variant = 0;
thread_local int t_last_by_lines = 0;

struct Plan {
    int variant = 0;
    int shape = 0;     // a TileShape
    int tile_m = 0, tile_n = 0;  // rows and columns of a tile
    int NT = 0, RB = 0;
    int grid = 0, rounds = 0, swz_sc_log2 = -1, nt_log2 = 0, grid_log2 = 0, round_rows = 0;
    int mt = 0, strips = 0;  // small-M
    size_t partial_off = 0, partial_bytes = 0;
    size_t g_off = 0, g_bytes = 0;
    size_t total_bytes = 0;
    int split_s = 0;             // split kernel: workgroups per tile, 0 = another kernel
    int split_shape = 0;         // a SplitShape
    double split_us = 0.0;       // its estimated time
    size_t sums_off = 0;
};

// Which plans a call may take, by the scratch memory that there is: any; those without the finer tiles, which need up to twice the
// row statistics of the tiles they replace, or partial products where those need none; those that need least, which cut no K and keep the
// larger tiles.
enum Scratch { kScratchAny, kScratchCoarse, kScratchLeast };

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int validate_shape(int64_t M, int64_t K, int64_t N, int dtype)
{
    if (dtype != FF_F32 && dtype != FF_BF16)
        return FF_ERR_DTYPE;
    if (M <= 0 || K <= 0 || N <= 0)
        return FF_ERR_SHAPE;
    // K is bounded so that 256 rows of X or W span less than 4 GiB (the kernels
    // address a tile's rows with 32-bit byte offsets)
    if (M > (int64_t)1 << 30 || K > (int64_t)1 << 21 || N > (int64_t)1 << 30)
        return FF_ERR_SHAPE;
    const int vec = dtype == FF_BF16 ? 8 : 4;
    if (K % vec != 0 || N % vec != 0)
        return FF_ERR_UNSUPPORTED;
    return FF_OK;
}

// Decides variant, tile size, grid and workspace layout for a shape.
// Workgroups of the chosen tile kernel that fit a compute unit at once, asked of the runtime once per
// kernel and device; 0 when unknown.
int resident_blocks_per_cu(DeviceState *st, bool bf16, int shape, int mode)
{
    if (st == nullptr)
        return 0;
    signed char &slot = st->blocks_per_cu[bf16 ? 1 : 0][shape][mode];
    if (slot == 0) {
        const int n = tile_kernel_blocks_per_cu(bf16, shape, mode);
        slot = (signed char)(n <= 0 ? -1 : (n > 100 ? 100 : n));
    }
    return slot < 0 ? 0 : slot;
}

int resident_split_blocks(DeviceState *st, bool bf16, int shape)
{
    if (st == nullptr)
        return 0;
    signed char &slot = st->split_blocks[bf16 ? 1 : 0][shape];
    if (slot == 0) {
        const int n = split_kernel_blocks_per_cu(bf16, shape);
        slot = (signed char)(n <= 0 ? -1 : (n > 100 ? 100 : n));
    }
    return slot < 0 ? 0 : slot;
}

// Split kernel: the (shape, S) with the smallest estimated time among those whose workgroups all fit the
// chip at once, or false if there is none.  The estimate (microseconds, one launch after another, inputs
// from HBM) adds up what the kernel does one after the other:
//     start + max(slabs of a workgroup * time of one, W from HBM at the chip's rate or the active units')
//     + epilogue of a tile's share + exchange with the NT tiles of the rows
//     + S > 1: meeting of the tile's S workgroups and one write and read of the partial products
// Its constants were fitted to 3 600 runs (420 shapes drawn over M 1..8192, K 128..16384, N 128..16384, every
// shape and S of each); those of the epilogue of the larger tiles, which run eight wavefronts, in bf16 to 4 800 runs more
// (400 shapes, M 33..2048): the configuration picked is 0.6 (bf16) and 0.8 % (fp32) slower than the best on average.
// A unit draws at most 32 (26) bytes a nanosecond of W from HBM, so a few workgroups cannot stream at the chip's
// rate: 4 x 9272 x 15096 bf16 takes 102 us in 118 workgroups of 128-column tiles, 66 in 236 of 64.
// The busiest unit's share counts up to 16 rows, where the streamer is the other choice: of a grid of a few more
// workgroups than units some units read twice what the others do (3 x 10232 x 17024: 127 us in 266 workgroups, 110
// in 532 smaller ones).
//
// 32 x 32 tiles have a model of their own, fitted to 2 300 runs of 1 132 shapes (M 1..2048, K 128..8192, N 128..8192, S 1 to 4; off by
// 2 (fp32) and 3 % (bf16) on average): two to sixteen times as many tiles as of the other shapes, so that K need not be cut and the
// tile's workgroups need not meet, at twice the bytes through a unit's load path and more.  256 x 512 x 512 fp32 11.6 us,
// now 9.6; 512 x 1024 x 512 bf16 10.7, 8.6.  They are taken where their estimate is 4 (bf16, whose estimates scatter more: 10) % below the others', which
// are 6 % high here, in bf16 uncut and over 16 rows only (fp32: 0.91 of the time over all these shapes, 0.5 % above the better of the two, at
// most 1.03; bf16, where taken, 0.87, at most 0.93; between 0.90 and 0.99 of the others' estimate 0.90 to 1.07).
// fp32 over 64 rows has 64 x 32 tiles beside them, up to three a unit, from eight slabs on: bound by the matrix units, it gains from
// finer tiles where larger ones fill the last round badly.  Their model was fitted to 1 500 runs of 980 shapes (off by 2.6 %);
// taken where it says 6 % less than the others, whose estimates are 5 % high here, 0.91 of the time, 1 % above the better of the
// two, at most 1.02 (2033 x 2560 x 632 88 us, 69; 855 x 2272 x 1024 49, 47).  Two whole ones a unit do not replace tiles up to 128 x 64 with K cut in
// two (67 shapes 1.03 to 1.07: 256 x 2560 x 3840 50.6 us, 53.7; but 206 x 3840 x 4372, 128 x 128 cut in two, 0.62), nor more than 2.3 a unit under
// ten slabs where a row has 80 and more (60 shapes 1.03, at most 1.05: 256 x 256 x 5888 18.4 us, 19.2; up to 2.3 0.96 to 1.00, with 60 to 79 tiles 0.96).
struct SmallTiles {
    int shape = kSplit32, s = 0;
    double us = 0.0;
};
SmallTiles small_tiles(int64_t M, int64_t K, int64_t N, bool bf16, int num_cus, DeviceState *st)
{
    struct Cost { double start, slab, slab2, unit_hbm, epi, tiles, exch, exch_s, hbm; };
    constexpr Cost kBf16 = {6.15, 0.096, 0.221, 44.0e3, 0.13, 0.0383, 0.0, 0.0, 7.5e6};
    constexpr Cost kF32 = {5.68, 0.168, 0.32, 26.6e3, 0.80, 0.0372, 1.70, 0.197, 5.7e6};
    const Cost &c = bf16 ? kBf16 : kF32;
    const int size = bf16 ? 2 : 4;
    const int64_t slabs = (K * size + 127) / 128, RB = (M + 31) / 32, NT = (N + 31) / 32;
    SmallTiles best;
    // Where rows lie off the line boundaries and N ends inside a tile the larger tiles stay.  (They need not: in fp32 these would take 0.91 of
    // their time there, against 0.89 for rows on line boundaries.)
    // bf16 of up to eight slabs, whose one load latency the larger tiles wait for as well, gains nothing on average (59 shapes 1.00),
    // nor does it beyond 32 (K 2048 to 4096: 1.05), nor with two workgroups a unit and rows on 64-byte boundaries (0.98 to 1.14 of the larger
    // tiles' time: 1995 x 1280 x 256 11.0 us, 12.6 in 504 of these; rows off them 0.90 to 1.05: 671 x 1992 x 768 16.8, 15.4).
    // fp32 of few rows in 80 and more tiles each has too many to merge (70 shapes 1.07, at most 1.12: 29 x 416 x 2560 10.4, 11.5).
    const bool two_a_unit = !bf16 || K % 32 != 0;
    if ((bf16 && (M <= 16 || slabs <= 8 || slabs > 32)) || RB * NT > (two_a_unit ? 2 : 1) * (int64_t)num_cus ||
        (K * size % 128 != 0 && N % 32 != 0) || (!bf16 && M <= 64 && NT >= 80))
        return best;
    const int resident = resident_split_blocks(st, bf16, kSplit32);
    for (int S = 1; S <= (bf16 ? 1 : 4); S *= 2) {
        const int64_t groups = RB * NT * S, rounds = (groups + num_cus - 1) / num_cus;
        if (groups > (int64_t)num_cus * (resident == 1 ? 1 : 2) || (S > 1 && slabs < 4 * S) ||
            (RB * NT + RB * S * kSplitWays) * kSplitCounterStride * 4 > (int64_t)(kCtrlBytes - 2 * kCounterOffset))
            break;
        const double stream = (double)N * K * size / std::min(c.hbm, std::min<double>((double)groups, num_cus) * c.unit_hbm);
        double t = c.start + std::max((double)((slabs + S - 1) / S) * (rounds == 1 ? c.slab : c.slab2), stream) +
                   c.epi * (double)rounds / S + c.tiles * (double)NT;
        if (S > 1)
            t += c.exch + c.exch_s * S + (double)groups * 32 * 32 * 4 / 2.6e6;
        if (best.s == 0 || t < best.us) {
            best.s = S;
            best.us = t;
        }
    }
    return best;
}

SmallTiles flat_tiles(int64_t M, int64_t K, int64_t N, int num_cus, DeviceState *st, const Plan &other)
{
    constexpr double kSlab[] = {0.313, 0.530, 0.784};  // of one, two and three workgroups a unit
    const int64_t slabs = (K + 31) / 32, RB = (M + 31) / 32, NT = (N + 63) / 64;
    SmallTiles best;
    best.shape = kSplit64x32;
    if (M <= 64 || slabs < 8 || (K % 32 != 0 && N % 32 != 0))  // (as above)
        return best;
    const int resident = resident_split_blocks(st, false, kSplit64x32);
    const int64_t most = resident > 0 && resident < 3 ? resident : 3;
    for (int S = 1; S <= 2; S *= 2) {
        const int64_t groups = RB * NT * S;
        if (groups > num_cus * most ||
            (RB * NT + RB * S * kSplitWays) * kSplitCounterStride * 4 > (int64_t)(kCtrlBytes - 2 * kCounterOffset))
            break;
        const int64_t rounds = (groups + num_cus - 1) / num_cus;
        if ((S == 1 && rounds == 2 && other.split_s == 2 && other.split_shape != kSplit128) || (groups * 10 > 23 * num_cus && NT >= 80 && slabs < 10))
            continue;
        double t = 6.29 + (double)((slabs + S - 1) / S) * kSlab[rounds - 1] + 0.766 * (double)rounds / S + 0.0344 * (double)NT;
        if (S > 1)
            t += 1.02 + (double)groups * 64 * 32 * 4 / 2.5e6;
        t = std::max(t, 6.29 + (double)N * K * 4 / 5.1e6);
        if (best.s == 0 || t < best.us) {
            best.s = S;
            best.us = t;
        }
    }
    return best;
}

bool plan_split(int64_t M, int64_t K, int64_t N, bool bf16, int num_cus, DeviceState *st, bool finer, Plan &pl)
{
    // workgroups per compute unit that the LDS allows (what the runtime reports is asked as well)
    constexpr int kPerCu[] = {3, 2, 2, 1, 1};
    struct Cost { double start, slab, mfma, hbm, fabric, unit_hbm, exch, exch_s, sums, epi, epi_large, epi128, tiles; };
    constexpr Cost kBf16 = {4.2, 0.0, 0.128, 5.1e6, 51.6e3, 32e3, 2.4, 0.25, 2.8e6, 2.3, 1.9, 0.9, 0.052};
    constexpr Cost kF32 = {4.5, 0.134, 0.48, 5.1e6, 1e9, 26e3, 2.5, 0.2, 2.5e6, 3.0, 3.0, 0.78, 0.056};
    const Cost &c = bf16 ? kBf16 : kF32;
    const int size = bf16 ? 2 : 4;
    const int64_t slabs = (K * size + 127) / 128;
    Plan narrow;
    double best = 0.0, narrow_us = 0.0;
    for (int shape = 0; shape <= kSplit128; ++shape) {
        const int bm = split_shape_rows(shape), bn = split_shape_cols(shape);
        // tiles of few rows pay only where they spare the padding of larger ones
        if (bm == 32 && M > 64)
            continue;
        // Two row blocks of 128 x 32 in bf16 take W through four wavefronts' loads twice, which the estimate does not
        // know and which pays in short products only, or against uncut tiles of 128 x 64 (below).  Up to 18
        // slabs they take 0.94 of the time of the next best (89 shapes; 48 x 176 x 8176 11.1 us, 12.8), in longer ones 1.08
        // (67 shapes; 51 x 5080 x 15984 65.1, 51.5; 48 x 3784 x 13976 47.5, 38.7).
        const bool apart = bf16 && shape == kSplit128x32 && M > 32 && slabs > 18;
        Plan &to = apart ? narrow : pl;
        double &least = apart ? narrow_us : best;
        const int64_t RB = (M + bm - 1) / bm, NT = (N + bn - 1) / bn;
        if (RB * NT > (int64_t)num_cus * kPerCu[shape])
            continue;
        int per_cu = resident_split_blocks(st, bf16, shape);
        per_cu = per_cu > 0 && per_cu < kPerCu[shape] ? per_cu : kPerCu[shape];
        for (int S = 1; S <= kSplitMaxS; S *= 2) {
            const int64_t groups = RB * NT * S;
            if (groups > (int64_t)num_cus * per_cu ||
                (RB * NT + RB * S * kSplitWays) * kSplitCounterStride * 4 > (int64_t)(kCtrlBytes - 2 * kCounterOffset))
                break;
            // A share of fewer than two slabs, or a bf16 product of under ten (fp32: four), is not worth
            // the meeting: 256 x 512 x 512 bf16 takes 9.8 us whole and 9.6 to 9.9 split.
            if (S > 1 && (slabs < 2 * S || slabs < (bf16 ? 10 : 4)))
                break;
            // One 128 x 128 tile per unit with the whole of K is the tile kernel's ground where the
            // product is short (3584 x 512 x 768 bf16: 18.2 us there, 18.8 here; from nine slabs on the
            // deeper ring wins, 2048 x 8192 x 2048: 114 against 96) and in fp32, which is bound by the
            // matrix units (7400 x 1792 x 384: 126 against 135).
            if (shape == kSplit128 && S == 1 && (!bf16 || slabs <= 8))
                continue;
            const double per = (double)((slabs + S - 1) / S), wpc = (double)((groups + num_cus - 1) / num_cus);
            const double unit = bm * bn / 4096.0;
            const double slab = c.slab + std::max(c.mfma * unit * wpc, (bn + bm) * 128 * wpc / c.fabric);
            const double busiest = M <= 16 && wpc > 1 ? wpc * per * bn * 128 / c.unit_hbm : 0.0;
            const double stream = std::max((double)N * K * size / std::min(c.hbm, std::min<double>((double)groups, num_cus) * c.unit_hbm), busiest);
            double t = c.start + std::max(per * slab, stream) + (shape >= kSplit128x64 ? c.epi_large : c.epi) * unit / S * wpc + c.tiles * (double)NT +
                       (shape == kSplit128 ? c.epi128 : 0.0);
            if (S > 1)
                t += c.exch + c.exch_s * S + (double)groups * bm * bn * 4 / c.sums;
            if (least != 0.0 && t >= least)
                continue;
            least = t;
            to.split_s = S;
            to.split_shape = shape;
            to.tile_m = bm;
            to.tile_n = bn;
            to.RB = (int)RB;
            to.NT = (int)NT;
            to.grid = (int)groups;
        }
    }
    if (pl.split_s == 0)
        return false;
    // (44 x 1440 x 14520 23.3 us in two row blocks, 25.9 in 114 tiles of 128 x 64, on half of the units; 33 x 2408 x 16192
    // 34.5, 38.0; 64 x 1608 x 16048 29.4, 32.3)
    if (narrow.split_s != 0 && narrow_us < best && pl.split_shape == kSplit128x64 && pl.split_s == 1) {
        pl = narrow;
        best = narrow_us;
    }
    SmallTiles small = finer ? small_tiles(M, K, N, bf16, num_cus, st) : SmallTiles();
    const SmallTiles flat = finer && !bf16 ? flat_tiles(M, K, N, num_cus, st, pl) : SmallTiles();
    bool takes = small.s != 0 && small.us < (bf16 ? 0.90 * (best - 0.5) : 0.96 * (best - 0.3));
    if (flat.s != 0 && flat.us < 0.893 * best && !(takes && small.us <= flat.us)) {
        small = flat;
        takes = true;
    }
    if (takes) {
        best = small.us;
        pl.split_s = small.s;
        pl.split_shape = small.shape;
        pl.tile_m = split_shape_rows(small.shape);
        pl.tile_n = split_shape_cols(small.shape);
        pl.RB = (int)((M + pl.tile_m - 1) / pl.tile_m);
        pl.NT = (int)((N + pl.tile_n - 1) / pl.tile_n);
        pl.grid = pl.RB * pl.NT * pl.split_s;
    }
    // 128 x 128 tiles of long bf16 rows that do not begin on 64-byte boundaries keep four wavefronts.  By slabs every line of
    // a slab is requested twice, and eight wavefronts go to HBM for half of W's lines a second time (147 x 10568 x 6016
    // 89 us, with four 76; K = 10560: 62, 66).  206 such shapes, all by slabs: up to 48 slabs a workgroup eight win (0.94 of the time),
    // beyond them four do (0.95, at best 0.80: 1284 x 9832 x 2432 150 us, 119).  By lines, as four go where rows come from HBM, they take 0.84 of
    // that, and eight by lines would take 0.80 to 0.97 of four's time (1284 x 9832 x 2432 101 us, 80): this line was drawn before there were any.
    if (bf16 && pl.split_shape == kSplit128 && K % 32 != 0 && (slabs + pl.split_s - 1) / pl.split_s > 48)
        pl.split_shape = kSplit128W4;
    pl.rounds = 1;
    pl.split_us = best;
    const size_t rows = (size_t)pl.tile_m / pl.split_s, tiles = (size_t)pl.RB * pl.NT;
    pl.partial_off = kCtrlBytes;
    pl.partial_bytes = round_up(tiles * pl.split_s * (rows < 16 ? 16 : rows) * sizeof(floatx2), 256);
    pl.sums_off = pl.partial_off + pl.partial_bytes;
    pl.total_bytes = pl.sums_off + (pl.split_s > 1 ? tiles * pl.split_s * pl.tile_m * pl.tile_n * sizeof(float) : 0);
    return true;
}

int make_plan(int64_t M, int64_t K, int64_t N, int dtype, int num_cus, DeviceState *st, int forced,
              bool linear_only, Plan &pl, Scratch scratch = kScratchAny)
{
    const bool bf16 = dtype == FF_BF16, finer = scratch == kScratchAny, roomy = scratch != kScratchLeast;
    const int64_t strips = (N + kSmallMStripCols - 1) / kSmallMStripCols;
    const bool smallm_ok = bf16 && M <= 32 && strips <= (int64_t)num_cus * kSmallMMaxStripsPerGroup;

    int variant = forced;
    if (linear_only)
        variant = FF_VARIANT_TILED_TWOPASS;  // layout only; the launch uses the linear-only mode
    else if (variant == FF_VARIANT_AUTO)
        variant = smallm_ok ? FF_VARIANT_SMALL_M : 0;

    if (variant == FF_VARIANT_SMALL_M && !smallm_ok)
        return FF_ERR_UNSUPPORTED;
    // The streamer keeps M <= 16 where its estimated time is at most 2 % above the split kernel's: launch and merge,
    // W at the rate of the chip, the rounds of strips of a unit at the unit's rate, a round's epilogue, the meeting
    // of the strips (fitted to 440 shapes, K 64..16384, N 64..40000; it is off by 3 % on average).  Both sides were
    // timed on all of them: with this choice a call takes 0.891 of the streamer's time on average, 6 of them more
    // than 1.03 (at most 1.06).  (With cut slabs of the split kernel loaded like the others: 104 more shapes 1.2 % above the
    // better of the two.)  The streamer wins mostly with nearly whole rounds of strips (16 x 8192 x 8192: 37.2
    // us, 39 split; 2 x 800 x 16280, 509 strips: 18.6, 20.6) and with few slabs to cut (9 x 840 x 7248: 13.7, 15.6), the
    // split kernel elsewhere (14 x 4608 x 12888, 403 strips: 40, 34; 2 x 16128 x 1904, 60: 41.7, 26).
    // Over 16 rows the streamer's registers no longer cover its loads (22 x 5888 x 6008: 34.6, 22; never faster).
    // (A forced variant, tile or wavefront count names the kernel it named before there was a split one.)
    const bool may_split = roomy && !linear_only && forced == FF_VARIANT_AUTO && g_forced_tile == 0 && g_forced_waves == 0;
    if (may_split && plan_split(M, K, N, bf16, num_cus, st, finer, pl)) {
        // (short rows of W that end inside a line: 3 x 136 x 7720 stays with the streamer; from 512 on no such shape gains)
        const double split_us = pl.split_us + (K % 64 != 0 && K < 512 ? 0.7 : 0.0);
        const double rounds = (double)((strips + num_cus - 1) / num_cus);
        const double streamer_us = 7.3 + (double)N * K * 2 / 20e6 + rounds * ((double)K * 64 / 31.6e3 + 1.36) + 0.0102 * (double)strips;
        if (!(variant == FF_VARIANT_SMALL_M && M <= 16 && streamer_us < 1.02 * split_us)) {
            pl.variant = variant == FF_VARIANT_SMALL_M ? FF_VARIANT_SMALL_M : FF_VARIANT_TILED_FUSED;
            return FF_OK;
        }
        pl = Plan();
    }
    if (variant == FF_VARIANT_SMALL_M) {
        pl.variant = FF_VARIANT_SMALL_M;
        pl.mt = M <= 16 ? 1 : 2;
        pl.strips = (int)strips;
        pl.grid = (int)(strips < num_cus ? strips : num_cus);
        pl.partial_off = kCtrlBytes;
        pl.partial_bytes = round_up((size_t)strips * 16 * pl.mt * sizeof(float) * 2, 256);
        pl.total_bytes = pl.partial_off + pl.partial_bytes;
        return FF_OK;
    }

    // Tiled variants, by how many tiles of a shape there are per compute unit:
    //   more 256 x 256 tiles than half the compute units (in fp32, which is bound by the matrix units, only
    //     when 128 x 128 tiles two per unit would not do in one round: 2927 x 2952 x 2692 takes 395 us with
    //     those, 688 with 132 tiles of 256): 256 x 256 tiles, one workgroup of eight
    //     wavefronts per unit.  Two wavefronts per SIMD hide each other's latencies in the epilogue, and their
    //     accumulators leave room for the blocks of 16 x 16, which draw less power than four wavefronts' of 32 x 32
    //     (4096^3 112 against 127 us; 65536 x 1024 x 1024 149, 171; 8192 x 4096 x 16384 833, 967);
    //   else, in bf16, if the 128 x 128 tiles outnumber the units but the 256-column x 128-row tiles do not:
    //     256 x 128 tiles, one per unit, in one round, with three slabs of LDS and eight wavefronts (in fp32 128 x 128
    //     tiles win by a third): 1024 x 4096 x 8192 68 us, 15 such shapes 1.25 times as fast as with two slabs and four
    //     wavefronts.  (Four wavefronts and three slabs: 34 shapes 6 % slower, and 28 of nearly full chips with cut rows of
    //     32 and more tiles 4 %; 256 x 4448 x 31976, 1 % faster, is the best of them.)  Up to a quarter more 128 x 128 tiles than units go two per unit where one of these holds:
    //     an odd number of them a row, which leaves half a 256-column tile empty (1843 x 5264 x 2312 85.5, with 256 x 128
    //     100.7; 1459 x 7640 x 2848 132, 145); at most eight more than 256 units and more than 4 a row (591 x 936 x 6560
    //     27.0, 31.3; with 4, 16891 x 3856 x 256, 113, 88); a short product (11899 x 72 x 344 13.9, 14.8).  They never do
    //     where twice the tiles of a row to merge
    //     outweigh the product (rows of more than 12 tiles of 256 columns with K < 32 times their number: 523 x 256 x
    //     7872 27.0, 22.8) or W is narrow and K long (9354 x 5680 x 512 147, 121).  Elsewhere 256 x 128: 5115 x 2688 x
    //     1024 46.3, 60.6; 18048 x 4416 x 256 71.1, 94.3.  98 shapes of 257 to 325 tiles 1 % above the better of the two.
    //     In several rounds 256 x 128 tiles lose to 256 x 256 (30 shapes 0.85);
    //   else 128 x 128 tiles, up to two per unit, which finish in one round; and for at most a
    //     quarter of the units' worth of those, 64 x 64 tiles, which spread them further.  (Most of these
    //     smaller problems go to the split kernel above; what is left is what does not fit it.)
    const int64_t tiles256 = ((M + 255) / 256) * ((N + 255) / 256);
    const int64_t tiles256x128 = ((M + 127) / 128) * ((N + 255) / 256);
    const int64_t tiles128 = ((M + 127) / 128) * ((N + 127) / 128);
    const int64_t across = (N + 255) / 256;
    const bool pays = across > 12 ? K >= 32 * across : (across > 2 || K < 4500);
    const bool half_empty = ((N + 127) / 128) % 2 != 0;
    const bool two_a_unit = tiles128 * 4 <= 5 * num_cus && pays &&
                            (half_empty || (tiles128 * 32 <= 33 * num_cus && across > 2) || K < 256);
    // (A plan for the least scratch memory splits nothing and keeps the larger tiles, which have half the row statistics.)
    // fp32 in several rounds: 128 x 128 tiles, two a unit, in plain order.  A round of them is two units of matrix time, one of at
    // most half as many 1.15 (a unit's lone workgroup does not quite fill its matrix pipes), where a round of 256 x 256 tiles is
    // four units, however few of the compute units have one.  Microseconds: matrix time, and the rest of a tile.  70 shapes (M, N
    // 512..8192, K 64..4096): 0.865 of the time with 256 x 256 tiles throughout, 0.2 % above the better of the two (7656 x
    // 1764 x 2144, two rounds of 135, 832 us, 443; 5632 x 2708 x 3072 1233, 798; 2999 x 1416 x 3436, one of 168, 344, 272).
    //
    // 64 x 64 tiles, four a unit, also in plain order, where even 128 x 128 tiles leave units half idle: a round of up to as many of these
    // as units is a unit of matrix time, of up to twice as many two, where 64 x 64 tiles count in quarters.  They take more for
    // each unit and for each tile of a row.  540 shapes of 129 to 520 tiles of 128 x 128: 0.89 of the time, 0.6 % above the
    // better of the two, at most 1.05 (2906 x 4056 x 740 254 us, 189; 655 x 1216 x 3008 84, 66; 2637 x 156 x 868 22.7, 18.8; in rows of 70 and
    // more tiles of 128 short products lose up to twofold: 982 x 172 x 7668 44, 99).
    bool in_turn = false, in_turn64 = false;
    // (the estimates below are of two and four workgroups a unit: not where the runtime says that a unit holds fewer)
    auto holds = [&](int shape, int workgroups) {
        const int fit = resident_blocks_per_cu(st, bf16, shape, kFused);
        return fit == 0 || fit >= workgroups;
    };
    // (Where the row statistics fit the entry point that allocates nothing, so that both have the same bits; the fewer row-blocks
    // of larger tiles for very long X.)
    const bool room128 = kCtrlBytes + (size_t)tiles128 * 128 * sizeof(floatx2) <= kNoAllocBytes && (M + 127) / 128 < kMaxRowBlocks &&
                         N <= 128 * (int64_t)num_cus;
    if (!bf16 && may_split && finer && room128 && tiles128 > 2 * num_cus) {
        const int64_t rest = tiles128 % (2 * num_cus);
        const double units = 2.0 * (double)(tiles128 / (2 * num_cus)) + (rest == 0 ? 0.0 : (rest <= num_cus ? 1.15 : 2.0));
        const int64_t rows256 = (M + 255) / 256;
        const double rounds256 = (double)(across * 2 <= num_cus ? (rows256 + num_cus / across - 1) / (num_cus / across)
                                                                : (tiles256 + num_cus - 1) / num_cus);
        const double us128 = 6.0 + units * (0.0561 * (double)K + 6.8 + 0.03 * (double)((N + 127) / 128));
        const double us256 = 6.0 + rounds256 * (0.216 * (double)K + 22.0);
        in_turn = us128 < 0.92 * us256 && holds(kTile128, 2);
    }
    const int64_t tiles64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (!bf16 && may_split && finer && (in_turn || (tiles128 <= 2 * num_cus && tiles128 * 4 > num_cus)) && N <= 128 * (int64_t)num_cus &&
        kCtrlBytes + (size_t)tiles64 * 64 * sizeof(floatx2) <= kNoAllocBytes && (M + 63) / 64 < kMaxRowBlocks) {
        const int64_t rest = tiles128 % (2 * num_cus), rest64 = tiles64 % (4 * num_cus);
        const double units128 = 2.0 * (double)(tiles128 / (2 * num_cus)) + (rest == 0 ? 0.0 : (rest <= num_cus ? 1.15 : 2.0));
        const double units64 = (double)(tiles64 / (4 * num_cus)) + 0.25 * (double)((rest64 + num_cus - 1) / num_cus);
        const double k = (double)K, nt128 = (double)((N + 127) / 128), nt64 = (double)((N + 63) / 64);
        in_turn64 = 9.1 - 0.126 * nt64 + units64 * (0.0595 * k + 1.8 + 0.342 * nt64) <
                    0.94 * (2.1 + units128 * (0.0541 * k + 9.1 + 0.034 * nt128)) && holds(kTile64, 4);
    }
    // bf16 where little more than half of the units would have a 256 x 256 tile: one round of tiles of half the height, one
    // a unit (22 shapes 0.83 of the time: 2616 x 512 x 2944 25.5 us, 19.9; 612 x 3984 x 12200 123, 92), or else of 128 x 128 tiles, two
    // a unit (27 shapes 0.85: 9190 x 256 x 880 22.6, 17.9; 16843 x 5376 x 296 124, 96; with rows of more than 64 of them 726 x
    // 2048 x 10856 52.7, 55.3).  So too two rounds of these for two of those, if a row has up to 16 (14 shapes 0.80: 9596 x 256 x
    // 1552 40.6, 30.3; 22038 x 7936 x 552 345, 291; with 40 and more 0.9 to 1.3).  Not where plain order (below) saves half a round.
    bool pair_half = false, pair128 = false;
    if (bf16 && may_split && finer && room128 && tiles256 * 2 > num_cus) {
        const int64_t rows256 = (M + 255) / 256, rows128 = (M + 127) / 128, across128 = (N + 127) / 128;
        const bool one = tiles256 <= num_cus, plain = across * 2 <= num_cus && rows256 == num_cus / across + 1 && K >= 2048;
        const bool two = !one && across * 2 <= num_cus && rows256 <= 2 * (num_cus / across) && !plain;
        pair_half = one && tiles256x128 <= num_cus;
        pair128 = !pair_half && ((one && tiles128 <= 2 * num_cus && across128 <= 64) ||
                                 (two && across128 <= 16 && rows128 <= 2 * (2 * num_cus / across128))) && holds(kTile128, 2);
    }
    if (in_turn64)
        pl.shape = kTile64;
    else if (in_turn || pair128)
        pl.shape = kTile128;
    else if (pair_half)
        pl.shape = kTile256x128;
    else if (tiles256 * 2 > num_cus && (bf16 || !roomy || tiles128 > 2 * num_cus))
        pl.shape = kTile256W8;
    else if (bf16 && tiles128 > num_cus && tiles256x128 <= num_cus && !(roomy && two_a_unit))
        pl.shape = kTile256x128;
    else
        pl.shape = tiles128 * 4 > num_cus ? kTile128 : kTile64;
    if (g_forced_tile != 0) {
        pl.shape = g_forced_tile == 64 ? kTile64 : (g_forced_tile == 128 ? kTile128 : kTile256);
        if (g_forced_tile == 256 && g_forced_wg_per_cu == 2)
            pl.shape = kTile256x128;
    }
    if (g_forced_waves != 0) {
        if (tile_shape_cols(pl.shape) != 256)
            return FF_ERR_UNSUPPORTED;
        pl.shape = g_forced_waves == 8 ? kTile256W8 : kTile256;
    }
    pl.tile_m = tile_shape_rows(pl.shape);
    pl.tile_n = tile_shape_cols(pl.shape);
    const int64_t RB = (M + pl.tile_m - 1) / pl.tile_m;
    const int64_t NT = (N + pl.tile_n - 1) / pl.tile_n;
    if (RB > kMaxRowBlocks - 1 || RB * NT > (int64_t)1 << 30)  // the last counter pair belongs to the cross-entropy kernel
        return FF_ERR_SHAPE;
    pl.RB = (int)RB;
    pl.NT = (int)NT;
    const int64_t total = RB * NT;
    // workgroups per compute unit: a tile of 256 columns takes a whole unit's LDS, the other shapes half or less
    int per_cu = tile_shape_cols(pl.shape) == 256 ? 1 : (in_turn64 ? 4 : 2);
    in_turn = in_turn || in_turn64;
    if (g_forced_wg_per_cu == 1)
        per_cu = 1;
    // The fused kernel's workgroups wait for one another inside the launch: never launch more of them
    // than the runtime says are resident at once.
    if (variant != FF_VARIANT_TILED_TWOPASS && !linear_only) {
        const int fit = resident_blocks_per_cu(st, bf16, pl.shape, kFused);
        if (fit > 0 && per_cu > fit)
            per_cu = fit;
    }
    const int64_t grid_cap = (int64_t)num_cus * per_cu;
    pl.grid = (int)(total < grid_cap ? total : grid_cap);
    pl.rounds = (int)((total + pl.grid - 1) / pl.grid);
    const bool fused_ok = NT <= pl.grid;
    if (variant == 0)
        variant = fused_ok ? FF_VARIANT_TILED_FUSED : FF_VARIANT_TILED_TWOPASS;
    if (variant == FF_VARIANT_TILED_FUSED && !fused_ok)
        return FF_ERR_UNSUPPORTED;
    if (variant != FF_VARIANT_TILED_FUSED && variant != FF_VARIANT_TILED_TWOPASS)
        return FF_ERR_UNSUPPORTED;
    pl.variant = variant;
    // XCD-aware tile order: needs 8 XCDs x 32 or 64 workgroups and NT a power of two that divides
    // the grid (the kernel's index arithmetic is then all shifts)
    pl.swz_sc_log2 = -1;
    pl.nt_log2 = 0;
    pl.grid_log2 = 0;
    if (!in_turn && (pl.grid == 256 || pl.grid == 512) && NT <= pl.grid && (NT & (NT - 1)) == 0) {
        int sc = (int)(NT / 8 > 8 ? NT / 8 : 8);
        if (sc > NT)
            sc = (int)NT;
        while ((1 << pl.nt_log2) < NT)
            ++pl.nt_log2;
        while ((1 << pl.grid_log2) < pl.grid)
            ++pl.grid_log2;
        pl.swz_sc_log2 = 0;
        while ((1 << pl.swz_sc_log2) < sc)
            ++pl.swz_sc_log2;
    }
    // Every other fused launch: rounds of whole row-blocks, as many in each.  A row-block whose tiles lie in
    // two rounds makes those of the first wait, accumulators and all, for the second (23040 x 408 x 9584, 37
    // tiles a row: 651 us, with whole row-blocks 492 in one round more); spreading the row-blocks evenly
    // costs nothing, as the chip's power sets the rate (24064 x 7056 x 768, 47 row-blocks in each of two
    // rounds instead of 85 and 9: 460 -> 436 us).  Rows of more than half the grid's tiles stay in plain order:
    // whole ones would leave up to half the chip idle.  So does a long bf16 product of one row-block more than a
    // round holds: a full round and a few tiles on a cool chip beat two half rounds (10823 x 4608 x 1536, 43 row-blocks
    // of which 42 fit: 240 us in halves, 223; 3614 x 2904 x 4584, 15 and 14: 204, 180; 20 such shapes with K >= 2048 take
    // 0.95 of the time on average, none more than 1.02.  With K below that, two row-blocks more, or three rounds
    // halves are as fast or faster: 3736 x 1656 x 8632, three rounds: 178, 211).
    // And so does a short fp32 product on more than one workgroup per unit but not two, where plain order already
    // gives an XCD whole columns (NT a multiple of 8): its row-blocks end one after the other, and their stores
    // run beside the products of the rest (652 x 172 x 8084, 384 tiles: 52.1 us in rounds, 44.0; 1227 x 204 x 4032:
    // 47.0, 42.7; 34 such shapes with K < 600 take 0.98 of the time on average, 36 longer ones 1.01).
    const bool staggered = !bf16 && total > num_cus && total == pl.grid && NT % 8 == 0 && K < 600;
    if (pl.swz_sc_log2 < 0 && NT * 2 <= pl.grid && variant == FF_VARIANT_TILED_FUSED && !linear_only && !staggered && !in_turn) {
        const int64_t most = pl.grid / NT < RB ? pl.grid / NT : RB, rounds = (RB + most - 1) / most;
        if (!(bf16 && RB == most + 1 && K >= 2048)) {
            pl.rounds = (int)rounds;
            pl.round_rows = (int)((RB + rounds - 1) / rounds);
            pl.grid = (int)(pl.round_rows * NT);
        }
    }
    pl.partial_off = kCtrlBytes;
    pl.partial_bytes = round_up((size_t)total * pl.tile_m * sizeof(float) * 2, 256);
    pl.g_off = pl.partial_off + pl.partial_bytes;
    pl.g_bytes = (variant == FF_VARIANT_TILED_TWOPASS && !linear_only)
                     ? round_up((size_t)M * (size_t)N * sizeof(float), 256)
                     : 0;
    pl.total_bytes = pl.g_off + pl.g_bytes;
    return FF_OK;
}

DeviceState *current_device_state(int *dev_out = nullptr)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    DeviceState &st = g_dev[dev];
    if (!st.probed) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            st.num_cus = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeWallClockRate, dev) == hipSuccess && v > 0)
            st.ticks_per_us = v / 1000 > 0 ? v / 1000 : 1;
        (void)hipGetLastError();
        st.probed = true;
    }
    if (dev_out)
        *dev_out = dev;
    return &st;
}

void note_recording(DeviceState &st, hipStream_t stream)
{
    if (!st.ws_owned || st.ws_recorded)
        return;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess)
        (void)hipGetLastError();
    else
        st.ws_recorded = capture != hipStreamCaptureStatusNone;
}

// Gives up the library's own workspace: kept if a graph may use it, else freed.
bool release_own(DeviceState &st)
{
    if (st.ws_recorded && st.n_kept < (int)(sizeof(st.kept) / sizeof(st.kept[0])))
        st.kept[st.n_kept++] = {st.ws, st.ws_bytes};
    else if (hipDeviceSynchronize() != hipSuccess || hipFree(st.ws) != hipSuccess)
        return false;
    st.ws = nullptr;
    st.ws_bytes = 0;
    st.ws_owned = st.ws_recorded = false;
    return true;
}

// Makes sure a workspace of at least `bytes` exists.  The control region of a workspace is zeroed,
// synchronously, when it is allocated here or bound by ff_set_workspace, never on a caller's stream;
// the kernels leave it zero behind them.  Allocating, freeing and synchronising are illegal while a
// stream is being captured, so a call that would have to grow the library's own workspace during a
// capture is refused instead.
//
// A graph holds the address of the workspace it was recorded with.  One of the library's own that a captured
// call has used is therefore never freed: outgrown, or replaced by a caller's, it is kept for the replays (and
// taken again where it is large enough).  Each is at least a quarter larger than the need that outgrew the one
// before, so they are few (64 reach from 1 MiB to beyond any device) and no more than five times the largest.
int prepare_workspace(DeviceState &st, size_t bytes, hipStream_t stream)
{
    if (st.ws != nullptr && st.ws_bytes >= bytes) {
        note_recording(st, stream);
        return FF_OK;
    }
    if (st.ws != nullptr && !st.ws_owned)
        return FF_ERR_WORKSPACE;  // the caller's workspace is too small
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return FF_ERR_WORKSPACE;
    }
    if (capture != hipStreamCaptureStatusNone)
        return FF_ERR_WORKSPACE;
    if (st.ws != nullptr && !release_own(st)) {
        (void)hipGetLastError();
        return FF_ERR_LAUNCH;
    }
    int fits = -1;  // the smallest kept one that is large enough
    for (int i = 0; i < st.n_kept; ++i)
        if (st.kept[i].bytes >= bytes && (fits < 0 || st.kept[i].bytes < st.kept[fits].bytes))
            fits = i;
    if (fits >= 0) {
        st.ws = st.kept[fits].ptr;
        st.ws_bytes = st.kept[fits].bytes;
        st.ws_owned = st.ws_recorded = true;
        st.kept[fits] = st.kept[--st.n_kept];
        return FF_OK;
    }
    const size_t want = round_up(bytes + bytes / 4, 1 << 20);
    void *mem = nullptr;
    if (hipMalloc(&mem, want) != hipSuccess) {
        (void)hipGetLastError();
        return FF_ERR_WORKSPACE;
    }
    if (init_control_region(mem) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(mem);
        return FF_ERR_LAUNCH;
    }
    st.ws = mem;
    st.ws_bytes = want;
    st.ws_owned = true;
    st.ws_recorded = false;
    return FF_OK;
}

// Host memory of at least `bytes` that kernels can write to, or null: up to 4 MiB a device.  It belongs to the library's own workspace: a
// caller who binds memory gets no allocation from a call, and binding or unbinding frees it.  Used under the lock from launch to
// synchronisation, so that nothing is in flight when it is freed or replaced by a larger one.
// (A copy into pageable memory behind the kernel: eight tasks of 10 x 300 take 15 us longer.)
constexpr size_t kPinnedMost = 4u << 20;
void release_pinned(DeviceState &st)
{
    if (st.pinned != nullptr && hipHostFree(st.pinned) != hipSuccess)
        (void)hipGetLastError();
    st.pinned = nullptr;
    st.pinned_bytes = 0;
}
void *pinned_results(DeviceState &st, size_t bytes, hipStream_t stream)
{
    if (bytes > kPinnedMost)
        return nullptr;
    if (st.pinned_bytes < bytes) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        void *mem = nullptr;
        const size_t want = std::min(kPinnedMost, round_up(2 * bytes, 64u << 10));
        if (hipStreamIsCapturing(stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone ||
            hipHostMalloc(&mem, want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        release_pinned(st);
        st.pinned = mem;
        st.pinned_bytes = want;
    }
    return st.pinned;
}

// The largest workspace a call on this stream can have: what a caller bound, or during a capture what the
// library already owns (growing it would be illegal), is fixed.
size_t workspace_limit(DeviceState &st, hipStream_t stream)
{
    if (st.ws != nullptr && !st.ws_owned)
        return st.ws_bytes;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return st.ws_bytes;
    }
    return capture != hipStreamCaptureStatusNone ? st.ws_bytes : SIZE_MAX;
}

bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// This device's copies of the static scratch arrays (asked of the runtime once per device, with that
// device current), or null if the runtime refuses.
void *no_alloc_scratch(DeviceState &st)
{
    if (st.no_alloc_ptr == nullptr) {
        void *ptr = nullptr;
        void *sums = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr ||
            hipGetSymbolAddress(&sums, HIP_SYMBOL(scratch_sums)) != hipSuccess || sums == nullptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        st.no_alloc_ptr = ptr;
        st.no_alloc_sums = sums;
    }
    return st.no_alloc_ptr;
}

int run(const void *X, const void *W, const void *b, const void *gamma, const void *beta, float eps,
        int64_t M, int64_t K, int64_t N, int dtype, void *Y, float *Z, bool linear_only,
        hipStream_t stream, bool no_alloc = false)
{
    int rc = validate_shape(M, K, N, dtype);
    if (rc != FF_OK)
        return rc;
    if (!X || !W || (!linear_only && !Y) || (linear_only && !Z))
        return FF_ERR_NULL;
    if (misaligned(X) || misaligned(W) || misaligned(b) || misaligned(gamma) || misaligned(beta) ||
        misaligned(Y) || misaligned(Z))
        return FF_ERR_ALIGN;

    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    // the first plan that the scratch memory holds, or else the one that needs least
    Plan pl;
    for (const Scratch scratch : {kScratchAny, kScratchCoarse, kScratchLeast}) {
        pl = Plan();
        rc = make_plan(M, K, N, dtype, st->num_cus, st, g_forced_variant, linear_only, pl, scratch);
        if (rc != FF_OK)
            return rc;
        const size_t held = pl.split_s > 0 ? pl.sums_off : pl.total_bytes;  // without the partial products
        if (no_alloc ? held <= kNoAllocBytes && pl.total_bytes - held <= kNoAllocSumBytes
                     : pl.total_bytes <= st->ws_bytes || pl.total_bytes <= workspace_limit(*st, stream))
            break;
    }
    char *ws = nullptr;
    if (no_alloc) {
        // the static array is the workspace; what the kernels expect to find zero (error word, the
        // arrival counters this plan uses) is cleared by a kernel on the caller's stream first
        if ((pl.split_s > 0 ? pl.sums_off : pl.total_bytes) > kNoAllocBytes)
            return FF_ERR_WORKSPACE;
        ws = static_cast<char *>(no_alloc_scratch(*st));
        if (ws == nullptr)
            return FF_ERR_LAUNCH;
        // the error word (offset 0) is cleared by the first call on a device only: later calls leave a
        // failure flagged by an earlier one for ff_check_device to report
        const size_t first = st->no_alloc_used ? kCounterOffset : 0;
        const size_t ctrl =
            kCounterOffset +
            sizeof(unsigned) * (pl.split_s > 0 ? ((size_t)pl.RB * pl.NT + (size_t)pl.RB * pl.split_s * kSplitWays) * kSplitCounterStride
                                : pl.variant == FF_VARIANT_SMALL_M ? (size_t)kSyncWays * kSyncStride
                                                                   : (size_t)row_counter_pairs(pl.RB) * 2);
        const size_t words = (ctrl - first + 3) / 4;
        hipLaunchKernelGGL(fill_words_kernel, dim3((unsigned)((words + 255) / 256 < 64 ? (words + 255) / 256 : 64)),
                           dim3(256), 0, stream, reinterpret_cast<unsigned *>(ws + first), words, 0u);
        if (hipGetLastError() != hipSuccess)
            return FF_ERR_LAUNCH;
        st->no_alloc_used = true;
    } else {
        rc = prepare_workspace(*st, pl.total_bytes, stream);
        if (rc != FF_OK)
            return rc;
        ws = static_cast<char *>(st->ws);
    }
    unsigned *err = reinterpret_cast<unsigned *>(ws);
    unsigned *counters = reinterpret_cast<unsigned *>(ws + kCounterOffset);
    const long long wait_ticks = g_wait_limit_us * st->ticks_per_us;
    const bool bf16 = dtype == FF_BF16;

    if (pl.variant == FF_VARIANT_SMALL_M && pl.split_s == 0) {
        SmallMParams p{};
        p.X = X; p.W = W; p.b = b; p.gamma = gamma; p.beta = beta; p.Y = Y;
        p.partials = reinterpret_cast<floatx2 *>(ws + pl.partial_off);
        p.counters = counters;
        p.err = err;
        p.eps = eps;
        p.M = (int)M; p.K = (int)K; p.N = (int)N;
        p.strips = pl.strips;
        p.extra_arrivals = g_extra_arrivals;
        p.wait_ticks = wait_ticks;
        p.timeline = (st->timeline != nullptr &&
                      st->timeline_bytes >= (size_t)pl.grid * kTimelineSlots * sizeof(unsigned long long))
                         ? st->timeline
                         : nullptr;
        if (launch_smallm_kernel(pl.mt, p, pl.grid, stream) != hipSuccess)
            return FF_ERR_LAUNCH;
        t_last_by_lines = 0;
        t_last_variant = pl.variant;
        return FF_OK;
    }

    if (pl.split_s > 0) {
        SplitParams p{};
        p.X = X; p.W = W; p.b = b; p.gamma = gamma; p.beta = beta; p.Y = Y;
        p.sums = static_cast<float *>(no_alloc ? st->no_alloc_sums : ws + pl.sums_off);
        p.partials = reinterpret_cast<floatx2 *>(ws + pl.partial_off);
        p.counters = counters;
        p.err = err;
        p.eps = eps;
        p.M = (int)M; p.K = (int)K; p.N = (int)N;
        p.NT = pl.NT; p.RB = pl.RB; p.S = pl.split_s;
        p.extra_arrivals = g_extra_arrivals;
        p.wait_ticks = wait_ticks;
        p.timeline = (st->timeline != nullptr &&
                      st->timeline_bytes >= (size_t)pl.grid * kTimelineSlots * sizeof(unsigned long long))
                         ? st->timeline
                         : nullptr;
        if (launch_split_kernel(bf16, pl.split_shape, p, pl.grid, stream) != hipSuccess)
            return FF_ERR_LAUNCH;
        t_last_by_lines = split_kernel_by_lines(bf16, pl.split_shape, p);
        t_last_variant = pl.variant;
        return FF_OK;
    }

    TileParams p{};
    p.X = X; p.W = W; p.b = b; p.gamma = gamma; p.beta = beta; p.Y = Y;
    p.F = linear_only ? Z : reinterpret_cast<float *>(ws + pl.g_off);
    p.partials = reinterpret_cast<floatx2 *>(ws + pl.partial_off);
    p.counters = counters;
    p.err = err;
    p.eps = eps;
    p.M = (int)M; p.K = (int)K; p.N = (int)N;
    p.NT = pl.NT; p.RB = pl.RB; p.rounds = pl.rounds; p.round_rows = pl.round_rows; p.swz_sc_log2 = pl.swz_sc_log2; p.nt_log2 = pl.nt_log2;
    p.grid_log2 = pl.grid_log2;
    p.extra_arrivals = g_extra_arrivals;
    p.wait_ticks = wait_ticks;
    p.timeline = nullptr;
    p.timeline_rounds = 0;
    if (st->timeline != nullptr) {
        const size_t per_round = (size_t)pl.grid * kTimelineSlots * sizeof(unsigned long long);
        const size_t rounds = st->timeline_bytes / per_round;
        p.timeline = rounds > 0 ? st->timeline : nullptr;
        p.timeline_rounds = (int)(rounds < (size_t)pl.rounds ? rounds : (size_t)pl.rounds);
    }
    const int mode = linear_only ? kLinearOnly
                                 : (pl.variant == FF_VARIANT_TILED_FUSED ? kFused : kTwoPass);
    if (launch_tile_kernel(bf16, pl.shape, mode, p, pl.grid, stream) != hipSuccess)
        return FF_ERR_LAUNCH;
    if (mode == kTwoPass) {
        FinalizeParams f{};
        f.G = p.F; f.partials = p.partials; f.gamma = gamma; f.beta = beta; f.Y = Y;
        f.eps = eps; f.M = (int)M; f.N = (int)N; f.NT = pl.NT; f.BM = pl.tile_m; f.BN = pl.tile_n;
        if (launch_finalize_kernel(bf16, f, stream) != hipSuccess)
            return FF_ERR_LAUNCH;
    }
    if (!linear_only) {
        t_last_variant = pl.variant;
        t_last_by_lines = tile_kernel_by_lines(bf16, pl.shape, mode, p);
    }
    return FF_OK;
}

}  // namespace

extern "C" {

int ff_fused_linear_gelu_ln(const void *X, const void *W, const void *b, const void *gamma,
                            const void *beta, float eps, int64_t M, int64_t K, int64_t N, int dtype,
                            void *Y, void *stream)
{
    return run(X, W, b, gamma, beta, eps, M, K, N, dtype, Y, nullptr, false,
               static_cast<hipStream_t>(stream));
}

int ff_fused_linear_gelu_ln_noalloc(const void *X, const void *W, const void *b, const void *gamma,
                                    const void *beta, float eps, int64_t M, int64_t K, int64_t N, int dtype,
                                    void *Y, void *stream)
{
    return run(X, W, b, gamma, beta, eps, M, K, N, dtype, Y, nullptr, false,
               static_cast<hipStream_t>(stream), true);
}

size_t ff_noalloc_max_bytes(void) { return kNoAllocBytes; }

int ff_debug_linear(const void *X, const void *W, const void *b, int64_t M, int64_t K, int64_t N,
                    int dtype, float *Z_f32, void *stream)
{
    return run(X, W, b, nullptr, nullptr, 0.0f, M, K, N, dtype, nullptr, Z_f32, true,
               static_cast<hipStream_t>(stream));
}

}  // extern "C"

namespace {

// Column strips and row chunks of the second chain's first phase: 128-byte strips, and the number of row
// chunks with the least estimated time, in rows of a workgroup (4 ns): its rounds of (strip, chunk) items, each
// worth its rows and 75 more for the reductions; 60 for a batch of four chunks in the second phase's sum (16 chunks
// or more share the work of adding); and the reading of the partial sums, which every unit does for itself.
// Fitted to 301 shapes (K 8..32768, N 64..2^20, up to 18 chunk counts of each): 0.6 % slower than the best count on
// average.  (256 / strips chunks at most: 2.7 %, with 160 strips of 256 x 5120 x 2072 fp32 whole on 160 of 256
// units; without the last two terms: 2.9 %, with 120 x 960 x 16036 fp32 20.6 us in 17 chunks, 19.0 in 8, and
// 64 x 6560 x 1816 23.1 in 6, 18.7 in one.)
// `most` bounds the scratch memory for the partial sums.
struct RowMeanPlan {
    int strips, k_pad, chunks, rows_per_chunk;
    size_t partial_bytes, cpart_bytes;
};

RowMeanPlan rowmean_plan(int64_t K, int64_t N, int dtype, int num_cus, size_t most = SIZE_MAX)
{
    RowMeanPlan r{};
    const int64_t strip_elems = 128 / (dtype == FF_BF16 ? 2 : 4);
    r.strips = (int)((K + strip_elems - 1) / strip_elems);
    r.k_pad = (int)(r.strips * strip_elems);
    const int64_t q = kRowMeanRowsPerStep;
    int64_t best = 0;
    // Up to 64 chunks; of very many rows, an item for every unit where there are fewer than four strips (2669 x 120 x
    // 961536 bf16, two strips, 99.7 us in 64, 84.8 in 128; 20 x 64 x 20000, one strip, 10.5 in 63, 11.1 in 105).
    const int64_t limit = r.strips < 4 && N >= (int64_t)1 << 17 ? 256 / r.strips : 64;
    for (int64_t want = 1; want <= limit; ++want) {
        const int64_t rows = ((N + want - 1) / want + q - 1) / q * q, chunks = (N + rows - 1) / rows;
        const int64_t cost = (r.strips * chunks + 255) / 256 * (rows + 75) + ((chunks < 16 ? chunks : 16) + 3) / 4 * 60 +
                             chunks * r.k_pad / 28;
        if (want > 1 && (cost >= best || (size_t)(chunks * r.k_pad) * sizeof(float) > most))
            continue;
        best = cost;
        r.rows_per_chunk = (int)rows;
        r.chunks = (int)chunks;
    }
    r.partial_bytes = round_up((size_t)r.chunks * (size_t)r.k_pad * sizeof(float), 256);
    r.cpart_bytes = round_up((size_t)num_cus * sizeof(float), 256);
    return r;
}

}  // namespace

extern "C" {

int ff_fused_linear_sub_rowmean_gelu_residual(const void *X, const void *W, const void *b, const void *s,
                                              int64_t M, int64_t K, int64_t N, int dtype, void *Out,
                                              void *stream)
{
    int rc = validate_shape(M, K, N, dtype);
    if (rc != FF_OK)
        return rc;
    if (!X || !W || !Out)
        return FF_ERR_NULL;
    if (misaligned(X) || misaligned(W) || misaligned(b) || misaligned(s) || misaligned(Out))
        return FF_ERR_ALIGN;
    if (K > kRowMeanMaxK)
        return FF_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    RowMeanParams p{};
    // a bound workspace, or the library's own during a capture, bounds the chunks; one chunk needs no more than before
    const size_t head = kCtrlBytes + round_up((size_t)st->num_cus * sizeof(float), 256);
    const size_t limit = workspace_limit(*st, static_cast<hipStream_t>(stream));
    const RowMeanPlan pl = rowmean_plan(K, N, dtype, st->num_cus, limit > head ? (limit - head) / 256 * 256 : 0);
    rc = prepare_workspace(*st, kCtrlBytes + pl.partial_bytes + pl.cpart_bytes, static_cast<hipStream_t>(stream));
    if (rc != FF_OK)
        return rc;
    char *ws = static_cast<char *>(st->ws);
    p.X = X; p.W = W; p.b = b; p.s = s; p.Out = Out;
    p.partial = reinterpret_cast<float *>(ws + kCtrlBytes);
    p.cpart = reinterpret_cast<float *>(ws + kCtrlBytes + pl.partial_bytes);
    p.counters = reinterpret_cast<unsigned *>(ws + kCounterOffset);
    p.err = reinterpret_cast<unsigned *>(ws);
    p.M = (int)M; p.K = (int)K; p.N = (int)N;
    p.strips = pl.strips; p.k_pad = pl.k_pad; p.chunks = pl.chunks; p.rows_per_chunk = pl.rows_per_chunk;
    p.grid = st->num_cus;  // one workgroup per compute unit, all resident: the phases meet inside the launch
    p.extra_arrivals = g_extra_arrivals;
    p.wait_ticks = g_wait_limit_us * st->ticks_per_us;
    if (launch_rowmean_chain(dtype == FF_BF16, p, static_cast<hipStream_t>(stream)) != hipSuccess)
        return FF_ERR_LAUNCH;
    return FF_OK;
}

}  // extern "C"

namespace {

size_t rowmean_workspace_bytes(int64_t K, int64_t N, int dtype)
{
    // sized for any device: the per-workgroup slices take at most 1024 compute units' worth
    const RowMeanPlan pl = rowmean_plan(K, N, dtype, 1024);
    return kCtrlBytes + pl.partial_bytes + pl.cpart_bytes;
}

}  // namespace

extern "C" {

size_t ff_rowmean_workspace_bytes(int64_t M, int64_t K, int64_t N, int dtype)
{
    if (validate_shape(M, K, N, dtype) != FF_OK)
        return 0;
    return rowmean_workspace_bytes(K, N, dtype);
}

int ff_cross_entropy_mean(const void *logits, const int64_t *targets, int64_t B, int64_t C, int dtype,
                          float *row_loss, float *mean_loss, void *stream)
{
    if (dtype != FF_F32 && dtype != FF_BF16)
        return FF_ERR_DTYPE;
    if (B <= 0 || C <= 0 || B > (int64_t)1 << 30 || C > (int64_t)1 << 30)
        return FF_ERR_SHAPE;
    if (!logits || !targets || !mean_loss)
        return FF_ERR_NULL;
    if (misaligned(logits) || (reinterpret_cast<uintptr_t>(targets) & 7u) ||
        (reinterpret_cast<uintptr_t>(row_loss) & 3u) || (reinterpret_cast<uintptr_t>(mean_loss) & 3u))
        return FF_ERR_ALIGN;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    XentParams p{};
    p.B = (int)B;
    p.C = (int)C;
    const int full = dtype == FF_BF16 ? 8 : 4;  // elements of a 16-byte load
    p.vec = C >= 4 * full ? full : 1;
    const int64_t chunks = C / p.vec;
    // Scratch memory: one pair per workgroup, or per segment and row.  A workspace of
    // ff_cross_entropy_workspace_bytes() holds either; a smaller one that a caller bound (or that the
    // library owns while the stream is captured) bounds the grid and rules segments out.
    const size_t limit = st->ws_bytes >= ff_cross_entropy_workspace_bytes(B, C, dtype)
                             ? st->ws_bytes
                             : workspace_limit(*st, static_cast<hipStream_t>(stream));
    // (in whole 256 bytes, as the need is rounded up to)
    const int64_t pairs = limit < kCtrlBytes + 256 ? 1 : (int64_t)std::min<size_t>((limit - kCtrlBytes) / 256 * 256 / sizeof(floatx2), 8192);
    int64_t groups, per_cu = 8;  // workgroups of four wavefronts: with 4 (2) per unit 65536 x 1000 fp32 takes 4 % (49 %) more
    if (chunks <= 512) {
        // A row in the registers of 4, 16 or 64 lanes, at most eight loads each.  (A wavefront per row whatever
        // its length, with the remainder of a batch loaded one after the other: 65536 x 16 fp32 41.4 us, now
        // 6.0; 65536 x 1000 106 -> 46.7; 56832 x 373 106 -> 24.)
        p.lanes = chunks <= 16 ? 4 : (chunks <= 64 ? 16 : 64);
        const int q = (int)((chunks + p.lanes - 1) / p.lanes);
        p.per_lane = q <= 1 && p.lanes == 4 ? 1 : (q <= 2 ? 2 : (q <= 4 ? 4 : 8));
        groups = (B * p.lanes + 255) / 256;
    } else {
        // A wavefront per row; fewer than six rows per unit are cut into segments, up to as many as make
        // about two wavefronts per SIMD (256 x 50257 fp32: 28.0 us whole, 14.1 in 8 segments, 14.8 in 12;
        // 512 x 32000 bf16: 16.0, 11.3 in 4, 12.3 in 8; 143 x 154624 fp32 28.7 in 8, 22.8 in 16) and down to 100 loads
        // each (26 x 5074 fp32 5.8 us in 4, 5.3 in 8, 6.1 in 16).  More rows than 2.5 per unit nearly fill the chip
        // themselves: two segments pay only for long ones in bf16 whose wavefronts still fit one round (963 x 50944
        // 26.4 whole, 23.9; but 1080 x 4899 fp32 9.6, 11.9; 1019 x 65536 fp32 48.8, 53.9; 1380 x 17976 bf16 14.9, 18.0).
        p.segs = 1;
        const int64_t cus = st->num_cus;
        const bool cut = B * 2 <= cus * 5 || (dtype == FF_BF16 && chunks >= 1024 && B <= cus * 4);
        while (cut && B * p.segs < cus * 6 && p.segs < kXentMaxSegs && chunks / (2 * p.segs) >= 100 && B * (2 * p.segs + 1) <= pairs)
            p.segs *= 2;
        const int64_t batch = 64 * 8;  // whole batches of loads per segment where there are enough
        p.seg_chunks = (int)((chunks + p.segs - 1) / p.segs);
        if (p.segs > 1 && p.seg_chunks > 4 * batch)
            p.seg_chunks = (int)((p.seg_chunks + batch - 1) / batch * batch);
        groups = (B * p.segs + 3) / 4;
        // Rows of two batches or more keep enough loads in flight with two workgroups per unit, and DRAM reads
        // few streams faster than many (32768 x 4096 fp32 84.7 against 86.9 us with eight, 4096 x 50257 bf16
        // 69.5 against 71.5), provided their rounds come out even (5120 x 13018 bf16, 2.5 rounds: 29.0, 26.8).
        const int64_t few = (int64_t)st->num_cus * 2, even = (groups + few - 1) / few * few;
        if (chunks >= 2 * batch && groups * 10 >= even * 9)
            per_cu = 2;
    }
    // as many rounds as the resident workgroups need, then as few workgroups as finish in that many
    const int64_t cap = std::min<int64_t>((int64_t)st->num_cus * per_cu, pairs);
    const int64_t rounds = (groups + cap - 1) / cap;
    p.grid = (int)((groups + rounds - 1) / rounds);
    const int64_t need = p.segs > 1 ? B * p.segs + B : p.grid;
    const int rc = prepare_workspace(*st, kCtrlBytes + round_up((size_t)need * sizeof(floatx2), 256),
                                     static_cast<hipStream_t>(stream));
    if (rc != FF_OK)
        return rc;
    char *ws = static_cast<char *>(st->ws);
    p.logits = logits;
    p.targets = reinterpret_cast<const long long *>(targets);
    p.row_loss = row_loss;
    p.mean_loss = mean_loss;
    p.partials = reinterpret_cast<floatx2 *>(ws + kCtrlBytes);
    p.picked = p.partials + B * p.segs;
    p.ways = reinterpret_cast<unsigned *>(ws + kCounterOffset);
    // the last counter pair of the control region; the tiled kernels never reach it
    p.counter = reinterpret_cast<unsigned *>(ws + kCounterOffset) + 2 * (kMaxRowBlocks - 1);
    if (launch_xent_kernel(dtype == FF_BF16, p, static_cast<hipStream_t>(stream)) != hipSuccess)
        return FF_ERR_LAUNCH;
    return FF_OK;
}

size_t ff_cross_entropy_workspace_bytes(int64_t B, int64_t C, int dtype)
{
    if ((dtype != FF_F32 && dtype != FF_BF16) || B <= 0 || C <= 0)
        return 0;
    // sized for the largest grid any device uses here (8 workgroups per compute unit, 1024 units)
    return kCtrlBytes + 8192 * sizeof(floatx2);
}

int ff_metric_select_host(const double *r, const uint8_t *keep, int64_t n_tasks, int64_t n_metrics,
                          int top_k, double percentile, int min_tasks, int32_t *top, double *score,
                          uint8_t *selected, double *threshold)
{
    if (!r)
        return FF_ERR_NULL;
    if (n_tasks <= 0 || n_metrics <= 0 || top_k <= 0 || n_tasks > 1 << 20 || n_metrics > 1 << 24 ||
        !(percentile >= 0.0 && percentile <= 100.0) || min_tasks < 1)
        return FF_ERR_SHAPE;
    try {
        metric_select_host(r, keep, (int)n_tasks, (int)n_metrics, top_k, percentile, min_tasks, top, score,
                           selected, threshold);
    } catch (...) {  // host allocation failed: nothing may leave through the C boundary
        return FF_ERR_WORKSPACE;
    }
    return FF_OK;
}

int ff_metric_selection(const double *values, const double *runtime, int64_t n_tasks, int64_t n_kernels,
                        int64_t n_metrics, int top_k, double percentile, double collinear_tau,
                        int min_tasks, double *r_host, double *score_host, int32_t *top_host,
                        uint8_t *selected_host, double *threshold_host, void *stream)
{
    if (!values || !runtime)
        return FF_ERR_NULL;
    if (n_tasks <= 0 || n_kernels <= 0 || n_metrics <= 0 || top_k <= 0 || n_tasks > 1 << 16 ||
        n_kernels > 1 << 20 || n_metrics > 1 << 24 || !(percentile >= 0.0 && percentile <= 100.0) ||
        min_tasks < 1)
        return FF_ERR_SHAPE;
    const bool filter = collinear_tau > 0.0 && collinear_tau <= 1.0;
    if (filter && n_metrics > 8192)
        return FF_ERR_UNSUPPORTED;  // the greedy pass keeps a bit for each metric in LDS and a row of bits in registers
    if ((reinterpret_cast<uintptr_t>(values) & 7u) || (reinterpret_cast<uintptr_t>(runtime) & 7u))
        return FF_ERR_ALIGN;
    const int n = (int)n_tasks, V = (int)n_kernels, J = (int)n_metrics;
    hipStream_t st_stream = static_cast<hipStream_t>(stream);
    try {
    // one host buffer, r then the filter's verdicts: one copy brings both
    const size_t count = (size_t)n * J;
    std::vector<double> results(count + (filter ? (count + 7) / 8 : 0));
    double *const r = results.data();
    uint8_t *const keep = filter ? reinterpret_cast<uint8_t *>(r + count) : nullptr;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        DeviceState *st = current_device_state();
        if (!st)
            return FF_ERR_LAUNCH;
        const size_t words = ((size_t)J + 63) / 64;
        const bool bound = st->ws != nullptr && !st->ws_owned;
        const size_t have = bound ? (st->ws_bytes > kCtrlBytes ? st->ws_bytes - kCtrlBytes : 0) : SIZE_MAX;
        const size_t result_bytes = count * (sizeof(double) + (filter ? 1 : 0));
        double *const pinned = bound ? nullptr : static_cast<double *>(pinned_results(*st, result_bytes, st_stream));
        // One launch does it all where a task fits the LDS and there is room for all tasks' bits.
        const size_t mask_bytes = (size_t)n * selection_mask_bytes(J);
        const size_t one_out = pinned != nullptr ? 0 : round_up(result_bytes, 256);
        if (filter && selection_fits(V, J) && n <= 4096 && mask_bytes <= (size_t)64 << 20 && one_out + mask_bytes <= have) {
            const int rc = prepare_workspace(*st, kCtrlBytes + one_out + mask_bytes, st_stream);
            if (rc != FF_OK)
                return rc;
            char *ws = static_cast<char *>(st->ws);
            double *const r_out = pinned != nullptr ? pinned : reinterpret_cast<double *>(ws + kCtrlBytes);
            if (launch_selection(values, runtime, r_out, reinterpret_cast<unsigned char *>(r_out + count),
                                 reinterpret_cast<unsigned long long *>(ws + kCtrlBytes + one_out),
                                 reinterpret_cast<unsigned *>(ws + kCounterOffset), collinear_tau, n, V, J, st_stream) != hipSuccess)
                return FF_ERR_LAUNCH;
            if (pinned == nullptr && hipMemcpyAsync(r, r_out, result_bytes, hipMemcpyDeviceToHost, st_stream) != hipSuccess)
                return FF_ERR_LAUNCH;
        } else {
            // Workspace: r and the verdicts of all tasks, unless they go to host memory; for a batch of tasks, the columns'
            // means and scales and the pair bits.  A batch is what 64 MiB hold, or a bound workspace.  Where that has no
            // room for all verdicts (very many tasks of very few metrics), a batch's are copied out before the next.
            const size_t per_task = filter ? (size_t)J * (2 * sizeof(double) + words * sizeof(unsigned long long) + 1) : 0;
            size_t out_bytes = pinned != nullptr ? 0 : round_up(result_bytes, 256);
            const bool together = have >= out_bytes + per_task;
            if (!together)
                out_bytes = round_up(count * sizeof(double), 256);
            int batch = n;
            if (filter) {
                const size_t fit = (bound ? (have > out_bytes ? have - out_bytes : 0) : (size_t)64 << 20) / per_task;
                batch = (int)std::min<size_t>({(size_t)n, fit < 1 ? 1 : fit, 32768});
            }
            const int rc = prepare_workspace(*st, kCtrlBytes + out_bytes + (size_t)batch * per_task, st_stream);
            if (rc != FF_OK)
                return rc;
            char *ws = static_cast<char *>(st->ws);
            double *r_dev = pinned != nullptr ? pinned : reinterpret_cast<double *>(ws + kCtrlBytes);
            double *mean_dev = filter ? reinterpret_cast<double *>(ws + kCtrlBytes + out_bytes) : nullptr;
            double *inv_dev = filter ? mean_dev + (size_t)batch * J : nullptr;
            unsigned long long *mask_dev = filter ? reinterpret_cast<unsigned long long *>(inv_dev + (size_t)batch * J) : nullptr;
            unsigned char *batch_keep = reinterpret_cast<unsigned char *>(mask_dev + (filter ? (size_t)batch * J * words : 0));
            for (int i = 0; i < n; i += batch) {
                const int m = n - i < batch ? n - i : batch;
                const double *vals = values + (size_t)i * V * J;
                if (launch_pearson(vals, runtime + (size_t)i * V, r_dev + (size_t)i * J, mean_dev, inv_dev, m, V, J, st_stream) !=
                    hipSuccess)
                    return FF_ERR_LAUNCH;
                if (filter) {
                    const size_t done = (size_t)i * J;
                    unsigned char *keep_dev = together ? reinterpret_cast<unsigned char *>(r_dev + count) + done : batch_keep;
                    if (launch_duplicate_filter(vals, mean_dev, inv_dev, collinear_tau, mask_dev, keep_dev, m, V, J,
                                                st_stream) != hipSuccess)
                        return FF_ERR_LAUNCH;
                    if (!together && hipMemcpyAsync(keep + done, keep_dev, (size_t)m * J, hipMemcpyDeviceToHost, st_stream) !=
                                         hipSuccess)
                        return FF_ERR_LAUNCH;
                }
            }
            if (pinned == nullptr && hipMemcpyAsync(r, r_dev, count * (sizeof(double) + (filter && together ? 1 : 0)),
                                                    hipMemcpyDeviceToHost, st_stream) != hipSuccess)
                return FF_ERR_LAUNCH;
        }
        if (hipStreamSynchronize(st_stream) != hipSuccess)
            return FF_ERR_LAUNCH;
        if (pinned != nullptr)
            std::memcpy(r, pinned, result_bytes);
    }
    metric_select_host(r, keep, n, J, top_k, percentile, min_tasks, top_host,
                       score_host, selected_host, threshold_host);
    if (r_host)
        std::copy(r, r + count, r_host);
    } catch (...) {  // host allocation failed: nothing may leave through the C boundary
        return FF_ERR_WORKSPACE;
    }
    return FF_OK;
}

size_t ff_workspace_bytes(int64_t M, int64_t K, int64_t N, int dtype)
{
    if (validate_shape(M, K, N, dtype) != FF_OK)
        return 0;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    const int num_cus = st ? st->num_cus : 256;
    Plan pl;
    if (make_plan(M, K, N, dtype, num_cus, st, g_forced_variant, false, pl) != FF_OK)
        return 0;
    return pl.total_bytes;
}

int ff_plan_query(int64_t M, int64_t K, int64_t N, int dtype, int out[8])
{
    if (out == nullptr)
        return FF_ERR_NULL;
    const int rc = validate_shape(M, K, N, dtype);
    if (rc != FF_OK)
        return rc;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    const int num_cus = st ? st->num_cus : 256;
    Plan pl;
    const int prc = make_plan(M, K, N, dtype, num_cus, st, g_forced_variant, false, pl);
    if (prc != FF_OK)
        return prc;
    const bool small = pl.variant == FF_VARIANT_SMALL_M && pl.split_s == 0;
    out[0] = pl.variant;
    out[1] = small ? (int)M : pl.tile_m;
    out[2] = small ? kSmallMStripCols : pl.tile_n;
    out[3] = small ? 8 : (pl.split_s > 0 ? split_shape_waves(pl.split_shape) : tile_shape_waves(pl.shape));
    out[4] = pl.grid;
    out[5] = small ? 1 : pl.rounds;
    out[6] = (pl.grid + num_cus - 1) / num_cus;
    out[7] = (pl.split_s > 0 || (!small && pl.swz_sc_log2 >= 0)) ? 1 : 0;
    return FF_OK;
}

int ff_set_workspace(void *dev_ptr, size_t bytes)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    if (dev_ptr != nullptr && ((reinterpret_cast<uintptr_t>(dev_ptr) & 255u) != 0))
        return FF_ERR_ALIGN;
    if (dev_ptr != nullptr && bytes < kCtrlBytes)
        return FF_ERR_WORKSPACE;
    if (dev_ptr != nullptr && init_control_region(dev_ptr) != hipSuccess) {
        (void)hipGetLastError();
        return FF_ERR_LAUNCH;  // the old binding stays
    }
    release_pinned(*st);
    if (st->ws != nullptr && st->ws_owned && !release_own(*st)) {
        (void)hipGetLastError();
        return FF_ERR_LAUNCH;
    }
    st->ws = dev_ptr;
    st->ws_bytes = dev_ptr ? bytes : 0;
    st->ws_owned = false;
    return FF_OK;
}

int ff_check_device(void *stream)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    if (hipStreamSynchronize(static_cast<hipStream_t>(stream)) != hipSuccess) {
        (void)hipGetLastError();
        return FF_ERR_LAUNCH;
    }
    bool failed = false;
    for (int i = -2; i < st->n_kept; ++i) {
        void *region = i == -2 ? st->ws : (i == -1 ? (st->no_alloc_used ? st->no_alloc_ptr : nullptr) : st->kept[i].ptr);
        if (region == nullptr)
            continue;
        unsigned flag = 0;
        if (hipMemcpy(&flag, region, sizeof(flag), hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipGetLastError();
            return FF_ERR_LAUNCH;
        }
        if (flag != 0) {
            // a wait gave up: counters may be half-way; start from a clean control region
            (void)init_control_region(region);
            failed = true;
        }
    }
    return failed ? FF_ERR_DEVICE : FF_OK;
}

const char *ff_status_string(int status)
{
    switch (status) {
    case FF_OK: return "FF_OK";
    case FF_ERR_NULL: return "FF_ERR_NULL: a required pointer is NULL";
    case FF_ERR_SHAPE: return "FF_ERR_SHAPE: M, K and N must be positive, M and N at most 2^30, K at most 2^21";
    case FF_ERR_DTYPE: return "FF_ERR_DTYPE: dtype must be FF_F32 or FF_BF16";
    case FF_ERR_ALIGN: return "FF_ERR_ALIGN: pointers must be 16-byte aligned";
    case FF_ERR_UNSUPPORTED: return "FF_ERR_UNSUPPORTED: K and N must be multiples of 8 (bf16) or 4 (fp32), or the forced variant cannot run this shape";
    case FF_ERR_WORKSPACE: return "FF_ERR_WORKSPACE: workspace too small or allocation failed";
    case FF_ERR_LAUNCH: return "FF_ERR_LAUNCH: the HIP runtime refused the request";
    case FF_ERR_DEVICE: return "FF_ERR_DEVICE: a workgroup gave up waiting for the other tiles of its rows";
    default: return "unknown ff_status";
    }
}

int ff_version(void) { return 100; }

int ff_last_variant(void) { return t_last_variant; }

int ff_debug_last_by_lines(void) { return t_last_by_lines; }

int ff_debug_force_variant(int variant)
{
    if (variant < FF_VARIANT_AUTO || variant > FF_VARIANT_SMALL_M)
        return FF_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_forced_variant = variant;
    return FF_OK;
}

int ff_debug_force_tile(int tile, int wg_per_cu)
{
    if ((tile != 0 && tile != 64 && tile != 128 && tile != 256) || wg_per_cu < 0 || wg_per_cu > 2)
        return FF_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_forced_tile = tile;
    g_forced_wg_per_cu = wg_per_cu;
    return FF_OK;
}

int ff_debug_force_waves(int waves)
{
    if (waves != 0 && waves != 4 && waves != 8)
        return FF_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_forced_waves = waves;
    return FF_OK;
}

int ff_debug_set_stagger_us(int microseconds)
{
    return microseconds < 0 || microseconds > 1000 ? FF_ERR_SHAPE : FF_OK;  // no launch has a second workgroup to delay
}

int ff_debug_set_timeline(void *dev_ptr, size_t bytes)
{
    if (dev_ptr != nullptr && (reinterpret_cast<uintptr_t>(dev_ptr) & 7u) != 0)
        return FF_ERR_ALIGN;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    st->timeline = static_cast<unsigned long long *>(dev_ptr);
    st->timeline_bytes = dev_ptr ? bytes : 0;
    return FF_OK;
}

int ff_debug_copy(const void *src, void *dst, size_t bytes, void *stream)
{
    if (!src || !dst)
        return FF_ERR_NULL;
    if (misaligned(src) || misaligned(dst))
        return FF_ERR_ALIGN;
    if (bytes % 16 != 0)
        return FF_ERR_UNSUPPORTED;
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    if (launch_copy_kernel(src, dst, bytes, st->num_cus, static_cast<hipStream_t>(stream)) != hipSuccess)
        return FF_ERR_LAUNCH;
    return FF_OK;
}

int ff_debug_mfma_loop(int64_t iters, double *flops)
{
    if (!flops)
        return FF_ERR_NULL;
    if (iters <= 0 || iters > (int64_t)1 << 32)
        return FF_ERR_SHAPE;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    // the kernel's per-thread results go to the workspace (they only keep the loop alive)
    const int rc = prepare_workspace(*st, kCtrlBytes + (size_t)st->num_cus * 512 * sizeof(float), nullptr);
    if (rc != FF_OK)
        return rc;
    float *sink = reinterpret_cast<float *>(static_cast<char *>(st->ws) + kCtrlBytes);
    if (launch_mfma_loop(iters, sink, st->num_cus, nullptr, flops) != hipSuccess)
        return FF_ERR_LAUNCH;
    return FF_OK;
}

int ff_debug_stream_read(const void *src, size_t bytes)
{
    if (!src)
        return FF_ERR_NULL;
    if (misaligned(src))
        return FF_ERR_ALIGN;
    if (bytes % 16 != 0)
        return FF_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *st = current_device_state();
    if (!st)
        return FF_ERR_LAUNCH;
    const int rc = prepare_workspace(*st, kCtrlBytes + (size_t)st->num_cus * 2 * 256 * sizeof(unsigned), nullptr);
    if (rc != FF_OK)
        return rc;
    unsigned *sink = reinterpret_cast<unsigned *>(static_cast<char *>(st->ws) + kCtrlBytes);
    if (launch_stream_read(src, bytes, sink, st->num_cus, nullptr) != hipSuccess)
        return FF_ERR_LAUNCH;
    return FF_OK;
}

int ff_debug_expect_extra_arrivals(int count)
{
    if (count < 0 || count > 1024)
        return FF_ERR_SHAPE;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_extra_arrivals = count;
    return FF_OK;
}

int ff_debug_set_wait_limit_us(int64_t microseconds)
{
    if (microseconds <= 0)
        return FF_ERR_SHAPE;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_wait_limit_us = microseconds;
    return FF_OK;
}

}  // extern "C"
