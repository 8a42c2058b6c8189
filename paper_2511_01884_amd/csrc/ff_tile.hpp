// Host/device interface of the kernels: parameter blocks and launch functions.
#pragma once
#include <type_traits>

#include "ff_device.hpp"

namespace ff {

enum { kFused = 0, kTwoPass = 1, kLinearOnly = 2 };

struct TileParams {
    const void *X;       // [M,K]
    const void *W;       // [N,K]
    const void *b;       // [N] or null
    const void *gamma;   // [N] or null
    const void *beta;    // [N] or null
    void *Y;             // kFused: [M,N] in the tensor dtype
    float *F;            // kTwoPass: fp32 G scratch [M,N]; kLinearOnly: fp32 Z out
    floatx2 *partials;   // [RB][NT][BM] (mean, M2) per tile row
    unsigned *counters;  // pairs (arrival, departure), a row-block's at row_counter()
    unsigned *err;       // error word
    float eps;
    int M, K, N;
    int NT;              // tiles along N
    int RB;              // row-blocks
    int rounds;          // ceil(RB * NT / grid), or ceil(RB / round_rows)
    int round_rows;      // row-blocks of a round when the grid is made of whole ones, else 0
    int swz_sc_log2;     // XCD-aware order: log2 of the super-block width in tiles, -1 = plain order
    int nt_log2;         // log2(NT) when the XCD-aware order is on
    int grid_log2;       // log2(grid) when the XCD-aware order is on
    int extra_arrivals;  // test hook: added to the arrival target (non-zero makes waits expire)
    long long wait_ticks;
    unsigned long long *timeline;  // test hook: phase timestamps, or null
    int timeline_rounds;           // rounds of tiles the timeline buffer has room for
};

// Timeline record of one tile: slots 0..6 wall-clock stamps (tile start, first slab landed, main
// loop done, statistics published, other tiles arrived, statistics merged, stores issued); slots
// kTimelineCycleSlot, +1 the shader clock at the start and end of the main loop.  Slot 7, split kernel only:
// the tile's partial products are summed.
constexpr int kTimelineSlots = 16;
constexpr int kTimelineCycleSlot = 8;

struct FinalizeParams {
    const float *G;
    const floatx2 *partials;
    const void *gamma;
    const void *beta;
    void *Y;
    float eps;
    int M, N, NT, BM, BN;
};

// Split kernel: counters in 128-byte lines of their own, one per tile (the S workgroups that share its
// K range), then kSplitWays per row slice (the workgroups that share its rows); word 0 of a line counts
// arrivals, word 1 (of a slice's first line) departures.
constexpr int kSplitCounterStride = 32;  // uint32 words
constexpr int kSplitWays = 8;
constexpr int kSplitMaxS = 16;

struct SplitParams {
    const void *X, *W, *b, *gamma, *beta;
    void *Y;
    float *sums;         // [tile][S][BM][BN] partial products (S > 1)
    floatx2 *partials;   // [RB][S][NT][max(BM / S, 16)] (mean, M2) per row of a slice and column tile
    unsigned *counters;
    unsigned *err;
    float eps;
    int M, K, N;
    int NT, RB;          // tiles along N, row blocks
    int S;               // workgroups that share a tile's K range
    int extra_arrivals;  // test hook: added to the arrival target (non-zero makes waits expire)
    long long wait_ticks;
    unsigned long long *timeline;  // test hook: phase timestamps, or null
};

// Shapes of the split kernel (columns x rows of a tile; W4: four wavefronts, bf16 only)
enum SplitShape { kSplit64x32 = 0, kSplit128x32 = 1, kSplit64 = 2, kSplit128x64 = 3, kSplit128 = 4, kSplit128W4 = 5, kSplit32 = 6, kNumSplitShapes = 7 };
constexpr int split_shape_cols(int shape) { return shape == kSplit32 ? 32 : shape == kSplit64x32 || shape == kSplit64 ? 64 : 128; }
constexpr int split_shape_rows(int shape) { return shape == kSplit32 ? 32 : shape >= kSplit128 ? 128 : (shape >= kSplit64 ? 64 : 32); }
constexpr int split_shape_waves(int shape) { return shape == kSplit128x64 || shape == kSplit128 ? 8 : 4; }
hipError_t launch_split_kernel(bool bf16, int shape, const SplitParams &p, int grid, hipStream_t stream);
int split_kernel_blocks_per_cu(bool bf16, int shape);
bool split_kernel_by_lines(bool bf16, int shape, const SplitParams &p);

struct SmallMParams {
    const void *X, *W, *b, *gamma, *beta;
    void *Y;
    floatx2 *partials;   // [strips][16 * MT] (mean, M2)
    unsigned *counters;  // [2]
    unsigned *err;
    float eps;
    int M, K, N;
    int strips;          // N / 32 rounded up
    int extra_arrivals;  // test hook: added to the arrival target (non-zero makes waits expire)
    long long wait_ticks;
    unsigned long long *timeline;  // test hook: phase timestamps, or null
};

// second chain: 512 threads; phase 1 covers 64 rows x 128 bytes of W per load instruction
constexpr int kRowMeanThreads = 512;
constexpr int kRowMeanRowsPerStep = 64;
constexpr int kRowMeanMaxK = 32768;  // the column means lie in LDS, four bytes each

struct RowMeanParams {
    const void *X, *W, *b, *s;
    void *Out;
    float *partial;      // [chunks][k_pad] partial column sums of W
    float *cpart;        // [grid] slices of sum(b - s)
    unsigned *counters;  // control-region counter array (zero before and after a launch)
    unsigned *err;
    int M, K, N;
    int strips;          // 128-byte column strips; k_pad = strips * (128 / sizeof T)
    int k_pad;
    int chunks, rows_per_chunk;  // row chunks of W; rows_per_chunk is a multiple of kRowMeanRowsPerStep
    int grid;            // one workgroup per compute unit: all co-resident
    int extra_arrivals;  // test hook
    long long wait_ticks;
};

constexpr int kXentMaxSegs = 16;  // segments of a long row

struct XentParams {
    const void *logits;        // [B][C]
    const long long *targets;  // [B]
    float *row_loss;           // [B] or null
    float *mean_loss;          // [1]
    floatx2 *partials;         // [grid]: one number per workgroup; with segments [B][segs]: (maximum, sum)
    floatx2 *picked;           // [B] with segments: the target's logit
    unsigned *counter, *ways;  // arrivals of this launch, final and in kSyncWays words; zero before and after
    int B, C;
    int grid;
    int vec;                   // elements per load: 16 bytes' worth, or 1 for rows of fewer than four such loads
    int lanes, per_lane;       // short rows: lanes per row and loads per lane; lanes = 0: a wavefront per row or segment
    int segs, seg_chunks;      // long rows: segments per row, 16-byte loads of a segment
};

hipError_t launch_copy_kernel(const void *src, void *dst, size_t bytes, int num_cus, hipStream_t stream);
hipError_t launch_mfma_loop(long long iters, float *sink, int num_cus, hipStream_t stream, double *flops);
hipError_t launch_stream_read(const void *src, size_t bytes, unsigned *sink, int num_cus, hipStream_t stream);

// profiling-metric selection: device correlations, host selection
hipError_t launch_pearson(const double *values, const double *runtime, double *r, double *mean, double *inv, int n,
                          int V, int J, hipStream_t stream);
hipError_t launch_duplicate_filter(const double *values, const double *mean, const double *inv, double tau,
                                   unsigned long long *mask, unsigned char *keep, int n, int V, int J, hipStream_t stream);
bool selection_fits(int V, int J);
size_t selection_mask_bytes(int J);
hipError_t launch_selection(const double *values, const double *runtime, double *r, unsigned char *keep, unsigned long long *mask,
                            unsigned *arrived, double tau, int n, int V, int J, hipStream_t stream);
void metric_select_host(const double *r, const unsigned char *keep, int n, int J, int k, double q,
                        int min_tasks, int *top, double *score, unsigned char *selected, double *threshold);

hipError_t launch_xent_kernel(bool bf16, const XentParams &p, hipStream_t stream);
hipError_t launch_rowmean_chain(bool bf16, const RowMeanParams &p, hipStream_t stream);
// Tile shapes of the tiled kernels (columns x rows of the output a workgroup owns).
enum TileShape {
    kTile64 = 0,       // 64 x 64, four wavefronts, up to four workgroups per compute unit
    kTile128 = 1,      // 128 x 128, four wavefronts, two workgroups per compute unit
    kTile256 = 2,      // 256 x 256, four wavefronts of 4 x 4 MFMA blocks, one workgroup per compute unit
    kTile256W8 = 3,    // 256 x 256, eight wavefronts of 4 x 2 blocks, one workgroup per compute unit
    kTile256x128 = 4,  // 256 columns x 128 rows, eight wavefronts of 64 x 64 outputs, one workgroup per compute unit
    kNumTileShapes = 5
};
inline int tile_shape_cols(int shape) { return shape == kTile64 ? 64 : (shape == kTile128 ? 128 : 256); }
inline int tile_shape_rows(int shape)
{
    return shape == kTile64 ? 64 : ((shape == kTile128 || shape == kTile256x128) ? 128 : 256);
}
inline int tile_shape_waves(int shape) { return shape == kTile256W8 || shape == kTile256x128 ? 8 : 4; }
hipError_t launch_tile_kernel(bool bf16, int shape, int mode, const TileParams &p, int grid, hipStream_t stream);
int tile_kernel_blocks_per_cu(bool bf16, int shape, int mode);
bool tile_kernel_by_lines(bool bf16, int shape, int mode, const TileParams &p);
hipError_t launch_finalize_kernel(bool bf16, const FinalizeParams &p, hipStream_t stream);
hipError_t launch_smallm_kernel(int mt, const SmallMParams &p, int grid, hipStream_t stream);

constexpr int kSmallMStripCols = 32;
constexpr int kSmallMMaxStripsPerGroup = 8;

}  // namespace ff
