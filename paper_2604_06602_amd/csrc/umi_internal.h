// Internal layout shared by the host launcher and the HIP kernels of the UMI
// library.  Nothing here is part of the public C ABI (include/umi.h).
#pragma once

#include <stdint.h>

namespace umi {

// Largest staged tile: output positions plus the W-1 halo.  The tile sort and
// the wavelet matrix work on power-of-two padded sizes up to this.
constexpr int kStageMax = 2048;
constexpr int kStageLog2 = 11;
constexpr int kWords = kStageMax / 64 + 1;  // bit-vector words incl. sentinel
constexpr int kMainThreads = 512;            // threads per main-kernel workgroup
constexpr int kMaxTile = 3 * kMainThreads;   // output positions per tile: <= 3 per lane
constexpr int kSplitMaxTile = kMainThreads / 2;  // tiles this small split windows
constexpr int kSmallW = 31;                  // full windows this small take register networks
// Paths of the estimate kernel a batch needs (bits of a kernel instance).
constexpr int kFeatSmall = 1;                // small-window networks (W <= kSmallW)
constexpr int kFeatSplit = 2;                // split tiles (tile <= kSplitMaxTile)
constexpr int kFeatExtra = 4;                // MAD ablation, time windows
constexpr int kFeatCore = 8;                 // sorted cores (wide windows)
constexpr int kFeatAll = kFeatSmall | kFeatSplit | kFeatExtra | kFeatCore;
constexpr int kFeatNoSplit = 16;             // with kFeatSplit: the small tiles all take cores,
                                             // so no instance with split windows is needed
constexpr int kFeatBits = 8;                 // the batch's largest core stands above these

// Sorted cores: 32 consecutive windows share all but at most 31 samples of
// each; the core is that shared run, a whole number of blocks of kCoreBlock.
// Narrower windows sum their samples directly: what a wave does for a group,
// and the 33 edge and 16 block samples of a window's iteration, cost the same
// whatever W.  One line for two: batches gain from about W = 97 (500 curves of
// 18,000: W = 97 737 us directly, 740 by cores; W = 113 818 and 731), one curve of
// 20,000, in small tiles whose windows several lanes share, from about 190 (W = 113
// 17 and 19 us; W = 161 18 and 19; W = 201 19.5 and 19; W = 361 24.5 and 19.5), so
// that lone curves lose some 1 us between.
constexpr int kCoreMinW = 117;
constexpr int kCoreBlock = 8;
// Tiles smaller than this (an explicit tile, or W > 1985) leave most of a
// workgroup's waves without a group of windows; the lanes that share a window
// directly use them all (us a call, by cores and directly: 838 curves of 1,740
// with ties at W = 2017, tiles of 32, one iteration 6,990 and 2,715; 40 of 18,000
// at W = 1987, tiles of 62, 1,129 and 1,096; 7 of 2,671 at W = 361 with tiles of one
// position 653 and 293; with tiles of 64, 40 of 18,000 at W = 117 take 229 and
// 232, at W = 361 247 and 500).
constexpr int kCoreMinTile = 64;
// Waves per SIMD the core instances are built for: three workgroups per CU, with
// 80 registers that spill little; at 4 waves (128 registers) two fit and W = 361
// took 3.3 ms against 2.5, with groups of 64 windows.  Up to about W = 480 LDS
// would allow four (39 KB: the wavelet build's 29 and 10), up to about 725 three,
// up to about 1250 two.
// (Edge samples in registers spill some of the tile's own values, outside the
// groups' loop.)
constexpr int kCoreWaves = 6;
constexpr int kCoreGroup = 32;               // windows that share a core
constexpr int kCoreEdge = 32 + kCoreBlock + 32;  // samples a wave sums one by one
__host__ __device__ constexpr int core_cap(int W)
{
    return W >= kCoreGroup ? W - (kCoreGroup - 1) : 0;
}
// the search tree over nb blocks' first values: levels of every 4^k-th value,
// each a whole number of fours.  The first level, of every 2^core_top-th value,
// stands in registers; the last, of every value, is the blocks' own.
__host__ __device__ constexpr int core_top(int nb)  // log2 of that stride
{
    return nb > 1 ? (31 - __builtin_clz((unsigned)(nb - 1))) & ~1 : 0;
}
__host__ __device__ constexpr int core_level_len(int nb, int sh)  // of every 2^sh-th value
{
    return (((nb + (1 << sh) - 1) >> sh) + 3) & ~3;
}
__host__ __device__ constexpr int core_tree(int nb)
{
    int len = 0;
    for (int sh = core_top(nb) - 2; sh > 0; sh -= 2) len += core_level_len(nb, sh);
    return len;
}
// floats of LDS one wave's core takes: values, edge samples, and the larger
// of the rank marks and the block table (search tree, five power sums per
// block edge)
constexpr int kCoreMin = 32;                 // samples of the smallest core (Phase 1's ranks lie inside)
constexpr int kCoreMarks = kStageMax / 16;   // words of the rank marks (and of Phase 1's masks)
static_assert(kCoreMarks >= 2 * 64, "masks fit");
constexpr int kRankBytes = 2 * kStageMax;    // the tile's ranks, ahead of the waves' cores
__host__ __device__ constexpr int core_floats_for(int cap)
{
    const int nb = cap / kCoreBlock;
    const int table = core_tree(nb) + 5 * (nb + 1);
    const int masks = kCoreMarks;
    return ((cap + 3) & ~3) + kCoreEdge + (((table > masks ? table : masks) + 3) & ~3);
}

// Lanes that share one window for a tile of `tile` output positions: 1 above
// kSplitMaxTile (each lane takes up to three windows), else the largest of 2,
// 4, 8 with tile * G <= kMainThreads.
__host__ __device__ constexpr int split_lanes(int tile)
{
    return tile > kSplitMaxTile ? 1 : (tile > kMainThreads / 4 ? 2 : (tile > kMainThreads / 8 ? 4 : 8));
}
constexpr int kSetupThreads = 256;           // threads per set-up workgroup
constexpr int kSetupGroups = 1024;           // set-up workgroups at most
constexpr int kPrepChunk = 1 << 20;          // samples a chunk of the table's chunk counts stands for
constexpr float kScaleConst = 0.6745f;       // Section 2.2, after Eq. 1
constexpr double kGapDays = 0.5;             // segment break threshold (days)

// Per-batch parameters, read by the kernels from device memory so that a
// captured launch sequence can be replayed for any batch (only the staged
// bytes change between replays).
struct BatchHeader {
    int32_t n_curves;   // entries in the curve table
    int32_t n_tiles;    // tiles over all curves
    int32_t iters;      // Phase 3 iterations
    int32_t scale;      // umi_scale: Phase 2 estimator
    int32_t n_chunks;   // chunks of kPrepChunk samples over all curves
    int32_t reserved;
    float* detrended;   // flux / trend output (curve offsets as for trend), or null
    const double* time; // the batch's times (read by the time-window scans), or null
};
static_assert(sizeof(BatchHeader) == 40, "BatchHeader layout");

// One curve of a packed batch, in the (cost-sorted) order tiles are issued.
struct CurveDesc {
    int64_t off;        // first sample in the packed arrays
    int32_t len;        // samples
    int32_t W;          // window (odd)
    int32_t tile;       // output positions per tile
    int32_t tile_base;  // index of this curve's first tile in the tile list
    float alpha;        // asymmetry factor (Eq. 2) of this curve
    float c;            // bisquare tuning constant of this curve
    double window_days; // > 0: time window of this length (W still bounds it)
    int32_t chunk_base; // index of this curve's first chunk
    int32_t core;       // its tiles sum windows by sorted cores
};
static_assert(sizeof(CurveDesc) == 48, "CurveDesc layout");

// A batch's table by value, as kernel arguments (n_curves 0: the table is in
// device memory).
constexpr int kSmallTable = 32;
struct SmallTable {
    int32_t n_curves;
    int32_t reserved;
    BatchHeader hdr;
    CurveDesc c[kSmallTable];
};
static_assert(sizeof(SmallTable) <= 2048, "SmallTable fits the kernel arguments");

// Workgroups of the estimate kernel that one launch may have: HIP counts a
// launch's threads in 32 bits.
__host__ __device__ constexpr bool grid_fits(int64_t groups)
{
    return groups * kMainThreads <= (int64_t)UINT32_MAX;
}

// One record per chunk of the launch interface (launch_prepass): two words.
constexpr int kSegWords = 1;
struct ChunkRec {
    uint64_t agg[kSegWords];
    uint64_t inc[kSegWords];
};

// Device counters of a workspace (zeroed when it is allocated).
struct Counters {
    uint32_t queue;     // estimate-kernel tile queue (cleared by the set-up)
    uint32_t tickets;
    uint32_t done;
    uint32_t reserved;
    uint64_t epoch;
    uint64_t reserved2;
};
static_assert(sizeof(Counters) == 32, "Counters layout");

// A list of copies for the copy kernel, passed by value as kernel arguments
// (so nothing on either side needs to outlive the launch): copy i moves
// bytes[i] bytes from src[i] to dst[i] and is cut into pieces of kCopyPieceBytes
// bytes, piece p of the launch belonging to the copy i with
// first[i] <= p < first[i + 1].
constexpr int kCopyMax = 64;
constexpr int kCopyPieceBytes = 32768;
struct CopyBatch {
    int32_t n;                   // copies
    int32_t reserved;
    int32_t first[kCopyMax + 1]; // first piece of each copy; first[n] = pieces
    const uint8_t* src[kCopyMax];
    uint8_t* dst[kCopyMax];
    int64_t bytes[kCopyMax];
};
static_assert(sizeof(CopyBatch) <= 2048, "CopyBatch fits the kernel arguments");

// Tile record written by the set-up: x = index into the curve table,
// y = first output position (curve-local).

}  // namespace umi
