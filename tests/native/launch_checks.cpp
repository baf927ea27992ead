// Driver for the contract between the library's host code and its kernels
// (test infrastructure): the host source, built with g++ against the host-only
// HIP stand-in (tests/native/fake_hip), with launch wrappers that do only what
// the kernels do.  A launch without a queue and a tile count takes its table
// by value: at most kSmallTable curves, one workgroup per tile, no tile list,
// and a grid that HIP's 32-bit thread count holds.  Any other estimate launch
// reads the table and the tile list that a set-up launch wrote.  Every tile is
// served by an instance that carries its path: sorted cores with room for the
// curve's core, split tiles without them, small windows, the extra options.
// Prints "launch checks ok" and exits 0 on success.
#include "umi_host.hip"

#include <random>

namespace {

int g_failures = 0;
long g_setup = 0, g_value = 0, g_staged = 0, g_per_curve = 0;
int g_tiles = 0;        // tiles of the last estimate launch
bool g_outputs = true;  // the stand-in writes the outputs (off for very long curves)

#define CHECK(cond)                                                               \
    do {                                                                          \
        if (!(cond)) {                                                            \
            std::fprintf(stderr, "CHECK failed at line %d: %s\n", __LINE__, #cond); \
            ++g_failures;                                                         \
        }                                                                         \
    } while (0)

}  // namespace

namespace umi {

hipError_t launch_prepass(const float*, const double*, uint8_t* block, const uint8_t* stage, int,
                          int grid, int32_t*, int2* tiles, Counters* ctr, ChunkRec*,
                          bool clear_queue, bool, const CurveDesc*, hipStream_t)
{
    if (!clear_queue) return hipSuccess;
    return fake_hip::record_or_run([=] {
        ++g_setup;
        CHECK(grid >= 1 && grid <= kSetupGroups);
        const int nc = reinterpret_cast<const BatchHeader*>(stage ? stage : block)->n_curves;
        if (stage) std::memcpy(block, stage, block_bytes(nc));
        const CurveDesc* c = reinterpret_cast<const CurveDesc*>(block + sizeof(BatchHeader));
        ctr->queue = 0u;
        for (int i = 0; i < nc; ++i)
            for (int t = 0; (int64_t)t * c[i].tile < c[i].len; ++t)
                tiles[c[i].tile_base + t] = make_int2(i, t * c[i].tile);
        return hipSuccess;
    });
}

hipError_t launch_copy(const CopyBatch&, hipStream_t) { return hipSuccess; }

void check_tile(const BatchHeader& hdr, const CurveDesc& cd, int t0, int feat, float* trend)
{
    const int cap = feat >> kFeatBits;
    feat &= (1 << kFeatBits) - 1;
    const bool no_split = (feat & kFeatNoSplit) != 0;
    const int h = (cd.W - 1) / 2, t1 = (int)std::min<int64_t>((int64_t)t0 + cd.tile, cd.len);
    CHECK(t0 >= 0 && t0 < cd.len && cd.tile >= 1 && cd.tile <= kMaxTile);
    CHECK(std::min<int64_t>((int64_t)t1 + h, cd.len) - std::max(t0 - h, 0) <= kStageMax);
    CHECK(cd.core == (core_window(cd.W, cd.alpha, hdr.scale) && cd.tile >= kCoreMinTile ? 1 : 0));
    if (cd.core) {
        CHECK((feat & kFeatCore) && cap >= core_cap(cd.W));
    } else if (cd.tile <= kSplitMaxTile) {
        CHECK((feat & kFeatSplit) && !no_split);
        CHECK(split_lanes(cd.tile) * cd.tile <= kMainThreads);
    }
    if (cd.W <= kSmallW) CHECK(feat & kFeatSmall);
    if (cd.window_days > 0.0 || hdr.scale != UMI_SCALE_UPPER_RMS) CHECK(feat & kFeatExtra);
    if (g_outputs)
        for (int p = t0; p < t1; ++p) trend[cd.off + p] = (float)cd.W;
}

hipError_t launch_main(const float*, const int32_t*, const BatchHeader* hdr,
                       const CurveDesc* curves, const int2* tiles, int tile_first, int tile_count,
                       uint32_t* counter, int grid, float* trend, float*, int feat, hipStream_t)
{
    if (counter == nullptr && tile_count < 0) {
        // by value: the arguments are read when the launch is made
        ++g_value;
        CHECK(hdr->n_curves >= 1 && hdr->n_curves <= kSmallTable);
        CHECK((int64_t)hdr->n_tiles * kMainThreads <= (int64_t)UINT32_MAX);
        for (int tile = 0; tile < hdr->n_tiles; ++tile) {
            int ci = 0;
            for (int i = 0; i < hdr->n_curves; ++i)
                if (curves[i].tile_base <= tile) ci = i;
            check_tile(*hdr, curves[ci], (tile - curves[ci].tile_base) * curves[ci].tile, feat,
                       trend);
        }
        return hipSuccess;
    }
    return fake_hip::record_or_run([=] {
        ++(tile_count < 0 ? g_staged : g_per_curve);
        g_tiles = hdr->n_tiles;
        CHECK(grid >= 1 && (int64_t)grid * kMainThreads <= (int64_t)UINT32_MAX);
        if (tile_count < 0)
            CHECK(*counter == 0u);
        else
            CHECK(grid == tile_count);
        const int end = tile_count < 0 ? hdr->n_tiles : tile_first + tile_count;
        CHECK(end <= hdr->n_tiles);
        for (int t = tile_first; t < end; ++t)
            check_tile(*hdr, curves[tiles[t].x], tiles[t].y, feat, trend);
        return hipSuccess;
    });
}

}  // namespace umi

namespace {

std::mt19937_64 rng(49ull);
int64_t uni(int64_t lo, int64_t hi) { return std::uniform_int_distribution<int64_t>(lo, hi)(rng); }

// Batches of every path, direct and through a plan: every position written once.
void check_batches()
{
    for (int round = 0; round < 200; ++round) {
        const int64_t n = uni(1, 45);
        std::vector<int64_t> len((size_t)n), off((size_t)n);
        std::vector<int32_t> W((size_t)n);
        std::vector<float> al((size_t)n);
        std::vector<double> wd((size_t)n);
        int64_t span = 0;
        for (int64_t b = 0; b < n; ++b) {
            len[b] = uni(0, 5) == 0 ? 0 : uni(1, 30000);
            W[b] = (int32_t)(2 * uni(0, uni(0, 2) ? 180 : 1023) + 1);
            al[b] = uni(0, 4) ? 2.0f : 20.0f;
            wd[b] = uni(0, 3) ? 0.0 : 0.3;
            off[b] = span;
            span += len[b];
        }
        std::vector<float> flux((size_t)span + 1, 1.0f), trend((size_t)span + 1, 0.0f);
        std::vector<double> time((size_t)span + 1, 0.0);
        umi_options o = {uni(0, 1) ? al.data() : nullptr, nullptr, (int32_t)(uni(0, 4) == 0), 0,
                         nullptr, uni(0, 2) ? nullptr : wd.data()};
        umi_launch lo = {uni(0, 5) ? UMI_MODE_PERSISTENT : UMI_MODE_PER_CURVE,
                         uni(0, 2) ? 0 : (int32_t)uni(1, 1600), uni(0, 3) ? 0 : (int32_t)uni(1, 4),
                         0, nullptr, nullptr};
        CHECK(umi_detrend_gather_ex(flux.data(), time.data(), off.data(), len.data(), n, W.data(),
                                    2.0f, 5.0f, 5, trend.data(), nullptr, &o, &lo,
                                    nullptr) == UMI_OK);
        for (int64_t b = 0; b < n; ++b)
            for (int64_t i = 0; i < len[b]; ++i) CHECK(trend[(size_t)(off[b] + i)] == (float)W[b]);
        if (span == 0) continue;
        umi_plan* p = nullptr;
        CHECK(umi_plan_create(&p, span, n, 2047, flux.data(), time.data(), trend.data(), nullptr,
                              reinterpret_cast<void*>(uintptr_t(0x1000))) == UMI_OK);
        for (int run = 0; run < 2; ++run) {
            std::fill(trend.begin(), trend.end(), 0.0f);
            CHECK(umi_plan_run_ex(p, off.data(), len.data(), W.data(), n, 2.0f, 5.0f, 5, &o) ==
                  UMI_OK);
            for (int64_t b = 0; b < n; ++b)
                for (int64_t i = 0; i < len[b]; ++i)
                    CHECK(trend[(size_t)(off[b] + i)] == (float)W[b]);
        }
        CHECK(umi_plan_destroy(p) == UMI_OK);
    }
    CHECK(g_setup > 0 && g_value > 0 && g_staged > 0 && g_per_curve > 0);
}

// A lone curve of more tiles than one launch may have workgroups runs through
// the tile queue, directly, with tiles given and as a plan's step; of one tile
// fewer, by value.
void check_many_tiles()
{
    g_outputs = false;
    const int64_t most = (int64_t)UINT32_MAX / umi::kMainThreads;  // workgroups of a launch
    for (int64_t tiles : {most, most + 1}) {
        const int64_t n = 2 * tiles;  // W = 2047: tiles of two positions
        const int32_t W = 2047;
        std::vector<float> flux((size_t)n, 1.0f), trend((size_t)n);
        const long value = g_value, staged = g_staged;
        CHECK(umi_detrend(flux.data(), nullptr, n, W, 2.0f, 5.0f, 5, trend.data(), nullptr,
                          nullptr) == UMI_OK);
        const bool fits = tiles <= most;
        CHECK(g_value == value + (fits ? 1 : 0) && g_staged == staged + (fits ? 0 : 1));
        const int64_t off = 0;
        umi_plan* p = nullptr;
        CHECK(umi_plan_create(&p, n, 1, W, flux.data(), nullptr, trend.data(), nullptr,
                              reinterpret_cast<void*>(uintptr_t(0x1000))) == UMI_OK);
        CHECK(umi_plan_run(p, &off, &n, &W, 1, 2.0f, 5.0f, 5) == UMI_OK);
        CHECK(g_value == value + (fits ? 2 : 0) && g_staged == staged + (fits ? 0 : 2));
        CHECK(umi_plan_destroy(p) == UMI_OK);
        const int32_t narrow = 25;
        const umi_launch lo = {UMI_MODE_PERSISTENT, 1, 0, 0, nullptr, nullptr};
        const int64_t len = tiles;
        CHECK(umi_detrend_batch(flux.data(), nullptr, &len, 1, &narrow, 2.0f, 5.0f, 5,
                                trend.data(), nullptr, &lo, nullptr) == UMI_OK);
        CHECK(g_value == value + (fits ? 3 : 0) && g_staged == staged + (fits ? 0 : 3));
    }
}

// A small batch is cut into no more tiles than the workgroups that the call
// lets run at once, where larger tiles leave it as few.
void check_limited_groups()
{
    g_outputs = false;
    const int64_t n = 40, len = 7662;
    std::vector<int64_t> lens((size_t)n, len);
    std::vector<float> flux((size_t)(n * len), 1.0f), trend((size_t)(n * len));
    for (int W : {61, 115, 241, 361}) {
        const std::vector<int32_t> Ws((size_t)n, W);
        for (float alpha : {2.0f, 0.1f})
            for (int groups = 1; groups <= 4; ++groups) {
                const umi_launch lo = {UMI_MODE_PERSISTENT, 0, groups, 0, nullptr, nullptr};
                CHECK(umi_detrend_batch(flux.data(), nullptr, lens.data(), n, Ws.data(), alpha, 5.0f,
                                        5, trend.data(), nullptr, &lo, nullptr) == UMI_OK);
                CHECK(g_tiles <= 256 * groups);
            }
    }
}

}  // namespace

int main()
{
    check_batches();
    check_limited_groups();
    check_many_tiles();
    umi_release();
    if (g_failures == 0) std::printf("launch checks ok\n");
    return g_failures == 0 ? 0 : 1;
}
