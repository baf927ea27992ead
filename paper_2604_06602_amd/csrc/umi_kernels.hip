// HIP kernels of the UMI library for CDNA4 (gfx950).
//
//   umi_main_kernel     tiles of consecutive output positions.  A workgroup
//                       stages a tile plus its W-1 halo from HBM once, finds
//                       the span's valid samples and segments (gap handling,
//                       minimum segment length W/3 of Section 4.4), keeps the
//                       valid samples compacted in LDS and sorts (value,
//                       index) pairs of them once.  Then, per window:
//                         Phase 1 (Section 2.1): the exact median, from the
//                           sorted tile;
//                         Phase 2 (Section 2.2, Eq. 1): upper-RMS scale;
//                         Phase 3 (Section 2.3, Eqs. 2-4): asymmetric bisquare
//                           iterations in the residual form
//                           mu <- mu + sum(w v) / (k sum(w)), v = k (x - mu),
//                           k = A/(c s), A = (1 + alpha)/2: Eq. 4 rewritten
//                           around the current mu, with Eq. 2's two branches
//                           folded into one expression of v.
//                       Windows of kCoreMinW samples or more share sorted
//                       cores with their neighbours and sum most of their
//                       samples by power sums.  Narrower ones take their
//                       medians from a wavelet matrix over the sorted ranks
//                       (full windows of W <= 31 from register networks) and
//                       sum sample by sample, a lane taking up to three
//                       consecutive windows and one LDS read feeding all of
//                       them; tiles of at most 256 positions split each window
//                       over 2, 4 or 8 lanes.  Launched with the curve table by
//                       value and one workgroup per tile (few curves),
//                       persistently (a grid sized to the chip pops tiles from
//                       a device counter), or per curve.
//
//   umi_setup_kernel    copies the staged curve table of a larger batch to
//                       the device, lists its tiles and clears the counter.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include <stdint.h>

#include "umi.h"
#include "umi_internal.h"

// Every fused multiply-add below is written out with __builtin_fmaf; the
// compiler may not contract anything else, so the same window gives the same
// bits whichever code path (fused multi-window or single-window) computes it.
#pragma clang fp contract(off)

namespace umi {

// ---------------------------------------------------------------------------
// Set-up of a batch whose curve table is in device memory (or in the caller's
// pinned staging block, which the device reads over the bus): copies the
// staged block to `to` for the estimate kernel, writes the tile list and
// clears the tile queue.  Batches of at most kSmallTable curves pass the
// table to the estimate kernel by value and need none of this.
__global__ __launch_bounds__(kSetupThreads) void umi_setup_kernel(
    const uint8_t* __restrict__ block, uint8_t* __restrict__ to, int2* __restrict__ tiles,
    uint32_t* __restrict__ queue)
{
    const BatchHeader* __restrict__ hdr = reinterpret_cast<const BatchHeader*>(block);
    const CurveDesc* __restrict__ curves =
        reinterpret_cast<const CurveDesc*>(block + sizeof(BatchHeader));
    if (blockIdx.x == 0 && threadIdx.x == 0) *queue = 0u;
    const int n_curves = hdr->n_curves;
    if (to != nullptr) {  // in 8-byte words, spread over the grid
        const int words = (int)((sizeof(BatchHeader) + (size_t)n_curves * sizeof(CurveDesc)) / 8);
        const uint64_t* s = reinterpret_cast<const uint64_t*>(block);
        uint64_t* d = reinterpret_cast<uint64_t*>(to);
        for (int i = (int)(blockIdx.x * kSetupThreads + threadIdx.x); i < words;
             i += (int)gridDim.x * kSetupThreads)
            d[i] = s[i];
    }
    for (int c = (int)blockIdx.x; c < n_curves; c += (int)gridDim.x) {
        const int len = curves[c].len, tile = curves[c].tile, base = curves[c].tile_base;
        for (int t = (int)threadIdx.x; (int64_t)t * tile < len; t += kSetupThreads)
            tiles[base + t] = make_int2(c, t * tile);
    }
}
static_assert(sizeof(BatchHeader) % 8 == 0 && sizeof(CurveDesc) % 8 == 0, "8-byte words");

// ---------------------------------------------------------------------------
// Main kernel.

// IEEE-754 totalOrder of float32 as an unsigned key, and back.
__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float key_value(uint32_t k)
{
    const uint32_t b = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(b);
}

// A pair of the tile sort, and of the sorted tile: the sample's totalOrder
// key, in the sorted tile the sample itself, above its compacted index.
__device__ __forceinline__ uint64_t sorted_pair(uint64_t keyed)
{
    return ((uint64_t)__float_as_uint(key_value((uint32_t)(keyed >> 32))) << 32) | (uint32_t)keyed;
}

__device__ __forceinline__ float sorted_value(uint64_t pair)
{
    return __uint_as_float((uint32_t)(pair >> 32));
}

struct MainSmem {
    float xv[kStageMax];                  // compacted valid samples
    uint64_t vbits[kWords];               // staged-sample validity
    uint32_t vpre[kWords];
    uint64_t sbits[kWords];               // valid samples a gap precedes: they start a segment
    uint64_t live[kWords];                // valid samples of segments of at least W/3
    double tfirst[kWords], tlast[kWords]; // times of each word's first and last valid sample
    int tile;
    int nvalid;
    int multi;                            // the span holds more than one segment
    int check;                            // some of them may be shorter than W/3
    int seg_n[2];                         // samples of the span's first and last segment (>= W/3: at least)
    int any_live;                         // some segment is live
    int walk;                             // bit 0, 1: short of W/3, and the segment goes on
                                          // beyond kNearSamples before, behind the span
    double walk_t[2];                     // time of its valid sample nearest to there
    uint32_t kmin, kmax;                  // smallest and largest staged key
    uint32_t wsum[kMainThreads / 64];     // per wave: bucket counts of its threads
};

// The sorted tile and the wavelet matrix over its ranks.  The sequences' space
// first holds the tile sort's bucket counters; tiles with sorted cores need
// only the ranks, and the waves' cores take all the space behind those.
struct Wavelet {
    uint16_t seq[2][kStageMax];           // level sequences; [0]: rank of each sample
    uint64_t bits[kStageLog2][kWords];    // level bit vectors
    uint32_t pre[kStageLog2][kWords];     // ones before each word
    uint32_t zeros[kStageLog2];           // zeros per level
    uint64_t sortbuf[kStageMax];          // pairs, (key or value << 32 | compacted index)
};
constexpr int kBuckets = kStageMax;       // counters of the tile sort
static_assert(sizeof(Wavelet::seq) >= kBuckets * sizeof(uint32_t), "counters fit");
static_assert(sizeof(Wavelet::seq[0]) == kRankBytes, "cores start behind the ranks");

__device__ __forceinline__ uint32_t rank1(const uint64_t* bits, const uint32_t* pre, uint32_t i)
{
    const uint32_t w = i >> 6;
    const uint64_t m = (1ull << (i & 63u)) - 1ull;
    return pre[w] + (uint32_t)__popcll(bits[w] & m);
}

// Wave-wide minimum and maximum by DPP, valid in lane 63.
__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
#define UMI_STEP(CTRL, ROWS)                                                                       \
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false))
    UMI_STEP(0x111, 0xF);
    UMI_STEP(0x112, 0xF);
    UMI_STEP(0x114, 0xF);
    UMI_STEP(0x118, 0xF);
    UMI_STEP(0x142, 0xA);
    UMI_STEP(0x143, 0xC);
#undef UMI_STEP
    return v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return ~wave_min(~v); }

// The thread's index in the workgroup, opaque to the compiler: it would keep
// every index and address it derives from threadIdx.x across the tiles of the
// estimate kernel's loop, and spill what does not fit (the instance with
// cores: 29 registers spilled against 8).
__device__ __forceinline__ int thread_index()
{
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The value of the lane before (lane 0 keeps its own).
__device__ __forceinline__ double wave_shift(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)u, (int)(uint32_t)u,
                                                              0x138, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(
        (int)(uint32_t)(u >> 32), (int)(uint32_t)(u >> 32), 0x138, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The same value in scalar registers (it is the wave's already).
template <class T>
__device__ __forceinline__ T uniform(const T& v)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    constexpr int n = sizeof(T) / 4;
    int w[n];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < n; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// Inclusive sum over the lanes of a wave by DPP.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
#define UMI_STEP(CTRL, ROWS)                                                                       \
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false)
    UMI_STEP(0x111, 0xF);
    UMI_STEP(0x112, 0xF);
    UMI_STEP(0x114, 0xF);
    UMI_STEP(0x118, 0xF);
    UMI_STEP(0x142, 0xA);
    UMI_STEP(0x143, 0xC);
#undef UMI_STEP
    return v;
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Ones-before prefix over `nw` words, computed by wave 0; returns total ones
// in lane 0's view through `total_out` (written to LDS by the caller).
__device__ __forceinline__ void word_prefix(const uint64_t* bits, uint32_t* pre, int nw, uint32_t* total_out)
{
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const int c = lane < nw ? __popcll(bits[lane]) : 0;
        const int incl = (int)wave_scan((uint32_t)c);
        if (lane < nw) pre[lane] = (uint32_t)(incl - c);
        if (lane == 63) *total_out = (uint32_t)incl;
    }
}

// ---------------------------------------------------------------------------
// Validity and segments of a tile's staged span (gap handling, minimum
// segment length W/3 of Section 4.4).
//
// A window reaches at most W-1 samples and never past its segment, so all it
// needs is inside the staged span: which samples are valid, and where a valid
// sample lies more than kGapDays after the valid one before it (strictly; no
// times, no breaks).  Only a segment's length can depend on samples outside
// the span, and only for the first and the last segment of the span, when
// they hold fewer than W/3 valid samples inside it: those are followed
// outwards until the count is reached or the segment ends.  So no pass over
// the curves precedes the estimate kernel (a scan that wrote one segment word
// per sample took 0.47 ms of 3.0 on 2,000 curves of 40,000-70,000 samples at
// W = 25, and 12 of 50 us on one of 20,000 at W = 361).

// The double in lane l, in scalar registers.
__device__ __forceinline__ double lane_double(double v, int l)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

constexpr int kNearSamples = 256;  // beyond the span, looked at by one wave

// What a wave found in a run of samples beyond the span, in the order away
// from it.
struct WalkPart {
    double first, last;  // times of its valid samples nearest to the span and furthest
    int count, head;     // valid samples, and those before the first break among them
    int cut;             // there is one
    int reserved;
};

// Adds K rows of 64 samples to a part: row u holds the samples of times t[u],
// valid where the lane's ok has bit u, lane after lane; dir > 0: times go up.  The
// predecessors' times come from the lanes for all rows first, so that their
// latencies overlap.
template <int K>
__device__ __forceinline__ void walk_rows(uint32_t ok, const double (&t)[K], int dir, WalkPart& p)
{
    const int lane = thread_index() & 63;
    const uint64_t lower = (1ull << lane) - 1ull;
    uint64_t m[K];
    double ts[K];
#pragma unroll
    for (int u = 0; u < K; ++u) {
        m[u] = __ballot(((ok >> u) & 1u) != 0 && isfinite(t[u]));
        const uint64_t nearer = m[u] & lower;
        ts[u] = __shfl(t[u], nearer ? 63 - (int)__builtin_clzll(nearer) : lane, 64);
    }
#pragma unroll
    for (int u = 0; u < K; ++u) {
        if (p.cut || m[u] == 0) continue;
        const bool none = (m[u] & lower) == 0;  // no valid sample before it in the row
        const double t_in = none ? p.last : ts[u];
        const uint64_t c = __ballot(((m[u] >> lane) & 1ull) != 0 && !(none && p.count == 0) &&
                                    (dir > 0 ? t[u] - t_in : t_in - t[u]) > kGapDays);
        if (c != 0) {
            p.head = p.count + (int)__popcll(m[u] & ((c & -c) - 1ull));
            p.cut = 1;
        }
        if (p.count == 0) p.first = lane_double(t[u], (int)__builtin_ctzll(m[u]));
        p.last = lane_double(t[u], 63 - (int)__builtin_clzll(m[u]));
        p.count += (int)__popcll(m[u]);
    }
}

// Joins a part to the n samples counted so far, the furthest of them at time
// tn; open: the segment goes on.
__device__ __forceinline__ void walk_join(const WalkPart& p, bool timed, int dir, int& n, double& tn,
                                          bool& open)
{
    if (p.count == 0) return;
    if (timed && (dir > 0 ? p.first - tn : tn - p.first) > kGapDays) {
        open = false;
        return;
    }
    n += p.cut ? p.head : p.count;
    open = p.cut == 0;
    tn = p.last;
}

// The 256 samples from curve sample e on in direction dir, added to the n that
// a segment has up to there.  Run by one wave.
__device__ __forceinline__ void walk_near(const float* __restrict__ flux,
                                          const double* __restrict__ time, int len, uint32_t e,
                                          int dir, int& n, double& tn, bool& open)
{
    constexpr int K = kNearSamples / 64;
    const int lane = thread_index() & 63;
    double t[K];
    float x[K];
    uint32_t ok = 0;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const uint32_t i = e + (uint32_t)(dir * (64 * u + lane));
        x[u] = flux[i < (uint32_t)len ? i : 0u];  // (outside the curve: sample 0, not counted)
        t[u] = time != nullptr ? time[i < (uint32_t)len ? i : 0u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < K; ++u)
        ok |= e + (uint32_t)(dir * (64 * u + lane)) < (uint32_t)len && isfinite(x[u]) ? 1u << u : 0u;
    WalkPart p = {0.0, 0.0, 0, 0, 0, 0};
    walk_rows<K>(ok, t, dir, p);
    walk_join(p, time != nullptr, dir, n, tn, open);
}

// Valid samples further beyond the span of the segments that reach its borders,
// added to sm.seg_n until W/3 are found or the segment ends.  By the whole workgroup,
// from the border outwards: 4,096 samples in the first step, 16,384 in the others,
// of which only times of rows with valid samples are read.  Indexes are unsigned:
// one before the curve's start lies beyond its end.
// By one wave, 256 samples a step, this set the time where valid samples are few
// and far apart (one curve without times, us a call: 118 valid samples among
// 2,000,000 at W = 361 10,200, now 605; one in 1,000 of 200,000 at W = 1441 1,735,
// now 108; one in 1,000 of 100,000 at W = 2047, in tiles of two positions, 20,900,
// now 2,090; with times, one in 16 of 18,000 at W = 1081 42, now 28; with a pass
// over the samples ahead 108, 45, 598 and 31).  What is left is latency: loads
// of 16 or 32 samples a lane, of the next while these are counted, or of eight
// consecutive ones a lane gained nothing or cost the ordinary tiles registers.
// At worst a tile reads the samples up to W/3 valid ones away.
__device__ __forceinline__ void walk_beyond(MainSmem& sm, WalkPart* parts,
                                         const float* __restrict__ flux,
                                         const double* __restrict__ time, int len, int s0, int N,
                                         int m_min)
{
    constexpr int K = 8;  // rows of 64 samples that a wave loads together
    const int tid = thread_index();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool multi = sm.multi != 0;
    const int walk = sm.walk;
    int n = sm.seg_n[0];
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {  // before the span, behind it
        if (side == 1 && multi) n = sm.seg_n[1];
        const uint32_t dir = side ? 1u : ~0u;
        uint32_t e = side ? (uint32_t)(s0 + N + kNearSamples) : (uint32_t)(s0 - 1 - kNearSamples);
        double tn = sm.walk_t[side];
        bool open = ((walk >> side) & 1) != 0;
        int turns = 1;
        while (open && n < m_min && e < (uint32_t)len) {
            WalkPart p = {0.0, 0.0, 0, 0, 0, 0};
            uint32_t i0 = e + dir * (uint32_t)(wave * 64 * K * turns + lane);
#pragma unroll 1
            for (int turn = 0; turn < turns && !p.cut && p.count < m_min - n;
                 ++turn, i0 += dir * (64u * K)) {
                float x[K];
#pragma unroll
                for (int u = 0; u < K; ++u)  // (outside the curve: sample 0, not counted)
                    x[u] = flux[i0 + dir * (64u * u) < (uint32_t)len ? i0 + dir * (64u * u) : 0u];
                uint32_t ok = 0;
#pragma unroll
                for (int u = 0; u < K; ++u)
                    ok |= i0 + dir * (64u * u) < (uint32_t)len && isfinite(x[u]) ? 1u << u : 0u;
                if (!__any(ok != 0)) continue;
                if (time == nullptr) {
                    p.count += __builtin_amdgcn_readlane((int)wave_scan((uint32_t)__popc(ok)), 63);
                    continue;
                }
#pragma unroll
                for (int u0 = 0; u0 < K; u0 += K / 2) {
                    double t[K / 2];
#pragma unroll
                    for (int u = 0; u < K / 2; ++u)
                        t[u] = time[((ok >> (u0 + u)) & 1u) != 0 ? i0 + dir * (64u * (u0 + u)) : 0u];
                    walk_rows<K / 2>(ok >> u0, t, side ? 1 : -1, p);
                }
            }
            if (lane == 0) parts[wave] = p;
            __syncthreads();
            for (int w = 0; w < kMainThreads / 64 && open && n < m_min; ++w)
                walk_join(parts[w], time != nullptr, side ? 1 : -1, n, tn, open);
            __syncthreads();
            e += dir * (uint32_t)(kMainThreads * K * turns);
            turns = 4;
        }
        if (tid == 0) sm.seg_n[multi ? side : 0] = n;
    }
    __syncthreads();
}

// From the span's validity and in-word start bits: the prefix counts, the
// starts at word borders, and the sizes of the span's first and last segment
// (the same one without starts), with the samples next to the span.  Run by
// wave 0.
__device__ __forceinline__ void resolve_segments(MainSmem& sm, const float* __restrict__ flux,
                                                 const double* __restrict__ time, int len, int s0,
                                                 int N, int nwv, int m_min)
{
    const int lane = thread_index() & 63;
    const uint64_t v = lane < nwv ? sm.vbits[lane] : 0ull;
    uint64_t s = lane < nwv ? sm.sbits[lane] : 0ull;
    const int c = __popcll(v);
    const int incl = (int)wave_scan((uint32_t)c);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const uint64_t some = __ballot(c > 0);
    if (time != nullptr) {
        // the first valid sample of a word against the last before the word
        const uint64_t earlier = some & ((1ull << lane) - 1ull);
        if (c > 0 && earlier != 0 &&
            sm.tfirst[lane] - sm.tlast[63 - __builtin_clzll(earlier)] > kGapDays) {
            s |= v & -v;
            sm.sbits[lane] = s;
        }
    }
    if (lane < nwv) {
        sm.vpre[lane] = (uint32_t)(incl - c);
        sm.live[lane] = v;
    }
    const uint64_t starts = __ballot(s != 0);
    const bool multi = starts != 0;
    const bool check = total > 0 && m_min > 1 && (multi || total < m_min);
    if (lane == 0) {
        sm.nvalid = total;
        sm.multi = multi ? 1 : 0;
        sm.check = check ? 1 : 0;
        sm.any_live = 0;
    }
    if (!check) return;
    wave_lds_sync();
    int n0 = total, n1 = total;
    if (multi) {  // samples before the first start, and from the last one on
        const int w0 = (int)__builtin_ctzll(starts), w1 = 63 - (int)__builtin_clzll(starts);
        const uint64_t sf = sm.sbits[w0], sl = sm.sbits[w1];
        n0 = (int)sm.vpre[w0] + (int)__popcll(sm.vbits[w0] & ((sf & -sf) - 1ull));
        n1 = total - (int)sm.vpre[w1] -
             (int)__popcll(sm.vbits[w1] & ((1ull << (63 - (int)__builtin_clzll(sl))) - 1ull));
    }
    // what lies next to the span decides most of them
    double t0 = 0.0, t1 = 0.0;
    bool open0 = n0 < m_min && s0 > 0, open1 = false;
    if (open0) {
        t0 = time != nullptr ? sm.tfirst[__builtin_ctzll(some)] : 0.0;
        walk_near(flux, time, len, (uint32_t)(s0 - 1), -1, n0, t0, open0);
    }
    if (!multi) n1 = n0;
    if (n1 < m_min && s0 + N < len) {
        open1 = true;
        t1 = time != nullptr ? sm.tlast[63 - (int)__builtin_clzll(some)] : 0.0;
        walk_near(flux, time, len, (uint32_t)(s0 + N), 1, n1, t1, open1);
    }
    if (!multi) n0 = n1;
    if (lane == 0) {
        sm.seg_n[0] = n0;
        sm.seg_n[1] = n1;
        sm.walk_t[0] = t0;
        sm.walk_t[1] = t1;
        sm.walk = (open0 && n0 < m_min && s0 > kNearSamples ? 1 : 0) |
                  (open1 && n1 < m_min && len - (s0 + N) > kNearSamples ? 2 : 0);
    }
}

// The live bits of a span with segments to check: every sample finds its
// segment by the nearest start bits, a word per wave at a time.  (A walk of one
// wave from segment to segment set the time where segments are many: 40 curves
// of 18,000 with a sample a day, 510 us a call at W = 25 and 615 at W = 361,
// against 48 and 34.)
__device__ __forceinline__ void live_segments(MainSmem& sm, int nwv, int m_min)
{
    const int lane = thread_index() & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint64_t starts = __ballot(lane < nwv && sm.sbits[lane < nwv ? lane : 0] != 0);
    for (int w = wave; w < nwv; w += kMainThreads / 64) {
        const uint64_t v = sm.vbits[w], s = sm.sbits[w];
        const int pre = (int)sm.vpre[w];
        // samples before the segment that reaches into the word, and before the
        // first one that starts after it (-1: the span's first, its last)
        int before = -1, after = -1;
        const uint64_t lower = starts & ((1ull << w) - 1ull);
        const uint64_t upper = starts & ~((2ull << w) - 1ull);
        if (lower != 0) {
            const int u = 63 - (int)__builtin_clzll(lower);
            const int b = 63 - (int)__builtin_clzll(sm.sbits[u]);
            before = (int)sm.vpre[u] + (int)__popcll(sm.vbits[u] & ((1ull << b) - 1ull));
        }
        if (upper != 0) {
            const int u = (int)__builtin_ctzll(upper);
            const uint64_t su = sm.sbits[u];
            after = (int)sm.vpre[u] + (int)__popcll(sm.vbits[u] & ((su & -su) - 1ull));
        }
        const uint64_t upto = s & (~0ull >> (63 - lane)), from = s & ~(~0ull >> (63 - lane));
        if (upto != 0)
            before = pre + (int)__popcll(v & ((1ull << (63 - (int)__builtin_clzll(upto))) - 1ull));
        if (from != 0) after = pre + (int)__popcll(v & ((from & -from) - 1ull));
        const int n = before < 0 ? sm.seg_n[0] : (after < 0 ? sm.seg_n[1] : after - before);
        const uint64_t bits = __ballot(((v >> lane) & 1ull) != 0 && n >= m_min);
        if (lane == 0) {
            sm.live[w] = bits;
            if (bits != 0) sm.any_live = 1;
        }
    }
}

// k-th smallest (0-based) value of the level-0 sequence within [s, e).
__device__ __forceinline__ uint32_t wavelet_kth(const Wavelet& wv, int levels, uint32_t s, uint32_t e, uint32_t k)
{
    uint32_t r = 0;
    for (int l = 0; l < levels; ++l) {
        const uint32_t os = rank1(wv.bits[l], wv.pre[l], s);
        const uint32_t oe = rank1(wv.bits[l], wv.pre[l], e);
        const uint32_t zs = s - os, ze = e - oe;
        const uint32_t nz = ze - zs;
        if (k < nz) {
            s = zs;
            e = ze;
        } else {
            k -= nz;
            s = wv.zeros[l] + os;
            e = wv.zeros[l] + oe;
            r |= 1u << (levels - 1 - l);
        }
    }
    return r;
}

// Number of level-0 values smaller than v within [s, e).
__device__ __forceinline__ uint32_t wavelet_count_less(const Wavelet& wv, int levels, uint32_t s,
                                                       uint32_t e, uint32_t v)
{
    if (v >> levels) return e - s;  // v beyond every stored value
    uint32_t cnt = 0;
    for (int l = 0; l < levels; ++l) {
        const uint32_t os = rank1(wv.bits[l], wv.pre[l], s);
        const uint32_t oe = rank1(wv.bits[l], wv.pre[l], e);
        if ((v >> (levels - 1 - l)) & 1u) {
            cnt += (e - oe) - (s - os);
            s = wv.zeros[l] + os;
            e = wv.zeros[l] + oe;
        } else {
            s -= os;
            e -= oe;
        }
    }
    return cnt;
}

// Phase 3 (Eqs. 2-4) with the asymmetry folded into one fma.  With
// u = (x - mu)/(c s), A = (1 + alpha)/2 and B = (1 - alpha)/2, the effective
// residual of Eq. 2 is A u + B |u| (u for u >= 0, alpha u for u < 0, any
// alpha > 0).  In the scaled variable v = A u = x*k + b, k = A/(c s), it is
// v + beta |v| with beta = B/A, one fma with an |.| source modifier.  The
// sums are sum(w) and sum(w v); Eq. 4 in residual form is then
// mu + sum(w v) / (k sum(w)).
__device__ __forceinline__ void bisquare_acc(float x, float k, float b, float beta, float& sw,
                                             float& swv)
{
    const float v = __builtin_fmaf(x, k, b);
    const float ue = __builtin_fmaf(__builtin_fabsf(v), beta, v);
    // Eq. 3: (1 - ue^2)^2 on |ue| < 1, else 0.  1 - ue^2 <= 1 always, so
    // clamping to [0, 1] is exactly max(., 0).
    const float t = __builtin_amdgcn_fmed3f(__builtin_fmaf(-ue, ue, 1.0f), 0.0f, 1.0f);
    const float w = t * t;
    sw += w;
    swv = __builtin_fmaf(w, v, swv);
}

// Eq. 4 in residual form: mu + sum(w v) / (k sum(w)), with the hardware
// reciprocal (1 ulp): the quotient is a correction of the order of the scale,
// so its last bit is far below the location's, and the errors against 64 bits
// do not change (3.73e-8 at W = 25).  A correctly rounded division took ten
// instructions more per window and iteration (2,000 x 40,000-70,000 samples at
// W = 25: 2.56 ms against 2.46).  Every path uses this same expression, so
// paths that sum in the same order agree bit for bit.
__device__ __forceinline__ float mu_update(float mu, float swv, float sw, float k)
{
    return __builtin_fmaf(swv, __builtin_amdgcn_rcpf(sw * k), mu);
}

// Eq. 1: s = 0.6745 sqrt(ssq / n+), with the hardware square root and
// reciprocal (1 ulp each): once per window, in place of a correctly rounded
// square root and division that cost some 30 instructions (7 % of the
// estimate kernel's time at W = 25).
__device__ __forceinline__ float upper_scale(float ssq, uint32_t nplus)
{
    return kScaleConst * __builtin_amdgcn_sqrtf(ssq * __builtin_amdgcn_rcpf((float)nplus));
}

// The scaled variable's factor k = A / (c s) (A = (1 + alpha) / 2).
__device__ __forceinline__ float bisquare_k(float kA, float c, float s)
{
    return kA * __builtin_amdgcn_rcpf(c * s);
}

// Phase 3 over the n samples xv[c0], ..., xv[c0 + n - 1] of one window, from
// the median m with the scaled k above.  The samples are summed in index
// order whatever the launch shape, so results do not depend on the tiling.
// `n` may be a per-lane count or a wave-uniform one; with a uniform count
// the loop runs on the scalar unit and only the LDS address stays per lane.
__device__ __forceinline__ float bisquare(const float* __restrict__ xv, int c0, int n, float m,
                                          float k, float beta, int iters)
{
    float mu = m;
    const float* x = xv + c0;
    for (int it = 0; it < iters; ++it) {
        const float b = -mu * k;
        float sw = 0.0f, swv = 0.0f;
#pragma unroll 8
        for (int j = 0; j < n; ++j) bisquare_acc(x[j], k, b, beta, sw, swv);
        if (!(sw > 0.0f)) break;  // no weight left: keep mu
        mu = mu_update(mu, swv, sw, k);
    }
    return mu;
}

// Phase 2 sum of squares above the median over xv[c0 .. c0 + n).
__device__ __forceinline__ float upper_ssq(const float* __restrict__ xv, int c0, int n, float m)
{
    float ssq = 0.0f;
    const float* x = xv + c0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) {
        const float d = __builtin_fmaxf(x[j] - m, 0.0f);
        ssq = __builtin_fmaf(d, d, ssq);
    }
    return ssq;
}

// R windows that start at consecutive compacted samples x[0], x[1], ...,
// x[R-1], each n samples long (n >= R): one LDS read feeds every window that
// contains the sample, and each window still sums its samples in index
// order, so the result equals R single-window sweeps bit for bit.
template <int R>
__device__ __forceinline__ void bisquare_multi(const float* __restrict__ x, int n, const float* k,
                                               float* mu, bool* act, float beta, int iters)
{
    for (int it = 0; it < iters; ++it) {
        float b[R], sw[R], swv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            b[r] = -mu[r] * k[r];
            sw[r] = 0.0f;
            swv[r] = 0.0f;
        }
#pragma unroll
        for (int j = 0; j < R - 1; ++j) {  // head: windows 0..j
            const float xj = x[j];
#pragma unroll
            for (int r = 0; r <= j; ++r) bisquare_acc(xj, k[r], b[r], beta, sw[r], swv[r]);
        }
#pragma unroll 8
        for (int j = R - 1; j < n; ++j) {  // every window
            const float xj = x[j];
#pragma unroll
            for (int r = 0; r < R; ++r) bisquare_acc(xj, k[r], b[r], beta, sw[r], swv[r]);
        }
#pragma unroll
        for (int d = 1; d < R; ++d) {  // tail: windows d..R-1 take sample n-1+d
            const float xj = x[n - 1 + d];
#pragma unroll
            for (int r = d; r < R; ++r) bisquare_acc(xj, k[r], b[r], beta, sw[r], swv[r]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (act[r]) {
                if (sw[r] > 0.0f)
                    mu[r] = mu_update(mu[r], swv[r], sw[r], k[r]);
                else
                    act[r] = false;  // no weight left: keep mu from now on
            }
        }
    }
}

// Phase 2 sums for R consecutive windows (see bisquare_multi).
template <int R>
__device__ __forceinline__ void upper_ssq_multi(const float* __restrict__ x, int n, const float* m,
                                                float* ssq)
{
#pragma unroll
    for (int r = 0; r < R; ++r) ssq[r] = 0.0f;
#pragma unroll
    for (int j = 0; j < R - 1; ++j) {
        const float xj = x[j];
#pragma unroll
        for (int r = 0; r <= j; ++r) {
            const float d = __builtin_fmaxf(xj - m[r], 0.0f);
            ssq[r] = __builtin_fmaf(d, d, ssq[r]);
        }
    }
#pragma unroll 4
    for (int j = R - 1; j < n; ++j) {
        const float xj = x[j];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float d = __builtin_fmaxf(xj - m[r], 0.0f);
            ssq[r] = __builtin_fmaf(d, d, ssq[r]);
        }
    }
#pragma unroll
    for (int d = 1; d < R; ++d) {
        const float xj = x[n - 1 + d];
#pragma unroll
        for (int r = d; r < R; ++r) {
            const float dd = __builtin_fmaxf(xj - m[r], 0.0f);
            ssq[r] = __builtin_fmaf(dd, dd, ssq[r]);
        }
    }
}

// The j-th smallest value (0-based) of the window held at compacted
// positions [ca, cb), from the wavelet matrix and the sorted tile.
__device__ __forceinline__ float window_value(const MainSmem& sm, const Wavelet& wv, int levels, uint32_t ca,
                                              uint32_t cb, uint32_t j)
{
    return sorted_value(wv.sortbuf[wavelet_kth(wv, levels, ca, cb, j)]);
}

// Scale ablation: the standard MAD, the lower median of |x - m| over a window
// of n samples with median m.  With the window sorted (v_0 <= ... <= v_{n-1})
// and m = v_q, q = (n-1)/2, the q+1 smallest deviations belong to a run
// v_lo .. v_{lo+q} with 0 <= lo <= q, so the q-th smallest deviation is the
// minimum over lo of max(m - v_lo, v_{lo+q} - m).  The first term falls and
// the second rises with lo: a binary search finds where they cross.  Float
// subtraction is monotone, so the result is the exact MAD rounded once.
__device__ __forceinline__ float window_mad(const MainSmem& sm, const Wavelet& wv, int levels, uint32_t ca,
                                         uint32_t n, float m)
{
    const uint32_t cb = ca + n;
    const uint32_t q = (n - 1) >> 1;
    uint32_t lo = 0, hi = q;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        const float below = m - window_value(sm, wv, levels, ca, cb, mid);
        const float above = window_value(sm, wv, levels, ca, cb, mid + q) - m;
        if (below <= above)
            hi = mid;
        else
            lo = mid + 1;
    }
    float mad = window_value(sm, wv, levels, ca, cb, lo + q) - m;
    if (lo > 0) mad = __builtin_fminf(mad, m - window_value(sm, wv, levels, ca, cb, lo - 1));
    return mad;
}


// Sort 32 keys in registers ascending: Batcher's merge exchange (Knuth, The Art
// of Computer Programming 3, 5.2.2, Algorithm M).  With 23 keys and four
// middle ranks asked for (W = 25) 193 minima and maxima are left of it, 245 of
// a bitonic network.
__device__ __forceinline__ void sort32(uint32_t (&k)[32])
{
#pragma unroll
    for (int p = 16; p > 0; p >>= 1) {
#pragma unroll
        for (int q = 16; q >= p; q >>= 1) {
            // comparators (i, i + d) at i & p == r: first d = p, r = 0, then
            // d = q' - p, r = p for q' = 32 / 2, 32 / 4, ..., 2 p
            const int d = q == 16 ? p : 2 * q - p;
            const int r = q == 16 ? 0 : p;
#pragma unroll
            for (int i = 0; i < 32 - d; ++i) {
                if ((i & p) == r) {
                    const uint32_t a = k[i], b = k[i + d];
                    k[i] = a < b ? a : b;
                    k[i + d] = a < b ? b : a;
                }
            }
        }
    }
}

// Phase 1 for up to three consecutive full windows kp[r .. r + W), r < nwin,
// of W <= kSmallW samples given by their totalOrder keys.  The W - 2 keys the
// three share, kp[2 .. W), are sorted once (padded with the largest key); each
// window is that core plus two keys lo <= hi, and its element of rank
// q = (W-1)/2 is min(A[q], max(A[q-1], lo), max(A[q-2], hi)) for the sorted
// core A (an index below 0 reads as the smallest key): the rank-q element of
// a union of two sorted lists, split over the at most two keys of the second.
// The element of the next rank comes the same way; unless it ties with the
// median, the points strictly above are those ranked after it, else they are
// counted on the unsorted keys.
// Keys past kp[lim] are never read.  Same results as the tile-sort path,
// without the tile sort and wavelet matrix.
// kW > 0 fixes W at compile time: the padding and the median rank are then
// constants, and the compiler drops every comparator that only moves padding
// or feeds ranks other than q-2 .. q.
template <int kW>
__device__ __forceinline__ void small_window_medians(const uint32_t* __restrict__ kp, int W_rt,
                                                     int nwin, int lim, float* pm, uint32_t* pn)
{
    const int W = kW > 0 ? kW : W_rt;
    const int q = (W - 1) >> 1;  // <= 15, the same for the whole tile
    uint32_t med[3], next[3];
    if (W == 1) {
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            med[r] = kp[min(r, lim)];
            next[r] = 0xffffffffu;
        }
    } else {
        uint32_t k[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) k[i] = i < W - 2 ? kp[2 + i] : 0xffffffffu;
        sort32(k);
        uint32_t a0 = k[0], a1 = 0u, a2 = 0u, a3 = k[1];  // A[q], A[q-1], A[q-2], A[q+1]
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            a3 = q == i ? k[i + 1] : a3;
            a0 = q == i ? k[i] : a0;
            a1 = q - 1 == i ? k[i] : a1;
            a2 = q - 2 == i ? k[i] : a2;
        }
        const uint32_t ex[4] = {kp[0], kp[1], kp[min(W, lim)], kp[min(W + 1, lim)]};
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const uint32_t lo = min(ex[r], ex[r + 1]), hi = max(ex[r], ex[r + 1]);
            med[r] = min(a0, min(max(a1, lo), max(a2, hi)));
            next[r] = min(a3, min(max(a0, lo), max(a1, hi)));
        }
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        if (r < nwin) {
            const float m = key_value(med[r]);
            // strictly above, numerically: -0 and +0 are equal
            const uint32_t T = m == 0.0f ? order_key(0.0f) : med[r];
            uint32_t cnt = (uint32_t)(W - 1 - q);
            if (next[r] <= T) {
                cnt = 0;
                for (int j = 0; j < W; ++j) cnt += kp[r + j] > T ? 1u : 0u;
            }
            pm[r] = m;
            pn[r] = cnt;
        }
    }
}

// How far from p, in direction dir and at most `reach` positions, a time
// window extends: up to the last valid sample whose time lies within `half` of
// ti, p's.  Valid samples' times are non-decreasing (the others' may be
// anything), so those samples are a run: its end is looked for around where an
// even cadence has it, in steps that double, then by halving.  Sample by sample
// from the index window's end, 40 curves of 18,000 took 930 us with windows of
// 36 samples and W = 1081, now 218; 100 of 4,408 with 108 and W = 121 75, now 74.
__device__ __forceinline__ int time_reach(const MainSmem& sm, const double* __restrict__ tc, int s0,
                                          int p, int dir, int reach, double ti, double half)
{
    int lo = 0, hi = reach;  // the window's end lies in [lo, hi]
    int d = hi, step = 1;
    int mode = 0;            // at the furthest, at the guess, outwards, inwards, halving
    while (lo < hi) {
        // the valid sample at distance d, or the first one nearer to p (p is one)
        const uint32_t i = (uint32_t)(p + dir * d - s0);
        uint32_t wi = i >> 6;
        uint64_t m = sm.vbits[wi] & (dir < 0 ? ~0ull << (i & 63u) : ~0ull >> (63u - (i & 63u)));
        while (m == 0ull) m = sm.vbits[wi -= (uint32_t)dir];
        const int v = s0 + (int)((wi << 6) + (dir < 0 ? (uint32_t)__builtin_ctzll(m)
                                                      : 63u - (uint32_t)__builtin_clzll(m)));
        const double dt = __builtin_fabs(tc[v] - ti);
        const bool in = dt <= half;
        if (in)
            lo = d;
        else
            hi = dir * (v - p) - 1;
        if (lo >= hi) break;
        if (mode == 0) {
            const float at = (float)half * __builtin_amdgcn_rcpf((float)dt) * (float)(hi + 1);
            d = (int)__builtin_fminf(at, (float)hi);
            mode = 1;
        } else {
            mode = mode == 1 ? (in ? 2 : 3) : (mode == (in ? 2 : 3) ? mode : 4);
            d = mode == 2 ? lo + step : (mode == 3 ? hi + 1 - step : (lo + hi + 1) >> 1);
            step *= 2;
        }
        d = max(min(d, hi), lo + 1);
    }
    return lo;
}

// The window of output position p: its valid samples are the compacted
// positions [ca, ca + n) of the staged tile.  False when p is invalid or in a
// dead segment (a NaN output).  kPair: lanes 2i and 2i + 1 ask for the same p.
template <int kFeat, bool kPair = false>
__device__ __forceinline__ bool window_range(const MainSmem& sm, const CurveDesc& cd,
                                             const double* __restrict__ time, bool multi, int h,
                                             int s0, int N, int p, uint32_t& ca, uint32_t& n)
{
    const uint32_t ip = (uint32_t)(p - s0);
    if (((sm.live[ip >> 6] >> (ip & 63u)) & 1ull) == 0ull) return false;
    int a = max(p - h, s0);
    int b = min(p + h, s0 + N - 1);
    if (multi) {
        // the segment starts at the last start bit up to p, and ends before
        // the first one after it, where these are within reach
        const uint32_t reach = (uint32_t)(a - s0);
        uint32_t wi = ip >> 6;
        uint64_t sb = sm.sbits[wi] & (~0ull >> (63u - (ip & 63u)));
        while (sb == 0ull && (wi << 6) > reach) sb = sm.sbits[--wi];
        if (sb != 0ull) a = max(a, s0 + (int)((wi << 6) + 63u - (uint32_t)__builtin_clzll(sb)));
        const uint32_t from = ip + 1u, lim = (uint32_t)(b - s0);
        wi = from >> 6;
        sb = sm.sbits[wi] & (~0ull << (from & 63u));
        while (sb == 0ull && (wi << 6) + 64u <= lim) sb = sm.sbits[++wi];
        if (sb != 0ull) b = min(b, s0 + (int)((wi << 6) + (uint32_t)__builtin_ctzll(sb)) - 1);
    }
    if ((kFeat & kFeatExtra) && cd.window_days > 0.0) {
        // time window: only the samples within half its length of p count
        const double* tc = time + cd.off;
        const double ti = tc[p];
        const double half = 0.5 * cd.window_days;
        if (kPair) {
            const int dir = (thread_index() & 1) ? 1 : -1;
            const int r = time_reach(sm, tc, s0, p, dir, dir < 0 ? p - a : b - p, ti, half);
            const int other = __builtin_amdgcn_update_dpp(0, r, 0xB1, 0xF, 0xF, false);
            a = p - (dir < 0 ? r : other);
            b = p + (dir < 0 ? other : r);
        } else {
            // a few positions first, both ends at once: windows of nearly W samples
            auto out = [&](int i) {
                const uint32_t q = (uint32_t)(i - s0);
                return !(((sm.vbits[q >> 6] >> (q & 63u)) & 1ull) != 0 &&
                         __builtin_fabs(tc[i] - ti) <= half);
            };
            bool more_a = true, more_b = true;
#pragma unroll 1
            for (int k = 0; k < 8 && (more_a || more_b); ++k) {
                more_a = more_a && out(a);
                more_b = more_b && out(b);
                a += more_a ? 1 : 0;
                b -= more_b ? 1 : 0;
            }
            if (more_a) a = p - time_reach(sm, tc, s0, p, -1, p - a, ti, half);
            if (more_b) b = p + time_reach(sm, tc, s0, p, 1, b - p, ti, half);
        }
    }
    ca = rank1(sm.vbits, sm.vpre, (uint32_t)(a - s0));
    n = rank1(sm.vbits, sm.vpre, (uint32_t)(b - s0 + 1)) - ca;  // >= 1: p is valid
    return true;
}

// Phase 1 of the window at compacted [ca, ca + n) from the sorted tile and
// the wavelet matrix: the median m, and either n+ (the points strictly
// above m, for Eq. 1) or, with the MAD ablation, the scale itself.
__device__ __forceinline__ void window_phase1(const MainSmem& sm, const Wavelet& wv, int levels, int nv, int scale,
                                              uint32_t ca, uint32_t n, float& m, float& sc,
                                              uint32_t& nplus)
{
    const uint32_t cb = ca + n;
    const uint32_t rk = wavelet_kth(wv, levels, ca, cb, (n - 1) >> 1);
    m = sorted_value(wv.sortbuf[rk]);
    if (scale == UMI_SCALE_MAD) {
        sc = window_mad(sm, wv, levels, ca, n, m);
        return;
    }
    // the points strictly above m are the window's elements ranked after
    // the last tile element numerically equal to m (ties and -0/+0 sit next
    // to m in the sorted order); a galloping search: one probe without ties,
    // O(log) with many
    uint32_t rh = rk, hi = rk + 1, step = 1;
    while (hi < (uint32_t)nv && sorted_value(wv.sortbuf[hi]) == m) {
        rh = hi;
        hi = rh + (step <<= 1);
    }
    if (hi > (uint32_t)nv) hi = (uint32_t)nv;
    while (hi - rh > 1u) {  // last equal in [rh, hi)
        const uint32_t mid = (rh + hi) >> 1;
        if (sorted_value(wv.sortbuf[mid]) == m)
            rh = mid;
        else
            hi = mid;
    }
    // exactly k + 1 window elements rank at or below rk (rk is the window's
    // k-th); of the tile elements tied with m after rk, count those in the
    // window directly when they are few, else with a wavelet descent
    const uint32_t k = (n - 1) >> 1;
    if (rh - rk <= 16u) {
        uint32_t tied = 0;
        for (uint32_t j = rk + 1; j <= rh; ++j)
            tied += ((uint32_t)(wv.sortbuf[j] & 0xffffffffull) - ca < n) ? 1u : 0u;
        nplus = n - k - 1 - tied;
    } else {
        nplus = n - wavelet_count_less(wv, levels, ca, cb, rh + 1);
    }
}

// Sorts the tile's (key, index) pairs: sortbuf[0, npad) ascending, as (value,
// index) pairs padded with ~0, and seq[0], the rank of each sample (with
// `ranks` only that), from xv[0, nv) and the keys' range in sm.kmin, sm.kmax; cnt holds
// kBuckets cleared counters.  The keys are dealt to kBuckets buckets of equal
// key range (counted with LDS atomics, placed by a block scan), and each pair
// then counts the pairs of its own bucket below it: seven barriers, where a
// bitonic network over 2,048 pairs has 66.  The pairs are distinct, so the
// order is the network's, whatever order the atomics ran in (the network took
// a third of an estimate launch at W = 121 and 361 without its sweeps: 200 x
// 18,000 samples at W = 121 went from 553 to 490 us with the buckets).  A tile with
// more than kBucketMost pairs in a bucket (long runs of ties, or a few far
// outliers) would count for longer than the network sorts; it takes the network.
constexpr uint32_t kBucketMost = 96;

__device__ __forceinline__ void sort_tile(MainSmem& sm, Wavelet& wv, int nv, int npad, bool ranks)
{
    uint32_t* const cnt = reinterpret_cast<uint32_t*>(wv.seq);
    const int tid = thread_index();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kPer = kStageMax / kMainThreads;
    const uint32_t kmin = sm.kmin;
    const uint32_t range = sm.kmax - kmin;
    const int shift = max(0, 32 - (int)__builtin_clz(range | 1u) - 11);
    static_assert(kBuckets == 1 << 11, "shift");
    uint32_t slot[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kMainThreads;
        if (i < nv) slot[q] = atomicAdd(&cnt[(order_key(sm.xv[i]) - kmin) >> shift], 1u);
    }
    __syncthreads();
    const uint4 c = reinterpret_cast<const uint4*>(cnt)[tid];
    const uint32_t own = c.x + c.y + c.z + c.w;
    const uint32_t incl = wave_scan(own);
    if ((tid & 63) == 63) sm.wsum[wave] = incl;
    if (__syncthreads_or(max(max(c.x, c.y), max(c.z, c.w)) > kBucketMost)) {
        for (int i = tid; i < npad; i += kMainThreads)
            wv.sortbuf[i] = i < nv ? ((uint64_t)order_key(sm.xv[i]) << 32) | (uint32_t)i : ~0ull;
        __syncthreads();
        for (int kk = 2; kk <= npad; kk <<= 1) {
            for (int jj = kk >> 1; jj > 0; jj >>= 1) {
                for (int cix = tid; cix < (npad >> 1); cix += kMainThreads) {
                    const int i = 2 * cix - (cix & (jj - 1));
                    const int l = i + jj;
                    const uint64_t a = wv.sortbuf[i], b = wv.sortbuf[l];
                    const bool asc = (i & kk) == 0;
                    if ((a > b) == asc) {
                        wv.sortbuf[i] = b;
                        wv.sortbuf[l] = a;
                    }
                }
                __syncthreads();
            }
        }
        for (int i = tid; i < npad; i += kMainThreads) {
            const uint64_t p = wv.sortbuf[i];
            wv.seq[0][i < nv ? (uint32_t)p : (uint32_t)i] = (uint16_t)(i < nv ? i : npad - 1);
            if (i < nv) wv.sortbuf[i] = sorted_pair(p);
        }
        __syncthreads();
        return;
    }
    uint32_t base = incl - own;
#pragma unroll
    for (int w = 0; w < kMainThreads / 64; ++w) base += w < wave ? sm.wsum[w] : 0u;
    reinterpret_cast<uint4*>(cnt)[tid] = make_uint4(base, base + c.x, base + c.x + c.y,
                                                    base + c.x + c.y + c.z);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kMainThreads;
        if (i < nv) {
            const uint32_t key = order_key(sm.xv[i]);
            wv.sortbuf[cnt[(key - kmin) >> shift] + slot[q]] = ((uint64_t)key << 32) | (uint32_t)i;
        }
    }
    __syncthreads();
    uint64_t e[kPer];
    uint32_t rank[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kMainThreads;
        if (i < nv) {
            e[q] = wv.sortbuf[i];
            const uint32_t b = ((uint32_t)(e[q] >> 32) - kmin) >> shift;
            const uint32_t lo = cnt[b];
            const uint32_t hi = b + 1 < (uint32_t)kBuckets ? cnt[b + 1] : (uint32_t)nv;
            uint32_t r = lo;
            for (uint32_t j = lo; j < hi; ++j) r += wv.sortbuf[j] < e[q] ? 1u : 0u;
            rank[q] = r;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kMainThreads;
        if (i < nv) {
            wv.seq[0][(uint32_t)e[q]] = (uint16_t)rank[q];
            if (!ranks) wv.sortbuf[rank[q]] = sorted_pair(e[q]);
        } else if (i < npad) {
            wv.seq[0][i] = (uint16_t)(npad - 1);
            wv.sortbuf[i] = ~0ull;
        }
    }
    __syncthreads();
}

// sort_tile as a call, for the instances with every path: inlined there it
// cost them 18 spilled registers (a replayed step of six curves, 89 us against 83).
__device__ __noinline__ void sort_tile_call(MainSmem& sm, Wavelet& wv, int nv, int npad, bool ranks)
{
    sort_tile(sm, wv, nv, npad, ranks);
}

// The windows of one tile: each lane takes R consecutive output positions.
template <int R, int kFeat>
__device__ __forceinline__ void tile_windows(const MainSmem& sm, const Wavelet& wv, int levels, int nv,
                                             const CurveDesc& cd, int h, int s0, int N, int t0,
                                             int t1,
                                             bool multi, float alpha, float c, int iters, int scale, bool simple,
                                             const float* pm, const uint32_t* pn,
                                             const double* __restrict__ time,
                                             float* __restrict__ trend,
                                             float* __restrict__ median,
                                             float* __restrict__ detrended)
{
    const int pfirst = t0 + thread_index() * R;
    uint32_t ca[R], n[R];
    bool live[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = pfirst + r;
        ca[r] = 0;
        n[r] = 0;
        if ((kFeat & kFeatSmall) && simple) {
            // a small-window tile: the whole span is valid and in one live
            // segment, so every window is full and its compacted range is its
            // staged range
            live[r] = p < t1;
            ca[r] = (uint32_t)(p - h - s0);
            n[r] = (uint32_t)cd.W;
        } else {
            live[r] = p < t1 &&
                      window_range<kFeat>(sm, cd, time, multi, h, s0, N, p, ca[r], n[r]);
        }
    }
    // The common case -- every window of the wave live, of one length, and
    // consecutive -- runs the fused loops with a wave-uniform trip count.
    const uint32_t n_u = __builtin_amdgcn_readfirstlane(n[0]);
    bool mine = live[0] && n[0] == n_u && n_u >= (uint32_t)R;
#pragma unroll
    for (int r = 1; r < R; ++r) mine = mine && live[r] && n[r] == n_u && ca[r] == ca[0] + r;
    const bool uniform = __all(mine);

    // Phase 1 (median) and Phase 2 (Eq. 1, or the MAD ablation) per window
    float m[R], sc[R];
    uint32_t nplus[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        m[r] = 0.0f;
        sc[r] = 0.0f;
        nplus[r] = 0;
        if (live[r] && simple) {
            m[r] = pm[r];  // from the small-window networks
            nplus[r] = pn[r];
        } else if (live[r]) {
            window_phase1(sm, wv, levels, nv, scale, ca[r], n[r], m[r], sc[r], nplus[r]);
        }
    }
    if (scale != UMI_SCALE_MAD) {
        float ssq[R];
        if (uniform) {
            upper_ssq_multi<R>(sm.xv + ca[0], (int)n_u, m, ssq);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
                ssq[r] = live[r] ? upper_ssq(sm.xv, (int)ca[r], (int)n[r], m[r]) : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (nplus[r] > 0) sc[r] = upper_scale(ssq[r], nplus[r]);
    }
    float k[R], mu[R];
    bool act[R];
    const float kA = 0.5f * (1.0f + alpha);         // A of the folded residual
    const float beta = (1.0f - alpha) / (1.0f + alpha);  // B / A
#pragma unroll
    for (int r = 0; r < R; ++r) {
        mu[r] = m[r];
        k[r] = 0.0f;
        act[r] = false;
        if (live[r] && sc[r] > 0.0f && iters > 0) {
            const float kk = bisquare_k(kA, c, sc[r]);
            if (isfinite(kk)) {
                k[r] = kk;
                act[r] = true;
            }
        }
    }
    // Phase 3 (Eqs. 2-4)
    if (uniform) {
        bisquare_multi<R>(sm.xv + ca[0], (int)n_u, k, mu, act, beta, iters);
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (act[r]) mu[r] = bisquare(sm.xv, (int)ca[r], (int)n[r], m[r], k[r], beta, iters);
    }
    const float nanf_ = __builtin_nanf("");
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = pfirst + r;
        if (p < t1) {
            trend[cd.off + p] = live[r] ? mu[r] : nanf_;
            if (median) median[cd.off + p] = live[r] ? m[r] : nanf_;
            if (detrended) {
                // normalisation stage: flux / trend (a live sample is valid,
                // so its compacted position is its rank among valid ones)
                float d = nanf_;
                if (live[r]) d = sm.xv[rank1(sm.vbits, sm.vpre, (uint32_t)(p - s0))] / mu[r];
                detrended[cd.off + p] = d;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Split windows: G lanes share one window (tiles of at most kMainThreads / G
// output positions).  Lane l of a group sums the window samples l, l + G,
// l + 2G, ... in order, and a butterfly over the group's G consecutive lanes
// combines the partial sums -- lane xor 1 and xor 2 by DPP quad permutes,
// xor 4 by a ds_swizzle -- in one fixed order.  Every lane of a group ends
// with the same bits (IEEE addition commutes), so the group's lanes iterate
// in step.  The sums are ordered differently from the one-lane-per-window
// path, so the two agree to rounding, not bit for bit; each is deterministic.

__device__ __forceinline__ float dpp_xor1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}

__device__ __forceinline__ float dpp_xor2(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));
}

__device__ __forceinline__ float swizzle_xor4(float v)
{
    // bitmask mode: and 0x1f, or 0, xor 4 (lanes within 32-lane halves)
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x101F));
}

template <int G>
__device__ __forceinline__ float group_sum(float v)
{
    static_assert(G == 2 || G == 4 || G == 8, "group of 2, 4 or 8 lanes");
    v = v + dpp_xor1(v);
    if (G >= 4) v = v + dpp_xor2(v);
    if (G >= 8) v = v + swizzle_xor4(v);
    return v;
}

// f(x[j]) for j = l, l + G, l + 2G, ... below n, in that order; eight loads
// are issued ahead of their use, so a lane waits on LDS once per eight
// samples rather than once per sample (the order of the sums is unchanged).
template <int G, class F>
__device__ __forceinline__ void strided_sweep(const float* __restrict__ x, int l, int n, F&& f)
{
    int j = l;
    for (; j + 7 * G < n; j += 8 * G) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x[j + u * G];
#pragma unroll
        for (int u = 0; u < 8; ++u) f(v[u]);
    }
    for (; j < n; j += G) f(x[j]);
}

// Sum over a group of G consecutive lanes (G = 2, 4, 8), integers.
template <int G>
__device__ __forceinline__ uint32_t group_sum_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
    if (G >= 4) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
    if (G >= 8) v += (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x101F);
    return v;
}

// Phase 1 of a split-tile window from the sorted tile alone (no wavelet
// matrix).  The window's G lanes walk the sorted (key, index) pairs from the
// smallest, 8G at a time (lane l takes the 8 consecutive pairs from 8l), and
// count the pairs whose compacted index lies in [ca, ca + n); the pair at
// which the count reaches k + 1 is the window's k-th smallest, the same
// position wavelet_kth gives.  Each lane's counts of a step travel packed 4
// bits per lane through one group sum, so every lane of the group sees them
// all and takes the same decisions.  Padding pairs (~0) lie in no window, and
// a step never reads past npad (a power of two >= 64, so a multiple of 8G).
// The walk takes about nv / 16G steps to a median, against a wavelet build
// of log2(npad) levels of four barriers each for the whole tile.  The median
// and n+ are the same integers as window_phase1's.
template <int G>
__device__ __forceinline__ void window_phase1_scan(const Wavelet& wv, int nv, uint32_t ca,
                                                   uint32_t n, float& m, uint32_t& nplus)
{
    const uint32_t l = (uint32_t)thread_index() & (G - 1);
    const uint32_t k = (n - 1) >> 1;
    uint32_t need = k + 1;  // window pairs still to pass, the k-th included
    uint32_t rk = 0;
    for (int j0 = 0; j0 < nv; j0 += 8 * G) {
        const int q0 = j0 + 8 * (int)l;
        uint64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = wv.sortbuf[q0 + u];
        uint32_t bits = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            bits |= ((uint32_t)(v[u] & 0xffffffffull) - ca < n ? 1u : 0u) << u;
        const uint32_t packed = group_sum_u32<G>((uint32_t)__popc(bits) << (4 * l));
        uint32_t below = 0, lane_hit = G;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t cg = (packed >> (4 * g)) & 15u;
            if (lane_hit == G) {
                if (below + cg >= need)
                    lane_hit = g;
                else
                    below += cg;
            }
        }
        if (lane_hit == G) {  // not in this step
            need -= below;
            continue;
        }
        // the (need - below)-th window pair of lane lane_hit's eight
        uint32_t pos = 0;
        if (l == lane_hit) {
            uint32_t b = bits;
            for (uint32_t r = need - below; r > 1u; --r) b &= b - 1u;
            pos = (uint32_t)q0 + (uint32_t)__builtin_ctz(b);
        }
        rk = group_sum_u32<G>(pos);
        break;
    }
    m = sorted_value(wv.sortbuf[rk]);
    // the points strictly above m: the window pairs after the last tile pair
    // numerically equal to m (ties sit next to m in the sorted order)
    uint32_t rh = rk, hi = rk + 1, step = 1;
    while (hi < (uint32_t)nv && sorted_value(wv.sortbuf[hi]) == m) {
        rh = hi;
        hi = rh + (step <<= 1);
    }
    if (hi > (uint32_t)nv) hi = (uint32_t)nv;
    while (hi - rh > 1u) {  // last equal in [rh, hi)
        const uint32_t mid = (rh + hi) >> 1;
        if (sorted_value(wv.sortbuf[mid]) == m)
            rh = mid;
        else
            hi = mid;
    }
    uint32_t tied = 0;
    for (uint32_t j = rk + 1 + l; j <= rh; j += G)
        tied += ((uint32_t)(wv.sortbuf[j] & 0xffffffffull) - ca < n) ? 1u : 0u;
    tied = group_sum_u32<G>(tied);
    nplus = n - k - 1 - tied;
}

template <int G, int kFeat>
__device__ __forceinline__ void tile_windows_split(const MainSmem& sm, const Wavelet& wv, int levels, int nv,
                                                   const CurveDesc& cd, int h, int s0, int N,
                                                   int t0, int t1,
                                                   bool multi, float alpha, float c, int iters, int scale,
                                                   const double* __restrict__ time,
                                                   float* __restrict__ trend,
                                                   float* __restrict__ median,
                                                   float* __restrict__ detrended, bool scan)
{
    const int tid = thread_index();
    const int l = tid & (G - 1);
    const int p = t0 + tid / G;
    uint32_t ca = 0, n = 0;
    const bool live =
        p < t1 && window_range<kFeat>(sm, cd, time, multi, h, s0, N, p, ca, n);
    float m = 0.0f, sc = 0.0f;
    uint32_t nplus = 0;
    if (live) {  // same on every lane
        if (scan)
            window_phase1_scan<G>(wv, nv, ca, n, m, nplus);
        else
            window_phase1(sm, wv, levels, nv, scale, ca, n, m, sc, nplus);
    }
    const float* x = sm.xv + ca;
    if (live && scale != UMI_SCALE_MAD) {
        // Phase 2 (Eq. 1)
        float ssq = 0.0f;
        strided_sweep<G>(x, l, (int)n, [&](float xj) {
            const float d = __builtin_fmaxf(xj - m, 0.0f);
            ssq = __builtin_fmaf(d, d, ssq);
        });
        ssq = group_sum<G>(ssq);
        if (nplus > 0) sc = upper_scale(ssq, nplus);
    }
    // Phase 3 (Eqs. 2-4), as in the one-lane path
    float mu = m;
    const float kA = 0.5f * (1.0f + alpha);
    const float beta = (1.0f - alpha) / (1.0f + alpha);
    const float kk = live && sc > 0.0f ? bisquare_k(kA, c, sc) : 0.0f;
    if (live && sc > 0.0f && iters > 0 && isfinite(kk)) {
        for (int it = 0; it < iters; ++it) {
            const float b = -mu * kk;
            float sw = 0.0f, swv = 0.0f;
            strided_sweep<G>(x, l, (int)n,
                             [&](float xj) { bisquare_acc(xj, kk, b, beta, sw, swv); });
            sw = group_sum<G>(sw);
            swv = group_sum<G>(swv);
            if (!(sw > 0.0f)) break;  // no weight left: keep mu
            mu = mu_update(mu, swv, sw, kk);
        }
    }
    if (p < t1 && l == 0) {
        const float nanf_ = __builtin_nanf("");
        trend[cd.off + p] = live ? mu : nanf_;
        if (median) median[cd.off + p] = live ? m : nanf_;
        if (detrended) {
            float d = nanf_;
            if (live) d = sm.xv[rank1(sm.vbits, sm.vpre, (uint32_t)(p - s0))] / mu;
            detrended[cd.off + p] = d;
        }
    }
}

// ---------------------------------------------------------------------------
// Wide windows by sorted cores.
//
// The 32 windows of an aligned group of consecutive positions share all but
// at most 31 samples of each.  One wave takes a group, a pair of lanes per
// window: it compacts the shared samples (the core) in value order out of the
// sorted tile, in blocks of kCoreBlock, and keeps at every block edge the
// first five power sums of the core's deviations from a value near its
// centre, counted from the centre outwards.  Eq. 3's weight is a polynomial of
// degree four in the sample on either side of the location and zero beyond
// the cut-offs, so the sums of Eq. 4 over the blocks strictly between two of
// the three break points (lower cut-off, location, upper cut-off) follow from
// two block edges' power sums, shifted to the location; the block that holds
// a break point and the window's own samples outside the core (its edge
// samples) are summed one by one as in the direct sweep.  Eq. 1's sum follows
// likewise.  An iteration of a 361-sample window takes some 33 + 16 samples
// instead of 361.
//
// The polynomial is exact; what it costs is rounding where the location lies
// far from the centre in units of the cut-off, so a window (or the part below
// its location) is summed directly when it does, and when the scales leave
// the range in which the powers neither overflow nor vanish.  A window's
// result depends only on the group and the window, never on the tile.
//
// What bounds it: VALU issue.  1,000 x 18,000 samples at W = 361: 14.0k lane
// instructions per window and 4.2 ms with every sample summed directly, 5.0k
// and 1.85 ms with groups of 64 windows (a lane each, twice the edge samples),
// 4.6k and 1.75 ms with pairs of lanes, which also keep twice the waves busy
// in a small batch (16 x 20,000: 98 us against 84).  The waves' cores take the
// LDS that the tile sort is done with, so three workgroups fit a CU up to about
// W = 725 (W = 721: 1.42 ms with two, 1.11 with three for 500 x 18,000).

struct CoreLds {
    float* cv;      // core samples in value order
    float* edge;    // samples before the core (32 slots), the core's samples
                    // beyond its last whole block, samples after the core (32)
    uint32_t* over; // the core's rank marks, then Phase 1's kCoreRanks masks,
                    // then (the same space) tree and g
    float* tree;    // first value of each block, by a search tree (core_find)
    float* g;       // five power sums per block edge
};

__device__ __forceinline__ CoreLds core_lds(float* base, int cap)
{
    CoreLds c;
    c.cv = base;
    c.edge = base + ((cap + 3) & ~3);
    c.tree = c.edge + kCoreEdge;
    c.over = reinterpret_cast<uint32_t*>(c.tree);
    c.g = c.tree + core_tree(cap / kCoreBlock);
    return c;
}

// v + (v of the lane a DPP control selects, 0 where it selects none)
template <int kCtrl, int kRows>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(
                   __builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, kRows, 0xF, false));
}

// Inclusive sum over each half of the wave (lanes 0-31, lanes 32-63).
__device__ __forceinline__ float half_scan(float v)
{
    v = dpp_add<0x111, 0xF>(v);  // row_shr:1
    v = dpp_add<0x112, 0xF>(v);  // row_shr:2
    v = dpp_add<0x114, 0xF>(v);  // row_shr:4
    v = dpp_add<0x118, 0xF>(v);  // row_shr:8
    return dpp_add<0x142, 0xA>(v);  // row_bcast:15 into the odd rows
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// The wave's core in value order, nc samples at compacted positions
// [cca, cca + nc), and the edge samples.  The core's samples mark their ranks
// in a bit vector; the marks before a sample's own are its place.
__device__ __forceinline__ void core_collect(const MainSmem& sm, const Wavelet& wv,
                                             const CoreLds& cw, int nv, int cca, int nc)
{
    const int lane = thread_index() & 63;
    const uint16_t* const rank = wv.seq[0] + cca;
    const float* const x = sm.xv + cca;
    uint2* const marks = reinterpret_cast<uint2*>(cw.over);  // (32 ranks, marks before them)
    marks[lane] = make_uint2(0u, 0u);
    wave_lds_sync();
#pragma unroll 4
    for (int j = lane; j < nc; j += 64) {
        const uint32_t r = rank[j];
        atomicOr(&marks[r >> 5].x, 1u << (r & 31u));
    }
    wave_lds_sync();
    const uint32_t c = (uint32_t)__popc(marks[lane].x);
    marks[lane].y = wave_scan(c) - c;
    wave_lds_sync();
#pragma unroll 4
    for (int j = lane; j < nc; j += 64) {
        const uint32_t r = rank[j];
        const uint2 b = marks[r >> 5];
        cw.cv[b.y + (uint32_t)__popc(b.x & ((1u << (r & 31u)) - 1u))] = x[j];
    }
    wave_lds_sync();
    const int rem = nc & (kCoreBlock - 1);
    const int i = cca - 32 + lane + (lane < 32 ? 0 : nc);
    cw.edge[lane + (lane < 32 ? 0 : rem)] = i >= 0 && i < nv ? sm.xv[i] : 0.0f;
    if (lane < rem) cw.edge[32 + lane] = cw.cv[nc - rem + lane];
    wave_lds_sync();
}
static_assert(kStageMax == 64 * 32, "a word of marks per lane");

// The tree's first level, the same for every lane: kept in scalar registers, a
// load less in each search's chain (one curve of 20,000 samples at W = 361:
// 20.5 -> 19.5 us; 200 x 19,440 at W = 1081: 614 -> 600 us).
struct CoreRoot {
    float v1, v2, v3;
};

__device__ __forceinline__ CoreRoot core_root(const CoreLds& cw, int nb)
{
    const int st = 1 << core_top(nb);
    const float nan = __builtin_nanf("");
    CoreRoot r;
    r.v1 = st < nb ? lane_value(cw.cv[kCoreBlock * st], 0) : nan;
    r.v2 = 2 * st < nb ? lane_value(cw.cv[2 * kCoreBlock * st], 0) : nan;
    r.v3 = 3 * st < nb ? lane_value(cw.cv[3 * kCoreBlock * st], 0) : nan;
    return r;
}

// What a curve's alpha fixes for its groups, formed once per tile.
struct CoreParams {
    float kA, beta;   // A = (1 + alpha)/2 and B/A of the folded residual
    float inv_alpha;  // the lower cut-off in units of the upper one
    float quantile;   // of the core, where its centre is taken: about half-way
                      // from the median to where the iterations end
};

__device__ __forceinline__ CoreParams core_params(float alpha)
{
    CoreParams q;
    q.kA = 0.5f * (1.0f + alpha);
    q.beta = (1.0f - alpha) / (1.0f + alpha);
    q.inv_alpha = 1.0f / alpha;
    q.quantile =
        alpha > 1.0f ? __builtin_fminf(0.5f + 0.1f * __builtin_log2f(alpha), 0.8f) : 0.5f;
    return q;
}

// The core's block table and power sums, of its values less the centre: the
// values and the edge samples are shifted by it in place, so that a
// residual's rounding is relative to the deviation and not to the flux
// (trends' error against 64 bits at alpha = 10, c = 2.5, W = 361: 6.61e-8
// without, 6.31e-8 with, 6.39e-8 for windows summed sample by sample; the
// shift is free, the table's pass reads every value anyway).
// The sums start at that edge of the centre's block behind which fewer of its
// values lie far away: where a step or an eclipse ends inside the block, sums
// that took in the far values would lose the near ones' digits (a step of 300
// times the scale: trends off by 6e-4 instead of 1e-7).  `gap` is how far the
// values on the other side reach, below the centre when `below`.  Of the other
// blocks between the centre and a window's location all values lie within its
// cut-offs.  False when the deviations' scale is unusable.
__device__ __forceinline__ bool core_build(const CoreLds& cw, int nc, float quantile, float& centre,
                                           float& unit, float& gap, bool& below)
{
    const int lane = thread_index() & 63;
    const int nb = nc / kCoreBlock;
    // the centre, and a power of two near the core's spread
    const int cq = (int)(quantile * (float)nc);
    const int block = cq / kCoreBlock;
    centre = cw.cv[cq];
    const float under = centre - cw.cv[kCoreBlock * block];
    const float over = cw.cv[kCoreBlock * block + kCoreBlock - 1] - centre;
    float spread = cw.cv[(27 * nc) >> 5] - cw.cv[(5 * nc) >> 5];
    // most of the core equal: the spread of the rest (summed sample by sample,
    // 100 curves of 18,000 with 75 or 97 of 100 samples equal took 2,900 us at
    // W = 1441 instead of 970 and 1,000)
    if (!(spread > 0.0f)) spread = cw.cv[(31 * nc) >> 5] - cw.cv[nc >> 5];
    if (!(spread > 0.0f)) spread = cw.cv[nc - 1] - cw.cv[0];
    const int ex = __builtin_amdgcn_frexp_expf(spread);
    if (!(spread > 0.0f) || ex < -60 || ex > 60) return false;
    unit = __builtin_amdgcn_ldexpf(1.0f, -ex);
    {
        float* t = cw.tree;
        for (int sh = core_top(nb) - 2; sh > 0; sh -= 2) {
            const int len = core_level_len(nb, sh);
            for (int i = lane; i < len; i += 64)
                t[i] = (i << sh) < nb ? cw.cv[(kCoreBlock * i) << sh] - centre : __builtin_nanf("");
            t += len;
        }
    }
    // (LDS operations of a wave keep their order, so the values may change now)
    const float e0 = cw.edge[lane], e1 = cw.edge[64 + (lane & 7)];
    cw.edge[lane] = e0 - centre;
    if (lane < kCoreEdge - 64) cw.edge[64 + lane] = e1 - centre;
    gap = __builtin_fminf(under, over);
    below = __builtin_amdgcn_readfirstlane(under <= over ? 1 : 0) != 0;
    const int bc = block + (below ? 0 : 1);
    // power sums from that edge outwards: upwards in the lower half of the
    // wave, downwards (with a minus sign) in the upper half
    const bool up = lane < 32;
    float carry[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int r0 = 0; r0 < max(nb - bc, bc); r0 += 32) {
        const int i = r0 + (lane & 31);
        const int b = up ? bc + i : bc - 1 - i;
        const bool act = up ? b < nb : b >= 0;
        float s[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (act) {
            float4* const at = reinterpret_cast<float4*>(cw.cv + kCoreBlock * b);
            float4 lo = at[0], hi = at[1];
            lo = make_float4(lo.x - centre, lo.y - centre, lo.z - centre, lo.w - centre);
            hi = make_float4(hi.x - centre, hi.y - centre, hi.z - centre, hi.w - centre);
            at[0] = lo;
            at[1] = hi;
            const float v[kCoreBlock] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int q = 0; q < kCoreBlock; ++q) {
                const float d = v[q] * unit;
                const float d2 = d * d;
                const float d4 = d2 * d2;
                s[0] += d;
                s[1] += d2;
                s[2] = __builtin_fmaf(d2, d, s[2]);
                s[3] += d4;
                s[4] = __builtin_fmaf(d4, d, s[4]);
            }
        }
        const bool more = r0 + 32 < max(nb - bc, bc);
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const float t = half_scan(s[k]) + carry[k];
            if (more) {
                const float lo = lane_value(t, 31), hi = lane_value(t, 63);
                carry[k] = up ? lo : hi;
            }
            if (act) cw.g[5 * (up ? b + 1 : b) + k] = up ? t : -t;
        }
    }
    if (lane < 5) cw.g[5 * bc + lane] = 0.0f;
    wave_lds_sync();
    return true;
}

// Inclusive "or" over each half of the wave, and over the wave.
__device__ __forceinline__ uint32_t half_or_scan(uint32_t v)
{
#define UMI_STEP(CTRL, ROWS)                                                                       \
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false)
    UMI_STEP(0x111, 0xF);
    UMI_STEP(0x112, 0xF);
    UMI_STEP(0x114, 0xF);
    UMI_STEP(0x118, 0xF);
    UMI_STEP(0x142, 0xA);
#undef UMI_STEP
    return v;
}

__device__ __forceinline__ uint32_t wave_or_scan(uint32_t v)
{
    v = half_or_scan(v);
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
}

// Phase 1 of a window by its samples' ranks in the sorted tile: those of a core
// of nc samples from cca on, which core_collect() left marked, and those of the
// nl samples before it and the nr after it, one by one (nc = 0: the nl samples
// from ca on).  The median has the first rank that k + 1 of them do not pass, by
// bisection.  For time windows whose lengths differ by more samples than a group
// has slots for, and groups without a core.  Run by pairs of lanes, which take
// every second sample.  (Over all samples of such windows, by both lanes and with
// two more passes, this took twice as long as all the sums; with those sample by
// sample too, 40 curves of 18,000 at random times, W = 1081 and 648 samples a
// window, took 1,700 us a call, now 305; in bursts of 60, W = 361, 697, now 204.)
__device__ __forceinline__ void rank_phase1(const MainSmem& sm, const Wavelet& wv,
                                            const CoreLds& cw, int nv, int cca, int nc, int ca,
                                            int nl, int nr, float& m, uint32_t& nplus)
{
    const int half = thread_index() & 1;
    const int k = (nl + nc + nr - 1) >> 1;
    const uint2* const marks = reinterpret_cast<const uint2*>(cw.over);
    const uint16_t* const rl = wv.seq[0] + ca;
    const uint16_t* const rr = wv.seq[0] + cca + nc;
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        const int at = (lo + hi) >> 1;
        uint32_t below = 0;
        if (nc > 0 && half == 0) {
            const uint2 b = marks[at >> 5];
            below = b.y + (uint32_t)__popc(b.x & (~0u >> (31u - ((uint32_t)at & 31u))));
        }
#pragma unroll 8
        for (int j = half; j < nl; j += 2) below += (int)rl[j] <= at ? 1u : 0u;
#pragma unroll 8
        for (int j = half; j < nr; j += 2) below += (int)rr[j] <= at ? 1u : 0u;
        if ((int)group_sum_u32<2>(below) > k)
            hi = at;
        else
            lo = at + 1;
    }
    // its value: the core's, or that of the one sample of this rank
    const float* const xl = sm.xv + ca;
    const float* const xr = sm.xv + cca + nc;
    int next = 0;  // core samples of this rank or below
    bool of_core = false;
    if (nc > 0) {
        const uint2 b = marks[lo >> 5];
        const uint32_t bit = 1u << ((uint32_t)lo & 31u);
        next = (int)(b.y + (uint32_t)__popc(b.x & (bit - 1u)));
        of_core = (b.x & bit) != 0;
        if (of_core) m = cw.cv[next++];
    }
    if (!of_core) {
        uint32_t v = 0;
#pragma unroll 8
        for (int j = half; j < nl; j += 2)
            if ((int)rl[j] == lo) v = __float_as_uint(xl[j]);
#pragma unroll 8
        for (int j = half; j < nr; j += 2)
            if ((int)rr[j] == lo) v = __float_as_uint(xr[j]);
        m = __uint_as_float(group_sum_u32<2>(v));
    }
    // n+: the core's from the first value above it, and the others above it
    if (next < nc && cw.cv[next] == m) {
        int last = next, end = nc;  // cv[last] == m
        while (end - last > 1) {
            const int at = (last + end) >> 1;
            if (cw.cv[at] == m)
                last = at;
            else
                end = at;
        }
        next = end;
    }
    uint32_t above = 0;
    auto count = [&](float v) { above += v > m ? 1u : 0u; };
    strided_sweep<2>(xl, half, nl, count);
    strided_sweep<2>(xr, half, nr, count);
    nplus = group_sum_u32<2>(above) + (uint32_t)(nc - next);
}

// Phase 1 (Section 2.1) of a group's windows.  A window is the core plus at
// most 31 edge samples (63 with time windows, which differ in length, and fewer
// than the core has), so its median lies at one of the kRanks core samples around
// the core's middle (of all, where a core behind which infinity stands has fewer),
// or between two of them.  For each of
// those core ranks the wave forms the set of edge samples below that core
// sample (a bit mask: the edge samples' ranks by binary search, set in LDS,
// then a prefix "or" over the lanes); a window counts its own ones with a mask
// of its edge samples, and a binary search over the ranks finds the core
// sample at or below the median.  The median is that sample or one of the few
// edge samples between it and the next.  No tile-wide structure beyond the
// sorted tile.  Values compare as floats; a median of zero takes its sign by
// counting.  Also n+ of Eq. 1.  Windows that do not fit the edge samples' slots,
// and groups without a core, take theirs from rank_phase1().
// Against the wavelet matrix (a build of 44 barriers, then a descent per
// window): 1,000 x 18,000 samples at W = 361 without iterations 1.50 -> 0.88 ms.
template <int kRanks>
__device__ __forceinline__ void core_phase1(const MainSmem& sm, const Wavelet& wv,
                                            const CoreLds& cw, int nv,
                                            bool core, bool fits, int nc, int cca, bool live,
                                            uint32_t ca, uint32_t n, float& m, uint32_t& nplus)
{
    static_assert(kRanks == 32 || kRanks == 64, "a rank per lane of a wave or of its half");
    const int lane = thread_index() & 63;
    const int k = (int)((n - 1) >> 1);
    bool zero = false;
    if (core) {
        const int r0 = max((nc >> 1) - kRanks / 2, 0);
        const float* const mid = cw.cv + r0;
        const int rem = nc & (kCoreBlock - 1);
        // masks of core rank r0 + r: words 2r (samples before the core) and
        // 2r + 1 (after it)
        cw.over[lane] = 0u;
        if (kRanks == 64) cw.over[64 + lane] = 0u;
        const int word = lane >> 5, slot = lane & 31;
        const float e = cw.edge[lane + (word ? rem : 0)];
        int rk = 0;
#pragma unroll
        for (int st = kRanks / 2; st > 0; st >>= 1) rk += mid[rk + st - 1] < e ? st : 0;
        rk += mid[rk] < e ? 1 : 0;
        wave_lds_sync();
        if (rk < kRanks) atomicOr(&cw.over[2 * rk + word], 1u << slot);
        wave_lds_sync();
        if (kRanks == 32) {
            const uint32_t below = half_or_scan(cw.over[2 * slot + word]);
            wave_lds_sync();
            cw.over[2 * slot + word] = below;
        } else {
            const uint32_t b0 = wave_or_scan(cw.over[2 * lane]);
            const uint32_t b1 = wave_or_scan(cw.over[2 * lane + 1]);
            wave_lds_sync();
            cw.over[2 * lane] = b0;
            cw.over[2 * lane + 1] = b1;
        }
        wave_lds_sync();
        const int nl = cca - (int)ca, nr = (int)n - nc - nl;
        const uint32_t own_l = live && fits && nl > 0 ? ~0u << (32 - nl) : 0u;
        const uint32_t own_r = live && fits && nr > 0 ? ~0u >> (32 - nr) : 0u;
        // the last rank r (from r0) with rank + own edge samples below <= k
        const uint2* const masks = reinterpret_cast<const uint2*>(cw.over);
        int r = 0;
#pragma unroll
        for (int st = kRanks / 2; st > 0; st >>= 1) {
            const uint2 b = masks[r + st];
            const int f = r0 + r + st + __popc(b.x & own_l) + __popc(b.y & own_r);
            r += f <= k ? st : 0;
        }
        if (live && fits) {
            // (past the last rank there is no gap: the median is that core
            // sample, as no edge sample lies below it)
            const uint2 b0 = masks[r], b1 = masks[min(r + 1, kRanks - 1)];
            const uint32_t lo_l = b0.x & own_l, lo_r = b0.y & own_r;
            // 0: the core sample; else the t-th of the gap
            int t = k - (r0 + r + __popc(lo_l) + __popc(lo_r));
            m = mid[r];
            nplus = n - (uint32_t)k - 1u;
            float last = -__builtin_inff();
            while (t > 0) {  // the gap's distinct values in turn
                float least = __builtin_inff();
                int cnt = 0;
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    for (uint32_t b = w ? b1.y & own_r & ~lo_r : b1.x & own_l & ~lo_l; b != 0;
                         b &= b - 1) {
                        const float x = cw.edge[(w ? 32 + rem : 0) + (int)__builtin_ctz(b)];
                        if (x > last) {
                            cnt = x < least ? 1 : cnt + (x == least ? 1 : 0);
                            least = __builtin_fminf(least, x);
                        }
                    }
                }
                m = least;
                if (cnt <= 0 || t <= cnt) {
                    nplus -= (uint32_t)(cnt - t);  // equal edge samples after it
                    break;
                }
                t -= cnt;
                last = least;
            }
            // an edge sample equal to a core sample ranks below it, so what
            // else ties with the median after it are the next core samples:
            // the first one above it by a galloping search
            const float* const c = mid + r + 1;
            const int left = nc - (r0 + r + 1);
            if (left > 0 && c[0] == m) {
                int lo = 0, hi = 1;  // c[lo] == m
                while (hi < left && c[hi] == m) {
                    lo = hi;
                    hi = 2 * hi + 1;
                }
                hi = min(hi, left);
                while (hi - lo > 1) {
                    const int at = (lo + hi) >> 1;
                    if (c[at] == m)
                        lo = at;
                    else
                        hi = at;
                }
                nplus -= (uint32_t)(lo + 1);
            }
            zero = m == 0.0f;
        }
        wave_lds_sync();  // the masks give way to the block table
    }
    if (zero) {
        // n+ by counting, and the negative zeros of a zero median; each lane
        // of the pair takes every second sample (one after the other by both:
        // one curve of 18,000 at W = 721 with values of three digits around
        // zero 66 us against 38, 100 at W = 361 480 against 310)
        uint32_t above = 0, negative = 0;
        strided_sweep<2>(sm.xv + ca, lane & 1, (int)n, [&](float v) {
            above += v > 0.0f ? 1u : 0u;
            negative += __float_as_uint(v) >> 31;
        });
        nplus = group_sum_u32<2>(above);
        m = k < (int)group_sum_u32<2>(negative) ? -0.0f : 0.0f;
    }
}

// The last block whose first value is <= the knot (0 where none is): four
// values per level of the tree, the first of which needs no test (a level
// holds every 4th value of the next; beyond the last value stands NaN), and
// at the end the blocks' own first values.  One load per level where a binary
// search takes two dependent ones.  A level's length comes by shifts: as a
// quotient by a stride that only the loop knew it cost a 30-instruction
// integer division per level, search and iteration (1,000 x 18,000 samples at
// W = 361: 1.72 ms against 1.62; 200 x 19,440 at W = 1081: 693 us against 626).
__device__ __forceinline__ int core_find(const CoreLds& cw, const CoreRoot& root, int nb,
                                         float knot)
{
    int b = (root.v1 <= knot ? 1 : 0) + (root.v2 <= knot ? 1 : 0) + (root.v3 <= knot ? 1 : 0);
    const float* tree = cw.tree;
    int sh = core_top(nb);
    if (sh == 0) return b;
    for (sh -= 2; sh > 0; sh -= 2) {
        const float4 v = reinterpret_cast<const float4*>(tree)[b];
        b = 4 * b + (v.y <= knot ? 1 : 0) + (v.z <= knot ? 1 : 0) + (v.w <= knot ? 1 : 0);
        tree += core_level_len(nb, sh);
    }
    b = 4 * b;
    const float* const v = cw.cv + kCoreBlock * b;
    const float v1 = v[kCoreBlock], v2 = v[2 * kCoreBlock], v3 = v[3 * kCoreBlock];
    const bool c1 = v1 <= knot, c2 = c1 && v2 <= knot, c3 = c2 && v3 <= knot;
    // (past the last block stand other values)
    return min(b + (c1 ? 1 : 0) + (c2 ? 1 : 0) + (c3 ? 1 : 0), nb - 1);
}

// Sums of w and w z over blocks [e0, e1) with z = (d - delta) kappa, |z| < 1:
// the blocks' power sums about the location, then (1 - z^2)^2 term by term.
__device__ __forceinline__ void core_poly(const float* __restrict__ g, int e0, int e1, float delta,
                                          float kappa, float& sw, float& swz)
{
    float d[6];
    d[0] = (float)(kCoreBlock * (e1 - e0));
#pragma unroll
    for (int k = 0; k < 5; ++k) d[k + 1] = g[5 * e1 + k] - g[5 * e0 + k];
#pragma unroll
    for (int i = 1; i <= 5; ++i) {
#pragma unroll
        for (int k = 5; k >= i; --k) d[k] = __builtin_fmaf(-delta, d[k - 1], d[k]);
    }
    const float k2 = kappa * kappa;
    sw = __builtin_fmaf(k2, __builtin_fmaf(k2, d[4], -2.0f * d[2]), d[0]);
    swz = kappa * __builtin_fmaf(k2, __builtin_fmaf(k2, d[5], -2.0f * d[3]), d[1]);
}

// f over this lane's half of block b, in value order
template <class F>
__device__ __forceinline__ void core_block(const float* __restrict__ cv, int b, int half, F&& f)
{
    const float4 v = reinterpret_cast<const float4*>(cv)[2 * b + half];
    f(v.x);
    f(v.y);
    f(v.z);
    f(v.w);
}

// Edge samples a lane keeps in registers: half of the most a group of index
// windows has (31 that the windows differ by, and 7 beyond the last block).
// Read from LDS in every iteration by a loop, a wave alone on its SIMD spent
// 1,000 cycles of an iteration on them, and 2,100 where the windows' counts
// differ (at a segment's ends, which set a small batch's time); from registers
// 620, absent ones as samples of no weight.  1,000 x 18,000 samples at W = 361:
// 1.62 -> 1.54 ms, at W = 191: 1.55 -> 1.40 ms; one curve of 9,337 at W = 721:
// 22.7 -> 21.0 us (both with the root above).
constexpr int kEdgeRegs = (kCoreGroup - 1 + kCoreBlock - 1 + 1) / 2;
static_assert(32 + 2 * kEdgeRegs <= kCoreEdge, "loads stay inside the edge samples");

// f over this lane's edge samples: e in registers (the last three only where
// a window has them), the rest of a time window's from xe
template <class F>
__device__ __forceinline__ void core_edges(const float (&e)[kEdgeRegs], const float* xe, int half,
                                           int ne, bool more, F&& f)
{
#pragma unroll
    for (int i = 0; i < kCoreGroup / 2; ++i) f(e[i]);
    if (more) {
#pragma unroll
        for (int i = kCoreGroup / 2; i < kEdgeRegs; ++i) f(e[i]);
        for (int j = 2 * kEdgeRegs + half; j < ne; j += 2) f(xe[j]);
    }
}

// Furthest a location may lie from the core's centre, in units of the
// cut-off of the side summed by power sums.
constexpr float kCoreReach = 0.5f;

// Where the next live segment starts after curve position p, which is staged
// (s0 + N or more: not within the next 63 positions).
__device__ __forceinline__ int next_segment(const MainSmem& sm, int s0, int N, int p)
{
    const uint32_t i = (uint32_t)(p + 1 - s0);
    const uint32_t w = i >> 6, b = i & 63u;
    uint64_t m = (sm.sbits[w] & sm.live[w]) >> b;
    if (b != 0u && 64u * (w + 1u) <= (uint32_t)N) m |= (sm.sbits[w + 1] & sm.live[w + 1]) << (64u - b);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)m);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(m >> 32));
    const uint64_t u = ((uint64_t)hi << 32) | lo;
    return u != 0 ? p + 1 + (int)__builtin_ctzll(u) : s0 + N;
}

// The windows of one group at positions [from, to), all of the group's of one
// segment, a pair of lanes each: the lanes take every second
// edge sample, half of each block summed one by one, and one side's power
// sums; their sums meet by DPP, so both hold the same bits and iterate in step.
template <int kFeat>
__device__ __forceinline__ void core_group(const MainSmem& sm, const Wavelet& wv, const CoreLds& cw,
                                           int nv, const CurveDesc& cd, int h, int s0, int N, int t0,
                                           int t1, int g0, int from, int to, bool multi,
                                           const CoreParams& q, float c, int iters, const double* __restrict__ time,
                                           float* __restrict__ trend, float* __restrict__ median,
                                           float* __restrict__ detrended)
{
    const int lane = thread_index() & 63;
    const int half = lane & 1;
    const int p = g0 + (lane >> 1);
    const bool part = p >= from && p < to;
    const bool mine = part && p >= t0 && p < t1;
    uint32_t ca = 0, n = 0;
    // the ranges of positions outside the tile count too (cut at the staged
    // span, which the core never reaches): the core is the group's
    const bool alive = part && window_range<kFeat, true>(sm, cd, time, multi, h, s0, N, p, ca, n);
    const bool live = alive && mine;
    const uint64_t alive_m = __ballot(alive);
    const uint64_t live_m = __ballot(live);
    float m = 0.0f, mu = 0.0f;
    if (live_m != 0) {
        uint32_t nplus = 0;
        float sc = 0.0f;
        // the core: from the last window's start to the first window's end
        const int lane_lo = (int)__builtin_ctzll(alive_m), lane_hi = 63 - (int)__builtin_clzll(alive_m);
        const int cca = __builtin_amdgcn_readlane((int)ca, lane_hi);
        const int ccb = __builtin_amdgcn_readlane((int)(ca + n), lane_lo);
        const int nc = min(ccb - cca, core_cap(cd.W));
        float centre = 0.0f, unit = 1.0f;
        bool core = nc >= kCoreMin;
        const bool timed = (kFeat & kFeatExtra) && cd.window_days > 0.0;
        if (core) core_collect(sm, wv, cw, nv, cca, nc);
        if (core && timed && nc < 2 * kCoreMin) {  // core_phase1's ranks beyond the core
            if (nc + lane < 2 * kCoreMin) cw.cv[nc + lane] = __builtin_inff();
            wave_lds_sync();
        }
        // nl edge samples before the core, nr after it; windows that differ in
        // length (time windows) may have more than there are slots
        const int nl = live ? cca - (int)ca : 0, nr = live ? (int)n - nc - nl : 0;
        const bool fits = !timed || ((uint32_t)nl <= 32u && (uint32_t)nr <= 32u &&
                                     nl + nr < min(2 * kCoreGroup, nc));
        // (a window that does not hold the core: times that decrease)
        const bool holds = core && nl >= 0 && nr >= 0;
        const bool ranked = live && !(core && fits);
        if (__any(ranked)) {
            if (ranked)
                rank_phase1(sm, wv, cw, nv, cca, holds ? nc : 0, (int)ca, holds ? nl : (int)n,
                            holds ? nr : 0, m, nplus);
            wave_lds_sync();
        }
        if ((kFeat & kFeatExtra) && timed)
            core_phase1<2 * kCoreGroup>(sm, wv, cw, nv, core, fits, nc, cca, live, ca, n, m, nplus);
        else
            core_phase1<kCoreGroup>(sm, wv, cw, nv, core, fits, nc, cca, live, ca, n, m, nplus);
        float gap = 0.0f;
        bool gap_below = false;
        core = core && core_build(cw, nc, q.quantile, centre, unit, gap, gap_below);
        const int nb = nc / kCoreBlock;
        // samples to sum one by one: those before the core, what the core
        // holds beyond its last whole block, and those after the core
        const bool edges = live && fits;
        const float* const xe = cw.edge + 32 - (edges ? nl : 0);
        const int ne = edges ? (int)n - nb * kCoreBlock : 0;
        const CoreRoot root = core_root(cw, nb);
        const bool full = __all(ne >= kCoreGroup - 1), more = __any(ne > kCoreGroup);
        float e[kEdgeRegs];
#pragma unroll
        for (int i = 0; i < kEdgeRegs; ++i) e[i] = xe[2 * i + half];
        auto take = [&](int i) { e[i] = 2 * i + half < ne ? e[i] : -__builtin_inff(); };
        if (!full) {
#pragma unroll
            for (int i = 0; i < kCoreGroup / 2 - 1; ++i) take(i);
        }
#pragma unroll
        for (int i = kCoreGroup / 2 - 1; i < kEdgeRegs; ++i) take(i);
        const float* const x = sm.xv + ca;
        // time windows with more edge samples than slots read theirs where
        // they are
        const bool more_edges = (kFeat & kFeatExtra) && core && live && holds && !fits;
        const bool any_more = (kFeat & kFeatExtra) && __any(more_edges);
        auto far_edges = [&](auto&& f) {
            auto centred = [&](float v) { f(v - centre); };
            strided_sweep<2>(x, half, more_edges ? nl : 0, centred);
            strided_sweep<2>(cw.edge + 32, half, more_edges ? nc - nb * kCoreBlock : 0, f);
            strided_sweep<2>(sm.xv + cca + nc, half, more_edges ? nr : 0, centred);
        };
        const bool served = (live && fits) || more_edges;

        // Phase 2 (Eq. 1)
        float ssq = 0.0f, rest = 0.0f;
        float at = m - centre;
        auto up2 = [&](float v) {
            const float d = __builtin_fmaxf(v - at, 0.0f);
            ssq = __builtin_fmaf(d, d, ssq);
        };
        bool direct = true;
        if (core) {
            core_edges(e, xe, half, ne, more, up2);
            if (any_more) far_edges(up2);
            const int b = core_find(cw, root, nb, at);
            core_block(cw.cv, b, half, up2);
            const int b1 = b + 1;
            const float d0 = (float)(kCoreBlock * (nb - b1));
            const float d1 = cw.g[5 * nb] - cw.g[5 * b1];
            const float d2 = cw.g[5 * nb + 1] - cw.g[5 * b1 + 1];
            const float delta = at * unit;
            const float whole = __builtin_fmaf(delta * delta, d0, d2);
            const float sum = __builtin_fmaf(-2.0f * delta, d1, whole);
            const float back = 1.0f / unit;  // a power of two
            rest = sum * back * back;
            direct = !(served && sum >= 0.125f * whole && whole < 1e30f);
        }
        if (live && direct) {
            at = m;
            ssq = 0.0f;
            rest = 0.0f;
            strided_sweep<2>(x, half, (int)n, up2);
        }
        ssq = group_sum<2>(ssq) + rest;
        if (live && nplus > 0) sc = upper_scale(ssq, nplus);

        // Phase 3 (Eqs. 2-4)
        mu = m;
        float k = 0.0f;
        bool act = false;
        if (live && sc > 0.0f && iters > 0) {
            const float kk = bisquare_k(q.kA, c, sc);
            if (isfinite(kk)) {
                k = kk;
                act = true;
            }
        }
        const float beta = q.beta;
        const float cs = c * sc;               // upper cut-off
        const float cl = cs * q.inv_alpha;     // lower cut-off
        // their inverses per unit of the power sums
        const float ka = __builtin_amdgcn_rcpf(cs * unit);
        const float kb = __builtin_amdgcn_rcpf(cl * unit);
        // (values of the centre's block that the sums of one side hold, though
        // they may lie beyond the cut-offs, are near enough)
        const bool scaled = ka > 1e-4f && ka < 1e4f && gap * unit * (gap_below ? ka : kb) <= 1.5f;
        const float vmax = core ? cw.cv[kCoreBlock * nb - 1] : 0.0f;
        // samples that are not there, and any as far out, weigh nothing
        const float lowest = -1e9f * __builtin_fmaxf(cs, cl);
        if (!full) {
#pragma unroll
            for (int i = 0; i < kCoreGroup / 2 - 1; ++i) e[i] = __builtin_fmaxf(e[i], lowest);
        }
#pragma unroll
        for (int i = kCoreGroup / 2 - 1; i < kEdgeRegs; ++i) e[i] = __builtin_fmaxf(e[i], lowest);
        // this lane's side of the power sums: above the location, or below
        const float kside = half ? ka : kb, fside = half ? q.kA : q.kA * q.inv_alpha;
        const float knot = half ? 0.0f : cl;
        for (int it = 0; it < iters; ++it) {
            const float mu_c = mu - centre;
            float bb = -mu_c * k;
            float sw = 0.0f, swv = 0.0f;
            auto acc = [&](float v) { bisquare_acc(v, k, bb, beta, sw, swv); };
            direct = true;
            if (core) {
                core_edges(e, xe, half, ne, more, acc);
                if (any_more) far_edges(acc);
                const int bm = core_find(cw, root, nb, mu_c - knot);
                const int bo = __float_as_int(dpp_xor1(__int_as_float(bm)));
                const int b0 = half ? bo : bm, b1 = half ? bm : bo;
                // the upper cut-off is rarely inside the core: past its
                // largest value every block above the location is whole
                int b2 = nb;
                if (!(mu_c + cs >= vmax)) {
                    b2 = core_find(cw, root, nb, mu_c + cs);
                    if (b2 != b1) core_block(cw.cv, b2, half, acc);
                }
                core_block(cw.cv, b0, half, acc);
                if (b1 != b0) core_block(cw.cv, b1, half, acc);
                const float delta = mu_c * unit;
                const float far = __builtin_fabsf(delta);
                int e0 = half ? min(b1 + 1, b2) : min(b0 + 1, b1);
                const int e1 = half ? b2 : b1;
                if (!(far * kb <= kCoreReach)) {
                    // too far for the side below: block by block
                    for (int b = min(b0 + 1, b1); b < b1; ++b) core_block(cw.cv, b, half, acc);
                    e0 = half ? e0 : e1;
                }
                float pw, pz;
                core_poly(cw.g, e0, e1, delta, kside, pw, pz);
                sw = group_sum<2>(sw + pw);
                swv = group_sum<2>(__builtin_fmaf(fside, pz, swv));
                direct = !(served && scaled && far * ka <= kCoreReach && sw > 0.03125f * (float)(int)n);
            }
            if (act && direct) {
                bb = -mu * k;
                sw = 0.0f;
                swv = 0.0f;
                strided_sweep<2>(x, half, (int)n, acc);
                sw = group_sum<2>(sw);
                swv = group_sum<2>(swv);
            }
            if (act) {
                if (sw > 0.0f)
                    mu = mu_update(mu, swv, sw, k);
                else
                    act = false;  // no weight left: keep mu from now on
            }
        }
        if (core) wave_lds_sync();  // the next group's core takes this one's place
    }
    if (mine) {
        const float nanf_ = __builtin_nanf("");
        if (half == 0)
            trend[cd.off + p] = live ? mu : nanf_;
        else if (median)
            median[cd.off + p] = live ? m : nanf_;
        if (detrended && half == 1)
            detrended[cd.off + p] =
                live ? sm.xv[rank1(sm.vbits, sm.vpre, (uint32_t)(p - s0))] / mu : nanf_;
    }
}

// kFeat (kFeat* bits) selects the paths an instance carries: the
// small-window networks, split tiles, and the MAD ablation with time windows.
// The host launches the smallest instance that covers the batch; fewer paths
// leave the compiler more registers for the rest, and every instance gives
// the same results on the batches it serves.
template <int kFeat>
__global__ __launch_bounds__(kMainThreads, (kFeat & kFeatCore) ? kCoreWaves : 8) void umi_main_kernel(
    const float* __restrict__ flux, const BatchHeader* __restrict__ hdr,
    const CurveDesc* __restrict__ curves, const int2* __restrict__ tiles, int tile_first,
    int tile_count, uint32_t* __restrict__ counter, float* __restrict__ trend,
    float* __restrict__ median, int core_floats, const SmallTable small)
{
    __shared__ MainSmem sm;
    Wavelet* wvp;
    float* cores = nullptr;
    if constexpr ((kFeat & kFeatCore) != 0) {
        extern __shared__ __align__(16) float dyn[];
        wvp = reinterpret_cast<Wavelet*>(dyn);
        cores = dyn;
    } else {
        __shared__ __align__(16) Wavelet wv_;
        wvp = &wv_;
    }
    Wavelet& wv = *wvp;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool by_value = small.n_curves > 0;
    const int iters = by_value ? small.hdr.iters : hdr->iters;
    const int scale = (kFeat & kFeatExtra) ? (by_value ? small.hdr.scale : hdr->scale)
                                           : (int)UMI_SCALE_UPPER_RMS;
    float* const detrended = by_value ? small.hdr.detrended : hdr->detrended;
    const double* const time = by_value ? small.hdr.time : hdr->time;
    // tile range [tile_first, tile_end): a count < 0 means "all tiles of the batch"
    const int tile_end = tile_count >= 0 ? tile_first + tile_count
                                         : (by_value ? small.hdr.n_tiles : hdr->n_tiles);

    for (int round = 0;; ++round) {
        const int tid = thread_index();
        const int lane = tid & 63;
        // Instances with split tiles serve small batches, where a workgroup
        // often has one tile: its first tile is its block index, and the
        // queue counter hands out the tiles after the grid's first round
        // (not touched at all when the first round covers every tile).
        constexpr bool kStaticFirst = (kFeat & kFeatSplit) != 0;
        if (tid == 0) {
            sm.kmin = ~0u;
            sm.kmax = 0u;
            if (counter && !(kStaticFirst && round == 0))
                sm.tile = (kStaticFirst && tile_first + (int)gridDim.x >= tile_end)
                              ? tile_end
                              : tile_first + (kStaticFirst ? (int)gridDim.x : 0) +
                                    (int)atomicAdd(counter, 1u);
            else
                sm.tile = tile_first + (int)blockIdx.x + round * (int)gridDim.x;
        }
        __syncthreads();
        const int tile = __builtin_amdgcn_readfirstlane(sm.tile);
        if (tile >= tile_end) break;

        CurveDesc cd;
        int t0;
        if (by_value) {
            // the tile's curve: the last table entry whose first tile is <= tile
            int ci = 0;
            if (small.n_curves > 1) {
                const bool le = lane < small.n_curves && small.c[lane].tile_base <= tile;
                ci = 63 - (int)__builtin_clzll(__ballot(le));
            }
            cd = uniform(small.c[ci]);
            t0 = (tile - cd.tile_base) * cd.tile;
        } else {
            const int2 td = tiles[tile];
            cd = uniform(curves[__builtin_amdgcn_readfirstlane(td.x)]);
            t0 = __builtin_amdgcn_readfirstlane(td.y);
        }
        const float alpha = cd.alpha;
        const float c = cd.c;
        const int h = (cd.W - 1) >> 1;
        const int t1 = min(t0 + cd.tile, cd.len);
        const int s0 = max(t0 - h, 0);
        const int s1 = min(t1 + h, cd.len);
        const int N = s1 - s0;  // <= kStageMax, guaranteed by the host
        const float* const f = flux + cd.off;
        const double* const tm = time ? time + cd.off : nullptr;

        // --- staging: validity (finite flux and time) and segment starts as
        // bit vectors, the span's samples in registers ---
        const int nwv = (N >> 6) + 1;
        constexpr int kPer = kStageMax / kMainThreads;
        float xs[kPer];
        {
            double ts[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int i = tid + u * kMainThreads;
                xs[u] = i < N ? f[s0 + i] : __builtin_nanf("");
                ts[u] = i < N && tm ? tm[s0 + i] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int wi = wave + u * (kMainThreads / 64);
                if (wi >= nwv) break;
                const bool ok = isfinite(xs[u]) && isfinite(ts[u]);
                const uint64_t bal = __ballot(ok);
                uint64_t st = 0;
                if (tm) {
                    // against the valid sample before it in the word (the
                    // first of a word: resolve_segments)
                    double before = wave_shift(ts[u]);
                    const uint64_t earlier = bal & ((1ull << lane) - 1ull);
                    const int prev = earlier ? 63 - (int)__builtin_clzll(earlier) : lane;
                    if (__any(ok && prev < lane - 1)) {
                        const double tp = __shfl(ts[u], prev, 64);
                        if (prev != lane - 1) before = tp;
                    }
                    st = __ballot(ok && earlier != 0 && ts[u] - before > kGapDays);
                    if (ok && earlier == 0) sm.tfirst[wi] = ts[u];
                    if (ok && (bal >> lane) == 1ull) sm.tlast[wi] = ts[u];
                }
                if (lane == 0) {
                    sm.vbits[wi] = bal;
                    sm.sbits[wi] = st;
                }
            }
            if (tid == 0 && nwv == kWords) {  // a full span's sentinel word
                sm.vbits[kWords - 1] = 0ull;
                sm.sbits[kWords - 1] = 0ull;
            }
        }
        // lanes per window (1: R windows per lane)
        const int G = (kFeat & kFeatSplit) && !cd.core ? split_lanes(cd.tile) : 1;
        __syncthreads();
        const int m_min = max(1, cd.W / 3);
        if (wave == 0) resolve_segments(sm, f, tm, cd.len, s0, N, nwv, m_min);
        __syncthreads();
        const bool check = __builtin_amdgcn_readfirstlane(sm.check) != 0;
        if (check) {
            if (__builtin_amdgcn_readfirstlane(sm.walk) != 0)
                walk_beyond(sm, reinterpret_cast<WalkPart*>(&wv), f, tm, cd.len, s0, N, m_min);
            live_segments(sm, nwv, m_min);
            __syncthreads();
        }
        // (of a span without a live sample nothing is sorted: its outputs are NaN)
        const int nv = check && __builtin_amdgcn_readfirstlane(sm.any_live) == 0
                           ? 0
                           : __builtin_amdgcn_readfirstlane(sm.nvalid);
        const bool multi = __builtin_amdgcn_readfirstlane(sm.multi) != 0;
        // A tile is "simple" when every one of its windows is full: a small
        // W, no curve end within reach, and the whole span valid and in
        // one segment.  Its medians then come from per-window networks.
        const bool simple = (kFeat & kFeatSmall) && nv == N && !multi && cd.W <= kSmallW &&
                            scale != UMI_SCALE_MAD && cd.window_days == 0.0 && t0 >= h &&
                            t1 + h <= cd.len && G == 1;
        int npad = 64;
        while (npad < nv) npad <<= 1;
        int levels = 6;
        while ((1 << levels) < npad) ++levels;
        const bool core_tile = (kFeat & kFeatCore) && cd.core;
        const bool scan_tile = (kFeat & kFeatSplit) && G > 1 && scale != UMI_SCALE_MAD;

        if (simple) {
            // every staged sample is valid: values and keys in index order
            uint32_t* keys = reinterpret_cast<uint32_t*>(wv.seq);
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int i = tid + u * kMainThreads;
                if (i < N) {
                    sm.xv[i] = xs[u];
                    keys[i] = order_key(xs[u]);
                }
            }
            __syncthreads();
        } else {
        // --- compaction: values in index order, (key, index) for the sort ---
        uint32_t kmin = ~0u, kmax = 0u;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + u * kMainThreads;
            if (i < N && ((sm.vbits[i >> 6] >> lane) & 1ull) != 0ull) {
                const uint32_t ci = rank1(sm.vbits, sm.vpre, (uint32_t)i);
                sm.xv[ci] = xs[u];
                const uint32_t key = order_key(xs[u]);
                kmin = min(kmin, key);
                kmax = max(kmax, key);
            }
        }
        kmin = wave_min(kmin);
        kmax = wave_max(kmax);
        if (lane == 63) {
            atomicMin(&sm.kmin, kmin);
            atomicMax(&sm.kmax, kmax);
        }
        // clear the tile sort's counters
        reinterpret_cast<uint4*>(&wv)[tid] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();

        if (kFeat & kFeatExtra)
            sort_tile_call(sm, wv, nv, npad, core_tile);
        else
            sort_tile(sm, wv, nv, npad, core_tile);

        // --- wavelet matrix over the sequence rank_of[compacted index]; split
        // tiles take their medians from the sorted tile directly ---
        if (!scan_tile && !core_tile) {
        const int nwl = (npad >> 6) + 1;
        for (int l = 0; l < levels; ++l) {
            const uint16_t* cur = wv.seq[l & 1];
            uint16_t* nxt = wv.seq[(l + 1) & 1];
            const int bit = levels - 1 - l;
            for (int i0 = wave * 64; i0 < nwl * 64; i0 += kMainThreads) {
                const int i = i0 + lane;
                const bool one = (i < npad) && (((cur[i < npad ? i : 0] >> bit) & 1) != 0);
                const uint64_t bal = __ballot(one);
                if (lane == 0) wv.bits[l][i0 >> 6] = bal;
            }
            __syncthreads();
            uint32_t ones_total;
            word_prefix(wv.bits[l], wv.pre[l], nwl, &wv.zeros[l]);
            __syncthreads();
            if (tid == 0) {
                ones_total = wv.zeros[l];
                wv.zeros[l] = (uint32_t)npad - ones_total;
            }
            __syncthreads();
            const uint32_t z = wv.zeros[l];
            for (int i = tid; i < npad; i += kMainThreads) {
                const uint16_t val = cur[i];
                const uint32_t o = rank1(wv.bits[l], wv.pre[l], (uint32_t)i);
                const bool one = ((val >> bit) & 1) != 0;
                nxt[one ? z + o : (uint32_t)i - o] = val;
            }
            __syncthreads();
        }
        }  // wavelet
        }  // not simple

        // --- the tile's windows: G lanes per position, or R consecutive
        // positions per lane ---
        if ((kFeat & kFeatSplit) && G > 1) {
            if (G == 2)
                tile_windows_split<2, kFeat>(sm, wv, levels, nv, cd, h, s0, N, t0, t1, multi, alpha, c, iters,
                                      scale, time, trend, median, detrended, scan_tile);
            else if (G == 4)
                tile_windows_split<4, kFeat>(sm, wv, levels, nv, cd, h, s0, N, t0, t1, multi, alpha, c, iters,
                                      scale, time, trend, median, detrended, scan_tile);
            else
                tile_windows_split<8, kFeat>(sm, wv, levels, nv, cd, h, s0, N, t0, t1, multi, alpha, c, iters,
                                      scale, time, trend, median, detrended, scan_tile);
            __syncthreads();
            continue;
        }
        if (core_tile) {
            const CoreLds cw = core_lds(cores + kRankBytes / 4 + wave * core_floats, core_cap(cd.W));
            const CoreParams cp = core_params(alpha);
            // where a segment ends inside a group, the windows on either side
            // share nothing and have a core each (as one group without a core,
            // 100 curves of 18,000 in segments of 500 took 1,470 us at W = 1441, now
            // 670, and one at W = 721 80, now 31)
            for (int from = (t0 & -kCoreGroup) + wave * kCoreGroup; from < t1;) {
                const int g0 = from & -kCoreGroup;
                int to = min(g0 + kCoreGroup, cd.len);
                if (multi) to = min(to, next_segment(sm, s0, N, from));
                core_group<kFeat>(sm, wv, cw, nv, cd, h, s0, N, t0, t1, g0, from, to, multi, cp, c,
                                  iters, time, trend, median, detrended);
                from = to - g0 == kCoreGroup ? g0 + kCoreGroup * (kMainThreads / 64) : to;
            }
            __syncthreads();
            continue;
        }
        const int R = (t1 - t0 + kMainThreads - 1) / kMainThreads;  // tile <= kMaxTile -> R <= 3
        // Simple tiles: Phase 1 of this lane's windows from the networks, run
        // here where few registers are live (every window is [p-h, p+h], all
        // of it valid, so its keys start at staged index p - h - s0).
        float pm[3] = {0.0f, 0.0f, 0.0f};
        uint32_t pn[3] = {0u, 0u, 0u};
        if (simple) {
            const uint32_t* keys = reinterpret_cast<const uint32_t*>(wv.seq);
            const int p0 = t0 + tid * R;
            if (p0 < t1) {
                const int b = p0 - h - s0;
                if (cd.W == 25)  // the Kepler long-cadence window
                    small_window_medians<25>(keys + b, 25, min(R, t1 - p0), N - 1 - b, pm, pn);
                else
                    small_window_medians<0>(keys + b, cd.W, min(R, t1 - p0), N - 1 - b, pm, pn);
            }
        }
        if (R == 3)
            tile_windows<3, kFeat>(sm, wv, levels, nv, cd, h, s0, N, t0, t1, multi, alpha, c, iters, scale,
                            simple, pm, pn, time, trend, median, detrended);
        else if (R == 2)
            tile_windows<2, kFeat>(sm, wv, levels, nv, cd, h, s0, N, t0, t1, multi, alpha, c, iters, scale,
                            simple, pm, pn, time, trend, median, detrended);
        else
            tile_windows<1, kFeat>(sm, wv, levels, nv, cd, h, s0, N, t0, t1, multi, alpha, c, iters, scale,
                            simple, pm, pn, time, trend, median, detrended);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Copy kernel (serving helper, not a step of the method): one workgroup per
// piece of a list of copies between device memory and pinned host memory,
// read and written directly over the bus rather than through the runtime's
// copy engines.

__global__ __launch_bounds__(256) void umi_copy_kernel(CopyBatch cb)
{
    __shared__ int sh_copy;
    const int piece = (int)blockIdx.x;
    if (threadIdx.x < 64) {  // the copy this piece belongs to: last i with first[i] <= piece
        const int lane = (int)threadIdx.x;
        const bool le = lane < cb.n && cb.first[lane] <= piece;
        const uint64_t m = __ballot(le);  // lane 0 always qualifies
        if (lane == 0) sh_copy = 63 - __builtin_clzll(m);
    }
    __syncthreads();
    const int i = sh_copy;
    const int64_t off = (int64_t)(piece - cb.first[i]) * kCopyPieceBytes;
    const int64_t len = min((int64_t)kCopyPieceBytes, cb.bytes[i] - off);
    const uint8_t* src = cb.src[i] + off;
    uint8_t* dst = cb.dst[i] + off;
    const uintptr_t align = (uintptr_t)src | (uintptr_t)dst | (uintptr_t)len;
    if ((align & 15u) == 0) {
        const uint4* s4 = reinterpret_cast<const uint4*>(src);
        uint4* d4 = reinterpret_cast<uint4*>(dst);
        for (int64_t k = threadIdx.x; k < len / 16; k += blockDim.x) d4[k] = s4[k];
    } else if ((align & 3u) == 0) {
        const uint32_t* s1 = reinterpret_cast<const uint32_t*>(src);
        uint32_t* d1 = reinterpret_cast<uint32_t*>(dst);
        for (int64_t k = threadIdx.x; k < len / 4; k += blockDim.x) d1[k] = s1[k];
    } else {
        for (int64_t k = threadIdx.x; k < len; k += blockDim.x) dst[k] = src[k];
    }
}

// ---------------------------------------------------------------------------
// Host-side launch wrappers (the host library calls only these).

// The set-up of a batch: with clear_queue one launch over the staged table (a
// staging block `stage`, or `block` itself in device memory).  Without, the
// estimate launch takes the table by value (kSmallTable) and finds its tiles
// itself: nothing to do.  Samples need no pass of their own, so the arrays of
// the interface that described one stay as they are.
hipError_t launch_prepass(const float*, const double*, uint8_t* block, const uint8_t* stage, int,
                          int grid, int32_t*, int2* tiles, Counters* ctr, ChunkRec*,
                          bool clear_queue, bool, const CurveDesc*, hipStream_t stream)
{
    if (grid <= 0 || !clear_queue) return hipSuccess;
    hipLaunchKernelGGL(umi_setup_kernel, dim3(grid), dim3(kSetupThreads), 0, stream,
                       stage ? stage : block, stage ? block : nullptr, tiles, &ctr->queue);
    return hipGetLastError();
}

hipError_t launch_copy(const CopyBatch& cb, hipStream_t stream)
{
    const int pieces = cb.first[cb.n];
    if (pieces <= 0) return hipSuccess;
    hipLaunchKernelGGL(umi_copy_kernel, dim3(pieces), dim3(256), 0, stream, cb);
    return hipGetLastError();
}

// Without a queue and a tile count, hdr and curves are host memory: a table of
// at most kSmallTable curves, passed by value, one workgroup per tile.
hipError_t launch_main(const float* flux, const int32_t*, const BatchHeader* hdr,
                       const CurveDesc* curves, const int2* tiles, int tile_first,
                       int tile_count, uint32_t* counter, int grid, float* trend, float* median,
                       int feat, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    SmallTable small;
    small.n_curves = 0;
    if (counter == nullptr && tile_count < 0) {
        if (hdr->n_curves < 1 || hdr->n_curves > kSmallTable) return hipErrorInvalidValue;
        small.n_curves = hdr->n_curves;
        small.hdr = *hdr;
        std::memcpy(small.c, curves, (size_t)hdr->n_curves * sizeof(CurveDesc));
        grid = hdr->n_tiles;
        hdr = nullptr;
        curves = nullptr;
    }
    if (!grid_fits(grid)) return hipErrorInvalidValue;
    // instances with sorted cores size their dynamic LDS for the batch's
    // largest core; it also holds the wavelet build's sequences
    const int core_floats = core_floats_for(feat >> kFeatBits);
    feat &= (1 << kFeatBits) - 1;
    if (feat & kFeatNoSplit) feat &= ~(kFeatSplit | kFeatNoSplit);
    const size_t dyn = (feat & kFeatCore)
                           ? std::max(sizeof(Wavelet),
                                      kRankBytes + (size_t)(kMainThreads / 64) * core_floats *
                                                       sizeof(float))
                           : 0;
#define UMI_LAUNCH_MAIN(F)                                                                       \
    hipLaunchKernelGGL(umi_main_kernel<F>, dim3(grid), dim3(kMainThreads), dyn, stream, flux, hdr, \
                        curves, tiles, tile_first, tile_count, counter, trend, median,       \
                       core_floats, small)
    // the instances built: none, small windows, split tiles, everything but
    // cores; cores, cores and small windows, everything
    if (feat == 0)
        UMI_LAUNCH_MAIN(0);
    else if (feat == kFeatSmall)
        UMI_LAUNCH_MAIN(kFeatSmall);
    else if (feat == kFeatSplit)
        UMI_LAUNCH_MAIN(kFeatSplit);
    else if (!(feat & kFeatCore))
        UMI_LAUNCH_MAIN(kFeatSmall | kFeatSplit | kFeatExtra);
    else if (feat == kFeatCore)
        UMI_LAUNCH_MAIN(kFeatCore);
    else if (feat == (kFeatCore | kFeatSmall))
        UMI_LAUNCH_MAIN(kFeatCore | kFeatSmall);
    else
        UMI_LAUNCH_MAIN(kFeatAll);
#undef UMI_LAUNCH_MAIN
    return hipGetLastError();
}

}  // namespace umi
