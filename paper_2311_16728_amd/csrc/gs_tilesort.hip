// Tile binning by per-tile depth sorts: the path gs_bin_sort takes unless the
// tiles are few for the number of records (use_tile_sort's rule).
//
// A (target, Gaussian) pair is counted, placed in its tile's stretch of the
// pair buffer, and only then put in depth order, tile by tile in LDS:
//   count   - a workgroup takes a chunk of one view's records; for every target
//             of the view it lists the visible ones (tile rectangle, record) and
//             counts its pairs per tile in LDS (one row of counts
//             per chunk);
//   columns - every tile's column of counts becomes the exclusive count over
//             the chunks before, and its total; a chunk with far more pairs
//             than others leaves its larger rectangles to be counted here;
//   starts  - every tile's first place (beyond kScanTilesMax tiles; otherwise
//             part of the scatter);
//   scatter - a chunk writes its pairs (key, record) to its slots of each tile,
//             in any order inside a tile's slots of the chunk;
//   order   - a tile's pairs are sorted by (depth key, record) and its records
//             written: lists of up to kSortSmall pairs by a workgroup each,
//             longer ones by a second launch, the longest by many workgroups.
// Four launches (one more where a list may be longer than the small sort
// holds, one for the starts, one more for several targets), against 15 for sorting the
// records by depth and then the pairs by tile: below a few hundred thousand pairs
// the latency of those launches is all there is.  Keys and tie-breaks are those of
// the other path, so the lists are the same: (depth, Gaussian index).  Where a record
// covers hundreds of tiles, sorting pairs is the more work: 100,000 Gaussians of 400 tiles
// at 1200x680 (39.7M pairs) 1,188 us, the records first 501; 20,000 of them 197 and 147.
#include "gs_binning.hpp"

namespace gs {
namespace {

// Pairs of a chunk beyond which its larger entries are taken from it: what a workgroup of
// 256 threads counts or places in 13 us, one of 1,024 in 35 us, and half as much again as
// a chunk's even share of pair_cap, so that calls whose chunks are all alike keep them
// (40,000 Gaussians over 400 tiles each: 1,457 us where all of them were taken, 332
// otherwise); up to kLargeAlways records, whatever the share.
constexpr uint32_t kBudgetFew = 32768, kBudgetMany = 131072;
constexpr int64_t kLargeAlways = 4096;
constexpr int kBinStage = 1024;           // list entries whose pairs are shared out at a time
constexpr uint32_t kSatSlot = 0xffff0000u;   // slots saturate here: a chunk's ranks cannot wrap past it
static_assert(kBinChunkMax <= 0xffff, "a chunk's ranks stay below 2^16");

// Waits until the wave's stores have reached the L2: a barrier does not wait for them, and
// a fence by another wave after it waits for that wave's alone.
__device__ __forceinline__ void stores_reached() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Pair offsets of up to kBinStage list entries (in LDS).
template <int kT>
struct BinStage {
    uint32_t off[kBinStage + 1];
    uint32_t wsum[kT / kWave];
};

__device__ __forceinline__ uint32_t rect_area(uint2 rc) {
    return ((rc.x >> 16) - (rc.x & 0xffffu) + 1u) * ((rc.y >> 16) - (rc.y & 0xffffu) + 1u);
}

// Rows and columns of the tiles [w0, w0 + wn) of a target (row-major, tx a row): of
// all columns where they reach over more than one row.
struct TileSpan {
    uint32_t x0, x1, y0, y1;
};
__device__ __forceinline__ TileSpan tile_span(int w0, int wn, uint32_t tx) {
    const uint32_t a = uint32_t(w0), b = uint32_t(w0 + wn - 1), y0 = a / tx, y1 = b / tx;
    return y0 == y1 ? TileSpan{a - y0 * tx, b - y0 * tx, y0, y1} : TileSpan{0u, tx - 1u, y0, y1};
}
// Cuts a rectangle down to a span; false if nothing is left.
__device__ __forceinline__ bool clip_rect(uint2 &rc, const TileSpan &p) {
    const uint32_t x0 = max(rc.x & 0xffffu, p.x0), x1 = min(rc.x >> 16, p.x1);
    const uint32_t y0 = max(rc.y & 0xffffu, p.y0), y1 = min(rc.y >> 16, p.y1);
    rc = make_uint2(x0 | (x1 << 16), y0 | (y1 << 16));
    return x0 <= x1 && y0 <= y1;
}

// Entries taken at a time from lists over a target of `tiles` tiles: their
// pairs stay below 2^31.
__device__ __forceinline__ uint32_t stage_entries(int tiles) {
    return min(uint32_t(kBinStage), 0x7fffffffu / uint32_t(tiles));
}

// Calls visit4(tile[4], entry[4], count) for the pairs of entries [0, en) of
// rect (en <= kBinStage), every pair once: the pairs, entry by entry and
// row-major in its rectangle, are shared out evenly over the workgroup's
// threads, so a near Gaussian over thousands of tiles takes as long as many
// small ones; a thread passes its consecutive pairs on four at a time.
// (Rectangles taken by 16 lanes each left the workgroup waiting for the
// largest: count 42 us and scatter 59 us for 2.6M pairs, 17-19 us and 32-34 us
// now.)  Barriers inside; ends with one.
template <int kT, class Visit4>
__device__ __forceinline__ void share_pairs(const uint2 *rect, uint32_t en, uint32_t tx, BinStage<kT> &L, Visit4 visit4) {
    constexpr int kPer = kBinStage / kT;
    const int tid = threadIdx.x, wave = tid / kWave;
    uint32_t a[kPer], sum = 0u;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t e = uint32_t(tid * kPer + j);
        a[j] = e < en ? rect_area(rect[e]) : 0u;
        sum += a[j];
    }
    const uint32_t inc = wave_inclusive_scan(sum);
    if (lane_id() == kWave - 1) L.wsum[wave] = inc;
    __syncthreads();
    uint32_t pre = inc - sum, total = 0u;
#pragma unroll
    for (int w = 0; w < kT / kWave; ++w) {
        const uint32_t x = L.wsum[w];
        pre += w < wave ? x : 0u;
        total += x;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        L.off[tid * kPer + j] = pre;
        pre += a[j];
    }
    if (tid == 0) L.off[kBinStage] = total;
    __syncthreads();
    const uint32_t share = (total + kT - 1) / kT;
    uint32_t k = min(total, tid * share);
    const uint32_t k1 = min(total, k + share);
    if (k < k1) {
        uint32_t lo = 0u, hi = en - 1u;   // the last entry that starts at or before k
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1u) / 2u;
            if (L.off[mid] <= k) lo = mid; else hi = mid - 1u;
        }
        uint32_t e = lo, next = L.off[e + 1];
        uint2 rc = rect[e];
        uint32_t x0 = rc.x & 0xffffu, x1 = rc.x >> 16;
        const uint32_t in = k - L.off[e], w = x1 - x0 + 1u, q = in / w;
        uint32_t x = x0 + (in - q * w), row = ((rc.y & 0xffffu) + q) * tx;
        while (k < k1) {
            uint32_t tile[4], entry[4];
            const int m = int(min(4u, k1 - k));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                tile[j] = row + x;
                entry[j] = e;
                ++k;
                if (k < next) {
                    if (++x > x1) { x = x0; row += tx; }
                } else if (k < k1) {
                    ++e;
                    next = L.off[e + 1];
                    rc = rect[e];
                    x0 = rc.x & 0xffffu;
                    x1 = rc.x >> 16;
                    x = x0;
                    row = (rc.y & 0xffffu) * tx;
                }
            }
            visit4(tile, entry, m);
        }
    }
    __syncthreads();
}

// A place after *count (in LDS) for every lane that asks for one, the wave's in a row.
__device__ __forceinline__ uint32_t append(bool wanted, uint32_t *count) {
    const uint64_t mask = __ballot(wanted);
    uint32_t at = 0u;
    if (mask != 0u && lane_id() == 0) at = atomicAdd(count, uint32_t(__popcll(mask)));
    return uint32_t(__builtin_amdgcn_readfirstlane(int(at))) + uint32_t(mask_rank(mask));
}

// A (target, chunk) list's length, and the most tiles of an entry whose pairs its own
// workgroup counts and places (0: any), in one word.  The limit is set where a chunk
// has more pairs than its budget: where large Gaussians are neighbours in the map, one
// workgroup had most pairs of the call.  The larger entries are counted by the
// columns kernel and placed by all of the scatter's workgroups, first in every tile's
// list: both take tiles instead of records and look for the entries that reach into theirs.
// Binning in us, all by the chunk's workgroup / this / sorting the records first: 1M
// Gaussians at 1200x680 with 4,000 of 200 tiles as neighbours 508 / 137 / 173, 300,000
// with 1,000 of 500 tiles 203 / 71 / 111, 300 over every tile 820 / 58 / 75 (of those,
// and of 2,000 over 480 tiles, 254 / 44 / 79, much by smaller chunks); 1M at 6400x3200
// with 4,000 of 5,000 tiles 4,390 / 695 / 705, 300 over every tile 5,111 / 299 / 602.
constexpr int kCountBits = 13, kLimitMax = (1 << (32 - kCountBits)) - 1;
static_assert(kBinChunkMax < 1 << kCountBits, "a list's length");
constexpr uint32_t kCountMask = (1u << kCountBits) - 1u;
__device__ __forceinline__ bool is_large(uint2 rc, uint32_t limit) { return limit != 0u && rect_area(rc) > limit; }

// The large entries of a target's chunks that reach into a span of its tiles: keep(place,
// rectangle in the span, entry) for each, then visit(count) whenever up to kHold of
// them are kept.  `which` holds kT words, S belongs to the call.  A wave takes a chunk, or
// several of them one.
struct LargeState {
    uint32_t chunks, held, more;
};
template <int kT, int kHold, class Keep, class Visit>
__device__ __forceinline__ void large_entries(const uint32_t *__restrict__ count, int64_t chunks, int chunk,
                                              const uint2 *__restrict__ rect, const TileSpan &span, uint32_t *which,
                                              LargeState &S, Keep keep, Visit visit) {
    static_assert(kHold % kT == 0, "steps of a round");
    const int tid = threadIdx.x, lane = lane_id();
    for (int64_t c0 = 0; c0 < chunks; c0 += kT) {
        __syncthreads();
        if (tid == 0) S.chunks = S.held = S.more = 0u;
        __syncthreads();
        const bool any = c0 + tid < chunks && count[c0 + tid] >> kCountBits != 0u;
        const uint32_t place = append(any, &S.chunks);
        if (any) which[place] = uint32_t(c0 + tid);
        __syncthreads();
        const uint32_t n = S.chunks;
        // the waves that share a chunk, and the chunks taken at a time
        const uint32_t wave = uint32_t(__builtin_amdgcn_readfirstlane(tid / kWave));
        const uint32_t parts = n != 0u && n < kT / kWave ? kT / kWave / n : 1u, step = kT / kWave / parts;
        const uint32_t first = wave % parts * kWave;
        uint32_t k = wave / parts < step ? wave / parts : n, e = first;
        for (bool more = n != 0u; more;) {   // uniform
#pragma unroll 1
            for (int j = 0; j < kHold / kT && k < n; ++j) {
                const uint32_t c = uint32_t(__builtin_amdgcn_readfirstlane(int(which[k]))), w = count[c], m = w & kCountMask;
                const int64_t at = int64_t(c) * chunk + e + lane;
                uint2 rc = make_uint2(0u, 0u);
                const bool in = e + lane < m && is_large(rc = rect[at], w >> kCountBits) && clip_rect(rc, span);
                const uint32_t to = append(in, &S.held);
                if (in) keep(to, rc, at);
                e += parts * kWave;
                if (e >= m) {
                    e = first;
                    k += step;
                }
            }
            if (k < n && lane == 0) S.more = 1u;
            __syncthreads();
            more = S.more != 0u;
            visit(S.held);
            __syncthreads();
            if (tid == 0) S.held = S.more = 0u;
            __syncthreads();
        }
    }
}

// The targets of view v: list entries [first, first + count) of view_list
// (kOne: target 0 alone, if its view is v).
template <bool kOne>
__device__ __forceinline__ void targets_of_view(int v, const gs_target *__restrict__ targets,
                                                const uint32_t *__restrict__ view_off, uint32_t &first,
                                                uint32_t &count) {
    first = kOne ? 0u : view_off[v];
    count = kOne ? uint32_t(targets[0].view == v) : view_off[v + 1] - first;
}

// Whether a record may touch the target's image: tile_rect's test with the
// hardware logarithm and square root (relative errors near 1e-6) and margins
// wider than its own by more than they can be off.  A third of tile_rect's
// instructions: the count tries every record of the view and is bound by them.
struct NearScale {
    float sc, sc2, inv_alpha, wmax, hmax;
};
__device__ __forceinline__ NearScale near_scale(const gs_settings &s, const gs_target &t) {
    const float sc = ldexpf(1.f, -t.level);
    return NearScale{sc, sc * sc, 1.f / s.alpha_min, float(t.width - 1), float(t.height - 1)};
}
__device__ __forceinline__ bool maybe_near(const gs_settings &s, const NearScale &c, double2 md, float4 cov_o) {
    const float mx = float(md.x) * c.sc, my = float(md.y) * c.sc;
    const float tq = fmaf(1.386294361f, __builtin_amdgcn_logf(cov_o.w * c.inv_alpha), 1e-5f);   // 2 ln(o / alpha_min)
    const float ex = fmaf(1.002f, __builtin_amdgcn_sqrtf(tq * fmaf(cov_o.x, c.sc2, s.dilation)), 0.1f);
    const float ey = fmaf(1.002f, __builtin_amdgcn_sqrtf(tq * fmaf(cov_o.z, c.sc2, s.dilation)), 0.1f);
    // (what compares false, as with a NaN, is left to tile_rect)
    return cov_o.w >= s.alpha_min && !(mx + ex < 0.f) && !(my + ey < 0.f) && !(mx - ex > c.wmax) && !(my - ey > c.hmax);
}

// Grid (chunks, n_views).  LDS: the counts of a window of the target's tiles
// (dynamic, `window` words) and the chunk's tile rectangles; of a target of several
// windows, the parts of them that lie in the window.
// kOne: a single target in the call; the kernel then also clears the counters
// and the raster queue (no set-up kernel runs).
// 64 registers, so that two workgroups of 1,024 threads share a CU and one works
// while the other waits at a barrier: 32 keyframes of three levels 721 -> 568 us,
// 8 keyframes 149 -> 119.
template <int kT, bool kOne>
__global__ void __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(8))) bin_count_kernel(
    gs_settings s, Proj proj, int64_t n, int64_t n_cap, int chunk, const gs_target *__restrict__ targets, int n_targets,
    const uint32_t *__restrict__ view_off, const uint32_t *__restrict__ view_list, int window, uint32_t budget, BinLists lists,
    uint32_t *__restrict__ thist, int64_t stride, int total_tiles, uint32_t *__restrict__ counters,
    uint32_t *__restrict__ queue) {
    extern __shared__ uint32_t hist[];
    constexpr int kChunkMax = kT == kBinThreadsFew ? kBinChunkMin : kBinChunkMax, kLoad = kChunkMax / kT;
    __shared__ uint2 srect[kChunkMax];
    __shared__ BinStage<kT> L;
    __shared__ uint16_t near[kChunkMax];
    __shared__ uint32_t s_count, s_near, s_pairs;
    const int tid = threadIdx.x;
    const int v = blockIdx.y;
    const int64_t g0 = int64_t(blockIdx.x) * chunk;
    if (kOne && blockIdx.x == 0 && v == 0) {
        if (tid < kNumCounters) counters[tid] = 0u;
        if (tid < kQueueWords) queue[tid] = 0u;
    }
    // tiles that no other workgroup counts have no pairs: those of targets of no view (an
    // index outside [0, n_views)), and those before, between and after the targets'
    // (total_tiles of a larger layout)
    if (v == 0) {
        uint32_t *row = thist + int64_t(blockIdx.x) * stride;
        auto clear = [&](int first, int count) {   // each lane's stretch, by the whole wave
            for (uint64_t m = __ballot(count > 0); m != 0ull; m &= m - 1) {
                const int j = __builtin_ctzll(m), f = __shfl(first, j, kWave), c = __shfl(count, j, kWave);
                for (int i = lane_id(); i < c; i += kWave) row[f + i] = 0u;
            }
        };
        for (int t0 = 0; t0 < n_targets; t0 += kT) {   // (whole waves take part)
            const int ti = t0 + tid;
            int first = 0, count = 0, before = 0;
            if (ti < n_targets) {
                const gs_target &t = targets[ti];
                const bool seen = t.view >= 0 && t.view < int(gridDim.y);
                first = t.tile_offset + (seen ? t.tiles_x * t.tiles_y : 0);
                count = (ti + 1 < n_targets ? targets[ti + 1].tile_offset : total_tiles) - first;
                if (ti == 0) before = t.tile_offset;
                if (!seen) lists.count[int64_t(ti) * gridDim.x + blockIdx.x] = 0u;
            }
            clear(first, count);
            clear(0, before);
        }
    }
    uint32_t q0, m;
    targets_of_view<kOne>(v, targets, view_off, q0, m);
    if (m == 0u) return;   // uniform
    // the chunk's records, held in registers for every target of the view
    const int held = int(min(int64_t(chunk), n - g0));
    double2 md[kLoad];
    float4 co[kLoad];
#pragma unroll
    for (int k = 0; k < kLoad; ++k) {
        const int i = tid + k * kT;
        const int64_t r = int64_t(v) * n_cap + (i < held ? g0 + i : 0);
        md[k] = proj.mean[r];
        co[k] = proj.cov_o[r];
    }
    for (uint32_t q = 0; q < m; ++q) {
        const uint32_t ti = kOne ? 0u : view_list[q0 + q];
        const gs_target t = targets[ti];
        const int tiles = t.tiles_x * t.tiles_y;
        const NearScale scale = near_scale(s, t);
        const int64_t lbase = int64_t(ti) * n_cap + g0;   // the chunk's list entries
        if (tid == 0) s_count = s_near = s_pairs = 0u;
        uint32_t limit = 0u;
        for (int w0 = 0; w0 < tiles; w0 += window) {
            const int wn = min(window, tiles - w0);
            for (int i = tid; i < wn; i += kT) hist[i] = 0u;
            __syncthreads();
            if (w0 == 0) {   // the list of the chunk's visible records: those that may be, then the exact test
                uint64_t mask[kLoad];
                uint32_t seen = 0u;
#pragma unroll
                for (int k = 0; k < kLoad; ++k) {
                    const int i = tid + k * kT;
                    mask[k] = __ballot(i < held && maybe_near(s, scale, md[k], co[k]));
                    seen += uint32_t(__popcll(mask[k]));
                }
                uint32_t at = 0u;
                if (seen != 0u && lane_id() == 0) at = atomicAdd(&s_near, seen);
                at = uint32_t(__builtin_amdgcn_readfirstlane(int(at)));
#pragma unroll
                for (int k = 0; k < kLoad; ++k) {
                    if ((mask[k] >> lane_id()) & 1u) near[at + uint32_t(mask_rank(mask[k]))] = uint16_t(tid + k * kT);
                    at += uint32_t(__popcll(mask[k]));
                }
                __syncthreads();
                const uint32_t near_n = s_near;
                uint32_t area = 0u;
                for (uint32_t e0 = 0; e0 < near_n; e0 += kT) {   // (whole waves take part)
                    const uint32_t i = e0 + tid < near_n ? near[e0 + tid] : 0u;
                    const int64_t r = int64_t(v) * n_cap + g0 + i;
                    Rect rc{0, 0, 0, 0};
                    const bool vis = e0 + tid < near_n && tile_rect(s, proj.mean[r], proj.cov_o[r], t, rc);
                    const uint32_t at = append(vis, &s_count);
                    if (vis) {
                        const uint2 packed = make_uint2(uint32_t(rc.x0) | (uint32_t(rc.x1) << 16),
                                                        uint32_t(rc.y0) | (uint32_t(rc.y1) << 16));
                        area += min(rect_area(packed), uint32_t(kLimitMax));
                        srect[at] = packed;
                        lists.rect[lbase + at] = packed;
                        lists.rec[lbase + at] = uint32_t(r);
                    }
                }
                area = wave_inclusive_scan(area);
                if (lane_id() == kWave - 1 && area != 0u) atomicAdd(&s_pairs, area);
                __syncthreads();
                if (s_pairs > budget) limit = max(min(budget / (4u * s_count), uint32_t(kLimitMax)), 1u);
            }
            uint32_t cnt = s_count;
            if (tiles > window || limit != 0u) {   // uniform
                const TileSpan span = tile_span(w0, wn, uint32_t(t.tiles_x));
                if (tid == 0) s_near = 0u;
                __syncthreads();
                for (uint32_t e0 = 0; e0 < cnt; e0 += kT) {   // (whole waves take part)
                    uint2 rc = make_uint2(0u, 0u);
                    const bool in = e0 + tid < cnt && !is_large(rc = lists.rect[lbase + e0 + tid], limit) && clip_rect(rc, span);
                    const uint32_t at = append(in, &s_near);
                    if (in) srect[at] = rc;
                }
                __syncthreads();
                cnt = s_near;
            }
            const uint32_t step = stage_entries(tiles);
            for (uint32_t e0 = 0; e0 < cnt; e0 += step)
                share_pairs<kT>(srect + e0, min(cnt - e0, step), uint32_t(t.tiles_x), L,
                                [&](const uint32_t (&tile)[4], const uint32_t (&)[4], int mm) {
#pragma unroll
                                    for (int j = 0; j < 4; ++j) {
                                        const uint32_t i = tile[j] - uint32_t(w0);
                                        if (j < mm && i < uint32_t(wn)) atomicAdd(&hist[i], 1u);
                                    }
                                });
            __syncthreads();
            uint32_t *row = thist + int64_t(blockIdx.x) * stride + t.tile_offset + w0;
            for (int i = tid; i < wn; i += kT) row[i] = hist[i];
        }
        if (tid == 0) {
            lists.count[int64_t(ti) * gridDim.x + blockIdx.x] = s_count | (limit << kCountBits);
            if (!kOne && limit != 0u) counters[kLarge] = 1u;
        }
        __syncthreads();   // s_count and srect are reused by the next target
    }
}

// Exclusive scan of every column of thist over the chunks, in place; column
// totals to total[t], and each workgroup's sum of them to group_total.  A workgroup takes 64 tiles, one per lane, so each load
// is a contiguous 256-byte piece of a row, and its kColWaves waves take
// consecutive runs of chunks.  Runs of up to kColHold chunks stay in registers
// between the sum and the prefixes (one batch of loads); longer ones are read
// twice, kColBatch loads at a time.
// Large entries come before all rows: the workgroup looks for those that reach into its
// tiles of each target, kColLarge at a time, and a lane counts its tile's.
constexpr int kColWaves = 16, kColHold = 16, kColBatch = 16, kColLarge = 4096;
__global__ void __launch_bounds__(kColWaves * kWave) bin_columns_kernel(
    int64_t rows, int64_t tiles, uint32_t *__restrict__ thist, int64_t stride, uint32_t *__restrict__ total,
    uint64_t *__restrict__ group_total, BinLists lists, int64_t n_cap, int chunk, const gs_target *__restrict__ targets,
    int n_targets, uint32_t *__restrict__ counters) {
    constexpr int kT = kColWaves * kWave;
    __shared__ uint32_t wsum[kColWaves][kWave], which[kT], s_targets[kWave], s_overlap;
    __shared__ uint2 rect[kColLarge];
    __shared__ LargeState state;
    __shared__ bool any_large[kColWaves];
    // whether a chunk has large entries: from the lists of a single target, whose counters
    // the count kernel cleared
    const bool one = n_targets == 1;
    const uint32_t some = one ? 0u : counters[kLarge];
    uint32_t mine = one && threadIdx.x < rows ? lists.count[threadIdx.x] >> kCountBits : 0u;
    if (one)   // (the first is waited for beside the counts)
        for (int64_t l = threadIdx.x + kT; l < rows; l += kT) mine |= lists.count[l] >> kCountBits;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    uint32_t *col = thist + int64_t(blockIdx.x) * kWave + lane;
    const int64_t per = (rows + kColWaves - 1) / kColWaves;
    const int64_t b0 = wave * per, b1 = b0 + per < rows ? b0 + per : rows;
    auto large_pairs = [&]() {   // of the lane's tile, shared out over the waves
        const int64_t g0 = int64_t(blockIdx.x) * kWave;
        if (threadIdx.x == 0) s_overlap = 0u;
        __syncthreads();
        for (int t0 = 0; t0 < n_targets; t0 += kT) {   // (whole waves take part)
            const int ti = t0 + threadIdx.x;
            bool in = false;
            if (ti < n_targets) {
                const int64_t first = targets[ti].tile_offset;
                in = first < g0 + kWave && first + targets[ti].tiles_x * targets[ti].tiles_y > g0;
            }
            const uint32_t at = append(in, &s_overlap);
            if (in && at < uint32_t(kWave)) s_targets[at] = uint32_t(ti);
        }
        __syncthreads();
        uint32_t found = 0u;
        for (uint32_t q = 0; q < min(s_overlap, uint32_t(kWave)); ++q) {
            const int64_t ti = s_targets[q];
            const gs_target &t = targets[ti];
            const int64_t tx = t.tiles_x, n = tx * t.tiles_y, a = max(g0 - t.tile_offset, int64_t(0));
            const int64_t b = min(g0 + kWave - t.tile_offset, n), tile = g0 + lane - t.tile_offset;
            const uint32_t y = uint32_t(tile / tx), x = uint32_t(tile - y * tx);
            const bool valid = tile >= a && tile < b;
            large_entries<kT, kColLarge>(
                lists.count + ti * rows, rows, chunk, lists.rect + ti * n_cap, tile_span(int(a), int(b - a), uint32_t(tx)), which,
                state, [&](uint32_t to, uint2 rc, int64_t) { rect[to] = rc; },
                [&](uint32_t held) {
                    for (uint32_t i = wave; i < held; i += kColWaves) {
                        const uint2 rc = rect[i];
                        found += valid && x >= (rc.x & 0xffffu) && x <= rc.x >> 16 && y >= (rc.y & 0xffffu) && y <= rc.y >> 16;
                    }
                });
        }
        return found;
    };
    auto cross_waves = [&](uint32_t s, uint32_t &run, uint32_t &all) {
        wsum[wave][lane] = s;
        if (one) {
            const bool large = __ballot(mine != 0u) != 0ull;
            if (lane == 0) any_large[wave] = large;
        }
        __syncthreads();
        run = 0u;
        all = 0u;
#pragma unroll
        for (int w = 0; w < kColWaves; ++w) {
            const uint32_t x = wsum[w][lane];
            run += w < wave ? x : 0u;
            all += x;
        }
        if (one ? __ballot(any_large[lane % kColWaves]) == 0ull : some == 0u) return;   // uniform
        if (one && blockIdx.x == 0 && threadIdx.x == 0) counters[kLarge] = 1u;   // for the scatter
        const uint32_t found = large_pairs();
        __syncthreads();
        wsum[wave][lane] = found;
        __syncthreads();
        uint32_t before = 0u;
#pragma unroll
        for (int w = 0; w < kColWaves; ++w) before += wsum[w][lane];
        run += before;
        all += before;
    };
    uint32_t run, all;
    if (per <= kColHold) {   // uniform over the workgroup
        uint32_t v[kColHold], s = 0u;
#pragma unroll
        for (int j = 0; j < kColHold; ++j) {
            v[j] = b0 + j < b1 ? col[(b0 + j) * stride] : 0u;
            s += v[j];
        }
        cross_waves(s, run, all);
#pragma unroll
        for (int j = 0; j < kColHold; ++j) {
            if (b0 + j < b1) col[(b0 + j) * stride] = run;
            run += v[j];
        }
    } else {
        uint32_t s = 0u;
        for (int64_t b = b0; b < b1; b += kColBatch) {
            uint32_t v[kColBatch];
#pragma unroll
            for (int j = 0; j < kColBatch; ++j) v[j] = b + j < b1 ? col[(b + j) * stride] : 0u;
#pragma unroll
            for (int j = 0; j < kColBatch; ++j) s += v[j];
        }
        cross_waves(s, run, all);
        for (int64_t b = b0; b < b1; b += kColBatch) {
            uint32_t v[kColBatch];
#pragma unroll
            for (int j = 0; j < kColBatch; ++j) v[j] = b + j < b1 ? col[(b + j) * stride] : 0u;
#pragma unroll
            for (int j = 0; j < kColBatch; ++j) {
                if (b + j < b1) col[(b + j) * stride] = run;
                run += v[j];
            }
        }
    }
    if (wave == 0) {
        const int64_t t = int64_t(blockIdx.x) * kWave + lane;
        total[t] = all;
        uint64_t sum = t < tiles ? all : 0u;
        sum = wave_inclusive_scan64(sum);
        if (lane == kWave - 1) group_total[blockIdx.x] = sum;
    }
}

// What is published about the tiles once their starts are known: ranges (clamped to
// the pair capacity), the tiles whose lists are longer than the small sort holds,
// those of which more than one workgroup sorts (with their slices and runs), and by
// the last tile's owner the pair counters.  A lane publishes the ranges of its tiles one by one
// and marks the longer lists; publish() then makes their entries, the whole wave at
// once, as each wait for an atomic takes microseconds.
constexpr int kPackBits = 21;   // (lists, slices and runs of 2^31 pairs: below 2^20 each)
struct Longer {
    uint32_t bits = 0u;   // the lane's tiles
    static __device__ __forceinline__ uint32_t slices(uint32_t n) { return (n + kSortLarge - 1) / kSortLarge; }
    static __device__ __forceinline__ uint32_t runs(uint32_t n) {
        return min(uint32_t(kRunsMax), (n + kRunTarget - 1) / kRunTarget);
    }
    // tile `first + j` of the lane
    __device__ __forceinline__ void range(uint32_t first, int j, uint64_t start, uint32_t count, uint32_t cap, uint2 *ranges) {
        const uint32_t a = uint32_t(start < cap ? start : cap);
        const uint64_t end = start + count;
        const uint32_t b = uint32_t(end < cap ? end : cap);
        ranges[first + j] = make_uint2(a, b);
        bits |= b - a > uint32_t(kSortSmall) ? 1u << j : 0u;
    }
    __device__ __forceinline__ void publish(uint32_t first, const uint2 *ranges, uint32_t *__restrict__ longs,
                                            const LongLists &lists, uint32_t *__restrict__ counters) {
        if (__ballot(bits != 0u) == 0ull) return;   // uniform
        uint32_t few = 0u;   // lists of one workgroup
        uint64_t many = 0;   // lists, slices and runs of the others, kPackBits each
#pragma unroll 1
        for (uint32_t b = bits; b != 0u; b &= b - 1u) {
            const uint2 r = ranges[first + __builtin_ctz(b)];
            const uint32_t n = r.y - r.x;
            if (n <= uint32_t(kSortAlone)) ++few;
            else many += (uint64_t(runs(n)) << (2 * kPackBits)) + (uint64_t(slices(n)) << kPackBits) + 1u;
        }
        const uint64_t all = wave_inclusive_scan64(many);
        const uint32_t all_few = wave_inclusive_scan(few);
        uint64_t at = 0;
        uint32_t at_few = 0u;
        if (lane_id() == kWave - 1) {
            if (all != 0) at = atomicAdd(reinterpret_cast<unsigned long long *>(counters + kLongLists), (unsigned long long)all);
            if (all_few != 0u) at_few = atomicAdd(&counters[kLongTiles], all_few);
        }
        at = (uint64_t(__builtin_amdgcn_readlane(uint32_t(at >> 32), kWave - 1)) << 32) |
             uint32_t(__builtin_amdgcn_readlane(uint32_t(at), kWave - 1));
        at += all - many;
        at_few = uint32_t(__builtin_amdgcn_readlane(at_few, kWave - 1)) + all_few - few;
#pragma unroll 1
        for (; bits != 0u; bits &= bits - 1u) {
            const uint32_t t = first + __builtin_ctz(bits);
            const uint2 r = ranges[t];
            const uint32_t n = r.y - r.x;
            if (n <= uint32_t(kSortAlone)) {
                longs[at_few++] = t;
                continue;
            }
            constexpr uint32_t kMask = (1u << kPackBits) - 1u;
            lists.list[uint32_t(at) & kMask] = make_uint4(t, n, uint32_t(at >> kPackBits) & kMask, uint32_t(at >> (2 * kPackBits)));
            at += (uint64_t(runs(n)) << (2 * kPackBits)) + (uint64_t(slices(n)) << kPackBits) + 1u;
        }
    }
};
__device__ __forceinline__ void publish_pairs(uint64_t pairs, uint32_t cap, uint32_t *__restrict__ counters,
                                              uint32_t *__restrict__ d_status) {
    counters[kPairs] = sat32(pairs);
    counters[kPairsClamped] = uint32_t(pairs < cap ? pairs : cap);
    if (pairs > cap && d_status) atomicOr(d_status, GS_STATUS_PAIR_OVERFLOW);
}

// Tile starts from the totals, for more tiles than the scatter's workgroups
// scan themselves (kScanTilesMax): a workgroup takes kStartTiles tiles, after
// the sum of group_total over those before.  start[t] (over total) is saturated.
// (One workgroup walking all tiles took 77 us for 80,606, this 7 us.)
constexpr int kStartPer = 4, kStartTiles = 256 * kStartPer;
__global__ void __launch_bounds__(256) bin_starts_kernel(int64_t tiles, uint32_t cap,
                                                         const uint64_t *__restrict__ group_total,
                                                         uint32_t *__restrict__ total, uint2 *ranges,
                                                         uint32_t *__restrict__ longs, LongLists long_lists,
                                                         uint32_t *__restrict__ counters,
                                                         uint32_t *__restrict__ d_status) {
    __shared__ uint64_t lds64[kScanThreads / kWave];
    const int tid = threadIdx.x;
    const int64_t groups = int64_t(blockIdx.x) * (kStartTiles / kWave);
    uint64_t before = 0, run, all;
    for (int64_t i = tid; i < groups; i += 256) before += group_total[i];
    block_exclusive_scan64(before, lds64, &run);
    const int64_t t0 = int64_t(blockIdx.x) * kStartTiles + tid * kStartPer;
    uint32_t v[kStartPer];
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < kStartPer; ++j) {
        v[j] = t0 + j < tiles ? total[t0 + j] : 0u;
        s += v[j];
    }
    uint64_t pre = run + block_exclusive_scan64(s, lds64, &all);
    Longer longer;
#pragma unroll
    for (int j = 0; j < kStartPer; ++j) {
        if (t0 + j < tiles) {
            longer.range(uint32_t(t0), j, pre, v[j], cap, ranges);
            total[t0 + j] = uint32_t(pre < kSatSlot ? pre : kSatSlot);
        }
        pre += v[j];
    }
    longer.publish(uint32_t(t0), ranges, longs, long_lists, counters);
    if (blockIdx.x == gridDim.x - 1 && tid == 0) publish_pairs(run + all, cap, counters, d_status);
}

// Exclusive sums of up to kScanTilesMax totals, to each(place of the thread's, tile, sum
// before it, total); returns the sum of all.  A barrier inside.
template <int kT, class Each>
__device__ __forceinline__ uint64_t scan_totals(const uint32_t *__restrict__ total, int64_t total_tiles, uint64_t *lds64,
                                                Each each) {
    constexpr int kPer = kScanTilesMax / kT;
    const int tid = threadIdx.x, wave = tid / kWave;
    uint32_t v[kPer];
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t g = int64_t(tid) * kPer + j;
        v[j] = g < total_tiles ? total[g] : 0u;
        s += v[j];
    }
    const uint64_t inc = wave_inclusive_scan64(s);
    if (lane_id() == kWave - 1) lds64[wave] = inc;
    __syncthreads();
    uint64_t pre = inc - s, all = 0;
#pragma unroll
    for (int w = 0; w < kT / kWave; ++w) {
        const uint64_t x = lds64[w];
        pre += w < wave ? x : 0u;
        all += x;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        each(j, int64_t(tid) * kPer + j, pre, v[j]);
        pre += v[j];
    }
    return all;
}

struct ScatterArgs {
    Proj proj;
    float znear;
    int64_t n_cap;
    int chunk;
    int64_t chunks;
    const gs_target *targets;
    int64_t total_tiles;
    int window;
    BinLists lists;
    uint32_t *thist;
    int64_t stride;
    const uint32_t *total;
    uint32_t cap;
    uint2 *pairs;
    uint2 *ranges;
    uint32_t *longs;
    LongLists long_lists;
    uint32_t *counters;
    uint32_t *d_status;
    KeepState *keep;
};
// The scatter's arguments, loaded again: what the rare parts use of them holds no
// registers before (with all loaded at the start, 107 spilled: 24 targets 141 us, so 132).
__device__ __forceinline__ const ScatterArgs &args_again() {
    auto p = (const __attribute__((address_space(4))) ScatterArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const ScatterArgs *)p;
}

// More pairs than the buffer holds: the first `cap` of them in the order (depth key,
// record, target, row-major in its rectangle) are kept, as where the records are sorted
// first, so every tile keeps its nearest Gaussians.  By the last kCrew workgroups of the
// scatter to get here, over the lists of the whole call: a radix selection, weighted by the
// rectangles' tiles, of the record that the cap-th pair belongs to, digit by digit; the pairs
// of every tile before it counted; the tile starts; and the pairs placed.  Each of these is a
// phase, whose items (some lists) are taken from a counter, and begins when the one
// before is done: the workgroup that ends its last item goes on at once, the others
// wait for it kWaits rounds (milliseconds) at most and then leave the rest to those that
// are there, so the launch ends whichever workgroups run at the same time.  `first`: the
// workgroup that got here last, which clears what the phases count with.  `tile` holds a word
// per tile, srect and sent (kBinStage entries each), L and lds64 are the caller's LDS.
// Bound: the phases' latency, some 20 us each, and the atomics on the tiles, in a call that
// raises the overflow flag and is to be repeated with a larger buffer.  By one workgroup / by
// these: 1M Gaussians at 1200x680, 2.6M pairs for 0.9M 2.9 / 0.34 ms (the sort of the records
// first, which only drops what is past the end, 0.1); 20,000 of 950 tiles, 18.9M pairs for
// 16.8M 15 / 2.2; 100,000 in 400 targets, 53M pairs for 34M 1,770 / 22.
constexpr int kSelectBits = 10, kCrew = 128, kWaits = 4096;
static_assert(kRankBits <= kKeepDigits * kSelectBits && (1 << kSelectBits) == kKeepBins, "digits of a rank");
static_assert(kKeepBins == kBinStage, "the selection's bins lie over srect");
template <int kT>
__device__ __forceinline__ void keep_first_pairs(const ScatterArgs &R, int n_targets, bool first, uint2 *srect, uint2 *sent,
                                                 BinStage<kT> &L, uint64_t *lds64) {
    constexpr int kWaves = kT / kWave, kPer = kKeepBins / kWave;
    constexpr int64_t kClear = 16384;   // tiles an item clears
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = lane_id();
    KeepState &K = *R.keep;
    uint32_t *tile = R.thist;
    const int64_t total_tiles = R.total_tiles, all_lists = R.chunks * n_targets;
    const uint32_t cap = R.cap;
    auto now = [](const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto wait_for = [&](const uint32_t *p, uint32_t n) {   // whether *p got to n
        __syncthreads();
        if (tid == 0) {
            for (int i = 0; i < kWaits && now(p) < n; ++i) __builtin_amdgcn_s_sleep(16);
            lds64[0] = now(p) >= n;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        const bool got = lds64[0] != 0;
        __syncthreads();
        return got;
    };
    auto phase = [&](int p, uint32_t items, auto work, auto end) {   // whether all items are done
        uint32_t did = 0u;
        for (;; ++did) {
            __syncthreads();
            if (tid == 0) lds64[0] = atomicAdd(&K.next[p], 1u);
            __syncthreads();
            const uint32_t item = uint32_t(lds64[0]);
            if (item >= items) break;   // uniform
            work(item);
        }
        end(did);
        stores_reached();
        __syncthreads();
        if (tid == 0 && did != 0u) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            atomicAdd(&K.done[p], did);
        }
        return wait_for(&K.done[p], items);
    };
    auto nothing = [](uint32_t) {};

    if (first) {
        uint32_t *words = reinterpret_cast<uint32_t *>(&K);
        for (uint32_t i = tid; i < sizeof(KeepState) / sizeof(uint32_t); i += kT) words[i] = 0u;
        if (tid == 0) R.counters[kLongTiles] = R.counters[kLongLists] = R.counters[kLongLists + 1] = 0u;
        stores_reached();
        __syncthreads();
        if (tid == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            atomicAdd(&R.counters[kGo], 1u);
        }
    }
    if (!wait_for(&R.counters[kGo], 1u)) return;   // uniform

    auto key_of = [&](uint32_t r) { return depth_key(R.proj.rgb_z[r].w, R.znear); };
    auto rank = [](uint32_t key, uint32_t r) { return (uint64_t(key) << 32) | r; };
    const int64_t per = (all_lists + 8 * kCrew - 1) / (8 * kCrew);   // lists an item
    const uint32_t items = uint32_t((all_lists + per - 1) / per);
    const int64_t parts = per < kWaves ? kWaves / per : 1;   // of a list, a wave each
    // digit by digit, the rank of the record that holds the cap-th pair, and the pairs before it
    unsigned long long *bins = reinterpret_cast<unsigned long long *>(srect);
    uint64_t last = 0, before = 0;
    for (int d = 0, hi = kRankBits; hi > 0; ++d) {
        const int lo = hi > kSelectBits ? hi - kSelectBits : 0;
        __syncthreads();
        for (int i = tid; i < kKeepBins; i += kT) bins[i] = 0ull;
        const bool done = phase(
            d, items + (d == 0 ? uint32_t((total_tiles + kClear - 1) / kClear) : 0u),
            [&](uint32_t item) {
                if (item >= items) {
                    const int64_t t0 = (item - items) * kClear, t1 = min(t0 + kClear, total_tiles);
                    for (int64_t t = t0 + tid; t < t1; t += kT) tile[t] = 0u;
                    return;
                }
                const int64_t l1 = min(all_lists, (item + 1) * per);
                for (int64_t i = wave; ; i += kWaves) {
                    const int64_t l = item * per + i / parts;
                    if (l >= l1) break;
                    const int64_t at = l / R.chunks * R.n_cap + l % R.chunks * R.chunk;
                    const uint32_t cnt = R.lists.count[l] & kCountMask;
                    for (uint32_t e = uint32_t(i % parts) * kWave + lane; e < cnt; e += uint32_t(parts) * kWave) {
                        const uint32_t r = R.lists.rec[at + e];
                        const uint64_t c = rank(key_of(r), r);
                        if (c >> hi == last >> hi)
                            atomicAdd(&bins[(c >> lo) & ((1u << (hi - lo)) - 1u)],
                                      (unsigned long long)rect_area(R.lists.rect[at + e]));
                    }
                }
            },
            [&](uint32_t) {
                __syncthreads();
                for (int i = tid; i < kKeepBins; i += kT)
                    if (bins[i] != 0ull) atomicAdd(&K.bins[d][i], bins[i]);
            });
        if (!done) return;   // uniform
        if (wave == 0) {
            auto bin = [&](int i) { return __hip_atomic_load(&K.bins[d][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            uint64_t sum = 0;
            for (int j = 0; j < kPer; ++j) sum += bin(lane * kPer + j);
            const uint64_t inc = wave_inclusive_scan64(sum);
            const uint64_t past = __ballot(before + inc > cap);   // (not empty: there are more than cap)
            if (past != 0ull && lane == __builtin_ctzll(past)) {
                uint64_t b = before + inc - sum;
                int i = lane * kPer;
                for (uint64_t x = bin(i); b + x <= cap; x = bin(++i)) b += x;
                lds64[0] = last | (uint64_t(i) << lo);
                lds64[1] = b;
            }
        }
        __syncthreads();
        last = lds64[0];
        before = lds64[1];
        hi = lo;
    }
    // visit(tile, pair) for the kept pairs of an item; of item `items`, those of the last record that still fit
    auto kept = [&](uint32_t item, auto visit) {
        if (item == items) {   // target by target
            const uint32_t r = uint32_t(last), v = uint32_t(r / uint64_t(R.n_cap));
            const int64_t b = int64_t(r - v * uint64_t(R.n_cap)) / R.chunk;
            uint32_t left = uint32_t(cap - before);
            for (int ti = 0; ti < n_targets && left != 0u; ++ti) {
                const gs_target &t = R.targets[ti];
                if (t.view != int(v)) continue;
                const uint32_t cnt = R.lists.count[ti * R.chunks + b] & kCountMask;
                const int64_t at = ti * R.n_cap + b * R.chunk;
                __syncthreads();
                if (tid == 0) lds64[2] = ~0ull;
                __syncthreads();
                for (uint32_t e = tid; e < cnt; e += kT)
                    if (R.lists.rec[at + e] == r) lds64[2] = e;
                __syncthreads();
                const uint64_t e = lds64[2];
                if (e == ~0ull) continue;
                const uint2 rc = R.lists.rect[at + int64_t(e)], pair = make_uint2(uint32_t(last >> 32), r);
                const uint32_t x0 = rc.x & 0xffffu, w = (rc.x >> 16) - x0 + 1u, take = min(left, rect_area(rc));
                for (uint32_t k = tid; k < take; k += kT)
                    visit(t.tile_offset + ((rc.y & 0xffffu) + k / w) * uint32_t(t.tiles_x) + x0 + k % w, pair);
                left -= take;
            }
            return;
        }
        for (int64_t l = item * per, l1 = min(all_lists, l + per); l < l1; ++l) {
            const int64_t ti = l / R.chunks, at = ti * R.n_cap + l % R.chunks * R.chunk;
            const gs_target &t = R.targets[ti];
            const uint32_t cnt = R.lists.count[l] & kCountMask, first_tile = uint32_t(t.tile_offset);
            for (uint32_t e0 = 0, step = stage_entries(t.tiles_x * t.tiles_y); e0 < cnt; e0 += step) {
                __syncthreads();
                if (tid == 0) lds64[2] = 0;
                __syncthreads();
                for (uint32_t e = e0 + tid; e < min(cnt, e0 + step); e += kT) {
                    const uint32_t r = R.lists.rec[at + e], key = key_of(r);
                    if (rank(key, r) < last) {
                        const uint32_t i = uint32_t(atomicAdd(reinterpret_cast<unsigned long long *>(&lds64[2]), 1ull));
                        srect[i] = R.lists.rect[at + e];
                        sent[i] = make_uint2(key, r);
                    }
                }
                __syncthreads();
                const uint32_t en = uint32_t(lds64[2]);
                if (en != 0u)   // (uniform)
                    share_pairs<kT>(srect, en, uint32_t(t.tiles_x), L, [&](const uint32_t (&t4)[4], const uint32_t (&e4)[4], int m) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (j < m) visit(first_tile + t4[j], sent[e4[j]]);
                    });
            }
        }
    };
    const bool counted = phase(
        kKeepCount, items + 1u, [&](uint32_t item) { kept(item, [&](uint32_t t, uint2) { atomicAdd(&tile[t], 1u); }); }, nothing);
    if (!counted) return;
    const bool started = phase(
        kKeepStarts, 1u,
        [&](uint32_t) {
            uint32_t run = 0u;
            for (int64_t t0 = 0; t0 < total_tiles; t0 += kT) {
                const int64_t t = t0 + tid;
                const uint32_t c = t < total_tiles ? now(&tile[t]) : 0u;
                const uint32_t inc = wave_inclusive_scan(c);
                if (lane == kWave - 1) L.wsum[wave] = inc;
                __syncthreads();
                uint32_t start = run + inc - c;
                for (int w = 0; w < kWaves; ++w) {
                    start += w < wave ? L.wsum[w] : 0u;
                    run += L.wsum[w];
                }
                __syncthreads();
                Longer longer;
                if (t < total_tiles) {
                    longer.range(uint32_t(t), 0, start, c, cap, R.ranges);
                    tile[t] = start;
                }
                longer.publish(uint32_t(t), R.ranges, R.longs, R.long_lists, R.counters);
            }
        },
        nothing);
    if (!started) return;
    phase(kKeepPlace, items + 1u, [&](uint32_t item) {
        kept(item, [&](uint32_t t, uint2 p) {
            const uint32_t at = atomicAdd(&tile[t], 1u);
            if (at < cap) R.pairs[at] = p;
        });
    }, nothing);
}

// Grid (chunks, or more for the large entries, n_targets, workgroups that share a
// target's windows).  kScan (at most kScanTilesMax tiles): total[]
// holds the tile totals, which every workgroup scans itself (workgroup 0 also
// publishes); otherwise it holds the tile starts.
//
// Bound by the writes: a chunk's few pairs of a tile land in as many partial lines.
// The chunks of an XCD fill each other's lines in its L2 while those fit there;
// beyond kStageFrom pairs in all (2 MB an XCD, half of its 4 MB L2, which
// the lists pass through too) lines left half written: 164 MB for 29 MB of pairs
// at 3.66M.  kStaged: the pairs are then placed by tile in LDS first (16 bits each,
// the place of their entry) and written tile by tile, kRunLanes lanes to a run, so
// that the chunks of an XCD write the same lines at about the same time.
// Measured, direct / staged in us (1200x680): 1.3M pairs 17.9 / 18.8; 1.8M 21.7 / 21.2;
// 2.6M 34.4 / 25.6; 5.2M 58.5 / 41.3; runs written by 2 lanes 27.2, by 8 24.9 and by 16
// 30.0 at 2.6M, 46.1, 41.8 and 52.3 at 5.2M.  Several targets are not staged: an XCD
// writes one target at a time, whose eighth fits its L2, and the LDS leaves one
// workgroup a CU (96 targets 670 / 814, 24 targets 125 / 189; now 699 and 132, direct).
constexpr uint32_t kStageFrom = 1u << 21, kStagePairs = 32768;
constexpr int kRunLanes = 4;
// With more chunks than CUs two workgroups without the staging's LDS share a CU, and
// with it take turns, so it is left out where the tiles are too few for so many pairs:
// 2M Gaussians over 260 tiles 13.9 us without, 19.2 with; 1,200 tiles 23.5 / 29.0;
// 3,225 tiles 58.5 / 41.3; 4M over 3,225 110 / 78.
constexpr int kStageTiles = 2048;
// (eight waves a SIMD: without the hint the overflow's part takes more than 100 SGPRs,
// two workgroups of 1,024 no longer share a CU, and 96 targets take 724 us for 672)
template <int kT, bool kScan, bool kStaged>
__global__ void __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(kStaged ? 4 : kT == kBinThreadsMany ? 8 : 5))) bin_scatter_kernel(
    const ScatterArgs A) {
    extern __shared__ uint32_t slot[];   // next slot of every tile of the window
    static_assert(kScan || !kStaged, "the pair count is known to the scan");
    __shared__ uint2 srect[kBinStage];
    __shared__ uint2 sent[kStaged ? kBinChunkMax : kBinStage];
    __shared__ BinStage<kT> L;
    __shared__ uint64_t lds64[kT / kWave];
    __shared__ uint32_t ends[kStaged ? kScanTilesMax : 1];    // a tile's place in staged: starts that advance to the ends
    __shared__ uint16_t staged[kStaged ? kStagePairs : 1];    // entries of the chunk's pairs, tile by tile
    __shared__ uint32_t s_en, cursor[kWave];
    __shared__ LargeState state;
    const int tid = threadIdx.x;
    // consecutive chunks to one XCD: their slots of a tile meet in the same
    // lines, which then fill up in one L2
    const int ti = blockIdx.y;
    const bool own = blockIdx.x < xcd_grid(A.chunks) && xcd_tile(blockIdx.x, A.chunks) < A.chunks;   // uniform
    const int64_t b = own ? xcd_tile(blockIdx.x, A.chunks) : 0;
    const uint32_t large = A.counters[kLarge];   // whether a chunk has large entries
    if (!own && large == 0u) return;   // uniform
    const uint32_t found = kScan ? 0u : A.counters[kPairs];   // (loaded beside the others, not after them)
    const gs_target t = A.targets[ti];
    const int tiles = t.tiles_x * t.tiles_y;
    const uint32_t word = A.lists.count[int64_t(ti) * A.chunks + b], cnt = word & kCountMask, limit = word >> kCountBits;
    const int64_t lbase = int64_t(ti) * A.n_cap + b * A.chunk;
    const uint32_t *row = A.thist + b * A.stride + t.tile_offset;
    const bool publisher = own && b == 0 && ti == 0;
    bool stage = false, over;   // uniform
    if (kScan) {   // (the window holds every tile of the target)
        Longer longer;
        const uint64_t all = scan_totals<kT>(A.total, A.total_tiles, lds64, [&](int j, int64_t g, uint64_t pre, uint32_t count) {
            if (publisher && g < A.total_tiles) longer.range(uint32_t(tid) * (kScanTilesMax / kT), j, pre, count, A.cap, A.ranges);
            const int64_t i = g - t.tile_offset;
            if (i >= 0 && i < tiles) slot[i] = uint32_t(pre < kSatSlot ? pre : kSatSlot);
        });
        longer.publish(uint32_t(tid) * (kScanTilesMax / kT), A.ranges, A.longs, A.long_lists, A.counters);
        if (publisher && tid == 0) publish_pairs(all, A.cap, A.counters, A.d_status);
        stage = kStaged && all > kStageFrom;
        over = all > A.cap;
        __syncthreads();
    } else {
        over = found > A.cap;
    }
    if (over) {   // the last workgroups with a chunk to get here keep the first pairs of the call
        if (!own) return;   // uniform
        const ScatterArgs &R = args_again();
        __threadfence();   // (their counts and ranges replace the publisher's)
        __syncthreads();
        if (tid == 0) lds64[0] = atomicAdd(&R.counters[kArrived], 1u);
        __syncthreads();
        const uint64_t before = lds64[0], all = uint64_t(R.chunks) * gridDim.y * gridDim.z;
        if (before + kCrew < all) return;   // uniform
        // (their counts by tile in the first row: a workgroup without a chunk may still sum the totals)
        keep_first_pairs<kT>(R, int(gridDim.y), before + 1 == all, srect, sent, L, lds64);
        return;
    }
    if (own && cnt != 0) {   // uniform
        if (kStaged && stage) {   // the chunk's counts, from its row of prefixes and the next
            constexpr int kPer = kScanTilesMax / kT;
            const uint32_t *next = b + 1 < A.chunks ? row + A.stride : A.total + t.tile_offset;
            uint32_t v[kPer], s = 0u;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const int i = tid * kPer + j;
                v[j] = i < tiles ? next[i] - row[i] : 0u;
                s += v[j];
            }
            const int wave = tid / kWave;
            const uint32_t inc = wave_inclusive_scan(s);
            if (lane_id() == kWave - 1) L.wsum[wave] = inc;
            __syncthreads();
            uint32_t pre = inc - s, all = 0u;
#pragma unroll
            for (int w = 0; w < kT / kWave; ++w) {
                const uint32_t x = L.wsum[w];
                pre += w < wave ? x : 0u;
                all += x;
            }
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                ends[tid * kPer + j] = pre;
                pre += v[j];
            }
            stage = all <= kStagePairs;   // (more: near Gaussians over many tiles, whose runs are long)
            __syncthreads();
        }
        for (uint32_t w = kScan ? 0u : blockIdx.z * A.window; w < uint32_t(tiles); w += gridDim.z * A.window) {
            const int w0 = int(w), wn = min(A.window, tiles - w0);
            for (int i = tid; i < wn; i += kT) {
                const uint64_t a = uint64_t(kScan ? slot[i] : A.total[t.tile_offset + w0 + i]) + row[w0 + i];
                slot[i] = uint32_t(a < kSatSlot ? a : kSatSlot);
            }
            const uint32_t step = stage_entries(tiles);
            for (uint32_t e0 = 0; e0 < cnt; e0 += step) {
                const uint32_t at0 = kStaged && stage ? e0 : 0u;
                uint32_t en = min(cnt - e0, step);
                if ((!kScan && tiles > A.window) || limit != 0u) {   // the entries' parts in the window (uniform)
                    const TileSpan span = tile_span(w0, wn, uint32_t(t.tiles_x));
                    if (tid == 0) s_en = 0u;
                    __syncthreads();
                    for (uint32_t i0 = 0; i0 < en; i0 += kT) {   // (whole waves take part)
                        uint2 rc = make_uint2(0u, 0u);
                        const bool in = i0 + tid < en && !is_large(rc = A.lists.rect[lbase + e0 + i0 + tid], limit) &&
                                        clip_rect(rc, span);
                        const uint32_t at = append(in, &s_en);
                        if (in) {
                            const uint32_t r = A.lists.rec[lbase + e0 + i0 + tid];
                            srect[at] = rc;
                            sent[at0 + at] = make_uint2(depth_key(A.proj.rgb_z[r].w, A.znear), r);
                        }
                    }
                    __syncthreads();
                    en = s_en;
                } else {
                    for (uint32_t e = tid; e < en; e += kT) {
                        const uint32_t r = A.lists.rec[lbase + e0 + e];
                        srect[e] = A.lists.rect[lbase + e0 + e];
                        sent[at0 + e] = make_uint2(depth_key(A.proj.rgb_z[r].w, A.znear), r);
                    }
                    __syncthreads();
                }
                if (kStaged && stage) {
                    share_pairs<kT>(srect, en, uint32_t(t.tiles_x), L,
                                    [&](const uint32_t (&tile)[4], const uint32_t (&entry)[4], int mm) {
                                        uint32_t at[4];
#pragma unroll
                                        for (int j = 0; j < 4; ++j)
                                            at[j] = j < mm ? atomicAdd(&ends[tile[j]], 1u) : kStagePairs;
#pragma unroll
                                        for (int j = 0; j < 4; ++j)
                                            if (at[j] < kStagePairs) staged[at[j]] = uint16_t(e0 + entry[j]);
                                    });
                    continue;
                }
                share_pairs<kT>(srect, en, uint32_t(t.tiles_x), L,
                                [&](const uint32_t (&tile)[4], const uint32_t (&entry)[4], int mm) {
                                    uint32_t at[4];   // (four ranks in flight)
#pragma unroll
                                    for (int j = 0; j < 4; ++j) {
                                        const uint32_t i = tile[j] - uint32_t(w0);
                                        at[j] = j < mm && i < uint32_t(wn) ? atomicAdd(&slot[i], 1u) : 0xffffffffu;
                                    }
#pragma unroll
                                    for (int j = 0; j < 4; ++j)
                                        if (at[j] < A.cap) A.pairs[at[j]] = sent[entry[j]];
                                });
            }
            __syncthreads();   // the next window reuses slot
        }
        if (kStaged && stage)
            for (int i = tid / kRunLanes; i < tiles; i += kT / kRunLanes) {
                const uint32_t s0 = i > 0 ? ends[i - 1] : 0u, m = ends[i] - s0, at = slot[i];
                for (uint32_t k = tid % kRunLanes; k < m; k += kRunLanes)
                    if (at + k < A.cap) A.pairs[at + k] = sent[staged[s0 + k]];
            }
    }
    if (large == 0u) return;   // uniform
    // The large entries, tiles 64 at a time, a wave to a tile, from its start on.
    const ScatterArgs &R = args_again();
    __syncthreads();
    if (kScan) {   // (the slots are used up)
        scan_totals<kT>(R.total, R.total_tiles, lds64, [&](int, int64_t g, uint64_t pre, uint32_t) {
            const int64_t i = g - t.tile_offset;
            if (i >= 0 && i < tiles) slot[i] = uint32_t(pre < kSatSlot ? pre : kSatSlot);
        });
    }
    const uint32_t tx = uint32_t(t.tiles_x);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = lane_id();
    for (int64_t i0 = (int64_t(gridDim.x) * blockIdx.z + blockIdx.x) * kWave; i0 < tiles;
         i0 += int64_t(gridDim.x) * gridDim.z * kWave) {
        const int a = int(i0), m = min(kWave, tiles - a);
        __syncthreads();
        if (tid < m) cursor[tid] = kScan ? slot[a + tid] : R.total[t.tile_offset + a + tid];
        large_entries<kT, kBinStage>(
            R.lists.count + int64_t(ti) * R.chunks, R.chunks, R.chunk, R.lists.rect + int64_t(ti) * R.n_cap,
            tile_span(a, m, tx), L.off, state,
            [&](uint32_t to, uint2 rc, int64_t e) {
                const uint32_t r = R.lists.rec[int64_t(ti) * R.n_cap + e];
                srect[to] = rc;
                sent[to] = make_uint2(depth_key(R.proj.rgb_z[r].w, R.znear), r);
            },
            [&](uint32_t held) {
                for (int i = wave; i < m; i += kT / kWave) {
                    const uint32_t y = uint32_t(a + i) / tx, x = uint32_t(a + i) - y * tx;
                    uint32_t at = cursor[i];
                    for (uint32_t e0 = 0; e0 < held; e0 += kWave) {
                        const uint32_t e = e0 + lane;
                        const uint2 rc = e < held ? srect[e] : make_uint2(1u, 1u);   // (empty)
                        const bool in = x >= (rc.x & 0xffffu) && x <= rc.x >> 16 && y >= (rc.y & 0xffffu) && y <= rc.y >> 16;
                        const uint64_t mask = __ballot(in);
                        const uint32_t to = at + uint32_t(mask_rank(mask));
                        if (in && to < R.cap) R.pairs[to] = sent[e];
                        at += uint32_t(__popcll(mask));
                    }
                    if (lane == 0) cursor[i] = at;
                }
            });
    }
}

__device__ __forceinline__ bool pair_less(uint2 a, uint2 b) { return a.x < b.x || (a.x == b.x && a.y < b.y); }

// Bitonic sort of p[0, n) in LDS by (key, record), padded to a power of two
// with the largest pair (capacity kCap).
template <int kThreads>
__device__ void bitonic_sort(uint2 *p, int n, int tid) {
    int m = 2;
    while (m < n) m <<= 1;
    for (int i = n + tid; i < m; i += kThreads) p[i] = make_uint2(0xffffffffu, 0xffffffffu);
    for (int size = 2; size <= m; size <<= 1)
        for (int d = size >> 1; d > 0; d >>= 1) {
            __syncthreads();
            for (int k = tid; k < m / 2; k += kThreads) {
                const int i = 2 * k - (k & (d - 1)), j = i + d;
                const uint2 a = p[i], b = p[j];
                if (pair_less(b, a) == ((i & size) == 0)) { p[i] = b; p[j] = a; }
            }
        }
    __syncthreads();
}

// Sorts p[0, n) of LDS, where ranking in equal parts of the depth range met crowds: by
// kSplits splitters out of a sorted sample (p is in the order of those parts, so an even
// sample is a fair one), into the places of which the pairs are dealt, to be ranked
// there.  work: 3 * kSplits + 1 words of LDS.  8,192 pairs: 20 us, bitonic 90.
constexpr int kSplits = 512;
template <int kThreads, int kCap, class Put>
__device__ __forceinline__ void split_sort(uint2 *p, int n, uint32_t *work, uint32_t *wsum, Put put) {
    constexpr int kItems = kCap / kThreads, kWaves = kThreads / kWave;
    static_assert(kThreads >= kSplits, "a thread per splitter");
    const int tid = threadIdx.x, wave = tid / kWave;
    uint2 *split = reinterpret_cast<uint2 *>(work);
    uint32_t *start = work + 2 * kSplits;
    if (tid < kSplits) {
        split[tid] = p[int(int64_t(n) * tid / kSplits)];
        start[tid + 1] = 0u;
    }
    if (tid == 0) start[0] = 0u;
    bitonic_sort<kThreads>(split, kSplits, tid);
    uint2 q[kItems];
    uint32_t part[kItems], at[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = tid + k * kThreads;
        if (i >= n) continue;
        q[k] = p[i];
        uint32_t lo = 0u;   // the splitters up to it (the last one aside)
#pragma unroll
        for (uint32_t step = kSplits / 2; step > 0; step >>= 1) lo += pair_less(q[k], split[lo + step - 1]) ? 0u : step;
        part[k] = lo;
        at[k] = atomicAdd(&start[lo + 1], 1u);
    }
    __syncthreads();
    uint32_t inc = 0u;   // counts -> starts
    if (tid < kSplits) {
        inc = wave_inclusive_scan(start[tid + 1]);
        if (lane_id() == kWave - 1) wsum[wave] = inc;
    }
    __syncthreads();
    if (tid < kSplits) {
        for (int w = 0; w < wave; ++w) inc += wsum[w];
        start[tid + 1] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        if (tid + k * kThreads < n) p[start[part[k]] + at[k]] = q[k];
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < kItems; ++k) {
        const int i = tid + k * kThreads;
        if (i >= n) break;
        const uint2 a = p[i];
        uint32_t lo = 0u;
        for (uint32_t step = kSplits / 2; step > 0; step >>= 1) lo += pair_less(a, split[lo + step - 1]) ? 0u : step;
        const uint32_t s = start[lo], e = start[lo + 1];
        uint32_t rank = s;
        for (uint32_t j = s; j < e; ++j) rank += pair_less(p[j], a) ? 1u : 0u;
        put(int(rank), a);
    }
}

// One workgroup's sort of at most kCap pairs get(0 .. n - 1) by (key, record);
// the sorted pairs are handed to put(i, pair), after every pair has been read.
//
// The depths of a tile spread over its range, so they are dealt into kCap
// buckets in proportion to their place in it (about one pair each), and a pair's
// place is the start of its bucket plus the pairs of the bucket that are
// smaller.  Where a bucket holds more than kCrowd pairs (equal depths, as on a
// plane facing the camera, or a few far off that stretch the range), the workgroup
// runs a bitonic sort instead, or (kDense) split_sort where there are many.
constexpr int kCrowd = 24;
template <int kThreads, int kCap>
struct SortLds {
    uint2 pair[kCap];
    uint32_t start[kCap + 1];
    uint32_t wsum[kThreads / kWave], lo[kThreads / kWave], hi[kThreads / kWave], rlo[kThreads / kWave], rhi[kThreads / kWave];
    uint32_t crowded;
};
template <bool kDense, int kThreads, int kCap, class Get, class Put>
__device__ __forceinline__ void sort_in_lds(int n, SortLds<kThreads, kCap> &L, Get get, Put put) {
    constexpr int kItems = kCap / kThreads, kWaves = kThreads / kWave;
    const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
    uint2 p[kItems];
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = tid + k * kThreads;
        p[k] = make_uint2(0u, 0u);
        if (i < n) {
            p[k] = get(i);
            lo = min(lo, p[k].x);
            hi = max(hi, p[k].x);
        }
    }
#pragma unroll
    for (int k = 0; k < kItems; k += 4)
        *reinterpret_cast<uint4 *>(&L.start[tid * kItems + k]) = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        lo = min(lo, uint32_t(__shfl_xor(int(lo), d, kWave)));
        hi = max(hi, uint32_t(__shfl_xor(int(hi), d, kWave)));
    }
    if (lane == 0) { L.lo[wave] = lo; L.hi[wave] = hi; }
    if (tid == 0) L.crowded = 0u;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        lo = min(lo, L.lo[w]);
        hi = max(hi, L.hi[w]);
    }
    // Bucket of a pair: monotone in its key (each conversion and product is).  kDense: many
    // pairs may share few depths; the record, as a fraction below one, tells those
    // apart (below 2^24 a key is exact and the sum below the next one; beyond,
    // the sum rounds to the key).
    const float scale = float(kCap - 1) / (float(hi - lo) + 1.f);
    const bool records = kDense && hi - lo < 8u * kCap;   // (uniform)
    uint32_t rlo = 0xffffffffu, rhi = 0u;
    if (records) {
#pragma unroll
        for (int k = 0; k < kItems; ++k)
            if (tid + k * kThreads < n) {
                rlo = min(rlo, p[k].y);
                rhi = max(rhi, p[k].y);
            }
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) {
            rlo = min(rlo, uint32_t(__shfl_xor(int(rlo), d, kWave)));
            rhi = max(rhi, uint32_t(__shfl_xor(int(rhi), d, kWave)));
        }
        if (lane == 0) { L.rlo[wave] = rlo; L.rhi[wave] = rhi; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            rlo = min(rlo, L.rlo[w]);
            rhi = max(rhi, L.rhi[w]);
        }
    }
    const float part = 0.99999f / (float(rhi - rlo) + 1.f);
    auto bucket = [&](uint2 q) {
        float x = float(q.x - lo);
        if (records) x += float(q.y - rlo) * part;
        return min(int(x * scale), kCap - 1);
    };
    uint32_t at[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        if (tid + k * kThreads < n) at[k] = atomicAdd(&L.start[bucket(p[k])], 1u);
    __syncthreads();
    {   // counts -> starts
        uint32_t c[kItems], sum = 0u, most = 0u;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            c[k] = L.start[tid * kItems + k];
            sum += c[k];
            most = max(most, c[k]);
        }
        if (most > uint32_t(kCrowd)) L.crowded = 1u;
        const uint32_t inc = wave_inclusive_scan(sum);
        if (lane == kWave - 1) L.wsum[wave] = inc;
        __syncthreads();
        uint32_t pre = inc - sum;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) pre += w < wave ? L.wsum[w] : 0u;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            L.start[tid * kItems + k] = pre;
            pre += c[k];
        }
        if (tid == 0) L.start[kCap] = uint32_t(n);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        if (tid + k * kThreads < n) L.pair[L.start[bucket(p[k])] + at[k]] = p[k];
    __syncthreads();
    if (L.crowded) {   // uniform
        if constexpr (kDense) {
            if (n > 2 * kSplits) {
                split_sort<kThreads, kCap>(L.pair, n, L.start, L.wsum, put);
                return;
            }
        }
        bitonic_sort<kThreads>(L.pair, n, tid);
        for (int i = tid; i < n; i += kThreads) put(i, L.pair[i]);
        return;
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = tid + k * kThreads;
        if (i < n) {
            const uint2 a = L.pair[i];
            const int b = bucket(a);
            const uint32_t s = L.start[b], e = L.start[b + 1];
            uint32_t rank = s;
            for (uint32_t j = s; j < e; ++j) rank += pair_less(L.pair[j], a) ? 1u : 0u;
            put(int(rank), a);
        }
    }
}

// Lists of up to kSortSmall pairs, kGroup tiles to a workgroup: each list by the whole
// workgroup in LDS, or, of several tiles, those of up to 64 pairs by a wave each, which
// ranks its pairs against one another in registers.
template <int kGroup>
__global__ void __launch_bounds__(kSortThreads) tile_order_small_kernel(const uint2 *__restrict__ ranges,
                                                                        const uint2 *__restrict__ pairs,
                                                                        uint32_t *__restrict__ out, int64_t tiles) {
    static_assert(kGroup == 1 || kGroup == kSortThreads / kWave, "a tile to a wave");
    __shared__ __attribute__((aligned(16))) SortLds<kSortThreads, kSortSmall> L;
    if (kGroup > 1) {
        const int64_t t = int64_t(blockIdx.x) * kGroup + __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
        const uint2 range = t < tiles ? ranges[t] : make_uint2(0u, 0u);
        const int n = __builtin_amdgcn_readfirstlane(int(range.y - range.x)), lane = lane_id();
        if (n > 0 && n <= kWave) {
            const uint2 p = lane < n ? pairs[range.x + lane] : make_uint2(0xffffffffu, 0xffffffffu);
            uint32_t rank = 0u;
            for (int j = 0; j < n; ++j)
                rank += pair_less(make_uint2(uint32_t(__builtin_amdgcn_readlane(int(p.x), j)),
                                             uint32_t(__builtin_amdgcn_readlane(int(p.y), j))), p) ? 1u : 0u;
            if (lane < n) out[range.x + rank] = p.y;
        }
    }
#pragma unroll 1
    for (int k = 0; k < kGroup; ++k) {
        const int64_t t = int64_t(blockIdx.x) * kGroup + k;
        if (kGroup > 1 && t >= tiles) return;   // uniform
        const uint2 range = ranges[t];
        const int n = int(range.y - range.x);
        if (n <= (kGroup > 1 ? kWave : 0) || n > kSortSmall) continue;   // uniform
        if (kGroup > 1) __syncthreads();   // the list before
        sort_in_lds<false, kSortThreads, kSortSmall>(
            n, L, [&](int i) { return pairs[range.x + i]; }, [&](int i, uint2 p) { out[range.x + i] = p.y; });
    }
}

// The longer lists, by a fixed grid.  Up to kSortLarge pairs: one workgroup each, in
// LDS.  Up to kSortAlone: one workgroup each, which deals them into buckets by the leading
// bits of their keys, from `pairs` into (key1, val1), and sorts runs of whole buckets.
// Longer ones by a sample sort over many workgroups:
//   count - the pairs are counted by run: the runs, of kRunTarget pairs or so, lie between
//           splitters out of a sorted sample of the list (kPerRun samples a run), by
//           (key, record), so that equal depths are cut too;
//   deal  - the pairs go from `pairs` to their runs' places in (key1, val1);
//   runs  - a run is sorted in LDS.
// The records end in val1.  A run or bucket of more than kSortLarge pairs (a poor sample,
// or depths within 2^-9 of each other) is merge sorted by its workgroup: stretches of
// kSortLarge sorted in LDS, then merged in pairs, doubling, by the threads in
// equal shares of the output (the split of each share found by bisection), back and forth
// between `pairs` and (key1, val1).
// The sample sort's slices of kSortLarge pairs (whose workgroups draw the same sample) and
// runs are items taken from counters.  A phase begins when the items of the one before
// are done: the workgroup that ends the last of them goes on at once, and the others wait
// for it kWaits rounds (milliseconds) at most and then leave the rest to those that are
// there, so the launch ends whichever workgroups run at the same time.
// Bound: the latency of its phases, 15 to 25 us each.  Binning of 1M Gaussians at 1200x680 in
// us, one workgroup per list of any length over buckets of leading key bits / sorting
// the records first / this: all within 40 pixels (nine tiles) 554 / 169 / 141, in one tile 17,281 / 174 / 158,
// in two at equal depths 41,815 / 158 / 155; half of them in two tiles and half spread 4,578 / 171 / 182;
// spread, over pyramid levels 0 to 4 636 / 291 / 324, 0 to 6 2,934 / 363 / 416; 2M at level 2 (lists of
// 11,300, up to 20,200) 144 / 237 / 145.  Lists that fit, taken where they were dealt out to 512
// workgroups before: 4,000 of 32 keyframes 137 / - / 119, 908 of 2M Gaussians 25.0 / - / 27.1.
constexpr int kPerRun = kSortLarge / kRunsMax;
using LargeLds = SortLds<kSortLargeThreads, kSortLarge>;
__shared__ __attribute__((aligned(16))) LargeLds s_large;   // (of tile_order_large_kernel)
__shared__ uint2 s_split[kRunsMax];                         // first pair of the next run

// An argument of a function that is not inlined, back in scalar registers (all lanes pass
// the same).
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return uint32_t(__builtin_amdgcn_readfirstlane(int(x))); }
template <typename T>
__device__ __forceinline__ T *uniform(T *p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<T *>((uint64_t(uniform(uint32_t(a >> 32))) << 32) | uniform(uint32_t(a)));
}

// (A list that fits is sorted in place in the kernel, without what dense ones need: 2,000 to
// 3,000 pairs 6.2 us, by this 7.7.)
// Sorts n <= kSortLarge pairs: of A, or of (K, V) without it, to `to` or, the records, to
// `records`; or n samples of A's `from` pairs, to the splitters.  Not inlined: its
// registers, five times over, left the kernel spilling.
__device__ __attribute__((noinline)) void sort_large(uint32_t n, const uint2 *A, const uint32_t *K, const uint32_t *V,
                                                     uint32_t from, uint2 *to, uint32_t *records) {
    n = uniform(n), from = uniform(from);
    A = uniform(A), K = uniform(K), V = uniform(V), to = uniform(to), records = uniform(records);
#ifdef __HIP_DEVICE_COMPILE__   // (all in global memory, which a function that is not inlined cannot see)
    auto global = [](const void *p) { __builtin_assume(!__builtin_amdgcn_is_shared(p) && !__builtin_amdgcn_is_private(p)); };
    global(A), global(K), global(V), global(to), global(records);
#endif
    const float stretch = float(from) / float(n);
    __syncthreads();   // s_large is reused
    sort_in_lds<true, kSortLargeThreads, kSortLarge>(
        int(n), s_large,
        [&](int i) {
            if (A == nullptr) return make_uint2(K[i], V[i]);
            if (from == 0u) return A[i];
            // one of the i-th of n equal stretches, by a multiplicative hash (with integer
            // divisions the sort is 50 KB of code, whose fetch takes 5 us)
            const uint32_t a = uint32_t(float(i) * stretch), b = uint32_t(float(i + 1) * stretch);
            return A[min(a + __umulhi(uint32_t(i + 1) * 2654435761u, b - a), from - 1u)];
        },
        [&](int i, uint2 p) {
            if (records != nullptr) records[i] = p.y;
            else if (to != nullptr) to[i] = p;
            else if (i % kPerRun == 0 && i > 0) s_split[i / kPerRun - 1] = p;
        });
}

// Sorts the n pairs of A; the records end in V.
__device__ __attribute__((noinline)) void merge_sort(uint2 *A, uint32_t *K, uint32_t *V, uint32_t n) {
    constexpr int kT = kSortLargeThreads;
    const int tid = threadIdx.x;
    n = uniform(n);
    A = uniform(A), K = uniform(K), V = uniform(V);
    for (uint32_t c = 0; c < n; c += kSortLarge)
        sort_large(min(n - c, uint32_t(kSortLarge)), A + c, nullptr, nullptr, 0u, A + c, nullptr);
    __syncthreads();
    bool in_a = true;   // the sorted runs are in A, else in (K, V)
    auto load = [&](uint32_t i) { return in_a ? A[i] : make_uint2(K[i], V[i]); };
    for (uint64_t run = kSortLarge; run < n; run <<= 1) {
        const uint32_t per = (n + kT - 1) / kT;
        uint32_t o = min(n, tid * per);
        const uint32_t o1 = min(n, o + per);
        while (o < o1) {   // the share's piece of each pair of runs it meets
            const uint32_t r0 = uint32_t(o / (2 * run) * (2 * run));
            const uint32_t ra = uint32_t(min(uint64_t(n), r0 + run)), rb = uint32_t(min(uint64_t(n), r0 + 2 * run));
            const uint32_t na = ra - r0, nb = rb - ra, d = o - r0, end = min(o1, rb);
            // the first d outputs take lo of the first run and d - lo of the second
            uint32_t lo = d > nb ? d - nb : 0u, hi = min(d, na);
            while (lo < hi) {
                const uint32_t mid = (lo + hi) / 2;
                if (pair_less(load(r0 + mid), load(ra + d - 1 - mid))) lo = mid + 1; else hi = mid;
            }
            uint32_t i = r0 + lo, j = ra + d - lo;
            for (; o < end; ++o) {
                const bool first = i < ra && (j >= rb || pair_less(load(i), load(j)));
                const uint2 p = load(first ? i : j);
                if (first) ++i; else ++j;
                if (in_a) { K[o] = p.x; V[o] = p.y; } else { A[o] = p; }
            }
        }
        __syncthreads();
        in_a = !in_a;
    }
    if (in_a)
        for (uint32_t i = tid; i < n; i += kT) V[i] = A[i].y;
    __syncthreads();
}

// The m pairs of a run, dealt to (K, V); the records end in V.  A: as many pairs of space.
__device__ __forceinline__ void sort_run(uint2 *A, uint32_t *K, uint32_t *V, uint32_t m) {
    if (m <= uint32_t(kSortLarge)) {
        if (m != 0u) sort_large(m, nullptr, K, V, 0u, nullptr, V);
        return;
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < m; i += kSortLargeThreads) A[i] = make_uint2(K[i], V[i]);
    merge_sort(A, K, V, m);
}

__global__ void __launch_bounds__(kSortLargeThreads) tile_order_large_kernel(
    uint32_t *counters, const uint32_t *__restrict__ longs, const uint2 *__restrict__ ranges, LongLists lists, uint2 *pairs,
    uint32_t *key1, uint32_t *val1) {
    constexpr int kT = kSortLargeThreads, kPer = kSortLarge / kT;
    static_assert(kRunsMax == 256 && kT == 4 * kRunsMax, "four threads a run sum the slices' counts");
    __shared__ uint32_t cursor[kRunsMax], total[kRunsMax], starts[kRunsMax + 1];
    constexpr int kKeyShift = kDepthKeyBits - 13;
    static_assert(kSortLarge == 1 << 13, "a bucket per value of the leading key bits");
    __shared__ uint32_t ends[kSortLarge];   // end of each bucket
    __shared__ uint32_t s_item;
    __shared__ uint4 s_list;
    const uint32_t n_long = counters[kLongTiles];
    const uint64_t packed = *reinterpret_cast<const uint64_t *>(counters + kLongLists);
    if (n_long == 0u && packed == 0u) return;   // uniform
    constexpr uint32_t kNone = 0xffffffffu;   // (of a pair past every other)
    constexpr uint32_t kMask = (1u << kPackBits) - 1u;
    const uint32_t n_lists = uint32_t(packed) & kMask, slices = uint32_t(packed >> kPackBits) & kMask,
                   runs = uint32_t(packed >> (2 * kPackBits));
    const int tid = threadIdx.x, wave = tid / kWave;
    auto run_of = [&](uint2 p) {   // the number of splitters up to p
        uint32_t q = 0u;
#pragma unroll
        for (uint32_t step = kRunsMax / 2; step > 0; step >>= 1) q += pair_less(p, s_split[q + step - 1]) ? 0u : step;
        return q;
    };
    // this thread's kPer pairs from A[first] on ((kNone, kNone) past the end)
    auto load_slice = [&](const uint2 *A, uint32_t first, uint32_t n, uint2 (&p)[kPer]) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t i = first + tid + j * kT;
            p[j] = A[min(i, n - 1u)];
            if (i >= n) p[j] = make_uint2(kNone, kNone);
        }
    };
    auto sample = [&](const uint2 *A, uint32_t n, uint32_t runs) {
        __syncthreads();
        if (tid < kRunsMax) s_split[tid] = make_uint2(kNone, kNone);
        sort_large(runs * kPerRun, A, nullptr, nullptr, n, nullptr, nullptr);   // (fewer samples than pairs)
        __syncthreads();
    };
    auto count_slice = [&](const uint2 *A, uint32_t first, uint32_t n) {
        uint2 p[kPer];
        load_slice(A, first, n, p);
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (p[j].x != kNone) atomicAdd(&total[run_of(p[j])], 1u);
    };
    auto scan_runs = [&] {   // starts[] of total[]
        uint32_t inc = 0u;
        if (tid < kRunsMax) {
            inc = wave_inclusive_scan(total[tid]);
            if (lane_id() == kWave - 1) s_large.wsum[wave] = inc;
        }
        __syncthreads();
        if (tid < kRunsMax) {
            for (int w = 0; w < wave; ++w) inc += s_large.wsum[w];
            starts[tid + 1] = inc;
        }
        if (tid == 0) starts[0] = 0u;
        __syncthreads();
    };
    auto deal_slice = [&](const uint2 *A, uint32_t first, uint32_t n, uint32_t *K, uint32_t *V) {
        uint2 p[kPer];
        load_slice(A, first, n, p);
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (p[j].x != kNone) {
                const uint32_t at = atomicAdd(&cursor[run_of(p[j])], 1u);
                K[at] = p[j].x;
                V[at] = p[j].y;
            }
    };
    // The list of a slice or run: its number, and in s_list tile, pairs, first slice, first
    // run (the lists' slices, and their runs, follow each other in the lists' order).
    auto find = [&](uint32_t item, bool by_run) {
        __syncthreads();
        for (uint32_t e = tid; e < n_lists; e += kT) {
            const uint4 l = lists.list[e];
            const uint32_t at = item - (by_run ? l.w : l.z);
            if (at < (by_run ? Longer::runs(l.y) : Longer::slices(l.y))) {
                s_list = l;
                s_item = e;
            }
        }
        __syncthreads();
        return s_item;
    };
    auto take = [&](int next) {
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(&counters[next], 1u);
        __syncthreads();
        return s_item;
    };
    // work(item) for items taken from a counter, each while the one before is worked on;
    // returns how many.
    auto each_item = [&](int next, uint32_t items, auto work) {
        uint32_t did = 0u;
        for (uint32_t item = take(next); item < items; ++did) {
            uint32_t ahead = 0u;
            if (tid == 0) ahead = atomicAdd(&counters[next], 1u);
            work(item);
            __syncthreads();
            if (tid == 0) s_item = ahead;
            __syncthreads();
            item = s_item;
        }
        return did;
    };
    // `did` items more are done; their writes are visible to who sees the count.  One fence
    // a workgroup: it writes back an L2 (one per wave and item took 400 us of a call), once
    // all waves' stores have reached it.
    auto ended = [&](int done, uint32_t did) {
        stores_reached();
        __syncthreads();
        if (did != 0u && tid == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            atomicAdd(&counters[done], did);
        }
    };
    auto wait_for = [&](int done) {   // whether all slices are done
        __syncthreads();
        if (tid == 0) {
            auto now = [&] { return __hip_atomic_load(&counters[done], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            for (int i = 0; i < kWaits && now() < slices; ++i) __builtin_amdgcn_s_sleep(16);
            s_item = now() >= slices;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        return s_item != 0u;
    };

    auto sort_alone = [&](uint2 range) {   // a list of up to kSortAlone pairs
        const uint32_t n = range.y - range.x;
        uint2 *A = pairs + range.x;
        uint32_t *K = key1 + range.x, *V = val1 + range.x;
        if (n <= uint32_t(kSortLarge)) {
            __syncthreads();   // s_large is reused
            sort_in_lds<false, kT, kSortLarge>(int(n), s_large, [&](int i) { return A[i]; }, [&](int i, uint2 p) { V[i] = p.y; });
            return;
        }
        // dealt into kSortLarge buckets by the leading bits of the keys, and runs of whole
        // buckets of up to kSortLarge pairs sorted
        __syncthreads();
        for (int i = tid; i < kSortLarge; i += kT) ends[i] = 0u;
        __syncthreads();
        auto bucket = [&](uint32_t key) { return min(key >> kKeyShift, uint32_t(kSortLarge - 1)); };
        for (uint32_t i0 = 0; i0 < n; i0 += kSortLarge) {
            uint2 p[kPer];
            load_slice(A, i0, n, p);
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (p[j].x != kNone) atomicAdd(&ends[bucket(p[j].x)], 1u);
        }
        __syncthreads();
        {   // counts -> starts
            uint32_t c[kPer], sum = 0u;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                c[j] = ends[tid * kPer + j];
                sum += c[j];
            }
            const uint32_t inc = wave_inclusive_scan(sum);
            if (lane_id() == kWave - 1) s_large.wsum[wave] = inc;
            __syncthreads();
            uint32_t pre = inc - sum;
#pragma unroll
            for (int w = 0; w < kT / kWave; ++w) pre += w < wave ? s_large.wsum[w] : 0u;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                ends[tid * kPer + j] = pre;
                pre += c[j];
            }
        }
        __syncthreads();
        for (uint32_t i0 = 0; i0 < n; i0 += kSortLarge) {   // the starts advance to the ends
            uint2 p[kPer];
            load_slice(A, i0, n, p);
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (p[j].x != kNone) {
                    const uint32_t at = atomicAdd(&ends[bucket(p[j].x)], 1u);
                    K[at] = p[j].x;
                    V[at] = p[j].y;
                }
        }
        __syncthreads();
        for (uint32_t g = 0; g < n;) {   // (uniform)
            // the buckets that end by g + kSortLarge, or else the next one alone
            auto first_past = [&](uint32_t limit) {
                uint32_t lo = 0u, hi = kSortLarge;   // the first bucket that ends past limit
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) / 2u;
                    if (ends[mid] > limit) hi = mid; else lo = mid + 1u;
                }
                return lo;
            };
            const uint32_t b = first_past(g + kSortLarge);
            uint32_t to = b > 0u ? ends[b - 1u] : 0u;
            if (to <= g) to = ends[first_past(g)];
            sort_run(A + g, K + g, V + g, to - g);
            g = to;
        }
    };

    // Consecutive slices (of one list mostly, which is sampled once) to a workgroup.  They are
    // taken, not given, as nobody may wait for a workgroup that has not begun, beside other
    // launches or among more of them than fit (512 of which 256 do, given: 2,400 us of waits).
    const uint32_t each = (slices + gridDim.x - 1u) / gridDim.x;
    uint32_t counted = 0u;
    for (uint32_t item = 0u, end = 0u, have = ~0u; slices != 0u; ++item) {
        if (item == end) {
            item = take(kNextCount) * each;
            end = min(slices, item + each);
            if (item >= slices) break;
        }
        const uint32_t e = find(item, false);
        const uint4 list = s_list;
        const uint2 *A = pairs + ranges[list.x].x;
        if (e != have) {
            sample(A, list.y, Longer::runs(list.y));
            have = e;
            // (workgroups of the same list write the same)
            if (tid < kRunsMax) lists.split[int64_t(e) * kRunsMax + tid] = s_split[tid];
        }
        if (tid < kRunsMax) total[tid] = 0u;
        __syncthreads();
        count_slice(A, (item - list.z) * kSortLarge, list.y);
        __syncthreads();
        if (tid < kRunsMax) lists.count[int64_t(item) * kRunsMax + tid] = total[tid];
        ++counted;
    }
    ended(kDoneCount, counted);
    // The lists of one workgroup: the first two are given, the others taken, each while the one
    // before the last is sorted, and its range read while the last one is.
    uint2 ahead = blockIdx.x < n_long ? ranges[longs[blockIdx.x]] : make_uint2(0u, 0u);
    for (uint32_t k = blockIdx.x, next = k + gridDim.x; k < n_long;) {
        const uint2 range = ahead;
        uint32_t taken = n_long;
        if (next < n_long) {
            ahead = ranges[longs[next]];
            if (tid == 0) taken = 2u * gridDim.x + atomicAdd(&counters[kNextAlone], 1u);
        }
        sort_alone(range);
        __syncthreads();
        if (tid == 0) s_item = taken;
        __syncthreads();
        k = next;
        next = s_item;
    }
    if (slices == 0u || !wait_for(kDoneCount)) return;
    ended(kDoneDeal, each_item(kNextDeal, slices, [&](uint32_t item) {
        const uint32_t e = find(item, false);
        const uint4 list = s_list;
        const uint2 range = ranges[list.x];
        const uint32_t n = list.y, mine = item - list.z, of = Longer::slices(n);
        // a run's pairs in all slices, and in those before
        const uint32_t q = tid % kRunsMax;
        if (tid < kRunsMax) {
            s_split[tid] = lists.split[int64_t(e) * kRunsMax + tid];
            total[tid] = cursor[tid] = 0u;
        }
        uint32_t all = 0u, before = 0u;
#pragma unroll 8
        for (uint32_t r = tid / kRunsMax; r < of; r += kT / kRunsMax) {
            const uint32_t c = lists.count[int64_t(list.z + r) * kRunsMax + q];
            all += c;
            before += r < mine ? c : 0u;
        }
        __syncthreads();
        atomicAdd(&total[q], all);
        atomicAdd(&cursor[q], before);
        __syncthreads();
        scan_runs();
        if (tid < kRunsMax) {
            cursor[tid] += starts[tid];
            if (mine == 0u) lists.start[int64_t(e) * kRunsMax + tid] = starts[tid];
        }
        __syncthreads();
        deal_slice(pairs + range.x, mine * kSortLarge, n, key1 + range.x, val1 + range.x);
    }));
    if (!wait_for(kDoneDeal)) return;
    each_item(kNextRun, runs, [&](uint32_t item) {
        const uint32_t e = find(item, true);
        const uint4 list = s_list;
        const uint2 range = ranges[list.x];
        const uint32_t n = list.y, q = item - list.w;
        const uint32_t *start = lists.start + int64_t(e) * kRunsMax + q;
        const uint32_t a = start[0], m = (q + 1u < Longer::runs(n) ? start[1] : n) - a, at = range.x + a;
        sort_run(pairs + at, key1 + at, val1 + at, m);
    });
}

}  // namespace

gs_status launch_tile_sort(const gs_settings &s, const Proj &proj, int64_t n, int64_t n_cap, int32_t n_views,
                           const gs_target *targets, int32_t n_targets, int32_t total_tiles, const SortBufs &B,
                           int64_t pair_cap, uint32_t *d_status, hipStream_t st) {
    const int chunk = bin_chunk(n, n_views, total_tiles);
    const int64_t chunks = n > 0 ? (n + chunk - 1) / chunk : 1;
    const BinLists lists{B.rects, B.rec, B.list_count};
    const int window = bin_window(total_tiles, n_targets);
    const size_t lds = sizeof(uint32_t) * window;
    const int splits = n_targets == 1 ? (total_tiles + window - 1) / window : 1;   // the scatter's windows
    const int64_t stride = B.tile_stride, tiles = total_tiles;
    const uint32_t cap = uint32_t(pair_cap);
    // small chunks (maps of up to kBinChunks * kBinChunkMin records): small
    // workgroups, whose barriers and start cost less, but for windows that take them long
    // to clear and to write (30,000 Gaussians over 80,000 tiles 305 us, 228 by large ones)
    constexpr int kFew = kBinThreadsFew, kMany = kBinThreadsMany;
    const bool few = chunk <= kBinChunkMin && window <= kBinWindow, one = n_targets == 1, scan = tiles <= kScanTilesMax;
    const int64_t share = n <= kLargeAlways ? 0 : 3 * pair_cap / (2 * chunks);
    const int64_t least = chunk <= kBinChunkMin ? kBudgetFew : kBudgetMany;
    const uint32_t budget = uint32_t(share > least ? share : least);
    // workgroups of a target in the scatter: for its chunks, and more where its large entries could keep them busy
    const int64_t groups = (tiles + int64_t(n_targets) * kWave - 1) / (int64_t(n_targets) * kWave), some = 256 / n_targets;
    const int64_t most = groups < some ? groups : some, grid = most > xcd_grid(chunks) ? most : xcd_grid(chunks);
    auto count = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(chunks, n_views), dim3(threads), lds, st, s, proj, n, n_cap, chunk, targets,
                           n_targets, B.view_off, B.view_list, window, budget, lists, B.thist, stride, total_tiles, B.counters,
                           B.queue);
    };
    const ScatterArgs args{proj, s.znear, n_cap, chunk, chunks, targets, tiles, window, lists, B.thist, stride, B.tile_total, cap,
                           B.pairs, B.ranges, B.longs, B.long_lists, B.counters, d_status, B.keep};
    auto scatter = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid, n_targets, splits), dim3(threads), lds, st, args);
    };
    if (few) one ? count(bin_count_kernel<kFew, true>, kFew) : count(bin_count_kernel<kFew, false>, kFew);
    else one ? count(bin_count_kernel<kMany, true>, kMany) : count(bin_count_kernel<kMany, false>, kMany);
    hipLaunchKernelGGL(bin_columns_kernel, dim3(stride / kWave), dim3(kColWaves * kWave), 0, st, chunks, tiles, B.thist,
                       stride, B.tile_total, B.group_total, lists, n_cap, chunk, targets, n_targets, B.counters);
    if (!scan)
        hipLaunchKernelGGL(bin_starts_kernel, dim3((tiles + kStartTiles - 1) / kStartTiles), dim3(256), 0, st, tiles, cap,
                           B.group_total, B.tile_total, B.ranges, B.longs, B.long_lists, B.counters, d_status);
    if (few) scan ? scatter(bin_scatter_kernel<kFew, true, false>, kFew) : scatter(bin_scatter_kernel<kFew, false, false>, kFew);
    else if (!scan) scatter(bin_scatter_kernel<kMany, false, false>, kMany);
    else if (one && (chunks <= kBinChunks || tiles > kStageTiles)) scatter(bin_scatter_kernel<kMany, true, true>, kMany);
    else scatter(bin_scatter_kernel<kMany, true, false>, kMany);
    constexpr int kGroup = kSortThreads / kWave;
    if (tiles <= int64_t(kOrderTiles) * n_targets)
        hipLaunchKernelGGL(tile_order_small_kernel<1>, dim3(total_tiles), dim3(kSortThreads), 0, st, B.ranges, B.pairs,
                           B.sorted, tiles);
    else
        hipLaunchKernelGGL(tile_order_small_kernel<kGroup>, dim3((total_tiles + kGroup - 1) / kGroup), dim3(kSortThreads), 0,
                           st, B.ranges, B.pairs, B.sorted, tiles);
    if (n > kSortSmall) {   // (a list holds each record of its view at most once)
        const int grid = n > kSortAlone || total_tiles > kSortLargeGrid ? kSortLargeGrid : total_tiles;
        hipLaunchKernelGGL(tile_order_large_kernel, dim3(grid), dim3(kSortLargeThreads), 0, st, B.counters, B.longs,
                           B.ranges, B.long_lists, B.pairs, B.other, B.sorted);
    }
    return GS_OK;
}

}  // namespace gs
