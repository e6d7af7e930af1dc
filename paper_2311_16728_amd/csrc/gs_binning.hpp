// Shared by the two binning paths (gs_sort.hip, gs_tilesort.hip): tile
// rectangles, depth keys, small scans and the workspace's buffers.
#pragma once

#include "gs_internal.hpp"

namespace gs {

// Conservative pixel bounding box of {alpha >= alpha_min} for a record at a
// pyramid level.  Returns false when the record cannot reach any pixel; records
// behind the near plane carry opacity 0 and are rejected by the opacity test.
struct Rect {
    int x0, x1, y0, y1;   // inclusive tile ranges
};

__device__ __forceinline__ bool tile_rect(const gs_settings &s, double2 md, float4 cov_o,
                                          const gs_target &t, Rect &r) {
    const float o = cov_o.w;
    if (!(o >= s.alpha_min)) return false;
    const float sc = ldexpf(1.f, -t.level);
    const float mx = float(md.x) * sc, my = float(md.y) * sc;
    const float c00 = cov_o.x * sc * sc + s.dilation;
    const float c11 = cov_o.z * sc * sc + s.dilation;
    const float tq = 2.f * logf(o / s.alpha_min);
    float ex = sqrtf(tq * c00), ey = sqrtf(tq * c11);
    ex += 0.05f + 1e-3f * ex;
    ey += 0.05f + 1e-3f * ey;
    const float fx0 = ceilf(mx - ex), fx1 = floorf(mx + ex);
    const float fy0 = ceilf(my - ey), fy1 = floorf(my + ey);
    if (!(fx1 >= 0.f) || !(fy1 >= 0.f) || !(fx0 <= float(t.width - 1)) ||
        !(fy0 <= float(t.height - 1)) || !(fx0 <= fx1) || !(fy0 <= fy1))
        return false;
    const int px0 = max(0, int(fx0)), px1 = min(t.width - 1, int(fx1));
    const int py0 = max(0, int(fy0)), py1 = min(t.height - 1, int(fy1));
    const TileShape ts = tile_shape(t.tile_w);
    r.x0 = px0 >> ts.wlog; r.x1 = px1 >> ts.wlog;
    r.y0 = py0 / ts.h; r.y1 = py1 / ts.h;
    return true;
}

// 64-bit wave scans for the pair offsets: a sum of per-record pair counts may
// pass 2^32, and is then saturated (a total past pair_cap <= 2^31 - 1 is an
// overflow, reported as such) instead of wrapping.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
    return (uint64_t(dpp_u32<kCtrl, kRowMask>(uint32_t(v >> 32))) << 32) | dpp_u32<kCtrl, kRowMask>(uint32_t(v));
}
// (the DPP steps of wave_inclusive_scan, on both halves)
__device__ __forceinline__ uint64_t wave_inclusive_scan64(uint64_t v) {
    v += dpp_u64<0x111, 0xf>(v);
    v += dpp_u64<0x112, 0xf>(v);
    v += dpp_u64<0x114, 0xf>(v);
    v += dpp_u64<0x118, 0xf>(v);
    v += dpp_u64<0x142, 0xa>(v);
    v += dpp_u64<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ uint32_t sat32(uint64_t v) {
    return v > 0xffffffffull ? 0xffffffffu : uint32_t(v);
}

// Exclusive scan over a 256-thread block in 64 bits; block total to *total.
// lds needs 4 words.
__device__ __forceinline__ uint64_t block_exclusive_scan64(uint64_t v, uint64_t *lds, uint64_t *total) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const uint64_t inc = wave_inclusive_scan64(v);
    if (lane == kWave - 1) lds[wave] = inc;
    __syncthreads();
    uint64_t base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / kWave; ++w) {
        const uint64_t x = lds[w];
        base += w < wave ? x : 0u;
        all += x;
    }
    __syncthreads();
    *total = all;
    return base + inc - v;
}

// Depth sort key of a visible record: the bit pattern of its (positive,
// float) depth minus that of the near plane, which orders depths exactly as
// the floats do while they stay within 2^27 ulps of the near plane (below
// znear * 2^16: 13 km at znear 0.2 m); deeper ones share the largest key and
// keep record order.  27 bits: three 9-bit radix passes.
constexpr int kDepthKeyBits = 27;
__device__ __forceinline__ uint32_t depth_key(float z, float znear) {
    const uint32_t a = __float_as_uint(z), b = __float_as_uint(znear);
    const uint32_t d = a > b ? a - b : 0u;
    return d < (1u << kDepthKeyBits) ? d : (1u << kDepthKeyBits) - 1u;
}

// q = k / w, r = k % w for k < 2^24, w >= 1: a float reciprocal estimate
// corrected by one step (exact: the estimate is off by at most one).
__device__ __forceinline__ void divmod_small(uint32_t k, uint32_t w, uint32_t &q, uint32_t &r) {
    q = uint32_t(float(k) * __builtin_amdgcn_rcpf(float(w)));
    int32_t rr = int32_t(k) - int32_t(q * w);
    if (rr < 0) { --q; rr += int32_t(w); }
    else if (rr >= int32_t(w)) { ++q; rr -= int32_t(w); }
    r = uint32_t(rr);
}

// Lists of the tile-sort path, one stretch per (target, chunk of records): the
// tile rectangle and record of each visible record, and their number (count[target * chunks + chunk]).  Stretches start at
// target * n_cap + chunk * (records per chunk).
struct BinLists {
    uint2 *rect;
    uint32_t *rec, *count;
};

// Lists of more than kSortAlone pairs: per list its tile, pairs, first slice and first run;
// the splitters between its runs and the runs' starts; per slice its pairs in each
// run (kRunsMax entries each).
struct LongLists {
    uint4 *list;
    uint2 *split;
    uint32_t *count, *start;
};

// What the phases count with that keep an overflowing call's first pairs
// (keep_first_pairs): the tiles of the entries by each digit of their rank, depth key and
// record, and for every phase the next item and those that are done.
constexpr int kRankBits = kDepthKeyBits + 32, kKeepBins = 1024;
enum KeepPhase { kKeepDigits = (kRankBits + 9) / 10, kKeepCount = kKeepDigits, kKeepStarts, kKeepPlace, kKeepPhases };
struct KeepState {
    unsigned long long bins[kKeepDigits][kKeepBins];
    uint32_t next[kKeepPhases], done[kKeepPhases];
};
static_assert(sizeof(KeepState) <= kKeepBytes, "the workspace's share");

struct SortBufs {
    uint32_t *counters, *counts, *vk[2], *vv[2], *voff, *pk[2], *pv[2], *bsum, *hist, *digit, *chunk_first,
        *view_off, *view_list;
    uint2 *ranges, *rects;
    uint32_t *order, *queue, *thist, *whist, *wdigit;
    int64_t max_blocks, tile_blocks, tile_stride, wstride;
    // tile sort: the lists' records, their lengths, the tile totals (then
    // starts) and their sums per 64 tiles, the tiles with long lists, the pairs (over both key
    // buffers), the sorted records' buffer and the other value buffer
    uint32_t *rec, *list_count, *tile_total, *longs, *sorted, *other;
    uint64_t *group_total;
    uint2 *pairs;
    LongLists long_lists;
    KeepState *keep;
};

static inline SortBufs sort_bufs(void *ws, int32_t n_views, int32_t n_targets, int64_t n_cap, int64_t pair_cap,
                          int32_t total_tiles) {
    SortLayout L = SortLayout::make(n_views, n_targets, n_cap, pair_cap, total_tiles);
    char *b = static_cast<char *>(ws);
    auto u = [&](size_t o) { return reinterpret_cast<uint32_t *>(b + o); };
    SortBufs B;
    B.counters = u(L.counters);
    B.counts = u(L.counts);
    B.vk[0] = u(L.vis_key0); B.vk[1] = u(L.vis_key1);
    B.vv[0] = u(L.vis_val0); B.vv[1] = u(L.vis_val1);
    B.voff = u(L.vis_off);
    B.pk[0] = u(L.pair_key0); B.pk[1] = u(L.pair_key1);
    B.pv[0] = u(L.pair_val0); B.pv[1] = u(L.pair_val1);
    B.bsum = u(L.bsum);
    B.hist = u(L.hist);
    B.digit = u(L.digit);
    B.chunk_first = u(L.chunk_first);
    B.view_off = u(L.view_off);
    B.view_list = u(L.view_list);
    B.ranges = reinterpret_cast<uint2 *>(b + L.ranges);
    B.rects = reinterpret_cast<uint2 *>(b + L.rects);
    B.max_blocks = L.max_blocks;
    B.thist = u(L.thist);
    B.whist = u(L.whist);
    B.wdigit = u(L.wdigit);
    B.wstride = L.wstride;
    B.tile_blocks = L.tile_blocks;
    B.tile_stride = L.tile_stride;
    B.order = u(L.order);
    B.queue = u(L.queue);
    B.rec = u(L.list_rec);
    B.list_count = u(L.list_count);
    B.tile_total = u(L.tile_total);
    B.longs = u(L.longs);
    B.group_total = reinterpret_cast<uint64_t *>(b + L.group_total);
    B.pairs = reinterpret_cast<uint2 *>(b + L.pair_key0);
    B.long_lists = LongLists{reinterpret_cast<uint4 *>(b + L.long_list), reinterpret_cast<uint2 *>(b + L.split),
                             u(L.slice_count), u(L.run_start)};
    B.keep = reinterpret_cast<KeepState *>(b + L.keep);
    const int at = sorted_buffer(total_tiles);
    B.sorted = B.pv[at];
    B.other = B.pv[at ^ 1];
    return B;
}

// gs_bin_sort's path by per-tile depth sorts (gs_tilesort.hip); the counters
// and view lists of several targets have been set up.
gs_status launch_tile_sort(const gs_settings &s, const Proj &proj, int64_t n, int64_t n_cap, int32_t n_views,
                           const gs_target *targets, int32_t n_targets, int32_t total_tiles, const SortBufs &B,
                           int64_t pair_cap, uint32_t *d_status, hipStream_t st);

}  // namespace gs
