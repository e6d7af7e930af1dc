// Tile rasteriser: Eq. 3 forward (front-to-back alpha compositing) and its
// reverse mode, recomputed back to front.
//
// One workgroup of one, two or four waves per tile of 256 pixels, four, two or one
// pixels per lane.  The tile's sorted list is consumed in batches: each thread
// gathers one Gaussian's record, converts it
// to the target's pyramid level (2D mean scaled by 2^-l, covariance by 4^-l
// plus the dilation, then inverted to the conic) and stages it in LDS; every
// pixel then reads the batch as LDS broadcasts.  The forward keeps, per
// pixel, only the final transmittance and one past the list position of the
// last composited Gaussian; the backward restarts from those, divides the
// transmittance back out Gaussian by Gaussian, and keeps a running dot
// product of what lies behind with dL/dC, so no per-pixel list is stored.
// Per Gaussian it sums over the tile's pixels the moments of dL/d(exponent)
// over the pixel offsets and the opacity and colour terms (registers, DPP
// and LDS), turns the moments into the gradients of the nine 2D quantities,
// and commits them with one atomic per quantity per tile.
#include "gs_internal.hpp"

#include <atomic>
#include <type_traits>

namespace gs {

// Finds the target owning global tile `tile` (targets sorted by tile_offset).
__device__ __forceinline__ int find_target(const gs_target *__restrict__ targets, int n_targets,
                                           int tile) {
    int lo = 0, hi = n_targets - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (targets[mid].tile_offset <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The record of source `src` as seen by a target at pyramid level `level`,
// with its 2D mean relative to the tile origin (ox, oy): the FP64 mean is
// reduced before rounding, so offsets inside the tile are accurate to a few
// 1e-7 px.  thr = ln(alpha_min / opacity): a pixel composites the Gaussian iff
// its exponent reaches thr.
__device__ __forceinline__ void stage_record(const gs_settings &s, const Proj &proj, int64_t n_cap,
                                             int view, int level, double ox, double oy, uint32_t src,
                                             float4 &A, float4 &B, float2 &C, int64_t &rec) {
    const int64_t g = int64_t(src % uint32_t(n_cap));
    const int64_t r = int64_t(view) * n_cap + g;
    rec = r;
    const float sc = ldexpf(1.f, -level);
    const double2 m = proj.mean[r];
    const float4 co = proj.cov_o[r];
    const float4 cz = proj.rgb_z[r];
    const float c00 = fmaf(co.x, sc * sc, s.dilation);
    const float c01 = co.y * (sc * sc);
    const float c11 = fmaf(co.z, sc * sc, s.dilation);
    const float det = c00 * c11 - c01 * c01;
    const float idet = 1.f / det;
    const double dsc = double(sc);
    A = make_float4(float(m.x * dsc - ox), float(m.y * dsc - oy), c11 * idet, -c01 * idet);
    B = make_float4(c00 * idet, co.w, cz.x, cz.y);
    C = make_float2(cz.z, __logf(s.alpha_min / co.w));
}

// Minimum of the quadratic form q(d) = a dx^2 + 2 b dx dy + c dy^2, d = p - m,
// over pixel centres p in [0, hx] x [0, hy] (tile-relative), relaxed to the
// rectangle.
__device__ __forceinline__ float qmin_tile(const float4 &A, const float4 &B, float hx, float hy) {
    const float mx = A.x, my = A.y, a = A.z, b = A.w, c = B.x;
    const float lo = 0.f;
    if (mx >= lo && mx <= hx && my >= lo && my <= hy) return 0.f;
    float best = 3.4e38f;
    // edges x = const: minimise over dy
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float dx = (e ? hx : lo) - mx;
        const float dy = fminf(fmaxf(-b * dx / c, lo - my), hy - my);
        best = fminf(best, a * dx * dx + 2.f * b * dx * dy + c * dy * dy);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float dy = (e ? hy : lo) - my;
        const float dx = fminf(fmaxf(-b * dy / a, lo - mx), hx - mx);
        best = fminf(best, a * dx * dx + 2.f * b * dx * dy + c * dy * dy);
    }
    return best;
}

// True when some pixel of the tile (ts) may reach the cutoff (conservative).
__device__ __forceinline__ bool touches_tile(const float4 &A, const float4 &B, const float2 &C,
                                             const TileShape &ts) {
    const float tq = -2.f * C.y;   // q <= tq  <=>  exponent >= thr
    return qmin_tile(A, B, float(ts.w - 1), float(ts.h - 1)) <= tq * 1.0001f + 1e-3f;
}

// The tile in kNx x kNy regions of bw x bh pixels; bit q (row by row): some pixel
// of region q may reach the cutoff (conservative, with the margin of
// touches_tile).  The minimum of q(d) over a region is 0 if it holds the mean,
// else on one of its edges; the regions' edges lie on a few lines, on each of
// which the free minimum is found once and clamped to the regions' ranges.  No
// bit is set unless touches_tile holds, which decides what the backward stages;
// it is evaluated itself only where this arithmetic may come out differently.
template <int kNx, int kNy>
__device__ __forceinline__ uint32_t regions_touched(const float4 &A, const float4 &B, const float2 &C,
                                                    const TileShape &ts, int bw, int bh) {
    const float mx = A.x, my = A.y, a = A.z, b = A.w, c = B.x;
    // the cutoff with its margin, and the rounding of q, whose terms, of
    // opposite signs, may be far larger than their sum
    const float ex = fabsf(mx) + 32.f, ey = fabsf(my) + 32.f;
    const float cut = -2.f * C.y * 1.0001f + 1e-3f, err = 2e-6f * (a * ex * ex + c * ey * ey);
    // free minimum along a vertical line dy = sy dx, along a horizontal dx = sx dy
    const float sy = -b * __builtin_amdgcn_rcpf(c), sx = -b * __builtin_amdgcn_rcpf(a);
    float best[kNx * kNy];
#pragma unroll
    for (int q = 0; q < kNx * kNy; ++q) best[q] = 3.4e38f;
#pragma unroll
    for (int l = 0; l < 2 * kNx; ++l) {   // vertical edges
        const float dx = float(bw * (l / 2) + (bw - 1) * (l & 1)) - mx;
        const float free = sy * dx, adx = a * dx * dx, bdx = 2.f * b * dx;
#pragma unroll
        for (int y = 0; y < kNy; ++y) {
            const float dy = __builtin_amdgcn_fmed3f(free, float(bh * y) - my, float(bh * y + bh - 1) - my);
            best[y * kNx + l / 2] = fminf(best[y * kNx + l / 2], adx + dy * (bdx + c * dy));
        }
    }
#pragma unroll
    for (int l = 0; l < 2 * kNy; ++l) {   // horizontal edges
        const float dy = float(bh * (l / 2) + (bh - 1) * (l & 1)) - my;
        const float free = sx * dy, cdy = c * dy * dy, bdy = 2.f * b * dy;
#pragma unroll
        for (int x = 0; x < kNx; ++x) {
            const float dx = __builtin_amdgcn_fmed3f(free, float(bw * x) - mx, float(bw * x + bw - 1) - mx);
            best[(l / 2) * kNx + x] = fminf(best[(l / 2) * kNx + x], cdy + dx * (bdy + a * dx));
        }
    }
    uint32_t bits = 0u;
    float tile = 3.4e38f;   // the tile's minimum
#pragma unroll
    for (int q = 0; q < kNx * kNy; ++q) {
        const float x = float(bw * (q % kNx)), y = float(bh * (q / kNx));
        const bool inside = mx >= x && mx <= x + float(bw - 1) && my >= y && my <= y + float(bh - 1);
        const float least = inside ? 0.f : best[q];
        if (least <= cut + err) bits |= 1u << q;
        tile = fminf(tile, least);
    }
    // (written so that a NaN cutoff is left to touches_tile)
    if (!(tile <= cut - err) && bits != 0u && !touches_tile(A, B, C, ts)) bits = 0u;
    return bits;
}

// The same over the regions of a tile's kWaves waves: two halves of 16x8 pixels
// (8x16 of an 8-wide tile), or four 8x8 blocks.
template <int kWaves>
__device__ __forceinline__ uint32_t waves_touched(const float4 &A, const float4 &B, const float2 &C, const TileShape &ts) {
    if (kWaves == 2)
        return ts.wlog == 5 ? regions_touched<2, 1>(A, B, C, ts, 16, 8)
                            : regions_touched<1, 2>(A, B, C, ts, ts.w, ts.h / 2);
    return ts.wlog == 4   ? regions_touched<2, 2>(A, B, C, ts, 8, 8)
           : ts.wlog == 3 ? regions_touched<1, 4>(A, B, C, ts, 8, 8)
                          : regions_touched<4, 1>(A, B, C, ts, 8, 8);
}

// alpha = min(opacity x exp(power), alpha_max) for the non-negative first
// argument, as one median instruction (an fminf canonicalises its operands
// on every use); forward and backward use the same instruction.
__device__ __forceinline__ float clamp_alpha(float at, float amax) {
    return __builtin_amdgcn_fmed3f(at, 0.f, amax);
}

// Staged records hold the conic in base-2 exponent form: A.z = -a log2(e) / 2,
// A.w = -b log2(e), B.x = -c log2(e) / 2 for the conic (a, b, c) of
// stage_record, and the cutoff C.y = ln(alpha_min / opacity) log2(e), so the
// exponent in base 2, -(a dx^2 + 2 b dx dy + c dy^2) log2(e) / 2, takes five
// operations and goes to the hardware exp2 as it is.  conic_a/b/c give the
// conic back (to a rounding or two: the gradients use it, the compositing
// decisions do not).
constexpr float kLog2e = 1.44269504088896341f, kLn2 = 0.693147180559945309f;
__device__ __forceinline__ void to_exponent_form(float4 &A, float4 &B, float2 &C) {
    A.z *= -0.5f * kLog2e;
    A.w *= -kLog2e;
    B.x *= -0.5f * kLog2e;
    C.y *= kLog2e;
}
__device__ __forceinline__ float conic_a(const float4 &A) { return A.z * (-2.f * kLn2); }
__device__ __forceinline__ float conic_b(const float4 &A) { return A.w * -kLn2; }
__device__ __forceinline__ float conic_c(const float4 &B) { return B.x * (-2.f * kLn2); }

// Base-2 exponent of a staged Gaussian at offset (dx, dy) = mean - pixel:
// dx (A.z dx) + dy (A.w dx + B.x dy).  The same instruction sequence serves
// the forward and the backward, so both take the same alpha_min decision.
__device__ __forceinline__ float eval_power(const float4 &A, const float4 &B, float dx, float dy) {
    const float u = fmaf(A.w, dx, B.x * dy);
    return fmaf(A.z * dx, dx, u * dy);
}

// Block-wide count of `flag` for kThreads threads (a multiple of 64): the
// number of threads before this one where it holds (ballots, no scan), and
// the block total.
template <int kThreads>
__device__ __forceinline__ uint32_t block_count_n(bool flag, uint32_t *lds, uint32_t *total) {
    constexpr int kW = kThreads / kWave;
    const uint64_t m = __ballot(flag);
    const uint32_t below = uint32_t(mask_rank(m));
    if (kW == 1) {
        *total = uint32_t(__popcll(m));
        return below;
    }
    const int wave = threadIdx.x / kWave;
    if (lane_id() == 0) lds[wave] = uint32_t(__popcll(m));
    __syncthreads();
    uint32_t base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
        const uint32_t s = lds[w];
        base += (w < wave) ? s : 0u;
        all += s;
    }
    __syncthreads();
    *total = all;
    return base + below;
}

// Per-pixel transmittance store of the store-all variant (the comparison
// point of the recompute backward): the transmittance in front of a pixel's
// k-th composited Gaussian sits at base[tile] + k * 256 + (pixel in tile), so
// each compositing step of a tile writes 256 consecutive floats.  base has
// total_tiles + 1 entries (the last is the floats needed); nothing is stored
// or read when that exceeds cap.
struct TStore {
    const int64_t *base;   // [total_tiles + 1]
    const int64_t *need;   // base + total_tiles: floats the store needs
    float *T;
    int64_t cap;
};

// More tiles than this: two waves a tile, not four.  A lane's second pixel shares
// the reads of LDS, which with one pixel a lane take the LDS pipe as long as the
// vector ALUs take for the step; fewer tiles leave the chip short of waves.
// Four / two waves, us: 209 tiles 28.7 / 54.5; 2,166 46.8 / 50.5; 2,520 49.3 / 54.0;
// 3,225 (three scenes) 42.3 / 40.4, 57.6 / 57.2, 59.4 / 59.3; 4,400 69.9 / 67.2; 34,160
// 537 / 485; 80,606 1,117 / 954.  One wave (four pixels a lane) gains only at the last, 929.
// With the tile queue (schedule 1), whose workgroups start by taking a tile one
// after the other, more workgroups cost more: 3,225 tiles (two scenes), four / two
// waves, 102 / 139 and 92 / 125; 34,160 with two 546 (598 by the earlier kernel of four).
constexpr int kFwdTilesFour = 3000, kFwdQueuedFour = 16384;

// Forward raster with kWaves waves per tile; a wave owns a region of the tile
// (waves_touched) and every lane kPix = 4 / kWaves pixels of one of its columns.
// kCount: per-pixel composited and evaluated counts (and, with tile_max, the
// largest composited count of each tile); kStore: the transmittance store, whose
// waves own strips of whole tile rows, so that a wave's 64 stores of a step fill
// consecutive lines (2M Gaussians at 1200x680, the storing differentiation's
// forward: 8x8 blocks 0.505 ms, strips 0.484; compacted batches 0.484 too).
//
// A staged Gaussian's slot is its place in the batch; each staging wave leaves,
// per region, a 64-bit mask of the slots that may touch it, and a wave walks its
// masks' bits: Gaussians that cover part of a tile cost only the regions they
// touch (the count variant walks every Gaussian that touches the tile, which
// is what it counts).  Lane masks (who has stopped, who composites) are kept in
// scalar registers.
//
// Bound: VALU issue, about 80 cycles a step and pixel (the backward's rates),
// and with one pixel a lane the LDS pipe as much (a step's 40 bytes to 64 lanes
// are 20 cycles of a pipe that four SIMDs share).  Most Gaussians of a list touch
// nearly the whole tile in dense scenes (75 of 88 composite), so the regions
// help sparse tiles and coarse levels most.
// Measured, before -> now in us: 2,000 Gaussians, 64 tiles 19 -> 13.6; 500,000 at
// 300x170, 209 tiles 46 -> 29.7; 1M at 1200x680, 3,225 tiles 55 -> 56; 32 keyframes x 3
// levels, 80,606 tiles 1,212 -> 1,036.  Not kept: compositing under the execution mask
// instead of selects (four waves, 209 tiles 43.4; 3,225 69.6), eight waves per SIMD (60.3),
// two steps at a time with four waves (60.7), one with two (63.8).
template <int kWaves, bool kCount = false, bool kStore = false, bool kQueued = false>
__global__ void __launch_bounds__(kWave *kWaves) __attribute__((amdgpu_waves_per_eu(kQueued ? 5 : 6))) render_fwd_kernel(
    gs_settings s, Proj proj, int64_t n_cap, Sorted srt, const gs_target *__restrict__ targets,
    int n_targets, float *__restrict__ out_rgb, float *__restrict__ out_T,
    int32_t *__restrict__ out_last, int32_t *__restrict__ out_nc, int32_t *__restrict__ out_ne,
    int32_t *__restrict__ tile_max = nullptr, TStore ts_store = TStore{nullptr, nullptr, nullptr, 0},
    const uint32_t *__restrict__ order = nullptr, uint32_t *__restrict__ queue = nullptr, int total_tiles = 0) {
    constexpr int kPix = 4 / kWaves, kThreads = kWave * kWaves;
    static_assert(!(kCount || kStore) || kPix == 1, "counts and stores are one pixel per lane");
    constexpr int kSlot = 48;   // bytes of a staged record: A, B, C and padding
    __shared__ float4 sRec[kThreads * kSlot / 16];
    __shared__ uint64_t sMask[kWaves][kWaves];   // [region][staging wave]
    constexpr bool queued = kQueued;
    const float amax = __builtin_canonicalizef(s.alpha_max);   // (once per launch)
    for (int round = 0;; ++round) {
        int tile;
        if (queued) {   // next tile of the cost-ordered queue
            __shared__ int s_item;
            if (threadIdx.x == 0) s_item = int(atomicAdd(&queue[kQueueNextFwd], 1u));
            __syncthreads();
            const int item = s_item;
            __syncthreads();
            if (item >= total_tiles) break;
            tile = int(order[item]);
            if (tile < 0 || tile >= total_tiles) continue;   // not a tile: order not built
        } else {
            if (round > 0) break;
            tile = blockIdx.x;
        }
        const int tid = threadIdx.x, lane = lane_id();
        const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
        const gs_target t = targets[find_target(targets, n_targets, tile)];
        const int local = tile - t.tile_offset;
        const int tx = local % t.tiles_x, ty = local / t.tiles_x;
        const TileShape ts = tile_shape(t.tile_w);
        // the wave's region, and the lane's first pixel; the next are `drow` rows down
        const int rlog = kStore ? ts.wlog : kWaves == 4 ? 3 : min(ts.wlog, 4);
        const int across = ts.w >> rlog, drow = kWave >> rlog;
        const int lxp = ((wave & (across - 1)) << rlog) + (lane & ((1 << rlog) - 1));
        const int lyp = (wave >> (ts.wlog - rlog)) * drow * kPix + (lane >> rlog);
        const int px = tx * ts.w + lxp, py = ty * ts.h + lyp;
        const uint2 range = srt.ranges[tile];
        const double ox = double(tx * ts.w), oy = double(ty * ts.h);

        float fpx = float(lxp), fpy[kPix];   // relative to the tile origin
        float T[kPix], C0[kPix], C1[kPix], C2[kPix];
        int32_t nc = 0, ne = 0, last[kPix];
        uint64_t done[kPix];   // lanes that have stopped
#pragma unroll
        for (int k = 0; k < kPix; ++k) {
            fpy[k] = float(lyp + k * drow);
            T[k] = 1.f;
            C0[k] = C1[k] = C2[k] = 0.f;
            last[k] = 0;
            done[k] = __ballot(!(px < t.width && py + k * drow < t.height));
        }
        auto all_done = [&]() {
            uint64_t m = done[0];
#pragma unroll
            for (int k = 1; k < kPix; ++k) m &= done[k];
            return m == ~0ull;
        };
        float *store_at = nullptr;   // this pixel's first slot (kStore), or none
        if (kStore && *ts_store.need <= ts_store.cap) store_at = ts_store.T + ts_store.base[tile] + lyp * ts.w + lxp;
        const int batch = min(s.batch, kThreads);
        for (uint32_t b0 = range.x; b0 < range.y; b0 += batch) {
            if (__syncthreads_and(all_done())) break;
            // stage the batch and mark the regions each Gaussian's cutoff ellipse meets
            const uint32_t idx = b0 + tid;
            uint32_t touched = 0u;
            if (tid < batch && idx < range.y) {
                float4 A, B;
                float2 Cc;
                int64_t rec;
                stage_record(s, proj, n_cap, t.view, t.level, ox, oy, srt.pair_val[idx], A, B, Cc, rec);
                touched = kCount   ? (touches_tile(A, B, Cc, ts) ? 0xfu : 0u)
                          : kStore ? regions_touched<1, 4>(A, B, Cc, ts, ts.w, kWave >> ts.wlog)
                                   : waves_touched<kWaves>(A, B, Cc, ts);
                to_exponent_form(A, B, Cc);
                float4 *slot = sRec + tid * (kSlot / 16);
                slot[0] = A;
                slot[1] = B;
                *reinterpret_cast<float2 *>(slot + 2) = Cc;
            }
#pragma unroll
            for (int q = 0; q < kWaves; ++q) {
                const uint64_t m = __ballot((touched >> q) & 1u);
                if (lane == 0) sMask[q][wave] = m;
            }
            __syncthreads();
            int32_t lj[kPix];   // where this batch's last composited Gaussian is staged
#pragma unroll
            for (int k = 0; k < kPix; ++k) lj[k] = -1;
            // Straight-line body: every lane evaluates every Gaussian of its
            // region and keeps the result only where it composites (a wave runs
            // the exponential whenever one of its lanes does); a lane that
            // stops compositing stays in the loop as a no-op until all of the
            // wave's lanes have stopped (checked every few Gaussians).
            auto step = [&](int at) {
                const char *slot = reinterpret_cast<const char *>(sRec) + at;
                const float4 A = *reinterpret_cast<const float4 *>(slot);
                const float4 B = *reinterpret_cast<const float4 *>(slot + 16);
                const float2 Cj = *reinterpret_cast<const float2 *>(slot + 32);
                const float dx = A.x - fpx;
#pragma unroll
                for (int k = 0; k < kPix; ++k) {
                    const float pw = eval_power(A, B, dx, A.y - fpy[k]);
                    if (kCount) ne += ((done[k] >> lane) & 1u) ? 0 : 1;
                    const uint64_t hit = __ballot(!(pw < Cj.y)) & ~done[k];
                    const float alpha = clamp_alpha(B.y * __builtin_amdgcn_exp2f(pw), amax);
                    const float Tn = T[k] * (1.f - alpha);
                    const uint64_t stop = __ballot(Tn < s.t_min) & hit;
                    done[k] |= stop;
                    const bool comp = __builtin_amdgcn_inverse_ballot_w64(hit & ~stop);
                    if (kStore && store_at && comp) store_at[int64_t(nc) * kTilePix] = T[k];
                    // a Gaussian that does not composite adds 0 x colour:
                    // colours and sums are finite and >= 0, so the sums keep
                    // their bits
                    const float w = comp ? alpha * T[k] : 0.f;
                    C0[k] = fmaf(w, B.z, C0[k]);
                    C1[k] = fmaf(w, B.w, C1[k]);
                    C2[k] = fmaf(w, Cj.x, C2[k]);
                    T[k] = comp ? Tn : T[k];
                    lj[k] = comp ? at : lj[k];
                    if (kCount || kStore) nc += comp ? 1 : 0;
                }
            };
            if (!all_done()) {
                constexpr int kTogether = kPix == 1 ? 4 : 2;
#pragma unroll 1
                for (int w = 0; w < kWaves && w * kWave < batch; ++w) {
                    uint64_t m = sMask[wave][w];
                    m = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(m >> 32)))) << 32) |
                        uint32_t(__builtin_amdgcn_readfirstlane(int(m)));
                    auto next = [&]() {
                        const int j = __builtin_ctzll(m);
                        m &= m - 1;
                        return (w * kWave + j) * kSlot;
                    };
                    for (int left = __popcll(m); left >= kTogether; left -= kTogether) {
                        int at[kTogether];
#pragma unroll
                        for (int i = 0; i < kTogether; ++i) at[i] = next();
#pragma unroll
                        for (int i = 0; i < kTogether; ++i) step(at[i]);
                        if (all_done()) m = 0, left = 0;
                    }
                    while (m != 0ull) step(next());
                    if (all_done()) break;
                }
                // one past the list position of the last composited Gaussian
#pragma unroll
                for (int k = 0; k < kPix; ++k)
                    if (lj[k] >= 0) last[k] = int32_t(b0 - range.x) + lj[k] / kSlot + 1;
            }
        }
        const int64_t HW = int64_t(t.width) * t.height;
        float *rgb = out_rgb + 3 * t.pix_offset;
#pragma unroll
        for (int k = 0; k < kPix; ++k) {
            if (px >= t.width || py + k * drow >= t.height) continue;
            const int64_t pix = int64_t(py + k * drow) * t.width + px;
            rgb[pix] = fmaf(T[k], t.bg[0], C0[k]);
            rgb[HW + pix] = fmaf(T[k], t.bg[1], C1[k]);
            rgb[2 * HW + pix] = fmaf(T[k], t.bg[2], C2[k]);
            out_T[t.pix_offset + pix] = T[k];
            out_last[t.pix_offset + pix] = last[k];
            if (kCount && out_nc) out_nc[t.pix_offset + pix] = nc;
            if (kCount && out_ne) out_ne[t.pix_offset + pix] = ne;
        }
        if (kCount && tile_max) {
            __shared__ int32_t tmax;
            if (tid == 0) tmax = 0;
            __syncthreads();
            if (nc > 0) atomicMax(&tmax, nc);
            __syncthreads();
            if (tid == 0) tile_max[tile] = tmax;
        }
    }
    if (queued) queue_retire(queue, kQueueNextFwd, kQueueDoneFwd);
}

// Exclusive scan of the per-tile store sizes (256 floats per compositing step
// of the tile's deepest pixel) into base[0..total_tiles]; one workgroup.
__global__ void __launch_bounds__(1024) store_base_kernel(const int32_t *__restrict__ tile_max,
                                                          int64_t total_tiles, int64_t *__restrict__ base) {
    __shared__ int64_t wsum[16];
    const int64_t per = (total_tiles + 1023) / 1024;
    const int64_t lo = int64_t(threadIdx.x) * per;
    int64_t local = 0;
    for (int64_t i = lo; i < lo + per && i < total_tiles; ++i) local += int64_t(tile_max[i]) * kTilePix;
    // inclusive scan over the block in 64 bits
    int64_t inc = local;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int64_t u = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += u;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    int64_t before = 0, all = 0;
    for (int w = 0; w < 16; ++w) {
        before += w < wave ? wsum[w] : 0;
        all += wsum[w];
    }
    int64_t run = before + inc - local;
    for (int64_t i = lo; i < lo + per && i < total_tiles; ++i) {
        base[i] = run;
        run += int64_t(tile_max[i]) * kTilePix;
    }
    if (threadIdx.x == 0) base[total_tiles] = all;
}

// Backward raster with kWaves waves per 16x16 tile; every lane owns
// kPix = 4 / kWaves pixels of one column (rows spaced by 4 * kWaves), or with
// four waves one pixel of its wave's 8x8 block, of which only the Gaussians that
// touch it are walked (regions_touched).
// Entries are staged bwd_stage(kWaves) at a time, back to front.
//
// Per Gaussian a lane forms nine sums over its pixels: the moments of
// n = dL/d(exponent) over the pixel offsets (sum n dx, sum n dy, sum n dx^2,
// sum n dx dy, sum n dy^2 and N = sum n; as the column shares dx, only N, sum n dy
// and sum n dy^2 are formed per pixel) and w dL/dC per channel.  They are added
// over the wave without a full butterfly per value: DPP adds that write half
// or a quarter of the banks of a register leave four values' sums over four
// lanes each in one register, so 14 adds reduce nine values to three registers
// of 16 parts per value; those go to an LDS transpose buffer, and once kGroup
// Gaussians are buffered every lane sums the parts of one of kGroup * 9 values.
//
// A pixel row that no lane composites is skipped; inside a row there are no
// branches: a pixel that does not composite the Gaussian takes alpha 0, which
// leaves its transmittance and what lies behind it as they are and adds zeros.
// Bound: VALU issue.  A wave64 add, multiply or move takes 2 cycles here, an FMA,
// compare, select, median or DPP add 4, a transcendental or lane swap 8
// (measured): about 106 cycles a pixel row and 80 a Gaussian.  A lone wave issues one
// only every 6 cycles, which is what few tiles are bound by: there a Gaussian's
// staged values are read one Gaussian ahead.
// Measured, the kernel alone in us: 2,000 Gaussians, 64 tiles, four waves 34.6; 500,000
// at 300x170, 209 tiles, four 73.7; 45,037 at 1200x680, 3,225 tiles, one 108; 1M there,
// one 136; 8 keyframes x 3 levels, 34,160 tiles, one 956; 32, 80,606 tiles, one 2,098.
// (Sums by butterflies, branches in the rows and every Gaussian of the tile walked, with
// about 9 us of clearing: 61, 135, -, 158, -, 2,329; every Gaussian walked, by the present
// body, at 64 and 209 tiles 42 and 91.)  Not kept: the sums by 16x16x4 FP32 matrix products with a one-hot
// operand (nine products of 32 cycles a Gaussian: 3,167 at one wave), by lane swaps (8
// cycles each: 2,368), and a second form of the loop without the two tests for
// Gaussians and tiles that cannot fail them (2,139, its registers cost more).
constexpr int kGroup = 6;                      // 6 * 9 = 54 values <= 64 lanes
constexpr int kParts = 16;                     // parts per value in the buffer
constexpr int kTStride = kParts + 4;           // 16-byte aligned rows on different banks
// Gaussians staged at a time.  With four waves (few tiles, whose latency
// counts) every thread stages one; otherwise 64, by the first wave, so that
// the LDS a workgroup takes does not limit how many are resident.
constexpr int bwd_stage(int waves) { return waves == 4 ? 256 : 64; }

// v[0..8] over the wave, in v[0], v[4] and v[8]: in every row of 16 lanes, the
// four banks of four lanes hold values 0, 2, 1, 3 (then 4, 6, 5, 7, then 8 in all
// banks), each lane the sum of four of the row's lanes.  First the lanes 8 apart
// are added (row_ror:8), two values to a register, then a half row's lane i and
// 7 - i (row_half_mirror), two such registers to one.  One block, as a DPP
// operand must not have been written by the last two instructions.
__device__ __forceinline__ void quarter_rows(float (&v)[9]) {
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %6, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %4, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %6, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %8, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %8, %8, %8 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %4, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xa"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]), "+v"(v[8]));
}

// What the branch-free body takes: loss gradients and colours that are finite and
// whose products and sums stay far from overflow (1e30 x 1e6 x 3).  Its zero weights
// would carry an infinity or NaN from a pixel into Gaussians that it does not
// composite, or from a Gaussian into pixels that do not composite it, so a tile is
// walked with branches (careful), where only the two that meet see each other, if a
// pixel's gradient, or what the background makes of it, is not plain, and from the
// batch on in which a Gaussian's colour is not.
__device__ __forceinline__ bool plain_gradient(float g) { return fabsf(g) < 1e30f; }
__device__ __forceinline__ bool plain_colour(float r, float g, float b) { return r < 1e6f && g < 1e6f && b < 1e6f; }

// kStored: the store-all variant, which reads each composited Gaussian's
// transmittance from the forward's store (in_nc: per-pixel composited counts)
// instead of dividing it back out.
template <int kWaves, bool kStored = false, bool kQueued = false>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(kWaves == 2 ? 5 : 4))) render_bwd_kernel(
    gs_settings s, Proj proj, int64_t n_cap, Sorted srt, const gs_target *__restrict__ targets,
    int n_targets, const float *__restrict__ in_T, const int32_t *__restrict__ in_last,
    const float *__restrict__ dL_drgb, float *__restrict__ acc,
    const int32_t *__restrict__ in_nc = nullptr, TStore ts_store = TStore{nullptr, nullptr, nullptr, 0},
    const uint32_t *__restrict__ order = nullptr, uint32_t *__restrict__ queue = nullptr, int total_tiles = 0) {
    constexpr int kThreads = 64 * kWaves;
    constexpr int kPix = kTilePix / kThreads;
    constexpr int kStage = bwd_stage(kWaves);
    // one pixel per lane: a wave owns an 8x8 block and walks the Gaussians that
    // touch it (the forward's masks), the next one read from LDS one ahead
    constexpr bool kMasked = kPix == 1;
    static_assert(!kMasked || kStage == kThreads, "a slot per staging thread");
    __shared__ float4 sA[kStage];
    __shared__ float4 sB[kStage];
    __shared__ float4 sC[kStage];       // blue, cutoff, list position
    __shared__ uint32_t sR[kStage];     // record view * n_cap + g (< 2^32)
    __shared__ uint32_t scan_lds[kMasked ? 1 : 8];
    __shared__ uint64_t sMask[kWaves][kMasked ? kWaves : 1];   // [region][staging wave]
    // The tile's sums per staged Gaussian.  The waves add to them in the order they
    // get there, so an array takes two waves' sums at most: 0 + a + b is the same
    // either way, and a Gaussian's sums over a tile are the same bits in every run.
    // (Four waves: 9 KB more leave three workgroups a CU instead of four, which only a
    // launch of more than 768 tiles has, 103 -> 115 us at 1,200; 209 tiles 74 -> 78.  With 128
    // staged at a time 110 and 85, with groups of three in the buffer 107 and 81.)
    constexpr int kSums = kStage * kAccRows, kSumArrays = (kWaves + 1) / 2;
    __shared__ float red[kSumArrays * kSums];
    __shared__ __attribute__((aligned(16))) float tbuf[kWaves][kGroup * kAccRows * kTStride];
    __shared__ uint32_t sK[kWaves][kGroup];
    __shared__ int sMaxLast, sPlain;
    if (kStored && !(*ts_store.need <= ts_store.cap)) return;   // the forward stored nothing
    constexpr bool queued = kQueued;
    const float amax = __builtin_canonicalizef(s.alpha_max);   // (once per launch)
    for (int round = 0;; ++round) {
        int tile;
        if (queued) {   // next tile of the cost-ordered queue
            __shared__ int s_item;
            if (threadIdx.x == 0) s_item = int(atomicAdd(&queue[kQueueNextBwd], 1u));
            __syncthreads();
            const int item = s_item;
            __syncthreads();
            if (item >= total_tiles) break;
            tile = int(order[item]);
            if (tile < 0 || tile >= total_tiles) continue;   // not a tile: order not built
        } else {
            if (round > 0) break;
            tile = blockIdx.x;
        }
        const int tid = threadIdx.x;
        const int lane = lane_id();
        const gs_target t = targets[find_target(targets, n_targets, tile)];
        const int local = tile - t.tile_offset;
        const int tx = local % t.tiles_x, ty = local / t.tiles_x;
        const TileShape ts = tile_shape(t.tile_w);
        const uint2 range = srt.ranges[tile];
        const double ox = double(tx * ts.w), oy = double(ty * ts.h);
        const float sc = ldexpf(1.f, -t.level);
        const int64_t HW = int64_t(t.width) * t.height;
        const float *dLt = dL_drgb + 3 * t.pix_offset;

        // S: the colour behind the current Gaussian (what the pixel shows from
        // there on, background included, at unit transmittance) dotted with
        // dL/dC; only that dot product enters the gradient, so the colour
        // itself is never formed.  At unit transmittance its error shrinks with
        // every Gaussian, and that of a recovered T is a relative error of the
        // gradient: weighted by the transmittances (S T, with dL/dalpha
        // T c . dL/dC - S T / (1 - alpha)) the two terms, of different roundings of
        // T, cancel: 1.4 to 2.3 times the error over 100 and 280 faint Gaussians a
        // pixel whose colours are close to the background's.
        float T[kPix], g0[kPix], g1[kPix], g2[kPix], S[kPix], fpy[kPix];
        int32_t last[kPix];
        int32_t kc[kPix];             // kStored: composited Gaussians not yet walked back
        const float *srow = nullptr;  // kStored: this tile's store
        int32_t steps = 0;            // kStored: compositing steps stored for the tile
        if (kStored) {
            srow = ts_store.T + ts_store.base[tile];
            steps = int32_t((ts_store.base[tile + 1] - ts_store.base[tile]) / kTilePix);
        }
        // the tile width divides 64, so a lane keeps its column in every row it owns
        const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
        const int lxp = kMasked ? (wave * 8 & (ts.w - 1)) + (lane & 7) : tid & (ts.w - 1);
        const float fpx = float(lxp);
        int my_max = 0;
        bool plain = true;
    #pragma unroll
        for (int i = 0; i < kPix; ++i) {
            const int ly = kMasked ? (wave * 8 >> ts.wlog) * 8 + (lane >> 3) : (tid + i * kThreads) >> ts.wlog;
            fpy[i] = float(ly);
            const int px = tx * ts.w + lxp, py = ty * ts.h + ly;
            T[i] = 0.f; g0[i] = g1[i] = g2[i] = 0.f; last[i] = 0;
            kc[i] = 0;
            if (px < t.width && py < t.height) {
                const int64_t pix = int64_t(py) * t.width + px;
                if (kStored)
                    kc[i] = min(in_nc[t.pix_offset + pix], steps);
                else
                    T[i] = in_T[t.pix_offset + pix];
                last[i] = in_last[t.pix_offset + pix];
                g0[i] = dLt[pix];
                g1[i] = dLt[HW + pix];
                g2[i] = dLt[2 * HW + pix];
            }
            // a restart position never exceeds the tile's list (guards stale input)
            last[i] = min(last[i], int32_t(range.y - range.x));
            my_max = max(my_max, last[i]);
            S[i] = fmaf(t.bg[0], g0[i], fmaf(t.bg[1], g1[i], t.bg[2] * g2[i]));   // the background
            plain &= plain_gradient(g0[i]) && plain_gradient(g1[i]) && plain_gradient(g2[i]) && fabsf(S[i]) < 1e36f;
        }
        if (tid == 0) { sMaxLast = 0; sPlain = 1; }
        __syncthreads();
        if (my_max > 0) atomicMax(&sMaxLast, my_max);
        if (!plain) sPlain = 0;
        __syncthreads();
        const int max_last = sMaxLast;

        // Orders this wave's LDS accesses around a hand-over between its lanes.
        auto wave_sync = [] {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        const int first = int(fpy[0]) * ts.w + lxp;   // tile-local index of this lane's first pixel
        float *tb = tbuf[wave];
        // this lane's places in a Gaussian's rows of the buffer (quarter_rows):
        // a row of the wave gives four parts; value 8 is in every bank, mirrored
        // in every other one
        const int bank = (lane >> 2) & 3;
        const int part = (((bank & 1) << 1) | (bank >> 1)) * kTStride + (lane >> 4) * 4 + (lane & 3);
        const int part8 = 8 * kTStride + (lane >> 4) * 4 + ((bank & 1) ? 3 - (lane & 3) : lane & 3);

        for (int end = max_last; end > 0; end -= kStage) {
            const int start = max(0, end - kStage);
            __syncthreads();
            float4 A, Bv;
            float2 Cc;
            int64_t rec;
            uint32_t keep = 0u;   // kMasked: the regions it touches, else whether it touches the tile
            if (tid < end - start) {
                stage_record(s, proj, n_cap, t.view, t.level, ox, oy, srt.pair_val[range.x + start + tid],
                             A, Bv, Cc, rec);
                keep = kMasked ? waves_touched<4>(A, Bv, Cc, ts) : touches_tile(A, Bv, Cc, ts) ? 1u : 0u;
                to_exponent_form(A, Bv, Cc);
            }
            uint32_t cnt = uint32_t(end - start), at_pos = tid;
            if (kMasked) {
#pragma unroll
                for (int q = 0; q < kWaves; ++q) {
                    const uint64_t m = __ballot((keep >> q) & 1u);
                    if (lane == 0) sMask[q][kMasked ? wave : 0] = m;
                }
            } else {
                at_pos = block_count_n<kThreads>(keep != 0u, scan_lds, &cnt);
            }
            if (keep) {
                sA[at_pos] = A;
                sB[at_pos] = Bv;
                sC[at_pos] = make_float4(Cc.x, Cc.y, __int_as_float(start + tid), 0.f);
                sR[at_pos] = uint32_t(rec);
                if (!plain_colour(Bv.z, Bv.w, Cc.x)) sPlain = 0;
            }
            for (int i = tid; i < kSumArrays * kSums; i += kThreads) red[i] = 0.f;
            __syncthreads();

            // a Gaussian's nine sums of the wave to the tile's sums
            auto put = [&](uint32_t k, int i, float v) {
                float *at = &red[wave / 2 * kSums + k * kAccRows + i];
                if (kWaves == 1) *at = v; else atomicAdd(at, v);
            };
            // the staged Gaussians of this wave, back to front
            auto walk_back = [&](auto visit) {
                if (!kMasked) {
                    for (int k = int(cnt) - 1; k >= 0; --k) {
                        const float4 A = sA[k];
                        const float4 Bv = sB[k];
                        const float4 Ck = sC[k];
                        visit(k, A, Bv, Ck);
                    }
                    return;
                }
#pragma unroll 1
                for (int w = (int(cnt) - 1) / kWave; w >= 0; --w) {
                    uint64_t m = sMask[wave][kMasked ? w : 0];
                    m = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(m >> 32)))) << 32) |
                        uint32_t(__builtin_amdgcn_readfirstlane(int(m)));
                    if (m == 0ull) continue;
                    int k = w * kWave + 63 - __builtin_clzll(m);
                    float4 A = sA[k], Bv = sB[k], Ck = sC[k];
                    do {
                        m ^= 1ull << (k & (kWave - 1));
                        const int next = m ? w * kWave + 63 - __builtin_clzll(m) : k;
                        const float4 An = sA[next], Bn = sB[next], Cn = sC[next];
                        visit(k, A, Bv, Ck);
                        A = An;
                        Bv = Bn;
                        Ck = Cn;
                        k = next;
                    } while (m);
                }
            };
            if (__builtin_amdgcn_readfirstlane(sPlain) == 0) {   // careful
                walk_back([&](int k, const float4 &A, const float4 &Bv, const float4 &Ck) {
                    const int pos = __float_as_int(Ck.z);
                    float v[kAccRows];
    #pragma unroll
                    for (int i = 0; i < kAccRows; ++i) v[i] = 0.f;
    #pragma unroll
                    for (int i = 0; i < kPix; ++i) {
                        const float dx = A.x - fpx, dy = A.y - fpy[i];
                        const float pw = eval_power(A, Bv, dx, dy);
                        if (pos < last[i] && !(pw < Ck.y)) {
                            const float at = Bv.y * __builtin_amdgcn_exp2f(pw);
                            const float alpha = clamp_alpha(at, amax);
                            const float oma = 1.f - alpha;
                            if (kStored) {
                                kc[i] = max(kc[i] - 1, 0);
                                T[i] = srow[int64_t(kc[i]) * kTilePix + first + i * kThreads];
                            } else {
                                T[i] *= __builtin_amdgcn_rcpf(oma);
                            }
                            const float cg = fmaf(Bv.z, g0[i], fmaf(Bv.w, g1[i], Ck.x * g2[i]));
                            const float w = alpha * T[i];
                            const float dal = T[i] * (cg - S[i]);
                            S[i] = fmaf(alpha, cg, oma * S[i]);   // (an infinity stays one)
                            const float n = -(at * (at < amax ? dal : 0.f));
                            v[0] = fmaf(n, dx, v[0]);
                            v[1] = fmaf(n, dy, v[1]);
                            v[2] = fmaf(n * dx, dx, v[2]);
                            v[3] = fmaf(n * dx, dy, v[3]);
                            v[4] = fmaf(n * dy, dy, v[4]);
                            v[5] += n;
                            v[6] = fmaf(w, g0[i], v[6]);
                            v[7] = fmaf(w, g1[i], v[7]);
                            v[8] = fmaf(w, g2[i], v[8]);
                        }
                    }
    #pragma unroll 1
                    for (int i = 0; i < kAccRows; ++i) {
                        float x = v[0];   // v[i], without indexing registers
    #pragma unroll
                        for (int j = 1; j < kAccRows; ++j) x = i == j ? v[j] : x;
                        x = wave_sum(x);
                        if (lane == 0) put(uint32_t(k), i, x);
                    }
                });
            } else {
                int slots = 0;   // Gaussians in the buffer (wave-uniform)
                // sums the buffered Gaussians' values: lane m < n * 9 owns value m
                auto flush = [&](int n) {
                    wave_sync();
                    if (lane < n * kAccRows) {
                        const float4 *row = reinterpret_cast<const float4 *>(tb + lane * kTStride);
                        const float4 a = row[0], b = row[1], c = row[2], d = row[3];
                        const int slot = lane / kAccRows;
                        put(sK[wave][slot], lane - slot * kAccRows,
                            (((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w))) +
                                (((c.x + c.y) + (c.z + c.w)) + ((d.x + d.y) + (d.z + d.w))));
                    }
                    wave_sync();
                };
                auto walk = [&](int k, const float4 &A, const float4 &Bv, const float4 &Ck) {
                    const int pos = __float_as_int(Ck.z);
                    const float dx = A.x - fpx;
                    const float qx = A.z * dx;
                    float N = 0.f, N1 = 0.f, N2 = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
                    bool some = false;   // (uniform)
    #pragma unroll
                    for (int i = 0; i < kPix; ++i) {
                        // eval_power, its terms of dx shared
                        const float dy = A.y - fpy[i];
                        const float u = fmaf(A.w, dx, Bv.x * dy);
                        const float pw = fmaf(qx, dx, u * dy);
                        const bool hit = pos < last[i] && !(pw < Ck.y);
                        if (__ballot(hit) == 0) continue;
                        some = true;
                        const float e = Bv.y * __builtin_amdgcn_exp2f(pw);
                        const float at = hit ? e : 0.f;
                        const float alpha = clamp_alpha(at, amax);
                        if (kStored) {   // transmittance in front of it, as stored
                            if (hit) {
                                kc[i] = max(kc[i] - 1, 0);
                                T[i] = srow[int64_t(kc[i]) * kTilePix + first + i * kThreads];
                            }
                        } else {
                            T[i] *= __builtin_amdgcn_rcpf(1.f - alpha);   // transmittance in front of it
                        }
                        // (the gradient sums use explicit FMAs: the build does
                        // not contract, so that both passes take the cutoff
                        // decisions with the same instructions)
                        // dL/dalpha = T (c - colour behind) . dL/dC; S becomes
                        // alpha cg + (1 - alpha) S
                        const float cg = fmaf(Bv.z, g0[i], fmaf(Bv.w, g1[i], Ck.x * g2[i]));
                        const float w = alpha * T[i];
                        const float dS = cg - S[i];
                        const float dal = T[i] * dS;
                        S[i] = fmaf(alpha, dS, S[i]);
                        const float n = at * (at < amax ? -dal : 0.f);
                        const float ny = n * dy;
                        N += n;
                        N1 += ny;
                        N2 = fmaf(ny, dy, N2);
                        c0 = fmaf(w, g0[i], c0);
                        c1 = fmaf(w, g1[i], c1);
                        c2 = fmaf(w, g2[i], c2);
                    }
                    if (!some) return;
                    const float nx = N * dx;
                    float v[kAccRows] = {nx, N1, nx * dx, N1 * dx, N2, N, c0, c1, c2};
                    quarter_rows(v);
                    float *slot = tb + slots * kAccRows * kTStride;
                    slot[part] = v[0];
                    slot[part + 4 * kTStride] = v[4];
                    slot[part8] = v[8];   // (lanes that hold the same part store the same bits)
                    if (lane == 0) sK[wave][slots] = uint32_t(k);
                    if (++slots == kGroup) {
                        flush(kGroup);
                        slots = 0;
                    }
                };
                walk_back(walk);
                if (slots > 0) flush(slots);
            }
            __syncthreads();
            // The conic gradient becomes the gradient of the dilated covariance
            // (-K dK K), both go back to level-0 units, and N becomes the
            // opacity's gradient (n = -dL/dalpha o exp(..)) ...
            for (int k = tid; k < int(cnt); k += kThreads) {
                if (kMasked && keep == 0u) continue;   // (k = tid: this thread's own)
                float *v = red + k * kAccRows;
                if (kSumArrays == 2)
    #pragma unroll
                    for (int i = 0; i < kAccRows; ++i) v[i] += v[kSums + i];
                const float a = conic_a(sA[k]), b = conic_b(sA[k]), c = conic_c(sB[k]);
                // mean gradient K (sum n d); conic gradient (sum n d d^T) / 2
                const float P = v[0], Q = v[1];
                const float ga = 0.5f * v[2], gb = 0.5f * v[3], gc = 0.5f * v[4];
                const float k00 = a * ga + b * gb, k01 = a * gb + b * gc;
                const float k10 = b * ga + c * gb, k11 = b * gb + c * gc;
                const float s2 = sc * sc;
                v[0] = (a * P + b * Q) * sc;
                v[1] = (b * P + c * Q) * sc;
                v[2] = -(k00 * a + k01 * b) * s2;
                v[3] = -(k00 * b + k01 * c) * s2;
                v[4] = -(k10 * b + k11 * c) * s2;
                v[5] = -v[5] / sB[k].y;
            }
            __syncthreads();
            // ... then one atomic per (Gaussian, quantity) for the whole tile, with
            // consecutive threads on consecutive accumulators of a record (a
            // record's nine accumulators are contiguous)
            for (int idx = tid; idx < int(cnt) * kAccRows; idx += kThreads) {
                const int k = idx / kAccRows, i = idx - k * kAccRows;
                const float v = red[idx];
                if (v != 0.f) atomicAdd(&acc[int64_t(sR[k]) * kAccRows + i], v);   // sR unsigned
            }
        }
    }
    if (queued) queue_retire(queue, kQueueNextBwd, kQueueDoneBwd);
}

__global__ void fill_f32_kernel(float *p, int64_t count, float v) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

// Four floats per thread, one 16-byte store each (p 16-byte aligned); the
// last thread also writes a tail of fewer than four.
__global__ void fill_f32x4_kernel(float *p, int64_t count, float v) {
    const int64_t e = 4 * (int64_t(blockIdx.x) * blockDim.x + threadIdx.x);
    if (e + 4 <= count) {
        *reinterpret_cast<float4 *>(p + e) = make_float4(v, v, v, v);
    } else {
        for (int64_t k = e; k < count; ++k) p[k] = v;
    }
}

// Workgroups of a persistent launch: as many as the chip holds at once (CUs x
// resident workgroups per CU for the kernel), looked up once per kernel.  Any
// count is correct (workgroups only take tiles from the queue); this one
// keeps every CU busy with no workgroup left waiting for a slot.
template <auto kKernel>
static int persistent_grid(int threads) {
    static std::atomic<int> cached{0};
    int g = cached.load(std::memory_order_relaxed);
    if (g > 0) return g;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kKernel, threads, 0) != hipSuccess || cus <= 0 ||
        per_cu <= 0)
        return 2048;
    g = cus * per_cu;
    cached.store(g, std::memory_order_relaxed);
    return g;
}

static void launch_fill(float *p, int64_t count, float v, hipStream_t st) {
    if (reinterpret_cast<uintptr_t>(p) % 16 == 0)
        hipLaunchKernelGGL(fill_f32x4_kernel, dim3((count + 1023) / 1024), dim3(256), 0, st, p, count, v);
    else
        hipLaunchKernelGGL(fill_f32_kernel, dim3((count + 255) / 256), dim3(256), 0, st, p, count, v);
}

gs_status launch_project_backward(const gs_settings &s, const float *params, int64_t n,
                                  int64_t n_cap, const gs_view *views, int32_t n_views,
                                  const float *acc, float *grad, hipStream_t st);
gs_status launch_project_backward_adam(const gs_settings &s, float *params, int64_t n, int64_t n_cap,
                                       const gs_view *views, int32_t n_views, const float *acc,
                                       float *m, float *v, const float *lr_rows, double beta1,
                                       double beta2, double eps, int32_t step, const int32_t *d_step,
                                       void *proj_out, hipStream_t st);

}  // namespace gs

extern "C" gs_status gs_render_fwd(const gs_settings *s, const void *proj_ws, int64_t n_cap,
                                   int32_t n_views, const void *sort_ws, int64_t pair_cap,
                                   const gs_target *targets, int32_t n_targets, int32_t total_tiles,
                                   float *out_rgb, float *out_T, int32_t *out_last,
                                   int32_t *out_ncontrib, int32_t *out_nevals, void *stream) {
    using namespace gs;
    if (!valid_settings(s) || !proj_ws || !sort_ws || !targets || n_cap <= 0 || n_cap % 64 ||
        n_views <= 0 || n_targets <= 0 || total_tiles <= 0 || pair_cap <= 0 || !out_rgb ||
        !out_T || !out_last || pair_cap > kMaxPairs || int64_t(n_views) * n_cap > kMaxRecords)
        return GS_ERR_INVALID_ARGUMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Sorted srt = sorted_at(sort_ws, n_views, n_targets, n_cap, pair_cap, total_tiles);
    const Proj proj = proj_at(const_cast<void *>(proj_ws), int64_t(n_views) * n_cap);
    auto launch = [&](auto waves) {
        constexpr int kWaves = decltype(waves)::value;
        if (s->schedule == 1)
            hipLaunchKernelGGL((render_fwd_kernel<kWaves, false, false, true>),
                               dim3(persistent_grid<render_fwd_kernel<kWaves, false, false, true>>(kWave * kWaves)),
                               dim3(kWave * kWaves), 0, st, *s, proj, n_cap, srt, targets, n_targets, out_rgb, out_T,
                               out_last, nullptr, nullptr, nullptr, TStore{nullptr, nullptr, nullptr, 0}, srt.order,
                               srt.queue, total_tiles);
        else
            hipLaunchKernelGGL(render_fwd_kernel<kWaves>, dim3(total_tiles), dim3(kWave * kWaves), 0, st, *s, proj,
                               n_cap, srt, targets, n_targets, out_rgb, out_T, out_last, nullptr, nullptr);
    };
    if (out_ncontrib || out_nevals)
        hipLaunchKernelGGL((render_fwd_kernel<4, true>), dim3(total_tiles), dim3(kTilePix), 0, st, *s, proj, n_cap,
                           srt, targets, n_targets, out_rgb, out_T, out_last, out_ncontrib, out_nevals);
    else if (total_tiles <= (s->schedule == 1 ? kFwdQueuedFour : kFwdTilesFour))
        launch(std::integral_constant<int, 4>{});
    else
        launch(std::integral_constant<int, 2>{});
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_raster_bwd(const gs_settings *s, const void *proj_ws, int64_t n_cap,
                                   int32_t n_views, const void *sort_ws, int64_t pair_cap,
                                   const gs_target *targets, int32_t n_targets, int32_t total_tiles,
                                   const float *out_T, const int32_t *out_last,
                                   const float *dL_drgb, void *accum_ws, void *stream) {
    using namespace gs;
    if (!valid_settings(s) || !proj_ws || !sort_ws || !targets || !out_T || !out_last || !dL_drgb ||
        !accum_ws || n_cap <= 0 || n_cap % 64 || n_views <= 0 || n_targets <= 0 ||
        total_tiles <= 0 || pair_cap <= 0 || pair_cap > kMaxPairs ||
        int64_t(n_views) * n_cap > kMaxRecords)
        return GS_ERR_INVALID_ARGUMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t records = int64_t(n_views) * n_cap;
    const Sorted srt = sorted_at(sort_ws, n_views, n_targets, n_cap, pair_cap, total_tiles);
    const Proj proj = proj_at(const_cast<void *>(proj_ws), records);
    float *acc = static_cast<float *>(accum_ws);
    const int64_t acc_n = int64_t(kAccRows) * records;
    launch_fill(acc, acc_n, 0.f, st);
    const TStore none{nullptr, nullptr, nullptr, 0};
    if (s->schedule >= 1) {   // persistent workgroups over the cost-ordered tile queue
        switch (s->bwd_waves) {
            case 1:
                hipLaunchKernelGGL((render_bwd_kernel<1, false, true>),
                                   dim3(persistent_grid<render_bwd_kernel<1, false, true>>(64)), dim3(64), 0, st,
                                   *s, proj, n_cap, srt, targets, n_targets, out_T, out_last, dL_drgb, acc,
                                   nullptr, none, srt.order, srt.queue, total_tiles);
                break;
            case 2:
                hipLaunchKernelGGL((render_bwd_kernel<2, false, true>),
                                   dim3(persistent_grid<render_bwd_kernel<2, false, true>>(128)), dim3(128), 0, st,
                                   *s, proj, n_cap, srt, targets, n_targets, out_T, out_last, dL_drgb, acc,
                                   nullptr, none, srt.order, srt.queue, total_tiles);
                break;
            default:
                hipLaunchKernelGGL((render_bwd_kernel<4, false, true>),
                                   dim3(persistent_grid<render_bwd_kernel<4, false, true>>(256)), dim3(256), 0, st,
                                   *s, proj, n_cap, srt, targets, n_targets, out_T, out_last, dL_drgb, acc,
                                   nullptr, none, srt.order, srt.queue, total_tiles);
                break;
        }
    } else {
        switch (s->bwd_waves) {
            case 1:
                hipLaunchKernelGGL(render_bwd_kernel<1>, dim3(total_tiles), dim3(64), 0, st, *s, proj, n_cap,
                                   srt, targets, n_targets, out_T, out_last, dL_drgb, acc);
                break;
            case 2:
                hipLaunchKernelGGL(render_bwd_kernel<2>, dim3(total_tiles), dim3(128), 0, st, *s, proj, n_cap,
                                   srt, targets, n_targets, out_T, out_last, dL_drgb, acc);
                break;
            default:
                hipLaunchKernelGGL(render_bwd_kernel<4>, dim3(total_tiles), dim3(256), 0, st, *s, proj, n_cap,
                                   srt, targets, n_targets, out_T, out_last, dL_drgb, acc);
                break;
        }
    }
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_render_fwd_store(const gs_settings *s, const void *proj_ws, int64_t n_cap,
                                         int32_t n_views, const void *sort_ws, int64_t pair_cap,
                                         const gs_target *targets, int32_t n_targets,
                                         int32_t total_tiles, float *out_rgb, float *out_T,
                                         int32_t *out_last, int32_t *out_ncontrib, int32_t *tile_steps,
                                         int64_t *store_base, float *store, int64_t store_cap,
                                         void *stream) {
    using namespace gs;
    if (!valid_settings(s) || !proj_ws || !sort_ws || !targets || n_cap <= 0 || n_cap % 64 ||
        n_views <= 0 || n_targets <= 0 || total_tiles <= 0 || pair_cap <= 0 || !out_rgb || !out_T ||
        !out_last || !out_ncontrib || !tile_steps || !store_base || !store || store_cap < 0 ||
        pair_cap > kMaxPairs || int64_t(n_views) * n_cap > kMaxRecords)
        return GS_ERR_INVALID_ARGUMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Sorted srt = sorted_at(sort_ws, n_views, n_targets, n_cap, pair_cap, total_tiles);
    const Proj proj = proj_at(const_cast<void *>(proj_ws), int64_t(n_views) * n_cap);
    // counts, the store layout, then the forward again writing the store
    hipLaunchKernelGGL((render_fwd_kernel<4, true>), dim3(total_tiles), dim3(kTilePix), 0, st, *s, proj, n_cap, srt,
                       targets, n_targets, out_rgb, out_T, out_last, out_ncontrib, nullptr, tile_steps,
                       TStore{nullptr, nullptr, nullptr, 0});
    hipLaunchKernelGGL(store_base_kernel, dim3(1), dim3(1024), 0, st, tile_steps, int64_t(total_tiles), store_base);
    hipLaunchKernelGGL((render_fwd_kernel<4, false, true>), dim3(total_tiles), dim3(kTilePix), 0, st, *s, proj,
                       n_cap, srt, targets, n_targets, out_rgb, out_T, out_last, nullptr, nullptr, nullptr,
                       TStore{store_base, store_base + total_tiles, store, store_cap});
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_raster_bwd_stored(const gs_settings *s, const void *proj_ws, int64_t n_cap,
                                          int32_t n_views, const void *sort_ws, int64_t pair_cap,
                                          const gs_target *targets, int32_t n_targets,
                                          int32_t total_tiles, const int32_t *out_last,
                                          const int32_t *out_ncontrib, const int64_t *store_base,
                                          const float *store, int64_t store_cap, const float *dL_drgb,
                                          void *accum_ws, void *stream) {
    using namespace gs;
    if (!valid_settings(s) || !proj_ws || !sort_ws || !targets || !out_last || !out_ncontrib ||
        !store_base || !store || store_cap < 0 || !dL_drgb || !accum_ws || n_cap <= 0 || n_cap % 64 ||
        n_views <= 0 || n_targets <= 0 || total_tiles <= 0 || pair_cap <= 0 || pair_cap > kMaxPairs ||
        int64_t(n_views) * n_cap > kMaxRecords)
        return GS_ERR_INVALID_ARGUMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t records = int64_t(n_views) * n_cap;
    const Sorted srt = sorted_at(sort_ws, n_views, n_targets, n_cap, pair_cap, total_tiles);
    const Proj proj = proj_at(const_cast<void *>(proj_ws), records);
    float *acc = static_cast<float *>(accum_ws);
    launch_fill(acc, int64_t(kAccRows) * records, 0.f, st);
    const TStore ts{store_base, store_base + total_tiles, const_cast<float *>(store), store_cap};
    switch (s->bwd_waves) {
        case 1:
            hipLaunchKernelGGL((render_bwd_kernel<1, true>), dim3(total_tiles), dim3(64), 0, st, *s, proj, n_cap,
                               srt, targets, n_targets, nullptr, out_last, dL_drgb, acc, out_ncontrib, ts);
            break;
        case 2:
            hipLaunchKernelGGL((render_bwd_kernel<2, true>), dim3(total_tiles), dim3(128), 0, st, *s, proj, n_cap,
                               srt, targets, n_targets, nullptr, out_last, dL_drgb, acc, out_ncontrib, ts);
            break;
        default:
            hipLaunchKernelGGL((render_bwd_kernel<4, true>), dim3(total_tiles), dim3(256), 0, st, *s, proj, n_cap,
                               srt, targets, n_targets, nullptr, out_last, dL_drgb, acc, out_ncontrib, ts);
            break;
    }
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_project_bwd(const gs_settings *s, const float *params, int64_t n,
                                    int64_t n_cap, const gs_view *views, int32_t n_views,
                                    const void *accum_ws, float *grad, void *stream) {
    using namespace gs;
    if (!valid_settings(s) || !params || !views || !accum_ws || !grad || n < 0 || n_cap <= 0 ||
        n > n_cap || n_cap % 64 || n_views <= 0)
        return GS_ERR_INVALID_ARGUMENT;
    return launch_project_backward(*s, params, n, n_cap, views, n_views,
                                   static_cast<const float *>(accum_ws), grad,
                                   static_cast<hipStream_t>(stream));
}

extern "C" gs_status gs_project_bwd_adam(const gs_settings *s, float *params, int64_t n,
                                         int64_t n_cap, const gs_view *views, int32_t n_views,
                                         const void *accum_ws, float *m, float *v,
                                         const float *lr_rows, double beta1, double beta2,
                                         double eps, int32_t step, const int32_t *d_step,
                                         void *proj_out, void *stream) {
    using namespace gs;
    if (!valid_settings(s) || !params || !views || !accum_ws || !m || !v || !lr_rows || n < 0 ||
        n_cap <= 0 || n > n_cap || n_cap % 64 || n_views <= 0 || (step < 1 && !d_step) ||
        !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps >= 0.0))
        return GS_ERR_INVALID_ARGUMENT;
    return launch_project_backward_adam(*s, params, n, n_cap, views, n_views,
                                        static_cast<const float *>(accum_ws), m, v, lr_rows, beta1,
                                        beta2, eps, step, step < 1 ? d_step : nullptr, proj_out,
                                        static_cast<hipStream_t>(stream));
}

extern "C" gs_status gs_render_bwd(const gs_settings *s, const float *params, int64_t n,
                                   int64_t n_cap, const gs_view *views, int32_t n_views,
                                   const void *proj_ws, const void *sort_ws, int64_t pair_cap,
                                   const gs_target *targets, int32_t n_targets, int32_t total_tiles,
                                   const float *out_T, const int32_t *out_last,
                                   const float *dL_drgb, void *accum_ws, float *grad,
                                   void *stream) {
    if (!params || !grad || n < 0 || n > n_cap || !views) return GS_ERR_INVALID_ARGUMENT;
    gs_status r = gs_raster_bwd(s, proj_ws, n_cap, n_views, sort_ws, pair_cap, targets, n_targets,
                                total_tiles, out_T, out_last, dL_drgb, accum_ws, stream);
    if (r != GS_OK) return r;
    return gs_project_bwd(s, params, n, n_cap, views, n_views, accum_ws, grad, stream);
}

extern "C" gs_status gs_render_bwd_adam(const gs_settings *s, float *params, int64_t n,
                                        int64_t n_cap, const gs_view *views, int32_t n_views,
                                        const void *proj_ws, const void *sort_ws, int64_t pair_cap,
                                        const gs_target *targets, int32_t n_targets,
                                        int32_t total_tiles, const float *out_T,
                                        const int32_t *out_last, const float *dL_drgb,
                                        void *accum_ws, float *m, float *v, const float *lr_rows,
                                        double beta1, double beta2, double eps, int32_t step,
                                        const int32_t *d_step, void *proj_out, void *stream) {
    if (!params || !m || !v || !lr_rows || n < 0 || n > n_cap || !views || (step < 1 && !d_step))
        return GS_ERR_INVALID_ARGUMENT;
    gs_status r = gs_raster_bwd(s, proj_ws, n_cap, n_views, sort_ws, pair_cap, targets, n_targets,
                                total_tiles, out_T, out_last, dL_drgb, accum_ws, stream);
    if (r != GS_OK) return r;
    return gs_project_bwd_adam(s, params, n, n_cap, views, n_views, accum_ws, m, v, lr_rows, beta1,
                               beta2, eps, step, d_step, proj_out, stream);
}

namespace gs {
__global__ void step_advance_kernel(int32_t *d_step) {
    if (threadIdx.x == 0) *d_step += 1;
}
}  // namespace gs

extern "C" gs_status gs_step_advance(int32_t *d_step, void *stream) {
    if (!d_step) return GS_ERR_INVALID_ARGUMENT;
    hipLaunchKernelGGL(gs::step_advance_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                       d_step);
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_fill(float *dst, int64_t count, float value, void *stream) {
    if (!dst || count < 0) return GS_ERR_INVALID_ARGUMENT;
    if (count == 0) return GS_OK;
    gs::launch_fill(dst, count, value, static_cast<hipStream_t>(stream));
    GS_CHECK_LAUNCH();
    return GS_OK;
}
