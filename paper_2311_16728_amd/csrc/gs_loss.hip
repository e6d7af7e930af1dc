// Gaussian pyramid (Section 3.4) and the photometric loss of Eq. 4 with its
// gradient, over every render target at once.
//
// The loss uses the rasteriser's tiling (the target's tile shape, 256 pixels):
// one 256-thread workgroup per tile stages the tile plus a 5-pixel halo of
// render and target
// in LDS, runs the separable 11-tap Gaussian window horizontally then
// vertically for the five SSIM moments, and writes per-pixel partial
// derivatives of the SSIM map (with respect to the window mean, the second
// moment and the cross moment).  A second pass filters those three maps with
// the same (self-adjoint) window, over larger blocks, and forms dL/dI.  Partial
// sums are reduced per tile and then per target in a fixed order, so the loss is
// deterministic.
#include "gs_internal.hpp"

namespace gs {

constexpr int kR = 5;                       // SSIM window radius (11 taps)

struct Window {
    float w[2 * kR + 1];
};

static Window ssim_window() {
    Window W;
    double v[2 * kR + 1], s = 0;
    for (int i = -kR; i <= kR; ++i) {
        v[i + kR] = std::exp(-double(i * i) / (2.0 * 1.5 * 1.5));
        s += v[i + kR];
    }
    for (int i = 0; i < 2 * kR + 1; ++i) W.w[i] = float(v[i] / s);
    return W;
}

__device__ __forceinline__ int find_target_loss(const gs_target *__restrict__ targets, int n,
                                                int tile) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (targets[mid].tile_offset <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Tile geometry of the loss kernels: the target's raster tile (TW x TH
// pixels, TW * TH = 256) plus an R-pixel halo, HX x HY.  Each kernel
// dispatches on the target's tile width to a body compiled for that shape;
// LDS is sized for the largest (16 x 16: 48 x 26 halo with its padded rows;
// 32 x 8: 18 x 32 horizontal pass).
// LDS row stride of a halo window: the horizontal passes read 32 / TW rows of
// TW consecutive floats per half wave; row strides that put those rows on
// disjoint banks keep the reads conflict-free (16-wide: 48, two rows 16
// banks apart; 8-wide: 24, four rows at bank offsets 0, 24, 16, 8).
template <int TW>
__host__ __device__ constexpr int halo_stride() {
    return TW == 16 ? 48 : TW == 8 ? 24 : TW + 2 * kR;
}
constexpr int kHaloMax = 48 * (16 + 2 * kR);   // the largest of the three shapes (16 x 16)
static_assert(halo_stride<8>() * (32 + 2 * kR) <= kHaloMax && halo_stride<32>() * (8 + 2 * kR) <= kHaloMax,
              "halo buffers");
constexpr int kHPassMax = 32 * (8 + 2 * kR);

// The HX x HY window of kP channel planes around the tile, zero outside the
// image: fetched into registers (kHaloRounds values per plane and thread,
// every load unconditional at a clamped address, so all are in flight
// together), then put into LDS (row stride halo_stride<TW>()).  Fetching
// the next channel while the current one is filtered hides the loads.
template <int TW>
__host__ __device__ constexpr int halo_rounds() {
    return ((TW + 2 * kR) * (kTilePix / TW + 2 * kR) + kTilePix - 1) / kTilePix;
}
template <int TW, int kP>
struct Halo {
    float v[kP][halo_rounds<TW>()];   // as loaded (clamped address)
    uint32_t in;                      // bit r: round r's pixel lies in the image
};
template <int TW, int kP>
__device__ __forceinline__ void fetch_halo(const float *const (&planes)[kP], int W, int H, int x0, int y0,
                                           Halo<TW, kP> &hv) {
    constexpr int TH = kTilePix / TW, HX = TW + 2 * kR, HY = TH + 2 * kR;
    constexpr int kRounds = halo_rounds<TW>();
    static_assert(kRounds <= 32, "one bit per round");
    hv.in = 0u;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int i = threadIdx.x + r * kTilePix;
        const int yy = i / HX, xx = i % HX;
        const int gx = x0 - kR + xx, gy = y0 - kR + yy;
        const bool in = i < HX * HY && gx >= 0 && gx < W && gy >= 0 && gy < H;
        const int64_t at = int64_t(min(max(gy, 0), H - 1)) * W + min(max(gx, 0), W - 1);
        hv.in |= uint32_t(in) << r;
        // (zeroed when put, so that nothing waits for the loads before then)
#pragma unroll
        for (int p = 0; p < kP; ++p) hv.v[p][r] = planes[p][at];
    }
}
template <int TW, int kP>
__device__ __forceinline__ void put_halo(const Halo<TW, kP> &hv, float *const (&dst)[kP]) {
    constexpr int HX = TW + 2 * kR, HY = kTilePix / TW + 2 * kR, HS = halo_stride<TW>();
#pragma unroll
    for (int r = 0; r < halo_rounds<TW>(); ++r) {
        const int i = threadIdx.x + r * kTilePix;
        if (i < HX * HY) {
            const bool in = (hv.in >> r) & 1u;
#pragma unroll
            for (int p = 0; p < kP; ++p) dst[p][(i / HX) * HS + i % HX] = in ? hv.v[p][r] : 0.f;
        }
    }
}

struct alignas(16) SsimLds {
    float sx[kHaloMax];
    float sy[kHaloMax];
    float h[5][kHPassMax];
    float red[2][kTilePix / kWave];
};

template <int TW>
__device__ __forceinline__ void ssim_fwd_tile(const float *__restrict__ render,
                                              const float *__restrict__ target, const gs_target &t,
                                              int tile, const Window &win, float *__restrict__ maps,
                                              float *__restrict__ partial, SsimLds &L) {
    constexpr int TH = kTilePix / TW, HY = TH + 2 * kR, HS = halo_stride<TW>();
    const float C1 = 0.01f * 0.01f, C2 = 0.03f * 0.03f;
    const int tid = threadIdx.x;
    const int local = tile - t.tile_offset;
    const int x0 = (local % t.tiles_x) * TW, y0 = (local / t.tiles_x) * TH;
    const int lx = tid % TW, ly = tid / TW;
    const int px = x0 + lx, py = y0 + ly;
    const bool inside = px < t.width && py < t.height;
    const int64_t HW = int64_t(t.width) * t.height;
    const int64_t pix = int64_t(py) * t.width + px;
    float l1 = 0.f, ss = 0.f;
    Halo<TW, 2> hv;
    auto fetch = [&](int c) {
        const float *const planes[2] = {render + 3 * t.pix_offset + c * HW, target + 3 * t.pix_offset + c * HW};
        fetch_halo<TW, 2>(planes, t.width, t.height, x0, y0, hv);
    };
    float *const dst[2] = {L.sx, L.sy};
    fetch(0);
    for (int c = 0; c < 3; ++c) {
        __syncthreads();   // the previous channel's reads of the windows are done
        put_halo<TW, 2>(hv, dst);
        __syncthreads();
        if (c + 1 < 3) fetch(c + 1);
        // two horizontally adjacent outputs per thread (one round for 16-
        // and 8-wide tiles): each input and its products are formed once;
        // every output sums its taps in the same order as one alone would
        constexpr int kTaps = 2 * kR + 1;
#pragma unroll
        for (int s2 = tid; s2 < HY * (TW / 2); s2 += kTilePix) {
            const int r = s2 / (TW / 2), cc = 2 * (s2 % (TW / 2));
            const float *rx = L.sx + r * HS + cc, *ry = L.sy + r * HS + cc;
            float m1[2] = {0, 0}, m2[2] = {0, 0}, e11[2] = {0, 0}, e22[2] = {0, 0}, e12[2] = {0, 0};
#pragma unroll
            for (int k = 0; k <= kTaps; ++k) {
                const float a = rx[k], b = ry[k];
                const float aa = a * a, bb = b * b, ab = a * b;
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int t = k - o;   // tap of output o
                    if (t < 0 || t >= kTaps) continue;
                    const float w = win.w[t];
                    m1[o] = fmaf(w, a, m1[o]);
                    m2[o] = fmaf(w, b, m2[o]);
                    e11[o] = fmaf(w, aa, e11[o]);
                    e22[o] = fmaf(w, bb, e22[o]);
                    e12[o] = fmaf(w, ab, e12[o]);
                }
            }
            const int i = r * TW + cc;
            *reinterpret_cast<float2 *>(&L.h[0][i]) = make_float2(m1[0], m1[1]);
            *reinterpret_cast<float2 *>(&L.h[1][i]) = make_float2(m2[0], m2[1]);
            *reinterpret_cast<float2 *>(&L.h[2][i]) = make_float2(e11[0], e11[1]);
            *reinterpret_cast<float2 *>(&L.h[3][i]) = make_float2(e22[0], e22[1]);
            *reinterpret_cast<float2 *>(&L.h[4][i]) = make_float2(e12[0], e12[1]);
        }
        __syncthreads();
        float mx = 0, my = 0, exx = 0, eyy = 0, exy = 0;
#pragma unroll
        for (int k = 0; k < 2 * kR + 1; ++k) {
            const float w = win.w[k];
            const int i = (ly + k) * TW + lx;
            mx = fmaf(w, L.h[0][i], mx);
            my = fmaf(w, L.h[1][i], my);
            exx = fmaf(w, L.h[2][i], exx);
            eyy = fmaf(w, L.h[3][i], eyy);
            exy = fmaf(w, L.h[4][i], exy);
        }
        if (inside) {
            const float vx = exx - mx * mx, vy = eyy - my * my, cxy = exy - mx * my;
            const float A1 = 2.f * mx * my + C1, A2 = 2.f * cxy + C2;
            const float B1 = mx * mx + my * my + C1, B2 = vx + vy + C2;
            // B1 >= C1 and B2 >= C2 (up to rounding of the variances): the
            // hardware reciprocal (1 ulp) instead of four IEEE divisions
            const float iB1 = __builtin_amdgcn_rcpf(B1), iB2 = __builtin_amdgcn_rcpf(B2);
            const float iB1B2 = iB1 * iB2;
            const float S = A1 * A2 * iB1B2;
            ss += S;
            const int ci = (ly + kR) * HS + lx + kR;
            l1 += fabsf(L.sx[ci] - L.sy[ci]);
            float *mp = maps + 9 * t.pix_offset + (3 * c) * HW;
            mp[pix] = 2.f * my * (A2 - A1) * iB1B2 - 2.f * mx * S * (iB1 - iB2);
            mp[HW + pix] = -S * iB2;
            mp[2 * HW + pix] = 2.f * A1 * iB1B2;
        }
    }
    l1 = wave_sum(l1);
    ss = wave_sum(ss);
    if (lane_id() == 0) { L.red[0][tid / kWave] = l1; L.red[1][tid / kWave] = ss; }
    __syncthreads();
    if (tid == 0) {
        float a = 0, b = 0;
        for (int w = 0; w < kTilePix / kWave; ++w) { a += L.red[0][w]; b += L.red[1][w]; }
        partial[2 * int64_t(tile)] = a;
        partial[2 * int64_t(tile) + 1] = b;
    }
}

// (seven workgroups per CU, as many as its LDS allows)
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7))) ssim_fwd_kernel(const float *__restrict__ render,
                                                       const float *__restrict__ target,
                                                       const gs_target *__restrict__ targets,
                                                       int n_targets, int total_tiles, Window win,
                                                       float *__restrict__ maps,
                                                       float *__restrict__ partial) {
    __shared__ SsimLds L;
    const int tile = int(xcd_tile(blockIdx.x, total_tiles));
    if (tile >= total_tiles) return;
    const gs_target t = targets[find_target_loss(targets, n_targets, tile)];
    switch (tile_shape(t.tile_w).w) {
        case 8: ssim_fwd_tile<8>(render, target, t, tile, win, maps, partial, L); break;
        case 32: ssim_fwd_tile<32>(render, target, t, tile, win, maps, partial, L); break;
        default: ssim_fwd_tile<16>(render, target, t, tile, win, maps, partial, L); break;
    }
}

// One block: per-target means from the tile partials (fixed order), then the
// weighted total.
// Eq. 4 per target (one workgroup each, tile partials summed in double in a
// fixed order), then the weighted sum over targets in target order.
__device__ __forceinline__ void loss_of_target(const gs_target *__restrict__ targets, int ti,
                                               float lambda, const float *__restrict__ partial,
                                               double *__restrict__ tloss, float *__restrict__ d_loss) {
    __shared__ double red[2][kTilePix / kWave];
    const gs_target t = targets[ti];
    const int nt = t.tiles_x * t.tiles_y;
    double a = 0, b = 0;
    // unrolled so that the loads of several tiles are in flight; the sums keep
    // their order
#pragma unroll 8
    for (int i = threadIdx.x; i < nt; i += blockDim.x) {
        a += partial[2 * int64_t(t.tile_offset + i)];
        b += partial[2 * int64_t(t.tile_offset + i) + 1];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if (lane_id() == 0) { red[0][threadIdx.x / kWave] = a; red[1][threadIdx.x / kWave] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sa = 0, sb = 0;
        for (int w = 0; w < kTilePix / kWave; ++w) { sa += red[0][w]; sb += red[1][w]; }
        const double n = 3.0 * double(t.width) * double(t.height);
        const double L = (1.0 - lambda) * sa / n + lambda * (1.0 - sb / n);
        tloss[ti] = double(t.weight) * L;
        if (d_loss) d_loss[ti] = float(L);
    }
    __syncthreads();   // red is reused by the next call
}

// The gradient filters the three maps over 32x32 blocks of one channel.
//
// Bound: VALU issue (a wave64 FMA takes 4 cycles here, an add 2, so the window's
// mirrored taps are added first: five adds and six FMAs per output, not eleven
// FMAs) and the latency of a block's steps, which as many workgroups as LDS and
// registers allow (six per CU) hide in part.  A thread filters four neighbours, in
// a row and then in a column, from registers: reading tap by tap from LDS took as
// long as the arithmetic.  32x32 blocks filter 1.3 rows per output row in the first
// pass (16x16 tiles: 1.6), and the maps go through two windows and row buffers one
// after the other.
// Measured, before -> now in us: 3 levels of 1200x680 27.4 -> 24.2; one level 23.1 ->
// 19.4; 32 keyframes of 3 levels 513 -> 407.  Not kept: the first pass as FP32 matrix
// products with the banded window (its 28 columns for 11 taps undo their rate: 34
// at 3 levels of 1200x680), 32x64 blocks of 512 threads (30), all row buffers at once
// with four workgroups per CU (26).  Nor is this layout kept for the forward: its
// moments have to be summed tap by tap (their rounding is what the gradient's
// error against 64 bits consists of), which leaves 37 against the tiles' 35; with
// mirrored taps and the moments taken about a value of the block it takes 28.5 and
// the error falls from 1.6e-5 to 4e-6, but results move by as much.

// A block's outputs, its staged window (rows and columns with the halo; the
// row count is rounded up to the staging's and the row stride to 16 bytes) and
// the rows of the first pass.
constexpr int kBlk = 32, kGroup = 4;            // a thread filters kGroup neighbours
constexpr int kWinRows = kBlk + 2 * kR;         // 42
constexpr int kStride = 44;
constexpr int kStageRounds = (kWinRows + 3) / 4;
constexpr int kWinSize = 4 * kStageRounds * kStride, kPassSize = kWinRows * kBlk;

// The work of a target's raster tile `local`, of nt: the items [begin, end) of the
// target's nb blocks in each of three channels (item i is block i % nb of channel
// i / nb), spread evenly and in order.  A tile has 256 pixels, so most take one
// item and some none.
struct Items {
    int nbx, nb, begin, end;
};
__device__ __forceinline__ Items loss_items(const gs_target &t, int local) {
    const int nbx = (t.width + kBlk - 1) / kBlk, nb = nbx * ((t.height + kBlk - 1) / kBlk);
    const uint32_t nt = uint32_t(t.tiles_x) * t.tiles_y;
    const double inv = 1.0 / double(nt);
    auto first = [&](uint32_t l) {   // floor(l m / nt), m = 3 nb
        const uint64_t p = uint64_t(l) * (3u * uint32_t(nb));
        uint64_t q = uint64_t(double(p) * inv);   // off by one at most
        if (q * nt > p) --q;
        if ((q + 1) * nt <= p) ++q;
        return int(q);
    };
    return Items{nbx, nb, first(uint32_t(local)), first(uint32_t(local) + 1)};
}

// The three maps around a block at (x0, y0), zero outside the image.  Wave w
// stages rows w, w + 4, ...: the row's part of address and test is scalar.
// Every load and store is unconditional, at a clamped address (stores that meet
// there store the same value), so that all loads are in flight together and
// none is moved to its store; put() waits for a plane's.
struct Stage {
    float v[3][kStageRounds];
    __device__ __forceinline__ void fetch(const float *maps, int64_t plane, int W, int H, int x0, int y0) {
        const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
        const uint32_t gx = uint32_t(min(max(x0 - kR + lane_id(), 0), W - 1));
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int k = 0; k < kStageRounds; ++k) {
                const int gy = min(max(y0 - kR + wave + 4 * k, 0), H - 1);
                v[p][k] = (maps + p * plane + int64_t(gy) * W)[gx];
            }
    }
    __device__ __forceinline__ void put(int p, int W, int H, int x0, int y0, float (&dst)[kWinSize]) const {
        const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
        const int lane = lane_id(), gx = x0 - kR + lane;
        const bool col = lane < kStride - 1 && gx >= 0 && gx < W;
        float *at = dst + min(lane, kStride - 1);
#pragma unroll
        for (int k = 0; k < kStageRounds; ++k) {
            const int r = wave + 4 * k, gy = y0 - kR + r;
            at[r * kStride] = col && gy >= 0 && gy < H ? v[p][k] : 0.f;
        }
    }
};

// The window over q[0 .. 10], mirrored taps added first.
__device__ __forceinline__ float window_at(const Window &win, const float *q) {
    float acc = win.w[kR] * q[kR];
#pragma unroll
    for (int k = kR - 1; k >= 0; --k) acc = fmaf(win.w[k], q[k] + q[2 * kR - k], acc);
    return acc;
}

// First pass, along rows: item s of kWinRows * (kBlk / kGroup) is kGroup outputs of
// one row, formed by filter(row, column).
template <typename Filter>
__device__ __forceinline__ void rows_pass(Filter filter) {
    constexpr int kPer = kBlk / kGroup;
#pragma unroll 1
    for (int s = threadIdx.x; s < kWinRows * kPer; s += kTilePix) filter(s / kPer, kGroup * (s % kPer));
}
// kGroup outputs of the window over q, to the row buffer.
__device__ __forceinline__ void row_out(const Window &win, const float *q, float *dst) {
    *reinterpret_cast<float4 *>(dst) = make_float4(window_at(win, q), window_at(win, q + 1), window_at(win, q + 2),
                                                   window_at(win, q + 3));
}
__device__ __forceinline__ void row_in(const float *src, float (&q)[16]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 v = reinterpret_cast<const float4 *>(src)[i];
        q[4 * i] = v.x, q[4 * i + 1] = v.y, q[4 * i + 2] = v.z, q[4 * i + 3] = v.w;
    }
}
// Second pass: kGroup outputs of a column of the row buffer.
__device__ __forceinline__ void column_out(const Window &win, const float *src, float (&f)[kGroup]) {
    float q[kGroup + 2 * kR];
#pragma unroll
    for (int k = 0; k < kGroup + 2 * kR; ++k) q[k] = src[k * kBlk];
#pragma unroll
    for (int o = 0; o < kGroup; ++o) f[o] = window_at(win, q + o);
}

struct alignas(16) SsimBwdLds {
    float s[2][kWinSize];
    float h[2][kPassSize];
};

// A few targets (kFold): workgroup 0 also forms the per-target losses and the
// total from the forward's tile partials before its tile (the sums and order
// of loss_few_kernel, one launch fewer).
constexpr int kLossOneBlockTargets = 8;
template <bool kFold>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) ssim_bwd_kernel(const float *__restrict__ render,
                                                       const float *__restrict__ target,
                                                       const gs_target *__restrict__ targets,
                                                       int n_targets, int total_tiles, Window win,
                                                       float lambda,
                                                       const float *__restrict__ maps,
                                                       float *__restrict__ dL,
                                                       const float *__restrict__ partial,
                                                       double *__restrict__ tloss,
                                                       float *__restrict__ d_loss,
                                                       float *__restrict__ d_total) {
    __shared__ SsimBwdLds L;
    if (kFold && blockIdx.x == 0) {   // uniform over the workgroup
        for (int ti = 0; ti < n_targets; ++ti) loss_of_target(targets, ti, lambda, partial, tloss, d_loss);
        if (threadIdx.x == 0 && d_total) {
            double total = 0.0;
            for (int ti = 0; ti < n_targets; ++ti) total += tloss[ti];
            *d_total = float(total);
        }
    }
    const int tile = int(xcd_tile(blockIdx.x, total_tiles));
    if (tile >= total_tiles) return;
    const gs_target t = targets[find_target_loss(targets, n_targets, tile)];
    const int local = tile - t.tile_offset;
    if (uint32_t(local) >= uint32_t(t.tiles_x) * t.tiles_y) return;   // a tile of no target of the call
    const Items items = loss_items(t, local);
    const int tid = threadIdx.x;
    const int64_t HW = int64_t(t.width) * t.height;
    const float inv = 1.f / (3.f * float(HW));
    for (int item = items.begin; item < items.end; ++item) {
        const int c = item / items.nb, blk = item - c * items.nb;
        const int x0 = blk % items.nbx * kBlk, y0 = blk / items.nbx * kBlk;
        const float *mp = maps + 9 * t.pix_offset + (3 * c) * HW;
        Stage st;
        st.fetch(mp, HW, t.width, t.height, x0, y0);
        __syncthreads();   // the previous item's reads are done
        const int lx = tid % kBlk, ly = tid / kBlk * kGroup;
        const int px = x0 + lx, py = y0 + ly;
        const int64_t at = 3 * t.pix_offset + c * HW + px;
        float x[kGroup], y[kGroup];
#pragma unroll
        for (int o = 0; o < kGroup; ++o) {
            const bool in = px < t.width && py + o < t.height;
            const int64_t a = at + int64_t(py + o) * t.width;
            x[o] = in ? render[a] : 0.f;
            y[o] = in ? target[a] : 0.f;
        }
        const float *const column = &L.h[0][ly * kBlk + lx];
        float f0[kGroup], f1[kGroup], f2[kGroup];
        auto rows = [&](int b) {
            rows_pass([&](int r, int cc) {
                float q[16];
                row_in(L.s[b] + r * kStride + cc, q);
                row_out(win, q, &L.h[b][r * kBlk + cc]);
            });
        };
        // the three maps one after the other, on two windows and row buffers
        st.put(0, t.width, t.height, x0, y0, L.s[0]);
        __syncthreads();
        st.put(1, t.width, t.height, x0, y0, L.s[1]);
        rows(0);
        __syncthreads();
        st.put(2, t.width, t.height, x0, y0, L.s[0]);
        column_out(win, column, f0);
        rows(1);
        __syncthreads();
        column_out(win, column + kPassSize, f1);
        rows(0);
        __syncthreads();
        column_out(win, column, f2);
#pragma unroll
        for (int o = 0; o < kGroup; ++o) {
            if (px >= t.width || py + o >= t.height) continue;
            const float d = x[o] - y[o];
            const float sgn = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
            const float dssim = f0[o] + 2.f * x[o] * f1[o] + y[o] * f2[o];
            dL[at + int64_t(py + o) * t.width] = t.weight * inv * ((1.f - lambda) * sgn - lambda * dssim);
        }
    }
}

__global__ void __launch_bounds__(256) loss_target_kernel(const gs_target *__restrict__ targets,
                                                          float lambda,
                                                          const float *__restrict__ partial,
                                                          double *__restrict__ tloss,
                                                          float *__restrict__ d_loss) {
    loss_of_target(targets, blockIdx.x, lambda, partial, tloss, d_loss);
}

// A few targets: one workgroup takes them in order and forms the total
// (the same sums in the same order as the two kernels above and below).
__global__ void __launch_bounds__(256) loss_few_kernel(const gs_target *__restrict__ targets,
                                                       int n_targets, float lambda,
                                                       const float *__restrict__ partial,
                                                       double *__restrict__ tloss,
                                                       float *__restrict__ d_loss,
                                                       float *__restrict__ d_total) {
    for (int ti = 0; ti < n_targets; ++ti) loss_of_target(targets, ti, lambda, partial, tloss, d_loss);
    if (threadIdx.x == 0 && d_total) {
        double total = 0.0;
        for (int ti = 0; ti < n_targets; ++ti) total += tloss[ti];
        *d_total = float(total);
    }
}

__global__ void __launch_bounds__(64) loss_total_kernel(int n_targets, const double *__restrict__ tloss,
                                                        float *__restrict__ d_total) {
    if (threadIdx.x != 0) return;
    double total = 0.0;
#pragma unroll 8
    for (int ti = 0; ti < n_targets; ++ti) total += tloss[ti];   // in target order
    if (d_total) *d_total = float(total);
}

// One pyramid level down: 5x5 binomial, reflected borders (edge not repeated),
// even rows/columns kept.
__device__ __forceinline__ int refl101(int i, int n) {
    if (n == 1) return 0;
    while (i < 0 || i >= n) {
        if (i < 0) i = -i;
        if (i >= n) i = 2 * (n - 1) - i;
    }
    return i;
}

// A workgroup forms 30x16 outputs of one channel from 63x35 staged inputs, rows
// first; a wave stages a row in one load.  kCopy: its 60x32 inputs are also copied
// (the pyramid's first level), on their way to LDS.
// Bound: memory and launch.  1200x680, 3 channels: copy and first level 8.1 us (a
// copy of 6.5 and 25 loads per output, 11, before), second level 3.4 (4.2).
constexpr int kPyrW = 30, kPyrH = 16, kPyrRows = 2 * kPyrH + 3;
template <bool kCopy>
__global__ void __launch_bounds__(256) pyr_down_kernel(const float *__restrict__ in, int channel, int H, int W,
                                                       float *__restrict__ out, float *__restrict__ same) {
    __shared__ float s[kPyrRows + 1][kWave];
    __shared__ float h[kPyrRows][kPyrW];
    const int Ho = (H + 1) / 2, Wo = (W + 1) / 2;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int blocks = (Wo + kPyrW - 1) / kPyrW;
    const int ox0 = blockIdx.x % blocks * kPyrW, oy0 = blockIdx.x / blocks * kPyrH;
    const int64_t HW = int64_t(H) * W;
    const int64_t c = int64_t(channel) + blockIdx.y;
    const float *src = in + c * HW;
    const int x = 2 * ox0 - 2 + lane, y0 = 2 * oy0 - 2;
    const int xr = refl101(min(x, W + 1), W);   // (no output needs more)
    constexpr int kRounds = (kPyrRows + 3) / 4;
    float v[kRounds];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) v[k] = src[int64_t(refl101(min(y0 + wave + 4 * k, H + 1), H)) * W + xr];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
        const int r = wave + 4 * k, y = y0 + r;
        s[r][lane] = v[k];
        if (kCopy && lane >= 2 && lane < 2 + 2 * kPyrW && x < W && r >= 2 && r < 2 + 2 * kPyrH && y < H)
            same[c * HW + int64_t(y) * W + x] = v[k];
    }
    __syncthreads();
    const float w[5] = {1.f / 16, 4.f / 16, 6.f / 16, 4.f / 16, 1.f / 16};
    for (int i = tid; i < kPyrRows * kPyrW; i += 256) {
        const int r = i / kPyrW, c = i % kPyrW;
        float row = 0.f;
#pragma unroll
        for (int b = 0; b < 5; ++b) row = fmaf(w[b], s[r][2 * c + b], row);
        h[r][c] = row;
    }
    __syncthreads();
    for (int i = tid; i < kPyrH * kPyrW; i += 256) {
        const int r = i / kPyrW, col = i % kPyrW;
        if (oy0 + r >= Ho || ox0 + col >= Wo) continue;
        float acc = 0.f;
#pragma unroll
        for (int a = 0; a < 5; ++a) acc = fmaf(w[a], h[2 * r + a][col], acc);
        out[c * (int64_t(Ho) * Wo) + int64_t(oy0 + r) * Wo + ox0 + col] = acc;
    }
}

__global__ void copy_f32_kernel(const float *__restrict__ a, float *__restrict__ b, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) b[i] = a[i];
}

}  // namespace gs

extern "C" gs_status gs_pyramid_build(const float *img, int32_t C, int32_t H, int32_t W,
                                      int32_t levels, float *out, void *stream) {
    using namespace gs;
    if (!img || !out || C <= 0 || H <= 0 || W <= 0 || levels <= 0 || levels > 16)
        return GS_ERR_INVALID_ARGUMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t n0 = int64_t(C) * H * W;
    if (levels == 1)
        hipLaunchKernelGGL(copy_f32_kernel, dim3((n0 + 255) / 256), dim3(256), 0, st, img, out, n0);
    const float *prev = img;
    float *cur = out + n0;
    int h = H, w = W;
    for (int l = 1; l < levels; ++l) {
        const int ho = (h + 1) / 2, wo = (w + 1) / 2;
        const int64_t blocks = int64_t((wo + kPyrW - 1) / kPyrW) * ((ho + kPyrH - 1) / kPyrH);
        for (int c = 0; c < C; c += 65535 < C - c ? 65535 : C - c) {
            const dim3 grid(blocks, C - c < 65535 ? C - c : 65535);
            if (l == 1)
                hipLaunchKernelGGL(pyr_down_kernel<true>, grid, dim3(256), 0, st, prev, c, h, w, cur, out);
            else
                hipLaunchKernelGGL(pyr_down_kernel<false>, grid, dim3(256), 0, st, prev, c, h, w, cur, nullptr);
        }
        prev = cur;
        cur += int64_t(C) * ho * wo;
        h = ho;
        w = wo;
    }
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_pyramid_loss(const float *render, const float *target,
                                     const gs_target *targets, int32_t n_targets,
                                     int32_t total_tiles, int64_t total_pixels, float lambda,
                                     void *loss_ws, float *d_loss, float *d_total,
                                     float *dL_drender, void *stream) {
    using namespace gs;
    if (!render || !target || !targets || !loss_ws || n_targets <= 0 || total_tiles <= 0 || n_targets > total_tiles ||
        total_pixels <= 0 || !(lambda >= 0.f && lambda <= 1.f))
        return GS_ERR_INVALID_ARGUMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    LossLayout L = LossLayout::make(total_pixels, total_tiles);
    char *b = static_cast<char *>(loss_ws);
    float *partial = reinterpret_cast<float *>(b + L.partial);
    float *maps = reinterpret_cast<float *>(b + L.maps);
    const Window win = ssim_window();
    const int64_t grid = xcd_grid(total_tiles);
    hipLaunchKernelGGL(ssim_fwd_kernel, dim3(grid), dim3(kTilePix), 0, st, render, target, targets,
                       n_targets, total_tiles, win, maps, partial);
    double *tloss = reinterpret_cast<double *>(b + L.tloss);
    const bool few = n_targets <= kLossOneBlockTargets;
    if (dL_drender && few) {
        hipLaunchKernelGGL(ssim_bwd_kernel<true>, dim3(grid), dim3(kTilePix), 0, st, render, target, targets,
                           n_targets, total_tiles, win, lambda, maps, dL_drender, partial, tloss, d_loss, d_total);
        GS_CHECK_LAUNCH();
        return GS_OK;
    }
    if (dL_drender)
        hipLaunchKernelGGL(ssim_bwd_kernel<false>, dim3(grid), dim3(kTilePix), 0, st, render, target, targets,
                           n_targets, total_tiles, win, lambda, maps, dL_drender, partial, tloss, d_loss, d_total);
    if (few) {
        hipLaunchKernelGGL(loss_few_kernel, dim3(1), dim3(256), 0, st, targets, n_targets, lambda, partial,
                           tloss, d_loss, d_total);
    } else {
        hipLaunchKernelGGL(loss_target_kernel, dim3(n_targets), dim3(256), 0, st, targets, lambda, partial,
                           tloss, d_loss);
        hipLaunchKernelGGL(loss_total_kernel, dim3(1), dim3(64), 0, st, n_targets, tloss, d_total);
    }
    GS_CHECK_LAUNCH();
    return GS_OK;
}
