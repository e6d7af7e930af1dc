// Initialisation of newly densified primitives (Section 3.3.1: temporary
// primitives are created at inactive 2D keypoints of a new keyframe, placed in
// 3D with the keypoint's depth).  Kernels:
//   features  - network input per keypoint: 7x7 RGB patch of the keyframe image
//               (edge-clamped), depth, keypoint scale, a one-hot of its
//               octave (8), the heuristic's log-scale and log depth,
//               zero-padded to 160, BF16;
//   heuristic - scale = mean distance to the 3 nearest means (existing and
//               new), isotropic, identity rotation, opacity 0.1, colour from
//               the pixel, higher SH zero;
//   decode    - network outputs (corrections to the heuristic's log-scale and
//               SH DC, a camera-frame quaternion, the opacity logit) to
//               world-frame parameters, falling back to the heuristic when the
//               predicted opacity is below 0.01;
//   append    - copy new columns into the parameter store, Adam moments zeroed.
// Keypoints are float4 (u, v, depth, scale) in pixels / metres; scale is
// 1.2^octave.
#include "gs_internal.hpp"

namespace gs {

constexpr int kFeat = 160, kPatch = 7;

__device__ __forceinline__ uint16_t f2bf_init(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

// One thread per (keypoint, feature), so a keypoint's row is written by
// consecutive threads and its 147 patch pixels are read side by side.  Bound:
// launch latency.  2,000 keypoints at 1200x680: 4.6 us (29.5 us with one
// thread per keypoint, which gathered and stored its 160 values one after the
// other in eight workgroups).
__global__ void __launch_bounds__(256) features_kernel(const float *__restrict__ img, int H, int W,
                                                       const float4 *__restrict__ kp, int B,
                                                       const float *__restrict__ heur,
                                                       uint16_t *__restrict__ x) {
    constexpr int kPix = kPatch * kPatch;
    const int64_t at = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (at >= int64_t(B) * kFeat) return;
    const int i = int(at / kFeat), f = int(at - int64_t(i) * kFeat);
    const float4 k = kp[i];
    float v = 0.f;
    if (f < 3 * kPix) {   // the patch, channel major
        const int cu = int(rintf(k.x)), cv = int(rintf(k.y));
        const int c = f / kPix, q = f - c * kPix, dy = q / kPatch - kPatch / 2, dx = q % kPatch - kPatch / 2;
        const int yy = min(max(cv + dy, 0), H - 1), xx = min(max(cu + dx, 0), W - 1);
        v = img[(int64_t(c) * H + yy) * W + xx];
    } else if (f == 3 * kPix) {
        v = k.z;                                                            // depth
    } else if (f == 3 * kPix + 1) {
        v = k.w;                                                            // scale
    } else if (f < 3 * kPix + 10) {                                         // octave, one-hot
        const int oct = min(max(int(rintf(__logf(fmaxf(k.w, 1.f)) / __logf(1.2f))), 0), 7);
        v = f - (3 * kPix + 2) == oct ? 1.f : 0.f;
    } else if (f == 3 * kPix + 10) {
        v = heur ? heur[int64_t(3) * B + i] : 0.f;                          // heuristic log-scale (metres)
    } else if (f == 3 * kPix + 11) {
        v = logf(k.z);                                                      // log depth
    }
    x[at] = f2bf_init(v);
}

// The heuristic column of new mean i whose three smallest squared distances
// to other means are d[0] <= d[1] <= d[2].
__device__ __forceinline__ void write_heuristic(const float *__restrict__ new_mu, const float *__restrict__ new_rgb,
                                                int B, int i, const float (&d)[3], float *__restrict__ out) {
    const float mean_d = (sqrtf(d[0]) + sqrtf(d[1]) + sqrtf(d[2])) / 3.f;
    const float ls = logf(fmaxf(mean_d, 1e-7f));
    const float c0 = 0.28209479177387814f;   // degree-0 real SH value
    float col[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) col[r] = 0.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        col[a] = new_mu[int64_t(a) * B + i];
        col[3 + a] = ls;
        col[11 + a] = (new_rgb[int64_t(a) * B + i] - 0.5f) / c0;
    }
    col[6] = 1.f;
    col[10] = logf(0.1f / 0.9f);
#pragma unroll
    for (int r = 0; r < kRows; ++r) out[int64_t(r) * B + i] = col[r];
}

// d joins the three smallest squared distances (kept in ascending order); a
// NaN is left out, as it compares false.
__device__ __forceinline__ void keep_smallest(float (&best)[3], float d) {
    const float x = d < best[2] ? d : best[2];
    best[2] = __builtin_amdgcn_fmed3f(best[1], best[2], x);
    best[1] = __builtin_amdgcn_fmed3f(best[0], best[1], x);
    best[0] = fminf(best[0], x);
}

// 3 nearest neighbours of every new mean among the n existing means and the
// other new means, by brute force.  A workgroup takes kKnnQueries new means,
// one per lane, and the blockIdx.y-th of gridDim.y shares of the points; its
// waves take the share's chunks of kKnnChunk points in turn, and the waves'
// results are merged in LDS.  A chunk's points are the same for all lanes, so
// they come through scalar loads and cost no vector instruction; their
// smallest distance is compared once with the third best so far, and only a
// chunk that improves some lane goes through the insertion.  With one share
// the workgroup writes the new columns, otherwise its three distances go to
// rows 3s .. 3s + 2 of `out` (share s; out is overwritten by the merge
// kernel), so no other memory is needed.
//
// Bound: VALU, six operations a pair and one comparison in kKnnChunk.  2,000
// new means against 300,000: 162 us and 14 us for the merge, against 33.6 ms for one thread per
// new mean over all points (eight workgroups on 256 CUs).
constexpr int kKnnQueries = kWave, kKnnWaves = 16, kKnnChunk = 8;
constexpr int kKnnShares = kRows / 3;       // three rows of `out` per share
constexpr int kKnnGroups = 512;             // workgroups wanted: two of 16 waves per CU
__global__ void __launch_bounds__(kKnnWaves * kWave) heuristic_kernel(
    const float *__restrict__ new_mu, const float *__restrict__ new_rgb, int B, const float *__restrict__ P,
    int64_t n, int64_t n_cap, float *__restrict__ out) {
    __shared__ float part[kKnnWaves][3][kWave];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int i = blockIdx.x * kKnnQueries + lane;
    const bool live = i < B;
    float px = 0, py = 0, pz = 0;
    if (live) { px = new_mu[i]; py = new_mu[int64_t(B) + i]; pz = new_mu[2 * int64_t(B) + i]; }
    float best[3] = {3.4e38f, 3.4e38f, 3.4e38f};
    auto distance = [&](float x, float y, float z) {
        const float dx = x - px, dy = y - py, dz = z - pz;
        return fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    };
    // points [0, count) of rows x, y, z; `self`: the point that is this lane's own
    auto scan = [&](const float *__restrict__ x, const float *__restrict__ y, const float *__restrict__ z,
                    int64_t count, int64_t self, bool has_self) {
        const int64_t chunks = (count + kKnnChunk - 1) / kKnnChunk;
        const int64_t step = int64_t(gridDim.y) * kKnnWaves;
        for (int64_t c = int64_t(blockIdx.y) * kKnnWaves + wave; c < chunks; c += step) {
            const int64_t j0 = c * kKnnChunk;
            float d[kKnnChunk], least = 3.4e38f;
            if (j0 + kKnnChunk <= count) {
#pragma unroll
                for (int t = 0; t < kKnnChunk; ++t) d[t] = distance(x[j0 + t], y[j0 + t], z[j0 + t]);
            } else {
#pragma unroll
                for (int t = 0; t < kKnnChunk; ++t) {
                    const int64_t j = j0 + t < count ? j0 + t : count - 1;
                    const float v = distance(x[j], y[j], z[j]);
                    d[t] = j0 + t < count ? v : 3.4e38f;
                }
            }
            if (has_self) {
#pragma unroll
                for (int t = 0; t < kKnnChunk; ++t) d[t] = j0 + t == self ? 3.4e38f : d[t];
            }
#pragma unroll
            for (int t = 0; t < kKnnChunk; ++t) least = fminf(least, d[t]);
            if (__any(least < best[2])) {
#pragma unroll
                for (int t = 0; t < kKnnChunk; ++t) keep_smallest(best, d[t]);
            }
        }
    };
    scan(P, P + n_cap, P + 2 * n_cap, n, 0, false);
    scan(new_mu, new_mu + B, new_mu + 2 * int64_t(B), B, i, true);
#pragma unroll
    for (int k = 0; k < 3; ++k) part[wave][k][lane] = best[k];
    __syncthreads();
    if (wave != 0 || !live) return;
    for (int w = 1; w < kKnnWaves; ++w)
#pragma unroll
        for (int k = 0; k < 3; ++k) keep_smallest(best, part[w][k][lane]);
    if (gridDim.y == 1) {
        write_heuristic(new_mu, new_rgb, B, i, best, out);
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) out[int64_t(3 * blockIdx.y + k) * B + i] = best[k];
    }
}

// The shares' distances of every new mean, merged; then its column.  (A thread
// reads and writes its own column only.)
__global__ void __launch_bounds__(kWave) heuristic_merge_kernel(const float *__restrict__ new_mu,
                                                                const float *__restrict__ new_rgb, int B, int shares,
                                                                float *out) {
    const int i = blockIdx.x * kWave + threadIdx.x;
    if (i >= B) return;
    float best[3] = {3.4e38f, 3.4e38f, 3.4e38f};
    for (int r = 0; r < 3 * shares; ++r) keep_smallest(best, out[int64_t(r) * B + i]);
    write_heuristic(new_mu, new_rgb, B, i, best, out);
}

// Rotation matrix (row-major) to unit quaternion (w, x, y, z).
__device__ __forceinline__ void mat_to_quat(const float R[9], float q[4]) {
    const float tr = R[0] + R[4] + R[8];
    if (tr > 0.f) {
        const float s = sqrtf(tr + 1.f) * 2.f;
        q[0] = 0.25f * s; q[1] = (R[7] - R[5]) / s; q[2] = (R[2] - R[6]) / s; q[3] = (R[3] - R[1]) / s;
    } else if (R[0] > R[4] && R[0] > R[8]) {
        const float s = sqrtf(1.f + R[0] - R[4] - R[8]) * 2.f;
        q[0] = (R[7] - R[5]) / s; q[1] = 0.25f * s; q[2] = (R[1] + R[3]) / s; q[3] = (R[2] + R[6]) / s;
    } else if (R[4] > R[8]) {
        const float s = sqrtf(1.f + R[4] - R[0] - R[8]) * 2.f;
        q[0] = (R[2] - R[6]) / s; q[1] = (R[1] + R[3]) / s; q[2] = 0.25f * s; q[3] = (R[5] + R[7]) / s;
    } else {
        const float s = sqrtf(1.f + R[8] - R[0] - R[4]) * 2.f;
        q[0] = (R[3] - R[1]) / s; q[1] = (R[2] + R[6]) / s; q[2] = (R[5] + R[7]) / s; q[3] = 0.25f * s;
    }
}

__global__ void __launch_bounds__(256) decode_kernel(const float *__restrict__ y, const float4 *__restrict__ kp,
                                                     gs_view view, int B, const float *__restrict__ heur,
                                                     float *__restrict__ out, int32_t *__restrict__ used_fallback) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    const float *yi = y + int64_t(i) * 16;
    const float opac = 1.f / (1.f + __expf(-yi[7]));
    if (opac < 0.01f) {
        for (int r = 0; r < kRows; ++r) out[int64_t(r) * B + i] = heur[int64_t(r) * B + i];
        if (used_fallback) used_fallback[i] = 1;
        return;
    }
    if (used_fallback) used_fallback[i] = 0;
    const float4 k = kp[i];
    // camera frame point, then world: mu = R^T (xc - t)
    const float xc[3] = {k.z * (k.x - view.cx) / view.fx, k.z * (k.y - view.cy) / view.fy, k.z};
    const float *R = view.R;
    float d[3] = {xc[0] - view.t[0], xc[1] - view.t[1], xc[2] - view.t[2]};
    float col[kRows];
    for (int r = 0; r < kRows; ++r) col[r] = 0.f;
    for (int a = 0; a < 3; ++a) col[a] = R[a] * d[0] + R[3 + a] * d[1] + R[6 + a] * d[2];
    // log-scale: the heuristic's plus the predicted correction
    for (int a = 0; a < 3; ++a) col[3 + a] = heur[int64_t(3 + a) * B + i] + yi[a];
    // camera-frame rotation to world: q_w = q(R^T) * q_c
    float Rt[9] = {R[0], R[3], R[6], R[1], R[4], R[7], R[2], R[5], R[8]};
    float qa[4];
    mat_to_quat(Rt, qa);
    const float qb[4] = {yi[3], yi[4], yi[5], yi[6]};
    col[6] = qa[0] * qb[0] - qa[1] * qb[1] - qa[2] * qb[2] - qa[3] * qb[3];
    col[7] = qa[0] * qb[1] + qa[1] * qb[0] + qa[2] * qb[3] - qa[3] * qb[2];
    col[8] = qa[0] * qb[2] - qa[1] * qb[3] + qa[2] * qb[0] + qa[3] * qb[1];
    col[9] = qa[0] * qb[3] + qa[1] * qb[2] - qa[2] * qb[1] + qa[3] * qb[0];
    col[10] = yi[7];
    // SH DC: the heuristic's (pixel colour) plus the predicted correction
    for (int c = 0; c < 3; ++c) col[11 + c] = heur[int64_t(11 + c) * B + i] + yi[8 + c];
    for (int r = 0; r < kRows; ++r) out[int64_t(r) * B + i] = col[r];
}

// Row blockIdx.y of the new columns (one workgroup per row and 256 columns:
// 2,000 columns 2.5-4.4 us, 17 us with a thread walking all rows of a column).
__global__ void __launch_bounds__(256) append_kernel(float *__restrict__ P, float *__restrict__ m,
                                                     float *__restrict__ v, int64_t n, int64_t n_cap,
                                                     const float *__restrict__ newp, int B) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    const int64_t dst = int64_t(blockIdx.y) * n_cap + n + i;
    P[dst] = newp[int64_t(blockIdx.y) * B + i];
    if (m) m[dst] = 0.f;
    if (v) v[dst] = 0.f;
}

}  // namespace gs

extern "C" gs_status gs_init_features(const float *img, int32_t H, int32_t W, const float *kp,
                                      int32_t B, const float *heuristic, void *x_bf16, void *stream) {
    if (!img || !kp || !x_bf16 || H <= 0 || W <= 0 || B <= 0) return GS_ERR_INVALID_ARGUMENT;
    hipLaunchKernelGGL(gs::features_kernel, dim3((int64_t(B) * gs::kFeat + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), img, H, W, reinterpret_cast<const float4 *>(kp), B,
                       heuristic, static_cast<uint16_t *>(x_bf16));
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_init_heuristic(const float *new_mu, const float *new_rgb, int32_t B,
                                       const float *params, int64_t n, int64_t n_cap, float *out,
                                       void *stream) {
    if (!new_mu || !new_rgb || !out || B <= 0 || n < 0 || (n > 0 && !params) || n > n_cap || n_cap % 64)
        return GS_ERR_INVALID_ARGUMENT;
    using namespace gs;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // shares of the points: enough workgroups to fill the chip, each wave with
    // at least a few chunks, and no more shares than `out` has rows for
    const int64_t groups = (int64_t(B) + kKnnQueries - 1) / kKnnQueries;
    const int64_t useful = (n + B) / (4 * kKnnWaves * kKnnChunk) + 1;
    const int64_t wanted = (kKnnGroups + groups - 1) / groups;
    const int64_t most = wanted < kKnnShares ? wanted : int64_t(kKnnShares);
    const int shares = int(useful < most ? useful : most);
    hipLaunchKernelGGL(heuristic_kernel, dim3(groups, shares), dim3(kKnnWaves * kWave), 0, st, new_mu, new_rgb, B,
                       params, n, n_cap, out);
    if (shares > 1)
        hipLaunchKernelGGL(heuristic_merge_kernel, dim3((int64_t(B) + kWave - 1) / kWave), dim3(kWave), 0, st, new_mu,
                           new_rgb, B, shares, out);
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_init_decode(const float *y, const float *kp, const gs_view *view, int32_t B,
                                    const float *heuristic, float *out, int32_t *used_fallback,
                                    void *stream) {
    if (!y || !kp || !view || !heuristic || !out || B <= 0) return GS_ERR_INVALID_ARGUMENT;
    hipLaunchKernelGGL(gs::decode_kernel, dim3((B + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), y, reinterpret_cast<const float4 *>(kp), *view, B,
                       heuristic, out, used_fallback);
    GS_CHECK_LAUNCH();
    return GS_OK;
}

extern "C" gs_status gs_append(float *params, float *m, float *v, int64_t n, int64_t n_cap,
                               const float *new_params, int32_t B, void *stream) {
    if (!params || !new_params || B < 0 || n < 0 || n + B > n_cap || n_cap % 64)
        return GS_ERR_INVALID_ARGUMENT;
    if (B == 0) return GS_OK;
    hipLaunchKernelGGL(gs::append_kernel, dim3((int64_t(B) + 255) / 256, gs::kRows), dim3(256), 0,
                       static_cast<hipStream_t>(stream), params, m, v, n, n_cap, new_params, B);
    GS_CHECK_LAUNCH();
    return GS_OK;
}
