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
    const int64_t at = wide_block() * blockDim.x + threadIdx.x;
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
// to other means are d[0] <= d[1] <= d[2] (of kParts parts the part-th).
template <int kParts>
__device__ __forceinline__ void write_heuristic(const float *__restrict__ new_mu, const float *__restrict__ new_rgb,
                                                int B, int i, const float (&d)[3], float *__restrict__ out,
                                                int part) {
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
    for (int r = 0; r < kRows; ++r)
        if (r % kParts == part) out[int64_t(r) * B + i] = col[r];
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
// other new means, by brute force.  A workgroup takes kAllQueries new means,
// one per lane, and the blockIdx.y-th of gridDim.y shares of the points; its
// waves take the share's chunks of kAllChunk points in turn, and the waves'
// results are merged in LDS.  A chunk's points are the same for all lanes, so
// they come through scalar loads and cost no vector instruction; their
// smallest distance is compared once with the third best so far, and only a
// chunk that improves some lane goes through the insertion.  With one share
// the workgroup writes the new columns, otherwise its three distances go to
// rows 3s .. 3s + 2 of `out` (share s), which heuristic_columns_kernel merges and
// overwrites, so no other memory is needed.
//
// Bound: VALU, eight operations a pair and one comparison in kAllChunk.  Up to
// kAllPoints points (above them heuristic_kernel measures fewer pairs).
constexpr int kAllQueries = kWave, kAllWaves = 16, kAllChunk = 8;
constexpr int kAllShares = kRows / 3;       // three rows of `out` per share
constexpr int kAllGroups = 512;             // workgroups wanted: two of 16 waves per CU
__global__ void __launch_bounds__(kAllWaves * kWave) heuristic_all_kernel(
    const float *__restrict__ new_mu, const float *__restrict__ new_rgb, int B, const float *__restrict__ P,
    int64_t n, int64_t n_cap, float *__restrict__ out) {
    __shared__ float part[kAllWaves][3][kWave];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int i = blockIdx.x * kAllQueries + lane;
    const bool live = i < B;
    float px = 0, py = 0, pz = 0;
    if (live) { px = new_mu[i]; py = new_mu[int64_t(B) + i]; pz = new_mu[2 * int64_t(B) + i]; }
    float best[3] = {3.4e38f, 3.4e38f, 3.4e38f};
    auto distance = [&](float x, float y, float z) {
        const float dx = x - px, dy = y - py, dz = z - pz;
        return dx * dx + dy * dy + dz * dz;
    };
    // points [0, count) of rows x, y, z; `self`: the point that is this lane's own
    auto scan = [&](const float *__restrict__ x, const float *__restrict__ y, const float *__restrict__ z,
                    int64_t count, int64_t self, bool has_self) {
        const int64_t chunks = (count + kAllChunk - 1) / kAllChunk;
        const int64_t step = int64_t(gridDim.y) * kAllWaves;
        for (int64_t c = int64_t(blockIdx.y) * kAllWaves + wave; c < chunks; c += step) {
            const int64_t j0 = c * kAllChunk;
            float d[kAllChunk], least = 3.4e38f;
            if (j0 + kAllChunk <= count) {
#pragma unroll
                for (int t = 0; t < kAllChunk; ++t) d[t] = distance(x[j0 + t], y[j0 + t], z[j0 + t]);
            } else {
#pragma unroll
                for (int t = 0; t < kAllChunk; ++t) {
                    const int64_t j = j0 + t < count ? j0 + t : count - 1;
                    const float v = distance(x[j], y[j], z[j]);
                    d[t] = j0 + t < count ? v : 3.4e38f;
                }
            }
            if (has_self) {
#pragma unroll
                for (int t = 0; t < kAllChunk; ++t) d[t] = j0 + t == self ? 3.4e38f : d[t];
            }
#pragma unroll
            for (int t = 0; t < kAllChunk; ++t) least = fminf(least, d[t]);
            if (__any(least < best[2])) {
#pragma unroll
                for (int t = 0; t < kAllChunk; ++t) keep_smallest(best, d[t]);
            }
        }
    };
    scan(P, P + n_cap, P + 2 * n_cap, n, 0, false);
    scan(new_mu, new_mu + B, new_mu + 2 * int64_t(B), B, i, true);
#pragma unroll
    for (int k = 0; k < 3; ++k) part[wave][k][lane] = best[k];
    __syncthreads();
    if (wave != 0 || !live) return;
    for (int w = 1; w < kAllWaves; ++w)
#pragma unroll
        for (int k = 0; k < 3; ++k) keep_smallest(best, part[w][k][lane]);
    if (gridDim.y == 1) {
        write_heuristic<1>(new_mu, new_rgb, B, i, best, out, 0);
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) out[int64_t(3 * blockIdx.y + k) * B + i] = best[k];
    }
}

// The same for many points.  A workgroup takes kKnnQueries new means and the blockIdx.y-th
// of gridDim.y shares of the points, which come in groups of 64 (existing and new
// means apart), up to kKnnRound groups a round:
//  1. A wave takes groups in turn.  With both shifted by the workgroup's first
//     mean, s = q.p - |p|^2 / 2 (the larger, the nearer) is a sum over four terms,
//     each with its factors cut into three BF16 parts h + m + l (exactly): one
//     16x16x32 matrix product for 16 points and 16 queries (a lane holds
//     A[lane % 16][8 (lane / 16) ..], B[8 (lane / 16) ..][lane % 16] and
//     D[4 (lane / 16) + r][lane % 16]), whose 8 slots per term are h h, m h, h m, m m,
//     l h, h l and two zeros.  A group's largest s per query goes to LDS.
//  2. A thread takes a query and every kKnnParts-th group.  s is off by e at most,
//     in proportion to |q| R + R^2 with R the group's largest |p|.  Four points (of
//     which one may be the query itself) are as near as the fourth largest of the
//     threads' largest (s - e) says, or of the workgroups', each of which joins its
//     largest to the four largest so far; so a group can hold one of the three
//     nearest only if its (largest s) + e reaches that.  Those that do are listed:
//     few, as the workgroups run together, and never too few.
//  3. The listed groups' points are measured exactly, a lane each, and those
//     within the bound join the query's three smallest distances.
// A group with a point that is far off or not finite has e = infinity: it counts
// for no bound and is always measured.  The four largest of a query's workgroups
// (in the last rows of `out`) and its three smallest distances (in LDS) are kept as
// unsigned numbers in the order of the floats and joined by chains of atomics: what
// a row turns away goes on to the next, so any order of joining ends with the same
// values.  The distances of share s then go to rows 3s .. 3s + 2 of `out`, which
// heuristic_columns_kernel merges and overwrites, so no other memory is needed.
//
// Bound: VALU issue (norms, cuts and maxima of step 1), beside which the matrix
// products (16 cycles for 256 pairs) run.
// 2,000 new means against 300,000, with the columns: 95 us (181 by measuring every
// pair, 33.6 ms by one thread per new mean over all points).  By 16x16x4 FP32
// products, which do not run beside vector instructions, 121; with the distances
// of all workgroups joined in one row of device atomics 180.
// More points than this (both kinds together) are taken by heuristic_kernel.  Every
// pair measured / groups, us: 1,000 + 50 points 11.0 / 18.5; 5,000 + 4,096 19.9 / 30.0;
// 20,000 + 200 24.9 / 24.4; 100,000 + 1,000 64.2 / 38.4; 300,000 + 50 87.0 / 54.8;
// 500,000 + 4,096 477 / 235.
constexpr int64_t kAllPoints = 20000;
constexpr int kKnnQueries = 128, kKnnTiles = kKnnQueries / 16, kKnnWaves = 16, kKnnThreads = kKnnWaves * kWave;
constexpr int kKnnParts = kKnnThreads / kKnnQueries;
constexpr int kKnnRound = 256;              // groups of 64 points per round
constexpr int kKnnStride = kKnnQueries + 1;
constexpr int kKnnList = 1024;              // listed (query, group) pairs at a time
constexpr int kKnnGroups = 256;             // workgroups wanted: one per CU
constexpr int kKnnNear = 3, kKnnBounds = 4; // distances kept per share; rows of bounds
constexpr int kKnnShares = (kRows - kKnnBounds) / kKnnNear;
// s by parts: each factor is within 2^-23 after the shift, the parts left out are
// 2^-23 of a product, and 24 products and their sum round to 2^-23 or so each.
constexpr float kKnnErr = 64.f / 16777216.f;
typedef float KnnAcc __attribute__((ext_vector_type(4)));
typedef __bf16 KnnFrag __attribute__((ext_vector_type(8)));
typedef uint32_t KnnWords __attribute__((ext_vector_type(4)));
// Sum or maximum over the four lanes that are equal modulo 16, in all of them.
template <typename Op>
__device__ __forceinline__ float across_rows(float x, Op op) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int kRotate>
__device__ __forceinline__ uint32_t row_rotated(uint32_t x) {   // within a row of 16 lanes
    return __builtin_amdgcn_update_dpp(0, x, 0x120 + kRotate, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t row_most(uint32_t x) {
    x = max(x, row_rotated<8>(x));
    x = max(x, row_rotated<4>(x));
    x = max(x, row_rotated<2>(x));
    return max(x, row_rotated<1>(x));
}
// m[k] joined by the four values of d[k]; the wait is for the last product
// (the compiler does not see reads inside the block, and fmaxf() would first
// quiet every operand by an instruction of its own).
__device__ __forceinline__ void join_largest(float *m, const KnnAcc (&d)[4]) {
    asm("s_nop 15\n\t"
        "v_max3_f32 %0, %0, %4, %5\n\t"
        "v_max3_f32 %1, %1, %8, %9\n\t"
        "v_max3_f32 %2, %2, %12, %13\n\t"
        "v_max3_f32 %3, %3, %16, %17\n\t"
        "v_max3_f32 %0, %0, %6, %7\n\t"
        "v_max3_f32 %1, %1, %10, %11\n\t"
        "v_max3_f32 %2, %2, %14, %15\n\t"
        "v_max3_f32 %3, %3, %18, %19"
        : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3])
        : "v"(d[0][0]), "v"(d[0][1]), "v"(d[0][2]), "v"(d[0][3]), "v"(d[1][0]), "v"(d[1][1]), "v"(d[1][2]),
          "v"(d[1][3]), "v"(d[2][0]), "v"(d[2][1]), "v"(d[2][2]), "v"(d[2][3]), "v"(d[3][0]), "v"(d[3][1]),
          "v"(d[3][2]), "v"(d[3][3]));
}
// The largest over the four rows of lanes of m[0 .. 3], in one register: rows 0, 1,
// 2, 3 hold that of m[0], m[2], m[1], m[3].
__device__ __forceinline__ float rows_largest(float m0, float m1, float m2, float m3) {
    asm("s_nop 1\n\t"
        "v_permlane32_swap_b32 %0, %1\n\t"
        "v_permlane32_swap_b32 %2, %3\n\t"
        "s_nop 1\n\t"
        "v_max_f32 %0, %0, %1\n\t"
        "v_max_f32 %2, %2, %3\n\t"
        "s_nop 1\n\t"
        "v_permlane16_swap_b32 %0, %2\n\t"
        "s_nop 1\n\t"
        "v_max_f32 %0, %0, %2"
        : "+v"(m0), "+v"(m1), "+v"(m2), "+v"(m3));
    return m0;
}
// Unsigned numbers in the order of floats; 0 is below them all.
__device__ __forceinline__ uint32_t ordered(float x) {
    const uint32_t u = __float_as_uint(x);
    return u >> 31 ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(uint32_t u) {
    return u == 0u ? __uint_as_float(0xff800000u) : __uint_as_float(u >> 31 ? u & 0x7fffffffu : ~u);
}
__device__ __forceinline__ uint32_t now(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// x in three parts of eight bits each (as the upper halves of floats).
struct Cut {
    uint32_t h, m, l;
    __device__ __forceinline__ explicit Cut(float x) {
        h = __float_as_uint(x) & 0xffff0000u;
        const float r = x - __uint_as_float(h);
        m = __float_as_uint(r) & 0xffff0000u;
        l = __float_as_uint(r - __uint_as_float(m));
    }
};
// The upper halves of lo and hi, in that order.
__device__ __forceinline__ uint32_t halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ bool tame(float x) { return fabsf(x) < 1e15f; }   // (not a NaN)
__global__ void __launch_bounds__(kKnnThreads) __attribute__((amdgpu_waves_per_eu(4))) heuristic_kernel(
    const float *__restrict__ new_mu, int B, const float *__restrict__ P, int64_t n, int64_t n_cap,
    float *__restrict__ out) {
    __shared__ float largest[kKnnRound * kKnnStride];   // [group][query]
    __shared__ float reach[kKnnRound];                  // R of the groups
    __shared__ float query[3][kKnnQueries], bound[kKnnQueries];
    __shared__ float most[kKnnParts][kKnnQueries];
    __shared__ uint32_t nearest[kKnnNear][kKnnQueries];
    __shared__ uint16_t list[kKnnList];                 // query * kKnnRound + group
    __shared__ uint32_t listed;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int q0 = blockIdx.x * kKnnQueries, row = lane / 16, col = lane % 16;
    const float inf = __uint_as_float(0x7f800000u);
    // the shift, and this lane's component of it
    float c[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float x = new_mu[int64_t(k) * B + q0];
        c[k] = tame(x) ? x : 0.f;
    }
    const float shift = row == 0 ? c[0] : row == 1 ? c[1] : c[2];
    KnnFrag Bq[kKnnTiles];
#pragma unroll
    for (int t = 0; t < kKnnTiles; ++t) {
        KnnWords w = {0x3f803f80u, 0u, 0x00003f80u, 0u};   // the fourth term: 1 times the parts of -|p|^2 / 2
        if (row < 3) {
            const Cut x(new_mu[int64_t(row) * B + min(q0 + 16 * t + col, B - 1)] - shift);
            w = KnnWords{halves(x.h, x.h), halves(x.m, x.m), halves(x.h, x.l), 0u};
        }
        Bq[t] = __builtin_bit_cast(KnnFrag, w);
    }
    const int tile = row == 1 ? 2 : row == 2 ? 1 : row;   // (rows_largest)
    // this thread's query in step 2, and which of its groups
    const int mine = threadIdx.x % kKnnQueries, part = threadIdx.x / kKnnQueries, id = min(q0 + mine, B - 1);
    const float qx = new_mu[id], qy = new_mu[int64_t(B) + id], qz = new_mu[2 * int64_t(B) + id];
    if (part == 0) {
        query[0][mine] = qx, query[1][mine] = qy, query[2][mine] = qz;
#pragma unroll
        for (int k = 0; k < kKnnNear; ++k) nearest[k][mine] = __float_as_uint(3.4e38f);
    }
    // (what is not finite is near nothing)
    const bool live = q0 + mine < B && fabsf(qx) < inf && fabsf(qy) < inf && fabsf(qz) < inf;
    const float sx = qx - c[0], sy = qy - c[1], sz = qz - c[2];
    const float qq = sx * sx + sy * sy + sz * sz, length = __builtin_amdgcn_sqrtf(qq);
    uint32_t *const bounds = reinterpret_cast<uint32_t *>(out) + int64_t(kRows - kKnnBounds) * B + q0 + mine;

    const float *const in_old = P + (row < 3 ? row : 0) * n_cap + col;   // this lane's coordinate of a group's first points
    const float *const in_new = new_mu + (row < 3 ? row : 0) * int64_t(B) + col;
    const int64_t old_groups = (n + kWave - 1) / kWave, groups = old_groups + (int64_t(B) + kWave - 1) / kWave;
    const int64_t g0 = groups * blockIdx.y / gridDim.y, g1 = groups * (blockIdx.y + 1) / gridDim.y;
    const int64_t rounds = (g1 - g0 + kKnnRound - 1) / kKnnRound;
    for (int64_t round = 0; round < rounds; ++round) {
        const int64_t r0 = g0 + (g1 - g0) * round / rounds;
        const int count = int(g0 + (g1 - g0) * (round + 1) / rounds - r0);
        __syncthreads();   // the last round's reads are done
        // 1. (a wave's next groups are loaded while one is worked on)
        auto fetch = [&](int g, float (&v)[4], int &points) {
            const int64_t at = r0 + g;
            const bool old = at < old_groups;
            const int64_t first = (old ? at : at - old_groups) * kWave, left = (old ? n : int64_t(B)) - first;
            const float *p = (old ? in_old : in_new) + first;
            points = int(left < kWave ? left : kWave);
            if (points == kWave) {
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = p[16 * t];
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = p[min(16 * t, points - 1 - col)];
            }
        };
        float v[4];
        int points = 0;
        if (wave < count) fetch(wave, v, points);
        for (int g = wave; g < count; g += kKnnWaves) {
            float next[4];
            int next_points = 0;
            if (g + kKnnWaves < count) fetch(g + kKnnWaves, next, next_points);
            float m[kKnnTiles];
            uint32_t far = 0u;   // (of non-negative values and NaNs, ordered as their bits)
#pragma unroll
            for (int t = 0; t < kKnnTiles; ++t) m[t] = -inf;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float x = row < 3 ? v[t] - shift : 0.f;
                const float pp = across_rows(x * x, [](float a, float b) { return a + b; });
                far = max(far, __float_as_uint(pp));
                float a = row < 3 ? x : -0.5f * pp;
                if (points < kWave) a = row == 3 && 16 * t + col >= points ? -1e30f : a;   // (uniform)
                const Cut cut(a);
                const uint32_t hm = halves(cut.h, cut.m);
                const KnnFrag parts = __builtin_bit_cast(KnnFrag, KnnWords{hm, hm, halves(cut.l, cut.h), 0u});
#pragma unroll
                for (int h = 0; h < kKnnTiles; h += 4) {
                    if (h > 0 && q0 + 16 * h >= B) break;   // (uniform)
                    KnnAcc d[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const KnnAcc zero = {0.f, 0.f, 0.f, 0.f};
                        d[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(parts, Bq[h + k], zero, 0, 0, 0);
                    }
                    join_largest(m + h, d);
                }
            }
#pragma unroll
            for (int h = 0; h < kKnnTiles; h += 4)
                largest[g * kKnnStride + 16 * (h + tile) + col] = rows_largest(m[h], m[h + 1], m[h + 2], m[h + 3]);
            far = row_most(far);   // (equal in the four lanes of a column)
            if (lane == 0) reach[g] = __builtin_amdgcn_sqrtf(__uint_as_float(far)) * 1.000001f;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = next[t];
            points = next_points;
        }
        __syncthreads();
        // 2. the bounds
        auto error = [&](int g) { return kKnnErr * reach[g] * (length + reach[g]) + 1e-30f; };
        float top = -inf;
#pragma unroll 4
        for (int g = part; g < count; g += kKnnParts) {
            const float e = error(g);
            if (e < 1e30f) top = fmaxf(top, largest[g * kKnnStride + mine] - e);   // (not for a NaN)
        }
        most[part][mine] = live ? top : -inf;
        __syncthreads();
        float four[kKnnBounds];
#pragma unroll
        for (int u = 0; u < kKnnBounds; ++u) four[u] = -inf;
#pragma unroll
        for (int p = 0; p < kKnnParts; ++p) {
            float x = most[p][mine];
#pragma unroll
            for (int u = 0; u < kKnnBounds; ++u) {
                const float y = fminf(four[u], x);
                four[u] = fmaxf(four[u], x);
                x = y;
            }
        }
        if (part == 0 && four[0] > -inf) {
            uint32_t x = ordered(four[0]);
            if (x > now(bounds + int64_t(kKnnBounds - 1) * B)) {   // (which only rises)
#pragma unroll
                for (int r = 0; r < kKnnBounds; ++r) x = min(x, atomicMax(bounds + int64_t(r) * B, x));
            }
        }
        __syncthreads();
        const float least =
            live ? fmaxf(four[kKnnBounds - 1], from_ordered(now(bounds + int64_t(kKnnBounds - 1) * B))) : inf;
        // three others at least are within this squared distance
        if (part == 0) bound[mine] = (qq - 2.f * least) + 4e-6f * (qq + fabsf(least)) + 1e-30f;
        // the list, as far as it holds, and 3., until all is done
        int g = live ? part : count;
        for (;;) {
            if (threadIdx.x == 0) listed = 0u;
            __syncthreads();
            for (; g < count; g += kKnnParts) {
                const float e = error(g);
                if (e < 1e30f && largest[g * kKnnStride + mine] + e < least) continue;
                const uint32_t at = atomicAdd(&listed, 1u);
                if (at >= kKnnList) break;
                list[at] = uint16_t(mine * kKnnRound + g);
            }
            __syncthreads();
            const int entries = int(min(listed, uint32_t(kKnnList)));
            constexpr int kTogether = 4;   // groups whose points are loaded together
            for (int e0 = wave * kTogether; e0 < entries; e0 += kKnnWaves * kTogether) {
                float p[kTogether][3];
                int k[kTogether], self[kTogether], have[kTogether];
#pragma unroll
                for (int e = 0; e < kTogether; ++e) {
                    const int entry = __builtin_amdgcn_readfirstlane(list[min(e0 + e, entries - 1)]);
                    k[e] = entry / kKnnRound;
                    const int64_t at = r0 + entry % kKnnRound;
                    const bool old = at < old_groups;
                    const float *base = old ? P : new_mu;
                    const int64_t stride = old ? n_cap : int64_t(B), first = (old ? at : at - old_groups) * kWave;
                    const int64_t left = (old ? n : int64_t(B)) - first;
                    have[e] = e0 + e < entries ? int(left < kWave ? left : kWave) : 0;
                    self[e] = old ? -1 : int(q0 + k[e] - first);   // (outside 0 .. 63: not here)
                    const int64_t j = first + min(lane, int(left < kWave ? left : kWave) - 1);
#pragma unroll
                    for (int a = 0; a < 3; ++a) p[e][a] = base[a * stride + j];
                }
#pragma unroll
                for (int e = 0; e < kTogether; ++e) {
                    const float dx = p[e][0] - query[0][k[e]], dy = p[e][1] - query[1][k[e]],
                                dz = p[e][2] - query[2][k[e]];
                    const float d = dx * dx + dy * dy + dz * dz;
                    if (!(lane < have[e] && lane != self[e] && d <= bound[k[e]])) continue;
                    uint32_t x = __float_as_uint(d);
                    if (x >= *static_cast<volatile uint32_t *>(&nearest[kKnnNear - 1][k[e]])) continue;   // (which only falls)
#pragma unroll
                    for (int r = 0; r < kKnnNear; ++r) x = max(x, atomicMin(&nearest[r][k[e]], x));
                }
            }
            if (!__syncthreads_or(g < count)) break;
        }
    }
    if (part < kKnnNear && q0 + mine < B)
        out[int64_t(kKnnNear * blockIdx.y + part) * B + q0 + mine] = __uint_as_float(nearest[part][mine]);
}
// The rows of bounds in `out`, empty.
__global__ void __launch_bounds__(256) heuristic_clear_kernel(uint32_t *__restrict__ bounds, int64_t count) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < count) bounds[i] = 0u;
}

// The shares' distances of every new mean, merged; then its column.  A workgroup
// takes 64 new means; its waves read every kColumnWaves-th row of their columns,
// merge in LDS and, once all have read, write every kColumnWaves-th row.
// (2,000 new means, 16 shares: 4.7 us; a wave per 64 alone took 14.)
constexpr int kColumnWaves = 8;
__global__ void __launch_bounds__(kColumnWaves * kWave) heuristic_columns_kernel(const float *__restrict__ new_mu,
                                                                                 const float *__restrict__ new_rgb,
                                                                                 int B, int shares, float *out) {
    __shared__ float part[kColumnWaves][3][kWave];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int i = blockIdx.x * kWave + lane, at = min(i, B - 1);
    float best[3] = {3.4e38f, 3.4e38f, 3.4e38f};
    constexpr int kMost = (3 * kAllShares + kColumnWaves - 1) / kColumnWaves;
    float d[kMost];
#pragma unroll
    for (int k = 0; k < kMost; ++k) {
        const int r = wave + kColumnWaves * k;
        d[k] = r < 3 * shares ? out[int64_t(r) * B + at] : 3.4e38f;
    }
#pragma unroll
    for (int k = 0; k < kMost; ++k) keep_smallest(best, d[k]);
#pragma unroll
    for (int k = 0; k < 3; ++k) part[wave][k][lane] = best[k];
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kColumnWaves; ++w)
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (w != wave) keep_smallest(best, part[w][k][lane]);
    if (i < B) write_heuristic<kColumnWaves>(new_mu, new_rgb, B, i, best, out, wave);
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
    hipLaunchKernelGGL(gs::features_kernel, gs::wide_grid((int64_t(B) * gs::kFeat + 255) / 256), dim3(256), 0,
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
    // shares of the points: enough workgroups to fill the chip, and no more than
    // `out` has rows for
    auto split = [&](int64_t blocks, int64_t wanted, int64_t useful, int64_t most) {
        const int64_t each = (wanted + blocks - 1) / blocks;
        most = most < each ? most : each;
        return int(useful < most ? useful : most);
    };
    int shares;
    if (n + B <= kAllPoints) {
        const int64_t blocks = (int64_t(B) + kAllQueries - 1) / kAllQueries;
        shares = split(blocks, kAllGroups, (n + B) / (4 * kAllWaves * kAllChunk) + 1, kAllShares);
        hipLaunchKernelGGL(heuristic_all_kernel, dim3(blocks, shares), dim3(kAllWaves * kWave), 0, st, new_mu, new_rgb, B,
                           params, n, n_cap, out);
    } else {
        const int64_t blocks = (int64_t(B) + kKnnQueries - 1) / kKnnQueries, cleared = kKnnBounds * int64_t(B);
        shares = split(blocks, kKnnGroups, (n + B) / (2 * kWave) + 1, kKnnShares);
        hipLaunchKernelGGL(heuristic_clear_kernel, dim3((cleared + 255) / 256), dim3(256), 0, st,
                           reinterpret_cast<uint32_t *>(out) + int64_t(kRows - kKnnBounds) * B, cleared);
        hipLaunchKernelGGL(heuristic_kernel, dim3(blocks, shares), dim3(kKnnThreads), 0, st, new_mu, B, params, n, n_cap,
                           out);
    }
    if (shares > 1 || n + B > kAllPoints)   // (one workgroup's own columns are written)
        hipLaunchKernelGGL(heuristic_columns_kernel, dim3((int64_t(B) + kWave - 1) / kWave), dim3(kColumnWaves * kWave), 0,
                           st, new_mu, new_rgb, B, shares, out);
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
