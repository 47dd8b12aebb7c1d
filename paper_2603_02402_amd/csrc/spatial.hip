// Spatial order of rows and the bounds of its segments, for the pruned exact
// screen (screen_split_grid.hpp).
//
// Order.  512 pivot rows at equal strides are grouped: a pivot takes the label
// of the first pivot within 2.5 times the median nearest-pivot distance (one
// label step more joins chains), so that the pivots of one cluster follow each
// other.  Every row goes to its nearest pivot (one split-screen pass over the
// 16 pivot blocks) and rows are sorted by (pivot rank, logarithm of the
// distance to the pivot, Morton code of the first three coordinates): rows of
// clusters that hold no pivot, far from the pivot they fall to, stay apart
// from its own.  512 pivots because a cluster of 1% of the rows is then missed
// once in 170 draws; the pass costs 16 blocks per query block.
//
// Segments.  seg_blocks consecutive packed blocks of the order have a centre
// (float32 mean) and a radius no row exceeds; rows with an infinite or NaN value
// are in no answer and left out of both.  They are packed like rows
// (their "norm" is ||c||^2 - r^2, and the tail's last slot holds r), so that
// the split screen's contraction with a query whose own last slot holds -2 T
// gives d(x, c)^2 - ||x||^2 - r^2 - 2 T r: above T^2 - ||x||^2 exactly when
// no row of the segment lies within T of the query.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "morton.hpp"
#include "order_sort.hpp"
#include "rsc_internal.hpp"
#include "screen_common.hpp"
#include "screen_split.hpp"

namespace rsc {
namespace {

using namespace scr;

constexpr int kPivots = 512;
constexpr int kKeyBits = 30;  // 9 pivot rank, 3 distance, 18 Morton

__global__ __launch_bounds__(kPivots) void k_sp_pivots(int64_t n, int32_t *__restrict__ pivot,
                                                       uint32_t *__restrict__ bounds) {
    const int i = threadIdx.x;
    pivot[i] = (int32_t)((2 * (int64_t)i + 1) * n / (2 * kPivots));
    if (i < 3) {
        bounds[2 * i] = 0xffffffffu;
        bounds[2 * i + 1] = 0u;
    }
}

// Squared distances of pivot blockIdx.x to every pivot, and the nearest other;
// the bounding box of the pivots' first three coordinates.
__global__ __launch_bounds__(kPivots) void k_sp_pairs(const float *__restrict__ X, int d,
                                                      const int32_t *__restrict__ pivot, float *__restrict__ D,
                                                      float *__restrict__ nearest, uint32_t *__restrict__ bounds) {
    __shared__ float x[256];
    __shared__ float best[kPivots / kWave];
    const int i = blockIdx.x, j = threadIdx.x;
    const float *xi = X + (int64_t)pivot[i] * d;
    for (int t = j; t < d; t += kPivots) x[t] = xi[t];
    __syncthreads();
    const float *y = X + (int64_t)pivot[j] * d;
    float s = 0.f;
    for (int t = 0; t < d; ++t) {
        const float e = x[t] - y[t];
        s = fmaf(e, e, s);
    }
    D[i * kPivots + j] = s;
    float m = i == j ? INFINITY : s;
    for (int o = 32; o > 0; o >>= 1) m = fminf(m, __shfl_xor(m, o, kWave));
    if ((j & (kWave - 1)) == 0) best[j / kWave] = m;
    __syncthreads();
    if (j == 0) {
        for (int w = 1; w < kPivots / kWave; ++w) m = fminf(m, best[w]);
        nearest[i] = m;
    }
    if (j < 3 && j < d && fabsf(x[j]) < INFINITY) {
        atomicMin(&bounds[2 * j], ordered_bits(x[j]));
        atomicMax(&bounds[2 * j + 1], ordered_bits(x[j]));
    }
}

// Ranks of the pivots: labels of many pivots first, then (label, index).  Rows
// of large clusters then come first in the order, and the query tiles that
// visit most are the first that the launch hands out.
__global__ __launch_bounds__(kPivots) void k_sp_rank(const float *__restrict__ D, const float *__restrict__ nearest,
                                                     int32_t *__restrict__ rank) {
    __shared__ __attribute__((aligned(16))) float nn[kPivots];
    __shared__ __attribute__((aligned(16))) int key[kPivots];
    __shared__ int label[kPivots], size[kPivots];
    __shared__ float cut;
    const int i = threadIdx.x;
    const float mine = nearest[i];
    nn[i] = mine;
    size[i] = 0;
    __syncthreads();
    int below = 0;
#pragma unroll 4
    for (int j = 0; j < kPivots; j += 4) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(&nn[j]);
#pragma unroll
        for (int u = 0; u < 4; ++u) below += v[u] < mine || (v[u] == mine && j + u < i) ? 1 : 0;
    }
    if (below == kPivots / 2) cut = 6.25f * mine;
    __syncthreads();
    int l = i;
#pragma unroll 16
    for (int j = kPivots - 1; j >= 0; --j)
        if (D[j * kPivots + i] <= cut) l = min(l, j);
    label[i] = l;
    __syncthreads();
    const int l2 = label[l];
    atomicAdd(&size[l2], 1);
    __syncthreads();
    const int k = (kPivots - size[l2]) << 18 | l2 << 9 | i;
    key[i] = k;
    __syncthreads();
    int r = 0;
#pragma unroll 4
    for (int j = 0; j < kPivots; j += 4) {
        const int4 v = *reinterpret_cast<const int4 *>(&key[j]);
        r += (v.x < k) + (v.y < k) + (v.z < k) + (v.w < k);
    }
    rank[i] = r;
}

// Sort keys of rows: their nearest pivot's rank, the distance, the Morton code.
template <int Q, int TC>
__global__ __launch_bounds__((SplitShape<Q, TC, 16>::NW * kWave), (SplitShape<Q, TC, 16>::W)) void k_sp_keys(
    const float *__restrict__ X, int64_t n, int d, const void *__restrict__ pivots, const int32_t *__restrict__ rank,
    const uint32_t *__restrict__ bounds, const KnnCounters *__restrict__ kc, uint32_t *__restrict__ key,
    int32_t *__restrict__ id) {
    using S = SplitShape<Q, TC, 16>;
    __shared__ __attribute__((aligned(16))) char ring0[S::RING];
    __shared__ __attribute__((aligned(16))) char ring1[S::RING];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int h = lane >> 5;
    int64_t row = ((int64_t)blockIdx.x * S::NW + wave) * 32 + (lane & 31);
    if (row >= n) row = -1;
    const float scale = ldexpf(1.f, split_exponent(kc));
    SplitQuery<Q, TC> qop;
    qop.load(X, d, row, h, scale);
    float best = INFINITY;
    int at = 0;
    split_stream<Q, TC, S::PH>(
        static_cast<const char *>(pivots), kPivots / 32, [](int i) { return i; }, ring0, ring1,
        [&](const f16x8(&A)[2 * Q + TC], int blk) {
            const f32x16 acc = split_keys<Q, TC>(A, qop);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = blk * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                if (acc[v] < best) {
                    best = acc[v];
                    at = i;
                }
            }
        });
    const float ob = __shfl_xor(best, 32, kWave);
    const int oa = __shfl_xor(at, 32, kWave);
    if (ob < best || (ob == best && oa < at)) {
        best = ob;
        at = oa;
    }
    if (row < 0 || h != 0) return;
    const float *x = X + row * d;
    float xx = 0.f;
    for (int t = 0; t < d; ++t) xx = fmaf(x[t] * scale, x[t] * scale, xx);
    const float d2 = best + xx;  // times the squared scale: at most 2^30
    const int b = d2 > 1.f ? min(7, max(0, (29 - ilogbf(d2)) / 2)) : 7;
    uint32_t code = 0;
    for (int t = 0; t < 3; ++t) {
        if (t >= d) break;
        const float lo = from_ordered(bounds[2 * t]), hi = from_ordered(bounds[2 * t + 1]);
        code |= spread3(quantise10(x[t], lo, scale10(lo, hi)) >> 4) << (2 - t);
    }
    key[row] = (uint32_t)rank[at] << 21 | (uint32_t)b << 18 | code;
    id[row] = (int32_t)row;
}

// Centre and radius of every segment: rows perm[32 seg_blocks s ..].
__global__ __launch_bounds__(256) void k_segments(const float *__restrict__ X, int64_t n, int d,
                                                  const int32_t *__restrict__ perm, int rows,
                                                  const KnnCounters *__restrict__ kc, bool one,
                                                  float *__restrict__ centre, float *__restrict__ radius) {
    __shared__ float part[4][256];
    __shared__ float c[256];
    __shared__ float far[4];
    const int64_t r0 = (int64_t)blockIdx.x * rows;
    const int m = (int)min<int64_t>(rows, n - r0);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    for (int t = lane; t < d; t += kWave) {
        float s = 0.f;
        for (int r = wave; r < m; r += 4) {
            const float v = X[(int64_t)perm[r0 + r] * d + t];
            s += fabsf(v) < INFINITY ? v : 0.f;
        }
        part[wave][t] = s;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < d; t += 256) {
        float v = (part[0][t] + part[1][t] + part[2][t] + part[3][t]) / (float)m;
        // any point is a valid centre: one that the packed form holds exactly
        if (one) v = ldexpf((float)(_Float16)ldexpf(v, split_exponent(kc)), -split_exponent(kc));
        c[t] = v;
        centre[(int64_t)blockIdx.x * d + t] = v;
    }
    __syncthreads();
    float worst = 0.f;
    for (int r = wave; r < m; r += 4) {
        const float *y = X + (int64_t)perm[r0 + r] * d;
        float s = 0.f;
        for (int t = lane; t < d; t += kWave) {
            const float e = y[t] - c[t];
            s = fmaf(e, e, s);
        }
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
        if (s < INFINITY) worst = fmaxf(worst, s);
    }
    if (lane == 0) far[wave] = worst;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float w = fmaxf(fmaxf(far[0], far[1]), fmaxf(far[2], far[3]));
        const float M = __uint_as_float(max(kc->max_norm_bits, kc->query_norm_bits));
        // upwards over the sums' and the packed centre's rounding
        radius[blockIdx.x] = sqrtf(w) * 1.00002f + M * 0x1p-19f;
    }
}

// Segment s as row s % 32 of packed block s / 32.
__global__ __launch_bounds__(256) void k_pack_segments(const float *__restrict__ centre,
                                                       const float *__restrict__ radius, int nseg, int d, int Q,
                                                       int TC, bool one, const KnnCounters *__restrict__ kc,
                                                       f16x8 *__restrict__ out) {
    const int NA = 2 * Q + TC;
    const int total = (nseg + 31) / 32 * NA * kWave;
    const float scale = ldexpf(1.f, split_exponent(kc));
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const int lane = i % kWave, s = i / kWave % NA, b = i / kWave / NA;
        const int h = lane >> 5, seg = 32 * b + (lane & 31);
        const bool live = seg < nseg;
        const float *c = centre + (int64_t)(live ? seg : 0) * d;
        f16x8 v;
        if (s < TC) {
            _Float16 p1 = (_Float16)INFINITY, p2 = (_Float16)0.f, p3 = (_Float16)0.f, rad = (_Float16)0.f;
            if (live) {
                rad = (_Float16)(radius[seg] * scale * 1.002f);
                double cc = 0.0;
                for (int t = 0; t < d; ++t) cc += (double)c[t] * (double)c[t];
                const float N = (float)(cc * (double)scale * (double)scale - (double)rad * (double)rad);
                p1 = (_Float16)(N * 0x1p-15f);
                const float r1 = N - (float)p1 * 32768.f;
                p2 = (_Float16)(r1 * 0x1p-4f);
                p3 = (_Float16)(r1 - (float)p2 * 16.f);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 16 * s + 8 * h + e;
                if (k < 3) {
                    v[e] = k == 0 ? p1 : k == 1 ? p2 : p3;
                } else if (k == 16 * TC - 1) {
                    v[e] = rad;
                } else {
                    const TailSlot at(k, Q, one);
                    _Float16 hi, lo;
                    split16(live && at.t < d ? c[at.t] * scale : 0.f, hi, lo);
                    v[e] = at.part == 2 ? lo : hi;
                }
            }
        } else {
            const bool low = s >= TC + Q;
            const int t0 = 16 * (low ? s - TC - Q : s - TC) + 8 * h;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                _Float16 hi, lo;
                split16(live && t0 + e < d ? c[t0 + e] * scale : 0.f, hi, lo);
                v[e] = low ? lo : hi;
            }
        }
        out[i] = v;
    }
}

// Segment of the references where the middle query of each tile belongs (some
// segment, where the keys are sorted in pieces).
__global__ __launch_bounds__(256) void k_sp_own(const uint32_t *__restrict__ qkey, int64_t nq, int qg, int tiles,
                                                const uint32_t *__restrict__ rkey, int64_t nr, int rows,
                                                int32_t *__restrict__ own) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= tiles) return;
    const uint32_t k = qkey[min((int64_t)i * qg + qg / 2, nq - 1)];
    int64_t lo = 0, hi = nr;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (rkey[mid] < k) lo = mid + 1; else hi = mid;
    }
    own[i] = (int32_t)(min(lo, nr - 1) / rows);
}

int sort_rows(const float *X, int64_t n, int d, const SpatialBuffers &b, uint32_t *sorted, int32_t *perm,
              const KnnCounters *kc, hipStream_t s) {
    const SplitGeom g = split_geom(d);
#define X_(Q, TC)                                                                                               \
    if (g.q == Q && g.tc == TC) {                                                                               \
        constexpr int NW = SplitShape<Q, TC, 16>::NW;                                                           \
        hipLaunchKernelGGL((k_sp_keys<Q, TC>), dim3((unsigned)((n + NW * 32 - 1) / (NW * 32))), dim3(NW * kWave), \
                           0, s, X, n, d, b.pivot_packed, b.rank, b.bounds, kc, b.key, b.id);                   \
    }
    RSC_SPLIT_GEOMS(X_)
#undef X_
    int st = launch_status("spatial keys");
    if (st != RSC_OK) return st;
    return order_sort<uint32_t>(b.tmp, b.tmp_bytes, b.key, sorted, b.id, perm, n, kKeyBits, "sort of the spatial order",
                                s);
}

}  // namespace

int spatial_seg_blocks(int64_t nblk) {
    int sb = 1;
    while ((nblk + sb - 1) / sb > kSegMax) sb *= 2;
    return sb;
}

size_t spatial_carve(int64_t nq, int64_t nr, int d, void *base, SpatialBuffers *out) {
    const int64_t nblk = (nr + 31) / 32;
    SpatialBuffers b{};
    b.seg_blocks = spatial_seg_blocks(nblk);
    b.nseg = (int)((nblk + b.seg_blocks - 1) / b.seg_blocks);
    const size_t most = (size_t)std::max(nq, nr);
    Carver cv(base);
    b.pivot = cv.take<int32_t>(kPivots);
    b.rank = cv.take<int32_t>(kPivots);
    b.nearest = cv.take<float>(kPivots);
    b.pairs = cv.take<float>((size_t)kPivots * kPivots);
    b.bounds = cv.take<uint32_t>(6);
    b.pivot_packed = cv.take<char>(split_packed_bytes(d, kPivots / 32));
    b.key = cv.take<uint32_t>(most);
    b.id = cv.take<int32_t>(most);
    b.rkey = cv.take<uint32_t>((size_t)nr);
    b.rperm = cv.take<int32_t>((size_t)nr);
    b.qkey = cv.take<uint32_t>((size_t)nq);
    b.qperm = cv.take<int32_t>((size_t)nq);
    b.own = cv.take<int32_t>((size_t)(nq + 127) / 128);
    b.centre = cv.take<float>((size_t)b.nseg * d);
    b.radius = cv.take<float>((size_t)b.nseg);
    b.seg_packed = cv.take<char>(split_packed_bytes(d, (b.nseg + 31) / 32));
    b.tmp_bytes = order_sort_bytes<uint32_t>((int64_t)most, kKeyBits);
    b.tmp = cv.take<char>(std::max<size_t>(b.tmp_bytes, 1));
    if (out) *out = b;
    return cv.used;
}

int spatial_refs(const float *R, const float *nrow, int64_t nr, int d, bool rounded, const SpatialBuffers &b,
                 KnnCounters *kc, hipStream_t s) {
    ScopedTimer timer("query_order", s);
    hipLaunchKernelGGL(k_sp_pivots, dim3(1), dim3(kPivots), 0, s, nr, b.pivot, b.bounds);
    hipLaunchKernelGGL(k_sp_pairs, dim3(kPivots), dim3(kPivots), 0, s, R, d, b.pivot, b.pairs, b.nearest, b.bounds);
    hipLaunchKernelGGL(k_sp_rank, dim3(1), dim3(kPivots), 0, s, b.pairs, b.nearest, b.rank);
    int st = split_pack(R, nrow, nr, d, kPivots / 32, b.pivot_packed, nullptr, nullptr, nullptr, b.pivot, kPivots, kc,
                        s);
    if (st != RSC_OK || (st = sort_rows(R, nr, d, b, b.rkey, b.rperm, kc, s)) != RSC_OK) return st;
    const SplitGeom g = rounded ? rounded_geom(d) : split_geom(d);
    hipLaunchKernelGGL(k_segments, dim3((unsigned)b.nseg), dim3(256), 0, s, R, nr, d, b.rperm, 32 * b.seg_blocks, kc,
                       rounded, b.centre, b.radius);
    const int total = (b.nseg + 31) / 32 * g.chunks() * kWave;
    hipLaunchKernelGGL(k_pack_segments, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, b.centre, b.radius,
                       b.nseg, d, g.q, g.tc, rounded, kc, static_cast<f16x8 *>(b.seg_packed));
    return launch_status("segments");
}

int spatial_queries(const float *Q, int64_t nq, int64_t nr, int d, int qg, const SpatialBuffers &b, KnnCounters *kc,
                    hipStream_t s) {
    ScopedTimer timer("query_order", s);
    int st = sort_rows(Q, nq, d, b, b.qkey, b.qperm, kc, s);
    if (st != RSC_OK) return st;
    const int tiles = (int)((nq + qg - 1) / qg);
    hipLaunchKernelGGL(k_sp_own, dim3((unsigned)((tiles + 255) / 256)), dim3(256), 0, s, b.qkey, nq, qg, tiles, b.rkey,
                       nr, 32 * b.seg_blocks, b.own);
    return launch_status("query tiles");
}

}  // namespace rsc
