// Split FP16 screen of the exact path: packing and the grid-mapped launch
// (the operand split, its layout and its arithmetic: screen_split.hpp).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "rsc_internal.hpp"
#include "screen_common.hpp"
#include "screen_fp32.hpp"
#include "screen_split_grid.hpp"

namespace rsc {

namespace {

using namespace scr;

// Packed block b of NA = 2 Q + TC chunks: chunk s, lane (c, h) holds the 8
// slots 16 s + 8 h .. of row 32 b + c -- first the tail (norm parts, then
// (h, h, l) triples of dimensions 16 Q ..), then the high and the low parts
// of dimensions 0 .. 16 Q - 1.  Rows past the end, and rows with an infinite or
// NaN value: zeros and an infinite norm.  One workgroup per block: the rows come in coalesced through LDS and
// leave as 16-byte stores.  Marks inputs whose norms spread too far (`wide`).
__global__ __launch_bounds__(256) void k_pack_split(const float *__restrict__ R, const float *__restrict__ nrow,
                                                    int64_t nr, int d, int Q, int TC, bool one,
                                                    int64_t nblk, f16x8 *__restrict__ Ap, const int32_t *__restrict__ blk_sample,
                                                    const int64_t *__restrict__ boff,
                                                    const int64_t *__restrict__ soff,
                                                    const int32_t *__restrict__ row_map, int64_t nmap,
                                                    KnnCounters *counters) {
    extern __shared__ float rows[];  // 32 x (d | 1)
    const int ld = d | 1;
    const int lane = threadIdx.x & (kWave - 1), c = lane & 31, h = lane >> 5;
    const int NA = 2 * Q + TC;
    const float scale = ldexpf(1.f, split_exponent(counters));
    const float M = __uint_as_float(max(counters->max_norm_bits, counters->query_norm_bits));
    const float small = M * M * 0x1p-32f;  // squared norm of 2^-16 M
    bool wide = !split_scale_ok(counters);
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
        // row of packed slot 32 b + i, or -1 (see k_pack)
        auto row_of = [&](int i) -> int64_t {
            int64_t pos = 32 * b + i, end = row_map ? nmap : nr;
            if (blk_sample) {
                const int smp = blk_sample[b];
                pos = soff[smp] + 32 * (b - boff[smp]) + i;
                end = soff[smp + 1];
            }
            if (pos >= end) return -1;
            return row_map ? row_map[pos] : pos;
        };
        __syncthreads();  // the previous block's rows are consumed
        if (row_map) {
            for (int e = threadIdx.x; e < 32 * d; e += blockDim.x) {
                const int i = e / d, t = e - i * d;
                const int64_t row = row_of(i);
                rows[i * ld + t] = row >= 0 ? R[row * d + t] : 0.f;
            }
        } else {
            const int64_t r0 = row_of(0);  // rows of a block are consecutive
            for (int e = threadIdx.x; e < 32 * d; e += blockDim.x) {
                const int i = e / d, t = e - i * d;
                rows[i * ld + t] = row_of(i) >= 0 ? R[r0 * d + e] : 0.f;
            }
        }
        __syncthreads();
        const int64_t row = row_of(c);
        const float n2 = row >= 0 ? nrow[row] : INFINITY;
        const bool live = n2 < INFINITY, below = n2 < small;
        const float *x = rows + c * ld;
        for (int s = threadIdx.x >> 6; s < NA; s += 4) {
            f16x8 v;
            if (s < TC) {
                const float N = n2 * scale * scale;
                const _Float16 p1 = (_Float16)(N * 0x1p-15f);
                const float r1 = N - (float)p1 * 32768.f;
                const _Float16 p2 = (_Float16)(r1 * 0x1p-4f);
                const _Float16 p3 = (_Float16)(r1 - (float)p2 * 16.f);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int k = 16 * s + 8 * h + e;
                    if (k < 3) {
                        v[e] = live ? (k == 0 ? p1 : k == 1 ? p2 : p3) : (_Float16)(k == 0 ? INFINITY : 0.f);
                    } else {
                        const TailSlot at(k, Q, one);
                        const float y = live && at.t < d ? x[at.t] : 0.f;
                        wide |= below && y != 0.f;
                        _Float16 hi, lo;
                        split16(y * scale, hi, lo);
                        v[e] = at.part == 2 ? lo : hi;
                    }
                }
            } else {
                const bool low = s >= TC + Q;
                const int t0 = 16 * (low ? s - TC - Q : s - TC) + 8 * h;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float y = live && t0 + e < d ? x[t0 + e] : 0.f;
                    wide |= below && y != 0.f;
                    _Float16 hi, lo;
                    split16(y * scale, hi, lo);
                    v[e] = low ? lo : hi;
                }
            }
            Ap[(b * NA + s) * kWave + lane] = v;
        }
    }
    if (__ballot(wide) != 0ull && lane == 0) atomicOr(&counters->wide, 1);
}

// Largest key (times `unit`) of a reference that can lie within dm of row `row`:
// the key's error bound added; Y bounds the norm of such a reference.
__device__ __forceinline__ float key_limit(const CollectArgs &a, double dm, int64_t row, double ymax, double M, double eps,
                                           double eps_abs, double cosine_eps, double unit) {
    const bool cosine = a.metric == RSC_COSINE;
    double xx = 0.0;
    for (int t = 0; t < a.d; ++t) xx += (double)a.Q[row * a.d + t] * (double)a.Q[row * a.d + t];
    const double xn = sqrt(xx) * (1.0 + 1e-12), Y = fmin(ymax, (xn + sqrt(dm)) * (1.0 + 1e-9));
    const double t = cosine ? 2.0 * dm - 1.0 + cosine_eps
                            : dm - xx + eps * (2.0 * xn * Y + Y * Y) + eps_abs * M * (2.0 * xn + Y);
    return (float)((t + 1e-6 * (fabs(t) + (cosine ? 0.0 : 1e-6 * xx))) * unit);
}

// Files a reference under listed row i.
__device__ __forceinline__ void file(const CollectArgs &a, int i, int32_t ref, float key, float &limit) {
    const int at = atomicAdd(&a.found[i], 1);
    if (at < a.width) {
        a.out_idx[(int64_t)i * a.width + at] = ref;
        a.out_key[(int64_t)i * a.width + at] = key;
    } else {
        limit = -INFINITY;  // too many: the row is scanned exhaustively
    }
}

// The collection on inputs marked wide, in the FP32 chain's keys: the wave's 32
// listed rows (this lane's: entry i, row `row` or -1) against packed blocks
// [b0, b1).  Four blocks share a reading of the query's values.  8192 rows
// against 100k x 50: 2.2 ms, where comparing each pair in float64 took 174.
__device__ __forceinline__ void collect_wide(const CollectArgs &a, int i, int64_t row, int b0, int b1) {
    const int lane = threadIdx.x & (kWave - 1), h = lane >> 5;
    const int folded = norm_folded(a.dh) ? 1 : 0, S4 = packed_s4(a.dh), steps = a.dh + folded;
    const double ymax = (double)__uint_as_float(a.kc->max_norm_bits) * (1.0 + 1e-6);
    // keys that could leave float32's range bound nothing: every listed row is scanned exhaustively
    if (!(fmax(ymax, (double)__uint_as_float(a.kc->query_norm_bits)) < 0x1p62)) {
        if (row >= 0 && b0 == 0 && h == 0) a.found[i] = a.width + 1;
        return;
    }
    float limit =
        row >= 0 ? key_limit(a, a.bound[i], row, ymax, 0.0, a.fp32_eps, 0.0, a.fp32_cosine_eps, 1.0) + 0x1p-140f : -INFINITY;
    const float *x = a.Q + (row >= 0 ? row : 0) * a.d;
    const f32x4 *A = static_cast<const f32x4 *>(a.packed32) + lane;
    constexpr int NB = 4;
    for (int b = b0; b < b1; b += NB) {
        f32x16 acc[NB] = {};
        for (int s4 = 0; s4 < S4; ++s4) {
            float q[4];
            f32x4 y[NB];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = 4 * s4 + u, t = h * a.dh + s - folded;
                q[u] = 0.f;
                if (folded && s == 0)
                    q[u] = h == 0 ? 1.f : 0.f;
                else if (s < steps && t < a.d)
                    q[u] = -2.f * x[t];
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) y[j] = A[((int64_t)min(b + j, b1 - 1) * S4 + s4) * kWave];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(y[j][u], q[u], acc[j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (b + j >= b1) break;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float key = folded ? acc[j][v] : acc[j][v] + a.norms32[(int64_t)(b + j) * 32 + h * 16 + v];
                const int ref = (b + j) * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                if (key <= limit && ref < a.nr) file(a, i, ref, key, limit);
            }
        }
    }
}

// Every reference that can lie within bound[i] of listed row i (Euclidean:
// squared): its key is at most bound - ||x||^2 plus the key's error bound.  A
// key passes for little more than the row's m neighbours, so the pass is the
// bare contraction (8192 rows against 1M: 1.7 ms; 45 rows: 60 us, where
// screening them again 64 wide over 16 ranges took 4.2 ms).  Work units are
// (256 listed rows, a range of blocks), enough ranges for every CU.
template <int Q, int TC>
__global__ __launch_bounds__((SplitShape<Q, TC, 16>::NW * kWave), (SplitShape<Q, TC, 16>::W)) void k_split_collect(
    CollectArgs a) {
    using S = SplitShape<Q, TC, 16>;
    __shared__ __attribute__((aligned(16))) char ring0[S::RING];
    __shared__ __attribute__((aligned(16))) char ring1[S::RING];
    const int n = min(*a.nrows, a.cap);
    if (n == 0) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6, h = lane >> 5;
    constexpr int QG = S::NW * 32;
    const int tiles = (n + QG - 1) / QG;
    const int ranges = (int)min((int64_t)((gridDim.x + tiles - 1) / tiles), a.nblk);
    const int per = (int)((a.nblk + ranges - 1) / ranges);
    if (a.kc->wide) {
        for (int u = blockIdx.x; u < tiles * ranges; u += gridDim.x) {
            const int b0 = u % ranges * per, b1 = (int)min(a.nblk, (int64_t)b0 + per);
            const int i = u / ranges * QG + wave * 32 + (lane & 31);
            collect_wide(a, i, i < n ? (int64_t)a.rows[i] : -1, b0, b1);
        }
        return;
    }
    const int e = split_exponent(a.kc);
    const float scale = ldexpf(1.f, e);
    const double unit = ldexp(1.0, 2 * e);
    const double ymax = (double)__uint_as_float(a.kc->max_norm_bits) * (1.0 + 1e-6);
    const double M = fmax((double)__uint_as_float(a.kc->query_norm_bits), ymax);
    for (int u = blockIdx.x; u < tiles * ranges; u += gridDim.x) {
        const int b0 = u % ranges * per, b1 = (int)min(a.nblk, (int64_t)b0 + per);
        const int i = u / ranges * QG + wave * 32 + (lane & 31);
        const int64_t row = i < n ? (int64_t)a.rows[i] : -1;
        SplitQuery<Q, TC> qop;
        qop.load(a.Q, a.d, row, h, scale);
        float limit = row >= 0 ? key_limit(a, a.bound[i], row, ymax, M, a.eps, a.eps_abs, a.cosine_eps, unit) : -INFINITY;
        split_stream<Q, TC, S::PH>(
            static_cast<const char *>(a.packed), max(0, b1 - b0), [&](int j) { return b0 + j; }, ring0, ring1,
            [&](const f16x8(&A)[2 * Q + TC], int blk) {
                const f32x16 acc = split_keys<Q, TC>(A, qop);
                float mn = acc[0];
#pragma unroll
                for (int v = 1; v < 16; ++v) mn = fminf(mn, acc[v]);
                if (__ballot(mn <= limit) == 0ull) return;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int slot = blk * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (acc[v] <= limit && slot < a.nr) file(a, i, a.ref_map ? a.ref_map[slot] : slot, acc[v], limit);
                }
            });
    }
}

}  // namespace

int split_collect(const CollectArgs &a, hipStream_t s) {
    return scr::split_dispatch(scr::split_geom(a.d), [&](auto q, auto tc) {
        hipLaunchKernelGGL((k_split_collect<q.value, tc.value>), dim3((unsigned)scr::kCUs),
                           dim3(SplitShape<q.value, tc.value, 16>::NW * kWave), 0, s, a);
        return launch_status("collect");
    });
}

template int scr::split_launch<16>(const scr::ScreenArgs &, const char *, hipStream_t);

size_t split_packed_bytes(int d, int64_t nblk) { return (size_t)nblk * split_geom(d).chunks() * 1024; }
size_t rounded_packed_bytes(int d, int64_t nblk) { return (size_t)nblk * scr::rounded_geom(d).chunks() * 1024; }

int split_queries_per_group(int d, int half_width) {
    int qg = 0;
    scr::split_dispatch(scr::split_geom(d), [&](auto q, auto tc) {
        qg = half_width == 16 ? SplitShape<q.value, tc.value, 16>::QG : SplitShape<q.value, tc.value, 32>::QG;
        return RSC_OK;
    });
    return qg;
}

int split_pack(const float *R, const float *nrow, int64_t nr, int d, int64_t nblk, void *packed,
               const int32_t *blk_sample, const int64_t *boff, const int64_t *soff, const int32_t *row_map,
               int64_t nmap, KnnCounters *counters, hipStream_t stream, bool rounded) {
    const SplitGeom g = rounded ? rounded_geom(d) : split_geom(d);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(nblk, 1 << 20));
    hipLaunchKernelGGL(k_pack_split, dim3(grid), dim3(256), 32 * (size_t)(d | 1) * sizeof(float), stream, R, nrow, nr,
                       d, g.q, g.tc, rounded, nblk, static_cast<f16x8 *>(packed), blk_sample, boff, soff, row_map,
                       nmap, counters);
    return launch_status("pack_split");
}

using scr::split_launch;

int split_screen(const scr::ScreenArgs &a, int half_width, const char *name, hipStream_t s) {
    return half_width == 16 ? split_launch<16>(a, name, s) : split_launch<32>(a, name, s);
}

int split_screen_pruned(const PrunedArgs &a, int half_width, const char *name, hipStream_t s) {
    if (a.rounded) return scr::rounded_launch(a, name, s);
    return half_width == 16 ? scr::pruned_launch<16>(a, name, s) : scr::pruned_launch<32>(a, name, s);
}

// Error bound of a split key, in units of roundoff u = 2^-24 of S = 2 ||x||
// ||y|| + ||y||^2, from the structure of v_mfma_f32_32x32x16_f16 (two groups of
// 8 exact products, each summed with what lies below u of the group's largest
// product cut off, then added to the accumulator one after the other with
// rounding to nearest; read off a probe of the instruction):
//   2 (TC + Q)  the roundings of the tail and the high parts' MFMAs, those of
//               the low parts before them are 2^-11 of that size (1 for all);
//   7           the cut-off products: 7 per group, over the groups at most u
//               (||y||^2 + the sum of |2 x_t y_t|);
//   8           the split: |x - xh - xl| <= 2^-23 |x| on either side and the
//               dropped xl yl <= 2^-22 |x y|;
// with half as much again for safety.  Operand parts below FP16's smallest
// step (2^-25 in scaled units) add split_abs M (2 ||x|| + ||y||), M the largest
// norm.
double split_eps_coefficient(int d) {
    const scr::SplitGeom g = scr::split_geom(d);
    return 1.5 * (2 * (g.tc + g.q) + 16) * std::ldexp(1.0, -24);
}
double split_abs_coefficient(int d) { return 2.0 * std::sqrt((double)d) * std::ldexp(1.0, -38); }

}  // namespace rsc
