// Split FP16 screen of the exact path: packing and the grid-mapped launch
// (the operand split, its layout and its arithmetic: screen_split.hpp).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "rsc_internal.hpp"
#include "screen_common.hpp"
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

// Every reference that can lie within bound[i] of listed row i (Euclidean:
// squared): its key is at most bound - ||x||^2 plus the key's error bound.  A
// key passes for little more than the row's m neighbours, so the pass is the
// bare contraction (8192 rows against 1M: 1.7 ms; 45 rows: 60 us, where
// screening them again 64 wide over 16 ranges took 4.2 ms).  Work units are
// (256 listed rows, a range of blocks), enough ranges for every CU.  Inputs
// marked wide are compared in float64 instead.
template <int Q, int TC>
__global__ __launch_bounds__((SplitShape<Q, TC, 16>::NW * kWave), (SplitShape<Q, TC, 16>::W)) void k_split_collect(
    CollectArgs a) {
    using S = SplitShape<Q, TC, 16>;
    __shared__ __attribute__((aligned(16))) char ring0[S::RING];
    __shared__ __attribute__((aligned(16))) char ring1[S::RING];
    const int n = min(*a.nrows, a.cap);
    if (n == 0) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6, h = lane >> 5;
    const bool cosine = a.metric == RSC_COSINE;
    if (a.kc->wide) {
        for (int i = 0; i < n; ++i) {
            const float *x = a.Q0 + (int64_t)a.rows[i] * a.d;
            const double bound = a.bound[i];
            double cxx = 0.0;
            if (cosine)
                for (int t = 0; t < a.d; ++t) cxx = __dadd_rn(cxx, __dmul_rn((double)x[t], (double)x[t]));
            for (int64_t j = (int64_t)blockIdx.x * blockDim.x + tid; j < a.nr; j += (int64_t)gridDim.x * blockDim.x) {
                const float *y = a.R0 + j * a.d;
                double v;
                if (cosine) {
                    double sxy = 0.0, syy = 0.0;
                    for (int t = 0; t < a.d; ++t) {
                        sxy = __dadd_rn(sxy, __dmul_rn((double)x[t], (double)y[t]));
                        syy = __dadd_rn(syy, __dmul_rn((double)y[t], (double)y[t]));
                    }
                    v = (cxx == 0.0 || syy == 0.0)
                            ? 1.0
                            : __dsub_rn(1.0, __ddiv_rn(sxy, __dmul_rn(__dsqrt_rn(cxx), __dsqrt_rn(syy))));
                } else {
                    v = exact_d2(x, y, a.d);
                }
                if (!(v <= bound)) continue;
                const int at = atomicAdd(&a.found[i], 1);
                if (at < a.width) {
                    a.out_idx[(int64_t)i * a.width + at] = (int32_t)j;
                    a.out_key[(int64_t)i * a.width + at] = NAN;  // no screened key
                }
            }
        }
        return;
    }
    const int e = split_exponent(a.kc);
    const float scale = ldexpf(1.f, e);
    const double unit = ldexp(1.0, 2 * e);
    const double ymax = (double)__uint_as_float(a.kc->max_norm_bits) * (1.0 + 1e-6);
    const double M = fmax((double)__uint_as_float(a.kc->query_norm_bits), ymax);
    constexpr int QG = S::NW * 32;
    const int tiles = (n + QG - 1) / QG;
    const int ranges = (int)min((int64_t)((gridDim.x + tiles - 1) / tiles), a.nblk);
    const int per = (int)((a.nblk + ranges - 1) / ranges);
    for (int u = blockIdx.x; u < tiles * ranges; u += gridDim.x) {
        const int b0 = u % ranges * per, b1 = (int)min(a.nblk, (int64_t)b0 + per);
        const int i = u / ranges * QG + wave * 32 + (lane & 31);
        const int64_t row = i < n ? (int64_t)a.rows[i] : -1;
        SplitQuery<Q, TC> qop;
        qop.load(a.Q, a.d, row, h, scale);
        float limit = -INFINITY;
        if (row >= 0) {
            const double dm = a.bound[i];
            double xx = 0.0;
            for (int t = 0; t < a.d; ++t) xx += (double)a.Q[row * a.d + t] * (double)a.Q[row * a.d + t];
            const double xn = sqrt(xx) * (1.0 + 1e-12), Y = fmin(ymax, (xn + sqrt(dm)) * (1.0 + 1e-9));
            const double t = cosine ? 2.0 * dm - 1.0 + a.cosine_eps
                                    : dm - xx + a.eps * (2.0 * xn * Y + Y * Y) + a.eps_abs * M * (2.0 * xn + Y);
            limit = (float)((t + 1e-6 * (fabs(t) + (cosine ? 0.0 : 1e-6 * xx))) * unit);
        }
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
                    if (acc[v] <= limit && slot < a.nr) {
                        const int at = atomicAdd(&a.found[i], 1);
                        if (at < a.width) {
                            a.out_idx[(int64_t)i * a.width + at] = a.ref_map ? a.ref_map[slot] : slot;
                            a.out_key[(int64_t)i * a.width + at] = acc[v];
                        } else {
                            limit = -INFINITY;  // too many: the row is scanned exhaustively
                        }
                    }
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
