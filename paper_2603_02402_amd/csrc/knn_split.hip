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
// of dimensions 0 .. 16 Q - 1.  Rows past the end: zeros and an infinite
// norm.  One workgroup per block: the rows come in coalesced through LDS and
// leave as 16-byte stores.  Marks inputs whose norms spread too far (`wide`).
__global__ __launch_bounds__(256) void k_pack_split(const float *__restrict__ R, const float *__restrict__ nrow,
                                                    int64_t nr, int d, int Q, int TC, int64_t nblk,
                                                    f16x8 *__restrict__ Ap, const int32_t *__restrict__ blk_sample,
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
        const float n2 = row >= 0 ? nrow[row] : 0.f;
        const bool below = row >= 0 && n2 < small;
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
                        v[e] = row >= 0 ? (k == 0 ? p1 : k == 1 ? p2 : p3) : (_Float16)(k == 0 ? INFINITY : 0.f);
                    } else {
                        const int t = 16 * Q + (k - 3) / 3;
                        const float y = t < d ? x[t] : 0.f;
                        wide |= below && y != 0.f;
                        _Float16 hi, lo;
                        split16(y * scale, hi, lo);
                        v[e] = (k - 3) % 3 == 2 ? lo : hi;
                    }
                }
            } else {
                const bool low = s >= TC + Q;
                const int t0 = 16 * (low ? s - TC - Q : s - TC) + 8 * h;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float y = t0 + e < d ? x[t0 + e] : 0.f;
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

}  // namespace

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
               int64_t nmap, KnnCounters *counters, hipStream_t stream) {
    const SplitGeom g = split_geom(d);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(nblk, 1 << 20));
    hipLaunchKernelGGL(k_pack_split, dim3(grid), dim3(256), 32 * (size_t)(d | 1) * sizeof(float), stream, R, nrow, nr,
                       d, g.q, g.tc, nblk, static_cast<f16x8 *>(packed), blk_sample, boff, soff, row_map,
                       nmap, counters);
    return launch_status("pack_split");
}

using scr::split_launch;

int split_screen(const scr::ScreenArgs &a, int half_width, const char *name, hipStream_t s) {
    return half_width == 16 ? split_launch<16>(a, name, s) : split_launch<32>(a, name, s);
}

// Error bound of a split key: per 32x32x16 MFMA two float32 roundings (its
// two groups of 8 products are summed and added one after the other), per
// group of 8 the products' truncation below 2^-24 of the group's largest (7
// units over the high parts' groups by Cauchy-Schwarz, 7 of the norm's
// group), and 8 units for the operands' split and the dropped low x low
// products: (2 MFMAs + 22) units of roundoff of (2 ||x|| ||y|| + ||y||^2),
// doubled for safety.  Operand parts below FP16's smallest step (2^-25 in
// scaled units) add split_abs * M (2 ||x|| + ||y||), M the largest norm.
double split_eps_coefficient(int d) {
    return 2.0 * (2 * split_geom(d).mfmas() + 22) * std::ldexp(1.0, -24);
}
double split_abs_coefficient(int d) { return 2.0 * std::sqrt((double)d) * std::ldexp(1.0, -38); }

}  // namespace rsc
