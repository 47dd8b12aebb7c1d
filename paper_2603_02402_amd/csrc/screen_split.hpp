// The exact path's distance screen on the 16-bit matrix cores: every float32
// operand is split into two FP16 parts whose products are accumulated in
// FP32, so the key keeps (in fact betters) the accuracy of an FP32 chain at
// a fifth of its matrix-core time.
//
// Split.  With a power-of-two scale a = 2^e that brings the largest row norm
// M into [2^13, 2^14),
//   a y = yh + yl + dy,  yh = fp16(a y), yl = fp16(a y - yh),
// |dy| <= max(2^-23 |a y|, 2^-25); the query side splits -2 a x likewise.
// A key is a^2 (||y||^2 - 2 x.y) = norm + xh.yh + xl.yh + xh.yl (the product
// of the two low parts, below 2^-22 of the term, is dropped).  The float32
// norm a^2 ||y||^2 < 2^28 rides as three FP16 parts (33 bits: exact) times
// 2^15, 2^4 and 1.
//
// Contraction.  d = 16 Q + r dimensions (r <= the tail's room): Q chunks of 16
// dimensions are held once as high and once as low parts and multiplied as
// hh, hl, lh (3 Q MFMAs over 2 Q operand chunks); the tail chunks hold the
// norm's three slots and (h, h, l) triples of the remaining r dimensions.
// d = 50: 10 MFMAs of v_mfma_f32_32x32x16_f16 (320 matrix cycles) per 32 x 32
// keys where v_mfma_f32_32x32x2_f32 needs 26 (1664 cycles).
//
// Measured (1M rows, d = 50, k = 15): 258 ms where the FP32 chain took 783 ms;
// 300k rows 26.1 against 78.8 ms.  What bounds it is the matrix cores' power:
// random operands sustain 1.54 PFLOP/s of this MFMA from registers and 1.35
// with the operand reads and the minimum of the epilogue beside it; the
// screen runs at 1.24, and at the same without its selection.  The largest
// key error against float64 over the candidates falls there from 3.6 to 2.9
// units of 2^-24 (2 ||x|| ||y|| + ||y||^2), and over 500 to 300k rows from
// 3.3-5.1 to 2.2-3.2.  (The pruned form of the screen skips most blocks where
// the data has clusters: screen_split_grid.hpp.)
//
// Rounded rows.  The BF16 form sees rows rounded to BF16, whose 8 bits one FP16
// part holds: its chain is the tail alone, the norm's slots and then one slot
// per dimension (ONE below; d = 50: 4 MFMAs).
//
// Range.  Rows whose norm lies below 2^-16 M would lose bits to the FP16
// exponent; prep marks such inputs (KnnCounters::wide) and they take the FP32
// chain of screen_fp32.hpp instead.
#pragma once

#include <type_traits>

#include "rsc_internal.hpp"
#include "screen_common.hpp"

namespace rsc {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace scr {

// Exponent field of the largest norm; the split's scale is 2^(140 - field).
__device__ __forceinline__ int split_scale_field(const KnnCounters *kc) {
    const uint32_t b = max(kc->max_norm_bits, kc->query_norm_bits);
    return (int)(b >> 23);
}
__device__ __forceinline__ int split_exponent(const KnnCounters *kc) { return 140 - split_scale_field(kc); }
// Largest norms outside this range (zero included) take the FP32 chain: the
// scaled norms and the unscaled keys would leave float32's range.
__device__ __forceinline__ bool split_scale_ok(const KnnCounters *kc) {
    const int f = split_scale_field(kc);
    return f >= 77 && f <= 187;
}

// Contraction slots of a split screen: Q full chunks and TC tail chunks.
// Every padded width is 16 Q + 4 (TC = 1) or 16 Q + 9 (TC = 2): three norm
// slots and three per remaining dimension.
struct SplitGeom {
    int q, tc;
    __host__ __device__ constexpr int chunks() const { return 2 * q + tc; }  // operand chunks of 16 slots
    __host__ __device__ constexpr int mfmas() const { return 3 * q + tc; }
    constexpr bool valid() const { return tc > 0; }
};

__host__ __device__ constexpr int split_tail_dims(int tc) { return (16 * tc - 3) / 3; }  // 4, 9

// The instantiated geometries: two per 16 dimensions to d = 57, one per 16
// to 132, then one per 32 (each costs at most one padded chunk triple).
#define RSC_SPLIT_GEOMS_128(X) \
    X(0, 1) X(0, 2) X(1, 1) X(1, 2) X(2, 1) X(2, 2) X(3, 1) X(3, 2) X(4, 1) X(5, 1) X(6, 1) X(7, 1) X(8, 1)
#define RSC_SPLIT_GEOMS(X) RSC_SPLIT_GEOMS_128(X) X(10, 1) X(12, 1) X(14, 1) X(16, 1)

inline SplitGeom split_geom(int d) {
#define X(q, tc) {q, tc},
    constexpr SplitGeom opts[] = {RSC_SPLIT_GEOMS(X)};
#undef X
    for (const SplitGeom &g : opts)
        if (d <= 16 * g.q + split_tail_dims(g.tc)) return g;
    return {0, 0};
}

// f(integral_constant q, integral_constant tc) of the geometry's instantiation.
template <class F>
int split_dispatch(const SplitGeom &g, F f) {
#define X(Q, TC) \
    if (g.q == Q && g.tc == TC) return f(std::integral_constant<int, Q>{}, std::integral_constant<int, TC>{});
    RSC_SPLIT_GEOMS(X)
#undef X
    set_error("internal: no split screen for this dimension");
    return RSC_ERR_UNSUPPORTED;
}

// The rounded rows' geometry: three norm slots, one per dimension, and the last
// one free for a segment's radius.
inline SplitGeom rounded_geom(int d) { return {0, (d + 4 + 15) / 16}; }
#define RSC_ROUNDED_CHUNKS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9)

// Dimension of tail slot k >= 3 and which part of it the slot holds (2: the
// reference's low part, 1: the query's).
struct TailSlot {
    int t, part;
    __device__ __forceinline__ TailSlot(int k, int Q, bool one)
        : t(one ? k - 3 : 16 * Q + (k - 3) / 3), part(one ? 0 : (k - 3) % 3) {}
};

// The two FP16 parts of a scaled float32 value.
__device__ __forceinline__ void split16(float v, _Float16 &hi, _Float16 &lo) {
    hi = (_Float16)v;
    lo = (_Float16)(v - (float)hi);
}

// Query operand of one lane (query c = lane % 32, contraction half h): slot
// 16 s + 8 h + e of chunk s, for -2 a x.
template <int Q, int TC, bool ONE = false>
struct SplitQuery {
    f16x8 hi[Q > 0 ? Q : 1], lo[Q > 0 ? Q : 1], tail[TC];

    __device__ __forceinline__ void load(const float *__restrict__ X, int d, int64_t row, int h, float scale) {
        const float *x = X + (row >= 0 ? row : 0) * d;
        const float m = row >= 0 ? -2.f * scale : 0.f;
#pragma unroll
        for (int s = 0; s < Q; ++s) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int t = 16 * s + 8 * h + e;
                _Float16 a, b;
                split16(t < d ? m * x[t] : 0.f, a, b);
                hi[s][e] = a;
                lo[s][e] = b;
            }
        }
#pragma unroll
        for (int s = 0; s < TC; ++s) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 16 * s + 8 * h + e;
                _Float16 v = (_Float16)0.f;
                if (k < 3) {
                    if (row >= 0) v = (_Float16)(k == 0 ? 32768.f : k == 1 ? 16.f : 1.f);
                } else {
                    const TailSlot at(k, Q, ONE);
                    _Float16 a, b;
                    split16(at.t < d ? m * x[at.t] : 0.f, a, b);
                    v = at.part == 1 ? b : a;
                }
                tail[s][e] = v;
            }
        }
    }
};

// Keys (times a^2) of one packed block for the lane's query.  The products
// with a low part come first, while the sums are 2^-11 of the key's size and
// round at that size; then the tail (with the norm) and the high parts, so
// that the partial sums stay near the key's size: only 2 (TC + Q) of the
// chain's roundings are at full size.  A: the block's operand chunks --
// tail, high parts, low parts.
template <int Q, int TC, bool ONE>
__device__ __forceinline__ f32x16 split_keys(const f16x8 (&A)[2 * Q + TC], const SplitQuery<Q, TC, ONE> &b) {
    f32x16 acc = f32x16{};
#pragma unroll
    for (int s = 0; s < Q; ++s) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[TC + s], b.lo[s], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[TC + Q + s], b.hi[s], acc, 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < TC; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[s], b.tail[s], acc, 0, 0, 0);
#pragma unroll
    for (int s = 0; s < Q; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[TC + s], b.hi[s], acc, 0, 0, 0);
    return acc;
}

// Shape of a split screen's workgroups: one of 4 W waves fills a CU, W waves
// per SIMD (the query operand, the lists and their merge take up to 256
// registers to d = 196, more beyond).  Its waves share a double-buffered LDS
// ring of PH packed blocks per phase that takes what the per-lane queues
// leave of the 160 KiB: the block's operands are read from L2 once per 256
// queries, and a barrier is met every 8 blocks at d = 50.  Measured at 1M
// rows, d = 50: 2 waves per SIMD 258 ms; 4 (spilling) 258 ms with one
// workgroup of 16 waves, 292 with two of 8, 357 with four of 4 (a barrier
// per block); 3 in workgroups of 4 waves 312 ms.
template <int Q, int TC, int L>
struct SplitShape {
    static constexpr int NA = 2 * Q + TC;
    static constexpr int W = NA <= 25 ? 2 : 1;  // waves per SIMD
    static constexpr int NW = 4 * W;            // waves per workgroup: one workgroup fills a CU
    static constexpr int QCAP = 8;
    static constexpr int WGS = 4 * W / NW;  // workgroups per CU
    static constexpr int QBYTES = QCAP * NW * kWave * 8;
    static constexpr int BLOCK = NA * 1024;
    static constexpr int ROOM = (160 * 1024 / WGS - QBYTES - 512) / (2 * BLOCK);
    static constexpr int PH = ROOM < 1 ? 1 : ROOM > 8 ? 8 : ROOM;  // blocks per phase
    // the pruned screen's segment list and bitmap take 20 KiB more
    static constexpr int ROOMP = (160 * 1024 / WGS - QBYTES - 20 * 1024) / (2 * BLOCK);
    static constexpr int PHP = ROOMP < 1 ? 1 : ROOMP > 8 ? 8 : ROOMP;
    static constexpr int RING = PH * BLOCK;
    static constexpr int QG = NW * 32;  // queries per workgroup
};

// Streams packed blocks phys(0) .. phys(count - 1) of Ab through the ring of
// the workgroup and hands each to use(A, block): every wave of the workgroup
// calls this together.  phys may name any block that exists.
template <int Q, int TC, int PH, class Phys, class Use>
__device__ __forceinline__ void split_stream(const char *Ab, int count, Phys phys, char *ring0, char *ring1, Use use) {
    constexpr int NA = 2 * Q + TC, BLOCK = NA * 1024;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int nw = blockDim.x / kWave;
    // this wave's share of the asynchronous loads of phase `ph` into `buf`
    // (positions past the end load the last block again: always in bounds)
    auto issue = [&](int ph, char *buf) {
#pragma unroll
        for (int j = 0; j < (PH * NA + 3) / 4; ++j) {
            const int i = j * nw + wave;
            if (i < PH * NA) {
                const int r = i / NA, s = i - r * NA;
                const int64_t blk = phys(min(ph * PH + r, count - 1));
                load_lds16(Ab + blk * BLOCK + s * 1024 + lane * 16, buf + i * 1024);
            }
        }
    };
    const int nph = (count + PH - 1) / PH;
    auto phase = [&](int ph, const char *cur, char *nxt) {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's loads of phase ph landed
        __syncthreads();                      // everyone's landed; phase ph-1 is fully consumed
        if (ph + 1 < nph) issue(ph + 1, nxt);
        const int n = min(PH, count - ph * PH);
#pragma unroll 1
        for (int r = 0; r < n; ++r) {
            const int blk = phys(ph * PH + r);
            const f16x8 *sl = reinterpret_cast<const f16x8 *>(cur + r * BLOCK) + lane;
            f16x8 A[NA];
#pragma unroll
            for (int s = TC; s < NA; ++s) A[s] = sl[s * kWave];
#pragma unroll
            for (int s = 0; s < TC; ++s) A[s] = sl[s * kWave];
            // all operand reads of the block are in flight before its first MFMA
            if constexpr (NA <= 9) __builtin_amdgcn_sched_barrier(0);
            use(A, blk);
        }
    };
    __syncthreads();  // the ring is free (the previous stream is done with it)
    if (nph > 0) issue(0, ring0);
    for (int ph = 0; ph < nph; ph += 2) {
        phase(ph, ring0, ring1);
        if (ph + 1 < nph) phase(ph + 1, ring1, ring0);
    }
}

// One tile of 32 queries per wave over `span` packed blocks, every `stride`-th from
// b0 on, starting at the `rot`-th and around: every wave of the workgroup calls this
// together.  slot / row: this lane's output slot and query row (or -1);
// ref_base: reference row of packed row 0.
template <int Q, int TC, int L>
__device__ __forceinline__ void screen_split_tile(const ScreenArgs &a, int64_t slot, int64_t row, int b0, int span,
                                                  int stride, int rot, int p, int64_t ref_base, char *ring0, char *ring1,
                                                  double *qbuf) {
    using S = SplitShape<Q, TC, L>;
    const int h = (threadIdx.x & (kWave - 1)) >> 5;
    SplitQuery<Q, TC> qop;
    qop.load(a.Q, a.d, row, h, ldexpf(1.f, split_exponent(a.kc)));
    PackTopK<L, S::QCAP> top;
    top.init();
    double *q = qbuf + threadIdx.x;
    const int qs = blockDim.x;
    split_stream<Q, TC, S::PH>(
        static_cast<const char *>(a.Ap), span,
        [&](int i) {  // packed block of position i of the scan
            int j = rot + i;
            if (j >= span) j -= span;
            return b0 + j * stride;
        },
        ring0, ring1, [&](const f16x8(&A)[2 * Q + TC], int blk) {
            top.offer(split_keys(A, qop), (int)(ref_base + (int64_t)blk * 32) + 4 * h, q, qs);
        });
    top.flush(q, qs);
    if (slot >= 0) top.store(a, slot, p, h, a.ref_map);
}

}  // namespace scr
}  // namespace rsc
