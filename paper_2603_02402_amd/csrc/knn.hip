// Exact kNN on gfx950: MFMA distance screen + float64 rerank + certificate.
//
// The paper's neighbour step needs, per cell, the k nearest cells of the
// PCA embedding under the squared Euclidean distance of Methods, "Custom
// GPU kernels" (d_ij = ||x_i - x_j||^2).  The work is a dense contraction
// (2 d flops per ordered pair), so the screen runs on the matrix cores:
//
//   key_ij = ||y_j||^2 - 2 x_i . y_j      (= d_ij - ||x_i||^2, same order per row)
//
// The screen.  Operands are split into two FP16 parts and the keys accumulated in
// float32 (screen_split.hpp): the references are packed once in MFMA operand
// order and pass through an LDS ring that a workgroup of 8 waves, 32 queries
// each, shares; a lane keeps, in registers, the 16 or 32 smallest keys of the
// half of the rows its contraction half sees.  Large problems are searched in a
// spatial order whose segments carry bounds (k_split_pruned); where bounds do
// not help, lists of 32 and the BF16 form go to a scan of everything.  Inputs
// whose norms spread too far for FP16 parts are marked, and the FP32 chain
// (screen_fp32.hpp) answers them: both are launched, one returns at once.
// A launch may split the references into P ranges (blockIdx.y) to give small
// problems enough workgroups and long answers enough lists.
//
// The screen is not the answer.  Its rounding error is bounded per query, every
// candidate is re-ranked with float64 distances summed from direct differences
// in dimension order, and a row is certified exact when its m-th re-ranked
// distance is below the smallest key any range could have rejected, minus the
// bound.  Rows that fail collect every reference whose key can lie below the
// distance found (answers to 64; k_split_collect) or go through a wider FP32
// screen over many ranges (longer ones), and an exhaustive float64 scan where
// that does not settle them either.  Ties are broken towards the lower index
// throughout.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>

#include "rsc_internal.hpp"
#include "screen_common.hpp"
#include "screen_fp32.hpp"
#include "screen_split_grid.hpp"

namespace rsc {

namespace {

using namespace scr;

constexpr int kMaxD = 256;       // exact FP32 path (reduced-precision screens: 128)
constexpr int kMaxK = 255;       // exact FP32 path (reduced-precision screens: 63)
constexpr int kMaxDLowp = 128;
constexpr int kMaxKLowp = 63;
// References and query-reference pairs from which the exact search is pruned:
// ordering them and bounding the segments costs 0.15 ms at 16k rows and 0.9 ms
// at 1M.  Screen, rerank and order at 16384 rows (20 clusters): 0.41 ms pruned,
// 0.46 without (in a Morton order); at 10k rows 0.39 against 0.21; rectangular:
// the pairs of that square.  The BF16 form's rows (64 candidates a query) take
// the same path from there: 16.5k rows 1.40 -> 0.72 ms, 40k 2.25 -> 1.02, 500k
// 44.4 -> 14.6 (100 clusters, with their graph).  Rows without clusters gain
// nothing from bounds: a sample of the tiles finds that out (pruned_args).
constexpr int64_t kPruneRows = 16384;
constexpr double kPrunePairs = 2.5e8;
// Foreign queries from which it is: fewer pay for ordering the references without
// a gain (in ms, not pruned and pruned, rows in 5 to 100 clusters: 600 of 1M rows,
// d = 20, k = 15, 1.04, 2.88; 2000 of 500k, d = 50, 1.15, 1.78; 4500 of 300k, d = 50,
// k = 30, 1.89, 1.80 to 2.39; of 800k, d = 90, 4.28, 4.70 to 4.94, d = 20 2.19, 1.86 to
// 2.13; 12,000 1.0 to 1.35 times as long without).
constexpr int64_t kPruneQueries = 4000;
// Rows from which answers longer than 64 are: near rows crowd a range's lists, and
// some rows are searched again (in ms, not pruned and pruned, rows in 5, 30 and 78
// clusters: 20k rows, d = 50, k = 100, 1.35; 1.74, 1.54, 1.02; d = 90, k = 100, 2.06;
// 2.60, 2.09, 2.25; 25k, d = 50, k = 255, 2.97; 2.68, 2.50, 2.67; d = 90, k = 100 32k
// 3.28; 3.72, 2.69, 2.64).
constexpr int64_t kPruneRowsLong = 20480;
// Foreign queries from which the BF16 form is pruned: fewer do not pay for ordering
// the references.  In ms, plain and pruned, rows in 100 clusters: 2500 queries of
// 100k rows 0.89, 1.05; 3500 1.24, 1.10; 3500 of 500k 2.27, 2.71; 5000 2.70, 2.70;
// 5000 of 1M 3.97, 4.82; 8000 5.01, 4.72.
inline int64_t prune_queries_bf16(int64_t nr) { return std::max<int64_t>(3000, 2500 + nr / 200); }
// Workgroups the split screen asks for before it stops splitting the
// references: fewer leave CUs idle, more multiply the candidate lists the
// rerank reads (10k rows: screen + rerank 0.34 ms at 128, 0.47 at 256, 0.74
// at 512; 50k rows: 2.15 / 2.08 ms at 128 / 256).
constexpr int64_t kSplitWant = 128;
constexpr int kEscalateCap = 8192;  // rows handled by the escalation screen
constexpr int kEscalateSplits = 16;
constexpr int kEscalateWidth = 64;

// Squared norms of the reference rows (float64 sum, rounded once) and the
// largest norm.  A workgroup takes norm_rows(d) rows (64 for d <= 128): they
// are contiguous in memory and come into LDS with coalesced loads, then four
// lanes sum each row.  Bound by reading the rows; one wave per 64 rows, a lane
// summing each, kept 5 waves on a CU (245 us at 640k x 50, now 58).
constexpr int kNormRows = 64;
constexpr int kNormThreads = 256;
constexpr int kNormBuf = kNormRows * 129;  // floats staged per block
__host__ __device__ inline int norm_rows(int d) { return d <= 128 ? kNormRows : kNormRows * 128 / d; }

__global__ __launch_bounds__(kNormThreads) void k_norms(const float *__restrict__ R, int64_t nr, int d,
                                                        float *__restrict__ nrow,
                                                        uint32_t *__restrict__ max_norm_bits) {
    // nrow may be null: only the largest norm is wanted.  A row with an infinite or
    // NaN value has such a norm, which packing takes for no row, and stays out of
    // the largest (a finite row whose norm overflows float32 does enter it).
    __shared__ float buf[kNormBuf];
    __shared__ float wmax[kNormThreads / kWave];
    const int nrb = norm_rows(d);
    const int64_t r0 = (int64_t)blockIdx.x * nrb;
    const int rows = (int)min<int64_t>(nrb, nr - r0);
    const int ld = d | 1;
    const float *src = R + r0 * d;
    for (int e = threadIdx.x; e < rows * d; e += kNormThreads) buf[e / d * ld + e % d] = src[e];
    __syncthreads();
    const int i = threadIdx.x >> 2, q = threadIdx.x & 3;
    double s = 0.0;
    if (i < rows)
        for (int t = q; t < d; t += 4) {
            const double x = (double)buf[i * ld + t];
            s += x * x;
        }
    s += __shfl_xor(s, 1, kWave);
    s += __shfl_xor(s, 2, kWave);
    const float nf = (float)s;
    if (nrow && i < rows && q == 0) nrow[r0 + i] = nf;
    const float m = wave_max(s < INFINITY ? sqrtf(nf) : 0.f);
    if ((threadIdx.x & (kWave - 1)) == 0) wmax[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t bits = __float_as_uint(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])));
        // an atomic only where the maximum grows: they all meet in one word
        if (bits > *(volatile uint32_t *)max_norm_bits) atomicMax(max_norm_bits, bits);
    }
}

// Unit-normalised rows for the cosine screen: x / ||x|| with the norm summed
// in float64 and rounded once to float32, then one float32 division per
// element (each element within 2 units of roundoff of x_t / ||x||); a row of
// zero norm stays zero.  Rows staged as in k_norms.
__global__ __launch_bounds__(kNormThreads) void k_normalize(const float *__restrict__ X, int64_t n, int d,
                                                            float *__restrict__ out) {
    __shared__ float buf[kNormBuf];
    __shared__ float norm[kNormRows];
    const int nrb = norm_rows(d);
    const int64_t r0 = (int64_t)blockIdx.x * nrb;
    const int rows = (int)min<int64_t>(nrb, n - r0);
    const int ld = d | 1;
    for (int e = threadIdx.x; e < rows * d; e += kNormThreads) buf[e / d * ld + e % d] = X[r0 * d + e];
    __syncthreads();
    const int i = threadIdx.x >> 2, q = threadIdx.x & 3;
    double s = 0.0;
    if (i < rows)
        for (int t = q; t < d; t += 4) {
            const double x = (double)buf[i * ld + t];
            s += x * x;
        }
    s += __shfl_xor(s, 1, kWave);
    s += __shfl_xor(s, 2, kWave);
    if (i < rows && q == 0) norm[i] = (float)sqrt(s);
    __syncthreads();
    for (int e = threadIdx.x; e < rows * d; e += kNormThreads) {
        const float nrm = norm[e / d];
        out[r0 * d + e] = nrm > 0.f ? buf[e / d * ld + e % d] / nrm : 0.f;
    }
}

// Packed reference layout for a contraction half-width DH.  Block b holds
// rows 32b..32b+31:
//   A[b][s4][lane] (float4): element u = step s = 4 s4 + u of lane (c, h).
//       With the norm folded, step 0 of half 0 is ||R[32b + c]||^2 (+inf
//       past the end; half 1 holds 0) and step 1 + t is R[32b + c][h DH + t];
//       otherwise step t is R[32b + c][h DH + t].  0 elsewhere.  Putting the
//       norm first keeps the partial sums of the key near its final size;
//   N[b][h][4g + j] (only when not folded): ||R[32b + 8g + 4h + j]||^2, the
//       accumulator order of the 32x32 output block (+inf past the end);
// so that MFMA step s of a wave reads 1 KiB of lane-contiguous data.
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ R, const float *__restrict__ nrow, int64_t nr,
                                              int d, int DH, int S4, int folded, int64_t nblk,
                                              f32x4 *__restrict__ Ap, float *__restrict__ Np,
                                              const int32_t *__restrict__ blk_sample, const int64_t *__restrict__ boff,
                                              const int64_t *__restrict__ soff, const int32_t *__restrict__ row_map,
                                              const KnnCounters *__restrict__ gate) {
    if (gate && gate->wide == 0) return;  // the split screen answers
    const int64_t total = nblk * S4 * kWave;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int lane = (int)(e % kWave);
        const int64_t bs = e / kWave;
        const int s4 = (int)(bs % S4);
        const int64_t b = bs / S4;
        // row of lane (c, h); batched: blocks of sample s start at boff[s] and
        // hold rows soff[s]..soff[s+1]-1 (the last block of a sample is padded)
        // routed form: packed row 32b + c holds row_map[32b + c] (-1: padding)
        int64_t row = 32 * b + (lane & 31), row_end = nr;
        if (blk_sample) {
            const int smp = blk_sample[b];
            row = soff[smp] + 32 * (b - boff[smp]) + (lane & 31);
            row_end = soff[smp + 1];
        }
        bool live = row < row_end;
        if (row_map) {
            row = row_map[32 * b + (lane & 31)];
            live = row >= 0;
        }
        const int h = lane >> 5;
        f32x4 v;
        const int off = folded ? 1 : 0;  // the norm occupies step 0 when folded
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = 4 * s4 + u;
            const int sd = s - off;        // dimension step
            const int t = h * DH + sd;
            float x = 0.f;
            if (folded && s == 0) {
                if (h == 0) x = live ? nrow[row] : INFINITY;
            } else if (sd < DH) {
                if (live && t < d) x = R[row * d + t];
            }
            v[u] = x;
        }
        Ap[e] = v;
        if (!folded && s4 == 0) {
            // lane (c, h) of block b also files the norm of row 32b + c into accumulator order
            if (h == 0) {
                const int i = lane & 31;
                const int g = i >> 3, hh = (i >> 2) & 1, j = i & 3;
                Np[b * 32 + hh * 16 + 4 * g + j] = live ? nrow[row] : INFINITY;
            }
        }
    }
}

__global__ void k_set_i32(int32_t *p, int32_t v) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

__global__ void k_init_counters(KnnCounters *c) {
    if (threadIdx.x == 0) {
        c->flagged = 0;
        c->max_ratio_bits = 0u;
        c->max_norm_bits = 0u;
        c->flagged2 = 0;
        c->rescanned = 0;
        c->query_norm_bits = 0u;
        c->wide = 0;
        c->verdict = 0;
        c->sampled = 0;
        c->sampled_segments = 0ull;
        c->visited = 0ull;
    }
}

// ---------------------------------------------------------------------------
// Screen.
//
// Lane l handles query c = l % 32 of its wave and contraction half
// h = l / 32: a step of the MFMA chain multiplies dimension h*DH + t (plus
// the norm step, first, when folded).
// Output register v of the 32x32 block holds reference row 8(v/4) + 4h +
// (v%4), so each lane sees half of the references of every block and keeps
// its own sorted list of the L smallest keys of that half.
// Query slot i of the launch is row i, or row qlist[i] for i < min(*qcount,
// qcap) when a list is given (the escalation pass).
// Output: cand[(slot * 2P + 2p + h) * L + i], i-th smallest key of half h
// of range p (index -1 / key +inf where fewer than L were seen).
// ---------------------------------------------------------------------------
template <int DH, int L, int W>
__global__ __launch_bounds__(256, W) void k_screen_fp32(ScreenArgs a) {
    // Per-lane queue of keys that beat the lane's threshold (see LaneTopK).
    __shared__ float2 qbuf[kQueueCap * 256];
    constexpr int QG = kScreenWaves * 32;
    if (a.only_wide && a.kc->wide == 0) return;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, c = tid & 31;
    const int p = blockIdx.y;
    const int64_t blk_per = (a.nblk + a.P - 1) / a.P;
    const int64_t blk0 = (int64_t)p * blk_per;
    const int64_t blk1 = std::min<int64_t>(a.nblk, blk0 + blk_per);
    const int64_t nslots = screen_slots(a);
    for (int64_t qblk = blockIdx.x; qblk * QG < nslots; qblk += gridDim.x) {
        const int64_t slot = qblk * QG + wave * 32 + c;
        int64_t row = -1;
        if (slot < nslots) row = a.qlist ? (int64_t)a.qlist[slot] : slot;
        screen_fp32_tile<DH, L>(a, slot < nslots ? slot : -1, row, blk0, blk1, p, 0, qbuf);
    }
}

// ---------------------------------------------------------------------------
// Rerank + certificate: one wave per query slot.  Candidates of all P ranges
// are streamed 64 at a time; the m best (d2, j) are kept sorted across the
// lanes (lane i = i-th smallest) by bitonic sort + merge.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void bitonic_sort64(double &d2, int &jj, int lane) {
#pragma unroll
    for (int size = 2; size <= kWave; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const double od = __shfl_xor(d2, stride, kWave);
            const int oj = __shfl_xor(jj, stride, kWave);
            const bool want_min = ((lane & stride) == 0) == ((lane & size) == 0);
            const bool other_first = lex_before(od, oj, d2, jj);
            if (want_min == other_first) {
                d2 = od;
                jj = oj;
            }
        }
    }
}

// Sort a bitonic 64-sequence (d2, jj) ascending in (d, j) order.
__device__ __forceinline__ void bitonic_clean64(double &d2, int &jj, int lane) {
#pragma unroll
    for (int stride = kWave >> 1; stride > 0; stride >>= 1) {
        const double xd = __shfl_xor(d2, stride, kWave);
        const int xj = __shfl_xor(jj, stride, kWave);
        const bool lower = (lane & stride) == 0;
        const bool other_first = lex_before(xd, xj, d2, jj);
        if (lower == other_first) {
            d2 = xd;
            jj = xj;
        }
    }
}

// The m smallest (d, j) seen so far, m <= 64 R, sorted across the wave:
// position p = 64 r + lane lives in register r of that lane (+inf / INT_MAX
// where fewer were seen).  A sorted 64-chunk is merged register by register:
// the 64 smallest of (register r, carry) stay in r, the rest carry on.
template <int R>
struct TopM {
    double d[R];
    int j[R];

    __device__ __forceinline__ void init() {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            d[r] = INFINITY;
            j[r] = INT_MAX;
        }
    }
    // (d, j) at position p (p wave-uniform)
    __device__ __forceinline__ void at(int p, double &pd, int &pj) const {
        double rd = d[0];
        int rj = j[0];
#pragma unroll
        for (int r = 1; r < R; ++r)
            if (p >> 6 == r) {
                rd = d[r];
                rj = j[r];
            }
        pd = __shfl(rd, p & (kWave - 1), kWave);
        pj = __shfl(rj, p & (kWave - 1), kWave);
    }
    // merge a sorted chunk (cd, cj), lane i = i-th smallest
    __device__ __forceinline__ void merge(double cd, int cj, int lane) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double od = __shfl(cd, kWave - 1 - lane, kWave);
            const int oj = __shfl(cj, kWave - 1 - lane, kWave);
            const bool take = lex_before(od, oj, d[r], j[r]);
            const double hd = take ? d[r] : od;
            const int hj = take ? j[r] : oj;
            if (take) {
                d[r] = od;
                j[r] = oj;
            }
            bitonic_clean64(d[r], j[r], lane);
            if (r + 1 < R) {
                cd = hd;
                cj = hj;
                if (__ballot(cd < INFINITY) == 0ull) break;  // nothing left to carry
                bitonic_clean64(cd, cj, lane);
            }
        }
    }
};

// Candidate rows are staged through LDS 32 dimensions at a time: for each
// batch of 64 candidates (one per lane) the wave copies the rows' chunk with
// coalesced loads (two 128-byte row segments per instruction), then every
// lane continues its own float64 sum in dimension order from LDS, so the
// distances are those of exact_d2 bit for bit.
constexpr int kRerankChunk = 32;

template <int R>
__global__ __launch_bounds__(256) void k_rerank(RerankArgs a) {
    __shared__ float tile[4][kWave][kRerankChunk + 1];
    __shared__ float qrow[4][kMaxD];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int64_t slot = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave;
    int64_t nslots = a.nq;
    if (a.qlist) nslots = std::min<int64_t>(std::min<int64_t>(*a.qcount, a.qcap), a.nq);
    if (slot >= nslots) return;
    const int64_t row = a.qlist ? (int64_t)a.qlist[slot] : slot;
    const float *x = a.Q + row * a.d;
    float(*T)[kRerankChunk + 1] = tile[wave];
    float *xs = qrow[wave];
    for (int t = lane; t < a.d; t += kWave) xs[t] = x[t];

    // ||x||^2 in float64 (only feeds the certificate's margin)
    double xx = 0.0;
    for (int t = lane; t < a.d; t += kWave) xx += (double)x[t] * (double)x[t];
    xx = wave_sum(xx);
    const double xn = sqrt(xx) * (1.0 + 1e-12);
    const double ymax = (double)__uint_as_float(a.counters->max_norm_bits) * (1.0 + 1e-6);
    const bool cosine = a.metric == RSC_COSINE;
    // units and error bound of the screened keys
    const bool split = a.split && a.counters->wide == 0 && (a.split == 1 || a.counters->verdict != kPlain);
    const double kscale = split ? ldexp(1.0, -2 * scr::split_exponent(a.counters)) : 1.0;
    const double eps_coef = split ? a.split_eps : a.eps_coef;
    const double cosine_eps = split ? a.split_cosine_eps : a.cosine_eps;
    const double eps_abs =
        split ? a.split_abs * fmax((double)__uint_as_float(a.counters->query_norm_bits), ymax) : 0.0;
    // cosine: the query's squared norm summed in dimension order (as every
    // pair's distance below and the oracle compute it)
    double cxx = 0.0;
    if (cosine) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
        for (int t = 0; t < a.d; ++t) {
            const double v = (double)xs[t];
            cxx = __dadd_rn(cxx, __dmul_rn(v, v));
        }
    }

    // Smallest key any full range could have rejected.
    float tau = INFINITY;
    const int64_t cbase = slot * a.P * a.KP;
    for (int p = 0; p < a.P; ++p) {
        int j = -1;
        float key = -INFINITY;
        if (lane < a.S) {
            j = a.cand_idx[cbase + p * a.KP + lane];
            key = a.cand_key[cbase + p * a.KP + lane];
        }
        const bool full = __ballot(lane < a.S && j < 0) == 0ull;
        const float root = wave_max(key);
        if (full) tau = fminf(tau, root);
    }

    TopM<R> top;
    top.init();
    float ratio = 0.f;
    const int total = a.P * a.S;
    for (int c0 = 0; c0 < total; c0 += kWave) {
        const int ci = c0 + lane;
        int j = -1;
        float key = 0.f;
        if (ci < total) {
            const int p = ci / a.S, e = ci - (ci / a.S) * a.S;
            j = a.cand_idx[cbase + p * a.KP + e];
            key = a.cand_key[cbase + p * a.KP + e];
        }
        const bool valid = j >= 0 && !(a.self_mode && j == row);
        const int jl = valid ? j : 0;  // a row of R that exists, loaded (and ignored) for empty slots
        double s2 = 0.0, yy = 0.0, sxy = 0.0;
        for (int k0 = 0; k0 < a.d; k0 += kRerankChunk) {
            const int w = min(kRerankChunk, a.d - k0);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");  // earlier reads of the tile are done
            __builtin_amdgcn_wave_barrier();
#pragma unroll 4
            for (int i = 0; i < kWave / 2; ++i) {
                const int r = 2 * i + (lane >> 5), cc = lane & (kRerankChunk - 1);
                const int jr = __shfl(jl, r, kWave);
                if (cc < w) T[r][cc] = a.R[(int64_t)jr * a.d + k0 + cc];
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");  // the tile is written
            __builtin_amdgcn_wave_barrier();
            if (cosine) {
                for (int t = 0; t < w; ++t) {
                    const double y = (double)T[lane][t];
                    sxy = __dadd_rn(sxy, __dmul_rn((double)xs[k0 + t], y));
                    yy = __dadd_rn(yy, __dmul_rn(y, y));
                }
            } else {
                for (int t = 0; t < w; ++t) {
                    const double y = (double)T[lane][t];
                    const double diff = __dsub_rn((double)xs[k0 + t], y);
                    s2 = __dadd_rn(s2, __dmul_rn(diff, diff));
                    yy += y * y;
                }
            }
        }
        double d2 = INFINITY;
        int jj = INT_MAX;
        if (valid) {
            jj = j;
            if (cosine) {
                // 1 - x.y / (||x|| ||y||); a row of zero norm is at distance 1
                const bool zero = cxx == 0.0 || yy == 0.0;
                d2 = zero ? 1.0 : __dsub_rn(1.0, __ddiv_rn(sxy, __dmul_rn(__dsqrt_rn(cxx), __dsqrt_rn(yy))));
                // the screen ranked 2 D - 1 (unit vectors) up to cosine_eps
                if (!zero) ratio = fmaxf(ratio, (float)(fabs((double)key * kscale - (2.0 * d2 - 1.0)) / cosine_eps));
            } else {
                d2 = s2;
                const double yn = sqrt(yy);
                const double err_bound = eps_coef * (2.0 * xn * yn + yy) + eps_abs * (2.0 * xn + yn) + 1e-300;
                ratio = fmaxf(ratio, (float)(fabs((double)key * kscale - (d2 - xx)) / err_bound));
            }
        }
        bitonic_sort64(d2, jj, lane);
        top.merge(d2, jj, lane);
    }
    ratio = wave_max(ratio);
    if (lane == 0 && ratio > 0.f) atomicMax(&a.counters->max_ratio_bits, __float_as_uint(ratio));

    const int m = a.self_mode ? a.k - 1 : a.k;  // neighbours to certify
    // norms whose squares overflow float32 leave the screen no keys: such inputs are scanned exhaustively
    bool ok = !a.certify || m == 0 || ymax < INFINITY;
    if (a.certify && m > 0 && tau < INFINITY && cosine) {
        // Unit vectors: a rejected reference y had a screened key >= tau, and
        // the key is 2 D_y - 1 up to cosine_eps, so D_y >= (tau + 1 - eps) / 2,
        // which must exceed D_m.  (A zero row's key may be far from its
        // D_y = 1 but never above it: the bound still holds for it.)
        double dm;
        int jm;
        top.at(m - 1, dm, jm);
        const double bound = ((double)tau * kscale + 1.0 - cosine_eps) * 0.5 - 1e-13;
        ok = ok && dm < bound;
    } else if (a.certify && m > 0 && tau < INFINITY) {
        // A rejected reference y had a screened key >= tau.  If ||y|| > Y =
        // ||x|| + D_m it lies farther than D_m (triangle inequality); else its
        // float32 key is off by at most eps(Y), so its true key is >= tau -
        // eps(Y), which must exceed D_m^2 - ||x||^2.
        double dm;
        int jm;
        top.at(m - 1, dm, jm);
        const double Y = fmin(ymax, (xn + sqrt(dm)) * (1.0 + 1e-9));
        const double eps = eps_coef * (2.0 * xn * Y + Y * Y) + eps_abs * (2.0 * xn + Y);
        const double t = (double)tau * kscale;
        const double bound = t + xx - eps - 1e-12 * (fabs(t) + xx);
        ok = ok && dm < bound;
    }

    int32_t *oi = a.out_idx + row * a.k;
    float *od = a.out_dist + row * a.k;
    const int off = a.self_mode ? 1 : 0;
    if (a.self_mode && lane == 0) {
        oi[0] = (int32_t)row;
        od[0] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int pos = r * kWave + lane;
        if (pos < m) {
            oi[off + pos] = top.j[r] == INT_MAX ? -1 : top.j[r];
            od[off + pos] = cosine ? (float)top.d[r] : (float)sqrt(top.d[r]);
        }
    }
    if (!ok && lane == 0) {
        const int pos = atomicAdd(a.flag_count, 1);
        a.flag_out[pos] = (int32_t)row;
    }
}

// ---------------------------------------------------------------------------
// Rerank of short answers (at most 64 neighbours): one group of G lanes per
// query slot, two queries per wave while 32 lanes hold their answers.
//
// Of the P S candidates only those whose screened key can still belong to
// the m nearest are compared in float64: the m-th smallest key plus twice
// the key's error bound is an upper bound for the key of any of the m
// nearest (m candidates have a true key below the m-th smallest plus one
// bound; a candidate whose key lies above that by more than another bound is
// farther than all of them).  At k = 15 that leaves about 16 of 32 candidates
// (of 224 with 7 reference ranges).  The bound on the m-th smallest comes from
// a bisection on the keys with ballots, to 2^-12 of their range.
//
// The survivors' rows come in through LDS, 32 dimensions at a time (16 lanes
// of 8 bytes per row when the rows allow it, else 32 of 4), then each lane
// sums its own candidate in dimension order (exact_d2's arithmetic), and the
// order of the answers is a count of smaller (distance, index) pairs in LDS.
// More survivors than lanes: pass by pass, against the best so far.
// ---------------------------------------------------------------------------
constexpr int kLeanAnswer = 64;            // neighbours a group of 64 lanes holds
constexpr int kLeanChunk = 32;             // dimensions staged per pass
constexpr int kLeanLd = kLeanChunk + 2;    // LDS row stride: 8-byte reads of 32 lanes meet 32 bank pairs

template <int G, int KR, int VEC>
__global__ __launch_bounds__(256) void k_rerank_lean(RerankArgs a) {
    constexpr int NG = 256 / G;     // groups of the workgroup
    constexpr int PW = kWave / G;   // groups of a wave
    constexpr int LPR = kLeanChunk / VEC;  // lanes loading one row's chunk
    constexpr int RPI = G / LPR;           // rows per load instruction of a group
    __shared__ __attribute__((aligned(16))) float tile[NG][G * kLeanLd];
    __shared__ double ed[NG][2 * G];
    __shared__ int ej[NG][2 * G];
    __shared__ int sj[NG][2 * G];   // survivors waiting (candidate rows and their keys)
    __shared__ float sk[NG][2 * G];
    extern __shared__ float xrow[];  // NG x (d | 1) + 1
    const int lane = threadIdx.x & (kWave - 1);
    const int gl = threadIdx.x & (G - 1), g = threadIdx.x / G;
    const int half = lane / G;       // group of the wave
    const int64_t slot = (int64_t)blockIdx.x * NG + g;
    int64_t nslots = a.nq;
    if (a.qlist) nslots = std::min<int64_t>(std::min<int64_t>(*a.qcount, a.qcap), a.nq);
    if (slot - half >= nslots) return;  // the wave's first slot
    const int64_t row = slot < nslots ? (a.qlist ? (int64_t)a.qlist[slot] : slot) : -1;
    const bool live = row >= 0;
    auto wave_sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
    };
    // bits of this group in a wave's ballot
    auto group_ballot = [&](bool v) -> unsigned long long {
        const unsigned long long b = __ballot(v);
        return PW == 1 ? b : (b >> (half * G)) & ((1ull << (G & 63)) - 1);
    };

    const float *x = a.Q + (live ? row : 0) * a.d;
    float *xs = xrow + g * (a.d | 1);
    for (int t = gl; t < a.d; t += G) xs[t] = x[t];
    // ||x||^2 in float64 (only feeds the certificate's margin)
    double xx = 0.0;
    for (int t = gl; t < a.d; t += G) xx += (double)x[t] * (double)x[t];
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) xx += __shfl_xor(xx, o, kWave);
    const double xn = sqrt(xx) * (1.0 + 1e-12);
    const double ymax = (double)__uint_as_float(a.counters->max_norm_bits) * (1.0 + 1e-6);
    const bool cosine = a.metric == RSC_COSINE;
    const bool split = a.split && a.counters->wide == 0 && (a.split == 1 || a.counters->verdict != kPlain);
    const double kscale = split ? ldexp(1.0, -2 * scr::split_exponent(a.counters)) : 1.0;
    const double eps_coef = split ? a.split_eps : a.eps_coef;
    const double cosine_eps = split ? a.split_cosine_eps : a.cosine_eps;
    const double eps_abs =
        split ? a.split_abs * fmax((double)__uint_as_float(a.counters->query_norm_bits), ymax) : 0.0;
    wave_sync();
    double cxx = 0.0;  // cosine: the query's squared norm summed in dimension order
    if (cosine)
        for (int t = 0; t < a.d; ++t) {
            const double v = (double)xs[t];
            cxx = __dadd_rn(cxx, __dmul_rn(v, v));
        }

    // the candidates: lists of S keys, ascending; tau: the smallest key a full list could have rejected
    const int m = a.self_mode ? a.k - 1 : a.k;
    const int found = a.counts && live ? a.counts[slot] : 0;
    // (a row with more than its room is scanned exhaustively: none of its entries are taken, or need be written)
    const int total = a.counts ? (found <= a.KP ? found : 0) : a.P * a.S;
    const int64_t cbase = (live ? slot : 0) * a.P * a.KP;
    float key[KR];
    int cj[KR];
    float tau = INFINITY, kmin = INFINITY, kmax = -INFINITY;
    int nvalid = 0;
#pragma unroll
    for (int i = 0; i < KR; ++i) {
        const int ci = i * G + gl;
        key[i] = INFINITY;
        cj[i] = -1;
        if (live && ci < total) {
            const int p = a.counts ? 0 : ci / a.S, e = ci - p * a.S;
            const int j = a.cand_idx[cbase + p * a.KP + e];
            const float v = a.cand_key[cbase + p * a.KP + e];
            if (e == a.S - 1 && j >= 0) tau = fminf(tau, v);
            if (j >= 0 && !(a.self_mode && j == row)) {
                key[i] = v;
                cj[i] = j;
                // cosine: the key of a zero row says nothing about its distance
                if (!(cosine && v == 0.f)) {
                    kmin = fminf(kmin, v);
                    kmax = fmaxf(kmax, v);
                }
            }
        }
        nvalid += __popcll(group_ballot(cj[i] >= 0 && !(cosine && key[i] == 0.f)));
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        tau = fminf(tau, __shfl_xor(tau, o, kWave));
        kmin = fminf(kmin, __shfl_xor(kmin, o, kWave));
        kmax = fmaxf(kmax, __shfl_xor(kmax, o, kWave));
    }
    // keys up to `cut` may belong to the answer
    float cut = INFINITY;
    const double slack =
        cosine ? 2.0 * cosine_eps : 2.0 * (eps_coef * (2.0 * xn + ymax) * ymax + eps_abs * (2.0 * xn + ymax));
    if (a.certify && nvalid > m && m > 0 && slack < INFINITY && kmax < INFINITY) {
        float lo = kmin, hi = kmax;  // at least m keys are <= hi
        for (int it = 0; it < 12; ++it) {
            const float mid = 0.5f * lo + 0.5f * hi;
            int c = 0;
#pragma unroll
            for (int i = 0; i < KR; ++i) c += __popcll(group_ballot(key[i] <= mid && !(cosine && key[i] == 0.f)));
            if (c >= m) hi = mid; else lo = mid;
        }
        const double t = (double)hi * kscale;
        cut = (float)((t + slack + 1e-6 * (fabs(t) + slack)) / kscale);
    }

    int mb = 0;       // best so far
    float ratio = 0.f;
    int waiting = 0;  // survivors in sj / sk (group-uniform)
    // Distances of the first min(waiting, G) survivors, merged into the best.
    // Every group of the wave calls this together.
    auto pass = [&]() {
        const int nc = min(waiting, G);
        double s2 = 0.0, yy = 0.0, sxy = 0.0;
        float *T = tile[g];
        const int ncw = PW == 1 ? nc : max(nc, __shfl_xor(nc, G & 63, kWave));  // either group's
        for (int k0 = 0; k0 < a.d; k0 += kLeanChunk) {
            const int w = min(kLeanChunk, a.d - k0);
            const int e = (gl % LPR) * VEC;
            float2 buf[G / RPI / 2];
#pragma unroll
            for (int hb = 0; hb < 2; ++hb) {  // the rows in two halves of loads in flight
                if (hb * (G / 2) >= ncw) break;
#pragma unroll
                for (int i = 0; i < G / RPI / 2; ++i) {
                    const int r = hb * (G / 2) + i * RPI + gl / LPR;
                    buf[i] = make_float2(0.f, 0.f);
                    if (r < nc && e < w) {
                        const float *y = a.R + (int64_t)sj[g][r] * a.d + k0 + e;
                        if constexpr (VEC == 2)
                            buf[i] = *reinterpret_cast<const float2 *>(y);
                        else
                            buf[i].x = *y;
                    }
                }
                if (hb == 0) wave_sync();  // earlier reads of the tile are done
#pragma unroll
                for (int i = 0; i < G / RPI / 2; ++i) {
                    const int r = hb * (G / 2) + i * RPI + gl / LPR;
                    if constexpr (VEC == 2)
                        *reinterpret_cast<float2 *>(&T[r * kLeanLd + e]) = buf[i];
                    else
                        T[r * kLeanLd + e] = buf[i].x;
                }
            }
            wave_sync();  // the tile is written
            if (cosine) {
                for (int t = 0; t < w; ++t) {
                    const double y = (double)T[gl * kLeanLd + t];
                    sxy = __dadd_rn(sxy, __dmul_rn((double)xs[k0 + t], y));
                    yy = __dadd_rn(yy, __dmul_rn(y, y));
                }
            } else {
                auto step = [&](float xv, float yv) {
                    const double diff = __dsub_rn((double)xv, (double)yv);
                    s2 = __dadd_rn(s2, __dmul_rn(diff, diff));
                    yy = fma((double)yv, (double)yv, yy);
                };
                int t = 0;
                for (; t + 1 < w; t += 2) {
                    const float2 y = *reinterpret_cast<const float2 *>(&T[gl * kLeanLd + t]);
                    step(xs[k0 + t], y.x);
                    step(xs[k0 + t + 1], y.y);
                }
                if (t < w) step(xs[k0 + t], T[gl * kLeanLd + t]);
            }
        }
        double d2 = INFINITY;
        int jj = INT_MAX;
        if (gl < nc) {
            jj = sj[g][gl];
            const double skey = (double)sk[g][gl] * kscale;
            if (cosine) {
                // 1 - x.y / (||x|| ||y||); a row of zero norm is at distance 1
                const bool zero = cxx == 0.0 || yy == 0.0;
                d2 = zero ? 1.0 : __dsub_rn(1.0, __ddiv_rn(sxy, __dmul_rn(__dsqrt_rn(cxx), __dsqrt_rn(yy))));
                // the screen ranked 2 D - 1 (unit vectors) up to cosine_eps
                if (!zero) ratio = fmaxf(ratio, (float)(fabs(skey - (2.0 * d2 - 1.0)) / cosine_eps));
            } else {
                d2 = s2;
                const double yn = sqrt(yy);
                const double err_bound =
                    eps_coef * (2.0 * xn * yn + yy) + eps_abs * (2.0 * xn + yn) + 1e-300;
                ratio = fmaxf(ratio, (float)(fabs(skey - (d2 - xx)) / err_bound));
            }
        }
        // the waiting list moves up; ranks among the best so far and the new ones
        double bd = INFINITY;
        int bj = INT_MAX;
        if (gl < mb) {
            bd = ed[g][gl];
            bj = ej[g][gl];
        }
        const int mj = sj[g][G + gl];
        const float mk = sk[g][G + gl];
        wave_sync();
        sj[g][gl] = mj;
        sk[g][gl] = mk;
        if (gl < nc) {
            ed[g][mb + gl] = d2;
            ej[g][mb + gl] = jj;
        }
        wave_sync();
        const int ne = mb + nc;
        const int new_ = PW == 1 ? ne : max(ne, __shfl_xor(ne, G & 63, kWave));
        int rn = 0, rb = 0;
        for (int e = 0; e < new_; ++e) {
            if (e < ne) {
                const double od = ed[g][e];
                const int oj = ej[g][e];
                rn += lex_before(od, oj, d2, jj) ? 1 : 0;
                rb += lex_before(od, oj, bd, bj) ? 1 : 0;
            }
        }
        wave_sync();
        if (gl < mb && rb < m) {
            ed[g][rb] = bd;
            ej[g][rb] = bj;
        }
        if (gl < nc && rn < m) {
            ed[g][rn] = d2;
            ej[g][rn] = jj;
        }
        mb = min(m, ne);
        waiting -= nc;
        wave_sync();
    };
#pragma unroll
    for (int i = 0; i < KR; ++i) {
        if (__ballot(i * G < total) == 0ull) break;
        const bool in = cj[i] >= 0 && (a.counts || key[i] <= cut || (cosine && key[i] == 0.f));
        const unsigned long long b = group_ballot(in);
        if (in) {
            const int at = waiting + __popcll(b & ((1ull << gl) - 1));
            sj[g][at] = cj[i];
            sk[g][at] = key[i];
        }
        waiting += __popcll(b);
        wave_sync();
        if (__ballot(waiting >= G) != 0ull) pass();
    }
    while (__ballot(waiting > 0) != 0ull) pass();

    ratio = wave_max(ratio);
    if (lane == 0 && ratio > 0.f && __float_as_uint(ratio) > *(volatile uint32_t *)&a.counters->max_ratio_bits)
        atomicMax(&a.counters->max_ratio_bits, __float_as_uint(ratio));
    if (!live) return;

    // the certificate of k_rerank
    const double dm = m > 0 && mb >= m ? ed[g][m - 1] : (double)INFINITY;
    bool ok = !a.certify || m == 0 || ymax < INFINITY;
    if (a.certify && m > 0 && tau < INFINITY) {
        const double t = (double)tau * kscale;
        if (cosine) {
            ok = ok && dm < (t + 1.0 - cosine_eps) * 0.5 - 1e-13;
        } else {
            const double Y = fmin(ymax, (xn + sqrt(dm)) * (1.0 + 1e-9));
            const double eps = eps_coef * (2.0 * xn * Y + Y * Y) + eps_abs * (2.0 * xn + Y);
            ok = ok && dm < t + xx - eps - 1e-12 * (fabs(t) + xx);
        }
    }
    int32_t *oi = a.out_idx + row * a.k;
    float *od = a.out_dist + row * a.k;
    const int off = a.self_mode ? 1 : 0;
    if (a.self_mode && gl == 0) {
        oi[0] = (int32_t)row;
        od[0] = 0.f;
    }
    for (int pos = gl; pos < m; pos += G) {
        const bool have = pos < mb;
        const double d = have ? ed[g][pos] : (double)INFINITY;
        oi[off + pos] = have ? ej[g][pos] : -1;
        od[off + pos] = cosine ? (float)d : (float)sqrt(d);
    }
    if (found > a.KP) ok = false;
    if (!ok && gl == 0) {
        const int pos = atomicAdd(a.flag_count, 1);
        a.flag_out[pos] = (int32_t)row;
        if (a.flag_bound && pos < a.flag_cap) {
            a.flag_bound[pos] = dm;
            a.flag_found[pos] = 0;
        }
    }
}

// ---------------------------------------------------------------------------
// Exhaustive float64 scan of the rows no screen could certify: rows
// list2[0..count2) and list1[cap..count1).  One wave per row: each step the
// 64 lanes compute the distances of 64 consecutive references; a step with
// a distance before the current m-th is sorted and merged into the row's
// wave-wide top-m (TopM).
// ---------------------------------------------------------------------------
template <int R>
__global__ __launch_bounds__(64) void k_rescan(const float *__restrict__ Q, const float *__restrict__ Rf, int64_t nr,
                                               int d, int k, int self_mode, const int32_t *__restrict__ list1,
                                               const int32_t *__restrict__ count1, int cap1,
                                               const int32_t *__restrict__ list2,
                                               const int32_t *__restrict__ count2, int32_t *__restrict__ out_idx,
                                               float *__restrict__ out_dist, KnnCounters *__restrict__ counters,
                                               const int64_t *__restrict__ soff, int nsamples, int metric) {
    const int lane = threadIdx.x;
    const int m = self_mode ? k - 1 : k;
    const int c2 = *count2;
    const int extra = std::max(0, *count1 - cap1);
    const int count = c2 + extra;
    if (blockIdx.x == 0 && lane == 0) counters->rescanned = count;
    for (int f = blockIdx.x; f < count; f += gridDim.x) {
        const int64_t q = f < c2 ? list2[f] : list1[cap1 + (f - c2)];
        const float *x = Q + q * d;
        // references: all rows, or the rows of q's own sample (batched form)
        int64_t j0 = 0, j1 = nr;
        if (soff) {
            int lo = 0, hi = nsamples - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) / 2;
                if (soff[mid] <= q) lo = mid; else hi = mid - 1;
            }
            j0 = soff[lo];
            j1 = soff[lo + 1];
        }
        double cxx = 0.0;  // cosine: the query's squared norm, dimensions in order
        if (metric == RSC_COSINE)
            for (int t = 0; t < d; ++t) cxx = __dadd_rn(cxx, __dmul_rn((double)x[t], (double)x[t]));
        TopM<R> top;
        top.init();
        for (int64_t jb = j0; jb < j1; jb += kWave) {
            const int64_t j = jb + lane;
            double v = INFINITY;
            int jj = INT_MAX;
            if (j < j1 && !(self_mode && j == q)) {
                const float *y = Rf + j * d;
                if (metric == RSC_COSINE) {
                    double sxy = 0.0, syy = 0.0;
                    for (int t = 0; t < d; ++t) {
                        sxy = __dadd_rn(sxy, __dmul_rn((double)x[t], (double)y[t]));
                        syy = __dadd_rn(syy, __dmul_rn((double)y[t], (double)y[t]));
                    }
                    v = (cxx == 0.0 || syy == 0.0)
                            ? 1.0
                            : __dsub_rn(1.0, __ddiv_rn(sxy, __dmul_rn(__dsqrt_rn(cxx), __dsqrt_rn(syy))));
                } else {
                    v = exact_d2(x, y, d);
                }
                jj = (int)j;
            }
            if (m < 1) continue;
            double md;
            int mj;
            top.at(m - 1, md, mj);
            if (__ballot(lex_before(v, jj, md, mj)) == 0ull) continue;
            bitonic_sort64(v, jj, lane);
            top.merge(v, jj, lane);
        }
        int32_t *oi = out_idx + q * k;
        float *od = out_dist + q * k;
        const int off = self_mode ? 1 : 0;
        if (self_mode && lane == 0) {
            oi[0] = (int32_t)q;
            od[0] = 0.f;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int pos = r * kWave + lane;
            if (pos < m) {
                oi[off + pos] = top.j[r] == INT_MAX ? -1 : top.j[r];
                od[off + pos] = metric == RSC_COSINE ? (float)top.d[r] : (float)sqrt(top.d[r]);
            }
        }
    }
}

// Registers per lane of the running top-m list.
int topm_regs(int m) { return m <= 64 ? 1 : m <= 128 ? 2 : 4; }

// sparse: a grid with few active workgroups (the escalation)
template <int DH, int L>
int launch_screen(const ScreenArgs &a, unsigned gx, bool sparse, const char *name, hipStream_t stream) {
    ScopedTimer timer(name, stream);
    constexpr int WF = tile_screen_waves(DH, L), WS = screen_min_waves(DH, L);
    if (sparse && WS != WF)
        hipLaunchKernelGGL((k_screen_fp32<DH, L, WS>), dim3(gx, (unsigned)a.P), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((k_screen_fp32<DH, L, WF>), dim3(gx, (unsigned)a.P), dim3(256), 0, stream, a);
    return launch_status(name);
}

template <int L>
int dispatch_screen(int dh, const ScreenArgs &a, unsigned gx, bool sparse, const char *name, hipStream_t s) {
    switch (dh) {
        case 4: return launch_screen<4, L>(a, gx, sparse, name, s);
        case 8: return launch_screen<8, L>(a, gx, sparse, name, s);
        case 16: return launch_screen<16, L>(a, gx, sparse, name, s);
        case 25: return launch_screen<25, L>(a, gx, sparse, name, s);
        case 32: return launch_screen<32, L>(a, gx, sparse, name, s);
        case 48: return launch_screen<48, L>(a, gx, sparse, name, s);
        case 64: return launch_screen<64, L>(a, gx, sparse, name, s);
        case 96: return launch_screen<96, L>(a, gx, sparse, name, s);
        case 128: return launch_screen<128, L>(a, gx, sparse, name, s);
        default: set_error("internal: no screen kernel for this dimension"); return RSC_ERR_UNSUPPORTED;
    }
}

// One launch of the screen; `half_width` is the list length per contraction
// half; `sparse` marks a grid with few active workgroups.
int screen(int dh, const ScreenArgs &a, unsigned gx, int half_width, bool sparse, const char *name, hipStream_t s) {
    if (half_width == 16) return dispatch_screen<16>(dh, a, gx, sparse, name, s);
    return dispatch_screen<32>(dh, a, gx, sparse, name, s);
}

constexpr int kQueriesPerGroup = kScreenWaves * 32;

int pick_dh(int d) {
    const int half = (d + 1) / 2;
    const int opts[] = {4, 8, 16, 25, 32, 48, 64, 96, 128};
    for (int o : opts)
        if (half <= o) return o;
    return -1;
}

// Reference ranges for the main screen: `want` workgroups to fill the chip
// while every range keeps at least 8 blocks.
int pick_splits(int64_t nq, int64_t nblk, int qg, int64_t want) {
    const int64_t qblocks = std::max<int64_t>((nq + qg - 1) / qg, 1);
    int64_t P = qblocks >= want ? 1 : (want + qblocks - 1) / qblocks;
    P = std::min<int64_t>(P, std::max<int64_t>(1, nblk / 8));
    P = std::min<int64_t>(P, 32);
    return (int)std::max<int64_t>(P, 1);
}

}  // namespace

// Bound on |screened key - (2 D - 1)| for the cosine screen: the key error of
// unit vectors (eps_coef (2 |x||y| + |y|^2) with norms within 4 units of 1)
// plus the normalisation: each unit vector is within 2 units of roundoff per
// element of the exact direction, which moves |y|^2 by at most 4 units and
// x.y by at most 4 units (doubled in the key), with a margin.
static double cosine_eps_of(double eps_coef) { return 3.0001 * eps_coef + 16.0 * std::ldexp(1.0, -24); }

// Error bound of the float32 key (the norm enters the MFMA sum or is added
// after it; norms rounded once from float64): 2 (d + 3) units of roundoff
// times (2 ||x|| ||y|| + ||y||^2).
double knn_eps_coefficient(int d) { return 2.0 * (d + 3) * std::ldexp(1.0, -24); }

void knn_split_bounds(RerankArgs &ra) {
    ra.split = 1;
    ra.split_eps = split_eps_coefficient(ra.d);
    ra.split_abs = split_abs_coefficient(ra.d);
    ra.split_cosine_eps = cosine_eps_of(ra.split_eps);
}

// The largest norm of a rectangular problem's queries.
static int query_norms(const KnnPlan &p, const float *Q, const KnnBuffers &b, hipStream_t stream) {
    hipLaunchKernelGGL(k_norms, dim3((unsigned)((p.nq + norm_rows(p.d) - 1) / norm_rows(p.d))), dim3(kNormThreads), 0,
                       stream, Q, p.nq, p.d, nullptr, &b.counters->query_norm_bits);
    return launch_status("query norms");
}

int knn_prep(const KnnPlan &p, const float *R, const float *Q, const KnnBuffers &b, hipStream_t stream) {
    ScopedTimer timer("prep_pack", stream);
    const int st = knn_norms(R, p.nr, p.d, b.nrow, b.counters, stream);
    return st == RSC_OK && Q && p.nq > 0 ? query_norms(p, Q, b, stream) : st;
}

int knn_pack_fp32(int dh, const float *R, const float *nrow, int64_t nr, int d, int64_t nblk, float *packed,
                  float *norms, const int32_t *blk_sample, const int64_t *boff, const int64_t *soff,
                  const int32_t *row_map, const KnnCounters *gate, hipStream_t stream) {
    const int s4 = packed_s4(dh);
    ScopedTimer timer("pack_wide", stream);
    const int64_t tot = nblk * s4 * kWave;
    // (gated: most often idle)
    const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((tot + 255) / 256, gate ? 2048 : 65536));
    hipLaunchKernelGGL(k_pack, dim3(g), dim3(256), 0, stream, R, nrow, nr, d, dh, s4, norm_folded(dh) ? 1 : 0, nblk,
                       reinterpret_cast<f32x4 *>(packed), norms, blk_sample, boff, soff, row_map, gate);
    return launch_status("pack_wide");
}

int knn_norms(const float *R, int64_t nr, int d, float *nrow, KnnCounters *counters, hipStream_t stream) {
    hipLaunchKernelGGL(k_init_counters, dim3(1), dim3(64), 0, stream, counters);
    hipLaunchKernelGGL(k_norms, dim3((unsigned)((nr + norm_rows(d) - 1) / norm_rows(d))), dim3(kNormThreads), 0, stream, R,
                       nr, d, nrow, &counters->max_norm_bits);
    return launch_status("norms");
}

size_t knn_packed_floats(int dh, int64_t nblk) { return (size_t)nblk * packed_s4(dh) * kWave * 4; }

template <int G, int KR>
void launch_rerank_lean(const RerankArgs &ra, int64_t slots, hipStream_t stream) {
    constexpr int NG = 256 / G;
    const dim3 grid((unsigned)((slots + NG - 1) / NG));
    const size_t lds = ((size_t)NG * (ra.d | 1) + 1) * sizeof(float);
    // 8-byte row loads need even rows from an 8-byte boundary
    if (ra.d % 2 == 0 && (reinterpret_cast<uintptr_t>(ra.R) & 7u) == 0)
        hipLaunchKernelGGL((k_rerank_lean<G, KR, 2>), grid, dim3(256), lds, stream, ra);
    else
        hipLaunchKernelGGL((k_rerank_lean<G, KR, 1>), grid, dim3(256), lds, stream, ra);
}

int knn_launch_rerank(const RerankArgs &ra, int64_t slots, const char *name, hipStream_t stream) {
    ScopedTimer timer(name, stream);
    const dim3 grid((unsigned)((slots + 3) / 4));
    const int m = ra.self_mode ? ra.k - 1 : ra.k, total = ra.P * ra.S;
    // two rows per wave while 32 lanes hold the answer and a lane few candidates;
    // candidates per lane in steps, as every pass over them counts all (128 in
    // 4 registers for 8: 70k rows, k = 30 230 -> 199 us; in 2 for 8: 300k rows,
    // k = 48 1.73 -> 1.43 ms)
    if (m <= 32 && total <= 32)
        launch_rerank_lean<32, 1>(ra, slots, stream);
    else if (m <= 32 && total <= 64)
        launch_rerank_lean<32, 2>(ra, slots, stream);
    else if (m <= 32 && total <= 128)
        launch_rerank_lean<32, 4>(ra, slots, stream);
    else if (m <= 32 && total <= 256)
        launch_rerank_lean<32, 8>(ra, slots, stream);
    else if (m <= kLeanAnswer && total <= 128)
        launch_rerank_lean<64, 2>(ra, slots, stream);
    else if (m <= kLeanAnswer && total <= 512)
        launch_rerank_lean<64, 8>(ra, slots, stream);
    else if (m <= kLeanAnswer && total <= 2048)
        launch_rerank_lean<64, 32>(ra, slots, stream);
    else if (m <= 128)
        hipLaunchKernelGGL(k_rerank<2>, grid, dim3(256), 0, stream, ra);
    else
        hipLaunchKernelGGL(k_rerank<4>, grid, dim3(256), 0, stream, ra);
    return launch_status(name);
}

int knn_launch_rescan(const KnnPlan &p, const float *Q, const float *R, const KnnBuffers &b, int esc_cap,
                      int32_t *out_idx, float *out_dist, const int64_t *soff, int nsamples, hipStream_t stream) {
    ScopedTimer timer("rescan", stream);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(1024), dim3(64), 0, stream, Q, R, p.nr, p.d, p.k, p.self_mode ? 1 : 0, b.flag1,
                           &b.counters->flagged, esc_cap, b.flag2, &b.counters->flagged2, out_idx, out_dist,
                           b.counters, soff, nsamples, p.metric);
    };
    switch (topm_regs(p.self_mode ? p.k - 1 : p.k)) {
        case 1: go(k_rescan<1>); break;
        case 2: go(k_rescan<2>); break;
        default: go(k_rescan<4>); break;
    }
    return launch_status("rescan");
}

int knn_plan(int64_t nq, int64_t nr, int d, int k, const rsc_knn_opts *opts, bool self_mode, KnnPlan *plan) {
    if (nq < 0 || nr < 1) {
        set_error("need n_query >= 0 and n_ref >= 1");
        return RSC_ERR_INVALID_ARG;
    }
    if (nq > INT32_MAX - 1 || nr > INT32_MAX - 1) {
        set_error("row counts above 2^31-2 cannot be indexed by int32");
        return RSC_ERR_OVERFLOW;
    }
    if (d < 1 || k < 1 || k > nr) {
        set_error("need d >= 1 and 1 <= k <= n_ref");
        return RSC_ERR_INVALID_ARG;
    }
    if (d > kMaxD) {
        set_error("d > 256 is not supported by this build");
        return RSC_ERR_UNSUPPORTED;
    }
    if (k > kMaxK) {
        set_error("k > 255 is not supported by this build");
        return RSC_ERR_UNSUPPORTED;
    }
    int precision = opts ? opts->precision : RSC_FP32;
    if (precision != RSC_FP32 && (d > kMaxDLowp || k > kMaxKLowp)) {
        set_error("reduced-precision screens support d <= 128 and k <= 63");
        return RSC_ERR_UNSUPPORTED;
    }
    int screen_w = opts ? opts->screen : 0;
    const int metric = opts ? opts->metric : RSC_EUCLIDEAN;
    if (metric != RSC_EUCLIDEAN && metric != RSC_COSINE) {
        set_error("unknown metric");
        return RSC_ERR_INVALID_ARG;
    }
    if (precision != RSC_FP32 && precision != RSC_BF16 && precision != RSC_FP8_E4M3) {
        set_error("unknown precision");
        return RSC_ERR_INVALID_ARG;
    }
    if (precision == RSC_FP32) {
        if (screen_w == 0) screen_w = k <= 16 ? 32 : 64;
        if ((screen_w != 32 && screen_w != 64) || (k < 64 && screen_w <= k) || (k >= 64 && screen_w != 64)) {
            set_error("screen width must be 32 or 64 and larger than k (64 for k >= 64)");
            return RSC_ERR_INVALID_ARG;
        }
    } else {
        if (screen_w == 0) screen_w = 64;
        if (screen_w != 64 && screen_w != 128 && screen_w != 256 && screen_w != 512) {
            set_error("reduced-precision screens keep 64, 128, 256 or 512 candidates per query");
            return RSC_ERR_INVALID_ARG;
        }
    }
    const int resid = opts ? opts->fp8_residual : 0;
    if (resid != 0) {
        if (precision != RSC_FP8_E4M3 || metric != RSC_EUCLIDEAN) {
            set_error("fp8_residual needs the FP8-e4m3 screen and the Euclidean metric");
            return RSC_ERR_INVALID_ARG;
        }
        if (resid < 2 || resid > 4096 || resid > nr) {
            set_error("fp8_residual: the partition count must lie in [2, min(4096, n_ref)]");
            return RSC_ERR_INVALID_ARG;
        }
    }
    const int lowp_ranges = precision == RSC_FP32 ? 1 : screen_w / 64;
    if (precision != RSC_FP32) screen_w = 64;  // per reference range; the ranges multiply it
    plan->nq = nq;
    plan->nr = nr;
    plan->d = d;
    plan->k = k;
    plan->screen = screen_w;
    plan->half = screen_w / 2;
    plan->dh = pick_dh(d);
    plan->self_mode = self_mode;
    plan->nblk = (nr + 31) / 32 + resid;  // residual variant: each partition's last block padded
    plan->precision = precision;
    plan->metric = metric;
    plan->resid = resid;
    plan->pruned = (precision == RSC_FP32 || (precision == RSC_BF16 && lowp_ranges == 1)) && nr >= kPruneRows &&
                   (double)nq * (double)nr >= kPrunePairs;
    if (!self_mode && nq < (precision == RSC_BF16 ? prune_queries_bf16(nr) : kPruneQueries)) plan->pruned = false;
    const int m = self_mode ? k - 1 : k;
    const bool long_answer = k > kLeanAnswer + 1;  // (either mode: one workspace serves both)
    if (long_answer && nr < kPruneRowsLong) plan->pruned = false;
    const bool split = precision == RSC_FP32 || plan->pruned;
    // the split screen's workgroups of 8 waves fill a CU each; the others run four of 4 waves
    plan->splits = split
                       ? pick_splits(nq, plan->nblk, split_queries_per_group(d, plan->half),
                                     plan->pruned ? kCUs : kSplitWant)
                       : pick_splits(nq, plan->nblk, lowp_queries_per_group(precision, d), 1024);
    // A tile of foreign queries spans several clusters where the queries are
    // sparser than the references, and costs up to ten times another.  Few tiles
    // take as many ranges as keep one workgroup per CU (5000 queries of 400k
    // rows: 12 ranges 0.98 ms, 13 1.45); more of them even out in a second and
    // third round (20k queries: 2.42 ms in 4 ranges, 1.99 in 7).
    if (plan->pruned && !self_mode) {
        const int64_t qg = split_queries_per_group(d, plan->half), tiles = std::max<int64_t>(1, (nq + qg - 1) / qg);
        const int64_t P = 4 * tiles <= kCUs ? kCUs / tiles : (576 + tiles / 2) / tiles;
        plan->splits = (int)std::max<int64_t>(1, std::min<int64_t>(32, P));
    }
    // (two ranges even out tiles of different cost while each CU gets about one)
    if (plan->pruned && nq < 512 * split_queries_per_group(d, plan->half)) plan->splits = std::max(plan->splits, 2);
    // One workgroup a CU at a time: few tiles take as many ranges as fill one round
    // (20k rows, 79 tiles, d = 10, k = 15, without clusters: 4 ranges 0.76 ms, 3 0.54;
    // in 78 clusters, d = 60, k = 30, 0.67, 0.51).  Two ranges beyond: three would fill
    // the second round of 129 to 170 tiles (42k rows without clusters 1.54 -> 1.29), but
    // in clusters, where the tiles differ, they cost up to a quarter (33k, d = 38, k = 50,
    // 0.60 -> 0.76).
    if (plan->pruned && self_mode && precision == RSC_FP32) {
        const int64_t qg = split_queries_per_group(d, plan->half), tiles = (nq + qg - 1) / qg;
        if (tiles <= kCUs / 2) plan->splits = (int)std::min<int64_t>(plan->splits, kCUs / tiles);
    }
    if (split) {
        // enough (range, half) lists that the m nearest fill each to about half; rows in
        // no order and more than 64 of them to four tenths, or a few of their lists
        // overflow (4000 rows, k = 255, d = 50: 8 ranges and a second search 0.66 ms, 11
        // ranges 0.39)
        const int fill = long_answer && !plan->pruned ? plan->half * 25 / 32 : plan->half;
        plan->splits = std::min(32, std::max(plan->splits, (m + fill - 1) / fill));
    } else {
        plan->splits = std::max(plan->splits, lowp_ranges);
    }
    return RSC_OK;
}

// Query tiles of the pruned screen.
static int64_t query_tiles(const KnnPlan &p) {
    const int64_t qg = split_queries_per_group(p.d, p.half);
    return (p.nq + qg - 1) / qg;
}

// Whether rows without a certificate collect their candidates (k_split_collect;
// else the FP32 chain screens them again).
static bool knn_collects(const KnnPlan &p) { return (p.self_mode ? p.k - 1 : p.k) <= kLeanAnswer; }

size_t knn_workspace(const KnnPlan &p, void *ws, KnnBuffers *out) {
    Carver cv(ws);
    KnnBuffers b{};
    const bool fp32 = p.precision == RSC_FP32, rounded = !fp32 && p.pruned;
    const int64_t esc_rows = p.precision == RSC_FP32 ? std::min<int64_t>(p.nq, kEscalateCap) : 0;
    b.counters = cv.take<KnnCounters>(1);
    if (fp32) {
        b.nrow = cv.take<float>((size_t)p.nr);
        b.norms = cv.take<float>(norm_folded(p.dh) ? 1 : (size_t)p.nblk * 32);
        // (the pruned screen loads whole segments: the last one may reach past the blocks)
        const size_t split = split_packed_bytes(p.d, p.nblk + (p.pruned ? spatial_seg_blocks(p.nblk) : 0));
        const size_t chain = knn_packed_floats(p.dh, p.nblk) * sizeof(float);
        if (knn_collects(p)) {  // one or the other is read
            b.split = cv.take<char>(std::max(split, chain));
            b.packed = static_cast<float *>(b.split);
        } else {
            b.split = cv.take<char>(split);
            b.packed = reinterpret_cast<float *>(cv.take<char>(chain));
        }
    } else if (rounded) {
        b.nrow = cv.take<float>((size_t)p.nr);
        // one or the other screen's packing
        b.split = cv.take<char>(std::max(rounded_packed_bytes(p.d, p.nblk + spatial_seg_blocks(p.nblk)),
                                         lowp_packed_bytes(p.precision, p.nblk, p.d)));
        b.packed = static_cast<float *>(b.split);
    } else {
        b.packed = reinterpret_cast<float *>(cv.take<char>(lowp_packed_bytes(p.precision, p.nblk, p.d)));
        b.norms = cv.take<float>((size_t)p.nblk * 32);
        b.scal = cv.take<float>(2 * 128 + 1);
        b.amax = cv.take<uint32_t>(256);
    }
    b.cand_idx = cv.take<int32_t>((size_t)p.nq * p.splits * p.screen);
    b.cand_key = cv.take<float>((size_t)p.nq * p.splits * p.screen);
    b.flag1 = cv.take<int32_t>((size_t)std::max<int64_t>(p.nq, 1));
    b.flag2 = cv.take<int32_t>((size_t)std::max<int64_t>(esc_rows, 1));
    b.esc_idx = cv.take<int32_t>((size_t)std::max<int64_t>(esc_rows, 1) * kEscalateSplits * kEscalateWidth);
    b.esc_key = cv.take<float>((size_t)std::max<int64_t>(esc_rows, 1) * kEscalateSplits * kEscalateWidth);
    b.esc_bound = cv.take<double>((size_t)std::max<int64_t>(esc_rows, 1));
    b.esc_found = cv.take<int32_t>((size_t)std::max<int64_t>(esc_rows, 1));
    if (p.metric == RSC_COSINE || rounded) {  // the rows as the screen sees them
        b.rn = cv.take<float>((size_t)p.nr * p.d);
        b.qn = p.self_mode ? b.rn : cv.take<float>((size_t)std::max<int64_t>(p.nq, 1) * p.d);
    }
    if (p.pruned) {
        b.qcount = cv.take<int32_t>(1);
        // (a workspace serves the square and the rectangular form alike: with the queries' part)
        const size_t need = spatial_carve(p.nq, p.nr, p.d, nullptr, nullptr);
        char *base = cv.take<char>(need);
        spatial_carve(p.nq, p.nr, p.d, base, &b.sp);
    } else if (!fp32 && p.resid == 0 && p.nq > 0) {
        // spatial order of the queries (perm) and its sort
        b.perm = cv.take<int32_t>((size_t)p.nq);
        b.qcount = cv.take<int32_t>(1);
        b.order_ws = cv.take<char>(query_order_workspace(p.nq));
    }
    if (p.resid > 0) {
        b.cent = cv.take<float>((size_t)p.resid * p.d);
        b.assign = cv.take<int32_t>((size_t)p.nr);
        b.perm = cv.take<int32_t>((size_t)p.nr);
        b.init = cv.take<int32_t>((size_t)p.resid);
        b.poff = cv.take<int64_t>((size_t)p.resid + 1);
        b.pblk = cv.take<int64_t>((size_t)p.resid + 1);
        b.blk_part = cv.take<int32_t>((size_t)p.nblk * 4);
        b.map = cv.take<int32_t>((size_t)p.nblk * 32);
        b.qcount = cv.take<int32_t>(1);
        b.kws_bytes = kmeans_workspace_bytes(p.nr, p.d, p.resid);
        b.kws = cv.take<char>(b.kws_bytes ? b.kws_bytes : 1);
    }
    if (out) *out = b;
    return cv.used;
}

// Cosine metric: the screen's inputs are the unit-normalised rows.
int normalize_inputs(const KnnPlan &p, const float *Q, const float *R, const KnnBuffers &b, hipStream_t stream) {
    ScopedTimer timer("normalize", stream);
    hipLaunchKernelGGL(k_normalize, dim3((unsigned)((p.nr + norm_rows(p.d) - 1) / norm_rows(p.d))), dim3(kNormThreads), 0,
                       stream, R, p.nr, p.d, b.rn);
    if (!p.self_mode && p.nq > 0)
        hipLaunchKernelGGL(k_normalize, dim3((unsigned)((p.nq + norm_rows(p.d) - 1) / norm_rows(p.d))), dim3(kNormThreads), 0,
                           stream, Q, p.nq, p.d, b.qn);
    return launch_status("normalize");
}

__global__ __launch_bounds__(256) void k_round_bf16(const float *__restrict__ X, int64_t n, float *__restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = (float)(__bf16)X[i];
}

// The BF16 form on the pruned screen: its inputs are the rows rounded to BF16.
int round_inputs(const KnnPlan &p, const float *Q, const float *R, const KnnBuffers &b, hipStream_t stream) {
    ScopedTimer timer("prep_lowp", stream);
    auto run = [&](const float *x, int64_t n, float *out) {
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192));
        hipLaunchKernelGGL(k_round_bf16, dim3(grid), dim3(256), 0, stream, x, n, out);
    };
    run(R, p.nr * p.d, b.rn);
    if (!p.self_mode && p.nq > 0) run(Q, p.nq * p.d, b.qn);
    return launch_status("round to BF16");
}

// The row count on the device; spatial order of a pruned problem's references (and of foreign queries).
int order_rows(const KnnPlan &p, const float *Qs, const float *Rs, const KnnBuffers &b, hipStream_t stream) {
    int st;
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(64), 0, stream, b.qcount, (int32_t)p.nq);
    if ((st = launch_status("set query count")) != RSC_OK) return st;
    if ((st = spatial_refs(Rs, b.nrow, p.nr, p.d, p.precision == RSC_BF16, b.sp, b.counters, stream)) != RSC_OK) return st;
    if (p.self_mode) return RSC_OK;
    return spatial_queries(Qs, p.nq, p.nr, p.d, split_queries_per_group(p.d, p.half), b.sp, b.counters, stream);
}

PrunedArgs pruned_args(const KnnPlan &p, const ScreenArgs &s, const KnnBuffers &b) {
    PrunedArgs pa{};
    pa.s = s;
    pa.segments = b.sp.seg_packed;
    pa.nseg = b.sp.nseg;
    while ((1 << pa.seg_shift) < b.sp.seg_blocks) ++pa.seg_shift;
    pa.own = p.self_mode ? nullptr : b.sp.own;
    pa.eps = split_eps_coefficient(p.d);
    pa.counters = b.counters;
    pa.rounded = p.precision == RSC_BF16;
    // Whether bounds help is sampled where that pays.
    // BF16 rows: with fewer than 256 blocks to a range a tile has screened most of
    // them by the time the samples know (16.5k rows without clusters, 4 ranges of 129:
    // 1.12 ms pruned, 1.23 with the verdict; 25k, 3 of 260: 1.71, 1.38); at 9 steps the
    // plain screen has one workgroup per CU and gains nothing (d = 128, 200k rows: 44.6
    // pruned, 46.4 plain; d = 126: 44.6, 25.1).
    // Exact, lists of 32: the pruned loop spills 59 registers at 5 chunks to a row and
    // 583 at 17, and the unpruned one is faster at the same work (100k rows without
    // clusters, k = 30, pruned and plain: d = 35 14.1, 8.2 ms; d = 50 14.5, 8.8; d = 100
    // 26.6, 18.1; d = 128 42.3, 16.6), but not without spills (d = 20, 3 chunks, 7.41,
    // 7.21; d = 200, 29 chunks, 32.1, 29.7) or with short ranges in one round of
    // workgroups.  With lists of 16 it gains at most a tenth, and the verdict costs more.
    // Foreign queries in one round of workgroups gain nothing (BF16: 16,384 of 500k rows
    // 5.09 and 5.20; 24,000 10.1 and 7.4; exact, k = 30: 24,000 16.7 and 10.6).
    const int64_t tiles = query_tiles(p);
    const int chunks = (int)(split_packed_bytes(p.d, 1) / 1024);
    const double blocks = (double)p.nblk / p.splits;
    const bool pays = pa.rounded ? blocks >= 256 && lowp_steps(p.precision, p.d) <= 8
                                 : p.half == 32 && chunks >= 5 && chunks <= 25 &&
                                       (blocks * chunks >= 1792 || tiles * p.splits >= 4 * scr::kCUs);
    if (pays && (p.self_mode || 4 * tiles > scr::kCUs)) {
        pa.samples = (int)std::min<int64_t>(pa.rounded ? 64 : 16, tiles);
        // (in their place among those that run at once: 36k rows in 5 clusters, d = 60, k = 30,
        // 1.70 ms with the samples first, 1.45 so)
        if (!pa.rounded && tiles <= 2 * scr::kCUs) pa.sample_step = (int)(std::min<int64_t>(tiles, scr::kCUs) / pa.samples);
        // Both take the same time, BF16 at about half of the segments (200k rows, d = 50:
        // 0.50 of them 11.8 ms pruned, 11.9 plain; 0.30 6.8 and 9.1); exact at 0.6 to 0.8
        // (100k, d = 80, 0.65 of them 8.1, 8.2; 40k, d = 50, 0.83 of them 2.10, 1.77), with
        // 15 chunks and more a quarter (d = 128, 100k, 0.33 of them 19.5, 13.2; 300k, 0.20
        // 48.6, 70.9).  Foreign queries' tiles span several clusters, but their lists settle
        // early: 24,000 of 500k BF16 rows in 100 clusters 4.8 pruned, 6.0 plain.
        const bool late = p.self_mode && !pa.rounded && chunks < 15;
        const double share = late ? 0.75 : !p.self_mode ? 0.95 : pa.rounded ? 0.55 : 0.25;
        pa.plain_over = (int)(share * b.sp.nseg / p.splits);
        pa.wait_over = late ? pa.plain_over / 2 : pa.plain_over;
    }
    return pa;
}

// The BF16 form from kPruneRows references on: the pruned screen over rounded
// rows, or, where it finds that bounds do not help or the norms spread too far,
// the plain BF16 screen over the same order (its launches end at once unless that
// is so).  Rerank without a certificate.  Rows without clusters, in ms, in a plain
// screen of Morton order / pruned / by verdict: 300k rows, d = 50: 30.0 / 33.9 /
// 26.4; 200k, d = 100: 24.7 / 38.3 / 23.3; 40k, d = 50: 2.53 / 2.63 / 1.92; 24,000
// queries of 500k rows: 7.0 / 10.2 / 7.4.
int knn_run_rounded(const KnnPlan &p, const float *Q, const float *R, int32_t *out_idx, float *out_dist,
                    const KnnBuffers &b, hipStream_t stream) {
    int st;
    const bool cosine = p.metric == RSC_COSINE;
    if (cosine && (st = normalize_inputs(p, Q, R, b, stream)) != RSC_OK) return st;
    if ((st = round_inputs(p, cosine ? b.qn : Q, cosine ? b.rn : R, b, stream)) != RSC_OK) return st;
    if ((st = knn_prep(p, b.rn, p.self_mode ? nullptr : b.qn, b, stream)) != RSC_OK) return st;
    if ((st = order_rows(p, b.qn, b.rn, b, stream)) != RSC_OK) return st;
    {
        ScopedTimer timer("pack_split", stream);
        if ((st = split_pack(b.rn, b.nrow, p.nr, p.d, p.nblk, b.split, nullptr, nullptr, nullptr, b.sp.rperm, p.nr,
                             b.counters, stream, true)) != RSC_OK)
            return st;
    }
    ScreenArgs sa{};
    sa.Q = b.qn;
    sa.nq = p.nq;
    sa.qlist = p.self_mode ? b.sp.rperm : b.sp.qperm;
    sa.qcount = b.qcount;
    sa.qcap = (int)p.nq;
    sa.Ap = b.split;
    sa.nblk = p.nblk;
    sa.d = p.d;
    sa.P = p.splits;
    sa.cand_idx = b.cand_idx;
    sa.cand_key = b.cand_key;
    sa.kc = b.counters;
    {
        ScopedTimer timer("screen_bf16", stream);
        ScreenArgs ss = sa;
        ss.ref_map = b.sp.rperm;
        PrunedArgs pa = pruned_args(p, ss, b);
        if ((st = split_screen_pruned(pa, p.half, "screen_bf16_pruned", stream)) != RSC_OK) return st;
        // (as in knn_run_lowp, references in the queries' order for a single range of one matrix)
        const int32_t *rmap = p.self_mode && p.splits == 1 ? b.sp.rperm : nullptr;
        if ((st = lowp_prepare(p, b.qn, b.rn, b.packed, nullptr, nullptr, nullptr, rmap, stream, b.counters)) != RSC_OK)
            return st;
        sa.only_plain = 1;
        sa.rotate = rmap ? 1 : 0;
        const int plain_qg = lowp_queries_per_group(p.precision, p.d);
        if ((st = lowp_screen(p, sa, (unsigned)((p.nq + plain_qg - 1) / plain_qg), stream)) != RSC_OK) return st;
        if (rmap && (st = lowp_unmap_rows(p, b, rmap, stream, b.counters)) != RSC_OK) return st;
    }
    RerankArgs ra{};
    ra.Q = Q;
    ra.nq = p.nq;
    ra.qlist = sa.qlist;
    ra.qcount = sa.qcount;
    ra.qcap = sa.qcap;
    ra.R = R;
    ra.d = p.d;
    ra.k = p.k;
    ra.S = p.half;
    ra.KP = p.half;
    ra.P = 2 * p.splits;
    ra.self_mode = p.self_mode ? 1 : 0;
    ra.certify = 0;
    ra.metric = p.metric;
    ra.cand_idx = b.cand_idx;
    ra.cand_key = b.cand_key;
    ra.counters = b.counters;
    ra.flag_out = b.flag1;
    ra.flag_count = &b.counters->flagged;
    ra.out_idx = out_idx;
    ra.out_dist = out_dist;
    ra.split = 2;
    ra.eps_coef = ra.cosine_eps = ra.split_eps = ra.split_cosine_eps = 1.0;
    return knn_launch_rerank(ra, p.nq, "rerank", stream);
}

// Reduced-precision form: screen, then rerank without a certificate.
int knn_run_lowp(const KnnPlan &p, const float *Q, const float *R, int32_t *out_idx, float *out_dist,
                 const KnnBuffers &b, hipStream_t stream) {
    int st;
    hipLaunchKernelGGL(k_init_counters, dim3(1), dim3(64), 0, stream, b.counters);
    if ((st = launch_status("init_counters")) != RSC_OK) return st;
    const bool cosine = p.metric == RSC_COSINE;
    if (cosine && (st = normalize_inputs(p, Q, R, b, stream)) != RSC_OK) return st;
    const float *Qs = cosine ? b.qn : Q, *Rs = cosine ? b.rn : R;  // what the screen sees
    // The queries are screened in an order that keeps neighbours together,
    // so that the 32 queries of a wave tend to take keys from the same
    // blocks and share the selection's queue flushes: the residual variant
    // on one matrix uses its partition order, the other forms a Morton order
    // of the first coordinates (query_order.hip).  On one matrix screened as
    // a single reference range the latter also packs the references in that
    // order, and every query group starts its scan at its own rows: the
    // nearest references come first and tighten the thresholds before the
    // rest streams past.  (With several ranges, references packed in that
    // order would put a query's near rows into one range, whose 64
    // candidates are then all it keeps of them: fewer true neighbours
    // survive the noisier FP8 keys.)
    bool ordered = false, rotate = false;
    if (p.resid == 0 && b.order_ws && p.nq > 0) {
        if ((st = query_order_run(Qs, p.nq, p.d, b.order_ws, b.perm, stream)) != RSC_OK) return st;
        ordered = true;
        rotate = p.self_mode && p.splits == 1;
    }
    if (p.resid > 0)
        st = lowp_prepare_resid(p, R, b, stream);
    else
        st = lowp_prepare(p, Qs, Rs, b.packed, b.norms, b.scal, b.amax, rotate ? b.perm : nullptr, stream);
    if (st != RSC_OK) return st;
    if (p.nq == 0) return RSC_OK;
    if (p.resid > 0) ordered = p.self_mode;
    if (ordered) {
        hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(64), 0, stream, b.qcount, (int32_t)p.nq);
        if ((st = launch_status("set query count")) != RSC_OK) return st;
    }
    ScreenArgs sa{};
    sa.Q = Qs;
    sa.nq = p.nq;
    sa.qlist = ordered ? b.perm : nullptr;
    sa.qcount = ordered ? b.qcount : nullptr;
    sa.qcap = (int)p.nq;
    sa.Ap = b.packed;
    sa.Np = b.norms;
    sa.qscale = b.scal;
    sa.blk_part = b.blk_part;
    sa.cent = b.cent;
    sa.nblk = p.nblk;
    sa.d = p.d;
    sa.P = p.splits;
    sa.rotate = rotate ? 1 : 0;
    sa.cand_idx = b.cand_idx;
    sa.cand_key = b.cand_key;
    const int qg = lowp_queries_per_group(p.precision, p.d);
    if ((st = lowp_screen(p, sa, (unsigned)((p.nq + qg - 1) / qg), stream)) != RSC_OK) return st;
    if (p.resid > 0 && (st = lowp_unmap(p, b, stream)) != RSC_OK) return st;
    if (rotate && (st = lowp_unmap_rows(p, b, b.perm, stream)) != RSC_OK) return st;
    RerankArgs ra{};
    ra.Q = Q;
    ra.nq = p.nq;
    ra.qlist = sa.qlist;
    ra.qcount = sa.qcount;
    ra.qcap = sa.qcap;
    ra.R = R;
    ra.d = p.d;
    ra.k = p.k;
    ra.S = p.half;
    ra.KP = p.half;
    ra.P = 2 * p.splits;
    ra.self_mode = p.self_mode ? 1 : 0;
    ra.certify = 0;
    ra.metric = p.metric;
    ra.cosine_eps = 1.0;
    ra.cand_idx = b.cand_idx;
    ra.cand_key = b.cand_key;
    ra.eps_coef = 1.0;
    ra.counters = b.counters;
    ra.flag_out = b.flag1;
    ra.flag_count = &b.counters->flagged;
    ra.out_idx = out_idx;
    ra.out_dist = out_dist;
    return knn_launch_rerank(ra, p.nq, "rerank", stream);
}

int knn_run(const KnnPlan &p, const float *Q, const float *R, int32_t *out_idx, float *out_dist, void *ws,
            hipStream_t stream, const int32_t *qlist, const int32_t *qcount) {
    KnnBuffers b;
    knn_workspace(p, ws, &b);
    if (p.precision != RSC_FP32) {
        if (qlist) {
            set_error("internal: row lists need the FP32 path");
            return RSC_ERR_UNSUPPORTED;
        }
        return p.pruned ? knn_run_rounded(p, Q, R, out_idx, out_dist, b, stream)
                        : knn_run_lowp(p, Q, R, out_idx, out_dist, b, stream);
    }
    int st;
    const bool cosine = p.metric == RSC_COSINE;
    if (cosine && (st = normalize_inputs(p, Q, R, b, stream)) != RSC_OK) return st;
    const float *Qs = cosine ? b.qn : Q;  // what the screen sees
    const float *Rs = cosine ? b.rn : R;
    if ((st = knn_prep(p, Rs, p.self_mode ? nullptr : Qs, b, stream)) != RSC_OK) return st;
    // Large problems are screened in a spatial order with its segments' bounds.
    // (Under stream capture every pair is screened instead.)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool captured = p.pruned && hipStreamIsCapturing(stream, &capture) == hipSuccess &&
                          capture != hipStreamCaptureStatusNone;
    const bool pruned = p.pruned && !captured && !qlist && p.nq > 0;
    const int32_t *ref_map = nullptr;
    if (pruned) {
        if ((st = order_rows(p, Qs, Rs, b, stream)) != RSC_OK) return st;
        ref_map = b.sp.rperm;
        qlist = p.self_mode ? b.sp.rperm : b.sp.qperm;
        qcount = b.qcount;
    }
    {
        ScopedTimer timer("pack_split", stream);
        if ((st = split_pack(Rs, b.nrow, p.nr, p.d, p.nblk, b.split, nullptr, nullptr, nullptr, ref_map, p.nr,
                             b.counters, stream)) != RSC_OK)
            return st;
    }
    if (p.nq == 0) return RSC_OK;

    const double eps_coef = knn_eps_coefficient(p.d);

    // Slots are rows 0..nq-1, or the first min(*qcount, nq) rows of qlist.
    ScreenArgs sa{};
    sa.Q = Qs;
    sa.nq = p.nq;
    sa.qlist = qlist;
    sa.qcount = qcount;
    sa.qcap = (int)p.nq;
    sa.Ap = b.packed;
    sa.Np = b.norms;
    sa.nblk = p.nblk;
    sa.d = p.d;
    sa.P = p.splits;
    sa.cand_idx = b.cand_idx;
    sa.cand_key = b.cand_key;
    sa.kc = b.counters;
    ScreenArgs ss = sa;  // the split screen; the FP32 chain takes the inputs it cannot (both see the mark)
    ss.Ap = b.split;
    ss.ref_map = ref_map;
    if (pruned) {
        PrunedArgs pa = pruned_args(p, ss, b);
        ScopedTimer timer("screen_fp32", stream);
        if ((st = split_screen_pruned(pa, p.half, "screen_pruned", stream)) != RSC_OK) return st;
        if (pa.samples > 0) {
            ss.only_plain = ss.rotate = 1;
            ss.own = pa.own;
            ss.own_q = split_queries_per_group(p.d, p.half);
            ss.own_shift = pa.seg_shift;
            st = split_screen(ss, p.half, "screen_plain", stream);
        }
    } else {
        st = split_screen(ss, p.half, "screen_fp32", stream);
    }
    if (st != RSC_OK) return st;
    // (short answers read this packing on inputs marked wide alone, in the memory of the other)
    const bool collect = knn_collects(p);
    if ((st = knn_pack_fp32(p.dh, Rs, b.nrow, p.nr, p.d, p.nblk, b.packed, b.norms, nullptr, nullptr, nullptr, nullptr,
                            collect ? b.counters : nullptr, stream)) != RSC_OK)
        return st;
    sa.only_wide = 1;
    const unsigned gq = (unsigned)((p.nq + kQueriesPerGroup - 1) / kQueriesPerGroup);
    if ((st = screen(p.dh, sa, gq, p.half, false, "screen_wide", stream)) != RSC_OK) return st;

    // Each (range, half) list is one candidate group of width `half`.
    RerankArgs ra{};
    ra.Q = Q;
    ra.nq = p.nq;
    ra.qlist = qlist;
    ra.qcount = qcount;
    ra.qcap = (int)p.nq;
    ra.R = R;
    ra.d = p.d;
    ra.k = p.k;
    ra.S = p.half;
    ra.KP = p.half;
    ra.P = 2 * p.splits;
    ra.self_mode = p.self_mode ? 1 : 0;
    ra.certify = 1;
    ra.metric = p.metric;
    ra.cosine_eps = cosine_eps_of(eps_coef);
    ra.cand_idx = b.cand_idx;
    ra.cand_key = b.cand_key;
    ra.eps_coef = eps_coef;
    ra.counters = b.counters;
    ra.flag_out = b.flag1;
    ra.flag_count = &b.counters->flagged;
    ra.out_idx = out_idx;
    ra.out_dist = out_dist;
    knn_split_bounds(ra);
    const int esc_cap = (int)std::min<int64_t>(p.nq, kEscalateCap);
    if (collect) {
        ra.flag_bound = b.esc_bound;
        ra.flag_found = b.esc_found;
        ra.flag_cap = esc_cap;
    }
    if ((st = knn_launch_rerank(ra, p.nq, "rerank", stream)) != RSC_OK) return st;

    // Escalation of the rows that failed.  The m-th distance found bounds the
    // true one: a row of a short answer collects every reference whose key
    // can lie below it and re-ranks those (the answer is then complete).
    // Rows of longer answers are screened again 64 wide over many ranges, in
    // the FP32 chain.
    RerankArgs re = ra;
    re.qlist = b.flag1;
    re.qcount = &b.counters->flagged;
    re.qcap = esc_cap;
    re.cand_idx = b.esc_idx;
    re.cand_key = b.esc_key;
    re.flag_out = b.flag2;
    re.flag_count = &b.counters->flagged2;
    re.flag_bound = nullptr;
    if (collect) {
        CollectArgs ca{};
        ca.Q = Qs;
        ca.d = p.d;
        ca.metric = p.metric;
        ca.rows = b.flag1;
        ca.nrows = &b.counters->flagged;
        ca.cap = esc_cap;
        ca.bound = b.esc_bound;
        ca.found = b.esc_found;
        ca.width = kEscalateSplits * kEscalateWidth;
        ca.out_idx = b.esc_idx;
        ca.out_key = b.esc_key;
        ca.packed = b.split;
        ca.ref_map = ref_map;
        ca.nr = p.nr;
        ca.nblk = p.nblk;
        ca.eps = ra.split_eps;
        ca.eps_abs = ra.split_abs;
        ca.cosine_eps = ra.split_cosine_eps;
        ca.packed32 = b.packed;
        ca.norms32 = b.norms;
        ca.dh = p.dh;
        ca.fp32_eps = ra.eps_coef;
        ca.fp32_cosine_eps = ra.cosine_eps;
        ca.kc = b.counters;
        {
            ScopedTimer timer("screen_escalate", stream);
            if ((st = split_collect(ca, stream)) != RSC_OK) return st;
        }
        re.certify = 0;
        re.P = 1;
        re.S = re.KP = ca.width;
        re.counts = b.esc_found;
    } else {
        ScreenArgs se = sa;
        se.qlist = b.flag1;
        se.qcount = &b.counters->flagged;
        se.qcap = esc_cap;
        se.only_wide = 0;
        se.P = (int)std::min<int64_t>(kEscalateSplits, std::max<int64_t>(1, p.nblk));
        se.cand_idx = b.esc_idx;
        se.cand_key = b.esc_key;
        const unsigned ge = (unsigned)((esc_cap + kQueriesPerGroup - 1) / kQueriesPerGroup);
        if ((st = screen(p.dh, se, ge, kEscalateWidth / 2, true, "screen_escalate", stream)) != RSC_OK) return st;
        re.split = 0;
        re.S = re.KP = kEscalateWidth / 2;
        re.P = 2 * se.P;
    }
    if ((st = knn_launch_rerank(re, esc_cap, "rerank_escalate", stream)) != RSC_OK) return st;
    return knn_launch_rescan(p, Q, R, b, esc_cap, out_idx, out_dist, nullptr, 0, stream);
}

}  // namespace rsc
