// Device pieces shared by the FP32 and the reduced-precision screens.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "rsc_internal.hpp"

namespace rsc {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace scr {

constexpr int kWave = 64;
constexpr int kScreenWaves = 4;  // waves per screen workgroup
constexpr int kDenseLanes = 32;  // lanes with a hit from which a block is merged whole (PackTopK)
constexpr int kQueueCap = 16;    // default queue entries per lane and query block (a block adds at most 16)

// (d2, j) lexicographic order: smaller distance first, lower index on ties.
__device__ __forceinline__ bool lex_before(double da, int ja, double db, int jb) {
    return da < db || (da == db && ja < jb);
}

// Squared distance of two float32 rows in float64, dimensions in order,
// every product and sum rounded separately (no contraction).
__device__ __forceinline__ double exact_d2(const float *__restrict__ x, const float *__restrict__ y, int d) {
    double s = 0.0;
    for (int t = 0; t < d; ++t) {
        double diff = __dsub_rn((double)x[t], (double)y[t]);
        s = __dadd_rn(s, __dmul_rn(diff, diff));
    }
    return s;
}

__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

__device__ __forceinline__ int wave_max_int(int v) {
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, kWave));
    return v;
}

// Arguments of a screen launch.  Query slot i of the launch is row i, or
// row qlist[i] for i < min(*qcount, qcap) when a list is given.
// Output: cand[(slot * 2P + 2p + h) * L + i] = i-th smallest key of
// contraction half h of reference range p (index -1 / key +inf where fewer
// than L were seen).
struct ScreenArgs {
    const float *Q;
    int64_t nq;
    const int32_t *qlist;   // optional gather list
    const int32_t *qcount;  // its device-side length
    int qcap;
    const void *Ap;         // packed references (layout depends on the precision)
    const float *Np;        // norms in accumulator order, where the layout needs them
    const float *qscale;    // per-dimension query scales (FP8 screen)
    const int32_t *blk_part;  // FP8 residual variant: partition of each packed block (4 copies per block)
    const float *cent;        // FP8 residual variant: partition centroids
    int64_t nblk;
    int d;
    int P;                  // reference ranges (gridDim.y)
    int rotate;             // references packed in the queries' order (or one that `own` relates to it): each
                            // query group starts its scan at its own block
    const int32_t *own;     // split screen: that block for every own_q queries, in units of 1 << own_shift (null:
    int own_q, own_shift;   // the queries are the references)
    const int32_t *ref_map; // split screen: packed slot -> row (null: row order)
    const KnnCounters *kc;  // exact path and large BF16 problems: the largest norms (the split screen's scale) and the mark
    int only_wide;          // FP32 chain: run only on inputs marked wide
    int only_plain;         // split and BF16 screen: run only where the pruned screen does not answer
    int32_t *cand_idx;
    float *cand_key;
};

// Asynchronous 16-byte load per lane straight into LDS (lane l lands at
// lds_base + 16 l).
__device__ __forceinline__ void load_lds16(const void *gsrc, void *lds_base) {
    __builtin_amdgcn_global_load_lds(gsrc, (void __attribute__((address_space(3))) *)lds_base, 16, 0, 0);
}

__device__ __forceinline__ int64_t screen_slots(const ScreenArgs &a) {
    if (!a.qlist) return a.nq;
    const int64_t cnt = *a.qcount;
    const int64_t m = cnt < a.qcap ? cnt : a.qcap;
    return m < a.nq ? m : a.nq;
}

// The L smallest keys (and their reference indices) one lane has seen, kept
// sorted in registers, plus this lane's queue of keys that beat the
// threshold of the last merge.  Keys enter the queue with one LDS write; all
// lanes of the wave merge their queues together when any queue could
// overflow, so the per-key cost stays a compare in the common case.
template <int L, int QCAP = kQueueCap>
struct LaneTopK {
    float lk[L];
    int li[L];
    float thr;  // lk[L-1] as of the last merge
    int count;  // queued entries

    __device__ __forceinline__ void init() {
#pragma unroll
        for (int i = 0; i < L; ++i) {
            lk[i] = INFINITY;
            li[i] = -1;
        }
        thr = INFINITY;
        count = 0;
    }

    // Unrolled compare-and-shift insertion that drops the largest entry.
    __device__ __forceinline__ void insert(float key, int idx) {
#pragma unroll
        for (int i = L - 1; i > 0; --i) {
            const bool shift = key < lk[i - 1];
            const bool here = key < lk[i];
            lk[i] = shift ? lk[i - 1] : (here ? key : lk[i]);
            li[i] = shift ? li[i - 1] : (here ? idx : li[i]);
        }
        if (key < lk[0]) {
            lk[0] = key;
            li[0] = idx;
        }
    }

    // queue entry e of this lane lives at q[e * stride]
    __device__ __forceinline__ void flush(const float2 *q, int stride) {
        const int maxc = wave_max_int(count);
        for (int e = 0; e < maxc; ++e) {
            if (e < count) {
                const float2 v = q[e * stride];
                if (v.x < lk[L - 1]) insert(v.x, __float_as_int(v.y));
            }
        }
        count = 0;
        thr = lk[L - 1];
    }

    // Offer the 16 keys of one 32x32 output block (register v holds
    // reference ref0 + 8 (v/4) + (v%4)).
    __device__ __forceinline__ void offer(const f32x16 &acc, int ref0, float2 *q, int stride) {
        float mn = acc[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mn = fminf(mn, acc[v]);
        if (__ballot(mn < thr) == 0ull) return;
        int hits = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) hits += acc[v] < thr ? 1 : 0;
        if (__ballot(count + hits > QCAP) != 0ull) {
            flush(q, stride);
            if constexpr (QCAP < 16) {
                hits = 0;
#pragma unroll
                for (int v = 0; v < 16; ++v) hits += acc[v] < thr ? 1 : 0;
                if (__ballot(hits > QCAP) != 0ull) {
                    // more keys than a queue holds (only while the lists fill up): insert directly
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (acc[v] < lk[L - 1]) insert(acc[v], ref0 + 8 * (v >> 2) + (v & 3));
                    thr = lk[L - 1];
                    return;
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (acc[v] < thr) {
                q[count * stride] = make_float2(acc[v], __int_as_float(ref0 + 8 * (v >> 2) + (v & 3)));
                ++count;
            }
        }
    }

    __device__ __forceinline__ void store(const ScreenArgs &a, int64_t slot, int p, int h) const {
        const int64_t base = ((slot * a.P + p) * 2 + h) * L;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            a.cand_key[base + i] = lk[i];
            a.cand_idx[base + i] = li[i];
        }
    }
};

// The L smallest (key, index) one lane has seen, as LaneTopK, each held as one
// float64 whose high word is the key's bits and whose low word the index: such
// doubles are ordered as the keys (an infinite key is a finite double), so an
// insertion is one float64 min and max per entry and a compare-exchange two
// instructions, where separate words cost a compare and four selects.  A block
// with few hits queues them under wave-uniform branches; while the lists fill
// (many lanes with hits) the block's 16 keys are sorted and merged at once.
template <int L, int QCAP>
struct PackTopK {
    double v[L];
    float thr;  // key of v[L-1] as of the last merge
    int count;  // queued entries

    static __device__ __forceinline__ double pack(float key, int idx) {
        return __hiloint2double(__float_as_int(key), idx);
    }
    static __device__ __forceinline__ float key_of(double x) { return __int_as_float(__double2hiint(x)); }
    static __device__ __forceinline__ void order(double &a, double &b) {
        const double lo = fmin(a, b);
        b = fmax(a, b);
        a = lo;
    }

    __device__ __forceinline__ void init() {
#pragma unroll
        for (int i = 0; i < L; ++i) v[i] = pack(INFINITY, -1);
        thr = INFINITY;
        count = 0;
    }

    __device__ __forceinline__ void insert(double x) {
#pragma unroll
        for (int i = L - 1; i > 0; --i) v[i] = fmax(v[i - 1], fmin(v[i], x));
        v[0] = fmin(v[0], x);
    }

    // queue entry e of this lane lives at q[e * stride]
    __device__ __forceinline__ void flush(const double *q, int stride) {
        const int maxc = wave_max_int(count);
        for (int e = 0; e < maxc; ++e) insert(e < count ? q[e * stride] : pack(INFINITY, -1));
        count = 0;
        thr = key_of(v[L - 1]);
    }

    // Sort the block's 16 keys and merge them into the list.
    __device__ __forceinline__ void merge16(const f32x16 &acc, int ref0) {
        double w[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) w[i] = pack(acc[i], ref0 + 8 * (i >> 2) + (i & 3));
#pragma unroll
        for (int size = 2; size <= 16; size <<= 1) {
#pragma unroll
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int j = i ^ stride;
                    if (j > i) {
                        if ((i & size) == 0) order(w[i], w[j]); else order(w[j], w[i]);
                    }
                }
            }
        }
        // the L smallest of both: a bitonic sequence, then cleaned
#pragma unroll
        for (int i = 0; i < 16; ++i) v[L - 1 - i] = fmin(v[L - 1 - i], w[i]);
#pragma unroll
        for (int stride = L >> 1; stride > 0; stride >>= 1) {
#pragma unroll
            for (int i = 0; i < L; ++i) {
                const int j = i ^ stride;
                if (j > i) order(v[i], v[j]);
            }
        }
        thr = key_of(v[L - 1]);
    }

    // Offer the 16 keys of one 32x32 output block (register i holds reference
    // ref0 + 8 (i/4) + (i%4)).
    __device__ __forceinline__ void offer(const f32x16 &acc, int ref0, double *q, int stride) {
        float g[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            g[j] = fminf(fminf(acc[4 * j], acc[4 * j + 1]), fminf(acc[4 * j + 2], acc[4 * j + 3]));
        const unsigned long long hit = __ballot(fminf(fminf(g[0], g[1]), fminf(g[2], g[3])) < thr);
        if (__builtin_expect(hit == 0ull, 1)) return;
        if (__popcll(hit) >= kDenseLanes) {
            merge16(acc, ref0);
            return;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (__ballot(g[j] < thr) == 0ull) continue;
            if (__ballot(count > QCAP - 4) != 0ull) flush(q, stride);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float key = acc[4 * j + u];
                if (__ballot(key < thr) != 0ull) {
                    if (key < thr) {
                        q[count * stride] = pack(key, ref0 + 8 * j + u);
                        ++count;
                    }
                }
            }
        }
    }

    // map: list entries are packed slots of these rows (null: they are rows)
    __device__ __forceinline__ void store(const ScreenArgs &a, int64_t slot, int p, int h, const int32_t *map) const {
        const int64_t base = ((slot * a.P + p) * 2 + h) * L;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            // an infinite key is an empty entry or a padded row merged with its block
            const float key = key_of(v[i]);
            const int idx = key < INFINITY ? __double2loint(v[i]) : -1;
            a.cand_key[base + i] = key;
            a.cand_idx[base + i] = map && idx >= 0 ? map[idx] : idx;
        }
    }
};

}  // namespace scr
}  // namespace rsc
