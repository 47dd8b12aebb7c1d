// The grid-mapped launch of the split screen, instantiated per list length in
// a translation unit of its own (knn_split.hip, knn_split_wide.hip).
#pragma once

#include "screen_split.hpp"

namespace rsc {

struct PrunedArgs {
    scr::ScreenArgs s;       // Ap: references packed in the spatial order (ref_map)
    const void *segments;    // packed segment bounds
    int nseg, seg_shift;     // segments, log2 of the blocks per segment
    const int32_t *own;
    double eps;              // error coefficient of a split key
    bool rounded;            // BF16 rows: one FP16 part each (lists of 32)
    int samples;             // tiles that tell whether a plain screen is to answer (none: it is not asked),
    int sample_step;         // every so many tiles from the first on (0: the samples come first, from all tiles),
    int plain_over;          // and the segments of a range, on their average, above which it is
    int wait_over;           // a tile with more of them waits for the verdict
    KnnCounters *counters;   // statistics; the mark for the plain screen
};

namespace scr {

constexpr int64_t kCUs = 256;  // MI355X
// Blocks on either side of a tile's own that are screened before the bounds
// (at least one segment).
constexpr int kNearBlocks = 8;

// Query slot i of the launch is row i, or row qlist[i] for i < min(*qcount,
// qcap) when a list is given; lists are filed as by k_screen_fp32, with keys
// times the squared scale.
template <int Q, int TC, int L>
__global__ __launch_bounds__((SplitShape<Q, TC, L>::NW * kWave), (SplitShape<Q, TC, L>::W)) void k_screen_split(
    ScreenArgs a) {
    using S = SplitShape<Q, TC, L>;
    // Two ring buffers as two LDS objects: the compiler can then tell that
    // the asynchronous loads into one never alias the reads of the other.
    __shared__ __attribute__((aligned(16))) char ring0[S::RING];
    __shared__ __attribute__((aligned(16))) char ring1[S::RING];
    __shared__ double qbuf[S::QCAP * S::NW * kWave];
    if (a.kc->wide || (a.only_plain && a.kc->verdict != kPlain)) return;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, c = tid & 31;
    const int p = blockIdx.y;
    // range p: a run of blocks; rotated: every P-th block, as near rows follow each other
    const int nblk = (int)a.nblk, per = (nblk + a.P - 1) / a.P;
    const int b0 = a.rotate ? p : p * per, stride = a.rotate ? a.P : 1;
    const int span = a.rotate ? (nblk - p + a.P - 1) / a.P : max(0, min(per, nblk - b0));
    const int64_t nslots = screen_slots(a);
    const int qg = blockDim.x / 2;  // queries of the workgroup
    for (int64_t qblk = blockIdx.x; qblk * qg < nslots; qblk += gridDim.x) {
        const int64_t slot = qblk * qg + wave * 32 + c;
        int64_t row = -1;
        if (slot < nslots) row = a.qlist ? (int64_t)a.qlist[slot] : slot;
        int rot = 0;
        if (a.rotate) {
            const int64_t own = a.own ? (int64_t)a.own[qblk * qg / a.own_q] << a.own_shift : qblk * qg / 32;
            rot = max(0, min((int)(own / a.P), span - 1));
        }
        screen_split_tile<Q, TC, L>(a, slot < nslots ? slot : -1, row, b0, span, stride, rot, p, 0, ring0, ring1, qbuf);
    }
}

template <int Q, int TC, int L>
int split_launch_geom(const ScreenArgs &a, const char *name, hipStream_t s) {
    using S = SplitShape<Q, TC, L>;
    ScopedTimer timer(name, s);
    // half-size workgroups while they all find a CU of their own: a wave alone
    // on its SIMD fills its lists faster
    const int nw = S::NW == 8 && (a.nq + 127) / 128 * a.P <= kCUs ? 4 : S::NW;
    const unsigned gx = (unsigned)((a.nq + nw * 32 - 1) / (nw * 32));
    hipLaunchKernelGGL((k_screen_split<Q, TC, L>), dim3(gx, (unsigned)a.P), dim3(nw * kWave), 0, s, a);
    return launch_status(name);
}

// The pruned screen.  A tile first screens the segments around its own rows,
// which gives every query a threshold T (no row beyond the distance T of its
// current L-th key can enter its list); a contraction with the segments'
// bounds then tells which segments any query of the tile has within T, and
// only those are screened.  A skipped row's true key is above the query's
// threshold of that moment, hence above its final one: exactly what the
// rerank's certificate assumes of every row outside the lists.
// A tile whose queries' T differ by more than 2 holds some whose neighbours
// are elsewhere: when it would visit many blocks (24 per block of bounds: two
// more passes over those cost less), it screens every query's nearest segment
// first and bounds again (1M rows: 42.6 -> 32.3 ms).
// With P ranges, range p holds the segments p, p + P, ..
// ONE: the BF16 form's rounded rows, a chain of one product per dimension (500k
// rows, d = 50: screen 40 -> 9 ms).
//
// Rows without clusters are answered by a plain screen: the BF16 form's, which
// merges its lists at three waves per SIMD where this one has two, or the exact
// form's unpruned one in the same order, without this one's spills (lists of 32).
// The first workgroups (PrunedArgs::samples) take tiles spread evenly over all;
// the last of these to know its segments gives the verdict: plain where they are
// more than PrunedArgs::plain_over on average.  A workgroup whose own last list is
// long (PrunedArgs::wait_over) waits for the verdict (those that start with the samples: they know
// theirs at about the same time) and ends if it is plain.  The plain screen then
// takes all queries, so the answer does not depend on who waited how long.
// Samples far from each other share no segments in the caches: 64 of the exact
// form's 782 workgroups of 100k rows (d = 35, 20 clusters) cost 9% of the call, 16
// of them 4.  Up to two rounds of tiles the exact form's stay in their place.
// (Looking for the verdict during the last list instead: the loop around the ring
// spills up to 77 registers more.  Leaving only the tiles with long lists to the
// plain screen: a few of them run for as long as many, 500k BF16 rows 10.4 -> 13.5
// ms.)
constexpr int kWaitLooks = 4000;  // looks for the verdict, about a microsecond each

// Tile of workgroup x: the samples i tiles / samples first, then the others in order.
__device__ __forceinline__ int sampled_tile(int x, int tiles, int samples) {
    if (samples == 0 || samples == tiles) return x;
    if (x < samples) return (int)((int64_t)x * tiles / samples);
    // of the samples' runs (a sample, then the tiles to the next one): the last whose others start at or before x
    int lo = 0, hi = samples - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if ((int64_t)mid * tiles / samples - mid <= x - samples) lo = mid; else hi = mid - 1;
    }
    return x - samples + lo + 1;
}

template <int Q, int TC, int L, bool ONE>
__global__ __launch_bounds__((SplitShape<Q, TC, L>::NW * kWave), (SplitShape<Q, TC, L>::W)) void k_split_pruned(
    PrunedArgs pa) {
    using S = SplitShape<Q, TC, L>;
    constexpr int RING = S::PHP * S::BLOCK;
    constexpr int NWORDS = kSegMax / 32;
    __shared__ __attribute__((aligned(16))) char ring0[RING];
    __shared__ __attribute__((aligned(16))) char ring1[RING];
    __shared__ double qbuf[S::QCAP * S::NW * kWave];
    __shared__ uint32_t mark[NWORDS];  // segments found by the last pass over the bounds
    __shared__ uint32_t done[NWORDS];  // segments screened
    __shared__ int count[NWORDS];
    __shared__ uint16_t list[kSegMax];
    __shared__ uint32_t tmin, tmax;    // float bits of the smallest and largest T
    __shared__ int verdict;
    const ScreenArgs &a = pa.s;
    if (a.kc->wide) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6, h = lane >> 5;
    // whether the verdict is plain, after at most `looks` looks: one answer for the workgroup
    auto plain = [&](int looks) {
        if (tid == 0) {
            int v = 0;
            for (int i = 0; i < looks; ++i) {
                v = __hip_atomic_load(&pa.counters->verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (v != 0) break;
                __builtin_amdgcn_s_sleep(8);
            }
            verdict = v;
        }
        __syncthreads();
        return verdict == kPlain;
    };
    if (pa.samples > 0 && plain(1)) return;
    const int p = blockIdx.y, P = a.P;
    const int nblk = (int)a.nblk, nseg = pa.nseg, sh = pa.seg_shift, nw = (nseg + 31) / 32;
    const int qg = blockDim.x / 2, qs = blockDim.x;
    const int64_t nslots = screen_slots(a);
    const int64_t tile = pa.sample_step ? (int)blockIdx.x : sampled_tile(blockIdx.x, gridDim.x, pa.samples);
    const int64_t slot = tile * qg + wave * 32 + (lane & 31);
    const int64_t row = slot < nslots ? (a.qlist ? (int64_t)a.qlist[slot] : slot) : -1;
    const float scale = ldexpf(1.f, split_exponent(a.kc));

    SplitQuery<Q, TC, ONE> qop;
    qop.load(a.Q, a.d, row, h, scale);
    PackTopK<L, S::QCAP> top;
    top.init();
    double *q = qbuf + tid;
    float xx = 0.f;  // ||a x||^2
    if (row >= 0)
        for (int t = h; t < a.d; t += 2) {
            const float v = a.Q[row * a.d + t] * scale;
            xx = fmaf(v, v, xx);
        }
    xx += __shfl_xor(xx, 32, kWave);
    // the key's error bound, ||a c|| <= 2^14, with the products of T and r and the rounding of xx
    const float slack = 1.5f * (float)pa.eps * (2.f * sqrtf(xx) * 16384.f + 268435456.f) + xx * 0x1p-18f;

    // first the range's segments around the tile's rows
    const int first = pa.own ? pa.own[tile] : (int)((tile * qg / 32) >> sh);
    const int last = pa.own ? first : (int)(min((int64_t)nblk - 1, ((tile + 1) * qg - 1) / 32) >> sh);
    const int reach = max(1, kNearBlocks >> sh) * P;
    const int lo = max(0, first - reach), hi = min(nseg - 1, last + reach);
    const int near0 = lo + (p + P - lo % P) % P;
    int total = near0 <= hi ? (hi - near0) / P + 1 : 0;
    for (int i = tid; i < total; i += qs) list[i] = (uint16_t)(near0 + i * P);
    for (int w = tid; w < NWORDS; w += qs) done[w] = 0u;
    if (tid == 0) {
        tmin = 0xffffffffu;
        tmax = 0u;
    }
    bool final = false;
    int visited = 0;
    for (int round = 0;; ++round) {
        __syncthreads();  // the list is written
        split_stream<Q, TC, S::PHP>(
            static_cast<const char *>(a.Ap), total << sh,
            [&](int i) { return ((int)list[i >> sh] << sh) + (i & ((1 << sh) - 1)); }, ring0, ring1,
            [&](const f16x8(&A)[2 * Q + TC], int blk) {
                if (blk < nblk) top.offer(split_keys(A, qop), blk * 32 + 4 * h, q, qs);
            });
        top.flush(q, qs);
        visited += total;
        if (final) break;
        for (int i = tid; i < total; i += qs) atomicOr(&done[list[i] >> 5], 1u << (list[i] & 31));

        // T of each query, over both halves of its list; a query whose lists are not full takes every segment
        const float thr = fmaxf(top.thr, __shfl_xor(top.thr, 32, kWave));
        const float T = (float)(_Float16)(sqrtf(fmaxf(thr + xx * 1.00001f, 0.f)) * 1.002f);
        const bool bounded = T < 30000.f;
        const float limit = row < 0 ? -INFINITY : bounded ? T * T - xx + slack : INFINITY;
        if (round == 0 && row >= 0 && h == 0) {
            atomicMin(&tmin, __float_as_uint(T));
            atomicMax(&tmax, __float_as_uint(T));
        }
        uint32_t mine = 0u;
        int w = tid + first / 32;  // this thread's word, from the tile's own on and around
        if (w >= nw) w -= nw;
        for (bool nearest = false;; nearest = true) {
            if (h == 1) qop.tail[TC - 1][7] = (_Float16)(bounded && !nearest ? -2.f * T : 0.f);
            for (int i = tid; i < NWORDS; i += qs) mark[i] = 0u;
            float best = INFINITY;
            int at = -1;
            split_stream<Q, TC, S::PHP>(
                static_cast<const char *>(pa.segments), nw, [](int i) { return i; }, ring0, ring1,
                [&](const f16x8(&A)[2 * Q + TC], int blk) {
                    const f32x16 acc = split_keys(A, qop);
                    if (nearest) {
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            if (acc[v] < best) {
                                best = acc[v];
                                at = 32 * blk + 8 * (v >> 2) + 4 * h + (v & 3);
                            }
                        return;
                    }
                    float mn = acc[0];
#pragma unroll
                    for (int v = 1; v < 16; ++v) mn = fminf(mn, acc[v]);
                    if (__ballot(mn <= limit) == 0ull) return;
                    uint32_t bits = 0u;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const unsigned long long b = __ballot(acc[v] <= limit);
                        const int r = 8 * (v >> 2) + (v & 3);
                        bits |= ((uint32_t)b != 0u ? 1u : 0u) << r | ((uint32_t)(b >> 32) != 0u ? 1u : 0u) << (r + 4);
                    }
                    if (lane == 0) atomicOr(&mark[blk], bits);
                });
            if (nearest && row >= 0 && at >= 0) atomicOr(&mark[at >> 5], 1u << (at & 31));
            __syncthreads();
            mine = 0u;
            if (tid < nw) {
                mine = mark[w] & ~done[w];
                for (int i = 0; i < 32; ++i)
                    if (32 * w + i >= nseg || (P > 1 && (32 * w + i) % P != p)) mine &= ~(1u << i);
                count[tid] = __popc(mine);
            }
            __syncthreads();
            total = 0;
            for (int i = 0; i < nw; ++i) total += count[i];
            // (the same for all threads)
            if (nearest || round > 0 || total << sh <= 24 * nw ||
                __uint_as_float(tmax) <= 2.f * __uint_as_float(tmin)) {
                final = !nearest;
                break;
            }
        }
        if (pa.samples > 0 && final) {
            const int x = blockIdx.x, step = pa.sample_step;
            if (p == 0 && tid == 0 && (step ? x % step == 0 && x / step < pa.samples : x < pa.samples)) {
                KnnCounters *kc = pa.counters;
                atomicAdd(&kc->sampled_segments, (unsigned long long)(visited + total));
                __threadfence();
                if (atomicAdd(&kc->sampled, 1) == pa.samples - 1) {
                    const double seen = (double)atomicAdd(&kc->sampled_segments, 0ull);
                    const int v = seen > (double)pa.plain_over * pa.samples ? kPlain : kPruned;
                    __hip_atomic_store(&kc->verdict, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (visited + total > pa.wait_over && plain(kWaitLooks)) return;
        }
        int at = 0;
        for (int i = 0; i < nw; ++i) at += i < tid ? count[i] : 0;
        while (mine) {
            list[at++] = (uint16_t)(32 * w + __builtin_ctz(mine));
            mine &= mine - 1;
        }
    }
    if (row >= 0) top.store(a, slot, p, h, a.ref_map);
    if (tid == 0) atomicAdd(&pa.counters->visited, (unsigned long long)visited);
}

template <int Q, int TC, int L, bool ONE = false>
int pruned_launch_geom(const PrunedArgs &a, const char *name, hipStream_t s) {
    using S = SplitShape<Q, TC, L>;
    ScopedTimer timer(name, s);
    const unsigned gx = (unsigned)((a.s.nq + S::QG - 1) / S::QG);
    hipLaunchKernelGGL((k_split_pruned<Q, TC, L, ONE>), dim3(gx, (unsigned)a.s.P), dim3(S::NW * kWave), 0, s, a);
    return launch_status(name);
}

template <int L>
int pruned_launch(const PrunedArgs &a, const char *name, hipStream_t s) {
    return split_dispatch(split_geom(a.s.d),
                          [&](auto q, auto tc) { return pruned_launch_geom<q.value, tc.value, L>(a, name, s); });
}
extern template int pruned_launch<16>(const PrunedArgs &, const char *, hipStream_t);
extern template int pruned_launch<32>(const PrunedArgs &, const char *, hipStream_t);

// The BF16 form's rows, in lists of 32.
int rounded_launch(const PrunedArgs &a, const char *name, hipStream_t s);

// One launch with lists of L keys per contraction half.
template <int L>
int split_launch(const ScreenArgs &a, const char *name, hipStream_t s) {
    return split_dispatch(split_geom(a.d), [&](auto q, auto tc) { return split_launch_geom<q.value, tc.value, L>(a, name, s); });
}
extern template int split_launch<16>(const ScreenArgs &, const char *, hipStream_t);
extern template int split_launch<32>(const ScreenArgs &, const char *, hipStream_t);

}  // namespace scr
}  // namespace rsc
