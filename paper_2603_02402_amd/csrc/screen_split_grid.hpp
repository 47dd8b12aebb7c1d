// The grid-mapped launch of the split screen, instantiated per list length in
// a translation unit of its own (knn_split.hip, knn_split_wide.hip).
#pragma once

#include "screen_split.hpp"

namespace rsc {
namespace scr {

constexpr int64_t kCUs = 256;  // MI355X

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
    if (a.kc->wide) return;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, c = tid & 31;
    const int p = blockIdx.y;
    // Range p holds a run of packed blocks, or, with references packed in the
    // queries' order, the blocks p, p + P, ..: every range gets a share of
    // every neighbourhood.
    const int nblk = (int)a.nblk, per = (nblk + a.P - 1) / a.P;
    const int step = a.rotate ? a.P : 1, b0 = a.rotate ? p : p * per;
    const int span = a.rotate ? (p < nblk ? (nblk - p + a.P - 1) / a.P : 0) : max(0, min(per, nblk - b0));
    const int64_t nslots = screen_slots(a);
    const int qg = blockDim.x / 2;  // queries of the workgroup
    for (int64_t qblk = blockIdx.x; qblk * qg < nslots; qblk += gridDim.x) {
        const int64_t slot = qblk * qg + wave * 32 + c;
        int64_t row = -1;
        if (slot < nslots) row = a.qlist ? (int64_t)a.qlist[slot] : slot;
        // near references first: start at the group's own rows
        const int rot = a.rotate && span > 0 ? min((int)(qblk * (qg / 32) / a.P), span - 1) : 0;
        screen_split_tile<Q, TC, L>(a, slot < nslots ? slot : -1, row, b0, step, span, rot, p, 0, ring0, ring1, qbuf);
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

// One launch with lists of L keys per contraction half.
template <int L>
int split_launch(const ScreenArgs &a, const char *name, hipStream_t s) {
    return split_dispatch(split_geom(a.d), [&](auto q, auto tc) { return split_launch_geom<q.value, tc.value, L>(a, name, s); });
}
extern template int split_launch<16>(const ScreenArgs &, const char *, hipStream_t);
extern template int split_launch<32>(const ScreenArgs &, const char *, hipStream_t);

}  // namespace scr
}  // namespace rsc
