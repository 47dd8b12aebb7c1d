// The sort behind the row orders (query_order.hip, spatial.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>

#include "rsc_internal.hpp"

namespace rsc {

// Rows one sort takes while its stream is being recorded into a graph: above
// 2^20 rows the library clears its counters by memset, which is recorded as
// memset nodes (9 of them at 2^20 + 1 rows, none at 2^20), and such nodes have
// given wrong results on replays.
constexpr int64_t kRecordedSortRows = (int64_t)1 << 20;

// Scratch of a sort of n pairs (it never shrinks as n grows); 0 on failure.
template <class Key>
size_t order_sort_bytes(int64_t n, int bits) {
    size_t tmp = 0;
    if (rocprim::radix_sort_pairs(nullptr, tmp, (const Key *)nullptr, (Key *)nullptr, (const int32_t *)nullptr,
                                  (int32_t *)nullptr, (size_t)n, 0, bits, (hipStream_t)0) != hipSuccess)
        return 0;
    return std::max<size_t>(tmp, 1);
}

// Sorts n (key, row) pairs by the low `bits` of the key.  On a stream that is
// being recorded the pieces of kRecordedSortRows are sorted one by one: still an
// order of all rows, which is all that its users rely on.
template <class Key>
int order_sort(void *tmp, size_t tmp_bytes, const Key *key, Key *sorted, const int32_t *row, int32_t *perm, int64_t n,
               int bits, const char *what, hipStream_t s) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool recorded = hipStreamIsCapturing(s, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone;
    const int64_t piece = recorded ? kRecordedSortRows : n;
    for (int64_t i = 0; i < n; i += piece) {
        size_t bytes = tmp_bytes;
        const int st = hip_status(rocprim::radix_sort_pairs(tmp, bytes, key + i, sorted + i, row + i, perm + i,
                                                            (size_t)std::min(piece, n - i), 0, bits, s),
                                  what);
        if (st != RSC_OK) return st;
    }
    return RSC_OK;
}

}  // namespace rsc
