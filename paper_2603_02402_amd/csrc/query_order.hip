// Spatial order of the query rows for the reduced-precision screens.
//
// The screens keep, per lane, a queue of keys that beat the lane's threshold
// and merge all lanes' queues together whenever one of them could overflow.
// When the 32 queries of a wave lie close together, the references that
// enter one query's list tend to enter its neighbours' too, so the queues
// fill together and fewer merges and fewer blocks with any key below a
// threshold occur.  The order is a Morton (Z-order) code of the first three
// coordinates, each quantised to 10 bits over its range, sorted by rocPRIM's
// radix sort (in pieces while a stream is recorded, order_sort.hpp); the rows'
// results are written back in row order, so the order changes which candidates
// a screen keeps only through the threshold history, never the rows of the
// answer.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "morton.hpp"
#include "order_sort.hpp"
#include "rsc_internal.hpp"

namespace rsc {
namespace {

constexpr int kOrderDims = 3;
constexpr int kOrderBits = 10;  // per coordinate (quantise10): 30-bit keys

__global__ void k_qo_init(uint32_t *bounds) {
    if (threadIdx.x < kOrderDims) {
        bounds[2 * threadIdx.x] = 0xffffffffu;  // running minimum (ordered bits)
        bounds[2 * threadIdx.x + 1] = 0u;       // running maximum
    }
}

__global__ __launch_bounds__(256) void k_qo_bounds(const float *__restrict__ Q, int64_t nq, int d, int D,
                                                   uint32_t *__restrict__ bounds) {
    uint32_t lo[kOrderDims], hi[kOrderDims];
#pragma unroll
    for (int t = 0; t < kOrderDims; ++t) {
        lo[t] = 0xffffffffu;
        hi[t] = 0u;
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq; i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int t = 0; t < kOrderDims; ++t) {
            if (t < D) {
                const uint32_t u = ordered_bits(Q[i * d + t]);
                lo[t] = min(lo[t], u);
                hi[t] = max(hi[t], u);
            }
        }
    }
    // Atomics only where a bound moves: they all meet in six words (one pair
    // per thread took 295 us at 500K rows).
#pragma unroll
    for (int t = 0; t < kOrderDims; ++t) {
        if (t < D) {
            for (int o = 32; o > 0; o >>= 1) {
                lo[t] = min(lo[t], (uint32_t)__shfl_xor((int)lo[t], o, 64));
                hi[t] = max(hi[t], (uint32_t)__shfl_xor((int)hi[t], o, 64));
            }
            if ((threadIdx.x & 63) == 0) {
                volatile uint32_t *seen = bounds;
                if (lo[t] < seen[2 * t]) atomicMin(&bounds[2 * t], lo[t]);
                if (hi[t] > seen[2 * t + 1]) atomicMax(&bounds[2 * t + 1], hi[t]);
            }
        }
    }
}

// Key: the Morton code, below the row's sample when sample offsets are given.
template <class Key>
__global__ __launch_bounds__(256) void k_qo_keys(const float *__restrict__ Q, int64_t nq, int d, int D,
                                                 const uint32_t *__restrict__ bounds, Key *__restrict__ key,
                                                 int32_t *__restrict__ row, const int64_t *__restrict__ soff, int S) {
    float lo[kOrderDims], scale[kOrderDims];
#pragma unroll
    for (int t = 0; t < kOrderDims; ++t) {
        lo[t] = 0.f;
        scale[t] = 0.f;
        if (t < D) {
            const float a = from_ordered(bounds[2 * t]), b = from_ordered(bounds[2 * t + 1]);
            lo[t] = a;
            scale[t] = scale10(a, b);
        }
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq; i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t k = 0;
#pragma unroll
        for (int t = 0; t < kOrderDims; ++t) {
            if (t < D) {
                k |= spread3(quantise10(Q[i * d + t], lo[t], scale[t])) << (kOrderDims - 1 - t);
            }
        }
        Key full = (Key)k;
        if constexpr (sizeof(Key) == 8) {
            int a = 0, b = S - 1;
            while (a < b) {
                const int mid = (a + b + 1) / 2;
                if (soff[mid] <= i) a = mid; else b = mid - 1;
            }
            full |= (Key)a << (kOrderDims * kOrderBits);
        }
        key[i] = full;
        row[i] = (int32_t)i;
    }
}

template <class Key>
struct OrderWs {
    uint32_t *bounds;
    Key *key, *key2;
    int32_t *row;
    void *tmp;
    size_t tmp_bytes;
};

template <class Key>
size_t carve_order(int64_t nq, int bits, void *base, OrderWs<Key> *out) {
    const size_t m = (size_t)std::max<int64_t>(nq, 1);
    const size_t tmp = order_sort_bytes<Key>((int64_t)m, bits);
    if (!tmp) return 0;
    Carver cv(base);
    OrderWs<Key> w{};
    w.bounds = cv.take<uint32_t>(2 * kOrderDims);
    w.key = cv.take<Key>(m);
    w.key2 = cv.take<Key>(m);
    w.row = cv.take<int32_t>(m);
    w.tmp_bytes = tmp;
    w.tmp = cv.take<char>(tmp);
    if (out) *out = w;
    return cv.used;
}

template <class Key>
int order_run(const float *Q, int64_t nq, int d, const int64_t *soff, int S, int ws_bits, int bits, void *ws,
              int32_t *perm, hipStream_t s) {
    if (nq <= 0) return RSC_OK;
    OrderWs<Key> w;
    if (!carve_order<Key>(nq, ws_bits, ws, &w)) {
        set_error("query order: rocPRIM sort sizing failed");
        return RSC_ERR_HIP;
    }
    ScopedTimer timer("query_order", s);
    const int D = std::min(d, kOrderDims);
    const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((nq + 255) / 256, 4096));
    hipLaunchKernelGGL(k_qo_init, dim3(1), dim3(64), 0, s, w.bounds);
    hipLaunchKernelGGL(k_qo_bounds, dim3(std::min(g, 1024u)), dim3(256), 0, s, Q, nq, d, D, w.bounds);
    hipLaunchKernelGGL(k_qo_keys<Key>, dim3(g), dim3(256), 0, s, Q, nq, d, D, w.bounds, w.key, w.row, soff, S);
    int st = launch_status("query order keys");
    if (st != RSC_OK) return st;
    return order_sort<Key>(w.tmp, w.tmp_bytes, w.key, w.key2, w.row, perm, nq, bits, "sort of the query order", s);
}

constexpr int kCodeBits = kOrderDims * kOrderBits;

}  // namespace

size_t query_order_workspace(int64_t nq) { return carve_order<uint32_t>(nq, kCodeBits, nullptr, nullptr); }

int query_order_run(const float *Q, int64_t nq, int d, void *ws, int32_t *perm, hipStream_t s) {
    return order_run<uint32_t>(Q, nq, d, nullptr, 0, kCodeBits, kCodeBits, ws, perm, s);
}

size_t sample_order_workspace(int64_t n) { return carve_order<uint64_t>(n, 64, nullptr, nullptr); }

int sample_order_run(const float *X, int64_t n, int d, const int64_t *soff, int S, void *ws, int32_t *perm,
                     hipStream_t s) {
    int bits = kCodeBits;
    while (bits < 64 && ((int64_t)1 << (bits - kCodeBits)) < S) ++bits;
    return order_run<uint64_t>(X, n, d, soff, S, 64, bits, ws, perm, s);
}

}  // namespace rsc
