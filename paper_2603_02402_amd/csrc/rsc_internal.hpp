// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "../../include/rsc.h"

namespace rsc {

// Thread-local error message behind rsc_last_error().
void set_error(const std::string &msg);
void clear_error();

// Record a HIP failure (if any) and turn it into RSC_ERR_HIP.
int hip_status(hipError_t e, const char *what);
// Check the last launch error.
int launch_status(const char *what);

// Optional per-kernel event timing (rsc_profile_*).  When enabled, a
// ScopedTimer records one event before and one after the launches made in
// its scope on `stream` and files the pair under `name`.
class ScopedTimer {
  public:
    ScopedTimer(const char *name, hipStream_t stream);
    ~ScopedTimer();
    ScopedTimer(const ScopedTimer &) = delete;
    ScopedTimer &operator=(const ScopedTimer &) = delete;

  private:
    std::string name_;
    hipStream_t stream_;
    void *start_;
};

// While a TimerPrefix lives, the timers this thread starts file their pairs
// under prefix + name (a stage that runs a whole kNN call inside another
// call, such as k-means' assignments, keeps its kernels apart from the
// outer call's own).
class TimerPrefix {
  public:
    explicit TimerPrefix(const char *prefix);
    ~TimerPrefix();
    TimerPrefix(const TimerPrefix &) = delete;
    TimerPrefix &operator=(const TimerPrefix &) = delete;

  private:
    const char *prev_;
};

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) & ~(kAlign - 1); }

// Carves 256-byte aligned sub-buffers out of a workspace, or only counts.
struct Carver {
    char *base;
    size_t used = 0;
    explicit Carver(void *b) : base(static_cast<char *>(b)) {}
    template <class T>
    T *take(size_t count) {
        size_t off = used;
        used = align_up(used + count * sizeof(T));
        return base ? reinterpret_cast<T *>(base + off) : nullptr;
    }
};

// ---- kNN stages (knn.hip) -------------------------------------------------

// Device counters of one kNN call, at the start of the workspace.
struct KnnCounters {
    int32_t flagged;          // rows whose first certificate failed (escalated)
    uint32_t max_ratio_bits;  // float bits of the largest error ratio seen
    uint32_t max_norm_bits;   // float bits of max_j ||y_j||
    int32_t flagged2;         // escalated rows whose second certificate failed
    int32_t rescanned;        // rows recomputed exhaustively
    uint32_t query_norm_bits; // float bits of the largest query norm (rectangular problem; else 0)
    int32_t wide;             // nonzero: norms spread too far for the split screen; the FP32 chain runs (the
                              // BF16 form: its plain screen)
    int32_t verdict;          // pruned screen: 0 none yet, kPruned, kPlain (a plain screen answers)
    unsigned long long visited;  // pruned screen: segments screened, over all query tiles (bench.py reads it here)
    int32_t sampled;          // sampled tiles that know their segments
    int32_t pad;
    unsigned long long sampled_segments;  // those segments
};

constexpr int kPruned = 1, kPlain = 2;  // KnnCounters::verdict

struct KnnPlan {
    int64_t nq, nr;
    int d, k, screen, half;  // screen width (32 or 64) = 2 x list length per contraction half
    int dh;                // half of the padded contraction length
    bool self_mode;        // queries are the references (self forced to slot 0)
    int64_t nblk;          // 32-row reference blocks
    int splits;            // reference ranges of the main screen
    int precision;         // rsc_precision of the screen
    int metric;            // rsc_metric
    int resid;             // FP8 residual variant: reference partitions (0 = off)
    bool pruned;           // exact path: room for the spatial order and its segments (knn_run)
};

// Spatial order of a reference matrix and of a query matrix (spatial.hip).
constexpr int kSegMax = 8192;  // segments of an order
struct SpatialBuffers {
    int nseg, seg_blocks;    // segments, packed blocks per segment (a power of two)
    int32_t *pivot, *rank;
    float *nearest, *pairs;
    uint32_t *bounds;
    void *pivot_packed;
    uint32_t *key, *rkey, *qkey;  // unsorted; sorted keys of references / queries
    int32_t *id, *rperm, *qperm;  // rows in order
    int32_t *own;                 // segment of the references where each query tile belongs
    float *centre, *radius;
    void *seg_packed;
    void *tmp;
    size_t tmp_bytes;
};
int spatial_seg_blocks(int64_t nblk);
size_t spatial_carve(int64_t nq, int64_t nr, int d, void *base, SpatialBuffers *out);
// Orders the references (norms and their maximum known) and bounds the segments.
// rounded: BF16 rows, whose segments are packed as one FP16 part.
int spatial_refs(const float *R, const float *nrow, int64_t nr, int d, bool rounded, const SpatialBuffers &b,
                 KnnCounters *kc, hipStream_t s);
// Orders the queries of a rectangular problem and places their tiles of qg.
int spatial_queries(const float *Q, int64_t nq, int64_t nr, int d, int qg, const SpatialBuffers &b, KnnCounters *kc,
                    hipStream_t s);

struct KnnBuffers {
    SpatialBuffers sp;  // pruned exact screen
    KnnCounters *counters;
    float *nrow, *packed, *norms;
    void *split;      // exact path: references packed for the split FP16 screen
    float *scal;      // FP8 per-dimension scales
    uint32_t *amax;   // FP8 per-dimension absmax bits
    int32_t *cand_idx;
    float *cand_key;
    int32_t *flag1, *flag2;
    int32_t *esc_idx;
    float *esc_key;
    double *esc_bound;  // flagged rows: bound of the m-th distance, candidates collected
    int32_t *esc_found;
    float *qn, *rn;   // the rows as screened: unit-normalised (cosine metric), rounded (large BF16 problems)
    // FP8 residual variant
    float *cent;          // partition centroids, resid x d
    int32_t *assign, *perm, *init, *map;
    int32_t *qcount;  // the number of queries screened through perm (device)
    void *order_ws;   // reduced-precision screens: workspace of the spatial query order
    int32_t *blk_part;    // partition of each packed block, 4 copies per block
    int64_t *poff, *pblk;
    void *kws;            // k-means workspace
    size_t kws_bytes;
};

// Arguments of the float64 rerank (knn.hip).
struct RerankArgs {
    const float *Q;
    int64_t nq;
    const int32_t *qlist;   // optional: slot -> row
    const int32_t *qcount;
    int qcap;
    const float *R;
    int d, k, S, KP, P;
    int self_mode;
    int certify;            // 0: approximate screen, never flag rows
    int metric;             // rsc_metric of the reported distances
    double cosine_eps;      // cosine: bound on |screened key - (2 D - 1)| for unit vectors
    const int32_t *cand_idx;
    const float *cand_key;
    double eps_coef;
    // keys of the split FP16 screen (times its squared scale, unless the
    // inputs were marked wide; 2: nor where the plain BF16 screen answered): its
    // error bound in place of eps_coef / cosine_eps
    int split;
    double split_eps, split_abs, split_cosine_eps;
    KnnCounters *counters;
    int32_t *flag_out;   // rows that fail the certificate
    int32_t *flag_count;
    // optional, for the first flag_cap flagged rows: the m-th distance found
    // (squared if Euclidean), an upper bound of the true one, and a zeroed count
    double *flag_bound;
    int32_t *flag_found;
    int flag_cap;
    // optional: candidates per slot, in any order and complete (k_split_collect);
    // more than KP of them flag the row
    const int32_t *counts;
    int32_t *out_idx;
    float *out_dist;
};

// Fill a plan; returns RSC_OK or an error status (with message set).
int knn_plan(int64_t nq, int64_t nr, int d, int k, const rsc_knn_opts *opts, bool self_mode, KnnPlan *plan);
// Bytes of workspace for a plan; with ws != nullptr also carves the buffers.
size_t knn_workspace(const KnnPlan &p, void *ws, KnnBuffers *out);
// With qlist (device rows) the query slots are the first min(*qcount, p.nq)
// rows of the list; outputs are written at those rows.
int knn_run(const KnnPlan &p, const float *Q, const float *R, int32_t *out_idx, float *out_dist, void *ws,
            hipStream_t stream, const int32_t *qlist = nullptr, const int32_t *qcount = nullptr);

// Pieces of the exact path reused by the batched form (knn.hip).
double knn_eps_coefficient(int d);
// Counters and norms.  Q: the queries of a rectangular problem (their largest
// norm enters the split's scale), else null.
int knn_prep(const KnnPlan &p, const float *R, const float *Q, const KnnBuffers &b, hipStream_t stream);
// Packs nblk blocks for the FP32 chain: rows in order, per sample (device tables
// blk_sample, boff, soff) or by row_map (-1: padding).  gate: only where its
// inputs were marked wide.
int knn_pack_fp32(int dh, const float *R, const float *nrow, int64_t nr, int d, int64_t nblk, float *packed,
                  float *norms, const int32_t *blk_sample, const int64_t *boff, const int64_t *soff,
                  const int32_t *row_map, const KnnCounters *gate, hipStream_t stream);
// The rerank's error bounds for keys of the split screen.
void knn_split_bounds(RerankArgs &ra);
int knn_launch_rerank(const RerankArgs &ra, int64_t slots, const char *name, hipStream_t stream);
// exhaustive float64 rescan of the rows flagged in b (first certificate only
// when there was no escalation); soff/nsamples restrict each row to its sample.
// (uses p.metric for the distances)
int knn_launch_rescan(const KnnPlan &p, const float *Q, const float *R, const KnnBuffers &b, int esc_cap,
                      int32_t *out_idx, float *out_dist, const int64_t *soff, int nsamples, hipStream_t stream);

namespace scr {
struct ScreenArgs;
}
// Squared norms of R's rows into nrow and their maximum into counters
// (counters re-initialised).
int knn_norms(const float *R, int64_t nr, int d, float *nrow, KnnCounters *counters, hipStream_t stream);
// FP32 packing of nblk blocks whose packed row 32b + c is row_map[32b + c]
// of R (-1: padding with an infinite norm).
size_t knn_packed_floats(int dh, int64_t nblk);
// Split FP16 screen of the exact path (knn_split.hip).
size_t split_packed_bytes(int d, int64_t nblk);
int split_queries_per_group(int d, int half_width);
// Packs nblk blocks (sample tables as knn_pack_fp32; row_map: the rows at
// the first nmap positions, -1 and the positions past them padded)
// and marks inputs whose norms spread too far; needs the norms of R.
int split_pack(const float *R, const float *nrow, int64_t nr, int d, int64_t nblk, void *packed,
               const int32_t *blk_sample, const int64_t *boff, const int64_t *soff, const int32_t *row_map,
               int64_t nmap, KnnCounters *counters, hipStream_t stream, bool rounded = false);
int split_screen(const scr::ScreenArgs &a, int half_width, const char *name, hipStream_t s);
// All references within a bound of each listed row (knn_split.hip).
struct CollectArgs {
    const float *Q;          // as screened (unit rows for the cosine metric)
    int d, metric;
    const int32_t *rows, *nrows;  // the listed rows and their count, at most cap
    int cap;
    const double *bound;     // per listed row: the m-th distance found (squared if Euclidean)
    int32_t *found;          // per listed row: references found (zeroed)
    int width;               // room per listed row
    int32_t *out_idx;
    float *out_key;
    const void *packed;
    const int32_t *ref_map;
    int64_t nr, nblk;
    double eps, eps_abs, cosine_eps;
    // inputs marked wide: the references packed for the FP32 chain (row order) and its keys' error bounds
    const void *packed32;
    const float *norms32;
    int dh;
    double fp32_eps, fp32_cosine_eps;
    const KnnCounters *kc;
};
int split_collect(const CollectArgs &a, hipStream_t s);
// The pruned screen over a spatial order: own = the segment of each query
// tile (null: the queries are the references in their order).
struct PrunedArgs;
int split_screen_pruned(const PrunedArgs &a, int half_width, const char *name, hipStream_t s);
size_t rounded_packed_bytes(int d, int64_t nblk);  // the BF16 form's rows
double split_eps_coefficient(int d);
double split_abs_coefficient(int d);
// Reduced-precision screens (knn_lowp.hip).
int lowp_steps(int precision, int d);
int lowp_qb(int precision, int d);
int lowp_queries_per_group(int precision, int d);
size_t lowp_packed_bytes(int precision, int64_t nblk, int d);
// Packs the references (rmap: packed slot -> row, or null for row order).
// gate (BF16): only where the plain screen is to answer.
int lowp_prepare(const KnnPlan &p, const float *Q, const float *R, void *packed, float *norms, float *scal,
                 uint32_t *amax, const int32_t *rmap, hipStream_t stream, const KnnCounters *gate = nullptr);
int lowp_screen(const KnnPlan &p, const scr::ScreenArgs &a, unsigned gx, hipStream_t s);
// FP8 residual variant: partitions, residual scales and the partition-ordered
// packing (into b.packed / b.norms, with b.map and b.blk_part); then, after
// the screen, the candidates' packed rows turned back into row ids.
int lowp_prepare_resid(const KnnPlan &p, const float *R, const KnnBuffers &b, hipStream_t stream);
int lowp_unmap(const KnnPlan &p, const KnnBuffers &b, hipStream_t stream);
// Candidates from packed slots to rows through the packing's row map.
int lowp_unmap_rows(const KnnPlan &p, const KnnBuffers &b, const int32_t *rmap, hipStream_t stream,
                    const KnnCounters *gate = nullptr);

// Spatial order of query rows (query_order.hip): perm = the rows sorted by a
// Morton code of their first three coordinates.
size_t query_order_workspace(int64_t nq);
int query_order_run(const float *Q, int64_t nq, int d, void *ws, int32_t *perm, hipStream_t s);
// The same within each of S samples (rows soff[s] .. soff[s+1]-1, device
// offsets): perm holds every sample's rows at its own positions.
size_t sample_order_workspace(int64_t n);
int sample_order_run(const float *X, int64_t n, int d, const int64_t *soff, int S, void *ws, int32_t *perm,
                     hipStream_t s);

// Batched form (knn_batched.hip).
size_t batched_workspace_bytes(const int64_t *offsets, int S, int d, int k);
int batched_run(const float *X, const int64_t *offsets, int S, int d, int k, int32_t *out_idx, float *out_dist,
                void *ws, size_t ws_bytes, hipStream_t s);
int batched_autotune(const float *X, const int64_t *offsets, int S, int d, int k, void *ws, size_t ws_bytes,
                     hipStream_t s, int32_t *chosen, float *times_ms);
const char *batched_policy_name(int pol);
const char *batched_trial_name(int trial);

// ---- routed form (partition.hip, router.hip, routed.hip) -----------------

size_t kmeans_workspace_bytes(int64_t n, int d, int P);
int kmeans_run(const float *X, int64_t n, int d, int P, const int32_t *init_rows, int iters, float *C,
               int32_t *assign, int64_t *offsets, int32_t *perm, int64_t *relocated, void *ws, size_t ws_bytes,
               hipStream_t s);
size_t partition_lists_workspace_bytes(int P);
int partition_lists(const int32_t *assign, int64_t n, int P, int64_t *offsets, int32_t *perm, void *ws,
                    size_t ws_bytes, hipStream_t s);
int partition_labels(const int32_t *idx, int64_t n, int k, const int32_t *assign, int64_t n_assign, int32_t *labels,
                     hipStream_t s);

int router_create(rsc_router **out, int d, int hidden, int parts, uint64_t seed);
void router_destroy(rsc_router *R);
int router_info(const rsc_router *R, int *d, int *hidden, int *parts, int64_t *n_params, int64_t *step);
size_t router_train_workspace(const rsc_router *R, int batch, int64_t n);
int router_train(rsc_router *R, const float *X, int64_t n, const int32_t *labels, int m, int epochs, int batch,
                 float lr, float *loss_log, void *ws, size_t ws_bytes, hipStream_t s);
size_t router_gradients_workspace(const rsc_router *R, int64_t n);
int router_gradients(const rsc_router *R, const float *X, int64_t n, const int32_t *labels, int m, float *grad_out,
                     float *loss_out, void *ws, size_t ws_bytes, hipStream_t s);
size_t router_infer_workspace(const rsc_router *R);
// Logits (logits != nullptr) or the top `probes` partitions and their mass
// of n rows (rows of X, or X[list[i]]).
int router_infer(const rsc_router *R, const float *X, int64_t n, const int32_t *list, float *logits, int probes,
                 int32_t *parts, float *mass, void *ws, size_t ws_bytes, hipStream_t s);
int router_save(const rsc_router *R, const char *path);
int router_load(rsc_router *R, const char *path);
int router_shape(const rsc_router *R, int *d, int *parts);

size_t probed_workspace_bytes(int64_t n, int d, int k, int P, int probes);
// mass/threshold: rows whose mass is below the threshold go to exact search
// (instead of, or besides, exact_rows).
int probed_run(const float *X, int64_t n, int d, int k, const int64_t *offsets, const int32_t *perm, int P,
               const int32_t *probe_parts, int probes, const uint8_t *exact_rows, const float *mass,
               float threshold, int32_t *out_idx, float *out_dist, uint8_t *out_route, rsc_routed_stats *stats,
               void *ws, size_t ws_bytes, hipStream_t s);

// ---- energy distance (edistance.hip) -------------------------------------

size_t edistance_sums_workspace_bytes(int64_t G, int64_t npairs, int64_t ncells, int d);
size_t edistance_pairwise_workspace_bytes(int64_t G, int64_t ncells, int d);
size_t edistance_onesided_workspace_bytes(int64_t G, int64_t ncells, int d);
size_t edistance_groups_workspace_bytes(int64_t n, int64_t G);
int edistance_groups(const int32_t *labels, int64_t n, int64_t G, int64_t *offsets, int32_t *cells, void *ws,
                     size_t ws_bytes, hipStream_t s);
int edistance_sums(const float *X, int64_t n, int d, const int64_t *offsets, int64_t G, const int32_t *cells,
                   const int32_t *pairs, int64_t npairs, double *sums, void *ws, size_t ws_bytes, hipStream_t s);
int edistance_pairwise(const float *X, int64_t n, int d, const int64_t *offsets, int64_t G, const int32_t *cells,
                       double *E, double *D, void *ws, size_t ws_bytes, hipStream_t s);
int edistance_onesided(const float *X, int64_t n, int d, const int64_t *offsets, int64_t G, const int32_t *cells,
                       int64_t ref, double *E, void *ws, size_t ws_bytes, hipStream_t s);

// ---- sparse PCA (pca.hip) -------------------------------------------------

size_t pca_workspace_bytes(int64_t n, int p, int k);
int pca_covariance(const int64_t *indptr, const int32_t *indices, const float *data, int64_t n, int p, double *mean,
                   double *cov, void *ws, size_t ws_bytes, hipStream_t s);
int pca_run(const int64_t *indptr, const int32_t *indices, const float *data, int64_t n, int p, int k, double *mean,
            double *cov, double *evals, double *loadings, float *Z, void *ws, size_t ws_bytes, hipStream_t s);

// ---- UMAP layout (umap.hip) -----------------------------------------------

size_t umap_workspace_bytes(int64_t n, int64_t nnz, int dim, int neg);
int umap_layout(const int64_t *indptr, const int32_t *indices, const float *weights, int64_t n, int64_t nnz,
                int dim, float *Y, int n_epochs, double a, double b, double gamma, double alpha0, int neg,
                uint64_t seed, void *ws, size_t ws_bytes, hipStream_t s);

// ---- graph stages (graph.hip) --------------------------------------------

// Workspace of a graph build over n rows of k slots; S > 0 adds room for
// the offsets of S samples (the batched form).
size_t graph_workspace_bytes(int64_t n, int k, int32_t S = 0);
int graph_run(const int32_t *idx, const float *dist, int64_t n, int k, int64_t *indptr, int32_t *indices,
              float *data, int64_t *nnz, double *rho, double *sigma, void *ws, hipStream_t stream);
// As graph_run, with every edge checked to stay inside its row's sample
// (seg_host: HOST int64 [S + 1] sample offsets, validated by the caller).
int graph_run_batched(const int32_t *idx, const float *dist, int64_t n, int k, const int64_t *seg_host, int32_t S,
                      int64_t *indptr, int32_t *indices, float *data, int64_t *nnz, void *ws, hipStream_t stream);
// As graph_run, with the workspace taken from a fixed device array of
// graph_noalloc_max_bytes() bytes instead of the caller (RSC_ERR_CAPACITY
// when the problem needs more).
size_t graph_noalloc_max_bytes();
int graph_run_noalloc(const int32_t *idx, const float *dist, int64_t n, int k, int64_t *indptr, int32_t *indices,
                      float *data, int64_t *nnz, double *rho, double *sigma, hipStream_t stream);

// ---- Leiden communities (leiden.hip) ----------------------------------------

size_t leiden_workspace_bytes(int64_t n, int64_t nnz);
int leiden_run(const int64_t *indptr, const int32_t *indices, const float *weights, int64_t n, int64_t nnz,
               double gamma, int32_t *labels, rsc_leiden_stats *stats, void *ws, hipStream_t s);

}  // namespace rsc
