// Index object and internal entry points shared by the library's host code.
#pragma once

#include <cmath>
#include <functional>
#include <memory>
#include <mutex>
#include <vector>

#include "common.h"

namespace scan {

// Tunable parameters of the intersection kernels (chosen per graph by the
// autotuner or the defaults).
struct IntersectConfig {
  int32_t small_max = 256;  // owners of degree <= small_max: one wavefront each
  // Row slots per chunk of a larger owner (builds with 512, 768 and 1024, R-MAT
  // of 60,000 vertices 493, 470 and 506 us, R-MAT-20 6.03, 5.94 and 6.00 ms).
  int32_t spc = 768;
  int32_t wbits = 20;       // LDS bitmap window of 2^wbits ids (clamped to LDS)
  // small_max and spc were left to the build, which then goes by the number of
  // vertices with neighbours (kWideRows).
  bool auto_shapes = true;
  bool search_windows = false;  // several windows: search row ranges instead of tabling them
  int32_t skip_deg = 0x7fffffff;  // edges whose endpoints both exceed this degree are left unwritten
                                  // (approximate builds overwrite them)
};

struct IntersectStats {
  int32_t wbits = 0;
  int32_t launches = 0;
  int32_t hub_rows = 0, hub_cols = 0;  // of the product over hub rows (0: none)
  // Optional pinned host int32[4]: receives (light vertices, bitmap chunks,
  // -, heavy vertices) asynchronously, in stream order.
  int32_t *host_counts = nullptr;
  // around the small-owner launches and around the large-owner launch (on
  // the streams that run them; the two may overlap)
  hipEvent_t ev_plan_end = nullptr;  // after the ownership plan
  hipEvent_t ev_small_begin = nullptr, ev_small_end = nullptr;
  hipEvent_t ev_big_begin = nullptr, ev_big_end = nullptr;
};

// a2: the ownership plan, enqueued on s. The work lists live in `arena`, which
// must outlive intersect_all; `counts` is kPlanCountBytes of device memory
// (PlanCounts, zero but for rows), and what follows it belongs to the caller: the plan's last step
// copies `words` int32 from `counts` to pinned `host` memory, and `ready` is
// recorded then. The caller waits for it before
// intersect_all.
//
// The shapes of a build that leaves them open follow from the number of
// vertices with neighbours, counted by the degree pass (PlanCounts::rows, set
// before the plan): above kWideRows, a window of the bitmap, the ids stay in
// several windows also when numbered without the isolated vertices; every
// chunk then sweeps the windows, so fewer, larger chunks pay (a thread per
// slot), and owners that one wavefront can take. Builds with small_max / spc
// of 256 / 768 and 512 / 1024, in ms: several windows, R-MAT-23 312 and 286,
// R-MAT of 4M vertices 42.6 and 38.7, of 2M (1.1M with neighbours) 15.5 and
// 15.5, of 2.2M 12.2 and 12.5, random graphs of 2.2M vertices and degree 300
// 276 and 158, degree 600 506 and 519; one window, R-MAT-20 among 4M ids 6.5
// and 7.0, R-MAT of 1.5M (0.8M with neighbours) 8.0 and 9.1, 100,000 vertices
// of degree 400 among 2.2M ids 8.2 and 10.5.
constexpr int32_t kWideRows = 1 << 20;
constexpr int32_t kWideSmallMax = 512, kWideSpc = 1024;
constexpr int32_t kDegBins = 192;  // eight per octave from degree 128 up
constexpr size_t kPlanCountBytes = 32 + 4 * (size_t)kDegBins;
// Least degree of bin b (b = kDegBins: past every degree).
__host__ __device__ inline int32_t deg_bin_low(int b) {
  const int64_t lo = (int64_t)(128 + 16 * (b & 7)) << (b >> 3);
  return lo > 0x7fffffff ? 0x7fffffff : (int32_t)lo;
}
__device__ __forceinline__ int deg_bin(int32_t d) {  // d >= 128
  const int o = 24 - __clz(d);
  return 8 * o + (int)(((uint32_t)d >> (o + 4)) & 7u);
}
constexpr int32_t kLightDeg = kWave;  // one wavefront per vertex up to this degree
struct PlanCounts {
  int32_t small;    // vertices of degree 1..kLightDeg
  int32_t big;      // chunks of the vertices of degree above small_max
  int32_t counter;  // work counter of the large-owner kernel
  int32_t heavy;    // vertices of degree kLightDeg+1..small_max
  int32_t done;     // workgroups of k_plan that have finished
  int32_t rows;     // vertices with neighbours (counted before the plan)
  int32_t small_max, spc;  // the shapes that the plan took
  int32_t bins[kDegBins];  // vertices by degree, from 128 up
};
static_assert(sizeof(PlanCounts) == kPlanCountBytes, "the maximum degrees follow the counts");
struct SmallOwner {
  int32_t h, dh;  // vertex, degree
  int64_t oh;     // first slot of its row
};
struct VertexRecord {  // what the large owners read of a neighbour, in one line
  int32_t deg, hub;    // degree, hub row or -1
  int64_t off;         // first slot of its row
};
struct BigChunk {
  int32_t h;
  int32_t k;    // slots [k*spc, (k+1)*spc) of row h
  int32_t dh;   // degree of h
  int32_t pad;
  int64_t oh;   // first slot of row h
};
struct IntersectPlan {
  int64_t n = 0, nnz = 0;
  bool one_graph = false;  // set by the caller
  bool weighted = false;   // the weighted kernels will run (set by the caller): no records
  SmallOwner *lists = nullptr;          // n entries: the light ones first, the heavy ones at the end
  VertexRecord *records = nullptr;      // n entries, for the intersection to fill
  void *big_list = nullptr, *counts = nullptr;  // device chunk list and counts
  const void *host = nullptr;                   // the host's copy of the counts
  // helper streams already ordered after the plan (set by the caller), used
  // for the two small-owner kernels; null: intersect_all orders its own
  hipStream_t helper[2] = {nullptr, nullptr};
  IntersectPlan() = default;
  IntersectPlan(const IntersectPlan &) = delete;
  IntersectPlan &operator=(const IntersectPlan &) = delete;
};
scan_status intersect_plan(const IntersectConfig &cfg, int64_t n, int64_t nnz, const int64_t *off,
                           const int32_t *deg, DevArena &arena, hipStream_t s, void *counts, int32_t words, void *host, hipEvent_t ready, IntersectPlan &plan);

// Common neighbours among hubs by matrix product (hubs.hip).
constexpr int32_t kHubMaxRows = 49152, kHubMaxCols = 65536;  // counts of common columns fit 16 bits
constexpr int32_t kHubMaxWindows = 63;
struct HubShape {
  int32_t rows = 0, cols = 0;        // their numbers (0: no product)
  int32_t row_deg = 0, col_deg = 0;  // least degrees
  int64_t slots = 0;                 // at least the rows' ids
};
struct HubRow {
  int64_t off;  // its ids outside the columns: rest[off, off + len)
  int32_t len;
  int32_t pad;
};
struct HubView {
  int32_t rows = 0, cols = 0;          // cols padded to a multiple of 256
  int32_t stride = 0;                  // rows padded to a multiple of 256
  const int32_t *col = nullptr;        // per vertex: its column, or -1
  const HubRow *row_of = nullptr;
  const int32_t *rest = nullptr;
  const uint4 *bits = nullptr;         // 128 columns of a row per entry (piece)
  const uint16_t *pre = nullptr;       // [row * cols / 128 + q]: bits before block q
  const uint16_t *D = nullptr;         // [i * stride + j], i >= j: common columns of rows i and j
  __host__ __device__ int64_t piece(int32_t r, int32_t q) const {
    return ((int64_t)(r >> 5) * (cols / 128) + q) * 32 + (r & 31);
  }
};
HubShape choose_hubs(const PlanCounts &pc, int64_t nnz, bool one_window);
// The rows' numbers go into records. win (several id windows): window starts of the rows' rests, rows x (nwin + 1).
scan_status prepare_hubs(const HubShape &shape, int64_t n, const int64_t *off, const int32_t *deg,
                         const int32_t *adj, const int32_t *radj, int32_t wbits, int32_t nwin, int32_t *win,
                         VertexRecord *records, DevArena &arena, hipStream_t s, HubView *out);

// a2-a4: ownership plan, then intersection + similarity for every edge,
// written into both CSR slots of sims (and counts if non-null).
// after_launch (may be empty) runs on the host once every intersection
// kernel is enqueued, so that the host enqueues other work (on streams it has
// ordered itself) while the device intersects. reserve (may be empty) takes
// the memory that after_launch needs: it runs before memory is taken that the
// intersection can do without, and may run again or not at all. plan is one made by
// intersect_plan on s with the same cfg, n, nnz and deg, whose counts are on
// the host.
scan_status intersect_all(const IntersectConfig &cfg, int64_t n, int64_t nnz, const int64_t *off,
                          const int32_t *deg, const int32_t *adj, int kind, double *sims,
                          int32_t *counts, int device, hipStream_t s, IntersectStats *stats,
                          const std::function<scan_status()> &reserve = {},
                          const std::function<scan_status()> &after_launch = {},
                          const IntersectPlan *plan = nullptr);

// Approximate similarities (lsh.hip): k samples, and the random draws on
// the device (gauss n x k for SimHash, perm for MinHash).
struct LshSpec {
  int32_t samples = 0;
  const double *gauss = nullptr;
  const uint32_t *perm = nullptr;
};

// Weighted cosine of every edge into both CSR slots of sims (weighted.hip);
// events (may be null) before the square sums, before the products, after.
// The square sums are timed as the "small" part, the owner products as the
// "big" part (stats may be null).
// plan: the ownership plan (weighted_config's shapes) where weighted_planned
// says so, else null.
IntersectConfig weighted_config(const IntersectConfig &cfg);
bool weighted_planned(int64_t n, int64_t nnz);
scan_status weighted_similarity_all(int64_t n, int64_t nnz, const int64_t *off, const int32_t *deg,
                                    const int32_t *adj, const double *w, double *sims, DevArena &tmp,
                                    hipStream_t s, const IntersectStats *stats, const IntersectPlan *plan,
                                    int device, int32_t skip_deg = 0x7fffffff);
// Overwrites sims of the edges between two high-degree vertices with their
// SimHash (cosine kinds) or k-partition MinHash (Jaccard) estimates; w may
// be null (unweighted). spec's pointers are device pointers.
scan_status lsh_overwrite(const LshSpec &spec, int64_t n, int64_t nnz, const int64_t *off, const int32_t *adj,
                          const double *w, int kind, double *sims, DevArena &tmp, hipStream_t s);
// SCAN_EGRAPH unless every weight is finite (waits for the stream).
scan_status check_weights(const double *w, int64_t nnz, DevArena &tmp, hipStream_t s);

// What k_q_cores finds out about a query, for the kernels after it.
struct QueryState {
  int64_t base;  // co_off[mu] (0 if mu > dmax + 1)
  int64_t K;     // number of cores
};

// Per-query device workspace (one slot of a batch): one allocation of
// kSlotStateBytes + 5 n bytes.
constexpr size_t kSlotStateBytes = 64;
struct QuerySlot {
  QueryState *st = nullptr;
  int32_t *parent = nullptr;  // int32[n] union-find parents (read for cores only)
  uint8_t *flag = nullptr;    // uint8[n] marks of epochs up to `epoch` (query.hip)
  int32_t epoch = 0;          // the epoch of the slot's last query
  size_t bytes = 0;
};

// Descriptor of one query of a batch (query.hip).
struct QueryDesc {
  int32_t mu;
  int32_t epoch;
  double eps;
  QueryState *st;
  int32_t *parent;
  uint8_t *flag;
  int32_t *memb;  // nullptr: unused batch entry
  uint8_t *is_core;
};

}  // namespace scan

namespace scan {

struct DevAlloc {
  void *p;
  size_t bytes;
};

// Device buffers shared by the indexes of one batched build (each index is a
// view into them); freed when the last index referring to it is freed.
struct SharedArena {
  hipStream_t stream = nullptr;
  std::vector<DevAlloc> allocs;
  int64_t bytes = 0;
  // Pinned staging of the build's host tables, returned to the pool once
  // `done` (recorded at the end of the build) has completed.
  std::vector<PinnedBlock> pinned;
  hipEvent_t done = nullptr;
  ~SharedArena();
};

// SCAN_PROFILE events of a build (shared by the indexes of a batch): start,
// prepare, plan, intersect, neighbour order, core order, then the begin and
// end of the small-owner launches (6, 7) and of the large-owner launch (8,
// 9), which may run concurrently on two streams.
struct BuildProfileEvents {
  hipEvent_t ev[10] = {};
  int32_t window_bits = 0;
  int32_t intersect_launches = 0;
  // (light owners, big chunks, -, heavy owners), written by the host when it
  // reads the plan's counts back
  int32_t plan_counts[4] = {0, 0, 0, 0};
  ~BuildProfileEvents();
};

}  // namespace scan

struct scan_index {
  int64_t n = 0, nnz = 0, dmax = 0;
  int32_t kind = 0;
  uint32_t flags = 0;
  hipStream_t stream = nullptr;
  int device = 0;
  int64_t *off = nullptr;      // int64[n+1]
  int32_t *no_ids = nullptr;   // int32[nnz]
  double *no_sim = nullptr;    // double[nnz]
  int64_t *co_off = nullptr;   // int64[dmax+3]
  int32_t *co_ids = nullptr;   // int32[nnz]
  double *co_thr = nullptr;    // double[nnz]
  double *sims = nullptr;      // double[nnz] (SCAN_KEEP_SIMS)
  int32_t *counts = nullptr;   // int32[nnz]  (SCAN_KEEP_COUNTS)
  std::shared_ptr<scan::SharedArena> arena;        // owns the arrays above
  std::shared_ptr<scan::BuildProfileEvents> prof;  // SCAN_PROFILE only
  int64_t bytes = 0;                               // device bytes of this index's arrays
  int32_t hub_rows = 0, hub_cols = 0;              // of the build's hub product
  // Query workspace pool: a slot may be reused once its last use completed
  // (event) or when the new use is on the same stream. The slots of one call
  // share its event.
  struct Done {
    hipEvent_t ev = nullptr;
    ~Done() {
      if (ev) (void)hipEventDestroy(ev);
    }
  };
  struct PooledSlot {
    scan::QuerySlot slot;
    std::shared_ptr<Done> done;
    hipStream_t last_stream = nullptr;
    bool busy = false;
  };
  std::mutex pool_mu;
  std::vector<PooledSlot *> pool;
};

namespace scan {

void index_release(scan_index *ix);

scan_status build_index(const scan_csr *g, int32_t kind, uint32_t flags, hipStream_t stream,
                        const IntersectConfig &cfg, scan_index **out);
// weights: per-slot edge weights (kind SCAN_SIM_WEIGHTED_COSINE, one graph
// only), on the same side (host or device) as the graph. lsh (one graph only):
// approximate the edges between high-degree vertices; its draws are on the
// graph's side too.
scan_status build_index_batch(const scan_csr *gs, int32_t count, int32_t kind, uint32_t flags,
                              hipStream_t stream, const IntersectConfig &cfg, scan_index **outs,
                              const double *weights = nullptr, const LshSpec *lsh = nullptr);

// Runs `count` queries. mu/eps host arrays; memberships[i] / is_core[i] are
// device pointers (is_core may hold nulls). Slots are workspaces, one per
// query; nothing is allocated and nothing waited for.
scan_status run_queries(const scan_index *ix, int32_t count, const int32_t *mu, const double *eps,
                        int32_t *const *memberships, uint8_t *const *is_core, QuerySlot *const *slots,
                        hipStream_t s);

scan_status alloc_query_slot(const scan_index *ix, QuerySlot *slot, hipStream_t s);

// Enqueues the query kernels for `count` descriptors in device memory.
void launch_query_kernels(const scan_index *ix, QueryDesc *d, int32_t count, hipStream_t s);
// Modularity terms (quality.hip) of `count` clusterings (memb[i * n ...]):
// terms[3 i] += s_in, terms[3 i + 1] += sd2; dsum (int64[count * n]) must be
// zero on entry and is zero on return.
void zero64(int64_t *p, int64_t count, hipStream_t s);
void launch_modularity_terms(const scan_index *ix, const int32_t *memb, int32_t count, int64_t *dsum,
                             int64_t *terms, hipStream_t s);
// The same for the clusterings of a sweep, kModLanes at a time, with the
// sweep's workspace (plan_modularity_sweep, allocated from tmp).
struct ModularitySweep {
  int32_t *T = nullptr;       // labels of up to 32 clusterings, transposed
  int32_t *row_of = nullptr;  // the row holding every 128th slot
};
scan_status plan_modularity_sweep(const scan_index *ix, DevArena &tmp, hipStream_t s, ModularitySweep *p);
void launch_modularity_sweep(const scan_index *ix, const ModularitySweep &p, const int32_t *memb, int32_t count,
                             int64_t *dsum, int64_t *terms, hipStream_t s);
double modularity_value(int64_t s_in, int64_t sd2, int64_t nnz);

// Hub / outlier roles of the unclustered vertices of one query's memberships.
void launch_roles(const scan_index *ix, const int32_t *memb, uint8_t *roles, hipStream_t s);
// One query whose workspace is the library's file-scope scratch array (no
// allocation); memberships / is_core are device pointers.
scan_status query_noalloc(const scan_index *ix, int32_t mu, double eps, int32_t *memberships, uint8_t *is_core,
                          hipStream_t s);
// The descriptor of the slot's next query, which runs on s (memb null: an
// unused entry).
QueryDesc make_query_desc(const scan_index *ix, int32_t mu, double eps, QuerySlot &slot, int32_t *memb,
                          uint8_t *is_core, hipStream_t s);
void free_query_slot(QuerySlot *slot, hipStream_t s);

IntersectConfig default_config();

scan_status similarity_values(int32_t kind, int64_t count, const int64_t *c, const int64_t *a_u,
                              const int64_t *a_v, double *out);

}  // namespace scan
