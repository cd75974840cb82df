// (mu, eps) clustering queries over the index (Section 4.2, Algorithms 3-5;
// connectivity by union-find as in Section 6.2; border vertices by the
// deterministic rule of Section 7.3.4).
//
// Per query, six grid-stride kernels over a batch (blockIdx.y = query). A
// byte per vertex (the slot's state array) marks cores and candidate borders
// of the slot's current epoch, so that no pass clears it between queries:
//   a7  k_q_cores   K = length of the eps-prefix of CO[mu] (64-way search);
//                   for the K cores: core mark, and parent = the smallest of
//                   the core and the core neighbours among the first
//                   kHookSpan entries of its eps-prefix
//   a9  k_q_jump    parent[u] = root of u for every core
//       k_q_hook, k_q_jump  the same once more for the trees' roots
//   a8+a9 k_q_union for each core u, scan the eps-prefix of NO[u]; a core
//                   neighbour whose root differs is united with u (larger
//                   root hooked under the smaller, so every root is its
//                   component's smallest id); a non-core neighbour is marked
//                   as a candidate border
//   a10 k_q_output  memberships: cores -> root; marked non-cores -> root of
//                   the first core in their own NO row (NO is sorted by sim
//                   desc, id asc, so that is the most similar eps-similar core,
//                   ties to the lower id); others -1.
// A vertex w is a core iff deg(w) >= mu-1 and NO_SIM[off[w] + mu - 2] >= eps,
// which is exactly membership in the eps-prefix of CO[mu] (the CO entry of w
// for mu carries that same threshold value).
//
// What bounds a query is the chain of dependent memory reads, not its bytes.
// Hooking every core, then every tree, before the exhaustive pass leaves that
// pass comparing two cached roots per neighbour instead of walking and
// swapping pointers across the chip (atomic accesses bypass the L2s). 32
// mixed queries of a 1M-vertex R-MAT index: k_q_union 1225 -> 386 us with
// 28 + 40 + 25 us of hooks and jumps before it; without the second round of
// hooks 670 us. Small indexes take one kernel (k_q_small).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include <cmath>
#include <mutex>
#include <vector>

#include "index.h"

namespace scan {

constexpr uint8_t kRoleClustered = SCAN_ROLE_CLUSTERED, kRoleHub = SCAN_ROLE_HUB, kRoleOutlier = SCAN_ROLE_OUTLIER;

struct IndexView {
  int64_t n, dmax;
  const int64_t *off;
  const int32_t *no_ids;
  const double *no_sim;
  const int64_t *co_off;
  const int32_t *co_ids;
  const double *co_thr;
};

// State bytes of a query's epoch e (1..kMaxEpoch).
constexpr int32_t kMaxEpoch = 127;
__device__ __forceinline__ uint8_t core_mark(int32_t e) { return (uint8_t)(2 * e + 1); }
__device__ __forceinline__ uint8_t border_mark(int32_t e) { return (uint8_t)(2 * e); }

// Length of the eps-prefix of CO[mu] (thresholds are sorted descending): a
// 64-way search by one wavefront, every lane sampling one position (4 rounds
// at a million entries, where halving takes 20 dependent reads).
__device__ __forceinline__ void core_prefix(const IndexView &ix, int32_t mu, double eps, int64_t &base,
                                            int64_t &K) {
  K = 0;
  base = 0;
  if ((int64_t)mu > ix.dmax + 1) return;
  const int lane = threadIdx.x & (kWave - 1);
  base = ix.co_off[mu];
  int64_t lo = 0, hi = ix.co_off[mu + 1] - base;
  while (hi - lo > kWave) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const int64_t p = lo + (int64_t)lane * step;
    const int c = __popcll(__ballot(p < hi && ix.co_thr[base + p] >= eps));  // a prefix of the lanes
    if (c == 0) return;  // only in the first round: the first threshold is below eps
    hi = min(hi, lo + (int64_t)c * step);
    lo += (int64_t)(c - 1) * step;  // this position is in the prefix
  }
  const int64_t p = lo + lane;
  K = lo + __popcll(__ballot(p < hi && ix.co_thr[base + p] >= eps));
}

// parent[] entries of the query's cores form a forest (hooks go from a root
// to a smaller root, halving moves a pointer to an ancestor); the step cap
// only guards against a corrupt index.
__device__ __forceinline__ int32_t uf_find(int32_t *parent, int32_t x) {
  int32_t cur = x;
  for (int guard = 0; guard < (1 << 26); ++guard) {
    int32_t nxt = __hip_atomic_load(&parent[cur], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (nxt == cur) return cur;
    int32_t nn = __hip_atomic_load(&parent[nxt], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (nn != nxt)  // path halving
      __hip_atomic_store(&parent[cur], nn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    cur = nxt;
  }
  return cur;
}

// The root of x without writing: k_q_jump needs every core's final pointer to
// be its root, and a halving step of another thread, based on pointers read
// before this thread stored the root, could overwrite it with an ancestor.
// Cached reads: an older pointer read here is an ancestor all the same, and
// the roots themselves do not change in the kernels that call this.
__device__ __forceinline__ int32_t cached(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ int32_t uf_root(const int32_t *parent, int32_t x) {
  int32_t cur = x;
  for (int guard = 0; guard < (1 << 26); ++guard) {
    const int32_t nxt = cached(&parent[cur]);
    if (nxt == cur) return cur;
    cur = nxt;
  }
  return cur;
}

__device__ __forceinline__ void uf_union(int32_t *parent, int32_t a, int32_t b) {
  for (;;) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a < b) {
      int32_t t = a;
      a = b;
      b = t;
    }
    // hook root a (larger) under b (smaller)
    if (atomicCAS(&parent[a], a, b) == a) return;
  }
}

// Where a kernel's descriptors come from: its arguments (the host's direct
// launches: nothing is copied to the device first) or device memory (batches
// replayed from a captured graph). A descriptor with memb == nullptr is an
// unused batch entry: every kernel skips it.
constexpr int kArgDescs = 32;
struct DescsInArgs {
  QueryDesc d[kArgDescs];
  __device__ __forceinline__ const QueryDesc &operator[](int i) const { return d[i]; }
};
struct DescsInMemory {
  const QueryDesc *d;
  __device__ __forceinline__ const QueryDesc &operator[](int i) const { return d[i]; }
};

// The smallest value of each row of 16 lanes, in all of them (rotations in the
// register path; a row's lanes are active together).
__device__ __forceinline__ int32_t row_min(int32_t v) {
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0xf, false));  // row_ror:8
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x124, 0xf, 0xf, false));  // row_ror:4
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x122, 0xf, 0xf, false));  // row_ror:2
  return min(v, __builtin_amdgcn_update_dpp(v, v, 0x121, 0xf, 0xf, false));  // row_ror:1
}

constexpr int kQThreads = 1024;
constexpr int kHookSpan = 16;  // lanes per core, and entries looked at, in k_q_cores

template <class Descs>
__global__ __launch_bounds__(kQThreads) void k_q_cores(IndexView ix, Descs qd) {
  const QueryDesc &q = qd[blockIdx.y];
  if (!q.memb) return;
  __shared__ int64_t sh[2];
  const int32_t mu = q.mu;
  const double eps = q.eps;
  if (threadIdx.x < kWave) {  // every block finds K itself (same addresses: cache hits)
    int64_t base, K;
    core_prefix(ix, mu, eps, base, K);
    if (threadIdx.x == 0) {
      sh[0] = base;
      sh[1] = K;
      if (blockIdx.x == 0) {
        q.st->K = K;
        q.st->base = base;
      }
    }
  }
  __syncthreads();
  const int64_t base = sh[0], K = sh[1];
  int32_t *parent = q.parent;
  uint8_t *flag = q.flag;
  const uint8_t mark = core_mark(q.epoch);
  const int pos = threadIdx.x % kHookSpan;
  // kHookSpan lanes per core. A neighbour's own threshold says whether it is
  // a core: its mark may not be written yet.
  for (int64_t i = (blockIdx.x * (int64_t)kQThreads + threadIdx.x) / kHookSpan; i < K;
       i += (int64_t)gridDim.x * (kQThreads / kHookSpan)) {
    const int32_t u = ix.co_ids[base + i];
    const int64_t k = ix.off[u] + pos;
    int32_t m = u;
    if (k < ix.off[u + 1] && ix.no_sim[k] >= eps) {
      const int32_t x = ix.no_ids[k];
      const int64_t t = ix.off[x] + mu - 2;
      if (x < u && t < ix.off[x + 1] && ix.no_sim[t] >= eps) m = x;
    }
    m = row_min(m);
    if (pos == 0) {
      parent[u] = m;
      flag[u] = mark;
    }
  }
}

template <class Descs>
__global__ __launch_bounds__(256) void k_q_jump(IndexView ix, Descs qd) {
  const QueryDesc &q = qd[blockIdx.y];
  if (!q.memb) return;
  const int64_t K = q.st->K, base = q.st->base;
  int32_t *parent = q.parent;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = ix.co_ids[base + i];
    __hip_atomic_store(&parent[u], uf_root(parent, u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A second round of hooks, of whole trees: every root met among the first
// kHookSpan entries of u's eps-prefix, and u's own, goes under the smallest
// of them (no value is read back). A hook may replace another; the exhaustive
// pass unites what that leaves apart. Pointers only ever go to smaller ids of
// the same component, so any mix of hooks is a forest.
template <class Descs>
__global__ __launch_bounds__(kQThreads) void k_q_hook(IndexView ix, Descs qd) {
  const QueryDesc &q = qd[blockIdx.y];
  if (!q.memb) return;
  const int64_t K = q.st->K, base = q.st->base;
  const double eps = q.eps;
  int32_t *parent = q.parent;
  const uint8_t *flag = q.flag;
  const uint8_t core = core_mark(q.epoch);
  const int pos = threadIdx.x % kHookSpan;
  for (int64_t i = (blockIdx.x * (int64_t)kQThreads + threadIdx.x) / kHookSpan; i < K;
       i += (int64_t)gridDim.x * (kQThreads / kHookSpan)) {
    const int32_t u = ix.co_ids[base + i];
    const int64_t k = ix.off[u] + pos;
    const int32_t ru = cached(&parent[u]);
    int32_t rx = ru;
    if (k < ix.off[u + 1] && ix.no_sim[k] >= eps) {
      const int32_t x = ix.no_ids[k];
      if (flag[x] == core) rx = cached(&parent[x]);
    }
    int32_t m = min(ru, rx);
    m = row_min(m);
    // (a read first: most of a tree's cores bring nothing smaller, and
    // swaps on one root queue up where reads of it do not)
    auto hook = [&](int32_t r) {
      if (__hip_atomic_load(&parent[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > m) atomicMin(&parent[r], m);
    };
    if (rx != m && rx != ru) hook(rx);
    if (pos == 0 && ru != m) hook(ru);
  }
}

// Rows by length: a group of kRowGroup lanes takes a core's first kRowShort
// entries; rows that go on are finished by a wavefront each up to kRowLong
// entries, and what is left of the longest by the whole workgroup, so that no
// hub row (tens of thousands of dependent 64-entry steps for one wavefront)
// holds the kernel. Every step's loads are issued together.
constexpr int kRowGroup = 16, kRowSteps = 4;
constexpr int kRowShort = 64;     // entries a group looks at
constexpr int kRowLong = 2048;    // entries a wavefront looks at

template <class Descs>
__global__ __launch_bounds__(kQThreads) void k_q_union(IndexView ix, Descs qd) {
  const QueryDesc &q = qd[blockIdx.y];
  if (!q.memb) return;
  const int64_t K = q.st->K, base = q.st->base;
  if (K == 0) return;
  constexpr int kCores = kQThreads / kRowGroup;  // cores per round
  __shared__ int32_t mid[kCores], far[kCores];
  __shared__ int32_t nmid, nfar;
  const double eps = q.eps;
  int32_t *parent = q.parent;
  uint8_t *flag = q.flag;
  const uint8_t core = core_mark(q.epoch), border = border_mark(q.epoch);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  // kRowSteps entries of core u's row, from k at `stride`: false once the
  // prefix (or the row) has ended for this lane. The marks and parents of all
  // of them are requested together (a parent is used only where the mark says
  // core). Parents are read as cached values: a stale one is an older
  // ancestor, so equal values mean one component.
  auto steps = [&](int32_t u, int32_t ru, int64_t k, int64_t e, int64_t stride) -> bool {
    double s[kRowSteps];
    int32_t x[kRowSteps], rx[kRowSteps];
    uint8_t f[kRowSteps];
#pragma unroll
    for (int j = 0; j < kRowSteps; ++j) {
      const int64_t p = k + j * stride < e ? k + j * stride : e - 1;
      s[j] = ix.no_sim[p];
      x[j] = ix.no_ids[p];
    }
    bool in[kRowSteps];
#pragma unroll
    for (int j = 0; j < kRowSteps; ++j) {
      in[j] = k + j * stride < e && s[j] >= eps;
      f[j] = 0;
      rx[j] = ru;
      if (in[j]) {
        f[j] = flag[x[j]];
        if (x[j] < u) rx[j] = cached(&parent[x[j]]);
      }
    }
#pragma unroll
    for (int j = 0; j < kRowSteps; ++j) {
      if (!in[j]) continue;
      if (f[j] != core) {
        if (f[j] != border) flag[x[j]] = border;
      } else if (rx[j] != ru) {
        uf_union(parent, ru, rx[j]);
      }
    }
    return in[kRowSteps - 1];
  };
  for (int64_t i0 = (int64_t)blockIdx.x * kCores; i0 < K; i0 += (int64_t)gridDim.x * kCores) {
    __syncthreads();  // the previous round's lists are read
    if (threadIdx.x == 0) nmid = nfar = 0;
    __syncthreads();
    const int64_t i = i0 + threadIdx.x / kRowGroup;
    if (i < K) {
      const int32_t u = ix.co_ids[base + i];
      const int pos = threadIdx.x % kRowGroup;
      const int64_t e = ix.off[u + 1];
      static_assert(kRowGroup * kRowSteps == kRowShort, "one batch of steps per group");
      const int32_t ru = cached(&parent[u]);
      const bool in = steps(u, ru, ix.off[u] + pos, e, kRowGroup);
      // the group's last lane saw the last entry: past it there may be more
      if (pos == kRowGroup - 1 && in) mid[atomicAdd(&nmid, 1)] = u;
    }
    __syncthreads();
    for (int32_t r = wave; r < nmid; r += kQThreads / kWave) {
      const int32_t u = mid[r];
      const int64_t b = ix.off[u], e = ix.off[u + 1];
      const int32_t ru = cached(&parent[u]);
      bool more = b + kRowShort < e;
      for (int64_t k0 = b + kRowShort; more && k0 < b + kRowLong; k0 += kRowSteps * kWave)
        more = __all(steps(u, ru, k0 + lane, e, kWave));
      if (more && lane == 0) far[atomicAdd(&nfar, 1)] = u;
    }
    __syncthreads();
    // the steps above end kRowShort past a multiple of kRowSteps * kWave
    constexpr int64_t kFarStart = kRowShort + (kRowLong - kRowShort + kRowSteps * kWave - 1) / (kRowSteps * kWave) *
                                                  (kRowSteps * kWave);
    for (int32_t r = 0; r < nfar; ++r) {
      const int32_t u = far[r];
      const int64_t e = ix.off[u + 1];
      const int32_t ru = cached(&parent[u]);
      bool more = true;
      for (int64_t k0 = ix.off[u] + kFarStart; more; k0 += kRowSteps * kQThreads)
        more = __syncthreads_and(steps(u, ru, k0 + threadIdx.x, e, kQThreads));
    }
  }
}

template <class Descs>
__global__ __launch_bounds__(256) void k_q_output(IndexView ix, Descs qd) {
  const QueryDesc &q = qd[blockIdx.y];
  if (!q.memb) return;
  const int64_t K = q.st->K;
  const double eps = q.eps;
  const int32_t *parent = q.parent;
  const uint8_t *flag = q.flag;
  int32_t *memb = q.memb;
  uint8_t *is_core = q.is_core;
  const uint8_t core = core_mark(q.epoch), border = border_mark(q.epoch);
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < ix.n; v += (int64_t)gridDim.x * blockDim.x) {
    const uint8_t st = K > 0 ? flag[v] : 0;
    int32_t m = -1;
    if (st == core) {
      m = uf_root(parent, v);
    } else if (st == border) {
      for (int64_t k = ix.off[v], e = ix.off[v + 1]; k < e && ix.no_sim[k] >= eps; ++k) {
        const int32_t x = ix.no_ids[k];
        if (flag[x] == core) {
          m = uf_root(parent, x);
          break;
        }
      }
    }
    memb[v] = m;
    if (is_core) is_core[v] = st == core ? 1 : 0;
  }
}

// Small indexes: a whole query in one workgroup, union-find and marks in LDS.
// The dependent launches above are then most of a query's time; kSmallN is
// what the LDS holds with kRowGroup edges per core. Its time goes with the
// slots that it reads, up to kSmallNnz of them (two queries, with every vertex
// a core and with few or none, this kernel and the launches in us: 2,048
// vertices of degree 8 42 and 51, 40 and 52; 16 78 and 61, 32 and 53; 64 112
// and 62, 17 and 29; the cores are few in most queries). Rows past kSmallRow
// entries are read by a wavefront each, most of them one after the other, so
// with such rows half of the slots are the limit (a clique of 256, 65,280
// slots, 47 and 38; of 362, 130,682 slots, 75 and 42; 2,048 vertices and 30
// hubs joined to all, 121,950 slots, 146 and 56).
constexpr int kSmallN = 2048;
constexpr int64_t kSmallNnz = 64 * kSmallN;
constexpr int64_t kSmallRow = 256, kSmallRowNnz = 32 * kSmallN;
constexpr int kSmallAhead = 4;  // cores that a lane group takes at once

__device__ __forceinline__ int32_t lds_find(int32_t *parent, int32_t x) {
  for (;;) {
    const int32_t p = __hip_atomic_load(&parent[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (p == x) return x;
    const int32_t g = __hip_atomic_load(&parent[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (g != p) __hip_atomic_store(&parent[x], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);  // path halving
    x = g;
  }
}
__device__ __forceinline__ void lds_union(int32_t *parent, int32_t a, int32_t b) {
  for (;;) {
    a = lds_find(parent, a);
    b = lds_find(parent, b);
    if (a == b) return;
    if (a < b) {
      const int32_t t = a;
      a = b;
      b = t;
    }
    if (atomicCAS(&parent[a], a, b) == a) return;
  }
}

template <class Descs>
__global__ __launch_bounds__(kQThreads) void k_q_small(IndexView ix, Descs qd) {
  const QueryDesc &q = qd[blockIdx.y];
  if (!q.memb) return;
  __shared__ int32_t off[kSmallN + 1], parent[kSmallN], cores[kSmallN];
  __shared__ uint8_t mark[kSmallN];  // 2 core, 1 candidate border
  __shared__ uint32_t edges[kSmallN * kRowGroup];
  __shared__ uint16_t longer[kSmallN];
  __shared__ int32_t nedges, nlonger;
  __shared__ int64_t sh[2];
  const int32_t n = (int32_t)ix.n;  // <= kSmallN
  const double eps = q.eps;
  for (int v = threadIdx.x; v <= n; v += kQThreads) {
    off[v] = (int32_t)ix.off[v];
    if (v < n) mark[v] = 0;
  }
  if (threadIdx.x < kWave) {
    int64_t base, K;
    core_prefix(ix, q.mu, eps, base, K);
    if (threadIdx.x == 0) {
      sh[0] = base;
      sh[1] = K;
      nedges = nlonger = 0;
    }
  }
  __syncthreads();
  const int64_t base = sh[0];
  const int32_t K = (int32_t)sh[1];
  for (int i = threadIdx.x; i < K; i += kQThreads) {
    const int32_t u = ix.co_ids[base + i];
    cores[i] = u;
    parent[u] = u;
    mark[u] = 2;
  }
  __syncthreads();
  // The first kRowGroup entries of every core's row, one lane each; those that
  // are smaller core neighbours go to a list of edges in LDS (the larger end's
  // row holds every edge once). A core past the last one stands for the last.
  constexpr int kGroups = kQThreads / kRowGroup;
  const int grp = threadIdx.x / kRowGroup, pos = threadIdx.x % kRowGroup, lane = threadIdx.x & (kWave - 1);
  const int32_t last = K - 1, rounds = (K + kSmallAhead * kGroups - 1) / (kSmallAhead * kGroups);
  for (int r = 0; r < rounds; ++r) {
    const int i0 = grp + r * kSmallAhead * kGroups;
    int32_t u[kSmallAhead], y[kSmallAhead];
    double s[kSmallAhead];
    bool in[kSmallAhead];
#pragma unroll
    for (int j = 0; j < kSmallAhead; ++j) {
      u[j] = cores[min(i0 + j * kGroups, last)];
      const int32_t k = off[u[j]] + pos, e = off[u[j] + 1];
      in[j] = k < e && i0 + j * kGroups < K;
      s[j] = ix.no_sim[min(k, e - 1)];
      y[j] = ix.no_ids[min(k, e - 1)];
    }
#pragma unroll
    for (int j = 0; j < kSmallAhead; ++j) {
      in[j] = in[j] && s[j] >= eps;
      const bool core = mark[y[j]] == 2;
      if (in[j] && !core) mark[y[j]] = 1;
      const bool edge = in[j] && core && y[j] < u[j];
      const uint64_t m = __ballot(edge);
      int32_t at = 0;
      if (lane == 0 && m) at = atomicAdd(&nedges, __popcll(m));
      at = __builtin_amdgcn_readfirstlane(at);
      if (edge) edges[at + __popcll(m & ((1ull << lane) - 1))] = (uint32_t)u[j] << 16 | (uint32_t)y[j];
      // the prefix may go on past these entries
      if (pos == kRowGroup - 1 && in[j]) longer[atomicAdd(&nlonger, 1)] = (uint16_t)u[j];
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nedges; i += kQThreads) lds_union(parent, edges[i] >> 16, edges[i] & 0xffffu);
  for (int i = threadIdx.x / kWave; i < nlonger; i += kQThreads / kWave) {  // a wavefront per longer row
    const int32_t u = longer[i];
    for (int32_t k = off[u] + kRowGroup + lane; k < off[u + 1] && ix.no_sim[k] >= eps;
         k += kWave) {
      const int32_t y = ix.no_ids[k];
      if (mark[y] != 2) mark[y] = 1;
      else if (cached(&parent[y]) != cached(&parent[u])) lds_union(parent, u, y);
    }
  }
  __syncthreads();
  for (int v = threadIdx.x; v < n; v += kQThreads) {
    int32_t m = -1;
    if (mark[v] == 2) {
      m = lds_find(parent, v);
    } else if (mark[v] == 1) {
      for (int32_t k = off[v]; k < off[v + 1] && ix.no_sim[k] >= eps; ++k) {
        const int32_t x = ix.no_ids[k];
        if (mark[x] == 2) {
          m = lds_find(parent, x);
          break;
        }
      }
    }
    q.memb[v] = m;
    if (q.is_core) q.is_core[v] = mark[v] == 2 ? 1 : 0;
  }
}

template <class Descs>
static void launch_queries(const scan_index *ix, const Descs &d, int32_t count, hipStream_t s) {
  IndexView v{ix->n, ix->dmax, ix->off, ix->no_ids, ix->no_sim, ix->co_off, ix->co_ids, ix->co_thr};
  if (ix->n <= kSmallN && ix->nnz <= (ix->dmax <= kSmallRow ? kSmallNnz : kSmallRowNnz)) {
    k_q_small<<<dim3(1, count), kQThreads, 0, s>>>(v, d);
    return;
  }
  const int64_t n = ix->n;
  // Blocks per query: enough for one heavy query to fill the chip, few
  // enough that the many light ones of a batch (no core at all) cost nothing.
  const dim3 gw(grid_for(n, kQThreads / kRowGroup, 256), count);
  const dim3 gt(grid_for(n, 256, count > 8 ? 512 : 2048), count);
  k_q_cores<<<gw, kQThreads, 0, s>>>(v, d);
  const dim3 gj(grid_for(n, 256, 256), count);
  k_q_jump<<<gj, 256, 0, s>>>(v, d);
  k_q_hook<<<gw, kQThreads, 0, s>>>(v, d);
  k_q_jump<<<gj, 256, 0, s>>>(v, d);
  k_q_union<<<gw, kQThreads, 0, s>>>(v, d);
  k_q_output<<<gt, 256, 0, s>>>(v, d);
}

void launch_query_kernels(const scan_index *ix, QueryDesc *d, int32_t count, hipStream_t s) {
  launch_queries(ix, DescsInMemory{d}, count, s);
}

// Hubs and outliers (Section 4.3): every unclustered vertex maps its
// neighbours to their clusters and checks whether two of them differ (the NO
// row holds the open neighbourhood). A wavefront takes kWave / kRoleGroup
// consecutive vertices, one per group of kRoleGroup lanes; a group scans its
// vertex's row kRoleGroup ids per step, reducing the step's smallest and
// largest cluster label within the group (lane exchanges stay inside the
// group, whose lanes are active together), and stops at a second cluster.
// Rows longer than kRoleGroupMax are scanned afterwards by the whole
// wavefront, kRoleSteps * 64 ids per step. A vertex in a cluster gets role 0
// without reading its row.
constexpr int kRoleGroup = 8;
constexpr int64_t kRoleGroupMax = 512;
constexpr int kRoleSteps = 8;

__device__ __forceinline__ int32_t group_min(int32_t x) {
#pragma unroll
  for (int m = kRoleGroup / 2; m > 0; m >>= 1) x = min(x, __shfl_xor(x, m, kWave));
  return x;
}
__device__ __forceinline__ int32_t group_max(int32_t x) {
#pragma unroll
  for (int m = kRoleGroup / 2; m > 0; m >>= 1) x = max(x, __shfl_xor(x, m, kWave));
  return x;
}

__global__ __launch_bounds__(256) void k_q_roles(IndexView ix, const int32_t *memb, uint8_t *roles) {
  constexpr int kPerWave = kWave / kRoleGroup;
  const int lane = threadIdx.x & (kWave - 1), pos = lane % kRoleGroup;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  for (int64_t v0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave * kPerWave; v0 < ix.n;
       v0 += nw * kPerWave) {
    const int64_t v = v0 + lane / kRoleGroup;
    int64_t b = 0, e = 0;
    bool unclustered = false;
    if (v < ix.n) {
      unclustered = memb[v] < 0;
      b = ix.off[v];
      e = ix.off[v + 1];
    }
    const bool group_row = unclustered && e - b <= kRoleGroupMax;
    uint8_t role = kRoleClustered;
    if (group_row) {  // the same for every lane of the group
      int32_t first = -1;
      bool hub = false;
      for (int64_t k0 = b; k0 < e && !hub; k0 += kRoleGroup) {
        const int64_t k = k0 + pos;
        const int32_t lab = k < e ? memb[ix.no_ids[k]] : -1;
        const int32_t lo = group_min(lab >= 0 ? lab : INT_MAX);
        const int32_t hi = group_max(lab);
        if (lo != INT_MAX) {
          if (first < 0) first = lo;
          hub = lo != first || hi != first;
        }
      }
      role = hub ? kRoleHub : kRoleOutlier;
    }
    // long unclustered rows: one at a time by the whole wavefront
    uint64_t longs = __ballot(unclustered && !group_row && pos == 0);
    while (longs) {
      const int src = __ffsll((unsigned long long)longs) - 1;
      longs &= longs - 1;
      const int64_t rb = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)b, src) |
                         ((int64_t)__builtin_amdgcn_readlane((int32_t)(b >> 32), src) << 32);
      const int64_t re = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)e, src) |
                         ((int64_t)__builtin_amdgcn_readlane((int32_t)(e >> 32), src) << 32);
      // kRoleSteps * kWave ids per iteration, all of their loads issued
      // before the labels are reduced (smallest and largest over the wave)
      int32_t first = -1;
      bool hub = false;
      for (int64_t k0 = rb; k0 < re && !hub; k0 += kRoleSteps * kWave) {  // uniform bounds and exit
        int32_t w[kRoleSteps];
#pragma unroll
        for (int j = 0; j < kRoleSteps; ++j) {
          const int64_t k = k0 + j * kWave + lane;
          w[j] = k < re ? ix.no_ids[k] : -1;
        }
        int32_t lo = INT_MAX, hi = -1;
#pragma unroll
        for (int j = 0; j < kRoleSteps; ++j) {
          const int32_t lab = w[j] >= 0 ? memb[w[j]] : -1;
          if (lab >= 0) {
            lo = min(lo, lab);
            hi = max(hi, lab);
          }
        }
#pragma unroll
        for (int m = kWave / 2; m > 0; m >>= 1) {
          lo = min(lo, __shfl_xor(lo, m, kWave));
          hi = max(hi, __shfl_xor(hi, m, kWave));
        }
        if (lo != INT_MAX) {
          if (first < 0) first = lo;
          hub = lo != first || hi != first;
        }
      }
      if (lane / kRoleGroup == src / kRoleGroup) role = hub ? kRoleHub : kRoleOutlier;
    }
    if (v < ix.n && pos == 0) roles[v] = role;
  }
}

void launch_roles(const scan_index *ix, const int32_t *memb, uint8_t *roles, hipStream_t s) {
  IndexView v{ix->n, ix->dmax, ix->off, ix->no_ids, ix->no_sim, ix->co_off, ix->co_ids, ix->co_thr};
  k_q_roles<<<grid_for((ix->n + kWave / kRoleGroup - 1) / (kWave / kRoleGroup) * kWave, 256), 256, 0, s>>>(
      v, memb, roles);
}

// ---------------------------------------------------------------------------
// Allocation-free query: the slot workspace lives in a file-scope device
// array instead of allocated memory. Layout: the query's state (K, base),
// then parent int32[n], then the state bytes uint8[n].

constexpr size_t kNoAllocStateBytes = 256;
constexpr int64_t kNoAllocMaxN = (int64_t)1 << 23;
constexpr size_t kNoAllocScratchBytes = kNoAllocStateBytes + (size_t)kNoAllocMaxN * 5;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

// The device address of `scratch` on each device, taken once per device with
// that device current (the host-side name of the array is not a device
// address).
static std::mutex g_scratch_mu;
static std::vector<void *> g_scratch_ptr;

static scan_status scratch_address(int device, unsigned char **out) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch_ptr.size() <= device) g_scratch_ptr.resize(device + 1, nullptr);
  if (!g_scratch_ptr[device]) {
    int cur = 0;
    SCAN_HIP_TRY(hipGetDevice(&cur));
    if (cur != device) SCAN_HIP_TRY(hipSetDevice(device));
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p)
      return fail(SCAN_EDEVICE, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    g_scratch_ptr[device] = p;
  }
  *out = (unsigned char *)g_scratch_ptr[device];
  return SCAN_OK;
}

// Clears a slot's state bytes (no memset node, so that it may be captured).
__global__ void k_q_clear(uint8_t *flag, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    flag[i] = 0;
}

scan_status query_noalloc(const scan_index *ix, int32_t mu, double eps, int32_t *memberships, uint8_t *is_core,
                          hipStream_t s) {
  if (ix->n > kNoAllocMaxN)
    return fail(SCAN_EINVAL, "scan_query_noalloc takes indexes of at most %lld vertices (this one has %lld)",
                (long long)kNoAllocMaxN, (long long)ix->n);
  unsigned char *base;
  SCAN_TRY(scratch_address(ix->device, &base));
  if (ix->n == 0) return SCAN_OK;
  int32_t *parent = (int32_t *)(base + kNoAllocStateBytes);
  uint8_t *flag = (uint8_t *)(parent + ix->n);
  k_q_clear<<<grid_for(ix->n, 256, 2048), 256, 0, s>>>(flag, ix->n);
  DescsInArgs d{};
  d.d[0] = QueryDesc{mu, 1, eps, (QueryState *)base, parent, flag, memberships, is_core};
  launch_queries(ix, d, 1, s);
  SCAN_HIP_TRY(hipGetLastError());
  return SCAN_OK;
}

QueryDesc make_query_desc(const scan_index *ix, int32_t mu, double eps, QuerySlot &slot, int32_t *memb,
                          uint8_t *is_core, hipStream_t s) {
  if (memb && slot.epoch == kMaxEpoch) {  // every mark value has been used: start over
    k_q_clear<<<grid_for(ix->n, 256, 2048), 256, 0, s>>>(slot.flag, ix->n);
    slot.epoch = 0;
  }
  if (memb) ++slot.epoch;
  return QueryDesc{mu, slot.epoch, eps, slot.st, slot.parent, slot.flag, memb, is_core};
}

// One allocation: the query's state, the parents, the state bytes.
scan_status alloc_query_slot(const scan_index *ix, QuerySlot *slot, hipStream_t s) {
  const size_t n = (size_t)(ix->n > 0 ? ix->n : 1);
  slot->bytes = kSlotStateBytes + n * 5;
  unsigned char *p = (unsigned char *)dev_alloc(slot->bytes, s);
  if (!p) return fail(SCAN_ENOMEM, "query workspace allocation failed");
  slot->st = (QueryState *)p;
  slot->parent = (int32_t *)(p + kSlotStateBytes);
  slot->flag = (uint8_t *)(slot->parent + n);
  slot->epoch = 0;
  hipError_t e = hipMemsetAsync(slot->flag, 0, n, s);
  if (e != hipSuccess) {
    free_query_slot(slot, s);
    return fail(SCAN_EDEVICE, "hipMemsetAsync: %s", hipGetErrorString(e));
  }
  return SCAN_OK;
}

void free_query_slot(QuerySlot *slot, hipStream_t s) {
  if (slot->st) dev_free(slot->st, slot->bytes, s);
  *slot = QuerySlot{};
}

scan_status run_queries(const scan_index *ix, int32_t count, const int32_t *mu, const double *eps,
                        int32_t *const *memberships, uint8_t *const *is_core, QuerySlot *const *slots,
                        hipStream_t s) {
  for (int32_t i0 = 0; i0 < count; i0 += kArgDescs) {
    const int32_t c = std::min<int32_t>(kArgDescs, count - i0);
    DescsInArgs d{};
    for (int32_t i = 0; i < c; ++i)
      d.d[i] = make_query_desc(ix, mu[i0 + i], eps[i0 + i], *slots[i0 + i], memberships[i0 + i],
                               is_core ? is_core[i0 + i] : nullptr, s);
    launch_queries(ix, d, c, s);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SCAN_EDEVICE, "query launch: %s", hipGetErrorString(e));
  return SCAN_OK;
}

}  // namespace scan
