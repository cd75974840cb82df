// Per-edge intersection |N(u) ∩ N(h)| and similarity (Algorithm 1 with its
// min-side rule), fused: the count c = t + 2 over closed neighbourhoods and
// the FP64 similarity are written into both CSR slots of the edge.
//
// Every undirected edge {u, h} is owned by its endpoint that is larger in the
// order (degree, id); the owner's row is the lookup structure and every lower
// neighbour u streams its own, shorter row through it, so an edge costs
// min-side work and no global atomics.
//
//   k_plan          per vertex, by degree: 1..small_max go to the lists of
//                   small vertices, larger ones are cut into chunks of `spc`
//                   row slots (block-scanned appends, one reservation per tile).
//   k_small_owner   one workgroup per small vertex: its row goes into an LDS
//                   hash table, and groups of 8 or 16 lanes stream a lower
//                   neighbour's row each through it.
//   k_big_owner     persistent workgroups (1024 threads) holding a bitmap of an
//                   id window (2^wbits ids) in LDS: the owner's ids in the
//                   window are set, every lower neighbour's ids in the window
//                   are tested with one LDS read each, and the bitmap is
//                   cleared as a whole for the next owner or window. Chunks
//                   are claimed from a global counter, short ranges four at a
//                   time and pieces of long ones by wavefronts from LDS
//                   counters.
//   k_window_table  (ids spanning several windows) the first position of
//                   every window in every row, so that chunks read each lower
//                   neighbour's range in a window instead of searching it.
//   k_id_flags, k_rename  (several windows) ids numbered without the isolated
//                   vertices, so that they span fewer windows.
//
// Where it pays, the common neighbours of two high-degree vertices come from a
// matrix product (hubs.hip) and k_big_owner streams what is left of their rows.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstddef>

#include "index.h"
#include "rows.h"

namespace scan {

__device__ __forceinline__ bool is_lower(int32_t u, int32_t du, int32_t h, int32_t dh) {
  return du < dh || (du == dh && u < h);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ uint64_t lanes_below() {
  return (1ull << lane_id()) - 1ull;
}

// Wave-uniform values. A value broadcast with __shfl or loaded from LDS lives
// in a vector register, and the compiler then treats a loop exit that depends
// on it as divergent; it may restructure such a loop so that lane 0 leaves it
// on a separate path from the other lanes, which breaks cross-lane operations
// inside it. readfirstlane puts the value in a scalar register, which makes the
// uniformity explicit (all lanes are active wherever these are used).
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Sum over the wavefront with DPP row shifts and row broadcasts
// (register-path lane exchanges, no LDS crossbar): after row_shr 1, 2, 4, 8
// each row's last lane holds the row total, row_bcast 15 and 31 carry the
// totals to lane 63, which is read into a scalar. All lanes must be active.
__device__ __forceinline__ int32_t dpp_wave_sum(int32_t v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);  // row_bcast:31 into rows 2, 3
  return __builtin_amdgcn_readlane(v, kWave - 1);
}

__device__ __forceinline__ int32_t wave_incl_sum(int32_t v) {
  const int lane = lane_id();
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int32_t t = __shfl_up(v, d, kWave);
    if (lane >= d) v += t;
  }
  return v;
}


// ---------------------------------------------------------------------------
// a2: ownership plan.

// Exclusive prefix sum over the workgroup (one value per thread, up to 1024
// threads); *total receives the sum. wsum holds one int per wavefront.
__device__ __forceinline__ int32_t block_excl_scan(int32_t v, int32_t *wsum, int32_t *total) {
  const int lane = lane_id(), wave = threadIdx.x / kWave, nw = blockDim.x / kWave;
  const int32_t incl = wave_incl_sum(v);
  if (lane == kWave - 1) wsum[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int32_t w = lane < nw ? wsum[lane] : 0;
    const int32_t wi = wave_incl_sum(w);
    if (lane < nw) wsum[lane] = wi - w;
    if (lane == nw - 1) *total = wi;
  }
  __syncthreads();
  return incl - v + wsum[wave];
}

constexpr int kPlanThreads = 256;
constexpr int kPlanPer = 8;  // consecutive vertices per thread and tile

// The shapes of a build, and those of one with more than wide_rows vertices
// with neighbours.
struct PlanShapes {
  int32_t small_max, spc;
  int32_t wide_rows, wide_small_max, wide_spc;
};

// Tiles of kPlanThreads * kPlanPer vertices: a vertex of degree 1..small_max
// goes to the small list, a larger one is cut into chunks of spc row slots.
// Whether a vertex owns any edge is left to the intersection kernels (they
// read the neighbour degrees anyway; a vertex that owns nothing costs one
// staging pass). The block scans its counts, reserves list space with one
// global atomic per list, and writes the entries in vertex order.
__global__ __launch_bounds__(kPlanThreads) void k_plan(const int32_t *deg, const int64_t *off, int64_t n,
                                                       PlanShapes shapes, SmallOwner *lists,
                                                       BigChunk *big_list, PlanCounts *pc, int32_t words,
                                                       int32_t *host) {
  __shared__ int32_t last;
  __shared__ int32_t wsum[kPlanThreads / kWave];
  __shared__ int32_t tot_small, tot_heavy, tot_big, base_small, base_heavy, base_big;
  __shared__ int32_t bins[kDegBins];
  static_assert(kDegBins <= kPlanThreads, "a thread per degree bin");
  const bool wide = pc->rows > shapes.wide_rows;
  const int32_t small_max = wide ? shapes.wide_small_max : shapes.small_max;
  const int32_t spc = wide ? shapes.wide_spc : shapes.spc;
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // (read by the last workgroup)
    __hip_atomic_store(&pc->small_max, small_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&pc->spc, spc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x < kDegBins) bins[threadIdx.x] = 0;
  __syncthreads();
  constexpr int64_t kTile = (int64_t)kPlanThreads * kPlanPer;
  for (int64_t t0 = (int64_t)blockIdx.x * kTile; t0 < n; t0 += (int64_t)gridDim.x * kTile) {
    const int64_t v0 = t0 + (int64_t)threadIdx.x * kPlanPer;
    int32_t code[kPlanPer];  // 0 nothing, -1 light, -2 heavy small, else number of chunks
    int32_t ns = 0, nh = 0, nb = 0;
#pragma unroll
    for (int k = 0; k < kPlanPer; ++k) {
      const int32_t dh = v0 + k < n ? deg[v0 + k] : 0;
      if (dh >= 128) atomicAdd(&bins[deg_bin(dh)], 1);
      code[k] = dh == 0 ? 0 : dh <= min(small_max, kLightDeg) ? -1 : dh <= small_max ? -2 : (dh + spc - 1) / spc;
      ns += code[k] == -1;
      nh += code[k] == -2;
      nb += code[k] > 0 ? code[k] : 0;
    }
    __syncthreads();  // wsum and the totals are reused across tiles
    const int32_t os = block_excl_scan(ns, wsum, &tot_small);
    const int32_t oh = block_excl_scan(nh, wsum, &tot_heavy);
    const int32_t ob = block_excl_scan(nb, wsum, &tot_big);
    if (threadIdx.x == 0) {
      base_small = tot_small ? atomicAdd(&pc->small, tot_small) : 0;
      base_heavy = tot_heavy ? atomicAdd(&pc->heavy, tot_heavy) : 0;
      base_big = tot_big ? atomicAdd(&pc->big, tot_big) : 0;
    }
    __syncthreads();
    int32_t ps = base_small + os, ph = base_heavy + oh, pb = base_big + ob;
#pragma unroll
    for (int k = 0; k < kPlanPer; ++k) {
      if (code[k] == -1) lists[ps++] = SmallOwner{(int32_t)(v0 + k), deg[v0 + k], off[v0 + k]};
      if (code[k] == -2) lists[n - 1 - ph++] = SmallOwner{(int32_t)(v0 + k), deg[v0 + k], off[v0 + k]};
      for (int32_t j = 0; j < code[k]; ++j) big_list[pb++] = BigChunk{(int32_t)(v0 + k), j, deg[v0 + k], 0, off[v0 + k]};
    }
  }
  __syncthreads();
  if (threadIdx.x < kDegBins && bins[threadIdx.x]) atomicAdd(&pc->bins[threadIdx.x], bins[threadIdx.x]);
  // The last block to finish hands the counts (and what follows them) to the
  // host's pinned copy: a copy would be a launch more before the host goes on.
  if (!last_workgroup(&pc->done, &last)) return;
  for (int i = threadIdx.x; i < words; i += blockDim.x) host[i] = load_agent((const int32_t *)pc + i);
}

// ---------------------------------------------------------------------------
// Writing one edge's result.

__device__ __forceinline__ void write_edge(int kind, int64_t s, int64_t mirror, int32_t t,
                                           int32_t du, int32_t dh, double *sims,
                                           int32_t *counts) {
  const int64_t c = (int64_t)t + 2;
  const double x = similarity(kind, c, (int64_t)du + 1, (int64_t)dh + 1);
  sims[s] = x;
  if (mirror >= 0) sims[mirror] = x;
  if (counts) {
    counts[s] = (int32_t)c;
    if (mirror >= 0) counts[mirror] = (int32_t)c;
  }
}

// ---------------------------------------------------------------------------
// Small owners (degree <= small_max): one workgroup per vertex, of one
// wavefront up to degree kLightDeg and of kSmallWaves wavefronts above. The
// vertex's row goes into an LDS hash table of buckets of four ids, its lower
// neighbours into an LDS list, and the lower neighbours' rows are streamed
// through the table: groups of lanes take one lower neighbour each (several
// rows per step, since these rows are short), kSmallLoads ids per lane and
// step, with the next step's ids in flight. Bound by the vector units (30
// instructions per 64 lookups) and by latency: a vertex is a chain of four
// dependent reads (list entry, ids, their offsets, rows) and a lookup should
// be one LDS read, so a bucket is read whole and several lookups are issued
// before the first is waited for. (One slot per read, a step's lookups one
// after the other, six dependent reads a vertex: builds of 12 SBM graphs 6.74
// ms, now 5.51; R-MAT of 60,000 vertices 546 and 500 us; R-MAT-20, beside the
// large owners, 6.60 and 6.32 ms. Groups of 16 and 32 lanes instead of 8 and
// 16, 5.79 ms for the SBM graphs; four lookups in flight, 5.65; a full 32-bit
// product in the hash, 5.54.)

constexpr int kSmallWaves = 4;
constexpr int kLightGroup = 8;   // lanes per lower neighbour in the one-wavefront kernel
constexpr int kHeavyGroup = 16;  // and in the kSmallWaves kernel
constexpr int kSmallLoads = 4;   // ids in flight per lane
constexpr int kSmallLookups = 2;  // LDS reads in flight per lane
constexpr int32_t kEmpty = -1;

__device__ __forceinline__ uint32_t hash_bucket(int32_t x, int bbits) {
  // Fibonacci hashing of the low 24 bits (a product at the full rate)
  return __builtin_amdgcn_ubfe(__umul24((uint32_t)x, 10368889u), 24 - bbits, bbits);
}

// Hash table slots per row entry (at least), the kernels' `spread`: a full
// bucket sends a lookup on to the next one (with a quarter of the slots taken
// one bucket in fifty is full, with an eighth one in five hundred), so sparse
// tables pay as long as the LDS holds several workgroups (builds with 4 and 8:
// R-MAT of 60,000 vertices 518 and 507 us, R-MAT-20 6.41 and 6.41 ms, 12 SBM
// graphs 6.10 and 6.08 ms); small_max = 4096 fits with 4.
constexpr int kSpread = 8, kSpreadLarge = 4;
constexpr size_t kSmallLdsMax = 32768;

struct LowRow {
  int64_t ou;     // row offset of a lower neighbour (an empty row's: 0, where reads for it go)
  int32_t du, e;  // its degree, its slot in the vertex's row
};

// LDS bytes of k_small_owner for a given small_max and spread.
static inline size_t small_lds_bytes(int small_max, int spread) {
  int tb = 6;
  while ((1 << tb) < spread * small_max) ++tb;
  return (size_t)small_max * sizeof(LowRow) + ((size_t)4 << tb) + 16;
}

// One block per list entry.
template <int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void k_small_owner(const SmallOwner *list, int small_max, int spread,
                                                               const int64_t *off, const int32_t *adj, int kind,
                                                               double *sims, int32_t *counts, int32_t skip) {
  extern __shared__ unsigned char smem[];
  int32_t &s_nlow = *(int32_t *)smem;
  LowRow *lows = (LowRow *)(smem + 16);        // [small_max] the lower neighbours
  int4 *buckets = (int4 *)(lows + small_max);  // hash table of the row
  int32_t *tab = (int32_t *)buckets;
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const SmallOwner o = list[blockIdx.x];
  const int32_t h = o.h, dh = o.dh;
  const int64_t oh = o.oh;
  int tbits = 6;
  while ((1 << tbits) < spread * dh) ++tbits;
  const int bbits = tbits - 2;
  const uint32_t bmask = (1u << bbits) - 1;
  for (int32_t i = threadIdx.x; i < 1 << bbits; i += WAVES * kWave) buckets[i] = int4{kEmpty, kEmpty, kEmpty, kEmpty};
  if (threadIdx.x == 0) s_nlow = 0;
  __syncthreads();
  for (int32_t i0 = 0; i0 < dh; i0 += WAVES * kWave) {
    const int32_t i = i0 + (int32_t)threadIdx.x;
    const int32_t u = adj[oh + min(i, dh - 1)];
    const int64_t ou = off[u];
    const int32_t d = (int32_t)(off[u + 1] - ou);
    if (i < dh) {
      // (a bucket fills from its first slot: one with an empty last slot ends a lookup)
      uint32_t sl = hash_bucket(u, bbits) * 4;
      while (atomicCAS(&tab[sl], kEmpty, u) != kEmpty) sl = (sl + 1) & (bmask * 4 + 3);
    }
    const bool low = i < dh && is_lower(u, d, h, dh) && d <= skip;
    const uint64_t m = __ballot(low);
    int32_t base = 0;
    if (m) {
      const int leader = __ffsll((unsigned long long)m) - 1;
      int32_t old = 0;
      if (lane == leader) old = atomicAdd(&s_nlow, __popcll(m));
      base = __builtin_amdgcn_readlane(old, leader);
    }
    if (low) lows[base + __popcll(m & lanes_below())] = LowRow{row_start(ou, d), d, i};
  }
  __syncthreads();
  const int32_t nlow = uniform(s_nlow);
  // Each group of G lanes takes one lower neighbour (NG per wavefront, the
  // wavefronts take successive sets); a missing row has length -1 (an empty one
  // is met in graphs that do not hold every edge in both directions). Reads
  // past a row's end read its last id again.
  constexpr int G = WAVES == 1 ? kLightGroup : kHeavyGroup, NG = kWave / G;
  constexpr int L = kSmallLoads, P = kSmallLookups;
  static_assert(G == 8 || G == 16, "sums within a row of 16 lanes");
  const int grp = lane / G, gl = lane % G;
  struct Rows {  // a step: the rows from j, ids from k
    int32_t j, k, longest;
    LowRow q;
  };
  auto rows_at = [&](int32_t j) {
    Rows r{j, 0, 0, lows[min(j + grp, nlow - 1)]};
    if (j + grp >= nlow) r.q.du = -1;
#pragma unroll
    for (int g = 0; g < NG; ++g) r.longest = max(r.longest, __builtin_amdgcn_readlane(r.q.du, g * G));
    return r;
  };
  auto after = [&](const Rows &r) {
    Rows n = r;
    n.k += G * L;
    if (n.k >= r.longest) {
      n.j += WAVES * NG;
      n.k = 0;
      if (n.j < nlow) n = rows_at(n.j);
    }
    return n;
  };
  auto fetch = [&](int32_t x[L], const Rows &r) {
#pragma unroll
    for (int j = 0; j < L; ++j) x[j] = adj[r.q.ou + row_position(r.k + gl + j * G, r.q.du)];
  };
  int32_t acc = 0, pos = -1;  // of this lane: common neighbours, the position of h
  auto probe = [&](const int32_t x[L], const Rows &r) {
#pragma unroll
    for (int j0 = 0; j0 < L; j0 += P) {
      if (j0 && r.k + j0 * G >= r.longest) break;  // uniform
      int4 v[P];
#pragma unroll
      for (int j = 0; j < P; ++j) v[j] = buckets[hash_bucket(x[j0 + j], bbits)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < P; ++j) {
        const int32_t i = r.k + gl + (j0 + j) * G, y = x[j0 + j];
        const bool valid = i < r.q.du;
        bool hit = v[j].x == y || v[j].y == y || v[j].z == y || v[j].w == y;
        if (__ballot(valid && !hit && v[j].w != kEmpty)) {
          uint32_t b = hash_bucket(y, bbits);
          int4 t = v[j];
          while (!hit && t.w != kEmpty) {  // ends at x or at a bucket with room
            b = (b + 1) & bmask;
            t = buckets[b];
            hit = t.x == y || t.y == y || t.z == y || t.w == y;
          }
        }
        acc += valid && hit;
        if (valid && y == h) pos = i;
      }
    }
  };
  auto finish = [&](const Rows &r) {
    int32_t t = acc;
    t += __builtin_amdgcn_update_dpp(0, t, 0x111, 0xf, 0xf, true);  // row_shr:1, 2, 4 (, 8)
    t += __builtin_amdgcn_update_dpp(0, t, 0x112, 0xf, 0xf, true);
    t += __builtin_amdgcn_update_dpp(0, t, 0x114, 0xf, 0xf, true);
    if (G == 16) t += __builtin_amdgcn_update_dpp(0, t, 0x118, 0xf, 0xf, true);
    t = __shfl(t, lane | (G - 1), kWave);
    if (r.q.du >= 0 && (gl == 0 || pos >= 0)) {
      const int64_t c = (int64_t)t + 2;
      const double x = similarity(kind, c, (int64_t)r.q.du + 1, (int64_t)dh + 1);
      if (gl == 0) {
        sims[oh + r.q.e] = x;
        if (counts) counts[oh + r.q.e] = (int32_t)c;
      }
      if (pos >= 0) {
        sims[r.q.ou + pos] = x;
        if (counts) counts[r.q.ou + pos] = (int32_t)c;
      }
    }
    acc = 0;
    pos = -1;
  };
  if (wave * NG >= nlow) return;
  int32_t xa[L], xb[L];
  Rows a = rows_at(wave * NG), b;
  fetch(xa, a);
  for (;;) {
    b = after(a);
    fetch(xb, b);
    probe(xa, a);
    if (b.j != a.j) finish(a);
    if (b.j >= nlow) break;
    a = after(b);
    fetch(xa, a);
    probe(xb, b);
    if (a.j != b.j) finish(b);
    if (a.j >= nlow) break;
  }
}

// ---------------------------------------------------------------------------
// Big owners: persistent workgroups with an LDS bitmap window.

constexpr int kBigThreads = 1024;
constexpr int kBigRun = 4;   // chunks per claim (one window)
constexpr int kUnroll = 4;   // LDS reads in flight per wavefront
constexpr int kDeep = 2;     // items of a wavefront, one probed and one in flight (3 and 4 measured the same)
// Short ranges are taken four per wavefront, by rows of lanes: a whole
// wavefront on one has most of its loads past the end (R-MAT-23, up to 64,
// 128 and 192 ids: 294, 284 and 304 ms; none: 330).
constexpr int kRow = 16;      // lanes per short range
constexpr int kShort = 128;   // its most ids

// Word of the owner bitmap holding id x's bit (x & 31), with the words' byte
// addresses under mask: ids of other windows are not asked for, and an id's
// place in its own window are its low bits. The bitmap starts the kernel's
// dynamic LDS, which starts at LDS address 0 because the kernel has no static
// LDS (the host checks), so the byte address takes two instructions, where a
// pointer to the bitmap costs a third (adding a base the compiler cannot fold).
__device__ __forceinline__ uint32_t bitmap_word(uint32_t x, uint32_t mask) {
  return *(const __attribute__((address_space(3))) uint32_t *)(size_t)((x >> 3) & mask);
}

struct BigShared {
  int32_t claim[2];  // chunk claimed for later, by iteration parity
  int32_t some[2];   // the last iteration whose chunk has lower neighbours, by parity
  int32_t nlong, nshort;
  int32_t next, snext;
  int32_t nextra;
  int32_t wsum[kBigThreads / kWave];
};

// First position in row[lo, hi) whose id is >= key, searched 64-wide by the
// whole wavefront (every lane returns the same value).
__device__ __forceinline__ int64_t wave_lower_bound(const int32_t *row, int64_t lo, int64_t hi,
                                                    int32_t key) {
  const int lane = lane_id();
  while (hi - lo > kWave) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const int64_t p = lo + (int64_t)lane * step;
    const bool less = p < hi && row[p] < key;
    const uint64_t m = __ballot(less);
    const int cnt = __popcll(m);  // positions lo, lo+step, ... below key are a prefix
    if (cnt == 0) return lo;
    const int64_t nlo = lo + (int64_t)(cnt - 1) * step + 1;
    const int64_t nhi = min(hi, lo + (int64_t)cnt * step);
    lo = nlo;
    hi = nhi;
  }
  const int64_t p = lo + lane;
  const bool less = p < hi && row[p] < key;
  return lo + __popcll(__ballot(less));
}

// One workgroup per chunk (owner h, up to spc row slots), persistent over a
// global chunk counter. Per id window: the owner's ids in the window are set
// in the LDS bitmap; each lower neighbour's ids in the window (its range) are
// looked up there, the short ranges four per wavefront, the long ones in items
// of kItem ids, which wavefronts claim from an LDS counter (item j < nlong is
// the first of long range j; later ones are the further items of ranges longer
// than that), so that one long row cannot hold the workgroup at the barrier
// that ends the window. Partial counts meet in LDS. Rows are streamed and set
// from radj: adj itself, or the same rows with ids numbered without the
// isolated vertices (cid), in the same order.
//
// Bound by the reads behind the L2s: on R-MAT-20, alone, 3.05 ms for 20 GB at
// 6.6 of the 7.6 TB/s that random kilobytes reach from the Infinity Cache; on
// R-MAT-23 1.45 TB at 6.7 of 6.9 TB/s. The vector units and the LDS are each
// at 48 %, and a quarter of the wavefronts' time is waiting to issue. What
// brought it there was fewer instructions and fewer waits per id and per range
// (before, with the hub product: R-MAT-20 4.13 ms, R-MAT-23 330; now 3.70 and
// 268): LDS reads in groups, short ranges together, ranges past the end read
// as id 0 and taken out of the sums, claims not waited for, the next chunk's
// data read ahead. Two workgroups of half the size where the
// bitmap leaves room (2^19 vertices) were slower, 3.29 against 3.12 ms a build.
template <bool kOneWindow>
__global__ __launch_bounds__(kBigThreads) void k_big_owner(
    const BigChunk *chunks, PlanCounts *pc, int spc, int wbits, int64_t n,
    const VertexRecord *records, const int32_t *adj, const int32_t *radj, const int64_t *cid, const int32_t *wt,
    int32_t nwin, HubView hub, int kind, double *sims, int32_t *counts, int32_t skip) {
  extern __shared__ unsigned char smem[];
  const int64_t W = (int64_t)1 << wbits;
  const int nwords = (int)(W >> 5);
  const uint32_t wmask = (uint32_t)(nwords - 1) * 4;
  uint32_t *bm = (uint32_t *)smem;
  // Per slot of the chunk, where it is a lower neighbour:
  struct Range {
    const int32_t *ids;  // what is streamed of the row
    int32_t b0, b1;      // positions in the current window
  };
  static_assert(sizeof(Range) == 16, "one LDS read");
  Range *le = (Range *)(bm + nwords);
  int32_t *le_cnt = (int32_t *)(le + spc);  // common neighbours found
  int32_t *le_lt = le_cnt + spc;  // ids below h in the row (searched windows: the row's length)
  int32_t *le_xp = le_lt + spc;   // exclusive prefix of the long ranges' extra segments
  BigShared *sh = (BigShared *)(le_xp + spc);
  uint16_t *le_ord = (uint16_t *)(sh + 1);  // slots with long ranges from the front, with short ones from the back
  const int tid = threadIdx.x, lane = lane_id();
  constexpr bool one_window = kOneWindow;  // the whole id space fits one window
  // Ids per work item: with several windows the ranges are shorter
  // (R-MAT-23, 512 and 1024: 284.0 and 284.2 ms; R-MAT-20: 3.76 and 3.74).
  constexpr int kItem = kOneWindow ? 1024 : 512;
  constexpr int kItemLoads = kItem / kWave;
  constexpr int kGroups = kItem / (kWave * kUnroll);

  const int32_t nchunks = pc->big;  // written by k_plan: no host round trip
  if (nchunks <= 0) return;
  // With one window, chunks are claimed in runs of kRun consecutive ones:
  // a high-degree owner's chunks are consecutive, so a run often keeps one
  // owner, and the owner's bits stay in the bitmap from chunk to chunk
  // (they are cleared only when the next chunk has another owner). The last
  // chunks are claimed one by one.
  constexpr int32_t kRun = kOneWindow ? kBigRun : 1;
  int32_t run_base = 0, run_pos = 0, run_len = 0;  // (of thread 0)
  // The bitmap is cleared as a whole: 128 KB are written in half a
  // microsecond, less than it takes to read back the ids that were set.
  auto wipe = [&]() {
    for (int i = tid; i < nwords / 4; i += kBigThreads) ((uint4 *)bm)[i] = uint4{0, 0, 0, 0};
  };
  struct Owner {
    int32_t ci, h, dh, m;  // chunk, vertex, degree, slots in the chunk
    int64_t oh, s0;        // first slot of the row, of the chunk
  };
  // (words: a chunk's descriptor spread over the lanes)
  auto owner_of = [&](int32_t ci, int32_t words) {
    Owner o;
    const bool ok = ci >= 0 && ci < nchunks;
    o.ci = ci;
    auto word = [&](size_t at) { return __builtin_amdgcn_readlane(words, (int)(at / 4)); };
    o.h = word(offsetof(BigChunk, h));
    o.dh = ok ? word(offsetof(BigChunk, dh)) : 0;
    o.oh = (int64_t)(uint32_t)word(offsetof(BigChunk, oh)) | (int64_t)word(offsetof(BigChunk, oh) + 4) << 32;
    o.s0 = o.oh + (int64_t)word(offsetof(BigChunk, k)) * spc;
    o.m = ok ? (int32_t)min((int64_t)spc, o.oh + o.dh - o.s0) : 0;
    return o;
  };
  const bool own_tab = !one_window && wt && nwin < kWave;
  constexpr int kOwn = 4;  // owner ids per thread in flight

  // A chunk's data come through a chain of dependent reads: claim,
  // descriptor, ids, their degrees and offsets, the hubs' counts. They are
  // made up to three chunks ahead, one step of the chain per chunk, so that
  // each is in flight while a whole chunk is handled (waiting for them in
  // turn took 10 of the 46 thousand cycles of a chunk of R-MAT-20). Thread t carries slot t
  // in registers. Iterations whose chunk is not there yet have no slots.
  Owner cur{-1, 0, 0, 0, 0, 0}, nxt = cur;  // this chunk and the next
  int32_t c2 = -1;                           // the chunk after
  int32_t d2 = 0;
  bool low = false;                          // this chunk's slot is a lower neighbour, and then:
  int32_t u = 0, du = 0, wrow = 0;           // it, its degree, its row of the window table
  int64_t ou = 0;                            // and its first slot
  int32_t un = 0, du_n = 0, r_n = -1;        // the next chunk's slot: vertex, degree, hub row
  int64_t ou_n = 0;
  int32_t of_n = -1;                         // the next owner's hub row and column, and its id among the streamed ones
  int32_t hc = 0, hx = 0;                    // this one's
  bool hubs = false;                         // this chunk's slot is an edge between hubs, and then:
  HubRow hq{0, 0, 0};
  int32_t hcnt = 0, hpre = 0;
  uint4 hbits{0, 0, 0, 0};
  int32_t ox[kOwn];              // the owner's ids at positions p + tid + j * kBigThreads
  int32_t own = 0, own_n = 0;    // the owner's row of the window table, spread over the lanes
  int32_t kw = 0, pe = 0;        // window, and end of its ids in the owner's row
  int32_t pf0 = 0, pf1 = 0;      // the slot's range in it
  int32_t held = -1;             // the owner whose bits the bitmap holds (one window)
#pragma unroll
  for (int j = 0; j < kOwn; ++j) ox[j] = 0;
  auto load_own = [&](const Owner &o, int32_t p, int32_t pe) {
#pragma unroll
    for (int j = 0; j < kOwn; ++j) ox[j] = radj[o.oh + p + min(tid + j * kBigThreads, pe - p - 1)];
  };
  auto set_own = [&](const Owner &o, int32_t p, int32_t pe, int32_t w0) {
    for (;;) {
#pragma unroll
      for (int j = 0; j < kOwn; ++j) {
        const int32_t x = ox[j] - w0;
        if (tid + j * kBigThreads < pe - p) atomicOr(&bm[x >> 5], 1u << (x & 31));
      }
      if (pe - p <= kOwn * kBigThreads) break;
      p += kOwn * kBigThreads;
      load_own(o, p, pe);
    }
  };
  // The window of position p of the owner's row, and where its ids end there.
  auto window_at = [&](const Owner &o, int32_t row, int32_t p, int32_t &k, int32_t &end) {
    if (own_tab) {
      k = __popcll(__ballot(row <= p)) - 1;
      end = __builtin_amdgcn_readlane(row, k + 1);
      return;
    }
    k = uniform(radj[o.oh + p] >> wbits);
    const int64_t w1 = (int64_t)(k + 1) << wbits;
    end = wt ? uniform(wt[(int64_t)o.h * (nwin + 1) + k + 1])
             : (int32_t)wave_lower_bound(radj + o.oh, p, o.dh, (int32_t)min(w1, (int64_t)INT32_MAX));
  };
  auto load_ranges = [&](bool is_low, int32_t row) {
    if (wt && is_low) {
      const int32_t *t = wt + (int64_t)row * (nwin + 1) + kw;
      pf0 = t[0];
      pf1 = t[1];
    }
  };

  wipe();
  if (tid == 0) {
    sh->claim[0] = -1;
    sh->some[0] = sh->some[1] = -1;
    sh->nlong = sh->nshort = sh->nextra = 0;
    sh->next = sh->snext = 0;
  }
  for (int32_t it = 0;; ++it) {
    __syncthreads();
    if (cur.ci >= nchunks) break;
    const int32_t c3 = uniform(sh->claim[it & 1]);
    const Owner own_c = cur;
    const int32_t h = own_c.h, dh = own_c.dh;
    if (tid < own_c.m) {
      // An edge between two hubs streams only the ids outside the product's
      // columns; the count of the others is in D, and of those below h in the
      // bits before its column.
      int32_t lt = !one_window && !wt && low ? du : 0;
      if (one_window && hubs) {
        const uint64_t lo = (uint64_t)hbits.y << 32 | hbits.x, hi = (uint64_t)hbits.w << 32 | hbits.z;
        const uint64_t below = (1ull << (hc & 63)) - 1;
        lt = hpre + ((hc & 64) ? __popcll(lo) + __popcll(hi & below) : __popcll(lo & below));
      }
      le_cnt[tid] = hubs ? hcnt : 0;
      le_lt[tid] = lt;
      le[tid] = Range{hubs ? hub.rest + hq.off : radj + ou, 0, !one_window || !low ? 0 : hubs ? hq.len : du};
    }
    // The next chunk's slots, and what follows of the chain.
    auto advance = [&]() {
      const VertexRecord q = records[un];  // (one line a neighbour instead of three)
      du_n = q.deg;
      r_n = q.hub;
      ou_n = q.off;
      if (own_tab) own_n = lane <= nwin ? wt[(int64_t)nxt.h * (nwin + 1) + lane] : INT32_MAX;
      c2 = c3;
      d2 = ((const int32_t *)(chunks + max(0, min(c3, nchunks - 1))))[min(lane, (int)(sizeof(BigChunk) / 4) - 1)];
      if (tid == 0 && run_pos == run_len) {
        run_len = run_base + 16 * (int32_t)gridDim.x < nchunks ? kRun : 1;
        run_base = atomicAdd(&pc->counter, run_len);
        run_pos = 0;
      }
    };
    if (one_window && own_c.m && h != held) {
      set_own(own_c, 0, dh, 0);
      held = h;
    }
    if (!one_window) advance();
    // Windows of ids [w0, w0 + W) that hold ids of N(h), in increasing order:
    // window kw holds positions [p, pe) of the owner's row. The owner's ids in
    // the next window and, with the table, the slot's range in it are read
    // while the current window's items run.
    int32_t p = 0;
    if (one_window) pe = dh;
    if (!one_window && uniform(sh->some[it & 1]) != it) p = dh;  // no lower neighbours
    if (one_window && dh == 0) advance();
    while (p < dh) {
      const int32_t w0 = one_window ? 0 : (int32_t)((int64_t)kw << wbits);
      if (!one_window) set_own(own_c, p, pe, w0);
      if (!one_window && wt) {
        // thread t alone writes and reads slot t's range before the barrier
        if (tid < own_c.m) {
          le[tid].b0 = low ? pf0 : 0;
          le[tid].b1 = low ? pf1 : 0;
        }
      } else if (!one_window) {
        // each lower neighbour's ids inside this window, after the last one
        __syncthreads();
        for (;;) {
          int32_t old = 0;
          if (lane == 0) old = atomicAdd(&sh->snext, 1);
          const int32_t i = __builtin_amdgcn_readlane(old, 0);
          if (i >= own_c.m) break;
          const int32_t len = uniform(le_lt[i]);
          const int32_t *row = (const int32_t *)(uintptr_t)uniform64((int64_t)(uintptr_t)le[i].ids);  // (no hubs here)
          const int64_t w1 = (int64_t)w0 + W;
          const int64_t b0 = wave_lower_bound(row, uniform(le[i].b1), len, w0);
          const int64_t b1 = wave_lower_bound(row, b0, len, (int32_t)min(w1, (int64_t)INT32_MAX));
          le[i].b0 = (int32_t)b0;
          le[i].b1 = (int32_t)b1;
        }
        __syncthreads();
        if (tid == 0) sh->snext = 0;
      }
      // Long and short ranges; empty ones need nothing.
      const int32_t range = tid < own_c.m ? le[tid].b1 - le[tid].b0 : 0;
      {
        const uint64_t ml = __ballot(range > kShort), ms = __ballot(range > 0 && range <= kShort);
        int32_t bl = 0, bs = 0;
        if (lane == 0) {
          if (ml) bl = atomicAdd(&sh->nlong, __popcll(ml));
          if (ms) bs = atomicAdd(&sh->nshort, __popcll(ms));
        }
        bl = uniform(bl) + __popcll(ml & lanes_below());
        bs = uniform(bs) + __popcll(ms & lanes_below());
        if (range > kShort) le_ord[bl] = (uint16_t)tid;
        else if (range > 0) le_ord[spc - 1 - bs] = (uint16_t)tid;
        if (range > kItem) sh->nextra = 1;
      }
      __syncthreads();
      if (one_window) advance();
      const int nlong = uniform(sh->nlong), nshort = uniform(sh->nshort);
      const bool bit0 = uniform((int32_t)bm[0]) & 1;
      int32_t nitems = nlong;
      if (uniform(sh->nextra)) {
        // Extra segments of the long ranges, as an exclusive prefix over them.
        int32_t ex = 0;
        if (tid < nlong) {
          const int32_t e = le_ord[tid];
          ex = (le[e].b1 - le[e].b0 - 1) / kItem;
        }
        const int32_t xp = block_excl_scan(ex, sh->wsum, &sh->nextra);
        if (tid < nlong) le_xp[tid] = xp;
        __syncthreads();
        nitems += uniform(sh->nextra);
      }
      const int32_t pn = pe;  // the next window's start
      if (!one_window && pn < dh) {
        window_at(own_c, own, pn, kw, pe);
        load_own(own_c, pn, pe);
        load_ranges(low, wrow);
      }
      // Work items are claimed from the LDS counter, one lane adding 1.
      // A claim is split in two: take() issues the LDS atomic, resolve()
      // turns its result into an item. Between the two the wavefront probes
      // its current item, so the atomic's round trip is not on its path.
      // (the address is made to look divergent, or the compiler would combine
      // the lanes' adds first and wait for the result at once)
      auto take_of = [&](int32_t *counter, int32_t count) -> int32_t {
        int32_t zero = 0, old = 0;
        asm("" : "+v"(zero));
        if (lane == 0) old = atomicAdd(counter + zero, count);
        return old;
      };
      auto take = [&]() { return take_of(&sh->next, 1); };
      auto resolve = [&](int32_t tok, int32_t &e, int32_t &lo, int32_t &hi, const int32_t *&ids) {
        const int32_t j = __builtin_amdgcn_readlane(tok, 0);
        if (j >= nitems) {
          e = -1;
          lo = hi = 0;
          ids = radj;
          return;
        }
        int32_t ee = j, sg = 0;
        if (j >= nlong) {
          // the last long range e with le_xp[e] <= jj (le_xp is non-decreasing and
          // le_xp[0] = 0): a 64-way search, every lane sampling one edge
          const int32_t jj = j - nlong;
          int32_t a0 = 0, na = nlong;
          while (na > 1) {
            const int32_t step = (na + kWave - 1) / kWave;
            const int32_t q = a0 + lane * step;
            const int32_t c = __popcll(__ballot(q < a0 + na && le_xp[q] <= jj));  // >= 1: lane 0
            const int32_t nb = a0 + (c - 1) * step;
            na = min(step, a0 + na - nb);
            a0 = nb;
          }
          ee = a0;
          sg = 1 + jj - uniform(le_xp[a0]);
        }
        ee = uniform((int32_t)le_ord[ee]);
        e = ee;
        const Range q = le[ee];
        ids = (const int32_t *)(uintptr_t)uniform64((int64_t)(uintptr_t)q.ids);
        lo = (one_window ? 0 : uniform(q.b0)) + sg * kItem;
        hi = min(uniform(q.b1), lo + kItem);
      };
      // Whole items are requested one item ahead, and the loop body is
      // unrolled so that the register sets swap roles without register
      // copies (a copy waits for its load). Every load of an item is
      // issued: a fixed count keeps the waits exact (the compiler waits for
      // an item's loads by counting the loads issued after them). The loads
      // are raw buffer loads over a resource of exactly the item's bytes, so
      // lanes past its end read 0 without touching memory (no line is
      // fetched for them, and no bound check or mask is needed). Addressing
      // is scalar base + lane offset + immediate: no vector instruction per
      // load.
      auto fetch_item = [&](int32_t x[kItemLoads], const int32_t *ids, int32_t lo, int32_t len) {
        // resource word 3: DATA_FORMAT 32 (a valid format enables the buffer)
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((void *)(ids + lo), (short)0, len * 4, 0x00020000);
        // (opaque here, so that the lane offset and the immediates are not added
        // up ahead of the loop, in a register each)
        int32_t at = lane * 4;
        asm("" : "+v"(at));
#pragma unroll
        for (int j = 0; j < kItemLoads; ++j) x[j] = __builtin_amdgcn_raw_buffer_load_b32(r, at + j * kWave * 4, 0, 0);
      };
      // Hits of an item's len ids and, with one window, how many are below h:
      // rows are sorted, so the position of h in the lower neighbour's row is
      // the sum of the latter over the row's items. kUnroll LDS reads are in
      // flight (left to itself the compiler waits for each in turn). Lanes
      // past the end hold id 0 and are taken out of the sums afterwards.
      auto probe_item = [&](const int32_t x[kItemLoads], int32_t e, int32_t len) {
        uint32_t acc = 0;
        int32_t below = 0, lanes = 0;
#pragma unroll
        for (int c = 0; c < kGroups; ++c)
          if (c == 0 || len > c * kWave * kUnroll) {
            uint32_t w[kUnroll];
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) w[k] = bitmap_word((uint32_t)x[c * kUnroll + k], wmask);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
              acc += __builtin_amdgcn_ubfe(w[k], (uint32_t)x[c * kUnroll + k], 1);
              if (kOneWindow) below += __popcll(__ballot(x[c * kUnroll + k] < hx));
            }
            lanes += kWave * kUnroll;
          }
        const int32_t past = lanes - len;
        const int32_t t = dpp_wave_sum((int32_t)acc) - (bit0 ? past : 0);
        // t is wave-uniform: lane 0 records it (no return value is used, so
        // no lane waits on another)
        if (lane == 0) {
          atomicAdd(&le_cnt[e], t);
          if (kOneWindow) atomicAdd(&le_lt[e], below - (hx > 0 ? past : 0));
        }
      };
      // Items are claimed one step further ahead: the claim's atomic goes
      // out before a probe and is resolved after it, when the probe has
      // freed its registers, so no claim waits on loads in flight.
      if (nitems) {
        int32_t e[kDeep], lo[kDeep], hi[kDeep];
        const int32_t *ids[kDeep];
        int32_t x[kDeep][kItemLoads];
#pragma unroll
        for (int d = 0; d < kDeep; ++d) {
          resolve(take(), e[d], lo[d], hi[d], ids[d]);
          if (d + 1 < kDeep) fetch_item(x[d], ids[d], lo[d], hi[d] - lo[d]);
        }
        for (bool more = true; more;) {
#pragma unroll
          for (int d = 0; d < kDeep; ++d) {
            const int f = (d + kDeep - 1) % kDeep;
            if (e[d] < 0) {
              more = false;
              break;
            }
            fetch_item(x[f], ids[f], lo[f], hi[f] - lo[f]);
            const int32_t t = take();
            probe_item(x[d], e[d], hi[d] - lo[d]);
            resolve(t, e[d], lo[d], hi[d], ids[d]);
          }
        }
      }
      // Short ranges: four per wavefront, one in each row of kRow lanes.
      constexpr int kShortLoads = kShort / kRow;
      const int rlane = lane & (kRow - 1), rowi = lane / kRow;
      auto stake = [&]() -> int32_t {
        return take_of(&sh->snext, kWave / kRow);
      };
      auto sresolve = [&](int32_t tok, int32_t &q, int32_t &e, int32_t &len, const int32_t *&ids) {
        q = __builtin_amdgcn_readlane(tok, 0);
        const bool ok = q + rowi < nshort;
        e = le_ord[ok ? spc - 1 - q - rowi : spc - 1];
        const Range r = le[e];
        len = ok ? r.b1 - r.b0 : 0;
        ids = r.ids + r.b0;
      };
      // (past its end a lane reads the range's last id again)
      auto sfetch = [&](int32_t x[kShortLoads], const int32_t *ids, int32_t len) {
#pragma unroll
        for (int j = 0; j < kShortLoads; ++j) x[j] = ids[max(min(rlane + j * kRow, len - 1), 0)];
      };
      auto sprobe = [&](const int32_t x[kShortLoads], int32_t e, int32_t len) {
        uint32_t acc = 0, w[kShortLoads];
#pragma unroll
        for (int j = 0; j < kShortLoads; ++j) w[j] = bitmap_word((uint32_t)x[j], wmask);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < kShortLoads; ++j) {
          const uint32_t hit = __builtin_amdgcn_ubfe(w[j], (uint32_t)x[j], 1) + (kOneWindow && x[j] < hx ? 0x10000u : 0u);
          acc += rlane + j * kRow < len ? hit : 0u;
        }
        int32_t v = (int32_t)acc;
        v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
        v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
        v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
        v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
        if (rlane == kRow - 1 && len > 0) {
          atomicAdd(&le_cnt[e], v & 0xffff);
          if (kOneWindow) atomicAdd(&le_lt[e], (int32_t)((uint32_t)v >> 16));
        }
      };
      if (nshort) {
        int32_t q[kDeep], e[kDeep], len[kDeep];
        const int32_t *ids[kDeep];
        int32_t x[kDeep][kShortLoads];
#pragma unroll
        for (int d = 0; d < kDeep; ++d) {
          sresolve(stake(), q[d], e[d], len[d], ids[d]);
          if (d + 1 < kDeep) sfetch(x[d], ids[d], len[d]);
        }
        for (bool more = true; more;) {
#pragma unroll
          for (int d = 0; d < kDeep; ++d) {
            const int f = (d + kDeep - 1) % kDeep;
            if (q[d] >= nshort) {
              more = false;
              break;
            }
            sfetch(x[f], ids[f], len[f]);
            const int32_t t = stake();
            sprobe(x[d], e[d], len[d]);
            sresolve(t, q[d], e[d], len[d], ids[d]);
          }
        }
      }
      __syncthreads();
      if (tid == 0) {
        sh->nlong = sh->nshort = sh->nextra = 0;
        sh->next = sh->snext = 0;
      }
      if (!one_window) {
        wipe();
        __syncthreads();
      }
      p = pn;
    }
    // Ahead: the next chunk's hub data, first window and owner ids, the ids
    // of the chunk after.
    const int32_t lt = le_lt[min(tid, spc - 1)], cnt = le_cnt[min(tid, spc - 1)];
    const bool low_c = low;
    const int32_t du_c = du;
    const int64_t ou_c = ou;
    const bool low_n = tid < nxt.m && is_lower(un, du_n, nxt.h, nxt.dh) && du_n <= skip;
    const int32_t hr = hub.rows ? uniform(of_n) : -1;
    hc = __builtin_amdgcn_readlane(of_n, 1);
    const int32_t hx_c = hx;
    hx = cid ? __builtin_amdgcn_readlane(of_n, 2) : nxt.h;
    hubs = low_n && hr >= 0 && r_n >= 0;
    wrow = un;
    if (hubs) {
      hq = hub.row_of[r_n];
      hcnt = hub.D[(int64_t)max(r_n, hr) * hub.stride + min(r_n, hr)];
      wrow = (int32_t)n + r_n;
      if (one_window) {
        hbits = hub.bits[hub.piece(r_n, hc >> 7)];
        hpre = hub.pre[(int64_t)r_n * (hub.cols / 128) + (hc >> 7)];
      }
    }
    if (!one_window && __ballot(low_n) && lane == 0) sh->some[(it + 1) & 1] = it + 1;
    const int32_t u_c = u;
    u = un;
    own = own_n;
    low = low_n;
    du = du_n;
    ou = ou_n;
    if (one_window) {
      if (nxt.m && nxt.h != held) {
        load_own(nxt, 0, nxt.dh);
        wipe();
      }
    } else if (nxt.m) {
      window_at(nxt, own, 0, kw, pe);
      load_own(nxt, 0, pe);
      load_ranges(low, wrow);
    }
    const Owner two = owner_of(c2, d2);
    if (two.m) {
      un = adj[two.s0 + min(tid, two.m - 1)];
      const int32_t *at = lane == 0 ? &records[two.h].hub : lane == 1 ? hub.col + two.h : (const int32_t *)(cid + two.h);
      if (lane == 0 || (lane == 1 && hub.rows) || (lane == 2 && cid)) of_n = *at;
    }
    // This chunk's edges.
    if (low_c) {
      int64_t mir = -1;
      if (one_window) {
        // h sits after the ids below it (absent only from an asymmetric row)
        if (lt < du_c && adj[ou_c + lt] == h) mir = ou_c + lt;
      } else {
        // h may lie in a window that holds no id of N(h): locate it directly,
        // with the table among the ids of its window and by interpolation in
        // every other step (rows are long and ids spread: four dependent
        // reads instead of eleven; 37 of the 345 thousand cycles of a chunk
        // of R-MAT-23 were spent here)
        int64_t a = 0, b = du_c, va = 0, vb = 0;
        if (wt) {
          const int32_t *t = wt + (int64_t)u_c * (nwin + 1) + (hx_c >> wbits);
          a = t[0];
          b = t[1];
          va = (int64_t)(hx_c >> wbits) << wbits;
          vb = va + W;
        }
        for (bool guess = wt != nullptr; a < b; guess = !guess && wt) {
          int64_t mid = (a + b) >> 1;
          if (guess) mid = min(b - 1, a + (int64_t)((float)(hx_c - va) * (float)(b - a) / (float)(vb - va)));
          const int32_t v = radj[ou_c + mid];
          if (v == hx_c) {
            mir = ou_c + mid;
            break;
          }
          if (v < hx_c) {
            a = mid + 1;
            va = v;
          } else {
            b = mid;
            vb = v;
          }
        }
      }
      // (nothing read for the chunks to come is waited for behind the stores)
      asm volatile("" ::"v"(un), "v"(of_n), "v"(hcnt), "v"(hq.off), "v"(hq.len));
      if (one_window) asm volatile("" ::"v"(hpre), "v"(hbits.x), "v"(hbits.y), "v"(hbits.z), "v"(hbits.w));
      else asm volatile("" ::"v"(pf0), "v"(pf1));
#pragma unroll
      for (int j = 0; j < kOwn; ++j) asm volatile("" ::"v"(ox[j]));
      write_edge(kind, own_c.s0 + tid, mir, cnt, du_c, dh, sims, counts);
    }
    if (tid == 0) sh->claim[(it + 1) & 1] = run_base + run_pos++;
    cur = nxt;
    nxt = two;
  }
}

// Window table of every row: wt[u * (nwin + 1) + k] = the first position in
// row u whose id is >= k * 2^wbits (k = 0..nwin), so that a lower
// neighbour's ids inside window k are positions [wt[k], wt[k + 1]) of its
// row. One wavefront per row; the next row's offsets are requested while a
// row is handled. Rows of up to kTableScan ids are streamed 64 ids per step:
// a lane whose id opens windows past its left neighbour's writes their
// starts (every entry is written once), and the step past the row's end
// closes the last windows. Longer rows find each window's start by a 64-way
// search (every lane samples one position, a few rounds per window), so that
// no wavefront walks a hub's whole row.
constexpr int32_t kTableScan = 2048;

__global__ __launch_bounds__(256) void k_window_table(const int64_t *off, const int32_t *adj, int64_t n,
                                                      int wbits, int32_t nwin, int32_t *wt) {
  const int lane = lane_id();
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  int64_t u = uniform64((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave);
  int64_t o_next = 0, e_next = 0;  // offsets of the wavefront's next row
  if (u < n) {
    o_next = off[u];
    e_next = off[u + 1];
  }
  for (; u < n; u += nw) {
    const int64_t o = uniform64(o_next);
    const int32_t d = uniform((int32_t)(uniform64(e_next) - o));
    if (u + nw < n) {
      o_next = off[u + nw];
      e_next = off[u + nw + 1];
    }
    int32_t *t = wt + u * (nwin + 1);
    if (d > kTableScan) {
      int32_t lo = 0;  // window starts do not decrease with k
      for (int32_t k = 1; k < nwin; ++k) {
        const int64_t bound = (int64_t)k << wbits;
        int32_t hi = d;  // the start is in [lo, hi]; position d stands for the end of the row
        while (lo < hi) {
          // (kWave - 1) * step >= hi - lo: the last lane samples at or past hi
          const int32_t step = (hi - lo + kWave - 2) / (kWave - 1);
          const int64_t p = (int64_t)lo + (int64_t)lane * step;
          const bool at = p >= hi || adj[o + p] >= bound;
          const int f = __ffsll((unsigned long long)__ballot(at)) - 1;  // >= 0: the last lane is true
          if (f == 0) break;  // the start is lo
          const int32_t nlo = lo + (f - 1) * step + 1;
          hi = uniform((int32_t)min((int64_t)hi, (int64_t)lo + (int64_t)f * step));
          lo = uniform(nlo);
        }
        if (lane == 0) t[k] = lo;
      }
      if (lane == 0) {
        t[0] = 0;
        t[nwin] = d;
      }
      continue;
    }
    int32_t prev = -1;  // window of the id before this step (wave-uniform)
    for (int32_t i0 = 0; i0 <= d; i0 += kWave) {
      const int32_t i = i0 + lane;
      const int32_t w = i < d ? adj[o + i] >> wbits : nwin;  // past the end: window nwin
      int32_t wl = __shfl_up(w, 1, kWave);
      if (lane == 0) wl = prev;
      for (int32_t k = wl + 1; k <= w; ++k) t[k] = i;
      prev = __shfl(w, kWave - 1, kWave);
    }
  }
}

__global__ void k_vertex_records(const int64_t *off, int64_t n, VertexRecord *records) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    const int64_t o = off[v];
    records[v] = VertexRecord{(int32_t)(off[v + 1] - o), -1, o};
  }
}

// Ids without the isolated vertices (`used` are left), in the same order.
__global__ void k_id_flags(const int32_t *deg, int64_t n, int32_t *flags) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
    flags[v] = deg[v] > 0;
}
__global__ __launch_bounds__(256) void k_rename(const int32_t *adj, int64_t nnz, const int64_t *cid, int32_t used,
                                                int32_t *out) {
  constexpr int kPer = 4;  // ids per thread in flight
  for (int64_t s0 = blockIdx.x * (int64_t)(kPer * 256) + threadIdx.x; s0 < nnz; s0 += (int64_t)gridDim.x * kPer * 256) {
    int32_t x[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) x[k] = s0 + k * 256 < nnz ? adj[s0 + k * 256] : 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) x[k] = used_number(cid[x[k]], used);
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (s0 + k * 256 < nnz) out[s0 + k * 256] = x[k];
  }
}

// ---------------------------------------------------------------------------
// Host side.

constexpr size_t kMaxWindowTable = (size_t)4 << 30;

static size_t big_lds_bytes(int wbits, int spc) {
  return ((size_t)1 << wbits) / 8 + (size_t)spc * (16 + 4 * 3 + 2) + sizeof(BigShared);
}

// The id window width of the large-owner kernel: cfg.wbits, no wider than
// the id space and narrowed until its LDS fits.
static int window_bits(const IntersectConfig &cfg, int64_t n, int lds_max) {
  int wbits = cfg.wbits;
  int nb = 0;
  while (((int64_t)1 << nb) < n) ++nb;
  if (nb < 10) nb = 10;
  if (wbits > nb) wbits = nb;
  while (wbits > 10 && big_lds_bytes(wbits, cfg.spc) > (size_t)lds_max) --wbits;
  return wbits;
}

scan_status intersect_plan(const IntersectConfig &cfg, int64_t n, int64_t nnz, const int64_t *off,
                           const int32_t *deg, DevArena &arena, hipStream_t s, void *counts, int32_t words, void *host, hipEvent_t ready, IntersectPlan &p) {
  p.n = n;
  p.nnz = nnz;
  if (nnz == 0) return SCAN_OK;
  BigChunk *big_list;
  PlanCounts *pc = (PlanCounts *)counts;
  SCAN_TRY(arena.alloc(&p.lists, n));
  if (!p.weighted) SCAN_TRY(arena.alloc(&p.records, n));
  PlanShapes shapes{cfg.small_max, cfg.spc, INT_MAX, cfg.small_max, cfg.spc};
  if (cfg.auto_shapes && n > kWideRows) {
    shapes.wide_rows = kWideRows;
    shapes.wide_small_max = kWideSmallMax;
    shapes.wide_spc = kWideSpc;
  }
  SCAN_TRY(arena.alloc(&big_list, nnz / std::min(shapes.spc, shapes.wide_spc) +
                                      std::min(n, nnz / std::min(shapes.small_max, shapes.wide_small_max)) + 1));
  p.big_list = big_list;
  p.counts = counts;
  p.host = host;
  k_plan<<<grid_for(n, kPlanThreads * kPlanPer, 2048), kPlanThreads, 0, s>>>(
      deg, off, n, shapes, p.lists, big_list, pc, words, (int32_t *)host);
  SCAN_HIP_TRY(hipEventRecord(ready, s));
  return SCAN_OK;
}

scan_status intersect_all(const IntersectConfig &asked, int64_t n, int64_t nnz, const int64_t *off,
                          const int32_t *deg, const int32_t *adj, int kind, double *sims,
                          int32_t *counts, int device, hipStream_t s, IntersectStats *stats,
                          const std::function<scan_status()> &reserve,
                          const std::function<scan_status()> &after_launch, const IntersectPlan *plan) {
  if (nnz == 0) return after_launch ? after_launch() : SCAN_OK;
  int lds_max = 65536, cus = 256;
  (void)hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  if (!plan || plan->n != n || plan->nnz != nnz || !plan->host)
    return fail(SCAN_EINVAL, "plan made for another graph");
  const BigChunk *big_list = (const BigChunk *)plan->big_list;
  PlanCounts *pc = (PlanCounts *)plan->counts;
  // The host reads the work counts to size the grids: one block per vertex
  // lets the hardware balance the uneven rows, which persistent grids with a
  // static split do not.
  const PlanCounts h = *(const PlanCounts *)plan->host;
  IntersectConfig cfg = asked;
  cfg.small_max = h.small_max;
  cfg.spc = h.spc;
  // Memory that the build can do without (ids numbered anew, the hub product)
  // is taken after what it needs, and given back where that is refused: a
  // build fits wherever it would fit without them.
  DevArena tmp(s), ids_mem(s), hub_mem(s);
  const int wbits_all = window_bits(cfg, n, lds_max);
  int wbits = wbits_all;
  auto windows = [](int64_t ids, int bits) { return (int32_t)((ids + ((int64_t)1 << bits) - 1) >> bits); };
  int32_t nwin = windows(n, wbits);
  int32_t *wt = nullptr, *renamed = nullptr;
  int64_t *cid = nullptr;
  if (h.big && nwin > 1) {
    // Ids spanning several windows. A chunk's cost is mostly its work items,
    // and each lower neighbour makes at least one per window, so ids are
    // numbered without the isolated vertices where that saves a window (half
    // of an R-MAT graph's: R-MAT-23 has 8 windows with them and 6 without, and
    // its large owners take 448 ms with them, 400 without; renaming takes 5).
    // Where there is no memory for the second adjacency, they stay.
    const int rbits = window_bits(cfg, h.rows, lds_max);
    int32_t *flags;
    int64_t *ws;
    if (windows(h.rows, rbits) < nwin) {
      if (reserve) SCAN_TRY(reserve());
      if (ids_mem.alloc(&renamed, nnz) == SCAN_OK && ids_mem.alloc(&flags, n) == SCAN_OK &&
          ids_mem.alloc(&cid, n + 1) == SCAN_OK && ids_mem.alloc(&ws, scan_workspace_elems(n)) == SCAN_OK) {
        k_id_flags<<<grid_for(n, 256), 256, 0, s>>>(deg, n, flags);
        SCAN_TRY(exclusive_scan(flags, cid, n, ws, s));
        k_rename<<<grid_for(nnz, 1024), 256, 0, s>>>(adj, nnz, cid, h.rows, renamed);
        wbits = rbits;
        nwin = windows(h.rows, rbits);
      } else {
        ids_mem.release();
        renamed = nullptr;
        cid = nullptr;
      }
    }
  }
  // Common neighbours among hubs by matrix product, where that saves enough.
  // (Not in approximate builds, which leave the hubs' edges out.)
  const bool table = nwin > 1 && !cfg.search_windows;
  HubShape shape;
  if (h.big && plan->one_graph && cfg.skip_deg == 0x7fffffff && (nwin == 1 || (table && nwin <= kHubMaxWindows)))
    shape = choose_hubs(h, nnz, nwin == 1);
  if (shape.rows && reserve) SCAN_TRY(reserve());
  if (h.big && table) {
    // The window table, unless it would exceed kMaxWindowTable bytes or the
    // searched ranges are asked for; then chunks search them per window.
    // The rows of the hubs' rests follow those of the vertices.
    auto table_for = [&](int64_t rows) -> scan_status {
      if ((size_t)(nwin + 1) * (size_t)n * 4 > kMaxWindowTable) return SCAN_OK;
      return tmp.alloc(&wt, (int64_t)(nwin + 1) * rows);
    };
    scan_status st = table_for(n + shape.rows);
    if (st == SCAN_ENOMEM && shape.rows) {
      shape = HubShape{};
      st = table_for(n);
    }
    if (st == SCAN_ENOMEM && renamed) {
      ids_mem.release();
      renamed = nullptr;
      cid = nullptr;
      wbits = wbits_all;
      nwin = windows(n, wbits);
      st = table_for(n);
    }
    SCAN_TRY(st);
    if (wt) k_window_table<<<grid_for(n * kWave, 256), 256, 0, s>>>(off, renamed ? renamed : adj, n, wbits, nwin, wt);
  }
  if (h.big) k_vertex_records<<<grid_for(n, 256, 4096), 256, 0, s>>>(off, n, plan->records);
  HubView hub;
  if (shape.rows && (nwin == 1 || wt)) {
    const scan_status st = prepare_hubs(shape, n, off, deg, adj, renamed ? renamed : adj, wbits, nwin,
                                        wt ? wt + (int64_t)(nwin + 1) * n : nullptr, plan->records, hub_mem, s, &hub);
    if (st != SCAN_OK && st != SCAN_ENOMEM) return st;
    if (st == SCAN_ENOMEM) hub_mem.release();  // every row is streamed whole
  }
  if (big_lds_bytes(wbits, cfg.spc) > (size_t)lds_max) return fail(SCAN_EINVAL, "chunk size too large for LDS");
  if (stats) {
    stats->wbits = wbits;
    stats->hub_rows = hub.rows;
    stats->hub_cols = hub.rows ? shape.cols : 0;
    stats->launches = (h.small > 0) + (h.heavy > 0) + (h.big > 0);
    if (stats->host_counts) {
      stats->host_counts[0] = h.small;
      stats->host_counts[1] = h.big;
      stats->host_counts[3] = h.heavy;
    }
  }
  auto mark = [&](hipEvent_t e, hipStream_t st) -> scan_status {
    if (e) SCAN_HIP_TRY(hipEventRecord(e, st));
    return SCAN_OK;
  };
  SCAN_TRY(mark(stats ? stats->ev_plan_end : nullptr, s));
  // The large-owner kernel is persistent (one 1024-thread workgroup per CU,
  // most of the LDS) and leaves wavefront slots, registers and some LDS free
  // on every CU; the small-owner kernels, independent of it, run on the
  // helper stream and fill them. The large one is launched first so that its
  // workgroups are placed before the small ones take CUs.
  // The two small-owner kernels take helper streams of their own, so that
  // neither waits for the other.
  auto fork = [&](int k, bool used) -> hipStream_t {
    if (!used || !h.big) return s;
    // Ordered after the plan by the caller; after the hub product they run
    // beside the large-owner kernel, which leaves room for them, and not
    // beside the product, which does not.
    if (plan->helper[k] && (!hub.rows || stream_wait(plan->helper[k], s) == SCAN_OK)) return plan->helper[k];
    hipStream_t hs = helper_stream(k);
    if (!hs || stream_wait(hs, s) != SCAN_OK) return s;
    return hs;
  };
  const hipStream_t sh = fork(0, h.heavy > 0), sl = fork(1, h.small > 0);
  JoinOnExit join_sh{s, sh}, join_sl{s, sl};  // before the plan lists are released
  if (h.big) {
    size_t lds = big_lds_bytes(wbits, cfg.spc);
    const bool one = nwin == 1;
    const int32_t *radj = renamed ? renamed : adj;
    const void *fn = one ? (const void *)k_big_owner<true> : (const void *)k_big_owner<false>;
    hipFuncAttributes fa;
    SCAN_HIP_TRY(hipFuncGetAttributes(&fa, fn));
    if (fa.sharedSizeBytes != 0)  // bitmap_word assumes the dynamic LDS starts at address 0
      return fail(SCAN_EDEVICE, "k_big_owner has %zu bytes of static LDS", (size_t)fa.sharedSizeBytes);
    if (lds > 65536)
      SCAN_HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(2, (size_t)lds_max / lds));
    const int grid = (int)std::min<int64_t>((int64_t)cus * per_cu, h.big);
    SCAN_TRY(mark(stats ? stats->ev_big_begin : nullptr, s));
    if (one)
      k_big_owner<true><<<grid, kBigThreads, lds, s>>>(big_list, pc, cfg.spc, wbits, n, plan->records, adj, radj, cid, nullptr,
                                                       nwin, hub, kind, sims, counts, cfg.skip_deg);
    else
      k_big_owner<false><<<grid, kBigThreads, lds, s>>>(big_list, pc, cfg.spc, wbits, n, plan->records, adj, radj, cid, wt,
                                                        nwin, hub, kind, sims, counts, cfg.skip_deg);
    SCAN_HIP_TRY(hipGetLastError());
    SCAN_TRY(mark(stats ? stats->ev_big_end : nullptr, s));
  } else {
    SCAN_TRY(mark(stats ? stats->ev_big_begin : nullptr, s));
    SCAN_TRY(mark(stats ? stats->ev_big_end : nullptr, s));
  }
  const hipStream_t ss = sh != s ? sh : sl;  // the small-owner events go on one of them
  SCAN_TRY(mark(stats ? stats->ev_small_begin : nullptr, ss));
  if (h.small || h.heavy) {
    const int cap = std::min<int>(cfg.small_max, kLightDeg);  // light rows: LDS sized for them
    const int spread = small_lds_bytes(cfg.small_max, kSpread) > kSmallLdsMax ? kSpreadLarge : kSpread;
    const size_t lds = small_lds_bytes(cfg.small_max, spread), lds1 = small_lds_bytes(cap, kSpread);
    if (lds > (size_t)lds_max || lds1 > (size_t)lds_max) return fail(SCAN_EINVAL, "small_max too large for LDS");
    if (lds > 65536)
      SCAN_HIP_TRY(hipFuncSetAttribute((const void *)k_small_owner<kSmallWaves>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    if (lds1 > 65536)
      SCAN_HIP_TRY(hipFuncSetAttribute((const void *)k_small_owner<1>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds1));
    if (h.heavy)  // the longer rows first
      k_small_owner<kSmallWaves><<<h.heavy, kSmallWaves * kWave, lds, sh>>>(
          plan->lists + (n - h.heavy), cfg.small_max, spread, off, adj, kind, sims, counts, cfg.skip_deg);
    if (h.small)
      k_small_owner<1><<<h.small, kWave, lds1, sl>>>(plan->lists, cap, kSpread, off, adj, kind, sims, counts,
                                                     cfg.skip_deg);
    SCAN_HIP_TRY(hipGetLastError());
  }
  if (sl != ss) SCAN_TRY(stream_wait(ss, sl));  // the end event covers both
  SCAN_TRY(mark(stats ? stats->ev_small_end : nullptr, ss));
  if (after_launch) SCAN_TRY(after_launch());
  return SCAN_OK;
}

}  // namespace scan
