// Weighted cosine similarity (Section 3.1; Algorithm 1 is written for this
// measure). For adjacent u, v:
//   sigma(u, v) = D(u, v) / sqrt(S_u * S_v),
//   D(u, v) = sum over x in N[u] ∩ N[v] of w(u, x) w(v, x),
//   S_v     = sum over x in N[v] of w(v, x)^2,
// over closed neighbourhoods with w(x, x) = 1; w(u, x) is the weight stored in
// u's CSR slot for x. The paper leaves the order of these floating-point sums
// open. Here every sum adds its terms one at a time in ascending x, so each
// similarity is one fixed FP64 value (no FP contraction, IEEE sqrt and
// division); with all weights 1 the sums are the integers c, a_u and a_v and
// the result is the unweighted cosine bit for bit.
//
// The sums are the cost: 1.27e9 products on R-MAT-20, each one dependent add.
// A row of 16 lanes takes one edge; the lanes' products are broadcast within
// the row one after the other (row_newbcast) and added by every lane, so one
// add instruction serves four edges, and lanes without a common id add +0.0,
// which changes nothing (a running sum is never -0).
//
//   k_w_square_sums  a row of lanes per vertex: the squares of its row, added
//                    in order with the self term 1 at its place.
// Up to 2^kWbMaxBits vertices, by the ownership plan of the unweighted path
// (each edge by the endpoint larger in (degree, id), the owner h; every lower
// neighbour l streams its row in ascending order):
//   k_w_big          owners above kWbSmallMax: h's row is a bitmap in LDS with
//                    counts per 128 bits, so that a common id gives its
//                    position in h's row, and with it w(h, x).
//   k_w_small        the others: h's row in an LDS hash table with its
//                    positions and weights.
// Above:
//   k_w_unit_rows    the row holding the first slot of every kWUnit-slot unit
//                    of the CSR.
//   k_w_owner        one workgroup per unit. The owner's ids and weights go
//                    into LDS in tiles of kWTile; every lower neighbour l
//                    streams its row through them, a lane finds its id by
//                    binary search in its bucket of the tile (kWBuckets
//                    buckets of equal id width, indexed per tile), and the
//                    wavefront adds the products of the common ids in
//                    ascending id.
// All insert the terms of x = h (1 * w(l, h)) and x = l (w(h, l) * 1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "index.h"
#include "rows.h"

namespace scan {
namespace {

constexpr int kWUnit = 128;                  // CSR slots per workgroup
constexpr int kWThreads = 256;
constexpr int kWWaves = kWThreads / kWave;
constexpr int kWTile = 1024;                 // owner ids (and weights) per LDS tile
constexpr int kWBuckets = 512;               // id buckets per tile (a lookup's first guess)
constexpr int kWRows = 64;                   // row offsets staged at a time
#ifndef SCAN_W_CHUNKS
#define SCAN_W_CHUNKS 4
#endif
constexpr int kWChunks = SCAN_W_CHUNKS;      // 64-id chunks of a lower row loaded at once

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
// Lane k's double (k wave-uniform).
__device__ __forceinline__ double lane_f64(double v, int k) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)b, k);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)(b >> 32), k);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// acc + p(lane 0) + p(lane 1) + ... of each row, added in that order. The add
// is fma(p, 1, acc), the same value: of the FP64 operations only the fused
// one reads a lane broadcast as an operand. (Two wait states between a
// register's write and its read by a broadcast.)
#define SCAN_ROW_ADD(n) "v_fmac_f64_dpp %0, %1, %2 row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ double row_sum(double acc, double p) {
  asm("s_nop 1\n\t" SCAN_ROW_ADD(0) SCAN_ROW_ADD(1) SCAN_ROW_ADD(2) SCAN_ROW_ADD(3) SCAN_ROW_ADD(4) SCAN_ROW_ADD(5)
          SCAN_ROW_ADD(6) SCAN_ROW_ADD(7) SCAN_ROW_ADD(8) SCAN_ROW_ADD(9) SCAN_ROW_ADD(10) SCAN_ROW_ADD(11)
              SCAN_ROW_ADD(12) SCAN_ROW_ADD(13) SCAN_ROW_ADD(14) SCAN_ROW_ADD(15)
      : "+&v"(acc)
      : "v"(p), "v"(1.0));
  return acc;
}
#undef SCAN_ROW_ADD
// The same with x added before lane `at`'s value (at = 16: not at all): the
// values before it, x, the others, each sum over all lanes (a lane that is not
// in it adds +0.0). Adding x or +0.0 before every lane took 112 instructions
// instead of 38, in one step of six on R-MAT-20 (builds 23.5 ms, now
// 22.9).
__device__ __forceinline__ double row_sum_with(double acc, double p, int at, double x) {
  const int gl = lane_id() & 15;
  acc = row_sum(acc, gl < at ? p : 0.0);
  acc += at < 16 ? x : 0.0;
  return row_sum(acc, gl < at ? 0.0 : p);
}
// This row's 16 bits of a ballot.
__device__ __forceinline__ uint32_t row_bits(uint64_t m) { return (uint32_t)(m >> (lane_id() & 48)) & 0xffffu; }

// A row of lanes per vertex, four vertices per wavefront in step (a hub's sum
// is its length in dependent adds; the others of its wavefront wait). The
// loads of kSqAhead steps are in flight, none of them behind a branch.
// R-MAT-20: 2.0 -> 0.64 ms.
constexpr int kSqAhead = 8;
__global__ __launch_bounds__(256) void k_w_square_sums(const int64_t *off, const int32_t *adj, const double *w,
                                                       int64_t n, double *S) {
  const int lane = lane_id(), row = lane / 16, gl = lane % 16;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  for (int64_t v0 = uniform64(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave * 4); v0 < n; v0 += waves * 4) {
    const int64_t v = v0 + row;
    int64_t o = 0, d = 0;
    if (v < n) {
      o = off[v];
      d = off[v + 1] - o;
      if (d <= 0) o = 0;
    }
    const int64_t top = max(d - 1, (int64_t)0);  // the last position (an empty row reads slot 0: o is 0)
    int64_t steps = (d + 15) / 16;
    steps = max(max(steps, (int64_t)__shfl_xor((int)steps, 16, kWave)), (int64_t)__shfl_xor((int)steps, 32, kWave));
    steps = uniform64(max(steps, (int64_t)__shfl_xor((int)steps, 48, kWave)));
    double acc = 0.0;
    bool self = false;
    int32_t x[kSqAhead];
    double wx[kSqAhead];
    auto fetch = [&](int64_t s, int32_t &xs, double &ws) {
      const int64_t q = o + min(s * 16 + gl, top);
      xs = adj[q];
      ws = w[q];
    };
#pragma unroll
    for (int k = 0; k < kSqAhead; ++k) fetch(k, x[k], wx[k]);
    for (int64_t s0 = 0; s0 < steps; s0 += kSqAhead) {
#pragma unroll
      for (int k = 0; k < kSqAhead; ++k) {  // (steps past the end add +0.0)
        const int64_t s = s0 + k;
        const bool in = s * 16 + gl < d;
        const double sq = in ? wx[k] * wx[k] : 0.0;
        const uint32_t above = row_bits(__ballot(in && x[k] > v));
        fetch(s + kSqAhead, x[k], wx[k]);
        int at = 16;  // the self term 1 goes before the first id above v
        if (!self && above) {
          at = __ffs(above) - 1;
          self = true;
        }
        acc = __any(at < 16) ? row_sum_with(acc, sq, at, 1.0) : row_sum(acc, sq);
      }
    }
    if (!self) acc += 1.0;
    if (gl == 0 && v < n) S[v] = acc;
  }
}

// One edge's sum, the state of a row of lanes.
struct WEdge {
  int32_t l, du;   // the lower neighbour and its degree (du 0: no edge)
  int64_t ou;      // its row
  double whl, acc; // w(h, l), the running sum
  bool ldone;      // the x = l term is in acc
};
// Adds a step's products (0.0 where there is none); at: the lane before which
// the x = l term goes, 16 if not in this step; some: whether any lane of the
// wavefront has a product. Without one the adds are left out: in random graphs
// of degree 200 to 330, whose rows have few ids in common, the builds were 4 to
// 11% behind k_w_owner's, which adds the common ids' products alone, and are
// now level to 8% behind (100,000 vertices of degree 250 10.3 -> 9.4 ms, 9.4
// with k_w_owner; 20,000 of degree 230 2.17 -> 2.11, 1.95); R-MAT-20 23.0 ms
// either way.
__device__ __forceinline__ void add_products(WEdge &e, double prod, int at, bool some) {
  if (__any(at < 16)) e.acc = row_sum_with(e.acc, prod, at, e.whl);
  else if (some) e.acc = row_sum(e.acc, prod);
}
// Where the x = l term goes among a step's ids (marks it done).
__device__ __forceinline__ int place_l(WEdge &e, bool valid, int32_t x) {
  if (__all(e.ldone)) return 16;
  const uint32_t above = row_bits(__ballot(valid && x > e.l));
  if (e.ldone || !above) return 16;
  e.ldone = true;
  return __ffs(above) - 1;
}
__device__ __forceinline__ int32_t quad_max(int32_t v) {  // v is the same within a row of lanes
  const int32_t a = max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
  return max(a, max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// ---------------------------------------------------------------------------
// Small owners. The next step's ids and weights are requested before a step is
// summed; owners without lower neighbours end after the staging.

constexpr int kWbSmallMax = 256;
constexpr int kWSmallSpread = 4;  // table slots per row entry (at least)
constexpr int32_t kWEmpty = -1;

__host__ __device__ inline int smem_table(int cap) {  // table slots for rows of up to cap ids
  int tb = 6;
  while ((1 << tb) < kWSmallSpread * cap) ++tb;
  return 1 << tb;
}
static inline size_t w_small_lds(int cap) {
  return (size_t)cap * (8 + 8 + 4 * 3 + 2) + (size_t)6 * smem_table(cap);
}

template <int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void k_w_small(const SmallOwner *list, int cap, const int64_t *off,
                                                           const int32_t *deg, const int32_t *adj, const double *w,
                                                           const double *S, double *sims, int32_t skip) {
  extern __shared__ unsigned char smem[];
  double *tw = (double *)smem;              // [cap] the vertex's weights
  int64_t *lou = (int64_t *)(tw + cap);     // [cap] row offset of the j-th lower neighbour
  int32_t *ids = (int32_t *)(lou + cap);    // [cap] the vertex's row
  int32_t *lid = ids + cap;                 // [cap] the j-th lower neighbour
  int32_t *ldu = lid + cap;                 // [cap] its degree
  int32_t *tab = ldu + cap;                 // [2^tbits] hash table of the row: ids
  uint16_t *le = (uint16_t *)(tab + smem_table(cap));  // [cap] the lower neighbour's slot
  uint16_t *tpos = le + cap;                // [2^tbits] their positions
  __shared__ int32_t s_nlow;
  const int lane = lane_id(), wave = threadIdx.x / kWave, row = lane / 16, gl = lane % 16;
  const int32_t h = list[blockIdx.x].h;
  const int32_t dh = deg[h];
  const int64_t oh = off[h];
  int tbits = 6;
  while ((1 << tbits) < kWSmallSpread * dh) ++tbits;
  const uint32_t tmask = (1u << tbits) - 1;
  if (threadIdx.x == 0) s_nlow = 0;
  __syncthreads();
  for (int32_t i0 = 0; i0 < dh; i0 += blockDim.x) {
    const int32_t i = i0 + (int32_t)threadIdx.x;
    int32_t u = 0, d = 0;
    if (i < dh) {
      u = adj[oh + i];
      d = deg[u];
      ids[i] = u;
      tw[i] = w[oh + i];
    }
    const bool low = i < dh && (d < dh || (d == dh && u < h)) && d <= skip;
    const uint64_t m = __ballot(low);
    int32_t base = 0;
    if (m && lane == 0) base = atomicAdd(&s_nlow, __popcll(m));
    base = uniform(base);
    if (low) {
      const int32_t j = base + __popcll(m & ((1ull << lane) - 1ull));
      le[j] = (uint16_t)i;
      lid[j] = u;
      ldu[j] = d;
      lou[j] = row_start(off[u], d);
    }
  }
  __syncthreads();
  const int32_t nlow = uniform(s_nlow);
  if (nlow == 0) return;  // owns no edge (uniform across the block)
  for (uint32_t i = threadIdx.x; i <= tmask; i += blockDim.x) tab[i] = kWEmpty;
  __syncthreads();
  for (int32_t i = threadIdx.x; i < dh; i += blockDim.x) {
    const int32_t x = ids[i];
    uint32_t sl = ((uint32_t)x * 2654435761u) >> (32 - tbits);
    while (atomicCAS(&tab[sl], kWEmpty, x) != kWEmpty) sl = (sl + 1) & tmask;
    tpos[sl] = (uint16_t)i;
  }
  __syncthreads();
  const double sh = S[h];
  for (int32_t j0 = wave * 4; j0 < nlow; j0 += WAVES * 4) {
    const int32_t j = min(j0 + row, nlow - 1);
    const bool has = j0 + row < nlow;
    WEdge e{lid[j], has ? ldu[j] : 0, lou[j], tw[le[j]], 0.0, false};
    const int32_t du = ldu[j], steps = (quad_max(e.du) + 15) / 16;
    int64_t mpos = -1;
    int32_t x;
    double wl;
    auto fetch = [&](int32_t s) {
      const int64_t q = e.ou + row_position(s * 16 + gl, du);
      x = adj[q];
      wl = w[q];
    };
    fetch(0);
    for (int32_t s = 0; s < steps; ++s) {
      const bool valid = s * 16 + gl < e.du;
      const int32_t xs = x;
      const double ws = wl;
      fetch(s + 1);
      double wh = 0.0;
      bool hit = false;
      if (valid) {
        uint32_t sl = ((uint32_t)xs * 2654435761u) >> (32 - tbits);
        for (;;) {  // ends at xs or at an empty slot (the table is at most a quarter full)
          const int32_t t = tab[sl];
          if (t == xs) {
            wh = tw[tpos[sl]];
            hit = true;
            break;
          }
          if (t == kWEmpty) break;
          sl = (sl + 1) & tmask;
        }
      }
      if (valid && xs == h) {
        wh = 1.0;
        hit = true;
        mpos = e.ou + s * 16 + gl;
      }
      const int at = place_l(e, valid, xs);
      add_products(e, hit ? wh * ws : 0.0, at, __any(hit));
    }
    if (!e.ldone) e.acc += e.whl;  // l is above every id of its row
    // the lane that met h writes the mirror slot too
    const double v = e.acc / sqrt(sh * S[e.l]);
    if (has && gl == 0) sims[oh + le[j]] = v;
    if (mpos >= 0) sims[mpos] = v;
  }
}

// ---------------------------------------------------------------------------
// Large owners: persistent workgroups claim chunks of kWbSpc slots of an
// owner's row (in runs, so that an owner's bitmap serves several chunks). The
// chunk's lower neighbours are ordered by length class, and every wavefront
// takes four of them at a time, one per row of lanes, in step; their ids are
// requested two steps ahead, the weights of a step's common ids one step
// before they are summed (a common id takes two scattered reads of 8 bytes;
// reading the weights of all ids takes 55 GB more on R-MAT-20). R-MAT-20, 1.0e8
// steps: 20.6 ms with the small owners beside it, where k_w_owner took 45; its
// vector instructions (87 a step, 16 of them the adds) are issued three
// quarters of the time. Weights requested one step ahead: 21.2 ms, and 24.2
// when the loop's exits made the compiler wait for every load.

constexpr int kWbMaxBits = 20;
constexpr int kWbThreads = 1024;
constexpr int kWbSpc = 256;
constexpr int32_t kWbRun = 4;
constexpr int kWbClasses = 64;  // four per octave of the lower neighbour's degree

struct WBigShared {
  int32_t chunk, run_next, run_left, nlow, next;
  int32_t cls[kWbClasses];
  int32_t wsum[kWbThreads / kWave];
};

static size_t w_big_lds(int wbits) {
  const size_t bits = (size_t)1 << wbits, blocks = bits / 128;
  return bits / 8 + blocks * 2 + 32 * 4 + (size_t)kWbSpc * (8 + 8 + 4 * 3 + 2 * 2) + sizeof(WBigShared);
}

__device__ __forceinline__ double load_f64(__amdgpu_buffer_rsrc_t r, uint32_t byte) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)byte, 0, 0);
  return __longlong_as_double((long long)((uint64_t)v[1] << 32 | v[0]));
}

__device__ __forceinline__ int length_class(int32_t d) {  // 0: the longest
  const int o = 31 - __clz(d);
  const int c = 4 * o + (o >= 2 ? (d >> (o - 2)) & 3 : 0);
  return kWbClasses - 1 - min(c, kWbClasses - 1);
}

__global__ __launch_bounds__(kWbThreads) void k_w_big(const BigChunk *chunks, PlanCounts *pc, int wbits,
                                                      const int64_t *off, const int32_t *deg, const int32_t *adj,
                                                      const double *w, int64_t nnz, const double *S, double *sims,
                                                      int32_t skip) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int nwords = (1 << wbits) >> 5, nblk = nwords >> 2;  // blocks of 128 bits
  uint32_t *bm = (uint32_t *)smem;
  int64_t *le_ou = (int64_t *)(bm + nwords);
  double *le_acc = (double *)(le_ou + kWbSpc);
  int32_t *le_l = (int32_t *)(le_acc + kWbSpc);
  int32_t *le_du = le_l + kWbSpc;
  int32_t *le_mpos = le_du + kWbSpc;
  int32_t *base = le_mpos + kWbSpc;         // [32] bits before every 32 * per blocks
  uint16_t *pre = (uint16_t *)(base + 32);  // [nblk] bits before a block, from its base
  uint16_t *le_e = pre + nblk;
  uint16_t *order = le_e + kWbSpc;
  WBigShared *sh = (WBigShared *)(order + kWbSpc);
  const int tid = threadIdx.x, lane = lane_id(), row = lane / 16, gl = lane % 16, wave = tid / kWave;
  const int per = max(1, nblk / kWbThreads);  // blocks per thread in the counts; a base per 32 threads
  const int bshift = 31 - __clz(32 * per);
  const int32_t nchunks = pc->big;
  // resource word 3: DATA_FORMAT 32 (a valid format enables the buffer)
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void *)w, (short)0, (int)(uint32_t)(nnz * 8), 0x00020000);
  const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc((void *)adj, (short)0, (int)(uint32_t)(nnz * 4), 0x00020000);
  for (int i = tid; i < nwords; i += kWbThreads) bm[i] = 0u;
  if (tid == 0) sh->run_left = 0;
  int32_t held = -1, held_dh = 0;  // the owner whose bits the bitmap holds
  int64_t held_oh = 0;
  for (;;) {
    __syncthreads();
    if (tid == 0) {
      if (sh->run_left == 0) {
        sh->run_next = atomicAdd(&pc->counter, kWbRun);
        sh->run_left = kWbRun;
      }
      sh->chunk = sh->run_next++;
      --sh->run_left;
      sh->nlow = 0;
      sh->next = 0;
    }
    if (tid < kWbClasses) sh->cls[tid] = 0;
    __syncthreads();
    const int32_t ci = uniform(sh->chunk);
    if (ci >= nchunks) break;
    const BigChunk ch = chunks[ci];
    const int32_t h = ch.h;
    const int32_t dh = deg[h];
    const int64_t oh = off[h];
    const int64_t s0 = oh + (int64_t)ch.k * kWbSpc;
    const int m = (int)min((int64_t)kWbSpc, oh + dh - s0);
    if (tid < kWbSpc) {  // the chunk's lower neighbours (whole wavefronts)
      int32_t u = 0, du = 0;
      if (tid < m) {
        u = adj[s0 + tid];
        du = deg[u];
      }
      const bool low = tid < m && (du < dh || (du == dh && u < h)) && du <= skip;
      const uint64_t mk = __ballot(low);
      int32_t b = 0;
      if (mk && lane == 0) b = atomicAdd(&sh->nlow, __popcll(mk));
      b = uniform(b);
      if (low) {
        const int k = b + __popcll(mk & ((1ull << lane) - 1ull));
        le_e[k] = (uint16_t)tid;
        le_l[k] = u;
        le_du[k] = du;
        le_ou[k] = row_start(off[u], du);
        le_mpos[k] = -1;
        atomicAdd(&sh->cls[length_class(du)], 1);
      }
    }
    __syncthreads();
    const int nlow = uniform(sh->nlow);
    if (nlow == 0) continue;
    if (h != held) {
      if (held >= 0) {
        for (int i = tid; i < held_dh; i += kWbThreads) bm[(uint32_t)adj[held_oh + i] >> 5] = 0u;
        __syncthreads();  // the new owner's bits may share words with the old one's
      }
      for (int i = tid; i < dh; i += kWbThreads) {
        const int32_t x = adj[oh + i];
        atomicOr(&bm[x >> 5], 1u << (x & 31));
      }
      held = h;
      held_oh = oh;
      held_dh = dh;
      __syncthreads();
      // counts: this thread's blocks, then an exclusive sum over the workgroup
      int32_t sum = 0;
      for (int k = 0; k < per; ++k)
        if (tid * per + k < nblk) {
          const uint4 b = ((const uint4 *)bm)[tid * per + k];
          sum += __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w);
        }
      int32_t incl = sum;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const int32_t t = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += t;
      }
      if (lane == kWave - 1) sh->wsum[wave] = incl;
      __syncthreads();
      int32_t e = incl - sum;
      for (int k = 0; k < wave; ++k) e += sh->wsum[k];
      const int32_t b0 = __shfl(e, lane & 32, kWave);
      if (tid % 32 == 0 && tid * per < nblk) base[tid / 32] = b0;
      for (int k = 0; k < per; ++k)
        if (tid * per + k < nblk) {
          pre[tid * per + k] = (uint16_t)(e - b0);
          const uint4 b = ((const uint4 *)bm)[tid * per + k];
          e += __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w);
        }
    }
    if (wave == 0) {  // class starts
      int32_t c = sh->cls[lane], incl = c;
      static_assert(kWbClasses == kWave, "a lane per class");
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const int32_t t = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += t;
      }
      sh->cls[lane] = incl - c;
    }
    __syncthreads();
    if (tid < nlow) order[atomicAdd(&sh->cls[length_class(le_du[tid])], 1)] = (uint16_t)tid;
    __syncthreads();
    for (;;) {
      int32_t q = 0;
      if (lane == 0) q = atomicAdd(&sh->next, 1);
      q = uniform(q) * 4;
      if (q >= nlow) break;
      const bool has = q + row < nlow;
      const int k = order[min(q + row, nlow - 1)];
      const int32_t ldu = le_du[k], top = row_position(INT_MAX, ldu);
      WEdge e{le_l[k], has ? ldu : 0, le_ou[k], w[s0 + le_e[k]], 0.0, false};
      const int32_t steps = (quad_max(e.du) + 15) / 16;
      // Slots fit 32 bits, their weights' bytes too. A step's position is a
      // scalar, so an id's byte takes one add and one clamp, and the same add
      // tells whether it lies in the row.
      const uint32_t eo = (uint32_t)e.ou, ho = (uint32_t)oh;
      const uint32_t id0 = (eo + gl) * 4u, id_top = (eo + (uint32_t)top) * 4u,
                     id_end = has && ldu > 0 ? id_top + 1 : 0;
      auto fetch = [&](int32_t s) -> int32_t {
        return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(ar, (int)min(id0 + (uint32_t)s * 64u, id_top), 0, 0);
      };
      // One step: probe its ids and request the weights of the common ones.
      // Every load is issued by every lane, so that the compiler can wait for
      // a step's loads by counting those issued after them (behind a branch it
      // waits for all: 29.7 instead of 24.6 ms on R-MAT-20): buffer loads, whose
      // offset is past the end where there is nothing to read, which gives 0
      // and touches no memory.
      auto probe = [&](int32_t x, int32_t s, double &wl, double &wh, bool &self, int &at,
                       bool &some) {
        const uint32_t id = id0 + (uint32_t)s * 64u;
        const bool valid = id < id_end;
        const uint4 b = ((const uint4 *)bm)[(uint32_t)x >> 7];
        const uint64_t lo = (uint64_t)b.y << 32 | b.x, hi = (uint64_t)b.w << 32 | b.z;
        const bool upper = (x & 64) != 0;
        const uint64_t half = upper ? hi : lo;
        const bool hit = valid && ((half >> (x & 63)) & 1);
        self = valid && x == h;
        some = __any(hit || self);
        // position of x in h's row, where x is in it
        const uint32_t blk = (uint32_t)x >> 7;
        const int32_t rank = base[blk >> bshift] + pre[blk] + (upper ? __popcll(lo) : 0) +
                             __popcll(half & ~(~0ull << (x & 63)));
        wl = load_f64(wr, hit || self ? id * 2u : ~7u);
        wh = load_f64(wr, hit ? (ho + (uint32_t)rank) * 8u : ~7u);
        if (self) le_mpos[k] = s * 16 + gl;
        at = place_l(e, valid, x);
      };
      int32_t x0 = fetch(0), x1 = fetch(1), x2 = fetch(2);
      double wl0, wh0, wl1, wh1, wl2, wh2;
      bool self0, self1, self2;  // x = h: w(h, h) = 1
      int at0, at1, at2;
      bool some0, some1, some2;
      probe(x0, 0, wl0, wh0, self0, at0, some0);
      x0 = fetch(3);
      probe(x1, 1, wl1, wh1, self1, at1, some1);
      x1 = fetch(4);
      // The three register sets change roles without copies; steps past the
      // rows' ends (no valid id) add nothing.
      for (int32_t s = 2; s - 2 < steps; s += 3) {
        probe(x2, s, wl2, wh2, self2, at2, some2);
        x2 = fetch(s + 3);
        add_products(e, wl0 * (self0 ? 1.0 : wh0), at0, some0);
        probe(x0, s + 1, wl0, wh0, self0, at0, some0);
        x0 = fetch(s + 4);
        add_products(e, wl1 * (self1 ? 1.0 : wh1), at1, some1);
        probe(x1, s + 2, wl1, wh1, self1, at1, some1);
        x1 = fetch(s + 5);
        add_products(e, wl2 * (self2 ? 1.0 : wh2), at2, some2);
      }
      if (has && gl == 0) le_acc[k] = e.ldone ? e.acc : e.acc + e.whl;  // (l above every id of its row)
    }
    __syncthreads();
    if (tid < nlow) {
      const double v = le_acc[tid] / sqrt(S[h] * S[le_l[tid]]);
      sims[s0 + le_e[tid]] = v;
      if (le_mpos[tid] >= 0) sims[le_ou[tid] + le_mpos[tid]] = v;
    }
  }
}

// row_of[k] = the row holding slot k * kWUnit (rows are non-empty there).
__global__ void k_w_unit_rows(const int64_t *off, int64_t n, int32_t *row_of) {
  for (int64_t h = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; h < n; h += (int64_t)gridDim.x * blockDim.x) {
    const int64_t a = off[h], b = off[h + 1];
    for (int64_t k = (a + kWUnit - 1) / kWUnit; k * kWUnit < b; ++k) row_of[k] = (int32_t)h;
  }
}

struct WShared {
  int32_t tid[kWTile];      // the owner's ids of the current tile
  double tw[kWTile];        // and their weights w(h, x)
  int32_t bst[kWBuckets + 1];  // first tile position of each id bucket (then tn)
  int64_t roff[kWRows + 1];  // off[base .. base + kWRows]
  int64_t lou[kWUnit];      // row offset of the j-th lower neighbour
  double acc[kWUnit];       // its running dot product
  double whl[kWUnit];       // w(h, l): the weight in h's slot for l
  int32_t le[kWUnit];       // that slot
  int32_t lid[kWUnit];      // l
  int32_t ldu[kWUnit];      // deg(l)
  int32_t cur[kWUnit];      // first position of l's row not yet streamed
  int32_t nxt[kWUnit];      // the id there (INT_MIN before the first tile)
  int32_t mpos[kWUnit];     // position of h in l's row (the mirror slot)
  int32_t ldone[kWUnit];    // 1 once the x = l term is added
  int32_t nlow;
};

__global__ __launch_bounds__(kWThreads) void k_w_owner(const int64_t *off, const int32_t *deg, const int32_t *adj,
                                                       const double *w, const double *S, const int32_t *row_of,
                                                       int64_t n, int64_t nnz, double *sims, int32_t skip) {
  __shared__ WShared sh;
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const int64_t s0 = (int64_t)blockIdx.x * kWUnit, s1 = s0 + kWUnit < nnz ? s0 + kWUnit : nnz;
  int64_t h = row_of[blockIdx.x], base = -1;
  for (;;) {
    if (base < 0 || h + 1 > base + kWRows) {  // stage the next kWRows row offsets
      __syncthreads();
      base = h;
      for (int i = threadIdx.x; i <= kWRows; i += blockDim.x) sh.roff[i] = off[base + i < n ? base + i : n];
      __syncthreads();
    }
    const int64_t ra = uniform64(sh.roff[h - base]), rb = uniform64(sh.roff[h + 1 - base]);
    if (ra >= s1) break;  // uniform across the block
    const int64_t a = ra > s0 ? ra : s0, b = rb < s1 ? rb : s1;
    if (a < b) {
      const int32_t dh = (int32_t)(rb - ra);
      if (threadIdx.x == 0) sh.nlow = 0;
      __syncthreads();
      // The lower neighbours among slots [a, b), compacted into LDS.
      {
        const int64_t slot = a + threadIdx.x;
        int32_t u = 0, du = 0;
        const bool in = slot < b;
        if (in) {
          u = adj[slot];
          du = deg[u];
        }
        const bool low = in && (du < dh || (du == dh && u < h)) && du <= skip;
        const uint64_t m = __ballot(low);
        int32_t j0 = 0;
        if (m) {
          const int leader = __ffsll((unsigned long long)m) - 1;
          j0 = __builtin_amdgcn_readlane(atomicAdd(&sh.nlow, lane == leader ? __popcll(m) : 0), leader);
        }
        if (low) {
          const int j = j0 + __popcll(m & ((1ull << lane) - 1ull));
          sh.le[j] = (int32_t)(slot - ra);
          sh.lid[j] = u;
          sh.ldu[j] = du;
          sh.lou[j] = off[u];
          sh.whl[j] = w[slot];
          sh.acc[j] = 0.0;
          sh.cur[j] = 0;
          sh.nxt[j] = INT_MIN;
          sh.mpos[j] = -1;
          sh.ldone[j] = 0;
        }
      }
      __syncthreads();
      const int32_t nlow = uniform(sh.nlow);
      for (int32_t t0 = 0; nlow > 0 && t0 < dh; t0 += kWTile) {
        const int32_t tn = dh - t0 < kWTile ? dh - t0 : kWTile;
        __syncthreads();  // the previous tile's readers are done
        for (int i = threadIdx.x; i < tn; i += blockDim.x) {
          sh.tid[i] = adj[ra + t0 + i];
          sh.tw[i] = w[ra + t0 + i];
        }
        __syncthreads();
        const int32_t tlo = uniform(sh.tid[0]), hi = uniform(sh.tid[tn - 1]);
        // Buckets of 2^tsh ids from tlo: bucket b holds positions
        // [bst[b], bst[b + 1]) (every entry written once, by the position
        // that opens it, or by the last position for the empty tail).
        int tsh = 0;
        while (((hi - tlo) >> tsh) >= kWBuckets) ++tsh;
        const int32_t nb = ((hi - tlo) >> tsh) + 1;
        for (int i = threadIdx.x; i < tn; i += blockDim.x) {
          const int32_t bi = (sh.tid[i] - tlo) >> tsh;
          const int32_t bp = i > 0 ? (sh.tid[i - 1] - tlo) >> tsh : -1;
          for (int32_t b = bp + 1; b <= bi; ++b) sh.bst[b] = i;
          if (i == tn - 1)
            for (int32_t b = bi + 1; b <= nb; ++b) sh.bst[b] = tn;
        }
        __syncthreads();
        const bool last = t0 + kWTile >= dh;
        for (int32_t j = wave; j < nlow; j += kWWaves) {
          if (!last && uniform(sh.nxt[j]) > hi) continue;  // nothing of l's row up to hi is left
          const int64_t ou = uniform64(sh.lou[j]);
          const int32_t du = uniform(sh.ldu[j]), l = uniform(sh.lid[j]);
          int32_t c = uniform(sh.cur[j]), mp = uniform(sh.mpos[j]), nx = INT_MAX;
          bool ldone = uniform(sh.ldone[j]) != 0;
          const double whl = sh.whl[j];
          double acc = sh.acc[j];
          // One chunk of 64 positions from c: returns how many were in
          // range (a prefix) and sets nx when the range ended inside it.
          auto chunk = [&](int32_t xq, double wq) {
            const bool in = c + lane < du;
            const int32_t x = in ? xq : INT_MAX;
            const double wl = in ? wq : 0.0;
            const bool valid = in && (last || x <= hi);
            // lower_bound of x in its bucket (x outside [tlo, hi]: no hit)
            const bool inr = x >= tlo && x <= hi;
            int32_t lo = 0, len = 0;
            if (inr) {
              const int32_t b = (x - tlo) >> tsh;
              lo = sh.bst[b];
              len = sh.bst[b + 1] - lo;
            }
            while (len > 0) {
              const int32_t half = len >> 1;
              if (sh.tid[lo + half] < x) {
                lo += half + 1;
                len -= half + 1;
              } else {
                len = half;
              }
            }
            const bool hit = valid && inr && lo < tn && sh.tid[lo] == x;
            const bool selfh = valid && x == (int32_t)h;
            const double prod = hit ? sh.tw[lo] * wl : wl;  // x = h: w(h, h) = 1
            const int cnt = __popcll(__ballot(valid));      // the valid lanes are a prefix
            const uint64_t hm = __ballot(selfh);
            if (hm) mp = c + __ffsll((unsigned long long)hm) - 1;
            // The products of the common ids, in lane (= ascending id)
            // order; the x = l term goes before the first of them above l.
            uint64_t cm = __ballot(hit || selfh);
            uint64_t after = 0;
            if (!ldone) {
              const uint64_t above = __ballot((hit || selfh) && x > l);
              if (above) {
                after = cm & ~((1ull << (__ffsll((unsigned long long)above) - 1)) - 1ull);
                cm &= ~after;
              }
            }
            for (; cm; cm &= cm - 1) acc += lane_f64(prod, __ffsll((unsigned long long)cm) - 1);
            if (after) {
              acc += whl;
              ldone = true;
              for (cm = after; cm; cm &= cm - 1) acc += lane_f64(prod, __ffsll((unsigned long long)cm) - 1);
            }
            if (cnt < kWave && c + cnt < du) nx = __builtin_amdgcn_readlane(x, cnt);
            return cnt;
          };
          // kWChunks chunks' loads are issued together (clamped into the
          // row, so unconditionally), then the chunks are taken in order.
          bool more = c < du;
          while (more) {
            int32_t xq[kWChunks];
            double wq[kWChunks];
#pragma unroll
            for (int u = 0; u < kWChunks; ++u) {
              const int32_t p = c + u * kWave + lane;
              const int64_t q = ou + (p < du ? p : du - 1);
              xq[u] = adj[q];
              wq[u] = w[q];
            }
#pragma unroll
            for (int u = 0; u < kWChunks; ++u) {
              if (more) {
                const int cnt = chunk(xq[u], wq[u]);
                c += cnt;
                more = cnt == kWave && c < du;
              }
            }
          }
          if (lane == 0) {
            sh.cur[j] = c;
            sh.nxt[j] = nx;
            sh.mpos[j] = mp;
            sh.ldone[j] = ldone ? 1 : 0;
            sh.acc[j] = acc;
          }
        }
      }
      __syncthreads();
      for (int32_t j = threadIdx.x; j < nlow; j += blockDim.x) {
        double acc = sh.acc[j];
        if (!sh.ldone[j]) acc += sh.whl[j];  // l is above every common id
        const int32_t l = sh.lid[j];
        const double x = acc / sqrt(S[h] * S[l]);
        sims[ra + sh.le[j]] = x;
        if (sh.mpos[j] >= 0) sims[sh.lou[j] + sh.mpos[j]] = x;
      }
      __syncthreads();  // before the next row reuses the arrays
    }
    ++h;
    if (h >= n) break;
  }
}

// err[0] = 1 if any weight is not finite.
__global__ void k_w_check(const double *w, int64_t nnz, int32_t *err) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * blockDim.x)
    if (!isfinite(w[i])) err[0] = 1;
}

}  // namespace

scan_status check_weights(const double *w, int64_t nnz, DevArena &tmp, hipStream_t s) {
  if (nnz == 0) return SCAN_OK;
  int32_t *d_err;
  SCAN_TRY(tmp.alloc(&d_err, 1));
  SCAN_HIP_TRY(hipMemsetAsync(d_err, 0, 4, s));
  k_w_check<<<grid_for(nnz, 256), 256, 0, s>>>(w, nnz, d_err);
  int32_t herr = 0;
  SCAN_HIP_TRY(hipMemcpyAsync(&herr, d_err, 4, hipMemcpyDeviceToHost, s));
  SCAN_HIP_TRY(hipStreamSynchronize(s));
  if (herr) return fail(SCAN_EGRAPH, "edge weights must be finite");
  return SCAN_OK;
}

// The bitmap path holds one id window and addresses the weights by 32-bit
// byte offsets; larger graphs take k_w_owner.
bool weighted_planned(int64_t n, int64_t nnz) {
  return n <= ((int64_t)1 << kWbMaxBits) && nnz * 8 < (int64_t)0xfffffff8u;
}
IntersectConfig weighted_config(const IntersectConfig &cfg) {
  IntersectConfig c = cfg;
  c.small_max = kWbSmallMax;
  c.spc = kWbSpc;
  c.wbits = kWbMaxBits;
  c.auto_shapes = false;
  return c;
}

static scan_status weighted_by_plan(const IntersectPlan &plan, int64_t n, int64_t nnz, const int64_t *off, const int32_t *deg,
                                    const int32_t *adj, const double *w, const double *S, double *sims, int device,
                                    hipStream_t s, int32_t skip) {
  const PlanCounts c = *(const PlanCounts *)plan.host;
  int wbits = 10;
  while (((int64_t)1 << wbits) < n) ++wbits;
  const size_t lds = w_big_lds(wbits);
  int lds_max = 65536, cus = 256;
  (void)hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, device);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  if (lds > (size_t)lds_max) return fail(SCAN_EDEVICE, "the weighted bitmap needs %zu bytes of LDS", lds);
  // As in the unweighted path: the persistent large-owner kernel first, the
  // small owners' on helper streams (ordered after the square sums).
  auto fork = [&](int k) -> hipStream_t {
    if (!c.big || !plan.helper[k] || stream_wait(plan.helper[k], s) != SCAN_OK) return s;
    return plan.helper[k];
  };
  const hipStream_t sh = fork(0), sl = fork(1);
  JoinOnExit join_sh{s, sh}, join_sl{s, sl};
  if (c.big) {
    SCAN_HIP_TRY(hipFuncSetAttribute((const void *)k_w_big, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int per_cu = (int)std::min<size_t>(2, (size_t)lds_max / lds);
    k_w_big<<<(unsigned)std::min<int64_t>((int64_t)cus * per_cu, c.big), kWbThreads, lds, s>>>(
        (const BigChunk *)plan.big_list, (PlanCounts *)plan.counts, wbits, off, deg, adj, w, nnz, S, sims, skip);
  }
  constexpr int kHeavyWaves = 4;
  if (c.heavy)
    k_w_small<kHeavyWaves><<<c.heavy, kHeavyWaves * kWave, w_small_lds(kWbSmallMax), sh>>>(
        plan.lists + (n - c.heavy), kWbSmallMax, off, deg, adj, w, S, sims, skip);
  if (c.small)
    k_w_small<1><<<c.small, kWave, w_small_lds(kLightDeg), sl>>>(plan.lists, kLightDeg, off, deg, adj, w, S,
                                                                 sims, skip);
  SCAN_HIP_TRY(hipGetLastError());
  return SCAN_OK;
}

scan_status weighted_similarity_all(int64_t n, int64_t nnz, const int64_t *off, const int32_t *deg,
                                    const int32_t *adj, const double *w, double *sims, DevArena &tmp,
                                    hipStream_t s, const IntersectStats *stats, const IntersectPlan *plan,
                                    int device, int32_t skip_deg) {
  auto mark = [&](hipEvent_t e) -> scan_status {
    if (e) SCAN_HIP_TRY(hipEventRecord(e, s));
    return SCAN_OK;
  };
  SCAN_TRY(mark(stats ? stats->ev_small_begin : nullptr));
  if (nnz > 0) {
    const int64_t units = (nnz + kWUnit - 1) / kWUnit;
    if (units > INT_MAX) return fail(SCAN_EINVAL, "graph too large for the weighted path");
    double *S;
    int32_t *row_of;
    SCAN_TRY(tmp.alloc(&S, n));
    k_w_square_sums<<<grid_for(n * 16, 256), 256, 0, s>>>(off, adj, w, n, S);
    SCAN_HIP_TRY(hipGetLastError());
    SCAN_TRY(mark(stats ? stats->ev_small_end : nullptr));
    SCAN_TRY(mark(stats ? stats->ev_big_begin : nullptr));
    if (plan) {
      SCAN_TRY(weighted_by_plan(*plan, n, nnz, off, deg, adj, w, S, sims, device, s, skip_deg));
    } else {
      SCAN_TRY(tmp.alloc(&row_of, units));
      k_w_unit_rows<<<grid_for(n, 256), 256, 0, s>>>(off, n, row_of);
      k_w_owner<<<(unsigned)units, kWThreads, 0, s>>>(off, deg, adj, w, S, row_of, n, nnz, sims, skip_deg);
    }
    SCAN_HIP_TRY(hipGetLastError());
    tmp.drop(S);
  } else {
    SCAN_TRY(mark(stats ? stats->ev_small_end : nullptr));
    SCAN_TRY(mark(stats ? stats->ev_big_begin : nullptr));
  }
  SCAN_TRY(mark(stats ? stats->ev_big_end : nullptr));
  return SCAN_OK;
}

}  // namespace scan
