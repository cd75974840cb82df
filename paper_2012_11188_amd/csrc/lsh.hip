// Approximate similarities (Section 5) with the degree heuristic of Section
// 6.3: only edges between two high-degree vertices (degree > k for cosine,
// > 3k/2 for Jaccard) are approximated; every other edge keeps the exact
// similarity computed before this pass. The random draws are inputs.
//
//   SimHash (cosine, optionally weighted): bit i of v's sketch is 1 iff the
//   dot product of N[v] (weights w(v, x), w(v, v) = 1) with direction i,
//   gauss[x * k + i], is >= 0, the dot product summed term by term in
//   ascending x. Estimate cos(pi h / k) for h differing bits, read from a
//   table of the k + 1 values computed once on the host.
//   k-partition MinHash (Jaccard): bin(x) = floor(perm[x] * k / n); entry b of
//   v's sketch is the least perm[x] over x in N[v] in bin b (0xffffffff when
//   none). Estimate: matching non-empty bins / (k - bins empty in both).
//
//   k_simhash_big  workgroups resident on every CU claim (high vertex, group
//                of 64 directions) items from a counter; per item its
//                wavefronts gather the coordinates of kShChunk row entries
//                into LDS, then one of them adds them in ascending x (lane i:
//                direction g * 64 + i); the signs form one 64-bit word by
//                ballot.
//   k_minhash    one workgroup per high vertex: k bins in LDS, atomicMin of
//                perm[x] over N[v].
//   k_estimate   one wavefront per piece of 64 slots of a high vertex's row
//                (pieces numbered by a prefix over the vertices): the slots
//                whose other end is high too are overwritten.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <vector>

#include "index.h"

namespace scan {
namespace {

constexpr int kLshThreads = 256;
constexpr int kLshWaves = kLshThreads / kWave;
constexpr int kLshPiece = 64;  // row slots per estimate work item
constexpr int kShChunk = 64;     // row entries staged in LDS per round of the block kernel
constexpr int kShThreads = 256;
constexpr int kShUnroll = 8;     // entries whose LDS values the summing wave reads ahead
constexpr int kShWaves = kShThreads / kWave;
constexpr int kMhGroup = 16;   // lanes comparing one pair of MinHash sketches
constexpr int kMhHeld = 256;   // bins of u's sketch that a group keeps in registers
constexpr int kMhPairs = 2;    // pairs whose sketches a group reads at once

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ bool high(int kind, int64_t deg, int64_t k) {
  return kind == SCAN_SIM_JACCARD ? 2 * deg > 3 * k : deg > k;
}

// The high vertices: those of degree above kLshLong to big[0, nhigh[0]), the
// others to big[n - nhigh[1], n), one reservation per wavefront and class.
constexpr int64_t kLshLong = 4096;
__global__ __launch_bounds__(256) void k_high_list(const int64_t *off, int64_t n, int kind, int32_t k, int32_t *big,
                                                   int32_t *nhigh) {
  const int lane = lane_id();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) - lane; v0 < n; v0 += stride) {
    const int64_t v = v0 + lane;
    const int64_t d = v < n ? off[v + 1] - off[v] : 0;
    const bool in = v < n && high(kind, d, k);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const bool mine = in && (d > kLshLong) == (c == 0);
      const uint64_t m = __ballot(mine);
      int32_t at = 0;
      if (m && lane == 0) at = atomicAdd(&nhigh[c], __popcll(m));
      at = uniform(at) + __popcll(m & ((1ull << lane) - 1));
      if (mine) big[c == 0 ? at : n - 1 - at] = (int32_t)v;
    }
  }
}
__device__ __forceinline__ int32_t high_vertex(const int32_t *big, int64_t n, int64_t nlong, int64_t i) {
  return i < nlong ? big[i] : big[n - 1 - (i - nlong)];
}

// SimHash words, words[v * (k / 64) + g] with bit i for direction g * 64 + i:
// one item per (high vertex, group of 64 directions). The long rows' items
// come first (their sums are the longest serial chains); the others go group
// by group, so that at any time the gathers fall into one group's 512 bytes
// per vertex, whose often-met rows stay in the
// last-level cache. R-MAT-20, k = 256 (41 GB of gathers): 8.1 ms vertex by
// vertex, 7.0 group by group, 5.95 with each round's gathers requested before
// the sum of the round before it. The grid is what the
// CUs hold at once, and each workgroup claims its next item from *claim as
// soon as it is done (item sizes follow the degrees, so a static split would
// leave most workgroups idle behind the longest lists). Per round, all waves
// gather the coordinates of kShChunk row entries into LDS (a wave's gathers
// are issued back to back, so hundreds are in flight at once), then wave 0
// adds them in ascending order, lane i for direction g * 64 + i, with the
// self term at its place.
__global__ __launch_bounds__(kShThreads) void k_simhash_big(const int64_t *off, const int32_t *adj, const double *w,
                                                            const double *gauss, int64_t n, int32_t k,
                                                            const int32_t *big, const int32_t *nhigh,
                                                            unsigned long long *claim, uint64_t *words) {
  extern __shared__ double st[];           // [kShChunk][64] coordinates
  __shared__ int32_t sid[kShChunk];        // the entries' ids
  __shared__ double sw[kShChunk];          // and weights
  __shared__ int64_t s_item;
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const int32_t groups = k / kWave;
  const int64_t nlong = uniform(nhigh[0]), nrest = uniform(nhigh[1]);
  const int64_t items = (nlong + nrest) * groups;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int64_t)atomicAdd(claim, 1ull);
    __syncthreads();
    const int64_t t = s_item;
    if (t >= items) break;  // uniform across the block
    const int64_t r = t - nlong * groups;
    const int64_t v = high_vertex(big, n, nlong, r < 0 ? t / groups : nlong + r % nrest);
    const int32_t g = (int32_t)(r < 0 ? t % groups : r / nrest);
    const int64_t o = uniform64(off[v]), d = uniform64(off[v + 1]) - o;
    const double *col = gauss + g * kWave + lane;
    const double gself = col[v * (int64_t)k];  // the self term's coordinate
    double acc = 0.0;
    bool self = false;
    // Entries wave, wave + kShWaves, ... of a round: ids by one vector load
    // (and weights), then every gather of the wave. A round's gathers are
    // requested before the round before it is summed, its ids one round
    // earlier still, so that the sums wait for neither.
    constexpr int kPer = kShChunk / kShWaves;
    const int jl = wave + kShWaves * lane;  // the entry whose id this lane loads (lanes below kPer)
    auto fetch_ids = [&](int64_t c, int32_t &x, double &wx) {
      const int64_t p = lane < kPer && c + jl < d ? c + jl : d - 1;  // (past the row: its last entry again)
      x = adj[o + p];
      wx = w ? w[o + p] : 1.0;
    };
    auto gather = [&](int32_t x, double gv[kPer]) {
#pragma unroll
      for (int q = 0; q < kPer; ++q) gv[q] = col[(int64_t)__builtin_amdgcn_readlane(x, q) * k];
    };
    int32_t x0, x1;
    double w0, w1, gv[kPer];
    fetch_ids(0, x0, w0);
    gather(x0, gv);
    fetch_ids(kShChunk, x1, w1);
    for (int64_t c = 0; c < d; c += kShChunk) {
      const int m = (int)(d - c < kShChunk ? d - c : kShChunk);
      __syncthreads();  // the previous round's readers are done
      if (lane < kPer) {
        sid[jl] = x0;
        sw[jl] = w0;
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) st[(wave + kShWaves * q) * kWave + lane] = gv[q];
      x0 = x1;
      w0 = w1;
      if (c + kShChunk < d) {
        gather(x0, gv);
        fetch_ids(c + 2 * kShChunk, x1, w1);
      }
      __syncthreads();
      if (wave == 0) {
        for (int j0 = 0; j0 < m; j0 += kShUnroll) {
          int32_t xs[kShUnroll];
          double ws[kShUnroll], gs[kShUnroll];
#pragma unroll
          for (int u = 0; u < kShUnroll; ++u) {  // entries past m are not added
            xs[u] = sid[j0 + u];
            ws[u] = sw[j0 + u];
            gs[u] = st[(j0 + u) * kWave + lane];
          }
#pragma unroll
          for (int u = 0; u < kShUnroll; ++u) {
            if (j0 + u < m) {
              if (!self && xs[u] > v) {
                acc += 1.0 * gself;
                self = true;
              }
              acc += ws[u] * gs[u];
            }
          }
        }
      }
    }
    if (wave == 0) {
      if (!self) acc += 1.0 * gself;
      const uint64_t bits = __ballot(acc >= 0.0);
      if (lane == 0) words[v * groups + g] = bits;
    }
    __syncthreads();  // every thread has read s_item before the next claim
  }
}

// sk[v * k + b]: a workgroup per high vertex, its bins in LDS (minima: any
// order gives the same sketch), so that a hub's row is read by all of its
// wavefronts. (With a wavefront per vertex the longest row, 65k entries, held
// the kernel: 830 us on R-MAT-20 with k = 256; this takes
// 280.)
constexpr int kMhThreads = 512;
constexpr int kMhSteps = 4;  // entries per thread requested together
__global__ __launch_bounds__(kMhThreads) void k_minhash(const int64_t *off, const int32_t *adj, const uint32_t *perm,
                                                        int64_t n, int32_t k, const int32_t *big,
                                                        const int32_t *nhigh, unsigned long long *claim,
                                                        uint32_t *sk) {
  extern __shared__ uint32_t bins[];  // [k]
  __shared__ int64_t s_item;
  const int64_t nlong = uniform(nhigh[0]), items = nlong + uniform(nhigh[1]);
  for (;;) {
    if (threadIdx.x == 0) s_item = (int64_t)atomicAdd(claim, 1ull);
    for (int32_t b = threadIdx.x; b < k; b += kMhThreads) bins[b] = 0xffffffffu;
    __syncthreads();
    const int64_t t = s_item;
    if (t >= items) break;  // uniform across the block
    const int64_t v = high_vertex(big, n, nlong, t);
    const int64_t o = off[v], d = off[v + 1] - o;
    for (int64_t c = threadIdx.x; c <= d; c += kMhSteps * kMhThreads) {  // position d is v itself
      int64_t x[kMhSteps];
      uint32_t px[kMhSteps];
#pragma unroll
      for (int j = 0; j < kMhSteps; ++j) {
        const int64_t p = c + j * kMhThreads;
        x[j] = p < d ? adj[o + p] : v;
      }
#pragma unroll
      for (int j = 0; j < kMhSteps; ++j) px[j] = perm[x[j]];  // (past the row: v again, which is in the set)
#pragma unroll
      for (int j = 0; j < kMhSteps; ++j) {
        if (c + j * kMhThreads <= d) atomicMin(&bins[(uint64_t)px[j] * (uint64_t)k / (uint64_t)n], px[j]);
      }
    }
    __syncthreads();
    for (int32_t b = threadIdx.x; b < k; b += kMhThreads) sk[v * k + b] = bins[b];
    __syncthreads();  // the bins and s_item are reused
  }
}

// cnt[u] = pieces of kLshPiece slots of u's row when u is high, else 0.
__global__ void k_lsh_pieces(const int64_t *off, int64_t n, int kind, int32_t k, int32_t *cnt) {
  for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
    const int64_t d = off[u + 1] - off[u];
    cnt[u] = high(kind, d, k) ? (int32_t)((d + kLshPiece - 1) / kLshPiece) : 0;
  }
}

// One wavefront per piece (P = exclusive prefix of the pieces, P[n] their
// number): the piece's slots whose other end is high too get the estimate.
// SimHash: a lane per slot. MinHash: four groups of 16 lanes, a group per
// slot; lane l of a group compares bins 4 (l + 16 i) .. 4 (l + 16 i) + 3, so
// each load instruction of a group reads 256 contiguous bytes of a sketch.
__global__ __launch_bounds__(kLshThreads) void k_estimate(const int64_t *off, const int32_t *adj, int64_t n,
                                                          int kind, int32_t k, const int64_t *P,
                                                          const uint64_t *words, const uint32_t *sk,
                                                          const double *table, double *sims) {
  __shared__ int32_t list[kLshWaves][kWave];
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const int64_t waves = (int64_t)gridDim.x * kLshWaves;
  const int64_t T = uniform64(P[n]);
  for (int64_t t = uniform64(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave); t < T; t += waves) {
    // the u with P[u] <= t < P[u + 1]: the last one with P[u] <= t, by a
    // 64-way search (every lane samples one position)
    int64_t lo = 0, cnt = n;
    while (cnt > 1) {
      const int64_t step = (cnt + kWave - 1) / kWave;
      const int64_t q = lo + lane * step;
      const int c = __popcll(__ballot(q < lo + cnt && P[q] <= t));  // >= 1: lane 0
      const int64_t nlo = lo + (c - 1) * step;
      cnt = min(step, lo + cnt - nlo);
      lo = nlo;
    }
    const int64_t u = lo, o = uniform64(off[u]), d = uniform64(off[u + 1]) - o;
    const int64_t p0 = (t - uniform64(P[u])) * kLshPiece;
    if (kind != SCAN_SIM_JACCARD) {
      const int64_t p = p0 + lane;
      if (p < d && p < p0 + kLshPiece) {
        const int64_t v = adj[o + p];
        if (high(kind, off[v + 1] - off[v], k)) {
          const int32_t groups = k / kWave;
          int32_t h = 0;
          for (int32_t i = 0; i < groups; ++i) h += __popcll(words[u * groups + i] ^ words[v * groups + i]);
          sims[o + p] = table[h];
        }
      }
      continue;
    }
    // The slots to compare, listed in lane order. u's sketch stays in
    // registers for the piece where it fits (kMhHeld bins).
    const int32_t v = p0 + lane < d ? adj[o + p0 + lane] : 0;
    const bool on = p0 + lane < d && high(kind, off[v + 1] - off[v], k);
    const uint64_t todo = __ballot(on);
    const int count = __popcll(todo);
    if (on) list[wave][__popcll(todo & ((1ull << lane) - 1))] = lane;
    const int grp = lane / kMhGroup, gl = lane % kMhGroup;
    const uint4 *a = (const uint4 *)(sk + u * k);
    constexpr int kHeld = kMhHeld / 4 / kMhGroup;
    uint4 ha[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) ha[i] = a[min(gl + i * kMhGroup, k / 4 - 1)];
    auto compare = [](const uint4 &ea, const uint4 &eb, int32_t &match, int32_t &empty) {
      const uint32_t av[4] = {ea.x, ea.y, ea.z, ea.w}, bv[4] = {eb.x, eb.y, eb.z, eb.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool same = av[j] == bv[j];
        empty += same && av[j] == 0xffffffffu ? 1 : 0;
        match += same ? 1 : 0;  // (the empty ones come off below)
      }
    };
    for (int r = 0; r < count; r += kWave / kMhGroup * kMhPairs) {
      const uint4 *b[kMhPairs];
      int src[kMhPairs];
      uint4 eb[kMhPairs][kHeld];
      int32_t match[kMhPairs], empty[kMhPairs];
#pragma unroll
      for (int q = 0; q < kMhPairs; ++q) {
        src[q] = list[wave][min(r + q * (kWave / kMhGroup) + grp, count - 1)];
        b[q] = (const uint4 *)(sk + (int64_t)__shfl(v, src[q], kWave) * k);
#pragma unroll
        for (int i = 0; i < kHeld; ++i) eb[q][i] = b[q][min(gl + i * kMhGroup, k / 4 - 1)];
      }
#pragma unroll
      for (int q = 0; q < kMhPairs; ++q) {
        match[q] = empty[q] = 0;
#pragma unroll
        for (int i = 0; i < kHeld; ++i)
          if (gl + i * kMhGroup < k / 4) compare(ha[i], eb[q][i], match[q], empty[q]);
        for (int32_t i = gl + kHeld * kMhGroup; i < k / 4; i += kMhGroup) compare(a[i], b[q][i], match[q], empty[q]);
#pragma unroll
        for (int m = kMhGroup / 2; m > 0; m >>= 1) {  // sums over the group (all lanes take part)
          match[q] += __shfl_xor(match[q], m, kWave);
          empty[q] += __shfl_xor(empty[q], m, kWave);
        }
        if (gl == 0 && r + q * (kWave / kMhGroup) + grp < count)
          sims[o + p0 + src[q]] = (double)(match[q] - empty[q]) / (double)(k - empty[q]);
      }
    }
  }
}

// err[0] = 1 if some perm value is not below n.
__global__ void k_perm_check(const uint32_t *perm, int64_t n, int32_t *err) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    if ((int64_t)perm[i] >= n) err[0] = 1;
}

}  // namespace

scan_status lsh_overwrite(const LshSpec &spec, int64_t n, int64_t nnz, const int64_t *off, const int32_t *adj,
                          const double *w, int kind, double *sims, DevArena &tmp, hipStream_t s) {
  const int32_t k = spec.samples;
  if (n == 0 || nnz == 0) return SCAN_OK;
  uint64_t *words = nullptr;
  uint32_t *sk = nullptr;
  double *table = nullptr;
  int device = 0, cus = 256;
  (void)hipGetDevice(&device);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  int32_t *big, *nhigh;  // the high vertices, and the numbers of long and other ones
  unsigned long long *claim;
  SCAN_TRY(tmp.alloc(&big, n));
  SCAN_TRY(tmp.alloc(&nhigh, 2));
  SCAN_TRY(tmp.alloc(&claim, 1));
  SCAN_HIP_TRY(hipMemsetAsync(nhigh, 0, 8, s));
  SCAN_HIP_TRY(hipMemsetAsync(claim, 0, 8, s));
  k_high_list<<<grid_for(n, 256, 2048), 256, 0, s>>>(off, n, kind, k, big, nhigh);
  if (kind == SCAN_SIM_JACCARD) {
    int32_t *d_err;
    SCAN_TRY(tmp.alloc(&d_err, 1));
    SCAN_HIP_TRY(hipMemsetAsync(d_err, 0, 4, s));
    k_perm_check<<<grid_for(n, 256), 256, 0, s>>>(spec.perm, n, d_err);
    int32_t herr = 0;
    SCAN_HIP_TRY(hipMemcpyAsync(&herr, d_err, 4, hipMemcpyDeviceToHost, s));
    SCAN_HIP_TRY(hipStreamSynchronize(s));
    if (herr) return fail(SCAN_EINVAL, "MinHash permutation values must lie in [0, n)");
    SCAN_TRY(tmp.alloc(&sk, n * (int64_t)k));
    k_minhash<<<cus * 4, kMhThreads, (size_t)k * 4, s>>>(off, adj, spec.perm, n, k, big, nhigh, claim, sk);
  } else {
    std::vector<double> t(k + 1);
    for (int32_t h = 0; h <= k; ++h) t[h] = std::cos(M_PI * (double)h / (double)k);
    SCAN_TRY(tmp.alloc(&table, k + 1));
    SCAN_HIP_TRY(hipMemcpyAsync(table, t.data(), t.size() * 8, hipMemcpyHostToDevice, s));
    SCAN_TRY(tmp.alloc(&words, n * (int64_t)(k / kWave)));
    const size_t lds = (size_t)kShChunk * kWave * 8;
    SCAN_HIP_TRY(hipFuncSetAttribute((const void *)k_simhash_big, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_simhash_big, kShThreads, lds) !=
            hipSuccess ||
        per_cu < 1) {
      (void)hipGetLastError();
      per_cu = 1;
    }
    k_simhash_big<<<cus * per_cu, kShThreads, lds, s>>>(off, adj, w, spec.gauss, n, k, big, nhigh, claim, words);
  }
  int32_t *cnt;
  int64_t *P, *ws;
  SCAN_TRY(tmp.alloc(&cnt, n));
  SCAN_TRY(tmp.alloc(&P, n + 1));
  SCAN_TRY(tmp.alloc(&ws, scan_workspace_elems(n)));
  k_lsh_pieces<<<grid_for(n, 256), 256, 0, s>>>(off, n, kind, k, cnt);
  SCAN_TRY(exclusive_scan(cnt, P, n, ws, s));
  k_estimate<<<grid_for(n * kWave / 16, kLshThreads), kLshThreads, 0, s>>>(off, adj, n, kind, k, P, words, sk, table,
                                                                          sims);
  SCAN_HIP_TRY(hipGetLastError());
  if (kind != SCAN_SIM_JACCARD) SCAN_HIP_TRY(hipStreamSynchronize(s));  // the host table stays alive until here
  return SCAN_OK;
}

}  // namespace scan
