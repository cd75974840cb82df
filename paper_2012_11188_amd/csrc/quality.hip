// Clustering quality on the device: the modularity of Section 7.2 (Newman's
// definition) with every unclustered vertex in a cluster of its own, the
// score by which Section 7.3.4 selects (mu, eps).
//
//   Q = 1/(2m) * sum over ordered pairs (u, v) of (A_uv - d_u d_v / 2m) delta_uv
//     = (s_in - sd2 / 2m) / 2m,
//   s_in = ordered neighbour pairs inside one cluster (a count of CSR slots),
//   sd2  = sum over clusters of (sum of degrees in the cluster)^2.
//
// Both terms are integers and are accumulated exactly (int64 atomics), so the
// host's final FP64 step gives the same bits as any other exact evaluation.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "index.h"

namespace scan {

constexpr int kModThreads = 256;
constexpr int kModGroup = 8;          // lanes per vertex
constexpr int64_t kModGroupMax = 512;  // longer rows: the whole wavefront
constexpr int kModSteps = 8;

static __device__ __forceinline__ int64_t block_sum64(int64_t v, int64_t *wsum) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int m = kWave / 2; m > 0; m >>= 1) {
    const int32_t lo = __shfl_xor((int32_t)(uint32_t)v, m, kWave);
    const int32_t hi = __shfl_xor((int32_t)(v >> 32), m, kWave);
    v += (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
  }
  __syncthreads();
  if (lane == 0) wsum[wave] = v;
  __syncthreads();
  int64_t t = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kModThreads / kWave; ++w) t += wsum[w];
  return t;  // thread 0
}

// The sums per cluster label of one workgroup: a direct-mapped table in LDS
// (an entry is claimed by the first label that needs it; a label that finds
// its entry taken adds to memory), written out at the end. One add per vertex
// to memory serialised on the labels of large clusters (100k-vertex R-MAT
// graph, one large cluster: 133 us a clustering, 16 us with the table).
constexpr int kModTable = 256;

// Clustering blockIdx.y of a batch: s_in, and per cluster label the degree
// sum (dsum, zero on entry); unclustered vertices add their squared degree to
// terms[1] directly. (terms[2] counts memberships outside [-1, n).)
__global__ __launch_bounds__(kModThreads) void k_mod_rows(const int64_t *off, const int32_t *ids, int64_t n,
                                                          const int32_t *memb_all, int64_t *dsum_all,
                                                          int64_t *terms_all) {
  __shared__ int64_t wsum[kModThreads / kWave];
  __shared__ int32_t key[kModTable];
  __shared__ unsigned long long sum[kModTable];
  const int32_t *memb = memb_all + (int64_t)blockIdx.y * n;
  int64_t *dsum = dsum_all + (int64_t)blockIdx.y * n, *terms = terms_all + 3 * (int64_t)blockIdx.y;
  for (int i = threadIdx.x; i < kModTable; i += kModThreads) {
    key[i] = -1;
    sum[i] = 0;
  }
  __syncthreads();
  auto add_degree = [&](int32_t c, int64_t d) {
    const int at = (int)(((uint32_t)c * 2654435761u) >> 24);
    static_assert(kModTable == 256, "the hash keeps 8 bits");
    const int32_t old = atomicCAS(&key[at], -1, c);
    if (old == -1 || old == c) atomicAdd(&sum[at], (unsigned long long)d);
    else atomicAdd((unsigned long long *)&dsum[c], (unsigned long long)d);
  };
  constexpr int kPerWave = kWave / kModGroup;
  const int lane = threadIdx.x & (kWave - 1), pos = lane % kModGroup;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) / kWave;
  int64_t in = 0, sq = 0;  // this lane's shares
  for (int64_t v0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave * kPerWave; v0 < n;
       v0 += nw * kPerWave) {
    const int64_t v = v0 + lane / kModGroup;
    int64_t b = 0, e = 0;
    int32_t c = -1;
    if (v < n) {
      c = memb[v];
      b = off[v];
      e = off[v + 1];
      if (c >= n || c < -1) {  // not a label of this graph: reported, counted as unclustered
        if (pos == 0) atomicAdd((unsigned long long *)&terms[2], 1ull);
        c = -1;
      }
      if (pos == 0) {
        if (c >= 0) add_degree(c, e - b);
        else sq += (e - b) * (e - b);
      }
    }
    if (c >= 0 && e - b <= kModGroupMax) {  // the same for every lane of the group
      // kModSteps steps' ids, then their labels, requested together
      for (int64_t k0 = b + pos; k0 < e; k0 += kModSteps * kModGroup) {
        int32_t w[kModSteps];
#pragma unroll
        for (int j = 0; j < kModSteps; ++j) {
          const int64_t k = k0 + j * kModGroup;
          w[j] = k < e ? ids[k] : -1;
        }
#pragma unroll
        for (int j = 0; j < kModSteps; ++j) in += (w[j] >= 0 && memb[w[j]] == c) ? 1 : 0;
      }
    }
    // long clustered rows: one at a time by the whole wavefront
    uint64_t longs = __ballot(c >= 0 && e - b > kModGroupMax && pos == 0);
    while (longs) {
      const int src = __ffsll((unsigned long long)longs) - 1;
      longs &= longs - 1;
      const int64_t rb = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)b, src) |
                         ((int64_t)__builtin_amdgcn_readlane((int32_t)(b >> 32), src) << 32);
      const int64_t re = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)e, src) |
                         ((int64_t)__builtin_amdgcn_readlane((int32_t)(e >> 32), src) << 32);
      const int32_t rc = __builtin_amdgcn_readlane(c, src);
      for (int64_t k0 = rb; k0 < re; k0 += kModSteps * kWave) {
        int32_t w[kModSteps];
#pragma unroll
        for (int j = 0; j < kModSteps; ++j) {
          const int64_t k = k0 + j * kWave + lane;
          w[j] = k < re ? ids[k] : -1;
        }
#pragma unroll
        for (int j = 0; j < kModSteps; ++j) in += (w[j] >= 0 && memb[w[j]] == rc) ? 1 : 0;
      }
    }
  }
  const int64_t bin = block_sum64(in, wsum);
  const int64_t bsq = block_sum64(sq, wsum);  // (its barriers also order the table's adds before the reads below)
  if (threadIdx.x == 0) {
    if (bin) atomicAdd((unsigned long long *)&terms[0], (unsigned long long)bin);
    if (bsq) atomicAdd((unsigned long long *)&terms[1], (unsigned long long)bsq);
  }
  for (int i = threadIdx.x; i < kModTable; i += kModThreads)
    if (key[i] >= 0 && sum[i]) atomicAdd((unsigned long long *)&dsum[key[i]], sum[i]);
}

// sd2 += dsum[c]^2 over every label, and dsum is cleared for the next call.
__global__ __launch_bounds__(kModThreads) void k_mod_squares(int64_t *dsum_all, int64_t n, int64_t *terms_all) {
  __shared__ int64_t wsum[kModThreads / kWave];
  int64_t *dsum = dsum_all + (int64_t)blockIdx.y * n, *terms = terms_all + 3 * (int64_t)blockIdx.y;
  int64_t sq = 0;
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n; c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t d = dsum[c];
    if (d) {
      sq += d * d;
      dsum[c] = 0;
    }
  }
  const int64_t b = block_sum64(sq, wsum);
  if (threadIdx.x == 0 && b) atomicAdd((unsigned long long *)&terms[1], (unsigned long long)b);
}

// Many clusterings of one graph (a parameter sweep): kModLanes of them side
// by side, their labels transposed to T[v * kModLanes + l], so that one read
// of a neighbour's labels (128 consecutive bytes) serves them all; lane l of
// a half wavefront counts clustering l. One clustering at a time reads a
// scattered 4-byte label per slot and clustering (100k-vertex R-MAT graph, 32
// clusterings: 495 us; this way 128 + 28 + 8 us for the pairs, the degrees
// and the transpose, the pairs at the rate of scattered 128-byte reads).
constexpr int kModLanes = 32;
constexpr int kModUnit = 128;   // CSR slots per half wavefront (rows are cut, so no hub row is one lane's work)
constexpr int kModAhead = 8;    // neighbours' labels in flight

// T from memb[l * n + v], l < count; labels of the other lanes are -1.
__global__ __launch_bounds__(kModThreads) void k_mod_transpose(const int32_t *memb, int64_t n, int32_t count,
                                                               int32_t *T) {
  __shared__ int32_t t[kModLanes][kModLanes + 1];
  const int x = threadIdx.x % kModLanes, y = threadIdx.x / kModLanes;
  constexpr int kRows = kModThreads / kModLanes;
  for (int64_t v0 = (int64_t)blockIdx.x * kModLanes; v0 < n; v0 += (int64_t)gridDim.x * kModLanes) {
    for (int l = y; l < kModLanes; l += kRows) t[l][x] = l < count && v0 + x < n ? memb[l * n + v0 + x] : -1;
    __syncthreads();
    for (int v = y; v < kModLanes; v += kRows)
      if (v0 + v < n) T[(v0 + v) * kModLanes + x] = t[x][v];
    __syncthreads();
  }
}

// row_of[k] = the row holding slot k * kModUnit.
__global__ void k_mod_unit_rows(const int64_t *off, int64_t n, int32_t *row_of) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
    for (int64_t k = (off[v] + kModUnit - 1) / kModUnit; k * kModUnit < off[v + 1]; ++k) row_of[k] = (int32_t)v;
}

// s_in of every lane's clustering: terms[3 l] += ordered neighbour pairs with
// one label.
__global__ __launch_bounds__(kModThreads) void k_mod_pairs(const int64_t *off, const int32_t *ids,
                                                           const int32_t *row_of, int64_t nnz, const int32_t *T,
                                                           int32_t count, int64_t *terms) {
  __shared__ int64_t part[kModThreads / kModLanes][kModLanes];
  const int l = threadIdx.x % kModLanes, half = threadIdx.x / kModLanes, half_of_wave = half % (kWave / kModLanes);
  constexpr int kHalves = kModThreads / kModLanes;
  const int64_t units = (nnz + kModUnit - 1) / kModUnit;
  int64_t in = 0;
  for (int64_t k = (int64_t)blockIdx.x * kHalves + half; k < units; k += (int64_t)gridDim.x * kHalves) {
    const int64_t s1 = min(nnz, (k + 1) * kModUnit);
    int64_t v = row_of[k], s = k * kModUnit, e = off[v + 1];
    int32_t c = T[v * kModLanes + l];
    for (;;) {  // the half's lanes go through its slots together
      const int64_t end = min(e, s1);
      // a row that no clustering of the lanes holds is passed over
      const bool any = (uint32_t)(__ballot(c >= 0) >> (half_of_wave * kModLanes)) != 0;
      for (; any && s < end; s += kModLanes) {
        const int m = (int)min((int64_t)kModLanes, end - s);
        const int32_t id = ids[s + min(l, m - 1)];
        for (int j0 = 0; j0 < m; j0 += kModAhead) {
          int32_t lab[kModAhead];
#pragma unroll
          for (int j = 0; j < kModAhead; ++j)
            lab[j] = T[(int64_t)__shfl(id, j0 + j, kModLanes) * kModLanes + l];  // past m: the last id again
#pragma unroll
          for (int j = 0; j < kModAhead; ++j) in += (j0 + j < m && c >= 0 && lab[j] == c) ? 1 : 0;
        }
      }
      if (e >= s1) break;
      s = e;
      do e = off[++v + 1];
      while (e == s);  // rows without neighbours (s < s1 <= nnz: a later row holds slot s)
      c = T[v * kModLanes + l];
    }
  }
  part[half][l] = in;
  __syncthreads();
  if (half == 0) {
    for (int h = 1; h < kHalves; ++h) in += part[h][l];
    if (l < count && in) atomicAdd((unsigned long long *)&terms[3 * l], (unsigned long long)in);
  }
}

// Per lane's clustering: the degree sums of its labels (tables as in
// k_mod_rows, one per clustering) and the squared degrees of its unclustered
// vertices.
constexpr int kModSmallTable = 64;
__global__ __launch_bounds__(kModThreads) void k_mod_degrees(const int64_t *off, int64_t n, const int32_t *T,
                                                             int32_t count, int64_t *dsum, int64_t *terms) {
  __shared__ int32_t key[kModSmallTable][kModLanes];
  __shared__ unsigned long long sum[kModSmallTable][kModLanes];
  __shared__ int64_t part[kModThreads / kModLanes][kModLanes];
  const int l = threadIdx.x % kModLanes, half = threadIdx.x / kModLanes;
  constexpr int kHalves = kModThreads / kModLanes;
  for (int i = half; i < kModSmallTable; i += kHalves) {
    key[i][l] = -1;
    sum[i][l] = 0;
  }
  __syncthreads();
  int64_t sq = 0;
  for (int64_t v = (int64_t)blockIdx.x * kHalves + half; v < n && l < count; v += (int64_t)gridDim.x * kHalves) {
    const int32_t c = T[v * kModLanes + l];
    const int64_t d = off[v + 1] - off[v];
    if (c < 0) {
      sq += d * d;
    } else {
      const int at = (int)(((uint32_t)c * 2654435761u) >> 26);
      static_assert(kModSmallTable == 64, "the hash keeps 6 bits");
      const int32_t old = atomicCAS(&key[at][l], -1, c);
      if (old == -1 || old == c) atomicAdd(&sum[at][l], (unsigned long long)d);
      else atomicAdd((unsigned long long *)&dsum[(int64_t)l * n + c], (unsigned long long)d);
    }
  }
  part[half][l] = sq;
  __syncthreads();
  if (l >= count) return;
  if (half == 0) {
    for (int h = 1; h < kHalves; ++h) sq += part[h][l];
    if (sq) atomicAdd((unsigned long long *)&terms[3 * l + 1], (unsigned long long)sq);
  }
  for (int i = half; i < kModSmallTable; i += kHalves)
    if (key[i][l] >= 0 && sum[i][l]) atomicAdd((unsigned long long *)&dsum[(int64_t)l * n + key[i][l]], sum[i][l]);
}

__global__ void k_zero64(int64_t *p, int64_t count) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

void zero64(int64_t *p, int64_t count, hipStream_t s) {
  if (count > 0) k_zero64<<<grid_for(count, 256, 4096), 256, 0, s>>>(p, count);
}

void launch_modularity_terms(const scan_index *ix, const int32_t *memb, int32_t count, int64_t *dsum,
                             int64_t *terms, hipStream_t s) {
  const int64_t n = ix->n;
  // Workgroups per clustering: all of the chip for one, and few enough for a
  // batch that a workgroup's table of label sums is shared by many vertices.
  // No power of two: the vertices of a wavefront lie that many apart, and ids
  // that are multiples of a large power of two are often hubs, whose rows it
  // reads one after the other (R-MAT-20, 232,644 clustered vertices, 6,196 of
  // them with more than 512 neighbours, with 4,096 and 4,095: 1,538 and 883
  // us; one cluster of 1M vertices of a random graph 150 and 150).
  const int64_t cap = std::max<int64_t>(64, 4096 / count) - 1;
  const int64_t groups = (n + kWave / kModGroup - 1) / (kWave / kModGroup);
  k_mod_rows<<<dim3(grid_for(groups * kWave, kModThreads, cap), count), kModThreads, 0, s>>>(ix->off, ix->no_ids, n,
                                                                                            memb, dsum, terms);
  k_mod_squares<<<dim3(grid_for(n, kModThreads, std::max<int64_t>(64, 2048 / count)), count), kModThreads, 0, s>>>(
      dsum, n, terms);
}

scan_status plan_modularity_sweep(const scan_index *ix, DevArena &tmp, hipStream_t s, ModularitySweep *p) {
  SCAN_TRY(tmp.alloc(&p->T, ix->n * kModLanes));
  SCAN_TRY(tmp.alloc(&p->row_of, ix->nnz / kModUnit + 1));
  k_mod_unit_rows<<<grid_for(ix->n, kModThreads), kModThreads, 0, s>>>(ix->off, ix->n, p->row_of);
  return SCAN_OK;
}

void launch_modularity_sweep(const scan_index *ix, const ModularitySweep &p, const int32_t *memb, int32_t count,
                             int64_t *dsum, int64_t *terms, hipStream_t s) {
  const int64_t n = ix->n;
  constexpr int kHalves = kModThreads / kModLanes;
  for (int32_t i = 0; i < count; i += kModLanes) {
    const int32_t c = std::min<int32_t>(kModLanes, count - i);
    int64_t *t = terms + 3 * (int64_t)i, *ds = dsum + i * n;
    k_mod_transpose<<<grid_for(n, kModLanes, 4096), kModThreads, 0, s>>>(memb + i * n, n, c, p.T);
    k_mod_degrees<<<grid_for(n, kHalves, 1024), kModThreads, 0, s>>>(ix->off, n, p.T, c, ds, t);
    if (ix->nnz)
      k_mod_pairs<<<grid_for((ix->nnz + kModUnit - 1) / kModUnit, kHalves, 4096), kModThreads, 0, s>>>(
          ix->off, ix->no_ids, p.row_of, ix->nnz, p.T, c, t);
    k_mod_squares<<<dim3(grid_for(n, kModThreads, std::max<int64_t>(64, 4096 / c)), c), kModThreads, 0, s>>>(ds, n, t);
  }
}

double modularity_value(int64_t s_in, int64_t sd2, int64_t nnz) {
  if (nnz == 0) return 0.0;
  const double two_m = (double)nnz;
  return ((double)s_in - (double)sd2 / two_m) / two_m;
}

}  // namespace scan
