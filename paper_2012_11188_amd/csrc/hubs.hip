// Common neighbours among the highest-degree vertices by matrix product.
//
// Most of the min-side work of a skewed graph lies between its hubs: in an
// R-MAT graph of scale 20 the 8,000 vertices of highest degree own half of
// all streamed ids among themselves. Their rows are dense over the columns of
// high degree, so that part of the intersection is a contraction: with B the
// 0/1 matrix of hub rows (degree >= row_deg) by columns (degree >= col_deg),
// D = B B^T holds, for every pair of hubs, their common neighbours among the
// columns. The large-owner kernel then streams only what is left of a lower
// hub's row and starts its count at D.
//
//   k_hub_flags / k_hub_maps  rows and columns, numbered in id order (a prefix
//                   sum of packed flags)
//   k_hub_rows      a workgroup per hub row: its column bits, counts of them
//                   before every 128 columns, and the rest of its ids in order
//   k_hub_product   D on the matrix cores: the bits are expanded to FP4 values
//                   in registers (0 and 0.5, products of 0.25), accumulated in
//                   FP32, exact since every sum is a small multiple of 0.25
#include <hip/hip_runtime.h>

#include <algorithm>

#include "index.h"

namespace scan {
namespace {

constexpr int kRowThreads = 1024;
constexpr int kRowPer = 4;
constexpr int kTile = 256;      // rows and columns of D per workgroup (128 x 128 per wavefront)
constexpr int kColBlock = 256;  // columns per product step of a wavefront

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

__global__ void k_hub_flags(const int32_t *deg, int64_t n, int32_t row_deg, int32_t col_deg, int64_t *flags) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    const int32_t d = deg[v];
    flags[v] = (int64_t)(d >= col_deg) | (int64_t)(d >= row_deg) << 32;
  }
}

__global__ void k_hub_maps(const int32_t *deg, int64_t n, int32_t row_deg, int32_t col_deg, const int64_t *P,
                           VertexRecord *records, int32_t *col, int32_t *verts) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    const int32_t d = deg[v];
    const int64_t p = P[v];
    col[v] = d >= col_deg ? (int32_t)(uint32_t)p : -1;
    if (d >= row_deg) {
      records[v].hub = (int32_t)(p >> 32);
      verts[p >> 32] = (int32_t)v;
    }
  }
}

// Row r of B and the rest of its ids (of radj, the numbering that is
// streamed), in order; rows past K are zero. win: with several id windows,
// where the rest's windows start.
__global__ __launch_bounds__(kRowThreads) void k_hub_rows(HubView hub, const int32_t *verts, const int64_t *off,
                                                          const int32_t *adj, const int32_t *radj, int32_t wbits,
                                                          int32_t nwin, int32_t *win, unsigned long long *cursor) {
  __shared__ uint32_t bm[kHubMaxCols / 32];
  __shared__ int32_t count[kHubMaxWindows + 1];
  __shared__ int32_t wsum[2][kRowThreads / kWave];
  __shared__ int64_t s_base;
  const int t = threadIdx.x, lane = lane_id(), wave = t / kWave;
  const int32_t r = blockIdx.x, blocks = hub.cols / 128;
  const bool real = r < hub.rows;
  const int64_t o = real ? off[verts[r]] : 0;
  const int32_t d = real ? (int32_t)(off[verts[r] + 1] - o) : 0;
  for (int i = t; i < hub.cols / 32; i += kRowThreads) bm[i] = 0;
  if (t <= nwin) count[t] = 0;
  if (t == 0 && real) s_base = (int64_t)atomicAdd(cursor, (unsigned long long)d);
  __syncthreads();
  const int64_t base = real ? s_base : 0;
  int32_t *rest = const_cast<int32_t *>(hub.rest) + base;
  // kRowPer ids per thread and step: their loads, and then those of their
  // columns, are in flight together (R-MAT-20: 118 us, one at a time 172).
  int32_t len = 0;
  int buf = 0;
  for (int32_t i0 = 0; i0 < d; i0 += kRowThreads * kRowPer) {
    int32_t v[kRowPer], x[kRowPer], c[kRowPer];
#pragma unroll
    for (int j = 0; j < kRowPer; ++j) v[j] = adj[o + min(i0 + j * kRowThreads + t, d - 1)];
#pragma unroll
    for (int j = 0; j < kRowPer; ++j) x[j] = radj[o + min(i0 + j * kRowThreads + t, d - 1)];
#pragma unroll
    for (int j = 0; j < kRowPer; ++j) c[j] = hub.col[v[j]];
#pragma unroll
    for (int j = 0; j < kRowPer; ++j) {
      if (i0 + j * kRowThreads >= d) break;  // uniform
      const bool in = i0 + j * kRowThreads + t < d, keep = in && c[j] < 0;
      if (in && !keep) atomicOr(&bm[c[j] >> 5], 1u << (c[j] & 31));
      if (keep && nwin > 1) atomicAdd(&count[x[j] >> wbits], 1);
      const uint64_t m = __ballot(keep);
      if (lane == 0) wsum[buf][wave] = __popcll(m);
      __syncthreads();  // (the other buffer is written next)
      int32_t before = 0, total = 0;
#pragma unroll
      for (int w = 0; w < kRowThreads / kWave; ++w) {
        const int32_t n = wsum[buf][w];
        if (w < wave) before += n;
        total += n;
      }
      if (keep) rest[len + before + __popcll(m & ((1ull << lane) - 1))] = x[j];
      len += total;
      buf ^= 1;
    }
  }
  __syncthreads();
  // the bits, in blocks of 128 columns, and the counts before each block
  uint4 b{0, 0, 0, 0};
  int32_t c = 0;
  static_assert(kHubMaxCols / 128 <= kRowThreads, "a thread per block of columns");
  if (t < blocks) {
    b = ((const uint4 *)bm)[t];
    c = __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w);
    const_cast<uint4 *>(hub.bits)[hub.piece(r, t)] = b;
  }
  int32_t incl = c;
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) {
    const int32_t y = __shfl_up(incl, k, kWave);
    if (lane >= k) incl += y;
  }
  if (lane == kWave - 1) wsum[0][wave] = incl;
  __syncthreads();
  int32_t pre = incl - c;
  for (int w = 0; w < wave; ++w) pre += wsum[0][w];
  if (real && t < blocks) const_cast<uint16_t *>(hub.pre)[(int64_t)r * blocks + t] = (uint16_t)pre;
  if (real && t == 0) {
    const_cast<HubRow *>(hub.row_of)[r] = HubRow{base, len, 0};
    if (nwin > 1) {
      int32_t s = 0;
      for (int w = 0; w <= nwin; ++w) {
        win[(int64_t)r * (nwin + 1) + w] = s;
        s += count[w];
      }
    }
  }
}

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// 32 bits as 32 FP4 values: a set bit becomes 0b0001 (0.5). Any order of the
// columns will do, as long as both operands have the same.
__device__ __forceinline__ i32x8 fp4_of(uint32_t w) {
  i32x8 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (int)((w >> j) & 0x11111111u);
  v[4] = v[5] = v[6] = v[7] = 0;  // (not read for 4-bit formats)
  return v;
}

// The lower triangle of D in tiles of 256 x 256, one per workgroup; each of
// the four wavefronts takes 128 x 128 (16 accumulators of 32 x 32, the whole
// register file of a SIMD), so that a step of 64 columns has 16 matrix
// instructions (512 cycles) to the 56 shifts and masks that expand its
// operands. The bits are laid out so that a fragment of 32 rows by 256 columns
// is one contiguous kilobyte, a 16-byte load per lane; the next 256 columns'
// loads are in flight. The product reads 8 bytes of bits per row and 64
// columns, so it is bound by the matrix cores and the expansion beside them:
// R-MAT-20, 5,008 rows by 51,785 columns, 356 us with 210 workgroups on the
// 256 CUs (4.0 PFLOP/s; all 256 would reach 4.9). It took k_big_owner, as it
// was then, from 4.8 to 3.9 ms beside the small owners.
__global__ __launch_bounds__(256, 1) void k_hub_product(HubView hub, uint16_t *D) {
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const int t = blockIdx.x;
  int I = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  while (I * (I + 1) / 2 > t) --I;
  const int J = t - I * (I + 1) / 2;
  const int ra = I * kTile + (wave >> 1) * 128, rb = J * kTile + (wave & 1) * 128;
  const int blocks = hub.cols / 128;
  const uint4 *pa = hub.bits + hub.piece(ra, lane >> 5) + (lane & 31);
  const uint4 *pb = hub.bits + hub.piece(rb, lane >> 5) + (lane & 31);
  const int64_t frag = (int64_t)blocks * 32;  // uint4 from one fragment of 32 rows to the next
  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.0f;
  uint4 na[4], nb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    na[i] = pa[i * frag];
    nb[i] = pb[i * frag];
  }
  const int chunks = hub.cols / kColBlock;
  for (int c = 0; c < chunks; ++c) {
    uint32_t a[4][4], b[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i][0] = na[i].x; a[i][1] = na[i].y; a[i][2] = na[i].z; a[i][3] = na[i].w;
      b[i][0] = nb[i].x; b[i][1] = nb[i].y; b[i][2] = nb[i].z; b[i][3] = nb[i].w;
    }
    const int64_t next = (int64_t)min(c + 1, chunks - 1) * 64;  // two blocks of 128 columns x 32 rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      na[i] = pa[i * frag + next];
      nb[i] = pb[i * frag + next];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      i32x8 vb[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) vb[j] = fp4_of(b[j][s]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const i32x8 va = fp4_of(a[i][s]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, vb[j], acc[i][j], 4, 4, 0, 0x7f7f7f7f, 0,
                                                                      0x7f7f7f7f);
      }
    }
  }
  // lane l holds, in register k, row 8 (k / 4) + 4 (l / 32) + k % 4, column l % 32
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int row = ra + i * 32 + 8 * (k / 4) + 4 * (lane >> 5) + k % 4, col = rb + j * 32 + (lane & 31);
        D[(int64_t)row * hub.stride + col] = (uint16_t)(acc[i][j][k] * 4.0f);
      }
}

}  // namespace

// Rows and columns by a model of what they save: edges between two vertices of
// degrees a and b number a b / nnz, an edge between two hubs saves the share
// of its lower end's ids that are columns (the columns' share of all slots),
// and the product takes rounds of 256 workgroups. On R-MAT-20 the model's
// edges and ids are within 12% of the counted ones. The rates are the
// large-owner kernel's time per streamed id and the product's measured one; a
// gain below 0.1 ms is left alone. Builds without it and with: R-MAT of 60,000
// vertices (not chosen) 0.53 ms, R-MAT-20 (5,008 rows) 6.98 and 6.80 ms,
// R-MAT-23 417 and 383 ms (11,520 rows); with the faster large-owner kernel,
// 11,520 and 44,418 rows 305 and 291 ms. kHubMaxRows bounds D to 4.8 GB.
HubShape choose_hubs(const PlanCounts &pc, int64_t nnz, bool one_window) {
  const double per_id = one_window ? 0.5e-12 : 0.6e-12;  // seconds
  const double per_round_col = 8.0 / 2.3e9 / 0.6;        // a round's seconds per column
  const double per_slot = 20e-12, fixed = 60e-6;         // building the rows; the launches
  double c[kDegBins], d[kDegBins];
  for (int b = 0; b < kDegBins; ++b) {
    c[b] = pc.bins[b];
    d[b] = 0.5 * ((double)deg_bin_low(b) + (double)deg_bin_low(b + 1));
  }
  HubShape best;
  double best_gain = 0.1e-3, ids = 0, rows = 0, row_slots = 0;
  for (int r = kDegBins - 1; r >= 0; --r) {
    rows += c[r];
    if (rows > kHubMaxRows) break;
    if (c[r] == 0) continue;
    for (int j = r + 1; j < kDegBins; ++j) ids += c[r] * c[j] * std::min(1.0, d[r] * d[j] / nnz) * d[r];
    ids += 0.5 * c[r] * c[r] * std::min(1.0, d[r] * d[r] / nnz) * d[r];
    row_slots += c[r] * deg_bin_low(r + 1);
    const double tiles = std::ceil(rows / kTile), rounds = std::ceil(tiles * (tiles + 1) / 2 / 256);
    double cols = 0, col_slots = 0;
    for (int q = kDegBins - 1; q >= 0; --q) {
      cols += c[q];
      col_slots += c[q] * d[q];
      if (cols > kHubMaxCols) break;
      if (q > r || c[q] == 0) continue;
      const double gain = ids * per_id * std::min(1.0, col_slots / nnz) - rounds * cols * per_round_col -
                          row_slots * per_slot - fixed;
      if (gain > best_gain) {
        best_gain = gain;
        best.row_deg = deg_bin_low(r);
        best.col_deg = deg_bin_low(q);
        best.rows = (int32_t)rows;
        best.cols = (int32_t)cols;
        best.slots = (int64_t)row_slots;
      }
    }
  }
  return best;
}

scan_status prepare_hubs(const HubShape &shape, int64_t n, const int64_t *off, const int32_t *deg,
                         const int32_t *adj, const int32_t *radj, int32_t wbits, int32_t nwin, int32_t *win,
                         VertexRecord *records, DevArena &arena, hipStream_t s, HubView *out) {
  HubView h;
  h.rows = shape.rows;
  h.cols = (shape.cols + kColBlock - 1) / kColBlock * kColBlock;
  h.stride = (shape.rows + kTile - 1) / kTile * kTile;
  int64_t *flags, *P, *ws;
  int32_t *col, *verts, *rest;
  HubRow *row_of;
  uint4 *bits;
  uint16_t *pre, *D;
  unsigned long long *cursor;
  SCAN_TRY(arena.alloc(&flags, n));
  SCAN_TRY(arena.alloc(&P, n + 1));
  SCAN_TRY(arena.alloc(&ws, scan_workspace_elems(n)));
  SCAN_TRY(arena.alloc(&col, n));
  SCAN_TRY(arena.alloc(&verts, h.rows));
  SCAN_TRY(arena.alloc(&row_of, h.rows));
  SCAN_TRY(arena.alloc(&rest, shape.slots));
  SCAN_TRY(arena.alloc(&bits, (int64_t)h.stride * (h.cols / 128)));
  SCAN_TRY(arena.alloc(&pre, (int64_t)h.rows * (h.cols / 128)));
  SCAN_TRY(arena.alloc(&D, (int64_t)h.stride * h.stride));
  SCAN_TRY(arena.alloc(&cursor, 1));
  h.col = col;
  h.row_of = row_of;
  h.rest = rest;
  h.bits = bits;
  h.pre = pre;
  h.D = D;
  SCAN_HIP_TRY(hipMemsetAsync(cursor, 0, 8, s));
  k_hub_flags<<<grid_for(n, 256, 4096), 256, 0, s>>>(deg, n, shape.row_deg, shape.col_deg, flags);
  SCAN_TRY(exclusive_scan64(flags, P, n, ws, s));
  k_hub_maps<<<grid_for(n, 256, 4096), 256, 0, s>>>(deg, n, shape.row_deg, shape.col_deg, P, records, col, verts);
  k_hub_rows<<<h.stride, kRowThreads, 0, s>>>(h, verts, off, adj, radj, wbits, nwin, win, cursor);
  const int tiles = h.stride / kTile;
  k_hub_product<<<tiles * (tiles + 1) / 2, 256, 0, s>>>(h, D);
  SCAN_HIP_TRY(hipGetLastError());
  *out = h;
  return SCAN_OK;
}

}  // namespace scan
