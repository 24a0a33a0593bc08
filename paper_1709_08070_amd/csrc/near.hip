// Cell list and FP64 near-field matrix of a band: what the mixed and treecode operators build
// once per geometry (every pair closer than r_c, in FP64), and the cell list the network's
// neighbour search walks.
//
// Cells are at least r_c wide, so a node's near sources lie in the 27 cells around it. A cell's
// nodes are kept in increasing index (counting sort by cell, then each node ranks itself
// within its cell), so every list, and with it every sum, has a fixed order. Positions, normals
// and the FP32 coordinates of the near predicate are copied in cell order: the nine
// contiguous ranges that hold a node's 27 cells are then read with coalesced loads.
#include <algorithm>
#include <cmath>
#include <vector>

#include "pair_kernels.hpp"

namespace pb {
namespace {

// Bounding box partials of the projections, 6 doubles per block, written to pinned host memory.
__global__ void __launch_bounds__(kBlock) k_bbox(int n, BandDev b, double* __restrict__ out) {
  __shared__ double s[6][kBlock];
  double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int j = blockIdx.x * kBlock + threadIdx.x; j < n; j += gridDim.x * kBlock) {
    v[0] = fmin(v[0], b.px[j]); v[1] = fmin(v[1], b.py[j]); v[2] = fmin(v[2], b.pz[j]);
    v[3] = fmax(v[3], b.px[j]); v[4] = fmax(v[4], b.py[j]); v[5] = fmax(v[5], b.pz[j]);
  }
  for (int q = 0; q < 6; ++q) s[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off)
      for (int q = 0; q < 6; ++q)
        s[q][threadIdx.x] = q < 3 ? fmin(s[q][threadIdx.x], s[q][threadIdx.x + off])
                                  : fmax(s[q][threadIdx.x], s[q][threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int q = 0; q < 6; ++q) out[6 * blockIdx.x + q] = s[q][0];
}

// FP32 coordinates of a node as k_pack_f32 writes them (the same expression, the same bits).
__device__ __forceinline__ float3 coords_f32(const BandDev& b, int j, double cx, double cy, double cz, double sigma) {
  return make_float3((float)(sigma * (b.px[j] - cx)), (float)(sigma * (b.py[j] - cy)),
                     (float)(sigma * (b.pz[j] - cz)));
}

// Bounding box of each aligned group of kGroup nodes in FP32 coordinates (one block per group):
// box[2g] = (lo, 0), box[2g + 1] = (hi, 0) over the group's live nodes.
__global__ void __launch_bounds__(kGroup) k_group_box(int n, BandDev b, double cx, double cy, double cz, double sigma,
                                                      float4* __restrict__ box) {
  __shared__ float s[6][kGroup / 64];
  const int i = blockIdx.x * kGroup + threadIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (i < n) {
    const float3 a = coords_f32(b, i, cx, cy, cz, sigma);
    v[0] = v[3] = a.x;
    v[1] = v[4] = a.y;
    v[2] = v[5] = a.z;
  }
  for (int off = 32; off > 0; off >>= 1)
    for (int q = 0; q < 6; ++q) {
      const float o = __shfl_xor(v[q], off);
      v[q] = q < 3 ? fminf(v[q], o) : fmaxf(v[q], o);
    }
  if (lane == 0)
    for (int q = 0; q < 6; ++q) s[q][w] = v[q];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int u = 1; u < kGroup / 64; ++u)
      for (int q = 0; q < 6; ++q) s[q][0] = q < 3 ? fminf(s[q][0], s[q][u]) : fmaxf(s[q][0], s[q][u]);
    box[2 * blockIdx.x] = make_float4(s[0][0], s[1][0], s[2][0], 0.f);
    box[2 * blockIdx.x + 1] = make_float4(s[3][0], s[4][0], s[5][0], 0.f);
  }
}

struct CellGrid {
  double lx, ly, lz, inv;
  int ncx, ncy, ncz;
};

// The node's cell and its (arrival-ordered) slot in it.
__global__ void __launch_bounds__(kBlock) k_cell_count(int n, BandDev b, CellGrid g, int* __restrict__ cell_of,
                                                       int* __restrict__ slot, int* __restrict__ counts) {
  const int j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= n) return;
  const int cx = min(g.ncx - 1, max(0, (int)((b.px[j] - g.lx) * g.inv)));
  const int cy = min(g.ncy - 1, max(0, (int)((b.py[j] - g.ly) * g.inv)));
  const int cz = min(g.ncz - 1, max(0, (int)((b.pz[j] - g.lz) * g.inv)));
  const int c = (cx * g.ncy + cy) * g.ncz + cz;
  cell_of[j] = c;
  slot[j] = atomicAdd(&counts[c], 1);
}

__global__ void __launch_bounds__(kBlock) k_cell_fill(int n, const int* __restrict__ cell_of,
                                                      const int* __restrict__ slot, const int* __restrict__ start,
                                                      int* __restrict__ tmp) {
  const int j = blockIdx.x * kBlock + threadIdx.x;
  if (j < n) tmp[start[cell_of[j]] + slot[j]] = j;
}

// Each node's rank among its cell's nodes gives its place in cell order; its record follows. A
// thread per node: 5 µs at 45,818 nodes where one thread per cell sorting by insertion took 48 µs.
template <bool kNear>
__global__ void __launch_bounds__(kBlock) k_cell_place(int n, BandDev b, const double* __restrict__ w,
                                                       const int* __restrict__ cell_of, const int* __restrict__ start,
                                                       const int* __restrict__ tmp, double cx, double cy, double cz,
                                                       double sigma, int* __restrict__ nodes, double4* __restrict__ pos,
                                                       double4* __restrict__ nrm, float4* __restrict__ key) {
  const int j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= n) return;
  const int c = cell_of[j], s = start[c], e = start[c + 1];
  int at = s;
  for (int q = s; q < e; ++q) at += tmp[q] < j;
  nodes[at] = j;
  pos[at] = make_double4(b.px[j], b.py[j], b.pz[j], w[j]);
  if (kNear) {
    nrm[at] = make_double4(b.nx[j], b.ny[j], b.nz[j], 0.0);
    const float3 a = coords_f32(b, j, cx, cy, cz, sigma);
    key[at] = make_float4(a.x, a.y, a.z, __int_as_float(j));
  }
}

constexpr int kNearWaves = kBlock / 64;  // targets per block of the near-list kernels
constexpr int kAhead = 4;                // steps of 64 candidates read at once
constexpr int kNearQueue = 64 * kAhead + 64;
constexpr int kHitSlots = 1024;          // counters of k_near_once, by target, so that few waves share one

// Visits the near sources of target i (FP32 distance below r_c) in a fixed order: the nine
// ranges of cell_ranges one after the other, 64 candidates at a time. Per step every lane calls
// f(hit, q, mask) with its candidate's place q in cell order and the ballot of the hits, and after each turn of
// kAhead steps turn(last). One wave
// per target. The ranges (30 to 45 candidates each) are read as one sequence, four steps' records at once:
// bound by the latency of those reads, of which a loop over the ranges has nine in a row.
template <typename F, typename T>
__device__ __forceinline__ void for_near_wave(const float3& t, int c, const float4* __restrict__ key,
                                              const CellsDev& cells, float rc2, F f, T turn) {
  const int lane = threadIdx.x & 63;
  int lo, hi;
  cell_ranges(cells, c, lo, hi);
  int first[9], shift[9], m = 0;  // range r holds candidates first[r] … of the sequence, at shift[r] + its number
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const int a = __builtin_amdgcn_readlane(lo, r), e = __builtin_amdgcn_readlane(hi, r);
    first[r] = m;
    shift[r] = a - m;
    m += e - a;
  }
  for (int f0 = 0; f0 < m; f0 += 64 * kAhead) {
    int q[kAhead];
    float4 k[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int g = min(f0 + 64 * u + lane, m - 1);
      int s = shift[0];
#pragma unroll
      for (int r = 1; r < 9; ++r) s = g >= first[r] ? shift[r] : s;
      q[u] = g + s;
      k[u] = key[q[u]];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (f0 + 64 * u >= m) break;
      const bool hit = f0 + 64 * u + lane < m && r2_f32(t.x, t.y, t.z, k[u].x, k[u].y, k[u].z) < rc2;
      f(hit, q[u], __ballot(hit));
    }
    turn(f0 + 64 * kAhead >= m);
  }
}

// Near sources per target, and a zero after the last for the scan's total.
__global__ void __launch_bounds__(kBlock) k_near_count(int n, BandDev b, double cx, double cy, double cz, double sigma,
                                                       const float4* __restrict__ key, CellsDev cells, float rc2,
                                                       int64_t* __restrict__ counts) {
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * kNearWaves + (threadIdx.x >> 6));
  if (i >= n) return;
  int64_t cnt = 0;
  for_near_wave(coords_f32(b, i, cx, cy, cz, sigma), cells.cell_of[i], key, cells, rc2,
                [&](bool, int, unsigned long long mask) { cnt += __popcll(mask); }, [](bool) {});
  if ((threadIdx.x & 63) == 0) {
    counts[i] = cnt;
    if (i == n - 1) counts[n] = 0;
  }
}

// The near pairs of target i, up to 64 at a time: hits (about 50 of 200 to 400 candidates) queue up in
// the wave's kNearQueue entries of LDS over a turn of kAhead steps, and pairs(q) is called by every lane that has
// one, with the source's place q in cell order, and full(cnt) by all lanes after each cnt ≤ 64 pairs. One place
// for the pairs' code, outside the unrolled steps. Whole waves; no block barrier.
template <typename P, typename F>
__device__ __forceinline__ void for_near_pairs(const float3& t, int c, const float4* __restrict__ key,
                                               const CellsDev& cells, float rc2, int* queue, P pairs, F full) {
  const int lane = threadIdx.x & 63;
  int pending = 0;
  auto lds_order = [] {  // this wave's queue entries are visible to its other lanes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for_near_wave(
      t, c, key, cells, rc2,
      [&](bool hit, int q, unsigned long long mask) {  // pending < 64 before a turn's first step
        if (hit) queue[pending + __popcll(mask & ((1ull << lane) - 1ull))] = q;
        pending += __popcll(mask);
      },
      [&](bool last) {
        lds_order();
        int at = 0;
        for (; pending - at >= (last ? 1 : 64); at += 64) {
          const int cnt = min(pending - at, 64);
          if (lane < cnt) pairs(queue[at + lane]);
          full(cnt);
        }
        if (last) return;
        pending -= at;
        const int rest = lane < pending ? queue[at + lane] : 0;
        lds_order();
        if (lane < pending) queue[lane] = rest;
      });
}

// Near-field block matrix: for each near pair the FP64 coefficients of
//   y1_i += c0 ψ_j + c1 ψn_j,  y2_i += c2 ψ_j + c3 ψn_j,  with s_j = h³ω_j/(4π)
//   c0 = 4πK11 s_j, c1 = −4πK12 s_j, c2 = 4πK21 s_j, c3 = −4πK22 s_j.
// The coefficients depend on geometry only, so a solve builds them once per band; formed 64 at a time,
// from the cell-ordered geometry.
__global__ void __launch_bounds__(kBlock) k_near_fill(int n, BandDev b, double cx, double cy, double cz, double sigma,
                                                      double scale, const float4* __restrict__ key,
                                                      const double4* __restrict__ nrm, CellsDev cells, float rc2,
                                                      KParams kp, const int64_t* __restrict__ row,
                                                      int* __restrict__ col, double4* __restrict__ coef) {
  __shared__ int queue[kNearWaves][kNearQueue];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * kNearWaves + wave);  // the wave's: scalar loads
  if (i >= n) return;
  const double xi = b.px[i], yi = b.py[i], zi = b.pz[i], nxi = b.nx[i], nyi = b.ny[i], nzi = b.nz[i];
  const double ci = b.curv ? b.curv[i] : 0.0;
  int64_t done = row[i];
  for_near_pairs(
      coords_f32(b, i, cx, cy, cz, sigma), cells.cell_of[i], key, cells, rc2, queue[wave],
      [&](int q) {
        const double4 x = cells.pos[q], m = nrm[q];
        double k[4];
        kern4_f64(xi, yi, zi, nxi, nyi, nzi, x.x, x.y, x.z, m.x, m.y, m.z, kp, ci, k);
        const double sj = scale * x.w;
        col[done + lane] = cells.nodes[q];
        coef[done + lane] = make_double4(k[0] * sj, -k[1] * sj, k[2] * sj, -k[3] * sj);
      },
      [&](int cnt) { done += cnt; });
}

// near = (near block matrix)·p without the matrix, for an operator that is applied once to its band: the
// same pairs and coefficients as k_near_fill's, multiplied where they are formed, the lanes' sums added in a
// fixed order. Each wave adds its pairs to one of kHitSlots counters (hits, may be null). At 13,393 nodes it
// takes 14 µs in place of count, scan, fill and product (9 + 12 + 19 + 8) and a synchronization between them; 141 at
// 185,127, 566 at 724,665 (17, 195 and 748 with four waves a SIMD).
__global__ void __launch_bounds__(kBlock) k_near_once(int n, BandDev b, double cx, double cy, double cz, double sigma,
                                                      double scale, const float4* __restrict__ key,
                                                      const double4* __restrict__ nrm, CellsDev cells, float rc2,
                                                      KParams kp, const double* __restrict__ p,
                                                      double* __restrict__ near, unsigned long long* __restrict__ hits) {
  __shared__ int queue[kNearWaves][kNearQueue];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * kNearWaves + wave);  // the wave's: scalar loads
  if (i >= n) return;
  const double xi = b.px[i], yi = b.py[i], zi = b.pz[i], nxi = b.nx[i], nyi = b.ny[i], nzi = b.nz[i];
  const double ci = b.curv ? b.curv[i] : 0.0;
  double s1 = 0.0, s2 = 0.0;
  int cnt = 0;
  for_near_pairs(
      coords_f32(b, i, cx, cy, cz, sigma), cells.cell_of[i], key, cells, rc2, queue[wave],
      [&](int q) {
        const int j = cells.nodes[q];
        const double4 x = cells.pos[q], m = nrm[q];
        const double ps = p[j], pn = p[n + j];
        double k[4];
        kern4_f64(xi, yi, zi, nxi, nyi, nzi, x.x, x.y, x.z, m.x, m.y, m.z, kp, ci, k);
        const double sj = scale * x.w;
        s1 += (k[0] * sj) * ps + (-k[1] * sj) * pn;
        s2 += (k[2] * sj) * ps + (-k[3] * sj) * pn;
      },
      [&](int c) { cnt += c; });
  for (int off = 32; off > 0; off >>= 1) {
    s1 += __shfl_down(s1, off);
    s2 += __shfl_down(s2, off);
  }
  if (lane == 0) {
    near[i] = s1;
    near[n + i] = s2;
    if (hits) atomicAdd(&hits[i & (kHitSlots - 1)], (unsigned long long)cnt);
  }
}

__global__ void __launch_bounds__(kHitSlots) k_hit_total(const unsigned long long* __restrict__ hits,
                                                         int64_t* __restrict__ total) {
  __shared__ unsigned long long s[kHitSlots];
  const int t = threadIdx.x;
  s[t] = hits[t];
  __syncthreads();
  for (int off = kHitSlots / 2; off > 0; off >>= 1) {
    if (t < off) s[t] += s[t + off];
    __syncthreads();
  }
  if (t == 0) *total = (int64_t)s[0];
}

}  // namespace

// Count and fill are bound by the waves in flight over a chain of five dependent reads (cell, ranges, keys, records,
// queue): with the pairs' code in one place and the target's data in scalar registers k_near_fill holds 76 vector
// registers instead of 112, six waves a SIMD instead of four: 40 µs at 45,818 nodes (52), the count 20 (22). At 185,127 nodes
// (9.3M pairs) the earlier form took 183 and 70 µs; 228 and 104 with a loop over the nine ranges, 558 and 345 with 27
// separate cells walked through index lists and the library's exp. Turns of 2, 3 and 6 steps are no faster (601, 563, 589 µs
// against 566 in k_near_once at 724,665 nodes), nor is a bound of eight waves, which spills.

// Geometry of the mixed operator for one band: centre and scale of the FP32 records, the
// cell list and the FP64 near-field CSR matrix. Buffers are named `<pfx>...` in the context
// workspace; the plan receives the sizes and pointers. The FP32 records themselves are written
// by k_pack_f32, with the weights, before each application.
pb_status near_build(pb_ctx* ctx, const pb_band* band, const Derived& d, const char* pfx, MixedPlan& P,
                     NearBuild what) {
  const int n = (int)band->n;
  auto name = [&](const char* s) {
    static thread_local char buf[64];
    snprintf(buf, sizeof(buf), "%s%s", pfx, s);
    return (const char*)buf;
  };
  const int nbb = std::min(256, (n + 4 * kBlock - 1) / (4 * kBlock));
  static_assert(6 * 256 <= kHostPin, "bounding box partials fit the pinned slots");
  PB_TRY(host_pin(ctx));
  k_bbox<<<nbb, kBlock, 0, ctx->stream>>>(n, band_dev(band), ctx->host_pin_dev);
  PB_TRY(launch_ok(ctx, "bbox"));
  PB_TRY(sync(ctx, "bbox"));
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  const volatile double* hb = ctx->host_pin;
  for (int q = 0; q < nbb; ++q)
    for (int a = 0; a < 3; ++a) {
      lo[a] = std::fmin(lo[a], hb[6 * q + a]);
      hi[a] = std::fmax(hi[a], hb[6 * q + 3 + a]);
    }
  for (int a = 0; a < 3; ++a) {
    P.lo[a] = lo[a];
    P.hi[a] = hi[a];
  }
  P.band_key = band->px;
  P.n = n;
  P.cx = 0.5 * (lo[0] + hi[0]);
  P.cy = 0.5 * (lo[1] + hi[1]);
  P.cz = 0.5 * (lo[2] + hi[2]);
  P.sigma = d.kappa > 0.0 ? d.kappa : 1.0;
  P.rc = d.rc;
  P.rc2f = f32params(d, P.sigma).rc2;
  // cells at least r_c wide (margin for the FP32 rounding of the coordinates), at most 2^26 cells
  double cell = d.rc * 1.001 + 1e-4;
  for (;;) {
    double nc = 1.0;
    for (int a = 0; a < 3; ++a) nc *= std::floor((hi[a] - lo[a]) / cell) + 1.0;
    if (nc <= 67108864.0) break;
    cell *= 1.25;
  }
  P.cell = cell;
  P.ncx = (int)std::floor((hi[0] - lo[0]) / cell) + 1;
  P.ncy = (int)std::floor((hi[1] - lo[1]) / cell) + 1;
  P.ncz = (int)std::floor((hi[2] - lo[2]) / cell) + 1;
  const int64_t ncell = (int64_t)P.ncx * P.ncy * P.ncz;
  int* start = (int*)workspace(ctx, name("cell_start"), sizeof(int) * (size_t)(ncell + 1));
  int* nodes = (int*)workspace(ctx, name("cell_nodes"), sizeof(int) * (size_t)n);
  int* tmp = (int*)workspace(ctx, name("cell_tmp"), sizeof(int) * 2 * (size_t)n);
  int* cell_of = (int*)workspace(ctx, name("cell_of"), sizeof(int) * (size_t)n);
  double4* pos = (double4*)workspace(ctx, name("cell_pos"), sizeof(double4) * (size_t)n);
  if (!start || !nodes || !tmp || !cell_of || !pos) return PB_ENOMEM;
  double4* nrm = nullptr;
  float4* key = nullptr;
  if (what != NearBuild::cells) {
    nrm = (double4*)workspace(ctx, name("cell_nrm"), sizeof(double4) * (size_t)n);
    key = (float4*)workspace(ctx, name("cell_key"), sizeof(float4) * (size_t)n);
    if (!nrm || !key) return PB_ENOMEM;
  }
  PB_HIP(ctx, hipMemsetAsync(start, 0, sizeof(int) * (size_t)(ncell + 1), ctx->stream));
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  const CellGrid cg{lo[0], lo[1], lo[2], 1.0 / cell, P.ncx, P.ncy, P.ncz};
  k_cell_count<<<nb, kBlock, 0, ctx->stream>>>(n, band_dev(band), cg, cell_of, tmp + n, start);
  PB_TRY(launch_ok(ctx, "cell count"));
  PB_TRY(exclusive_scan_i32(ctx, start, ncell + 1));
  k_cell_fill<<<nb, kBlock, 0, ctx->stream>>>(n, cell_of, tmp + n, start, tmp);
  auto place = what == NearBuild::cells ? k_cell_place<false> : k_cell_place<true>;
  place<<<nb, kBlock, 0, ctx->stream>>>(n, band_dev(band), band->w, cell_of, start, tmp, P.cx, P.cy, P.cz, P.sigma,
                                        nodes, pos, nrm, key);
  PB_TRY(launch_ok(ctx, "cell list"));
  P.cell_start = start;
  P.cell_nodes = nodes;
  P.cell_of = cell_of;
  P.cell_pos = pos;
  P.cell_nrm = nrm;
  P.cell_key = key;
  P.row = nullptr;
  P.col = nullptr;
  P.coef = nullptr;
  P.nnz = 0;
  if (what == NearBuild::cells) return PB_OK;
  float4* A = (float4*)workspace(ctx, name("A"), sizeof(float4) * n);
  float4* M = (float4*)workspace(ctx, name("M"), sizeof(float4) * n);
  float4* N = (float4*)workspace(ctx, name("N"), sizeof(float4) * n);
  const int ngroup = (n + kGroup - 1) / kGroup;
  float4* box = (float4*)workspace(ctx, name("box"), sizeof(float4) * 2 * (size_t)ngroup);
  if (!A || !M || !N || !box) return PB_ENOMEM;
  k_group_box<<<(unsigned)ngroup, kGroup, 0, ctx->stream>>>(n, band_dev(band), P.cx, P.cy, P.cz, P.sigma, box);
  P.A = A;
  P.M = M;
  P.N = N;
  P.box = box;
  if (what == NearBuild::once) return launch_ok(ctx, "group boxes");
  int64_t* row = (int64_t*)workspace(ctx, name("near_row"), sizeof(int64_t) * (size_t)(n + 1));
  if (!row) return PB_ENOMEM;
  const CellsDev cells = cells_dev(P);
  const unsigned nbw = (unsigned)((n + kNearWaves - 1) / kNearWaves);
  k_near_count<<<nbw, kBlock, 0, ctx->stream>>>(n, band_dev(band), P.cx, P.cy, P.cz, P.sigma, key, cells, P.rc2f, row);
  PB_TRY(launch_ok(ctx, "near count"));
  int64_t nnz = 0;
  PB_TRY(exclusive_scan_i64(ctx, row, n + 1, &nnz));
  P.nnz = nnz;
  int* col = (int*)workspace(ctx, name("near_col"), sizeof(int) * (size_t)std::max<int64_t>(nnz, 1));
  double4* coef = (double4*)workspace(ctx, name("near_coef"), sizeof(double4) * (size_t)std::max<int64_t>(nnz, 1));
  if (!col || !coef) return PB_ENOMEM;
  k_near_fill<<<nbw, kBlock, 0, ctx->stream>>>(n, band_dev(band, d.curved), P.cx, P.cy, P.cz, P.sigma,
                                               d.h3 / (4.0 * kPi), key, nrm, cells, P.rc2f, kparams(d), row, col, coef);
  PB_TRY(launch_ok(ctx, "near fill"));
  P.row = row;
  P.col = col;
  P.coef = coef;
  return PB_OK;
}

// near = (near block matrix)·p of a prepared band: from the matrix if the plan holds one, else straight from
// the cells (a plan made for one application).
pb_status near_apply(pb_ctx* ctx, const pb_band* band, const Derived& d, const MixedPlan& P, const double* p,
                     double* near, int64_t* total_dev) {
  const int n = (int)band->n;
  if (P.row) {
    k_near_spmv<<<(unsigned)(((int64_t)n * kRowLanes + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
        n, P.row, P.col, P.coef, p, near);
    return PB_OK;
  }
  unsigned long long* hits = nullptr;
  if (total_dev) {
    hits = (unsigned long long*)workspace(ctx, "near_hits", sizeof(unsigned long long) * kHitSlots);
    if (!hits) return PB_ENOMEM;
    PB_HIP(ctx, hipMemsetAsync(hits, 0, sizeof(unsigned long long) * kHitSlots, ctx->stream));
  }
  k_near_once<<<(unsigned)((n + kNearWaves - 1) / kNearWaves), kBlock, 0, ctx->stream>>>(
      n, band_dev(band, d.curved), P.cx, P.cy, P.cz, P.sigma, d.h3 / (4.0 * kPi), P.cell_key, P.cell_nrm,
      cells_dev(P), P.rc2f, kparams(d), p, near, hits);
  if (hits) k_hit_total<<<1, kHitSlots, 0, ctx->stream>>>(hits, total_dev);
  return PB_OK;
}

}  // namespace pb
