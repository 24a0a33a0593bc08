// Octree, target batches and interaction lists of the treecode (tree.hip), built on the GPU once per
// band and plan.
//
// Tree. Nodes are sorted by the Morton code of their FP32 (scaled) coordinates, 21 bits per axis,
// ties by index (a stable LSD radix sort), so that every octree node owns a contiguous range.
// Nodes with more than kLeaf points split level by level; each level's nodes are contiguous.
// `skip` threads the depth-first order: the node that follows a subtree.
//
// Target batches are runs of consecutive leaves in Morton order of at most kBatch nodes whose
// union box has a radius of at most kPackRadius times that of their largest leaf: a run that
// straddles a jump of the curve would have a wide box and interpolate almost nothing, while
// neighbouring leaves of different parents fill the wave's lanes (a batch costs one wave
// whatever its size). The runs are taken greedily from the first leaf on. Where a run that starts
// at leaf i ends depends on i alone, so every leaf finds its successor in parallel, and the run
// starts are the orbit of leaf 0, found by pointer doubling (the t-th start applies the powers in
// t's binary digits). On bands too small to give every compute unit kMinWavesPerCU such batches,
// runs of sibling leaves (smaller, more waves) are used instead.
//
// Lists. Each batch walks the tree once to count and once to fill: a cluster with more than
// (p+1)³ sources goes to the batch's proxy list when (r_B + r_C) < θ·dist and the two balls are at
// least 1.01·r_c apart (so it holds no near pair); leaves that fail the test go to the direct list,
// consecutive ones with the same predicate flag merged into one range. A wave walks for a batch, 64
// nodes at a time from a stack; the leaves it reaches out of order set bits, from which the ranges
// are read in order. The lists are cut into segments of about equal work, one wave each: a batch
// with a wide box can hold ten times the average work, and one wave per batch took 17.1 ms for the far
// field of 185,127 nodes (5046 batches) against 3.9 ms in segments.
//
// All decisions are taken in FP64 from the exact FP32 coordinates, products and sums rounded as
// written. At 724,665 nodes a plan takes about 1.5 ms, 0.6 ms of it the two walks; the same built by
// the host (16 threads, the coordinates copied down and the lists up) took about 35 ms.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "pair_kernels.hpp"

#pragma clang fp contract(off)

namespace pb {

// Device tree of one band (buffers th_* of the context workspace).
struct TreeDev {
  int n = 0, n_nodes = 0, n_leaf = 0, n_batch = 0;
  int* perm = nullptr;
  float4* xyz = nullptr;        // FP32 coordinates in tree order
  struct TreeNode* node = nullptr;
  double* box = nullptr;        // per node lo, hi
  int* leaf = nullptr;          // leaves in Morton order
  int* leaf_at = nullptr;       // index of the leaf that starts at a position
  int2* batch = nullptr;
};

struct alignas(64) TreeNode {
  int b, e;        // tree-order range
  int kid, skip;   // first child (−1: leaf; the children are consecutive), node after the subtree (−1: none)
  double c[3], r;  // centre and radius of the tight box
  int nk;          // children
};

namespace {

constexpr double kPackRadius = 4.0;  // batch box radius / largest leaf radius in the batch
constexpr int kMinWavesPerCU = 16;   // packed batches per compute unit below which siblings are used
constexpr int kLeaf = 64;            // source leaves hold at most this many nodes
static_assert(kLeaf <= kBatch, "a leaf fits one target batch");
constexpr int kLevels = 21;          // bits per axis of the Morton codes
constexpr unsigned long long kMaxSegs = 1 << 20;  // work segments of a plan beyond one per batch

// Device counters of one build, copied to pinned host memory at its synchronization points.
struct TreeCount {
  int level[kLevels + 1];  // nodes per level
  int n_leaf, n_raw, n_batch, n_dir, n_app, n_cl, n_items, n_sib;
  unsigned long long dir_pairs, app_pairs, work;
};
static_assert(sizeof(TreeCount) <= sizeof(double) * kHostPin, "the counters fit the pinned slots");

// ---------------------------------------------------------------- Morton order

__device__ __forceinline__ uint64_t spread3(uint64_t v) {  // 21 bits → every third bit
  v &= 0x1fffff;
  v = (v | v << 32) & 0x1f00000000ffffULL;
  v = (v | v << 16) & 0x1f0000ff0000ffULL;
  v = (v | v << 8) & 0x100f00f00f00f00fULL;
  v = (v | v << 4) & 0x10c30c30c30c30c3ULL;
  v = (v | v << 2) & 0x1249249249249249ULL;
  return v;
}

struct MortonFrame {
  double cx, cy, cz, sigma;  // of the FP32 records
  double lo[3], size;        // of the scaled FP32 coordinates
};

__device__ __forceinline__ void scaled_f32(const BandDev& b, int j, const MortonFrame& f, float v[3]) {
  v[0] = (float)(f.sigma * (b.px[j] - f.cx));
  v[1] = (float)(f.sigma * (b.py[j] - f.cy));
  v[2] = (float)(f.sigma * (b.pz[j] - f.cz));
}

__global__ void __launch_bounds__(kBlock) k_morton(int n, BandDev b, MortonFrame f, uint64_t* __restrict__ code,
                                                   int* __restrict__ idx) {
  const int j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= n) return;
  float v[3];
  scaled_f32(b, j, f, v);
  uint64_t m = 0;
  for (int a = 0; a < 3; ++a) {
    const double q = ((double)v[a] - f.lo[a]) / f.size * 2097152.0;
    m |= spread3((uint64_t)fmin(fmax(q, 0.0), 2097151.0)) << (2 - a);
  }
  code[j] = m;
  idx[j] = j;
}

// Stable LSD radix sort, 8 bits per pass. A block takes a tile of kSortTile keys, each of its four
// waves kSortTile/4 consecutive ones in rounds of 64; the lanes of a round that share a digit
// find each other by eight ballots.
constexpr int kSortTile = 2048, kSortRounds = kSortTile / 256;

__device__ __forceinline__ unsigned long long digit_peers(int d, bool live) {
  unsigned long long m = __ballot(live);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const unsigned long long v = __ballot(live && ((d >> bit) & 1));
    m &= (d >> bit) & 1 ? v : ~v;
  }
  return m;
}

__global__ void __launch_bounds__(256) k_sort_hist(int n, const uint64_t* __restrict__ key, int shift, int nb,
                                                   int* __restrict__ hist) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = blockIdx.x * kSortTile + r * 256 + threadIdx.x;
    if (i < n) atomicAdd(&h[(key[i] >> shift) & 255], 1);
  }
  __syncthreads();
  hist[threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// hist: exclusive scan over (digit, block).
__global__ void __launch_bounds__(256) k_sort_scatter(int n, const uint64_t* __restrict__ key,
                                                      const int* __restrict__ idx, int shift, int nb,
                                                      const int* __restrict__ hist, uint64_t* __restrict__ key_out,
                                                      int* __restrict__ idx_out) {
  __shared__ int cnt[4][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int base = blockIdx.x * kSortTile + w * (kSortTile / 4);
  const unsigned long long below = (1ull << lane) - 1ull;
  auto lds_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for (int d = lane; d < 256; d += 64) cnt[w][d] = 0;
  lds_order();
  uint64_t k[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = base + r * 64 + lane;
    k[r] = i < n ? key[i] : 0;
    const int d = (int)((k[r] >> shift) & 255);
    const unsigned long long m = digit_peers(d, i < n);
    if (i < n && (m & below) == 0) cnt[w][d] += __popcll(m);  // the first peer counts for all
    lds_order();
  }
  __syncthreads();
  {  // each wave's first place per digit
    const int d = threadIdx.x;
    int at = hist[d * nb + blockIdx.x];
    for (int v = 0; v < 4; ++v) {
      const int c = cnt[v][d];
      cnt[v][d] = at;
      at += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = base + r * 64 + lane;
    const int d = (int)((k[r] >> shift) & 255);
    const unsigned long long m = digit_peers(d, i < n);
    int at = 0;
    if (i < n) at = cnt[w][d] + __popcll(m & below);
    lds_order();
    if (i < n) {
      if ((m & below) == 0) cnt[w][d] += __popcll(m);
      key_out[at] = k[r];
      idx_out[at] = idx[i];
    }
    lds_order();
  }
}

__global__ void __launch_bounds__(kBlock) k_tree_xyz(int n, const int* __restrict__ perm, BandDev b, MortonFrame f,
                                                     float4* __restrict__ xyz) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t >= n) return;
  float v[3];
  scaled_f32(b, perm[t], f, v);
  xyz[t] = make_float4(v[0], v[1], v[2], 0.f);
}

// ---------------------------------------------------------------- octree

__global__ void k_tree_root(int n, TreeNode* __restrict__ node, TreeCount* __restrict__ ct) {
  node[0].b = 0;
  node[0].e = n;
  node[0].kid = -1;
  node[0].skip = -1;
  ct->level[0] = 1;
}

// First node of a level.
__device__ __forceinline__ int level_base(const TreeCount* ct, int level) {
  int s = 0;
  for (int l = 0; l < level; ++l) s += ct->level[l];
  return s;
}

// Splits the nodes of `level` that hold more than kLeaf points: eight lanes per node, lane o finding
// where octant o ends (binary search over the sorted codes).
__global__ void __launch_bounds__(kBlock) k_tree_level(int level, const uint64_t* __restrict__ code,
                                                       TreeNode* __restrict__ node, TreeCount* __restrict__ ct) {
  const int base = level_base(ct, level), m = ct->level[level];
  const int o = threadIdx.x & 7, lane = threadIdx.x & 63;
  const int shift = 3 * (kLevels - 1 - level);
  for (int q = (blockIdx.x * kBlock + threadIdx.x) >> 3; q < m; q += (gridDim.x * kBlock) >> 3) {
    const TreeNode nd = node[base + q];
    if (nd.e - nd.b <= kLeaf) continue;  // the eight lanes of a node stay together
    int lo = nd.b, hi = nd.e;            // first position whose octant exceeds o
    while (lo < hi) {
      const int mid = lo + ((hi - lo) >> 1);
      if ((int)((code[mid] >> shift) & 7) <= o) lo = mid + 1;
      else hi = mid;
    }
    const int end = lo, prev = __shfl_up(end, 1, 8), begin = o == 0 ? nd.b : prev;
    const bool live = end > begin;
    const unsigned kids = (unsigned)(__ballot(live) >> (lane & 56)) & 255u;
    const int nk = __popc(kids), rank = __popc(kids & ((1u << o) - 1u));
    int first = 0;
    if (o == 0) first = base + m + atomicAdd(&ct->level[level + 1], nk);
    first = __shfl(first, 0, 8);
    if (live) {
      TreeNode& c = node[first + rank];
      c.b = begin;
      c.e = end;
      c.kid = -1;
      c.skip = rank + 1 < nk ? first + rank + 1 : nd.skip;
    }
    if (o == 0) {
      node[base + q].kid = first;
      node[base + q].nk = nk;
    }
  }
}

__device__ __forceinline__ double box_radius(const double lo[3], const double hi[3]) {
  double r2 = 0.0;
  for (int a = 0; a < 3; ++a) r2 += 0.25 * (hi[a] - lo[a]) * (hi[a] - lo[a]);
  return sqrt(r2);
}

__device__ __forceinline__ void put_box(TreeNode& nd, double* __restrict__ out, const double lo[3],
                                        const double hi[3]) {
  for (int a = 0; a < 3; ++a) {
    out[a] = lo[a];
    out[3 + a] = hi[a];
    nd.c[a] = 0.5 * (lo[a] + hi[a]);
  }
  nd.r = box_radius(lo, hi);
}

// Tight boxes of the leaves, eight lanes per node, and the leaf flags by first point.
__global__ void __launch_bounds__(kBlock) k_leaf_box(int n_nodes, const float4* __restrict__ xyz,
                                                     TreeNode* __restrict__ node, double* __restrict__ box,
                                                     int* __restrict__ flag) {
  const int q = (blockIdx.x * kBlock + threadIdx.x) >> 3, o = threadIdx.x & 7;
  if (q >= n_nodes) return;
  const int b = node[q].b, e = node[q].e;
  if (node[q].kid >= 0) return;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int t = b + o; t < e; t += 8) {
    const float4 x = xyz[t];
    const float v[3] = {x.x, x.y, x.z};
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], v[a]);
      hi[a] = fmaxf(hi[a], v[a]);
    }
  }
  for (int off = 4; off > 0; off >>= 1)
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], __shfl_xor(lo[a], off, 8));
      hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off, 8));
    }
  if (o == 0) {
    const double l[3] = {lo[0], lo[1], lo[2]}, h[3] = {hi[0], hi[1], hi[2]};
    put_box(node[q], box + 6 * (size_t)q, l, h);
    flag[b] = 1;
  }
}

// Boxes of the internal nodes of one level from their children's (levels from the deepest up).
__global__ void __launch_bounds__(kBlock) k_union_box(int first, int m, TreeNode* __restrict__ node,
                                                      double* __restrict__ box) {
  const int q = blockIdx.x * kBlock + threadIdx.x;
  if (q >= m || node[first + q].kid < 0) return;
  TreeNode& nd = node[first + q];
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int k = nd.kid; k != nd.skip; k = node[k].skip) {  // the children, in order
    const double* __restrict__ bx = box + 6 * (size_t)k;
    for (int a = 0; a < 3; ++a) {
      lo[a] = fmin(lo[a], bx[a]);
      hi[a] = fmax(hi[a], bx[3 + a]);
    }
  }
  put_box(nd, box + 6 * (size_t)(first + q), lo, hi);
}

// leaf[i] = the i-th leaf in Morton order (at: exclusive scan of the leaf flags).
__global__ void __launch_bounds__(kBlock) k_leaf_list(int n_nodes, int n, const TreeNode* __restrict__ node,
                                                      const int* __restrict__ at, int* __restrict__ leaf,
                                                      TreeCount* __restrict__ ct) {
  const int q = blockIdx.x * kBlock + threadIdx.x;
  if (q == 0) ct->n_leaf = at[n];
  if (q < n_nodes && node[q].kid < 0) leaf[at[node[q].b]] = q;
}

// ---------------------------------------------------------------- target batches

// next[i]: the leaf after the run that starts at leaf i.
__global__ void __launch_bounds__(kBlock) k_run_next(int n_leaf, const int* __restrict__ leaf,
                                                     const TreeNode* __restrict__ node, const double* __restrict__ box,
                                                     int* __restrict__ next) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i > n_leaf) return;
  if (i == n_leaf) {
    next[i] = n_leaf;
    return;
  }
  const int f = leaf[i], cb = node[f].b;
  double lo[3], hi[3], maxr = node[f].r;
  for (int a = 0; a < 3; ++a) {
    lo[a] = box[6 * (size_t)f + a];
    hi[a] = box[6 * (size_t)f + 3 + a];
  }
  int k = i + 1;
  for (; k < n_leaf; ++k) {
    const int q = leaf[k];
    if (node[q].e - cb > kBatch) break;
    double ul[3], uh[3];
    for (int a = 0; a < 3; ++a) {
      ul[a] = fmin(lo[a], box[6 * (size_t)q + a]);
      uh[a] = fmax(hi[a], box[6 * (size_t)q + 3 + a]);
    }
    const double mr = fmax(maxr, node[q].r);
    if (!(box_radius(ul, uh) <= kPackRadius * mr)) break;
    for (int a = 0; a < 3; ++a) {
      lo[a] = ul[a];
      hi[a] = uh[a];
    }
    maxr = mr;
  }
  next[i] = k;
}

// Pointer doubling: out[i] = in[in[i]].
__global__ void __launch_bounds__(kBlock) k_jump(int n_leaf, const int* __restrict__ in, int* __restrict__ out) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i <= n_leaf) out[i] = in[in[i]];
}

// Run t starts at leaf J_0^t(0), composed from the powers jump[p·stride] = J_0^(2^p). raw[t] is its
// range and cnt[t] the batches it gives: one, or several for a leaf of more than kBatch coincident codes.
__global__ void __launch_bounds__(kBlock) k_run_start(int n_leaf, int n_pow, const int* __restrict__ jump, int stride,
                                                      const int* __restrict__ leaf, const TreeNode* __restrict__ node,
                                                      int2* __restrict__ raw, int* __restrict__ cnt,
                                                      TreeCount* __restrict__ ct) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t > n_leaf) return;
  int pos = 0;
  for (int p = 0; p < n_pow && pos < n_leaf; ++p)
    if ((t >> p) & 1) pos = jump[(size_t)p * stride + pos];
  if (t == n_leaf || pos >= n_leaf) {
    cnt[t] = 0;
    return;
  }
  const int nx = jump[pos], b = node[leaf[pos]].b, e = node[leaf[nx - 1]].e;
  raw[t] = make_int2(b, e);
  cnt[t] = (e - b + kBatch - 1) / kBatch;
  if (nx >= n_leaf) ct->n_raw = t + 1;
}

__global__ void __launch_bounds__(kBlock) k_run_write(int n_leaf, const int2* __restrict__ raw,
                                                      const int* __restrict__ at, int2* __restrict__ batch,
                                                      TreeCount* __restrict__ ct) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t == 0) ct->n_batch = at[n_leaf];
  if (t >= n_leaf) return;
  for (int k = at[t], b = raw[t].x; k < at[t + 1]; ++k, b += kBatch)
    batch[k] = make_int2(b, min(raw[t].y, b + kBatch));
}

// Runs of sibling leaves under one node (the root alone when it is a leaf): counted (batch = null) or
// written from at[q] on. One thread per node.
__global__ void __launch_bounds__(kBlock) k_sibling_runs(int n_nodes, const TreeNode* __restrict__ node,
                                                         int* __restrict__ at, int2* __restrict__ batch,
                                                         TreeCount* __restrict__ ct) {
  const int q = blockIdx.x * kBlock + threadIdx.x;
  if (q > n_nodes) return;
  if (batch && q == 0) ct->n_sib = at[n_nodes];
  int n = 0, w = batch && q < n_nodes ? at[q] : 0;
  auto put = [&](int b, int e) {
    for (; b < e; b += kBatch, ++n)
      if (batch) batch[w + n] = make_int2(b, min(e, b + kBatch));
  };
  if (q < n_nodes) {
    const TreeNode nd = node[q];
    if (nd.kid < 0) {
      if (q == 0) put(nd.b, nd.e);
    } else {
      int cb = -1, ce = -1;
      for (int k = nd.kid; k != nd.skip; k = node[k].skip) {
        const TreeNode ch = node[k];
        if (ch.kid < 0 && cb >= 0 && ce == ch.b && ch.e - cb <= kBatch) {
          ce = ch.e;
          continue;
        }
        if (cb >= 0) put(cb, ce);
        cb = ce = -1;
        if (ch.kid < 0) {
          cb = ch.b;
          ce = ch.e;
        }
      }
      if (cb >= 0) put(cb, ce);
    }
  }
  if (!batch) at[q] = n;
}

// ---------------------------------------------------------------- interaction lists

struct WalkArgs {
  int n_batch, P3, n_leaf;
  double theta, rcs, clear2;
  const int2* batch;
  const float4* xyz;
  const TreeNode* node;
  const double* box;
  const int* leaf;
  const int* leaf_at;
};

// Walks the tree for batch q, one thread: app(node) per proxy cluster, dir(range) per direct range (the sign bit
// of its end: it may hold near pairs).
template <typename FApp, typename FDir>
__device__ __forceinline__ void walk_tree(const WalkArgs& w, int q, FApp app, FDir dir) {
  const int2 bt = w.batch[q];
  double blo[3] = {INFINITY, INFINITY, INFINITY}, bhi[3] = {-INFINITY, -INFINITY, -INFINITY}, bc[3];
  for (int t = bt.x; t < bt.y; ++t) {
    const float4 x = w.xyz[t];
    const double v[3] = {x.x, x.y, x.z};
    for (int a = 0; a < 3; ++a) {
      blo[a] = fmin(blo[a], v[a]);
      bhi[a] = fmax(bhi[a], v[a]);
    }
  }
  for (int a = 0; a < 3; ++a) bc[a] = 0.5 * (blo[a] + bhi[a]);
  const double br = box_radius(blo, bhi);
  int2 run = make_int2(-1, -1);
  for (int k = 0; k >= 0;) {
    const TreeNode nd = w.node[k];
    const double dist = sqrt((bc[0] - nd.c[0]) * (bc[0] - nd.c[0]) + (bc[1] - nd.c[1]) * (bc[1] - nd.c[1]) +
                             (bc[2] - nd.c[2]) * (bc[2] - nd.c[2]));
    if (nd.e - nd.b > w.P3 && br + nd.r < w.theta * dist && dist - br - nd.r > w.rcs) {
      app(k, nd);
      k = nd.skip;
    } else if (nd.kid < 0) {
      // a leaf whose box is at least √clear2 from the batch's box holds no pair that the FP32
      // predicate calls near (its rounding is far below the margin)
      const double* __restrict__ bx = w.box + 6 * (size_t)k;
      double gap2 = 0.0;
      for (int a = 0; a < 3; ++a) {
        const double g = fmax(0.0, fmax(bx[a] - bhi[a], blo[a] - bx[3 + a]));
        gap2 += g * g;
      }
      const int flag = gap2 >= w.clear2 ? 0 : (int)0x80000000u;
      if (run.x >= 0 && (run.y & 0x7fffffff) == nd.b && (run.y & (int)0x80000000u) == flag) {
        run.y = nd.e | flag;
      } else {
        if (run.x >= 0) dir(run);
        run = make_int2(nd.b, nd.e | flag);
      }
      k = nd.skip;
    } else {
      k = nd.kid;
    }
  }
  if (run.x >= 0) dir(run);
}

__device__ __forceinline__ int range_len(int2 r) { return (r.y & 0x7fffffff) - r.x; }

// Work of a batch's lists in units of one proxy interaction; a direct pair costs about two.
__global__ void __launch_bounds__(64) k_walk_count(WalkArgs w, int* __restrict__ n_dir, int* __restrict__ n_app,
                                                   int* __restrict__ used, TreeCount* __restrict__ ct) {
  const int q = blockIdx.x * 64 + threadIdx.x;
  if (q >= w.n_batch) return;
  int nd = 0, na = 0, src = 0;
  walk_tree(
      w, q,
      [&](int k, const TreeNode&) {
        ++na;
        used[k] = 1;
      },
      [&](int2 r) {
        ++nd;
        src += range_len(r);
      });
  n_dir[q] = nd;
  n_app[q] = na;
  const unsigned long long cnt = w.batch[q].y - w.batch[q].x;
  atomicAdd(&ct->dir_pairs, cnt * (unsigned long long)src);
  atomicAdd(&ct->app_pairs, cnt * (unsigned long long)na * (unsigned long long)w.P3);
  atomicAdd(&ct->work, (unsigned long long)na * w.P3 + 2ull * (unsigned long long)src);
}

__global__ void __launch_bounds__(64) k_walk_fill(WalkArgs w, const int* __restrict__ dir_ptr,
                                                  const int* __restrict__ app_ptr, const int* __restrict__ cl_of,
                                                  int2* __restrict__ dir_rng, int* __restrict__ app_cl) {
  const int q = blockIdx.x * 64 + threadIdx.x;
  if (q >= w.n_batch) return;
  int d = dir_ptr[q], a = app_ptr[q];
  walk_tree(
      w, q, [&](int k, const TreeNode&) { app_cl[a++] = cl_of[k]; }, [&](int2 r) { dir_rng[d++] = r; });
}

// The same lists with one wave per batch (block): counted (kFill = false) or written. Dynamic LDS: a
// stack of kWalkStack nodes and two bits per leaf, which limits it to kWalkLeaves leaves (beyond, the
// one-thread walks above). The leaves that fail the acceptance test set bit D (and F when they may
// hold near pairs); leaves that follow each other in Morton order are contiguous, so a direct range is
// a run of D bits with equal F bits. One thread per batch took 2.2 ms per walk at 724,665 nodes
// and, for a batch with a wide box, up to 5 ms alone at 185,127: a chain of dependent node loads.
constexpr int kWalkStack = 1024, kWalkReserve = 160, kWalkLeaves = 196608;
// A pop of one node pushes at most 7 more than it takes per level below it.
static_assert(kWalkReserve >= 7 * kLevels + 8, "depth-first steps fit the reserve");

template <bool kFill>
__global__ void __launch_bounds__(64) k_walk_wave(WalkArgs w, int* __restrict__ n_dir, int* __restrict__ n_app,
                                                  int* __restrict__ used, const int* __restrict__ cl_of,
                                                  int2* __restrict__ dir_rng, int* __restrict__ app_cl,
                                                  TreeCount* __restrict__ ct) {
  extern __shared__ unsigned lds[];
  int* stack = (int*)lds;
  const int nw = (w.n_leaf + 31) / 32;
  unsigned *D = lds + kWalkStack, *F = D + nw;
  const int q = blockIdx.x, lane = threadIdx.x;
  const unsigned long long below = (1ull << lane) - 1ull;
  auto lds_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for (int i = lane; i < nw; i += 64) D[i] = F[i] = 0u;
  const int2 bt = w.batch[q];
  double blo[3], bhi[3], bc[3];
  {
    const float4 x = w.xyz[min(bt.x + lane, bt.y - 1)];
    float v[3] = {x.x, x.y, x.z};
    for (int a = 0; a < 3; ++a) {
      float l = v[a], h = v[a];
      for (int off = 32; off > 0; off >>= 1) {
        l = fminf(l, __shfl_xor(l, off));
        h = fmaxf(h, __shfl_xor(h, off));
      }
      blo[a] = l;
      bhi[a] = h;
      bc[a] = 0.5 * (blo[a] + bhi[a]);
    }
  }
  const double br = box_radius(blo, bhi);
  int napp = 0, top = 1;
  const int a0 = kFill ? n_app[q] : 0;
  if (lane == 0) stack[0] = 0;
  lds_order();
  while (top > 0) {
    int cnt = min(64, top);
    if (top + 7 * cnt > kWalkStack - kWalkReserve) cnt = max(1, min(cnt, (kWalkStack - kWalkReserve - top) / 7));
    const bool mine = lane < cnt;
    const int k = mine ? stack[top - 1 - lane] : 0;
    top -= cnt;
    lds_order();
    const TreeNode nd = w.node[k];
    const double dist = sqrt((bc[0] - nd.c[0]) * (bc[0] - nd.c[0]) + (bc[1] - nd.c[1]) * (bc[1] - nd.c[1]) +
                             (bc[2] - nd.c[2]) * (bc[2] - nd.c[2]));
    const bool acc = mine && nd.e - nd.b > w.P3 && br + nd.r < w.theta * dist && dist - br - nd.r > w.rcs;
    const unsigned long long ma = __ballot(acc);
    if (acc) {
      if (kFill) app_cl[a0 + napp + __popcll(ma & below)] = cl_of[k];
      else used[k] = 1;
    }
    napp += __popcll(ma);
    if (mine && !acc && nd.kid < 0) {
      const double* __restrict__ bx = w.box + 6 * (size_t)k;
      double gap2 = 0.0;
      for (int a = 0; a < 3; ++a) {
        const double g = fmax(0.0, fmax(bx[a] - bhi[a], blo[a] - bx[3 + a]));
        gap2 += g * g;
      }
      const int li = w.leaf_at[nd.b];
      atomicOr(&D[li >> 5], 1u << (li & 31));
      if (!(gap2 >= w.clear2)) atomicOr(&F[li >> 5], 1u << (li & 31));
    }
    const int nk = mine && !acc && nd.kid >= 0 ? nd.nk : 0;
    if (__ballot(nk > 0))
      for (int c = 0; c < 8; ++c) {
        const unsigned long long mk = __ballot(c < nk);
        if (c < nk) stack[top + __popcll(mk & below)] = nd.kid + c;
        top += __popcll(mk);
      }
    lds_order();
  }
  // ranges: the r-th begins at the r-th set bit of S and ends with the r-th set bit of E
  const int d0 = kFill ? n_dir[q] : 0;
  int ns = 0, ne = 0;
  long long src = 0;
  for (int i0 = 0; i0 < nw; i0 += 64) {
    const int i = i0 + lane;
    const unsigned d = i < nw ? D[i] : 0u;
    if (!__ballot(d != 0u)) continue;
    const unsigned f = i < nw ? F[i] : 0u;
    const unsigned dp = i > 0 && i <= nw ? D[i - 1] >> 31 : 0u, fp = i > 0 && i <= nw ? F[i - 1] >> 31 : 0u;
    const unsigned dn = i + 1 < nw ? D[i + 1] << 31 : 0u, fn = i + 1 < nw ? F[i + 1] << 31 : 0u;
    const unsigned S = d & ~(((d << 1) | dp) & ~(f ^ ((f << 1) | fp)));
    const unsigned E = d & ~(((d >> 1) | dn) & ~(f ^ ((f >> 1) | fn)));
    int ps = __popc(S), pe = __popc(E);
    const int cs = ps, ce = pe;
    for (int off = 1; off < 64; off <<= 1) {
      const int us = __shfl_up(ps, off), ue = __shfl_up(pe, off);
      if (lane >= off) {
        ps += us;
        pe += ue;
      }
    }
    int r = d0 + ns + ps - cs;
    for (unsigned m = S; m; m &= m - 1u, ++r) {
      const int b = w.node[w.leaf[i * 32 + __ffs(m) - 1]].b;
      src -= b;
      if (kFill) dir_rng[r].x = b;
    }
    r = d0 + ne + pe - ce;
    for (unsigned m = E; m; m &= m - 1u, ++r) {
      const int bit = __ffs(m) - 1, e = w.node[w.leaf[i * 32 + bit]].e;
      src += e;
      if (kFill) dir_rng[r].y = e | ((f >> bit) & 1u ? (int)0x80000000u : 0);
    }
    ns += __shfl(ps, 63);
    ne += __shfl(pe, 63);
  }
  if (kFill) return;
  for (int off = 32; off > 0; off >>= 1) src += __shfl_xor(src, off);
  if (lane == 0) {
    n_dir[q] = ns;
    n_app[q] = napp;
    const unsigned long long t = bt.y - bt.x;
    atomicAdd(&ct->dir_pairs, t * (unsigned long long)src);
    atomicAdd(&ct->app_pairs, t * (unsigned long long)napp * (unsigned long long)w.P3);
    atomicAdd(&ct->work, (unsigned long long)napp * w.P3 + 2ull * (unsigned long long)src);
  }
}

// Proxy work items per cluster (0 for nodes no list uses).
__global__ void __launch_bounds__(kBlock) k_cluster_count(int n_nodes, const TreeNode* __restrict__ node,
                                                          const int* __restrict__ used, int* __restrict__ items) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  if (k > n_nodes) return;
  items[k] = k < n_nodes && used[k] ? (node[k].e - node[k].b + kProxyChunk - 1) / kProxyChunk : 0;
}

__global__ void k_list_totals(int n_batch, int n_nodes, const int* __restrict__ dir_ptr,
                              const int* __restrict__ app_ptr, const int* __restrict__ cl_of,
                              const int* __restrict__ item_at, TreeCount* __restrict__ ct) {
  ct->n_dir = dir_ptr[n_batch];
  ct->n_app = app_ptr[n_batch];
  ct->n_cl = cl_of[n_nodes];
  ct->n_items = item_at[n_nodes];
}

// Proxy clusters: the tree nodes some list uses, in node order; half-widths kept away from zero.
__global__ void __launch_bounds__(kBlock) k_cluster_write(int n_nodes, const TreeNode* __restrict__ node,
                                                          const double* __restrict__ box, const int* __restrict__ cl_of,
                                                          const int* __restrict__ item_at, float4* __restrict__ half,
                                                          double* __restrict__ ccen, int* __restrict__ item_ptr,
                                                          int4* __restrict__ items) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  if (k > n_nodes) return;
  const int cl = cl_of[k];
  if (k == n_nodes) {
    item_ptr[cl] = item_at[k];
    return;
  }
  if (cl_of[k + 1] == cl) return;  // not used
  const TreeNode nd = node[k];
  const double* __restrict__ bx = box + 6 * (size_t)k;
  double ext = 0.0, hw[3];
  for (int a = 0; a < 3; ++a) ext = fmax(ext, bx[3 + a] - bx[a]);
  for (int a = 0; a < 3; ++a) {
    hw[a] = fmax(0.5 * (bx[3 + a] - bx[a]), fmax(1e-3 * ext, 1e-6));
    ccen[3 * (size_t)cl + a] = nd.c[a];
  }
  half[cl] = make_float4((float)hw[0], (float)hw[1], (float)hw[2], 0.f);
  item_ptr[cl] = item_at[k];
  for (int i = item_at[k], t = nd.b; t < nd.e; t += kProxyChunk, ++i)
    items[i] = make_int4(cl, t, min(nd.e, t + kProxyChunk), 0);
}

// Cuts a batch's lists into segments that close once they hold W units of work: counted (seg =
// null) or written from at[q] on. One thread per batch; at least one segment each.
__global__ void __launch_bounds__(64) k_segments(int n_batch, int P3, int W, const int* __restrict__ dir_ptr,
                                                 const int* __restrict__ app_ptr, const int2* __restrict__ dir_rng,
                                                 int* __restrict__ at, TreeSeg* __restrict__ seg) {
  const int q = blockIdx.x * 64 + threadIdx.x;
  if (q > n_batch) return;
  if (q == n_batch) {
    if (!seg) at[q] = 0;
    return;
  }
  const int d1 = dir_ptr[q + 1], a1 = app_ptr[q + 1];
  int n = 0;
  TreeSeg s{q, dir_ptr[q], dir_ptr[q], app_ptr[q], app_ptr[q]};
  const int base = seg ? at[q] : 0;
  int work = 0;
  while (s.d1 < d1 || s.a1 < a1) {
    if (s.d1 < d1) {
      work += 2 * range_len(dir_rng[s.d1++]);
    } else {  // whole clusters up to W
      const int take = min(a1 - s.a1, max(1, (W - work + P3 - 1) / P3));
      s.a1 += take;
      work += take * P3;
    }
    if (work >= W && (s.d1 < d1 || s.a1 < a1)) {
      if (seg) seg[base + n] = s;
      ++n;
      s.d0 = s.d1;
      s.a0 = s.a1;
      work = 0;
    }
  }
  if (seg) seg[base + n] = s;
  else at[q] = n + 1;
}

unsigned blocks_for(int64_t m, int per) { return (unsigned)((m + per - 1) / per); }

// The build's counters on the host, after a synchronization.
pb_status read_counts(pb_ctx* ctx, const TreeCount* dev, TreeCount* out) {
  PB_HIP(ctx, hipMemcpyAsync(ctx->host_pin, dev, sizeof(TreeCount), hipMemcpyDeviceToHost, ctx->stream));
  PB_TRY(sync(ctx, "tree build"));
  std::memcpy(out, ctx->host_pin, sizeof(TreeCount));
  return PB_OK;
}

pb_status tree_build(pb_ctx* ctx, const pb_band* band, const MixedPlan& P, TreeDev& H) {
  const int n = (int)band->n;
  H.n = n;
  PB_TRY(host_pin(ctx));
  MortonFrame f{P.cx, P.cy, P.cz, P.sigma, {}, 0.0};
  {
    // the extremes of the scaled FP32 coordinates are those of the projections, scaled and rounded
    const double c[3] = {P.cx, P.cy, P.cz};
    double size = 1e-12;
    for (int a = 0; a < 3; ++a) {
      f.lo[a] = (double)(float)(P.sigma * (P.lo[a] - c[a]));
      size = std::max(size, (double)(float)(P.sigma * (P.hi[a] - c[a])) - f.lo[a]);
    }
    f.size = size * (1.0 + 1e-9);
  }
  const int nb = (int)blocks_for(n, kSortTile);
  // internal nodes hold more than kLeaf points, at most n/(kLeaf + 1) per level; the leaves are
  // disjoint and not empty
  const int64_t cap = (int64_t)n + (int64_t)kLevels * (n / (kLeaf + 1) + 1) + 1;
  uint64_t* key[2] = {(uint64_t*)workspace(ctx, "th_key0", sizeof(uint64_t) * (size_t)n),
                      (uint64_t*)workspace(ctx, "th_key1", sizeof(uint64_t) * (size_t)n)};
  int* idx[2] = {(int*)workspace(ctx, "th_perm", sizeof(int) * (size_t)n),
                 (int*)workspace(ctx, "th_idx1", sizeof(int) * (size_t)n)};
  int* hist = (int*)workspace(ctx, "th_hist", sizeof(int) * (256 * (size_t)nb + 1));
  TreeCount* ct = (TreeCount*)workspace(ctx, "th_count", sizeof(TreeCount));
  H.xyz = (float4*)workspace(ctx, "th_xyz", sizeof(float4) * (size_t)n);
  H.node = (TreeNode*)workspace(ctx, "th_node", sizeof(TreeNode) * (size_t)cap);
  H.box = (double*)workspace(ctx, "th_box", sizeof(double) * 6 * (size_t)cap);
  int* flag = (int*)workspace(ctx, "th_flag", sizeof(int) * (size_t)(n + 1));
  if (!key[0] || !key[1] || !idx[0] || !idx[1] || !hist || !ct || !H.xyz || !H.node || !H.box || !flag)
    return PB_ENOMEM;
  H.perm = idx[0];
  PB_HIP(ctx, hipMemsetAsync(ct, 0, sizeof(TreeCount), ctx->stream));
  PB_HIP(ctx, hipMemsetAsync(flag, 0, sizeof(int) * (size_t)(n + 1), ctx->stream));
  k_morton<<<blocks_for(n, kBlock), kBlock, 0, ctx->stream>>>(n, band_dev(band), f, key[0], idx[0]);
  static_assert(3 * kLevels <= 64, "eight passes of eight bits, an even number: the result is in key[0], idx[0]");
  for (int pass = 0; pass < 8; ++pass) {
    const int from = pass & 1, to = from ^ 1;
    k_sort_hist<<<nb, 256, 0, ctx->stream>>>(n, key[from], 8 * pass, nb, hist);
    PB_TRY(exclusive_scan_i32(ctx, hist, 256 * (int64_t)nb));
    k_sort_scatter<<<nb, 256, 0, ctx->stream>>>(n, key[from], idx[from], 8 * pass, nb, hist, key[to], idx[to]);
  }
  k_tree_xyz<<<blocks_for(n, kBlock), kBlock, 0, ctx->stream>>>(n, H.perm, band_dev(band), f, H.xyz);
  k_tree_root<<<1, 1, 0, ctx->stream>>>(n, H.node, ct);
  for (int l = 0; l < kLevels; ++l)
    k_tree_level<<<std::min<unsigned>(blocks_for(8 * (int64_t)(n / (kLeaf + 1) + 1), kBlock), 1024), kBlock, 0,
                   ctx->stream>>>(l, key[0], H.node, ct);
  PB_TRY(launch_ok(ctx, "octree"));
  TreeCount hc;
  PB_TRY(read_counts(ctx, ct, &hc));
  int depth = 0;
  H.n_nodes = 0;
  for (int l = 0; l <= kLevels; ++l) {
    if (hc.level[l] > 0) depth = l;
    H.n_nodes += hc.level[l];
  }
  if (H.n_nodes > cap) return ctx->fail(PB_EDEVICE, "octree: %d nodes, room for %lld", H.n_nodes, (long long)cap);
  const int nn = H.n_nodes;
  k_leaf_box<<<blocks_for(8 * (int64_t)nn, kBlock), kBlock, 0, ctx->stream>>>(nn, H.xyz, H.node, H.box, flag);
  for (int l = depth - 1, first = nn - hc.level[depth]; l >= 0; --l) {
    first -= hc.level[l];
    k_union_box<<<blocks_for(hc.level[l], kBlock), kBlock, 0, ctx->stream>>>(first, hc.level[l], H.node, H.box);
  }
  PB_TRY(exclusive_scan_i32(ctx, flag, n + 1));
  int* leaf = (int*)workspace(ctx, "th_leaf", sizeof(int) * (size_t)nn);
  if (!leaf) return PB_ENOMEM;
  H.leaf = leaf;
  H.leaf_at = flag;
  k_leaf_list<<<blocks_for(nn, kBlock), kBlock, 0, ctx->stream>>>(nn, n, H.node, flag, leaf, ct);
  PB_TRY(launch_ok(ctx, "octree boxes"));
  PB_TRY(read_counts(ctx, ct, &hc));
  const int nl = H.n_leaf = hc.n_leaf;
  // packed runs
  int n_pow = 1;
  while ((1ll << n_pow) <= nl) ++n_pow;
  const int stride = nl + 1;
  int* jump = (int*)workspace(ctx, "th_jump", sizeof(int) * (size_t)n_pow * stride);
  int2* raw = (int2*)workspace(ctx, "th_raw", sizeof(int2) * (size_t)stride);
  int* at = (int*)workspace(ctx, "th_at", sizeof(int) * (size_t)std::max(stride, nn + 1));
  H.batch = (int2*)workspace(ctx, "th_batch", sizeof(int2) * ((size_t)nl + (size_t)n / kBatch + 1));
  if (!jump || !raw || !at || !H.batch) return PB_ENOMEM;
  const unsigned bl = blocks_for(stride, kBlock);
  k_run_next<<<bl, kBlock, 0, ctx->stream>>>(nl, leaf, H.node, H.box, jump);
  for (int p = 1; p < n_pow; ++p)
    k_jump<<<bl, kBlock, 0, ctx->stream>>>(nl, jump + (size_t)(p - 1) * stride, jump + (size_t)p * stride);
  k_run_start<<<bl, kBlock, 0, ctx->stream>>>(nl, n_pow, jump, stride, leaf, H.node, raw, at, ct);
  PB_TRY(exclusive_scan_i32(ctx, at, stride));
  k_run_write<<<bl, kBlock, 0, ctx->stream>>>(nl, raw, at, H.batch, ct);
  PB_TRY(launch_ok(ctx, "target batches"));
  PB_TRY(read_counts(ctx, ct, &hc));
  H.n_batch = hc.n_batch;
  if ((int64_t)hc.n_raw < (int64_t)kMinWavesPerCU * ctx->n_cu) {  // sibling runs
    const unsigned bn = blocks_for(nn + 1, kBlock);
    k_sibling_runs<<<bn, kBlock, 0, ctx->stream>>>(nn, H.node, at, nullptr, ct);
    PB_TRY(exclusive_scan_i32(ctx, at, nn + 1));
    k_sibling_runs<<<bn, kBlock, 0, ctx->stream>>>(nn, H.node, at, H.batch, ct);
    PB_TRY(launch_ok(ctx, "sibling batches"));
    PB_TRY(read_counts(ctx, ct, &hc));
    H.n_batch = hc.n_sib;
  }
  return PB_OK;
}

}  // namespace

pb_status tree_prepare(pb_ctx* ctx, const pb_band* band, const Derived& d, int degree, double theta, TreePlan& T,
                       const char* pfx, const MixedPlan* near, std::shared_ptr<TreeDev>* tree, NearBuild what) {
  const int n = (int)band->n;
  const std::string px_ = pfx;
  if (near) T.near = *near;  // the near field depends on the geometry only: shared between plans
  else PB_TRY(near_build(ctx, band, d, (px_ + "n_").c_str(), T.near, what));
  const MixedPlan& P = T.near;
  const int P1 = degree + 1, P3 = P1 * P1 * P1;
  std::shared_ptr<TreeDev> hp = tree && *tree && (*tree)->n == n ? *tree : nullptr;
  if (!hp) {
    hp = std::make_shared<TreeDev>();
    PB_TRY(tree_build(ctx, band, P, *hp));
    if (tree) *tree = hp;
  }
  const TreeDev& H = *hp;
  const int nbt = H.n_batch, nn = H.n_nodes;
  auto ws = [&](const char* nm, size_t bytes) { return workspace(ctx, (px_ + nm).c_str(), std::max<size_t>(bytes, 16)); };
  TreeCount* ct = (TreeCount*)workspace(ctx, "th_count", sizeof(TreeCount));
  int* cl_of = (int*)workspace(ctx, "th_cl", sizeof(int) * 2 * (size_t)(nn + 1));  // clusters | items
  int* dir_ptr = (int*)ws("dir_ptr", sizeof(int) * (size_t)(nbt + 1));
  int* app_ptr = (int*)ws("app_ptr", sizeof(int) * (size_t)(nbt + 1));
  if (!ct || !cl_of || !dir_ptr || !app_ptr) return PB_ENOMEM;
  int* item_at = cl_of + (nn + 1);
  PB_HIP(ctx, hipMemsetAsync(ct, 0, sizeof(TreeCount), ctx->stream));
  PB_HIP(ctx, hipMemsetAsync(cl_of, 0, sizeof(int) * (size_t)(nn + 1), ctx->stream));
  PB_HIP(ctx, hipMemsetAsync(dir_ptr + nbt, 0, sizeof(int), ctx->stream));
  PB_HIP(ctx, hipMemsetAsync(app_ptr + nbt, 0, sizeof(int), ctx->stream));
  const WalkArgs w{nbt,     P3,    H.n_leaf, theta, P.sigma * P.rc * 1.01, (double)P.rc2f * (1.0 + 1e-3),
                   H.batch, H.xyz, H.node,   H.box, H.leaf,                H.leaf_at};
  const bool waves = H.n_leaf <= kWalkLeaves;
  const size_t lds = sizeof(unsigned) * ((size_t)kWalkStack + 2 * (size_t)((H.n_leaf + 31) / 32));
  const unsigned bb = blocks_for(nbt, 64), bn = blocks_for(nn + 1, kBlock);
  if (waves)
    k_walk_wave<false><<<nbt, 64, lds, ctx->stream>>>(w, dir_ptr, app_ptr, cl_of, nullptr, nullptr, nullptr, ct);
  else
    k_walk_count<<<bb, 64, 0, ctx->stream>>>(w, dir_ptr, app_ptr, cl_of, ct);
  k_cluster_count<<<bn, kBlock, 0, ctx->stream>>>(nn, H.node, cl_of, item_at);
  PB_TRY(exclusive_scan_i32(ctx, dir_ptr, nbt + 1));
  PB_TRY(exclusive_scan_i32(ctx, app_ptr, nbt + 1));
  PB_TRY(exclusive_scan_i32(ctx, cl_of, nn + 1));
  PB_TRY(exclusive_scan_i32(ctx, item_at, nn + 1));
  k_list_totals<<<1, 1, 0, ctx->stream>>>(nbt, nn, dir_ptr, app_ptr, cl_of, item_at, ct);
  PB_TRY(launch_ok(ctx, "tree lists"));
  TreeCount hc;
  PB_TRY(read_counts(ctx, ct, &hc));
  const int n_cl = hc.n_cl, n_items = hc.n_items;
  // about 64 segments per compute unit, so that no wave outlasts the rest by much, but each large
  // enough (a quarter of a typical batch at least) that its set-up stays small; no more than kMaxSegs beyond one per
  // batch, whose sums are kept (1 KB each): with nearly all pairs direct (θ = 0.001 on 1.2 million nodes) segments of
  // 8192 were 6.9 million
  const int64_t W64 = std::min<int64_t>(8192, std::max<int64_t>(256, (int64_t)(hc.work / (64ull * ctx->n_cu))));
  const int W = (int)std::max<int64_t>(W64, (int64_t)(hc.work / kMaxSegs) + 1);
  const int64_t seg_max = (int64_t)(hc.work / (unsigned long long)W) + nbt;
  T.perm = H.perm;
  T.batch = H.batch;
  T.dir_rng = (int2*)ws("dir_rng", sizeof(int2) * (size_t)hc.n_dir);
  T.app_cl = (int*)ws("app_cl", sizeof(int) * (size_t)hc.n_app);
  T.half = (float4*)ws("half", sizeof(float4) * (size_t)n_cl);
  T.ccen = (double*)ws("ccen", sizeof(double) * 3 * (size_t)n_cl);
  T.items = (int4*)ws("items", sizeof(int4) * (size_t)n_items);
  T.item_ptr = (int*)ws("item_ptr", sizeof(int) * (size_t)(n_cl + 1));
  T.seg_ptr = (int*)ws("seg_ptr", sizeof(int) * (size_t)(nbt + 1));
  T.seg = (TreeSeg*)ws("seg", sizeof(TreeSeg) * (size_t)seg_max);
  T.seg_sum = (double*)ws("seg_sum", sizeof(double) * 2 * kBatch * (size_t)seg_max);
  T.At = (float4*)ws("At", sizeof(float4) * (size_t)n);
  T.Mt = (float4*)ws("Mt", sizeof(float4) * (size_t)n);
  T.Nt = (float4*)ws("Nt", sizeof(float4) * (size_t)n);
  T.Gt = (float4*)ws("Gt", sizeof(float4) * (size_t)n);
  T.St = (double*)ws("St", sizeof(double) * 3 * (size_t)n);
  T.anc = (double*)ws("anc", sizeof(double) * 3 * (size_t)((n + kAnchor - 1) / kAnchor));
  T.PX = (float4*)ws("PX", sizeof(float4) * (size_t)n_cl * P3);
  T.PM = (float*)ws("PM", sizeof(float) * (size_t)n_cl * P3);
  T.part = (double2*)ws("part", sizeof(double2) * (size_t)n_items * P3);
  T.far = (double*)ws("far", sizeof(double) * 2 * (size_t)n);
  if (!T.dir_rng || !T.app_cl || !T.half || !T.ccen || !T.items || !T.item_ptr || !T.seg_ptr || !T.seg ||
      !T.seg_sum || !T.At || !T.Mt || !T.Nt || !T.Gt || !T.St || !T.anc || !T.PX || !T.PM || !T.part || !T.far)
    return PB_ENOMEM;
  if (waves)
    k_walk_wave<true><<<nbt, 64, lds, ctx->stream>>>(w, dir_ptr, app_ptr, nullptr, cl_of, T.dir_rng, T.app_cl, ct);
  else
    k_walk_fill<<<bb, 64, 0, ctx->stream>>>(w, dir_ptr, app_ptr, cl_of, T.dir_rng, T.app_cl);
  k_cluster_write<<<bn, kBlock, 0, ctx->stream>>>(nn, H.node, H.box, cl_of, item_at, T.half, T.ccen, T.item_ptr,
                                                  T.items);
  const unsigned bs = blocks_for(nbt + 1, 64);
  k_segments<<<bs, 64, 0, ctx->stream>>>(nbt, P3, W, dir_ptr, app_ptr, T.dir_rng, T.seg_ptr, nullptr);
  PB_TRY(exclusive_scan_i32(ctx, T.seg_ptr, nbt + 1));
  k_segments<<<bs, 64, 0, ctx->stream>>>(nbt, P3, W, dir_ptr, app_ptr, T.dir_rng, T.seg_ptr, T.seg);
  PB_TRY(launch_ok(ctx, "tree segments"));
  T.band_key = band->px;
  T.n = n;
  T.rc = d.rc;
  T.theta = theta;
  T.degree = degree;
  T.n_batch = nbt;
  T.n_cl = n_cl;
  T.n_items = n_items;
  T.n_seg_max = (int)seg_max;
  T.n_dir_pairs = (int64_t)hc.dir_pairs;
  T.n_app_pairs = (int64_t)hc.app_pairs;
  for (int a = 0; a <= degree; ++a) T.u[a] = (float)std::cos(kPi * a / degree);
  return tree_coords(ctx, band, T);
}

}  // namespace pb
