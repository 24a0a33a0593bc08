// Learned initial guess and right preconditioner for the IBIM system (not part of the
// paper's method): a point-convolution network over the band nodes, served and trained with
// BF16 MFMA kernels (FP32 accumulation, FP32 master weights, Adam).
//
// Network. Each node has 16 neighbour slots: itself and its 15 nearest band nodes by
// projection distance |x_i* − x_j*| (ties by index). Layer l maps the gathered slot features
// [16 × C_l] of a node to C_{l+1} channels: Z = G·W_l + b_l, X = leaky-ReLU(Z) (slope 0.01),
// with widths 16 → 64 → 64 → 64 → 16 (outputs 0 and 1 used). Layer-1 slot features of
// neighbour j seen from node i (10 used of 16): φ_j/ε, n_j, H_j·ε (H: mean curvature from the
// normals of the neighbours), v1_j/s1, v2_j/s2, (x_j* − x_i*)/ε, where v is the vector the
// network is applied to and s1, s2 the RMS of its two halves.
//
// Map. M(v) = Λ⁻¹ (v + s ⊙ O(v)) per node (s = (s1, s2)), i.e. the paper's diagonal solve
// plus a learned correction; a zero network is exactly Λ⁻¹. M is positively homogeneous
// (M(αv) = αM(v), α > 0). Served as x0 = M(g) and as a right preconditioner inside FGMRES.
//
// Training target for a pair (v, u = A⁻¹v): T = (Λu − v)/s per node; the loss is
// Σ|O − T|² / Σ|T|² over the band.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <type_traits>
#include <vector>

#include "pair_kernels.hpp"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef short short8_t __attribute__((ext_vector_type(8)));

struct pb_nn {
  int device = 0;
  int64_t n_params = 0;
  float* params = nullptr;  // FP32 master: per layer W[K][Cout] (k-major) then b[Cout]
  float* grads = nullptr;
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  uint16_t* wt = nullptr;   // BF16 W^T per layer: [Cout][K]
  uint16_t* wk = nullptr;   // BF16 W per layer: [K][Cout]
  int64_t step = 0;
};

namespace pb {
namespace nnk {

constexpr int kSlots = 16;
constexpr int kLayers = 4;
constexpr int kCin[kLayers] = {16, 64, 64, 64};
constexpr int kCout[kLayers] = {64, 64, 64, 16};
constexpr float kSlope = 0.01f;

constexpr int kdim(int l) { return kSlots * kCin[l]; }

// parameter offsets (floats) of W_l and b_l in the flat buffer, and of the BF16 copies
inline int64_t w_off(int l) {
  int64_t o = 0;
  for (int q = 0; q < l; ++q) o += (int64_t)kdim(q) * kCout[q] + kCout[q];
  return o;
}
inline int64_t b_off(int l) { return w_off(l) + (int64_t)kdim(l) * kCout[l]; }
inline int64_t wbf_off(int l) {
  int64_t o = 0;
  for (int q = 0; q < l; ++q) o += (int64_t)kdim(q) * kCout[q];
  return o;
}
inline int64_t n_params() { return w_off(kLayers); }
inline int64_t n_wbf() { return wbf_off(kLayers); }

// FP32 → BF16 bits, round to nearest even (NaN kept quiet).
__host__ __device__ __forceinline__ uint16_t bf16_bits(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ bf16x8_t pack8(const float* v) {
  short8_t s;
#pragma unroll
  for (int r = 0; r < 8; ++r) s[r] = (short)bf16_bits(v[r]);
  return __builtin_bit_cast(bf16x8_t, s);
}

__device__ __forceinline__ bf16x8_t load8_bf16(const uint16_t* p) {
  short8_t s = *reinterpret_cast<const short8_t*>(p);
  return __builtin_bit_cast(bf16x8_t, s);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  const uint32_t u = (uint32_t)b << 16;
  float f;
  memcpy(&f, &u, 4);
  return f;
}

__device__ __forceinline__ float act(float z) { return z > 0.f ? z : kSlope * z; }
__device__ __forceinline__ float dact(float x) { return x > 0.f ? 1.f : kSlope; }

// ---------------------------------------------------------------- geometry

// 16 nearest band nodes by projection distance (ties by index; self first), from the cell list:
// one wave per node.
//  1. The lanes form the squared distances of the node's candidates (the nine ranges of its 27
//     cells, up to kKnnCand) in registers, 64 a row.
//  2. Bisection on a squared radius, by ballots, for one that holds 16 to 64 candidates (all
//     of them where there are no more than 64).
//  3. Those are compacted, and each ranks itself among them by (distance, index): rank s < 16 is
//     slot s.
// Where a node has more than kKnnCand candidates or no such radius exists (48 equal distances),
// the wave takes the least (distance, index) beyond the last sixteen times over the candidates.
// Bound by the waves in flight over the chain of reads and ballots: 57 µs at 55,111 nodes, with the ranges
// read as one sequence, four rows at once, and 59 registers, eight waves a SIMD. A loop over the nine ranges
// through 24 KB of LDS a block took 115 µs, a sorted list per thread 594. The general case takes
// 6.7 ms where 40,000 nodes fill a ball of 2.8 Å (15.7 with a sorted list in one lane).
constexpr int kKnnCand = 512;
constexpr int kKnnWaves = 4;

__device__ __forceinline__ double dist2_rn(double dx, double dy, double dz) {
  return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}

__global__ void __launch_bounds__(64 * kKnnWaves) k_knn(int n, BandDev b, CellsDev cells, int* __restrict__ nbr) {
  __shared__ double sd[kKnnWaves][64];
  __shared__ int sq[kKnnWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * kKnnWaves + w);
  if (i >= n) return;  // whole waves; the kernel has no block barrier
  auto lds_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const double xi = b.px[i], yi = b.py[i], zi = b.pz[i];
  int lo, hi;
  cell_ranges(cells, cells.cell_of[i], lo, hi);
  int first[9], shift[9], m = 0;  // range r holds candidates first[r] … of one sequence, at shift[r] + their number
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const int a = __builtin_amdgcn_readlane(lo, r), e = __builtin_amdgcn_readlane(hi, r);
    first[r] = m;
    shift[r] = a - m;
    m += e - a;
  }
  int* __restrict__ out = nbr + (int64_t)i * kSlots;
  bool done = false;
  if (m <= kKnnCand) {
    constexpr int kRows = kKnnCand / 64, kAhead = 4;  // rows read at once
    double d[kRows];
    int q[kRows];
#pragma unroll
    for (int r0 = 0; r0 < kRows; r0 += kAhead) {
#pragma unroll
      for (int r = r0; r < r0 + kAhead; ++r) {
        d[r] = INFINITY;
        q[r] = 0;
      }
      if (r0 * 64 < m) {
        double4 x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int g = min((r0 + u) * 64 + lane, m - 1);
          int s = shift[0];
#pragma unroll
          for (int r = 1; r < 9; ++r) s = g >= first[r] ? shift[r] : s;
          q[r0 + u] = g + s;
          x[u] = cells.pos[q[r0 + u]];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          if ((r0 + u) * 64 + lane < m) d[r0 + u] = dist2_rn(xi - x[u].x, yi - x[u].y, zi - x[u].z);
      }
    }
    // cells are at least r_c wide: (2 cells)² bounds what the bisection starts from
    const double top = 12.0 / (cells.inv * cells.inv);
    double t = m <= 64 ? INFINITY : top, tl = 0.0, th = INFINITY;
    int cnt = m;
    for (int it = 0; m > 64 && it < 48; ++it) {
      t = th < INFINITY ? 0.5 * (tl + th) : (it == 0 ? top * 0.0625 : t * 4.0);
      cnt = 0;
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        if (r * 64 < m) cnt += __popcll(__ballot(d[r] <= t));
      if (cnt < kSlots) tl = t;
      else if (cnt > 64) th = t;
      else break;
    }
    if (cnt <= 64 && (cnt >= kSlots || m <= 64)) {
      // compact the survivors, at most 64, into the wave's LDS slots
      int base = 0;
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        if (r * 64 < m) {
          const bool in = r * 64 + lane < m && d[r] <= t;
          const unsigned long long mask = __ballot(in);
          if (in) {
            const int at2 = base + __popcll(mask & ((1ull << lane) - 1ull));
            sd[w][at2] = d[r];
            sq[w][at2] = cells.nodes[q[r]];
          }
          base += __popcll(mask);
        }
      lds_order();
      cnt = base;  // a NaN distance is in no radius
      const double dm = lane < cnt ? sd[w][lane] : INFINITY;
      const int jm = lane < cnt ? sq[w][lane] : 0;
      int rank = 0;
      for (int k = 0; k < cnt; ++k) {
        const double dk = sd[w][k];
        const int jk = sq[w][k];
        rank += dk < dm || (dk == dm && jk < jm);
      }
      if (lane < cnt && rank < kSlots) out[rank] = jm;
      if (lane >= cnt && lane < kSlots) out[lane] = i;  // fewer than 16 candidates
      done = true;
    }
  }
  if (done) return;
  // the general case: slot by slot, the least (distance, index) after the last one's
  double ld = -1.0;
  int lj = -1;
  for (int t = 0; t < kSlots; ++t) {
    double bd = INFINITY;
    int bj = INT_MAX;
    for (int g = lane; g < m; g += 64) {
      int s = shift[0];
#pragma unroll
      for (int r = 1; r < 9; ++r) s = g >= first[r] ? shift[r] : s;
      const double4 x = cells.pos[g + s];
      const int j = cells.nodes[g + s];
      const double d2 = dist2_rn(xi - x.x, yi - x.y, zi - x.z);
      if ((d2 > ld || (d2 == ld && j > lj)) && (d2 < bd || (d2 == bd && j < bj))) {
        bd = d2;
        bj = j;
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      const double od = __shfl_xor(bd, off);
      const int oj = __shfl_xor(bj, off);
      if (od < bd || (od == bd && oj < bj)) {
        bd = od;
        bj = oj;
      }
    }
    if (lane == 0) out[t] = bd < INFINITY ? bj : i;
    ld = bd;
    lj = bj;
  }
}

// Per-node geometry features: φ/ε, n (3), H·ε with H = (2/m) Σ_{j≠i} (n_j − n_i)·(x_j − x_i)/|x_j − x_i|².
__global__ void __launch_bounds__(kBlock) k_geom(int n, BandDev b, const double* __restrict__ phi, double eps,
                                                 const int* __restrict__ nbr, float* __restrict__ feat) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  double H = 0.0;
  int m = 0;
  for (int s = 0; s < kSlots; ++s) {
    const int j = nbr[(int64_t)i * kSlots + s];
    const double dx = b.px[j] - b.px[i], dy = b.py[j] - b.py[i], dz = b.pz[j] - b.pz[i];
    const double d2 = dx * dx + dy * dy + dz * dz;
    if (j == i || d2 < 1e-12 * eps * eps) continue;
    H += ((b.nx[j] - b.nx[i]) * dx + (b.ny[j] - b.ny[i]) * dy + (b.nz[j] - b.nz[i]) * dz) / d2;
    ++m;
  }
  H = m ? 2.0 * H / m : 0.0;
  float* f = feat + (int64_t)i * 5;
  f[0] = (float)(phi[i] / eps);
  f[1] = (float)b.nx[i];
  f[2] = (float)b.ny[i];
  f[3] = (float)b.nz[i];
  f[4] = (float)(H * eps);
}

// s[0..1] = RMS of the two halves of v (1 when zero); partial sums per block, then one block.
__global__ void __launch_bounds__(kBlock) k_rms_partial(int n, const double* __restrict__ v, double* __restrict__ part) {
  __shared__ double r1[kBlock], r2[kBlock];
  double a = 0.0, c = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    a += v[i] * v[i];
    c += v[n + i] * v[n + i];
  }
  r1[threadIdx.x] = a;
  r2[threadIdx.x] = c;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      r1[threadIdx.x] += r1[threadIdx.x + off];
      r2[threadIdx.x] += r2[threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = r1[0];
    part[2 * blockIdx.x + 1] = r2[0];
  }
}

// The two inputs of a node as the network reads them: v/s per half, BF16, the first in the low bits.
__device__ __forceinline__ uint32_t input_pair(double v1, double v2, double s1, double s2) {
  return (uint32_t)bf16_bits((float)(v1 / s1)) | (uint32_t)bf16_bits((float)(v2 / s2)) << 16;
}

// s from the partial sums of k_rms_partial (strided sums per thread, then a fixed tree: every block forms
// it for itself, block 0 stores it), and the scaled inputs of every node.
__global__ void __launch_bounds__(kBlock) k_pack_in(int n, int nb, const double* __restrict__ part,
                                                    const double* __restrict__ v, double* __restrict__ s,
                                                    uint32_t* __restrict__ vs) {
  __shared__ double r1[kBlock], r2[kBlock];
  double a = 0.0, c = 0.0;
  for (int q = threadIdx.x; q < nb; q += kBlock) {
    a += part[2 * q];
    c += part[2 * q + 1];
  }
  r1[threadIdx.x] = a;
  r2[threadIdx.x] = c;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      r1[threadIdx.x] += r1[threadIdx.x + off];
      r2[threadIdx.x] += r2[threadIdx.x + off];
    }
    __syncthreads();
  }
  a = sqrt(r1[0] / n);
  c = sqrt(r2[0] / n);
  a = a > 0.0 ? a : 1.0;
  c = c > 0.0 ? c : 1.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    s[0] = a;
    s[1] = c;
  }
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) vs[i] = input_pair(v[i], v[n + i], a, c);
}

// Layer-1 input rows G1[i] = 16 slots × 16 features (BF16), all but features 5 and 6, the neighbour's scaled
// inputs, which layer 1 puts in from vs: a solve applies the network to many inputs on one geometry.
__global__ void __launch_bounds__(kBlock) k_build_g1(int n, BandDev b, const int* __restrict__ nbr,
                                                     const float* __restrict__ feat, double eps,
                                                     uint16_t* __restrict__ G1) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t >= n * kSlots) return;
  const int i = t / kSlots, slot = t % kSlots;
  const int j = nbr[(int64_t)i * kSlots + slot];
  const float* fj = feat + (int64_t)j * 5;
  const float lo[8] = {fj[0], fj[1], fj[2], fj[3], fj[4], 0.f, 0.f, (float)((b.px[j] - b.px[i]) / eps)};
  const float hi[8] = {(float)((b.py[j] - b.py[i]) / eps), (float)((b.pz[j] - b.pz[i]) / eps), 0.f, 0.f, 0.f, 0.f, 0.f,
                       0.f};
  bf16x8_t* out = reinterpret_cast<bf16x8_t*>(G1 + (int64_t)t * 16);
  out[0] = pack8(lo);
  out[1] = pack8(hi);
}

// ---------------------------------------------------------------- forward

// Z = A·W + b for 16-node wave tiles; A rows are G1 (dense, BF16, K = 256) with the neighbours' inputs
// vs put in (and, for the weight gradient, stored back into G1 if asked), or the gathered BF16
// activations of the 16 neighbour slots (8 channels, one 16-byte load per lane and step). kAct (hidden
// layers) applies the leaky ReLU and stores BF16, rounded to nearest even once here (the rounding every
// consumer applies: the next layer's MFMA operand and the weight gradient's); the output layer stores
// FP32. The BF16 weights are staged in LDS in chunks of kWChunk columns and shared by the block's W waves
// (each wave would otherwise stream the whole matrix from the caches); rows are padded by 8 elements so
// that the 16 rows a wave reads at one column offset fall on different banks. Bound by the latency of the
// gathers, chunk after chunk, so by the waves in flight: chunks of 128 columns leave room for four a SIMD
// (256 columns, 150 VGPRs with the weights loaded ahead: two), and the weights of the next chunk are loaded
// before this one's products. A layer of 64 → 64 at 45,818 nodes 27.8 → 18.0 µs, 64 → 16 17.8 → 13.5.
constexpr int kWChunk = 128;
constexpr int kWPad = 8;

template <bool kDense, int CIN, int COUT, bool kAct, int W>
__global__ void __launch_bounds__(64 * W) k_layer_fwd(int n, uint16_t* __restrict__ G1,
                                                      const uint32_t* __restrict__ vs, int store,
                                                      const uint16_t* __restrict__ X, const int* __restrict__ nbr,
                                                      const uint16_t* __restrict__ Wt, const float* __restrict__ bias,
                                                      std::conditional_t<kAct, uint16_t, float>* __restrict__ Y,
                                                      const int* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int K = kSlots * CIN;
  constexpr int NT = COUT / 16;
  constexpr int KC = K < kWChunk ? K : kWChunk, KU = KC / 32;
  constexpr int kThreads = 64 * W, kParts = COUT * KC / 8, kMine = (kParts + kThreads - 1) / kThreads;
  static_assert(K % KC == 0 && KC % 32 == 0, "whole chunks of 32-column steps");
  __shared__ uint16_t sW[COUT][KC + kWPad];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int node0 = (blockIdx.x * W + wave) * 16;
  const int node = node0 + (lane & 15), row = min(node, n - 1);  // beyond the last node: its row, not stored
  const int kq = 8 * (lane >> 4);
  f32x4_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  short8_t w[kMine];  // the thread's part of a chunk of weights
  auto load_w = [&](int k0) {
#pragma unroll
    for (int r = 0; r < kMine; ++r) {
      const int e = threadIdx.x + r * kThreads;
      if (e < kParts)
        w[r] = *reinterpret_cast<const short8_t*>(Wt + (int64_t)(e / (KC / 8)) * K + k0 + (e % (KC / 8)) * 8);
    }
  };
  load_w(0);
  // the node's neighbour rows, looked up once
  int rows[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; q += 4) {
    const int4 v = *reinterpret_cast<const int4*>(nbr + (int64_t)row * kSlots + q);
    rows[q] = v.x, rows[q + 1] = v.y, rows[q + 2] = v.z, rows[q + 3] = v.w;
  }
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += KC) {
    // this chunk's A operands, loaded before the weights are staged so that the gathers' latency
    // overlaps the staging
    bf16x8_t a[KU];
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int slot = (k0 + u * 32) / CIN;
      if (kDense) {
        uint16_t* g = G1 + (int64_t)row * K + k0 + u * 32 + kq;
        short8_t x = *reinterpret_cast<const short8_t*>(g);
        if (!(kq & 8)) {  // features 0..7 of a slot
          const uint32_t in = vs[kq ? rows[slot + 1] : rows[slot]];
          x[5] = (short)(in & 0xffffu);
          x[6] = (short)(in >> 16);
          if (store && node < n) *reinterpret_cast<short8_t*>(g) = x;
        }
        a[u] = __builtin_bit_cast(bf16x8_t, x);
      } else {
        a[u] = load8_bf16(X + (int64_t)rows[slot] * CIN + (u * 32) % CIN + kq);
      }
    }
    if (k0) __syncthreads();  // the previous chunk is no longer read
#pragma unroll
    for (int r = 0; r < kMine; ++r) {
      const int e = threadIdx.x + r * kThreads;
      if (e < kParts) *reinterpret_cast<short8_t*>(&sW[e / (KC / 8)][(e % (KC / 8)) * 8]) = w[r];
    }
    if (k0 + KC < K) load_w(k0 + KC);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KU; ++u) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bf16x8_t bw = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const short8_t*>(
                                                             &sW[t * 16 + (lane & 15)][u * 32 + kq]));
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], bw, acc[t], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int j = t * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int nd = node0 + 4 * (lane >> 4) + r;
      if (nd < n) {
        const float z = acc[t][r] + bias[j];
        if constexpr (kAct)
          Y[(int64_t)nd * COUT + j] = bf16_bits(act(z));
        else
          Y[(int64_t)nd * COUT + j] = z;
      }
    }
  }
}

// p = Λ⁻¹(v + s ⊙ O[:, 0:2])
__global__ void __launch_bounds__(kBlock) k_apply_out(int n, const double* __restrict__ v, const float* __restrict__ O,
                                                      const double* __restrict__ s, double lam1, double lam2,
                                                      double* __restrict__ p) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  p[i] = (v[i] + s[0] * (double)O[(int64_t)i * 16]) / lam1;
  p[n + i] = (v[n + i] + s[1] * (double)O[(int64_t)i * 16 + 1]) / lam2;
}

// ---------------------------------------------------------------- loss and backward

// T = (Λu − v)/s, partial Σ|T|² per block.
__global__ void __launch_bounds__(kBlock) k_target(int n, const double* __restrict__ v, const double* __restrict__ u,
                                                   const double* __restrict__ s, double lam1, double lam2,
                                                   float* __restrict__ T, double* __restrict__ part) {
  __shared__ double red[kBlock];
  double a = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const double t1 = (lam1 * u[i] - v[i]) / s[0], t2 = (lam2 * u[n + i] - v[n + i]) / s[1];
    T[2 * (int64_t)i] = (float)t1;
    T[2 * (int64_t)i + 1] = (float)t2;
    a += t1 * t1 + t2 * t2;
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// dO = 2(O − T)/Σ|T|² on the two used channels (0 elsewhere); partial Σ|O − T|².
__global__ void __launch_bounds__(kBlock) k_loss(int n, const float* __restrict__ O, const float* __restrict__ T,
                                                 const double* __restrict__ tpart, int ntp, float* __restrict__ dO,
                                                 double* __restrict__ part) {
  __shared__ double red[kBlock];
  __shared__ double denom;
  if (threadIdx.x == 0) {
    double d = 0.0;
    for (int q = 0; q < ntp; ++q) d += tpart[q];
    denom = d > 0.0 ? d : 1.0;
  }
  __syncthreads();
  double a = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    for (int c = 0; c < 16; ++c) {
      float g = 0.f;
      if (c < 2) {
        const double e = (double)O[(int64_t)i * 16 + c] - (double)T[2 * (int64_t)i + c];
        a += e * e;
        g = (float)(2.0 * e / denom);
      }
      dO[(int64_t)i * 16 + c] = g;
    }
  }
  red[threadIdx.x] = a / denom;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// The pre-activation gradients dZ reach the MFMA kernels in BF16 (rounded to nearest even once,
// here) in two layouts: row-major dZr[node][j] for the input gradient and transposed
// dZt[j][ld] for the weight gradient, whose inner dimension is the node (rows padded with
// zeros to whole tiles of kGradNodes, so every 16-byte operand load is aligned and in bounds).
constexpr int kGradNodes = 64;  // nodes per block of the kernels that write dZ

// One tile of kGradNodes nodes: tile[nd][j] (FP32, zero beyond n) is in LDS; writes its
// BF16 transpose and the tile's bias gradient dbp[block][j] = Σ_nodes dZ (FP32, fixed order).
// Every thread of the 256-thread block calls it after a barrier.
template <int C>
__device__ __forceinline__ void write_dz_tile(const float (*tile)[C + 1], int node0, int64_t ld,
                                              uint16_t* __restrict__ dZt, float* __restrict__ dbp) {
  for (int e = threadIdx.x; e < C * kGradNodes / 8; e += 256) {
    const int j = e / (kGradNodes / 8), q = (e % (kGradNodes / 8)) * 8;
    float v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = tile[q + r][j];
    *reinterpret_cast<short8_t*>(dZt + (int64_t)j * ld + node0 + q) = __builtin_bit_cast(short8_t, pack8(v));
  }
  if (threadIdx.x < C) {
    float b = 0.f;
    for (int nd = 0; nd < kGradNodes; ++nd) b += tile[nd][threadIdx.x];
    dbp[(int64_t)blockIdx.x * C + threadIdx.x] = b;
  }
}

// Output layer: dZ = dO (n × 16), no activation.
__global__ void __launch_bounds__(256) k_dz_out(int n, int64_t ld, const float* __restrict__ dO,
                                                uint16_t* __restrict__ dZr, uint16_t* __restrict__ dZt,
                                                float* __restrict__ dbp) {
  __shared__ float tile[kGradNodes][17];
  const int node0 = blockIdx.x * kGradNodes;
  for (int e = threadIdx.x; e < kGradNodes * 16; e += 256) {
    const int nd = e / 16, j = e % 16;
    const float v = node0 + nd < n ? dO[(int64_t)(node0 + nd) * 16 + j] : 0.f;
    tile[nd][j] = v;
    if (node0 + nd < n) dZr[(int64_t)(node0 + nd) * 16 + j] = bf16_bits(v);
  }
  __syncthreads();
  write_dz_tile<16>(tile, node0, ld, dZt, dbp);
}

// 8×8 transpose of 16-bit elements in registers: x[r] holds 8 channels of node r, f[t] the 8
// nodes of channel t. Two byte permutes per pair of dwords, 32 in all.
__device__ __forceinline__ void transpose8(const short8_t (&x)[8], bf16x8_t (&f)[8]) {
  typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
  uint4_t in[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) in[r] = __builtin_bit_cast(uint4_t, x[r]);
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    uint4_t o;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      o[q] = __builtin_amdgcn_perm(in[2 * q + 1][t / 2], in[2 * q][t / 2], t & 1 ? 0x07060302u : 0x05040100u);
    f[t] = __builtin_bit_cast(bf16x8_t, o);
  }
}

// Weight gradient partials over a chunk of nodes (a multiple of 32):
// dW_part[chunk][k][j] = Σ_nodes A[node][k]·dZ[node][j], an MFMA product with the nodes as the
// inner dimension. A wave takes 128 rows k (two neighbour slots of 64 channels, or 128
// columns of the dense first layer) against all COUT columns: per step of 32 nodes each lane
// reads 8 consecutive channels of 8 nodes (16-byte loads, 8 lanes to a 128-byte activation
// row) and transposes them in registers into the A fragments of 8 tiles; lane q of a 16-row tile
// t then stands for row (q >> 3)·64 + 8(q & 7) + t. The B fragments are 16-byte loads of dZt.
// Bound by the gathers' latency; 128 chunks (512 for the small products) give about one wave per SIMD
// with the next step's rows in flight. One 16×16 tile per wave with scalar 2-byte gathers, 18
// to 27 blocks of 2048 nodes, took 10.4 ms per 64 → 64 layer at 55,111 nodes; this takes 38 µs.
template <bool kDense, int COUT>
__global__ void __launch_bounds__(256) k_wgrad(int n, int chunk, int64_t ld, const uint16_t* __restrict__ X,
                                               const int* __restrict__ nbr, const uint16_t* __restrict__ dZt,
                                               float* __restrict__ dWp) {
  constexpr int K = kDense ? 256 : 1024, NT = COUT / 16;
  const int lane = threadIdx.x & 63;
  const int kb = blockIdx.y * (blockDim.x >> 6) + (threadIdx.x >> 6);  // 128-row block of dW
  const int n0 = blockIdx.x * chunk, n1 = min(n, n0 + chunk);
  const int nq = 8 * (lane >> 4);                   // the lane's nodes within a step
  const int half = (lane >> 3) & 1, c0 = 8 * (lane & 7);
  f32x4_t acc[8][NT];
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const short8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
  auto load = [&](int nb, short8_t (&x)[8]) {
    int64_t at[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int nd = min(nb + nq + r, n - 1);
      at[r] = kDense ? (int64_t)nd * K + kb * 128 + half * 64 : (int64_t)nbr[(int64_t)nd * kSlots + 2 * kb + half] * 64;
    }
#pragma unroll
    for (int r = 0; r < 8; ++r)
      x[r] = nb + nq + r < n1 ? *reinterpret_cast<const short8_t*>(X + at[r] + c0) : zero;
  };
  short8_t x[8];
  load(n0, x);
  for (int nb = n0; nb < n1; nb += 32) {
    bf16x8_t f[8], b[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = load8_bf16(dZt + (int64_t)(j * 16 + (lane & 15)) * ld + nb + nq);
    transpose8(x, f);
    if (nb + 32 < n1) load(nb + 32, x);
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[t], b[j], acc[t][j], 0, 0, 0);
  }
  float* __restrict__ out = dWp + (int64_t)blockIdx.x * K * COUT;
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = 4 * (lane >> 4) + r;
      const int k = kb * 128 + (q >> 3) * 64 + 8 * (q & 7) + t;
#pragma unroll
      for (int j = 0; j < NT; ++j) out[(int64_t)k * COUT + j * 16 + (lane & 15)] = acc[t][j][r];
    }
}

// grads[off + e] = Σ_blocks part[blk·count + e] (fixed order): 64 elements per block, the
// partials split over its four waves and combined in wave order.
__global__ void __launch_bounds__(kBlock) k_sum_parts(int64_t count, int nblk, const float* __restrict__ part,
                                                      float* __restrict__ out) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  const int q0 = (int)((int64_t)nblk * w / 4), q1 = (int)((int64_t)nblk * (w + 1) / 4);
  float s = 0.f;
  if (e < count) {
#pragma unroll 8
    for (int q = q0; q < q1; ++q) s += part[(int64_t)q * count + e];
  }
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && e < count) out[e] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// Bias gradient: out[j] = Σ_tiles part[tile·count + j], one block per j (fixed order).
__global__ void __launch_bounds__(kBlock) k_sum_bias(int count, int ntile, const float* __restrict__ part,
                                                     float* __restrict__ out) {
  __shared__ float red[kBlock];
  float s = 0.f;
  for (int q = threadIdx.x; q < ntile; q += kBlock) s += part[(int64_t)q * count + blockIdx.x];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// dA[node][k] = Σ_j dZ[node][j]·W[k][j] as the MFMA product W·dZᵀ (W rows as A, nodes as columns),
// so that a lane holds four consecutive k of one node: 16-byte stores. A block takes 64
// nodes; each of its waves a quarter of the rows k, every W fragment serving four node tiles.
// Bound by writing dA (4 KB per node): 64 µs per 64 → 64 layer at 55,111 nodes (3.5 TB/s), 104 µs
// with 4-byte stores and one node tile per W fragment.
template <int COUT>
__global__ void __launch_bounds__(256) k_dgrad(int n, const uint16_t* __restrict__ dZr,
                                               const uint16_t* __restrict__ Wk, float* __restrict__ dA) {
  constexpr int K = kSlots * 64, JS = (COUT + 31) / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int jq = 8 * (lane >> 4);
  const bf16x8_t none = __builtin_bit_cast(bf16x8_t, short8_t{0, 0, 0, 0, 0, 0, 0, 0});
  bf16x8_t b[4][JS];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int nd = blockIdx.x * 64 + u * 16 + (lane & 15);
#pragma unroll
    for (int s = 0; s < JS; ++s)
      b[u][s] = nd < n && s * 32 + jq < COUT ? load8_bf16(dZr + (int64_t)nd * COUT + s * 32 + jq) : none;
  }
  for (int kt = wave * (K / 64); kt < (wave + 1) * (K / 64); ++kt) {
    bf16x8_t a[JS];
#pragma unroll
    for (int s = 0; s < JS; ++s)
      a[s] = s * 32 + jq < COUT ? load8_bf16(Wk + (int64_t)(kt * 16 + (lane & 15)) * COUT + s * 32 + jq) : none;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < JS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[u][s], acc, 0, 0, 0);
      const int nd = blockIdx.x * 64 + u * 16 + (lane & 15);
      if (nd < n) *reinterpret_cast<f32x4_t*>(dA + (int64_t)nd * K + kt * 16 + 4 * (lane >> 4)) = acc;
    }
  }
}

// dX[j][c] = Σ_{(i, slot) with nbr[i][slot] = j} dA[i][slot·64 + c] over the reverse lists (sorted,
// so the sum order is fixed), then dZ = dX ⊙ act'(X) of the layer below (X its stored BF16
// activation, whose sign is that of the pre-activation) in both layouts. 16 lanes read a
// node's 256-byte rows of dA, four entries in flight; 16 nodes at a time, 64 per block. 58 µs at
// 55,111 nodes (3.9 TB/s of dA), against 93 µs for the sum alone with one 4-byte channel per lane.
__global__ void __launch_bounds__(256) k_scatter_back(int n, int64_t ld, const int64_t* __restrict__ rrow,
                                                      const int* __restrict__ rent, const float* __restrict__ dA,
                                                      const uint16_t* __restrict__ X, uint16_t* __restrict__ dZr,
                                                      uint16_t* __restrict__ dZt, float* __restrict__ dbp) {
  __shared__ float tile[kGradNodes][65];
  typedef short short4_t __attribute__((ext_vector_type(4)));
  const int node0 = blockIdx.x * kGradNodes, c = 4 * (threadIdx.x & 15);
  for (int g = threadIdx.x >> 4; g < kGradNodes; g += 16) {
    const int j = node0 + g;
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
    if (j < n) {
      const int64_t e = rrow[j + 1];
      int64_t q = rrow[j];
      for (; q + 4 <= e; q += 4) {
        f32x4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)  // entry i·16 + slot is row i·16 + slot of dA's 64-channel rows
          v[u] = *reinterpret_cast<const f32x4_t*>(dA + (int64_t)rent[q + u] * 64 + c);
#pragma unroll
        for (int u = 0; u < 4; ++u) s += v[u];
      }
      for (; q < e; ++q) s += *reinterpret_cast<const f32x4_t*>(dA + (int64_t)rent[q] * 64 + c);
      const short4_t y = *reinterpret_cast<const short4_t*>(X + (int64_t)j * 64 + c);
      short4_t o;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] *= dact(bf16_to_f32((uint16_t)y[r]));
        o[r] = (short)bf16_bits(s[r]);
      }
      *reinterpret_cast<short4_t*>(dZr + (int64_t)j * 64 + c) = o;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) tile[g][c + r] = s[r];
  }
  __syncthreads();
  write_dz_tile<64>(tile, node0, ld, dZt, dbp);
}

// Reverse lists: entries e = i·16 + slot by neighbour nbr[e], increasing within a row. The
// arrival-ordered slot of each entry comes with the count; each entry then ranks itself in its row.
__global__ void __launch_bounds__(kBlock) k_rev_count(int64_t ne, const int* __restrict__ nbr, int* __restrict__ slot,
                                                      int64_t* __restrict__ cnt) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e < ne) slot[e] = (int)atomicAdd((unsigned long long*)&cnt[nbr[e]], 1ull);
}

__global__ void __launch_bounds__(kBlock) k_rev_fill(int64_t ne, const int* __restrict__ nbr,
                                                     const int64_t* __restrict__ row, const int* __restrict__ slot,
                                                     int* __restrict__ tmp) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e < ne) tmp[row[nbr[e]] + slot[e]] = (int)e;
}

__global__ void __launch_bounds__(kBlock) k_rev_place(int64_t ne, const int* __restrict__ nbr,
                                                      const int64_t* __restrict__ row, const int* __restrict__ tmp,
                                                      int* __restrict__ ent) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= ne) return;
  const int j = nbr[e];
  const int64_t s = row[j], t = row[j + 1];
  int64_t at = s;
  for (int64_t q = s; q < t; ++q) at += tmp[q] < (int)e;
  ent[at] = (int)e;
}

// Adam on the FP32 master parameters (bias-corrected), then the BF16 copies of the weights.
__global__ void __launch_bounds__(kBlock) k_adam(int64_t np, float* __restrict__ w, const float* __restrict__ g,
                                                 float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                                 float b2, float eps, float c1, float c2) {
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < np; e += (int64_t)gridDim.x * kBlock) {
    const float ge = g[e];
    const float me = b1 * m[e] + (1.f - b1) * ge;
    const float ve = b2 * v[e] + (1.f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    w[e] -= lr * (me / c1) / (sqrtf(ve / c2) + eps);
  }
}

__global__ void __launch_bounds__(kBlock) k_cast(int K, int COUT, const float* __restrict__ W, uint16_t* __restrict__ wt,
                                                 uint16_t* __restrict__ wk) {
  const int e = blockIdx.x * kBlock + threadIdx.x;
  if (e >= K * COUT) return;
  const int k = e / COUT, j = e % COUT;
  const uint16_t b = bf16_bits(W[e]);
  wk[e] = b;
  wt[(int64_t)j * K + k] = b;
}

}  // namespace nnk
}  // namespace pb

// ---------------------------------------------------------------- host side

namespace pb {
namespace {

using namespace nnk;

struct NNBufs {
  int* nbr;
  float* feat;
  int64_t* rrow;
  int* rent;
  double* s;
  double* spart;
  uint32_t* vs;  // the scaled inputs of every node (k_pack_in)
  uint16_t* G1;
  uint16_t* X[kLayers];  // BF16; X[0] unused (layer 0 reads G1); X[l] = input of layer l
  float* T;
  float* dO;
  uint16_t* dZr;  // BF16 pre-activation gradients, row-major and transposed (see k_dz_out)
  uint16_t* dZt;
  int64_t ld;     // row length of dZt
  float* dA;
  float* dWp;
  float* dbp;
  double* lpart;
};

constexpr int kRedBlocks = 256;
// Node chunks of a weight gradient with `rows` rows and COUT columns: at least 256 nodes each
// (8 MFMA steps) and at most 32 MB of partial products in all.
int wgrad_chunk(int n, int rows, int cout) {
  const int most = (32 << 20) / (4 * rows * cout);
  const int c = std::max(256, (n + most - 1) / most);
  return (c + 31) / 32 * 32;
}

// The buffers of one application, and with `train` those of the backward pass.
pb_status bufs(pb_ctx* ctx, int n, NNBufs& B, bool train = false) {
  auto ws = [&](const char* name, size_t bytes) { return workspace(ctx, name, bytes); };
  B.nbr = (int*)ws("nn_nbr", sizeof(int) * (size_t)n * kSlots);
  B.feat = (float*)ws("nn_feat", sizeof(float) * (size_t)n * 5);
  B.s = (double*)ws("nn_s", sizeof(double) * 2);
  B.spart = (double*)ws("nn_spart", sizeof(double) * 2 * kRedBlocks);
  B.vs = (uint32_t*)ws("nn_vs", sizeof(uint32_t) * (size_t)n);
  B.G1 = (uint16_t*)ws("nn_G1", sizeof(uint16_t) * (size_t)n * kdim(0));
  B.X[0] = nullptr;
  B.X[1] = (uint16_t*)ws("nn_X1", sizeof(uint16_t) * (size_t)n * 64);
  B.X[2] = (uint16_t*)ws("nn_X2", sizeof(uint16_t) * (size_t)n * 64);
  B.X[3] = (uint16_t*)ws("nn_X3", sizeof(uint16_t) * (size_t)n * 64);
  if (!B.nbr || !B.feat || !B.s || !B.spart || !B.vs || !B.G1 || !B.X[1] || !B.X[2] || !B.X[3]) return PB_ENOMEM;
  if (!train) return PB_OK;
  B.rrow = (int64_t*)ws("nn_rrow", sizeof(int64_t) * (size_t)(n + 1));
  B.rent = (int*)ws("nn_rent", sizeof(int) * (size_t)n * kSlots);
  B.T = (float*)ws("nn_T", sizeof(float) * (size_t)n * 2);
  B.dO = (float*)ws("nn_dO", sizeof(float) * (size_t)n * 16);
  const int nt = (n + kGradNodes - 1) / kGradNodes;
  B.ld = (int64_t)nt * kGradNodes;
  B.dZr = (uint16_t*)ws("nn_dZr", sizeof(uint16_t) * (size_t)n * 64);
  B.dZt = (uint16_t*)ws("nn_dZt", sizeof(uint16_t) * (size_t)B.ld * 64);
  B.dA = (float*)ws("nn_dA", sizeof(float) * (size_t)n * 1024);
  const int cw = wgrad_chunk(n, 1024, 64), cs = wgrad_chunk(n, 256, 64);
  B.dWp = (float*)ws("nn_dWp", sizeof(float) * std::max((size_t)((n + cw - 1) / cw) * 1024 * 64,
                                                        (size_t)((n + cs - 1) / cs) * 256 * 64));
  B.dbp = (float*)ws("nn_dbp", sizeof(float) * (size_t)nt * 64);
  B.lpart = (double*)ws("nn_lpart", sizeof(double) * 2 * kRedBlocks);
  if (!B.rrow || !B.rent || !B.T || !B.dO || !B.dZr || !B.dZt || !B.dA || !B.dWp || !B.dbp || !B.lpart)
    return PB_ENOMEM;
  return PB_OK;
}

float* out_buf(pb_ctx* ctx, int n) { return (float*)workspace(ctx, "nn_O", sizeof(float) * (size_t)n * 16); }

}  // namespace

// Neighbour lists and geometry features of a band, cached on the context for the band last
// prepared. The reverse lists, which only the backward pass reads, are built by its first use.
pb_status nn_prepare(pb_ctx* ctx, const pb_band* band, const Derived& d) {
  const int n = (int)band->n;
  NNBufs B;
  PB_TRY(bufs(ctx, n, B));
  if (!band->phi) return ctx->fail(PB_EINVAL, "the learned path needs the band's phi array");
  MixedPlan P;
  PB_TRY(near_build(ctx, band, d, "nn_", P, NearBuild::cells));
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  k_knn<<<(unsigned)((n + kKnnWaves - 1) / kKnnWaves), 64 * kKnnWaves, 0, ctx->stream>>>(n, band_dev(band), cells_dev(P),
                                                                                       B.nbr);
  k_geom<<<nb, kBlock, 0, ctx->stream>>>(n, band_dev(band), band->phi, d.eps, B.nbr, B.feat);
  PB_TRY(launch_ok(ctx, "nn prepare"));
  ctx->nn_key = band->px;
  ctx->nn_n = n;
  ctx->nn_rev = false;
  return PB_OK;
}

// Reverse lists of (node, slot) per neighbour, of the lists nn_prepare left on the context.
static pb_status nn_reverse(pb_ctx* ctx, int n, const NNBufs& B) {
  if (ctx->nn_rev) return PB_OK;
  const int64_t ne = (int64_t)n * kSlots;
  int* slot = (int*)workspace(ctx, "nn_rslot", sizeof(int) * 2 * (size_t)ne);
  if (!slot) return PB_ENOMEM;
  int* tmp = slot + ne;
  PB_HIP(ctx, hipMemsetAsync(B.rrow, 0, sizeof(int64_t) * (size_t)(n + 1), ctx->stream));
  const unsigned nbe = (unsigned)((ne + kBlock - 1) / kBlock);
  k_rev_count<<<nbe, kBlock, 0, ctx->stream>>>(ne, B.nbr, slot, B.rrow);
  PB_TRY(launch_ok(ctx, "nn reverse count"));
  PB_TRY(exclusive_scan_i64(ctx, B.rrow, n + 1, nullptr));
  k_rev_fill<<<nbe, kBlock, 0, ctx->stream>>>(ne, B.nbr, B.rrow, slot, tmp);
  k_rev_place<<<nbe, kBlock, 0, ctx->stream>>>(ne, B.nbr, B.rrow, tmp, B.rent);
  PB_TRY(launch_ok(ctx, "nn reverse lists"));
  ctx->nn_rev = true;
  return PB_OK;
}

static pb_status nn_check_prepared(pb_ctx* ctx, const pb_band* band) {
  if (ctx->nn_key != band->px || ctx->nn_n != band->n)
    return ctx->fail(PB_EINVAL, "the learned path was not prepared for this band");
  return PB_OK;
}

// The four layers over n nodes in blocks of W waves: X[1..3] and O from the layer-1 rows and inputs.
template <int W>
static void forward_w(hipStream_t st, const pb_nn* net, int n, uint16_t* G1, const uint32_t* vs, bool store,
                      const int* nbr, uint16_t* const* X, float* O, const int* skip) {
  const unsigned blocks = (unsigned)((n + 16 * W - 1) / (16 * W));
  const uint16_t* wt = net->wt;
  const float* prm = net->params;
  k_layer_fwd<true, 16, 64, true, W><<<blocks, 64 * W, 0, st>>>(n, G1, vs, store, nullptr, nbr, wt + wbf_off(0),
                                                                prm + b_off(0), X[1], skip);
  for (int l = 1; l < 3; ++l)
    k_layer_fwd<false, 64, 64, true, W><<<blocks, 64 * W, 0, st>>>(n, nullptr, nullptr, 0, X[l], nbr, wt + wbf_off(l),
                                                                   prm + b_off(l), X[l + 1], skip);
  k_layer_fwd<false, 64, 16, false, W><<<blocks, 64 * W, 0, st>>>(n, nullptr, nullptr, 0, X[3], nbr, wt + wbf_off(3),
                                                                  prm + b_off(3), O, skip);
}

// Eight waves share the weights where the nodes fill the chip several times over, four spread fewer
// nodes more evenly: one application 105 µs with four waves a block and 113 with eight at 43,035 nodes (8591
// nodes: 71 and 80), 166 and 154 at 86,513, 249 and 234 at 156,535.
static void forward(hipStream_t st, const pb_nn* net, int n, uint16_t* G1, const uint32_t* vs, bool store,
                    const int* nbr, uint16_t* const* X, float* O, const int* skip) {
  if (n < 65536) forward_w<4>(st, net, n, G1, vs, store, nbr, X, O, skip);
  else forward_w<8>(st, net, n, G1, vs, store, nbr, X, O, skip);
}

// The geometry's part of the layer-1 rows of the band last prepared.
pb_status nn_rows(pb_ctx* ctx, const pb_band* band, const Derived& d) {
  PB_TRY(nn_check_prepared(ctx, band));
  const int n = (int)band->n;
  NNBufs B;
  PB_TRY(bufs(ctx, n, B));
  Scope t(ctx, "nn");
  k_build_g1<<<(unsigned)(((int64_t)n * kSlots + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
      n, band_dev(band), B.nbr, B.feat, d.eps, B.G1);
  return launch_ok(ctx, "nn rows");
}

// p = M(v), after nn_rows on the same band; keeps the activations of this application in the workspace,
// with `train` its layer-1 rows too.
pb_status nn_apply(pb_ctx* ctx, const pb_nn* net, const pb_band* band, const Derived& d, const double* v, double* p,
                   bool train) {
  PB_TRY(nn_check_prepared(ctx, band));
  const int n = (int)band->n;
  NNBufs B;
  PB_TRY(bufs(ctx, n, B));
  float* O = out_buf(ctx, n);
  if (!O) return PB_ENOMEM;
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  Scope t(ctx, "nn");
  k_rms_partial<<<kRedBlocks, kBlock, 0, ctx->stream>>>(n, v, B.spart);
  k_pack_in<<<nb, kBlock, 0, ctx->stream>>>(n, kRedBlocks, B.spart, v, B.s, B.vs);
  forward(ctx->stream, net, n, B.G1, B.vs, train, B.nbr, B.X, O, ctx->skip);
  k_apply_out<<<nb, kBlock, 0, ctx->stream>>>(n, v, O, B.s, d.lam1, d.lam2, p);
  return launch_ok(ctx, "nn apply");
}

// Loss and gradients (into net->grads) of the pair (v, u = A⁻¹v); loss to host.
pb_status nn_grads(pb_ctx* ctx, pb_nn* net, const pb_band* band, const Derived& d, const double* v, const double* u,
                   double* loss) {
  const int n = (int)band->n;
  double* ptmp = (double*)workspace(ctx, "nn_ptmp", sizeof(double) * 2 * (size_t)n);
  if (!ptmp) return PB_ENOMEM;
  PB_TRY(nn_rows(ctx, band, d));
  PB_TRY(nn_apply(ctx, net, band, d, v, ptmp, true));
  NNBufs B;
  PB_TRY(bufs(ctx, n, B, true));
  PB_TRY(nn_reverse(ctx, n, B));
  float* O = out_buf(ctx, n);
  const unsigned nt = (unsigned)((n + kGradNodes - 1) / kGradNodes);
  Scope t(ctx, "nn");
  k_target<<<kRedBlocks, kBlock, 0, ctx->stream>>>(n, v, u, B.s, d.lam1, d.lam2, B.T, B.lpart);
  k_loss<<<kRedBlocks, kBlock, 0, ctx->stream>>>(n, O, B.T, B.lpart, kRedBlocks, B.dO, B.lpart + kRedBlocks);
  float* g = net->grads;
  k_dz_out<<<nt, 256, 0, ctx->stream>>>(n, B.ld, B.dO, B.dZr, B.dZt, B.dbp);
  // layers 3 to 1 gather X[l] (dX_l ⊙ act'(X_l) is the layer below's dZ); layer 0 reads G1 and
  // has no input gradient
  for (int l = kLayers - 1; l >= 0; --l) {
    const int rows = kdim(l), cout = kCout[l];
    const int chunk = wgrad_chunk(n, rows, cout), nc = (n + chunk - 1) / chunk;
    if (l == 0)
      k_wgrad<true, 64><<<dim3(nc, 1), 128, 0, ctx->stream>>>(n, chunk, B.ld, B.G1, B.nbr, B.dZt, B.dWp);
    else if (l == kLayers - 1)
      k_wgrad<false, 16><<<dim3(nc, 2), 256, 0, ctx->stream>>>(n, chunk, B.ld, B.X[l], B.nbr, B.dZt, B.dWp);
    else
      k_wgrad<false, 64><<<dim3(nc, 2), 256, 0, ctx->stream>>>(n, chunk, B.ld, B.X[l], B.nbr, B.dZt, B.dWp);
    k_sum_parts<<<(unsigned)(rows * cout / 64), kBlock, 0, ctx->stream>>>((int64_t)rows * cout, nc, B.dWp, g + w_off(l));
    k_sum_bias<<<(unsigned)cout, kBlock, 0, ctx->stream>>>(cout, (int)nt, B.dbp, g + b_off(l));
    if (l == 0) break;
    if (l == kLayers - 1)
      k_dgrad<16><<<nt, 256, 0, ctx->stream>>>(n, B.dZr, net->wk + wbf_off(l), B.dA);
    else
      k_dgrad<64><<<nt, 256, 0, ctx->stream>>>(n, B.dZr, net->wk + wbf_off(l), B.dA);
    k_scatter_back<<<nt, 256, 0, ctx->stream>>>(n, B.ld, B.rrow, B.rent, B.dA, B.X[l], B.dZr, B.dZt, B.dbp);
  }
  PB_TRY(launch_ok(ctx, "nn backward"));
  if (loss) {
    std::vector<double> lp(kRedBlocks);
    PB_HIP(ctx, hipMemcpyAsync(lp.data(), B.lpart + kRedBlocks, sizeof(double) * kRedBlocks, hipMemcpyDeviceToHost,
                               ctx->stream));
    PB_TRY(sync(ctx, "nn loss"));
    double s = 0.0;
    for (double x : lp) s += x;
    *loss = s;
  }
  return PB_OK;
}

pb_status nn_cast(pb_ctx* ctx, pb_nn* net) {
  for (int l = 0; l < kLayers; ++l) {
    const int K = kdim(l), C = kCout[l];
    k_cast<<<(unsigned)((K * C + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
        K, C, net->params + w_off(l), net->wt + wbf_off(l), net->wk + wbf_off(l));
  }
  return launch_ok(ctx, "nn cast");
}

// ---------------------------------------------------------------- batch of bands

namespace {

// Per molecule: s[2m], s[2m + 1] = RMS of the two halves of its segment of v (1 when zero).
// One block per molecule, fixed summation order.
__global__ void __launch_bounds__(kBlock) k_rms_batch(int n_mol, const int* __restrict__ off, const int* __restrict__ cnt,
                                                      const double* __restrict__ V, int64_t ldv,
                                                      const int* __restrict__ kptr, int kmax, double* __restrict__ s) {
  __shared__ double r1[kBlock], r2[kBlock];
  const int m = blockIdx.x;
  if (m >= n_mol) return;
  if (kptr && *kptr >= kmax) return;
  const double* v = V + (kptr ? (int64_t)(*kptr) * ldv : 0) + 2 * (int64_t)off[m];
  const int n = cnt[m];
  double a = 0.0, c = 0.0;
  for (int i = threadIdx.x; i < n; i += kBlock) {
    a += v[i] * v[i];
    c += v[n + i] * v[n + i];
  }
  r1[threadIdx.x] = a;
  r2[threadIdx.x] = c;
  __syncthreads();
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      r1[threadIdx.x] += r1[threadIdx.x + o];
      r2[threadIdx.x] += r2[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double q1 = sqrt(r1[0] / n), q2 = sqrt(r2[0] / n);
    s[2 * m] = q1 > 0.0 ? q1 : 1.0;
    s[2 * m + 1] = q2 > 0.0 ? q2 : 1.0;
  }
}

// The scaled inputs of every node of the batch.
__global__ void __launch_bounds__(kBlock) k_pack_in_batch(int ntot, const int* __restrict__ mol_of,
                                                          const int* __restrict__ off, const int* __restrict__ cnt,
                                                          const double* __restrict__ V, int64_t ldv,
                                                          const int* __restrict__ kptr, int kmax,
                                                          const double* __restrict__ s, uint32_t* __restrict__ vs) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= ntot) return;
  if (kptr && *kptr >= kmax) return;
  const int m = mol_of[i], n = cnt[m], l = i - off[m];
  const double* v = V + (kptr ? (int64_t)(*kptr) * ldv : 0) + 2 * (int64_t)off[m];
  vs[i] = input_pair(v[l], v[n + l], s[2 * m], s[2 * m + 1]);
}

// p = Λ⁻¹(v + s_m ⊙ O[:, 0:2]) over every molecule's segment.
__global__ void __launch_bounds__(kBlock) k_apply_out_batch(int ntot, const int* __restrict__ mol_of,
                                                            const int* __restrict__ off, const int* __restrict__ cnt,
                                                            const double* __restrict__ V, double* __restrict__ Z,
                                                            int64_t ldv, const int* __restrict__ kptr, int kmax,
                                                            const float* __restrict__ O, const double* __restrict__ s,
                                                            double lam1, double lam2) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= ntot) return;
  if (kptr && *kptr >= kmax) return;
  const int m = mol_of[i];
  const int n = cnt[m], l = i - off[m];
  const int64_t base = (kptr ? (int64_t)(*kptr) * ldv : 0) + 2 * (int64_t)off[m];
  Z[base + l] = (V[base + l] + s[2 * m] * (double)O[(int64_t)i * 16]) / lam1;
  Z[base + n + l] = (V[base + n + l] + s[2 * m + 1] * (double)O[(int64_t)i * 16 + 1]) / lam2;
}

// Local neighbour indices of one molecule → global node indices.
__global__ void __launch_bounds__(kBlock) k_batch_nbr(int64_t ne, int off, int* __restrict__ nbr) {
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (t < ne) nbr[t] += off;
}

}  // namespace

pb_status nn_batch_prepare(pb_ctx* ctx, int n_mol, const pb_band* bands, const int* off_host, const int* mol_of,
                           const Derived& d, NNBatch& nb) {
  int64_t ntot64 = 0;
  std::vector<int> cnt_host(n_mol);
  for (int m = 0; m < n_mol; ++m) {
    if (!bands[m].phi) return ctx->fail(PB_EINVAL, "the learned path needs each band's phi array (molecule %d)", m);
    cnt_host[m] = (int)bands[m].n;
    ntot64 += bands[m].n;
  }
  const int ntot = (int)ntot64;
  auto ws = [&](const char* name, size_t bytes) { return workspace(ctx, name, bytes); };
  nb.n_mol = n_mol;
  nb.ntot = ntot;
  nb.mol_of = mol_of;
  nb.off = (int*)ws("nnb_off", sizeof(int) * n_mol);
  nb.cnt = (int*)ws("nnb_cnt", sizeof(int) * n_mol);
  nb.vs = (uint32_t*)ws("nnb_vs", sizeof(uint32_t) * (size_t)ntot);
  nb.nbr = (int*)ws("nnb_nbr", sizeof(int) * kSlots * (size_t)ntot);
  nb.feat = (float*)ws("nnb_feat", sizeof(float) * 5 * (size_t)ntot);
  nb.s = (double*)ws("nnb_s", sizeof(double) * 2 * n_mol);
  nb.G1 = (uint16_t*)ws("nnb_G1", sizeof(uint16_t) * (size_t)ntot * kdim(0));
  nb.X[0] = nullptr;
  nb.X[1] = (uint16_t*)ws("nnb_X1", sizeof(uint16_t) * 64 * (size_t)ntot);
  nb.X[2] = (uint16_t*)ws("nnb_X2", sizeof(uint16_t) * 64 * (size_t)ntot);
  nb.X[3] = (uint16_t*)ws("nnb_X3", sizeof(uint16_t) * 64 * (size_t)ntot);
  nb.O = (float*)ws("nnb_O", sizeof(float) * 16 * (size_t)ntot);
  if (!nb.off || !nb.cnt || !nb.vs || !nb.nbr || !nb.feat || !nb.s || !nb.G1 || !nb.X[1] || !nb.X[2] || !nb.X[3] ||
      !nb.O)
    return PB_ENOMEM;
  PB_HIP(ctx, hipMemcpyAsync(nb.off, off_host, sizeof(int) * n_mol, hipMemcpyHostToDevice, ctx->stream));
  PB_HIP(ctx, hipMemcpyAsync(nb.cnt, cnt_host.data(), sizeof(int) * n_mol, hipMemcpyHostToDevice, ctx->stream));
  for (int m = 0; m < n_mol; ++m) {
    const pb_band* band = &bands[m];
    const int n = (int)band->n, o = off_host[m];
    MixedPlan P;
    PB_TRY(near_build(ctx, band, d, "nnb_", P, NearBuild::cells));
    const unsigned nbk = (unsigned)((n + kBlock - 1) / kBlock);
    int* nbr_m = nb.nbr + (int64_t)o * kSlots;
    k_knn<<<(unsigned)((n + kKnnWaves - 1) / kKnnWaves), 64 * kKnnWaves, 0, ctx->stream>>>(n, band_dev(band),
                                                                                         cells_dev(P), nbr_m);
    k_geom<<<nbk, kBlock, 0, ctx->stream>>>(n, band_dev(band), band->phi, d.eps, nbr_m, nb.feat + (int64_t)o * 5);
    const int64_t ne = (int64_t)n * kSlots;
    const unsigned nbe = (unsigned)((ne + kBlock - 1) / kBlock);
    k_build_g1<<<nbe, kBlock, 0, ctx->stream>>>(n, band_dev(band), nbr_m, nb.feat + (int64_t)o * 5, d.eps,
                                                nb.G1 + (int64_t)o * kdim(0));
    k_batch_nbr<<<nbe, kBlock, 0, ctx->stream>>>(ne, o, nbr_m);
    PB_TRY(launch_ok(ctx, "nn batch prepare"));
  }
  return PB_OK;
}

void nn_batch_apply(hipStream_t stream, const pb_nn* net, const NNBatch& nb, const double* V, double* Z, int64_t ldv,
                    const int* kptr, int kmax, double lam1, double lam2) {
  const int ntot = nb.ntot;
  k_rms_batch<<<nb.n_mol, kBlock, 0, stream>>>(nb.n_mol, nb.off, nb.cnt, V, ldv, kptr, kmax, nb.s);
  k_pack_in_batch<<<(unsigned)((ntot + kBlock - 1) / kBlock), kBlock, 0, stream>>>(ntot, nb.mol_of, nb.off, nb.cnt, V, ldv,
                                                                                 kptr, kmax, nb.s, nb.vs);
  forward(stream, net, ntot, nb.G1, nb.vs, false, nb.nbr, nb.X, nb.O, nullptr);
  k_apply_out_batch<<<(unsigned)((ntot + kBlock - 1) / kBlock), kBlock, 0, stream>>>(
      ntot, nb.mol_of, nb.off, nb.cnt, V, Z, ldv, kptr, kmax, nb.O, nb.s, lam1, lam2);
}

}  // namespace pb

// ---------------------------------------------------------------- C-ABI

extern "C" {

pb_status pb_nn_create(pb_ctx* ctx, uint64_t seed, pb_nn** out) {
  using namespace pb;
  using namespace pb::nnk;
  if (!ctx || !out) return PB_EINVAL;
  PB_HIP(ctx, hipSetDevice(ctx->device));
  pb_nn* net = new pb_nn();
  net->device = ctx->device;
  net->n_params = n_params();
  const size_t pb = sizeof(float) * (size_t)net->n_params;
  if (hipMalloc(&net->params, pb) != hipSuccess || hipMalloc(&net->grads, pb) != hipSuccess ||
      hipMalloc(&net->adam_m, pb) != hipSuccess || hipMalloc(&net->adam_v, pb) != hipSuccess ||
      hipMalloc(&net->wt, sizeof(uint16_t) * (size_t)n_wbf()) != hipSuccess ||
      hipMalloc(&net->wk, sizeof(uint16_t) * (size_t)n_wbf()) != hipSuccess) {
    pb_nn_destroy(net);
    return ctx->fail(PB_ENOMEM, "pb_nn_create: allocation failed");
  }
  // He-uniform weights from a SplitMix64 stream; biases zero; the output layer starts at zero
  // so an untrained network is exactly the diagonal solve Λ⁻¹.
  std::vector<float> h((size_t)net->n_params, 0.f);
  uint64_t st = seed;
  auto next = [&]() {
    uint64_t z = (st += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
  };
  for (int l = 0; l < kLayers - 1; ++l) {
    const double a = std::sqrt(6.0 / kdim(l));
    for (int64_t e = 0; e < (int64_t)kdim(l) * kCout[l]; ++e) h[w_off(l) + e] = (float)((2.0 * next() - 1.0) * a);
  }
  PB_HIP(ctx, hipMemcpy(net->params, h.data(), pb, hipMemcpyHostToDevice));
  PB_HIP(ctx, hipMemset(net->adam_m, 0, pb));
  PB_HIP(ctx, hipMemset(net->adam_v, 0, pb));
  PB_HIP(ctx, hipMemset(net->grads, 0, pb));
  PB_TRY(nn_cast(ctx, net));
  PB_TRY(sync(ctx, "pb_nn_create"));
  *out = net;
  return PB_OK;
}

void pb_nn_destroy(pb_nn* net) {
  if (!net) return;
  (void)hipSetDevice(net->device);
  for (void* p : {(void*)net->params, (void*)net->grads, (void*)net->adam_m, (void*)net->adam_v, (void*)net->wt,
                  (void*)net->wk})
    if (p) (void)hipFree(p);
  delete net;
}

int64_t pb_nn_param_count(void) { return pb::nnk::n_params(); }

pb_status pb_nn_get_params(pb_ctx* ctx, const pb_nn* net, float* host, float* grads_host) {
  if (!ctx || !net || (!host && !grads_host)) return PB_EINVAL;
  PB_HIP(ctx, hipSetDevice(ctx->device));
  PB_TRY(pb::sync(ctx, "pb_nn_get_params"));
  const size_t bytes = sizeof(float) * (size_t)net->n_params;
  if (host) PB_HIP(ctx, hipMemcpy(host, net->params, bytes, hipMemcpyDeviceToHost));
  if (grads_host) PB_HIP(ctx, hipMemcpy(grads_host, net->grads, bytes, hipMemcpyDeviceToHost));
  return PB_OK;
}

pb_status pb_nn_set_params(pb_ctx* ctx, pb_nn* net, const float* host) {
  if (!ctx || !net || !host) return PB_EINVAL;
  for (int64_t e = 0; e < net->n_params; ++e)
    if (!std::isfinite(host[e])) return ctx->fail(PB_EINVAL, "pb_nn_set_params: non-finite parameter %lld", (long long)e);
  PB_HIP(ctx, hipSetDevice(ctx->device));
  PB_HIP(ctx, hipMemcpy(net->params, host, sizeof(float) * (size_t)net->n_params, hipMemcpyHostToDevice));
  PB_TRY(pb::nn_cast(ctx, net));
  return pb::sync(ctx, "pb_nn_set_params");
}

pb_status pb_nn_prepare(pb_ctx* ctx, const pb_band* band, const pb_params* prm) {
  using namespace pb;
  if (!ctx) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  PB_HIP(ctx, hipSetDevice(ctx->device));
  PB_TRY(nn_prepare(ctx, band, derive(*prm)));
  return sync(ctx, "pb_nn_prepare");
}

pb_status pb_nn_apply(pb_ctx* ctx, const pb_nn* net, const pb_band* band, const pb_params* prm, const double* v,
                      double* p) {
  using namespace pb;
  if (!ctx || !net || !v || !p) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  PB_HIP(ctx, hipSetDevice(ctx->device));
  PB_TRY(nn_rows(ctx, band, derive(*prm)));
  PB_TRY(nn_apply(ctx, net, band, derive(*prm), v, p));
  return sync(ctx, "pb_nn_apply");
}

pb_status pb_nn_train_step(pb_ctx* ctx, pb_nn* net, const pb_band* band, const pb_params* prm, const double* v,
                           const double* u, float lr, double* loss) {
  using namespace pb;
  if (!ctx || !net || !v || !u || !(lr >= 0.f)) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  PB_HIP(ctx, hipSetDevice(ctx->device));
  PB_TRY(nn_grads(ctx, net, band, derive(*prm), v, u, loss));
  if (lr > 0.f) {
    net->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - std::pow(b1, (float)net->step), c2 = 1.f - std::pow(b2, (float)net->step);
    k_adam<<<1024, kBlock, 0, ctx->stream>>>(net->n_params, net->params, net->grads, net->adam_m, net->adam_v, lr, b1,
                                             b2, 1e-8f, c1, c2);
    PB_TRY(nn_cast(ctx, net));
  }
  return sync(ctx, "pb_nn_train_step");
}

pb_status pb_nn_geometry(pb_ctx* ctx, const pb_band* band, int* nbr_host, float* feat_host) {
  if (!ctx || !band) return PB_EINVAL;
  PB_TRY(pb::nn_check_prepared(ctx, band));
  PB_TRY(pb::sync(ctx, "pb_nn_geometry"));
  const size_t n = (size_t)band->n;
  if (nbr_host)
    PB_HIP(ctx, hipMemcpy(nbr_host, ctx->bufs["nn_nbr"].ptr, sizeof(int) * n * pb::nnk::kSlots, hipMemcpyDeviceToHost));
  if (feat_host) PB_HIP(ctx, hipMemcpy(feat_host, ctx->bufs["nn_feat"].ptr, sizeof(float) * n * 5, hipMemcpyDeviceToHost));
  return PB_OK;
}

}  // extern "C"
