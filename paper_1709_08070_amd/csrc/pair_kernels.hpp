// Device code shared by the single-molecule and batched operators: the per-pair kernels
// of eq. IBIM-PBE with the regularization subsection, and the LDS-tiled source loops.
//
// With d = x_i* − y_j*, r = |d|, E = e^{−κr}, a = E(1+κr), b = E(3+3κr+κ²r²), the four
// kernels times 4π are
//   4πK11 = (d·n_j)(1 − θ1 a)/r³            4πK12 = (1 − E)/r
//   4πK21 = (n_i·n_j)(1 − a)/r³ − (d·n_i)(d·n_j)(3 − b)/r⁵
//   4πK22 = −(d·n_i)(1 − θ2 a)/r³
// and pairs inside the tangent disc of radius τ take the disc averages (0, K̄12, 0, 0).
#pragma once

#include <hip/hip_runtime.h>

#include "fp64_math.hpp"
#include "pb_internal.hpp"

namespace pb {

struct KParams {
  double th1, th2, kappa, tau2, four_tau2, k12bar4pi;
  double k11c, k22c, k21bar4pi;  // regularized pairs: 4πK11 = k11c·c_i, 4πK22 = k22c·c_i, 4πK21 = k21bar4pi
  int metric;
  int curved;                     // curvature-corrected disc averages (the kernels then read b.curv)
};

inline KParams kparams(const Derived& d) {
  return KParams{d.th1, d.th2, d.kappa, d.tau2, d.four_tau2, 4.0 * kPi * d.k12bar,
                 d.curved ? d.k11c : 0.0, d.curved ? d.k22c : 0.0, d.curved ? d.k21bar4pi : 0.0, d.metric,
                 d.curved ? 1 : 0};
}

// ---------------------------------------------------------------- FP64

// The four kernels times 4π for one pair in FP64. The regularization predicate uses the
// products and sums exactly as written (no contraction).
__device__ __forceinline__ void kern4_f64(double xi, double yi, double zi, double nxi, double nyi, double nzi,
                                          double xj, double yj, double zj, double nxj, double nyj, double nzj,
                                          const KParams& kp, double ci, double k[4]) {
  double dx = xi - xj, dy = yi - yj, dz = zi - zj;
  double r2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
  double dnx = __dadd_rn(__dadd_rn(__dmul_rn(dx, nxi), __dmul_rn(dy, nyi)), __dmul_rn(dz, nzi));
  double t2 = __dadd_rn(r2, -__dmul_rn(dnx, dnx));
  bool reg;
  if (kp.metric == PB_REG_EUCLIDEAN) reg = r2 < kp.tau2;
  else if (kp.metric == PB_REG_TANGENT) reg = t2 < kp.tau2;
  else reg = t2 < kp.tau2 && r2 < kp.four_tau2;
  if (reg) {  // disc averages; ci = κ1 + κ2 at the target (0 with the paper's averages)
    k[0] = kp.k11c * ci;
    k[1] = kp.k12bar4pi;
    k[2] = kp.k21bar4pi;
    k[3] = kp.k22c * ci;
    return;
  }
  double dny = dx * nxj + dy * nyj + dz * nzj;
  double nn = nxi * nxj + nyi * nyj + nzi * nzj;
  const double rinv = rsqrt_f64(r2);
  double r = r2 * rinv;
  double r3 = rinv * rinv * rinv;
  double r5 = r3 * rinv * rinv;
  double z = kp.kappa * r;
  double E = exp_neg_f64(z);
  double a = E * (1.0 + z);
  double b = E * (3.0 + 3.0 * z + z * z);
  k[0] = dny * (1.0 - kp.th1 * a) * r3;
  k[1] = (1.0 - E) * rinv;
  k[2] = nn * (1.0 - a) * r3 - dnx * dny * (3.0 - b) * r5;
  k[3] = -dnx * (1.0 - kp.th2 * a) * r3;
}

// s1 += 4πK11·wψ − 4πK12·wψn, s2 += 4πK21·wψ − 4πK22·wψn.
__device__ __forceinline__ void pair_f64(double xi, double yi, double zi, double nxi, double nyi, double nzi,
                                         double xj, double yj, double zj, double nxj, double nyj, double nzj,
                                         double wpsi, double wpsn, const KParams& kp, double ci, double& s1,
                                         double& s2) {
  double k[4];
  kern4_f64(xi, yi, zi, nxi, nyi, nzi, xj, yj, zj, nxj, nyj, nzj, kp, ci, k);
  s1 += k[0] * wpsi - k[1] * wpsn;
  s2 += k[2] * wpsi - k[3] * wpsn;
}

// ---------------------------------------------------------------- FP32

// FP32 records, coordinates centred on the band and scaled by σ = κ (σ = 1 when κ = 0):
//   A_j = (σ(x_j − c), w̃n_j),  M_j = σ·w̃_j·n_j,  N_j = (n_j, σ·w̃_j),
// with w̃_j = h³ω_jψ_j/(4π) and w̃n_j = h³ω_jψn_j/(4π). In scaled coordinates r' = κr = z, so
// e^{−κr} = exp2(−log2(e)·r') needs no extra product, and the sums come out as y1 = σ·S1,
// y2 = σ²·S2 (the scale is applied in FP64 afterwards). Folding the ψ weight into the source
// normal (M) lets one dot product give (d·n_j)·w̃_j and another (n_i·n_j)·w̃_j.
struct F32Params {
  float th1, th2, mlog2e, rc2;  // rc2: squared near-field radius in scaled units
  float far2;                   // rc2·(1 + 1e-3): a tile whose bounding box is at least this far
                                // (squared) from the target block holds no near pair
};

constexpr int kGroup = 256;  // records per bounding box (groups aligned at multiples of kGroup)

// Squared gap between two axis-aligned boxes (0 when they overlap).
__device__ __forceinline__ float box_gap2(const float4& lo1, const float4& hi1, const float4& lo2, const float4& hi2) {
  const float gx = fmaxf(0.f, fmaxf(lo2.x - hi1.x, lo1.x - hi2.x));
  const float gy = fmaxf(0.f, fmaxf(lo2.y - hi1.y, lo1.y - hi2.y));
  const float gz = fmaxf(0.f, fmaxf(lo2.z - hi1.z, lo1.z - hi2.z));
  return gx * gx + gy * gy + gz * gz;
}

// Union of the boxes of groups [g0, g1).
__device__ __forceinline__ void box_union(const float4* __restrict__ box, int g0, int g1, float4& lo, float4& hi) {
  lo = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
  hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.f);
  for (int g = g0; g < g1; ++g) {
    const float4 l = box[2 * g], h = box[2 * g + 1];
    lo.x = fminf(lo.x, l.x); lo.y = fminf(lo.y, l.y); lo.z = fminf(lo.z, l.z);
    hi.x = fmaxf(hi.x, h.x); hi.y = fmaxf(hi.y, h.y); hi.z = fmaxf(hi.z, h.z);
  }
}

// Squared distance in FP32 with a fixed operation sequence; every kernel that separates
// near from far pairs calls it on the same FP32 records.
__device__ __forceinline__ float r2_f32(float xi, float yi, float zi, float xj, float yj, float zj) {
  float dx = xi - xj, dy = yi - yj, dz = zi - zj;
  return __fmaf_rn(dz, dz, __fmaf_rn(dy, dy, __fmul_rn(dx, dx)));
}

// One far pair in FP32 (target record ta with normal tn, source records sa, sm). Near pairs
// (r'² < rc2, which includes the self pair and every regularized pair) contribute exactly
// zero: 1/r' is replaced by 0 and every term carries a factor of it. With d = x_i − x_j,
// D = d·M_j = (d·n_j)σw̃_j, Nw = n_i·M_j = (n_i·n_j)σw̃_j, a = E(1+z):
//   a1 += (1 − θ1 a) D/r'³ − (1 − E) w̃n_j/r'
//   a2 += [(1 − a) Nw + (1 − θ2 a)(d·n_i) w̃n_j + (d·n_i) D (E z² − 3(1 − a))/r'²]/r'³,
// the second line being K21 r'³ = (n_i·n_j)(1 − a) − (d·n_i)(d·n_j)(3 − b)/r'² with
// 3 − b = 3(1 − a) − E z², b = E(3 + 3z + z²).
// kCheck = false is for tiles known to hold no near pair (the predicate is then skipped).
template <bool kScreened, bool kCheck = true>
__device__ __forceinline__ void pair_f32(const float4& ta, const float4& tn, const float4& sa, const float4& sm,
                                         const F32Params& fp, float& a1, float& a2) {
  const float dx = ta.x - sa.x, dy = ta.y - sa.y, dz = ta.z - sa.z;
  const float r2 = r2_f32(ta.x, ta.y, ta.z, sa.x, sa.y, sa.z);
  float rinv = __builtin_amdgcn_rsqf(r2);
  if (kCheck && r2 < fp.rc2) rinv = 0.f;
  float E = 1.f, z = 0.f;
  if (kScreened) {
    z = r2 * rinv;
    E = __builtin_amdgcn_exp2f(fp.mlog2e * z);
  }
  const float a = __fmaf_rn(E, z, E);  // E(1 + r')
  const float dnx = __fmaf_rn(dz, tn.z, __fmaf_rn(dy, tn.y, dx * tn.x));
  const float D = __fmaf_rn(dz, sm.z, __fmaf_rn(dy, sm.y, dx * sm.x));
  const float Nw = __fmaf_rn(tn.z, sm.z, __fmaf_rn(tn.y, sm.y, tn.x * sm.x));
  const float ri2 = rinv * rinv;
  const float r3 = ri2 * rinv;
  const float c1 = __fmaf_rn(-fp.th1, a, 1.f);
  const float c2 = __fmaf_rn(-fp.th2, a, 1.f);
  a1 = __fmaf_rn(c1 * D, r3, a1);
  float t;
  if (kScreened) {
    const float f0w = __fmaf_rn(-E, sa.w, sa.w);  // (1 − E) w̃n_j
    a1 = __fmaf_rn(-f0w, rinv, a1);
    const float gr = __fmaf_rn(__fmaf_rn(3.f, a, -3.f), ri2, E);  // g/r'² = E − 3(1 − a)/r'²
    t = __fmaf_rn(-a, Nw, Nw);
    t = __fmaf_rn(c2 * dnx, sa.w, t);
    t = __fmaf_rn(dnx * D, gr, t);
  } else {  // κ = 0: E = a = 1 and z = 0, so only the θ terms remain
    t = c2 * dnx * sa.w;
  }
  a2 = __fmaf_rn(t, r3, a2);
}

// Targets [t0, t0 + kBlk·TPL) against sources [j0, j1) of the same record arrays; per-tile
// FP32 partial sums flushed into FP64. out1/out2 receive σ·S1 and σ²·S2 for each live target
// (index relative to t0). Every thread of the block must call it (it synchronizes).
// box: bounding boxes of the record groups (k_group_box); full source tiles whose box is
// farther than √far2 from the target block's box skip the near-pair predicate.
template <int kBlk, int TILE, int TPL, bool kScreened>
__device__ __forceinline__ void far_tile_loop(const float4* __restrict__ A, const float4* __restrict__ M,
                                              const float4* __restrict__ N, const float4* __restrict__ box, int t0,
                                              int t_end, int j0, int j1, const F32Params& fp, double sig1,
                                              double sig2, float4* sA, float4* sM, double* __restrict__ out1,
                                              double* __restrict__ out2) {
  static_assert(TILE % kGroup == 0, "source tiles are whole groups");
  float4 tlo, thi;
  box_union(box, t0 / kGroup, (min(t0 + kBlk * TPL, t_end) - 1) / kGroup + 1, tlo, thi);
  float4 ta[TPL], tn[TPL];
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    const int i = t0 + t * kBlk + (int)threadIdx.x;
    ta[t] = i < t_end ? A[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    tn[t] = i < t_end ? N[i] : make_float4(0.f, 0.f, 1.f, 0.f);
  }
  double acc1[TPL], acc2[TPL];
#pragma unroll
  for (int t = 0; t < TPL; ++t) acc1[t] = acc2[t] = 0.0;
  for (int base = j0; base < j1; base += TILE) {
    for (int q = threadIdx.x; q < TILE; q += kBlk) {
      const int j = base + q;
      if (j < j1) {
        sA[q] = A[j];
        sM[q] = M[j];
      } else {  // padding: zero weights, every value they meet is finite
        sA[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        sM[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    // block-uniform: the tile is full and its box is clear of the target block's box
    int clear = 0;
    if (base + TILE <= j1) {
      float4 slo, shi;
      box_union(box, base / kGroup, (base + TILE) / kGroup, slo, shi);
      clear = box_gap2(tlo, thi, slo, shi) >= fp.far2;
    }
    clear = __builtin_amdgcn_readfirstlane(clear);
    __syncthreads();
    float a1[TPL], a2[TPL];
#pragma unroll
    for (int t = 0; t < TPL; ++t) a1[t] = a2[t] = 0.f;
    if (clear) {
#pragma unroll 4
      for (int q = 0; q < TILE; ++q) {
        const float4 sa = sA[q], sm = sM[q];
#pragma unroll
        for (int t = 0; t < TPL; ++t) pair_f32<kScreened, false>(ta[t], tn[t], sa, sm, fp, a1[t], a2[t]);
      }
    } else {
#pragma unroll 4
      for (int q = 0; q < TILE; ++q) {
        const float4 sa = sA[q], sm = sM[q];
#pragma unroll
        for (int t = 0; t < TPL; ++t) pair_f32<kScreened, true>(ta[t], tn[t], sa, sm, fp, a1[t], a2[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
      acc1[t] += (double)a1[t];
      acc2[t] += (double)a2[t];
    }
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    const int i = t0 + t * kBlk + (int)threadIdx.x;
    if (i < t_end) {
      out1[i - t0] = sig1 * acc1[t];
      out2[i - t0] = sig2 * acc2[t];
    }
  }
}


// ---------------------------------------------------------------- kernels

constexpr int kBlock = 256;

struct BandDev {
  const double *px, *py, *pz, *nx, *ny, *nz;
  const double* curv;  // κ1 + κ2 at the projections, or null (flat disc averages)
};

// The band's geometry; the curvature only where the curvature-corrected averages use it.
inline BandDev band_dev(const pb_band* b, bool with_curv = false) {
  return BandDev{b->px, b->py, b->pz, b->nx, b->ny, b->nz, with_curv ? b->curv : nullptr};
}

// Source weights h³ω_j ψ_j/(4π), h³ω_j ψn_j/(4π) in FP64.
static __global__ void __attribute__((unused)) __launch_bounds__(kBlock) k_weights_f64(int n, const double* __restrict__ w,
                                                               const double* __restrict__ p, double scale,
                                                               double* __restrict__ wpsi, double* __restrict__ wpsn) {
  int j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= n) return;
  double s = scale * w[j];
  wpsi[j] = s * p[j];
  wpsn[j] = s * p[n + j];
}

// FP64 targets [t0, t0 + kBlk) against sources [j0, j1) of the band arrays b with source
// weights wpsi/wpsn (h³ωψ/4π, h³ωψn/4π); out1/out2 receive the sums for each live target
// (index relative to t0). Every thread of the block must call it (it synchronizes).
template <int kBlk>
__device__ __forceinline__ void far64_tile_loop(const BandDev& b, const double* __restrict__ wpsi,
                                                const double* __restrict__ wpsn, int t0, int t_end, int j0, int j1,
                                                const KParams& kp, double* smem, double* __restrict__ out1,
                                                double* __restrict__ out2) {
  double *sx = smem, *sy = sx + kBlk, *sz = sy + kBlk, *snx = sz + kBlk, *sny = snx + kBlk, *snz = sny + kBlk,
         *sw1 = snz + kBlk, *sw2 = sw1 + kBlk;
  const int i = t0 + (int)threadIdx.x;
  const bool live = i < t_end;
  double xi = 0, yi = 0, zi = 0, nxi = 0, nyi = 0, nzi = 1, ci = 0;
  if (live) {
    xi = b.px[i]; yi = b.py[i]; zi = b.pz[i];
    nxi = b.nx[i]; nyi = b.ny[i]; nzi = b.nz[i];
    ci = b.curv ? b.curv[i] : 0.0;
  }
  double s1 = 0.0, s2 = 0.0;
  for (int base = j0; base < j1; base += kBlk) {
    const int j = base + (int)threadIdx.x;
    if (j < j1) {
      sx[threadIdx.x] = b.px[j]; sy[threadIdx.x] = b.py[j]; sz[threadIdx.x] = b.pz[j];
      snx[threadIdx.x] = b.nx[j]; sny[threadIdx.x] = b.ny[j]; snz[threadIdx.x] = b.nz[j];
      sw1[threadIdx.x] = wpsi[j]; sw2[threadIdx.x] = wpsn[j];
    }
    __syncthreads();
    const int m = min(kBlk, j1 - base);
    if (live)
      for (int q = 0; q < m; ++q)
        pair_f64(xi, yi, zi, nxi, nyi, nzi, sx[q], sy[q], sz[q], snx[q], sny[q], snz[q], sw1[q], sw2[q], kp, ci, s1,
                 s2);
    __syncthreads();
  }
  if (live) {
    out1[i - t0] = s1;
    out2[i - t0] = s2;
  }
}

// FP64 operator, one target per lane; block (x: target block, y: source chunk).
static __global__ void __attribute__((unused)) __launch_bounds__(kBlock) k_p2p_f64(BandDev b, const double* __restrict__ wpsi,
                                                           const double* __restrict__ wpsn, int n, int chunk,
                                                           double* __restrict__ partial, KParams kp,
                                                           const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ double smem[8 * kBlock];
  const int t0 = blockIdx.x * kBlock;
  const int j0 = blockIdx.y * chunk;
  const int j1 = min(n, j0 + chunk);
  double* out = partial + (size_t)blockIdx.y * 2 * n;
  far64_tile_loop<kBlock>(b, wpsi, wpsn, t0, n, j0, j1, kp, smem, out + t0, out + n + t0);
}

// y = Λp + Σ_chunks partial (+ near), in a fixed order: eight sums over every eighth chunk, then those
// pairwise. One sum over all chunks, up to 256 of them, would round that often at the size of the result: on a
// sphere of 45,818 nodes with a smooth density (179 chunks) the two halves of the FP64 operator have a relative
// error of 0.7e-16 and 1.5e-16, with one sum 2.3e-16 and 2.8e-16. Bound by the reads of the partial sums, eight in
// flight a thread.
static __global__ void __attribute__((unused)) __launch_bounds__(kBlock) k_reduce(int n, int n_chunks, const double* __restrict__ partial,
                                                          const double* __restrict__ near,
                                                          const double* __restrict__ p, double lam1, double lam2,
                                                          double* __restrict__ y) {
  constexpr int kSums = 8;
  int e = blockIdx.x * kBlock + threadIdx.x;
  if (e >= 2 * n) return;
  double s[kSums] = {}, v[kSums];
  int c = 0;
  for (; c + kSums <= n_chunks; c += kSums)
#pragma unroll
    for (int u = 0; u < kSums; ++u) s[u] += partial[(size_t)(c + u) * 2 * n + e];
  // the rest, all read before any is added
#pragma unroll
  for (int u = 0; u < kSums; ++u) v[u] = c + u < n_chunks ? partial[(size_t)(c + u) * 2 * n + e] : 0.0;
#pragma unroll
  for (int u = 0; u < kSums; ++u) s[u] += v[u];
#pragma unroll
  for (int k = kSums / 2; k > 0; k /= 2)
#pragma unroll
    for (int u = 0; u < k; ++u) s[u] += s[u + k];
  if (near) s[0] += near[e];
  y[e] = (e < n ? lam1 : lam2) * p[e] + s[0];
}

// FP32 records of a band (layout above); with p == nullptr only the geometry is written
// (weights zero).
static __global__ void __attribute__((unused)) __launch_bounds__(kBlock) k_pack_f32(int n, BandDev b, const double* __restrict__ w,
                                                            const double* __restrict__ p, double scale, double cx,
                                                            double cy, double cz, double sigma,
                                                            float4* __restrict__ A, float4* __restrict__ M,
                                                            float4* __restrict__ N) {
  int j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= n) return;
  const double s = scale * w[j];
  const double w1 = p ? sigma * s * p[j] : 0.0, w2 = p ? s * p[n + j] : 0.0;
  A[j] = make_float4((float)(sigma * (b.px[j] - cx)), (float)(sigma * (b.py[j] - cy)), (float)(sigma * (b.pz[j] - cz)),
                     (float)w2);
  M[j] = make_float4((float)(w1 * b.nx[j]), (float)(w1 * b.ny[j]), (float)(w1 * b.nz[j]), 0.f);
  N[j] = make_float4((float)b.nx[j], (float)b.ny[j], (float)b.nz[j], (float)w1);
}

// FP32 far field of one band: block (x: kBlock·TPL targets, y: source chunk).
template <int TILE, int TPL, bool kScreened>
static __global__ void __attribute__((unused)) __launch_bounds__(kBlock) k_p2p_f32(const float4* __restrict__ A, const float4* __restrict__ M,
                                                           const float4* __restrict__ N,
                                                           const float4* __restrict__ box, int n, int chunk,
                                                           F32Params fp, double sig1, double sig2,
                                                           double* __restrict__ partial,
                                                           const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ float4 sA[TILE], sM[TILE];
  const int t0 = blockIdx.x * kBlock * TPL;
  const int j0 = blockIdx.y * chunk;
  const int j1 = min(n, j0 + chunk);
  double* out = partial + (size_t)blockIdx.y * 2 * n;
  far_tile_loop<kBlock, TILE, TPL, kScreened>(A, M, N, box, t0, n, j0, j1, fp, sig1, sig2, sA, sM, out + t0,
                                              out + n + t0);
}

// ----------------------------------------------------------------- near field

// Cell list of a band (near.hip): cells in lexicographic order, the nodes of a cell in
// increasing index, with their positions (and h³ω/4π's ω in w) in the same order.
struct CellsDev {
  const int* start;     // ncell + 1
  const int* nodes;     // n
  const int* cell_of;   // n
  const double4* pos;   // n, cell order
  int ncx, ncy, ncz;
  double inv;           // 1 / cell width
};

inline CellsDev cells_dev(const MixedPlan& P) {
  return CellsDev{P.cell_start, P.cell_nodes, P.cell_of, P.cell_pos, P.ncx, P.ncy, P.ncz, 1.0 / P.cell};
}

// The 27 cells around cell c are nine runs of cells contiguous in z, so nine contiguous ranges
// of the cell-ordered arrays: lane r < 9 of the wave gets range r (empty outside the grid), in
// lexicographic cell order.
__device__ __forceinline__ void cell_ranges(const CellsDev& cells, int c, int& lo, int& hi) {
  const int lane = threadIdx.x & 63;
  const int cz = c % cells.ncz, cy = (c / cells.ncz) % cells.ncy, cx = c / (cells.ncz * cells.ncy);
  const int ax = cx - 1 + lane / 3, ay = cy - 1 + lane % 3;
  lo = hi = 0;
  if (lane < 9 && ax >= 0 && ax < cells.ncx && ay >= 0 && ay < cells.ncy) {
    const int line = (ax * cells.ncy + ay) * cells.ncz;
    lo = cells.start[line + max(cz - 1, 0)];
    hi = cells.start[line + min(cz + 1, cells.ncz - 1) + 1];
  }
}

constexpr int kRowLanes = 16;  // lanes cooperating on one CSR row

// near = (near block matrix)·p, 16 lanes per row, fixed-order lane reduction.
static __global__ void __attribute__((unused)) __launch_bounds__(kBlock) k_near_spmv(int n, const int64_t* __restrict__ row,
                                                      const int* __restrict__ col, const double4* __restrict__ coef,
                                                      const double* __restrict__ p, double* __restrict__ near) {
  const int i = (blockIdx.x * kBlock + threadIdx.x) / kRowLanes;
  const int lane = threadIdx.x % kRowLanes;
  double s1 = 0.0, s2 = 0.0;
  if (i < n) {
    const int64_t e = row[i + 1];
    for (int64_t q = row[i] + lane; q < e; q += kRowLanes) {
      const int j = col[q];
      const double4 c = coef[q];
      const double ps = p[j], pn = p[n + j];
      s1 += c.x * ps + c.y * pn;
      s2 += c.z * ps + c.w * pn;
    }
  }
  for (int off = kRowLanes / 2; off > 0; off >>= 1) {
    s1 += __shfl_down(s1, off, kRowLanes);
    s2 += __shfl_down(s2, off, kRowLanes);
  }
  if (i < n && lane == 0) {
    near[i] = s1;
    near[n + i] = s2;
  }
}


}  // namespace pb
