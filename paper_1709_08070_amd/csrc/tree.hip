// Treecode far field of the mixed operator: the paper accelerates the operator with a
// kernel-independent fast multipole method (section "Fast linear solvers"); this is the
// cluster–particle form of the same idea, built for the GPU.
//
// Sources are clustered by an octree over the FP32 (scaled) coordinates, nodes renumbered in
// Morton order so that every tree node owns a contiguous range. A source cluster C far from
// a target batch is replaced by (p+1)³ proxy points ŷ_k, the tensor-product Chebyshev points
// of the second kind on C's bounding box, carrying the interpolation weights of its sources.
// With L_k the Lagrange basis of those points, interpolating the kernels in the source
// variable and differentiating the interpolant for the source normal derivatives gives
//   Q_k = Σ_j σw̃_j (n_j · ∇L_k(y_j)),   M_k = Σ_j w̃n_j L_k(y_j),
// and, for a target x with normal n_x, d = x − ŷ_k, r = |d| (scaled by σ = κ), E = e^{−r},
// a = E(1 + r):
//   S1 += [(1 − θ1 E) Q_k − (1 − E) M_k] / r
//   S2 += −(d · n_x)[(1 − a) Q_k − (1 − θ2 a) M_k] / r³,
// which are the four kernels of eq. IBIM-PBE (K11 and K21 as source-normal derivatives of
// G0 − θ1Gκ and G0 − Gκ, K12 = G0 − Gκ, K22 as the target-normal derivative of G0 − θ2Gκ)
// applied to the interpolated density. y1 = σS1 and y2 = σ²S2 as for the dense FP32 kernel.
//
// Octree, target batches and interaction lists are built once per band in tree_build.hip; each
// application packs the records, computes the proxy weights and runs one fused far-field kernel
// over the batches' lists, cut into segments of about equal work. Direct sources are evaluated
// with the dense FP32 pair function (near pairs excluded by the shared FP32 predicate, the FP64 near
// field supplies them). Fixed orders throughout: the operator is bitwise reproducible.
//
// Local coordinates. The FP32 records hold σ(x − c) relative to the band's centre; their
// rounding, about 6e-8·|σ(x − c)|, is a relative error of |x − c|/r in the difference d of a
// pair at distance r, and the double-layer kernel amplifies it into the residual (at 2.57M
// band nodes it puts the FP32 operator about 1.2e-6·‖g‖ from the FP64 one, nearly all of it
// from pairs closer than 1 Å). The treecode therefore forms every difference from FP32
// coordinates local to an FP64 origin near the pair: a source of a direct range is stored
// as its offset from the centre of its aligned group of kAnchor tree-order nodes (a compact
// patch in Morton order) and the target is converted to the same origin, once per group, from
// its FP64 position; a proxy is stored as its offset from its cluster's FP64 centre, and the
// target converted to that centre once per cluster. The error in d is then about 6e-8 times
// the pair's own scale. Which pairs are near stays the shared FP32 predicate on the global
// records, evaluated on the direct ranges that can hold a near pair (marked when the lists are
// built); the other ranges skip it.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "pair_kernels.hpp"

namespace pb {
namespace {

constexpr int kProxyBlock = 256;
constexpr int kProxyTile = 64;

// 1D Chebyshev points of the second kind on [−1, 1], u_a = cos(πa/p), for degree p.
struct ChebNodes {
  float u[kTreeMaxDegree + 1];
};

// ℓ_a(u) and ℓ'_a(u) of the degree-(P1 − 1) Lagrange basis on the nodes u (product form).
template <int P1>
__device__ __forceinline__ void lagrange(float x, const ChebNodes& cn, float* L, float* dL) {
#pragma unroll
  for (int a = 0; a < P1; ++a) {
    float l = 1.f, dl = 0.f;
#pragma unroll
    for (int b = 0; b < P1; ++b) {
      if (b == a) continue;
      const float inv = 1.f / (cn.u[a] - cn.u[b]);
      const float f = (x - cn.u[b]) * inv;
      dl = dl * f + l * inv;
      l *= f;
    }
    L[a] = l;
    dL[a] = dl;
  }
}

// Tree-order records gathered from the band-order ones: At = (offset from the node's group
// anchor, w̃n ψn), Mt and Nt as in band order, and Gt = the FP32 global coordinates (the same
// bits the near-field predicate was evaluated on).
__global__ void __launch_bounds__(kBlock) k_tree_gather(int n, const int* __restrict__ perm,
                                                        const float4* __restrict__ A, const float4* __restrict__ M,
                                                        const float4* __restrict__ N, const double* __restrict__ St,
                                                        const double* __restrict__ anc, float4* __restrict__ At,
                                                        float4* __restrict__ Mt, float4* __restrict__ Nt,
                                                        float4* __restrict__ Gt) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t >= n) return;
  const int j = perm[t];
  const float4 a = A[j];
  const double* o = anc + 3 * (size_t)(t / kAnchor);
  const double* x = St + 3 * (size_t)t;
  At[t] = make_float4((float)(x[0] - o[0]), (float)(x[1] - o[1]), (float)(x[2] - o[2]), a.w);
  Mt[t] = M[j];
  Nt[t] = N[j];
  Gt[t] = make_float4(a.x, a.y, a.z, 0.f);
}

// Exact scaled coordinates in tree order, St[t] = σ(x − c) of band node perm[t] in FP64.
__global__ void __launch_bounds__(kBlock) k_tree_coords(int n, const int* __restrict__ perm, BandDev b, double cx,
                                                        double cy, double cz, double sigma, double* __restrict__ St) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t >= n) return;
  const int j = perm[t];
  St[3 * (size_t)t] = sigma * (b.px[j] - cx);
  St[3 * (size_t)t + 1] = sigma * (b.py[j] - cy);
  St[3 * (size_t)t + 2] = sigma * (b.pz[j] - cz);
}

// Anchor of each aligned group of kAnchor tree-order nodes: the centre of its bounding box.
__global__ void __launch_bounds__(kBlock) k_tree_anchor(int n, const double* __restrict__ St,
                                                        double* __restrict__ anc) {
  const int g = blockIdx.x * kBlock + threadIdx.x;
  if ((int64_t)g * kAnchor >= n) return;
  const int e = min(n, (g + 1) * kAnchor);
  for (int a = 0; a < 3; ++a) {
    double lo = INFINITY, hi = -INFINITY;
    for (int t = g * kAnchor; t < e; ++t) {
      lo = fmin(lo, St[3 * (size_t)t + a]);
      hi = fmax(hi, St[3 * (size_t)t + a]);
    }
    anc[3 * (size_t)g + a] = 0.5 * (lo + hi);
  }
}

// Partial proxy weights of one work item (cluster c, sources [b, e)): part[item][k] =
// (Q_k, M_k) summed over the item's sources in FP64. Cluster box: FP64 centre ccen[c],
// half-widths half[c]; the basis variable is u = (y − centre)/half per axis, formed in FP64
// from the exact coordinates St. Block of kProxyBlock threads; a tile of kProxyTile sources
// has its 1D bases evaluated once (three axes) and shared through LDS.
template <int P1>
__global__ void __launch_bounds__(kProxyBlock) k_proxy(const int4* __restrict__ items, const double* __restrict__ ccen,
                                                       const float4* __restrict__ half, const double* __restrict__ St,
                                                       const float4* __restrict__ At, const float4* __restrict__ Nt,
                                                       ChebNodes cn, double2* __restrict__ part,
                                                       const int* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int P3 = P1 * P1 * P1;
  constexpr int kPer = (P3 + kProxyBlock - 1) / kProxyBlock;
  __shared__ float sL[kProxyTile][3][P1], sD[kProxyTile][3][P1];
  __shared__ float4 sN[kProxyTile];
  __shared__ float sW[kProxyTile];
  const int4 it = items[blockIdx.x];  // (cluster, begin, end, unused)
  const float4 hw = half[it.x];
  const double* mid = ccen + 3 * (size_t)it.x;
  int ka[kPer], kb[kPer], kc[kPer];
  double q[kPer], m[kPer];
#pragma unroll
  for (int s = 0; s < kPer; ++s) {
    const int k = threadIdx.x + s * kProxyBlock;
    ka[s] = k / (P1 * P1);
    kb[s] = (k / P1) % P1;
    kc[s] = k % P1;
    q[s] = m[s] = 0.0;
  }
  for (int base = it.y; base < it.z; base += kProxyTile) {
    const int cnt = min(kProxyTile, it.z - base);
    if (threadIdx.x < 3 * kProxyTile) {
      const int j = threadIdx.x / 3, ax = threadIdx.x % 3;
      float L[P1], dL[P1];
      if (j < cnt) {
        const double ihd = 1.0 / (double)(ax == 0 ? hw.x : (ax == 1 ? hw.y : hw.z));
        const float s = (float)ihd;
        lagrange<P1>((float)((St[3 * (size_t)(base + j) + ax] - mid[ax]) * ihd), cn, L, dL);
#pragma unroll
        for (int b = 0; b < P1; ++b) dL[b] *= s;
      } else {
#pragma unroll
        for (int b = 0; b < P1; ++b) L[b] = dL[b] = 0.f;
      }
#pragma unroll
      for (int b = 0; b < P1; ++b) {
        sL[j][ax][b] = L[b];
        sD[j][ax][b] = dL[b];
      }
    }
    if (threadIdx.x < kProxyTile) {
      const int j = threadIdx.x;
      sN[j] = j < cnt ? Nt[base + j] : make_float4(0.f, 0.f, 0.f, 0.f);
      sW[j] = j < cnt ? At[base + j].w : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kPer; ++s) {
      if (threadIdx.x + s * kProxyBlock >= P3) continue;
      float qf = 0.f, mf = 0.f;
      for (int j = 0; j < cnt; ++j) {
        const float lx = sL[j][0][ka[s]], ly = sL[j][1][kb[s]], lz = sL[j][2][kc[s]];
        const float dx = sD[j][0][ka[s]], dy = sD[j][1][kb[s]], dz = sD[j][2][kc[s]];
        const float4 nw = sN[j];
        const float lyz = ly * lz;
        const float g = nw.x * dx * lyz + lx * (nw.y * dy * lz + nw.z * ly * dz);
        qf = fmaf(nw.w, g, qf);
        mf = fmaf(sW[j], lx * lyz, mf);
      }
      q[s] += (double)qf;
      m[s] += (double)mf;
    }
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < kPer; ++s) {
    const int k = threadIdx.x + s * kProxyBlock;
    if (k < P3) part[(size_t)blockIdx.x * P3 + k] = make_double2(q[s], m[s]);
  }
}

// Proxies of cluster c: position ŷ_k = centre + half·(u_a, u_b, u_c) and the weights Q_k, M_k,
// the sum of the cluster's item partials in item order. PX[k] = (ŷ_k − centre, Q_k) (the
// offset from the FP64 centre), PM[k] = M_k.
__global__ void __launch_bounds__(kBlock) k_proxy_sum(int n_cl, int P1, const int* __restrict__ item_ptr,
                                                      const double2* __restrict__ part, const float4* __restrict__ half,
                                                      ChebNodes cn, float4* __restrict__ PX, float* __restrict__ PM) {
  const int P3 = P1 * P1 * P1;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= (int64_t)n_cl * P3) return;
  const int c = (int)(g / P3), k = (int)(g % P3);
  double q = 0.0, m = 0.0;
  for (int it = item_ptr[c]; it < item_ptr[c + 1]; ++it) {
    const double2 v = part[(size_t)it * P3 + k];
    q += v.x;
    m += v.y;
  }
  const float4 hw = half[c];
  const int a = k / (P1 * P1), b = (k / P1) % P1, cc = k % P1;
  PX[g] = make_float4(hw.x * cn.u[a], hw.y * cn.u[b], hw.z * cn.u[cc], (float)q);
  PM[g] = (float)m;
}

// One target–proxy interaction (scaled coordinates, no near pair possible).
template <bool kScreened>
__device__ __forceinline__ void proxy_f32(const float4& ta, const float4& tn, const float4& sp, float sm,
                                          const F32Params& fp, float& a1, float& a2) {
  const float dx = ta.x - sp.x, dy = ta.y - sp.y, dz = ta.z - sp.z;
  const float r2 = __fmaf_rn(dz, dz, __fmaf_rn(dy, dy, dx * dx));
  const float rinv = __builtin_amdgcn_rsqf(r2);
  float E = 1.f, a = 1.f;
  if (kScreened) {
    const float z = r2 * rinv;
    E = __builtin_amdgcn_exp2f(fp.mlog2e * z);
    a = __fmaf_rn(E, z, E);
  }
  const float dn = __fmaf_rn(dz, tn.z, __fmaf_rn(dy, tn.y, dx * tn.x));
  // [(1 − θ1E)Q − (1 − E)M]/r and −dn[(1 − a)Q − (1 − θ2 a)M]/r³
  const float t1 = __fmaf_rn(__fmaf_rn(-fp.th1, E, 1.f), sp.w, -__fmaf_rn(-E, sm, sm));
  const float t2 = __fmaf_rn(-a, sp.w, sp.w) - __fmaf_rn(-fp.th2 * a, sm, sm);
  a1 = __fmaf_rn(t1, rinv, a1);
  a2 = __fmaf_rn(-dn * t2, rinv * rinv * rinv, a2);
}

// A direct pair in local coordinates (tl − sl = d) on a range that may hold near pairs: the
// shared FP32 predicate on the global coordinates tg, sg decides, and a near pair is replaced
// by a far stand-in with zero weights, which contributes exactly zero.
template <bool kScreened>
__device__ __forceinline__ void pair_local_checked(const float4& tl, const float4& tn, const float4& sl,
                                                   const float4& sm, const float4& tg, const float4& sg,
                                                   const F32Params& fp, float& a1, float& a2) {
  const bool near = r2_f32(tg.x, tg.y, tg.z, sg.x, sg.y, sg.z) < fp.rc2;
  const float4 s = near ? make_float4(tl.x + 1.f, tl.y, tl.z, 0.f) : sl;
  const float4 m = near ? make_float4(0.f, 0.f, 0.f, 0.f) : sm;
  pair_f32<kScreened, false>(tl, tn, s, m, fp, a1, a2);
}

// Far field of one work segment per wave (TreeSeg: some of the direct source ranges of a target
// batch, then some of its proxy clusters), the ranges with the dense pair function. Sources and proxies are staged 64 at a time in LDS (one
// record per lane, coalesced) and read back by every lane at the same address: an FP32
// instruction with a scalar-register operand issues at little more than half the rate of one on
// vector registers (4.1 against 2.2–2.6 cycles per wave), and about ten of a proxy's 26 instructions
// would have one if the records came through the scalar cache. Far field of 724,665 nodes: 14.1 ms
// through the scalar cache, 11.9 ms through LDS (one wave per batch both), 10.5 ms in segments. Differences
// are formed in local coordinates: per anchor group of a direct range and per proxy cluster, each
// lane converts its target's FP64 position to that origin. A range whose end carries the sign bit
// may hold near pairs and runs the predicate. FP32 sums per range and per cluster, flushed
// into FP64: seg_sum[segment][2][lane], unscaled.
template <bool kScreened>
__global__ void __launch_bounds__(kBatch) k_tree_far(const int2* __restrict__ batch, const TreeSeg* __restrict__ seg,
                                                     const int* __restrict__ seg_ptr, int n_batch,
                                                     const int2* __restrict__ dir_rng,
                                                     const int* __restrict__ app_cl, int P3,
                                                     const float4* __restrict__ PX, const float* __restrict__ PM,
                                                     const double* __restrict__ ccen, const float4* __restrict__ At,
                                                     const float4* __restrict__ Mt, const float4* __restrict__ Nt,
                                                     const float4* __restrict__ Gt, const double* __restrict__ St,
                                                     const double* __restrict__ anc, F32Params fp,
                                                     double* __restrict__ seg_sum, const int* __restrict__ skip) {
  if (skip && *skip) return;
  if ((int)blockIdx.x >= seg_ptr[n_batch]) return;  // the grid is an upper bound
  static_assert(kBatch == 64 && 64 % kAnchor == 0, "one wave per batch, whole anchor groups per stage");
  __shared__ float4 sA[64], sM[64], sG[64];
  __shared__ float sW[64];
  // staged records are read by all lanes of the wave that wrote them
  auto lds_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int lane = threadIdx.x;
  const TreeSeg sg = seg[blockIdx.x];
  const int2 bt = batch[sg.batch];
  const int t = bt.x + lane;
  const int tt = t < bt.y ? t : bt.x;  // idle lanes shadow the batch's first target (results unused)
  const double tx = St[3 * (size_t)tt], ty = St[3 * (size_t)tt + 1], tz = St[3 * (size_t)tt + 2];
  const float4 tn = Nt[tt], tg = Gt[tt];
  double acc1 = 0.0, acc2 = 0.0;
  for (int r = sg.d0; r < sg.d1; ++r) {
    const int2 rg = dir_rng[r];
    const bool check = rg.y < 0;
    const int end = rg.y & 0x7fffffff;
    float f1 = 0.f, f2 = 0.f;
    for (int base = rg.x / kAnchor * kAnchor; base < end; base += 64) {
      const int q = min(base + lane, end - 1);
      const float4 a = At[q], m = Mt[q];
      lds_order();
      sA[lane] = a;
      sM[lane] = m;
      if (check) sG[lane] = Gt[q];
      lds_order();
      for (int j = max(rg.x, base); j < min(end, base + 64);) {
        const int je = min(end, (j / kAnchor + 1) * kAnchor);
        const double* o = anc + 3 * (size_t)(j / kAnchor);
        const float4 tl = make_float4((float)(tx - o[0]), (float)(ty - o[1]), (float)(tz - o[2]), 0.f);
        if (check) {
          for (; j < je; ++j)
            pair_local_checked<kScreened>(tl, tn, sA[j - base], sM[j - base], tg, sG[j - base], fp, f1, f2);
        } else {
          for (; j + 4 <= je; j += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              pair_f32<kScreened, false>(tl, tn, sA[j - base + u], sM[j - base + u], fp, f1, f2);
          }
          for (; j < je; ++j) pair_f32<kScreened, false>(tl, tn, sA[j - base], sM[j - base], fp, f1, f2);
        }
      }
    }
    acc1 += (double)f1;
    acc2 += (double)f2;
  }
  for (int r = sg.a0; r < sg.a1; ++r) {
    const int cl = app_cl[r];
    const size_t base = (size_t)cl * P3;
    const double* o = ccen + 3 * (size_t)cl;
    const float4 tl = make_float4((float)(tx - o[0]), (float)(ty - o[1]), (float)(tz - o[2]), 0.f);
    float f1 = 0.f, f2 = 0.f;
    for (int k0 = 0; k0 < P3; k0 += 64) {
      const int q = min(k0 + lane, P3 - 1), cnt = min(64, P3 - k0);
      const float4 x = PX[base + q];
      const float m = PM[base + q];
      lds_order();
      sA[lane] = x;
      sW[lane] = m;
      lds_order();
      int k = 0;
      for (; k + 4 <= cnt; k += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) proxy_f32<kScreened>(tl, tn, sA[k + u], sW[k + u], fp, f1, f2);
      }
      for (; k < cnt; ++k) proxy_f32<kScreened>(tl, tn, sA[k], sW[k], fp, f1, f2);
    }
    acc1 += (double)f1;
    acc2 += (double)f2;
  }
  seg_sum[(size_t)blockIdx.x * 2 * kBatch + lane] = acc1;
  seg_sum[(size_t)blockIdx.x * 2 * kBatch + kBatch + lane] = acc2;
}

// The far field of a batch: its segments' sums in order, scaled by σ and σ², in band order.
__global__ void __launch_bounds__(kBatch) k_tree_sum(const int2* __restrict__ batch, const int* __restrict__ seg_ptr,
                                                     const double* __restrict__ seg_sum, const int* __restrict__ perm,
                                                     int n, double sig1, double sig2, double* __restrict__ out) {
  const int2 bt = batch[blockIdx.x];
  const int lane = threadIdx.x, t = bt.x + lane;
  if (t >= bt.y) return;
  double a1 = 0.0, a2 = 0.0;
  const int s1 = seg_ptr[blockIdx.x + 1];
  for (int s = seg_ptr[blockIdx.x]; s < s1; ++s) {
    a1 += seg_sum[(size_t)s * 2 * kBatch + lane];
    a2 += seg_sum[(size_t)s * 2 * kBatch + kBatch + lane];
  }
  const int i = perm[t];
  out[i] = sig1 * a1;
  out[n + i] = sig2 * a2;
}

}  // namespace

namespace {

template <int P1>
void launch_proxy(pb_ctx* ctx, const TreePlan& T, const ChebNodes& cn) {
  k_proxy<P1><<<(unsigned)T.n_items, kProxyBlock, 0, ctx->stream>>>(T.items, T.ccen, T.half, T.St, T.At, T.Nt, cn,
                                                                        T.part, ctx->skip);
}

void launch_tree(pb_ctx* ctx, const TreePlan& T, bool screened, const F32Params& fp, double sig1, double sig2) {
  ChebNodes cn{};
  const int P1 = T.degree + 1, P3 = P1 * P1 * P1;
  for (int a = 0; a < P1; ++a) cn.u[a] = T.u[a];
  if (T.n_items > 0) {
    switch (P1) {
      case 3: launch_proxy<3>(ctx, T, cn); break;
      case 4: launch_proxy<4>(ctx, T, cn); break;
      case 5: launch_proxy<5>(ctx, T, cn); break;
      case 6: launch_proxy<6>(ctx, T, cn); break;
      case 7: launch_proxy<7>(ctx, T, cn); break;
      case 8: launch_proxy<8>(ctx, T, cn); break;
      default: launch_proxy<9>(ctx, T, cn); break;
    }
    k_proxy_sum<<<(unsigned)(((int64_t)T.n_cl * P3 + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
        T.n_cl, P1, T.item_ptr, T.part, T.half, cn, T.PX, T.PM);
  }
  auto far = screened ? k_tree_far<true> : k_tree_far<false>;
  far<<<(unsigned)T.n_seg_max, kBatch, 0, ctx->stream>>>(T.batch, T.seg, T.seg_ptr, T.n_batch, T.dir_rng, T.app_cl, P3,
                                                          T.PX, T.PM, T.ccen, T.At, T.Mt, T.Nt, T.Gt, T.St, T.anc, fp,
                                                          T.seg_sum, ctx->skip);
  k_tree_sum<<<(unsigned)T.n_batch, kBatch, 0, ctx->stream>>>(T.batch, T.seg_ptr, T.seg_sum, T.perm, (int)T.n, sig1,
                                                              sig2, T.far);
}

}  // namespace

pb_status tree_coords(pb_ctx* ctx, const pb_band* band, const TreePlan& T) {
  const int n = (int)band->n, n_anc = (n + kAnchor - 1) / kAnchor;
  k_tree_coords<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
      n, T.perm, band_dev(band), T.near.cx, T.near.cy, T.near.cz, T.near.sigma, T.St);
  k_tree_anchor<<<(unsigned)((n_anc + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(n, T.St, T.anc);
  return launch_ok(ctx, "tree coordinates");
}

pb_status matvec_tree(pb_ctx* ctx, const pb_band* band, const Derived& d, const double* p, double* y,
                      const TreePlan& T, int64_t* near_total_dev) {
  const MixedPlan& P = T.near;
  const int n = (int)band->n;
  if (T.band_key != band->px || T.n != n || T.rc != d.rc)
    return ctx->fail(PB_EINVAL, "treecode operator used before its tree was prepared");
  double* near = (double*)workspace(ctx, "tc_near", sizeof(double) * 2 * (size_t)n);
  if (!near) return PB_ENOMEM;
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  k_pack_f32<<<nb, kBlock, 0, ctx->stream>>>(n, band_dev(band), band->w, p, d.h3 / (4.0 * kPi), P.cx, P.cy, P.cz,
                                             P.sigma, P.A, P.M, P.N);
  k_tree_gather<<<nb, kBlock, 0, ctx->stream>>>(n, T.perm, P.A, P.M, P.N, T.St, T.anc, T.At, T.Mt, T.Nt, T.Gt);
  const F32Params fp = f32params(d, P.sigma);
  const bool screened = d.kappa > 0.0;
  {
    Scope t(ctx, &T == &ctx->tree_fine ? "tree_fine_f32" : "tree_f32");
    launch_tree(ctx, T, screened, fp, P.sigma, P.sigma * P.sigma);
  }
  {
    Scope t(ctx, "near_f64");
    PB_TRY(near_apply(ctx, band, d, P, p, near, near_total_dev));
  }
  {
    Scope t(ctx, "reduce");
    k_reduce<<<(unsigned)((2 * n + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(n, 1, T.far, near, p, d.lam1,
                                                                                    d.lam2, y);
  }
  return launch_ok(ctx, "matvec_tree");
}

}  // namespace pb
