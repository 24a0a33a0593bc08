// The IBIM operator y = Λp + KWp (eq. final-lin-sys) between the band nodes of one molecule.
//
// FP64 path: one target per lane, sources staged through LDS in tiles of 256, the source
// range split into chunks so that small bands still fill the 256 CUs; chunk partial sums are
// reduced in a fixed order (no atomics, bitwise reproducible).
//
// Mixed path: the FP32 far field (k_p2p_f32, rsq and exp2 on the transcendental unit, 32 B
// source records in LDS, FP32 partials per tile flushed to FP64) plus the FP64 near field, a
// CSR matrix of 2×2 blocks for every pair closer than r_c (≥ 2τ, so every regularized pair).
// Both sides decide "near" with the same FP32 function of the same FP32 records, so each pair
// is counted exactly once. The near matrix depends only on the geometry and is built once per
// band; each application is then an SpMV. The far kernel's tile shape (sources per LDS tile,
// targets per lane) or the symmetric kernel (each unordered pair once, both directions) is chosen by
// the band's size (far_choice). The near-field matrix and its cell list are built in near.hip.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "pair_kernels.hpp"
#include "sym64_kernels.hpp"
#include "sym_kernels.hpp"

namespace pb {
namespace {

struct FarCfg {
  int tile, tpl;
};
constexpr FarCfg kFarCfgs[] = {{256, 1}, {512, 1}, {256, 2}, {512, 2}};
constexpr int kNumTiled = sizeof(kFarCfgs) / sizeof(kFarCfgs[0]);
constexpr int kSymCfg = kNumTiled;  // the symmetric kernel
constexpr int kNumFarCfgs = kNumTiled + 1;

// Tiles of the symmetric kernels for a band of n nodes: F nodes per tile (512, 256 or 128: blocks of
// 4 × 1, 2 × 2 or 1 × 2 waves), chunks of nsub tiles. Small bands take small tiles: tiles of 512 give
// (n/512)²/2 blocks, too few for 256 CUs below about 40,000 nodes and in few, uneven rounds. Measured,
// tiles of 512 / 256 / 128, FP32 operator with its near field: at 13,393 nodes (far field alone) 148 /
// 110 / 111 µs, at 35,214 787 / 747 / –, at 43,035 1074 / 1040 / –, at 54,655 1589 / 1581 / –, at 61,591
// 1980 / 1985 / –; FP64 at 8725 nodes 356 / 192 / 170 µs, at 12,300 – / 264 / 260, at 16,020 – / 391 /
// 395, at 55,111 3947 / 3879 / –, at 105,085 equal.
struct SymShape {
  int F, nsub, chunks;
};
SymShape sym_shape(int n, bool f64) {
  const int F = n >= 61440 ? 512 : f64 && n < 13312 ? 128 : 256;
  const int C = F == kSymSub ? F * sym_nsub(n) : F;
  return {F, C / F, (n + C - 1) / C};
}

// Work items (Ic, Jc) of a symmetric kernel: chunk pairs within a sub-block first, which are
// one-directional (both orders) and the longer ones (last, they end the FP64 operator 3 to 6% later
// below 20,000 nodes), then those of different sub-blocks (Ic < Jc).
std::vector<int2> sym_items(const SymShape& sh) {
  const int nc = sh.chunks, per = std::max(1, kSymSub / (sh.F * sh.nsub));
  std::vector<int2> v;
  v.reserve((size_t)nc * (nc + 1) / 2 + (size_t)nc * per);
  for (int i = 0; i < nc; ++i)
    for (int j = i / per * per; j < std::min(nc, (i / per + 1) * per); ++j) v.push_back(make_int2(i, j));
  for (int i = 0; i < nc; ++i)
    for (int j = (i / per + 1) * per; j < nc; ++j) v.push_back(make_int2(i, j));
  return v;
}

// The item list on the device for a band of n nodes (rebuilt when n changes; one list per tile
// size).
const int2* sym_items_dev(pb_ctx* ctx, int n, const SymShape& sh, int* n_items) {
  char nm[32];
  snprintf(nm, sizeof(nm), "sym_items%d", sh.F);
  pb_ctx::SymList& l = ctx->sym_list[sh.F];
  if (l.n != n) {
    l.n = -1;
    const std::vector<int2> v = sym_items(sh);
    int2* d = (int2*)workspace(ctx, nm, sizeof(int2) * v.size());
    if (!d || hipMemcpyAsync(d, v.data(), sizeof(int2) * v.size(), hipMemcpyHostToDevice, ctx->stream) != hipSuccess)
      return nullptr;
    l.n = n;
    l.n_items = (int)v.size();
    l.dev = d;
  }
  *n_items = l.n_items;
  return l.dev;
}

// Source chunks for a launch: at least ~8 blocks per CU, chunks a multiple of the tile.
int far_chunks(pb_ctx* ctx, int n, int targets_per_block, int tile, int* chunk) {
  int tb = (n + targets_per_block - 1) / targets_per_block;
  int want = (8 * ctx->n_cu + tb - 1) / tb;
  int max_chunks = (n + tile - 1) / tile;
  int s = std::max(1, std::min(want, max_chunks));
  int c = (n + s - 1) / s;
  c = (c + tile - 1) / tile * tile;
  *chunk = c;
  return (n + c - 1) / c;
}

template <int TILE, int TPL>
int launch_far_t(pb_ctx* ctx, bool screened, const float4* A, const float4* M, const float4* N, const float4* box,
                 int n, const F32Params& fp, double sig1, double sig2, double* partial, const int* skip) {
  int chunk = 0;
  const int S = far_chunks(ctx, n, kBlock * TPL, TILE, &chunk);
  dim3 grid((unsigned)((n + kBlock * TPL - 1) / (kBlock * TPL)), (unsigned)S);
  if (screened)
    k_p2p_f32<TILE, TPL, true><<<grid, kBlock, 0, ctx->stream>>>(A, M, N, box, n, chunk, fp, sig1, sig2, partial, skip);
  else
    k_p2p_f32<TILE, TPL, false><<<grid, kBlock, 0, ctx->stream>>>(A, M, N, box, n, chunk, fp, sig1, sig2, partial, skip);
  return S;
}

int launch_far(pb_ctx* ctx, int cfg, bool screened, const float4* A, const float4* M, const float4* N,
               const float4* box, int n, const F32Params& fp, double sig1, double sig2, double* partial,
               const int* skip) {
  if (cfg == kSymCfg) {
    const SymShape sh = sym_shape(n, false);
    int n_items = 0;
    const int2* items = sym_items_dev(ctx, n, sh, &n_items);
    if (!items) return -1;
    auto k = sh.F == 512 ? (screened ? k_p2p_f32_sym<true, 4, 1> : k_p2p_f32_sym<false, 4, 1>)
                         : (screened ? k_p2p_f32_sym<true, 2, 2> : k_p2p_f32_sym<false, 2, 2>);
    k<<<(unsigned)n_items, kBlock, 0, ctx->stream>>>(A, N, box, n, sh.nsub, items, n_items, fp, sig1, sig2, partial,
                                                     skip);
    return sh.chunks;
  }
  switch (cfg) {
    case 0: return launch_far_t<256, 1>(ctx, screened, A, M, N, box, n, fp, sig1, sig2, partial, skip);
    case 1: return launch_far_t<512, 1>(ctx, screened, A, M, N, box, n, fp, sig1, sig2, partial, skip);
    case 2: return launch_far_t<256, 2>(ctx, screened, A, M, N, box, n, fp, sig1, sig2, partial, skip);
    default: return launch_far_t<512, 2>(ctx, screened, A, M, N, box, n, fp, sig1, sig2, partial, skip);
  }
}

int far_max_chunks(pb_ctx* ctx, int n) {
  int m = sym_shape(n, false).chunks, c = 0;
  for (int k = 0; k < kNumTiled; ++k)
    m = std::max(m, far_chunks(ctx, n, kBlock * kFarCfgs[k].tpl, kFarCfgs[k].tile, &c));
  return m;
}

}  // namespace

// The far-field kernel of a band of n nodes: symmetric from 12,800 nodes on (16,384 unscreened, whose
// pairs are cheaper), one-directional in tiles of 256 below. At 2924 nodes the two take 28 and 33 µs,
// at 8725 nodes 85 and 65, at 12,056 nodes 158 and 99: the line lies above where the symmetric
// kernel's small tiles overtake, at the size where its tiles of 512 did, since the two group their FP32
// partial sums differently (about 2e-8 of the result) and the operator keeps its values. A fixed
// rule, so that the operator does not depend on timing. PB_FAR_CFG=<index> in the environment fixes the choice instead.
int far_choice(pb_ctx* ctx, int n, bool screened) {
  int cfg = n < (screened ? 12800 : 16384) ? 0 : kSymCfg;
  if (const char* env = std::getenv("PB_FAR_CFG")) {
    const int c = std::atoi(env);
    if (c >= 0 && c < kNumFarCfgs) cfg = c;
  }
  return ctx->far_cfg[n] = cfg;  // kept for pb_far_kernel
}

namespace {

// FP64 operator kernel: 0 = one target per lane over source chunks, 1 = symmetric.
int launch_f64(pb_ctx* ctx, int cfg, const pb_band* band, const double* wpsi, const double* wpsn, const KParams& kp,
               double* partial, const int* skip) {
  const int n = (int)band->n;
  if (cfg == 1) {
    const SymShape sh = sym_shape(n, true);
    int n_items = 0;
    const int2* items = sym_items_dev(ctx, n, sh, &n_items);
    if (!items) return -1;
    auto k = sh.F == 512 ? k_p2p_f64_sym<4, 1> : sh.F == 256 ? k_p2p_f64_sym<2, 2> : k_p2p_f64_sym<1, 2>;
    k<<<(unsigned)n_items, sh.F == 128 ? 128 : 256, 0, ctx->stream>>>(band_dev(band), wpsi, wpsn, n, sh.nsub, items,
                                                                      n_items, kp, kp.kappa * kp.kappa, partial, skip);
    return sh.chunks;
  }
  int chunk = 0;
  const int S = far_chunks(ctx, n, kBlock, kBlock, &chunk);
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  k_p2p_f64<<<dim3(nb, S), kBlock, 0, ctx->stream>>>(band_dev(band, kp.curved), wpsi, wpsn, n, chunk, partial, kp,
                                                                     skip);
  return S;
}

// The FP64 kernel: the symmetric one, which is faster at every size (2924
// nodes: 70 against 91 µs; 45,818 nodes: 2.74 against 6.19 ms), unless PB_F64_CFG=0 asks for the
// one-directional one or the curvature-corrected averages need it.
int f64_choice(bool curved) {
  if (curved) return 0;
  const char* env = std::getenv("PB_F64_CFG");
  return env && !std::strcmp(env, "0") ? 0 : 1;
}

}  // namespace

pb_status matvec_fp64(pb_ctx* ctx, const pb_band* band, const Derived& d, const double* p, double* y) {
  const int n = (int)band->n;
  int chunk = 0;
  const int S64 = std::max(far_chunks(ctx, n, kBlock, kBlock, &chunk), sym_shape(n, true).chunks);
  double* wpsi = (double*)workspace(ctx, "mv_wpsi", sizeof(double) * n);
  double* wpsn = (double*)workspace(ctx, "mv_wpsn", sizeof(double) * n);
  double* partial = (double*)workspace(ctx, "mv_partial64", sizeof(double) * 2 * (size_t)n * S64);
  if (!wpsi || !wpsn || !partial) return PB_ENOMEM;
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  k_weights_f64<<<nb, kBlock, 0, ctx->stream>>>(n, band->w, p, d.h3 / (4.0 * kPi), wpsi, wpsn);
  const KParams kp = kparams(d);
  const int cfg = f64_choice(d.curved);
  int S = 0;
  {
    Scope t(ctx, "p2p_f64");
    S = launch_f64(ctx, cfg, band, wpsi, wpsn, kp, partial, ctx->skip);
  }
  if (S < 0) return ctx->fail(PB_ENOMEM, "FP64 work list");
  {
    Scope t(ctx, "reduce");
    k_reduce<<<(unsigned)((2 * n + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(n, S, partial, nullptr, p, d.lam1,
                                                                                    d.lam2, y);
  }
  return launch_ok(ctx, "matvec_fp64");
}

F32Params f32params(const Derived& d, double sigma) {
  const double rcs = sigma * d.rc;
  return F32Params{(float)d.th1, (float)d.th2, (float)(-1.4426950408889634), (float)(rcs * rcs),
                   (float)(rcs * rcs * 1.001)};
}

pb_status mixed_prepare(pb_ctx* ctx, const pb_band* band, const Derived& d, NearBuild what) {
  PB_TRY(near_build(ctx, band, d, "mx_", ctx->mixed, what));
  const int n = (int)band->n;
  MixedPlan& P = ctx->mixed;
  P.far_cfg = far_choice(ctx, n, d.kappa > 0.0);
  return PB_OK;
}

pb_status matvec_mixed(pb_ctx* ctx, const pb_band* band, const Derived& d, const double* p, double* y) {
  const int n = (int)band->n;
  const MixedPlan& P = ctx->mixed;
  if (P.band_key != band->px || P.n != n || P.rc != d.rc)
    return ctx->fail(PB_EINVAL, "mixed operator used before its geometry was prepared");
  double* partial = (double*)workspace(ctx, "mv_partial", sizeof(double) * 2 * (size_t)n * far_max_chunks(ctx, n));
  double* near = (double*)workspace(ctx, "mx_near", sizeof(double) * 2 * (size_t)n);
  if (!partial || !near) return PB_ENOMEM;
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  k_pack_f32<<<nb, kBlock, 0, ctx->stream>>>(n, band_dev(band), band->w, p, d.h3 / (4.0 * kPi), P.cx, P.cy, P.cz,
                                             P.sigma, P.A, P.M, P.N);
  int S;
  {
    Scope t(ctx, "p2p_f32");
    S = launch_far(ctx, P.far_cfg, d.kappa > 0.0, P.A, P.M, P.N, P.box, n, f32params(d, P.sigma), P.sigma,
                   P.sigma * P.sigma, partial, ctx->skip);
  }
  if (S < 0) return ctx->fail(PB_ENOMEM, "far-field work list");
  {
    Scope t(ctx, "near_f64");
    PB_TRY(near_apply(ctx, band, d, P, p, near));
  }
  {
    Scope t(ctx, "reduce");
    k_reduce<<<(unsigned)((2 * n + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(n, S, partial, near, p, d.lam1,
                                                                                    d.lam2, y);
  }
  return launch_ok(ctx, "matvec_mixed");
}

}  // namespace pb

extern "C" pb_status pb_ibim_matvec(pb_ctx* ctx, const pb_band* band, const pb_params* prm, int precision,
                                    const double* p, double* y) {
  using namespace pb;
  if (!ctx) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  if (!p || !y) return ctx->fail(PB_EINVAL, "pb_ibim_matvec: NULL vector");
  if (p == y) return ctx->fail(PB_EINVAL, "pb_ibim_matvec: p and y must not alias");
  if (precision != PB_FP64 && precision != PB_MIXED && precision != PB_TREE)
    return ctx->fail(PB_EINVAL, "unknown precision %d", precision);
  if (precision != PB_FP64 && prm->reg_metric == PB_REG_TANGENT)
    return ctx->fail(PB_EINVAL, "the mixed path needs a bounded regularization radius (guarded or Euclidean metric)");
  PB_TRY(check_curv(ctx, band, prm));
  PB_HIP(ctx, hipSetDevice(ctx->device));
  Derived d = derive(*prm);
  if (precision == PB_FP64) {
    PB_TRY(matvec_fp64(ctx, band, d, p, y));
  } else if (precision == PB_MIXED) {
    PB_TRY(mixed_prepare(ctx, band, d, NearBuild::once));
    PB_TRY(matvec_mixed(ctx, band, d, p, y));
  } else {
    PB_TRY(tree_prepare(ctx, band, d, prm->tree_degree, prm->tree_theta, ctx->tree, "tc_", nullptr, nullptr,
                        NearBuild::once));
    PB_TRY(matvec_tree(ctx, band, d, p, y, ctx->tree, (int64_t*)ctx->host_pin_dev));
    PB_TRY(sync(ctx, "pb_ibim_matvec"));
    ctx->tree.near.nnz = *(volatile int64_t*)ctx->host_pin;
    return PB_OK;
  }
  return sync(ctx, "pb_ibim_matvec");
}
