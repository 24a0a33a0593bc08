// Right-hand side at the projections and Stage 4 (area and polarization energy).
//
// RHS (eq. IBIM-PBE): g1_i = Σ_k q_k/ε_I G0(x_i*, z_k),
//                     g2_i = Σ_k q_k/ε_I ∂G0(x_i*, z_k)/∂n(x_i*) = −Σ_k q_k (x_i*−z_k)·n_i/(4π ε_I |x_i*−z_k|³).
// Energy (eq. G pol): ψ_rxn(z_k) = h³ Σ_j ω_j [(θ1 ∂Gκ/∂n(y) − ∂G0/∂n(y)) ψ̄_j + (G0 − Gκ) ψ̄n_j]
//   at y = y_j*, with ρ = |z − y|, s = (z − y)·n_j: ∂G0/∂n(y) = s/(4πρ³),
//   ∂Gκ/∂n(y) = e^{−κρ}(1+κρ) s/(4πρ³). G_pol = ½ Σ_k q_k ψ_rxn(z_k); area = h³ Σ_j ω_j.
// All FP64. Reductions are fixed-order block trees (bitwise reproducible).
//
// pb_solvation_energy_noalloc runs the same kernels with no device allocation: ψ_rxn goes to
// the caller's array or to the file-scope `scratch` array below, and the three results to a
// caller-owned device array.
#include <cmath>
#include <mutex>

#include "fp64_math.hpp"
#include "pb_internal.hpp"

// ψ_rxn per atom for pb_solvation_energy_noalloc when the caller passes no array: 1 MiB
// per device, held until the process ends. Host code never names it in a launch or copy;
// it uses the address from hipGetSymbolAddress (pb::scratch_dev below).
constexpr int kNoallocMaxAtoms = 1 << 17;
static __device__ __align__(256) double scratch[kNoallocMaxAtoms];

namespace pb {
namespace {

constexpr int kMaxDevices = 64;
double* scratch_dev[kMaxDevices];  // device address of `scratch` per device ordinal
std::mutex scratch_mu;

// A block takes 64·NW nodes; AW waves share the atoms of each LDS tile out among themselves and add their
// sums up at the end in wave order. Bound by FP64 issue (some 20 instructions and a reciprocal square root a
// pair): by nodes alone the 1343 waves of 85,870 nodes leave SIMDs idle, so eight waves share the
// atoms of 64 nodes (1991 atoms 213 → 153 µs with the call, 500 atoms on 35,214 nodes 46 → 35). Few atoms do not
// pay for that many waves' set-up (rhs_splits).
template <int NW, int AW>
__global__ void __launch_bounds__(64 * NW * AW) k_rhs(int n, const double* __restrict__ px, const double* __restrict__ py,
                                                      const double* __restrict__ pz, const double* __restrict__ nx,
                                                      const double* __restrict__ ny, const double* __restrict__ nz,
                                                      const double* __restrict__ atoms, int n_atoms, double eps_in,
                                                      double* __restrict__ g) {
  static_assert(NW == 1 || AW == 1, "waves share out the nodes or the atoms");
  constexpr int kTile = 64 * NW * AW;
  __shared__ double4 tile[kTile];
  __shared__ double part[2][AW > 1 ? AW : 1][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wa = AW > 1 ? wave : 0;
  const int i = (AW > 1 ? blockIdx.x : blockIdx.x * NW + wave) * 64 + lane, r = min(i, n - 1);
  const double x = px[r], y = py[r], z = pz[r], a = nx[r], b = ny[r], c = nz[r];
  double s1 = 0.0, s2 = 0.0;
  const double c4 = 1.0 / (4.0 * kPi);
  for (int base = 0; base < n_atoms; base += kTile) {
    const int k = base + (int)threadIdx.x, m = min(kTile, n_atoms - base);
    // the charge enters as q/ε_I/(4π), formed once per atom (the same operations, hoisted)
    if (k < n_atoms)
      tile[threadIdx.x] = make_double4(atoms[5 * k], atoms[5 * k + 1], atoms[5 * k + 2], atoms[5 * k + 4] / eps_in * c4);
    __syncthreads();
#pragma unroll 4
    for (int q = wa; q < m; q += AW) {
      const double4 at = tile[q];
      const double dx = x - at.x, dy = y - at.y, dz = z - at.z;
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double rinv = rsqrt_f64(r2);
      const double dn = dx * a + dy * b + dz * c;
      const double t = at.w * rinv;
      s1 += t;
      s2 -= dn * (rinv * rinv) * t;
    }
    __syncthreads();
  }
  if (AW == 1) {
    if (i < n) {
      g[i] = s1;
      g[(int64_t)n + i] = s2;
    }
    return;
  }
  part[0][wa][lane] = s1;
  part[1][wa][lane] = s2;
  __syncthreads();
  if (wave < 2 && i < n) {
    double s = 0.0;
    for (int w = 0; w < AW; ++w) s += part[wave][w][lane];
    g[(int64_t)wave * n + i] = s;
  }
}

constexpr int kPsiBlock = 1024, kPsiHalf = 512;

// The sums of A values over a block of B threads in a fixed order: thread a < A gets that of v[a]. red: A doubles per
// wave, not in use by the block.
template <int B, int A>
__device__ __forceinline__ double block_sums(double (&v)[A], double (&red)[B / 64][A]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the halvings leave lane l with value l & (A − 1) summed over its group of A lanes
#pragma unroll
  for (int len = A / 2; len > 0; len /= 2) {
    const bool up = lane & len;
#pragma unroll
    for (int u = 0; u < len; ++u) v[u] = (up ? v[len + u] : v[u]) + __shfl_xor(up ? v[u] : v[len + u], len);
  }
  double s = v[0];
  for (int off = A; off < 64; off <<= 1) s += __shfl_xor(s, off);
  if (lane < A) red[wave][lane] = s;
  __syncthreads();
  s = 0.0;
  if (wave == 0) {
    for (int w = lane / A; w < B / 64; w += 64 / A) s += red[w][lane & (A - 1)];
    for (int off = A; off < 64; off <<= 1) s += __shfl_xor(s, off);
  }
  return s;
}

// ψ_rxn of A atoms per block: every thread reads the data of each of its nodes once and adds that
// node's term to the sums of all the block's atoms, then one fixed-order block reduction of them all (one per
// atom, of two barriers and a serial sum each, took a fifth of the time of 20,000 atoms on 2924 nodes).
// 1/ρ is rsqrt_f64 and e^{−κρ} exp_neg_f64 (fp64_math.hpp). Per pair, times 4π:
// (s(θ1 E(1 + κρ) − 1)/ρ² · ψ̄_j + (1 − E) · ψ̄n_j)/ρ, with the weight h³ω_j/4π, ψ̄_j's in the normal. Block 0 sums the area
// h³ Σ_j ω_j instead. Bound by FP64 issue (about 40 instructions a
// pair); one block of 512 threads per CU left two waves per SIMD to hide the loads of a node behind, and the area,
// summed afterwards by one block, took 76 µs of its own: 1991 atoms on 85,870 nodes 414 → 306 µs with
// the call.
template <int B, int A>
__global__ void __launch_bounds__(B) k_psi_rxn(int n, const double* __restrict__ px, const double* __restrict__ py,
                                                    const double* __restrict__ pz, const double* __restrict__ nx,
                                                    const double* __restrict__ ny, const double* __restrict__ nz,
                                                    const double* __restrict__ w, const double* __restrict__ p,
                                                    const double* __restrict__ atoms, int n_atoms, double th1,
                                                    double kappa, double h3, double* __restrict__ psi,
                                                    double* __restrict__ area) {
  __shared__ double red[B / 64][A], red1[B / 64][1];
  if (blockIdx.x == 0) {
    double s[1] = {0.0};
#pragma unroll 8
    for (int j = threadIdx.x; j < n; j += B) s[0] += w[j];
    const double t = block_sums<B>(s, red1);
    if (threadIdx.x == 0) *area = h3 * t;
    return;
  }
  const int k0 = (blockIdx.x - 1) * A;
  double za[A][3];
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) za[a][c] = atoms[5 * min(k0 + a, n_atoms - 1) + c];  // a missing atom's sum is not stored
  const double c4 = h3 / (4.0 * kPi);
  double acc[A];
#pragma unroll
  for (int a = 0; a < A; ++a) acc[a] = 0.0;
  for (int j = threadIdx.x; j < n; j += B) {
    const double yx = px[j], yy = py[j], yz = pz[j];
    const double ww = c4 * w[j];
    const double w1 = ww * p[j], w2 = ww * p[n + j];
    const double mx = w1 * nx[j], my = w1 * ny[j], mz = w1 * nz[j];
#pragma unroll
    for (int a = 0; a < A; ++a) {
      const double dx = za[a][0] - yx, dy = za[a][1] - yy, dz = za[a][2] - yz;
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double rinv = rsqrt_f64(r2);
      const double z = kappa * (r2 * rinv);
      const double E = exp_neg_f64(z);
      const double s = dx * mx + dy * my + dz * mz;
      const double t = fma(s * (rinv * rinv), fma(th1, fma(E, z, E), -1.0), fma(-E, w2, w2));
      acc[a] = fma(rinv, t, acc[a]);
    }
  }
  const double s = block_sums<B>(acc, red);
  if (threadIdx.x < A && k0 + (int)threadIdx.x < n_atoms) psi[k0 + threadIdx.x] = s;
}

// The fields of pb_energy in order: out[0] = G_pol = ½ Σ_k q_k ψ_k, out[1] = G_pol in kcal/mol (one
// block, fixed order); out[2], the area, is k_psi_rxn's.
__global__ void __launch_bounds__(kPsiBlock) k_finish(int n_atoms, const double* __restrict__ atoms,
                                                   const double* __restrict__ psi, double* __restrict__ out) {
  __shared__ double red[kPsiBlock / 64][1];
  double a[1] = {0.0};
  for (int k = threadIdx.x; k < n_atoms; k += kPsiBlock) a[0] += atoms[5 * k + 4] * psi[k];
  const double t = block_sums<kPsiBlock>(a, red);
  if (threadIdx.x == 0) {
    const double gpol = 0.5 * t;
    out[0] = gpol;
    out[1] = gpol * 4.0 * kPi * 332.0637;
  }
}

// ψ_rxn at every atom and the energy and area into out (3 doubles, device), on ctx->stream.
void energy_launch(pb_ctx* ctx, const pb_band* band, const double* atoms, int n_atoms, const Derived& d,
                   const double* p, double* psi, double* out) {
  const int n = (int)band->n;
  auto launch = [&](auto kernel, int A, int threads) {
    kernel<<<1 + (n_atoms + A - 1) / A, threads, 0, ctx->stream>>>(n, band->px, band->py, band->pz, band->nx, band->ny,
                                                                     band->nz, band->w, p, atoms, n_atoms, d.th1,
                                                                     d.kappa, d.h3, psi, out + 2);
  };
  // One block of 1024 threads fits a CU at a time; a turn over the nodes costs about its atoms and two thirds (the
  // loads). So the atoms per block that need the least in turns of all CUs: for 1000 atoms 4 (121 µs; 8: 194,
  // 2: 152), for 1991 8 (306; 4: 329), for 5000 4 (1382; 8: 1505), for 500 2 (69; 4: 84, 8: 136).
  int best = 8;
  double cost = INFINITY;
  for (int A = 8; A >= 1; A /= 2) {
    const double c = (double)(((n_atoms + A - 1) / A + ctx->n_cu - 1) / ctx->n_cu) * (A + 2.0 / 3.0);
    if (c < cost) cost = c, best = A;
  }
  // More than a block per CU: half the threads, so that a block's set-up and sums run beside another's pairs. 20,000 atoms
  // on 492, 2924, 13,628 and 105,366 nodes 66, 136, 427 and 2975 µs with the call; 82, 171, 495 and 3374 in blocks of 1024. With
  // a block per CU or fewer the half would leave the CU two waves per SIMD: 1000 atoms on 105,366 nodes 240 and 215.
  const bool half = (n_atoms + best - 1) / best > ctx->n_cu;
  if (best == 8) half ? launch(k_psi_rxn<kPsiHalf, 8>, 8, kPsiHalf) : launch(k_psi_rxn<kPsiBlock, 8>, 8, kPsiBlock);
  else if (best == 4) half ? launch(k_psi_rxn<kPsiHalf, 4>, 4, kPsiHalf) : launch(k_psi_rxn<kPsiBlock, 4>, 4, kPsiBlock);
  else if (best == 2) half ? launch(k_psi_rxn<kPsiHalf, 2>, 2, kPsiHalf) : launch(k_psi_rxn<kPsiBlock, 2>, 2, kPsiBlock);
  else launch(k_psi_rxn<kPsiBlock, 1>, 1, kPsiBlock);
  k_finish<<<1, kPsiBlock, 0, ctx->stream>>>(n_atoms, atoms, psi, out);
}

}  // namespace

pb_status noalloc_init(pb_ctx* ctx) {
  if (ctx->device < 0 || ctx->device >= kMaxDevices)
    return ctx->fail(PB_EDEVICE, "device ordinal %d beyond %d", ctx->device, kMaxDevices);
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (scratch_dev[ctx->device]) return PB_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr)
    return ctx->fail(PB_EDEVICE, "address of the energy scratch array on device %d: %s", ctx->device,
                     hipGetErrorString(e));
  scratch_dev[ctx->device] = (double*)ptr;
  return PB_OK;
}

// Whether eight waves share the atoms of 64 nodes: where the nodes alone give few waves and the atoms are enough to
// share. The two cross at about 8 atoms up to 16,000 nodes, 64 at 105,366 (24.1 µs both with the call), 90 at 169,205 and
// 200 at 371,268 (68.3); one atom on 724,665 nodes takes 37.9 µs split and 22.6 not, 1000 on 105,366 96 and 110.
static bool rhs_splits(int n, int n_atoms) { return n_atoms >= 8 && n_atoms >= n / 2048; }

pb_status rhs(pb_ctx* ctx, const pb_band* band, const double* atoms, int n_atoms, const Derived& d, double* g) {
  const int n = (int)band->n;
  Scope t(ctx, "rhs");
  const int nodes = rhs_splits(n, n_atoms) ? 64 : 256;
  (nodes == 64 ? k_rhs<1, 8> : k_rhs<4, 1>)<<<(unsigned)((n + nodes - 1) / nodes), nodes == 64 ? 512 : 256, 0, ctx->stream>>>(
      n, band->px, band->py, band->pz, band->nx, band->ny, band->nz, atoms, n_atoms, d.eps_in, g);
  return launch_ok(ctx, "rhs");
}

}  // namespace pb

extern "C" pb_status pb_ibim_rhs(pb_ctx* ctx, const pb_band* band, const double* atoms, int n_atoms,
                                 const pb_params* prm, double* g) {
  using namespace pb;
  if (!ctx) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  if (!atoms || n_atoms <= 0 || !g) return ctx->fail(PB_EINVAL, "pb_ibim_rhs: NULL or empty input");
  PB_HIP(ctx, hipSetDevice(ctx->device));
  PB_TRY(rhs(ctx, band, atoms, n_atoms, derive(*prm), g));
  return sync(ctx, "pb_ibim_rhs");
}

extern "C" pb_status pb_solvation_energy(pb_ctx* ctx, const pb_band* band, const double* atoms, int n_atoms,
                                         const pb_params* prm, const double* p, pb_energy* out, double* psi_rxn) {
  using namespace pb;
  if (!ctx) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  if (!atoms || n_atoms <= 0 || !p || !out) return ctx->fail(PB_EINVAL, "pb_solvation_energy: NULL or empty input");
  PB_HIP(ctx, hipSetDevice(ctx->device));
  Derived d = derive(*prm);
  double* psi = psi_rxn ? psi_rxn : (double*)workspace(ctx, "en_psi", sizeof(double) * n_atoms);
  double* res = (double*)workspace(ctx, "en_out", 3 * sizeof(double));
  if (!psi || !res) return PB_ENOMEM;
  {
    Scope t(ctx, "energy");
    energy_launch(ctx, band, atoms, n_atoms, d, p, psi, res);
  }
  PB_TRY(launch_ok(ctx, "energy"));
  double h[3];
  PB_HIP(ctx, hipMemcpyAsync(h, res, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
  PB_TRY(sync(ctx, "pb_solvation_energy"));
  out->g_pol = h[0];
  out->g_pol_kcal = h[1];
  out->area = h[2];
  return PB_OK;
}

extern "C" pb_status pb_solvation_energy_noalloc(pb_ctx* ctx, const pb_band* band, const double* atoms, int n_atoms,
                                                 const pb_params* prm, const double* p, double* out,
                                                 double* psi_rxn) {
  using namespace pb;
  if (!ctx) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  PB_TRY(check_band(ctx, band));
  if (!atoms || n_atoms <= 0 || !p || !out)
    return ctx->fail(PB_EINVAL, "pb_solvation_energy_noalloc: NULL or empty input");
  if (!psi_rxn && n_atoms > kNoallocMaxAtoms)
    return ctx->fail(PB_EINVAL,
                     "pb_solvation_energy_noalloc: %d atoms exceed the scratch array (%d); pass psi_rxn",
                     n_atoms, kNoallocMaxAtoms);
  double* psi = psi_rxn;
  if (!psi) {
    // set at pb_create for this device
    psi = ctx->device >= 0 && ctx->device < kMaxDevices ? scratch_dev[ctx->device] : nullptr;
    if (!psi) return ctx->fail(PB_EDEVICE, "pb_solvation_energy_noalloc: no scratch address for device %d",
                               ctx->device);
  }
  PB_HIP(ctx, hipSetDevice(ctx->device));
  energy_launch(ctx, band, atoms, n_atoms, derive(*prm), p, psi, out);
  return launch_ok(ctx, "pb_solvation_energy_noalloc");
}
