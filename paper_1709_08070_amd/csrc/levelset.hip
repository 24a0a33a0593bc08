// Stage 1: level set of the solvent excluded surface on the Cartesian grid.
//
// vdW union F (eq. vdW-levelset-fn), SAS = F − ρ0, inward eikonal flow φ_t = |∇φ| to
// t = ρ0, cavity removal by flood fill from the grid boundary, and reinitialization
// φ_t + sgn_h(φ0)(|∇φ| − 1) = 0 (eqs. reinit, signum). Time stepping is third-order TVD
// Runge–Kutta; |∇φ| is the Godunov Hamiltonian on fifth-order WENO one-sided derivatives.
//
// Layout: φ is one FP64 array, k fastest. Consecutive threads are consecutive k, so the ±k neighbours
// are coalesced and the ±i/±j neighbours are served from L2. Products and sums are rounded as written (no FMA
// contraction) except in the Godunov Hamiltonian of the stage kernel, where the compiler
// fuses them into FMAs; either way the grid values are the same to the last bit from run
// to run.
#include <algorithm>
#include <cmath>
#include <utility>

#include "fp64_math.hpp"
#include "pb_internal.hpp"
#include "stencil.hpp"

#pragma clang fp contract(off)

namespace pb {
namespace {

constexpr int kBlock = 256;

struct GridDev {
  int nx, ny, nz;
  double ox, oy, oz, h;
};

__device__ __forceinline__ double sq(double a) { return a * a; }

// F(x) − shift, F = min over atoms of |x − z| − r, on tiles of kTI × kTJ × kTK nodes (k fastest inside
// the tile). The tile's nodes lie within R of its centre c, so for every node F ≤ U + R with
// U = min_k(|c − z_k| − r_k), and an atom can attain the minimum at a node of the tile only if
// |c − z_k| ≤ U + 2R + r_k. The block keeps those atoms (with a margin far above the rounding of both
// sides) in LDS and takes the minimum over them, with the same per-atom arithmetic as a scan over all
// atoms, so F is the same to the last bit; a tile that keeps more than kVdwList atoms scans them all.
// TWO: a block takes 2 × 2 × 2 tiles and first filters the atoms once for all of them in the same way
// (the box of 8 × 16 × 16 nodes), so that a tile's filter reads some hundred atoms from LDS instead of
// all; a box that keeps more than kVdwBox atoms filters its tiles from all of them.
// Bound by the reads of the filter: 5000 atoms on 286 × 253 × 217 nodes 1.30 ms in one level, 0.55 ms in
// two.
constexpr int kTI = 4, kTJ = 8, kTK = 8;  // kTI·kTJ·kTK = kBlock
constexpr int kVdwList = 512, kVdwBox = 1024;
static_assert(kTI * kTJ * kTK == kBlock, "one node per thread");

// One atom's candidate for F at x, with the skip of atoms that cannot lower best (their
// distance exceeds best + r by a relative margin far above the rounding of both sides).
__device__ __forceinline__ void vdw_update(double x, double y, double z, const double4& at, double& best) {
  const double d2 = (sq(x - at.x) + sq(y - at.y)) + sq(z - at.z);
  const double lim = best + at.w;
  if (lim > 0.0 && d2 < lim * lim * (1.0 + 1e-12)) {
    const double dist = sqrt(d2) - at.w;
    best = dist < best ? dist : best;
  }
}

// The atoms of src(0..m−1) that can attain F within R of c, appended to list (the first cap of them);
// returns how many there are. Called by the whole block; red and count are its scratch. The minimum's
// exchange is by one wave (kOneWave), which leaves the LDS to the other blocks, or, with one barrier less,
// by each wave: 200³ nodes with 300 atoms 72 and 78 µs in one level, 107 and 104 in two.
template <bool kOneWave, class Src>
__device__ __forceinline__ int vdw_filter(const Src& src, int m, double cx, double cy, double cz, double R, double h,
                                          double4* list, int cap, double* red, int* count) {
  const int t = threadIdx.x;
  double u = INFINITY;
  for (int a = t; a < m; a += kBlock) {
    const double4 q = src(a);
    const double dc = sqrt((sq(cx - q.x) + sq(cy - q.y)) + sq(cz - q.z)) - q.w;
    u = dc < u ? dc : u;
  }
  if (t == 0) *count = 0;
  if (kOneWave) {
    red[t] = u;
    __syncthreads();
    if (t < 64) {
      for (int w = 1; w < kBlock / 64; ++w) u = fmin(u, red[t + 64 * w]);
      for (int off = 32; off > 0; off >>= 1) u = fmin(u, __shfl_xor(u, off));
      if (t == 0) red[0] = u;
    }
    __syncthreads();
    u = red[0];
  } else {
    for (int off = 32; off > 0; off >>= 1) u = fmin(u, __shfl_xor(u, off));
    if ((t & 63) == 0) red[t >> 6] = u;
    __syncthreads();
    for (int w = 0; w < kBlock / 64; ++w) u = fmin(u, red[w]);
  }
  const double reach = u + 2.0 * R;  // an atom matters only within reach + r of c
  for (int a = t; a < m; a += kBlock) {
    const double4 q = src(a);
    const double lim = (reach + q.w) * (1.0 + 1e-9) + 1e-9 * (1.0 + h);
    if (lim > 0.0 && (sq(cx - q.x) + sq(cy - q.y)) + sq(cz - q.z) <= lim * lim) {
      const int p = atomicAdd(count, 1);
      if (p < cap) list[p] = q;
    }
  }
  __syncthreads();
  const int kept = *count;
  __syncthreads();  // red, count and a source in LDS may be written again
  return kept;
}

template <bool TWO>
__global__ void __launch_bounds__(kBlock) k_vdw(GridDev g, const double* __restrict__ atoms, int n_atoms,
                                                double shift, double* __restrict__ phi) {
  __shared__ double4 box[TWO ? kVdwBox : 1], list[kVdwList];
  __shared__ double red[TWO ? kBlock / 64 : kBlock];
  __shared__ int count;
  constexpr int T = TWO ? 2 : 1;  // tiles per axis
  const int nbk = (g.nz + T * kTK - 1) / (T * kTK), nbj = (g.ny + T * kTJ - 1) / (T * kTJ);
  const int bk = blockIdx.x % nbk, bj = (blockIdx.x / nbk) % nbj, bi = blockIdx.x / (nbk * nbj);
  auto global = [&](int a) { return make_double4(atoms[5 * a], atoms[5 * a + 1], atoms[5 * a + 2], atoms[5 * a + 3]); };
  auto local = [&](int a) { return box[a]; };
  // centre and radius of a box of ni × nj × nk nodes whose first node is (i0, j0, k0)
  auto centre = [&](double o, int i0, int ni) { return o + g.h * (i0 + 0.5 * (ni - 1)); };
  auto radius = [&](int ni, int nj, int nk) {
    return g.h * 0.5 * sqrt((double)((ni - 1) * (ni - 1) + (nj - 1) * (nj - 1) + (nk - 1) * (nk - 1)));
  };
  int mb = kVdwBox + 1;
  if (TWO)
    mb = vdw_filter<false>(global, n_atoms, centre(g.ox, bi * T * kTI, T * kTI), centre(g.oy, bj * T * kTJ, T * kTJ),
                    centre(g.oz, bk * T * kTK, T * kTK), radius(T * kTI, T * kTJ, T * kTK), g.h, box, kVdwBox, red,
                    &count);
  const int t = threadIdx.x;
  for (int sub = 0; sub < T * T * T; ++sub) {
    const int i0 = (bi * T + (sub >> 2)) * kTI, j0 = (bj * T + ((sub >> 1) & 1)) * kTJ, k0 = (bk * T + (sub & 1)) * kTK;
    if (i0 >= g.nx || j0 >= g.ny || k0 >= g.nz) continue;  // the whole block
    const double cx = centre(g.ox, i0, kTI), cy = centre(g.oy, j0, kTJ), cz = centre(g.oz, k0, kTK),
                 R = radius(kTI, kTJ, kTK);
    const int m = TWO && mb <= kVdwBox
                      ? vdw_filter<!TWO>(local, mb, cx, cy, cz, R, g.h, list, kVdwList, red, &count)
                      : vdw_filter<!TWO>(global, n_atoms, cx, cy, cz, R, g.h, list, kVdwList, red, &count);
    const int i = i0 + t / (kTJ * kTK), j = j0 + (t / kTK) % kTJ, k = k0 + t % kTK;
    const double x = g.ox + g.h * (double)i, y = g.oy + g.h * (double)j, z = g.oz + g.h * (double)k;
    double best = INFINITY;
    if (m <= kVdwList) {
      for (int q = 0; q < m; ++q) vdw_update(x, y, z, list[q], best);
    } else {
      for (int a = 0; a < n_atoms; ++a) vdw_update(x, y, z, global(a), best);
    }
    if (i < g.nx && j < g.ny && k < g.nz) phi[((int64_t)i * g.ny + j) * g.nz + k] = best - shift;
    __syncthreads();  // the list is rewritten by the next tile
  }
}

// One side of an axis: the WENO5 one-sided derivative, times 6h, as a quotient n/d with d > 0.
struct Frac {
  double n, d;
};

// v: the middle difference of the side's five; c1..c3: its candidates minus 6v; b = ε + β of the
// three candidates. Weights 1/b₁² : 6/b₂² : 3/b₃², over their common denominator.
__device__ __forceinline__ Frac weno_side(double v, double c1, double c2, double c3, double b1, double b2, double b3) {
#pragma clang fp contract(fast)
  const double q1 = 3.0 * sq(b1), q2 = sq(b2), q3 = sq(b3), d3 = q3 + q3, A = q2 * q3;
  const double D = fma(q1, q2 + d3, A);
  const double N = fma(q1, fma(c2, d3, c3 * q2), c1 * A);
  return {fma(6.0 * v, D, N), D};
}

// n/d for d > 0 (not subnormal): the hardware reciprocal (2^-24 or better) and one Newton step (2^-47),
// then one correction of the quotient, whose own error is the square of that.
__device__ __forceinline__ double div_pos(double n, double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  const double q = n * r;
  return fma(fma(-d, q, n), r, q);
}

// One axis of the Godunov Hamiltonian sg·|∇φ| (sg = ±1) from the seven values f[0..6] centred
// on the node: the WENO5 one-sided derivatives a (differences d0..d4) and b (d5..d1), then
// max((a⁺)², (b⁻)²) for sg > 0 and max((a⁻)², (b⁺)²) for sg < 0. It works on the differences
// d = h·D instead of the divided differences D and on their differences e: the smoothness indicators
// are taken ×4h² (13t²/3 + u², ε entering as e4 = 4h²ε, the same weights) and the candidates ×6h, the
// middle difference split off (a = 6d2 + a convex combination of c1..c3), so that what is added to acc is
// (6h)² times the axis's term; the larger of the two quotients is chosen by cross multiplication
// (their denominators are positive), one division instead of two.
__device__ __forceinline__ double godunov_axis(const double f[7], double e4, double sg, double acc) {
#pragma clang fp contract(fast)
  const double d0 = f[1] - f[0], d1 = f[2] - f[1], d2 = f[3] - f[2], d3 = f[4] - f[3], d4 = f[5] - f[4],
               d5 = f[6] - f[5];
  const double e0 = d1 - d0, e1 = d2 - d1, e2 = d3 - d2, e3 = d4 - d3, e_4 = d5 - d4;
  const double g = 13.0 / 3.0;
  const double t1 = e2 - e1, t2 = e3 - e2;
  const double s1 = fma(g * t1, t1, e4), s2 = fma(g * t2, t2, e4);
  const double t0 = e1 - e0, s0 = fma(g * t0, t0, e4), t3 = e_4 - e3, s3 = fma(g * t3, t3, e4);
  const double ua1 = 3.0 * e1 - e0, ua2 = e1 + e2, ua3 = e3 - 3.0 * e2;
  const double ub1 = 3.0 * e3 - e_4, ub2 = e2 + e3, ub3 = e1 - 3.0 * e2;
  // the candidates from the same differences as the indicators: 5e1 − 2e0, e1 + 2e2, 4e2 − e3 and mirrored
  const Frac a = weno_side(d2, 2.0 * ua1 - e1, ua2 + e2, e2 - ua3, fma(ua1, ua1, s0), fma(ua2, ua2, s1),
                           fma(ua3, ua3, s2));
  const Frac b = weno_side(d3, e3 - 2.0 * ub1, -e2 - ub2, ub3 - e2, fma(ub1, ub1, s3), fma(ub2, ub2, s2),
                           fma(ub3, ub3, s1));
  const double A = fmax(sg * a.n, 0.0), B = fmax(-sg * b.n, 0.0);
  const bool left = A * b.d >= B * a.d;
  const double x = div_pos(left ? A : B, left ? a.d : b.d);
  return fma(x, x, acc);
}

// One TVD-RK3 stage: L = L(φ_in), then
//   stage 0: out = φ_in + dt·L
//   stage 1: out = 0.75 φ_n + 0.25 (φ_in + dt·L)
//   stage 2: out = φ_n / 3 + (2/3)(φ_in + dt·L)
// MODE 0: eikonal flow (L = |∇φ| with Hamiltonian −|∇φ|); MODE 1: reinit (L = −S(|∇φ| − 1)).
// |∇φ| is the Godunov Hamiltonian with zero-Neumann ghosts (even reflection about the boundary
// node, −m ↦ m and n−1+m ↦ n−1−m). stage_value finishes a node from the sum of its axes' terms.
template <int MODE>
__device__ __forceinline__ double stage_value(double acc, double c, double s, double phi, double dt, double phi_n,
                                              int stage) {
  // √acc from the reciprocal square root with one correction; acc = 0 where φ is flat
  const double rs = rsqrt_f64(acc), r0 = acc * rs;
  const double G = acc > 0.0 ? fma(fma(-r0, r0, acc), 0.5 * rs, r0) * c : acc * c;
  const double L = MODE == 0 ? G : -s * (G - 1.0);
  const double v0 = phi + dt * L;
  return stage == 0 ? v0 : stage == 1 ? 0.75 * phi_n + 0.25 * v0 : phi_n * (1.0 / 3.0) + (2.0 / 3.0) * v0;
}

// The node that position q (−3 … n + 2) stands for.
__device__ __forceinline__ int reflect(int q, int n) { return min(abs(q), 2 * (n - 1) - abs(q)); }

constexpr int kXcds = 8;

// t / d for t < 2^32 from m = ⌈2^64 / d⌉ (d ≥ 2): m·d exceeds 2^64 by less than d < 2^32, so the product
// with t is right to the last bit of its high word.
struct Div {
  uint32_t hi, lo;
};
inline Div div_by(uint64_t d) {
  const uint64_t m = ~0ull / d + 1;
  return {(uint32_t)(m >> 32), (uint32_t)m};
}
__device__ __forceinline__ unsigned div_u32(unsigned t, Div m) {
  return (unsigned)(((uint64_t)t * m.hi + __umulhi(t, m.lo)) >> 32);
}

// The stage with one thread per node: e = 4h²ε and c = 1/(6h) undo the scaling of godunov_axis. 32-bit
// node indexing (grids hold fewer than 2^31 nodes). The XCDs take slabs of ny/8 rows, so that the
// planes of a node's x neighbours lie in the L2 of its own XCD; on grids of less than 32 rows (kRows = false),
// where one XCD would have up to twice the rows of another, slabs of an eighth of the (y, z) columns instead
// (300 × 9 × 300 nodes 3.23 ms by rows, 2.21 by columns; from 32 rows on either is ahead, by up to 3 or 10%
// as the shape has it).
// Small grids wait on launches (an empty one takes 4 µs, a stage here under 6) and on one chain of index
// arithmetic, loads and FP64 work (two waves per SIMD at 135,000 nodes): no divisions, no branch that a wave
// takes both ways, 250 FP64 instructions a node. Level set of 54 × 51 × 49 nodes (150 stages; cavities
// included) 1270 → 900 µs, of 85 × 79 × 70 2.11 → 1.56 ms, of 117 × 106 × 93 3.9 → 2.9 ms.
template <int MODE, bool kRows>
__global__ void __launch_bounds__(kBlock) k_rk_node(GridDev g, const double* __restrict__ phi_in,
                                                    const double* __restrict__ phi_n, const double* __restrict__ S,
                                                    double* __restrict__ out, int stage, double dt, double e,
                                                    double c, Div by_less, Div by_more, Div by_nz) {
  const unsigned xcd = blockIdx.x % kXcds, t = blockIdx.x / kXcds * kBlock + threadIdx.x;
  int i, j, k;
  unsigned uid;
  if (kRows) {
    const unsigned j0 = (unsigned)g.ny * xcd / kXcds, j1 = (unsigned)g.ny * (xcd + 1) / kXcds;
    const unsigned slab = (j1 - j0) * (unsigned)g.nz;
    if (t >= slab * (unsigned)g.nx) return;
    i = (int)div_u32(t, j1 - j0 == (unsigned)g.ny / kXcds ? by_less : by_more);
    const int r = (int)(t - i * slab), row = (int)div_u32((unsigned)r, by_nz);
    j = (int)j0 + row;
    k = r - row * g.nz;
    uid = ((unsigned)i * g.ny + j) * g.nz + k;
  } else {
    const unsigned plane = (unsigned)g.ny * g.nz, c0 = plane * xcd / kXcds, slab = plane * (xcd + 1) / kXcds - c0;
    if (t >= slab * (unsigned)g.nx) return;
    i = (int)div_u32(t, slab == plane / kXcds ? by_less : by_more);
    const unsigned col = c0 + (t - i * slab);
    j = (int)div_u32(col, by_nz);
    k = (int)col - j * g.nz;
    uid = i * plane + col;
  }
  const double* __restrict__ p = phi_in + uid;
  const double s = MODE == 1 ? S[uid] : -1.0;
  const double sg = s >= 0.0 ? 1.0 : -1.0;
  // all values before any arithmetic; ghosts by index in z and y, where a wave mostly has some, by branch
  // in x, where it has them as a whole
  double f[3][7];
#pragma unroll
  for (int m = 0; m < 7; ++m) {
    f[2][m] = p[reflect(k + m - 3, g.nz) - k];
    if (m != 3) f[1][m] = p[(reflect(j + m - 3, g.ny) - j) * g.nz];
  }
  f[1][3] = f[2][3];
  const int plane_x = g.ny * g.nz;
  if ((unsigned)(i - 3) <= (unsigned)(g.nx - 7)) {
#pragma unroll
    for (int m = 0; m < 7; ++m) f[0][m] = p[(m - 3) * plane_x];
  } else {
#pragma unroll
    for (int m = 0; m < 7; ++m) f[0][m] = p[(reflect(i + m - 3, g.nx) - i) * plane_x];
  }
  double acc = 0.0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) acc = godunov_axis(f[ax], e, sg, acc);
  out[uid] = stage_value<MODE>(acc, c, s, f[2][3], dt, stage > 0 ? phi_n[uid] : 0.0, stage);
}

// The stage on large grids (stage_marches): a thread takes two nodes consecutive in k (16-byte loads, 8-byte aligned
// only: rows may be odd) and marches len nodes in i with the seven x values of both in registers, a
// block a tile of 32 (k) × 16 (j) columns: 11 loads for two nodes and a step instead of 38, and the
// loads from far away (next x plane, S, φ_n) are issued a step ahead. Tiles go to the XCDs in
// contiguous runs along j.
// With one thread per node the L1 serves 19 values a node, 72% of the kernel's cycles beside 65%
// VALU; here it is bound by FP64 issue and the reads of φ, φ_n and S (at 15.7M nodes 250 FP64
// instructions a node, 145 µs, and 0.6 GB, 125 µs; a stage takes 185). Level set of 286 × 253 × 217 nodes:
// 53 ms before, 40.8 ms with k_rk_node, 33.9 ms with this kernel; 208 × 185 × 159: 18.4, 14.3, 12.2 ms.
constexpr int kStageK = 32, kStageJ = 2 * kBlock / kStageK;

struct D2 {
  double v[2];
};
__device__ __forceinline__ D2 load2(const double* p) {
  typedef double vec __attribute__((ext_vector_type(2), aligned(8)));
  return __builtin_bit_cast(D2, *reinterpret_cast<const vec*>(p));
}

template <int MODE>
__global__ void __launch_bounds__(kBlock) k_rk_march(GridDev g, const double* __restrict__ phi_in,
                                                     const double* __restrict__ phi_n, const double* __restrict__ S,
                                                     double* __restrict__ out, int stage, double dt, double e,
                                                     double c, int len, int nkt, int nic, int nb) {
  const int per = gridDim.x / kXcds, id = (int)(blockIdx.x % kXcds) * per + (int)(blockIdx.x / kXcds);
  if (id >= nb) return;
  constexpr int KT = kStageK / 2;  // threads along k
  const int kt = id % nkt, ic = id / nkt % nic, jt = id / (nkt * nic);
  const int j = jt * kStageJ + (int)threadIdx.x / KT, k0 = kt * kStageK + 2 * ((int)threadIdx.x % KT);
  const int jc = min(j, g.ny - 1), kk = min(k0, g.nz - 2);  // nodes kk and kk + 1; beyond the grid: not stored
  const bool live = j < g.ny && k0 < g.nz;
  const int plane = g.ny * g.nz, col = jc * g.nz + kk;
  int yo[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) yo[m] = (reflect(jc + (m < 3 ? m - 3 : m - 2), g.ny) - jc) * g.nz;
  const bool kin = kk >= 3 && kk + 4 < g.nz;
  const int i0 = ic * len, i1 = min(g.nx, i0 + len);
  D2 w[7];
#pragma unroll
  for (int m = 0; m < 7; ++m) w[m] = load2(phi_in + (int64_t)reflect(i0 + m - 3, g.nx) * plane + col);
  D2 s_next{}, pn_next{};
  if (MODE == 1) s_next = load2(S + (int64_t)i0 * plane + col);
  if (stage > 0) pn_next = load2(phi_n + (int64_t)i0 * plane + col);
#pragma unroll 2
  for (int i = i0; i < i1; ++i) {
    const int64_t uid = (int64_t)i * plane + col;
    const double* __restrict__ p = phi_in + uid;
    D2 y[6];
    const D2 s = s_next, pn = pn_next;
    double z[8];
#pragma unroll
    for (int m = 0; m < 6; ++m) y[m] = load2(p + yo[m]);
    if (kin) {
      const D2 l = load2(p - 3), h = load2(p + 2);
      z[0] = l.v[0], z[1] = l.v[1], z[2] = p[-1], z[5] = h.v[0], z[6] = h.v[1], z[7] = p[4];
    } else {
#pragma unroll
      for (int m = 0; m < 8; ++m) z[m] = p[reflect(kk + m - 3, g.nz) - kk];
    }
    z[3] = w[3].v[0], z[4] = w[3].v[1];
    D2 w7{};
    if (i + 1 < i1) {
      if (MODE == 1) s_next = load2(S + uid + plane);
      if (stage > 0) pn_next = load2(phi_n + uid + plane);
      w7 = load2(phi_in + (int64_t)reflect(i + 4, g.nx) * plane + col);
    }
    double v[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const double su = MODE == 1 ? s.v[u] : -1.0, sg = su >= 0.0 ? 1.0 : -1.0;
      double f[7];
#pragma unroll
      for (int m = 0; m < 7; ++m) f[m] = w[m].v[u];
      double acc = godunov_axis(f, e, sg, 0.0);
#pragma unroll
      for (int m = 0; m < 3; ++m) f[m] = y[m].v[u], f[4 + m] = y[3 + m].v[u];
      f[3] = w[3].v[u];
      acc = godunov_axis(f, e, sg, acc);
#pragma unroll
      for (int m = 0; m < 7; ++m) f[m] = z[m + u];
      acc = godunov_axis(f, e, sg, acc);
      v[u] = stage_value<MODE>(acc, c, su, w[3].v[u], dt, pn.v[u], stage);
    }
    if (live) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (kk + u >= k0) out[uid + u] = v[u];
    }
#pragma unroll
    for (int m = 0; m < 6; ++m) w[m] = w[m + 1];
    w[6] = w7;
  }
}

// Whether a grid marches, and how far a thread then goes.
// Marching pays once it has some 1300 blocks; below that too few waves are in flight: 161 × 145 × 127
// nodes (2.97M) 6.95 ms marching, 7.15 ms by nodes; 137 × 120 × 103 (1.69M) 5.00 and 4.18 ms. And its tiles of columns
// have to be filled, 85% of them: 140 × 140 × 140 (2.7M, 85%) 6.24 ms marching, 6.12 by nodes; 180 × 170 × 90 (91%)
// 5.67 and 6.13; 300 × 200 × 103 (6.2M, 77%) 13.9 and 13.0; 340 × 330 × 140 (15.7M, 86%) 31.8 and 34.9. On flat grids most
// lanes would idle: 620 × 610 × 7 (21%) 18.9 and 5.8 ms, 300 × 260 × 34 (51%) 8.6 and 5.8. A longer
// march loads the seven starting planes less often but needs a larger grid for as many blocks: 4, 8 and 16
// nodes take 12.4, 12.8, 13.6 ms at 6.1M nodes and 35.5, 34.2, 33.7 ms at 15.7M.
bool stage_marches(const GridDev& g) {
  const int64_t cols = (int64_t)g.ny * g.nz, tiles = (int64_t)((g.ny + kStageJ - 1) / kStageJ) * ((g.nz + kStageK - 1) / kStageK);
  return cols * g.nx >= (int64_t)5 << 19 && 100 * cols >= 85 * tiles * (kStageJ * kStageK);
}
int march_len(int64_t total) { return (int)std::min<int64_t>(std::max<int64_t>(total >> 20, 4), 16); }

__global__ void __launch_bounds__(kBlock) k_sign(int64_t total, const double* __restrict__ phi, double h,
                                                 double* __restrict__ S) {
  int64_t id = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (id < total) S[id] = phi[id] / sqrt(phi[id] * phi[id] + h * h);
}

// ---- cavity removal
//
// On bit masks: word w of the row (i, j) holds its nodes k = 64w … 64w + 63 (nw words a row). P marks
// φ > 0, O the exterior found so far, P's nodes on the boundary of the grid at first. A sweep along an
// axis joins to O every P-node that is reachable through P along its line from an O-node or from a
// P-node with an O-neighbour across the line. Bits only go 0 → 1 and a word is written by one thread of a
// sweep, so reads of neighbours that other lines are updating are harmless; repeated sweeps over the
// three axes reach the unique fixed point, the 6-connected component of {φ > 0} that touches the grid
// boundary. A flood with one wave per grid line on φ itself and a
// search of every unreached node's ball took 0.94 and 1.70 ms on 286 × 253 × 217 nodes; this takes 0.11 ms,
// of which 49 µs read φ.

// One wave per word.
__global__ void __launch_bounds__(kBlock) k_cav_masks(GridDev g, int nw, int words, const double* __restrict__ phi,
                                                      uint64_t* __restrict__ P, uint64_t* __restrict__ O) {
  const int word = (int)(blockIdx.x * (kBlock / 64) + threadIdx.x / 64), lane = threadIdx.x & 63;
  if (word >= words) return;
  const int row = word / nw, w = word - row * nw, i = row / g.ny, j = row - i * g.ny, k = 64 * w + lane;
  const bool pos = k < g.nz && phi[(int64_t)row * g.nz + k] > 0.0;
  const bool edge = i == 0 || j == 0 || k == 0 || i == g.nx - 1 || j == g.ny - 1 || k == g.nz - 1;
  const uint64_t p = __ballot(pos), o = __ballot(pos && edge);
  if (lane == 0) {
    P[word] = p;
    O[word] = o;
  }
}

// Bits t of F (< 64) that some seed s ≤ t (reach_up) or s ≥ t (reach_down) reaches through set bits of
// P: a doubling scan (Kogge–Stone; bits shifted in are 0).
__device__ __forceinline__ uint64_t reach_up(uint64_t S, uint64_t P) {
  uint64_t F = S, A = P;
  for (int d = 1; d < 64; d <<= 1) {
    F |= (F << d) & A;
    A &= A << d;
  }
  return F;
}
__device__ __forceinline__ uint64_t reach_down(uint64_t S, uint64_t P) {
  uint64_t F = S, A = P;
  for (int d = 1; d < 64; d <<= 1) {
    F |= (F >> d) & A;
    A &= A >> d;
  }
  return F;
}

// Sweep along z, one thread per row: up its words with the carry of the last node, then down.
__global__ void __launch_bounds__(64) k_cav_z(GridDev g, int nw, const uint64_t* __restrict__ P, uint64_t* O,
                                              int* changed) {
  const int row = (int)(blockIdx.x * 64 + threadIdx.x);
  if (row >= g.nx * g.ny) return;
  const int i = row / g.ny, j = row - i * g.ny;
  const int64_t at = (int64_t)row * nw, plane = (int64_t)g.ny * nw;
  bool any = false;
  uint64_t carry = 0;
  for (int w = 0; w < nw; ++w) {
    const uint64_t p = P[at + w], o = O[at + w];
    uint64_t s = o | carry;
    if (i > 0) s |= O[at + w - plane];
    if (i < g.nx - 1) s |= O[at + w + plane];
    if (j > 0) s |= O[at + w - nw];
    if (j < g.ny - 1) s |= O[at + w + nw];
    const uint64_t f = reach_up(s & p, p);
    carry = f >> 63;
    if (f != o) O[at + w] = f, any = true;
  }
  carry = 0;
  for (int w = nw - 1; w >= 0; --w) {
    const uint64_t p = P[at + w], o = O[at + w], f = reach_down((o | carry << 63) & p, p);
    carry = f & 1;
    if (f != o) O[at + w] = f, any = true;
  }
  if (any) *changed = 1;
}

// Sweep along x or y, one wave per line of words (n of them, `step` apart) and 64 of its words at a time,
// one per lane, first up, then down, the carry between chunks held by every lane. Lines: n2 × nw, `step2`
// apart in the first index, and one word in the second; across the line are the words step2 away and, in z,
// the neighbouring bits.
__global__ void __launch_bounds__(kBlock) k_cav_xy(int nw, int n, int64_t step, int n2, int64_t step2,
                                                   const uint64_t* __restrict__ P, uint64_t* O, int* changed) {
  const int line = (int)(blockIdx.x * (kBlock / 64) + threadIdx.x / 64), lane = threadIdx.x & 63;
  if (line >= n2 * nw) return;  // the whole wave
  const int l2 = line / nw, w = line - l2 * nw, chunks = (n + 63) / 64;
  const int64_t at0 = l2 * step2 + w;
  bool any = false;
  uint64_t carry = 0;
  for (int ch = 0; ch < chunks; ++ch) {
    const int q = ch * 64 + lane;
    const int64_t at = at0 + q * step;
    uint64_t p = 0, o = 0, s = 0;
    if (q < n) {
      p = P[at];
      o = O[at];
      s = o | o << 1 | o >> 1;
      if (w > 0) s |= O[at - 1] >> 63;
      if (w < nw - 1) s |= O[at + 1] << 63;
      if (l2 > 0) s |= O[at - step2];
      if (l2 < n2 - 1) s |= O[at + step2];
    }
    uint64_t f = (lane == 0 ? s | carry : s) & p, a = p;
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t fu = __shfl_up(f, d), au = __shfl_up(a, d);
      if (lane >= d) f |= fu & a, a &= au;
    }
    carry = __shfl(f, 63);
    if (f != o) O[at] = f, any = true;
  }
  carry = 0;
  for (int ch = chunks - 1; ch >= 0; --ch) {
    const int q = ch * 64 + lane;
    const int64_t at = at0 + q * step;
    uint64_t p = 0, o = 0;
    if (q < n) p = P[at], o = O[at];
    uint64_t f = (lane == 63 ? o | carry : o) & p, a = p;
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t fd = __shfl_down(f, d), ad = __shfl_down(a, d);
      if (lane + d < 64) f |= fd & a, a &= ad;
    }
    carry = __shfl(f, 0);
    if (f != o) O[at] = f, any = true;
  }
  if (any) *changed = 1;
}

// Cavity nodes (unreached, φ > 0) get −ε; those with a neighbour along an axis that is none go into the
// list, in any order. The balls of the listed ones cover what the balls of all would: a path from a
// cavity node to any node of its ball by steps that come closer leaves the cavity at a listed node.
__global__ void __launch_bounds__(kBlock) k_cav_list(GridDev g, int nw, int words, const uint64_t* __restrict__ P,
                                                     const uint64_t* __restrict__ O, double eps,
                                                     double* __restrict__ phi, unsigned* __restrict__ list, int* count) {
  const int word = (int)(blockIdx.x * kBlock + threadIdx.x);
  if (word >= words) return;
  auto cavity = [&](int q) { return P[q] & ~O[q]; };
  const uint64_t c = cavity(word);
  if (!c) return;
  const int row = word / nw, w = word - row * nw, i = row / g.ny, j = row - i * g.ny, plane = g.ny * nw;
  uint64_t in = (c << 1 | (w > 0 ? cavity(word - 1) >> 63 : 1)) & (c >> 1 | (w < nw - 1 ? cavity(word + 1) << 63 : 0));
  if (i > 0) in &= cavity(word - plane);
  if (i < g.nx - 1) in &= cavity(word + plane);
  if (j > 0) in &= cavity(word - nw);
  if (j < g.ny - 1) in &= cavity(word + nw);
  const unsigned first = (unsigned)row * (unsigned)g.nz + 64u * (unsigned)w;
  uint64_t out = c & ~in;
  unsigned at = out ? (unsigned)atomicAdd(count, __popcll(out)) : 0;
  for (uint64_t q = c; q; q &= q - 1) {
    const unsigned id = first + (unsigned)(__ffsll((long long)q) - 1);
    phi[id] = -eps;
    if (out & q & -q) list[at++] = id;
  }
}

// Unreached nodes within (ε + h) of a listed node get −ε: a block per node and turn, over the ball
// around it (rr2: its squared radius in nodes, m: the whole of its radius).
__global__ void __launch_bounds__(kBlock) k_cav_fill(GridDev g, int nw, const uint64_t* __restrict__ O,
                                                     const unsigned* __restrict__ list, const int* __restrict__ count,
                                                     double eps, int m, double rr2, double* __restrict__ phi) {
  const int n = *count, side = 2 * m + 1;
  for (int q = blockIdx.x; q < n; q += gridDim.x) {
    const unsigned id = list[q];
    const int k0 = (int)(id % (unsigned)g.nz), j0 = (int)(id / (unsigned)g.nz % (unsigned)g.ny),
              i0 = (int)(id / ((unsigned)g.nz * (unsigned)g.ny));
    for (int64_t t = threadIdx.x; t < (int64_t)side * side * side; t += kBlock) {
      const int a = (int)(t / ((int64_t)side * side)) - m, b = (int)(t / side % side) - m, c = (int)(t % side) - m;
      if ((double)a * a + (double)b * b + (double)c * c > rr2) continue;
      const int i = i0 + a, j = j0 + b, k = k0 + c;
      if (i < 0 || j < 0 || k < 0 || i >= g.nx || j >= g.ny || k >= g.nz) continue;
      const int64_t row = (int64_t)i * g.ny + j;
      if (!(O[row * nw + k / 64] >> (k & 63) & 1)) phi[row * g.nz + k] = -eps;
    }
  }
}

constexpr int kMaxAxis = 4096;

unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Whether k_vdw filters in two levels. The box's eight tiles follow one another in a block, which
// pays when there are boxes enough and when a scan of the atoms costs more than a tile's own work, the
// sooner the more boxes there are (µs, one level against two): 4.25M nodes 66 and 89 with 513 atoms, 135 and
// 143 with 1400, 179 and 160 with 2000; 8M nodes 111 and 132 with 700 atoms, 144 and 146 with 1000, 205 and 181 with
// 1400; 5000 atoms on 286 × 253 × 217 nodes 1300 and 550, 2000 atoms on 161 × 145 × 127 nodes (2.97M) 145 and 167.
bool vdw_two_levels(int64_t total, int n_atoms) {
  return total >= (int64_t)1 << 22 && n_atoms > (total >= (int64_t)1 << 23 ? 4 : 6) * kBlock;
}

// Three-stage TVD-RK3 for `steps` steps of size dt on φ in cur. A step's result goes to the buffer its
// first stage used, which then holds φ: the two swap every step.
pb_status tvd_rk3(pb_ctx* ctx, const GridDev& g, double*& cur, double*& spare, double* p2, const double* S, int mode,
                  int steps, double dt) {
  const int64_t plane = (int64_t)g.ny * g.nz, total = plane * g.nx;
  const double e = 4.0 * g.h * g.h * kWenoEps, c = 1.0 / (6.0 * g.h);
  const bool march = stage_marches(g);
  const bool rows = g.ny >= 32;
  const int64_t unit = rows ? g.nz : 1;  // what k_rk_node deals out to the XCDs: rows or columns, at least four each
  const int len = march_len(total), nkt = (g.nz + kStageK - 1) / kStageK, njt = (g.ny + kStageJ - 1) / kStageJ,
            nic = (g.nx + len - 1) / len, nb = nkt * njt * nic;
  const unsigned blocks = kXcds * (march ? (unsigned)((nb + kXcds - 1) / kXcds)
                                         : blocks_for((plane / unit + kXcds - 1) / kXcds * unit * g.nx));
  const int64_t own = plane / unit / kXcds;  // an XCD's units, or one more
  const Div by_less = div_by(own * unit), by_more = div_by((own + 1) * unit), by_nz = div_by(g.nz);
  auto stage = [&](const double* in, const double* phi_n, double* out, int st) {
    if (march)
      (mode == 0 ? k_rk_march<0> : k_rk_march<1>)<<<blocks, kBlock, 0, ctx->stream>>>(g, in, phi_n, S, out, st, dt, e,
                                                                                     c, len, nkt, nic, nb);
    else
      (rows ? mode == 0 ? k_rk_node<0, true> : k_rk_node<1, true>
            : mode == 0 ? k_rk_node<0, false> : k_rk_node<1, false>)<<<blocks, kBlock, 0, ctx->stream>>>(
          g, in, phi_n, S, out, st, dt, e, c, by_less, by_more, by_nz);
  };
  for (int s = 0; s < steps; ++s) {
    Scope t(ctx, "levelset");
    stage(cur, cur, spare, 0);
    stage(spare, cur, p2, 1);
    stage(p2, cur, spare, 2);
    std::swap(cur, spare);
  }
  return launch_ok(ctx, "levelset rk3");
}

}  // namespace
}  // namespace pb

extern "C" pb_status pb_build_levelset(pb_ctx* ctx, const double* atoms, int n_atoms, const pb_params* prm,
                                       const pb_grid* grid, double* phi, size_t cap, size_t* needed) {
  using namespace pb;
  if (!ctx) return PB_EINVAL;
  PB_TRY(check_params(ctx, prm));
  if (!grid) return ctx->fail(PB_EINVAL, "pb_build_levelset: NULL grid");
  if (grid->nx < 7 || grid->ny < 7 || grid->nz < 7)
    return ctx->fail(PB_EINVAL, "pb_build_levelset: grid must be at least 7 nodes per axis");
  if (grid->nx > kMaxAxis || grid->ny > kMaxAxis || grid->nz > kMaxAxis)
    return ctx->fail(PB_EINVAL, "pb_build_levelset: grid axes hold at most %d nodes", kMaxAxis);
  if (!std::isfinite(grid->origin[0]) || !std::isfinite(grid->origin[1]) || !std::isfinite(grid->origin[2]))
    return ctx->fail(PB_EINVAL, "pb_build_levelset: non-finite grid origin");
  if (std::fabs(grid->h - prm->h) > 1e-12 * prm->h)
    return ctx->fail(PB_EINVAL, "pb_build_levelset: grid spacing differs from params.h");
  const size_t count = (size_t)grid->nx * (size_t)grid->ny * (size_t)grid->nz;
  if (count >= ((size_t)1 << 31)) return ctx->fail(PB_EINVAL, "pb_build_levelset: grid of 2^31 nodes or more");
  if (needed) *needed = count;
  if (!phi) return PB_OK;  // size query
  if (cap < count)
    return ctx->fail(PB_ECAPACITY, "pb_build_levelset: phi holds %zu doubles, the grid needs %zu", cap, count);
  if (!atoms || n_atoms <= 0) return ctx->fail(PB_EINVAL, "pb_build_levelset: NULL or empty atoms");
  PB_HIP(ctx, hipSetDevice(ctx->device));
  GridDev g{grid->nx, grid->ny, grid->nz, grid->origin[0], grid->origin[1], grid->origin[2], grid->h};
  const int64_t total = (int64_t)g.nx * g.ny * g.nz;
  const double h = prm->h;
  const bool ses = prm->ls_mode == PB_LS_SES;

  // steps of the inward eikonal flow to t = ρ0 (equal, no longer than cfl·h) and of the reinitialization;
  // φ starts in the buffer from which so many swaps end in the caller's
  const int n_e = ses && prm->probe > 0.0 ? (int)std::ceil(prm->probe / (prm->cfl * h) - 1e-9) : 0;
  const int n_r = prm->reinit_steps > 0 ? prm->reinit_steps : 2 * (int)std::ceil((prm->band_k + 4.0) / prm->cfl - 1e-9);
  double *cur = phi, *spare = nullptr, *p2 = nullptr, *S = nullptr;
  int* flags = nullptr;
  if (ses) {
    spare = (double*)workspace(ctx, "ls_p1", sizeof(double) * total);
    p2 = (double*)workspace(ctx, "ls_p2", sizeof(double) * total);
    S = (double*)workspace(ctx, "ls_S", sizeof(double) * total);
    flags = (int*)workspace(ctx, "ls_flags", 4 * sizeof(int));
    if (!spare || !p2 || !S || !flags) return PB_ENOMEM;
    if ((n_e + n_r) % 2) std::swap(cur, spare);
  }
  {
    Scope t(ctx, "levelset");
    const bool two = vdw_two_levels(total, n_atoms);
    const int T = two ? 2 : 1;
    const unsigned blocks = (unsigned)(((g.nx + T * kTI - 1) / (T * kTI)) * (int64_t)((g.ny + T * kTJ - 1) / (T * kTJ)) *
                                       ((g.nz + T * kTK - 1) / (T * kTK)));
    (two ? k_vdw<true> : k_vdw<false>)<<<blocks, kBlock, 0, ctx->stream>>>(g, atoms, n_atoms, ses ? prm->probe : 0.0,
                                                                           cur);
  }
  PB_TRY(launch_ok(ctx, "vdw"));
  if (!ses) return sync(ctx, "pb_build_levelset");
  if (n_e) PB_TRY(tvd_rk3(ctx, g, cur, spare, p2, nullptr, 0, n_e, prm->probe / n_e));

  // cavity removal; masks and list in the buffers of the flows (a row's words are no more than its nodes)
  const int nw = (g.nz + 63) / 64, words = g.nx * g.ny * nw;
  uint64_t *P = (uint64_t*)spare, *O = (uint64_t*)p2;
  unsigned* list = (unsigned*)S;
  auto per = [](int64_t n, int q) { return (unsigned)((n + q - 1) / q); };
  PB_HIP(ctx, hipMemsetAsync(flags, 0, 3 * sizeof(int), ctx->stream));
  {
    Scope t(ctx, "levelset");
    k_cav_masks<<<per(words, kBlock / 64), kBlock, 0, ctx->stream>>>(g, nw, words, cur, P, O);
  }
  PB_TRY(launch_ok(ctx, "cavity masks"));
  // two rounds of sweeps at a time: the last round of any fill only finds that nothing changes
  for (int it = 0;; it += 2) {
    if (it > 100000) return ctx->fail(PB_EDEVICE, "cavity flood fill did not converge");
    if (it) PB_HIP(ctx, hipMemsetAsync(flags, 0, 2 * sizeof(int), ctx->stream));
    for (int r = 0; r < 2; ++r) {
      Scope t(ctx, "levelset");
      const int64_t plane = (int64_t)g.ny * nw;
      k_cav_xy<<<per((int64_t)g.ny * nw, kBlock / 64), kBlock, 0, ctx->stream>>>(nw, g.nx, plane, g.ny, nw, P, O,
                                                                                flags + r);
      k_cav_xy<<<per((int64_t)g.nx * nw, kBlock / 64), kBlock, 0, ctx->stream>>>(nw, g.ny, nw, g.nx, plane, P, O,
                                                                                flags + r);
      k_cav_z<<<per((int64_t)g.nx * g.ny, 64), 64, 0, ctx->stream>>>(g, nw, P, O, flags + r);
    }
    PB_TRY(launch_ok(ctx, "cavity sweep"));
    int changed = 0;
    PB_HIP(ctx, hipMemcpyAsync(&changed, flags + 1, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    PB_TRY(sync(ctx, "cavity sweep"));
    if (!changed) break;
  }
  const double eps = prm->band_k * h;
  const double rr = (eps + h) / h;
  const int m = (int)std::min(std::floor(rr), (double)kMaxAxis);
  {
    Scope t(ctx, "levelset");
    k_cav_list<<<per(words, kBlock), kBlock, 0, ctx->stream>>>(g, nw, words, P, O, eps, cur, list, flags + 2);
    k_cav_fill<<<1024, kBlock, 0, ctx->stream>>>(g, nw, O, list, flags + 2, eps, m, rr * rr, cur);
  }
  PB_TRY(launch_ok(ctx, "cavity fill"));

  // reinitialization with the frozen smoothed sign of the post-removal φ
  {
    Scope t(ctx, "levelset");
    k_sign<<<per(total, kBlock), kBlock, 0, ctx->stream>>>(total, cur, h, S);
  }
  PB_TRY(launch_ok(ctx, "sign"));
  PB_TRY(tvd_rk3(ctx, g, cur, spare, p2, S, 1, n_r, prm->cfl * h));
  return sync(ctx, "pb_build_levelset");
}
