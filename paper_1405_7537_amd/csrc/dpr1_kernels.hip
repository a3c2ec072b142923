// Forward-stable DPR1 eigensolver: gfx950 kernels and the C ABI.
//
// Paper: Jakovcevic Stor, Slapnicar, Barlow, "Forward stable eigenvalue
// decomposition of rank-one modifications of diagonal matrices" (Alg. 1).
//
// Kernels (all FP64; double-double where the paper asks for double the
// working precision):
//   k_prep  -- per problem: checks of Sec. 1, the rho < 0 reduction, staging
//              of (d_j, zeta_j^2) pairs and the low parts of zeta_j^2.
//   k_eig   -- one lane per eigenvalue, 64 eigenvalues per block; W waves of
//              a block split the inner index j.  All lanes of a wave read the
//              same (d_j, zeta_j^2) at the same time, so the data arrive
//              through scalar loads and feed the FP64 VALU as SGPR operands.
//              Per eigenvalue: shift test, tip b in double-double, extreme
//              root of the arrowhead secular function (model passes, the
//              last one with compensated summation), near-zero test, ||x||.
//              From order FAR_MIN on only the poles near the block's
//              eigenvalues are summed one by one; the others enter through
//              expansions whose moments k_far has formed.
//              Instances for 4, 6 and 8 waves per SIMD (register budgets);
//              the split W, the budget and the pass count are options that
//              dpr1_autotune / dpr1_batched_autotune choose by timing.
//   k_far   -- moments of the far-field expansions, one per block of 64
//              eigenvalues and (from FAR_MIN2) one per 512.
//   k_fix   -- one 256-thread block at a time per flagged eigenpair: root
//              search continued past k_eig's pass budget, double-double
//              Newton polish, and the near-zero recomputation of eq. (gamma).
//   k_fixvec -- k_fix's work and the eigenvector writer in one launch: a few
//              blocks finish the flagged eigenpairs while the others write V,
//              a block per tile of rows and columns, non-temporal stores
//              in windows aligned to whole cache lines; a flagged column is
//              written by the block that finishes its eigenpair.
#include <float.h>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <memory>
#include <vector>

#include "../../include/dpr1.h"
#include "dd.h"
#include "far_sizes.h"

namespace dpr1 {

constexpr int MAXW = 16;
constexpr double GROW = 1.0 + 0x1p-40;

typedef const __attribute__((address_space(4))) double cdouble;

// Wave-uniform load through the scalar data cache (idx must be uniform).
__device__ __forceinline__ double ldu(const double* base, int64_t idx) {
  return ((cdouble*)base)[idx];
}

struct Meta {
  int64_t off;   // first element of the problem in the packed arrays
  int32_t n;
  int32_t neg;   // rho < 0: solved as (-d reversed, z reversed, -rho)
  int32_t info;
  int32_t pad;
  double rho;    // |rho|
  double zz;     // sum zeta_j^2
  double zabs;   // sum |zeta_j| (K_z of eq. knu2)
};

enum : int32_t { FIX_POLISH = 1, FIX_NEARZERO = 2, FIX_CONTINUE = 4 };

// A flagged eigenpair: polish, near-zero rule, or a rational iteration still
// running when the eigenvalue kernel reached its pass budget (then cnu, cL,
// cU, cprev, iters hold the iteration's state).
struct FixItem {
  int32_t p, k, i, flags;
  int32_t iters, pad;
  double nu0, nu1, bhi, blo, lo, hi;
  double cnu, cL, cU, cprev;
};

struct KArgs {
  const Meta* meta;
  const double* pairs;  // [2N]: (d'_j, zeta'_j^2)
  const double* z2lo;   // [N]  low part of zeta'_j^2
  const double* sd;     // [N]  d'
  const double* sz;     // [N]  zeta'
  int32_t* ii;          // [N]  shift index (within the problem)
  double* mu;           // [N]
  double* xs;           // [N]  |mu| * ||x||_2
  double* lam;          // [N]
  FixItem* fix;         // [N]
  uint8_t* vflag;       // [N]  1: eigenpair finished in k_fix (its V column written after)
  int32_t* ctr;         // [0] fix count, [1] queue head, [2] k_fix queue head
  int32_t* stats;       // nullable
  const int4* items;    // batched queue (p, k0, record of the wide level or -1, its slices), or nullptr
  int32_t nitems;
  const double* far;    // far-field records (FAR_REC doubles each; a batch: record of item e at e), or
                        // nullptr: every pole summed directly
  int32_t far_wide, far_slices;  // one problem: first record of the wide level (0: none), its slices
  int32_t far_min;      // a batch: smallest order with records
  int32_t nfixcap;  // capacity of `fix` (one slot per eigenvalue)
  int32_t W;
  int32_t mode_b, root, polish;
  int32_t main_passes;
  double kappa_polish, nearzero;
  int32_t g0;           // single problem: first group of 64 eigenvalues of this launch
  int32_t remedy;       // apply (R1)/(R2) where K_nu > knu_thr
  double knu_thr;
  double* knu;          // optional output: K_nu per eigenpair (caller's order)
  // the caller's outputs (all but lam_out and info_out may be null) and the
  // eigenvector writer's per-column constants
  double* lam_out;
  int32_t* idx_out;
  double* mu_out;
  double* xn_out;
  int32_t* info_out;
  double* V;
  const int64_t* voffs;
  int64_t ldv;
  double* csig;         // [N]  sigma_k
  double* cinv;         // [N]  1/||x_k||
};

// ------------------------------------------------------------ bit helpers
__device__ __forceinline__ uint64_t bits(double x) { return (uint64_t)__double_as_longlong(x); }
__device__ __forceinline__ double unbits(uint64_t u) { return __longlong_as_double((long long)u); }

// midpoint in the order of binary64 numbers, 0 < lo < hi
__device__ __forceinline__ double fmid(double lo, double hi) {
  uint64_t a = bits(lo), b = bits(hi);
  return unbits(a + (b - a) / 2);
}
__device__ __forceinline__ bool adjacent(double lo, double hi) { return bits(hi) - bits(lo) <= 1; }
// the same for lo < hi of one sign (both negative: the bit patterns run backwards)
__device__ __forceinline__ bool adjacent_signed(double lo, double hi) {
  return lo > 0.0 ? bits(hi) - bits(lo) <= 1 : bits(lo) - bits(hi) <= 1;
}
__device__ __forceinline__ double fmid_signed(double lo, double hi) {
  return lo > 0.0 ? fmid(lo, hi) : -fmid(-hi, -lo);
}

// Reciprocal from the hardware estimate refined by one Newton step: for the
// signs that steer bisection, and as the seed of a quotient that is then
// corrected by its residual (within about half an ulp more than correct
// rounding).  v_rcp_f64 is specified to 2^29 ulp (2^-23 relative) and
// measured at 2^-24.4 on gfx950 over random normal inputs; one Newton step
// gives 2^-48.7.  The IEEE divide costs about twice as many instructions on
// this ISA.
__device__ __forceinline__ double rcp_1nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE); }
__device__ __forceinline__ int lane_id() { return threadIdx.x % WAVE; }
__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0; }

// lane l's value to every lane (an SGPR), l a compile-time constant
__device__ __forceinline__ double lane_value(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// ------------------------------------------------- cross-wave reductions
// Every wave of the block ends with the same sums, added in the same order,
// so all waves keep identical per-lane state.
template <int NV>
__device__ __forceinline__ void wg_sum(double (&v)[NV], int W, int wv, int lane, double* red) {
  static_assert(NV <= 4, "the reduction buffer holds four values per lane and wave");
  if (W == 1) return;
#pragma unroll
  for (int q = 0; q < NV; ++q) red[(q * W + wv) * WAVE + lane] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double s = red[(q * W) * WAVE + lane];
    for (int w = 1; w < W; ++w) s += red[(q * W + w) * WAVE + lane];
    v[q] = s;
  }
  __syncthreads();
}

// (s, c) Neumaier partials -> combined with TwoSum in wave order.
__device__ __forceinline__ void wg_sum_comp(double& s, double& c, int W, int wv, int lane, double* red) {
  if (W == 1) return;
  red[(0 * W + wv) * WAVE + lane] = s;
  red[(1 * W + wv) * WAVE + lane] = c;
  __syncthreads();
  double S = red[lane], C = red[W * WAVE + lane];
  for (int w = 1; w < W; ++w) {
    dd t = two_sum(S, red[w * WAVE + lane]);
    S = t.hi;
    C += red[(W + w) * WAVE + lane] + t.lo;
  }
  s = S;
  c = C;
  __syncthreads();
}

// same-signed double-double partials
__device__ __forceinline__ void wg_sum_dd(dd& a, int W, int wv, int lane, double* red) {
  if (W == 1) return;
  red[(0 * W + wv) * WAVE + lane] = a.hi;
  red[(1 * W + wv) * WAVE + lane] = a.lo;
  __syncthreads();
  dd s = {red[lane], red[W * WAVE + lane]};
  for (int w = 1; w < W; ++w) s = dd_add_same(s, dd{red[w * WAVE + lane], red[(W + w) * WAVE + lane]});
  a = s;
  __syncthreads();
}

// Walk the wave's slice [j0, j1) of the inner index in three segments:
// below the window of shift indices this wave can own (seg 0: every lane has
// j < i), inside it (seg 1: per-lane test), above it (seg 2: every lane has
// j > i).  j is wave-uniform in all three loops.  f(j, seg, d_j, zeta_j^2,
// low part of zeta_j^2 (0 unless asked for), u) with u the position of the
// pair in its block (a compile-time constant once unrolled), or -1 for the
// pairs after the last whole block.
template <bool LO, class F>
__device__ __forceinline__ void sweep_seg(const double* P, const double* Zl, int a, int b, int seg, F& f) {
  // Blocks of B pairs (with LO also the B low parts of zeta_j^2), software-
  // pipelined: the scalar loads of the next block are issued before the
  // current block is computed, so their latency hides behind that work.  A
  // wait for scalar loads covers all of them, so no load may be waited for
  // inside the computation; with LO the blocks are halved to keep both
  // blocks in scalar registers.
  constexpr int B = LO ? 4 : 8;
  constexpr int NV = LO ? 3 * B : 2 * B;
  auto load = [](double (&c)[NV], const double* q, const double* ql) {
#pragma unroll
    for (int t = 0; t < 2 * B; ++t) c[t] = ldu(q, t);
    if constexpr (LO) {
#pragma unroll
      for (int t = 0; t < B; ++t) c[2 * B + t] = ldu(ql, t);
    }
  };
  const double* q = P + 2 * (int64_t)a;
  const double* ql = LO ? Zl + a : nullptr;
  int j = a;
  if (j + B <= b) {
    double c[NV];
    load(c, q, ql);
    // wait for the first block here (s_waitcnt lgkmcnt(0)): otherwise the wait
    // for it lands inside the loop, where it also waits for the prefetch
    __builtin_amdgcn_s_waitcnt(0xC07F);
    for (; j + 2 * B <= b; j += B, q += 2 * B, ql += LO ? B : 0) {
      double nx[NV];
      load(nx, q + 2 * B, LO ? ql + B : nullptr);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < B; ++u) f(j + u, seg, c[2 * u], c[2 * u + 1], LO ? c[2 * B + u] : 0.0, u);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < NV; ++t) c[t] = nx[t];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) f(j + u, seg, c[2 * u], c[2 * u + 1], LO ? c[2 * B + u] : 0.0, u);
    j += B;
    q += 2 * B;
    ql += LO ? B : 0;
  }
  for (; j < b; ++j, q += 2, ql += LO ? 1 : 0)
    f(j, seg, ldu(q, 0), ldu(q, 1), LO ? ldu(ql, 0) : 0.0, -1);
}

template <class F>
__device__ __forceinline__ void sweep(const double* P, int j0, int j1, int wlo, int whi, F&& f) {
  sweep_seg<false>(P, nullptr, j0, min(j1, wlo), 0, f);
  sweep_seg<false>(P, nullptr, max(j0, wlo), min(j1, whi), 1, f);
  sweep_seg<false>(P, nullptr, max(j0, whi), j1, 2, f);
}

// the same walk, also handing f the low part of zeta_j^2 from Zl
template <class F>
__device__ __forceinline__ void sweep_lo(const double* P, const double* Zl, int j0, int j1, int wlo, int whi,
                                         F&& f) {
  sweep_seg<true>(P, Zl, j0, min(j1, wlo), 0, f);
  sweep_seg<true>(P, Zl, max(j0, wlo), min(j1, whi), 1, f);
  sweep_seg<true>(P, Zl, max(j0, whi), j1, 2, f);
}

// ------------------------------------------------------------------ prep
// nsplit == 1: block p stages problem p and writes its meta.  nsplit > 1 (a
// single problem): block b stages one slice and leaves its partial sums and
// flags in `part`, which k_meta adds in slice order (the last block of k_prep
// doing it behind a fence cost 20 us at n = 32768: the fence writes back the
// XCD's L2).  Block 0 also clears the counters and the stats.
constexpr int PREP_MAX_SPLIT = 64;
__device__ __forceinline__ void put_meta(int p, int64_t off, int64_t n, double rho, double zz, double za, int fl,
                                         Meta* meta, int32_t* info) {
  int code = 0;
  if (!isfinite(rho) || rho == 0.0) code = DPR1_INFO_BAD_RHO;
  else if (fl & 4) code = DPR1_INFO_NONFINITE;
  else if (fl & 1) code = DPR1_INFO_UNSORTED;
  else if (fl & 2) code = DPR1_INFO_ZERO_Z;
  else if (fl & 8) code = DPR1_INFO_RANGE;
  Meta m;
  m.off = off;
  m.n = (int32_t)n;
  m.neg = rho < 0;
  m.info = code;
  m.pad = 0;
  m.rho = fabs(rho);
  m.zz = zz;
  m.zabs = za;
  meta[p] = m;
  if (info) info[p] = code;
}
__global__ void __launch_bounds__(256) k_prep(int nprob, int nsplit, const int64_t* __restrict__ offs,
                                              int64_t n_single, const double* __restrict__ d,
                                              const double* __restrict__ z, const double* __restrict__ rho_dev,
                                              double rho_host, Meta* __restrict__ meta, double* __restrict__ sd,
                                              double* __restrict__ sz, double* __restrict__ pairs,
                                              double* __restrict__ z2lo, int32_t* __restrict__ info,
                                              double* __restrict__ part, int32_t* __restrict__ ctr,
                                              int32_t* __restrict__ stats) {
  const int p = nsplit == 1 ? (int)blockIdx.x : 0;
  const int bs = nsplit == 1 ? 0 : (int)blockIdx.x;
  if (blockIdx.x == 0 && threadIdx.x < 16) {
    ctr[threadIdx.x] = 0;
    if (stats && threadIdx.x < DPR1_NSTATS) stats[threadIdx.x] = 0;
  }
  if (p >= nprob) return;
  const int64_t off = offs ? offs[p] : 0;
  const int64_t n = offs ? offs[p + 1] - offs[p] : n_single;
  const double rho = rho_dev ? rho_dev[p] : rho_host;
  const int neg = rho < 0;
  const int64_t chunk = (n + nsplit - 1) / nsplit;
  const int64_t ja = min(n, (int64_t)bs * chunk), jb = min(n, ja + chunk);
  __shared__ double red[256], red2[256];
  __shared__ int flags;
  if (threadIdx.x == 0) flags = 0;
  __syncthreads();
  int f = 0;
  double acc = 0.0, acc2 = 0.0;
  for (int64_t j = ja + threadIdx.x; j < jb; j += blockDim.x) {
    int64_t src = neg ? n - 1 - j : j;
    double dj = d[off + src], zj = z[off + src];
    if (!isfinite(dj) || !isfinite(zj)) f |= 4;
    if (zj == 0.0) f |= 2;
    // zeta_j^2 must be a normal number (the sums are taken in squares), and
    // two poles closer than 2^-1000 would put 1/(d_j - d_i) and nu beyond the
    // binary64 range
    if (zj != 0.0 && fabs(zj) < 0x1p-511) f |= 8;
    if (j + 1 < n) {
      double dn = d[off + src + (neg ? -1 : 1)];
      // staged order must be strictly decreasing: d_j > d_{j+1} (or -d reversed)
      if (!(neg ? (-dj > -dn) : (dj > dn))) f |= 1;
      else if (fabs(dj - dn) < 0x1p-1000) f |= 8;
    }
    double ds = neg ? -dj : dj;
    double z2 = zj * zj;
    sd[off + j] = ds;
    sz[off + j] = zj;
    pairs[2 * (off + j)] = ds;
    pairs[2 * (off + j) + 1] = z2;
    z2lo[off + j] = __builtin_fma(zj, zj, -z2);
    acc += z2;
    acc2 += fabs(zj);
  }
  if (f) atomicOr(&flags, f);
  red[threadIdx.x] = acc;
  red2[threadIdx.x] = acc2;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[threadIdx.x] += red[threadIdx.x + s];
      red2[threadIdx.x] += red2[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  if (nsplit > 1) {
    // part: (sum zeta^2, sum |zeta|, flags) per slice
    part[3 * bs] = red[0];
    part[3 * bs + 1] = red2[0];
    part[3 * bs + 2] = (double)flags;
  } else {
    put_meta(p, off, n, rho, red[0], red2[0], flags, meta, info);
  }
}
__global__ void __launch_bounds__(64) k_meta(int nsplit, const int64_t* __restrict__ offs, int64_t n_single,
                                             const double* __restrict__ rho_dev, double rho_host,
                                             const double* __restrict__ part, Meta* __restrict__ meta,
                                             int32_t* __restrict__ info) {
  __shared__ double lp[3 * PREP_MAX_SPLIT];
  for (int t = threadIdx.x; t < 3 * nsplit; t += 64) lp[t] = part[t];
  __syncthreads();
  if (threadIdx.x != 0) return;
  double zz = 0.0, za = 0.0;
  int fl = 0;
  for (int q = 0; q < nsplit; ++q) {
    zz += lp[3 * q];
    za += lp[3 * q + 1];
    fl |= (int)lp[3 * q + 2];
  }
  put_meta(0, offs ? offs[0] : 0, offs ? offs[1] - offs[0] : n_single, rho_dev ? rho_dev[0] : rho_host, zz, za, fl,
           meta, info);
}

// ------------------------------------------------------------------- out
// The shifted representation of an eigenpair is usable when lambda is finite,
// mu is a normal number and |mu| ||x|| is finite and positive.  It leaves the
// binary64 range when |delta_j / mu| exceeds it (mu beside a pole with zeta
// near 1e-150 while the poles spread over many decades): the problem's info
// then reports DPR1_INFO_RANGE instead of returning NaN silently.
__device__ __forceinline__ bool range_ok(double lam, double mu, double xs) {
  return fabs(lam) < INFINITY && fabs(mu) >= 2.2250738585072014e-308 && fabs(mu) < INFINITY && xs > 0.0 &&
         xs < INFINITY;
}
// An eigenpair's values in the caller's order (rho < 0 maps k -> n-1-k,
// lambda -> -lambda); final: checked for range too.
__device__ __forceinline__ void put_outputs(const KArgs& A, const Meta& M, int p, int k, int i, double lam, double mu,
                                            double xs, bool final) {
  const int64_t b = M.off + (M.neg ? M.n - 1 - k : k);
  const double sg = M.neg ? -1.0 : 1.0;
  A.lam_out[b] = sg * lam;
  if (A.idx_out) A.idx_out[b] = M.neg ? M.n - 1 - i : i;
  if (A.mu_out) A.mu_out[b] = sg * mu;
  if (A.xn_out) A.xn_out[b] = xs / fabs(mu);
  if (final && !range_ok(lam, mu, xs)) A.info_out[p] = DPR1_INFO_RANGE;
}

// ------------------------------------------------------------------- eig
// Step from the current iterate m to the root of the model of g.  Written in
// poles, g(t) = b' - t + sum_j w_j/(t - xi_j) with xi_j = 1/delta'_j and
// w_j = zeta_j^2/(delta'_j^2 zeta_i^2); the wanted root lies right of every
// pole.  The model keeps the nearest pole xm with its exact weight sw^2 and
// replaces the rest of the sum by one pole p fitted to value, slope and
// curvature at m (Spz, Sppz are the moments sum w/(m - xi)^2, sum
// w/(m - xi)^3).  Every other pole lies left of xm, so the fitted pole does
// too.  With D = t - m and g the value at m the model's root satisfies
//   D (1 + a^2/(1 + D e) + r/(1 + D f)) = g,
// e = 1/(m - xm), a = sw e, r the rest of the slope, f = 1/(m - p): D comes
// with the relative accuracy of g whatever its size, so refined reciprocal
// estimates serve.  Solved in steps x from the residual h at the current D:
// one quotient of the slope and curvature there, x (1 + sl/(1 + x be)) = -h, a
// quadratic in x; inside the bracket (L, U), until a step is below 2^-20 of D,
// which leaves less than 2^-40 of it.  Two to five steps where Newton's method
// doubles D step by step beside a small zeta_i.  (Newton's method for t itself to 2^-52 with IEEE quotients
// took up to 20 us a call: single lanes ran 40 steps at the rounding level,
// and the wave waits for the last.)  The model matches g to second order at m,
// so the outer iteration converges cubically.  The weight enters as its square
// root: with zeta_i near 1e-148 beside a pole 1e-13 away a weight reaches
// 1e322 while weight/(t - pole) is finite.  A model whose parameters are not
// finite says nothing: NaN makes the caller take a bisection step.
__device__ __forceinline__ double model_delta(double m, double g, double Spz, double Sppz, double xm, double sw,
                                              double L, double U) {
  const double e = rcp_1nr(m - xm);
  const double a = sw * e;
  const double a2 = a * a;
  double r = Spz - a2;
  const double rpp = Sppz - a2 * e;
  double f = 0.0;
  // (slopes below 2^-80 count for nothing beside the 1, and have no reciprocal
  // where they are subnormal)
  if (r > 0x1p-80 && rpp > 0.0)
    f = fmin(rpp * rcp_1nr(r), e);
  else
    r = 0.0;
  if (!(fabs(g) < INFINITY) || !(e < INFINITY) || !(a2 + r < INFINITY)) return NAN;
  double lo = fmax(L, xm) - m, hi = U - m;
  double D = 0.0, h = -g, u1 = 1.0, u2 = 1.0;
  for (int q = 0; q < 40; ++q) {
    const double A1 = a2 * (u1 * u1), R1 = r * (u2 * u2);
    const double sl = A1 + R1;
    double x;
    if (sl > 0x1p-80) {
      // be x^2 + B x + h = 0, the root that goes to 0 with h
      const double be = __builtin_fma(A1 * u1, e, R1 * u2 * f) * rcp_1nr(sl);
      const double B = __builtin_fma(h, be, 1.0 + sl);
      const double iB = rcp_1nr(B);
      const double t = -h * iB;
      const double w = __builtin_fma(4.0 * be * t, iB, 1.0);
      const double y = __builtin_amdgcn_rsq(w);
      double S = w * y;
      S = __builtin_fma(__builtin_fma(-S, S, w), 0.5 * y, S);
      x = B > 0.0 ? 2.0 * t * rcp_1nr(1.0 + S) : -0.5 * B * (1.0 + S) * rcp_1nr(be);
    } else {
      x = -h;  // no slope beside t's own
    }
    double n = D + x;
    // (tested before the bracket: D may sit on the end that it has just set)
    if (fabs(x) <= 0x1p-20 * fabs(n)) {
      D = n;
      break;
    }
    // outside the bracket: a point just inside the end passed; where the
    // model's root lies beyond that too, it is the answer if the end is within
    // 2^20 of m (else the caller halves the bracket in the exponent)
    const int out = n <= lo ? -1 : n >= hi ? 1 : 0;
    if (out) n = out < 0 ? __builtin_fma(0x1p-45, D - lo, lo) : __builtin_fma(0x1p-45, D - hi, hi);
    if (!(n != D)) return NAN;
    D = n;
    u1 = rcp_1nr(__builtin_fma(D, e, 1.0));
    u2 = rcp_1nr(__builtin_fma(D, f, 1.0));
    h = __builtin_fma(D, 1.0 + __builtin_fma(a2, u1, r * u2), -g);
    if (!(h == h)) return NAN;
    if ((out < 0 && h > 0.0) || (out > 0 && h < 0.0)) {
      const double t = m + D;
      return t > 0x1p-19 * m && t < 0x1p20 * m ? D : NAN;
    }
    if (h == 0.0) break;
    if (h < 0.0) lo = D; else hi = D;
  }
  return D;
}

// g(m) = b' - m + S/zeta_i^2 of an accurate pass: b' = bh + bl, S = sh + sl,
// every sum and the quotient carried with its rounding error, so that only the
// errors of the terms of S are left (Sz: the quotient in working precision).
__device__ __forceinline__ double g_value(double bh, double bl, double m, double sh, double sl, double zi,
                                          double& Sz) {
  const double z2 = zi * zi, z2l = __builtin_fma(zi, zi, -z2);
  Sz = (sh + sl) / z2;
  double e = __builtin_fma(-Sz, z2, sh);
  e = __builtin_fma(-Sz, z2l, e + sl);
  const dd a = two_sum(bh, -m);
  const dd b = two_sum(a.hi, Sz);
  const double g = b.hi + (((a.lo + b.lo) + bl) + e / z2);
  return g == g ? g : (bh - m) + Sz;
}

// One step of the safeguarded iteration for the rightmost root of g from its
// value g and moments at m (the bracket [L, U] already updated with the sign
// of g).  A model root outside (L, U) is replaced by the bit midpoint, and so
// is the next iterate of a two-cycle: g changed sign at the last two steps
// while |g| fell by less than a factor 10 on the same side (g1, g2 keep the
// two previous values of g).
__device__ __forceinline__ void model_step(double m, double g, double Spz, double Sppz, double xm, double sw,
                                           int iters, double L, double U, double& nu, double& nu0, double& prevstep,
                                           double& g1, double& g2, bool& done, double tol = 0x1p-20) {
  if (g == 0.0) {
    done = true;
    nu0 = m;
    return;
  }
  const bool cycle = (g * g1 < 0.0) && (g1 * g2 < 0.0) && (fabs(g) > 0.1 * fabs(g2));
  g2 = g1;
  g1 = g;
  const double dm = model_delta(m, g, Spz, Sppz, xm, sw, L, U);
  double nn = m + dm;
  const double step = fabs(dm);
  // Cubic convergence: a step e leaves a model error of about 8 e^3 (the
  // shift keeps every pole at least nu/2 from the root), so after a step
  // below 2^-20 the new iterate is exact to rounding.  The same tolerance
  // accepts the step of the accurate last pass.
  if (step <= tol * m) {
    done = true;
    nu0 = (nn >= L && nn <= U) ? nn : m;
    return;
  }
  if (!(nn > L && nn < U) || cycle) {
    if (adjacent(L, U)) {
      done = true;
      nu0 = U;
      return;
    }
    nn = fmid(L, U);
  } else if (iters >= 8 && step > 0.5 * prevstep) {
    done = true;  // rounding noise dominates g: leave it to the checks after
    nu0 = nn;
    return;
  }
  if (iters >= 40) {
    done = true;
    nu0 = nn;
    return;
  }
  prevstep = fabs(nn - m);
  nu = nn;
}

// ------------------------------------------------------------- far field
// The sums of the method over the poles far from a block's 64 eigenvalues.
// With c the middle and R = 1/iR the half-width of the interval that holds the
// block's eigenvalues and shift poles, D_j = (d_j - c)/R, x = (t - c)/R,
//   sum_far zeta_j^2/(d_j - t) = f(x) = sum_q m_q T_q(x),
//   m_0 = sum a_j, m_q = 2 sum a_j u_j^q,
//   u = 1/(D + sign(D) sqrt(D^2 - 1)), a = (zeta^2 iR)/(sign(D) sqrt(D^2 - 1))
// (Chebyshev expansion of 1/(D - x) on [-1, 1]; geometric in u).  A pole is
// far when |D| >= FAR_T = 2.5, so |u| <= 1/4.79 and FAR_P = 48 orders leave
// less than 2^-106 of the sum of magnitudes; orders below FAR_Q = 24 are
// accumulated in double-double, the others (together below 2^-52 of it) in
// binary64.  The tip takes all 48.  The shift test and the passes that only
// steer take FAR_ND = 26: values to 2^-56, slopes to 2^-46 (worst at the end of
// the interval away from a pole at the cut).  The accurate pass, whose slope
// gives ||x||, takes FAR_NA = 31: values to 2^-68, slopes to 2^-57.
// The moments cost about 450 instructions per pole and block instead of the
// 64 x 71 of the direct sums, and what the eigenvalue kernel does per
// eigenvalue no longer grows with n.  A second, wide level (FAR_WIDE blocks
// share an expansion, cut into slices of poles) takes the poles far from
// those; the block's own level then covers only the poles between the two
// windows.  Each pole is in exactly one of: the near window [a, b) (summed
// directly), the block's level, the wide level.  The windows come from the
// poles' positions alone, so any distribution is covered: where poles cluster
// so that nothing is far, the window is the whole problem.  Bound by FP64
// issue; measured at n = 32768 (uniform poles): k_far 72 us and k_eig 126 us
// where the direct sums took 2520 us; the 2048-problem mix 400 and 770 us
// against 3560 us.  Errors against extended precision, all eigenvalues of 17
// distributions, rms in eps: mu 0.30 to 0.49 (direct sums 0.36 to 0.76), ||x||
// 0.45 to 0.57 (0.50 to 0.87).
constexpr int FAR_P = 48, FAR_Q = 24, FAR_ND = 26, FAR_NA = 31;
constexpr double FAR_T = 2.5;
// record: m_q (FAR_P), their low parts (FAR_Q), the moments of the
// magnitudes sum zeta_j^2/|d_j - t| (FAR_ND), c, iR, the window a, b, and the
// number of poles in the level
constexpr int FR_LO = FAR_P, FR_ABS = FR_LO + FAR_Q, FR_C = FR_ABS + FAR_ND, FR_IR = FR_C + 1, FR_A = FR_C + 2,
              FR_B = FR_C + 3, FR_CNT = FR_C + 4, FAR_REC = 104;
static_assert(FR_CNT < FAR_REC, "far record");

struct FarGeo {
  double c, ir;
  int a, b;  // near window: poles a .. b-1
};

// first j in [0, n) with (d_j - c) iR < t (STRICT) or <= t; the products
// decrease with j, so one wave narrows 64-fold per step
template <bool STRICT>
__device__ __forceinline__ int far_first(const double* Dv, int n, double c, double ir, double t, int lane) {
  int lo = 0, len = n;
  while (len > 0) {
    const int step = (len + WAVE - 1) / WAVE;
    const int end = lo + len;
    const int64_t j = lo + (int64_t)(lane + 1) * step - 1;
    bool hit = true;
    if (j < end) {
      const double x = (Dv[j] - c) * ir;
      hit = STRICT ? x < t : x <= t;
    }
    const int cnt = __popcll(__ballot(!hit));
    lo = (int)min((int64_t)end, lo + (int64_t)cnt * step);
    len = min(step - 1, end - lo);
  }
  return lo;
}

// Interval and near window of the eigenvalues e0 .. e0+ne-1.  Where the
// positions leave the range in which the moments are safe (poles further than
// 2^400 half-widths, or an interval that over- or underflows) every pole is
// near.
__device__ __forceinline__ FarGeo far_geo(const double* Dv, int n, int e0, int ne, int lane) {
  FarGeo g;
  const double dl = Dv[max(e0 - 1, 0)], dh = Dv[min(e0 + ne - 1, n - 1)];
  g.c = 0.5 * dl + 0.5 * dh;
  g.ir = 1.0 / fmax(dl - g.c, g.c - dh);
  g.a = 0;
  g.b = n;
  const double x0 = (Dv[0] - g.c) * g.ir, x1 = (Dv[n - 1] - g.c) * g.ir;
  if (g.ir < 0x1p500 && g.ir > 0x1p-500 && fabs(x0) < 0x1p400 && fabs(x1) < 0x1p400) {
    g.a = far_first<true>(Dv, n, g.c, g.ir, FAR_T, lane);
    g.b = far_first<false>(Dv, n, g.c, g.ir, -FAR_T, lane);
  }
  return g;
}

// t (hi, lo) to the accumulator (s, e): TwoSum into s, the rest into e
__device__ __forceinline__ void far_acc(double& s, double& e, double th, double tl) {
  const dd y = two_sum(s, th);
  s = y.hi;
  e += y.lo + tl;
}

// One exchange of a reduce-scatter over 2 H values: lanes with bit M set keep
// the upper half.
template <int H, int M, bool DD>
__device__ __forceinline__ void far_halve(double (&h)[32], double (&l)[32], int lane) {
  const bool up = (lane & M) != 0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double kh = up ? h[i + H] : h[i], sh = up ? h[i] : h[i + H];
    const double oh = __shfl_xor(sh, M);
    if (DD) {
      const double kl = up ? l[i + H] : l[i], sl = up ? l[i] : l[i + H];
      const double ol = __shfl_xor(sl, M);
      const dd y = two_sum(kh, oh);
      h[i] = y.hi;
      l[i] = y.lo + (kl + ol);
    } else {
      h[i] = kh + oh;
    }
  }
}
// After it lanes 2q and 2q+1 hold the wave's sum of value q in h[0] (and, with
// DD, its low part in l[0]; without DD l is not touched).
template <bool DD>
__device__ __forceinline__ void far_reduce(double (&h)[32], double (&l)[32], int lane) {
  far_halve<16, 32, DD>(h, l, lane);
  far_halve<8, 16, DD>(h, l, lane);
  far_halve<4, 8, DD>(h, l, lane);
  far_halve<2, 4, DD>(h, l, lane);
  far_halve<1, 2, DD>(h, l, lane);
  const double oh = __shfl_xor(h[0], 1);
  if (DD) {
    const double ol = __shfl_xor(l[0], 1);
    const dd y = two_sum(h[0], oh);
    h[0] = y.hi;
    l[0] = y.lo + (l[0] + ol);
  } else {
    h[0] = h[0] + oh;
  }
}

// Moments of one (level, group, slice): the block's waves are dealt to the
// poles above and below the window in proportion to their numbers (at least
// one each), so that the sums of magnitudes come from the same accumulators.
__device__ __forceinline__ void far_item(const Meta& M, const double* sd, const double* pairs, const double* z2lo, int e0, bool wide,
                         int slice, int nsl, bool two, double* rec, double* lds) {
  const int lane = lane_id(), wv = wave_id();
  const int n = M.n;
  const double* Dv = sd + M.off;
  const FarGeo g = far_geo(Dv, n, e0, wide ? FAR_WIDE * WAVE : WAVE, lane);
  int pa = 0, pb = n;
  int a = g.a, b = g.b;
  if (two && !wide) {
    const FarGeo w = far_geo(Dv, n, e0 / (FAR_WIDE * WAVE) * (FAR_WIDE * WAVE), FAR_WIDE * WAVE, lane);
    pa = w.a;
    pb = w.b;
    a = max(a, pa);
    b = min(b, pb);
  }
  // this slice's part of the poles above [pa, a) and below [b, pb)
  const int la = a - pa, lb = pb - b;
  const int ua = pa + (int)((int64_t)la * slice / nsl), ub = pa + (int)((int64_t)la * (slice + 1) / nsl);
  const int va = b + (int)((int64_t)lb * slice / nsl), vb = b + (int)((int64_t)lb * (slice + 1) / nsl);
  constexpr int NW = FAR_BLK / WAVE;
  const int cu = ub - ua, cv = vb - va;
  int wu = 0;  // waves on the upper side
  if (cu > 0) wu = cv == 0 ? NW : min(NW - 1, max(1, (int)(((int64_t)NW * cu + (cu + cv) / 2) / (cu + cv))));
  const bool upper = wv < wu;
  const int j0 = upper ? ua + wv * WAVE + lane : va + (wv - wu) * WAVE + lane;
  const int j1 = upper ? ub : vb;
  const int stride = (upper ? wu : NW - wu) * WAVE;

  double mh[32], ml[32], md[32];
#pragma unroll
  for (int q = 0; q < 32; ++q) mh[q] = ml[q] = md[q] = 0.0;
  for (int j = j0; j < j1; j += stride) {
    const double dj = pairs[2 * (M.off + j)], z2 = pairs[2 * (M.off + j) + 1], z2l = z2lo[M.off + j];
    // D and v = 1/D in double-double
    const dd D = dd_mul_d(two_sum(dj, -g.c), g.ir);
    const double r = rcp_1nr(D.hi);
    const double ev = __builtin_fma(-r, D.lo, __builtin_fma(-r, D.hi, 1.0));
    const dd v = fast_two_sum(r, r * ev);
    // s = sqrt(1 - v^2) (0.91 < s <= 1), rs = 1/s to working precision
    const dd vv = dd_mul(v, v);
    dd E = fast_two_sum(1.0, -vv.hi);
    E.lo -= vv.lo;
    double rs = __builtin_amdgcn_rsq(E.hi);
    rs = __builtin_fma(rs, __builtin_fma(-0.5 * E.hi * rs, rs, 0.5), rs);
    rs = __builtin_fma(rs, __builtin_fma(-0.5 * E.hi * rs, rs, 0.5), rs);
    const double s0 = E.hi * rs;
    const dd sq = fast_two_sum(s0, (__builtin_fma(-s0, s0, E.hi) + E.lo) * (0.5 * rs));
    // u = v/(1 + s)
    dd den = fast_two_sum(1.0, sq.hi);
    den.lo += sq.lo;
    const double ru = rcp_1nr(den.hi);
    const double u1 = v.hi * ru;
    const double eu = __builtin_fma(-u1, den.lo, __builtin_fma(-u1, den.hi, v.hi) + v.lo);
    const dd u = fast_two_sum(u1, eu * ru);
    // a = zeta^2 (v iR)/s
    const dd w = dd_mul(dd_mul_d(v, g.ir), dd{z2, z2l});
    const double a1 = w.hi * rs;
    const double ea = __builtin_fma(-a1, sq.lo, __builtin_fma(-a1, sq.hi, w.hi) + w.lo);
    const dd t = fast_two_sum(a1, ea * rs);
    far_acc(mh[0], ml[0], t.hi, t.lo);
    double th = 2.0 * t.hi, tl = 2.0 * t.lo;
#pragma unroll
    for (int q = 1; q < FAR_Q; ++q) {
      const double p = th * u.hi;
      tl = __builtin_fma(tl, u.hi, __builtin_fma(th, u.lo, __builtin_fma(th, u.hi, -p)));
      th = p;
      far_acc(mh[q], ml[q], th, tl);
    }
#pragma unroll
    for (int q = 0; q < FAR_P - FAR_Q; ++q) {
      th *= u.hi;
      md[q] += th;
    }
  }
  far_reduce<true>(mh, ml, lane);
  const double h0 = mh[0], l0 = ml[0];
  far_reduce<false>(md, ml, lane);
  __syncthreads();  // the previous item's sums are no longer read
  if ((lane & 1) == 0) {
    lds[(wv * 3) * 32 + lane / 2] = h0;
    lds[(wv * 3 + 1) * 32 + lane / 2] = l0;
    lds[(wv * 3 + 2) * 32 + lane / 2] = md[0];
  }
  __syncthreads();
  // waves in order; the sum of magnitudes takes the lower side's terms negated
  const int t = threadIdx.x;
  if (t < FAR_Q) {
    dd s = {0.0, 0.0};
    double ab = 0.0;
    for (int w = 0; w < NW; ++w) {
      const double h = lds[(w * 3) * 32 + t], l = lds[(w * 3 + 1) * 32 + t];
      const dd y = two_sum(s.hi, h);
      s = {y.hi, s.lo + (y.lo + l)};
      ab += w < wu ? h : -h;
    }
    s = fast_two_sum(s.hi, s.lo);
    rec[t] = s.hi;
    rec[FR_LO + t] = s.lo;
    rec[FR_ABS + t] = ab;
  } else if (t < FAR_P) {
    double s = 0.0, ab = 0.0;
    for (int w = 0; w < NW; ++w) {
      const double h = lds[(w * 3 + 2) * 32 + t - FAR_Q];
      s += h;
      ab += w < wu ? h : -h;
    }
    rec[t] = s;
    if (t < FAR_ND) rec[FR_ABS + t] = ab;
  } else if (t == FAR_P) {
    rec[FR_C] = g.c;
    rec[FR_IR] = g.ir;
    rec[FR_A] = (double)a;
    rec[FR_B] = (double)b;
    rec[FR_CNT] = (double)(la + lb);
  }
}

// A batch's list, left in the workspace by the plan (the plan struct does not
// hold it): the first nown items of the eigenvalue queue have a record of
// their own (record = item), the wide level's entries are (problem, first
// eigenvalue, slice | slices << 16, record).
struct FarHdr {
  int64_t nown, nwide, wide_off;  // wide_off: bytes from the start of the workspace
};
// The first wide block of one problem (blocks in order: the wide level's
// (group, slice) pairs, then the blocks of 64), or of a batch the wide items,
// then the items of the queue.
struct FarArgs {
  const Meta* meta;
  const double* sd;
  const double* pairs;
  const double* z2lo;
  double* rec;
  int32_t ng, wide, slices;  // one problem: blocks of 64, first record of the wide level (0: none), its slices
  const int4* items;         // a batch
  const FarHdr* hdr;
  const char* work;
};
__global__ void __launch_bounds__(FAR_BLK, 2) k_far(FarArgs F) {
  __shared__ double lds[3 * 32 * (FAR_BLK / WAVE)];
  const bool one = F.items == nullptr;
  const int64_t nwide = one ? (F.wide ? (int64_t)((F.ng + FAR_WIDE - 1) / FAR_WIDE) * F.slices : 0) : F.hdr->nwide;
  const int64_t cnt = nwide + (one ? F.ng : F.hdr->nown);
  const int4* wi = one ? nullptr : reinterpret_cast<const int4*>(F.work + F.hdr->wide_off);
  for (int64_t e = blockIdx.x; e < cnt; e += gridDim.x) {
    const bool wide = e < nwide;
    const int w = (int)(wide ? e : e - nwide);
    int p = 0, e0, slice = 0, nsl = 1;
    int64_t rec;
    bool two = true;
    if (one) {
      e0 = wide ? w / F.slices * (FAR_WIDE * WAVE) : w * WAVE;
      if (wide) {
        slice = w % F.slices;
        nsl = F.slices;
      }
      rec = wide ? F.wide + (int64_t)w : w;
      two = F.wide != 0;
    } else {
      const int4 it = wide ? wi[w] : F.items[w];
      p = it.x;
      e0 = it.y;
      rec = wide ? it.w : w;
      if (wide) {
        slice = it.z & 0xffff;
        nsl = it.z >> 16;
      } else {
        two = it.z >= 0;
      }
    }
    const Meta M = F.meta[p];
    if (M.info != 0) continue;
    far_item(M, F.sd, F.pairs, F.z2lo, e0, wide, slice, nsl, two, F.rec + rec * FAR_REC, lds);
  }
}

// Values of an expansion held in LDS (the layout of a record) by Clenshaw's
// recurrence, differentiated for the slopes.
// The orders P-1 .. L (26 - 1 = 5 x 5, 31 - 1 = 6 x 5) run in fives, whose
// coefficients are loaded together: one LDS latency per five steps.
template <int P, int L = 1, class F>
__device__ __forceinline__ void far_orders(const double* cf, F&& step) {
  static_assert((P - L) % 5 == 0, "orders in fives");
#pragma unroll 1
  for (int c = P - 5; c >= L; c -= 5) {
    double k[5];
#pragma unroll
    for (int u = 0; u < 5; ++u) k[u] = cf[c + u];
#pragma unroll
    for (int u = 4; u >= 0; --u) step(k[u]);
  }
}
template <class F>
__device__ __forceinline__ void far_orders2(const double* cf, const double* cg, F&& step) {
#pragma unroll 1
  for (int c = FAR_ND - 5; c >= 1; c -= 5) {
    double k[5], l[5];
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      k[u] = cf[c + u];
      l[u] = cg[c + u];
    }
#pragma unroll
    for (int u = 4; u >= 0; --u) step(k[u], l[u]);
  }
}
// f, f' and f''/2 at x, and the sum of magnitudes fa
__device__ __forceinline__ void far_eval(const double* cf, double x, double& f, double& f1, double& f2, double& fa) {
  const double x2 = 2.0 * x;
  double b1 = 0.0, b2 = 0.0, p1 = 0.0, p2 = 0.0, h1 = 0.0, h2 = 0.0, m1 = 0.0, m2 = 0.0;
  far_orders2(cf, cf + FR_ABS, [&](double a, double am) {
    const double h0 = __builtin_fma(x2, h1, __builtin_fma(2.0, p1, -h2));
    const double p0 = __builtin_fma(x2, p1, __builtin_fma(2.0, b1, -p2));
    const double b0 = __builtin_fma(x2, b1, a - b2);
    const double m0 = __builtin_fma(x2, m1, am - m2);
    b2 = b1;
    b1 = b0;
    p2 = p1;
    p1 = p0;
    h2 = h1;
    h1 = h0;
    m2 = m1;
    m1 = m0;
  });
  f = __builtin_fma(x, b1, cf[0] - b2);
  f1 = __builtin_fma(x, p1, b1 - p2);
  f2 = __builtin_fma(x, h1, p1 - h2);
  fa = __builtin_fma(x, m1, cf[FR_ABS] - m2);
}
// the divided difference f[x, y], and f', f''/2 and the third derivative / 6 at
// y, from P orders
template <int P>
__device__ __forceinline__ void far_diff(const double* cf, double x, double y, double& fxy, double& f1, double& f2,
                                         double& f3) {
  const double x2 = 2.0 * x, y2 = 2.0 * y;
  double a1 = 0.0, a2 = 0.0, c1 = 0.0, c2 = 0.0;
  double b1 = 0.0, b2 = 0.0, p1 = 0.0, p2 = 0.0, h1 = 0.0, h2 = 0.0, g1 = 0.0, g2 = 0.0;
  far_orders<P>(cf, [&](double k) {
    const double c0 = __builtin_fma(y2, c1, __builtin_fma(2.0, a1, -c2));
    const double a0 = __builtin_fma(x2, a1, k - a2);
    const double g0 = __builtin_fma(y2, g1, __builtin_fma(2.0, h1, -g2));
    const double h0 = __builtin_fma(y2, h1, __builtin_fma(2.0, p1, -h2));
    const double p0 = __builtin_fma(y2, p1, __builtin_fma(2.0, b1, -p2));
    const double b0 = __builtin_fma(y2, b1, k - b2);
    a2 = a1;
    a1 = a0;
    c2 = c1;
    c1 = c0;
    b2 = b1;
    b1 = b0;
    p2 = p1;
    p1 = p0;
    h2 = h1;
    h1 = h0;
    g2 = g1;
    g1 = g0;
  });
  fxy = __builtin_fma(y, c1, a1 - c2);
  f1 = __builtin_fma(y, p1, b1 - p2);
  f2 = __builtin_fma(y, h1, p1 - h2);
  f3 = __builtin_fma(y, g1, h1 - g2);
}
// f[x, y] in double-double at double-doubles x, y, from FAR_NA orders: the
// recurrence of far_diff for the accurate pass, whose sum is carried with its
// rounding errors.  The orders from FAR_QD on are below 2^-5 of f[x, y] (worst, a
// pole at the cut seen from the block's other end), so binary64 there leaves 0.1
// eps; the lower ones take the moments' low parts.  (All orders below FAR_Q in
// double-double: 2 to 4 % of a batch's time.)
constexpr int FAR_QD = 6;
__device__ __forceinline__ dd far_pair(const double* cf, dd x, dd y) {
  const double x2 = 2.0 * x.hi, y2 = 2.0 * y.hi;
  double a1 = 0.0, a2 = 0.0, c1 = 0.0, c2 = 0.0;
  far_orders<FAR_NA, FAR_QD>(cf, [&](double k) {
    const double c0 = __builtin_fma(y2, c1, __builtin_fma(2.0, a1, -c2));
    const double a0 = __builtin_fma(x2, a1, k - a2);
    a2 = a1;
    a1 = a0;
    c2 = c1;
    c1 = c0;
  });
  const dd X2 = {x2, 2.0 * x.lo}, Y2 = {y2, 2.0 * y.lo};
  dd A1 = {a1, 0.0}, A2 = {a2, 0.0}, C1 = {c1, 0.0}, C2 = {c2, 0.0};
  double kh = cf[FAR_QD - 1], kl = cf[FR_LO + FAR_QD - 1];
#pragma unroll 1
  for (int q = FAR_QD - 1; q >= 1; --q) {
    // the next order's coefficients while this one's are used
    const double nh = cf[q - 1], nl = cf[FR_LO + q - 1];
    const dd C0 = dd_add_same(dd_add_same(dd{2.0 * A1.hi, 2.0 * A1.lo}, dd_neg(C2)), dd_mul(Y2, C1));
    const dd A0 = dd_add_same(dd_add_same(dd{kh, kl}, dd_neg(A2)), dd_mul(X2, A1));
    A2 = A1;
    A1 = A0;
    C2 = C1;
    C1 = C0;
    kh = nh;
    kl = nl;
  }
  return dd_add_same(dd_add_same(A1, dd_neg(C2)), dd_mul(y, C1));
}
// f in double-double at a double-double x, and the sum of magnitudes fa
__device__ __forceinline__ dd far_value(const double* cf, dd x, double& fa) {
  const double x2 = 2.0 * x.hi;
  double b1 = 0.0, b2 = 0.0;
  static_assert((FAR_P - FAR_Q) % 6 == 0 && (FAR_Q - 1) == 23, "orders in groups");
#pragma unroll 1
  for (int c = FAR_P - 6; c >= FAR_Q; c -= 6) {
    double k[6];
#pragma unroll
    for (int u = 0; u < 6; ++u) k[u] = cf[c + u];
#pragma unroll
    for (int u = 5; u >= 0; --u) {
      const double b0 = __builtin_fma(x2, b1, k[u] - b2);
      b2 = b1;
      b1 = b0;
    }
  }
  const dd X2 = {x2, 2.0 * x.lo};
  dd B1 = {b1, 0.0}, B2 = {b2, 0.0};
  double m1 = 0.0, m2 = 0.0;
  double kh = cf[FAR_Q - 1], kl = cf[FR_LO + FAR_Q - 1], km = cf[FR_ABS + FAR_Q - 1];
#pragma unroll 1
  for (int q = FAR_Q - 1; q >= 1; --q) {
    // the next order's coefficients while this one's are used (order 0 last)
    const double nh = cf[q - 1], nl = cf[FR_LO + q - 1], nm = cf[FR_ABS + q - 1];
    const dd B0 = dd_add_same(dd_add_same(dd{kh, kl}, dd_neg(B2)), dd_mul(X2, B1));
    B2 = B1;
    B1 = B0;
    const double m0 = __builtin_fma(x2, m1, km - m2);
    m2 = m1;
    m1 = m0;
    kh = nh;
    kl = nl;
    km = nm;
  }
  fa = __builtin_fma(x.hi, m1, km - m2);
  return dd_add_same(dd_add_same(dd{kh, kl}, dd_neg(B2)), dd_mul(x, B1));
}

template <bool B>
struct Bool {
  static constexpr bool value = B;
};

// Expansions of one block: the levels that hold poles (their records in LDS,
// FAR_REC doubles each) and the near window.
struct Far {
  const double* cf;
  int lev, na, nb;
};

// The record of the block's own level, and the wide level's slices added in
// order, to LDS; every thread of the block calls it.
__device__ __forceinline__ Far far_load(const double* r0, const double* r1, int nsl, int n, double* cf) {
  const int t = threadIdx.x;
  Far F;
  F.cf = cf;
  F.lev = 0;
  F.na = 0;
  F.nb = n;
  if (!r0) return F;
  F.na = (int)ldu(r0, FR_A);
  F.nb = (int)ldu(r0, FR_B);
  if (ldu(r0, FR_CNT) != 0.0) {
    for (int q = t; q < FR_A; q += blockDim.x) cf[q] = r0[q];
    F.lev = 1;
  }
  if (r1 && ldu(r1, FR_CNT) != 0.0) {
    double* c1 = cf + F.lev * FAR_REC;
    if (t < FAR_Q) {
      dd s = {0.0, 0.0};
#pragma unroll 4
      for (int w = 0; w < nsl; ++w) {
        const double* q = r1 + (int64_t)w * FAR_REC;
        const dd y = two_sum(s.hi, q[t]);
        s = {y.hi, s.lo + (y.lo + q[FR_LO + t])};
      }
      s = fast_two_sum(s.hi, s.lo);
      c1[t] = s.hi;
      c1[FR_LO + t] = s.lo;
    } else if (t < FAR_P) {
      double s = 0.0;
      for (int w = 0; w < nsl; ++w) s += r1[(int64_t)w * FAR_REC + t];
      c1[t] = s;
    } else if (t < FAR_P + 2) {
      c1[FR_C + t - FAR_P] = r1[FR_C + t - FAR_P];
    }
    if (t < FAR_ND) {
      double s = 0.0;
      for (int w = 0; w < nsl; ++w) s += r1[(int64_t)w * FAR_REC + FR_ABS + t];
      c1[FR_ABS + t] = s;
    }
    F.lev += 1;
  }
  __syncthreads();
  return F;
}

// The exterior eigenvalue (k = 1) lies outside its block's interval: its sums
// over the poles outside the near window are taken directly, the block's
// threads along the poles.  All threads call it; every thread receives the
// totals.  COMP: v[0], v[1] are Neumaier partials, combined with TwoSum.  red: 5
// doubles per wave.
template <bool COMP>
__device__ __forceinline__ void ext_total(double (&v)[5], int W, int wv, int lane, double* red) {
  auto add = [](double (&a)[5], const double (&b)[5]) {
    if (COMP) {
      const dd t = two_sum(a[0], b[0]);
      a[0] = t.hi;
      a[1] = a[1] + b[1] + t.lo;
    } else {
      a[0] += b[0];
      a[1] += b[1];
    }
    a[2] += b[2];
    a[3] += b[3];
    a[4] += b[4];
  };
  for (int o = 32; o > 0; o >>= 1) {
    double x[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) x[q] = __shfl_xor(v[q], o);
    add(v, x);
  }
  __syncthreads();
  if (lane == 0)
    for (int q = 0; q < 5; ++q) red[5 * wv + q] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 5; ++q) v[q] = red[q];
  for (int w = 1; w < W; ++w) {
    double x[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) x[q] = red[5 * w + q];
    add(v, x);
  }
}
// f, f', f''/2 of the far poles at sigma + tau
__device__ __forceinline__ void ext_eval(const double* P, int n, const Far& F, double sigma, double tau, double (&v)[5],
                                         int W, int wv, int lane, double* red) {
  for (int q = 0; q < 5; ++q) v[q] = 0.0;
  const int len = F.na + (n - F.nb);
#pragma unroll 4
  for (int e = threadIdx.x; e < len; e += blockDim.x) {
    const int j = e < F.na ? e : e - F.na + F.nb;
    const double den = (P[2 * j] - sigma) - tau, z2 = P[2 * j + 1];
    const double r = rcp_1nr(den);
    double t = z2 * r;
    t = __builtin_fma(__builtin_fma(-t, den, z2), r, t);
    v[0] += t;
    v[1] += t * r;
    v[2] = __builtin_fma(t * r, r, v[2]);
  }
  ext_total<false>(v, W, wv, lane, red);
}
// the sums of a root-finder pass over the far poles at nu = m (s = 1):
// sum zeta^2/(delta pp) (Neumaier sum in v[0], v[1]), and those of
// zeta^2/pp^2, zeta^2 delta/pp^3, zeta^2 delta^2/pp^4
__device__ __forceinline__ void ext_sums(const double* P, int n, const Far& F, double sigma, double m, double (&v)[5],
                                         int W, int wv, int lane, double* red) {
  for (int q = 0; q < 5; ++q) v[q] = 0.0;
  const int len = F.na + (n - F.nb);
#pragma unroll 4
  for (int e = threadIdx.x; e < len; e += blockDim.x) {
    const int j = e < F.na ? e : e - F.na + F.nb;
    const double dl = P[2 * j] - sigma, z2 = P[2 * j + 1];
    const double pp = __builtin_fma(m, dl, -1.0);
    const double q = fmin(dl * pp, DBL_MAX);
    const double r = rcp_1nr(q);
    double t = z2 * r;
    t = __builtin_fma(__builtin_fma(-t, q, z2), r, t);
    const double u = (dl * r) * dl;
    const double tp = t * u, tp3 = tp * u;
    const double hi = fmax(v[0], t), lo = fmin(v[0], t);
    const double y = hi + lo;
    v[1] += (hi - y) + lo;
    v[0] = y;
    v[2] += tp;
    v[3] += tp3;
    v[4] = __builtin_fma(tp3, u, v[4]);
  }
  ext_total<true>(v, W, wv, lane, red);
}

// One block of 64 eigenvalues (k0 .. k0+63) of problem p, W waves.  r0, r1: the
// far-field records of the block's own level and of the wide level (nsl
// slices), or nullptr; cf: LDS for two records, er: 5 doubles per wave.
__device__ __forceinline__ void eig_block(const KArgs& A, int p, int k0, double* red, const double* r0, const double* r1, int nsl,
                          double* cf, double* er) {
  const int W = A.W;
  const int wv = wave_id();
  const int lane = lane_id();
  const Meta M = A.meta[p];
  if (M.info != 0) {
    // rejected problem: defined outputs (NaN values, in-range shift indices)
    if (wv == 0 && k0 + lane < M.n) {
      const int64_t b = M.off + k0 + lane;
      A.lam_out[b] = NAN;
      if (A.idx_out) A.idx_out[b] = k0 + lane;
      if (A.mu_out) A.mu_out[b] = NAN;
      if (A.xn_out) A.xn_out[b] = NAN;
    }
    return;
  }
  const int n = M.n;
  const int64_t off = M.off;
  const double* P = A.pairs + 2 * off;
  const double* Zl = A.z2lo + off;
  const double* Dv = A.sd + off;
  const double* Zv = A.sz + off;
  const double rho = M.rho;
  const int k = k0 + lane;
  const bool valid = k < n;
  const int kk = valid ? k : n - 1;

  if (n == 1) {
    // 1x1: lambda = d_1 + rho zeta_1^2, x = zeta_1/(d_1 - lambda)
    if (wv == 0 && lane == 0) {
      double z0 = Zv[0];
      double m = rho * (z0 * z0);
      A.ii[off] = 0;
      A.vflag[off] = 0;
      A.mu[off] = m;
      A.xs[off] = fabs(z0);
      A.lam[off] = Dv[0] + m;
      A.csig[off] = Dv[0];
      A.cinv[off] = fabs(m) / fabs(z0);
      put_outputs(A, M, p, 0, 0, Dv[0] + m, m, fabs(z0), true);
    }
    return;
  }

  // the near window, the wave's slice of it and the range of possible shift
  // indices; poles outside the window enter through the expansions
  const Far FF = far_load(r0, r1, nsl, n, cf);
  const int chunk = (FF.nb - FF.na + W - 1) / W;
  const int j0 = min(FF.nb, FF.na + wv * chunk);
  const int j1 = min(FF.nb, j0 + chunk);
  const int wlo = max(0, k0 - 1);
  const int whi = min(n, k0 + WAVE);
  const bool ext = FF.lev > 0 && k0 == 0;  // this block holds the exterior eigenvalue

  const double dk = Dv[kk];
  const double dkm1 = kk > 0 ? Dv[kk - 1] : 0.0;

  // bracket of the exterior root (k = 1): d_1 + rho zeta_1^2 <= lambda_1 <=
  // d_1 + rho ||z||^2, in nu = 1/(lambda_1 - d_1)
  double Lx = 0.0, Ux = 0.0, nux = 0.0;
  if (kk == 0) {
    const double z0 = Zv[0];
    Lx = (1.0 / (rho * M.zz)) / GROW;
    Ux = (1.0 / (rho * (z0 * z0))) * GROW;
    nux = A.root ? Ux : fmid(Lx, Ux);
  }

  // ---- shift (Alg. 1): F = 1 + rho sum zeta_j^2/((d_j - d_k) - tau)
  // The same pass also sums |terms| and terms/den (f' at the midpoint): the
  // midpoint is the first probe of the root finder, so its evaluation is reused.
  // For k = 1 there is no shift to choose; the pass evaluates f at the first
  // point of the root search instead, lambda = d_1 + 1/nux.
  const double tau = kk > 0 ? (dkm1 - dk) / 2 : 1.0 / nux;
  // Only the sign of F and a first model step are taken from these sums, so
  // the reciprocal is the hardware estimate alone (relative error below
  // 2^-23): the bounds taken from the probe allow for it.
  // The terms are positive for j < k (pole above the midpoint) and negative
  // for j >= k, so their sum and the sum of their magnitudes come from the
  // two one-signed partial sums Fs[0] (j < k) and Fs[1] (j >= k); below the
  // window every lane has j < k, above it j > k.
  double Fs[4] = {0.0, 0.0, 0.0, 0.0};
  sweep(P, j0, j1, wlo, whi, [&](int j, int seg, double dj, double z2, double, int) {
    double r = __builtin_amdgcn_rcp((dj - dk) - tau);
    double t = z2 * r;
    double tr = t * r;
    if (seg == 0) {
      Fs[0] += t;
    } else if (seg == 2) {
      Fs[1] += t;
    } else {
      const bool up = j < kk;
      Fs[0] += up ? t : 0.0;
      Fs[1] += up ? 0.0 : t;
    }
    Fs[2] += tr;
    Fs[3] = __builtin_fma(tr, r, Fs[3]);
  });
  double Ff = 0.0;  // the far poles' part of the sum
  for (int l = wv; l < FF.lev; l += W) {  // (one wave per level where there are two)
    const double* q = FF.cf + l * FAR_REC;
    const double ir = q[FR_IR], x = kk > 0 ? ((dk - q[FR_C]) + tau) * ir : 0.0;
    double f, f1, f2, fa;
    far_eval(q, x, f, f1, f2, fa);
    if (kk > 0) {
      Ff += f;
      Fs[0] += 0.5 * (f + fa);
      Fs[1] += 0.5 * (f - fa);
      Fs[2] = __builtin_fma(f1, ir, Fs[2]);
      Fs[3] = __builtin_fma(f2 * ir, ir, Fs[3]);
    }
  }
  wg_sum<4>(Fs, W, wv, lane, red);
  if (ext) {
    double v[5];
    ext_eval(P, n, FF, lane_value(dk, 0), lane_value(tau, 0), v, W, wv, lane, er);
    if (lane == 0) {  // every far pole lies below: negative terms
      Fs[1] += v[0];
      Fs[2] += v[1];
      Fs[3] += v[2];
    }
  }
  {
    const double sp = Fs[0], sn = Fs[1];
    Fs[0] = sp + sn;  // sum of the terms
    Fs[1] = sp - sn;  // sum of their magnitudes
  }
  double F = 1.0 + rho * Fs[0];
  // The estimated reciprocals leave the sign of F open when |F| is within
  // their error (2^-23 of the sum of |terms|, taken with a margin of 8): such
  // lanes repeat the test with corrected quotients, so that the shift pole
  // differs from a serial IEEE evaluation only where F is zero to rounding
  // (the eigenvalue at the midpoint of its gap: either pole is then nearest).
  // Every wave of the block holds the same per-lane state, so all take the
  // branch together.
  const bool open = valid && kk > 0 && fabs(F) <= 0x1p-20 * (1.0 + rho * Fs[1]);
  if (wave_any(open)) {
    double Fr[1] = {0.0};
    sweep(P, j0, j1, wlo, whi, [&](int, int, double dj, double z2, double, int) {
      const double den = (dj - dk) - tau;
      const double r = rcp_1nr(den);
      double t = z2 * r;
      t = __builtin_fma(__builtin_fma(-t, den, z2), r, t);
      Fr[0] += t;
    });
    Fr[0] += Ff;
    wg_sum<1>(Fr, W, wv, lane, red);
    if (open) F = 1.0 + rho * Fr[0];
  }
  const bool right = (kk == 0) || (F > 0);
  const int i = right ? kk : kk - 1;
  const double s = right ? 1.0 : -1.0;
  const double sigma = right ? dk : dkm1;
  const double zi = Zv[i];
  const double zi2 = zi * zi;

  // ---- tip b of A_i^{-1} (eq. b_ob) in double-double, plus the binary64 sums
  // of eq. (knu2).  P collects j < i (delta > 0), N collects j > i.
  // Each term zeta_j^2/(d_j - sigma) is formed as q1 + q2 from the exact
  // difference (TwoSum), the exact square (hi + lo) and one residual
  // correction, relative error about 2^-100.  P and N each add terms of one
  // sign (N adds the negated terms), so max/min by value orders the operands
  // by magnitude: each sum is a Neumaier compensated sum of the q1 whose
  // compensation also collects the q2.  Its error is O(n eps^2) of the sum,
  // as for a double-double accumulation, at 7 operations a term instead of 11.
  double ps = 0.0, pc = 0.0, ns = 0.0, nc = 0.0;
  auto acc = [](double& a, double& c, double q1, double q2) {
    const double hi = fmax(a, q1), lo = fmin(a, q1);
    const double y = hi + lo;
    c += ((hi - y) + lo) + q2;
    a = y;
  };
  sweep_lo(P, Zl, j0, j1, wlo, whi, [&](int j, int seg, double dj, double z2, double z2l, int) {
    dd dl = two_sum(dj, -sigma);  // exact d_j - sigma
    double r = rcp_1nr(dl.hi);
    double q1 = z2 * r;
    double e = __builtin_fma(-q1, dl.hi, z2);
    e = __builtin_fma(-q1, dl.lo, e + z2l);
    double q2 = e * r;
    if (seg == 0) {
      acc(ps, pc, q1, q2);
    } else if (seg == 2) {
      acc(ns, nc, -q1, -q2);
    } else {
      // selects, no branch: the shift pole's own term (not finite) adds 0
      const bool up = j < i;
      if (j == i) q1 = q2 = 0.0;
      double a = up ? ps : ns, c = up ? pc : nc;
      acc(a, c, up ? q1 : -q1, up ? q2 : -q2);
      ps = up ? a : ps;
      pc = up ? c : pc;
      ns = up ? ns : a;
      nc = up ? nc : c;
    }
  });
  dd Pd = fast_two_sum(ps, pc);
  dd Nd = fast_two_sum(-ns, -nc);
  // the far poles' f = P + N in double-double, cut with the sum of magnitudes
  // P - N so that P and N keep their meaning in K_b (the split is exact: P
  // rounded, N the rest)
  for (int l = wv; l < FF.lev; l += W) {
    const double* q = FF.cf + l * FAR_REC;
    double fa;
    const dd f = far_value(q, dd_mul_d(two_sum(sigma, -q[FR_C]), q[FR_IR]), fa);
    const double pf = 0.5 * (f.hi + fa);
    dd nf = two_sum(f.hi, -pf);
    nf.lo += f.lo;
    Pd = dd_add_same(Pd, dd{pf, 0.0});
    Nd = dd_add_same(Nd, nf);
  }
  wg_sum_dd(Pd, W, wv, lane, red);
  wg_sum_dd(Nd, W, wv, lane, red);
  const dd rr = dd_div(dd{1.0, 0.0}, dd{rho, 0.0});
  const dd num = dd_add(dd_add_same(rr, Pd), Nd);
  const dd bdd = dd_div_sq(num, zi);
  const double Pr = rho * Pd.hi, Nr = rho * Nd.hi;
  const double Kb64 = (1.0 + Pr - Nr) / fabs(1.0 + Pr + Nr);
  bool use_ext = A.mode_b == 0 || (A.mode_b == 1 && Kb64 > 100.0);
  if (A.mode_b == 3) {
    // Algorithm 1's gate: the bound of eq. (knu2) from the standard-precision
    // K_b above 100 (n+4) sqrt(n) (K_b > 100 unless K_z shows that b cannot
    // influence ||A_i^{-1}||)
    const double sn = sqrt((double)n), azi = fabs(zi);
    const double Kz = (M.zabs - azi) / azi;
    const double k1 = (n + 4) * sn * Kb64, k2 = 3.0 * sn + (n + 4) * (1.0 + 2.0 * Kz);
    use_ext = fmin(k1, k2) > 100.0 * (n + 4) * sn;
  }
  const double rzi = 1.0 / zi;
  const double b64 = ((1.0 / rho + Pd.hi) + Nd.hi) * (rzi * rzi);
  const double bh = use_ext ? bdd.hi : b64;
  const double bl = use_ext ? bdd.lo : 0.0;
  const double bp = s * bh;  // b' of the mirrored (rightmost) problem

  // ---- extreme root nu' > 0 of g(nu') = b' - nu' + S(nu')/zeta_i^2,
  // S(nu') = sum_{j!=i} zeta_j^2/(delta'_j (nu' delta'_j - 1)), delta' = s (d_j - sigma).
  const double nss = -s * sigma;
  const bool interior = kk > 0;
  const double xm = interior ? 1.0 / (dkm1 - dk) : 0.0;  // pole nearest to the root
  // the square root of its weight zeta_jm^2/(delta'_jm^2 zeta_i^2), jm the
  // other end of the gap
  const double zjm = interior ? Zv[right ? kk - 1 : kk] : 0.0;
  const double sw = interior ? fabs(zjm * xm) / fabs(zi) : 0.0;
  double L, U, nu;
  if (interior) {
    L = xm;
    U = INFINITY;
    nu = 2.0 * xm;  // mu at the midpoint of the gap: the nearest-pole bound
  } else {
    L = Lx;
    U = Ux;
    nu = nux;
  }
  // the rigorous bracket [L0, U0] (set below) is kept for the double-double
  // polish: the signs of g seen by the binary64 iteration can be wrong when g
  // is badly conditioned
  bool done = !valid;
  int iters = 0;
  double nu0 = nu, prevstep = INFINITY, g1 = 0.0, g2 = 0.0;
  const double rz2 = 1.0 / zi2;

  // First probe from the shift pass: g(nu') = f(lambda)/(rho zeta_i^2) up to
  // the sign s (eqs. secAi, Pick).  For an interior root lambda is the gap
  // midpoint, so g >= 0 there by the choice of the shift; b' + S/zeta_i^2 =
  // g + nu' is then an upper bound of the root (S decreases).  If rounding
  // leaves the sign of g open the pole is kept as the lower end.  For k = 1
  // the probe may lie on either side of the root.
  bool pre = valid;
  double pre_Spz = 0.0, pre_Sppz = 0.0, pre_g = 0.0;
  if (pre) {
    // error of f(lambda) from the estimated reciprocals: 2^-23 of |terms|,
    // taken with a margin of 8
    const double gerr = 0x1p-20 * (1.0 + rho * Fs[1]) / (rho * zi2);
    pre_g = s * (1.0 + rho * Fs[0]) / (rho * zi2);
    // g' = -F2/(zeta_i^2 nu^2) and g'' = 2 (s F3/nu^4 + F2/nu^3)/zeta_i^2 with
    // F2, F3 the sums of zeta_j^2/(d_j - lambda)^2 and ^3 (lambda = sigma + s/nu)
    const double inu = 1.0 / nu;
    pre_Spz = fmax(Fs[2] / (zi2 * nu * nu) - 1.0, 0.0);
    pre_Sppz = (((s * Fs[3]) * inu + Fs[2]) * (inu * inu * inu)) / zi2;
    if (interior) {
      U = (nu + fmax(pre_g, 0.0) + gerr) * GROW;
      if (pre_g > gerr) L = nu;
    } else if (pre_g > gerr) {
      L = nu;
      U = fmin(U, (nu + pre_g + gerr) * GROW);
    } else if (pre_g < -gerr) {
      U = nu;
    }
  }
  const double L0 = L, U0 = U;

  // The far poles' part of a pass at nu = m, one wave per level (the other
  // waves add 0): with mu = s/m, zeta^2/(delta' pp) = |mu| zeta^2/((d - sigma)(d - lambda)),
  // a divided difference of f, and zeta^2/pp^2, zeta^2 delta'/pp^3, zeta^2
  // delta'^2/pp^4 are its derivatives at lambda times powers of |mu|.  The
  // exterior eigenvalue takes its direct sums instead.  `last`: the accurate
  // pass, where the first sum comes in double-double (its low part in v0l),
  // as the near poles' does, and the slopes from more orders, each a wave's
  // job.
  auto far_sums = [&](double m, double (&v)[4], double& v0l, auto last) {
    constexpr bool LAST = decltype(last)::value;
    v[0] = v[1] = v[2] = v[3] = v0l = 0.0;
    const int jobs = LAST ? 2 * FF.lev : FF.lev;
    if (wv < jobs) {
      const dd ad = LAST ? dd_div(dd{1.0, 0.0}, dd{m, 0.0}) : dd{fabs(s / m), 0.0};
      const double am = ad.hi, muv = s * am;
      for (int l = wv; l < jobs; l += W) {
        const bool pair = LAST && l >= FF.lev;
        const double* q = FF.cf + (pair ? l - FF.lev : l) * FAR_REC;
        const double ir = q[FR_IR];
        if (pair) {
          const dd X = dd_mul_d(two_sum(sigma, -q[FR_C]), ir), md = dd_mul_d(ad, ir);
          const dd Y = interior ? dd_add(X, dd{s * md.hi, s * md.lo}) : X;
          const dd t = dd_add_same(dd{v[0], v0l}, dd_mul(far_pair(q, X, Y), md));
          v[0] = t.hi;
          v0l = t.lo;
          continue;
        }
        const double x = (sigma - q[FR_C]) * ir;
        const double y = interior ? __builtin_fma(muv, ir, x) : x;
        const double mi = am * ir, ms = muv * ir;  // in units of the half-width
        double fxy, f1, f2, f3;
        far_diff<LAST ? FAR_NA : FAR_ND>(q, x, y, fxy, f1, f2, f3);
        if (!LAST) v[0] = __builtin_fma(fxy, mi, v[0]);
        v[1] = __builtin_fma(f1 * am, mi, v[1]);
        v[2] = __builtin_fma(__builtin_fma(ms, f2, f1) * am, am * mi, v[2]);
        v[3] = __builtin_fma(__builtin_fma(ms, __builtin_fma(ms, f3, 2.0 * f2), f1) * am, am * (am * mi), v[3]);
      }
    }
    if (ext) {
      double e[5];
      ext_sums(P, n, FF, lane_value(sigma, 0), lane_value(m, 0), e, W, wv, lane, er);
      if (lane == 0) {
        const bool first = wv == 0;
        v[0] = first ? e[0] : 0.0;
        v0l = first ? e[1] : 0.0;
        v[1] = first ? e[2] : 0.0;
        v[2] = first ? e[3] : 0.0;
        v[3] = first ? e[4] : 0.0;
      }
    }
  };

  if (A.root == 0) {
    // -------- bisection in the order of the binary64 numbers
    while (wave_any(!done)) {
      double m = nu;
      double S[1] = {0.0};
      if (wave_any(!done && !pre)) {
        sweep(P, j0, j1, wlo, whi, [&](int j, int seg, double dj, double z2, double, int) {
          double dl = __builtin_fma(s, dj, nss);
          double pp = __builtin_fma(m, dl, -1.0);
          double t = z2 * rcp_1nr(dl * pp);
          if (seg == 1 && j == i) t = 0.0;
          S[0] += t;
        });
        double fs[4], fl;
        far_sums(m, fs, fl, Bool<false>{});
        S[0] += fs[0] + fl;
        wg_sum<1>(S, W, wv, lane, red);
        ++iters;
      }
      if (!done) {
        double Sz = S[0] * rz2;
        double g = (bp - m) + Sz;
        if (pre) {
          g = pre_g;
          pre = false;  // bracket already set from the probe
        } else {
          if (g > 0) L = m; else U = m;
        }
        if (adjacent(L, U) || iters >= 200) {
          done = true;
          nu0 = U;
        } else {
          nu = fmid(L, U);
        }
      }
    }
  } else {
    // -------- safeguarded model iteration: every pass gives the value, slope
    // and curvature of the sum term at nu; the root of the model built from
    // them (the nearest pole exact, the rest one fitted pole) is the next
    // iterate.  The last pass of the budget is the accurate one below.
    // The step from the probe costs no pass and is always taken.
    const int budget = max(A.main_passes, 1);
    int passes = 0;
    while (wave_any(!done) && (passes < budget - 1 || wave_any(pre))) {
      double m = nu;
      double S[3] = {0.0, 0.0, 0.0};
      if (wave_any(!done && !pre)) {
        sweep(P, j0, j1, wlo, whi, [&](int j, int seg, double dj, double z2, double, int) {
          double dl = __builtin_fma(s, dj, nss);
          double pp = __builtin_fma(m, dl, -1.0);
          double rq = __builtin_amdgcn_rcp(dl * pp);
          double t = z2 * rq;           // w_j/(m - xi_j)
          double u = (dl * rq) * dl;    // delta'_j/pp = 1/(m - xi_j)
          double tp = t * u;            // w_j/(m - xi_j)^2
          if (seg == 1 && j == i) {     // (dl = 0 there: u is NaN)
            t = 0.0;
            tp = 0.0;
            u = 0.0;
          }
          S[0] += t;
          S[1] += tp;
          S[2] = __builtin_fma(tp, u, S[2]);  // w_j/(m - xi_j)^3
        });
        double fs[4], fl;
        far_sums(m, fs, fl, Bool<false>{});
        S[0] += fs[0] + fl;
        S[1] += fs[1];
        S[2] += fs[2];
        wg_sum<3>(S, W, wv, lane, red);
        ++iters;
        ++passes;
      }
      if (!done) {
        double Sz = S[0] * rz2;
        double Spz = S[1] * rz2;  // -dS/dnu / zeta_i^2
        double Sppz = S[2] * rz2;
        double g = (bp - m) + Sz;
        if (pre) {
          Spz = pre_Spz;
          Sppz = pre_Sppz;
          g = pre_g;
          pre = false;  // bracket already set from the probe
        } else {
          // the terms of a plain pass carry the error of the estimated
          // reciprocal (below 2^-23, all terms positive): a sign of g within
          // that error leaves the bracket as it is
          const double gtol = 0x1p-20 * Sz + 0x1p-50 * fabs(bp);
          if (g > gtol) L = m; else if (g < -gtol) U = m;
        }
        model_step(m, g, Spz, Sppz, xm, sw, iters, L, U, nu, nu0, prevstep, g1, g2, done);
      }
    }
  }

  // ---- accurate pass at m: compensated sum of the secular terms (each a
  // corrected quotient), the moments for the last step, the amplification
  // estimate kappa_g = (|b| + |nu| + S)/(|nu| |g'|) and ||x||.  After
  // bisection m is the converged bracket end and the last step is Newton's;
  // in the model iteration m is the converged iterate (or the next one for a
  // lane that has not converged) and the last step is the model's, which is
  // accepted when it is below 2^-20 relative.  Right of every pole all terms
  // are positive: the eight terms of a block are added as a tree of depth 3
  // (error at most 3 eps of the block sum), and the block sums go into a
  // Neumaier sum, which takes the larger operand first by value.
  const double m = (A.root == 0 || done) ? nu0 : nu;
  double cs = 0.0, cc = 0.0;
  double Sp[3] = {0.0, 0.0, 0.0};
  double ga = 0.0, gb = 0.0, gc = 0.0;
  auto neu = [&](double t) {
    const double hi = fmax(cs, t), lo = fmin(cs, t);
    const double y = hi + lo;
    cc += (hi - y) + lo;
    cs = y;
  };
  sweep(P, j0, j1, wlo, whi, [&](int j, int seg, double dj, double z2, double, int ub) {
    double dl = __builtin_fma(s, dj, nss);
    double pp = __builtin_fma(m, dl, -1.0);
    // q > 0; beyond binary64 (a far pole with nu near 1e300) it is held at the
    // largest finite number, where the quotient is 0 to working precision and
    // the correction below stays finite (0 * inf would be NaN)
    double q = fmin(dl * pp, DBL_MAX);
    double r = rcp_1nr(q);
    double t = z2 * r;
    t = __builtin_fma(__builtin_fma(-t, q, z2), r, t);  // corrected quotient
    double u = (dl * r) * dl;                           // 1/(m - xi_j)
    double tp = t * u;                                  // zeta_j^2/pp^2
    double tp3 = tp * u;                                // zeta_j^2 delta'_j/pp^3
    if (seg == 1 && j == i) {                           // (dl = 0 there: u is NaN)
      t = 0.0;
      tp = 0.0;
      tp3 = 0.0;
      u = 0.0;
    }
    switch (ub) {
      case 0: ga = t; break;
      case 1: ga += t; break;
      case 2: gb = t; break;
      case 3: gb += t; ga += gb; break;
      case 4: gb = t; break;
      case 5: gb += t; break;
      case 6: gc = t; break;
      case 7: gc += t; gb += gc; ga += gb; neu(ga); break;
      default: neu(t);
    }
    Sp[0] += tp;
    Sp[1] += tp3;
    Sp[2] = __builtin_fma(tp3, u, Sp[2]);               // zeta_j^2 delta'_j^2/pp^4
  });
  {
    double fs[4], fl;
    far_sums(m, fs, fl, Bool<true>{});
    neu(fs[0]);
    cc += fl;
    Sp[0] += fs[1];
    Sp[1] += fs[2];
    Sp[2] += fs[3];
  }
  wg_sum_comp(cs, cc, W, wv, lane, red);
  wg_sum<3>(Sp, W, wv, lane, red);
  double Sz;
  const double g = g_value(bp, s * bl, m, cs, cc, zi, Sz);
  const double gp = -1.0 - Sp[0] / zi2;
  // divided in two steps: m |g'| overflows when nu nears 1e304
  const double kap = ((fabs(bp) + m + Sz) / m) / fabs(gp);
  double nu1 = m;
  bool fin = true;
  if (A.root == 0) {
    nu1 = m - g / gp;
  } else if (valid) {
    fin = false;
    if (g > 0) L = m; else if (g < 0) U = m;
    double nn = m;
    model_step(m, g, Sp[0] / zi2, Sp[1] / zi2, xm, sw, iters, L, U, nu, nn, prevstep, g1, g2, fin);
    if (fin) nu1 = nn;
  }
  const bool cont = valid && !fin;  // unfinished: continued in k_fix
  double muv = s / nu1;
  double lam = sigma + muv;
  double amp = fabs(muv / lam);
  if (!(amp > 1.0)) amp = 1.0;
  const bool pol = valid && !cont && A.polish && (kap * amp > A.kappa_polish);
  bool nz = false;
  if (valid && !cont && !pol && A.nearzero > 0) {
    double gap = fabs(lam - dk);
    if (kk > 0) gap = fmin(gap, fabs(lam - dkm1));
    nz = A.nearzero * fabs(lam) < gap;
  }

  // ---- ||x|| scaled by |mu|: with delta_j - mu = s (delta'_j - 1/nu) one has
  // mu/(delta_j - mu) = 1/(nu delta'_j - 1), so |mu|^2 ||x||^2 =
  // zeta_i^2 + sum_{j != i} zeta_j^2/pp_j^2, the S' sum of the accurate pass.
  // That sum is taken at m and carried to nu1 = m + h by its Taylor series to
  // second order (derivatives -2 sum zeta^2 delta'/pp^3 and 6 sum zeta^2
  // delta'^2/pp^4; |h|/(m - xi_j) <= 2^-19, so the error is below 2^-55).
  // The products are formed as h (h S) so that an h near 1e300 (nu = 1/mu
  // for a mu near 1e-300, beside a zeta_i near 1e-150) meets the underflowed
  // sums before it is squared: h h would overflow and inf * 0 be NaN.
  const double h = nu1 - m;
  double Nx[1] = {zi2 + ((Sp[0] - 2.0 * (h * Sp[1])) + 3.0 * (h * (h * Sp[2])))};
  if (wv == 0 && valid) {
    A.ii[off + k] = i;
    A.vflag[off + k] = (pol || nz || cont) ? 1 : 0;
    A.mu[off + k] = muv;
    // a tip b' beyond binary64 (zeta_i near 1e-150 beside a pole 1e-13 away
    // with an O(1) zeta) leaves g undefined: the NaN norm makes the output
    // check report DPR1_INFO_RANGE instead of a wrong vector
    const double xs = fabs(bp) < INFINITY ? sqrt(Nx[0]) : NAN;
    A.xs[off + k] = xs;
    A.lam[off + k] = lam;
    // per-column constants of the eigenvector writer: sigma_k and
    // w_k = 1/||x_k|| = |mu|/(|mu| ||x||), so that v_j = zeta_j (w_k/(delta_j -
    // mu)).  The quotient w/(delta_j - mu) = v_j/zeta_j is at most 1/|zeta_j|
    // and underflows only where v_j/zeta_j does; mu/(delta_j - mu) alone would
    // be subnormal beside a distant pole when mu is tiny (1e-304 against
    // delta_j = 1e10) and lose bits although v_j is a normal number
    A.csig[off + k] = sigma;
    A.cinv[off + k] = fabs(muv) / xs;
    // flagged pairs are finished, checked and written by k_fix
    if (!(pol || nz || cont)) put_outputs(A, M, p, k, i, lam, muv, xs, true);
    if (pol || nz || cont) {
      // the long items (polish, near-zero recomputation) fill the list from
      // the front, roots only continued fill it from the back, so that the
      // queue of k_fix hands out the long ones first
      const bool longer = pol || nz;
      int e = longer ? atomicAdd(&A.ctr[0], 1) : A.nfixcap - 1 - atomicAdd(&A.ctr[3], 1);
      FixItem it;
      it.p = p;
      it.k = k;
      it.i = i;
      it.flags = (pol ? FIX_POLISH : 0) | (nz ? FIX_NEARZERO : 0) | (cont ? FIX_CONTINUE : 0);
      it.iters = iters;
      it.pad = 0;
      it.nu0 = m;
      it.nu1 = nu1;
      it.bhi = bp;
      it.blo = s * bl;
      it.lo = L0;
      it.hi = U0;
      it.cnu = nu;
      it.cL = L;
      it.cU = U;
      it.cprev = prevstep;
      A.fix[e] = it;
    }
  }
  if (A.stats && wv == 0) {
    bool kb = valid && Kb64 > 100.0;
    unsigned long long bal = __ballot(kb);
    const unsigned long long bext = __ballot(valid && use_ext);
    int itv = valid ? iters : 0;
    int imax = itv, isum = itv;
    for (int o = 32; o > 0; o >>= 1) {
      imax = max(imax, __shfl_xor(imax, o));
      isum += __shfl_xor(isum, o);
    }
    if (lane == 0) {
      if (bal) atomicAdd(&A.stats[DPR1_STAT_KB_GT_100], __popcll(bal));
      if (bext) atomicAdd(&A.stats[DPR1_STAT_EXT_B], __popcll(bext));
      atomicMax(&A.stats[DPR1_STAT_ITERS_MAX], imax);
      atomicAdd(&A.stats[DPR1_STAT_ITERS_SUM], isum);
    }
  }
}

// OCC: waves per SIMD the register allocation is made for (4: up to 128
// VGPRs; 6: 80; 8: 64, the outer state then partly in scratch, the inner
// sweeps unchanged), so that more waves can hide the FP64 latencies.
template <int OCC>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(OCC, OCC))) k_eig(KArgs A) {
  extern __shared__ double red[];
  __shared__ double cf[2 * FAR_REC], er[5 * MAXW];
  // one problem: block b solves group g0 + b; a batch: persistent blocks take
  // (problem, first eigenvalue) items from the queue
  __shared__ int item;
  const bool one = A.items == nullptr;
  for (;;) {
    int p = 0, k0, nsl = A.far_slices;
    const double *r0 = nullptr, *r1 = nullptr;
    if (one) {
      const int g = A.g0 + (int)blockIdx.x;
      k0 = g * WAVE;
      if (A.far) r0 = A.far + (int64_t)g * FAR_REC;
      if (A.far_wide) r1 = A.far + (A.far_wide + (int64_t)(g / FAR_WIDE) * nsl) * FAR_REC;
    } else {
      if (threadIdx.x == 0) item = atomicAdd(&A.ctr[1], 1);
      __syncthreads();
      const int it = __builtin_amdgcn_readfirstlane(item);
      __syncthreads();
      if (it >= A.nitems) break;
      const int4 pk = A.items[it];
      p = pk.x;
      k0 = pk.y;
      nsl = pk.w;
      if (A.far && A.meta[p].n >= A.far_min) {
        r0 = A.far + (int64_t)it * FAR_REC;
        if (pk.z >= 0) r1 = A.far + (int64_t)pk.z * FAR_REC;
      }
    }
    eig_block(A, p, k0, red, r0, r1, nsl, cf, er);
    if (one) break;
  }
}

// ------------------------------------------------------------------- fix
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ double wave_min(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ dd wave_sum_same(dd a) {
  for (int o = 32; o > 0; o >>= 1) {
    dd b = {__shfl_xor(a.hi, o), __shfl_xor(a.lo, o)};
    a = dd_add_same(a, b);
  }
  return a;
}
__device__ __forceinline__ dd wave_sum_dd(dd a) {
  for (int o = 32; o > 0; o >>= 1) {
    dd b = {__shfl_xor(a.hi, o), __shfl_xor(a.lo, o)};
    a = dd_add(a, b);
  }
  return a;
}

// Block-wide sums over FIXT threads (4 waves) in a fixed order; every thread
// receives the total.
constexpr int FIXT = 256;
__device__ __forceinline__ double block_sum(double v, double* sm) {
  v = wave_sum(v);
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) sm[wv] = v;
  __syncthreads();
  return (sm[0] + sm[1]) + (sm[2] + sm[3]);
}
__device__ __forceinline__ double block_min(double v, double* sm) {
  v = wave_min(v);
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) sm[wv] = v;
  __syncthreads();
  return fmin(fmin(sm[0], sm[1]), fmin(sm[2], sm[3]));
}
__device__ __forceinline__ dd block_sum_same(dd a, double* sm) {
  a = wave_sum_same(a);
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) {
    sm[wv] = a.hi;
    sm[4 + wv] = a.lo;
  }
  __syncthreads();
  dd r = dd_add_same(dd{sm[0], sm[4]}, dd{sm[1], sm[5]});
  r = dd_add_same(r, dd{sm[2], sm[6]});
  return dd_add_same(r, dd{sm[3], sm[7]});
}
__device__ __forceinline__ dd block_sum_dd(dd a, double* sm) {
  a = wave_sum_dd(a);
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) {
    sm[wv] = a.hi;
    sm[4 + wv] = a.lo;
  }
  __syncthreads();
  dd r = dd_add(dd{sm[0], sm[4]}, dd{sm[1], sm[5]});
  r = dd_add(r, dd{sm[2], sm[6]});
  return dd_add(r, dd{sm[3], sm[7]});
}
__device__ __forceinline__ double block_sum_comp(double s, double c, double* sm) {
  // Neumaier partials: wave butterflies, then the four wave results in order
  for (int o = 32; o > 0; o >>= 1) {
    double s2 = __shfl_xor(s, o), c2 = __shfl_xor(c, o);
    dd t = two_sum(s, s2);
    s = t.hi;
    c = c + c2 + t.lo;
  }
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) {
    sm[wv] = s;
    sm[4 + wv] = c;
  }
  __syncthreads();
  double S = sm[0], C = sm[4];
  for (int w = 1; w < 4; ++w) {
    dd t = two_sum(S, sm[w]);
    S = t.hi;
    C += sm[4 + w] + t.lo;
  }
  return S + C;
}

// The four sums of a continued pass in one exchange: the Neumaier partials
// (s, c) combined as in block_sum_comp (returned, its compensation in c) and
// three plain sums a, b, e as in block_sum, with one pair of barriers instead
// of four.  sm holds 20 values.
__device__ __forceinline__ double block_sum_comp3(double s, double& c, double& a, double& b, double& e,
                                                  double* sm) {
  for (int o = 32; o > 0; o >>= 1) {
    const double s2 = __shfl_xor(s, o), c2 = __shfl_xor(c, o);
    const dd t = two_sum(s, s2);
    s = t.hi;
    c = c + c2 + t.lo;
  }
  a = wave_sum(a);
  b = wave_sum(b);
  e = wave_sum(e);
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) {
    sm[wv] = s;
    sm[4 + wv] = c;
    sm[8 + wv] = a;
    sm[12 + wv] = b;
    sm[16 + wv] = e;
  }
  __syncthreads();
  double S = sm[0], C = sm[4];
  for (int w = 1; w < 4; ++w) {
    dd t = two_sum(S, sm[w]);
    S = t.hi;
    C += sm[4 + w] + t.lo;
  }
  a = (sm[8] + sm[9]) + (sm[10] + sm[11]);
  b = (sm[12] + sm[13]) + (sm[14] + sm[15]);
  e = (sm[16] + sm[17]) + (sm[18] + sm[19]);
  c = C;
  return S;
}

// The block's threads along the n poles of a problem, in rounds of U per
// thread whose loads (pairs and, with LO, the low parts of zeta_j^2) are all
// issued before the first is used: a block has its CU nearly to itself, so
// one load latency per pole and pass was most of its time.  f(j, d_j,
// zeta_j^2, low part, j < n) for consecutive rounds of FIXT poles; past the end
// it gets the last pole again.
template <int U, bool LO, class F>
__device__ __forceinline__ void fix_poles(const double2* Z2v, const double* Zl, int n, F&& f) {
  for (int b = threadIdx.x; b < n; b += U * FIXT) {
    double2 p[U];
    double l[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(b + u * FIXT, n - 1);
      p[u] = Z2v[j];
      l[u] = LO ? Zl[j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) f(b + u * FIXT, p[u].x, p[u].y, l[u], b + u * FIXT < n);
  }
}

// The sums of a polish step in one exchange: the same-signed double-doubles a
// and the plain sums b, c, in the orders of block_sum_same and block_sum.
__device__ __forceinline__ dd block_sum_polish(dd a, double& b, double& c, double* sm) {
  a = wave_sum_same(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int wv = threadIdx.x / WAVE;
  __syncthreads();
  if (threadIdx.x % WAVE == 0) {
    sm[wv] = a.hi;
    sm[4 + wv] = a.lo;
    sm[8 + wv] = b;
    sm[12 + wv] = c;
  }
  __syncthreads();
  b = (sm[8] + sm[9]) + (sm[10] + sm[11]);
  c = (sm[12] + sm[13]) + (sm[14] + sm[15]);
  dd r = dd_add_same(dd{sm[0], sm[4]}, dd{sm[1], sm[5]});
  r = dd_add_same(r, dd{sm[2], sm[6]});
  return dd_add_same(r, dd{sm[3], sm[7]});
}

// Safeguarded iteration for the extreme root of g (eq. secAi) at the shift
// pole d_i (side s), g evaluated in double-double: far from the root the
// model step of the main solver, close to it Newton (g exact to
// ~2^-100, so the last step lands on the rounded root).  b' = s b in
// double-double, xm the nearest pole of g (in nu) and sw the square root of its
// weight (one pole and a constant, the model used before, took up to 34 steps
// beside poles 1e-10 apart: 180 us for one root), (lo0, hi0) a rigorous
// bracket, cur the start.  Returns the last iterate.  With `confirm` the
// iteration goes on until a step no longer changes it, *last then receives the
// Newton correction at it (nu = cur + *last to about 2^-100); without, a Newton
// step below 2^-36 relative is the last (its own error is below 2^-70) and is
// not followed by an evaluation that only confirms it.  *steps: the number of
// double-double evaluations less one.  All threads of the block call it and
// return the same values.
__device__ double dd_polish(const double2* Z2v, const double* Zl, int n, int i, double s, double sigma, double zi,
                           dd bdd, double xm, double sw, double lo0, double hi0, double cur, bool confirm, double* last,
                           int* steps, double* sm) {
  const double zi2 = zi * zi;
  double lo = lo0, hi = hi0;
  if (!(cur > lo && cur < hi)) cur = fmid(lo, hi);
  // progress guard: when |g| has not halved over two steps away from the
  // final Newton phase, the model is not describing g (a pole one ulp from
  // the shift pole dominates it), and the step is a bisection
  double gprev = INFINITY, newton = 0.0;
  int slow = 0, pit;
  for (pit = 0; pit < 100; ++pit) {
    dd acc = {0.0, 0.0};
    double sp = 0.0, sp3 = 0.0;
    fix_poles<4, true>(Z2v, Zl, n, [&](int j, double dj, double z2, double z2l, bool in) {
      const dd dl = two_sum(s * dj, -s * sigma);               // delta'_j exactly
      const dd pp = dd_add(dd_mul_d(dl, cur), dd{-1.0, 0.0});  // nu delta' - 1
      dd q = dd_mul(dl, pp);
      if (!(q.hi < DBL_MAX)) q = {DBL_MAX, 0.0};  // beyond binary64: the term is 0
      // (zeta_j^2 hi + lo)/q: leading quotient from the refined reciprocal
      // (2^-48.7) and one residual correction, about 2^-97
      const double r = rcp_1nr(q.hi);
      const double q1 = z2 * r;
      double e = __builtin_fma(-q1, q.hi, z2);
      e = __builtin_fma(-q1, q.lo, e + z2l);
      dd t = fast_two_sum(q1, e * r);
      const double rp = rcp_1nr(pp.hi);
      double u = (z2 * rp) * rp, u3 = u * (dl.hi * rp);  // the derivatives only steer the step
      if (j == i || !in) {
        t = {0.0, 0.0};
        u = u3 = 0.0;
      }
      acc = dd_add_same(acc, t);
      sp += u;
      sp3 += u3;
    });
    acc = block_sum_polish(acc, sp, sp3, sm);
    dd Sdd = dd_div_sq(acc, zi);
    dd gd = dd_add(dd_add(bdd, dd{-cur, 0.0}), Sdd);
    double Spz = sp / zi2;
    double gpv = -1.0 - Spz;
    newton = 0.0;
    if (gd.hi == 0.0) break;
    if (gd.hi > 0) lo = cur; else hi = cur;
    const double ag = fabs(gd.hi);
    slow = ag > 0.5 * gprev ? slow + 1 : 0;
    gprev = ag;
    newton = -(gd.hi + gd.lo) / gpv;
    double t;
    bool last_one = !confirm && fabs(newton) <= 0x1p-36 * cur;
    if (fabs(newton) <= 0x1p-30 * cur) {
      t = cur + newton;
    } else {
      t = cur + model_delta(cur, gd.hi, Spz, sp3 / zi2, xm, sw, lo, hi);
    }
    // stay inside the sign bracket and off the pole / rigorous lower end
    if (!(t >= lo && t <= hi) || !(t > lo0) || !(t < INFINITY) || (slow >= 2 && fabs(newton) > 0x1p-30 * cur)) {
      t = fmid(lo, hi);
      slow = 0;
      last_one = false;
    }
    if (t == cur) break;
    cur = t;
    if (last_one) break;
  }
  *last = fabs(newton) <= 0x1p-30 * cur ? newton : 0.0;
  *steps = pit;
  return cur;
}

// The polish of the exterior eigenvalue (k = 1): mu = lambda_1 - d_1 from
// rho sum zeta_j^2/(mu + (d_1 - d_j)) = 1, whose terms all have one sign, so
// that nothing cancels whatever mu against the poles' spread.  (g cancels by
// mu/spread: in double-double a ratio beyond 1e16 left any point of the bracket,
// up to n times off.)  The reciprocal of the sum is concave in mu and close to linear
// from mu = spread on: Newton's steps on it come from the left after the first, two or
// three in all.  cur: the start; returns mu.
__device__ double ext_polish(const double2* Z2v, const double* Zl, int n, double sigma, double zi2, double zz,
                             double rho, double cur, int* steps, double* sm) {
  double lo = rho * zi2 / GROW, hi = rho * zz * GROW;
  if (!(cur > lo && cur < hi)) cur = fmid(lo, hi);
  int pit;
  for (pit = 0; pit < 100; ++pit) {
    dd acc = {0.0, 0.0};
    double s2 = 0.0, unused = 0.0;
    fix_poles<4, true>(Z2v, Zl, n, [&](int, double dj, double z2, double z2l, bool in) {
      const dd den = dd_add_same(two_sum(sigma, -dj), dd{cur, 0.0});
      const double r = rcp_1nr(den.hi);
      const double q1 = z2 * r;
      double e = __builtin_fma(-q1, den.hi, z2);
      e = __builtin_fma(-q1, den.lo, e + z2l);
      if (!in) return;
      acc = dd_add_same(acc, fast_two_sum(q1, e * r));
      s2 += q1 * r;
    });
    acc = block_sum_polish(acc, s2, unused, sm);
    const dd S = dd_mul_d(acc, rho), h = dd_add(S, dd{-1.0, 0.0});
    if (h.hi == 0.0) break;
    if (h.hi > 0.0) lo = cur; else hi = cur;
    const double step = (S.hi / (rho * s2)) * (h.hi + h.lo);
    double t = cur + step;
    const bool last = fabs(step) <= 0x1p-36 * cur;
    if (!(t >= lo && t <= hi)) {
      if (adjacent(lo, hi)) break;
      t = fmid(lo, hi);
    } else if (last) {
      cur = t;
      break;
    }
    cur = t;
  }
  *steps = pit;
  return cur;
}

// One block of FIXT threads per flagged eigenpair at a time; the inner index
// is strided over the block and every pass ends in a block-wide sum.
// Item e of the list: the n0 long items sit at the front, the others at the
// back in reverse order.
__device__ __forceinline__ int fix_slot(const KArgs& A, int n0, int e) {
  return e < n0 ? e : A.nfixcap - 1 - (e - n0);
}

__device__ void fix_items(const KArgs& A) {
  __shared__ double sm[20];
  __shared__ int next;
  const int tid = threadIdx.x;
  const int n0 = A.ctr[0];
  const int cnt = n0 + A.ctr[3];
  for (bool first = true;; first = false) {
    // items are taken from a queue, long ones first, so a block that drew
    // cheap items takes more of them (polish steps cost several times a
    // continued root's); a block that comes to an empty queue only reads it,
    // since atomics on one address take their turns (512 blocks, 15 us).  One
    // thread looks, for the whole block: others may see later values
    if (tid == 0) {
      const bool empty = first && __hip_atomic_load(&A.ctr[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= cnt;
      next = empty ? cnt : atomicAdd(&A.ctr[2], 1);
    }
    __syncthreads();
    const int e = next;
    __syncthreads();
    if (e >= cnt) break;
    const FixItem it = A.fix[fix_slot(A, n0, e)];
    const Meta M = A.meta[it.p];
    const int n = M.n;
    const int64_t off = M.off;
    const double* Dv = A.sd + off;
    const double* Zv = A.sz + off;
    const double* Z2 = A.pairs + 2 * off;
    const double2* Z2v = reinterpret_cast<const double2*>(Z2);  // (d_j, zeta_j^2), 16-byte aligned
    const double* Zl = A.z2lo + off;
    const double rho = M.rho;
    const int k = it.k, i = it.i;
    const double s = (i == k) ? 1.0 : -1.0;
    const double sigma = Dv[i];
    const double zi = Zv[i];
    const double zi2 = zi * zi;
    double muv = A.mu[off + k];
    double lam = A.lam[off + k];
    bool nz = (it.flags & FIX_NEARZERO) != 0;
    bool pol = (it.flags & FIX_POLISH) != 0;
    bool polished = false;
    int singular = 0;
    int pit = 0;  // double-double steps of the polish
    double nu0 = it.nu0, nu1 = it.nu1;
    double xsv = 0.0;
    bool have_xs = false;

    if (it.flags & FIX_CONTINUE) {
      // the root search continued with block-wide sums; every pass is the
      // accurate one of the eigenvalue kernel (compensated sum, corrected
      // quotients, derivative sums up to the third), so the pass whose model
      // step is accepted also gives kappa_g and ||x||
      const double xm = (k > 0) ? 1.0 / (Dv[k - 1] - Dv[k]) : 0.0;
      const double zjm = (k > 0) ? Zv[i == k ? k - 1 : k] : 0.0;
      const double sw = (k > 0) ? fabs(zjm * xm) / fabs(zi) : 0.0;
      const double bp = it.bhi;
      double nu = it.cnu, L = it.cL, U = it.cU, prevstep = it.cprev, g1 = 0.0, g2 = 0.0;
      int iters = it.iters;
      bool done = false;
      double m = nu, Sz = 0.0, sp = 0.0, sp3 = 0.0, sp4 = 0.0;
      while (!done) {
        m = nu;
        double cs = 0.0, cc = 0.0;
        sp = 0.0;
        sp3 = 0.0;
        sp4 = 0.0;
        fix_poles<8, false>(Z2v, nullptr, n, [&](int j, double dj, double z2, double, bool in) {
          const double dl = __builtin_fma(s, dj, -s * sigma);
          const double pp = __builtin_fma(m, dl, -1.0);
          const double q = fmin(dl * pp, DBL_MAX);  // as in k_eig's accurate pass
          const double r = rcp_1nr(q);
          double t = z2 * r;
          t = __builtin_fma(__builtin_fma(-t, q, z2), r, t);  // corrected quotient
          double u = (dl * r) * dl;                           // 1/(m - xi_j)
          if (j == i || !in) t = u = 0.0;
          const double tp = t * u;
          const double tp3 = tp * u;
          const double hi = fmax(cs, t), lo = fmin(cs, t);    // positive terms
          const double y = hi + lo;
          cc += (hi - y) + lo;
          cs = y;
          sp += tp;
          sp3 += tp3;
          sp4 = __builtin_fma(tp3, u, sp4);
        });
        cs = block_sum_comp3(cs, cc, sp, sp3, sp4, sm);
        ++iters;
        const double g = g_value(bp, it.blo, m, cs, cc, zi, Sz);
        if (g > 0) L = m; else if (g < 0) U = m;
        model_step(m, g, sp / zi2, sp3 / zi2, xm, sw, iters, L, U, nu, nu0, prevstep, g1, g2, done);
      }
      nu1 = nu0;
      const double gp = -1.0 - sp / zi2;
      const double kap = ((fabs(bp) + m + Sz) / m) / fabs(gp);  // as in k_eig
      muv = s / nu1;
      lam = sigma + muv;
      double amp = fabs(muv / lam);
      if (!(amp > 1.0)) amp = 1.0;
      pol = A.polish && (kap * amp > A.kappa_polish);
      if (!pol && A.nearzero > 0) {
        double gap = fabs(lam - Dv[k]);
        if (k > 0) gap = fmin(gap, fabs(lam - Dv[k - 1]));
        nz = A.nearzero * fabs(lam) < gap;
      }
      // ||x|| carried from m to the root to second order, as in k_eig
      const double h = nu1 - m;
      xsv = sqrt(zi2 + ((sp - 2.0 * (h * sp3)) + 3.0 * (h * (h * sp4))));
      nu0 = m;
      have_xs = true;
    }

    if (pol) {
      if (k == 0) {
        muv = ext_polish(Z2v, Zl, n, sigma, zi2, M.zz, rho, 1.0 / nu1, &pit, sm);
      } else {
        const dd bdd = {it.bhi, it.blo};
        const double xm = 1.0 / (Dv[k - 1] - Dv[k]);
        double cur = nu1;
        if (!(cur > it.lo && cur < it.hi)) cur = nu0;
        double last;
        const double sw = fabs(Zv[i == k ? k - 1 : k] * xm) / fabs(zi);
        cur = dd_polish(Z2v, Zl, n, i, s, sigma, zi, bdd, xm, sw, it.lo, it.hi, cur, false, &last, &pit, sm);
        muv = s / cur;
      }
      lam = sigma + muv;
      polished = true;
      if (A.nearzero > 0) {
        double gap = fabs(lam - Dv[k]);
        if (k > 0) gap = fmin(gap, fabs(lam - Dv[k - 1]));
        nz = A.nearzero * fabs(lam) < gap;
      }
    }

    if (nz) {
      // eq. (gamma): f(0) = 1 + rho z^T D^{-1} z in double-double
      dd f0 = {0.0, 0.0};
      double uu = 0.0, dmin = INFINITY;
      fix_poles<4, true>(Z2v, Zl, n, [&](int, double dj, double z2, double z2l, bool in) {
        const dd t = dd_div(dd{z2, z2l}, dd{dj, 0.0});
        if (in) {
          f0 = dd_add(f0, t);
          uu += (z2 / dj) / dj;
          dmin = fmin(dmin, fabs(dj));
        }
      });
      f0 = block_sum_dd(f0, sm);
      uu = block_sum(uu, sm);
      dmin = block_min(dmin, sm);
      f0 = dd_add(dd{1.0, 0.0}, dd_mul_d(f0, rho));
      double f0d = f0.hi + f0.lo;
      if (f0d == 0.0) {
        lam = 0.0;
        singular = 1;
      } else {
        const double gam = -rho / f0d;
        const double sh = (f0d < 0) ? 1.0 : -1.0;  // sign of lambda
        const double gt = sh * gam;
        // eta~ = sh/lambda > 0 on the right branch of
        // h(eta~) = 1 + gt sum zeta_j^2/(d~_j (1 - eta~ d~_j)),  d~ = sh d
        double lo;
        if (sh > 0) lo = (k > 0) ? 1.0 / Dv[k - 1] : 4.9406564584124654e-324;
        else lo = -1.0 / Dv[k];
        double hi = (1.0 / dmin + fabs(gam) * uu) * GROW;
        if (!(lo > 0)) lo = 4.9406564584124654e-324;
        if (!(hi > lo)) hi = lo * 2.0;
        // h rises and is concave right of its poles: Newton steps from the
        // eigenvalue found so far, inside the bracket that the signs of h
        // narrow (bisection alone took 60 passes over the poles, 1.1 ms for one
        // eigenpair at n = 32768).  The compensated step below follows.
        double e0 = sh / lam;
        if (!(e0 > lo && e0 < hi)) e0 = fmid(lo, hi);
        for (int hit = 0; hit < 200; ++hit) {
          double acc = 0.0, der = 0.0;
          fix_poles<8, false>(Z2v, nullptr, n, [&](int, double dj, double z2, double, bool in) {
            const double dt = sh * dj;
            const double om = __builtin_fma(-e0, dt, 1.0);
            const double t = z2 / (dt * om);
            acc += in ? t : 0.0;
            der += in ? t * dt / om : 0.0;
          });
          acc = block_sum(acc, sm);
          der = block_sum(der, sm);
          const double hv = 1.0 + gt * acc;
          if (hv < 0) lo = e0; else hi = e0;
          const double step = -hv / (gt * der);
          double t = e0 + step;
          const bool near = fabs(step) <= 0x1p-30 * e0;
          if (adjacent(lo, hi)) {
            e0 = hi;
            break;
          }
          if (!(t > lo && t < hi)) {
            if (near) break;
            t = fmid(lo, hi);
          }
          e0 = t;
          if (near) break;
        }
        double cs = 0.0, cc = 0.0, sp = 0.0;
        fix_poles<4, false>(Z2v, nullptr, n, [&](int, double dj, double z2, double, bool in) {
          const double dt = sh * dj;
          const double om = __builtin_fma(-e0, dt, 1.0);
          const double t = in ? z2 / (dt * om) : 0.0;
          const double y = cs + t;
          cc += (fabs(cs) >= fabs(t)) ? ((cs - y) + t) : ((t - y) + cs);
          cs = y;
          sp += in ? z2 / (om * om) : 0.0;
        });
        double S = block_sum_comp(cs, cc, sm);
        sp = block_sum(sp, sm);
        double hv = 1.0 + gt * S;
        double hp = gt * sp;
        double e1 = e0 - hv / hp;
        lam = sh / e1;
      }
    }

    if (polished) {
      double acc = 0.0;
      fix_poles<8, false>(Z2v, nullptr, n, [&](int, double dj, double z2, double, bool in) {
        const double den = (dj - sigma) - muv;
        const double rc = rcp_1nr(den);
        double r = muv * rc;
        r = __builtin_fma(__builtin_fma(-r, den, muv), rc, r);  // corrected quotient
        acc = __builtin_fma(in ? z2 * r : 0.0, r, acc);
      });
      xsv = sqrt(block_sum(acc, sm));
    }
    const double xs = polished || have_xs ? (fabs(it.bhi) < INFINITY ? xsv : NAN) : A.xs[off + k];
    if (A.V) {
      // the pair's column, in the writer's arithmetic
      const int64_t ko = M.neg ? n - 1 - k : k;
      const double sg = M.neg ? -1.0 : 1.0;
      const double iv = fabs(muv) / xs;  // 1/||x||
      double* col = A.V + (A.voffs ? A.voffs[it.p] : 0) + ko * (A.voffs ? (int64_t)n : A.ldv);
#pragma unroll 8
      for (int pos = tid; pos < n; pos += FIXT) {
        const int j = M.neg ? n - 1 - pos : pos;
        const double den = (Dv[j] - sigma) - muv;
        const double rc = rcp_1nr(den);
        double q = iv * rc;
        q = __builtin_fma(__builtin_fma(-q, den, iv), rc, q);  // corrected quotient
        __builtin_nontemporal_store((sg * Zv[j]) * q, &col[pos]);
      }
    }
    if (tid == 0) {
      put_outputs(A, M, it.p, k, i, lam, muv, xs, true);
      A.lam[off + k] = lam;
      if (nz) A.vflag[off + k] = 2;  // lambda from eq. (gamma): no remedy of K_nu
      A.mu[off + k] = muv;
      A.xs[off + k] = xs;
      if (A.stats) {
        if (polished) {
          atomicAdd(&A.stats[DPR1_STAT_POLISHED], 1);
          atomicMax(&A.stats[DPR1_STAT_POLISH_STEPS_MAX], min(pit + 1, 100));
        }
        if (it.flags & FIX_CONTINUE) atomicAdd(&A.stats[DPR1_STAT_CONTINUED], 1);
        if (nz) atomicAdd(&A.stats[DPR1_STAT_NEARZERO], 1);
        if (singular) atomicAdd(&A.stats[DPR1_STAT_SINGULAR], 1);
      }
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(FIXT, 4) k_fix(KArgs A) { fix_items(A); }

// ------------------------------------------------------------------- vec
// v_j = zeta_j w/(delta_j - mu), w = 1/||x|| (eq. eigenvecAi).  A block owns up
// to VEC_C columns of one problem over up to VEC_ROWS consecutive positions of
// each column.  The (d_j, zeta_j) of those positions are staged in LDS once; each
// wave then writes 128-element windows aligned to 1 KB of V (64 elements where
// columns are shorter), so every store covers whole lines at any column offset
// (a packed ragged batch puts most columns at odd offsets; misaligned
// non-temporal stores write partial lines and halve the write bandwidth).
// Only the first and last window of a column segment are partial.  The block
// reads (problem, first column, columns, first row) from a table built by the
// plan.
constexpr int VEC_T = 256;
constexpr int VEC_ROWS = 2048;
// most columns per block
constexpr int VEC_C = 32;
// Fewer, VEC_C_MIN at least, where they would be more than VEC_ELEMS elements,
// and in memory order, for the same reason as the tiles below: 300 problems of
// n = 700 .. 800 647 us a call (686 in 32 columns, largest problems first), 64
// of n = 1000 293 (311); twice the elements 670 and 306, half 696 and 300.
constexpr int VEC_C_MIN = 4, VEC_ELEMS = 8192;
// Where blocks of that many columns leave the GPU idle their width is halved,
// to 4 at least, until VEC_BLOCKS run (a problem of n = 1501: 47 blocks of 32
// columns took 54 us for 18 MB).
constexpr int64_t VEC_BLOCKS = 1024;
// most chunks of the overlapped single-problem solve (opts.vwrite)
constexpr int VEC_CHUNKS_MAX = 8;

// Arguments of the eigenvector writer.  Columns flagged in vflag belong to
// eigenpairs that k_fix finishes; they are skipped here and written there once
// their values are final.
struct VArgs {
  const Meta* meta;
  const int4* groups;  // batched: (problem, first column, columns, first row) per block
  const double* sd;
  const double* sz;
  const double* mu;
  const double* csig;
  const double* cinv;
  const uint8_t* vflag;
  double* V;
  const int64_t* voffs;
  int64_t ldv;
  int32_t cbase, cend;  // single problem: columns cbase .. cend-1
  int32_t prio;         // k_vec: raise the waves' issue priority
  int32_t n, neg;       // single problem: its order, rho < 0 (-1: in meta)
};

__device__ void vec_block(unsigned bid, const VArgs& v) {
  __shared__ double ld_d[VEC_ROWS], ld_z[VEC_ROWS];
  __shared__ double lsig[VEC_C], lmu[VEC_C], linv[VEC_C];
  __shared__ uint8_t lskip[VEC_C];
  const Meta* __restrict__ meta = v.meta;
  const double* __restrict__ sd = v.sd;
  const double* __restrict__ sz = v.sz;
  double* __restrict__ V = v.V;
  const int4 grp = v.groups[bid];
  const int p = grp.x, c0 = grp.y, nc = grp.z;
  const int64_t r0 = grp.w;
  const Meta M = meta[p];
  if (M.info != 0) return;
  const int n = M.n;
  const int nr = (int)min((int64_t)VEC_ROWS, (int64_t)n - r0);
  if (nc <= 0 || nr <= 0) return;
  const double sg = M.neg ? -1.0 : 1.0;
  // stage positions r0 .. r0+nr-1 (position = row in memory order; a
  // reversed problem stores row j at position n-1-j)
  for (int t = threadIdx.x; t < nr; t += VEC_T) {
    const int64_t pos = r0 + t;
    const int64_t j = M.neg ? n - 1 - pos : pos;
    ld_d[t] = sd[M.off + j];
    ld_z[t] = sg * sz[M.off + j];
  }
  if (threadIdx.x < nc) {
    const int64_t a = M.off + c0 + threadIdx.x;
    lsig[threadIdx.x] = v.csig[a];
    lmu[threadIdx.x] = v.mu[a];
    linv[threadIdx.x] = v.cinv[a];
    lskip[threadIdx.x] = v.vflag ? v.vflag[a] : 0;
  }
  const bool skipping = __syncthreads_or(threadIdx.x < nc && v.vflag && v.vflag[M.off + c0 + threadIdx.x]);
  typedef double vdbl2 __attribute__((ext_vector_type(2)));
  constexpr int WE = 2 * WAVE;
  const int64_t ld = n, base = v.voffs[p];
  const int wv = wave_id(), lane = threadIdx.x % WAVE;
  constexpr int NW = VEC_T / WAVE;
  if (nr == n) {
    // Whole columns of a packed block: the group's columns are one
    // contiguous range of nc n elements, written in aligned windows with
    // (column, position) recovered per element.  nc n <= CB VEC_ROWS < 2^24,
    // so the float quotient is off by at most one and corrected exactly.
    const int64_t kolo = M.neg ? (int64_t)n - c0 - nc : c0;
    const int64_t S = base + kolo * n;
    const int len = nc * n;
    if (n >= WE) {
      // windows of 128 elements aligned to 1 KB, two elements per lane in one
      // 16-byte store; a window meets two columns at most, and the wave keeps
      // the column and position of its first element
      const int skew = (int)(((uintptr_t)(V + S) >> 3) & (WE - 1));
      int l0 = wv * WE - skew, q = l0 > 0 ? l0 / n : 0, pos0 = l0 - q * n;
      const int dq = NW * WE / n, dr = NW * WE - dq * n;
      auto value = [&](int x, bool& ok) {  // element x of the window's column or of the next
        int c = q;
        ok = l0 + x >= 0 && l0 + x < len;
        int pos = pos0 + x;
        if (pos >= n) {
          pos -= n;
          ++c;
        }
        pos = max(pos, 0);
        c = min(c, nc - 1);
        if (M.neg) c = nc - 1 - c;
        if (skipping) ok = ok && !lskip[c];
        const double w = linv[c];
        const double den = (ld_d[pos] - lsig[c]) - lmu[c];
        const double rc = rcp_1nr(den);
        double qq = w * rc;
        qq = __builtin_fma(__builtin_fma(-qq, den, w), rc, qq);  // corrected quotient
        return ld_z[pos] * qq;
      };
      for (; l0 < len; l0 += NW * WE) {
        bool a0, a1;
        const double v0 = value(2 * lane, a0), v1 = value(2 * lane + 1, a1);
        double* vp = V + S + l0 + 2 * lane;
        if (a0 && a1) {
          const vdbl2 vv = {v0, v1};
          __builtin_nontemporal_store(vv, reinterpret_cast<vdbl2*>(vp));
        } else if (a0) {
          __builtin_nontemporal_store(v0, vp);
        } else if (a1) {
          __builtin_nontemporal_store(v1, vp + 1);
        }
        q += dq;
        pos0 += dr;
        if (pos0 >= n) {
          pos0 -= n;
          ++q;
        } else if (pos0 < 0) {  // the first window started before the range
          pos0 += n;
          --q;
        }
      }
      return;
    }
    const int64_t Sal = S & ~(int64_t)(WAVE - 1);
    const int nwin = (int)((S + len - Sal + WAVE - 1) / WAVE);
    const float inv_n = 1.0f / (float)n;
    for (int w = wv; w < nwin; w += NW) {
      const int64_t e = Sal + (int64_t)w * WAVE + lane;
      const int64_t l64 = e - S;
      if (l64 >= 0 && l64 < len) {
        const int local = (int)l64;
        int q = (int)((float)local * inv_n);
        int pos = local - q * n;
        if (pos < 0) {
          pos += n;
          --q;
        } else if (pos >= n) {
          pos -= n;
          ++q;
        }
        const int ko = (int)kolo + q;
        const int c = (M.neg ? n - 1 - ko : ko) - c0;
        if (lskip[c]) continue;
        const double w = linv[c];
        const double den = (ld_d[pos] - lsig[c]) - lmu[c];
        const double rc = rcp_1nr(den);
        double qq = w * rc;
        qq = __builtin_fma(__builtin_fma(-qq, den, w), rc, qq);  // corrected quotient
        __builtin_nontemporal_store(ld_z[pos] * qq, &V[e]);
      }
    }
    return;
  }
  // Column segments: wave w writes columns w, w + NW, ... of the group, each
  // in windows of 128 elements aligned to 1 KB, two consecutive elements per
  // lane in one 16-byte store (the column's address set up once, then a plain
  // loop; a window's lane with only one element in the segment stores it
  // alone).
  for (int c = wv; c < nc; c += NW) {
    if (lskip[c]) continue;
    const int k = c0 + c;
    const int64_t ko = M.neg ? n - 1 - k : k;
    const int64_t s0 = base + ko * ld + r0;  // element index of the segment's first position
    // windows aligned on the address (V itself need only be 8-byte aligned)
    const int64_t sal = s0 - (int64_t)(((uintptr_t)(V + s0) >> 3) & (WE - 1));
    const int nwin = (int)((s0 + nr - sal + WE - 1) / WE);
    const double m = lmu[c], sc = lsig[c], iv = linv[c];
    double* vp = V + sal + 2 * lane;
    int rel = (int)(sal - s0) + 2 * lane;
    for (int w = 0; w < nwin; ++w, vp += WE, rel += WE) {
      const bool a0 = rel >= 0 && rel < nr, a1 = rel + 1 >= 0 && rel + 1 < nr;
      if (!a0 && !a1) continue;
      const int r0c = a0 ? rel : rel + 1, r1c = a1 ? rel + 1 : rel;
      const double den0 = (ld_d[r0c] - sc) - m, den1 = (ld_d[r1c] - sc) - m;
      const double rc0 = rcp_1nr(den0), rc1 = rcp_1nr(den1);
      double q0 = iv * rc0, q1 = iv * rc1;
      q0 = __builtin_fma(__builtin_fma(-q0, den0, iv), rc0, q0);  // corrected quotients
      q1 = __builtin_fma(__builtin_fma(-q1, den1, iv), rc1, q1);
      const double v0 = ld_z[r0c] * q0, v1 = ld_z[r1c] * q1;
      if (a0 && a1) {
        const vdbl2 vv = {v0, v1};
        __builtin_nontemporal_store(vv, reinterpret_cast<vdbl2*>(vp));
      } else if (a0) {
        __builtin_nontemporal_store(v0, vp);
      } else {
        __builtin_nontemporal_store(v1, vp + 1);
      }
    }
  }
}


// The eigenvector writer of one problem (batches take vec_block): a block
// writes TILE_ROWS positions of TILE_C columns, two consecutive positions per
// thread in one 16-byte non-temporal store, and ends; blocks go down the
// columns first, in memory order.  HBM takes writes fastest when the whole
// GPU's write front moves through memory in order, as a fill does, and blocks
// that start in order and end soon hold it together better than resident waves
// that loop over columns: n = 32768, the writer alone 1230 us (7.0 TB/s; a fill
// 1270) against 1430 to 1780 for 1024 or 2048 looping waves, and 1440 with 8
// blocks per CU in place of the 4 that k_fix's registers leave.  A call: n =
// 32768 1497 us (1622 with looping waves), n = 24000 841 (930).  A tile's
// columns pay for its start-up: 8 columns, 6 and 10 are 1 to 3 % slower, 4 10 %.
// The arithmetic is vec_block's.
// Where every column starts on a 128-byte line a thread's d and zeta stay in
// registers.  Else (SH) a column's windows are shifted back to whole lines, by
// up to LINE - 1 positions, and the block keeps the positions that it may meet
// in LDS; the last range also writes the up to LINE - 1 positions behind its
// window.  A call: n = 32767 1700 us (2020 with 2048 rows by 32 columns a block,
// windows aligned but each block's columns far apart), n = 16001 474 (562).
constexpr int TILE_ROWS = 2 * VEC_T;
constexpr int TILE_C = 8;
constexpr int LINE = 16;  // doubles of a line
template <bool SH>
__device__ void vec_tile(const VArgs& v, unsigned bid) {
  constexpr int C = TILE_C;
  // rho's sign on the host: the loads below need not wait for the meta record
  Meta M;
  const int info = v.meta[0].info;
  if (v.neg >= 0) {
    M.off = 0;
    M.n = v.n;
    M.neg = v.neg;
  } else {
    M = v.meta[0];
  }
  const int n = M.n, t = threadIdx.x;
  const int rt = (n + TILE_ROWS - 1) / TILE_ROWS;
  const int r = (int)(bid % rt), r0 = r * TILE_ROWS;
  // columns in memory order: ko of the caller's, k = n - 1 - ko when reversed
  const int ce = min(n, v.cend);
  const int kb = M.neg ? n - ce : v.cbase, ke = M.neg ? n - v.cbase : ce;
  const int64_t ko0 = kb + (int64_t)(bid / rt) * C;
  if (ko0 >= ke) return;
  const double sg = M.neg ? -1.0 : 1.0;
  // (d, zeta) of a position, 0 outside the column
  auto entry = [&](int at, double& d, double& z) {
    const bool in = at >= 0 && at < n;
    const int64_t j = M.off + (M.neg ? n - 1 - at : at);
    d = in ? v.sd[j] : 0.0;
    z = in ? sg * v.sz[j] : 0.0;
  };
  double sc[C], mm[C], iv[C];
  bool skip[C];  // past the range, or a column k_fix writes
#pragma unroll
  for (int u = 0; u < C; ++u) {
    const int ko = (int)min(ko0 + u, (int64_t)ke - 1);
    const int64_t a = M.off + (M.neg ? n - 1 - ko : ko);
    sc[u] = v.csig[a];
    mm[u] = v.mu[a];
    iv[u] = v.cinv[a];
    skip[u] = ko0 + u >= ke || (v.vflag && v.vflag[a]);
  }
  constexpr int NB = TILE_ROWS + 2 * LINE;
  __shared__ double ld_d[SH ? NB : 1], ld_z[SH ? NB : 1];
  double d0, z0, d1, z1;
  if (SH) {
    for (int i = t; i < NB - 1; i += VEC_T) entry(r0 - (LINE - 1) + i, ld_d[i], ld_z[i]);
    __syncthreads();
  } else {
    entry(r0 + 2 * t, d0, z0);
    entry(r0 + 2 * t + 1, d1, z1);
  }
  if (info != 0) return;
#pragma unroll
  for (int u = 0; u < C; ++u) {
    if (skip[u]) continue;
    double* col = v.V + (ko0 + u) * v.ldv;
    const int s = SH ? (int)(((uintptr_t)col >> 3) & (LINE - 1)) : 0;
    if (SH) {
      const int i = LINE - 1 - s + 2 * t;
      d0 = ld_d[i];
      d1 = ld_d[i + 1];
      z0 = ld_z[i];
      z1 = ld_z[i + 1];
    }
    const double den0 = (d0 - sc[u]) - mm[u], den1 = (d1 - sc[u]) - mm[u];
    const double rc0 = rcp_1nr(den0), rc1 = rcp_1nr(den1);
    double q0 = iv[u] * rc0, q1 = iv[u] * rc1;
    q0 = __builtin_fma(__builtin_fma(-q0, den0, iv[u]), rc0, q0);  // corrected quotients
    q1 = __builtin_fma(__builtin_fma(-q1, den1, iv[u]), rc1, q1);
    typedef double vdbl2 __attribute__((ext_vector_type(2)));
    const vdbl2 vv = {z0 * q0, z1 * q1};
    const int at = r0 - s + 2 * t;
    const bool a0 = at >= 0 && at < n, a1 = at + 1 >= 0 && at + 1 < n;
    if (a0 && a1)
      __builtin_nontemporal_store(vv, reinterpret_cast<vdbl2*>(col + at));
    else if (a0)
      __builtin_nontemporal_store(vv.x, col + at);
    else if (a1)
      __builtin_nontemporal_store(vv.y, col + at + 1);
    const int tail = r0 + TILE_ROWS - s + t;
    if (SH && r == rt - 1 && t < LINE && tail < n) {
      const int i = LINE - 1 - s + TILE_ROWS + t;
      const double den = (ld_d[i] - sc[u]) - mm[u], rc = rcp_1nr(den);
      double q = iv[u] * rc;
      q = __builtin_fma(__builtin_fma(-q, den, iv[u]), rc, q);
      __builtin_nontemporal_store(ld_z[i] * q, col + tail);
    }
  }
}
static int64_t tile_blocks(int64_t n, int64_t columns) {
  return (n + TILE_ROWS - 1) / TILE_ROWS * ((columns + TILE_C - 1) / TILE_C);
}

// The eigenvector writer alone (single problem, a range of columns); launched
// with VEC_PAD bytes of LDS, which leave 4 blocks per CU.
constexpr size_t VEC_PAD = 28 << 10;
// The writer's table of a batch, in memory order, from an entry a problem:
// (its first block, columns a block, order).  Made and copied by the host it was
// most of a large plan, us: the 2048-problem mix (100 000 blocks) 300 against
// 117, one problem of n = 32768 143 / 26, 8 of 8000 85 / 26; 256 of 512 (8192
// blocks) 30 / 30, and below a kernel costs more than it saves (100 of 300 17 /
// 22, 64 of 64 15 / 21): PLAN_HOST.
constexpr int64_t PLAN_HOST = 8192;
__global__ void __launch_bounds__(256) k_plan_groups(int nprob, int ngroups, const int4* __restrict__ prob,
                                                     int4* __restrict__ groups) {
  const int e = (int)(blockIdx.x * 256 + threadIdx.x);
  if (e >= ngroups) return;
  int lo = 0, hi = nprob - 1;  // the last problem whose first block is not behind e
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (prob[mid].x <= e)
      lo = mid;
    else
      hi = mid - 1;
  }
  const int4 q = prob[lo];
  const int rt = (q.z + VEC_ROWS - 1) / VEC_ROWS, l = e - q.x;
  const int c0 = l / rt * q.y, r0 = l % rt * VEC_ROWS;
  groups[e] = make_int4(lo, c0, min(q.y, q.z - c0), r0);
}

template <bool SH>
__global__ void __launch_bounds__(VEC_T) k_vec(VArgs v) {
  // beside the eigenvalue kernel of the next chunk its waves issue first, so
  // that the stores keep flowing while the sweeps take the remaining issue
  // slots; beside k_fix (the last chunk) they do not, since k_fix is latency-
  // bound and would starve
  if (v.prio) __builtin_amdgcn_s_setprio(3);
  vec_tile<SH>(v, blockIdx.x);
}

// k_fix and the eigenvector writer in one launch, so that the two overlap: the
// first nfix blocks take flagged eigenpairs from the queue (latency-bound
// work), then come the blocks that write V (HBM-bound), and the last ntail take
// what is left of the queue when the writers run out.
// Where the writers are more than the GPU's places few blocks go in front: 256
// there hold a quarter of the places for little when few eigenpairs are flagged.
// Where all blocks are resident together the tail only costs its launch.  A call
// with FIX_SMALL in front / FIX_HEAD and FIX_TAIL, us: n = 300 57 / 60, 1000 76 / 81,
// 1400 77 / 82, 1700 83 / 83, 2000 89 / 88, 4000 107 / 103, 8000 181 / 169, 20000
// 696 / 666; every eigenpair polished, 6000 472 / 361.
constexpr int FIX_HEAD = 64, FIX_TAIL = 448, FIX_SMALL = 256;
constexpr int64_t FIX_RESIDENT = 1024;  // 256 CUs, 4 blocks each
// A batch: few blocks in front where its flagged eigenpairs are few (at least one
// a problem, the exterior one) or little against what the writer has to do, for
// which its blocks per 64 eigenvalues stand where they are full ones (4 for
// problems of n = 257 .. 512, 8 above); the line lies at order 490, inside the
// orders of 4 blocks, so also by the mean order.  512 blocks in front /
// BATCH_HEAD and BATCH_TAIL, us (graded poles in brackets): 400 problems of n = 64
// 72 / 86, 100 of 200 82 / 103, 1000 of n = 104 .. 156 208 / 238 (202 / 234), 200 of
// 300 158 / 207, 300 of n = 264 .. 396 270 / 304 (270 / 308), 200 of 480 264 / 274
// (335 / 348), 256 of 512 (398 / 383), 200 of 540 297 / 293 (384 / 380), 300 of n =
// 600 .. 900 625 / 603 (799 / 776); 30 of 200 65 / 62, 30 of 300 72 / 69, 40 of 300
// 73 / 77, 10 of 1000 94 / 92 (132 / 130); 300 of n = 100 .. 700 257 / 285, 1024 of n = 16 .. 2048
// 1304 / 1288.
constexpr int FIX_BATCH = 512, BATCH_HEAD = 128, BATCH_TAIL = 384;
constexpr int64_t BATCH_FEW = 6, BATCH_FEW_MEAN = 490, BATCH_FEW_PROB = 32;
static bool batch_few(int64_t nprob, int64_t N, int64_t ngroups) {
  return nprob <= BATCH_FEW_PROB || N >= BATCH_FEW_MEAN * nprob ||
         (ngroups > 2 * VEC_BLOCKS && WAVE * ngroups >= BATCH_FEW * N);
}
enum { VEC_BATCH, VEC_ALIGNED, VEC_SHIFTED };
template <int KIND>
__global__ void __launch_bounds__(VEC_T, 4) k_fixvec(KArgs A, VArgs v, int nfix, int ntail) {
  if (blockIdx.x < (unsigned)nfix || blockIdx.x >= gridDim.x - ntail)
    fix_items(A);
  else if (KIND == VEC_BATCH)
    vec_block(blockIdx.x - nfix, v);
  else
    vec_tile<KIND == VEC_SHIFTED>(v, blockIdx.x - nfix);
}

// ------------------------------------------------------- K_nu, remedies
// K_nu of eq. (K0) for eigenpair k shifted to d_i: ||A_i^{-1}||_2 =
// 1/min_j |lambda_j - d_i|, and by the interlacing (eq. interlace) the
// minimum is taken at lambda_k or at the other eigenvalue beside the pole,
// lambda_o (o = k+1 if i = k, o = k-1 if i = k-1), so
// K_nu = |lambda_k - d_i| / min(|lambda_k - d_i|, |lambda_o - d_i|), with the
// distances from the shifted representations in double-double.  knu_pole
// gives it for any neighbouring pole p of lambda_k (remedy (R1) compares the
// two).
__device__ double knu_pole(const double* Dv, const int32_t* ii, const double* mu, int n, int k, int p) {
  const dd lk = dd_add(two_sum(Dv[ii[k]], -Dv[p]), dd{mu[k], 0.0});
  const double ak = fabs(lk.hi + lk.lo);
  const int o = (p == k) ? k + 1 : k - 1;
  if (o < 0 || o >= n || ak == 0.0) return 1.0;
  const dd lo = dd_add(two_sum(Dv[ii[o]], -Dv[p]), dd{mu[o], 0.0});
  const double ao = fabs(lo.hi + lo.lo);
  if (ao >= ak) return 1.0;
  return ao > 0.0 ? ak / ao : INFINITY;
}

// A remedy: eigenpair k of problem p, nearest pole i; po the other
// neighbouring pole for (R1), -1 for (R2).
struct RemItem {
  int32_t p, k, i, po;
};

// One thread per eigenpair (a batch: block p takes problem p): K_nu to the
// optional output, the count of K_nu > knu_thr, and with opts.remedy the
// remedy list (in the eigenpair list's memory, free once k_fix has run).
// Pairs whose eigenvalue came from eq. (gamma) (vflag 2) keep it.
__global__ void __launch_bounds__(256) k_knu(KArgs A, int nprob) {
  const int p = nprob > 1 ? (int)blockIdx.x : 0;
  const int k0 = nprob > 1 ? (int)threadIdx.x : (int)(blockIdx.x * blockDim.x + threadIdx.x);
  const int kstep = nprob > 1 ? (int)blockDim.x : (int)(gridDim.x * blockDim.x);
  if (p >= nprob) return;
  const Meta M = A.meta[p];
  if (M.info != 0) return;
  const int n = M.n;
  const int64_t off = M.off;
  const double* Dv = A.sd + off;
  const int32_t* ii = A.ii + off;
  const double* mu = A.mu + off;
  RemItem* list = reinterpret_cast<RemItem*>(A.fix);
  for (int k = k0; k < n; k += kstep) {
    const int i = ii[k];
    const double K = n > 1 ? knu_pole(Dv, ii, mu, n, k, i) : 1.0;
    if (A.knu) A.knu[off + (M.neg ? n - 1 - k : k)] = K;
    if (!(K > A.knu_thr)) continue;
    if (A.stats) atomicAdd(&A.stats[DPR1_STAT_KNU_GT], 1);
    if (!A.remedy || A.vflag[off + k] == 2) continue;
    const int po = (i == k) ? k - 1 : k;  // the other neighbouring pole
    int use = -1;
    if (k >= 1 && po >= 0) {
      const double K2 = knu_pole(Dv, ii, mu, n, k, po);
      if (K2 < K && K2 <= A.knu_thr) use = po;
    }
    const int e = atomicAdd(&A.ctr[4], 1);
    list[e] = RemItem{p, k, i, use};
  }
}

// Remedies of Sec. 2 (Algorithm 1, last branch), one block of FIXT threads
// per listed eigenpair:
//  (R1) the other neighbouring pole d_po: its tip b (eq. b_ob) in
//       double-double, the extreme root of its g refined in double-double
//       (dd_polish from the current eigenvalue), and mu_i = (d_po - d_i) +
//       mu_po in double-double: mu_i inherits mu_po's absolute error, so the
//       root is carried to about 2^-100;
//  (R2) A - sigma I with sigma = d_i + mu (1 - 2^-e) between d_i and lambda
//       (e = 20, or smaller when the sign of f(sigma) shows sigma past
//       lambda): its inverse E + gamma u u^T with e_j = 1/(d_j - sigma), u_j =
//       zeta_j e_j, gamma = -rho/f(sigma), f(sigma) = 1 + rho sum
//       zeta_j^2/(d_j - sigma) in double-double from the exact differences;
//       eta = 1/(lambda - sigma) is its exterior eigenvalue (right of every
//       e_j when mu > 0, left when mu < 0), found by safeguarded Newton steps
//       from the current estimate; mu_i = (sigma - d_i) + 1/eta.
// The eigenpair keeps its nearest pole; ||x||, the outputs and its column of
// V are recomputed from the new mu.
__global__ void __launch_bounds__(FIXT) k_remedy(KArgs A) {
  __shared__ double sm[20];
  const int tid = threadIdx.x;
  const int cnt = A.ctr[4];
  const RemItem* list = reinterpret_cast<const RemItem*>(A.fix);
  for (int e = blockIdx.x; e < cnt; e += gridDim.x) {
    const RemItem it = list[e];
    const Meta M = A.meta[it.p];
    const int n = M.n;
    const int64_t off = M.off;
    const double* Dv = A.sd + off;
    const double* Zv = A.sz + off;
    const double2* Z2v = reinterpret_cast<const double2*>(A.pairs + 2 * off);
    const double* Zl = A.z2lo + off;
    const double rho = M.rho;
    const int k = it.k, i = it.i;
    const double muk = A.mu[off + k];
    double newmu = NAN;
    int how = 0;
    if (it.po >= 0) {
      // ---- (R1)
      const int po = it.po;
      const double s = (po == k) ? 1.0 : -1.0;
      const double sigma = Dv[po], zp = Zv[po];
      dd acc = {0.0, 0.0};
      for (int j = tid; j < n; j += FIXT) {
        if (j == po) continue;
        const double2 pj = Z2v[j];
        const dd dl = two_sum(pj.x, -sigma);
        const double r = rcp_1nr(dl.hi);
        const double q1 = pj.y * r;
        double er = __builtin_fma(-q1, dl.hi, pj.y);
        er = __builtin_fma(-q1, dl.lo, er + Zl[j]);
        acc = dd_add(acc, fast_two_sum(q1, er * r));
      }
      acc = block_sum_dd(acc, sm);
      const dd num = dd_add(dd_div(dd{1.0, 0.0}, dd{rho, 0.0}), acc);
      const dd b = dd_div_sq(num, zp);
      const dd bdd = {s * b.hi, s * b.lo};
      const double xm = 1.0 / (Dv[k - 1] - Dv[k]);
      // nu at d_po from the current eigenvalue: 1/(s (lambda - d_po))
      const dd lp = dd_add(two_sum(Dv[i], -sigma), dd{muk, 0.0});
      double cur = 1.0 / (s * (lp.hi + lp.lo));
      double last;
      int steps;
      const double sw = fabs(Zv[po == k ? k - 1 : k] * xm) / fabs(zp);
      cur = dd_polish(Z2v, Zl, n, po, s, sigma, zp, bdd, xm, sw, xm, INFINITY, cur, true, &last, &steps, sm);
      const dd nu = fast_two_sum(cur, last);
      const dd mup = dd_div(dd{s, 0.0}, nu);
      const dd mi = dd_add(two_sum(sigma, -Dv[i]), mup);
      newmu = mi.hi + mi.lo;
      how = 1;
    } else {
      // ---- (R2)
      const bool pos = muk > 0;
      for (int ex = 20; ex >= 2; ex -= 6) {
        const double ms = muk * (1.0 - ldexp(1.0, -ex));  // sigma - d_i
        dd fs = {0.0, 0.0};
        double uu = 0.0, emax = -INFINITY, emin = INFINITY, emag = 0.0;
        for (int j = tid; j < n; j += FIXT) {
          const double2 pj = Z2v[j];
          const dd dl = dd_add(two_sum(pj.x, -Dv[i]), dd{-ms, 0.0});  // d_j - sigma
          const double r = rcp_1nr(dl.hi);
          const double q1 = pj.y * r;
          double er = __builtin_fma(-q1, dl.hi, pj.y);
          er = __builtin_fma(-q1, dl.lo, er + Zl[j]);
          fs = dd_add(fs, fast_two_sum(q1, er * r));
          const double dr = dl.hi + dl.lo, ej = 1.0 / dr, uj = Zv[j] / dr;
          uu += uj * uj;
          emax = fmax(emax, ej);
          emin = fmin(emin, ej);
          emag = fmax(emag, fabs(ej));
        }
        fs = block_sum_dd(fs, sm);
        uu = block_sum(uu, sm);
        emax = -block_min(-emax, sm);
        emin = block_min(emin, sm);
        emag = -block_min(-emag, sm);
        const dd F = dd_add(dd{1.0, 0.0}, dd_mul_d(fs, rho));
        if (pos ? !(F.hi < 0.0) : !(F.hi > 0.0)) continue;  // sigma is past lambda
        const double gam = -rho / (F.hi + F.lo);
        const double ub = (emag + fabs(gam) * uu) * GROW;
        double lo, hi;
        if (pos) {
          lo = emax > 0.0 ? emax : 4.9406564584124654e-324;
          hi = ub;
        } else {
          lo = -ub;
          hi = emin < 0.0 ? emin : -4.9406564584124654e-324;
        }
        // eta from the current estimate 1/(mu - ms), kept in the bracket
        double cur = 1.0 / (muk - ms);
        for (int st = 0; st < 80; ++st) {
          if (!(cur > lo && cur < hi)) cur = fmid_signed(lo, hi);
          double hs = 0.0, hc = 0.0, hp = 0.0;
          for (int j = tid; j < n; j += FIXT) {
            const double2 pj = Z2v[j];
            const dd dl = dd_add(two_sum(pj.x, -Dv[i]), dd{-ms, 0.0});
            const double dr = dl.hi + dl.lo, ej = 1.0 / dr, uj = Zv[j] / dr;
            const double den = ej - cur;
            const double t = (uj * uj) / den;
            const double y = hs + t;
            hc += (fabs(hs) >= fabs(t)) ? ((hs - y) + t) : ((t - y) + hs);
            hs = y;
            hp += (uj * uj) / (den * den);
          }
          const double S = block_sum_comp(hs, hc, sm);
          hp = block_sum(hp, sm);
          const double h = 1.0 + gam * S;
          if (h == 0.0) break;
          // right branch: h rises, the root is above where h < 0; left branch:
          // h falls, the root is above where h > 0
          if (pos ? (h < 0.0) : (h > 0.0)) lo = cur; else hi = cur;
          const double step = -h / (gam * hp);
          double t = cur + step;
          if (!(t > lo && t < hi)) t = fmid_signed(lo, hi);
          if (t == cur || fabs(step) <= 0x1p-53 * fabs(cur) || adjacent_signed(lo, hi)) {
            cur = t > lo && t < hi ? t : cur;
            break;
          }
          cur = t;
        }
        newmu = ms + 1.0 / cur;
        how = 2;
        break;
      }
    }
    if (!(newmu == newmu) || newmu == 0.0 || !(fabs(newmu) < INFINITY)) continue;
    // ||x|| scaled by |mu| from the new mu, as after the polish
    double acc = 0.0;
    for (int j = tid; j < n; j += FIXT) {
      const double r = (j == i) ? -1.0 : newmu / ((Dv[j] - Dv[i]) - newmu);
      acc = __builtin_fma(Z2v[j].y * r, r, acc);
    }
    const double xsv = sqrt(block_sum(acc, sm));
    const double lam = Dv[i] + newmu;
    const int ko = M.neg ? n - 1 - k : k;
    const double sg = M.neg ? -1.0 : 1.0;
    if (tid == 0) {
      A.mu[off + k] = newmu;
      A.xs[off + k] = xsv;
      A.lam[off + k] = lam;
      put_outputs(A, M, it.p, k, i, lam, newmu, xsv, true);
      if (A.stats) atomicAdd(&A.stats[how == 1 ? DPR1_STAT_REMEDY_R1 : DPR1_STAT_REMEDY_R2], 1);
    }
    if (A.V) {
      const double sc = Dv[i];
      const double iv = fabs(newmu) / xsv;
      const int64_t ld = A.voffs ? (int64_t)n : A.ldv;
      double* col = A.V + (A.voffs ? A.voffs[it.p] : 0) + (int64_t)ko * ld;
      for (int pos = tid; pos < n; pos += FIXT) {
        const int j = M.neg ? n - 1 - pos : pos;
        const double den = (Dv[j] - sc) - newmu;
        const double rc = rcp_1nr(den);
        double q = iv * rc;
        q = __builtin_fma(__builtin_fma(-q, den, iv), rc, q);
        __builtin_nontemporal_store((sg * Zv[j]) * q, &col[pos]);
      }
    }
  }
}

// ===================================================================== host
struct Layout {
  size_t meta, sd, sz, pairs, z2lo, ii, mu, xs, lam, csig, cinv, fix, vflag, prob, items, witems, groups, part, ctr,
      far, total;
};

static constexpr size_t al(size_t x) { return (x + 255) & ~size_t(255); }

// nrec: far-field records; nwide: entries of a batch's list of wide items, whose
// offset is in the header at FAR_HDR behind the counters.
constexpr size_t FAR_HDR = 128;
static constexpr Layout layout(int64_t nprob, int64_t N, int64_t nitems, int64_t ngroups, int64_t nrec,
                               int64_t nwide) {
  Layout L{};
  size_t o = 0;
  L.meta = o; o = al(o + sizeof(Meta) * nprob);
  L.sd = o; o = al(o + 8 * N);
  L.sz = o; o = al(o + 8 * N);
  L.pairs = o; o = al(o + 16 * N);
  L.z2lo = o; o = al(o + 8 * N);
  L.ii = o; o = al(o + 4 * N);
  L.mu = o; o = al(o + 8 * N);
  L.xs = o; o = al(o + 8 * N);
  L.lam = o; o = al(o + 8 * N);
  L.csig = o; o = al(o + 8 * N);
  L.cinv = o; o = al(o + 8 * N);
  L.fix = o; o = al(o + sizeof(FixItem) * N);
  L.vflag = o; o = al(o + N);
  L.part = o; o = al(o + 3 * sizeof(double) * PREP_MAX_SPLIT);
  L.ctr = o; o = al(o + FAR_HDR + sizeof(FarHdr));  // the plan's header, problems, queue and wide items: one copy
  L.prob = o; o = al(o + (nitems ? sizeof(int4) * nprob : 0));
  L.items = o; o = al(o + sizeof(int4) * nitems);
  L.witems = o; o = al(o + sizeof(int4) * nwide);
  L.groups = o; o = al(o + sizeof(int4) * ngroups);
  L.far = o; o = al(o + 8 * (size_t)FAR_REC * nrec);
  L.total = o;
  return L;
}

// One problem: a record per block of 64 eigenvalues and the wide level's.
static constexpr Layout layout_single(int64_t n) {
  return layout(1, n, 0, 0, n < FAR_MIN ? 0 : (n + WAVE - 1) / WAVE + far_wide_room(n), 0);
}
// A batch, from what its plan holds.  The wide level's records lie behind the
// queue's.  Halving the columns of the writer's blocks at most doubles a count
// below VEC_BLOCKS, so 2 VEC_BLOCKS entries hold the table wherever it is not
// the one of full blocks: the size grows with the problems and their number.
static int64_t batch_items(int64_t nprob, int64_t N) { return N / WAVE + nprob; }  // >= sum ceil(n_p/64)
static Layout layout_batch(int64_t nprob, int64_t N, int64_t nmax, int64_t ngroups) {
  const int64_t nitems = batch_items(nprob, N), nwide = far_batch_wide(N, nmax);
  return layout(nprob, N, nitems, std::max(ngroups, 2 * VEC_BLOCKS), far_batch_own(N, nmax, nitems) + nwide, nwide);
}

static void fill_opts(const dpr1_opts* in, dpr1_opts* o) {
  dpr1_default_opts(o);
  if (in) {
    *o = *in;
    if (!(o->kappa_polish > 0)) o->kappa_polish = 16.0;
    if (o->nearzero < 0) o->nearzero = 10.0;
    if (!(o->knu_thr > 0)) o->knu_thr = 32.0;
  }
}

// The split when the options leave it open.  What a block does between its
// sums (the tip's quotients, the model steps, the expansions) does not shrink
// with W, so W only pays while the GPU has idle issue slots: few blocks.
// Measured, k_eig with W = 1 / 2 / 4 / 8 in us: n = 256 (4 blocks) 72 / 51 / 39
// / 40, n = 1501 (24) 64 / 51 / 44 / 50, n = 4096 (64) 107 / 74 / 58 / 59, 512
// problems of n = 100 (1024) 89 / 67 / 72 / -, 256 of n = 512 (2048) 168 / 142
// / 162 / -, the 2048-problem mix (14 700) 641 / 694 / 820 / -.  From n = 2048
// on few blocks take 8, which costs nothing there and halves the time of a
// block whose poles are all near (steeply graded poles).  A slice has at least
// 16 poles.
static int pick_split(int64_t nblocks, int64_t nmax) {
  int w = nblocks <= 640 ? (nmax >= 2048 ? 8 : 4) : nblocks <= 6144 ? 2 : 1;
  while (w > 1 && nmax / w < 16) w /= 2;
  return w;
}

// k_eig occupancy variant of the options: 4 (default), 6 or 8 waves per SIMD.
static int occ_of(const dpr1_opts& o) { return o.waves_per_simd == 0 ? 4 : o.waves_per_simd; }
static bool occ_valid(int32_t w) { return w == 0 || w == 4 || w == 6 || w == 8; }

// Blocks of the persistent batched k_eig: as many W-wave blocks as the 256
// CUs hold at the variant's occupancy (4 SIMDs x occ waves per CU), never
// more blocks than work items.
static int32_t persistent_grid_for(int64_t nitems, int W, int occ) {
  const int64_t per_cu = std::max<int64_t>(1, (4 * occ) / W);
  return (int32_t)std::min<int64_t>(nitems, 256 * per_cu);
}

// ------------------------------------------------------------ autotuning
// Mean duration in ms of `reps` calls of `solve` after one untimed call,
// between two events on stream st.
template <class F>
static int time_calls(F&& solve, int reps, hipStream_t st, double* ms) {
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return DPR1_EHIP;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return DPR1_EHIP;
  }
  int rc = solve();
  if (rc == 0 && hipEventRecord(e0, st) != hipSuccess) rc = DPR1_EHIP;
  for (int r = 0; r < reps && rc == 0; ++r) rc = solve();
  if (rc == 0 && hipEventRecord(e1, st) != hipSuccess) rc = DPR1_EHIP;
  if (rc == 0 && hipEventSynchronize(e1) != hipSuccess) rc = DPR1_EHIP;
  float t = 0.0f;
  if (rc == 0 && hipEventElapsedTime(&t, e0, e1) != hipSuccess) rc = DPR1_EHIP;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *ms = (double)t / reps;
  return rc;
}

// Candidate splits for the largest order nmax: W waves share one block of 64
// eigenvalues (W threads per eigenvalue), 64 poles of the problem or more each
// (they split the near poles, which are fewer from order FAR_MIN on).  Candidate
// occupancy variants of k_eig: 4, 6 and 8 waves per SIMD.
static int split_candidates(int64_t nmax, int* out) {
  static const int cand[6] = {1, 2, 4, 8, 12, 16};
  int c = 0;
  for (int w : cand)
    if (w <= MAXW && (w == 1 || nmax / w >= 64)) out[c++] = w;
  return c;
}
static const int OCC_CAND[3] = {4, 6, 8};
// The 6- and 8-wave register budgets spill part of k_eig's state to scratch
// (about 7 to 18 times the HBM bytes of the 4-wave variant at n = 32768):
// they are chosen only when at least 4 % faster, beyond the 2-3 % by which
// one shape's time moves between runs, not on timing noise.
static double occ_margin(int oc) { return oc > 4 ? 0.96 : 1.0; }

// Number of (problem, column group, row tile) blocks of the batched
// eigenvector launch with cb columns each, and its columns per block.
static int group_columns(int64_t np, int cb) {
  while (cb > VEC_C_MIN && cb * std::min<int64_t>(np, VEC_ROWS) > VEC_ELEMS) cb /= 2;
  return cb;
}
static int64_t group_blocks(int64_t np, int g) {  // (g a power of two: a plan may have many problems)
  return ((np + g - 1) >> __builtin_ctz(g)) * ((np + VEC_ROWS - 1) / VEC_ROWS);
}
static int64_t count_groups(int64_t nprob, const int64_t* offs, int cb) {
  int64_t c = 0;
  for (int64_t p = 0; p < nprob; ++p) {
    const int64_t np = offs[p + 1] - offs[p];
    c += group_blocks(np, group_columns(np, cb));
  }
  return c;
}
// The columns of a batch's blocks; full: the number of full ones, which becomes
// the number of blocks.
static int batch_columns(int64_t nprob, const int64_t* offs, int64_t& full) {
  int cb = VEC_C;
  while (cb > 4 && full < VEC_BLOCKS) full = count_groups(nprob, offs, cb /= 2);
  return cb;
}

// LDS of k_eig's cross-wave reductions: the widest, wg_sum<RED_NV>, stores
// RED_NV values per lane and wave.
constexpr int RED_NV = 4;
static size_t red_bytes(int W) { return W > 1 ? sizeof(double) * RED_NV * W * WAVE : 0; }

// Workspace of dpr1_eig_noalloc: a device array of the library, sized for the
// largest problem it accepts.  Every GPU holds its own copy for the life of
// the process; host code reaches it only through the address that
// hipGetSymbolAddress returns on that device (the name itself is a host-side
// stand-in, not a device address).
constexpr size_t NOALLOC_BYTES = layout_single(DPR1_NOALLOC_MAX_N).total;
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
static std::mutex scratch_mutex;
static void* scratch_ptr[NOALLOC_MAX_DEVICES];

// Device address of `scratch` on the current device, resolved once per device
// (nullptr on a HIP error or an out-of-range device index).
static void* scratch_on_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    scratch_ptr[dev] = p;
  }
  return scratch_ptr[dev];
}

}  // namespace dpr1

using namespace dpr1;

extern "C" {

void dpr1_default_opts(dpr1_opts* o) {
  o->mode_b = 0;
  o->root = 1;
  o->polish = 1;
  o->split = 0;
  o->kappa_polish = 16.0;
  o->nearzero = 10.0;
  o->main_passes = 0;
  o->waves_per_simd = 0;
  o->events = nullptr;
  o->vwrite = 0;
  o->remedy = 0;
  o->knu_thr = 32.0;
  o->knu = nullptr;
}

size_t dpr1_workspace_size(int64_t n) {
  if (n < 1) return 0;
  return layout_single(n).total;
}

#define HIPCHECK(x)                           \
  do {                                        \
    if ((x) != hipSuccess) return DPR1_EHIP;  \
  } while (0)

// Second stream of the current device for the overlapped eigenvector write:
// created once per device (default priority, non-blocking) and kept until the
// process ends; nullptr if it cannot be created.
constexpr int AUX_MAX_DEVICES = 64;
static std::mutex aux_mutex;
static hipStream_t aux_streams[AUX_MAX_DEVICES];
static hipStream_t aux_stream() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= AUX_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(aux_mutex);
  if (!aux_streams[dev]) {
    hipStream_t s = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return nullptr;
    aux_streams[dev] = s;
  }
  return aux_streams[dev];
}

static int launch_solve(const Layout& L, char* w, int64_t nprob, int64_t N, int64_t nmax, const int64_t* offs,
                        int64_t n_single, const double* d, const double* z, const double* rho_dev,
                        double rho_host, double* lambda, double* V, const int64_t* voffs, int64_t ldv,
                        int32_t* shift_idx, double* mu, double* xnorm, int32_t* info, int32_t* stats,
                        const dpr1_opts& o, int W, int64_t nitems, int persistent_grid, int64_t ngroups,
                        hipStream_t st, bool aux_ok = true) {
  Meta* meta = (Meta*)(w + L.meta);
  KArgs A;
  A.meta = meta;
  A.pairs = (const double*)(w + L.pairs);
  A.z2lo = (const double*)(w + L.z2lo);
  A.sd = (const double*)(w + L.sd);
  A.sz = (const double*)(w + L.sz);
  A.ii = (int32_t*)(w + L.ii);
  A.mu = (double*)(w + L.mu);
  A.xs = (double*)(w + L.xs);
  A.lam = (double*)(w + L.lam);
  A.fix = (FixItem*)(w + L.fix);
  A.vflag = (uint8_t*)(w + L.vflag);
  A.ctr = (int32_t*)(w + L.ctr);
  A.stats = stats;
  A.items = persistent_grid ? (const int4*)(w + L.items) : nullptr;
  const bool far = nmax >= FAR_MIN;
  A.far = far ? (const double*)(w + L.far) : nullptr;
  A.far_wide = far && !persistent_grid && far_wide_records(N) ? (int32_t)nitems : 0;
  A.far_slices = (int32_t)far_slices(N);
  A.far_min = FAR_MIN;
  A.nitems = (int32_t)nitems;
  A.nfixcap = (int32_t)N;
  A.W = W;
  A.mode_b = o.mode_b;
  A.root = o.root;
  A.polish = o.polish;
  A.kappa_polish = o.kappa_polish;
  A.nearzero = o.nearzero;
  // Default budget: two plain passes and the accurate one, which leave 0.2 to
  // 0.4 % of the roots to k_fix (one plain pass leaves 8 %: eigenvalues only
  // 99 against 101 us at n = 1501 but 2050 against 1230 us on the 2048-problem
  // mix; three cost 5 us at small orders and win nothing elsewhere).
  A.main_passes = o.main_passes > 0 ? o.main_passes : 3;
  A.remedy = o.remedy;
  A.knu_thr = o.knu_thr;
  A.knu = o.knu;

  A.lam_out = lambda;
  A.idx_out = shift_idx;
  A.mu_out = mu;
  A.xn_out = xnorm;
  A.info_out = info;
  A.V = V;
  A.voffs = voffs;
  A.ldv = ldv;
  A.csig = (double*)(w + L.csig);
  A.cinv = (double*)(w + L.cinv);

  const int nsplit = nprob == 1 ? (int)std::min<int64_t>(PREP_MAX_SPLIT, std::max<int64_t>(1, N / 512)) : 1;
  hipLaunchKernelGGL(k_prep, dim3((unsigned)(nsplit > 1 ? nsplit : nprob)), dim3(256), 0, st, (int)nprob, nsplit,
                     offs, n_single, d, z, rho_dev, rho_host, meta, (double*)A.sd, (double*)A.sz,
                     (double*)A.pairs, (double*)A.z2lo, info, (double*)(w + L.part), A.ctr,
                     stats);
  if (nsplit > 1)
    hipLaunchKernelGGL(k_meta, dim3(1), dim3(64), 0, st, nsplit, offs, n_single, rho_dev, rho_host,
                       (const double*)(w + L.part), meta, info);
  if (far) {
    FarArgs F;
    F.meta = meta;
    F.sd = A.sd;
    F.pairs = A.pairs;
    F.z2lo = A.z2lo;
    F.rec = (double*)(w + L.far);
    F.ng = (int32_t)nitems;
    F.wide = A.far_wide;
    F.slices = A.far_slices;
    F.items = A.items;
    F.hdr = (const FarHdr*)(w + L.ctr + FAR_HDR);
    F.work = w;
    const int64_t blocks = persistent_grid ? std::min<int64_t>(nitems, 2048) : far_grid(nitems + far_wide_records(N));
    hipLaunchKernelGGL(k_far, dim3((unsigned)blocks), dim3(FAR_BLK), 0, st, F);
  }
  HIPCHECK(hipGetLastError());
  hipEvent_t* ev = (hipEvent_t*)o.events;
  VArgs va;
  va.meta = meta;
  va.sd = A.sd;
  va.sz = A.sz;
  va.mu = A.mu;
  va.csig = A.csig;
  va.cinv = A.cinv;
  va.vflag = A.vflag;
  va.V = V;
  va.voffs = voffs;
  va.ldv = ldv;
  va.cbase = 0;
  va.cend = (int32_t)N;
  va.prio = 0;
  va.n = (int32_t)N;
  va.neg = rho_dev ? -1 : rho_host < 0;
  // one problem: some column starts off a 128-byte line
  const bool shift = ((uintptr_t)V & (8 * LINE - 1)) != 0 || ldv % LINE != 0;
  auto launch_eig = [&](unsigned grid, int g0, int occ) {
    A.g0 = g0;
    switch (occ) {
      case 6: hipLaunchKernelGGL(k_eig<6>, dim3(grid), dim3(64 * W), red_bytes(W), st, A); break;
      case 8: hipLaunchKernelGGL(k_eig<8>, dim3(grid), dim3(64 * W), red_bytes(W), st, A); break;
      default: hipLaunchKernelGGL(k_eig<4>, dim3(grid), dim3(64 * W), red_bytes(W), st, A); break;
    }
  };
  // K_nu of every eigenpair and, with opts.remedy, the remedies (after every
  // eigenpair and column is final, on `stream`)
  auto launch_knu = [&]() {
    if (!o.knu && !o.remedy && !stats) return;  // nobody reads it
    hipLaunchKernelGGL(k_knu, dim3(nprob > 1 ? (unsigned)nprob : (unsigned)std::min<int64_t>((N + 255) / 256, 1024)),
                       dim3(256), 0, st, A, (int)nprob);
    if (o.remedy)
      hipLaunchKernelGGL(k_remedy, dim3((unsigned)std::min<int64_t>(std::max<int64_t>(N / 16, 1), 2048)),
                         dim3(FIXT), 0, st, A);
  };
  auto launch_vec = [&](int64_t cb, int64_t ce, hipStream_t s2, bool prio) {
    VArgs vb = va;
    vb.cbase = (int32_t)cb;
    vb.cend = (int32_t)ce;
    vb.prio = prio ? 1 : 0;
    const dim3 grid((unsigned)tile_blocks(N, ce - cb));
    if (shift)
      hipLaunchKernelGGL(k_vec<true>, grid, dim3(VEC_T), VEC_PAD, s2, vb);
    else
      hipLaunchKernelGGL(k_vec<false>, grid, dim3(VEC_T), VEC_PAD, s2, vb);
  };

  // A single problem with eigenvectors and opts.vwrite = K >= 2: the
  // eigenvalue kernel runs in K launches over consecutive chunks of its
  // groups of 64 eigenvalues, and the columns of chunk c are written on a
  // second stream while chunk c + 1 is solved, so that the HBM-bound stores
  // overlap the ALU-bound sweeps; the last chunk's columns are written beside
  // k_fix.  Flagged columns are left to k_fix, as in the sequential path.
  // The default (0 or 1) writes V after the eigenvalue kernel, which measured
  // faster at every order tried (n = 8192 .. 65536) since the address-ordered
  // writer; below 8192 eigenpairs the write is short and the fork costs more
  // than it hides in any case.
  const int nchunks = o.vwrite <= 1 ? 1 : o.vwrite;
  bool overlap = V && !persistent_grid && nchunks >= 2 && aux_ok && N >= 8192 && nitems >= nchunks;
  hipStream_t st2 = overlap ? aux_stream() : nullptr;
  if (overlap && !st2) overlap = false;
  if (overlap) {
    hipEvent_t evs[VEC_CHUNKS_MAX + 1];
    int nev = 0, rc = DPR1_OK;
    for (; nev <= nchunks; ++nev)
      if (hipEventCreateWithFlags(&evs[nev], hipEventDisableTiming) != hipSuccess) {
        rc = DPR1_EHIP;
        break;
      }
    if (rc == DPR1_OK && ev && hipEventRecord(ev[0], st) != hipSuccess) rc = DPR1_EHIP;
    for (int c = 0; c < nchunks && rc == DPR1_OK; ++c) {
      const int64_t ga = nitems * c / nchunks, gb = nitems * (c + 1) / nchunks;
      const int64_t ka = ga * WAVE, kb = std::min<int64_t>(gb * WAVE, N);
      // the chunks solved beside the writer take at least the 6-wave register
      // budget, so that writer waves fit next to a 16-wave block
      launch_eig((unsigned)(gb - ga), (int)ga, c == 0 ? occ_of(o) : std::max(occ_of(o), 6));
      if (c == nchunks - 1 && ev && hipEventRecord(ev[1], st) != hipSuccess) rc = DPR1_EHIP;
      if (hipGetLastError() != hipSuccess || hipEventRecord(evs[c], st) != hipSuccess ||
          hipStreamWaitEvent(st2, evs[c], 0) != hipSuccess)
        rc = DPR1_EHIP;
      if (rc == DPR1_OK) launch_vec(ka, kb, st2, c < nchunks - 1);
    }
    if (rc == DPR1_OK && ev && hipEventRecord(ev[2], st) != hipSuccess) rc = DPR1_EHIP;
    if (rc == DPR1_OK) {
      unsigned fgrid = (unsigned)std::min<int64_t>(std::max<int64_t>(N, 1), 2048);
      hipLaunchKernelGGL(k_fix, dim3(fgrid), dim3(FIXT), 0, st, A);
      if (hipGetLastError() != hipSuccess || hipEventRecord(evs[nchunks], st2) != hipSuccess ||
          hipStreamWaitEvent(st, evs[nchunks], 0) != hipSuccess || (ev && hipEventRecord(ev[3], st) != hipSuccess))
        rc = DPR1_EHIP;
    }
    if (rc == DPR1_OK) {
      launch_knu();
      if (hipGetLastError() != hipSuccess) rc = DPR1_EHIP;
    }
    for (int e = 0; e < nev; ++e) (void)hipEventDestroy(evs[e]);
    return rc;
  }

  unsigned grid = persistent_grid ? (unsigned)persistent_grid : (unsigned)nitems;
  if (ev) HIPCHECK(hipEventRecord(ev[0], st));
  launch_eig(grid, 0, occ_of(o));
  HIPCHECK(hipGetLastError());
  if (ev) HIPCHECK(hipEventRecord(ev[1], st));
  if (ev) HIPCHECK(hipEventRecord(ev[2], st));
  if (V) {
    // k_fix overlapped with the eigenvector writer: a few blocks take the
    // flagged eigenpairs, the rest write every other column
    if (persistent_grid) {
      va.groups = (const int4*)(w + L.groups);
      const bool few = batch_few(nprob, N, ngroups);
      const int nfix = few ? BATCH_HEAD : FIX_BATCH, ntail = few ? BATCH_TAIL : 0;
      hipLaunchKernelGGL(k_fixvec<VEC_BATCH>, dim3((unsigned)(nfix + ngroups + ntail)), dim3(VEC_T), 0, st, A, va,
                         nfix, ntail);
    } else {
      const int64_t tiles = tile_blocks(N, N);
      const bool many = tiles > FIX_RESIDENT;
      const int nfix = many ? FIX_HEAD : FIX_SMALL, ntail = many ? FIX_TAIL : 0;
      const dim3 grid((unsigned)(nfix + tiles + ntail));
      if (shift)
        hipLaunchKernelGGL(k_fixvec<VEC_SHIFTED>, grid, dim3(VEC_T), 0, st, A, va, nfix, ntail);
      else
        hipLaunchKernelGGL(k_fixvec<VEC_ALIGNED>, grid, dim3(VEC_T), 0, st, A, va, nfix, ntail);
    }
  } else {
    unsigned fgrid = (unsigned)std::min<int64_t>(std::max<int64_t>(N, 1), 2048);
    hipLaunchKernelGGL(k_fix, dim3(fgrid), dim3(FIXT), 0, st, A);
  }
  HIPCHECK(hipGetLastError());
  if (ev) HIPCHECK(hipEventRecord(ev[3], st));
  launch_knu();
  HIPCHECK(hipGetLastError());
  return DPR1_OK;
}

int dpr1_eig(const double* d, const double* z, double rho, int64_t n, double* lambda, double* V, int64_t ldv,
             int32_t* shift_idx, double* mu, double* xnorm, int32_t* info, int32_t* stats,
             const dpr1_opts* opts, void* work, size_t work_bytes, void* stream) {
  if (!d) return -1;
  if (!z) return -2;
  if (!(rho == rho) || rho == 0.0 || rho == INFINITY || rho == -INFINITY) return -3;
  if (n < 1 || n > (int64_t)INT32_MAX / 2) return -4;
  if (!lambda) return -5;
  if (V && ldv < n) return -7;
  if (!info) return -11;
  Layout L = layout_single(n);
  if (!work) return -14;
  if (work_bytes < L.total) return -15;
  dpr1_opts o;
  fill_opts(opts, &o);
  if (!occ_valid(o.waves_per_simd) || o.vwrite < 0 || o.vwrite > VEC_CHUNKS_MAX || o.mode_b < 0 || o.mode_b > 3)
    return -13;
  int64_t nblocks = (n + WAVE - 1) / WAVE;
  int W = o.split > 0 ? std::min(o.split, MAXW) : pick_split(nblocks, n);
  return launch_solve(L, (char*)work, 1, n, n, nullptr, n, d, z, nullptr, rho, lambda, V, nullptr, ldv, shift_idx,
                      mu, xnorm, info, stats, o, W, nblocks, 0, 0, (hipStream_t)stream);
}

size_t dpr1_noalloc_scratch_bytes(void) { return NOALLOC_BYTES; }

// dpr1_eig on the library's static device scratch instead of a workspace
// argument: the same checks, kernels and results; no allocation of any kind.
int dpr1_eig_noalloc(const double* d, const double* z, double rho, int64_t n, double* lambda, double* V,
                     int64_t ldv, int32_t* shift_idx, double* mu, double* xnorm, int32_t* info, int32_t* stats,
                     const dpr1_opts* opts, void* stream) {
  if (!d) return -1;
  if (!z) return -2;
  if (!(rho == rho) || rho == 0.0 || rho == INFINITY || rho == -INFINITY) return -3;
  if (n < 1) return -4;
  if (n > DPR1_NOALLOC_MAX_N) return DPR1_ETOOBIG;
  if (!lambda) return -5;
  if (V && ldv < n) return -7;
  if (!info) return -11;
  dpr1_opts o;
  fill_opts(opts, &o);
  if (!occ_valid(o.waves_per_simd) || o.vwrite < 0 || o.vwrite > VEC_CHUNKS_MAX || o.mode_b < 0 || o.mode_b > 3)
    return -13;
  void* work = scratch_on_current_device();
  if (!work) return DPR1_EHIP;
  const Layout L = layout_single(n);
  int64_t nblocks = (n + WAVE - 1) / WAVE;
  int W = o.split > 0 ? std::min(o.split, MAXW) : pick_split(nblocks, n);
  return launch_solve(L, (char*)work, 1, n, n, nullptr, n, d, z, nullptr, rho, lambda, V, nullptr, ldv, shift_idx,
                      mu, xnorm, info, stats, o, W, nblocks, 0, 0, (hipStream_t)stream,
                      /*aux_ok=*/false);
}

// ------------------------------------------------------------ batched
size_t dpr1_batched_workspace_size(int64_t nprob, const int64_t* offs_host) {
  if (nprob < 1 || !offs_host || offs_host[0] != 0) return 0;
  for (int64_t p = 0; p < nprob; ++p)
    if (offs_host[p + 1] - offs_host[p] < 1) return 0;
  int64_t nmax = 0;
  for (int64_t p = 0; p < nprob; ++p) nmax = std::max(nmax, offs_host[p + 1] - offs_host[p]);
  return layout_batch(nprob, offs_host[nprob], nmax, count_groups(nprob, offs_host, VEC_C)).total;
}

int dpr1_batched_plan(int64_t nprob, const int64_t* offs_host, const dpr1_opts* opts, dpr1_plan* plan,
                      void* work, size_t work_bytes, void* stream) {
  if (nprob < 1 || nprob > (1 << 24)) return -1;
  if (!offs_host) return -2;
  if (!plan) return -4;
  if (!work) return -5;
  if (offs_host[0] != 0) return -2;
  int64_t nmax = 0;
  for (int64_t p = 0; p < nprob; ++p) {
    int64_t np = offs_host[p + 1] - offs_host[p];
    if (np < 1 || np > (int64_t)INT32_MAX / 2) return -2;
    nmax = std::max(nmax, np);
  }
  int64_t N = offs_host[nprob];
  if (N > (int64_t)INT32_MAX) return -2;
  int64_t ngroups = count_groups(nprob, offs_host, VEC_C);
  const Layout L0 = layout_batch(nprob, N, nmax, ngroups);
  if (work_bytes < L0.total) return -6;
  dpr1_opts o;
  fill_opts(opts, &o);
  if (!occ_valid(o.waves_per_simd) || o.mode_b < 0 || o.mode_b > 3) return -3;
  // longest-processing-time order: larger problems first
  std::vector<int32_t> order(nprob);
  for (int64_t p = 0; p < nprob; ++p) order[p] = (int32_t)p;
  const auto larger = [&](int32_t a, int32_t b) {
    return offs_host[a + 1] - offs_host[a] > offs_host[b + 1] - offs_host[b];
  };
  if (!std::is_sorted(order.begin(), order.end(), larger)) std::stable_sort(order.begin(), order.end(), larger);
  // the queue, and the far-field records: item e's own record is e, the wide
  // level's lie behind the queue's
  std::vector<int4> items, witems;
  items.reserve(batch_items(nprob, N));
  FarHdr hdr{0, 0, (int64_t)L0.witems};
  const int64_t rec0 = far_batch_own(N, nmax, batch_items(nprob, N));
  for (int32_t p : order) {
    const int64_t np = offs_host[p + 1] - offs_host[p];
    const int nsl = np >= FAR_MIN2 ? (int)far_slices(np) : 1;
    const int64_t w0 = rec0 + (int64_t)witems.size();
    if (np >= FAR_MIN2)
      for (int64_t k0 = 0; k0 < np; k0 += FAR_WIDE * WAVE)
        for (int sl = 0; sl < nsl; ++sl)
          witems.push_back(make_int4(p, (int)k0, sl | nsl << 16, (int)(rec0 + (int64_t)witems.size())));
    for (int64_t k0 = 0; k0 < np; k0 += WAVE)
      items.push_back(make_int4(p, (int)k0, np >= FAR_MIN2 ? (int)(w0 + k0 / (FAR_WIDE * WAVE) * nsl) : -1, nsl));
    if (np >= FAR_MIN) hdr.nown = (int64_t)items.size();
  }
  const int64_t nwide = hdr.nwide = (int64_t)witems.size();
  int64_t nitems = (int64_t)items.size();
  int W = o.split > 0 ? std::min(o.split, MAXW) : pick_split(nitems, nmax);
  // the eigenvector kernel's blocks
  const int cb = batch_columns(nprob, offs_host, ngroups);
  const bool on_host = ngroups <= PLAN_HOST;
  // [far header, problems, items, wide items, groups] in one copy: each from
  // pageable memory costs some 15 us (a tridiagonal solve of n = 4096, a plan
  // per depth, 3310 us with three, 3255 with one; n = 300 823 and 785)
  const size_t h0 = L0.ctr + FAR_HDR;
  const size_t bytes = (on_host ? L0.groups + sizeof(int4) * ngroups
                        : nwide ? L0.witems + sizeof(int4) * nwide
                                : L0.items + sizeof(int4) * nitems) - h0;
  std::unique_ptr<char[]> mir(new char[bytes]);
  memcpy(mir.get(), &hdr, sizeof hdr);
  memcpy(mir.get() + (L0.items - h0), items.data(), sizeof(int4) * nitems);
  if (nwide) memcpy(mir.get() + (L0.witems - h0), witems.data(), sizeof(int4) * nwide);
  int4* prob = (int4*)(mir.get() + (L0.prob - h0));
  int4* groups = (int4*)(mir.get() + (on_host ? L0.groups - h0 : 0));
  int64_t g0 = 0;
  for (int32_t p = 0; p < nprob; ++p) {
    const int64_t np = offs_host[p + 1] - offs_host[p];
    const int g = group_columns(np, cb);
    if (on_host) {
      for (int64_t c0 = 0; c0 < np; c0 += g)
        for (int64_t r0 = 0; r0 < np; r0 += VEC_ROWS)
          *groups++ = make_int4(p, (int)c0, (int)std::min<int64_t>(g, np - c0), (int)r0);
    } else {
      prob[p] = make_int4((int)g0, g, (int)np, 0);
      g0 += group_blocks(np, g);
    }
  }
  hipStream_t st = (hipStream_t)stream;
  HIPCHECK(hipMemcpyAsync((char*)work + h0, mir.get(), bytes, hipMemcpyHostToDevice, st));
  if (!on_host && ngroups <= INT32_MAX)  // beyond (64 kB a block) no V fits any memory
    hipLaunchKernelGGL(k_plan_groups, dim3((unsigned)((ngroups + 255) / 256)), dim3(256), 0, st, (int)nprob,
                       (int)ngroups, (const int4*)((char*)work + L0.prob), (int4*)((char*)work + L0.groups));
  const bool launched = hipGetLastError() == hipSuccess;
  if (hipStreamSynchronize(st) != hipSuccess || !launched) return DPR1_EHIP;
  plan->ngroups = ngroups;
  plan->nprob = nprob;
  plan->ntotal = N;
  plan->nitems = nitems;
  plan->nmax = nmax;
  plan->split = W;
  plan->grid = persistent_grid_for(nitems, W, occ_of(o));
  plan->opts = o;
  return DPR1_OK;
}

int dpr1_eig_batched(const dpr1_plan* plan, const int64_t* offs, const double* d, const double* z,
                     const double* rho, double* lambda, double* V, const int64_t* voffs, int32_t* shift_idx,
                     double* mu, double* xnorm, int32_t* info, int32_t* stats, void* work, size_t work_bytes,
                     void* stream) {
  if (!plan || plan->nprob < 1) return -1;
  if (!offs) return -2;
  if (!d) return -3;
  if (!z) return -4;
  if (!rho) return -5;
  if (!lambda) return -6;
  if (V && !voffs) return -8;
  if (!info) return -12;
  if (!work) return -14;
  const Layout L = layout_batch(plan->nprob, plan->ntotal, plan->nmax, plan->ngroups);
  if (work_bytes < L.total) return -15;
  return launch_solve(L, (char*)work, plan->nprob, plan->ntotal, plan->nmax, offs, 0, d, z, rho, 0.0, lambda, V, voffs, 0,
                      shift_idx, mu, xnorm, info, stats, plan->opts, plan->split, plan->nitems, plan->grid,
                      plan->ngroups, (hipStream_t)stream);
}

// Autotuning: every candidate (split, occupancy variant, pass budget) is
// timed on the caller's data and the fastest kept; ties keep the earlier
// candidate.
int dpr1_autotune(const double* d, const double* z, double rho, int64_t n, double* lambda, double* V,
                  int64_t ldv, int32_t* shift_idx, double* mu, double* xnorm, int32_t* info, dpr1_opts* opts,
                  int32_t reps, double* best_ms, void* work, size_t work_bytes, void* stream) {
  if (!opts) return -12;
  if (reps < 0) return -13;
  if (reps == 0) reps = 3;
  dpr1_opts o;
  fill_opts(opts, &o);
  o.events = nullptr;
  int ws[8];
  const int nw = split_candidates(n, ws);
  const int passes[2] = {2, 3};
  const int np = o.root == 1 ? 2 : 1;
  // with eigenvectors at n >= 8192 also the write: after the eigenvalue
  // kernel (0) or overlapped in two chunks (2)
  const int vws[2] = {0, 2};
  const int nv = (V && n >= 8192) ? 2 : 1;
  double best = INFINITY;
  int bw = ws[0], bp = o.main_passes, bo = 4, bv = o.vwrite;
  for (int a = 0; a < nw; ++a)
    for (int oc : OCC_CAND)
      for (int b = 0; b < np; ++b)
        for (int e = 0; e < nv; ++e) {
        dpr1_opts c = o;
        c.split = ws[a];
        c.waves_per_simd = oc;
        if (o.root == 1) c.main_passes = passes[b];
        if (nv > 1) c.vwrite = vws[e];
        double ms = 0.0;
        int rc = time_calls([&]() { return dpr1_eig(d, z, rho, n, lambda, V, ldv, shift_idx, mu, xnorm, info,
                                                    nullptr, &c, work, work_bytes, stream); },
                            reps, (hipStream_t)stream, &ms);
        if (rc != 0) return rc;
        if (ms < best * occ_margin(oc)) {
          best = ms;
          bw = c.split;
          bp = c.main_passes;
          bo = oc;
          bv = c.vwrite;
        }
      }
  opts->split = bw;
  opts->main_passes = bp;
  opts->waves_per_simd = bo;
  opts->vwrite = bv;
  if (best_ms) *best_ms = best;
  return DPR1_OK;
}

int dpr1_batched_autotune(dpr1_plan* plan, const int64_t* offs, const double* d, const double* z,
                          const double* rho, double* lambda, double* V, const int64_t* voffs,
                          int32_t* shift_idx, double* mu, double* xnorm, int32_t* info, int32_t reps,
                          double* best_ms, void* work, size_t work_bytes, void* stream) {
  if (!plan || plan->nprob < 1) return -1;
  if (reps < 0) return -13;
  if (reps == 0) reps = 3;
  const dpr1_plan base = *plan;
  int ws[8];
  const int nw = split_candidates(base.nmax, ws);
  const int passes[3] = {2, 3, 4};
  const int np = base.opts.root == 1 ? 3 : 1;
  double best = INFINITY;
  dpr1_plan bestp = base;
  for (int a = 0; a < nw; ++a)
    for (int oc : OCC_CAND)
      for (int b = 0; b < np; ++b) {
        dpr1_plan c = base;
        c.split = ws[a];
        c.opts.waves_per_simd = oc;
        c.grid = persistent_grid_for(c.nitems, ws[a], oc);
        c.opts.events = nullptr;
        if (base.opts.root == 1) c.opts.main_passes = passes[b];
        double ms = 0.0;
        int rc = time_calls([&]() { return dpr1_eig_batched(&c, offs, d, z, rho, lambda, V, voffs, shift_idx, mu,
                                                            xnorm, info, nullptr, work, work_bytes, stream); },
                            reps, (hipStream_t)stream, &ms);
        if (rc != 0) return rc;
        if (ms < best * occ_margin(oc)) {
          best = ms;
          bestp = c;
        }
      }
  bestp.opts.events = base.opts.events;
  *plan = bestp;
  if (best_ms) *best_ms = best;
  return DPR1_OK;
}

const char* dpr1_strerror(int code) {
  switch (code) {
    case DPR1_OK: return "ok";
    case DPR1_EHIP: return "a HIP runtime call or kernel launch failed";
    case DPR1_ETOOBIG: return "n exceeds DPR1_NOALLOC_MAX_N, the size of the static scratch of dpr1_eig_noalloc";
    case DPR1_INFO_UNSORTED: return "info: d is not strictly decreasing";
    case DPR1_INFO_ZERO_Z: return "info: some z_j is zero (reducible problem)";
    case DPR1_INFO_NONFINITE: return "info: non-finite input";
    case DPR1_INFO_BAD_RHO: return "info: rho is zero or not finite";
    case DPR1_INFO_RANGE: return "info: a shifted representation left the binary64 range";
    default: return code < 0 ? "invalid argument (see the argument position -code)" : "unknown code";
  }
}

}  // extern "C"
