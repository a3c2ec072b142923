// Front end for reducible inputs (Sec. 1 of the paper): any finite d (any
// order, repeated values) and any finite z (zeros allowed); and the Hermitian
// case A = D + rho z z^H with complex z, which a diagonal unitary similarity
// turns into the real problem with |z| (the extension the paper's closing
// remarks mention).
//
// The reduction: sort the poles decreasingly, deflate a pole whose z_j is zero
// (eigenpair (d_j, e_j)), and merge a group of equal poles by a Householder
// reflection of its block that maps its part w of z onto a multiple of e_first:
// the pole enters the reduced problem once, with z = ||w||, and the other
// columns of the reflection are eigenvectors for the same eigenvalue.  The
// reduced problem (strictly decreasing, no zero z) is solved by dpr1_eig
// without eigenvectors; k_front_columns orders its eigenvalues among the
// deflated poles and k_assemble writes every column of V in the caller's row
// order.  All of it runs on the GPU; the host reads back the reduced problem's
// order, on which the solver's launches depend.  (On the host, with the copies
// there and back, the reduction and the ordering took 1.1 ms at n = 32768 and
// 0.3 ms at n = 4099, complex z.)
//
// A column k of the reduced problem needs no gather: in the caller's rows its
// components are those of eq. (eigenvecAi) evaluated on the original d and z,
//   v_k[i] = z_i / (((d_i - sigma_k) - mu_k) ||x_k||),
// because a member i of a merged group has d_i = the group's pole and carries
// z_i = (w_i / ||w||) ||w||, and a deflated row has z_i = 0.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "../../include/dpr1.h"
#define DPR1_HD __device__ __forceinline__
#include "columns.h"

namespace dpr1 {
namespace gen {

// Per original row i: rgrp its group id, rpos its position in the group, ru
// the reflection vector's component there (0 for groups without reflection).
// Per final column c, an eigenvector of the reduced problem (cgrp = -1):
//   csig = sigma_k (the shift pole), cmu = mu_k, cic = 1 / ||x_k||
// or a column of the reduction, column ct of the reflection of group cgrp:
//   cub = beta u_t (0 for a deflated pole: a unit vector)
struct AsmArgs {
  int64_t n, ldv;
  const double* d;
  const double* z;
  const int32_t* rgrp;
  const int32_t* rpos;
  const double* ru;
  const int32_t* cgrp;
  const int32_t* ct;
  const double* csig;
  const double* cmu;
  const double* cic;
  const double* cub;
  const double* ph;  // [2n] unit phases z_i / |z_i| (Hermitian case), else null
  double* V;
};

__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// A block writes ASM_T E rows of ASM_C columns in 16-byte streaming stores, E
// rows a thread (a complex element fills 16 bytes), and ends; blocks go down
// the columns first, in memory order, 5 to a CU (ASM_LDS bytes of LDS each,
// more than they use), which holds the GPU's write front together as the eigenvector
// writer's tiles do.  A column's windows are shifted back to whole 128-byte
// lines, by up to LINE - 1 rows; the block keeps what it needs of the rows
// that it may meet in LDS, and the last row range also writes the rows behind its window.
// Bound by HBM writes.  A call, against 2048 waves that loop over columns: n =
// 32768 1890 us (1925), 32767 1853 (2845), 16000 665 (711), 16001 706 (893),
// complex n = 4099 281 (293).  8 columns 2 to 5 % slower, 12 and 16 more.
// CPLX: V is complex (interleaved re, im; element (i, c) at 2 (i + c ldv)) and
// row i is multiplied by the phase of z_i.
constexpr int ASM_T = 256, ASM_C = 6;
constexpr size_t ASM_LDS = 30 << 10;

typedef double dbl2 __attribute__((ext_vector_type(2)));

template <bool CPLX>
__global__ void __launch_bounds__(ASM_T) k_assemble(AsmArgs a, int rtiles) {
  constexpr int E = CPLX ? 1 : 2, ROWS = ASM_T * E, LINE = 16 / (CPLX ? 2 : 1), NB = ROWS + 2 * LINE;
  __shared__ double ld_d[NB], ld_z[NB], ld_u[NB];
  __shared__ int2 ld_g[NB];
  __shared__ dbl2 ld_p[CPLX ? NB : 1];
  const int t = threadIdx.x, r = (int)(blockIdx.x % rtiles);
  const int64_t n = a.n, r0 = (int64_t)r * ROWS, c0 = (int64_t)(blockIdx.x / rtiles) * ASM_C;
  double sg[ASM_C], mu[ASM_C], ic[ASM_C], ub[ASM_C];
  int grp[ASM_C], ct[ASM_C];
#pragma unroll
  for (int u = 0; u < ASM_C; ++u) {
    const int64_t c = min(c0 + u, n - 1);
    sg[u] = a.csig[c];
    mu[u] = a.cmu[c];
    ic[u] = a.cic[c];
    ub[u] = a.cub[c];
    grp[u] = a.cgrp[c];
    ct[u] = a.ct[c];
  }
  for (int i = t; i < NB - 1; i += ASM_T) {
    const int64_t at = r0 - (LINE - 1) + i;
    const bool in = at >= 0 && at < n;
    ld_d[i] = in ? a.d[at] : 0.0;
    ld_z[i] = in ? a.z[at] : 0.0;
    ld_u[i] = in ? a.ru[at] : 0.0;
    ld_g[i] = in ? int2{a.rgrp[at], a.rpos[at]} : int2{-2, 0};
    if (CPLX) ld_p[i] = in ? *(const dbl2*)(a.ph + 2 * at) : dbl2{0.0, 0.0};
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < ASM_C; ++u) {
    if (c0 + u >= n) break;
    double* col = a.V + (CPLX ? 2 : 1) * (c0 + u) * a.ldv;
    const int s = (int)(((uintptr_t)col / (CPLX ? 16 : 8)) & (LINE - 1));
    auto value = [&](int i) {
      // mu / den with one residual correction, then the scaled norm; a row
      // with z_i == 0 (deflated, or a zero member of a merged group) is
      // exactly 0 whatever den is
      const double den = (ld_d[i] - sg[u]) - mu[u];
      const double rc = rcp_nr(den), z = ld_z[i];
      double w = ic[u] * rc;
      w = __builtin_fma(__builtin_fma(-w, den, ic[u]), rc, w);
      double v = z != 0.0 ? z * w : 0.0;
      if (grp[u] >= 0) {
        // column ct of H = I - beta u u^T restricted to the group
        const int2 g = ld_g[i];
        v = g.x == grp[u] ? (g.y == ct[u] ? 1.0 : 0.0) - ub[u] * ld_u[i] : 0.0;
      }
      return v;
    };
    auto put = [&](int i, int64_t at, double v) {  // one row, entry i of LDS
      if (at < 0 || at >= n) return;
      if (CPLX) {
        const dbl2 cv = {v * ld_p[i].x, v * ld_p[i].y};
        __builtin_nontemporal_store(cv, (dbl2*)(col + 2 * at));
      } else {
        __builtin_nontemporal_store(v, col + at);
      }
    };
    const int i = LINE - 1 - s + E * t;
    const int64_t at = r0 - s + E * t;
    const double v0 = value(i);
    if (CPLX) {
      put(i, at, v0);
    } else {
      const double v1 = value(i + 1);
      const dbl2 v = {v0, v1};
      if (at >= 0 && at + 1 < n) {
        __builtin_nontemporal_store(v, (dbl2*)(col + at));
      } else {
        put(i, at, v0);
        put(i + 1, at + 1, v1);
      }
    }
    if (r == rtiles - 1 && t < LINE) {
      const int q = LINE - 1 - s + ROWS + t;
      put(q, r0 + ROWS - s + t, value(q));
    }
  }
}

// ------------------------------------------------------------- reduction
// Sort: runs of FR rows by rank counting in LDS (all pairs of a run, 0.5 M
// comparisons a block), then FW runs at a time by binary searches in lock step
// (an element's place is its own index plus its rank in each of the other
// runs: FW independent loads a step, so a pass costs about as many load
// latencies as a merge of two runs would).  A block first takes FS samples of
// each run to LDS: only the steps between two samples, next to each other in
// memory, are loads (n = 32768: 36 us for
// the two passes, 59 with every step a load).  Keys
// are the poles as integers that increase as the poles decrease (-0 as +0, any
// NaN in some place, so that the order is a permutation whatever the input);
// equal poles keep their row order.
constexpr int FR = 512, FW = 16, FS = 128;

__device__ __forceinline__ uint64_t pole_key(double x) {
  const uint64_t b = x == 0.0 ? 0 : (uint64_t)__double_as_longlong(x);
  return ~((b >> 63) ? ~b : (b | ((uint64_t)1 << 63)));
}

// Block b also leaves in bad[b] whether one of its rows is not finite, and
// writes the deflated z: |z_j| < 2^-511 counts as zero (its square is not a
// normal number, and the eigenvalue beside d_j would lie within rho z_j^2 of
// it).  CPLX: z is complex; with Phi = diag(z_j / |z_j|) unitary (1 where z_j =
// 0) Phi D Phi^H = D, A = Phi (D + rho |z| |z|^T) Phi^H, so the eigenvalues are
// those of the real problem with |z| and v = Phi v_real.
template <bool CPLX>
__global__ void __launch_bounds__(FR) k_front_sort(const double* d, const double* z, int64_t n, double* zd,
                                                   double* ph, uint64_t* key, int32_t* idx, int32_t* bad) {
  __shared__ uint64_t s[FR];
  const int t = threadIdx.x;
  const int64_t b0 = (int64_t)blockIdx.x * FR, i = b0 + t;
  const bool in = i < n;
  uint64_t k = ~(uint64_t)0;  // rows beyond the last: behind every row
  bool ok = true;
  if (in) {
    const double x = d[i];
    k = pole_key(x);
    ok = isfinite(x);
    double r;
    if (CPLX) {
      const double re = z[2 * i], im = z[2 * i + 1];
      ok = ok && isfinite(re) && isfinite(im);
      r = hypot(re, im);
      ph[2 * i] = r > 0.0 ? re / r : 1.0;
      ph[2 * i + 1] = r > 0.0 ? im / r : 0.0;
    } else {
      r = z[i];
      ok = ok && isfinite(r);
    }
    zd[i] = fabs(r) < 0x1p-511 ? 0.0 : r;
  }
  s[t] = k;
  const int any = __syncthreads_or(!ok);
  if (t == 0) bad[blockIdx.x] = any;
  const int w0 = t & ~63;
  int rank = 0;
  for (int j = 0; j < w0; ++j) rank += s[j] <= k;
  for (int j = w0; j < w0 + 64; ++j) rank += s[j] < k || (s[j] == k && j < t);
  for (int j = w0 + 64; j < FR; ++j) rank += s[j] < k;
  if (in) {
    key[b0 + rank] = k;
    idx[b0 + rank] = (int32_t)i;
  }
}

// One pass: every FW runs of `len` (FR FW^p) rows become one.
__global__ void __launch_bounds__(256) k_front_merge(int64_t n, int64_t len, const uint64_t* key, const int32_t* idx,
                                                     uint64_t* key2, int32_t* idx2) {
  const int64_t b0 = (int64_t)blockIdx.x * 256;  // one run: len is a multiple of 256
  const int64_t run = b0 / len, base = run / FW * FW * len;
  const int r = (int)(run % FW);
  const int64_t i = b0 + threadIdx.x;
  const int stride = (int)(len / FS);
  __shared__ uint64_t smp[FW][FS];
  __shared__ int cnt[FW];  // rows of the run
  if (threadIdx.x < FW)
    cnt[threadIdx.x] = (int)min(max(n - (base + threadIdx.x * len), (int64_t)0), len);
  for (int e = threadIdx.x; e < FW * FS; e += 256) {
    const int64_t at = base + (e / FS) * len + (int64_t)(e % FS + 1) * stride - 1;
    smp[e / FS][e % FS] = at < n ? key[at] : ~(uint64_t)0;
  }
  __syncthreads();
  if (i >= n) return;
  const uint64_t k = key[i];
  int lo[FW];
#pragma unroll
  for (int q = 0; q < FW; ++q) lo[q] = 0;
  // samples that lie before k, then the rows between two samples
  for (int h = FS; h > 0; h >>= 1) {
#pragma unroll
    for (int q = 0; q < FW; ++q) {
      const int at = lo[q] + h;
      const uint64_t x = smp[q][min(at, FS) - 1];
      if (at <= cnt[q] / stride && (x < k || (x == k && q < r))) lo[q] = at;
    }
  }
#pragma unroll
  for (int q = 0; q < FW; ++q) lo[q] *= stride;
  for (int h = stride / 2; h > 0; h >>= 1) {
#pragma unroll
    for (int q = 0; q < FW; ++q) {
      const int at = lo[q] + h;
      const bool inside = at <= cnt[q];
      if (!inside) continue;
      const uint64_t x = key[base + q * len + at - 1];
      if (x < k || (x == k && q < r)) lo[q] = at;
    }
  }
  int64_t pos = i - (base + r * len);
#pragma unroll
  for (int q = 0; q < FW; ++q)
    if (q != r) pos += lo[q];
  key2[base + pos] = k;
  idx2[base + pos] = idx[i];
}

// What the reduction leaves for the host and for k_front_columns.
struct FrontHdr {
  int32_t m, bad;  // order of the reduced problem; an input is not finite
};

__device__ __forceinline__ double wave_sum(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Groups of equal poles, in sorted positions.  A group of at most FT is taken by
// the thread of its first position, a larger one by that thread's wave, 256
// members in flight at a time (n = 32768 with pairs among the poles: 39 us with
// every group by a wave, 6 so): the largest |w_t|, ||w|| scaled by it (no square
// overflows), then u = w/||w|| + sign(u_first) e_first and beta = 2/(u^T u).
// Per row: rgrp (the group's first position), rpos, ru; per group, at its first
// position: gnw = ||w|| (z itself for a pole alone), gbeta.  cnt[b] = poles of
// block b's positions that enter the reduced problem.
constexpr int FT = 8;
constexpr int FG = 4;  // members a lane has in flight
__global__ void __launch_bounds__(FR) k_front_groups(int64_t n, const uint64_t* key, const int32_t* idx,
                                                     const double* zd, int32_t* rgrp, int32_t* rpos, double* ru,
                                                     double* gnw, double* gbeta, int32_t* cnt) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * FR + threadIdx.x;
  const bool in = s < n;
  const uint64_t k = in ? key[s] : 0;
  const bool head = in && (s == 0 || key[s - 1] != k);
  int size = 0;  // members, FT + 1 for more than FT
  if (head)
    for (size = 1; size <= FT && s + size < n && key[s + size] == k; ++size) {
    }
  const bool small = head && size <= FT;
  double nw = 0.0;
  if (small) {
    int32_t row[FT];
    double wt[FT];
    double big = 0.0, uu = 0.0;
#pragma unroll
    for (int t = 0; t < FT; ++t) row[t] = t < size ? idx[s + t] : 0;
#pragma unroll
    for (int t = 0; t < FT; ++t) {
      wt[t] = t < size ? zd[row[t]] : 0.0;
      big = fmax(big, fabs(wt[t]));
    }
    if (size == 1) {
      nw = wt[0];
    } else if (big > 0.0) {
      double acc = 0.0;
#pragma unroll
      for (int t = 0; t < FT; ++t) {
        const double q = wt[t] / big;
        acc += q * q;
      }
      nw = big * sqrt(acc);
    }
#pragma unroll
    for (int t = 0; t < FT; ++t) {
      if (t >= size) continue;
      double u = 0.0;
      if (size > 1 && nw != 0.0) {
        u = wt[t] / nw;
        if (t == 0) u += u >= 0.0 ? 1.0 : -1.0;
      }
      uu += u * u;
      rgrp[row[t]] = (int32_t)s;
      rpos[row[t]] = t;
      ru[row[t]] = u;
    }
    gnw[s] = nw;
    gbeta[s] = uu != 0.0 ? 2.0 / uu : 0.0;
  }
  for (uint64_t todo = __ballot(head && !small); todo; todo &= todo - 1) {
    const int l = __ffsll((unsigned long long)todo) - 1;
    const int64_t h = s - lane + l;
    const uint64_t kk = key[h];
    double big = 0.0;
    int64_t e = h;  // one behind the group's last
    for (int64_t j = h;; j += 64 * FG) {
      int same = 0;
#pragma unroll
      for (int g = 0; g < FG; ++g) {
        const int64_t p = j + 64 * g + lane;
        const bool mine = p < n && key[p] == kk;
        if (mine) big = fmax(big, fabs(zd[idx[p]]));
        same += __popcll(__ballot(mine));
      }
      e += same;
      if (same < 64 * FG) break;
    }
    for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
    double norm = 0.0;
    if (big > 0.0) {
      double acc = 0.0;
      for (int64_t j = h + lane; j < e; j += 64 * FG)
#pragma unroll
        for (int g = 0; g < FG; ++g) {
          const int64_t p = j + 64 * g;
          const double q = p < e ? zd[idx[p]] / big : 0.0;
          acc += q * q;
        }
      norm = big * sqrt(wave_sum(acc));
    }
    double uu = 0.0;
    for (int64_t j = h + lane; j < e; j += 64 * FG)
#pragma unroll
      for (int g = 0; g < FG; ++g) {
        const int64_t p = j + 64 * g;
        if (p >= e) continue;
        const int32_t row = idx[p];
        double u = 0.0;
        if (norm != 0.0) {
          u = zd[row] / norm;
          if (p == h) u += u >= 0.0 ? 1.0 : -1.0;
        }
        uu += u * u;
        rgrp[row] = (int32_t)h;
        rpos[row] = (int32_t)(p - h);
        ru[row] = u;
      }
    uu = wave_sum(uu);
    if (lane == l) {
      nw = norm;
      gnw[h] = norm;
      gbeta[h] = norm != 0.0 ? 2.0 / uu : 0.0;
    }
  }
  __shared__ int part[FR / 64];
  const int c = __popcll(__ballot(head && !(nw == 0.0)));
  if (lane == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int sum = 0;
    for (int w = 0; w < FR / 64; ++w) sum += part[w];
    cnt[blockIdx.x] = sum;
  }
}

// The reduced problem and the columns that do not come from it, both in
// decreasing pole order: a sorted position either enters the reduced problem
// (the first of a group whose ||w|| is not 0) or gives a column, that of its
// place in its group's reflection (the identity where ||w|| = 0).
struct FrontCols {
  double* val;   // the eigenvalue
  double* ub;    // beta u_t
  int32_t* grp;
  int32_t* t;
};
__global__ void __launch_bounds__(FR) k_front_reduce(int64_t n, const double* d, const int32_t* idx,
                                                     const int32_t* rgrp, const double* ru, const double* gnw,
                                                     const double* gbeta, const int32_t* cnt, const int32_t* bad,
                                                     double* rd, double* rz, FrontCols fc, FrontHdr* hdr) {
  __shared__ int part[FR / 64], sums[FR / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t s = (int64_t)blockIdx.x * FR + t;
  const bool last = blockIdx.x == gridDim.x - 1;
  int before = 0, nf = 0;
  for (int64_t b = t; b < (int64_t)blockIdx.x; b += FR) before += cnt[b];
  if (last)
    for (int64_t b = t; b < (int64_t)gridDim.x; b += FR) nf |= bad[b];
  const bool in = s < n;
  const int32_t row = in ? idx[s] : 0;
  const int32_t h = in ? rgrp[row] : 0;
  const double nw = in ? gnw[h] : 0.0;
  const bool red = in && h == s && !(nw == 0.0);
  const uint64_t mask = __ballot(red);
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  if (lane == 0) {
    part[w] = before;
    sums[w] = __popcll(mask);
  }
  const int anybad = __syncthreads_or(nf);
  int64_t r = __popcll(mask & (((uint64_t)1 << lane) - 1));
  int64_t m = 0;
  for (int q = 0; q < FR / 64; ++q) {
    r += part[q] + (q < w ? sums[q] : 0);
    m += part[q] + sums[q];
  }
  if (last && t == 0) {
    hdr->m = (int32_t)m;
    hdr->bad = anybad;
  }
  if (!in) return;
  if (red) {
    rd[r] = d[row];
    rz[r] = nw;
  } else {
    const int64_t c = s - r;
    fc.val[c] = d[idx[h]];
    fc.grp[c] = h;
    fc.t[c] = (int32_t)(s - h);
    fc.ub[c] = gbeta[h] * ru[row];  // 0 where ||w|| = 0
  }
}

// The columns in decreasing order of their eigenvalues, those of the reduction
// first among equal ones.
__global__ void __launch_bounds__(256) k_front_columns(int64_t n, int64_t m, bool neg, FrontCols fc,
                                                       const double* rd,
                                                       const double* lamr, const int32_t* sidx, const double* mu,
                                                       const double* xn, const int32_t* inf, double* lambda,
                                                       int32_t* info, bool vectors, int32_t* cgrp, int32_t* ct,
                                                       double* csig, double* cmu, double* cic, double* cub) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int32_t code = m > 0 ? inf[0] : 0;
  if (t == 0) info[0] = code;
  if (t >= n || code != 0) return;  // the solve left its outputs unspecified
  const bool red = t < m;
  const int64_t own = red ? t : t - m;
  const double v = red ? lamr[own] : fc.val[own];
  const int64_t c = column_place(t, n, m, lamr, rd, neg, [&](int64_t q) { return fc.val[q]; });
  lambda[c] = v;
  if (!vectors) return;
  cgrp[c] = red ? -1 : fc.grp[own];
  ct[c] = red ? 0 : fc.t[own];
  csig[c] = red ? rd[sidx[own]] : 0.0;
  cmu[c] = red ? mu[own] : 0.0;
  cic[c] = red ? 1.0 / xn[own] : 0.0;
  cub[c] = red ? 0.0 : fc.ub[own];
}

static size_t al(size_t x) { return (x + 255) & ~size_t(255); }

struct GLayout {
  size_t dr, zr, lamr, sidx, mu, xn, inf, rgrp, rpos, ru, cgrp, ct, csig, cmu, cic, cub, zabs, ph, val0, ub0,
      grp0, t0, cnt, bad, hdr, solver, total;
};
static GLayout glayout(int64_t n) {
  GLayout L;
  size_t o = 0;
  L.dr = o; o = al(o + 8 * n);
  L.zr = o; o = al(o + 8 * n);
  L.lamr = o; o = al(o + 8 * n);
  L.sidx = o; o = al(o + 4 * n);
  L.mu = o; o = al(o + 8 * n);
  L.xn = o; o = al(o + 8 * n);
  L.inf = o; o = al(o + 8);
  L.rgrp = o; o = al(o + 4 * n);
  L.rpos = o; o = al(o + 4 * n);
  L.ru = o; o = al(o + 8 * n);
  L.cgrp = o; o = al(o + 4 * n);
  L.ct = o; o = al(o + 4 * n);
  L.csig = o; o = al(o + 8 * n);
  L.cmu = o; o = al(o + 8 * n);
  L.cic = o; o = al(o + 8 * n);
  L.cub = o; o = al(o + 8 * n);
  L.zabs = o; o = al(o + 8 * n);
  L.ph = o; o = al(o + 16 * n);
  L.val0 = o; o = al(o + 8 * n);
  L.ub0 = o; o = al(o + 8 * n);
  L.grp0 = o; o = al(o + 4 * n);
  L.t0 = o; o = al(o + 4 * n);
  L.cnt = o; o = al(o + 4 * ((n + FR - 1) / FR));
  L.bad = o; o = al(o + 4 * ((n + FR - 1) / FR));
  L.hdr = o; o = al(o + sizeof(FrontHdr));
  L.solver = o; o = al(o + dpr1_workspace_size(n));
  L.total = o;
  return L;
}

}  // namespace gen
}  // namespace dpr1

using namespace dpr1::gen;

#define GCHECK(x)                            \
  do {                                       \
    if ((x) != hipSuccess) return DPR1_EHIP; \
  } while (0)

extern "C" {

size_t dpr1_general_workspace_size(int64_t n) {
  if (n < 1) return 0;
  return glayout(n).total;
}

}  // extern "C"

// Argument checks shared by the two entry points (same positions).
static int check_args(const double* d, const void* z, double rho, int64_t n, const double* lambda,
                      const double* V, int64_t ldv, const int32_t* info, const dpr1_opts* opts, const void* work,
                      size_t work_bytes) {
  if (!d) return -1;
  if (!z) return -2;
  if (!(rho == rho) || rho == 0.0 || rho == INFINITY || rho == -INFINITY) return -3;
  if (n < 1 || n > (int64_t)INT32_MAX / 2) return -4;
  if (!lambda) return -5;
  if (V && ldv < n) return -7;
  if (!info) return -8;
  if (opts && opts->waves_per_simd != 0 && opts->waves_per_simd != 4 && opts->waves_per_simd != 6 &&
      opts->waves_per_simd != 8)
    return -9;
  if (!work) return -10;
  if (work_bytes < glayout(n).total) return -11;
  return 0;
}

static int set_info(int32_t* info, int32_t code, hipStream_t st) {
  GCHECK(hipMemcpyAsync(info, &code, 4, hipMemcpyHostToDevice, st));
  GCHECK(hipStreamSynchronize(st));
  return DPR1_OK;
}

// The reduction, the reduced solve and the assembly.
template <bool CPLX>
static int front_end(const double* d, const double* z, double rho, int64_t n, double* lambda, double* V, int64_t ldv,
                     int32_t* info, const dpr1_opts* opts, char* w, hipStream_t st) {
  const GLayout L = glayout(n);
  auto f64 = [&](size_t off) { return (double*)(w + off); };
  auto i32 = [&](size_t off) { return (int32_t*)(w + off); };
  double *zd = f64(L.zabs), *ph = f64(L.ph), *rd = f64(L.dr), *rz = f64(L.zr);
  // the sort and the groups work in the room of arrays that are written later
  uint64_t *key = (uint64_t*)(w + L.lamr), *key2 = (uint64_t*)(w + L.csig);
  int32_t *idx = i32(L.sidx), *idx2 = i32(L.cgrp);
  double *gnw = f64(L.cmu), *gbeta = f64(L.cic);
  const FrontCols fc = {f64(L.val0), f64(L.ub0), i32(L.grp0), i32(L.t0)};
  FrontHdr* dhdr = (FrontHdr*)(w + L.hdr);
  const dim3 runs((unsigned)((n + FR - 1) / FR)), rows((unsigned)((n + 255) / 256));
  hipLaunchKernelGGL(k_front_sort<CPLX>, runs, dim3(FR), 0, st, d, z, n, zd, ph, key, idx, i32(L.bad));
  for (int64_t len = FR; len < n; len *= FW) {
    hipLaunchKernelGGL(k_front_merge, rows, dim3(256), 0, st, n, len, (const uint64_t*)key, (const int32_t*)idx, key2,
                       idx2);
    std::swap(key, key2);
    std::swap(idx, idx2);
  }
  hipLaunchKernelGGL(k_front_groups, runs, dim3(FR), 0, st, n, (const uint64_t*)key, (const int32_t*)idx,
                     (const double*)zd, i32(L.rgrp), i32(L.rpos), f64(L.ru), gnw, gbeta, i32(L.cnt));
  hipLaunchKernelGGL(k_front_reduce, runs, dim3(FR), 0, st, n, d, (const int32_t*)idx, (const int32_t*)i32(L.rgrp),
                     (const double*)f64(L.ru), (const double*)gnw, (const double*)gbeta, (const int32_t*)i32(L.cnt),
                     (const int32_t*)i32(L.bad), rd, rz, fc, dhdr);
  GCHECK(hipGetLastError());
  FrontHdr h;
  GCHECK(hipMemcpyAsync(&h, dhdr, sizeof(h), hipMemcpyDeviceToHost, st));
  GCHECK(hipStreamSynchronize(st));
  if (h.bad) return set_info(info, DPR1_INFO_NONFINITE, st);
  const int64_t m = h.m;

  // the reduced problem: eigenvalues and the shifted representation (sigma_k,
  // mu_k, ||x_k||) from which k_assemble evaluates the vectors
  if (m > 0) {
    const int rc = dpr1_eig(rd, rz, rho, m, f64(L.lamr), nullptr, m, V ? i32(L.sidx) : nullptr,
                            V ? f64(L.mu) : nullptr, V ? f64(L.xn) : nullptr, i32(L.inf), nullptr, opts,
                            w + L.solver, dpr1_workspace_size(m), (void*)st);
    if (rc != DPR1_OK) return rc;
  }
  hipLaunchKernelGGL(k_front_columns, rows, dim3(256), 0, st, n, m, rho < 0.0, fc, (const double*)rd, (const double*)f64(L.lamr),
                     (const int32_t*)i32(L.sidx), (const double*)f64(L.mu), (const double*)f64(L.xn),
                     (const int32_t*)i32(L.inf), lambda, info, V != nullptr, i32(L.cgrp), i32(L.ct), f64(L.csig),
                     f64(L.cmu), f64(L.cic), f64(L.cub));
  GCHECK(hipGetLastError());
  if (V) {
    AsmArgs a;
    a.n = n;
    a.ldv = ldv;
    a.d = d;
    a.z = zd;
    a.ph = CPLX ? ph : nullptr;
    a.rgrp = i32(L.rgrp);
    a.rpos = i32(L.rpos);
    a.ru = f64(L.ru);
    a.cgrp = i32(L.cgrp);
    a.ct = i32(L.ct);
    a.csig = f64(L.csig);
    a.cmu = f64(L.cmu);
    a.cic = f64(L.cic);
    a.cub = f64(L.cub);
    a.V = V;
    const int64_t span = CPLX ? ASM_T : 2 * ASM_T;  // rows of a block
    const int64_t rtiles = (n + span - 1) / span, ctiles = (n + ASM_C - 1) / ASM_C;
    hipLaunchKernelGGL(k_assemble<CPLX>, dim3((unsigned)(rtiles * ctiles)), dim3(ASM_T),
                       ASM_LDS - (CPLX ? 48 * 272 : 32 * 544), st, a, (int)rtiles);
    GCHECK(hipGetLastError());
  }
  GCHECK(hipStreamSynchronize(st));
  return DPR1_OK;
}

extern "C" {

int dpr1_eig_general(const double* d, const double* z, double rho, int64_t n, double* lambda, double* V,
                     int64_t ldv, int32_t* info, const dpr1_opts* opts, void* work, size_t work_bytes,
                     void* stream) {
  const int bad = check_args(d, z, rho, n, lambda, V, ldv, info, opts, work, work_bytes);
  if (bad) return bad;
  return front_end<false>(d, z, rho, n, lambda, V, ldv, info, opts, (char*)work, (hipStream_t)stream);
}

int dpr1_eig_hermitian(const double* d, const double* z, double rho, int64_t n, double* lambda, double* V,
                       int64_t ldv, int32_t* info, const dpr1_opts* opts, void* work, size_t work_bytes,
                       void* stream) {
  const int bad = check_args(d, z, rho, n, lambda, V, ldv, info, opts, work, work_bytes);
  if (bad) return bad;
  return front_end<true>(d, z, rho, n, lambda, V, ldv, info, opts, (char*)work, (hipStream_t)stream);
}

}  // extern "C"
