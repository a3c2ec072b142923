// Reverse mode of the DPR1 eigendecomposition on gfx950.
//
// For L(Lambda, V):  Abar = V X V^T,  X = diag(lambda_bar) + F o (V^T V_bar),
// F_lk = 1/(lambda_k - lambda_l) for l != k (first-order perturbation of a
// symmetric eigendecomposition with simple eigenvalues; the interlacing of
// Sec. 1 makes every eigenvalue of an irreducible DPR1 matrix simple).  With
// dA = diag(dd) + drho z z^T + rho (dz z^T + z dz^T):
//   d_bar_j = Abar_jj = sum_k (V X)_jk V_jk
//   rho_bar = z^T Abar z = y^T X y,            y = V^T z
//   z_bar   = rho (Abar + Abar^T) z = rho V (X + X^T) y
// and y_k = v_k^T z = -1/(rho ||x_k||) because f(lambda_k) = 0 (eq. Pick,
// Aeigenvec), which avoids the cancellation of the sum v_k^T z.  The gaps
// lambda_k - lambda_l come from the shifted representation
// (d_{i_k} + mu_k) - (d_{i_l} + mu_l), added in double-double, so clustered
// eigenvalues keep their relative gap accuracy.
//
// Kernels:
//   k_gemm<EPI_X>  P = V^T V_bar on FP64 matrix cores, epilogue X = F o P +
//                  diag(lambda_bar), partial sums of X y (rows) and X^T y (cols)
//   k_bwd_u        u = (X + X^T) y and parts of rho_bar = y^T X y from those
//                  partials
//   k_gemm<EPI_D>  Q = V X on FP64 matrix cores, epilogue partial row sums of
//                  Q o V (for d_bar) and of V diag(u) (for z_bar)
//   k_bwd_final    d_bar, z_bar = rho V u and rho_bar from the partials
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/dpr1.h"
#include "dd.h"

namespace dpr1 {
namespace bwd {

// Block tile TB x TB: 128 (2 x 4 waves of 64 x 32) or 64 (2 x 2 waves of 32 x
// 32), in blocks of the 16x16x4 FP64 MFMA, K staged through LDS in slices of
// 16, double-buffered; tile_of chooses.
constexpr int BK = 16;
constexpr int PAD = 2;   // LDS row padding (doubles)
constexpr int NXCD = 8;  // workgroups are dealt round-robin to the 8 XCDs

typedef double double4_t __attribute__((ext_vector_type(4)));

enum { EPI_X = 0, EPI_D = 1 };

struct GArgs {
  int64_t n;
  int nb;
  const double* A;   // V (both GEMMs), or null: V recomputed from (z, shift, mu, ||x||)
  const double* z;      // [nb*n]  (used when A is null)
  const double* sig;    // [nb*n]  d_{i_k}, the shift of eigenvalue k (used when A is null)
  const double* ixn;    // [nb*n]  1/||x_k|| (used when A is null)
  const double* B;   // V_bar (EPI_X, column-major) or X (EPI_D, row-major)
  double* C;         // X (EPI_X), stored row-major
  // EPI_X
  const double* lam_bar;  // [nb*n] or null
  const double* d;        // [nb*n]
  const int32_t* sidx;    // [nb*n]
  const double* mu;       // [nb*n]
  const double* y;        // [nb*n]
  double* part_r;         // [nb][ntile][n]  sum_k X_lk y_k over the tile's k range
  double* part_c;         // [nb][ntile][n]  sum_l X_lk y_l over the tile's l range
  // EPI_D
  const double* u;        // [nb*n]  (X + X^T) y
  double* part_d;         // [nb][ntile][n]  sum_k Q_jk V_jk
  double* part_z;         // [nb][ntile][n]  sum_k V_jk u_k
  int has_B;              // 0: V_bar is null, P = 0
  int64_t lda;            // leading dimension of V (A), column-major
  int64_t ldb;            // leading dimension of B: V_bar's (columns, or rows with BR), n for X
};

// Element (j, k) of V for problem offset vo, recomputed from the forward's
// shifted representation: v_k[j] = z_j / (((d_j - d_{i_k}) - mu_k) ||x_k||)
// (eq. eigenvecAi), so that a caller short of memory need not keep V between
// the forward and the backward.  d_{i_k} and 1/||x_k|| come precomputed
// (k_bwd_y); the quotient is the refined reciprocal with one residual
// correction, as in the forward's eigenvector writer.
__device__ __forceinline__ double v_from(double dj, double zj, double sk, double mk, double ik) {
  const double den = (dj - sk) - mk;
  double r = __builtin_amdgcn_rcp(den);
  r = __builtin_fma(r, __builtin_fma(-den, r, 1.0), r);
  double q = zj * r;
  q = __builtin_fma(__builtin_fma(-q, den, zj), r, q);
  return q * ik;
}
__device__ __forceinline__ double v_elem(const GArgs& g, int64_t vo, int64_t j, int64_t k) {
  return v_from(g.d[vo + j], g.z[vo + j], g.sig[vo + k], g.mu[vo + k], g.ixn[vo + k]);
}

// Column-major n x n matrices (V with ld = lda, V_bar with ld = ldb; a
// batch's problems lda * n and ldb * n apart; X row-major with ld = n).
// EPI_X computes op(A) = A^T (A = V),
// EPI_D op(A) = A.
// RV: V is not passed in; its elements are rebuilt by v_elem (a separate
// instance, so that the path with V keeps its plain loads).
// BR (EPI_X): V_bar comes row by row, V_bar(j, c) at j ldb + c, as autograd
// hands it over; it is loaded as EPI_D loads X instead of being transposed
// first (256 x 512: the copy took 680 us of a 4.0 ms step).
// Two blocks per CU (66.5 KB of LDS each, 68 KB where V^T is rebuilt) are 4
// waves per SIMD, which leaves 128 VGPRs a lane: the bound asks for that
// budget.
template <int TB, int EPI, bool RV, bool BR = EPI == EPI_D>
__global__ void __launch_bounds__(4 * TB, 4) k_gemm(GArgs g) {
  constexpr int BM = TB, BN = TB;
  constexpr int WNW = TB / 32;          // waves along n (2 along m)
  constexpr int TN = BN / WNW;          // columns per wave
  constexpr int NBT = TN / 16;          // MFMA blocks per wave along n
  constexpr int MAT = BM / 32;          // and along m
  constexpr int NT = 128 * WNW;
  static_assert(NT == 4 * TB, "launch bounds");
  const int64_t n = g.n;
  const int tiles = (int)((n + BM - 1) / BM);
  const int T = tiles * tiles;
  // (problem, tile) pairs in one list, cut into NXCD consecutive pieces of
  // equal length, one per XCD: a problem's tiles still share an XCD's L2, and
  // few problems fill all XCDs (a whole problem per XCD left 7 of 8 idle for
  // one problem: n = 2000, 2.25 ms a product against 0.33)
  const int64_t total = (int64_t)g.nb * T;
  const int64_t piece = (total + NXCD - 1) / NXCD;
  const int64_t it = (int64_t)(blockIdx.x % NXCD) * piece + blockIdx.x / NXCD;
  if (blockIdx.x / NXCD >= piece || it >= total) return;
  const int pb = (int)(it / T), t = (int)(it % T);
  const int tm = t % tiles, tn = t / tiles;
  const int64_t mo = (int64_t)pb * n * n;
  const int64_t vo = (int64_t)pb * n;
  const double* A = RV ? nullptr : g.A + (int64_t)pb * g.lda * n;
  const double* Bm = g.B + (EPI == EPI_X ? (int64_t)pb * g.ldb * n : mo);
  const int64_t lda = g.lda, ldb = EPI == EPI_X ? g.ldb : n;
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x;
  const int wv = tid / 64, lane = tid % 64;
  const int wm = (wv & 1) * (BM / 2), wn = (wv >> 1) * TN;

  // one LDS buffer: the double-buffered operand tiles during the K loop,
  // the epilogue's per-row / per-column arrays after it
  constexpr int TILE_D = 2 * BK * (BM + PAD);
  constexpr int EPI_D_N = 3 * BM + 4 * BN + 2 * WNW * BM + 2 * BN;
  constexpr int SMEM_D = 2 * TILE_D > EPI_D_N ? 2 * TILE_D : EPI_D_N;
  __shared__ double smem[SMEM_D];
  double(*As)[BK][BM + PAD] = reinterpret_cast<double(*)[BK][BM + PAD]>(smem);
  double(*Bs)[BK][BN + PAD] = reinterpret_cast<double(*)[BK][BN + PAD]>(smem + TILE_D);

  double4_t acc[MAT][NBT];
#pragma unroll
  for (int a = 0; a < MAT; ++a)
#pragma unroll
    for (int b = 0; b < NBT; ++b) acc[a][b] = (double4_t){0.0, 0.0, 0.0, 0.0};

  constexpr int PER = (BM * BK) / NT;  // elements of each operand per thread
  static_assert(BM == BN && NT % BM == 0 && NT % BK == 0, "tile shape");
  // Element e2 of a thread: EPI_X: k = ek, m (or c) = em + STEP e2; EPI_D: m (or
  // c) = em, k = ek + STEP e2.  The per-thread part of each address is formed
  // once; what changes with k0 and e2 is uniform across the block.
  // The same for B, whose contiguous index is k where it comes column by column
  // and c (BR) where it comes row by row.
  constexpr int STEP = EPI == EPI_X ? NT / BK : NT / BM, STEPB = BR ? NT / BN : NT / BK;
  const int ek = EPI == EPI_X ? tid % BK : tid / BM;
  const int em = EPI == EPI_X ? tid / BK : tid % BM;
  const int bk = BR ? tid / BN : tid % BK, bc = BR ? tid % BN : tid / BK;
  const double* pA = RV ? nullptr : (EPI == EPI_X ? A + ek + (m0 + em) * lda : A + (m0 + em) + ek * lda);
  const double* pB = BR ? Bm + bk * ldb + (n0 + bc) : Bm + bk + (n0 + bc) * ldb;
  double ra[PER], rb[PER];
  // V^T rebuilt (EPI_X): the tile's columns k = m0 .. m0 + BM - 1 keep their
  // (d_{i_k}, mu_k, 1/||x_k||) in LDS for the whole K loop, and a thread's
  // elements of one K step share their row j, so d_j and z_j load once
  __shared__ double colc[RV && EPI == EPI_X ? 3 : 1][RV && EPI == EPI_X ? BM : 1];
  // V rebuilt (EPI_D): a thread's elements all lie in its row j = m0 + em
  double djr = 0.0, zjr = 0.0;
  if constexpr (RV && EPI == EPI_D) {
    if (m0 + em < n) {
      djr = g.d[vo + m0 + em];
      zjr = g.z[vo + m0 + em];
    }
  }
  if constexpr (RV && EPI == EPI_X) {
    for (int t = tid; t < BM; t += NT) {
      const int64_t gm = m0 + t;
      const bool ok = gm < n;
      colc[0][t] = ok ? g.sig[vo + gm] : 0.0;
      colc[1][t] = ok ? g.mu[vo + gm] : 0.0;
      colc[2][t] = ok ? g.ixn[vo + gm] : 0.0;
    }
    __syncthreads();
  }
  // indices are below 2^20 + 128 (n is at most 2^20): 32 bits
  const int ni = (int)n;
  auto gload = [&](int k0) {
    double dj = 0.0, zj = 0.0;
    if constexpr (RV && EPI == EPI_X) {
      if (k0 + ek < ni) {
        dj = g.d[vo + k0 + ek];
        zj = g.z[vo + k0 + ek];
      }
    }
#pragma unroll
    for (int e2 = 0; e2 < PER; ++e2) {
      if (EPI == EPI_X) {
        // A^T(m, k) = V[k + m lda], contiguous along k
        const int ml = em + STEP * e2;
        ra[e2] = (m0 + ml < ni && k0 + ek < ni)
                     ? (RV ? v_from(dj, zj, colc[0][RV ? ml : 0], colc[1][RV ? ml : 0], colc[2][RV ? ml : 0])
                           : pA[k0 + STEP * e2 * lda])
                     : 0.0;
      } else {
        // A(m, k) = V[m + k lda], contiguous along m
        const int gk = k0 + ek + STEP * e2;
        ra[e2] = (m0 + em < ni && gk < ni)
                     ? (RV ? v_from(djr, zjr, g.sig[vo + gk], g.mu[vo + gk], g.ixn[vo + gk])
                           : pA[(k0 + STEP * e2) * lda])
                     : 0.0;
      }
      // B(k, c): X[k n + c] (EPI_D), V_bar[k ldb + c] (BR) or V_bar[k + c ldb]
      const int hk = k0 + bk + (BR ? STEPB * e2 : 0), hc = n0 + bc + (BR ? 0 : STEPB * e2);
      rb[e2] = (hk < ni && hc < ni) ? (BR ? pB[(k0 + STEPB * e2) * ldb] : pB[k0 + STEPB * e2 * ldb]) : 0.0;
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int e2 = 0; e2 < PER; ++e2) {
      int e = tid + e2 * NT;
      if (EPI == EPI_X) {
        As[buf][e % BK][e / BK] = ra[e2];
      } else {
        As[buf][e / BM][e % BM] = ra[e2];
      }
      if (BR) Bs[buf][e / BN][e % BN] = rb[e2];
      else Bs[buf][e % BK][e / BK] = rb[e2];
    }
  };

  const bool doB = (EPI == EPI_D) || g.has_B;
  if (doB) {
    gload(0);
    sstore(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < ni; k0 += BK) {
      const bool more = k0 + BK < ni;
      if (more) gload(k0 + BK);  // next slice in flight during this one
#pragma unroll
      for (int ks = 0; ks < BK; ks += 4) {
        // 16x16x4 FP64 MFMA: lane holds A(row = lane%16, k = lane/16) and
        // B(k = lane/16, col = lane%16)
        const int r = lane % 16, q = lane / 16;
        double af[MAT], bf[NBT];
#pragma unroll
        for (int x = 0; x < MAT; ++x) af[x] = As[buf][ks + q][wm + 16 * x + r];
#pragma unroll
        for (int x = 0; x < NBT; ++x) bf[x] = Bs[buf][ks + q][wn + 16 * x + r];
#pragma unroll
        for (int a = 0; a < MAT; ++a)
#pragma unroll
          for (int b = 0; b < NBT; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[a], bf[b], acc[a][b], 0, 0, 0);
      }
      if (more) {
        sstore(buf ^ 1);
        __syncthreads();
        buf ^= 1;
      }
    }
  }

  // Epilogue (256 x 512: the matrix cores are busy 60 % of a product's time, other
  // vector instructions, most of them this, 12 to 18 %; one V load per element in
  // turn and IEEE quotients cost 90 us a product).  Accumulator element q of a lane holds row lane/16 + 4q,
  // column lane%16 of its 16x16 block (checked on gfx950 with a probe that
  // multiplies A(:,0) = 2^i by B(0,:) = 3^j).  The per-row and per-column
  // quantities of this tile are staged in LDS first; per-row / per-column
  // partial sums go back through LDS.
  __syncthreads();  // every wave is done with the operand tiles
  double* rsig = smem;
  double* rmu = rsig + BM;
  double* ry = rmu + BM;
  double* csig = ry + BM;
  double* cmu = csig + BN;
  double* cy = cmu + BN;
  double* clb = cy + BN;
  double(*rowp)[WNW][BM] = reinterpret_cast<double(*)[WNW][BM]>(clb + BN);  // [quantity][wave along n][row]
  double(*colp)[BN] = reinterpret_cast<double(*)[BN]>(clb + BN + 2 * WNW * BM);  // [wave along m][col]
  // shift indices come from the caller: clamped so that a bad one cannot
  // address outside the problem
  auto sidx = [&](int64_t k) { return (int64_t)min(max(g.sidx[vo + k], 0), (int)(n - 1)); };
  if (tid < BM) {
    int64_t row = m0 + tid;
    if (row < n) {
      if (EPI == EPI_X) {
        rsig[tid] = g.d[vo + sidx(row)];
        rmu[tid] = g.mu[vo + row];
        ry[tid] = g.y[vo + row];
      }
    }
  } else if (tid < BM + BN) {
    int c = tid - BM;
    int64_t col = n0 + c;
    if (col < n) {
      if (EPI == EPI_X) {
        csig[c] = g.d[vo + sidx(col)];
        cmu[c] = g.mu[vo + col];
        cy[c] = g.y[vo + col];
        clb[c] = g.lam_bar ? g.lam_bar[vo + col] : 0.0;
      } else {
        cy[c] = g.u[vo + col];
      }
    }
  }
  __syncthreads();
  const int half_n = wv >> 1, half_m = wv & 1;  // wave index along n, along m
  double cs[NBT];
#pragma unroll
  for (int b = 0; b < NBT; ++b) cs[b] = 0.0;
#pragma unroll
  for (int a = 0; a < MAT; ++a) {
    double rs1[4] = {0.0, 0.0, 0.0, 0.0}, rs2[4] = {0.0, 0.0, 0.0, 0.0};
    // V(row, col) of the 4 NBT elements, all loads in flight together (indices
    // past the matrix are clamped; their products are dropped)
    double vj[NBT][4];
    if (EPI == EPI_D) {
#pragma unroll
      for (int b = 0; b < NBT; ++b) {
        const int col = min(n0 + wn + b * 16 + lane % 16, ni - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = min(m0 + wm + a * 16 + (lane / 16) + 4 * q, ni - 1);
          vj[b][q] = RV ? v_elem(g, vo, row, col) : A[row + col * lda];
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NBT; ++b) {
      const int cl = wn + b * 16 + lane % 16;
      const int col = n0 + cl;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int rl = wm + a * 16 + (lane / 16) + 4 * q;
        const int row = m0 + rl;
        if (row >= ni || col >= ni) continue;
        const double v = acc[a][b][q];
        if (EPI == EPI_X) {
          // X(row = l, col = k), stored row-major (consecutive lanes on
          // consecutive columns)
          double x;
          if (row == col) {
            x = clb[cl];
          } else {
            // the gap from the shifted representation: both differences and
            // their sum with their rounding errors; the quotient corrected
            const dd ds = two_sum(csig[cl], -rsig[rl]), dm = two_sum(cmu[cl], -rmu[rl]);
            const dd t = two_sum(ds.hi, dm.hi);
            const double gap = t.hi + (t.lo + (ds.lo + dm.lo));
            double r = __builtin_amdgcn_rcp(gap);
            r = __builtin_fma(r, __builtin_fma(-gap, r, 1.0), r);
            x = v * r;
            if (fabs(x) < INFINITY) x = __builtin_fma(__builtin_fma(-x, gap, v), r, x);
          }
          g.C[mo + (int64_t)row * n + col] = x;
          rs1[q] += x * cy[cl];
          cs[b] += x * ry[rl];
        } else {
          // Q(row = j, col = k) V(j, k) for d_bar, V(j, k) u_k for z_bar
          rs1[q] += v * vj[b][q];
          rs2[q] += vj[b][q] * cy[cl];
        }
      }
    }
    // reduce over the 16 lanes sharing a row (same lane/16)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double s1 = rs1[q], s2 = rs2[q];
      for (int o = 1; o < 16; o <<= 1) {
        s1 += __shfl_xor(s1, o);
        if (EPI == EPI_D) s2 += __shfl_xor(s2, o);
      }
      if (lane % 16 == 0) {
        int r = wm + a * 16 + (lane / 16) + 4 * q;
        rowp[0][half_n][r] = s1;
        rowp[1][half_n][r] = s2;
      }
    }
  }
  if (EPI == EPI_X) {
    // columns: reduce over the 4 lane groups sharing a column (same lane%16)
#pragma unroll
    for (int b = 0; b < NBT; ++b) {
      double c = cs[b];
      c += __shfl_xor(c, 16);
      c += __shfl_xor(c, 32);
      if (lane < 16) colp[half_m][wn + b * 16 + lane] = c;
    }
  }
  __syncthreads();
  const int ntile = tiles;
  if (tid < BM) {
    int64_t row = m0 + tid;
    if (row < n) {
      int64_t a = ((int64_t)pb * ntile + tn) * n + row;
      double s1 = rowp[0][0][tid], s2 = rowp[1][0][tid];
      for (int w = 1; w < WNW; ++w) {
        s1 += rowp[0][w][tid];
        s2 += rowp[1][w][tid];
      }
      if (EPI == EPI_X) {
        g.part_r[a] = s1;
      } else {
        g.part_d[a] = s1;
        g.part_z[a] = s2;
      }
    }
  } else if (EPI == EPI_X && tid < BM + BN) {
    int c = tid - BM;
    int64_t col = n0 + c;
    if (col < n) g.part_c[((int64_t)pb * ntile + tm) * n + col] = colp[0][c] + colp[1][c];
  }
}

// y_k = v_k^T z = -1/(rho ||x_k||); for the products without a stored V also
// the shift d_{i_k} (index clamped to the problem) and 1/||x_k||
__global__ void __launch_bounds__(256) k_bwd_y(int64_t n, int64_t nb, const double* __restrict__ rho,
                                               const double* __restrict__ xnorm, const double* __restrict__ d,
                                               const int32_t* __restrict__ sidx, double* __restrict__ y,
                                               double* __restrict__ sig, double* __restrict__ ixn) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * nb) return;
  int64_t p = t / n;
  y[t] = -1.0 / (rho[p] * xnorm[t]);
  if (sig) {
    const int64_t ik = (int64_t)min(max(sidx[t], 0), (int)(n - 1));
    sig[t] = d[p * n + ik];
    ixn[t] = 1.0 / xnorm[t];
  }
}

// u = X y + X^T y from the partials of the first GEMM, and the parts of
// rho_bar = y^T X y that the block's 256 rows give (k_bwd_final adds them in
// order; one block per problem took 42 us for one problem of n = 2000)
__global__ void __launch_bounds__(256) k_bwd_u(int64_t n, int ntile, const double* __restrict__ part_r,
                                               const double* __restrict__ part_c, const double* __restrict__ y,
                                               double* __restrict__ u, double* __restrict__ rho_part) {
  const int64_t pb = blockIdx.y;
  const int64_t vo = pb * n;
  __shared__ double red[256];
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double acc = 0.0;
  if (j < n) {
    double r = 0.0, c = 0.0;
#pragma unroll 4
    for (int t = 0; t < ntile; ++t) {
      const int64_t a = (pb * ntile + t) * n + j;
      r += part_r[a];
      c += part_c[a];
    }
    u[vo + j] = r + c;
    acc = y[vo + j] * r;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) rho_part[pb * gridDim.x + blockIdx.x] = red[0];
}

// d_bar_j = sum_k (V X)_jk V_jk and z_bar = rho V u from the second GEMM's partials
__global__ void __launch_bounds__(256) k_bwd_final(int64_t n, int64_t nb, int ntile, const double* __restrict__ rho,
                                                   const double* __restrict__ part_d,
                                                   const double* __restrict__ part_z,
                                                   const double* __restrict__ rho_part, double* __restrict__ d_bar,
                                                   double* __restrict__ z_bar, double* __restrict__ rho_bar) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * nb) return;
  int64_t pb = t / n, j = t % n;
  if (j == 0) {
    const int nr = (int)((n + 255) / 256);
    double r = 0.0;
    for (int q = 0; q < nr; ++q) r += rho_part[pb * nr + q];
    rho_bar[pb] = r;
  }
  double sd = 0.0, sz = 0.0;
  for (int q = 0; q < ntile; ++q) {
    int64_t a = (pb * ntile + q) * n + j;
    sd += part_d[a];
    sz += part_z[a];
  }
  d_bar[t] = sd;
  z_bar[t] = rho[pb] * sz;
}

// Without V_bar only the eigenvalue part remains, in closed form (O(n^2) per
// problem instead of two n^3 products): d_bar_j = sum_k lam_bar_k v_jk^2,
// z_bar_j = -2 sum_k lam_bar_k v_jk / ||x_k|| (from v_k^T z = -1/(rho ||x_k||)),
// rho_bar = sum_k lam_bar_k / (rho ||x_k||)^2.  Grid (row blocks, problems,
// pieces of k); the constants of EIG_K eigenvalues at a time are staged in
// LDS and read by every row of the block.  With one piece per row block the
// sum over k is one serial chain on few CUs (n = 4096, V rebuilt: 16 blocks,
// 967 us); eigonly_pieces cuts it until about 1024 blocks run, and
// k_bwd_eigsum adds the pieces in order.  More than one piece: row sums to
// part_d, part_z [problem][piece][n].
constexpr int EIG_K = 64;
static int64_t eigonly_pieces(int64_t n, int64_t nb) {
  const int64_t rows = (n + 255) / 256 * nb;
  return std::max<int64_t>(1, std::min<int64_t>((1024 + rows - 1) / rows, n / 128));
}
__global__ void __launch_bounds__(256) k_bwd_eigonly(GArgs g, const double* __restrict__ lam_bar,
                                                     const double* __restrict__ xnorm,
                                                     const double* __restrict__ rho, double* __restrict__ d_bar,
                                                     double* __restrict__ z_bar, double* __restrict__ rho_bar) {
  __shared__ double red[256];
  __shared__ double c_lb[EIG_K], c_lx[EIG_K], c_sig[EIG_K], c_mu[EIG_K], c_ix[EIG_K];
  const int64_t n = g.n;
  const int64_t p = blockIdx.y;
  const int64_t vo = p * n;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int pieces = gridDim.z;
  if (blockIdx.x == 0 && blockIdx.z == 0) {
    double acc = 0.0;
    for (int64_t k = threadIdx.x; k < n; k += blockDim.x) {
      const double lb = lam_bar ? lam_bar[vo + k] : 0.0;
      const double yk = 1.0 / (rho[p] * xnorm[vo + k]);
      acc += lb * (yk * yk);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) rho_bar[p] = red[0];
  }
  const int64_t chunk = (n + pieces - 1) / pieces;
  const int64_t ka = min(n, (int64_t)blockIdx.z * chunk), kb = min(n, ka + chunk);
  const bool ok = j < n;
  const double dj = ok && !g.A ? g.d[vo + j] : 0.0, zj = ok && !g.A ? g.z[vo + j] : 0.0;
  double sd = 0.0, sz = 0.0;
  for (int64_t k0 = ka; k0 < kb; k0 += EIG_K) {
    const int nk = (int)min((int64_t)EIG_K, kb - k0);
    __syncthreads();  // the previous constants are no longer read
    if ((int)threadIdx.x < nk) {
      const int64_t k = vo + k0 + threadIdx.x;
      const double lb = lam_bar ? lam_bar[k] : 0.0;
      c_lb[threadIdx.x] = lb;
      c_lx[threadIdx.x] = lb / xnorm[k];
      if (!g.A) {
        c_sig[threadIdx.x] = g.sig[k];
        c_mu[threadIdx.x] = g.mu[k];
        c_ix[threadIdx.x] = g.ixn[k];
      }
    }
    __syncthreads();
    if (!ok) continue;
    if (g.A) {
      const double* col = g.A + p * g.lda * n + j + k0 * g.lda;
#pragma unroll 8
      for (int q = 0; q < nk; ++q) {
        const double v = col[q * g.lda];
        sd = __builtin_fma(c_lb[q] * v, v, sd);
        sz = __builtin_fma(c_lx[q], v, sz);
      }
    } else {
#pragma unroll 4
      for (int q = 0; q < nk; ++q) {
        const double v = v_from(dj, zj, c_sig[q], c_mu[q], c_ix[q]);
        sd = __builtin_fma(c_lb[q] * v, v, sd);
        sz = __builtin_fma(c_lx[q], v, sz);
      }
    }
  }
  if (!ok) return;
  if (pieces == 1) {
    d_bar[vo + j] = sd;
    z_bar[vo + j] = -2.0 * sz;
  } else {
    const int64_t a = (p * pieces + blockIdx.z) * n + j;
    g.part_d[a] = sd;
    g.part_z[a] = sz;
  }
}
__global__ void __launch_bounds__(256) k_bwd_eigsum(int64_t n, int64_t nb, int pieces,
                                                    const double* __restrict__ part_d,
                                                    const double* __restrict__ part_z, double* __restrict__ d_bar,
                                                    double* __restrict__ z_bar) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * nb) return;
  const int64_t p = t / n, j = t % n;
  double sd = 0.0, sz = 0.0;
  for (int q = 0; q < pieces; ++q) {
    const int64_t a = (p * pieces + q) * n + j;
    sd += part_d[a];
    sz += part_z[a];
  }
  d_bar[t] = sd;
  z_bar[t] = -2.0 * sz;
}

// rho of the single-problem call, moved to the device as a kernel argument
// (no copy from host memory, so the call can be captured in a graph)
__global__ void k_set_rho(double* __restrict__ dst, double v) { *dst = v; }

struct BLayout {
  size_t X, y, u, pr, pc, pd, pz, sig, ixn, rho, rp, total;
};
static size_t al(size_t x) { return (x + 255) & ~size_t(255); }
// Tile size of the two products for nb problems of order n: the size whose
// tiles the fullest of the 256 CUs finishes first.  A tile of 128 alone on its
// CU takes 1 (two waves per SIMD), two together 1.72, a tile of 64 0.26.
// Measured, the whole backward with tiles of 64 / 128 in us: n = 400 73 / 156,
// 1200 259 / 408, 1600 444 / 539, 2000 688 / 664, 2400 1244 / 1373, 2800 1819
// / 1596; 16 problems of n = 128 40 / 72, 40 of n = 300 133 / 210.
static int tile_of(int64_t n, int64_t nb) {
  const int64_t t = (n + 127) / 128, h = (n + 63) / 64;
  const int64_t u = (t * t * nb + 255) / 256, v = (h * h * nb + 255) / 256;
  return 0.26 * (double)v < (u == 1 ? 1.0 : 0.86 * (double)u) ? 64 : 128;
}
static BLayout blayout(int64_t n, int64_t nb) {
  BLayout L;
  // partials for the smaller tile whichever runs: the size then grows with n
  // and nb, and a workspace holds every smaller call too
  const int64_t nt = (n + 63) / 64;
  size_t o = 0;
  L.X = o; o = al(o + sizeof(double) * n * n * nb);
  L.y = o; o = al(o + sizeof(double) * n * nb);
  L.u = o; o = al(o + sizeof(double) * n * nb);
  L.pr = o; o = al(o + sizeof(double) * n * nt * nb);
  L.pc = o; o = al(o + sizeof(double) * n * nt * nb);
  L.pd = o; o = al(o + sizeof(double) * n * nt * nb);
  L.pz = o; o = al(o + sizeof(double) * n * nt * nb);
  L.sig = o; o = al(o + sizeof(double) * n * nb);
  L.ixn = o; o = al(o + sizeof(double) * n * nb);
  L.rho = o; o = al(o + sizeof(double));
  L.rp = o; o = al(o + sizeof(double) * ((n + 255) / 256) * nb);
  L.total = o;
  return L;
}

// The launches of both entry points (arguments checked there).
static int run_backward(int64_t nbatch, int64_t n, const double* d, const double* z, const double* rho,
                        const int32_t* shift_idx, const double* mu, const double* xnorm, const double* V, int64_t lda,
                        const double* lambda_bar, const double* V_bar, int64_t ldb, bool rows, double* d_bar,
                        double* z_bar, double* rho_bar, void* work, const BLayout& L, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  char* w = (char*)work;
  double* X = (double*)(w + L.X);
  double* y = (double*)(w + L.y);
  double* u = (double*)(w + L.u);
  double* pr = (double*)(w + L.pr);
  double* pc = (double*)(w + L.pc);
  double* pd = (double*)(w + L.pd);
  double* pz = (double*)(w + L.pz);
  double* rp = (double*)(w + L.rp);
  const int tb = tile_of(n, nbatch);
  const int tiles = (int)((n + tb - 1) / tb);
  const unsigned ggrid = (unsigned)((nbatch * tiles * tiles + NXCD - 1) / NXCD * NXCD);

  double* sig = V ? nullptr : (double*)(w + L.sig);
  double* ixn = V ? nullptr : (double*)(w + L.ixn);
  hipLaunchKernelGGL(k_bwd_y, dim3((unsigned)((n * nbatch + 255) / 256)), dim3(256), 0, st, n, nbatch, rho, xnorm, d,
                     shift_idx, y, sig, ixn);
  GArgs g;
  g.n = n;
  g.nb = (int)nbatch;
  g.A = V;
  g.z = z;
  g.sig = sig;
  g.ixn = ixn;
  g.B = V_bar;
  g.C = X;
  g.lam_bar = lambda_bar;
  g.d = d;
  g.sidx = shift_idx;
  g.mu = mu;
  g.y = y;
  g.part_r = pr;
  g.part_c = pc;
  g.u = u;
  g.part_d = pd;
  g.part_z = pz;
  g.has_B = V_bar != nullptr;
  g.lda = lda;
  g.ldb = ldb;
  if (!V_bar) {
    const int64_t pieces = eigonly_pieces(n, nbatch);  // <= tiles, the capacity of the partials
    g.part_d = pd;
    g.part_z = pz;
    hipLaunchKernelGGL(k_bwd_eigonly, dim3((unsigned)((n + 255) / 256), (unsigned)nbatch, (unsigned)pieces),
                       dim3(256), 0, st, g, lambda_bar, xnorm, rho, d_bar, z_bar, rho_bar);
    if (pieces > 1)
      hipLaunchKernelGGL(k_bwd_eigsum, dim3((unsigned)((n * nbatch + 255) / 256)), dim3(256), 0, st, n, nbatch,
                         (int)pieces, pd, pz, d_bar, z_bar);
    if (hipGetLastError() != hipSuccess) return DPR1_EHIP;
    return DPR1_OK;
  }
  const auto product = [&](auto small, auto large) {
    if (tb == 64)
      hipLaunchKernelGGL(small, dim3(ggrid), dim3(256), 0, st, g);
    else
      hipLaunchKernelGGL(large, dim3(ggrid), dim3(512), 0, st, g);
  };
  if (V && rows)
    product(k_gemm<64, EPI_X, false, true>, k_gemm<128, EPI_X, false, true>);
  else if (V)
    product(k_gemm<64, EPI_X, false, false>, k_gemm<128, EPI_X, false, false>);
  else if (rows)
    product(k_gemm<64, EPI_X, true, true>, k_gemm<128, EPI_X, true, true>);
  else
    product(k_gemm<64, EPI_X, true, false>, k_gemm<128, EPI_X, true, false>);
  if (hipGetLastError() != hipSuccess) return DPR1_EHIP;
  hipLaunchKernelGGL(k_bwd_u, dim3((unsigned)((n + 255) / 256), (unsigned)nbatch), dim3(256), 0, st, n, tiles, pr, pc,
                     y, u, rp);
  g.B = X;
  if (V)
    product(k_gemm<64, EPI_D, false>, k_gemm<128, EPI_D, false>);
  else
    product(k_gemm<64, EPI_D, true>, k_gemm<128, EPI_D, true>);
  if (hipGetLastError() != hipSuccess) return DPR1_EHIP;
  hipLaunchKernelGGL(k_bwd_final, dim3((unsigned)((n * nbatch + 255) / 256)), dim3(256), 0, st, n, nbatch, tiles,
                     rho, pd, pz, rp, d_bar, z_bar, rho_bar);
  if (hipGetLastError() != hipSuccess) return DPR1_EHIP;
  return DPR1_OK;
}

}  // namespace bwd
}  // namespace dpr1

using namespace dpr1::bwd;

extern "C" {

size_t dpr1_backward_workspace_size(int64_t n, int64_t nbatch) {
  if (n < 1 || nbatch < 1) return 0;
  return blayout(n, nbatch).total;
}

int dpr1_eig_backward_batched(int64_t nbatch, int64_t n, const double* d, const double* z, const double* rho,
                              const int32_t* shift_idx, const double* mu, const double* xnorm, const double* V,
                              const double* lambda_bar, const double* V_bar, double* d_bar, double* z_bar,
                              double* rho_bar, void* work, size_t work_bytes, void* stream) {
  if (nbatch < 1 || nbatch > 65535) return -1;
  if (n < 1 || n > (1 << 20)) return -2;
  if (!d) return -3;
  if (!z && !V) return -4;
  if (!rho) return -5;
  if (!shift_idx) return -6;
  if (!mu) return -7;
  if (!xnorm) return -8;
  if (!d_bar) return -12;
  if (!z_bar) return -13;
  if (!rho_bar) return -14;
  if (!work) return -15;
  BLayout L = blayout(n, nbatch);
  if (work_bytes < L.total) return -16;
  return run_backward(nbatch, n, d, z, rho, shift_idx, mu, xnorm, V, n, lambda_bar, V_bar, n, false, d_bar, z_bar,
                      rho_bar, work, L, stream);
}

int dpr1_eig_backward(const double* d, const double* z, double rho, int64_t n, const int32_t* shift_idx,
                      const double* mu, const double* xnorm, const double* V, int64_t ldv, const double* lambda_bar,
                      const double* V_bar, int64_t ldvb, double* d_bar, double* z_bar, double* rho_bar, void* work,
                      size_t work_bytes, void* stream) {
  if (!d) return -1;
  if (!z && !V) return -2;
  if (!(rho == rho) || rho == 0.0 || rho == INFINITY || rho == -INFINITY) return -3;
  if (n < 1 || n > (1 << 20)) return -4;
  if (!shift_idx) return -5;
  if (!mu) return -6;
  if (!xnorm) return -7;
  if (V && ldv < n) return -9;
  if (V_bar && ldvb < n) return -12;
  if (!d_bar) return -13;
  if (!z_bar) return -14;
  if (!rho_bar) return -15;
  if (!work) return -16;
  BLayout L = blayout(n, 1);
  if (work_bytes < L.total) return -17;
  double* drho = (double*)((char*)work + L.rho);
  hipLaunchKernelGGL(k_set_rho, dim3(1), dim3(1), 0, (hipStream_t)stream, drho, rho);
  if (hipGetLastError() != hipSuccess) return DPR1_EHIP;
  return run_backward(1, n, d, z, drho, shift_idx, mu, xnorm, V, V ? ldv : n, lambda_bar, V_bar, V_bar ? ldvb : n,
                      false, d_bar, z_bar, rho_bar, work, L, stream);
}

int dpr1_eig_backward_strided(int64_t nbatch, int64_t n, const double* d, const double* z, const double* rho,
                              const int32_t* shift_idx, const double* mu, const double* xnorm, const double* V,
                              int64_t ldv, const double* lambda_bar, const double* V_bar, int64_t vb_row,
                              int64_t vb_col, double* d_bar, double* z_bar, double* rho_bar, void* work,
                              size_t work_bytes, void* stream) {
  if (nbatch < 1 || nbatch > 65535) return -1;
  if (n < 1 || n > (1 << 20)) return -2;
  if (!d) return -3;
  if (!z && !V) return -4;
  if (!rho) return -5;
  if (!shift_idx) return -6;
  if (!mu) return -7;
  if (!xnorm) return -8;
  if (V && ldv < n) return -10;
  const bool rows = V_bar && vb_row != 1;
  if (rows && (vb_row < n || vb_col != 1)) return -13;
  if (V_bar && !rows && vb_col < n) return -14;
  if (!d_bar) return -15;
  if (!z_bar) return -16;
  if (!rho_bar) return -17;
  if (!work) return -18;
  BLayout L = blayout(n, nbatch);
  if (work_bytes < L.total) return -19;
  return run_backward(nbatch, n, d, z, rho, shift_idx, mu, xnorm, V, V ? ldv : n, lambda_bar, V_bar,
                      V_bar ? (rows ? vb_row : vb_col) : n, rows, d_bar, z_bar, rho_bar, work, L, stream);
}

}  // extern "C"
