// Places of the columns of a reduced problem: its m eigenvalues and the n - m
// columns of the reduction (deflated and reflected poles, in decreasing
// order), the latter first among equal values.  A column's place is its own
// index plus its rank in the other list, which is a permutation only if both
// lists are non-increasing.  The solver's eigenvalues are ranked as held in
// the interval that interlacing gives each of them (eq. interlace: between
// d_k and d_k-1 for rho > 0, d_k+1 and d_k for rho < 0; consecutive intervals
// share an end), so they are non-increasing whatever was computed: an
// eigenvalue that options without a polish leave a rounding error outside its
// interval, or any value after a range report.
#pragma once

#include <math.h>
#include <stdint.h>

#ifndef DPR1_HD
#define DPR1_HD static inline
#endif

namespace dpr1 {

// lambda_k in its interval (NaN: the interval's lower end); d: the reduced
// problem's poles
DPR1_HD double held(const double* lam, const double* d, int64_t m, int64_t k, bool neg) {
  const double lo = neg ? (k + 1 < m ? d[k + 1] : -INFINITY) : d[k];
  const double hi = neg ? d[k] : (k > 0 ? d[k - 1] : INFINITY);
  return fmin(fmax(lam[k], lo), hi);
}

// The place of entry t: eigenvalue t for t < m, the reduction's column t - m
// from there on (val(c): its value).
template <class Val>
DPR1_HD int64_t column_place(int64_t t, int64_t n, int64_t m, const double* lam, const double* d, bool neg,
                             const Val& val) {
  int64_t lo = 0;
  if (t < m) {
    const double v = held(lam, d, m, t, neg);
    for (int64_t hi = n - m; lo < hi;) {  // the reduction's columns that come first
      const int64_t mid = (lo + hi) / 2;
      if (val(mid) >= v)
        lo = mid + 1;
      else
        hi = mid;
    }
    return t + lo;
  }
  // the eigenvalues that come first: the intervals above v hold those, the one
  // around it may (a search among the poles and one look at an eigenvalue)
  const double v = val(t - m);
  for (int64_t hi = m; lo < hi;) {
    const int64_t mid = (lo + hi) / 2;
    if (d[mid] > v)
      lo = mid + 1;
    else
      hi = mid;
  }
  if (neg && lo > 0) --lo;
  if (lo < m && held(lam, d, m, lo, neg) > v) ++lo;
  return t - m + lo;
}

}  // namespace dpr1
