// C entry point over the places of a reduced problem's columns (columns.h), for CPU tests.
#include "../../paper_1405_7537_amd/csrc/columns.h"

extern "C" void shim_places(int64_t n, int64_t m, const double* lam, const double* d, int neg, const double* val,
                            int64_t* place) {
  for (int64_t t = 0; t < n; ++t)
    place[t] = dpr1::column_place(t, n, m, lam, d, neg != 0, [&](int64_t c) { return val[c]; });
}
