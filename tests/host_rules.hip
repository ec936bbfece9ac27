// Host-side rules of the library's kernels and launches, made callable for test_host_rules.py.
#include "dfisher_internal.h"

extern "C" __attribute__((visibility("default"))) int rules_row_records(int rows, int lds, int cols) {
  return dfi::row_records(rows, lds, cols);
}

#include "gram.hip"

extern "C" __attribute__((visibility("default"))) void rules_gram_plan(int64_t n, int64_t m, int64_t lds, int prec, int aligned,
                                                                       int q, int mode, int64_t* nslice, int64_t* kslice) {
  const dfi::GramPlan p = dfi::gram_plan(n, m, lds, prec, aligned != 0, q, mode);
  *nslice = p.nslice;
  *kslice = p.kslice;
}
