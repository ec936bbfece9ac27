// Host-side rules of the library's kernels and launches, made callable for test_host_rules.py.
#include "dfisher_internal.h"

extern "C" __attribute__((visibility("default"))) int rules_row_records(int rows, int lds, int cols) {
  return dfi::row_records(rows, lds, cols);
}
