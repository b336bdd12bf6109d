// C entry point to sym_pinv_solve of csrc/sw_linalg.h for tests/test_pinv.py.
#include <vector>

#include "sw_linalg.h"

extern "C" int pinv(int n, const double* a, const double* h, double* theta, double cut) {
  std::vector<double> A(a, a + (size_t)n * n);
  return sw::sym_pinv_solve(n, A, h, theta, cut);
}
