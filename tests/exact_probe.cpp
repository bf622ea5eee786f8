// Test harness (host code): the library's exact determinant signs
// (paper_1908_06909_amd/csrc/exact.h) on caller-given columns.  Built by the
// tests with hipcc; the library itself never uses this file.
#include "exact.h"

using namespace tct;

// n cases of det[A1 - A0, B1 - B0, C1 - C0], points [n][6][3] in the order A1,
// A0, B1, B0, C1, C0; a point with null[6k + i] set is passed as null.
//   sign[k]  det_diff_sign
//   ints[k]  1 when all three columns fit the integer route
//   slow[k]  expansion_det_diff_sign
extern "C" void probe_exact(long long n, const float* pts, const int* null, int* sign, int* ints, int* slow) {
  for (long long k = 0; k < n; ++k) {
    const float* p[6];
    for (int i = 0; i < 6; ++i) p[i] = null[6 * k + i] ? nullptr : pts + 18 * k + 3 * i;
    sign[k] = det_diff_sign(p[0], p[1], p[2], p[3], p[4], p[5], nullptr);
    slow[k] = expansion_det_diff_sign(p[0], p[1], p[2], p[3], p[4], p[5]);
    long long c[3];
    ints[k] = column_to_int(p[0], p[1], c) && column_to_int(p[2], p[3], c) && column_to_int(p[4], p[5], c);
  }
}
