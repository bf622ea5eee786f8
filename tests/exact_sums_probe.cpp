// Test harness (host code): the digits of the exact backprojection sums
// (paper_1908_06909_amd/csrc/kernels.h, the code that the walk's flush and the
// final conversion inline).  Built by the tests with hipcc; the library itself
// never uses this file.
#include "kernels.h"

using namespace tct;

extern "C" {

int probe_digit_bits(long long rays) { return exact_digit_bits(rays); }
int probe_words(int bits) { return exact_words(bits); }

// Adds n partial sums m 2^-scale to the accumulator words[exact_words(bits)]
// and returns its value.
double probe_sum(int bits, long long n, const int* scale, const long long* m, unsigned long long* words) {
  const int nw = exact_words(bits);
  for (long long k = 0; k < n; ++k)
    exact_add(bits, nw, scale[k], m[k], [&](int w, long long d) { words[w] += (unsigned long long)d; });
  return exact_total(bits, nw, [&](int l) { return (long long)words[l]; });
}
}
