// Test harness (host code): the walk step's test that all three exit signs are
// certain under the mesh's longest edge (paper_1908_06909_amd/csrc/walk_filter.h).
// Built by the tests with hipcc; the library itself never uses this file.
#include "walk_filter.h"

using namespace tct;

namespace {
float3 f3(const float* p) { return make_float3(p[0], p[1], p[2]); }
}  // namespace

// n steps as in filter_probe.cpp; factor: the mesh's longest edge in units of
// the step's own longest.
//   certain[k]    step_signs_certain
//   sign[3k + i]  sign of the estimate of E(v, a_i) that the step then uses
extern "C" void probe_certain(long long n, const float* S, const float* P, const float* extent, const double* s,
                              const float* v, const float* a0, const float* a1, const float* a2, float factor,
                              int* certain, int* sign) {
  for (long long k = 0; k < n; ++k) {
    Ray r{};
    r.S = f3(S + 3 * k);
    r.P = f3(P + 3 * k);
    finish_ray(r, extent[k]);
    StepEdges g;
    step_edges(r, s[k], f3(v + 3 * k), f3(a0 + 3 * k), f3(a1 + 3 * k), f3(a2 + 3 * k), g);
    certain[k] = step_signs_certain(g, factor * fmaxf(g.m0, fmaxf(g.m1, g.m2)));
    const float E[3] = {g.E0, g.E1, g.E2};
    for (int i = 0; i < 3; ++i) sign[3 * k + i] = E[i] < 0.f ? -1 : 1;
  }
}
