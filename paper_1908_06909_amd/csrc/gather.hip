// Deterministic backprojection: xhat_i = sum_j a_ij y_j (Eq. 3), every
// tetrahedron's sum exact, so the result is bitwise reproducible and, unlike
// the reproducible scatter's, as precise for weak rays as for strong ones.
//
// The paper scatters with atomics (Section II-F), having found a variant
// that kept the rays' contributions apart slower on its GPU; the same holds
// here.  The walk sums the segments of a wavefront and window per tetrahedron
// in its LDS table, exactly, in 64-bit fixed point at the wavefront's own
// power-of-two scale (walk.hip).  A flush does not keep these integers apart:
// it adds each into the tetrahedron's accumulator, an integer wide enough for
// every scale (255 bits above a unit of 2^-120) whose digits lie in
// separate 64-bit words.  A partial sum has 57 bits, so it is two or three
// digits, each one integer atomic, and no order of the additions can change
// the total; digits carry into each other only once, at the end.
//
// What bounds it: the walk and its table, then the atomics, two or three where
// the float scatter makes one.  The words lie word by word, not tetrahedron by
// tetrahedron: the lanes of a flush hold neighbouring tetrahedra, whose equal
// words then share a line (21.9 ms for 90 angles of the 512 x 512 benchmark,
// 30.8 the other way, with the walk and windows of then; now 18.4, and 16.6 for
// the float scatter).  Records written to memory,
// counted, moved into a list per tetrahedron and added up from there, with a
// wait of the host per chunk of angles, took 48.6 ms for these, and 90 for 48^3
// 256 x 256 x 120 (walked twice, the buffer being sized from a guess), which
// now takes 6.6.
#include "common.h"
#include "kernels.h"

namespace tct {

namespace {

__global__ void zero_words_kernel(unsigned long long* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

__global__ void exact_finish_kernel(ExactSums g, float* xhat, int nt, int accumulate) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nt) return;
  const double sum = exact_total(g.bits, g.words, [&](int l) { return (long long)g.acc[(int64_t)l * nt + t]; });
  xhat[t] = accumulate ? (float)((double)xhat[t] + sum) : (float)sum;
}

}  // namespace

tct_status backproject_gather(const tct_mesh* m, const tct_geom* g, const float* proj, float* xhat, int accumulate,
                              const int32_t* entry, int tile_u, int a_begin, int a_count, hipStream_t s) {
  const int nt = m->nt;
  ExactSums sums{};
  sums.bits = exact_digit_bits((int64_t)g->cone.nu * g->cone.nv * a_count);
  sums.words = exact_words(sums.bits);
  const int64_t n = (int64_t)sums.words * nt;
  TCT_HIP(hipMallocAsync((void**)&sums.acc, sizeof(unsigned long long) * (size_t)std::max<int64_t>(1, n), s));
  hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)std::max<int64_t>(1, (n + 255) / 256)), dim3(256), 0, s,
                     sums.acc, n);
  tct_status st = TCT_OK;
  // As many angles at once as the launch limit admits.
  const int64_t per_angle = std::max<int64_t>(1, pixel_walk_waves(g, 1, tile_u) / 4);
  const int chunk = (int)std::max<int64_t>(1, std::min<int64_t>(std::max(1, a_count), 0x7fffffff / per_angle));
  for (int a0 = a_begin; a0 < a_begin + a_count && st == TCT_OK; a0 += chunk)
    st = launch_pixel_walk(kModeBackExact, m, g, a0, std::min(chunk, a_begin + a_count - a0), entry, proj, nullptr,
                           nullptr, &sums, tile_u, s);
  if (st == TCT_OK)
    hipLaunchKernelGGL(exact_finish_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, sums, xhat, nt,
                       accumulate);
  const hipError_t e = hipGetLastError();
  (void)hipFreeAsync(sums.acc, s);
  if (st == TCT_OK && e != hipSuccess) return hip_fail(e, "exact backprojection launch");
  return st;
}

}  // namespace tct
