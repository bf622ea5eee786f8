// Kernel launchers (walk.hip, gather.hip, shadow.hip, paper_mode.hip) used by the C interface.
#pragma once

#include "common.h"

namespace tct {

enum WalkMode {
  kModeEntry = 0,
  kModeForward = 1,
  kModeBackAtomic = 2,
  kModeCountAll = 3,
  kModeTrace = 5,
  kModeBackExact = 6,   // backprojection through the wavefront tables into exact wide sums
  kModeBackDirect = 7,  // backprojection with one global atomic per segment
  kModeEntryRstar = 8,  // entry search through the R*-tree
  kModeBackFixed = 9,   // backprojection through the block table into 64-bit fixed-point sums (reproducible)
};

// What the reproducible scatter's scale follows from (TCT_BP_FIXED): the
// largest |y_j| of the launch, as float bits in device memory, a bound on the
// rays' length and the bits a term may have.
struct FixedScale {
  const unsigned* max_bits;
  float max_dlen;
  int bits;
};

// Exact sums per tetrahedron (TCT_BP_GATHER).  Tetrahedron t's sum is
// sum_l acc[l nt + t] 2^(l bits) in units of 2^-kExactUnit.  A partial sum
// m 2^-scale (|m| < 2^57; scale at least -78 from the largest float and at most
// kExactUnit, set by the walk) is added as balanced digits of `bits` bits to
// consecutive words.  A ray crosses a tetrahedron once, so a word receives at
// most one digit per ray of the launch: with bits <= 62 - ceil(log2 rays) it
// cannot overflow.
constexpr int kExactUnit = 120;
struct ExactSums {
  unsigned long long* acc;
  int bits, words;
};

// 36 bits up to 2^26 rays: 8 words, and a partial sum is mostly two digits.
__host__ __device__ constexpr int exact_digit_bits(int64_t rays) {
  int log2 = 0;
  while (log2 < 40 && ((int64_t)1 << log2) < rays) ++log2;
  return 62 - log2 < 36 ? 62 - log2 : 36;
}

// Words for the bits 0 .. 254 that partial sums occupy and the one above.
__host__ __device__ constexpr int exact_words(int bits) { return (kExactUnit + 78 + 57) / bits + 1; }

// The lowest digit of v, in [-2^(bits - 1), 2^(bits - 1)), and what remains:
// v = *digit + 2^bits * (returned).
__host__ __device__ __forceinline__ long long exact_digit(long long v, int bits, long long* digit) {
  *digit = (long long)((unsigned long long)v << (64 - bits)) >> (64 - bits);
  return (v >> bits) + (*digit < 0 ? 1 : 0);
}

// Calls add(word, digit) for the non-zero digits of m 2^-scale.
template <class Add>
__host__ __device__ __forceinline__ void exact_add(int bits, int words, int scale, long long m, const Add& add) {
  const int pos = kExactUnit - scale < 0 ? 0 : (kExactUnit - scale > kExactUnit + 78 ? kExactUnit + 78 : kExactUnit - scale);
  const int shift = pos % bits;
  int w = pos / bits;
  // The lowest digit of m 2^shift, from m's low bits; the rest is below 2^58.
  long long d = (long long)((unsigned long long)m << (64 - bits + shift)) >> (64 - bits);
  long long rest = (m >> (bits - shift)) + (d < 0 ? 1 : 0);
  for (;;) {
    if (d != 0 && w < words) add(w, d);
    if (rest == 0 || ++w >= words) return;
    rest = exact_digit(rest, bits, &d);
  }
}

// The value of the accumulator whose words are word(0), word(1), ...: the
// words' excess over a digit is carried upwards, the digits are summed in
// float64 from the lowest up.
template <class Word>
__host__ __device__ __forceinline__ double exact_total(int bits, int words, const Word& word) {
  long long carry = 0;
  double sum = 0.0;
  for (int l = 0; l < words; ++l) {
    long long d;
    carry = exact_digit(word(l) + carry, bits, &d);
    sum += ldexp((double)d, l * bits - kExactUnit);
  }
  return sum + ldexp((double)carry, words * bits - kExactUnit);
}

tct_status launch_pixel_walk(int mode, const tct_mesh* m, const tct_geom* g, int a0, int na_chunk,
                             const int32_t* entry, const float* in, float* out_f32, int32_t* out_i32,
                             const ExactSums* exact, int tile_u, hipStream_t s, int lds_table = 0,
                             unsigned long long* acc64 = nullptr, const FixedScale* scale = nullptr);

tct_status backproject_atomic(const tct_mesh* m, const tct_geom* g, const float* proj, float* xhat, int accumulate,
                              const int32_t* entry, int tile_u, int lds_table, hipStream_t s);

tct_status launch_list_walk(int mode, const tct_mesh* m, const tct_geom* g, const int64_t* ids, const float* S,
                            const float* P, const float* U, const float* V, int32_t n, int64_t* counts,
                            const int64_t* offsets, int32_t* tets, float* lens, hipStream_t s);

tct_status launch_fill(float* p, int64_t n, float v, hipStream_t s);
// Wavefronts of a pixel-walk launch over na_chunk angles (four per block).
int64_t pixel_walk_waves(const tct_geom* g, int na_chunk, int tile_u);
tct_status entry_raster(const tct_mesh* m, const tct_geom* g, int32_t* entry, hipStream_t s);
tct_status launch_permute(const float* in, float* out, const int32_t* perm, int n, int scatter, hipStream_t s);

tct_status backproject_fixed(const tct_mesh* m, const tct_geom* g, const float* proj, float* xhat, int accumulate,
                             const int32_t* entry, int tile_u, int a_begin, int a_count, hipStream_t s);
tct_status backproject_fixed_noalloc(const tct_mesh* m, const tct_geom* g, const float* proj, float* xhat,
                                     int accumulate, const int32_t* entry, int tile_u, hipStream_t s);

tct_status backproject_gather(const tct_mesh* m, const tct_geom* g, const float* proj, float* xhat, int accumulate,
                              const int32_t* entry, int tile_u, int a_begin, int a_count, hipStream_t s);

tct_status backproject_shadow(const tct_mesh* m, const tct_geom* g, const float* proj, float* xhat, int accumulate,
                              int a_begin, int a_count, hipStream_t s);

tct_status forward_paper(const tct_mesh* m, const tct_geom* g, const float* x, float* proj, const int32_t* entry,
                         int precision, tct_paper_stats* stats, hipStream_t s);

tct_status batch_build(const tct_mesh* const* meshes, const tct_geom* const* geoms, int32_t n, const int32_t* tile_u,
                       int32_t* const* entries, tct_batch** out);
void batch_free(tct_batch* b);
tct_status batch_walk(tct_batch* b, int mode, const tct_vecset* in, const tct_vecset* out, hipStream_t s);

tct_status vecset_dot(const tct_vecset* a, const tct_vecset* b, double* results, double* workspace, hipStream_t s);
tct_status vecset_axpy_ratio(const tct_vecset* y, const tct_vecset* x, const double* num, const double* den,
                             double sign, hipStream_t s);
tct_status vecset_xpay_ratio(const tct_vecset* p, const tct_vecset* x, const double* num, const double* den,
                             hipStream_t s);
tct_status vecset_fill(const tct_vecset* y, float v, hipStream_t s);

// Host-side builders (mesh.cpp).
tct_status mesh_build(const float* verts, int32_t nv, const int32_t* tets, int32_t nt, const int32_t* nbrs,
                      uint32_t flags, int device, tct_mesh** out);
void mesh_free_device(tct_mesh* m);
tct_status geom_build(const tct_cone* cone, const double* angles, int32_t na, int device, tct_geom** out);
tct_status check_geometry(const tct_mesh* m, const tct_geom* g);

int default_tile_u();

tct_status blas_dot(const float* a, const float* b, int64_t n, double* result, double* workspace, hipStream_t s);
tct_status blas_axpy_ratio(float* y, const float* x, int64_t n, const double* num, const double* den, double sign,
                           hipStream_t s);
tct_status blas_xpay_ratio(float* p, const float* x, int64_t n, const double* num, const double* den, hipStream_t s);
tct_status blas_axpby(float* y, const float* x, int64_t n, float a, float b, hipStream_t s);
tct_status blas_mul(float* y, const float* a, const float* b, int64_t n, hipStream_t s);
tct_status blas_recip(float* y, const float* a, int64_t n, float eps, hipStream_t s);
tct_status blas_copy_f64(double* dst, const double* src, int n, hipStream_t s);

}  // namespace tct
