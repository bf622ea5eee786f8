// Exact sign of 3x3 determinants of float32 point differences.
//
// Used for every decision of the walk that a floating-point estimate cannot
// certify: orientation of tetrahedra and faces at mesh creation, and the
// edge signs of rays through vertices, along edges or inside face planes
// (the near-degenerate cases the paper's Section II-C-1 and Fig. 9 show
// breaking float32 intersection code).
//
// Method: error-free transformations on float64 (Knuth's two-sum; the fused
// multiply-add two-product), accumulated into a non-overlapping expansion
// with zero elimination (Shewchuk 1997, "Adaptive precision floating-point
// arithmetic and fast robust geometric predicates").  Inputs are float32, so
// the product of two coordinates is exact in float64 and the product of three
// is exactly the sum of two float64 values; the determinant of differences is
// expanded by multilinearity into at most 48 such triple products and summed
// exactly.  The sign of a non-overlapping expansion is the sign of its
// largest component.
//
// Nearly all determinants that get here have columns whose entries, scaled by
// a power of two of the column's own, are integers below 2^42 (mesh and
// detector coordinates of similar size).  Those are decided in integer
// arithmetic: some 400 instructions in registers, against several thousand
// dependent ones on an array in scratch memory for the expansion.  What bounds
// a small launch is the latency of these signs, which one ray through an edge
// makes its whole wavefront wait for, some 30 times in a row along a diagonal
// of a regular mesh: a walk of 65,536 rays through 3,072 tetrahedra takes
// 0.03 ms without a tie and, with 1,082, 0.37 ms with the expansion, 0.09 with
// 128-bit integers in a function of their own, and 0.07 with 30-bit digits
// inline in the walk, whose registers then need not be saved around a call;
// one of 2.9M rays with 3.1M ties 8.1, 5.0 and 4.0 ms.
#pragma once

#include <hip/hip_runtime.h>

namespace tct {

__host__ __device__ inline void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  double bv = s - a;
  double av = s - bv;
  e = (a - av) + (b - bv);
}

__host__ __device__ inline void two_prod(double a, double b, double& p, double& e) {
  p = a * b;
  e = fma(a, b, -p);
}

// e[0..n) is non-overlapping with increasing magnitude; add b in place.
__host__ __device__ inline int expansion_grow(double* e, int n, double b) {
  double q = b;
  int k = 0;
  for (int i = 0; i < n; ++i) {
    double s, h;
    two_sum(q, e[i], s, h);
    if (h != 0.0) e[k++] = h;
    q = s;
  }
  if (q != 0.0) e[k++] = q;
  return k;
}

__host__ __device__ inline int expansion_add_triple(double* e, int n, float x, float y, float z, bool negate) {
  double xy = (double)x * (double)y;  // exact: 24 + 24 significant bits
  double p, r;
  two_prod(xy, (double)z, p, r);
  if (negate) {
    p = -p;
    r = -r;
  }
  n = expansion_grow(e, n, r);
  return expansion_grow(e, n, p);
}

// det[X, Y, Z] (columns) added exactly into the expansion, times sgn.
__host__ __device__ inline int expansion_add_det(double* e, int n, const float* X, const float* Y, const float* Z,
                                                 bool neg) {
  // + X0 Y1 Z2 - X0 Y2 Z1 - X1 Y0 Z2 + X1 Y2 Z0 + X2 Y0 Z1 - X2 Y1 Z0
  n = expansion_add_triple(e, n, X[0], Y[1], Z[2], neg);
  n = expansion_add_triple(e, n, X[0], Y[2], Z[1], !neg);
  n = expansion_add_triple(e, n, X[1], Y[0], Z[2], !neg);
  n = expansion_add_triple(e, n, X[1], Y[2], Z[0], neg);
  n = expansion_add_triple(e, n, X[2], Y[0], Z[1], neg);
  n = expansion_add_triple(e, n, X[2], Y[1], Z[0], !neg);
  return n;
}

// Exact sign of det[A1 - A0, B1 - B0, C1 - C0].  A null pointer stands for the
// zero vector.  By multilinearity the determinant is the signed sum of
// det[X, Y, Z] over X in {A1, A0}, Y in {B1, B0}, Z in {C1, C0}, the sign
// being (-1)^(number of *0 picks); picks of a null pointer or of the same
// point twice contribute exactly zero and are skipped.
__host__ __device__ __attribute__((noinline)) inline int expansion_det_diff_sign(const float* A1, const float* A0,
                                                                                 const float* B1, const float* B0,
                                                                                 const float* C1, const float* C0) {
  double e[96];
  int n = 0;
  const float* As[2] = {A1, A0};
  const float* Bs[2] = {B1, B0};
  const float* Cs[2] = {C1, C0};
  for (int ia = 0; ia < 2; ++ia)
    for (int ib = 0; ib < 2; ++ib)
      for (int ic = 0; ic < 2; ++ic) {
        const float *X = As[ia], *Y = Bs[ib], *Z = Cs[ic];
        if (!X || !Y || !Z || X == Y || Y == Z || X == Z) continue;
        n = expansion_add_det(e, n, X, Y, Z, ((ia + ib + ic) & 1) != 0);
      }
  if (n == 0) return 0;
  return e[n - 1] > 0.0 ? 1 : -1;
}

// The column a1 - a0 times a power of two as integers, |c| < 2^42; false when
// a scaled coordinate is not an integer.  (The scale puts the largest
// coordinate into [2^40, 2^41); a0 = null is zero.)
__host__ __device__ inline bool column_to_int(const float* a1, const float* a0, long long* c) {
  double m = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i) m = fmax(m, fmax(fabs((double)a1[i]), a0 ? fabs((double)a0[i]) : 0.0));
  int e = 0;
  (void)frexp(m, &e);  // m = 0 (a zero column): e = 0
  bool ok = m < 0x1p1000;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    // y = x + 1.5 2^52 rounds x to an integer, whose value is the difference
    // of the bit patterns of y and 1.5 2^52.  (A NaN equals nothing.)
    const double p = ldexp((double)a1[i], 41 - e), q = a0 ? ldexp((double)a0[i], 41 - e) : 0.0;
    const double yp = p + 0x1.8p52, yq = q + 0x1.8p52;
    ok = ok & (yp - 0x1.8p52 == p) & (yq - 0x1.8p52 == q);
    c[i] = __builtin_bit_cast(long long, yp) - __builtin_bit_cast(long long, yq);
  }
  return ok;
}

// Sign of det[a, b, c] for |entries| < 2^42, exactly, in digits of 30 bits, so
// that every product is one of two 32-bit integers: entries h 2^30 + l with
// |h| <= 2^12, minors m0 + m1 2^30 + m2 2^60 with |m2| < 2^26, and digit sums
// of the determinant below 2^62.  (128-bit integers would have to carry from
// product to product.)
__host__ __device__ inline int int_det_sign(const long long* a, const long long* b, const long long* c) {
  constexpr int kMask = (1 << 30) - 1;
  int al[3], ah[3], bl[3], bh[3], cl[3], ch[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    al[i] = (int)a[i] & kMask;
    ah[i] = (int)(a[i] >> 30);
    bl[i] = (int)b[i] & kMask;
    bh[i] = (int)(b[i] >> 30);
    cl[i] = (int)c[i] & kMask;
    ch[i] = (int)(c[i] >> 30);
  }
  long long d0 = 0, d1 = 0, d2 = 0, d3 = 0;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int j = (i + 1) % 3, k = (i + 2) % 3;
    const int nl = -bl[k], nh = -bh[k];
    const long long s0 = (long long)bl[j] * cl[k] + (long long)nl * cl[j];
    long long s1 = (long long)bl[j] * ch[k] + (long long)bh[j] * cl[k] + (long long)nl * ch[j] + (long long)nh * cl[j];
    s1 += s0 >> 30;
    const int m0 = (int)s0 & kMask, m1 = (int)s1 & kMask;
    const int m2 = (int)((long long)bh[j] * ch[k] + (long long)nh * ch[j] + (s1 >> 30));
    d0 += (long long)al[i] * m0;
    d1 += (long long)al[i] * m1 + (long long)ah[i] * m0;
    d2 += (long long)al[i] * m2 + (long long)ah[i] * m1;
    d3 += (long long)ah[i] * m2;
  }
  d1 += d0 >> 30;
  d2 += d1 >> 30;
  d3 += d2 >> 30;
  return d3 < 0 ? -1 : ((d3 | ((d0 | d1 | d2) & kMask)) != 0 ? 1 : 0);
}

// Float64 estimate of the same determinant with a certified error bound.
// det = A . (B x C); every one of its six monomials goes through at most
// eight roundings (three input differences, the product and difference
// inside B x C, the product with A, two additions), so
// |computed - exact| <= gamma_8 * sum|monomials| < 9 * 2^-53 * perm; 12 * 2^-53
// is used.  Returns 2 when the estimate cannot decide.
__host__ __device__ inline int filtered_det_diff_sign(const float* A1, const float* A0, const float* B1,
                                                      const float* B0, const float* C1, const float* C0) {
  double A[3], B[3], C[3];
  for (int i = 0; i < 3; ++i) {
    A[i] = (double)A1[i] - (A0 ? (double)A0[i] : 0.0);
    B[i] = (double)B1[i] - (B0 ? (double)B0[i] : 0.0);
    C[i] = (double)C1[i] - (C0 ? (double)C0[i] : 0.0);
  }
  double cx = B[1] * C[2] - B[2] * C[1];
  double cy = B[2] * C[0] - B[0] * C[2];
  double cz = B[0] * C[1] - B[1] * C[0];
  double det = A[0] * cx + A[1] * cy + A[2] * cz;
  double px = fabs(B[1] * C[2]) + fabs(B[2] * C[1]);
  double py = fabs(B[2] * C[0]) + fabs(B[0] * C[2]);
  double pz = fabs(B[0] * C[1]) + fabs(B[1] * C[0]);
  double perm = fabs(A[0]) * px + fabs(A[1]) * py + fabs(A[2]) * pz;
  const double bound = 12.0 * 1.1102230246251565e-16 * perm;  // 12 * 2^-53 * perm
  if (det > bound) return 1;
  if (det < -bound) return -1;
  return 2;
}

enum SignFlags : unsigned { kFlagExact = 1u, kFlagPerturbed = 2u };

// The same sign from the filter or, behind it, the integers alone; 2 when
// neither applies (a column without an integer form).
// p: A1, A0, B1, B0, C1, C0 (absent points as zeros).
__host__ __device__ inline int quick_det_sign(const float (&p)[6][3], unsigned* flags) {
  int s = filtered_det_diff_sign(p[0], p[1], p[2], p[3], p[4], p[5]);
  if (s != 2) return s;
  if (flags) *flags |= kFlagExact;
  long long a[3], b[3], c[3];
  const bool ka = column_to_int(p[0], p[1], a);
  const bool kb = column_to_int(p[2], p[3], b);
  const bool kc = column_to_int(p[4], p[5], c);
  return (ka & kb & kc) ? int_det_sign(a, b, c) : 2;
}

__host__ __device__ inline int det_diff_sign(const float* A1, const float* A0, const float* B1, const float* B0,
                                             const float* C1, const float* C0, unsigned* flags) {
  const float* const from[6] = {A1, A0, B1, B0, C1, C0};
  float p[6][3];
  for (int k = 0; k < 6; ++k)
    for (int i = 0; i < 3; ++i) p[k][i] = from[k] ? from[k][i] : 0.f;
  const int s = quick_det_sign(p, flags);
  return s != 2 ? s : expansion_det_diff_sign(A1, A0, B1, B0, C1, C0);
}

// orient3d(a, b, c, d) = sign det[b - a, c - a, d - a].
__host__ __device__ inline int orient3d_sign(const float* a, const float* b, const float* c, const float* d) {
  return det_diff_sign(b, a, c, a, d, a, nullptr);
}

// Sign of the edge (p, q) seen by the ray S -> P translated by eps U + eps^2 V:
// det[P - S, p - S, q - S], else det[P - S, U, p - q], else det[P - S, V, p - q].
// Zero only for an edge parallel to P - S.  By the filter and the expansion,
// which decide every input.
__host__ __device__ inline int perturbed_edge_sign(const float* S, const float* P, const float* U, const float* V,
                                                   const float* p, const float* q, unsigned* flags) {
  const float *B1 = p, *B0 = S, *C1 = q, *C0 = S;
  int s = 0;
#pragma unroll 1
  for (int level = 0; level < 3; ++level) {
    s = filtered_det_diff_sign(P, S, B1, B0, C1, C0);
    if (s == 2) {
      *flags |= kFlagExact;
      s = expansion_det_diff_sign(P, S, B1, B0, C1, C0);
    }
    if (s != 0) break;
    *flags |= kFlagPerturbed;
    B1 = level == 0 ? U : V;
    B0 = nullptr;
    C1 = p;
    C0 = q;
  }
  return s;
}

// The same by the filter and the integers: 2 where a determinant has no integer
// form.  One determinant in a loop over the levels, and no call: a walk has
// this inline beside its step.
__host__ __device__ inline int quick_perturbed_edge_sign(const float* S, const float* P, const float* U,
                                                         const float* V, const float* p, const float* q,
                                                         unsigned* flags) {
  float x[6][3];
  for (int i = 0; i < 3; ++i) {
    x[0][i] = P[i];
    x[1][i] = x[3][i] = x[5][i] = S[i];
    x[2][i] = p[i];
    x[4][i] = q[i];
  }
  int s = 0;
#pragma unroll 1
  for (int level = 0; level < 3; ++level) {
    s = quick_det_sign(x, flags);
    if (s != 0) break;
    *flags |= kFlagPerturbed;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (level == 0) {
        x[5][i] = x[4][i];
        x[4][i] = x[2][i];
        x[3][i] = 0.f;
      }
      x[2][i] = level == 0 ? U[i] : V[i];
    }
  }
  return s;
}

}  // namespace tct
