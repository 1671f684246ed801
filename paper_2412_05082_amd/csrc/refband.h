// Band products of the 1D factors with compile-time reference rows (default
// penalty gamma = k(k+1), unit cells).  On a uniform mesh M = h M^, L = L^ / h,
// B = B^ / h^3 exactly (h is a power of two), so every term of the operator
// carries one power of h, applied to the output.  With boundary nodes staged
// as 0, every interior row is the periodic row of its cell position, but for
// the k rows of B next to either end.
#pragma once

#include <hip/hip_runtime.h>

#include "refcoef.h"
#include "tiles.h"

namespace c0ip {
namespace ref {

using tile::Band;

// a b + c in one rounding, spelled out: left to the compiler, the first two
// products of a sum may be contracted either way round, and kernels with
// different tiles would differ in the last bit.
template <typename T>
__device__ __forceinline__ T mad(T a, T b, T c) {
  if constexpr (sizeof(T) == 8)
    return __builtin_fma(a, b, c);
  else
    return __builtin_fmaf(a, b, c);
}

// The error of s = a + b (Knuth's two-sum): a + b = s + the result, exactly.
template <typename T>
__device__ __forceinline__ T sum_error(T a, T b, T s) {
  const T c = s - a;
  return (a - (s - c)) + (b - c);
}

// 1 / (d + e) for d > 0 and |e| within half a unit in the last place of d,
// rounded once: Newton's iteration from the hardware reciprocal, with e in its
// last residual.  With e the error of the eigenvalue sum d, a mode times this
// is rounded as often as a mode divided by the rounded sum.
template <typename T>
__device__ __forceinline__ T recip(T d, T e) {
  T r;
  if constexpr (sizeof(T) == 8) {
    r = __builtin_amdgcn_rcp(d);  // 24 bits or more
    r = mad(mad(-d, r, T(1)), r, r);
  } else {
    r = __builtin_amdgcn_rcpf(d);
  }
  return mad(mad(-e, r, mad(-d, r, T(1))), r, r);
}
template <typename T>
__device__ __forceinline__ T recip_sum(T a, T b) {
  const T d = a + b;
  return recip(d, sum_error(a, b, d));
}

// Reference row of factor OP (0 = M, 1 = L, 2 = B) at cell position p.
template <int K, int OP>
__device__ __forceinline__ constexpr double ref_coef(int p, int j) {
  if constexpr (OP == 0)
    return RefCoef<K>::m[p][j];
  else if constexpr (OP == 1)
    return RefCoef<K>::l[p][j];
  else
    return RefCoef<K>::b[p][j];
}

// Band product with the reference row (constants) of the periodic class at
// cell position p; v centred on the row.
template <typename T, int OP, int K>
__device__ __forceinline__ T band_ref(const T* v, int p) {
  constexpr int H = 2 * K;
  const int lo = Band<OP, K>::lo(p);
  T a = (T)ref_coef<K, OP>(p, H + lo) * v[lo];
#pragma unroll
  for (int o = lo + 1; o <= Band<OP, K>::hi(p); ++o) a = mad((T)ref_coef<K, OP>(p, H + o), v[o], a);
  return a;
}

// Rows of B in the boundary cells: a[p] = the row's own product for the
// nodes of cell c at position p, where it differs from the periodic one; v[j]
// = the input at the cell's node j.  The first cell holds rows 1..k-1, the
// next one row k; the last cell holds the k mirrored rows.  (Adding the
// difference of the coefficients to the periodic product would round at the
// size of the larger of the two.)
template <typename T, int K>
__device__ __forceinline__ void boundary_b(T (&a)[K], const T* v, int c, int N) {
  if (c == 0) {
#pragma unroll
    for (int p = 1; p < K; ++p) {
      a[p] = (T)RefCoef<K>::bl[p - 1][0] * v[1];
#pragma unroll
      for (int j = 2; j <= 2 * K; ++j) a[p] = mad((T)RefCoef<K>::bl[p - 1][j - 1], v[j], a[p]);
    }
  }
  if (c == N - 1) {
#pragma unroll
    for (int p = 1; p < K; ++p) {
      a[p] = (T)RefCoef<K>::bl[K - 1 - p][2 * K - 1] * v[-K];
#pragma unroll
      for (int j = 2 * K - 1; j >= 1; --j) a[p] = mad((T)RefCoef<K>::bl[K - 1 - p][j - 1], v[K - j], a[p]);
    }
    if (N == 2) {  // the one inner vertex: both boundary terms
      a[0] = (T)RefCoef<K>::bl[K - 1][0] * v[1 - K];
#pragma unroll
      for (int j = 2; j < 2 * K; ++j) a[0] = mad((T)RefCoef<K>::bl[K - 1][j - 1], v[j - K], a[0]);
#pragma unroll
      for (int j = 0; j < K; ++j) a[0] = mad((T)RefCoef<K>::db[K - 1][K - 1 - j], v[j], a[0]);
    } else {
      a[0] = (T)RefCoef<K>::bl[K - 1][3 * K - 1] * v[-2 * K];
#pragma unroll
      for (int j = 3 * K - 1; j >= 1; --j) a[0] = mad((T)RefCoef<K>::bl[K - 1][j - 1], v[K - j], a[0]);
    }
  } else if (c == 1) {
    a[0] = (T)RefCoef<K>::bl[K - 1][0] * v[1 - K];
#pragma unroll
    for (int j = 2; j <= 3 * K; ++j) a[0] = mad((T)RefCoef<K>::bl[K - 1][j - 1], v[j - K], a[0]);
  }
}

}  // namespace ref
}  // namespace c0ip
