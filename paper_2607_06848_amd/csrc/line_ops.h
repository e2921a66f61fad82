// Products of short 1-D matrices with the lines of a cell (tensor-product
// operators): y = M x, P values a line, on the even and odd parts of x.
#pragma once

#include <stdint.h>

#include <vector>

// 1-D matrices of one axis in even/odd form: with H = ceil(P/2), Q = floor(P/2),
// e[q H + i] = (M[q][i] + M[q][P-1-i]) / 2 (M itself for i or q the middle),
// o[q Q + i] = (M[q][i] - M[q][P-1-i]) / 2; the transposed product reads the
// same numbers transposed.
constexpr int TP_MAT = 25;   // doubles per matrix: e (16), o (9)

// The matrices are read through the scalar cache.  fresh() hides where the
// pointer comes from, so that every phase loads its own 50 numbers again
// instead of keeping all six matrices in scalar registers (which spilled).
typedef const __attribute__((address_space(4))) double cdouble;
__device__ __forceinline__ cdouble *fresh(cdouble *m) {
  asm volatile("" : "+s"(m));
  return m;
}

// y = M x (T: M^T x) for matrix k of the table (axis, or 3 + axis)
template <int P, bool T>
__device__ __forceinline__ void mul1d(cdouble *m, int k, const double (&x)[P], double (&y)[P]) {
  cdouble *e = m + k * TP_MAT, *o = e + 16;
  constexpr int H = (P + 1) / 2, Q = P / 2;
  double xe[H], xo[Q > 0 ? Q : 1];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    xe[i] = x[i] + x[P - 1 - i];
    xo[i] = x[i] - x[P - 1 - i];
  }
  if (H > Q) xe[Q] = x[Q];
#pragma unroll
  for (int q = 0; q < H; ++q) {
    double s = (T ? e[q] : e[q * H]) * xe[0];
#pragma unroll
    for (int i = 1; i < H; ++i) s = fma(T ? e[i * H + q] : e[q * H + i], xe[i], s);
    if (q < Q) {
      double d = (T ? o[q] : o[q * Q]) * xo[0];
#pragma unroll
      for (int i = 1; i < Q; ++i) d = fma(T ? o[i * Q + q] : o[q * Q + i], xo[i], d);
      y[q] = s + d;
      y[P - 1 - q] = s - d;
    } else {
      y[q] = s;
    }
  }
}

// the even/odd form of the P x P matrix M
template <class T>
static inline void even_odd(int P, const std::vector<T> &M, double *e, double *o) {
  const int H = (P + 1) / 2, Q = P / 2;
  for (int q = 0; q < H; ++q)
    for (int i = 0; i < H; ++i)
      e[q * H + i] = i < Q ? T(0.5) * (M[q * P + i] + M[q * P + P - 1 - i]) : M[q * P + i];
  for (int q = 0; q < H && H > Q; ++q)   // middle row: M[mid][i] = M[mid][P-1-i]
    for (int i = 0; i < Q; ++i)
      if (q == Q) e[q * H + i] = T(0.5) * (M[q * P + i] + M[q * P + P - 1 - i]);
  for (int q = 0; q < Q; ++q)
    for (int i = 0; i < Q; ++i) o[q * Q + i] = T(0.5) * (M[q * P + i] - M[q * P + P - 1 - i]);
}
