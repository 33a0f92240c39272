// Conditional expectation of 16 rows of a count block as a matrix product on
// the FP64 matrix cores: S(16 rows x 16 columns) = C(16 x len) V(len x 16),
// v_mfma_f64_16x16x4_f64 with the int32 counts converted on the fly.
//
// Operand layout: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] of a
// K-step of four columns, and D[l / 16 + 4 r][l % 16], r = 0..3.  The K order
// is free, so lane group g = l / 16 takes columns 16 s + 4 g .. + 3 of chunk
// s with one 16-byte load of its row, and the chunk's four K-steps use one
// of them each.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qtree {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Four consecutive values at their own type's alignment (count rows start at
// any entry; global loads of 16 bytes need 4-byte alignment).
struct __attribute__((packed, aligned(4))) Int4U {
  int32_t v[4];
};
struct __attribute__((packed, aligned(8))) Dbl4U {
  double v[4];
};

// Elements d .. d + 3 of (x, 0, 0, ...), d >= 0 (a lane's own).
template <class T>
__device__ __forceinline__ void drop_front(T (&x)[4], int d) {
  const bool one = (d & 1) != 0, two = (d & 2) != 0;
#pragma unroll
  for (int u = 0; u < 3; ++u) x[u] = one ? x[u + 1] : x[u];
  x[3] = one ? (T)0 : x[3];
#pragma unroll
  for (int u = 0; u < 4; ++u) x[u] = d >= 4 ? (T)0 : (two ? (u < 2 ? x[u + 2] : (T)0) : x[u]);
}

// Columns j .. j + 3 of a row of n >= 4 entries, zero past its end: a load
// that would run past it starts four entries before the end, and what it
// brings too early is dropped.  (Loads under a lane's own branch are each
// waited for inside it; these stay in flight together.)
struct Cols4 {
  int at, drop;
  __device__ Cols4(int j, int n) : at(min(j, n - 4)), drop(j - at) {}
};

// A chunks, this lane's columns j + stride a .. + 3 of each (as Cols4): the
// loads, and the drops where a chunk of the wave crosses the end.
template <int A>
__device__ __forceinline__ void load_cols(const int32_t* __restrict__ row, int n, int j, int stride,
                                          int32_t (&c)[A][4]) {
#pragma unroll
  for (int a = 0; a < A; ++a) {
    const Int4U q = *reinterpret_cast<const Int4U*>(row + Cols4(j + stride * a, n).at);
#pragma unroll
    for (int u = 0; u < 4; ++u) c[a][u] = q.v[u];
  }
}
template <int A>
__device__ __forceinline__ void load_cols(const double* __restrict__ v, int n, int j, int stride,
                                          double (&x)[A][4]) {
#pragma unroll
  for (int a = 0; a < A; ++a) {
    const Dbl4U y = *reinterpret_cast<const Dbl4U*>(v + Cols4(j + stride * a, n).at);
#pragma unroll
    for (int u = 0; u < 4; ++u) x[a][u] = y.v[u];
  }
}
template <int A, class T>
__device__ __forceinline__ void drop_tails(int n, int j, int stride, T (&x)[A][4]) {
#pragma unroll
  for (int a = 0; a < A; ++a) drop_front(x[a], Cols4(j + stride * a, n).drop);
}

// Elements 0 .. 3 - d of x behind d zeros, d >= 0 (a lane's own).
template <class T>
__device__ __forceinline__ void drop_back(T (&x)[4], int d) {
  const bool one = (d & 1) != 0, two = (d & 2) != 0;
#pragma unroll
  for (int u = 3; u > 0; --u) x[u] = one ? x[u - 1] : x[u];
  x[0] = one ? (T)0 : x[0];
#pragma unroll
  for (int u = 3; u >= 0; --u) x[u] = d >= 4 ? (T)0 : (two ? (u > 1 ? x[u - 2] : (T)0) : x[u]);
}

// Counts of A chunks from a row that holds columns [lo, hi), hi > lo, at
// row[lo .. hi) (a band, or a row too short for Cols4), zero outside.  Rows of
// four columns and more (`wide`, the same for the wave) are loaded four at a
// time, as by Cols4 but at both ends.
template <int A>
__device__ __forceinline__ void load_band(const int32_t* __restrict__ row, int lo, int hi, int j,
                                          int stride, bool wide, int32_t (&c)[A][4]) {
  if (wide) {
    int shift[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
      const int t = j + stride * a, at = min(max(t, lo), hi - 4);
      shift[a] = t - at;
      const Int4U q = *reinterpret_cast<const Int4U*>(row + at);
#pragma unroll
      for (int u = 0; u < 4; ++u) c[a][u] = q.v[u];
    }
#pragma unroll
    for (int a = 0; a < A; ++a)
      if (__any(shift[a] != 0)) {
        drop_front(c[a], max(shift[a], 0));
        drop_back(c[a], max(-shift[a], 0));
      }
    return;
  }
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int u = 0; u < 4; ++u) c[a][u] = row[min(max(j + stride * a + u, lo), hi - 1)];
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = j + stride * a + u;
      c[a][u] = (t >= lo && t < hi) ? c[a][u] : 0;
    }
}

__device__ __forceinline__ bool finite4(const double (&x)[4]) {
  bool ok = true;
#pragma unroll
  for (int u = 0; u < 4; ++u) ok = ok && __builtin_isfinite(x[u]);
  return ok;
}

// acc += the chunk's 16 x 16 (columns) by 16 x 16 product.  A zero count adds
// nothing whatever its value is; 0 x inf is not zero, so a chunk with a value
// that is not finite goes entry by entry.
__device__ __forceinline__ void chunk_product(const int32_t (&c)[4], const double (&x)[4], int lane,
                                              f64x4& acc) {
  if (!__any((c[0] | c[1] | c[2] | c[3]) != 0)) return;
  if (__all(finite4(x))) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)c[u], x[u], acc, 0, 0, 0);
    return;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    for (int g = 0; g < 4; ++g) {
      const double v = __shfl(x[u], 16 * g + (lane & 15), 64);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int32_t cr = __shfl(c[u], 16 * g + (lane >> 4) + 4 * r, 64);
        if (cr != 0) acc[r] = fma((double)cr, v, acc[r]);
      }
    }
}

}  // namespace qtree
