// One bucket of the d = 2 cell search: which points beat which all over it,
// and its row (layout at LayerDev in qtree_internal.hpp).
#pragma once
#include "qtree_internal.hpp"

namespace qtree {

// A bucket [a0, b0] x [a1, b1] and the bound E on a key's error over it.
struct BucketBox {
  double a0, b0, a1, b1, E;
  // Squared distance from q to the farthest corner, and to the bucket.
  __device__ __forceinline__ double far2(float x, float y) const {
    const double d0 = fmax(fabs(a0 - (double)x), fabs(b0 - (double)x));
    const double d1 = fmax(fabs(a1 - (double)y), fabs(b1 - (double)y));
    return d0 * d0 + d1 * d1;
  }
  __device__ __forceinline__ double near2(float x, float y) const {
    const double e0 = fmax(0.0, fmax(a0 - (double)x, (double)x - b0));
    const double e1 = fmax(0.0, fmax(a1 - (double)y, (double)y - b1));
    return e0 * e0 + e1 * e1;
  }
  // E from the largest half norm and coordinates of the points.
  __device__ __forceinline__ void set_error(double hmax, double G0, double G1) {
    const double X0 = fmax(fabs(a0), fabs(b0)), X1 = fmax(fabs(a1), fabs(b1));
    E = 2.0 * 4.1 * 0x1p-24 * (hmax + X0 * G0 + X1 * G1);
  }
  // Largest near2 of a point that can win, min far2 being U.
  __device__ __forceinline__ double limit(double U) const {
    return U * (1.0 + 1e-9) + 4.0 * E;
  }
  // Whether q is nearer than p by more than 4 E at all four corners.
  __device__ __forceinline__ bool beaten(float px, float py, float qx, float qy) const {
    // |x - p|^2 - |x - q|^2 = 2 <x, q - p> + |p|^2 - |q|^2, least over the corners
    const double u0 = (double)qx - (double)px, u1 = (double)qy - (double)py;
    const double c = (double)px * (double)px + (double)py * (double)py -
                     (double)qx * (double)qx - (double)qy * (double)qy;
    return c + 2.0 * (fmin(a0 * u0, b0 * u0) + fmin(a1 * u1, b1 * u1)) > 4.0 * E;
  }
};

// Row of a bucket whose `kept` candidates are entry(0), entry(1), ... (`fits`:
// all of them are there).  Entries are byte offsets of 8-byte pairs (at most
// 4096 points); the pads all name one record, so the lanes of a wave that
// read it share one LDS access.  More than kBucketCap candidates go to a pool
// row (counted in row 0's first word); false where they do not fit there.
template <class ENTRY>
__device__ __forceinline__ bool write_bucket_row(uint16_t* out, uint16_t* longs, int pool, int N,
                                                 bool fits, int kept, ENTRY&& entry) {
  const uint16_t pad = (uint16_t)(8 * N);
  int size = kBucketRow;
  if (!fits || kept > kBucketCap) {
    for (int e = 1; e < kBucketRow; ++e) out[e] = pad;
    uint32_t at = 0;
    if (fits && kept <= kLongCap) at = 1u + atomicAdd(reinterpret_cast<uint32_t*>(longs), 1u);
    if (at == 0 || at >= (uint32_t)pool) {
      out[0] = kBucketFull;
      return false;
    }
    out[0] = kBucketLong;
    out[6] = (uint16_t)(at & 0xFFFFu);
    out[7] = (uint16_t)(at >> 16);
    out = longs + (int64_t)at * kLongRow;
    size = kLongRow;
  }
  out[0] = (uint16_t)kept;
  for (int e = 0; e < kept; ++e) out[1 + e] = (uint16_t)(8 * entry(e));
  for (int e = 1 + kept; e < size; ++e) out[e] = pad;
  return true;
}

}  // namespace qtree
