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

// The rows of a tile of kListTile x kListTile buckets (i0, j0) .. of a layer,
// by one workgroup.  One thread per bucket would loop over the N points twice,
// and over its candidates' pairs (30 ms for 31 layers of 2000 points, 23 for 366
// of 500; a whole plan of them now takes 1.9 and 2.6 ms); here the
// workgroup first lists the points that can win anywhere in the tile (a
// bucket's limit is at most its tile's), in increasing index, and 16 lanes per
// bucket then share those.  Per step of the grid optimizer (128 x 128
// buckets, 500 points) 10 us; tiles of 8 x 8 and 4 lanes take 24, the corner
// tests of the crowded buckets being the longest chain, and tiles of 2 x 2
// read all points too often.
// g: the layer's N records; list: LDS, [N].  Returns false in the lane whose
// bucket's candidates did not fit.
constexpr int kListTile = 4, kListThreads = 256;
constexpr int kListBuckets = kListTile * kListTile;
constexpr int kPerBucket = kListThreads / kListBuckets;
constexpr int kTileCand = 64;  // candidates of a bucket before the corner test
struct ListLds {
  uint16_t cand[kListBuckets][kTileCand];
  double red[4][kListThreads / 64];
  int wave_n[kListThreads / 64];
};
__device__ __forceinline__ bool list_tile(float4* list, ListLds& lds, const float4* g, int N,
                                          const float* lo, const float* scale, const int32_t* B,
                                          int i0, int j0, uint16_t* rows, uint16_t* longs,
                                          int pool) {
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  const double w0 = 1.0 / (double)scale[0], w1 = 1.0 / (double)scale[1];
  auto box_of = [&](int i, int j, int n) {
    BucketBox b;
    b.a0 = (double)lo[0] + (double)i * w0 - w0 / 64.0;
    b.b0 = (double)lo[0] + (double)(i + n) * w0 + w0 / 64.0;
    b.a1 = (double)lo[1] + (double)j * w1 - w1 / 64.0;
    b.b1 = (double)lo[1] + (double)(j + n) * w1 + w1 / 64.0;
    return b;
  };
  BucketBox tile = box_of(i0, j0, kListTile);
  double U = __builtin_huge_val(), hmax = 0.0, G0 = 0.0, G1 = 0.0;
  for (int p = t; p < N; p += kListThreads) {
    const float4 q = g[p];
    U = fmin(U, tile.far2(q.x, q.y));
    hmax = fmax(hmax, (double)q.w);
    G0 = fmax(G0, fabs((double)q.x));
    G1 = fmax(G1, fabs((double)q.y));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    U = fmin(U, __shfl_xor(U, off, 64));
    hmax = fmax(hmax, __shfl_xor(hmax, off, 64));
    G0 = fmax(G0, __shfl_xor(G0, off, 64));
    G1 = fmax(G1, __shfl_xor(G1, off, 64));
  }
  if (lane == 0) {
    lds.red[0][wave] = U;
    lds.red[1][wave] = hmax;
    lds.red[2][wave] = G0;
    lds.red[3][wave] = G1;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kListThreads / 64; ++w) {
    U = fmin(U, lds.red[0][w]);
    hmax = fmax(hmax, lds.red[1][w]);
    G0 = fmax(G0, lds.red[2][w]);
    G1 = fmax(G1, lds.red[3][w]);
  }
  tile.set_error(hmax, G0, G1);
  const double tile_thr = tile.limit(U);
  int n = 0;
  for (int p0 = 0; p0 < N; p0 += kListThreads) {
    const int p = p0 + t;
    float4 q = g[p < N ? p : 0];
    const bool in = p < N && tile.near2(q.x, q.y) <= tile_thr;
    const uint64_t mask = __ballot(in);
    if (lane == 0) lds.wave_n[wave] = __popcll(mask);
    __syncthreads();
    int at = n + __popcll(mask & ((1ull << lane) - 1));
#pragma unroll
    for (int w = 0; w < kListThreads / 64; ++w) {
      if (w < wave) at += lds.wave_n[w];
      n += lds.wave_n[w];
    }
    if (in) {
      q.z = __int_as_float(p);
      list[at] = q;
    }
    __syncthreads();
  }
  const int b = t / kPerBucket, sub = t % kPerBucket;
  const int bi = i0 + b / kListTile, bj = j0 + b % kListTile;
  BucketBox box = box_of(bi, bj, 1);
  box.set_error(hmax, G0, G1);
  U = __builtin_huge_val();
  float nx = list[0].x, ny = list[0].y;  // n >= 1: the point that sets the tile's U
  for (int p = sub; p < n; p += kPerBucket) {
    const float4 q = list[p];
    const double d = box.far2(q.x, q.y);
    nx = d < U ? q.x : nx;
    ny = d < U ? q.y : ny;
    U = fmin(U, d);
  }
#pragma unroll
  for (int off = 1; off < kPerBucket; off <<= 1) {
    const double o = __shfl_xor(U, off, 64);
    const float ox = __shfl_xor(nx, off, 64), oy = __shfl_xor(ny, off, 64);
    nx = o < U ? ox : nx;
    ny = o < U ? oy : ny;
    U = fmin(U, o);
  }
  // (on equal U the lanes may hold different points; each is a valid witness)
  const double thr = box.limit(U);
  constexpr uint64_t kGroup = ~0ull >> (64 - kPerBucket);
  const int shift = lane & ~(kPerBucket - 1);
  int c = 0;
  for (int p0 = 0; p0 < n; p0 += kPerBucket) {
    const float4 q = list[min(p0 + sub, n - 1)];
    const bool in = p0 + sub < n && box.near2(q.x, q.y) <= thr && !box.beaten(q.x, q.y, nx, ny);
    const uint64_t group = __ballot(in) >> shift & kGroup;
    const int at = c + __popcll(group & ((1ull << sub) - 1));
    if (in && at < kTileCand) lds.cand[b][at] = (uint16_t)(p0 + sub);
    c += __popcll(group);
  }
  __syncthreads();
  const int listed = c <= kTileCand ? c : 0;
  uint64_t keep = 0;
  for (int p = sub; p < listed; p += kPerBucket) {
    const float4 gp = list[lds.cand[b][p]];
    bool out = false;
    for (int q = 0; q < listed && !out; ++q) {
      const float4 gq = list[lds.cand[b][q]];
      out = q != p && box.beaten(gp.x, gp.y, gq.x, gq.y);
    }
    keep |= out ? 0ull : 1ull << p;
  }
#pragma unroll
  for (int off = 1; off < kPerBucket; off <<= 1) keep |= __shfl_xor(keep, off, 64);
  if (sub != 0 || bi >= B[0] || bj >= B[1]) return true;
  return write_bucket_row(rows + (int64_t)(bi * B[1] + bj) * kBucketRow, longs, pool, N,
                          c <= kTileCand, __popcll(keep), [&](int) {
                            // called in order
                            const int p = __ffsll((unsigned long long)keep) - 1;
                            keep &= keep - 1;
                            return __float_as_int(list[lds.cand[b][p]].z);
                          });
}

}  // namespace qtree
