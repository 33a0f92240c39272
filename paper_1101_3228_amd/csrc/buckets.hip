// Candidate lists of the d = 2 bucketed cell search.  A layer's reachable
// box is cut into buckets; bucket R lists every grid point p that can be the
// FP32 argmin of the half-norm key k_p(x) = h_p - <x, g_p> for some x in R.
// With u = 2^-24 the key carries an error below
// E(x) = 4.1 u (max_p h_p + |x_0| max_p |g_0| + |x_1| max_p |g_1|), so the
// FP32 winner p* for x has |x - g_p*|^2 <= min_q |x - g_q|^2 + 4 E(x) (both
// keys may err by E).  Over R, min_q |x - g_q|^2 <= U = min_q max over R's
// corners of |c - g_q|^2, and |x - g_p|^2 >= lo_p, the squared distance from
// g_p to R; so only p with lo_p <= U + 4 E_R (E_R the bound over R, doubled
// here for margin) can win.  Of these, p is struck out when some q is nearer
// by more than 4 E_R all over R: |x - g_p|^2 - |x - g_q|^2 is linear in x, so
// its least value over R is at a corner.  (That proof does not need q to stay
// on the list; equal points never strike out each other.)  What remains are
// the points whose cells meet R, 1.x on average where the first test alone
// kept about 3.  R is the bucket widened by 1/64 of its width on every side,
// more than the FP32 rounding of the bucket index can move a point.  FP64
// throughout.  Rows as described at LayerDev.
#include "bucket_list.hpp"

namespace qtree {

namespace {
constexpr int kBlock = 256;
}

__global__ __launch_bounds__(kBlock) void bucket_build_kernel(const LayerDev* layers, int nl,
                                                              int total, const float4* pts,
                                                              uint16_t* rows, uint16_t* longs,
                                                              int pool) {
  __shared__ uint16_t cand[kBlock][kLongCap];
  const int t = (int)(blockIdx.x * kBlock + threadIdx.x);
  if (t >= total) return;
  int lo = 0, hi = nl - 1;  // the layer holding bucket t: largest k with bk_off_k <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (layers[mid].bk_off <= t) lo = mid; else hi = mid - 1;
  }
  const LayerDev& L = layers[lo];
  const int r = t - L.bk_off;
  const int i = r / L.bk_B[1], j = r - i * L.bk_B[1];
  const double w0 = 1.0 / (double)L.bk_scale[0], w1 = 1.0 / (double)L.bk_scale[1];
  BucketBox box;
  box.a0 = (double)L.bk_lo[0] + (double)i * w0 - w0 / 64.0;
  box.b0 = (double)L.bk_lo[0] + (double)(i + 1) * w0 + w0 / 64.0;
  box.a1 = (double)L.bk_lo[1] + (double)j * w1 - w1 / 64.0;
  box.b1 = (double)L.bk_lo[1] + (double)(j + 1) * w1 + w1 / 64.0;
  const float4* g = pts + L.pt_off;
  double U = __builtin_huge_val(), hmax = 0.0, G0 = 0.0, G1 = 0.0;
  float4 near = g[0];  // a point whose farthest corner distance is U
  for (int p = 0; p < L.N; ++p) {
    const float4 q = g[p];
    const double d = box.far2(q.x, q.y);
    near = d < U ? q : near;
    U = fmin(U, d);
    hmax = fmax(hmax, (double)q.w);
    G0 = fmax(G0, fabs((double)q.x));
    G1 = fmax(G1, fabs((double)q.y));
  }
  box.set_error(hmax, G0, G1);
  const double thr = box.limit(U);
  uint16_t* list = cand[threadIdx.x];
  int c = 0;
  for (int p = 0; p < L.N; ++p) {
    const float4 q = g[p];
    if (box.near2(q.x, q.y) <= thr && !box.beaten(q.x, q.y, near.x, near.y)) {
      if (c < kLongCap) list[c] = (uint16_t)p;
      ++c;
    }
  }
  const int listed = c < kLongCap ? c : kLongCap;
  int kept = 0;  // ends >= 1: the nearest point at some corner stays
  uint32_t keep = 0;
  for (int p = 0; p < listed; ++p) {
    bool out = false;
    for (int q = 0; q < listed; ++q) {
      const float4 gp = g[list[p]], gq = g[list[q]];
      out = out || (q != p && box.beaten(gp.x, gp.y, gq.x, gq.y));
    }
    keep |= out ? 0u : 1u << p;
  }
  for (int p = 0; p < listed; ++p)
    if (keep >> p & 1) list[kept++] = list[p];
  write_bucket_row(rows + (int64_t)t * kBucketRow, longs, pool, L.N, c <= kLongCap, kept,
                   [&](int e) { return (int)list[e]; });
}

hipError_t launch_bucket_build(const LayerDev* layers, int n_layers_total, int total_buckets,
                               const float4* pts, uint16_t* rows, uint16_t* longs,
                               hipStream_t s) {
  if (total_buckets <= 0) return hipSuccess;
  const hipError_t e = launch_zero_i32(reinterpret_cast<int32_t*>(longs), 1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(bucket_build_kernel, dim3((unsigned)((total_buckets + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, layers, n_layers_total, total_buckets, pts, rows, longs,
                     (int)long_rows(total_buckets));
  return hipGetLastError();
}

}  // namespace qtree
