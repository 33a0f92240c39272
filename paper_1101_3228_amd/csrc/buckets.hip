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
#include "qtree_internal.hpp"

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
  const double a0 = (double)L.bk_lo[0] + (double)i * w0 - w0 / 64.0;
  const double b0 = (double)L.bk_lo[0] + (double)(i + 1) * w0 + w0 / 64.0;
  const double a1 = (double)L.bk_lo[1] + (double)j * w1 - w1 / 64.0;
  const double b1 = (double)L.bk_lo[1] + (double)(j + 1) * w1 + w1 / 64.0;
  const float4* g = pts + L.pt_off;
  double U = __builtin_huge_val(), hmax = 0.0, G0 = 0.0, G1 = 0.0;
  float4 near = g[0];  // a point whose farthest corner distance is U
  for (int p = 0; p < L.N; ++p) {
    const float4 q = g[p];
    const double d0 = fmax(fabs(a0 - (double)q.x), fabs(b0 - (double)q.x));
    const double d1 = fmax(fabs(a1 - (double)q.y), fabs(b1 - (double)q.y));
    const double d = d0 * d0 + d1 * d1;
    near = d < U ? q : near;
    U = fmin(U, d);
    hmax = fmax(hmax, (double)q.w);
    G0 = fmax(G0, fabs((double)q.x));
    G1 = fmax(G1, fabs((double)q.y));
  }
  const double X0 = fmax(fabs(a0), fabs(b0)), X1 = fmax(fabs(a1), fabs(b1));
  const double E = 2.0 * 4.1 * 0x1p-24 * (hmax + X0 * G0 + X1 * G1);
  const double thr = U * (1.0 + 1e-9) + 4.0 * E;
  // whether q beats p by more than 4 E at all four corners
  auto beaten = [&](const float4& p, const float4& q) {
    // |x - p|^2 - |x - q|^2 = 2 <x, q - p> + |p|^2 - |q|^2, least over the corners
    const double u0 = (double)q.x - (double)p.x, u1 = (double)q.y - (double)p.y;
    const double c = (double)p.x * (double)p.x + (double)p.y * (double)p.y -
                     (double)q.x * (double)q.x - (double)q.y * (double)q.y;
    return c + 2.0 * (fmin(a0 * u0, b0 * u0) + fmin(a1 * u1, b1 * u1)) > 4.0 * E;
  };
  uint16_t* list = cand[threadIdx.x];
  int c = 0;
  for (int p = 0; p < L.N; ++p) {
    const float4 q = g[p];
    const double e0 = fmax(0.0, fmax(a0 - (double)q.x, (double)q.x - b0));
    const double e1 = fmax(0.0, fmax(a1 - (double)q.y, (double)q.y - b1));
    if (e0 * e0 + e1 * e1 <= thr && !beaten(q, near)) {
      if (c < kLongCap) list[c] = (uint16_t)p;
      ++c;
    }
  }
  uint32_t keep = 0;
  const int listed = c < kLongCap ? c : kLongCap;
  for (int p = 0; p < listed; ++p) {
    bool out = false;
    for (int q = 0; q < listed; ++q) out = out || (q != p && beaten(g[list[p]], g[list[q]]));
    keep |= out ? 0u : 1u << p;
  }
  const int kept = __popc(keep);  // >= 1: the nearest point at some corner stays
  // entries are byte offsets of 8-byte pairs (at most 4096 points); the pads
  // all name one record, so the lanes of a wave that read it share one LDS
  // access
  const uint16_t pad = (uint16_t)(8 * L.N);
  uint16_t* out = rows + (int64_t)t * kBucketRow;
  int size = kBucketRow;
  if (c > kLongCap || kept > kBucketCap) {
    for (int e = 1; e < kBucketRow; ++e) out[e] = pad;
    // a pool row; they are counted in row 0's first word
    uint32_t at = 0;
    if (c <= kLongCap) at = 1u + atomicAdd(reinterpret_cast<uint32_t*>(longs), 1u);
    if (at == 0 || at >= (uint32_t)pool) {
      out[0] = kBucketFull;
      return;
    }
    out[0] = kBucketLong;
    out[6] = (uint16_t)(at & 0xFFFFu);
    out[7] = (uint16_t)(at >> 16);
    out = longs + (int64_t)at * kLongRow;
    size = kLongRow;
  }
  out[0] = (uint16_t)kept;
  int e = 1;
  for (int p = 0; p < listed; ++p)
    if (keep >> p & 1) out[e++] = (uint16_t)(8 * list[p]);
  for (; e < size; ++e) out[e] = pad;
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
