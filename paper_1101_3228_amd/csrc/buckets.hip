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
#include <algorithm>

#include "bucket_list.hpp"
#include "qtree_search.hpp"

namespace qtree {

namespace {
constexpr int kBlock = 256;
}

// Workgroup (x, k): tile x of layer k.
__global__ __launch_bounds__(kListThreads) void bucket_build_kernel(const LayerDev* layers,
                                                                    const float4* pts,
                                                                    uint16_t* rows,
                                                                    uint16_t* longs, int pool) {
  extern __shared__ float4 list[];
  __shared__ ListLds lds;
  const LayerDev& L = layers[blockIdx.y];
  const int t0 = (L.bk_B[0] + kListTile - 1) / kListTile;
  const int t1 = (L.bk_B[1] + kListTile - 1) / kListTile;
  if ((int)blockIdx.x >= t0 * t1) return;
  list_tile(list, lds, pts + L.pt_off, L.N, L.bk_lo, L.bk_scale, L.bk_B,
            (int)blockIdx.x / t1 * kListTile, (int)blockIdx.x % t1 * kListTile,
            rows + (int64_t)L.bk_off * kBucketRow, longs, pool);
}

hipError_t launch_bucket_build(const LayerDev* layers, int n_layers_total, int maxN,
                               int64_t total_buckets, const float4* pts, uint16_t* rows,
                               uint16_t* longs, hipStream_t s) {
  if (total_buckets <= 0) return hipSuccess;
  hipError_t e = launch_zero_i32(reinterpret_cast<int32_t*>(longs), 1, s);
  if (e != hipSuccess) return e;
  const size_t lds = sizeof(float4) * (size_t)maxN;
  if (lds + sizeof(ListLds) > 65536) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(bucket_build_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const unsigned tiles = (unsigned)((bucket_side(maxN) + kListTile - 1) / kListTile);
  for (int k0 = 0; k0 < n_layers_total; k0 += 65535) {
    const unsigned layers_now = (unsigned)std::min(65535, n_layers_total - k0);
    hipLaunchKernelGGL(bucket_build_kernel, dim3(tiles * tiles, layers_now), dim3(kListThreads),
                       lds, s, layers + k0, pts, rows, longs, (int)long_rows(total_buckets));
  }
  return hipGetLastError();
}

// The d = 3 tables, by the same rules (E with three products: 6.2 u).  As a
// box has tens of thousands of buckets, a workgroup takes a tile of 4 x 4 x 4 of
// them, first lists the points that can win anywhere in the tile (a bucket's
// limit is at most its tile's), in increasing index, and 4 lanes per bucket
// then share those (12 layers of 990 points, 5.6 10^5 buckets: 0.27 ms).
namespace {
struct CubeBox {
  double a[3], b[3], E;
  __device__ __forceinline__ void place(const Cubes& C, const int* i, int n) {
    for (int r = 0; r < 3; ++r) {
      const double w = 1.0 / (double)C.scale[r];
      a[r] = (double)C.lo[r] + (double)i[r] * w - w / 64.0;
      b[r] = (double)C.lo[r] + (double)(i[r] + n) * w + w / 64.0;
    }
  }
  __device__ __forceinline__ void set_error(double hmax, const double* G) {
    E = hmax;
    for (int r = 0; r < 3; ++r) E += fmax(fabs(a[r]), fabs(b[r])) * G[r];
    E *= 2.0 * 6.2 * 0x1p-24;
  }
  __device__ __forceinline__ double far2(const float4& q) const {
    const double c[3] = {(double)q.x, (double)q.y, (double)q.z};
    double d = 0.0;
    for (int r = 0; r < 3; ++r) {
      const double e = fmax(fabs(a[r] - c[r]), fabs(b[r] - c[r]));
      d += e * e;
    }
    return d;
  }
  __device__ __forceinline__ double near2(const float4& q) const {
    const double c[3] = {(double)q.x, (double)q.y, (double)q.z};
    double d = 0.0;
    for (int r = 0; r < 3; ++r) {
      const double e = fmax(0.0, fmax(a[r] - c[r], c[r] - b[r]));
      d += e * e;
    }
    return d;
  }
  __device__ __forceinline__ double limit(double U) const {
    return U * (1.0 + 1e-9) + 4.0 * E;
  }
  // Whether q is nearer than p by more than 4 E at all eight corners.
  __device__ __forceinline__ bool beaten(const float4& p, const float4& q) const {
    const double pc[3] = {(double)p.x, (double)p.y, (double)p.z};
    const double qc[3] = {(double)q.x, (double)q.y, (double)q.z};
    double c = 0.0;
    for (int r = 0; r < 3; ++r) {
      const double u = qc[r] - pc[r];
      c += pc[r] * pc[r] - qc[r] * qc[r] + 2.0 * fmin(a[r] * u, b[r] * u);
    }
    return c > 4.0 * E;
  }
};
constexpr int kCubesPerTile = kCubeTile * kCubeTile * kCubeTile;
constexpr int kPerCube = kBlock / kCubesPerTile;
constexpr int kCubeCand = 64;  // candidates of a bucket before the corner test
constexpr int kMaxCubeN = 4096;
}  // namespace

__global__ __launch_bounds__(kBlock) void cube_build_kernel(const Cubes* cubes, int nl,
                                                            const float4* pts, uint16_t* rows) {
  __shared__ uint16_t list[kMaxCubeN];
  __shared__ uint16_t cand[kCubesPerTile][kCubeCand];
  __shared__ double red[5][kBlock / 64];
  __shared__ int wave_n[kBlock / 64];
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  const int row0 = (int)blockIdx.x * kCubesPerTile;
  int lo = 0, hi = nl - 1;  // the layer of the tile: largest k with off_k <= row0
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cubes[mid].off <= row0) lo = mid; else hi = mid - 1;
  }
  const Cubes& C = cubes[lo];
  if (C.B[0] == 0) return;  // rows of a layer without a box
  const int N = C.N;
  const float4* g = pts + C.pt_off;
  const int nt1 = C.B[1] / kCubeTile, nt2 = C.B[2] / kCubeTile;
  const int tile_id = (row0 - C.off) / kCubesPerTile;
  const int i0[3] = {tile_id / (nt1 * nt2) * kCubeTile, tile_id / nt2 % nt1 * kCubeTile,
                     tile_id % nt2 * kCubeTile};
  CubeBox tile;
  tile.place(C, i0, kCubeTile);
  double v[5] = {-__builtin_huge_val(), 0.0, 0.0, 0.0, 0.0};  // -U, h, |g_r|: maxima
  for (int p = t; p < N; p += kBlock) {
    const float4 q = g[p];
    v[0] = fmax(v[0], -tile.far2(q));
    v[1] = fmax(v[1], (double)q.w);
    v[2] = fmax(v[2], fabs((double)q.x));
    v[3] = fmax(v[3], fabs((double)q.y));
    v[4] = fmax(v[4], fabs((double)q.z));
  }
#pragma unroll
  for (int e = 0; e < 5; ++e) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[e] = fmax(v[e], __shfl_xor(v[e], off, 64));
    if (lane == 0) red[e][wave] = v[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 5; ++e)
    for (int w = 0; w < kBlock / 64; ++w) v[e] = fmax(v[e], red[e][w]);
  tile.set_error(v[1], v + 2);
  const double tile_thr = tile.limit(-v[0]);
  int n = 0;
  for (int p0 = 0; p0 < N; p0 += kBlock) {
    const int p = p0 + t;
    const bool in = p < N && tile.near2(g[p < N ? p : 0]) <= tile_thr;
    const uint64_t mask = __ballot(in);
    if (lane == 0) wave_n[wave] = __popcll(mask);
    __syncthreads();
    int at = n + __popcll(mask & ((1ull << lane) - 1));
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
      if (w < wave) at += wave_n[w];
      n += wave_n[w];
    }
    if (in) list[at] = (uint16_t)p;
    __syncthreads();
  }
  const int b = t / kPerCube, sub = t % kPerCube;
  const int ib[3] = {i0[0] + b / (kCubeTile * kCubeTile), i0[1] + b / kCubeTile % kCubeTile,
                     i0[2] + b % kCubeTile};
  CubeBox box;
  box.place(C, ib, 1);
  box.set_error(v[1], v + 2);
  double U = __builtin_huge_val();
  int near = list[0];  // n >= 1: the point that sets the tile's U
  for (int p = sub; p < n; p += kPerCube) {
    const double d = box.far2(g[list[p]]);
    near = d < U ? list[p] : near;
    U = fmin(U, d);
  }
#pragma unroll
  for (int off = 1; off < kPerCube; off <<= 1) {
    const double o = __shfl_xor(U, off, 64);
    const int on = __shfl_xor(near, off, 64);
    near = o < U ? on : near;
    U = fmin(U, o);
  }
  const float4 gn = g[near];
  const double thr = box.limit(U);
  constexpr uint64_t kGroup = ~0ull >> (64 - kPerCube);
  const int shift = lane & ~(kPerCube - 1);
  int c = 0;
  for (int p0 = 0; p0 < n; p0 += kPerCube) {
    const int p = list[min(p0 + sub, n - 1)];
    const float4 q = g[p];
    const bool in = p0 + sub < n && box.near2(q) <= thr && !box.beaten(q, gn);
    const uint64_t group = __ballot(in) >> shift & kGroup;
    const int at = c + __popcll(group & ((1ull << sub) - 1));
    if (in && at < kCubeCand) cand[b][at] = (uint16_t)p;
    c += __popcll(group);
  }
  __syncthreads();
  const int listed = c <= kCubeCand ? c : 0;
  uint64_t keep = 0;
  for (int p = sub; p < listed; p += kPerCube) {
    const float4 gp = g[cand[b][p]];
    bool out = false;
    for (int q = 0; q < listed && !out; ++q)
      out = q != p && box.beaten(gp, g[cand[b][q]]);
    keep |= out ? 0ull : 1ull << p;
  }
#pragma unroll
  for (int off = 1; off < kPerCube; off <<= 1) keep |= __shfl_xor(keep, off, 64);
  if (sub != 0) return;
  uint16_t* out = rows + (size_t)(C.off + (ib[0] * C.B[1] + ib[1]) * C.B[2] + ib[2]) * kCubeRow;
  const int kept = __popcll(keep);  // >= 1: the nearest point at some corner stays
  const bool fits = c <= kCubeCand && kept <= kCubeCap;
  out[0] = fits ? (uint16_t)kept : kCubeFull;
  for (int e = 1; e < kCubeRow; ++e) {
    uint16_t p = (uint16_t)N;
    if (fits && keep) {
      p = cand[b][__ffsll((unsigned long long)keep) - 1];
      keep &= keep - 1;
    }
    out[e] = p;
  }
}

// Workgroup k: the samples of layer k's pairs whose bucket has no list, or that
// are outside the box.
__global__ __launch_bounds__(kBlock) void cube_probe_kernel(const LayerDev* layers, Cubes* cubes,
                                                            const uint16_t* rows) {
  const int k = (int)blockIdx.x;
  unsigned int miss[2] = {0u, 0u};
  for (int m = (int)threadIdx.x; m < kCubeProbes; m += kBlock) {
    float z[3], e[3], x[2][3];
    layer_normals<3>(0u, 0u, 0u, k, (uint64_t)m, z, e);
    layer_pair<3>(layers[k], z, e, x[0], x[1]);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int r = cube_of(cubes[k + q], x[q]);
      const bool no = r < 0 || rows[(size_t)r * kCubeRow] == kCubeFull;
      miss[q] += (unsigned int)__popcll(__ballot(no));
    }
  }
  if ((threadIdx.x & 63) < 2)
    atomicAdd(&cubes[k + (int)(threadIdx.x & 63)].misses, miss[threadIdx.x & 63]);
}

hipError_t launch_cube_build(const LayerDev* layers, Cubes* cubes, int n_layers_total, int total,
                             const float4* pts, uint16_t* rows, hipStream_t s) {
  if (total <= 0) return hipSuccess;
  if (total % kCubesPerTile) return hipErrorInvalidValue;
  hipLaunchKernelGGL(cube_build_kernel, dim3((unsigned)(total / kCubesPerTile)), dim3(kBlock), 0, s,
                     cubes, n_layers_total, pts, rows);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cube_probe_kernel, dim3((unsigned)(n_layers_total - 1)), dim3(kBlock), 0, s,
                     layers, cubes, rows);
  return hipGetLastError();
}

}  // namespace qtree
