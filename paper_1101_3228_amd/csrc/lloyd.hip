// Grid optimization on the device: randomized Lloyd iteration for the
// quadratic quantization error E min_i |X - x_i|^2 of X = L z, z ~ N(0, I_d)
// (Sec. 2, eq. Qerr).  The paper takes precomputed optimal grids for
// Gaussian marginals and moment-matching grids otherwise; here a grid is
// improved by Lloyd steps, each moving every point to the mean of the
// samples of its Voronoi cell (the stationarity condition of eq. Qerr).
//
// One step on the device:
//   tables (d = 2 on Philox samples): the bucket lists of the tree's 2-D cell
//     search for the current grid over the box of the samples.
//   accumulate: a persistent grid of workgroups; each stages the current grid
//     (d >= 2: records (g, |g|^2 / 2), or pairs where there are tables; d = 1:
//     midpoints padded with +inf) in LDS, draws samples (Philox counter
//     (m, step, 0, 2), Box-Muller, X = L z as fused multiply-add chains from
//     0), assigns them with the tree's own cell search, and adds to LDS
//     accumulators: the count, each coordinate as the integer rint(x 2^24) and
//     the squared distance to the cell's point as rint(|x - g|^2 2^16) (FP64).
//     The workgroup stores its totals, zeros included, as row b of a partial
//     table with plain stores.
//   update: each workgroup sums the columns of 4 cells over the table's rows
//     (integer sums make the result independent of the order of the samples
//     and of the workgroups; the table replaces device atomics from every
//     workgroup onto the same ~N d words, which serialized at the L2), and
//     moves them: new point = (sum 2^-24) / count in FP64, rounded once to
//     FP32 (an empty cell keeps its point), or the point moved a fraction
//     gamma of the way there; one more workgroup forms the distortion.
//
// The samples may instead be windows of a caller's sample set (Lloyd's
// method on an empirical measure, for marginals of any law): step t takes
// samples (t batch + j) mod M, and samples with a coordinate outside
// [-64, 64] (or not a number) are skipped and counted.
//
// Moment-matching grids (Sec. 2, the sub-optimal grids for marginals without
// an optimal grid): exact integer sums of x and x x' over the admissible
// samples of a set, then, in one workgroup, the mean, covariance and lower
// Cholesky factor in FP64 and the grid mean + chol base.
#include "bucket_list.hpp"
#include "qtree_internal.hpp"
#include "qtree_rng.hpp"
#include "qtree_search.hpp"

namespace qtree {

namespace {

constexpr int kBlock = 256;
constexpr int kSamplesNd = 8;  // samples per lane per round, d >= 2 (share each record read)

__device__ __forceinline__ long long fixed_of(double v, double scale) {
  return (long long)__builtin_rint(v * scale);
}

// Sample j of the step's window of the caller's set; false (and x = 0) when
// a coordinate is outside [-64, 64] or not a number.
template <int D>
__device__ __forceinline__ bool set_sample(const LloydArgs& a, uint64_t j, float* x) {
  uint64_t q = a.start + j;
  if (q >= a.Ms) q %= a.Ms;
  bool ok = true;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    x[c] = a.xs[q * D + c];
    ok = ok && fabsf(x[c]) <= 64.0f;
  }
  if (!ok) {
#pragma unroll
    for (int c = 0; c < D; ++c) x[c] = 0.0f;
  }
  return ok;
}

// X = L z for sample m of the step (z from one Philox block).
template <int D>
__device__ __forceinline__ void lloyd_sample(const LloydArgs& a, uint64_t m, float* x) {
  const U4 r = philox4x32_10(U4{(uint32_t)m, a.it_ctr, 0u, 2u}, a.key0, a.key1);
  float z[4];
  box_muller(r.x, r.y, z[0], z[1]);
  box_muller(r.z, r.w, z[2], z[3]);
#pragma unroll
  for (int row = 0; row < D; ++row) {
    float v = 0.0f;
#pragma unroll
    for (int c = 0; c < D; ++c) v = fmaf(a.L[row * D + c], z[c], v);
    x[row] = v;
  }
}

__device__ __forceinline__ float4 record_of(const float* g, int d) {
  float h = g[0] * g[0];
  for (int c = 1; c < d; ++c) h = fmaf(g[c], g[c], h);
  return make_float4(g[0], g[1], d > 2 ? g[2] : 0.f, 0.5f * h);
}

// Adds a sample of cell i (point g) to the workgroup's sums; returns its
// squared distance in units of 2^-16.
template <int D>
__device__ __forceinline__ unsigned long long add_sample(unsigned long long* sum,
                                                         unsigned int* cnt, int i, const float* x,
                                                         const float* g) {
  double d2 = 0.0;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double dx = (double)x[c] - (double)g[c];
    d2 = d2 + dx * dx;
    atomicAdd(&sum[(size_t)i * D + c], (unsigned long long)fixed_of((double)x[c], 0x1p24));
  }
  atomicAdd(&cnt[i], 1u);
  return (unsigned long long)fixed_of(d2, 0x1p16);
}

// The workgroup's row of the partial table: its sums and counts, and the
// totals of its BLOCK threads' distances, admissible and inadmissible samples.
template <int BLOCK>
__device__ __forceinline__ void store_partials(const LloydArgs& a, const unsigned long long* sum,
                                               const unsigned int* cnt, unsigned long long dist,
                                               unsigned long long used, unsigned long long rej) {
  __shared__ unsigned long long part[3][BLOCK / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    dist += __shfl_xor(dist, off, 64);
    used += __shfl_xor(used, off, 64);
    rej += __shfl_xor(rej, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = dist;
    part[1][threadIdx.x >> 6] = used;
    part[2][threadIdx.x >> 6] = rej;
  }
  __syncthreads();
  unsigned long long* row = a.part + (size_t)blockIdx.x * a.E;
  const int nd = a.N * a.d;
  if (threadIdx.x < 3) {
    unsigned long long t = 0ull;
    for (int w = 0; w < BLOCK / 64; ++w) t += part[threadIdx.x][w];
    row[nd + a.N + threadIdx.x] = t;
  }
  for (int i = threadIdx.x; i < nd; i += BLOCK) row[i] = sum[i];
  for (int i = threadIdx.x; i < a.N; i += BLOCK) row[nd + i] = cnt[i];
}

}  // namespace

// Records of the start grid (d >= 2), and an empty pool of longer rows.
__global__ void lloyd_records_kernel(LloydArgs a) {
  const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
  if (i < 2 && a.bk_longs) reinterpret_cast<uint32_t*>(a.bk_longs)[i] = 0u;
  if (i >= a.Npad) return;
  a.recs[i] = i < a.N ? record_of(a.grid + (size_t)i * a.d, a.d)
                      : make_float4(0.f, 0.f, 0.f, __builtin_huge_valf());
}

// Bucket tables of the current grid.  A bucket whose candidates fit nowhere is
// counted in the pool's second word, and the step then scans: tables pay only
// where they answer nearly every sample.
__global__ __launch_bounds__(kListThreads) void lloyd_tables_kernel(LloydArgs a) {
  extern __shared__ float4 list[];  // [N]
  __shared__ ListLds lds;
  const int tiles = (a.bk_B[1] + kListTile - 1) / kListTile;
  const bool ok = list_tile(list, lds, a.recs, a.N, a.bk_lo, a.bk_scale, a.bk_B,
                            (int)(blockIdx.x / tiles) * kListTile,
                            (int)(blockIdx.x % tiles) * kListTile, a.bk_rows, a.bk_longs,
                            a.bk_pool);
  if (!ok) atomicAdd(reinterpret_cast<uint32_t*>(a.bk_longs) + 1, 1u);
}

// LDS: d = 1: midpoints [P], points [N]; d >= 2: records [Npad]; then the
// counts [N] and the sums [N][d] (8-byte aligned).
template <int D, bool SET>
__global__ __launch_bounds__(kBlock) void lloyd_accum_kernel(LloydArgs a) {
  extern __shared__ float4 lds4[];
  float* ldsf = reinterpret_cast<float*>(lds4);
  float* mids = ldsf;                      // d = 1
  float* pts1 = ldsf + a.P;                // d = 1
  float4* recs = lds4;                     // d >= 2
  const size_t grid_words = D == 1 ? (size_t)a.P + a.N : (size_t)a.Npad * 4;
  unsigned long long* sum =
      reinterpret_cast<unsigned long long*>(ldsf + ((grid_words + 1) & ~(size_t)1));
  unsigned int* cnt = reinterpret_cast<unsigned int*>(sum + (size_t)a.N * D);

  if (D == 1) {
    for (int i = threadIdx.x; i < a.P; i += kBlock) {
      float m = __builtin_huge_valf();
      if (i + 1 < a.N) {
        m = 0.5f * (a.grid[i] + a.grid[i + 1]);
        if (m == 0.0f) m = 0.0f;
      }
      mids[i] = m;
    }
    for (int i = threadIdx.x; i < a.N; i += kBlock) pts1[i] = a.grid[i];
  } else {
    for (int i = threadIdx.x; i < a.Npad; i += kBlock) recs[i] = a.recs[i];
  }
  for (int i = threadIdx.x; i < a.N * D; i += kBlock) sum[i] = 0ull;
  for (int i = threadIdx.x; i < a.N; i += kBlock) cnt[i] = 0u;
  __syncthreads();

  constexpr int S = D == 1 ? 1 : kSamplesNd;
  const uint64_t per_round = (uint64_t)gridDim.x * kBlock * S;
  unsigned long long dist = 0ull, used = 0ull, rej = 0ull;
  for (uint64_t base = (uint64_t)blockIdx.x * kBlock * S; base < a.M; base += per_round) {
    float xs[S][D];
    bool live[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const uint64_t m = base + (uint64_t)s * kBlock + threadIdx.x;
      live[s] = m < a.M;
      if (SET) {
        const bool ok = set_sample<D>(a, live[s] ? m : 0, xs[s]);
        rej += (live[s] && !ok) ? 1ull : 0ull;
        live[s] = live[s] && ok;
      } else {
        lloyd_sample<D>(a, live[s] ? m : 0, xs[s]);
      }
      used += live[s] ? 1ull : 0ull;
    }
    int idx[S];
    if (D == 1) {
      idx[0] = cell_1d(mids, a.logP, xs[0][0]);
    } else {
      argmin_scan_tiled<D, S, 4>(recs, a.Npad, xs, idx);
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (!live[s]) continue;
      const int i = idx[s];
      float g[D];
      if (D == 1) {
        g[0] = pts1[i];
      } else {
        const float4 r = recs[i];
        g[0] = r.x;
        if (D > 1) g[1] = r.y;
        if (D > 2) g[2] = r.z;
      }
      dist += add_sample<D>(sum, cnt, i, xs[s], g);
    }
  }
  store_partials<kBlock>(a, sum, cnt, dist, used, rej);
}

// The same with the step's bucket tables.  LDS: the points as pairs and the
// pad pair (or the records, where the tables do not answer), sums, counts.
// A sample's search is then its row (16 bytes from the L2, 64 KB of them at
// N = 500) and four pairs instead of N records, and what is left is latency:
// 16 waves a workgroup, 2 samples of a lane in flight (4: 3 us more a step).
// 10^6 samples, N = 500: 60 -> 12.4 us.
__global__ __launch_bounds__(kLloydWideThreads) void lloyd_accum_wide_kernel(LloydArgs a) {
  constexpr int S = kLloydWideSamples, kThreads = kLloydWideThreads;
  extern __shared__ float4 lds4[];
  float2* pairs = reinterpret_cast<float2*>(lds4);
  unsigned long long* sum = reinterpret_cast<unsigned long long*>(lds4 + a.Npad);
  unsigned int* cnt = reinterpret_cast<unsigned int*>(sum + (size_t)a.N * 2);
  const BucketTab tab{reinterpret_cast<const uint4*>(a.bk_rows),
                      reinterpret_cast<const uint4*>(a.bk_longs)};
  const bool scan = reinterpret_cast<const uint32_t*>(a.bk_longs)[1] != 0u;
  if (scan) {
    for (int i = threadIdx.x; i < a.Npad; i += kThreads) lds4[i] = a.recs[i];
  } else {
    const float nan = __builtin_nanf("");
    for (int i = threadIdx.x; i <= a.N; i += kThreads)
      pairs[i] = i < a.N ? make_float2(a.grid[2 * i], a.grid[2 * i + 1]) : make_float2(nan, nan);
  }
  for (int i = threadIdx.x; i < a.N * 2; i += kThreads) sum[i] = 0ull;
  for (int i = threadIdx.x; i < a.N; i += kThreads) cnt[i] = 0u;
  __syncthreads();
  unsigned long long dist = 0ull, used = 0ull;
  if (scan) {
    // as many samples a lane as the kernel without tables; a wave's are
    // consecutive, and the first turns go to different workgroups
    constexpr int kPerWave = 64 * kSamplesNd;
    const int lane = (int)(threadIdx.x & 63);
    for (uint64_t t = blockIdx.x + (uint64_t)gridDim.x * (threadIdx.x >> 6); t * kPerWave < a.M;
         t += (uint64_t)gridDim.x * (kThreads / 64)) {
      float xs[kSamplesNd][2];
      int idx[kSamplesNd];
#pragma unroll
      for (int s = 0; s < kSamplesNd; ++s) {
        const uint64_t m = t * kPerWave + (uint64_t)(64 * s + lane);
        lloyd_sample<2>(a, m < a.M ? m : 0, xs[s]);
      }
      argmin_scan_tiled<2, kSamplesNd, 4>(lds4, a.Npad, xs, idx);
#pragma unroll
      for (int s = 0; s < kSamplesNd; ++s) {
        if (t * kPerWave + (uint64_t)(64 * s + lane) >= a.M) continue;
        const float4 r = lds4[idx[s]];
        const float g[2] = {r.x, r.y};
        dist += add_sample<2>(sum, cnt, idx[s], xs[s], g);
        used += 1ull;
      }
    }
    store_partials<kThreads>(a, sum, cnt, dist, used, 0ull);
    return;
  }
  const uint64_t per_round = (uint64_t)gridDim.x * kThreads * S;
  for (uint64_t base = (uint64_t)blockIdx.x * kThreads * S; base < a.M; base += per_round) {
    float xs[S][2];
    bool live[S];
    int idx[S];
    uint4 w[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const uint64_t m = base + (uint64_t)s * kThreads + threadIdx.x;
      live[s] = m < a.M;
      lloyd_sample<2>(a, live[s] ? m : 0, xs[s]);
      used += live[s] ? 1ull : 0ull;
    }
    bucket_rows<S>(a, a.N, tab, xs, w);
    bucket_argmin<S>(pairs, a.N, tab, xs, w, idx);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (!live[s]) continue;
      const float2 r = pairs[idx[s]];
      const float g[2] = {r.x, r.y};
      dist += add_sample<2>(sum, cnt, idx[s], xs[s], g);
    }
  }
  store_partials<kThreads>(a, sum, cnt, dist, used, 0ull);
}

// Workgroup b sums the columns of cells [4 b, 4 b + 4) over the `rows` rows of
// the partial table (thread t: column t mod 16, rows t / 16 + 16 i, so that
// the loads of a row are one or two segments and a thread's loads are all in
// flight) and gives these cells their new points: the mean, or the old point
// moved the fraction gamma towards it, or the old point of an empty cell.  The
// last workgroup sums the three totals.  Sum, update and the next grid's
// records were three launches of 9, 4.5 and 4.7 us a step (N = 500);
// this one takes 4.3, and the whole step went from 68 to 25 us.
constexpr int kCells = 4;
template <int D>
__global__ __launch_bounds__(kBlock) void lloyd_update_kernel(LloydArgs a, int rows) {
  constexpr int kCols = 16;
  static_assert(kCells * (D + 1) <= kCols, "a row's columns fit the threads");
  __shared__ unsigned long long red[kBlock / 64][kCols];
  const int col = (int)threadIdx.x % kCols, grp = (int)threadIdx.x / kCols;
  const int nd = a.N * D, c0 = (int)blockIdx.x * kCells;
  const bool totals = blockIdx.x == gridDim.x - 1;
  int column = -1;
  if (totals) column = col < 3 ? nd + a.N + col : -1;
  else if (col < kCells * D) column = c0 * D + col < nd ? c0 * D + col : -1;
  else if (col < kCells * (D + 1) && c0 + col - kCells * D < a.N)
    column = nd + c0 + col - kCells * D;
  unsigned long long acc = 0ull;
  if (column >= 0) {
#pragma unroll 8
    for (int r = grp; r < rows; r += kBlock / kCols) acc += a.part[(size_t)r * a.E + column];
  }
  acc += __shfl_xor(acc, 16, 64);
  acc += __shfl_xor(acc, 32, 64);
  if ((threadIdx.x & 63) < kCols) red[threadIdx.x >> 6][col] = acc;
  __syncthreads();
  auto total = [&](int c) {
    unsigned long long t = 0ull;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) t += red[w][c];
    return t;
  };
  if (totals) {
    if (threadIdx.x == 0) {
      const unsigned long long dist = total(0), used = total(1);
      if (a.distortion)
        a.distortion[a.it] =
            used > 0ull ? ((double)(long long)dist * 0x1p-16) / (double)(long long)used : 0.0;
      if (a.xs) {
        const unsigned long long rej = (a.it > 0 ? *a.rej_total : 0ull) + total(2);
        *a.rej_total = rej;
        if (a.rejected) *a.rejected = (long long)rej;
      }
      if (a.bk_longs) {  // the next tables start with an empty pool
        reinterpret_cast<uint32_t*>(a.bk_longs)[0] = 0u;
        reinterpret_cast<uint32_t*>(a.bk_longs)[1] = 0u;
      }
    }
    return;
  }
  const int i = c0 + (int)threadIdx.x;
  if (threadIdx.x >= kCells || i >= a.N) return;
  const unsigned int n = (unsigned int)total(kCells * D + (int)threadIdx.x);
  float g[kMaxDim] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < D; ++c) {
    g[c] = a.grid[(size_t)i * D + c];
    if (n == 0u) continue;
    const double mean =
        ((double)(long long)total((int)threadIdx.x * D + c) * 0x1p-24) / (double)n;
    g[c] = a.gamma == 1.0 ? (float)mean : (float)((double)g[c] + a.gamma * (mean - (double)g[c]));
    a.grid[(size_t)i * D + c] = g[c];
  }
  if (D > 1) a.recs[i] = record_of(g, D);
}

size_t lloyd_lds_bytes(int d, int N, int Npad, int P) {
  const size_t grid_words = d == 1 ? (size_t)P + N : (size_t)Npad * 4;
  return sizeof(float) * ((grid_words + 1) & ~(size_t)1) + sizeof(unsigned long long) * N * d +
         sizeof(unsigned int) * N;
}

hipError_t launch_lloyd_records(const LloydArgs& a, hipStream_t s) {
  if (a.d == 1) return hipSuccess;
  hipLaunchKernelGGL(lloyd_records_kernel, dim3((a.Npad + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                     a);
  return hipGetLastError();
}

template <class KERNEL>
static hipError_t launch_accum(KERNEL* k, const LloydArgs& a, int blocks, int threads, size_t lds,
                               hipStream_t s) {
  hipError_t e = hipSuccess;
  if (lds > 65536)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess) hipLaunchKernelGGL(k, dim3(blocks), dim3(threads), lds, s, a);
  return e;
}

hipError_t launch_lloyd_step(const LloydArgs& a, int blocks, hipStream_t s) {
  const bool wide = a.bk_B[0] > 0;
  if (blocks < 1 || blocks > (wide ? kLloydMaxWide : kLloydMaxBlocks)) return hipErrorInvalidValue;
  const size_t lds = lloyd_lds_bytes(a.d, a.N, a.Npad, a.P);
  const bool set = a.xs != nullptr;
  hipError_t e;
  if (wide) {
    const int tiles = (a.bk_B[0] + kListTile - 1) / kListTile;
    hipLaunchKernelGGL(lloyd_tables_kernel, dim3(tiles * tiles), dim3(kListThreads),
                       sizeof(float4) * a.N, s, a);
    e = launch_accum(lloyd_accum_wide_kernel, a, blocks, kLloydWideThreads, lds, s);
  } else if (a.d == 1) {
    e = launch_accum(set ? lloyd_accum_kernel<1, true> : lloyd_accum_kernel<1, false>, a, blocks,
                     kBlock, lds, s);
  } else if (a.d == 2) {
    e = launch_accum(set ? lloyd_accum_kernel<2, true> : lloyd_accum_kernel<2, false>, a, blocks,
                     kBlock, lds, s);
  } else {
    e = launch_accum(set ? lloyd_accum_kernel<3, true> : lloyd_accum_kernel<3, false>, a, blocks,
                     kBlock, lds, s);
  }
  if (e != hipSuccess) return e;
  const dim3 groups((a.N + kCells - 1) / kCells + 1);
  if (a.d == 1) hipLaunchKernelGGL(lloyd_update_kernel<1>, groups, dim3(kBlock), 0, s, a, blocks);
  else if (a.d == 2)
    hipLaunchKernelGGL(lloyd_update_kernel<2>, groups, dim3(kBlock), 0, s, a, blocks);
  else hipLaunchKernelGGL(lloyd_update_kernel<3>, groups, dim3(kBlock), 0, s, a, blocks);
  return hipGetLastError();
}

// ------------------------------------------------- moment-matching grids

// Exact integer sums over the admissible samples: the count, rint(x_r 2^24)
// and rint(x_r x_c 2^16) (the product exact in FP64); per-lane sums over a
// grid-stride loop, wave sums, one 64-bit device atomic per wave and value
// (integer addition, so the totals do not depend on the order).
template <int D>
__global__ __launch_bounds__(kBlock) void moments_kernel(const float* __restrict__ x, uint64_t M,
                                                         unsigned long long* sums) {
  unsigned long long acc[1 + D + D * D] = {};
  for (uint64_t m = (uint64_t)blockIdx.x * kBlock + threadIdx.x; m < M;
       m += (uint64_t)gridDim.x * kBlock) {
    float v[D];
    bool ok = true;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      v[c] = x[m * D + c];
      ok = ok && fabsf(v[c]) <= 64.0f;
    }
    if (!ok) continue;
    acc[0] += 1ull;
#pragma unroll
    for (int r = 0; r < D; ++r) {
      acc[1 + r] += (unsigned long long)fixed_of((double)v[r], 0x1p24);
#pragma unroll
      for (int c = 0; c < D; ++c)
        acc[1 + D + r * D + c] +=
            (unsigned long long)fixed_of((double)v[r] * (double)v[c], 0x1p16);
    }
  }
#pragma unroll
  for (int q = 0; q < 1 + D + D * D; ++q) {
    unsigned long long t = acc[q];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if ((threadIdx.x & 63) == 0 && t != 0ull) atomicAdd(&sums[q], t);
  }
}

__global__ void zero_u64_kernel(unsigned long long* p, int n) {
  const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
  if (i < n) p[i] = 0ull;
}

// One workgroup: thread 0 forms the mean, covariance and Cholesky factor in
// FP64 (the lower factor column by column; a non-positive pivot gives a zero
// column), then every thread maps grid points base[i] to
// mean + chol base[i] (FP64, left to right, rounded once).
__global__ __launch_bounds__(kBlock) void moment_grid_kernel(int d, const long long* sums,
                                                             const float* base, int N, float* grid,
                                                             double* moments) {
  __shared__ double mean[kMaxDim], chol[kMaxDim * kMaxDim];
  if (threadIdx.x == 0) {
    double cov[kMaxDim * kMaxDim] = {}, L[kMaxDim * kMaxDim] = {}, mu[kMaxDim] = {};
    const long long count = sums[0];
    if (count > 0) {
      for (int r = 0; r < d; ++r) mu[r] = ((double)sums[1 + r] * 0x1p-24) / (double)count;
      for (int r = 0; r < d; ++r)
        for (int c = 0; c < d; ++c)
          cov[r * d + c] =
              ((double)sums[1 + d + r * d + c] * 0x1p-16) / (double)count - mu[r] * mu[c];
    }
    for (int r = 0; r < d; ++r) {
      for (int c = 0; c <= r; ++c) {
        double v = cov[r * d + c];
        for (int q = 0; q < c; ++q) v = v - L[r * d + q] * L[c * d + q];
        if (r == c) L[r * d + c] = v > 0.0 ? sqrt(v) : 0.0;
        else L[r * d + c] = L[c * d + c] > 0.0 ? v / L[c * d + c] : 0.0;
      }
    }
    for (int r = 0; r < d; ++r) mean[r] = mu[r];
    for (int q = 0; q < d * d; ++q) chol[q] = L[q];
    if (moments) {
      for (int r = 0; r < d; ++r) moments[r] = mu[r];
      for (int q = 0; q < d * d; ++q) {
        moments[d + q] = cov[q];
        moments[d + d * d + q] = L[q];
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += kBlock) {
    for (int r = 0; r < d; ++r) {
      double v = mean[r];
      for (int c = 0; c <= r; ++c) v = v + chol[r * d + c] * (double)base[(size_t)i * d + c];
      grid[(size_t)i * d + r] = (float)v;
    }
  }
}

hipError_t launch_sample_moments(int d, const float* x, uint64_t M, long long* sums,
                                 hipStream_t s) {
  const int words = 1 + d + d * d;
  auto* u = reinterpret_cast<unsigned long long*>(sums);
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(kBlock), 0, s, u, words);
  if (M > 0) {
    const uint64_t want = (M + kBlock - 1) / kBlock;
    const unsigned blocks = (unsigned)(want < 2048 ? want : 2048);
    if (d == 1) hipLaunchKernelGGL(moments_kernel<1>, dim3(blocks), dim3(kBlock), 0, s, x, M, u);
    else if (d == 2) hipLaunchKernelGGL(moments_kernel<2>, dim3(blocks), dim3(kBlock), 0, s, x, M, u);
    else hipLaunchKernelGGL(moments_kernel<3>, dim3(blocks), dim3(kBlock), 0, s, x, M, u);
  }
  return hipGetLastError();
}

hipError_t launch_moment_grid(int d, const long long* sums, const float* base, int N,
                              float* grid, double* moments, hipStream_t s) {
  hipLaunchKernelGGL(moment_grid_kernel, dim3(1), dim3(kBlock), 0, s, d, sums, base, N, grid,
                     moments);
  return hipGetLastError();
}

}  // namespace qtree
