// Backward dynamic programming on the quantization tree (Sec. 2), FP64:
//   V_n = phi_n,  V_k(i) = max(phi_k(i), sum_j c_ij V_{k+1}(j) / p_i),
// with pi^k_ij = c_ij / p_i estimated by the forward counts.  The
// conditional expectation on the tree is the row reduction
// sum_j pi_ij f(x_j) of Sec. 2: a product of the count block with the value
// vectors of up to kPay payoffs, on the FP64 matrix cores.  Also the
// obstacle phi_k on the grid points.
#include "bdp_tile.hpp"
#include "qtree_batch.hpp"
#include "qtree_internal.hpp"

namespace qtree {

namespace {
constexpr int kBlock = 256;
constexpr int kPay = 16;     // payoffs per pass: the columns of a matrix-core tile
constexpr int kRows = 16;    // rows per workgroup: the rows of a tile
constexpr int kLayerWaves = 8;
constexpr int kFewPay = 2;   // payoffs a pass of the few-payoff path takes
constexpr int kFewRows = 4;  // ... and rows per workgroup
constexpr int kFewWaves = 4;

// The rows of a tile: this lane's row (lane % 16), a pointer indexed by
// column, and the columns [lo, hi) it holds; [from, to) covers every row.
struct TileRows {
  const int32_t* row;
  int lo, hi, from, to;
};

// One tile of kRows rows by one workgroup of W waves: wave w takes the
// chunks of 16 columns w, w + W, ..., AHEAD of them in flight, and the waves'
// products and row totals meet in LDS.  Thread t < 256 returns S of row
// t / 16 and payoff t % 16, and the row's total.  x: the values of this
// lane's payoff (lane % 16) by column, n1 of them (a lane without a payoff
// repeats another's: its sums are dropped).  DENSE: the rows hold all n1 >= 4
// columns.
//
// What bounds a layer is the latency of one launch: counts and values are
// one round trip, and nothing is reduced across lanes.  N = 500, 12
// payoffs: 4.7 us a layer, against 14.0 when a wave walked one row and
// reduced its 16 sums over the lanes with about 200 shuffles; N = 256: 3.8
// against 12.1; N = 2000: 13.0 against 39.8.
template <int W, int AHEAD, bool DENSE>
__device__ __forceinline__ bool tile_sums(const TileRows& R, const double* __restrict__ x, int n1,
                                          double& sum, int64_t& total) {
  __shared__ double part[W][kRows][kPay];
  __shared__ int64_t part_p[W][kRows];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = lane >> 4;
  const bool wide = !DENSE && n1 >= 4 && __all(R.hi - R.lo >= 4);
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  int64_t p = 0;
  for (int j0 = R.from + 16 * wave; j0 < R.to; j0 += 16 * W * AHEAD) {
    int32_t c[AHEAD][4];
    double v[AHEAD][4];
    const int j = j0 + 4 * g;
    if (DENSE) {
      load_cols(R.row, n1, j, 16 * W, c);
      load_cols(x, n1, j, 16 * W, v);
      if (j0 + 16 * W * (AHEAD - 1) + 16 > n1) {
        drop_tails(n1, j, 16 * W, c);
        drop_tails(n1, j, 16 * W, v);
      }
    } else {
      if (wide) {
        load_cols(x, n1, j, 16 * W, v);
      } else {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
#pragma unroll
          for (int u = 0; u < 4; ++u) v[a][u] = x[min(j + 16 * W * a + u, n1 - 1)];
      }
      load_band(R.row, R.lo, R.hi, j, 16 * W, wide, c);
      if (wide && j0 + 16 * W * (AHEAD - 1) + 16 > n1) drop_tails(n1, j, 16 * W, v);
    }
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) {
      p += (int64_t)c[a][0] + c[a][1] + c[a][2] + c[a][3];
      chunk_product(c[a], v[a], lane, acc);
    }
  }
  p += __shfl_xor(p, 16, 64);
  p += __shfl_xor(p, 32, 64);
#pragma unroll
  for (int r = 0; r < 4; ++r) part[wave][g + 4 * r][lane & 15] = acc[r];
  if (lane < kRows) part_p[wave][lane] = p;
  __syncthreads();
  const int t = (int)threadIdx.x;
  if (t >= kRows * kPay) return false;
  sum = 0.0;
  total = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    sum += part[w][t >> 4][t & 15];
    total += part_p[w][t >> 4];
  }
  return true;
}

// Sum over the 64 lanes of v[0 .. M): lane exchanges halve the values while
// they halve the lanes, so that lane l ends with the sum of value
// sum_slot<M>(l) (repeated over the lanes of a slot).
template <int M>
__device__ __forceinline__ double lane_sums(const double (&v)[M], int lane, int off) {
  if constexpr (M == 1) {
    double s = v[0];
    for (; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    return s;
  } else {
    constexpr int H = M / 2;
    double w[H];
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double keep = up ? v[H + i] : v[i], give = up ? v[i] : v[H + i];
      w[i] = keep + __shfl_xor(give, off, 64);
    }
    return lane_sums<H>(w, lane, off >> 1);
  }
}

// kFewRows rows by one workgroup for Q <= kFewPay payoffs on vector FMAs: a
// wave takes blocks of 256 columns (four consecutive ones per lane, the
// values loaded once for all rows), the lanes' sums and the waves' meet by
// exchange and LDS.  Thread t < kFewRows Q returns S of row t / Q and payoff
// t % Q, and the row's total (exact in FP64: below 2^53).  A tile on the
// matrix cores would spend 14 of its 16 columns on nothing and leave half of
// the chip without a row tile (N = 2000, 2 payoffs: 11.4 us a layer).  Here
// 6.5 us, against 12.7 with one wave per row; N = 990: 4.1 against 6.9; N =
// 500, 1 payoff: 3.1 against 6.4; N = 100: 3.6 against 6.5, launch included.
template <int Q>
__device__ __forceinline__ bool few_sums(const int32_t* __restrict__ rows, int nrows,
                                         const double* __restrict__ x, int64_t P, int n1,
                                         double& sum, double& total) {
  constexpr int kVals = kFewRows * (Q == 1 ? 2 : 4);  // per row: Q sums, the total (and a pad)
  __shared__ double part[kFewWaves][kVals];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  double s[kVals];
#pragma unroll
  for (int i = 0; i < kVals; ++i) s[i] = 0.0;
  constexpr int kPer = kVals / kFewRows;
  for (int j0 = 256 * wave; j0 < n1; j0 += 256 * kFewWaves) {
    const int j = j0 + 4 * lane;
    int32_t c[kFewRows][4];
    double v[Q][4];
    const Cols4 t(j, n1);
#pragma unroll
    for (int r = 0; r < kFewRows; ++r) {
      const int i = r < nrows ? r : nrows - 1;  // rows past the end repeat the last one
      const Int4U y = *reinterpret_cast<const Int4U*>(rows + (int64_t)i * n1 + t.at);
#pragma unroll
      for (int u = 0; u < 4; ++u) c[r][u] = y.v[u];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const Dbl4U y = *reinterpret_cast<const Dbl4U*>(x + q * P + t.at);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[q][u] = y.v[u];
    }
    if (j0 + 256 > n1) {
#pragma unroll
      for (int r = 0; r < kFewRows; ++r) drop_front(c[r], t.drop);
#pragma unroll
      for (int q = 0; q < Q; ++q) drop_front(v[q], t.drop);
    }
    bool finite = true;
#pragma unroll
    for (int q = 0; q < Q; ++q) finite = finite && finite4(v[q]);
    if (__all(finite)) {
#pragma unroll
      for (int r = 0; r < kFewRows; ++r)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double cd = (double)c[r][u];
          s[r * kPer + Q] += cd;
#pragma unroll
          for (int q = 0; q < Q; ++q) s[r * kPer + q] = fma(cd, v[q][u], s[r * kPer + q]);
        }
    } else {  // a zero count adds nothing, whatever its value is
#pragma unroll
      for (int r = 0; r < kFewRows; ++r)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double cd = (double)c[r][u];
          s[r * kPer + Q] += cd;
#pragma unroll
          for (int q = 0; q < Q; ++q)
            if (c[r][u] != 0) s[r * kPer + q] = fma(cd, v[q][u], s[r * kPer + q]);
        }
    }
  }
  const double mine = lane_sums<kVals>(s, lane, 32);
  // the halving gives value i to the lanes whose top bits spell i
  constexpr int kLanes = 64 / kVals;
  if (lane % kLanes == 0) part[wave][lane / kLanes] = mine;
  __syncthreads();
  const int t = (int)threadIdx.x;
  if (t >= kFewRows * Q) return false;
  sum = total = 0.0;
#pragma unroll
  for (int w = 0; w < kFewWaves; ++w) {
    sum += part[w][(t / Q) * kPer + t % Q];
    total += part[w][(t / Q) * kPer + Q];
  }
  return true;
}
}  // namespace

// One layer for every payoff: workgroup (x, y) takes rows 16 x .. + 15 and
// payoffs 16 y .. + 15 (the count rows are re-read per group of payoffs, from
// L2 for all but the first).
template <int AHEAD, bool DENSE>
__global__ __launch_bounds__(64 * kLayerWaves) void bdp_layer_kernel(
    BdpArgs a, int N_k, int N_k1, int64_t pt_k, int64_t pt_k1, int64_t cnt_k) {
  const int lane = threadIdx.x & 63;
  const int q0 = blockIdx.y * kPay;
  const int nq = (a.n_pay - q0) < kPay ? (a.n_pay - q0) : kPay;
  const int i0 = blockIdx.x * kRows;
  // rows past the end repeat the last one (their results are dropped)
  const int i = i0 + (lane & 15) < N_k ? i0 + (lane & 15) : N_k - 1;
  TileRows R;
  if (!DENSE && a.band_off) {
    // the band of columns band_lo .. of every row; the tile covers them all
    const int64_t r = pt_k + i;
    const int64_t o = a.band_off[r];
    R.lo = a.band_lo[r];
    R.hi = R.lo + (int)(a.band_off[r + 1] - o);
    R.row = a.counts + o - R.lo;
    R.from = R.lo;
    R.to = R.hi;
#pragma unroll
    for (int m = 8; m > 0; m >>= 1) {
      R.from = min(R.from, __shfl_xor(R.from, m, 64));
      R.to = max(R.to, __shfl_xor(R.to, m, 64));
    }
    R.from = __builtin_amdgcn_readfirstlane(R.from);
    R.to = __builtin_amdgcn_readfirstlane(R.to);
  } else {
    R.row = a.counts + cnt_k + (int64_t)i * N_k1;
    R.lo = R.from = 0;
    R.hi = R.to = N_k1;
  }
  const int q = lane & 15;
  double s;
  int64_t p;
  if (!tile_sums<kLayerWaves, AHEAD, DENSE>(R, a.V + (int64_t)(q0 + (q < nq ? q : 0)) * a.P + pt_k1, N_k1,
                                  s, p))
    return;
  const int row = i0 + (int)(threadIdx.x >> 4), col = (int)(threadIdx.x & 15);
  if (row < N_k && col < nq) {
    const double cont = p > 0 ? s / (double)p : 0.0;
    const int64_t at = (int64_t)(q0 + col) * a.P + pt_k + row;
    const double f = a.phi[at];
    a.V[at] = f > cont ? f : cont;
  }
}

// The same for Q <= kFewPay payoffs and rows of at least four columns, dense.
template <int Q>
__global__ __launch_bounds__(64 * kFewWaves) void bdp_few_kernel(BdpArgs a, int N_k, int N_k1,
                                                                 int64_t pt_k, int64_t pt_k1,
                                                                 int64_t cnt_k) {
  const int i0 = blockIdx.x * kFewRows;
  double s, p;
  if (!few_sums<Q>(a.counts + cnt_k + (int64_t)i0 * N_k1, min(kFewRows, N_k - i0), a.V + pt_k1,
                   a.P, N_k1, s, p))
    return;
  const int row = i0 + (int)threadIdx.x / Q;
  if (row < N_k) {
    const double cont = p > 0.0 ? s / p : 0.0;
    const int64_t at = (int64_t)((int)threadIdx.x % Q) * a.P + pt_k + row;
    const double f = a.phi[at];
    a.V[at] = f > cont ? f : cont;
  }
}

// The same for banded rows: a wave per row, its columns four at a time a lane.
// 1 / 2 payoffs, a layer of the recursion: N = 250 3.6 / 3.8 us, 2000 8.1 / 9.0,
// against 4.9 and 15.3 by tiles, whose lanes load 16 rows of different bands
// (and 7.0 and 12.6 by a wave per row and one column a lane).
template <int Q>
__global__ __launch_bounds__(64 * kFewWaves) void bdp_few_band_kernel(BdpArgs a, int N_k, int64_t pt_k,
                                                                      int64_t pt_k1) {
  const int lane = threadIdx.x & 63;
  const int i = (int)(blockIdx.x * kFewWaves + (threadIdx.x >> 6));
  if (i >= N_k) return;
  const int64_t r = pt_k + i, o = a.band_off[r];
  const int len = (int)(a.band_off[r + 1] - o);
  const int32_t* row = a.counts + o;
  const double* x = a.V + pt_k1 + a.band_lo[r];
  double s[Q + 1];
#pragma unroll
  for (int q = 0; q <= Q; ++q) s[q] = 0.0;
  for (int j0 = 4 * lane; j0 < len; j0 += 256) {
    int32_t c[4];
    double v[Q][4];
    if (len >= 4) {
      const Cols4 t(j0, len);
      const Int4U y = *reinterpret_cast<const Int4U*>(row + t.at);
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = y.v[e];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const Dbl4U z = *reinterpret_cast<const Dbl4U*>(x + q * a.P + t.at);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[q][e] = z.v[e];
      }
      if (__any(t.drop != 0)) {
        drop_front(c, t.drop);
#pragma unroll
        for (int q = 0; q < Q; ++q) drop_front(v[q], t.drop);
      }
    } else {  // lane 0 alone
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        c[e] = e < len ? row[e] : 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q][e] = e < len ? x[q * a.P + e] : 0.0;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double cd = (double)c[e];
      s[Q] += cd;
#pragma unroll
      for (int q = 0; q < Q; ++q)  // a zero count adds nothing, whatever its value is
        s[q] = c[e] != 0 ? fma(cd, v[q][e], s[q]) : s[q];
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q <= Q; ++q) s[q] += __shfl_xor(s[q], off, 64);
  if (lane >= Q) return;
  const double sq = Q == 1 || lane == 0 ? s[0] : s[Q - 1];
  const double cont = s[Q] > 0.0 ? sq / s[Q] : 0.0;
  const int64_t at = (int64_t)lane * a.P + pt_k + i;
  const double f = a.phi[at];
  a.V[at] = f > cont ? f : cont;
}

__global__ void copy_last_layer_kernel(BdpArgs a, int64_t pt_n, int N_n) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)a.n_pay * N_n;
  if (t >= total) return;
  const int64_t q = t / N_n, i = t - q * N_n;
  const int64_t at = q * a.P + pt_n + i;
  a.V[at] = a.phi[at];
}

hipError_t launch_bdp_layer(const BdpArgs& a, int k, int N_k, int N_k1, int64_t pt_k,
                            int64_t pt_k1, int64_t cnt_k, hipStream_t s) {
  (void)k;
  if (a.band_off && a.n_pay <= kFewPay) {
    const dim3 grid((unsigned)((N_k + kFewWaves - 1) / kFewWaves)), block(64 * kFewWaves);
    if (a.n_pay == 1)
      hipLaunchKernelGGL(bdp_few_band_kernel<1>, grid, block, 0, s, a, N_k, pt_k, pt_k1);
    else
      hipLaunchKernelGGL(bdp_few_band_kernel<2>, grid, block, 0, s, a, N_k, pt_k, pt_k1);
    return hipGetLastError();
  }
  const bool dense = !a.band_off && N_k1 >= 4;
  if (dense && a.n_pay <= kFewPay) {
    const dim3 grid((unsigned)((N_k + kFewRows - 1) / kFewRows)), block(64 * kFewWaves);
    if (a.n_pay == 1)
      hipLaunchKernelGGL(bdp_few_kernel<1>, grid, block, 0, s, a, N_k, N_k1, pt_k, pt_k1, cnt_k);
    else
      hipLaunchKernelGGL(bdp_few_kernel<2>, grid, block, 0, s, a, N_k, N_k1, pt_k, pt_k1, cnt_k);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((N_k + kRows - 1) / kRows), (unsigned)((a.n_pay + kPay - 1) / kPay));
  // kLayerWaves waves cover 128 columns at a time, one chunk each; two in
  // flight per wave where a row is longer than two such turns.  More chunks
  // or waves bring a row in sooner, but their registers and slots are what a
  // sampling pass on another stream leaves free: four chunks (68 registers more)
  // take 4.2 / 5.2 / 7.2 / 13.9 us at N = 256 / 500 / 1000 / 2000 against 3.8 /
  // 4.7 / 6.8 / 13.0, and a 50-layer forward beside it 1.84 against 1.74 ms.
  const dim3 block(64 * kLayerWaves);
  if (!dense)
    hipLaunchKernelGGL((bdp_layer_kernel<2, false>), grid, block, 0, s, a, N_k, N_k1, pt_k, pt_k1,
                       cnt_k);
  else if (N_k1 <= 2 * 16 * kLayerWaves)
    hipLaunchKernelGGL((bdp_layer_kernel<1, true>), grid, block, 0, s, a, N_k, N_k1, pt_k, pt_k1,
                       cnt_k);
  else
    hipLaunchKernelGGL((bdp_layer_kernel<2, true>), grid, block, 0, s, a, N_k, N_k1, pt_k, pt_k1,
                       cnt_k);
  return hipGetLastError();
}

// Results of layer 0 to `out` in pinned host memory: V[q stride], or of the jobs
// of a batch.
__global__ void v0_kernel(const double* V, int64_t stride, int n, double* out) {
  for (int q = threadIdx.x; q < n; q += blockDim.x) out[q] = V[(int64_t)q * stride];
}
__global__ void v0_jobs_kernel(const BdpJob* jobs, double* out) {
  const BdpJob& J = jobs[blockIdx.x];
  if ((int)threadIdx.x < J.nq)
    out[J.v0_at + (int)threadIdx.x] = as_global(J.V)[(int64_t)(J.q0 + (int)threadIdx.x) * J.P];
}

hipError_t launch_v0(const double* V, int64_t stride, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(v0_kernel, dim3(1), dim3(kBlock), 0, s, V, stride, n, out);
  return hipGetLastError();
}

hipError_t launch_v0_jobs(const BdpJob* jobs, int n_jobs, double* out, hipStream_t s) {
  hipLaunchKernelGGL(v0_jobs_kernel, dim3(n_jobs), dim3(64), 0, s, jobs, out);
  return hipGetLastError();
}

hipError_t launch_copy_last_layer(const BdpArgs& a, int64_t pt_n, int N_n, hipStream_t s) {
  const int64_t total = (int64_t)a.n_pay * N_n;
  const unsigned blocks = (unsigned)((total + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(copy_last_layer_kernel, dim3(blocks), dim3(kBlock), 0, s, a, pt_n, N_n);
  return hipGetLastError();
}

// Batched BDP.  The recursion is sequential in k, so it runs as backward
// steps: step j takes layer n - 1 - j of every contract with n > j, its rows
// cut into tasks of kBdpTaskRows rows; a launch boundary separates the steps.
// Every contract's work is spread over the whole chip at every step.  A task
// is one tile for the job's up to kPay payoffs; a batch whose jobs all have
// at most kFewPay payoffs and no layer below four points cuts a task into
// workgroups of kFewRows rows instead.
static_assert(kBdpTaskRows == kRows, "a task is one tile");
static_assert(kBdpTaskRows % kFewRows == 0, "a task is whole few-payoff workgroups");

__global__ void bdp_batch_copy_kernel(const BdpJob* jobs) {
  const BdpJob& J = jobs[blockIdx.y];
  const LayerDev& Ln = as_global(J.layers)[J.n];
  const double* phi = as_global(J.phi);
  double* V = as_global(J.V);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < J.nq * Ln.N; t += gridDim.x * blockDim.x) {
    const int q = t / Ln.N, i = t - q * Ln.N;
    const int64_t at = (int64_t)(J.q0 + q) * J.P + Ln.pt_off + i;
    V[at] = phi[at];
  }
}

template <bool DENSE>
__global__ __launch_bounds__(64 * kLayerWaves) void bdp_step_kernel(const BdpTask* tasks) {
  const BdpTask& T = tasks[blockIdx.x];
  const int lane = threadIdx.x & 63;
  const int n1 = T.n1, nrows = T.nrows, nq = T.nq;
  const int64_t P = T.P;
  const int r = lane & 15;  // rows past the end repeat the last one
  TileRows R;
  R.row = as_global(T.counts) + (int64_t)(r < nrows ? r : nrows - 1) * n1;
  R.lo = R.from = 0;
  R.hi = R.to = n1;
  const double* x = as_global(T.next) + (int64_t)(r < nq ? r : 0) * P;
  double s;
  int64_t p;
  if (!tile_sums<kLayerWaves, 2, DENSE>(R, x, n1, s, p)) return;
  const int row = (int)(threadIdx.x >> 4), col = (int)(threadIdx.x & 15);
  if (row < nrows && col < nq) {
    const double cont = p > 0 ? s / (double)p : 0.0;
    const int64_t at = (int64_t)col * P + row;
    const double f = as_global(T.phi)[at];
    as_global(T.V)[at] = f > cont ? f : cont;
  }
}

__global__ __launch_bounds__(64 * kFewWaves) void bdp_step_few_kernel(const BdpTask* tasks) {
  constexpr int kParts = kBdpTaskRows / kFewRows;
  const BdpTask& T = tasks[blockIdx.x / kParts];
  const int r0 = (int)(blockIdx.x % kParts) * kFewRows;
  const int n1 = T.n1, nrows = T.nrows, nq = T.nq;
  const int64_t P = T.P;
  if (r0 >= nrows) return;
  // a one-payoff job repeats its payoff as the second one
  double s, p;
  if (!few_sums<kFewPay>(as_global(T.counts) + (int64_t)r0 * n1, min(kFewRows, nrows - r0),
                         as_global(T.next), nq > 1 ? P : 0, n1, s, p))
    return;
  const int row = r0 + (int)threadIdx.x / kFewPay, q = (int)threadIdx.x % kFewPay;
  if (row < nrows && q < nq) {
    const double cont = p > 0.0 ? s / p : 0.0;
    const int64_t at = (int64_t)q * P + row;
    const double f = as_global(T.phi)[at];
    as_global(T.V)[at] = f > cont ? f : cont;
  }
}

hipError_t launch_bdp_steps(const BdpJob* jobs, int n_jobs, int max_last, int max_nq, int min_n1,
                            const BdpTask* tasks, const int* step_off, int n_steps,
                            hipStream_t s) {
  if (n_jobs <= 0) return hipSuccess;
  const unsigned cx = (unsigned)((max_last + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(bdp_batch_copy_kernel, dim3(cx < 1 ? 1 : cx, (unsigned)n_jobs), dim3(kBlock),
                     0, s, jobs);
  const bool few = max_nq <= kFewPay && min_n1 >= 4;
  for (int j = 0; j < n_steps; ++j) {
    const int cnt = step_off[j + 1] - step_off[j];
    if (cnt <= 0) continue;
    if (few)
      hipLaunchKernelGGL(bdp_step_few_kernel, dim3((unsigned)(cnt * (kBdpTaskRows / kFewRows))),
                         dim3(64 * kFewWaves), 0, s,
                         tasks + step_off[j]);
    else if (min_n1 >= 4)
      hipLaunchKernelGGL(bdp_step_kernel<true>, dim3((unsigned)cnt), dim3(64 * kLayerWaves), 0, s,
                         tasks + step_off[j]);
    else
      hipLaunchKernelGGL(bdp_step_kernel<false>, dim3((unsigned)cnt), dim3(64 * kLayerWaves), 0, s,
                         tasks + step_off[j]);
  }
  return hipGetLastError();
}

// Discounted obstacle phi_k(x) = exp(-r t_k) payoff(S_{t_k}(x)) on every grid
// point, S^a_t(x) = S0 exp((r - sigma_a^2 / 2) t + sigma_a x_a), FP64, for a
// group of contracts (blockIdx.z).
__global__ void payoff_kernel(PayoffArgs a) {
  const int k = blockIdx.y;
  const Contract& C = a.c[blockIdx.z];
  const LayerDev& L = a.layers[k];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= L.N) return;
  const double t = C.Tm * (double)k / (double)a.n;
  const double disc = exp(-C.r * t);
  const int64_t at = (int64_t)L.pt_off + i;
  const float4 g = a.d == 1 ? make_float4(a.pts1[at], 0.f, 0.f, 0.f) : a.pts[at];
  const float xs[3] = {g.x, g.y, g.z};
  double y[3];
  for (int c = 0; c < a.d; ++c) {
    if (!C.has_mix) {
      y[c] = (double)xs[c];
      continue;
    }
    y[c] = 0.0;
    for (int e = 0; e < a.d; ++e) y[c] += C.mix[c * a.d + e] * (double)xs[e];
  }
  double v;
  if (C.kind & 1) {
    double smax = -__builtin_huge_val();
    for (int c = 0; c < a.d; ++c) {
      const double sc = C.S0 * exp((C.r - 0.5 * C.sigma[c] * C.sigma[c]) * t + C.sigma[c] * y[c]);
      smax = sc > smax ? sc : smax;
    }
    v = disc * fmax(smax - C.K, 0.0);
  } else {
    const double sc =
        C.S0 * exp((C.r - 0.5 * C.sigma[0] * C.sigma[0]) * t + C.sigma[0] * y[0]);
    v = disc * fmax(C.K - sc, 0.0);
  }
  if ((C.kind & 2) && k < a.n) v = -__builtin_huge_val();
  a.phi[(int64_t)blockIdx.z * a.P + at] = v;
}

hipError_t launch_payoff(const PayoffArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.maxN + kBlock - 1) / kBlock), (unsigned)(a.n + 1),
                  (unsigned)a.count);
  hipLaunchKernelGGL(payoff_kernel, grid, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}


// ------------------------------------------------- many contracts, one tree
//
// The conditional expectation of the quantized BDP (Sec. 2) is a product of
// the transition matrix pi^k (N_k x N_{k+1}) with the values V_{k+1} of every
// contract priced on the tree; its cost is sum_k N_k N_{k+1} multiply-adds
// per contract.  pi_kernel turns the counts into pi^k_ij = c_ij / p_i once
// (FP64, rows padded with zeros to a multiple of 4 columns) and records the
// range of the nonzero columns of every row; bdp_many_kernel then runs the
// whole backward recursion of 64 contracts per workgroup with their V_{k+1}
// resident in LDS ([point][contract]), the products on the FP64 matrix cores
// and the obstacle phi_k computed where it is used.  One launch may cover
// many trees (a table of trees, one per number of layers for instance):
// workgroup b then prices 64 contracts of the tree whose range of workgroups
// holds b, the trees with the most layers first.

__global__ __launch_bounds__(256) void pi_kernel(PiArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // row over layers 0..n-1
  if (r >= a.rows) return;
  int lo = 0, hi = a.n - 1;  // the layer k with pt_off_k <= r < pt_off_k + N_k
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.layers[mid].pt_off <= r) lo = mid; else hi = mid - 1;
  }
  const LayerDev& L = a.layers[lo];
  const int i = (int)(r - L.pt_off);
  const int N1 = L.N1, N1p = (N1 + 3) & ~3;
  const int32_t* row = a.counts + L.cnt_off + (int64_t)i * N1;
  int64_t p = 0;
  int jlo = N1p, jhi = 0;
  for (int j = lane; j < N1; j += 64) {
    const int32_t c = row[j];
    p += c;
    if (c != 0) {
      jlo = j < jlo ? j : jlo;
      jhi = j + 1;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    p += __shfl_xor(p, off, 64);
    const int l2 = __shfl_xor(jlo, off, 64), h2 = __shfl_xor(jhi, off, 64);
    jlo = l2 < jlo ? l2 : jlo;
    jhi = h2 > jhi ? h2 : jhi;
  }
  double* out = a.pi + a.pi_off[lo] + (int64_t)i * N1p;
  const double inv_p = p > 0 ? (double)p : 1.0;
  for (int j = lane; j < N1p; j += 64) {
    const int32_t c = j < N1 ? row[j] : 0;
    out[j] = p > 0 ? (double)c / inv_p : 0.0;
  }
  if (lane == 0) {
    // whole groups of 4 columns; an empty row scans nothing (continuation 0)
    a.band[r] = p > 0 ? make_int2(jlo & ~3, (jhi + 3) & ~3) : make_int2(0, 0);
  }
}

// pi_off[k] = sum_{l < k} N_l N1p_l (one thread; n is at most a few thousand).
__global__ void pi_offsets_kernel(const LayerDev* layers, int n, int64_t* pi_off) {
  int64_t o = 0;
  for (int k = 0; k < n; ++k) {
    pi_off[k] = o;
    o += (int64_t)layers[k].N * (int64_t)((layers[k].N1 + 3) & ~3);
  }
}

hipError_t launch_pi(const PiArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(pi_offsets_kernel, dim3(1), dim3(1), 0, s, a.layers, a.n,
                     const_cast<int64_t*>(a.pi_off));
  hipLaunchKernelGGL(pi_kernel, dim3((unsigned)((a.rows + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

namespace {

// Obstacle of contract C on layer k (the arithmetic of payoff_kernel, so
// both give the same phi bit for bit): the layer's discount and drifts once,
// then one exponential per asset and grid point.
struct LayerObstacle {
  double disc;
  double drift[3];  // (r - sigma_c^2 / 2) t_k
  bool euro;        // European before maturity: phi = -inf
};

template <int D>
__device__ __forceinline__ LayerObstacle layer_obstacle(const Contract& C, int n, int k) {
  LayerObstacle o;
  const double t = C.Tm * (double)k / (double)n;
  o.disc = exp(-C.r * t);
#pragma unroll
  for (int c = 0; c < 3; ++c)
    o.drift[c] = c < D ? (C.r - 0.5 * C.sigma[c] * C.sigma[c]) * t : 0.0;
  o.euro = (C.kind & 2) && k < n;
  return o;
}

template <int D>
__device__ __forceinline__ double obstacle(const Contract& C, const LayerObstacle& o,
                                           const float* xs) {
  double y[D];
#pragma unroll
  for (int c = 0; c < D; ++c) {
    double v = 0.0;
#pragma unroll
    for (int e = 0; e < D; ++e) v += C.mix[c * D + e] * (double)xs[e];
    y[c] = C.has_mix ? v : (double)xs[c];
  }
  double v;
  if (C.kind & 1) {
    double smax = -__builtin_huge_val();
#pragma unroll
    for (int c = 0; c < D; ++c) {
      const double sc = C.S0 * exp(o.drift[c] + C.sigma[c] * y[c]);
      smax = sc > smax ? sc : smax;
    }
    v = o.disc * fmax(smax - C.K, 0.0);
  } else {
    const double sc = C.S0 * exp(o.drift[0] + C.sigma[0] * y[0]);
    v = o.disc * fmax(C.K - sc, 0.0);
  }
  return o.euro ? -__builtin_huge_val() : v;
}

// The grid is read through global pointers: taken from the tree table, the
// generic ones were read with flat loads, which count against the same wait
// counter as the kernel's scalar weight loads.
template <int D>
__device__ __forceinline__ void grid_point(const ManyTree& a, int64_t pt_off, int i,
                                           float* xs) {
  const int64_t at = pt_off + i;
  typedef const float __attribute__((address_space(1)))* GlobalF32;
  if (D == 1) {
    xs[0] = ((GlobalF32)a.pts1)[at];
  } else {
    const GlobalF32 g = (GlobalF32)(a.pts + at);  // the point's x, y (, z)
    xs[0] = g[0];
    xs[1] = g[1];
    if (D == 3) xs[2] = g[2];
  }
}

}  // namespace

// Read-only device memory in the global address space: uniform loads through
// such pointers may become scalar loads (a generic pointer taken from the
// tree table would be read with flat vector loads).
typedef const double __attribute__((address_space(1)))* GlobalF64;
typedef const int32_t __attribute__((address_space(1)))* GlobalI32;
typedef const int64_t __attribute__((address_space(1)))* GlobalI64;
typedef const uint64_t __attribute__((address_space(1)))* GlobalU64;


// Workgroup b prices 16 CTS contracts.  Wave w of 8 has contracts 16 (w % CTS)
// .. + 15 (one per lane % 16, for the whole recursion) and the tiles of 16
// rows w / CTS, w / CTS + 8 / CTS, ... of every layer: at most TILES of them,
// whose new values stay in registers until every wave has read V_{k+1}.
// A tile's product covers the columns of its rows' bands, 16 at a time, with
// the K order of bdp_tile.hpp (lane group g takes columns 4 g .. + 3 of the
// 16, 32 bytes of its row).
//
// R: a lane has rows g, g + 4, ... of a tile; layers of at most 4 R points have R
// of them, and no others' obstacles are computed (50 layers of 4 points, one
// contract 77 -> 60 us, 20000 138 -> 75).
//
// The products (64 clocks of a matrix core for 1024 multiply-adds, the rate
// of the vector units) run beside the obstacles' exponentials of other waves.
// With lane = contract, vector multiply-adds and the weights as scalar
// operands, every 16 of them waited for four scalar loads, and the four rows
// of a step were 8 apart, their bands' union half as wide again.
constexpr int kManyWaves = 8;

// V_0 of one contract by the workgroup's waves, a row at a time, where a weight
// of zero adds nothing whatever the value is.  A tile's product has many of
// them (columns of other rows' bands, the rest of a group of 16, rows of Vs past
// the layer), and where an obstacle overflowed they are 0 x inf, NaN.  A NaN
// stays one through every later product and maximum, so a price that is not
// NaN met none, and only contracts of finite parameters whose price is NaN come
// here.  (Tests of the values or of the products within the tiles: 6 % of the
// whole call.)  v: LDS, 2 a.np_max doubles.
template <int D>
__device__ __forceinline__ double price_by_rows(const ManyTree& T, const Contract& C, double* v,
                                                int np_max) {
  const GlobalI32 lay = (GlobalI32)T.layers;
  constexpr int kLayWords = (int)(sizeof(LayerDev) / 4);
  constexpr int kN = (int)(offsetof(LayerDev, N) / 4), kN1 = (int)(offsetof(LayerDev, N1) / 4),
                kPt = (int)(offsetof(LayerDev, pt_off) / 4);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  double *now = v, *next = v + np_max;
  for (int k = T.n; k >= 0; --k) {
    const int Nk = lay[k * kLayWords + kN];
    const int64_t pt = lay[k * kLayWords + kPt];
    const LayerObstacle ob = layer_obstacle<D>(C, T.n, k);
    const int N1p = k < T.n ? (lay[k * kLayWords + kN1] + 3) & ~3 : 0;
    const GlobalF64 P = (GlobalF64)T.pi + (k < T.n ? ((GlobalI64)T.pi_off)[k] : 0);
    __syncthreads();  // `now` is not read any more
#pragma unroll 1
    for (int i = wave; i < Nk; i += kManyWaves) {
      double sum = -__builtin_huge_val();
      if (k < T.n) {
        const GlobalF64 row = P + (int64_t)i * N1p;
        sum = 0.0;
#pragma unroll 1
        for (int j = lane; j < N1p; j += 64) {
          const double w = row[j];
          if (w != 0.0) sum = fma(w, next[j], sum);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
      }
      float xs[3];
      grid_point<D>(T, pt, i, xs);
      const double f = obstacle<D>(C, ob, xs);
      if (lane == 0) now[i] = k == T.n || f > sum ? f : sum;
    }
    __syncthreads();
    double* const t = now;
    now = next;
    next = t;
  }
  return next[0];
}

__device__ __forceinline__ bool finite_parameters(const Contract& C, int d) {
  bool ok = __builtin_isfinite(C.S0) && __builtin_isfinite(C.K) && __builtin_isfinite(C.r) &&
            __builtin_isfinite(C.Tm);
  for (int c = 0; c < d; ++c) ok = ok && __builtin_isfinite(C.sigma[c]);
  for (int c = 0; c < d * d; ++c) ok = ok && (!C.has_mix || __builtin_isfinite(C.mix[c]));
  return ok;
}

template <int D, int CTS, int TILES, int R = 4, int SPLIT = 1>
__global__ __launch_bounds__(64 * kManyWaves) void bdp_many_kernel(ManyArgs a) {
  constexpr int kCols = 16 * CTS, kRowWaves = kManyWaves / CTS, kRowTiles = kRowWaves / SPLIT;
  extern __shared__ double Vs[];  // [np_max][kCols]
  const int lane = threadIdx.x & 63, g = lane >> 4, m = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ct = wave % CTS, rw = wave / CTS;
  const int rt0 = SPLIT > 1 ? rw % kRowTiles : rw, r0 = SPLIT > 1 ? R * (rw / kRowTiles) : 0;
  // the workgroup's tree: the one tree, or the last table entry with
  // blk0 <= blockIdx.x
  ManyTree T;
  int64_t qb = (int64_t)blockIdx.x * kCols, qe = a.nq;
  if (a.trees) {
    // the table is read through a global pointer, so the record's values are
    // known to be uniform (a generic load could be a per-lane one)
    constexpr int kWords = (int)(sizeof(ManyTree) / 8);
    const GlobalU64 tab = (GlobalU64)a.trees;
    constexpr int kBlk0 = (int)(offsetof(ManyTree, blk0) / 4);
    int lo = 0, hi = a.n_trees - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (((GlobalI32)tab)[mid * 2 * kWords + kBlk0] <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    uint64_t raw[kWords];
#pragma unroll
    for (int w = 0; w < kWords; ++w) raw[w] = tab[lo * kWords + w];
    __builtin_memcpy(&T, raw, sizeof(ManyTree));
    qb = T.q0 + ((int64_t)blockIdx.x - T.blk0) * kCols;
    qe = T.q0 + T.nq;
  } else {
    T.layers = a.layers;
    T.pts1 = a.pts1;
    T.pts = a.pts;
    T.pi_off = a.pi_off;
    T.pi = a.pi;
    T.band = a.band;
    T.n = a.n;
  }
  const int col = 16 * ct + m;
  const int64_t q = qb + col;
  const Contract C = a.specs[q < qe ? q : qe - 1];
  // zero the padding rows once (they meet only zero weights, but must be finite)
  for (int j = threadIdx.x; j < kCols * a.np_max; j += 64 * kManyWaves) Vs[j] = 0.0;
  __syncthreads();
  // per-layer fields through global pointers (uniform values)
  const GlobalI32 lay = (GlobalI32)T.layers;
  constexpr int kLayWords = (int)(sizeof(LayerDev) / 4);
  constexpr int kN = (int)(offsetof(LayerDev, N) / 4), kN1 = (int)(offsetof(LayerDev, N1) / 4),
                kPt = (int)(offsetof(LayerDev, pt_off) / 4);
  {
    const int Nn = lay[T.n * kLayWords + kN];
    const int64_t pt = lay[T.n * kLayWords + kPt];
    const LayerObstacle ob = layer_obstacle<D>(C, T.n, T.n);
    for (int i = 4 * rw + g; i < Nn; i += 4 * kRowWaves) {
      float xs[3];
      grid_point<D>(T, pt, i, xs);
      Vs[i * kCols + col] = obstacle<D>(C, ob, xs);
    }
  }
  __syncthreads();
  for (int k = T.n - 1; k >= 0; --k) {
    const int Nk = lay[k * kLayWords + kN], N1p = (lay[k * kLayWords + kN1] + 3) & ~3;
    const int64_t pt = lay[k * kLayWords + kPt];
    const GlobalF64 P = (GlobalF64)T.pi + ((GlobalI64)T.pi_off)[k];
    const GlobalI32 B = (GlobalI32)(T.band + pt);  // (lo, hi) pairs
    const LayerObstacle ob = layer_obstacle<D>(C, T.n, k);
    f64x4 res[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const int i0 = 16 * (rt0 + kRowTiles * t);
      if (i0 + 4 * r0 >= Nk) break;
      // the tile's band: whole groups of 4 columns, empty rows (lo = hi) apart
      const int i = min(i0 + m, Nk - 1);  // rows past the end repeat the last one
      int lo = B[2 * i], hi = B[2 * i + 1];
      lo = hi > lo ? lo : 1 << 30;
#pragma unroll
      for (int s = 8; s > 0; s >>= 1) {
        lo = min(lo, __shfl_xor(lo, s, 64));
        hi = max(hi, __shfl_xor(hi, s, 64));
      }
      lo = __builtin_amdgcn_readfirstlane(lo);
      hi = __builtin_amdgcn_readfirstlane(hi);
      const GlobalF64 row = P + (int64_t)i * N1p;
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      for (int j0 = lo; j0 < hi; j0 += 16) {
        // a group past the row's end reads its last columns, times nothing
        const int j = j0 + 4 * g, jc = min(j, N1p - 4);
        double w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = row[jc + u];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(j < N1p ? w[u] : 0.0,
                                                     Vs[(jc + u) * kCols + col], acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        double cont = acc[r];
#pragma unroll
        for (int w = 1; w < SPLIT; ++w) cont = r0 == R * w ? acc[R * w + r] : cont;
        const int ir = min(i0 + g + 4 * (r0 + r), Nk - 1);
        float xs[3];
        grid_point<D>(T, pt, ir, xs);
        const double f = obstacle<D>(C, ob, xs);
        res[t][r] = f > cont ? f : cont;
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const int i0 = 16 * (rt0 + kRowTiles * t);
      if (i0 + 4 * r0 >= Nk) break;
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (i0 + g + 4 * (r0 + r) < Nk) Vs[(i0 + g + 4 * (r0 + r)) * kCols + col] = res[t][r];
    }
    __syncthreads();
  }
  bool again = false;
  if (threadIdx.x < kCols && qb + threadIdx.x < qe) {
    const double v0 = Vs[threadIdx.x];
    a.V0[qb + threadIdx.x] = v0;
    again = v0 != v0;
  }
  // (kCols <= 64: wave 0 has read its values, the row after them is free)
  uint64_t& redo = reinterpret_cast<uint64_t*>(Vs)[kCols];
  if (wave == 0) {
    const uint64_t mask = __ballot(again);
    if (lane == 0) redo = mask;
  }
  __syncthreads();
  uint64_t mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(redo >> 32));
  mask = mask << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)redo);
  for (; mask != 0; mask &= mask - 1) {
    const int64_t qc = qb + __ffsll((unsigned long long)mask) - 1;
    const Contract one = a.specs[qc];
    if (!finite_parameters(one, D)) continue;
    const double v0 = price_by_rows<D>(T, one, Vs, a.np_max);
    if (threadIdx.x == 0) a.V0[qc] = v0;
  }
}

bool bdp_many_fits(int max_n) { return max_n <= 256; }

// A layer of a workgroup is a chain (products, obstacles, two barriers): 16
// contracts and a tile of rows per wave make it short and the workgroups many,
// 64 and four tiles load each weight once for four products.  Trees of 10 to
// 100 layers of 100 points, 16 / 64 contracts a workgroup: 1000 contracts 324 /
// 904 us, 15000 470 / 894, 30000 767 / 970, 100000 2338 / 2162 (the lane =
// contract kernel: 6470 us).
// Up to 48 points a layer (on average) a layer's work is small beside its chain,
// and the workgroups are better few: from 192 of 64 on (d = 1) those win.  60
// layers, 12000 / 16000 / 20000 contracts, 16 against 64: 12 points 97/102,
// 168/102, 169/123 us; 43 points 189/198, 249/201, 287/311; sizes of 1 to 44
// 113/118, 187/118, 190/164; 62 points 220/287, 292/289, 335/453.  That is where
// the workgroups of 16 are more than three per CU, as many as are resident; for
// d > 1, two.  20 layers, 6000 / 12000 contracts, 16 against 64, d = 2: 8 points
// 44/45, 70/46, 16 points 47/58, 63/59, up to 32 points 57/67, 73/68; d = 3 47/49,
// 79/49, 52/65, 84/66 and 62/77, 91/79.
int bdp_many_cols(int d, int64_t blocks64, int64_t points, int64_t layers) {
  const int64_t small = d == 1 ? 192 : 128;
  return blocks64 < (points <= 48 * layers ? small : 1024) ? 16 : 64;
}

template <int D>
static hipError_t launch_bdp_many_d(const ManyArgs& a, hipStream_t s) {
  const dim3 grid(a.trees ? (unsigned)a.blocks : (unsigned)((a.nq + a.cols - 1) / a.cols));
  const size_t lds = sizeof(double) * (size_t)a.cols * (size_t)a.np_max;
  auto go = [&](auto* kernel) {
    hipError_t e = hipSuccess;
    if (lds > 65536)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * kManyWaves), lds, s, a);
    return hipGetLastError();
  };
  if (!bdp_many_fits(a.max_n)) return hipErrorInvalidValue;
  if (a.max_n <= 4)
    return a.cols == 16 ? go(bdp_many_kernel<D, 1, 1, 1>) : go(bdp_many_kernel<D, 4, 1, 1>);
  if (a.max_n <= 8)
    return a.cols == 16 ? go(bdp_many_kernel<D, 1, 1, 2>) : go(bdp_many_kernel<D, 4, 1, 2>);
  if constexpr (D > 1) {
    if (a.max_n <= 32 && a.cols == 16) return go(bdp_many_kernel<D, 1, 1, 1, 4>);
    if (a.max_n <= 16) return go(bdp_many_kernel<D, 4, 1, 2, 2>);
  }
  const bool small = a.max_n <= 128;
  if (a.cols == 16) return small ? go(bdp_many_kernel<D, 1, 1>) : go(bdp_many_kernel<D, 1, 2>);
  return small ? go(bdp_many_kernel<D, 4, 4>) : go(bdp_many_kernel<D, 4, 8>);
}

hipError_t launch_bdp_many(const ManyArgs& a, hipStream_t s) {
  if (a.trees ? a.blocks <= 0 : a.nq <= 0) return hipSuccess;
  if (a.d == 1) return launch_bdp_many_d<1>(a, s);
  if (a.d == 2) return launch_bdp_many_d<2>(a, s);
  return launch_bdp_many_d<3>(a, s);
}

}  // namespace qtree
