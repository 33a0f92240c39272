// Swing option on the quantization tree (Sec. 2: the stochastic control
// problem whose optimal control is bang-bang) and its obstacle, the forward
// on the sum of the factors of the Gaussian model (Sec. 3), FP64.
//
// The state of the recursion is the volume c consumed before date k, and P
// is stored point major ([point][level]) so that the levels of one grid
// point are contiguous.  cont(i, c) = sum_j c_ij P_{k+1}(j, c) / p_i is a
// product of the count block with P_{k+1}, on the FP64 matrix cores; then, for
// every c, the best feasible exercise x in {0, 1}:
//   P_k(i, c) = max_x  x v_k(i) + cont(i, c + x),
// x feasible when c + x <= Qmax and c + x + (n - k - 1) >= Qmin.
#include "bdp_tile.hpp"
#include "qtree_internal.hpp"

namespace qtree {

namespace {
constexpr int kBlock = 256;
constexpr int kRows = 16;   // rows per workgroup
constexpr int kWaves = 8;   // waves sharing a workgroup's columns
constexpr int kAhead = 2;   // chunks of 16 columns a wave takes at once
}  // namespace

__global__ void forward_payoff_kernel(ForwardArgs a) {
  const int k = blockIdx.y;
  const LayerDev& L = a.layers[k];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= L.N) return;
  const int d = a.d;
  // variance of w . X_k under X_k = mu_k + L_k z, and the mean term
  double var = 0.0, wm = 0.0;
  for (int c = 0; c < d; ++c) {
    double u = 0.0;
    for (int b = 0; b < d; ++b) u += a.w[b] * (double)L.L[b * d + c];
    var += u * u;
  }
  for (int b = 0; b < d; ++b) wm += a.w[b] * (double)L.mu[b];
  const int64_t at = (int64_t)L.pt_off + i;
  const float4 g = d == 1 ? make_float4(a.pts1[at], 0.f, 0.f, 0.f) : a.pts[at];
  const float xs[3] = {g.x, g.y, g.z};
  double s = 0.0;
  for (int b = 0; b < d; ++b) s += a.w[b] * (double)xs[b];
  const double t = a.Tm * (double)k / (double)a.n;
  a.v[at] = exp(-a.r * t) * (a.S0 * exp(s - wm - 0.5 * var) - a.K);
}

__global__ void swing_init_kernel(SwingArgs a) {
  const LayerDev& L = a.layers[a.n];
  const int64_t total = (int64_t)(a.Qmax + 1) * L.N;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(t / L.N), i = (int)(t - (int64_t)c * L.N);
    a.P[((int64_t)L.pt_off + i) * (a.Qmax + 1) + c] =
        (c >= a.Qmin && c <= a.Qmax) ? 0.0 : -__builtin_huge_val();
  }
}

// Workgroup (x, y): kLevels = 16 TILES levels from (kLevels - 1) x on (the last
// feeds the x = 1 choice of the one before and is not written), rows 16 y ..
// + 15; wave w takes the chunks of 16 columns w, w + 8, ....  A chunk without
// a count (most of them: a step of the factors reaches few cells) is known
// before its values are asked for.  A level that no feasible choice reads
// (c + rest < Qmin) holds -inf in P_{k+1} and is taken as zero.
//
// What bounds a layer is the latency of a launch and of its round trips
// (counts, then values), so the code is short and its registers few: with
// four chunks at once and 128 registers a layer of 500 points took 10.5 us,
// with two 7.3; 3 or 4 tiles 7.2 - 8.0, 16 waves 7.5 - 9.7.  n = 365, volume
// up to 250: 2.67 ms at 500 points a layer (one tile: 2.82), 1.55 ms at 100
// (two tiles: 1.68), against 11.7 and 3.3 ms with one wave per row and 63
// levels walking the row's counts.
template <int TILES>
__global__ __launch_bounds__(64 * kWaves, 4) void swing_layer_kernel(SwingArgs a, int k, int N,
                                                                     int N1, int64_t pt,
                                                                     int64_t pt1, int64_t cnt) {
  constexpr int kLevels = 16 * TILES, kSpan = kLevels - 1;
  __shared__ double part[kWaves][kRows][kLevels + 1];
  __shared__ int64_t part_p[kWaves][kRows];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = lane >> 4, m = lane & 15;
  const int levels = a.Qmax + 1;
  const int rest = a.n - k - 1;  // dates after this one
  const int c0 = kSpan * (int)blockIdx.x, i0 = kRows * (int)blockIdx.y;
  const int i = min(i0 + m, N - 1);  // rows past the end repeat the last one
  const int32_t* row = a.counts + cnt + (int64_t)i * N1;
  double vi[kRows / kWaves];  // obstacles of the rows this wave finishes
#pragma unroll
  for (int e = 0; e < kRows / kWaves; ++e) vi[e] = a.v[pt + min(i0 + wave + kWaves * e, N - 1)];
  // the lane's levels of a point: byte offsets in its row of P_{k+1}
  // (below 2^32: at most 16384 points of 2047 levels, 8 bytes each)
  const char* next = reinterpret_cast<const char*>(a.P + pt1 * levels);
  bool used[TILES];
  uint32_t lev[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    const int ct = c0 + 16 * t + m;
    used[t] = ct < levels && ct + rest >= a.Qmin;
    lev[t] = 8u * (uint32_t)min(ct, levels - 1);
  }
  auto value = [&](int col, int t) {
    const uint32_t at = 8u * (uint32_t)levels * (uint32_t)col + lev[t];
    return *reinterpret_cast<const double*>(next + at);
  };
  f64x4 acc[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  int64_t p = 0;
  for (int j0 = 16 * wave; j0 < N1; j0 += 16 * kWaves * kAhead) {
    const int j = j0 + 4 * g;
    int32_t cn[kAhead][4];
    if (N1 >= 4) {
      load_cols(row, N1, j, 16 * kWaves, cn);
      if (j0 + 16 * kWaves * (kAhead - 1) + 16 > N1) drop_tails(N1, j, 16 * kWaves, cn);
    } else {  // one chunk
#pragma unroll
      for (int s = 0; s < kAhead; ++s)
#pragma unroll
        for (int u = 0; u < 4; ++u) cn[s][u] = (s == 0 && j + u < N1) ? row[j + u] : 0;
    }
    double x[kAhead][TILES][4];
    uint32_t hit = 0, slow = 0;  // chunks with a count, with a value that is not finite
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      p += (int64_t)cn[s][0] + cn[s][1] + cn[s][2] + cn[s][3];
      if (__any((cn[s][0] | cn[s][1] | cn[s][2] | cn[s][3]) != 0)) hit |= 1u << s;
    }
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      if (!(hit >> s & 1)) continue;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < TILES; ++t)
          x[s][t][u] = value(min(j + 16 * kWaves * s + u, N1 - 1), t);
    }
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      if (!(hit >> s & 1)) continue;
#pragma unroll
      for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) x[s][t][u] = used[t] ? x[s][t][u] : 0.0;
      bool finite = true;
#pragma unroll
      for (int t = 0; t < TILES; ++t) finite = finite && finite4(x[s][t]);
      if (!__all(finite)) {
        slow |= 1u << s;
        continue;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < TILES; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)cn[s][u], x[s][t][u], acc[t], 0, 0,
                                                        0);
    }
    // obstacles that are not finite (a caller's): column by column, so that a
    // zero count adds nothing
    for (int s = 0; slow != 0; ++s, slow >>= 1) {
      if (!(slow & 1)) continue;
      const int j1 = j0 + 16 * kWaves * s;
      for (int col = j1; col < min(j1 + 16, N1); ++col) {
        const int32_t mine = row[col];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
          const double v = used[t] ? value(col, t) : 0.0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int32_t ce = __shfl(mine, g + 4 * e, 64);
            if (ce != 0) acc[t][e] = fma((double)ce, v, acc[t][e]);
          }
        }
      }
    }
  }
  p += __shfl_xor(p, 16, 64);
  p += __shfl_xor(p, 32, 64);
#pragma unroll
  for (int t = 0; t < TILES; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][g + 4 * e][16 * t + m] = acc[t][e];
  if (lane < kRows) part_p[wave][lane] = p;
  __syncthreads();
  // wave w finishes rows w, w + 8; lane = level
  const int c = c0 + lane;
#pragma unroll
  for (int r = wave; r < kRows; r += kWaves) {
    if (i0 + r >= N) break;
    double s = 0.0;
    int64_t total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      s += part[w][r][min(lane, kLevels - 1)];
      total += part_p[w][r];
    }
    const double cont = total > 0 ? s / (double)total : 0.0;
    const double cont1 = __shfl_down(cont, 1, 64);  // level c + 1
    if (lane >= kSpan || c >= levels) continue;
    double best = -__builtin_huge_val();
    if (c + rest >= a.Qmin) best = cont;
    if (c + 1 <= a.Qmax && c + 1 + rest >= a.Qmin) {
      const double e = vi[r / kWaves] + cont1;
      best = e > best ? e : best;
    }
    a.P[(pt + i0 + r) * levels + c] = best;
  }
}

hipError_t launch_forward_payoff(const ForwardArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.maxN + kBlock - 1) / kBlock), (unsigned)(a.n + 1));
  hipLaunchKernelGGL(forward_payoff_kernel, grid, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_swing(const SwingArgs& a, const int32_t* N_host, hipStream_t s) {
  hipLaunchKernelGGL(swing_init_kernel, dim3(256), dim3(kBlock), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int64_t pt = 0, cnt = 0;  // first point and count of layer k
  for (int k = 0; k < a.n; ++k) {
    pt += N_host[k];
    cnt += (int64_t)N_host[k] * N_host[k + 1];
  }
  auto spans = [&](int tiles) {
    return (unsigned)((a.Qmax + 1 + 16 * tiles - 2) / (16 * tiles - 1));
  };
  for (int k = a.n - 1; k >= 0; --k) {
    const int N = N_host[k], N1 = N_host[k + 1];
    const int64_t pt1 = pt;
    pt -= N;
    cnt -= (int64_t)N * N1;
    const unsigned rows = (unsigned)((N + kRows - 1) / kRows);
    // one tile of levels while that fills the chip (256 CUs) about once, two
    // beyond (half of the count loads)
    if (spans(1) * rows <= 320)
      hipLaunchKernelGGL(swing_layer_kernel<1>, dim3(spans(1), rows), dim3(64 * kWaves), 0, s, a, k,
                         N, N1, pt, pt1, cnt);
    else
      hipLaunchKernelGGL(swing_layer_kernel<2>, dim3(spans(2), rows), dim3(64 * kWaves), 0, s, a, k,
                         N, N1, pt, pt1, cnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace qtree
