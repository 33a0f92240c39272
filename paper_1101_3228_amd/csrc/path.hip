// Pathwise estimate (Sec. 3, Algorithms I/II): one lane per path walks all
// layers.  The cells a path visits either go to scratch (uint16, [layer]
// [path]) for a counting pass in which one workgroup owns 16384 entries of a
// count block in LDS, or are counted on the spot with one device-scope atomic
// per step (no scratch, or count blocks of too many tiles).
//
// A device-scope atomic costs about 50 ps of the whole chip; reading a cell
// pair once per super tile of its block, 0.7 ps, the walk's two bytes, and a
// read and a write of every count in each pass (through_cells in api.cpp
// weighs them).
#include "qtree_internal.hpp"
#include "qtree_rng.hpp"
#include "qtree_search.hpp"

namespace qtree {

namespace {

constexpr int kBlock = 256;
constexpr int kStep = 4;        // d = 1: layers whose midpoints are staged together
constexpr int kStageP = 1024;   // ... where the largest is no larger (padded)
constexpr int kCountBlock = 1024;
constexpr size_t kLdsBytes = 160 * 1024;  // of a CU

// Where a path's cells go.
struct Visits {
  uint16_t* cells;  // [n][stride]: cell of layer k + 1 at row k (STORE kernels)
  int64_t stride;
};

// Path t (of this launch) moved from cell i of layer k to cell j of layer k + 1.
template <bool STORE>
__device__ __forceinline__ void visit(const FwdArgs& a, const Visits& v, int k, uint64_t t,
                                      bool live, int i, int j) {
  if (!live) return;
  if (STORE) {
    v.cells[(int64_t)k * v.stride + (int64_t)t] = (uint16_t)j;
  } else {
    const LayerDev& L = a.layers[k];
    __hip_atomic_fetch_add(a.counts + L.cnt_off + (int64_t)i * L.N1 + j, 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

// d = 1: kStep layers at a time (one Philox block gives kStep normals): the
// states first, a chain of fused multiply-adds, then the searches of all
// kStep cells side by side over midpoints staged in LDS while the normals
// are drawn.  STAGE = false (layers above kStageP points): the searches read
// the midpoints from memory, as a workgroup's 256 paths would not use what it
// stages (32 KB for 2048 points; 20 layers of 1448 points, 2 10^4 paths 114 us
// staged, 103 not; 50 of 500 points 116 and 142).
template <bool STAGE, bool STORE>
__global__ __launch_bounds__(kBlock) void walk_1d(FwdArgs a, Visits v) {
  extern __shared__ float lds[];  // [kStep][maxP]
  const uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool live = t < a.M;
  const uint32_t mc = (uint32_t)(a.m0 + (live ? t : 0));
  const uint32_t k0 = vgpr_copy(a.key0), k1 = vgpr_copy(a.key1);
  float x = a.layers[0].x0[0];
  int i = 0;
  for (int k = 0; k < a.n; k += kStep) {
    const int steps = a.n - k < kStep ? a.n - k : kStep;
    if (STAGE) {
      __syncthreads();  // the searches of the layers before
      for (int s = 0; s < steps; ++s) {
        const LayerDev& L1 = a.layers[k + 1 + s];
        for (int q = threadIdx.x; q < L1.P; q += kBlock)
          lds[s * a.maxP + q] = a.mids[L1.aux_off + q];
      }
    }
    const U4 r = philox4x32_10(U4{mc, (uint32_t)(k >> 2), a.contract, 1u}, k0, k1);
    float e[kStep], y[kStep];
    box_muller(r.x, r.y, e[0], e[1]);
    box_muller(r.z, r.w, e[2], e[3]);
#pragma unroll
    for (int s = 0; s < kStep; ++s) {
      const LayerDev& L = a.layers[min(k + s, a.n - 1)];
      x = fmaf(L.T[0], e[s], fmaf(L.A[0], x, L.b[0]));
      y[s] = x;
    }
    if (STAGE) __syncthreads();
    int lg[kStep], top = 0;
    const float* m[kStep];
#pragma unroll
    for (int s = 0; s < kStep; ++s) {
      const LayerDev& L1 = a.layers[min(k + 1 + s, a.n)];
      m[s] = STAGE ? lds + s * a.maxP : a.mids + L1.aux_off;
      lg[s] = s < steps ? L1.logP : 0;
      top = max(top, lg[s]);
    }
    if (!STORE) {
      // one after the other: the atomics of a step run beside the next search
      // (5 layers of 3000 points, 10^5 paths 71 us, side by side 79)
#pragma unroll
      for (int s = 0; s < kStep; ++s)
        if (s < steps) {
          const int c = cell_1d(m[s], lg[s], y[s]);
          visit<STORE>(a, v, k + s, t, live, i, c);
          i = c;
        }
      continue;
    }
    // the deepest search of the kStep layers serves all: a midpoint past a
    // layer's own padded array is not read (its steps are skipped)
    int c[kStep] = {};
    for (int h = top - 1; h >= 0; --h) {
#pragma unroll
      for (int s = 0; s < kStep; ++s)
        if (h < lg[s]) {
          const int w = 1 << h;
          c[s] = m[s][c[s] + w - 1] < y[s] ? c[s] + w : c[s];
        }
    }
#pragma unroll
    for (int s = 0; s < kStep; ++s)
      if (s < steps) {
        visit<STORE>(a, v, k + s, t, live, i, c[s]);
        i = c[s];
      }
  }
}

// X_{k+1} = b + A x + T e, in the order of layer_pair.
__device__ __forceinline__ void step_2d(const float* A, const float* T, const float* b, float e0,
                                        float e1, float& x0, float& x1) {
  const float z0 = fmaf(A[1], x1, fmaf(A[0], x0, b[0]));
  const float z1 = fmaf(A[3], x1, fmaf(A[2], x0, b[1]));
  x0 = fmaf(T[1], e1, fmaf(T[0], e0, z0));
  x1 = fmaf(T[3], e1, fmaf(T[2], e0, z1));
}

// What step k needs of the records of layers k and k + 1, in LDS.
struct alignas(16) StepRec {
  float A[4], T[4], b[2];
  float bk_lo[2], bk_scale[2];
  int32_t bk_B[2];
  int32_t bk_off, N, pt_off, pad;
};
constexpr int kRecWords = sizeof(StepRec) / 4;
// Word w of the record of step k.
__device__ __forceinline__ uint32_t step_word(const FwdArgs& a, int k, int w) {
  constexpr int kLay = sizeof(LayerDev) / 4;
#define QTREE_W(f) ((int)(offsetof(LayerDev, f) / 4))
  int at;
  if (w < 4) at = QTREE_W(A) + w;
  else if (w < 8) at = QTREE_W(T) + w - 4;
  else if (w < 10) at = QTREE_W(b) + w - 8;
  else if (w < 16) at = kLay + QTREE_W(bk_lo) + w - 10;  // lo, scale and B are adjacent
  else if (w == 16) at = kLay + QTREE_W(bk_off);
  else if (w == 17) at = kLay + QTREE_W(N);
  else at = kLay + QTREE_W(pt_off);
#undef QTREE_W
  return reinterpret_cast<const uint32_t*>(a.layers + k)[at];
}
static_assert(offsetof(LayerDev, bk_scale) == offsetof(LayerDev, bk_lo) + 8 &&
                  offsetof(LayerDev, bk_B) == offsetof(LayerDev, bk_lo) + 16,
              "copied as one run");

// d = 2 with bucket tables, cells to scratch.  A path's normals and its cell
// searches are independent of each other; only the state X_k is a chain, of
// four fused multiply-adds a step.  So a workgroup takes kWidePaths paths and
// kWideSteps steps at a time, and the kSegments waves of the same 64 paths
// share them: each draws the normals of its two steps (one Philox block) into
// LDS, walks the whole chain, and searches the cells of its own two layers,
// whose points the waves of one segment stage together.
//
// One wave per 64 paths and all of their work (1e5 paths: 1.5 waves per SIMD)
// took 1.4 us a step at 240 points, 312 instructions at 11 clocks each: a
// serial chain on an idle chip.  64 VGPRs let 1024 of these workgroups be
// resident while the LDS holds four of them per CU, up to 490 points a layer
// (1e5 paths are 782; at 80 VGPRs 14 of them ran after the others, 611 us for
// 365 steps of 240 points against 408), and the layers' records come through
// LDS a turn ahead (333 us; as scalar loads, every step of the chain waited
// for its own).  At 500 points three fit and 14 of the 782 run after the rest.
constexpr int kWidePaths = 128, kSegments = 4, kWideSteps = 2 * kSegments;
constexpr int kWideBlock = kWidePaths * kSegments;
static_assert(kWideSteps * kRecWords <= kWideBlock, "one word of the records per thread");

// LDS of a workgroup, 64 bytes per point of the largest layer: more than a CU
// has from 2412 points on, whatever the count blocks are.
size_t wide_lds(int maxN) {
  return 2 * sizeof(StepRec) * kWideSteps + sizeof(float) * 2 * kWideSteps * kWidePaths +
         sizeof(float2) * kWideSteps * (size_t)((maxN + 2) & ~1);
}

__global__ __launch_bounds__(kWideBlock) __attribute__((amdgpu_waves_per_eu(8)))
void walk_2d_wide(FwdArgs a, Visits v) {
  extern __shared__ float4 lds4[];
  StepRec* recs = reinterpret_cast<StepRec*>(lds4);  // [2][kWideSteps]
  float* eps = reinterpret_cast<float*>(recs + 2 * kWideSteps);  // [2 kWideSteps][kWidePaths]
  float2* points = reinterpret_cast<float2*>(eps + 2 * kWideSteps * kWidePaths);
  const int buf = (a.maxN + 2) & ~1;
  const int seg = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWidePaths);
  const int p = (int)threadIdx.x % kWidePaths;
  const uint64_t t = (uint64_t)blockIdx.x * kWidePaths + (uint64_t)p;
  const bool live = t < a.M;
  const uint32_t mc = (uint32_t)(a.m0 + (live ? t : 0));
  const float2* pts = reinterpret_cast<const float2*>(a.pts);  // x, y of point q at 2 q
  const float2 nan2 = make_float2(__builtin_nanf(""), __builtin_nanf(""));
  float x0 = a.layers[0].x0[0], x1 = a.layers[0].x0[1];
  float2* mine = points + 2 * seg * buf;
  // this thread's word of the records of kWideSteps steps (clamped to the last)
  const int rw = (int)threadIdx.x % kRecWords, rs = (int)threadIdx.x / kRecWords;
  auto fetch = [&](int kb) {
    return rs < kWideSteps ? step_word(a, min(kb + rs, a.n - 1), rw) : 0u;
  };
  auto keep = [&](int half, uint32_t word) {
    if (rs < kWideSteps)
      reinterpret_cast<uint32_t*>(recs + half * kWideSteps)[rs * kRecWords + rw] = word;
  };
  keep(0, fetch(0));
  __syncthreads();
  int half = 0;
  for (int kb = 0; kb < a.n; kb += kWideSteps, half ^= 1) {
    const StepRec* R = recs + half * kWideSteps;
    const uint32_t ahead = fetch(kb + kWideSteps);
    const int ks = kb + 2 * seg;  // this segment's steps ks, ks + 1
    const int steps = min(max(a.n - ks, 0), 2);
    float e[4] = {0.f, 0.f, 0.f, 0.f};
    if (steps > 0) {
      const U4 r = philox4x32_10_vk(U4{mc, (uint32_t)(ks >> 1), a.contract, 1u}, a.key0, a.key1);
      box_muller(r.x, r.y, e[0], e[1]);
      box_muller(r.z, r.w, e[2], e[3]);
    }
    __syncthreads();  // the searches of the steps before
    keep(half ^ 1, ahead);
#pragma unroll
    for (int u = 0; u < 4; ++u) eps[(4 * seg + u) * kWidePaths + p] = e[u];
    for (int s = 0; s < steps; ++s) {
      const int N1 = __builtin_amdgcn_readfirstlane(R[2 * seg + s].N);
      const int pt = __builtin_amdgcn_readfirstlane(R[2 * seg + s].pt_off);
      float2* to = mine + s * buf;
      for (int q0 = p; q0 <= N1; q0 += 2 * kWidePaths) {
        const int q1 = q0 + kWidePaths;
        const float2 r0 = pts[2 * (pt + min(q0, N1 - 1))], r1 = pts[2 * (pt + min(q1, N1 - 1))];
        to[q0] = q0 < N1 ? r0 : nan2;
        if (q1 <= N1) to[q1] = q1 < N1 ? r1 : nan2;
      }
    }
    __syncthreads();
    // the chain; this segment's states on the way
    float xs[2][1][2];
#pragma unroll
    for (int s = 0; s < kWideSteps; ++s) {
      if (kb + s < a.n)
        step_2d(R[s].A, R[s].T, R[s].b, eps[(2 * s) * kWidePaths + p],
                eps[(2 * s + 1) * kWidePaths + p], x0, x1);
      if (s >> 1 == seg) {
        xs[s & 1][0][0] = x0;
        xs[s & 1][0][1] = x1;
      }
    }
    if (steps == 0) continue;
    uint4 w[2][1];
#pragma unroll
    for (int s = 0; s < 2; ++s) bucket_rows<1>(R[2 * seg + s], R[2 * seg + s].N, a.bk, xs[s], w[s]);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (s >= steps) break;
      int j[1];
      bucket_argmin<1, true>(mine + s * buf, R[2 * seg + s].N, a.bk, xs[s], w[s], j);
      if (live) v.cells[(int64_t)(ks + s) * v.stride + (int64_t)t] = (uint16_t)j[0];
    }
  }
}

// d = 2 with bucket tables, one lane per path: the next layer's points staged
// in LDS (pairs, as in the time-layer kernels).  For paths counted on the spot,
// and for layers whose points walk_2d_wide cannot stage.
template <bool STORE>
__global__ __launch_bounds__(kBlock) void walk_2d(FwdArgs a, Visits v) {
  extern __shared__ float2 xy[];
  const uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool live = t < a.M;
  const uint32_t mc = (uint32_t)(a.m0 + (live ? t : 0));
  const uint32_t k0 = vgpr_copy(a.key0), k1 = vgpr_copy(a.key1);
  const float2* pts = reinterpret_cast<const float2*>(a.pts);  // x, y of point q at 2 q
  const float2 nan2 = make_float2(__builtin_nanf(""), __builtin_nanf(""));
  const LayerDev* layers = a.layers;
  float x[1][2] = {{layers[0].x0[0], layers[0].x0[1]}};
  float eb[4];
  int i = 0;
  for (int k = 0; k < a.n; ++k) {
    const int N1 = layers[k + 1].N, pt = layers[k + 1].pt_off;
    __syncthreads();  // the search of the step before
    for (int q = threadIdx.x; q <= N1; q += kBlock)
      xy[q] = q < N1 ? pts[2 * (pt + q)] : nan2;
    if ((k & 1) == 0) {
      const U4 r = philox4x32_10(U4{mc, (uint32_t)(k >> 1), a.contract, 1u}, k0, k1);
      box_muller(r.x, r.y, eb[0], eb[1]);
      box_muller(r.z, r.w, eb[2], eb[3]);
    }
    const LayerDev& L = a.layers[k];
    step_2d(L.A, L.T, L.b, (k & 1) ? eb[2] : eb[0], (k & 1) ? eb[3] : eb[1], x[0][0], x[0][1]);
    int j[1];
    uint4 w[1];
    bucket_rows<1>(layers[k + 1], N1, a.bk, x, w);
    __syncthreads();
    bucket_argmin<1, true>(xy, N1, a.bk, x, w, j);
    visit<STORE>(a, v, k, t, live, i, j[0]);
    i = j[0];
  }
}

// d = 2 without tables, d = 3: the full scan over the next layer's grid,
// staged in LDS at every step (the whole block walks the layers together).
template <int D, bool STORE, bool BK = false>
__global__ __launch_bounds__(kBlock) void walk_scan(FwdArgs a, Visits v) {
  extern __shared__ float4 g[];
  const uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool live = t < a.M;
  const uint32_t mc = (uint32_t)(a.m0 + (live ? t : 0));
  float x[D];
#pragma unroll
  for (int c = 0; c < D; ++c) x[c] = a.layers[0].x0[c];
  int i = 0;
  float eb[4];
  for (int k = 0; k < a.n; ++k) {
    const LayerDev& L = a.layers[k];
    const LayerDev& L1 = a.layers[k + 1];
    __syncthreads();
    for (int q = threadIdx.x; q < L1.N; q += kBlock) g[q] = a.pts[L1.pt_off + q];
    if (BK && threadIdx.x == 0) g[L1.N] = make_float4(0.f, 0.f, 0.f, __builtin_huge_valf());
    __syncthreads();
    float e[D];
    if (D == 2) {
      if ((k & 1) == 0) {
        const U4 r = philox4x32_10(U4{mc, (uint32_t)(k >> 1), a.contract, 1u}, a.key0, a.key1);
        box_muller(r.x, r.y, eb[0], eb[1]);
        box_muller(r.z, r.w, eb[2], eb[3]);
      }
      e[0] = eb[(k & 1) * 2];
      e[1] = eb[(k & 1) * 2 + 1];
    } else {
      const U4 r = philox4x32_10(U4{mc, (uint32_t)k, a.contract, 1u}, a.key0, a.key1);
      float unused;
      box_muller(r.x, r.y, e[0], e[1]);
      box_muller(r.z, r.w, e[D - 1], unused);
    }
    float y[1][D];
#pragma unroll
    for (int r = 0; r < D; ++r) {
      float z = L.b[r];
#pragma unroll
      for (int c = 0; c < D; ++c) z = fmaf(L.A[r * D + c], x[c], z);
#pragma unroll
      for (int c = 0; c < D; ++c) z = fmaf(L.T[r * D + c], e[c], z);
      y[0][r] = z;
    }
    int j;
    if constexpr (BK && D == 3) {
      uint4 w[1][2];
      cube_rows<1>(a.cubes[k + 1], a.cube_rows, y, w);
      cube_cells<1>(a.cubes[k + 1], g, y, w, &j);
    } else {
      argmin_scan<D, 1>(g, L1.N, y, &j);
    }
    visit<STORE>(a, v, k, t, live, i, j);
    i = j;
#pragma unroll
    for (int c = 0; c < D; ++c) x[c] = y[0][c];
  }
}

// Counting pass: workgroup = super tile (kSuper entries) of one layer's count
// block.  It reads the cells of every path on layers k and k + 1 (16 bytes, 8
// paths, at a time), counts the pairs that fall into its entries in LDS and
// stores them (adds them: first = 0).
__global__ __launch_bounds__(kCountBlock) void path_count(FwdArgs a, Visits v, int first) {
  __shared__ uint32_t hist[kSuper];
  // consecutive super tiles, which read the same cells, on one XCD (workgroup
  // b runs on XCD b mod 8)
  const int per = (int)((gridDim.x + 7) / 8);
  const int b = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (b >= a.total_tiles) return;
  int lo = 0, hi = a.n - 1;  // largest k with tile_off_k <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.layers[mid].tile_off <= b) lo = mid; else hi = mid - 1;
  }
  const LayerDev& L = a.layers[lo];
  const int64_t base = (int64_t)(b - L.tile_off) * kSuper;
  const int64_t left = (int64_t)L.N * L.N1 - base;
  const uint32_t bins = (uint32_t)(left < kSuper ? left : kSuper);
  const uint32_t N1 = (uint32_t)L.N1;
  for (uint32_t q = threadIdx.x; q < kSuper; q += kCountBlock) hist[q] = 0;
  __syncthreads();
  // keys fit 32 bits (at most kPathTiles super tiles a block): an entry before
  // base wraps past bins
  const uint32_t off = (uint32_t)base;
  const uint4* from = reinterpret_cast<const uint4*>(v.cells + (int64_t)(lo - 1) * v.stride);
  const uint4* to = reinterpret_cast<const uint4*>(v.cells + (int64_t)lo * v.stride);
  const uint32_t M = (uint32_t)a.M, vecs = (M + 7) / 8;
  for (uint32_t q = threadIdx.x; q < vecs; q += kCountBlock) {
    const uint4 zero = make_uint4(0, 0, 0, 0);
    const uint4 wi = lo > 0 ? from[q] : zero;  // layer 0 is one cell
    const uint4 wj = to[q];
    const uint32_t ii[4] = {wi.x, wi.y, wi.z, wi.w}, jj[4] = {wj.x, wj.y, wj.z, wj.w};
    const bool whole = 8 * q + 8 <= M;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t i = (ii[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
      const uint32_t j = (jj[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
      const uint32_t key = i * N1 + j - off;
      if (key < bins && (whole || 8 * q + (uint32_t)e < M)) atomicAdd(&hist[key], 1u);
    }
  }
  __syncthreads();
  int32_t* dst = a.counts + L.cnt_off + base;
  for (uint32_t q = threadIdx.x; q < bins; q += kCountBlock)
    dst[q] = (int32_t)hist[q] + (first ? 0 : dst[q]);
}

template <bool STORE>
static hipError_t launch_walk(const FwdArgs& a, const Visits& v, hipStream_t s) {
  const dim3 grid((unsigned)((a.M + kBlock - 1) / kBlock)), block(kBlock);
  auto go = [&](auto* kernel, size_t lds) {
    if (lds > 65536) {  // the default limit (gfx950 has 160 KiB per CU)
      const hipError_t e =
          hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, grid, block, lds, s, a, v);
    return hipGetLastError();
  };
  if (a.d == 1)
    return a.maxP <= kStageP ? go(walk_1d<true, STORE>, sizeof(float) * kStep * (size_t)a.maxP)
                          : go(walk_1d<false, STORE>, 0);
  if (a.d == 2 && a.bucketed && STORE && wide_lds(a.maxN) <= kLdsBytes) {
    const size_t lds = wide_lds(a.maxN);
    if (lds > 65536) {
      const hipError_t e =
          hipFuncSetAttribute(reinterpret_cast<const void*>(walk_2d_wide),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(walk_2d_wide, dim3((unsigned)((a.M + kWidePaths - 1) / kWidePaths)),
                       dim3(kWideBlock), lds, s, a, v);
    return hipGetLastError();
  }
  if (a.d == 2 && a.bucketed) return go(walk_2d<STORE>, sizeof(float2) * (size_t)(a.maxN + 1));
  const size_t lds = sizeof(float4) * (size_t)(a.maxN + 1);
  if (a.d == 3 && a.cubes) return go(walk_scan<3, STORE, true>, lds);
  return a.d == 2 ? go(walk_scan<2, STORE>, lds) : go(walk_scan<3, STORE>, lds);
}

hipError_t launch_fwd_path(const FwdArgs& a, hipStream_t s) {
  return launch_walk<false>(a, Visits{nullptr, 0}, s);
}

hipError_t launch_path_counts(const FwdArgs& a, uint16_t* cells, int64_t stride, bool first,
                              hipStream_t s) {
  const Visits v{cells, stride};
  hipError_t e = launch_walk<true>(a, v, s);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)((a.total_tiles + 7) / 8 * 8);
  hipLaunchKernelGGL(path_count, dim3(grid), dim3(kCountBlock), 0, s, a, v, first ? 1 : 0);
  return hipGetLastError();
}

}  // namespace qtree
