// Device-side sample construction and cell search shared by the forward
// kernels and the per-sample diagnostics.
#pragma once
#include "qtree_internal.hpp"
#include "qtree_rng.hpp"

namespace qtree {

// Number of midpoints strictly below x in a sorted array padded with +inf to
// 2^logP entries (2^logP >= N > number of real midpoints).
__device__ __forceinline__ int cell_1d(const float* mids, int logP, float x) {
  int c = 0;
  for (int s = (1 << logP) >> 1; s > 0; s >>= 1) {
    c = (mids[c + s - 1] < x) ? c + s : c;
  }
  return c;
}

// Breadth-first (Eytzinger) order of the 2^LOGP padded midpoints of a layer:
// node i (1 <= i < 2^LOGP) at depth t = floor(log2 i) holds the sorted
// midpoint (2 (i - 2^t) + 1) 2^(LOGP-t-1) - 1, so binary lifting from the
// root visits the same midpoints as cell_1d.  Nodes of one depth are
// adjacent in LDS: the lanes of a wave at a shallow depth read a few
// consecutive words instead of words one power of two apart (which share a
// bank).  Slot 0 is unused.
template <int LOGP>
__device__ __forceinline__ int bfs_source(int i) {
  const int t = 31 - __clz(i);
  return ((2 * (i - (1 << t)) + 1) << (LOGP - t - 1)) - 1;
}

// cell_1d over a breadth-first LDS copy, the depth fixed at compile time:
// i <- 2 i + (e_i < x) from the root, count = i - 2^LOGP.  The comparison is
// the sign bit of e_i - x, which equals (e_i < x) for every finite x and
// every midpoint that is +inf or finite and not -0 (zero midpoints are stored
// as +0): with denormals kept the difference of two distinct floats never
// rounds to zero, and m - m = +0.  The LDS address a = base + 4 i is carried:
// the child's address is 2 a + (4 b - base), b the sign bit.  A step after
// the load is five vector operations (subtract, arithmetic shift, and, add,
// and one shift-add, the only half-rate one) instead of a compare and a
// select; they form one asm block so that the compiler keeps these forms and
// puts no wait states between them (plain VALU dependences interlock).
template <int LOGP>
__device__ __forceinline__ int cell_1d_bfs(const float* e, float x) {
  typedef __attribute__((address_space(3))) const float lds_float;
  const uint32_t base = (uint32_t)(uintptr_t)(lds_float*)e;
  const uint32_t nbase = vgpr_copy(0u - base);
  uint32_t addr = base + 4;
#pragma unroll
  for (int t = 0; t < LOGP; ++t) {
    const float m = *(lds_float*)(uintptr_t)addr;
    uint32_t tmp;
    asm("v_sub_f32_e32 %[t], %[m], %[x]\n\t"
        "v_ashrrev_i32_e32 %[t], 31, %[t]\n\t"
        "v_and_b32_e32 %[t], 4, %[t]\n\t"
        "v_add_u32_e32 %[t], %[t], %[nb]\n\t"
        "v_lshl_add_u32 %[a], %[a], 1, %[t]"
        : [a] "+v"(addr), [t] "=&v"(tmp)
        : [m] "v"(m), [x] "v"(x), [nb] "v"(nbase));
  }
  return (int)((addr - base) >> 2) - (1 << LOGP);
}

// cell_1d by a guide table: bucket b = (int)clamp(fma(x, scale, shift), 0,
// B - 1) (bmax = B - 1), then c = tab[b] + #{r < K : m[tab[b] + r] < x}.
// Exact when tab[b] counts the midpoints below the first float of bucket b
// and K bounds the midpoints inside any bucket (the host builds both from
// the same float formula), with m padded by K entries of +inf.  The clamp is
// one median-of-three (x is finite, so it equals max then min); each
// comparison is the sign bit of m - x (subtract, shift: full-rate
// operations, where a compare and select issue at half rate).  Written as
// plain arithmetic, the searches of neighbouring samples are free to be
// scheduled together: the compiler issues the table reads of several samples,
// then their paired candidate reads, before the first wait.
template <int K>
__device__ __forceinline__ int cell_1d_guide(const float* m, const uint16_t* tab, float scale,
                                             float shift, float bmax, float x) {
  const float t = __builtin_amdgcn_fmed3f(fmaf(x, scale, shift), 0.0f, bmax);
  const int c0 = tab[(int)t];
  int c = c0;
#pragma unroll
  for (int r = 0; r < K; ++r) c += (int)(__float_as_uint(m[c0 + r] - x) >> 31);
  return c;
}

// X_k = mu + L z and X_{k+1} = b + A X_k + T eps, row by row, left-to-right
// chains of fused multiply-adds (the AR(1) proposition of Sec. 3).
template <int D>
__device__ __forceinline__ void layer_pair(const LayerDev& L, const float* z, const float* e,
                                           float* x, float* y) {
#pragma unroll
  for (int r = 0; r < D; ++r) {
    float v = L.mu[r];
#pragma unroll
    for (int c = 0; c < D; ++c) v = fmaf(L.L[r * D + c], z[c], v);
    x[r] = v;
  }
#pragma unroll
  for (int r = 0; r < D; ++r) {
    float v = L.b[r];
#pragma unroll
    for (int c = 0; c < D; ++c) v = fmaf(L.A[r * D + c], x[c], v);
#pragma unroll
    for (int c = 0; c < D; ++c) v = fmaf(L.T[r * D + c], e[c], v);
    y[r] = v;
  }
}

// Argmin over N grid records (g_0..g_{D-1}, h) of h - <x, g>, lowest index on
// ties, for S query points at once.
template <int D, int S>
__device__ __forceinline__ void argmin_scan(const float4* __restrict__ g, int N,
                                            const float (*xs)[D], int* idx) {
  float best[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    best[s] = __builtin_huge_valf();
    idx[s] = 0;
  }
  for (int p = 0; p < N; ++p) {
    const float4 q = g[p];
    const float gc[3] = {q.x, q.y, q.z};
#pragma unroll
    for (int s = 0; s < S; ++s) {
      float key = q.w;
#pragma unroll
      for (int c = 0; c < D; ++c) key = fmaf(-xs[s][c], gc[c], key);
      const bool lt = key < best[s];
      best[s] = lt ? key : best[s];
      idx[s] = lt ? p : idx[s];
    }
  }
}

// The same argmin, by tiles of TL records: a running minimum per tile
// (fminf chains -> v_min3_f32) and only the index of the first tile whose
// minimum is strictly smaller than the best so far; the winning tile is then
// rescanned for the first record whose key equals the minimum.  Bit-identical
// to argmin_scan (same keys, lowest index among the minimal ones).  The
// record array must be padded to a multiple of TL with records whose key is
// +inf for every x (g = 0, h = +inf).
template <int D, int S, int TL>
__device__ __forceinline__ void argmin_scan_tiled(const float4* __restrict__ g, int Npad,
                                                  const float (*xs)[D], int* idx) {
  float best[S];
  int tile[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    best[s] = __builtin_huge_valf();
    tile[s] = 0;
  }
  // the records of the next tile are loaded while the current one is
  // scanned (the last iteration reloads its own tile, which stays in bounds)
  float4 cur[TL];
#pragma unroll
  for (int q = 0; q < TL; ++q) cur[q] = g[q];
  for (int p0 = 0; p0 < Npad; p0 += TL) {
    float4 nxt[TL];
    const int pn = p0 + TL < Npad ? p0 + TL : p0;
#pragma unroll
    for (int q = 0; q < TL; ++q) nxt[q] = g[pn + q];
    float m[S];
#pragma unroll
    for (int s = 0; s < S; ++s) m[s] = __builtin_huge_valf();
#pragma unroll
    for (int q = 0; q < TL; ++q) {
      const float4 r = cur[q];
      const float gc[3] = {r.x, r.y, r.z};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        float key = r.w;
#pragma unroll
        for (int c = 0; c < D; ++c) key = fmaf(-xs[s][c], gc[c], key);
        m[s] = fminf(m[s], key);
      }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const bool lt = m[s] < best[s];
      best[s] = lt ? m[s] : best[s];
      tile[s] = lt ? p0 : tile[s];
    }
#pragma unroll
    for (int q = 0; q < TL; ++q) cur[q] = nxt[q];
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    int found = tile[s] + TL - 1;
    // rolled: unrolled, the loads of every record of every sample's tile
    // would be hoisted together (TL x S float4 registers)
#pragma unroll 1
    for (int q = TL - 1; q >= 0; --q) {
      const float4 r = g[tile[s] + q];
      const float gc[3] = {r.x, r.y, r.z};
      float key = r.w;
#pragma unroll
      for (int c = 0; c < D; ++c) key = fmaf(-xs[s][c], gc[c], key);
      found = key == best[s] ? tile[s] + q : found;
    }
    idx[s] = found;
  }
}

// The full scan for the lanes of `need`, one after the other, each by the
// whole wave (the points split over its lanes): a lane scanning alone holds its
// workgroup up for 15 us at N = 990, the wave for less than one.  key(p, x) is
// the key of point p at x; the result is idx for the other lanes.  (All lanes
// of the wave come here together.)
template <int D, class KEY>
__device__ __forceinline__ int wave_scan(KEY key, int N, const float* x, uint64_t need, int idx) {
  const int lane = (int)(threadIdx.x & 63);
  while (need) {
    const int from = __ffsll((unsigned long long)need) - 1;
    need &= need - 1;
    float q[D];
#pragma unroll
    for (int c = 0; c < D; ++c) q[c] = __shfl(x[c], from, 64);
    float best = __builtin_huge_valf();
    int at = 0x7FFFFFFF;
#pragma unroll(D == 3 ? 2 : 1)
    for (int p = lane; p < N; p += 64) {
      const float v = key(p, q);
      const bool lt = v < best;
      best = lt ? v : best;
      at = lt ? p : at;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float o = __shfl_xor(best, off, 64);
      const int oat = __shfl_xor(at, off, 64);
      const bool lt = o < best || (o == best && oat < at);
      best = lt ? o : best;
      at = lt ? oat : at;
    }
    if (at == 0x7FFFFFFF) at = 0;  // no key below +inf
    idx = lane == from ? at : idx;
  }
  return idx;
}
constexpr int kWaveScans = 16;  // more lanes than this scan side by side

// d = 2 cells by the layer's bucket tables, in two steps so that the row
// loads of many points are in flight together.  A bucket's row (16 bytes)
// holds its candidate count c in entry 0 and, from entry 1 on, every point
// that can be the FP32 argmin of h - <x, g> anywhere in the bucket, in
// increasing index, then pads; more than kBucketCap of them are in a row of
// the pool.  The first minimum over the list is the full scan's cell (the
// lowest index of the minimal key).  Outside the box, in a bucket whose
// candidates did not fit (c = kBucketFull), or in a layer without tables, the
// full scan over the N points decides.
//
// The points are (x, y) pairs in LDS, 8 bytes each, with a pad pair (NaN,
// NaN) at index N: its key is NaN, which never wins a comparison, and the
// lanes that read it share one LDS access.  Entries are byte offsets of the
// pairs, and so is the cell (cell_index gives its index).  Consecutive points
// fall in different bank pairs, where 16-byte records would share a quarter
// of the banks (and 12-byte (x, y, h) triples take two reads).  The half norm
// is recomputed as h = (x x + y y) / 2 with one product, one fma and one
// halving, the order in which the records' own half norms are formed, so
// the key is bit for bit the scan's.
__device__ __forceinline__ float half_norm_key(float2 r, float x0, float x1) {
  const float h = 0.5f * fmaf(r.y, r.y, r.x * r.x);
  return fmaf(-x1, r.y, fmaf(-x0, r.x, h));
}

__device__ __forceinline__ int cell_index(int offset) { return offset >> 3; }

// The bucket of a point (FP32) in a layer's tables, -1 outside the box, for
// NaN and for a layer without tables (bk_B = 0).
template <class LAYER>
__device__ __forceinline__ int bucket_of(LAYER& L, float x0, float x1) {
  const float f0 = (x0 - L.bk_lo[0]) * L.bk_scale[0];
  const float f1 = (x1 - L.bk_lo[1]) * L.bk_scale[1];
  const bool in = f0 >= 0.0f && f1 >= 0.0f && f0 < (float)L.bk_B[0] && f1 < (float)L.bk_B[1];
  return in ? L.bk_off + (int)f0 * L.bk_B[1] + (int)f1 : -1;
}

// bucket_rows: the row of each of S points in a layer of N points; pads and
// the count kBucketFull where it has none (every point loads a row, row 0
// then, so that the load is not under a branch and all S stay in flight).
template <int S, class LAYER>
__device__ __forceinline__ void bucket_rows(LAYER& L, int N, const BucketTab& t,
                                            const float (*xs)[2], uint4* w) {
  const uint32_t pads = 8u * (uint32_t)N * 0x10001u;
  int r[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    r[s] = bucket_of(L, xs[s][0], xs[s][1]);
    w[s] = t.rows[(uint32_t)max(r[s], 0)];
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    w[s].x = r[s] < 0 ? pads | 0xFFFFu : w[s].x;
    w[s].y = r[s] < 0 ? pads : w[s].y;
    w[s].z = r[s] < 0 ? pads : w[s].z;
  }
}

// Entry e of 8.
__device__ __forceinline__ int bucket_entry(const uint4& w, int e) {
  const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
  return (int)((e & 1) ? ww[e >> 1] >> 16 : ww[e >> 1] & 0xFFFFu);
}
__device__ __forceinline__ float bucket_key(const float2* __restrict__ g, int at, float x0,
                                            float x1) {
  return half_norm_key(*reinterpret_cast<const float2*>(reinterpret_cast<const char*>(g) + at), x0,
                       x1);
}

// Entries e0 .. 7 (candidates or pads).
__device__ __forceinline__ void bucket_group(const float2* __restrict__ g, const uint4& w, int e0,
                                             float x0, float x1, float& best, int& at) {
#pragma unroll
  for (int e = e0; e < 8; ++e) {
    const int p = bucket_entry(w, e);
    const float key = bucket_key(g, p, x0, x1);
    const bool lt = key < best;
    best = lt ? key : best;
    at = lt ? p : at;
  }
}

// bucket_first: the minimum over the first kFirst candidates of each of S
// points' rows, in straight-line code so that the LDS reads of all S points
// can be in flight together.  The first entry is always a candidate of a
// listed row.  (Cells meet at most four at a time on the usual grids, and of
// a wave's 64 points one lies near such a corner in most rounds: with three,
// the branch for the fourth was taken almost always.)
constexpr int kFirst = 4;
template <int S>
__device__ __forceinline__ void bucket_first(const float2* __restrict__ g, const float (*xs)[2],
                                             const uint4* w, int* at) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    at[s] = bucket_entry(w[s], 1);
    float best = bucket_key(g, at[s], xs[s][0], xs[s][1]);
#pragma unroll
    for (int e = 2; e <= kFirst; ++e) {
      const int p = bucket_entry(w[s], e);
      const float key = bucket_key(g, p, xs[s][0], xs[s][1]);
      const bool lt = key < best;
      best = lt ? key : best;
      at[s] = lt ? p : at[s];
    }
  }
}

// bucket_rest: the rows of more candidates from their start, and the full
// scan; at then holds the cells.  A lane that scans alone waits for the LDS,
// eight points at a time (two samples a lane: four): 2500 points on a line, 1000
// and 10^5 paths of 12 steps 870 and 920 us, 1060 and 1096 with four.  WAVE: up
// to kWaveScans lanes without a list are scanned for by their wave (all of it
// comes here together).  That is for a caller's points, which may be outside the
// box (10^5 of them, a grid of 900 points on a circle 629 -> 34 us), and for paths,
// whose waves are few (1000 on five rows of 500 points 1072 -> 189; 365 layers
// whose lists answer 444 and 443); the time layers' samples hardly are outside,
// and the question alone would cost them 0.4 % of a call.
template <int S, bool WAVE = false>
__device__ __forceinline__ void bucket_rest(const float2* __restrict__ g, int N,
                                            const BucketTab& t, const float (*xs)[2],
                                            const uint4* w, int* at) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t c = w[s].x & 0xFFFFu;
    uint64_t alone = 0;
    if (WAVE) {
      alone = __ballot(c == (uint32_t)kBucketFull);
      if (__popcll(alone) > kWaveScans) alone = 0;
      if (alone != 0)
        at[s] = 8 * wave_scan<2>(
                        [&](int p, const float* q) { return half_norm_key(g[p], q[0], q[1]); }, N,
                        xs[s], alone, cell_index(at[s]));
    }
    if (c <= (uint32_t)kFirst) continue;
    float best = __builtin_huge_valf();
    int found = 0;
    if (c <= (uint32_t)kBucketCap) {
      bucket_group(g, w[s], 1, xs[s][0], xs[s][1], best, found);
    } else if (c == kBucketLong) {
      const uint4* row = t.longs + (size_t)w[s].w * (kLongRow / 8);
      const int cl = (int)(row[0].x & 0xFFFFu);
      bucket_group(g, row[0], 1, xs[s][0], xs[s][1], best, found);
      for (int q = 8; q <= cl; q += 8)
        bucket_group(g, row[q >> 3], 0, xs[s][0], xs[s][1], best, found);
    } else {
      if (alone != 0) continue;
#pragma unroll(S == 2 ? 4 : 8)
      for (int p = 0; p < 8 * N; p += 8) {
        const float key = bucket_key(g, p, xs[s][0], xs[s][1]);
        const bool lt = key < best;
        best = lt ? key : best;
        found = lt ? p : found;
      }
    }
    at[s] = found;
  }
}

// bucket_argmin: the cells of the S points whose rows bucket_rows fetched.
template <int S, bool WAVE = false>
__device__ __forceinline__ void bucket_argmin(const float2* __restrict__ g, int N,
                                              const BucketTab& t, const float (*xs)[2],
                                              const uint4* w, int* idx) {
  bucket_first<S>(g, xs, w, idx);
  bucket_rest<S, WAVE>(g, N, t, xs, w, idx);
#pragma unroll
  for (int s = 0; s < S; ++s) idx[s] = cell_index(idx[s]);
}

// d = 3 cells by the layer's bucket tables (rows at Cubes): the first minimum
// over the bucket's list, the full scan's cell.  g holds the layer's records
// and, at N, a pad whose key is +inf and wins no comparison; the entries are
// taken in groups of 4, 4 and 7 (cells of a product grid meet at most eight at
// a time).  Outside the box, for NaN, in a full bucket and in a layer without
// tables the scan over the N records decides.
__device__ __forceinline__ float record_key(const float4& r, const float* x) {
  return fmaf(-x[2], r.z, fmaf(-x[1], r.y, fmaf(-x[0], r.x, r.w)));
}
__device__ __forceinline__ int cube_of(const Cubes& C, const float* x) {
  float f[3];
  bool in = true;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    f[r] = (x[r] - C.lo[r]) * C.scale[r];
    in = in && f[r] >= 0.0f && f[r] < (float)C.B[r];
  }
  return in ? C.off + ((int)f[0] * C.B[1] + (int)f[1]) * C.B[2] + (int)f[2] : -1;
}
template <int E0, int E1>
__device__ __forceinline__ void cube_group(const float4* g, const uint4* w, const float* x,
                                           float& best, int& idx) {
#pragma unroll
  for (int e = E0; e < E1; ++e) {
    const int p = bucket_entry(w[e >> 3], e & 7);
    const float key = record_key(g[p], x);
    const bool lt = key < best;
    best = lt ? key : best;
    idx = lt ? p : idx;
  }
}
// The rows of S points (row 0 where there is none, so that the loads are not
// under a branch), then their cells.
template <int S>
__device__ __forceinline__ void cube_rows(const Cubes& C, const uint4* rows, const float (*xs)[3],
                                          uint4 (*w)[2]) {
  int r[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    r[s] = cube_of(C, xs[s]);
    const uint4* row = rows + 2 * (size_t)max(r[s], 0);
    w[s][0] = row[0];
    w[s][1] = row[1];
  }
  const uint32_t pads = (uint32_t)C.N * 0x10001u;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    w[s][0].x = r[s] < 0 ? pads | 0xFFFFu : w[s][0].x;
    w[s][0].y = r[s] < 0 ? pads : w[s][0].y;
    w[s][0].z = r[s] < 0 ? pads : w[s][0].z;
  }
}
// (All lanes of the wave come here together.)
template <int S>
__device__ __forceinline__ void cube_cells(const Cubes& C, const float4* g, const float (*xs)[3],
                                           const uint4 (*w)[2], int* idx) {
  const int N = C.N;
  if (C.B[0] == 0) {  // the layer has no tables
    argmin_scan<3, S>(g, N, xs, idx);
    return;
  }
  float best[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    best[s] = __builtin_huge_valf();
    idx[s] = 0;
    cube_group<1, 5>(g, w[s], xs[s], best[s], idx[s]);
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t c = w[s][0].x & 0xFFFFu;
    if (c > 4 && c != kCubeFull) {
      cube_group<5, 9>(g, w[s], xs[s], best[s], idx[s]);
      if (c > 8) cube_group<9, 16>(g, w[s], xs[s], best[s], idx[s]);
    }
    const uint64_t need = __ballot(c == kCubeFull);
    if (need == 0) continue;
    if (__popcll(need) <= kWaveScans) {
      idx[s] = wave_scan<3>([&](int p, const float* q) { return record_key(g[p], q); }, N, xs[s],
                            need, idx[s]);
    } else if (c == kCubeFull) {
      argmin_scan<3, 1>(g, N, xs + s, idx + s);
    }
  }
}

// Standard normals z (for X_k) and eps (for the innovation) of LAYERWISE
// sample m of layer k.  Philox counter (block, k, contract, tag): d = 1 uses
// block m >> 1 and the Box-Muller pair m & 1; d = 2 block m; d = 3 blocks
// (m, tag 0) and (m, tag 16).
template <int D>
__device__ __forceinline__ void layer_normals(uint32_t key0, uint32_t key1, uint32_t contract,
                                              int k, uint64_t m, float* z, float* e) {
  if (D == 1) {
    const U4 r = philox4x32_10(U4{(uint32_t)(m >> 1), (uint32_t)k, contract, 0u}, key0, key1);
    if (m & 1) box_muller(r.z, r.w, z[0], e[0]);
    else box_muller(r.x, r.y, z[0], e[0]);
  } else if (D == 2) {
    const U4 r = philox4x32_10(U4{(uint32_t)m, (uint32_t)k, contract, 0u}, key0, key1);
    box_muller(r.x, r.y, z[0], z[1]);
    box_muller(r.z, r.w, e[0], e[1]);
  } else {
    const U4 r = philox4x32_10(U4{(uint32_t)m, (uint32_t)k, contract, 0u}, key0, key1);
    box_muller(r.x, r.y, z[0], z[1]);
    box_muller(r.z, r.w, z[2], e[0]);
    const U4 r2 = philox4x32_10(U4{(uint32_t)m, (uint32_t)k, contract, 16u}, key0, key1);
    box_muller(r2.x, r2.y, e[1], e[2]);
  }
}

}  // namespace qtree
