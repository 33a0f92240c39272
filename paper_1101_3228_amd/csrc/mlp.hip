// Pricing-surrogate kernels for gfx950: inference, forward and back-propagation
// of a training tile in one kernel, the weight gradients of the two 256x256
// layers as an MFMA reduction over the batch, the remaining sums, and Adam
// with the refresh of the BF16 weight copies.
//
// MFMA mapping.  A tile is 32 samples.  A 256x256 layer is computed as
// Z^T = W H^T with the weights as the A operand (rows = output units) and
// the activations as the B operand (columns = samples), 8 output blocks x
// 16 K-steps of v_mfma_f32_32x32x16_bf16.  Lane l holds accumulator r of
// output block jb for unit 32 jb + 8 (r / 4) + 4 (l / 32) + r % 4 and sample
// l % 32.  The K order inside a dot product is free, so K-step t is defined
// to take, for lane half h and element e, the unit
//     unit(t, h, e) = 32 (t / 2) + 16 (t % 2) + 8 (e / 4) + 4 h + e % 4,
// which is exactly accumulator r = 8 (t % 2) + e of block t / 2 of the lane:
// a layer's output, once activated, is the next layer's B operand without
// leaving the registers.  The weights are stored pre-permuted to match
// (fragment (ib, t) of lane l = W[32 ib + l % 32][unit(t, l / 32, e)],
// e = 0..7, 16 contiguous bytes per lane).
//
// Layer 1 (6 inputs) is one K-step per output block as well: the 16 K-slots
// hold the normalised inputs as two BF16 terms, (u_hi[0..5], u_lo[0..5], 0 x4)
// for lane halves h = 0 (slots 0..7) and h = 1 (slots 8..15), against
// (W1[i][0..5], W1[i][0..5], 0 x4); the accumulators start from the biases.
#include <hip/hip_runtime.h>

#include "qtree_mlp_internal.hpp"

namespace qtree {
namespace mlp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

__device__ __forceinline__ float silu(float z) {
  return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}

__device__ __forceinline__ float dsilu(float z) {
  const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-z));
  return s * fmaf(z, 1.0f - s, 1.0f);
}

__device__ __forceinline__ uint16_t bf16_bits(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ float bf16_float(uint16_t b) {
  return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// Position of W1[i][c] in the layer-1 fragments: K-slot c (hi term) and
// K-slot 6 + c (lo term); slot s lives in lane half s / 8, element s % 8.
__host__ __device__ __forceinline__ int frag1_index(int i, int slot) {
  return (((i >> 5) * 64) + 32 * (slot >> 3) + (i & 31)) * 8 + (slot & 7);
}

// Index of W[i][k] in the fragment layout described at the top.
__host__ __device__ __forceinline__ int frag_index(int i, int k) {
  const int t = 2 * (k >> 5) + ((k >> 4) & 1);
  const int rem = k & 15;
  const int e = 4 * (rem >> 3) + (rem & 3);
  const int lane = 32 * ((rem >> 2) & 1) + (i & 31);
  return (((i >> 5) * 16 + t) * 64 + lane) * 8 + e;
}

// The 16 accumulators of an output block (already activated) as the B
// operands of its two K-steps, in TERMS BF16 parts.
template <int TERMS>
__device__ __forceinline__ void operand_pair(const float (&v)[16], bf16x8 (&one)[TERMS][2]) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const __bf16 p = (__bf16)v[8 * k + e];
      one[0][k][e] = p;
      if (TERMS == 2) one[TERMS - 1][k][e] = (__bf16)(v[8 * k + e] - (float)p);
    }
}

__device__ __forceinline__ int unit_of(int jb, int r, int h) {
  return 32 * jb + 8 * (r >> 2) + 4 * h + (r & 3);
}

// Elements of a tile (32 samples) of a per-unit training array: accumulator r
// of block jb of a lane is at (16 jb + r) 64 + lane.
constexpr int kWaveTile = 8 * 16 * 64;

// Tile-layout offset of (unit, sample s) (for kernels that walk units).
__device__ __forceinline__ int64_t tile_index(int unit, int64_t s) {
  const int u = unit & 31;
  const int r = 4 * (u >> 3) + (u & 3);
  const int h = (u >> 2) & 1;
  return (s >> 5) * kWaveTile + ((unit >> 5) * 16 + r) * 64 + 32 * h + (s & 31);
}

// Black-Scholes European put per unit strike on (S0/K, sigma, r, T).
__device__ __forceinline__ float bs_put(float s, float sig, float r, float T) {
  const float v = sig * sqrtf(T);
  const float d1 = (logf(s) + (r + 0.5f * sig * sig) * T) / v;
  const float d2 = d1 - v;
  return expf(-r * T) * 0.5f * erfcf(d2 * 0.70710678f) - s * 0.5f * erfcf(d1 * 0.70710678f);
}

// Inputs of row `row` (dead rows: the box's lower corner, u = 0): u the
// normalised ones, raw the first four; whether all lie in the box.
__device__ __forceinline__ bool normalise(const Weights& W, const float* __restrict__ x,
                                          int64_t row, bool live, float (&u)[kIn],
                                          float (&raw)[4]) {
  bool inside = true;
#pragma unroll
  for (int c = 0; c < kIn; ++c) {
    const float xv = live ? x[row * kIn + c] : W.lo[c];
    if (c < 4) raw[c] = xv;
    inside = inside && xv >= W.lo[c] && xv <= W.hi[c];
    u[c] = live ? fmaf(xv - W.lo[c], W.scale[c], W.shift[c]) : 0.0f;
  }
  return inside;
}

// Layer 1's B operand: the inputs as two BF16 terms in the 16 K-slots.
__device__ __forceinline__ bf16x8 input_operand(const float (&u)[kIn], int h) {
  float q[16];
#pragma unroll
  for (int c = 0; c < kIn; ++c) {
    const __bf16 a = (__bf16)u[c];
    q[c] = (float)a;
    q[kIn + c] = (float)(__bf16)(u[c] - (float)a);
  }
#pragma unroll
  for (int c = 2 * kIn; c < 16; ++c) q[c] = 0.0f;
  bf16x8 ub;
#pragma unroll
  for (int e = 0; e < 8; ++e) ub[e] = (__bf16)(h ? q[8 + e] : q[e]);
  return ub;
}

// The network's output from the head's sum.
__device__ __forceinline__ float output(const Weights& W, float part, bool base,
                                        const float (&raw)[4]) {
  float y = W.out_scale * (part + W.master[kOffB4]);
  if (W.baseline && base) y += bs_put(raw[0], raw[1], raw[2], raw[3]);
  return y;
}

struct FwdIO {
  const float* x;
  int64_t B;
  float* y;
  uint8_t* in_range;
};

// Eight waves share the 32 samples of a tile: wave ib computes output block
// ib of every layer (32 units), and the activations pass through LDS as the
// next layer's B operands.  A wave that owned a tile and all eight blocks read
// every weight from L2 for 32 samples (8.5 TB at 1e6 queries, 0.59 ms), and
// put a batch of 4096 on 32 CUs, each in a chain of 256 products and 768
// activations per lane (forward 89 us, backward 159 us; a single query 38 us).

constexpr int kTileBlock = 512;
constexpr int kOps = 16 * 64;  // B operands of a layer (one term)
constexpr int64_t kCus = 256;  // workgroups that hold the weights: one per CU

// The 16 activations of this wave's block as B operands of K-steps 2 ib, 2 ib
// + 1, in TERMS BF16 parts: ops[term][t][lane].
template <int TERMS>
__device__ __forceinline__ void share_operand(const float (&v)[16], bf16x8* ops, int ib, int lane) {
  bf16x8 one[TERMS][2];
  operand_pair<TERMS>(v, one);
#pragma unroll
  for (int q = 0; q < TERMS; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) ops[q * kOps + (2 * ib + e) * 64 + lane] = one[q][e];
}

// This wave's 16 weight fragments of a layer, and their product with ops.
__device__ __forceinline__ void load_frags(const uint16_t* __restrict__ frags, int ib, int lane,
                                           bf16x8 (&f)[16]) {
  const bf16x8* wf = reinterpret_cast<const bf16x8*>(frags);
#pragma unroll
  for (int t = 0; t < 16; ++t) f[t] = wf[(ib * 16 + t) * 64 + lane];
}
template <int TERMS>
__device__ __forceinline__ f32x16 tile_layer(const bf16x8 (&f)[16], const bf16x8* ops, int lane) {
  f32x16 acc = f32x16{};
#pragma unroll
  for (int t = 0; t < 16; ++t)
#pragma unroll
    for (int q = 0; q < TERMS; ++q)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[t], ops[q * kOps + t * 64 + lane], acc, 0, 0,
                                                    0);
  return acc;
}

// Four values of this lane's units 32 ib + 8 g + 4 h .. + 3 for g = 0..3.
__device__ __forceinline__ void load_units(const float* __restrict__ p, int ib, int h,
                                           float (&v)[16]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float4 q = *reinterpret_cast<const float4*>(p + unit_of(ib, 4 * g, h));
    v[4 * g] = q.x;
    v[4 * g + 1] = q.y;
    v[4 * g + 2] = q.z;
    v[4 * g + 3] = q.w;
  }
}

// This wave's part of the head, sum of w4 h3 over its 32 units, for the
// samples lane % 32 (in both lane halves).
__device__ __forceinline__ float head_part(const float (&w4)[16], const float (&h3)[16]) {
  float part = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) part = fmaf(w4[r], h3[r], part);
  return part + __shfl_xor(part, 32);
}

// Inference, one tile per workgroup (batches of up to a tile per CU).
template <int TERMS>
__global__ __launch_bounds__(kTileBlock) void mlp_forward(Weights W, FwdIO io) {
  extern __shared__ bf16x8 lds[];  // [2][TERMS][kOps]
  __shared__ float head[kTileBlock / 64][kWaveRows];
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int ib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  bf16x8* const opsA = lds;
  bf16x8* const opsB = lds + TERMS * kOps;
  const int64_t s = (int64_t)blockIdx.x * kWaveRows + (lane & 31);
  const bool live = s < io.B;
  float u[kIn], raw[4], b[16], w4[16], v[16];
  bf16x8 f2[16], f3[16];
  const bool inside = normalise(W, io.x, s, live, u, raw);
  load_frags(W.w2f, ib, lane, f2);
  load_units(W.master + kOffB1, ib, h, b);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = b[r];
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
      reinterpret_cast<const bf16x8*>(W.w1)[ib * 64 + lane], input_operand(u, h), acc, 0, 0, 0);
  load_frags(W.w3f, ib, lane, f3);
  load_units(W.master + kOffB2, ib, h, b);
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = silu(acc[r]);
  share_operand<TERMS>(v, opsA, ib, lane);
  __syncthreads();
  acc = tile_layer<TERMS>(f2, opsA, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = silu(acc[r] + b[r]);
  share_operand<TERMS>(v, opsB, ib, lane);
  load_units(W.master + kOffB3, ib, h, b);
#pragma unroll
  for (int r = 0; r < 16; ++r) w4[r] = bf16_float(W.w4[unit_of(ib, r, h)]);
  __syncthreads();
  acc = tile_layer<TERMS>(f3, opsB, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = silu(acc[r] + b[r]);
  const float part = head_part(w4, v);
  if (h == 0) head[ib][lane] = part;
  __syncthreads();
  if (ib != 0 || h != 0 || !live) return;
  float sum = 0.0f;
#pragma unroll
  for (int w = 0; w < kTileBlock / 64; ++w) sum += head[w][lane];
  io.y[s] = output(W, sum, inside, raw);
  if (io.in_range) io.in_range[s] = inside ? 1 : 0;
}

// Inference, large batches.  A workgroup keeps the weight fragments of layers
// 2 and 3 in registers (128 of them) and goes through its share of the batch
// two tiles at a time, two barriers a turn.  The outputs of a turn are finished
// by one wave, another each time, after the next turn's first barrier.
//
// 1e6 queries: 366 us a call with one activation term, 13.6 k clocks a turn of
// 64 samples; the exponentials and reciprocals of SiLU (6.1 k), the matrix cores
// (4.2 k) and the LDS reads of the operands (4.1 k) follow one another.  One
// tile's products interleaved with the other's SiLU by the scheduler's
// groups, at a barrier per product, is slower: 360 against 345 us where the two
// were compared, launches back to back.
constexpr int S = 2;
template <int TERMS>
__global__ __launch_bounds__(kTileBlock) void mlp_forward_pairs(Weights W, FwdIO io,
                                                                int64_t groups) {
  extern __shared__ bf16x8 lds[];  // [2][S][TERMS][kOps]
  __shared__ float head[S][kTileBlock / 64][kWaveRows];
  constexpr int kBuf = TERMS * kOps;
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int ib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  bf16x8* const opsA = lds;
  bf16x8* const opsB = lds + S * kBuf;
  const bf16x8 f1 = reinterpret_cast<const bf16x8*>(W.w1)[ib * 64 + lane];
  bf16x8 f2[16], f3[16];
  load_frags(W.w2f, ib, lane, f2);
  load_frags(W.w3f, ib, lane, f3);
  float b1[16], b2[16], b3[16], w4[16];
  load_units(W.master + kOffB1, ib, h, b1);
  load_units(W.master + kOffB2, ib, h, b2);
  load_units(W.master + kOffB3, ib, h, b3);
#pragma unroll
  for (int r = 0; r < 16; ++r) w4[r] = bf16_float(W.w4[unit_of(ib, r, h)]);
  // samples 32 S g .. of group g: lanes 0 .. 32 S - 1 of the wave whose turn it is
  auto finish = [&](int64_t g) {
    if (lane >= kWaveRows * S) return;
    const int64_t s = g * (kWaveRows * S) + lane;
    if (s >= io.B) return;
    float u[kIn], raw[4];
    const bool inside = normalise(W, io.x, s, true, u, raw);
    float part = 0.0f;
#pragma unroll
    for (int w = 0; w < kTileBlock / 64; ++w) part += head[lane >> 5][w][lane & 31];
    io.y[s] = output(W, part, inside, raw);
    if (io.in_range) io.in_range[s] = inside ? 1 : 0;
  };
  int turn = 0;
  int64_t g = blockIdx.x;
  for (; g < groups; g += gridDim.x, ++turn) {
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const int64_t s = (g * S + q) * kWaveRows + (lane & 31);
      float u[kIn], raw[4], v[16];
      normalise(W, io.x, s, s < io.B, u, raw);
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = b1[r];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1, input_operand(u, h), acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = silu(acc[r]);
      share_operand<TERMS>(v, opsA + q * kBuf, ib, lane);
    }
    __syncthreads();
    if (turn > 0 && ib == (turn & 7)) finish(g - gridDim.x);
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const f32x16 acc = tile_layer<TERMS>(f2, opsA + q * kBuf, lane);
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = silu(acc[r] + b2[r]);
      share_operand<TERMS>(v, opsB + q * kBuf, ib, lane);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const f32x16 acc = tile_layer<TERMS>(f3, opsB + q * kBuf, lane);
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = silu(acc[r] + b3[r]);
      const float part = head_part(w4, v);
      if (h == 0) head[q][ib][lane] = part;
    }
  }
  __syncthreads();
  if (turn > 0 && ib == (turn & 7)) finish(g - gridDim.x);
}

// Forward of a training tile: z1, z2, z3 of this wave's block, h1 and h2 to
// memory, and the tile's head sum (after a barrier).  lds: 64 KiB.
struct TileForward {
  float z1[16], z2[16], z3[16];
  float head;
};
template <int TERMS>
__device__ __forceinline__ void tile_forward(const Weights& W, const Train& T, const float (&u)[kIn],
                                             const float (&w4)[16], int64_t tile, bf16x8* lds,
                                             float (*head)[kWaveRows], int ib, int lane,
                                             TileForward& o) {
  const int h = lane >> 5;
  bf16x8* const opsA = lds;
  bf16x8* const opsB = lds + 2 * kOps;
  const int64_t at = tile * kWaveTile + (int64_t)ib * 1024 + lane;
  bf16x8 f2[16], f3[16];
  load_frags(W.w2f, ib, lane, f2);
  float b[16], v[16];
  load_units(W.master + kOffB1, ib, h, b);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = b[r];
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
      reinterpret_cast<const bf16x8*>(W.w1)[ib * 64 + lane], input_operand(u, h), acc, 0, 0, 0);
  load_frags(W.w3f, ib, lane, f3);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    o.z1[r] = acc[r];
    v[r] = silu(acc[r]);
    T.h1[at + 64 * r] = bf16_bits(v[r]);
  }
  share_operand<TERMS>(v, opsA, ib, lane);
  load_units(W.master + kOffB2, ib, h, b);
  __syncthreads();
  acc = tile_layer<TERMS>(f2, opsA, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    o.z2[r] = acc[r] + b[r];
    v[r] = silu(o.z2[r]);
    T.h2[at + 64 * r] = bf16_bits(v[r]);
  }
  share_operand<TERMS>(v, opsB, ib, lane);
  load_units(W.master + kOffB3, ib, h, b);
  __syncthreads();
  acc = tile_layer<TERMS>(f3, opsB, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    o.z3[r] = acc[r] + b[r];
    v[r] = silu(o.z3[r]);
  }
  const float part = head_part(w4, v);
  if (h == 0) head[ib][lane] = part;
  __syncthreads();
  o.head = 0.0f;
#pragma unroll
  for (int w = 0; w < kTileBlock / 64; ++w) o.head += head[w][lane & 31];
}

// Sums over the tile's 32 samples of v[r] (and of v[r] u[c]) for every unit
// of this wave's block, through its own 4 KiB of LDS: unit lane % 32 sums
// samples 16 (lane / 32) .. + 15, then the halves meet.
template <int C>
__device__ __forceinline__ void unit_sums(const float (&v)[16], float* tr,
                                          const float* __restrict__ us, int lane, float (&sum)[C]) {
  const int h = lane >> 5, s = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int unit = 8 * (r >> 2) + 4 * h + (r & 3);
    tr[32 * unit + (s ^ unit)] = v[r];
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int c = 0; c < C; ++c) sum[c] = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int q = 16 * h + i;
    const float x = tr[32 * s + (q ^ s)];
    sum[0] += x;
#pragma unroll
    for (int c = 1; c < C; ++c) sum[c] = fmaf(x, us[8 * q + c - 1], sum[c]);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int c = 0; c < C; ++c) sum[c] += __shfl_xor(sum[c], 32);
}

// Forward and backward of one tile: the pre-activations stay in registers;
// what leaves the workgroup are the BF16 operands of the weight-gradient
// products (h1, h2, dz2, dz3) and the tile's sums of every other gradient.
template <int TERMS>
__global__ __launch_bounds__(kTileBlock) void mlp_grad_tile(Weights W, Train T) {
  extern __shared__ bf16x8 lds[];  // two layers' operands, then the waves' transposes
  __shared__ float us[kWaveRows][8], dys[kWaveRows], head[kTileBlock / 64][kWaveRows];
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int ib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  float* tr = reinterpret_cast<float*>(lds + 4 * kOps) + 1024 * ib;
  const int64_t tile = blockIdx.x;
  const int64_t s = tile * kWaveRows + (lane & 31);
  const bool live = s < T.B;
  const int64_t row = (live && T.idx) ? (int64_t)T.idx[s] : s;
  float u[kIn], raw[4];
  const bool inside = normalise(W, T.x, row, live, u, raw);
  if (ib == 0 && h == 0) {
#pragma unroll
    for (int c = 0; c < kIn; ++c) us[lane][c] = u[c];
  }
  float w4[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) w4[r] = bf16_float(W.w4[unit_of(ib, r, h)]);
  TileForward o;
  tile_forward<TERMS>(W, T, u, w4, tile, lds, head, ib, lane, o);
  bf16x8 f[16];
  load_frags(W.w3t, ib, lane, f);
  if (ib == 0) {
    const float y = output(W, o.head, live && inside, raw);
    float lc = 0.0f, g = 0.0f;
    if (h == 0 && live) {
      const float wv = T.w ? T.w[row] : 1.0f;
      const float res = y - T.t[row];
      g = 2.0f * wv * res * T.inv_b;
      lc = wv * res * res * T.inv_b;
    }
    if (h == 0) dys[lane] = g;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      lc += __shfl_xor(lc, m);
      g += __shfl_xor(g, m);
    }
    if (lane == 0) {
      T.tsum[2 * tile] = g;
      T.tsum[2 * tile + 1] = lc;
    }
  }
  __syncthreads();
  const float dy = dys[lane & 31];
  const float gy = W.out_scale * dy;
  const int64_t at = tile * kWaveTile + (int64_t)ib * 1024 + lane;
  float* out = T.usum + (tile * kHid + 32 * ib) * kUnitSums;
  bf16x8* const opsA = lds;
  bf16x8* const opsB = lds + 2 * kOps;
  float v[16], one[1], in[kIn + 1];
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = dy * silu(o.z3[r]);
  unit_sums<1>(v, tr, nullptr, lane, one);
  const float dw4 = one[0];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    v[r] = w4[r] * gy * dsilu(o.z3[r]);
    T.dz3[at + 64 * r] = bf16_bits(v[r]);
  }
  share_operand<1>(v, opsB, ib, lane);
  unit_sums<1>(v, tr, nullptr, lane, one);
  const float db3 = one[0];
  __syncthreads();
  f32x16 acc = tile_layer<1>(f, opsB, lane);  // dh2 = W3^T dz3
  load_frags(W.w2t, ib, lane, f);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    v[r] = acc[r] * dsilu(o.z2[r]);
    T.dz2[at + 64 * r] = bf16_bits(v[r]);
  }
  share_operand<1>(v, opsA, ib, lane);
  unit_sums<1>(v, tr, nullptr, lane, one);
  const float db2 = one[0];
  __syncthreads();
  acc = tile_layer<1>(f, opsA, lane);  // dh1 = W2^T dz2
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = acc[r] * dsilu(o.z1[r]);
  unit_sums<kIn + 1>(v, tr, us[0], lane, in);
  if (h == 0) {
    float* q = out + lane * kUnitSums;
#pragma unroll
    for (int c = 0; c < kIn; ++c) q[c] = in[c + 1];
    q[6] = in[0];
    q[7] = db2;
    q[8] = db3;
    q[9] = dw4;
  }
}

// Partial weight gradients dW[i][k] = sum_s dz[i][s] h[k][s] of layers 2 and
// 3 over one chunk of kChunk samples, the samples as the K dimension: a
// workgroup takes 128 x 128 of the matrix, each of its four waves 64 x 64 (an
// operand row is loaded once for two products, where a wave per 32 x 32 tile
// loaded it for one: 100 MB through the L2s at 4096 samples, 15 us).
__global__ __launch_bounds__(kBlock) void mlp_wgrad(Train T) {
  const int nchunks = (int)(T.Bp / kChunk);
  const int q = (int)blockIdx.x % nchunks;
  const int quad = ((int)blockIdx.x / nchunks) & 3;
  const int L = (int)blockIdx.x / (nchunks * 4);
  const int wave = threadIdx.x >> 6;
  const int ib = 4 * (quad >> 1) + 2 * (wave >> 1), kb = 4 * (quad & 1) + 2 * (wave & 1);
  const int lane = threadIdx.x & 63, h = lane >> 5, row = lane & 31;
  const uint16_t* dz = L ? T.dz3 : T.dz2;
  const uint16_t* hh = L ? T.h2 : T.h1;
  f32x16 acc[2][2] = {{f32x16{}, f32x16{}}, {f32x16{}, f32x16{}}};
#pragma unroll 8
  for (int s0 = 0; s0 < kChunk; s0 += 16) {
    // 8 consecutive samples of one unit are contiguous in the tile layout
    const int64_t sa = (int64_t)q * kChunk + s0 + 8 * h;
    bf16x8 a[2], b[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      a[e] = *reinterpret_cast<const bf16x8*>(dz + tile_index(32 * (ib + e) + row, sa));
      b[e] = *reinterpret_cast<const bf16x8*>(hh + tile_index(32 * (kb + e) + row, sa));
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        acc[e][g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[e], b[g], acc[e][g], 0, 0, 0);
  }
  float* out = T.part + ((size_t)(L * nchunks + q) << 16);
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        out[(32 * (ib + e) + 8 * (r >> 2) + 4 * h + (r & 3)) * kHid + 32 * (kb + g) + row] =
            acc[e][g][r];
}

__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.0f;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) t += red[w];
  return t;
}

// Gradient sums in a fixed order: blocks [0, 512) add the partials of dW2 and
// dW3; the next kSumBlocks the tiles' sums of dW1, db1, db2, db3 and dw4, 16
// of them each, 16 threads to a sum; the last block db4 and the loss.
constexpr int kSumBlocks = kHid * kUnitSums / 16;
__global__ __launch_bounds__(kBlock) void mlp_reduce(Weights W, Train T, float* grad,
                                                     float* loss) {
  __shared__ float red[kBlock];
  const int nchunks = (int)(T.Bp / kChunk);
  const int64_t tiles = T.Bp / kWaveRows;
  const int b = blockIdx.x;
  if (b < 512) {
    const int e = b * kBlock + threadIdx.x;
    const int L = e >> 16, at = e & 0xFFFF;
    float sum = 0.0f;
#pragma unroll 8
    for (int q = 0; q < nchunks; ++q) sum += T.part[((size_t)(L * nchunks + q) << 16) + at];
    grad[(L ? kOffW3 : kOffW2) + at] = sum;
    return;
  }
  if (b < 512 + kSumBlocks) {
    const int e = (b - 512) * 16 + (int)(threadIdx.x & 15), part = (int)(threadIdx.x >> 4);
    float sum = 0.0f;
#pragma unroll 8
    for (int64_t t = part; t < tiles; t += 16) sum += T.usum[t * (kHid * kUnitSums) + e];
    red[threadIdx.x] = sum;
    __syncthreads();
    if (part != 0) return;
#pragma unroll
    for (int p = 1; p < 16; ++p) sum += red[16 * p + threadIdx.x];
    const int unit = e / kUnitSums, c = e - unit * kUnitSums;
    if (c < kIn) grad[kOffW1 + unit * kIn + c] = sum;
    else if (c == 6) grad[kOffB1 + unit] = sum;
    else if (c == 7) grad[kOffB2 + unit] = sum;
    else if (c == 8) grad[kOffB3 + unit] = sum;
    else grad[kOffW4 + unit] = W.out_scale * sum;
    return;
  }
  float gy = 0.0f, l = 0.0f;
  for (int64_t t = threadIdx.x; t < tiles; t += kBlock) {
    gy += T.tsum[2 * t];
    l += T.tsum[2 * t + 1];
  }
  gy = block_sum(gy, red);
  l = block_sum(l, red);
  if (threadIdx.x == 0) {
    grad[kOffB4] = W.out_scale * gy;
    if (loss) *loss = l;
  }
}

// Adam on the FP32 master parameters (when a.update), then every matrix
// weight's BF16 copy, in the forward and the transposed fragment layouts.
__global__ __launch_bounds__(kBlock) void mlp_adam(AdamArgs a) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= kParams) return;
  float v = a.master[p];
  if (a.update) {
    const float g = a.grad[p];
    const float m = fmaf(a.beta1, a.mom[p], (1.0f - a.beta1) * g);
    const float q = fmaf(a.beta2, a.vel[p], (1.0f - a.beta2) * g * g);
    a.mom[p] = m;
    a.vel[p] = q;
    v -= a.lr * (m * a.c1) / (sqrtf(q * a.c2) + a.eps);
    a.master[p] = v;
  }
  const uint16_t bits = bf16_bits(v);
  if (p < kOffB1) {
    const int i = p / kIn, c = p % kIn;
    a.w1[frag1_index(i, c)] = bits;
    a.w1[frag1_index(i, kIn + c)] = bits;
    if (c == 0)
      for (int z = 2 * kIn; z < 16; ++z) a.w1[frag1_index(i, z)] = 0;
  } else if (p >= kOffW2 && p < kOffB2) {
    const int i = (p - kOffW2) >> 8, k = (p - kOffW2) & 255;
    a.w2f[frag_index(i, k)] = bits;
    a.w2t[frag_index(k, i)] = bits;
  } else if (p >= kOffW3 && p < kOffB3) {
    const int i = (p - kOffW3) >> 8, k = (p - kOffW3) & 255;
    a.w3f[frag_index(i, k)] = bits;
    a.w3t[frag_index(k, i)] = bits;
  } else if (p >= kOffW4 && p < kOffB4) {
    a.w4[p - kOffW4] = bits;
  }
}

// ------------------------------------------------------------- launchers

// Dynamic LDS beyond the 64 KiB default (gfx950 has 160 KiB per CU).
template <typename F>
static hipError_t allow_lds(F* kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_forward(const Weights& W, int terms, const float* x, int64_t B, float* y,
                          uint8_t* in_range, hipStream_t s) {
  const FwdIO io{x, B, y, in_range};
  const int64_t tiles = (B + kWaveRows - 1) / kWaveRows;
  const size_t lds = sizeof(bf16x8) * 2 * (size_t)terms * kOps;
  if (tiles <= kCus) {
    if (terms == 2)
      hipLaunchKernelGGL(mlp_forward<2>, dim3((unsigned)tiles), dim3(kTileBlock), lds, s, W, io);
    else
      hipLaunchKernelGGL(mlp_forward<1>, dim3((unsigned)tiles), dim3(kTileBlock), lds, s, W, io);
    return hipGetLastError();
  }
  const int64_t pairs = (tiles + 1) / 2;
  const dim3 grid((unsigned)(pairs < kCus ? pairs : kCus));
  auto go = [&](auto* kernel) {
    const hipError_t e = allow_lds(kernel, 2 * lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, grid, dim3(kTileBlock), 2 * lds, s, W, io, pairs);
    return hipGetLastError();
  };
  return terms == 2 ? go(mlp_forward_pairs<2>) : go(mlp_forward_pairs<1>);
}

hipError_t launch_train_grad(const Weights& W, int terms, const Train& T, float* grad,
                             float* loss, hipStream_t s) {
  const dim3 tiles((unsigned)(T.Bp / kWaveRows));
  const size_t lds = sizeof(bf16x8) * 4 * kOps + sizeof(float) * 1024 * (kTileBlock / 64);
  hipError_t e;
  if (terms == 2) {
    if ((e = allow_lds(mlp_grad_tile<2>, lds)) != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_grad_tile<2>, tiles, dim3(kTileBlock), lds, s, W, T);
  } else {
    if ((e = allow_lds(mlp_grad_tile<1>, lds)) != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_grad_tile<1>, tiles, dim3(kTileBlock), lds, s, W, T);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(mlp_wgrad, dim3((unsigned)(2 * 4 * (T.Bp / kChunk))), dim3(kBlock), 0, s, T);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(mlp_reduce, dim3(512 + kSumBlocks + 1), dim3(kBlock), 0, s, W, T, grad, loss);
  return hipGetLastError();
}

hipError_t launch_adam(const AdamArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(mlp_adam, dim3((kParams + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace mlp
}  // namespace qtree
