// Internal layout shared by the host side of the library and its kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qtree {

constexpr int kMaxDim = 3;

// Two-pass LAYERWISE counting.  Pass A sorts each chunk of kChunk samples of
// a layer by tile (kTile consecutive entries of the layer's count block) and
// stores every key as its 16-bit offset inside its super tile (kSuper
// consecutive entries, kSuper / kTile tiles); pass B gives every (layer,
// super tile) to one workgroup that histograms its keys in LDS and writes the
// super tile with plain stores.
// One tile per super tile: the sort's scan and a chunk's segment table have
// one entry per super tile, all that pass B reads.
constexpr int kTileBits = 14;
constexpr int kTile = 1 << kTileBits;
constexpr int kSuperBits = 14;
constexpr int kSuper = 1 << kSuperBits;
constexpr int kTilesPerSuper = kSuper / kTile;
constexpr int kChunk = 4096;          // samples per pass-A workgroup

// A pointer read from device memory (a batch or job record, a kernel
// argument's struct field) is a generic address to the compiler, which then
// loads through it with flat instructions: a 64-bit address in VGPRs, no
// scalar loads of uniform fields, and waits shared with LDS operations.
// Every table such a field points to is device memory: reading the field as
// a global pointer and converting it gives global and scalar loads.
template <class T>
__device__ __forceinline__ T* as_global(T* const& field) {
  typedef __attribute__((address_space(1))) T* G;
  return (T*)*reinterpret_cast<const G*>(&field);
}
constexpr int kMaxTiles = 4096;       // larger count blocks use direct atomics
constexpr int kDefaultBatch = 1 << 22;  // samples per layer per pass by default
constexpr int kScanTile = 8;            // records per tile of the d >= 2 argmin scan
constexpr int kGuideMax = 8192;         // largest guide table of a 1-D layer (entries)
constexpr int kGuideKMax = 4;           // most midpoints one guide bucket may add

// One record per layer k = 0..n, stored in the plan's device workspace.
// Model coefficients are the FP32 inputs of the AR(1) proposition (Sec. 3);
// A, b, T are unused on the last layer.
struct alignas(16) LayerDev {
  int64_t cnt_off;  // first entry of counts block k (k < n)
  int32_t N;        // N_k
  int32_t N1;       // N_{k+1} (0 on the last layer)
  int32_t pt_off;   // first point of layer k in the point array
  int32_t aux_off;  // 1-D: first padded midpoint of layer k
  int32_t P;        // 1-D: padded midpoint slots, a power of two >= N_k
  int32_t logP;     // log2(P)
  int32_t tiles;    // ceil(N_k N_{k+1} / kTile) (0 on the last layer)
  int32_t tile_off; // super tiles of the layers before k
  // Histogram pass: each super tile of layer k is split into `split` parts
  // over the chunks (layers with few super tiles, such as a one-point first
  // layer, would otherwise give all their keys to a few workgroups); the
  // parts of a split layer add into its count block atomically, zeroed first.
  int32_t split;    // parts per super tile (1: one workgroup stores the tile)
  int32_t unit_off; // histogram-pass units (super tiles x parts) of the layers before k
  int32_t edge_off; // 1-D: first of the N_k + 1 cell-edge probabilities of layer k
  // 1-D guide table of the cell search: bucket b = (int)clamp(fma(x, gt_scale,
  // gt_shift), 0, gt_B - 1); the cell is tab[b] + #{r < K : m[tab[b] + r] < x}
  // for K >= gt_K (the table holds the count of midpoints below the bucket's
  // first float; gt_K bounds the midpoints a bucket can add).
  int32_t gt_off;   // first entry of the layer's table (16-bit entries)
  int32_t gt_B, gt_K;
  float gt_scale, gt_shift;
  float A[9], b[3], T[9], mu[3], L[9];
  float x0[3];      // start point of the pathwise mode (layer 0 record)
  // d = 2 bucketed cell search (bk_B[0] = 0: none): the layer's reachable box
  // from bk_lo in bk_B[0] x bk_B[1] buckets; x is in bucket
  // (floor((x_0 - bk_lo[0]) bk_scale[0]), floor((x_1 - bk_lo[1]) bk_scale[1]))
  // in FP32, and bucket (i, j) owns row bk_off + i bk_B[1] + j of the row
  // array (kBucketRow entries): entry 0 its candidate count c, entries 1..c
  // every point that can be the FP32 argmin anywhere in it, in increasing
  // index, the others the pad N (the search's pad record, whose key is NaN);
  // points and pad as byte offsets of 8-byte pairs.  A bucket of more
  // candidates has c = kBucketLong, pads, and in entries 6 and 7 the index
  // (low half first) of a row of the plan's pool of longer ones (kLongRow
  // entries, the same layout); where they do not fit there either, c =
  // kBucketFull, and the full scan decides.
  float bk_lo[2], bk_scale[2];
  int32_t bk_B[2];
  int32_t bk_off;
  // split and unit_off for few samples (FwdArgs::few)
  int32_t few_split, few_off;
};
constexpr int kBucketRow = 8;             // uint16 entries of a bucket row (16 bytes)
constexpr int kBucketCap = kBucketRow - 1; // candidates it holds
constexpr int kLongRow = 32;              // uint16 entries of a pool row (64 bytes)
constexpr int kLongCap = kLongRow - 1;    // candidates it holds
constexpr uint16_t kBucketFull = 0xFFFF;  // row count: candidates did not fit
constexpr uint16_t kBucketLong = 0xFFFE;  // row count: in a pool row
// Rows of the pool: one for every kBucketsPerLong buckets and row 0, whose
// first word counts the rows taken.  (On product grids about one bucket in
// thousands needs one.)
constexpr int64_t kBucketsPerLong = 8;
inline int64_t long_rows(int64_t buckets) { return buckets > 0 ? 1 + buckets / kBucketsPerLong : 0; }
// Buckets per side of a d = 2 layer of N points: about 36 buckets per point,
// at most 512 per side.  Denser buckets list fewer candidates, but four are
// looked at anyway, and the rows of two layers (2.3 MB at N = 2000) have to
// stay in an XCD's 4 MB L2.  Buckets per point 24 / 36 / 64 / 128 / 256: the
// 2-D max-call (n = 30, N = 2000, 1e7 pairs) 3.24 / 3.14 / 3.43 / 3.40 / 3.41
// ms a call, n = 365, N = 500, 1e5 pairs 0.42 / 0.40 / 0.42 / 0.47 / 0.51 ms,
// a ragged book of N up to 1000 2.54 / 2.49 / 2.43 / 2.49 / 2.48 ms.
inline int bucket_side(int N) {
  if (N <= 1) return 1;
  int b = 1;
  while ((double)b * b < 36.0 * N) ++b;
  return b < 512 ? b : 512;
}

// d = 3 bucketed cell search of a layer (B[0] = 0: none), on the same rule: the
// box from lo in B[0] x B[1] x B[2] buckets, bucket (i0, i1, i2) owns row
// off + (i0 B[1] + i1) B[2] + i2 of kCubeRow entries: its candidate count, then
// the candidates' indices in increasing order, then the pad N (a record whose
// key is +inf); kCubeFull where they do not fit, and the full scan decides.
struct Cubes {
  float lo[3], scale[3];
  int32_t B[3];
  int32_t off;
  int32_t N, pt_off;
  uint32_t misses;  // of the samples asked for at the build
};
constexpr int kCubeRow = 16;               // uint16 entries (32 bytes)
constexpr int kCubeCap = kCubeRow - 1;
constexpr uint16_t kCubeFull = 0xFFFF;
// Smaller layers scan: 50 layers, 10^6 pairs, tables / scan at 12 / 18 / 27 / 48
// points 790 / 739, 789 / 788, 789 / 842, 768 / 909 us; 10^5 paths 143 / 109, 145 /
// 113, 147 / 128, 140 / 144.
constexpr int kCubeMinN = 24;
constexpr int kCubeTile = 4;               // B is a multiple of it
// Two-pass chunks (2^15 samples) that the tables leave in a workspace: in more
// passes, each reading and writing all counts, they cost more than they save.  8
// layers of 1600 points, 3 10^5 samples, 4 / 8 / 16 chunks beside the tables:
// 1157 / 616 / 316 us, the full scan in one pass 805; 10^6 samples 3765 / 1915 /
// 1004 against 2387; 4 layers of 4096 points 1408 / 848 / 468 against 1460.
constexpr int64_t kCubeChunks = 8;
constexpr int64_t kMaxCubes = 1ll << 23;   // rows of a plan (256 MB)
// Buckets per axis of a layer of N points: about `per` per point, at most 64 per
// axis.  16 / 32 / 64 per point: 294 / 289 / 288 us for a 12-layer tree of
// 990 points and 3 10^5 pairs per layer (the full scan: 927 us).  A plan takes
// 32, or 16 where those would be too many rows, and beyond that no tables: the
// layers of a plan that had tables for some only scanned alone at the end of a
// launch (290 layers of 1000 points, 3 10^4 samples 2584 us, the scan 1998).
inline int cube_side(int N, int per) {
  int b = kCubeTile;
  while ((double)b * b * b < (double)per * N) b += kCubeTile;
  return b < 64 ? b : 64;
}
// 32, 16 or 0.
int cubes_per_point(int n, const int32_t* N);

// Workspace layout (byte offsets from the workspace base).
struct WsLayout {
  size_t layers;   // LayerDev[n+1]
  size_t points;   // d == 1: float[sum N]; d >= 2: float4[sum N] = (g0, g1, g2, h)
  size_t aux;      // d == 1: float[sum P] midpoints padded with +inf
  size_t edges;    // d == 1: double[sum (N_k + 1)] marginal probabilities below the cell edges
  size_t guide;    // d == 1: uint16[(n + 1) kGuideMax] guide tables of the cell search
  size_t band;     // d == 1: int64[R + 1] band offsets, then int32[R] first band columns
                   // of the R = sum_{k<n} N_k count rows (banded stratified counts)
  size_t bk_rows;  // d == 2: uint16[buckets][kBucketRow] bucket rows (count, candidates)
  size_t bk_long;  // d == 2: uint16[long_rows][kLongRow] pool of longer rows
  size_t cubes;    // d == 3: Cubes[n + 1], where the plan has tables
  size_t cube_rows; // d == 3: uint16[buckets][kCubeRow]
  size_t path;     // uint16[n][path cells] cells of the pathwise mode
  size_t keys;     // uint16[n][batch chunks][kChunk] pass-A keys
  size_t segs;     // uint32[n][batch chunks][max tiles + 1] segment starts
  size_t total;
};

// Pathwise scratch: a cell of 2 bytes per path and layer, for up to 2^17
// paths a pass (a path's walk is a serial chain: 2^17 fill the chip) in at
// most 96 MiB (n = 365 still takes 2^17); no scratch where that is under 4096
// paths, or where a count block has more than kPathTiles super tiles (about
// 1450 points a layer), each of which reads every cell pair.
constexpr int64_t kPathCells = 1 << 17;
constexpr int64_t kPathBytes = 96ll << 20;
constexpr int kPathTiles = 128;
int64_t path_cells(int n, const int32_t* N);

// Layout for a scratch that holds `batch_chunks` chunks per layer (0: none),
// `cells` path cells per layer (path_cells or 0) and `cubes` buckets of the
// d = 3 search (0: none).
WsLayout ws_layout(int d, int n, const int32_t* N, int64_t batch_chunks, int64_t cells,
                   int64_t cubes);
bool two_pass_fits(int d, int n, const int32_t* N);

// The rows of the d = 2 bucketed cell search of a plan.
struct BucketTab {
  const uint4* rows;   // a row per bucket
  const uint4* longs;  // pool rows, kLongRow / 8 words of 16 bytes each
};

struct FwdArgs {
  const LayerDev* layers;
  const float* mids;     // 1-D midpoints (padded per layer)
  const uint16_t* guide; // 1-D guide tables (kGuideMax entries per layer)
  int gt_Kmax;           // 1-D: largest guide K over the layers, -1 without tables
  int gt_Bmax;           // 1-D: largest guide table
  const float4* pts;     // d >= 2 points with half norm
  const float* pts1;     // 1-D points
  int32_t* counts;
  uint64_t m0, M;
  uint32_t key0, key1, contract;
  int32_t n, d;
  // launch decomposition: unit u = (layer, chunk); `chunks` per layer
  int32_t chunks;
  int32_t units;          // n * chunks
  int32_t units_per_xcd;  // ceil(units / 8)
  int32_t xcd_map;        // 1: keep a layer's chunks on one XCD
  uint64_t chunk_len;     // samples per chunk (even)
  int32_t maxP;           // largest padded midpoint count (1-D LDS sizing)
  int32_t maxN;           // largest layer size (d >= 2 LDS sizing)
  // two-pass counting
  uint16_t* keys;
  uint32_t* segs;
  int32_t seg_stride;     // max tiles + 1
  int32_t max_tiles;
  int32_t total_tiles;    // histogram units of this launch (pass-B grid)
  int32_t first_batch;    // pass B overwrites instead of adding
  int32_t few;            // pass B split as for few samples
  int32_t layer0;         // first layer of this launch (units and tiles)
  int32_t nd_samples;     // d >= 2: samples per lane sharing each grid read (8 or 4)
  int32_t tile0;          // first histogram unit of this launch
  // d = 2 bucketed cell search (bucketed = 0: the full scan)
  int32_t bucketed;
  BucketTab bk;
  // d = 3 bucketed cell search (null: the full scan)
  const Cubes* cubes;
  const uint4* cube_rows;
};

// Forward obstacle on the sum of the factors (see qtree_payoff_forward).
struct ForwardArgs {
  const LayerDev* layers;
  const float* pts1;
  const float4* pts;
  double* v;
  int32_t n, d, maxN;
  double S0, K, r, Tm;
  double w[kMaxDim];  // mix' sigma
};

// Swing BDP: P is [Pts][Qmax + 1] (point major, the levels of a point
// contiguous).
constexpr int kSwingMaxQ = 2046;
struct SwingArgs {
  const LayerDev* layers;
  const int32_t* counts;
  const double* v;
  double* P;
  int64_t Pts;
  int32_t n, Qmin, Qmax;
};

hipError_t launch_forward_payoff(const ForwardArgs& a, hipStream_t s);
hipError_t launch_swing(const SwingArgs& a, const int32_t* N_host, hipStream_t s);

hipError_t launch_zero_i32(int32_t* p, int64_t count, hipStream_t s);
hipError_t launch_fwd_layer_1d(const FwdArgs& a, hipStream_t s);
hipError_t launch_fwd_layer_nd(const FwdArgs& a, hipStream_t s);
// Pathwise counts of paths a.m0 .. + a.M - 1: with a device-scope atomic per
// step, or through a.M <= stride cells per layer (stride a multiple of 8) in
// `cells`, stored (first) or added.  a.total_tiles: super tiles of all layers.
hipError_t launch_fwd_path(const FwdArgs& a, hipStream_t s);
hipError_t launch_path_counts(const FwdArgs& a, uint16_t* cells, int64_t stride, bool first,
                              hipStream_t s);
hipError_t launch_fwd_keys(const FwdArgs& a, hipStream_t s);
hipError_t launch_count_tiles(const FwdArgs& a, hipStream_t s);
// Zero the count blocks of the split layers in [layer0, layer0 + nl).
hipError_t launch_zero_split(const FwdArgs& a, int nl, hipStream_t s);

struct BdpArgs {
  const LayerDev* layers;
  const int32_t* counts;
  const double* phi;
  double* V;
  int64_t P;  // points per payoff vector (sum N_k)
  int32_t n_pay;
  // banded counts (else null): row r = pt_off_k + i holds columns
  // band_lo[r] + w, w < band_off[r + 1] - band_off[r], at counts[band_off[r] + w]
  const int64_t* band_off;
  const int32_t* band_lo;
};
hipError_t launch_bdp_layer(const BdpArgs& a, int k, int N_k, int N_k1, int64_t pt_k,
                            int64_t pt_k1, int64_t cnt_k, hipStream_t s);
hipError_t launch_v0(const double* V, int64_t stride, int n, double* out, hipStream_t s);
hipError_t launch_copy_last_layer(const BdpArgs& a, int64_t pt_n, int N_n, hipStream_t s);

struct Contract {
  double S0, K, r, Tm;
  double sigma[kMaxDim];
  double mix[kMaxDim * kMaxDim];  // Brownian factors y = mix x (row-major d x d)
  int32_t kind;
  int32_t has_mix;                // 0: y = x
};
constexpr int kPayoffGroup = 16;  // contracts per payoff launch (kernel-argument size)

struct PayoffArgs {
  const LayerDev* layers;
  const float* pts1;
  const float4* pts;
  double* phi;      // [count][P]
  int64_t P;
  int32_t n, d, maxN, count;
  Contract c[kPayoffGroup];
};
hipError_t launch_payoff(const PayoffArgs& a, hipStream_t s);

// Transition weights pi^k = c / p (FP64, rows padded to N1p = multiple of 4)
// and the nonzero column range of every row, for the many-contract BDP.
struct PiArgs {
  const LayerDev* layers;
  const int32_t* counts;
  const int64_t* pi_off;  // [n] first weight of layer k (device)
  double* pi;
  int2* band;             // [rows] columns [x, y) hold every nonzero weight of the row
  int64_t rows;           // sum_{k<n} N_k
  int32_t n;
};
hipError_t launch_pi(const PiArgs& a, hipStream_t s);

// Backward recursion of many contracts on one tree (`cols` per workgroup).
// One tree of a many-tree launch: its tables and weights, and the contracts
// q0 .. q0 + nq - 1 it prices (workgroups blk0 .. blk0 + ceil(nq / cols) - 1).
struct alignas(16) ManyTree {
  const LayerDev* layers;
  const float* pts1;
  const float4* pts;
  const int64_t* pi_off;
  const double* pi;
  const int2* band;
  int64_t q0, nq;
  int32_t blk0, n;
};
struct ManyArgs {
  const LayerDev* layers;
  const float* pts1;
  const float4* pts;
  const int64_t* pi_off;
  const double* pi;
  const int2* band;
  const Contract* specs;  // [nq] (device)
  double* V0;             // [nq] (device)
  int64_t nq;
  int32_t n, d, max_n, np_max;  // np_max: largest N_k rounded up to a multiple of 4
  // many trees (else null): the table of n_trees trees, ordered by blk0;
  // the fields above then come from the workgroup's tree (max_n, np_max: the
  // largest over the trees)
  const ManyTree* trees;
  int32_t n_trees, blocks;
  int32_t cols;  // contracts per workgroup (bdp_many_cols)
};
bool bdp_many_fits(int max_n);  // layers of up to 256 points
// Contracts per workgroup when 64 of them would make `blocks64` workgroups, for
// layers of points / layers points on average.
int bdp_many_cols(int d, int64_t blocks64, int64_t points, int64_t layers);
hipError_t launch_bdp_many(const ManyArgs& a, hipStream_t s);

// Stratified time-layer counts (d = 1): Ms samples per cell of layer k.
struct StratArgs {
  const LayerDev* layers;
  const float* mids;      // sorted midpoints, padded per layer
  const uint16_t* guide;  // guide tables of the cell search (kGuideMax entries per layer)
  int gt_Kmax, gt_Bmax;   // largest guide K (-1: no tables) and table over the layers
  const double* edges;    // cell-edge probabilities per layer
  uint32_t key0, key1, contract;
  uint64_t M;             // samples per row (alloc 0) or per layer (alloc 1)
  int alloc;              // 0 equal, 1 proportional allocation
  int32_t* counts;        // the plan's count blocks, or the band values
  int n, maxP, maxN;      // layers; largest padded midpoint count; largest N_k
  // banded output (else null): row r = pt_off_k + i keeps columns
  // band_lo[r] .. band_lo[r] + W_r - 1 at counts[band_off[r] ..], W_r =
  // band_off[r + 1] - band_off[r]; counts outside the band go to *overflow
  const int64_t* band_off;
  const int32_t* band_lo;
  uint32_t* overflow;
};
constexpr int kStratRows = 4;            // rows (strata) per tile
constexpr uint64_t kStratSegment = 65536;  // samples per workgroup at most
// A workgroup's share: samples [s0, s1) of the tile of rows [i0, i0 + 4) of
// layer k (in the tile's own order: row by row); split: the tile is shared
// by several workgroups (its counts are added with atomics onto zeros).
struct alignas(16) StratUnit {
  int32_t k, i0, split, pad;
  uint64_t s0, s1;
};
size_t strat_lds_bytes(int maxP, int maxN);
hipError_t launch_strat(const StratArgs& a, const StratUnit* units, int n_units, hipStream_t s);
hipError_t launch_strat_samples(const StratArgs& a, int k, int i, uint64_t t0, int64_t count,
                                float* x, float* y, hipStream_t s);

// Randomized Lloyd iteration (Sec. 2, eq. Qerr) on a device grid.
struct LloydArgs {
  int d, N;
  int Npad;                  // d >= 2: records padded to whole scan tiles
  int P, logP;               // d = 1: midpoint slots (power of two >= N)
  float L[9];                // X = L z, row-major [d][d]
  uint32_t key0, key1;       // Philox key (seed)
  uint32_t it_ctr;           // counter word 1 of the step (the step, or 0)
  int it;                    // step index (distortion slot)
  uint64_t M;                // samples per step
  float* grid;               // [N][d], updated in place
  float4* recs;              // d >= 2: [Npad] (g, |g|^2 / 2)
  double* distortion;        // [steps] or null
  // d = 2 on Philox samples: bucket tables of the current grid over the
  // samples' box (fields as at LayerDev), rebuilt every step; bk_B[0] = 0: none
  float bk_lo[2], bk_scale[2];
  int32_t bk_B[2];
  int32_t bk_off;            // 0
  uint16_t *bk_rows, *bk_longs;
  int bk_pool;
  // per-workgroup partials of the accumulation: row b holds workgroup b's
  // sums [N d], counts [N], distortion, admissible and inadmissible samples
  // (E = N d + N + 3 words)
  unsigned long long* part;
  int E;
  // samples of a caller's set instead of Philox draws: step window
  // (start + m) mod Ms, m < M; samples with a coordinate outside [-64, 64]
  // (or NaN) are skipped and counted
  const float* xs;           // [Ms][d] device, or null (Philox samples)
  uint64_t Ms;
  uint64_t start;
  double gamma;              // new point g + gamma (mean - g); 1: the mean
  unsigned long long* rej_total;  // running total over the steps
  long long* rejected;       // caller's copy of the total, or null
};
constexpr int kLloydMaxBlocks = 512;  // accumulation workgroups per step at most
// With bucket tables: half as many, four times as wide, and the tables take
// the place of the other half of their partials.
constexpr int kLloydMaxWide = kLloydMaxBlocks / 2;
constexpr int kLloydWideThreads = 1024, kLloydWideSamples = 2;  // samples per thread and round
// Buckets per side, a multiple of 4: about 32 per point over the
// samples' whole box (a fifth of them where the points are), at most 192.
// More make the lists short and the corner tests few, but all have to be
// filled in every step: 8 / 16 / 32 / 64 per point take 32 / 25 / 23 / 27 us a
// step at N = 500 and 10^5 samples, and at N = 2048 42 / 42 / 54 / 87.
inline int lloyd_side(int N) {
  int b = 4;
  while ((double)b * b < 32.0 * N) b += 4;
  return b < 192 ? b : 192;
}
size_t lloyd_lds_bytes(int d, int N, int Npad, int P);
// Bucket rows of the d = 2 bucketed cell search of every layer (records
// and LayerDev already in the workspace).
hipError_t launch_bucket_build(const LayerDev* layers, int n_layers_total, int maxN,
                               int64_t total_buckets, const float4* pts, uint16_t* rows,
                               uint16_t* longs, hipStream_t s);
// Rows of the d = 3 search of every layer, `total` of them; and how many of
// kCubeProbes pairs (X_k, X_{k+1}) per layer k find no list, counted in `misses`
// of both layers.
constexpr int kCubeProbes = 1024;
hipError_t launch_cube_build(const LayerDev* layers, Cubes* cubes, int n_layers_total, int total,
                             const float4* pts, uint16_t* rows, hipStream_t s);
hipError_t launch_lloyd_records(const LloydArgs& a, hipStream_t s);
hipError_t launch_lloyd_step(const LloydArgs& a, int blocks, hipStream_t s);
// Moment-matching grids: exact integer moment sums of a device sample set,
// sums = [count, s1 (d), s2 (d d)], and the grid mean + chol(cov) base.
hipError_t launch_sample_moments(int d, const float* x, uint64_t M, long long* sums,
                                 hipStream_t s);
hipError_t launch_moment_grid(int d, const long long* sums, const float* base, int N,
                              float* grid, double* moments, hipStream_t s);

hipError_t launch_pi_quarter_disc(uint32_t key0, uint32_t key1, uint32_t rep0, int reps,
                                  uint64_t blocks, unsigned long long* inside, hipStream_t s);
hipError_t launch_box_muller(const uint32_t* ra, const uint32_t* rb, int64_t count, float* z0,
                             float* z1, hipStream_t s);
hipError_t launch_layer_samples(const FwdArgs& a, int k, int64_t count, float* x, float* y,
                                hipStream_t s);
hipError_t launch_cells(const FwdArgs& a, int k, const float* x, int64_t count, int32_t* cell,
                        hipStream_t s);

}  // namespace qtree
