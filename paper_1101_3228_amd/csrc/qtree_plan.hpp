// Host-side plan object shared by the C-ABI implementation files.
#pragma once
#include <hip/hip_runtime.h>

#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "qtree.h"
#include "qtree_internal.hpp"

struct qtree_plan {
  int d = 0, n = 0;
  std::vector<int32_t> N;
  std::vector<int64_t> pt_off, cnt_off, aux_off;
  std::vector<int32_t> P;
  int64_t points = 0, entries = 0;
  int32_t maxN = 0, maxP = 0;
  char* ws = nullptr;
  qtree::WsLayout lay{};
  int64_t tune_chunk = 0;  // 0: automatic
  int32_t tune_xcd_map = 1;
  int32_t tune_count = 0;  // 0 automatic, 1 direct atomics, 2 two-pass
  int32_t tune_groups = 0;  // layer groups of the two-pass forward (0: automatic)
  int32_t tune_nd_samples = 8;  // d >= 2 pass A: samples per lane sharing each grid read
  int32_t tune_tail = 100;      // last layer group's share, percent of the others
  int32_t tune_buckets = 1;     // d = 2, 3: cells through the bucket tables
  int64_t buckets = 0;          // d = 2: buckets over all layers (0: no tables)
  int64_t cubes = 0;            // d = 3: the same
  double cube_misses = 0.0;     // ... and the share of the search they leave to scans
  int64_t st_max = 1;           // super tiles of the largest count block
  uint64_t few_keys = 0;        // keys of a super tile below which it is not split in two
  int32_t max_tiles = 0, total_tiles = 0;
  std::vector<int32_t> tile_off;  // first super tile of every layer (host copy)
  std::vector<int32_t> unit_off;  // first histogram unit of every layer (host copy)
  std::vector<int32_t> few_split, few_off;  // split and unit_off for few samples
  std::vector<int32_t> split;     // histogram parts per super tile of every layer
  std::vector<float> marg_L;      // d = 1: the marginal factor L_k of every layer
  std::vector<double> edges;      // d = 1: host copy of the cell-edge probabilities
  std::vector<int64_t> band_off;  // d = 1: banded stratified counts, row offsets [R + 1]
  std::vector<int32_t> band_lo;   // d = 1: first band column of every row [R]
  int32_t gt_Kmax = -1;           // d = 1: largest guide K over the layers (-1: no tables)
  int32_t gt_Bmax = 1;            // d = 1: largest guide table
  int64_t batch_chunks = 0;      // scratch chunks per layer per pass
  int64_t all_chunks = 0;        // ... with the path cells' room (from lay.path on)
  int64_t path_cells = 0;        // pathwise scratch: cells per layer (0: none)
  bool two_pass_ok = false;       // the workspace holds two-pass scratch
  bool two_pass_shape = false;    // the count blocks and LDS allow two-pass counting
  hipEvent_t trace_keys = nullptr;
  // stream and events of the overlapped histogram passes (made on first use)
  static constexpr int kMaxGroups = 8;
  mutable hipStream_t aux = nullptr;
  mutable hipEvent_t fork[kMaxGroups] = {};
  mutable hipEvent_t join = nullptr;

  // The path cells' room serves one call at a time: each waits on the device for
  // the event of the one before.
  struct PathUse {
    std::mutex lock;
    hipEvent_t done = nullptr;  // recorded after each use
    ~PathUse() {
      if (done) (void)hipEventDestroy(done);
    }
  };
  std::shared_ptr<PathUse> path_use = std::make_shared<PathUse>();

  ~qtree_plan() {
    if (aux) (void)hipStreamSynchronize(aux);
    for (hipEvent_t& e : fork)
      if (e) (void)hipEventDestroy(e);
    if (join) (void)hipEventDestroy(join);
    if (aux) (void)hipStreamDestroy(aux);
  }
};

namespace qtree {
// A few results on their way to the host: a kernel writes them to a slot of
// pinned memory, and a blocking call copies them out when its stream is done.
// A copy into the caller's pageable memory costs 12 us, a strided one 7 us a
// row more (97 us for 12 payoffs); the kernel and the wait cost 16.  One array
// of kSlots slots, made with the first plan and kept until the process ends,
// serves all plans, threads and devices; a call holds a slot while it waits,
// and one that finds none free, or has more results, copies as before.
class HostSlot {
 public:
  static constexpr int kSlots = 16;
  static constexpr int64_t kDoubles = 2048;
  static void reserve();            // at plan creation
  explicit HostSlot(int64_t n);     // ptr() is null without a slot
  ~HostSlot();
  HostSlot(const HostSlot&) = delete;
  HostSlot& operator=(const HostSlot&) = delete;
  double* ptr() const { return p_; }
  // An error for a stream under capture, which nothing can wait for (the wait
  // would end the capture, and finish() would keep the slot).
  static hipError_t can_wait(hipStream_t s);
  // Waits for the stream and copies n results out.  After an error the slot
  // stays taken: the kernel may still write to it.
  hipError_t finish(double* out, int64_t n, hipStream_t s);

 private:
  double* p_ = nullptr;
  int i_ = -1;
};
// n results, `stride` apart, to host memory; waits for the stream.
hipError_t results_to_host(const double* V, int64_t stride, int64_t n, double* out, hipStream_t s);
}  // namespace qtree

namespace qtree {
// Record a failure for qtree_last_error and return its status.
qtree_status set_error(qtree_status s, const std::string& msg);

// Scratch of the two-pass counting: keys and segment starts for `chunks`
// chunks per layer per pass, and the most layer groups a call may use.
struct CountScratch {
  uint16_t* keys = nullptr;
  uint32_t* segs = nullptr;
  int64_t chunks = 0;
  int max_groups = 1;
};
qtree_status transitions_on_scratch(const qtree_plan* plan, uint64_t m0, uint64_t M,
                                    uint64_t seed, uint32_t contract_id, qtree_mode mode,
                                    int32_t* counts, void* stream, void* base, size_t bytes);
}  // namespace qtree
