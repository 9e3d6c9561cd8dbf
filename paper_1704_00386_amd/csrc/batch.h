// batch.h -- the multi-graph sweep engine shared by nd_batch_decompose and
// the server.  Internal header.
#pragma once

#include <memory>
#include <vector>

#include "internal.h"

namespace nd {

constexpr int kBatchRing = 32;    // per-graph sweep counters kept
constexpr int kPollMax = 16;      // epochs between host polls, at most

// Device descriptor of one graph in a batch.
struct BGraph {
  const int64_t *inc_off;
  const int32_t *inc_ids;
  void *tau[2];        // sweep number t reads tau[t & 1] (SND)
  SweepStats *ring;    // counters of sweep t at ring[t % kBatchRing]
  int64_t t0;          // epoch at which the graph joined
  int64_t max_local;   // sweeps allowed
  uint8_t *act[2];     // frontier stamps: sweep t reads act[t & 1]
  uint8_t *act_sum[2]; // one stamp per 64 r-cliques, set with any of their flags
  void *slack;         // support counting (NULL: flags); act is then its counters
  int64_t lost_shift;  // log2 of the bytes per counter
  unsigned long long notify_below;  // start notifying at <= this many changes
};

// A run of r-cliques of one graph and one sweep bin.
struct BTile {
  int32_t g;
  int32_t type;  // SweepBin
  int64_t lo, hi;
};

// Device-resident launch state: every kernel of an epoch reads it, so a
// chunk of epochs built as a HIP graph stays valid when the tables change.
struct BState {
  int64_t epoch;
  int32_t ntiles;
  int32_t ng;
};

// The tile kernel of k = K and tau of type T (16 or 32 bits), instantiated in
// sweep_inst.hip.
template <int K, typename T>
const void *batch_kernel(bool and_mode, bool fr);

// Tile length: an epoch is cut into about grid * tiles_per_group tiles of
// about equal work (one workgroup each).
struct BatchConfig {
  int grid = 2048;
  int tiles_per_group = 2;
};

// One graph taking part in a batch.
struct Member {
  nd_graph *g = nullptr;
  void *user = nullptr;
  int64_t t0 = 0;
  int64_t max_local = 0;
  int64_t sweeps = 0;
  bool converged = false;
  bool finished = false;
  int slot = -1;          // index in the device descriptor table
  int64_t ntiles = 0;     // tiles it contributes
  // one allocation: the values, slack words, and from `zero` on what starts
  // out cleared
  DArr<uint8_t> mem;
  uint8_t *tau[2] = {nullptr, nullptr};  // AND: the second is NULL
  uint8_t *slack = nullptr;              // support counting, or NULL
  uint8_t *zero = nullptr;
  int64_t zero_bytes = 0;                // a multiple of 16
  SweepStats *ring = nullptr;
  uint8_t *act[2] = {nullptr, nullptr};  // frontier: flags, or counters
  uint8_t *sum[2] = {nullptr, nullptr};  // one stamp per 64 r-cliques
  int lost_shift = 0;
};

class Batch {
 public:
  static constexpr int kGraphEpochs = 8;  // epochs per HIP graph

  // Work is issued on a private stream ordered after `caller`.  `support`:
  // members may count support, where that has room (see add).
  Batch(nd_ctx *ctx, nd_kind kind, nd_mode mode, bool tau16, bool frontier,
        bool support, hipStream_t caller);
  ~Batch();
  Batch(const Batch &) = delete;
  Batch &operator=(const Batch &) = delete;

  // Add a prepared graph; it starts at the current epoch.
  Member *add(nd_graph *g, int32_t max_iters, void *user);
  // Drop finished members (their memory is released by the caller).
  std::vector<std::unique_ptr<Member>> take_finished();
  void run_epochs(int count);
  // Update sweeps/converged/finished of every member from the device.
  void poll(int epochs_run);
  // Pick tile and grid sizes (cached per shape).  Returns the number of
  // real epochs it ran (0 or 1), which the caller then polls.
  int autotune();
  static constexpr float kTuneSkipMs = 2.0f;
  const void *result_tau(const Member &m) const;
  bool tau16() const { return tau16_; }
  bool frontier() const { return frontier_; }
  nd_kind kind() const { return kind_; }
  nd_mode mode() const { return mode_; }
  hipStream_t stream() const { return s_; }
  size_t size() const { return members_.size(); }
  // Epochs run so far (the next epoch's number).
  int64_t epoch() const { return epoch_; }
  // Members still being swept (not finished).
  std::vector<Member *> live() const {
    std::vector<Member *> v;
    for (auto &m : members_)
      if (!m->finished) v.push_back(m.get());
    return v;
  }
  bool use_graph = true;
  float tuned_ms = 0;
  BatchConfig config() const { return cfg_; }
  static BatchConfig default_config(nd_ctx *ctx);

 private:
  void init_member_tau(Member &m);
  void rebuild();
  void upload_state(int64_t epoch);
  void set_config(const BatchConfig &c);
  void launch_epoch();
  void build_graph();
  void drop_graph();

  nd_ctx *ctx_;
  nd_kind kind_;
  nd_mode mode_;
  bool tau16_;
  bool frontier_;
  bool support_;
  hipStream_t s_ = nullptr;
  BatchConfig cfg_;
  std::vector<std::unique_ptr<Member>> members_;
  // launch state, graph table and tile table, one buffer filled by one copy
  DArr<uint8_t> tables_;
  BState *state_ = nullptr;
  BGraph *gs_ = nullptr;
  BTile *tiles_ = nullptr;
  DArr<int64_t> poll_buf_;
  int64_t gs_cap_ = 0, tiles_cap_ = 0;  // tiles_cap_: also the sweep's grid
  int ntiles_ = 0, ng_ = 0;
  int64_t work_ = 0;
  int64_t epoch_ = 0;
  int64_t dead_tiles_ = 0;  // tiles of finished members still in the table
  bool dirty_ = true;
  hipGraphExec_t graph_exec_ = nullptr;
};

}  // namespace nd
