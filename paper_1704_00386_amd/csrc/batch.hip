// batch.hip -- many graphs swept together.
//
// Every graph of a batch keeps its own internal numbering, incidence lists,
// tau buffers and per-sweep counters.  Their r-cliques are cut into tiles
// (graph, bin, id range) that form one combined work list; one epoch is one
// sweep of every graph still running, one workgroup per tile, heaviest
// tiles first (dispatched first, so the tail of an epoch is short).  A
// graph whose
// previous sweep changed nothing is skipped tile by tile and dropped from the
// table at the next poll; graphs may join at any epoch (the server uses
// this), each counting its own sweeps from the epoch it joined.  All launch
// arguments are fixed device pointers and grid sizes -- the epoch number and
// table sizes live in device memory -- so a chunk of epochs is built once
// in a HIP graph and replayed until the table outgrows its buffers.
//
// Tile sizes come from a small autotuner, cached by (kind, mode,
// tau width, frontier, work bucket): a batch whose first sweep is short
// (launch-bound) times one trial sweep per candidate on scratch state and
// keeps the fastest; a longer one keeps the default, since there the
// configuration hardly matters and each trial would cost a whole sweep.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <deque>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include "api_util.h"
#include "batch.h"
#include "sweep_dev.h"

namespace nd {

namespace {

using namespace dev;

// r-cliques of one pass of a 256-thread workgroup, per bin type.
__host__ __device__ constexpr int rclq_per_pass(int type) {
  return type == kBinG1 ? 256
         : type == kBinG4 ? 64
         : type == kBinG16 ? 16
         : type >= kBinWave16 ? 4
                              : 1;
}

// Largest incidence count of one pass, in units of 1024 (hubs: a round one).
constexpr int pass_units(int type) {
  return type == kBinBlock ? 4 : type == kBinWave ? 2 : type == kBinWave16 ? 4
         : type == kBinWave8 ? 2 : 1;
}

// A tile's work at most.  With two tiles a resident workgroup a batch of large
// graphs ends each epoch on a partly filled round of long tiles (four k-trusses
// of 500,000 edges with lists of 590: 280 ms in tiles of 290 units, 251 of 64,
// 244 of 16; 16 gained nothing more on two of 10^6 edges with lists of 1200, 373 /
// 331 / 326 ms, and lost 4% in AND).
constexpr int64_t kMaxUnits = 64;

// After an epoch, one workgroup: each graph's changed total (read by its
// tiles of the next epoch and by the poll), the next sweep's counters
// cleared, the epoch advanced.  16 lanes a graph, one counter part each.
constexpr int kStepThreads = 1024;
static_assert(kStatParts == 16, "one lane per counter part");

__global__ __launch_bounds__(kStepThreads) void k_epoch_step(
    const BGraph *__restrict__ gs, BState *__restrict__ st) {
  const int64_t e = st->epoch;
  const int ng = st->ng;
  const int part = threadIdx.x % kStatParts;
  for (int i = threadIdx.x / kStatParts; i < ng; i += kStepThreads / kStatParts) {
    const int64_t local = e - gs[i].t0;
    if (local < 0 || local >= gs[i].max_local) continue;  // uniform over the 16
    SweepStats &z = gs[i].ring[local % kBatchRing];
    SweepStats &next = gs[i].ring[(local + 1) % kBatchRing];
    unsigned long long c = z.part[part].changed;
#pragma unroll
    for (int off = kStatParts / 2; off > 0; off >>= 1) c += __shfl_xor(c, off, kStatParts);
    next.part[part].changed = 0;
    next.part[part].evaluated = 0;
    if (part == 0) {
      z.total = c;
      next.notified = 0;
      next.total = 0;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) st->epoch = e + 1;
}

// How far each graph got in the last `n` epochs (ending before `e_end`): 2 x
// its sweeps so far, plus 1 when the last of them changed nothing; 0 when it
// ran none of them.
__global__ void k_collect(const BGraph *__restrict__ gs, int ng, int64_t e_end,
                          int n, int64_t *__restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ng) return;
  int64_t r = 0;
  for (int q = 0; q < n && !(r & 1); q++) {
    const int64_t local = e_end - n + q - gs[i].t0;
    if (local >= 0 && local < gs[i].max_local)
      r = 2 * (local + 1) + (gs[i].ring[local % kBatchRing].total == 0);
  }
  out[i] = r;
}

// A member's start: tau_0 = d_s in its one or two arrays; no counts, stamps
// or losses.
template <typename T>
__global__ __launch_bounds__(256) void k_member_init(
    const int32_t *__restrict__ ds, int64_t nr, T *__restrict__ tau0,
    T *__restrict__ tau1, uint4 *__restrict__ zero, int64_t nzero) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = t0; i < nr; i += stride) {
    const T v = (T)ds[i];
    tau0[i] = v;
    if (tau1 != nullptr) tau1[i] = v;
  }
  for (int64_t i = t0; i < nzero; i += stride) zero[i] = make_uint4(0, 0, 0, 0);
}

struct TuneKey {
  int kind, mode, t16, fr, bucket;
  bool operator<(const TuneKey &o) const {
    return std::tie(kind, mode, t16, fr, bucket) <
           std::tie(o.kind, o.mode, o.t16, o.fr, o.bucket);
  }
};
std::mutex g_tune_mu;
std::map<TuneKey, BatchConfig> g_tune_cache;

int work_bucket(int64_t P) {
  int b = 0;
  while (P > 1) {
    P >>= 1;
    b++;
  }
  return b;
}

}  // namespace

// ------------------------------------------------------------ Batch

Batch::Batch(nd_ctx *ctx, nd_kind kind, nd_mode mode, bool tau16,
             bool frontier, bool support, hipStream_t caller)
    : ctx_(ctx), kind_(kind), mode_(mode), tau16_(tau16), frontier_(frontier),
      support_(support) {
  cfg_ = default_config(ctx);
  if (const char *v = getenv("ND_BATCH_NO_GRAPH")) use_graph = v[0] != '1';
  ND_HIP(hipStreamCreateWithFlags(&s_, hipStreamNonBlocking));
  hipEvent_t ev;
  ND_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
  ND_HIP(hipEventRecord(ev, caller));
  ND_HIP(hipStreamWaitEvent(s_, ev, 0));
  (void)hipEventDestroy(ev);
  StreamScope scope(s_);
}

Batch::~Batch() {
  (void)hipStreamSynchronize(s_);
  drop_graph();
  {
    StreamScope scope(s_);
    members_.clear();
    tables_.free();
    poll_buf_.free();
  }
  ctx_->alloc.forget_stream(s_);
  (void)hipStreamDestroy(s_);
}

void Batch::drop_graph() {
  if (graph_exec_) {
    (void)hipGraphExecDestroy(graph_exec_);
    graph_exec_ = nullptr;
  }
}

BatchConfig Batch::default_config(nd_ctx *ctx) {
  BatchConfig c;
  c.grid = ctx->num_cu * 8;
  c.tiles_per_group = 2;
  return c;
}

Member *Batch::add(nd_graph *g, int32_t max_iters, void *user) {
  StreamScope scope(s_);
  KindState &ks = g->ks[kind_];
  ND_REQUIRE(ks.ready, ND_ERR_INVALID, "graph not prepared for the batch");
  ND_REQUIRE(ks.tau16 || !tau16_, ND_ERR_INVALID,
             "a 16-bit batch cannot hold a graph needing 32-bit tau");
  auto m = std::make_unique<Member>();
  m->g = g;
  m->user = user;
  m->t0 = epoch_;
  const int64_t cap = ks.nr + 1;  // Lemma 2: enough to observe convergence
  m->max_local = (max_iters < 0 || max_iters > cap) ? cap : max_iters;
  // The arrays in one block of memory: a batch of many small graphs would
  // spend milliseconds in allocations and fills of a few bytes.
  const int64_t nr = std::max<int64_t>(ks.nr, 1);
  const int64_t ng = (nr + (1 << kGroupShift) - 1) >> kGroupShift;
  auto place = [&](bool support) {
    int64_t at = 0;
    auto take = [&](int64_t bytes) {
      uint8_t *p = m->mem.p ? m->mem.p + at : nullptr;
      at += (bytes + 255) / 256 * 256;
      return p;
    };
    const int64_t tb = tau16_ ? 2 : 4;
    m->lost_shift = support ? lost_shift(ks) : 0;
    m->tau[0] = take(tb * nr);
    m->tau[1] = mode_ == ND_SND ? take(tb * nr) : nullptr;
    m->slack = support ? take(tb * nr) : nullptr;
    const int64_t z = at;
    m->ring = (SweepStats *)take((int64_t)sizeof(SweepStats) * kBatchRing);
    if (frontier_)
      for (int i = 0; i < 2; i++) {
        m->act[i] = take(nr << m->lost_shift);
        m->sum[i] = take(ng);
      }
    m->zero = m->mem.p ? m->mem.p + z : nullptr;
    m->zero_bytes = at - z;
    return at;
  };
  // Counting support takes more memory than flags do: under a budget at most a
  // quarter of what is left, so that outputs and other work on the context keep
  // room.
  const Allocator &al = ctx_->alloc;
  const size_t live = al.live_bytes();
  bool support = support_ && frontier_ && counts_support(ks) &&
                 (al.budget() == 0 ||
                  (live < al.budget() && (size_t)place(true) <= (al.budget() - live) / 4));
  if (support) {
    try {
      m->mem.reset(ctx_->alloc, place(true));
    } catch (const Err &e) {
      if (e.code != ND_ERR_OOM) throw;
      clear_error();
      support = false;
    }
  }
  if (!support) m->mem.reset(ctx_->alloc, place(false));
  place(support);
  init_member_tau(*m);
  if (ks.nr == 0 || m->max_local == 0) {
    m->finished = true;
    m->converged = ks.nr == 0;
  }
  Member *raw = m.get();
  members_.push_back(std::move(m));
  dirty_ = true;
  return raw;
}

void Batch::init_member_tau(Member &m) {
  const KindState &ks = m.g->ks[kind_];
  if (ks.nr == 0) return;
  const unsigned grid = (unsigned)std::min<int64_t>(
      grid_for(std::max<int64_t>(ks.nr, m.zero_bytes / 16), 256), 4096);
  if (tau16_)  // ks.tau16 holds (checked in add)
    k_member_init<uint16_t><<<grid, 256, 0, s_>>>(
        ks.ds.p, ks.nr, (uint16_t *)m.tau[0], (uint16_t *)m.tau[1],
        (uint4 *)m.zero, m.zero_bytes / 16);
  else
    k_member_init<int32_t><<<grid, 256, 0, s_>>>(
        ks.ds.p, ks.nr, (int32_t *)m.tau[0], (int32_t *)m.tau[1],
        (uint4 *)m.zero, m.zero_bytes / 16);
  ND_LAUNCHED();
}

std::vector<std::unique_ptr<Member>> Batch::take_finished() {
  std::vector<std::unique_ptr<Member>> out;
  std::vector<std::unique_ptr<Member>> keep;
  for (auto &m : members_)
    (m->finished ? out : keep).push_back(std::move(m));
  members_ = std::move(keep);
  if (!out.empty()) dirty_ = true;
  return out;
}

void Batch::rebuild() {
  StreamScope scope(s_);
  std::vector<BGraph> hg;
  std::vector<BTile> ht[kBinZero];  // per bin type; heaviest bins first
  int64_t work = 0;
  // Tile length: tiles hold about equal work bounds (pass_units) and an
  // epoch has about grid * tiles_per_group of them -- each a workgroup of
  // its own -- but never less than one block pass.
  int64_t units_total = 0;
  for (auto &mp : members_) {
    if (mp->finished) continue;
    const KindState &ks = mp->g->ks[kind_];
    for (int b = kBinBlock; b < kBinZero; b++)
      units_total += (ks.bin_hi[b] - ks.bin_lo[b] + rclq_per_pass(b) - 1) /
                     rclq_per_pass(b) * pass_units(b);
  }
  const int64_t target = (int64_t)cfg_.grid * cfg_.tiles_per_group;
  const int64_t units = std::min(
      kMaxUnits, std::max<int64_t>(1, units_total / std::max<int64_t>(target, 1)));
  for (auto &mp : members_) {
    Member &m = *mp;
    m.slot = -1;
    m.ntiles = 0;
    if (m.finished) continue;
    const KindState &ks = m.g->ks[kind_];
    const int32_t gi = (int32_t)hg.size();
    m.slot = gi;
    BGraph G{};
    G.inc_off = ks.inc_off.p;
    G.inc_ids = ks.inc_ids.p;
    G.tau[0] = m.tau[0];
    G.tau[1] = mode_ == ND_SND ? m.tau[1] : m.tau[0];
    G.ring = m.ring;
    G.t0 = m.t0;
    G.max_local = m.max_local;
    if (frontier_) {
      for (int i = 0; i < 2; i++) {
        G.act[i] = m.act[i];
        G.act_sum[i] = m.sum[i];
      }
      G.slack = m.slack;
      G.lost_shift = m.lost_shift;
      // (an epoch sweeps every member: the gathers of many graphs)
      const int div = frontier_switch(notifies_late(ks, INT64_MAX));
      G.notify_below = div <= 0 ? ~0ull
                                : (unsigned long long)(ks.bin_lo[kBinZero] / div);
    }
    hg.push_back(G);
    work += ks.P;
    for (int b = kBinBlock; b < kBinZero; b++) {
      const int64_t lo = ks.bin_lo[b], hi = ks.bin_hi[b];
      int64_t passes = std::max<int64_t>(1, units / pass_units(b));
      // whole runs of the flat sweep (4 passes) where a tile has several
      if (b >= kBinG64 && passes > 4) passes = passes / 4 * 4;
      const int64_t step = (int64_t)rclq_per_pass(b) * passes;
      for (int64_t x = lo; x < hi; x += step) {
        ht[b].push_back(BTile{gi, b, x, std::min(hi, x + step)});
        m.ntiles++;
      }
    }
  }
  int64_t nt = 0;
  for (int b = kBinBlock; b < kBinZero; b++) nt += (int64_t)ht[b].size();
  ntiles_ = (int)nt;
  ng_ = (int)hg.size();
  work_ = work;
  dead_tiles_ = 0;
  // Grow the device tables (capacities double); a new buffer, or a larger
  // grid, invalidates the epoch graph, whose kernel nodes hold them.
  if (tables_.p == nullptr || ng_ > gs_cap_ || nt > tiles_cap_) {
    if (ng_ > gs_cap_ || gs_cap_ == 0) gs_cap_ = std::max<int64_t>(std::max(ng_, 1), 2 * gs_cap_);
    if (nt > tiles_cap_ || tiles_cap_ == 0)
      tiles_cap_ = std::max<int64_t>(std::max<int64_t>(nt, 1), 2 * tiles_cap_);
    const int64_t gs_at = 256;
    const int64_t tiles_at = (gs_at + (int64_t)sizeof(BGraph) * gs_cap_ + 255) / 256 * 256;
    tables_.reset(ctx_->alloc, tiles_at + (int64_t)sizeof(BTile) * tiles_cap_);
    poll_buf_.reset(ctx_->alloc, gs_cap_);
    state_ = (BState *)tables_.p;
    gs_ = (BGraph *)(tables_.p + gs_at);
    tiles_ = (BTile *)(tables_.p + tiles_at);
    drop_graph();
  }
  // one copy: state, graphs, tiles heaviest bins first
  const size_t tiles_at = (uint8_t *)tiles_ - tables_.p;
  std::vector<uint8_t> host(tiles_at + sizeof(BTile) * (size_t)nt);
  const BState z{epoch_, ntiles_, ng_};
  memcpy(host.data(), &z, sizeof z);
  memcpy(host.data() + ((uint8_t *)gs_ - tables_.p), hg.data(), sizeof(BGraph) * hg.size());
  size_t at = tiles_at;
  for (int b = kBinBlock; b < kBinZero; b++) {
    if (ht[b].empty()) continue;
    memcpy(host.data() + at, ht[b].data(), sizeof(BTile) * ht[b].size());
    at += sizeof(BTile) * ht[b].size();
  }
  ND_HIP(hipMemcpyAsync(tables_.p, host.data(), host.size(), hipMemcpyHostToDevice, s_));
  ND_HIP(hipStreamSynchronize(s_));  // the host vectors go out of scope
  dirty_ = false;
}

void Batch::upload_state(int64_t epoch) {
  const BState z{epoch, ntiles_, ng_};
  ND_HIP(hipMemcpyAsync(state_, &z, sizeof z, hipMemcpyHostToDevice, s_));
  ND_HIP(hipStreamSynchronize(s_));
}

// The kernels of one epoch, in launch order, for the batch's instance.
struct EpochKernels {
  const void *fn[2];  // tiles, step
};

static EpochKernels epoch_kernels(int k, bool tau16, bool and_mode, bool fr) {
  const void *f = nullptr;
  switch (k * 2 + (tau16 ? 1 : 0)) {
    case 2: f = batch_kernel<1, int32_t>(and_mode, fr); break;
    case 3: f = batch_kernel<1, uint16_t>(and_mode, fr); break;
    case 4: f = batch_kernel<2, int32_t>(and_mode, fr); break;
    case 5: f = batch_kernel<2, uint16_t>(and_mode, fr); break;
    case 6: f = batch_kernel<3, int32_t>(and_mode, fr); break;
    case 7: f = batch_kernel<3, uint16_t>(and_mode, fr); break;
    case 10: f = batch_kernel<5, int32_t>(and_mode, fr); break;
    case 11: f = batch_kernel<5, uint16_t>(and_mode, fr); break;
    default:
      ND_REQUIRE(false, ND_ERR_INVALID, "no batch kernel for k=%d", k);
  }
  return {{f, (const void *)k_epoch_step}};
}

// Grid, block and arguments of kernel i of an epoch.  The argument values
// live in *this (table pointers), so `args` stays valid while they do.
struct EpochLaunch {
  const BGraph *gs;
  const BTile *tiles;
  BState *st;
  void *a_tiles[3], *a_step[2];
  dim3 grid[2], block[2];
  void **args[2];
  EpochLaunch(const BGraph *g, const BTile *t, BState *s, int64_t tile_grid)
      : gs(g), tiles(t), st(s) {
    a_tiles[0] = &gs;
    a_tiles[1] = &tiles;
    a_tiles[2] = &st;
    a_step[0] = &gs;
    a_step[1] = &st;
    args[0] = a_tiles;
    args[1] = a_step;
    grid[0] = dim3((unsigned)tile_grid);
    grid[1] = dim3(1);
    block[0] = dim3(256);
    block[1] = dim3(kStepThreads);
  }
  EpochLaunch(const EpochLaunch &) = delete;
};

void Batch::launch_epoch() {
  const EpochKernels ek =
      epoch_kernels(kind_rs(kind_).k, tau16_, mode_ == ND_AND, frontier_);
  EpochLaunch el(gs_, tiles_, state_, tiles_cap_);
  for (int i = 0; i < 2; i++) {
    ND_HIP(hipLaunchKernel(ek.fn[i], el.grid[i], el.block[i], el.args[i], 0, s_));
  }
}

// Build kGraphEpochs epochs as a HIP graph, node by node (no stream
// capture, so other threads stay free to use any stream, the legacy one
// included, while it is built); on failure this batch launches its epochs
// directly from then on.
void Batch::build_graph() {
  const EpochKernels ek =
      epoch_kernels(kind_rs(kind_).k, tau16_, mode_ == ND_AND, frontier_);
  EpochLaunch el(gs_, tiles_, state_, tiles_cap_);
  hipGraph_t gr = nullptr;
  bool ok = hipGraphCreate(&gr, 0) == hipSuccess;
  hipGraphNode_t prev = nullptr;
  for (int e = 0; ok && e < kGraphEpochs; e++)
    for (int i = 0; ok && i < 2; i++) {
      hipKernelNodeParams np{};
      np.func = const_cast<void *>(ek.fn[i]);
      np.gridDim = el.grid[i];
      np.blockDim = el.block[i];
      np.sharedMemBytes = 0;
      np.kernelParams = el.args[i];
      np.extra = nullptr;
      hipGraphNode_t node = nullptr;
      ok = hipGraphAddKernelNode(&node, gr, prev ? &prev : nullptr, prev ? 1 : 0,
                                 &np) == hipSuccess;
      prev = node;
    }
  if (ok && hipGraphInstantiate(&graph_exec_, gr, nullptr, nullptr, 0) != hipSuccess) {
    graph_exec_ = nullptr;
    ok = false;
  }
  if (gr) (void)hipGraphDestroy(gr);
  if (!ok) {
    (void)hipGetLastError();
    graph_exec_ = nullptr;
    use_graph = false;
  }
}

void Batch::run_epochs(int count) {
  if (dirty_) rebuild();
  if (ng_ == 0) return;
  if (use_graph && count == kGraphEpochs && !graph_exec_) build_graph();
  if (use_graph && count == kGraphEpochs && graph_exec_) {
    ND_HIP(hipGraphLaunch(graph_exec_, s_));
  } else {
    for (int i = 0; i < count; i++) launch_epoch();
  }
  epoch_ += count;
}

void Batch::poll(int epochs_run) {
  if (ng_ == 0 || epochs_run <= 0) return;
  ND_REQUIRE(epochs_run <= kPollMax, ND_ERR_INVALID, "poll window too large");
  k_collect<<<grid_for(ng_, 256), 256, 0, s_>>>(gs_, ng_, epoch_, epochs_run,
                                                 poll_buf_.p);
  ND_LAUNCHED();
  PinnedChunk pc;
  std::vector<int64_t> many;
  const int64_t *h;
  if (sizeof(int64_t) * ng_ <= PinnedChunk::kBytes) {
    h = pc.read(poll_buf_.p, (size_t)ng_, s_);
  } else {
    many.resize(ng_);
    ND_HIP(hipMemcpyAsync(many.data(), poll_buf_.p, sizeof(int64_t) * many.size(),
                          hipMemcpyDeviceToHost, s_));
    ND_HIP(hipStreamSynchronize(s_));
    h = many.data();
  }
  for (auto &mp : members_) {
    Member &m = *mp;
    if (m.finished || m.slot < 0) continue;
    const int64_t v = h[m.slot];
    if (v != 0) m.sweeps = v / 2;
    if (v & 1) {
      m.converged = true;
      m.finished = true;
    }
    if (!m.finished && m.sweeps >= m.max_local) m.finished = true;
    if (m.finished) dead_tiles_ += m.ntiles;
  }
  // drop finished graphs' tiles once they are a quarter of the table
  if (dead_tiles_ * 4 > ntiles_ && dead_tiles_ > 0) dirty_ = true;
}

const void *Batch::result_tau(const Member &m) const {
  return m.tau[mode_ == ND_SND ? m.sweeps & 1 : 0];
}

void Batch::set_config(const BatchConfig &c) {
  if (c.grid != cfg_.grid || c.tiles_per_group != cfg_.tiles_per_group) {
    cfg_ = c;
    dirty_ = true;
    drop_graph();
  }
}

// Pick the launch configuration.  The first epoch runs under the default
// configuration and counts as a real sweep; if it took kTuneSkipMs or more
// the batch is in the bandwidth-bound regime where the configuration hardly
// matters, and the default is kept (trials would cost whole sweeps).  A
// shorter (launch-bound) batch times one trial epoch per candidate on
// scratch state, then restores tau_0 and the epoch, so no epoch counts.
// Returns the real epochs run (0 or 1); the caller polls them.
int Batch::autotune() {
  StreamScope scope(s_);
  if (dirty_) rebuild();
  if (ng_ == 0) return 0;
  TuneKey key{(int)kind_, (int)mode_, tau16_ ? 1 : 0, frontier_ ? 1 : 0,
              work_bucket(work_)};
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune_cache.find(key);
    if (it != g_tune_cache.end()) {
      set_config(it->second);
      return 0;
    }
  }
  hipEvent_t a, b;
  ND_HIP(hipEventCreate(&a));
  ND_HIP(hipEventCreate(&b));
  auto time_epoch = [&]() {
    ND_HIP(hipEventRecord(a, s_));
    launch_epoch();
    ND_HIP(hipEventRecord(b, s_));
    ND_HIP(hipEventSynchronize(b));
    float ms = 0;
    ND_HIP(hipEventElapsedTime(&ms, a, b));
    return ms;
  };
  const int64_t e0 = epoch_;
  const BatchConfig dflt = default_config(ctx_);
  set_config(dflt);
  if (dirty_) rebuild();
  const float first = time_epoch();
  int real = 0;
  BatchConfig best_cfg = dflt;
  float best = first;
  if (first >= kTuneSkipMs) {
    epoch_ += 1;
    real = 1;
  } else {
    const int cus = ctx_->num_cu;
    for (int gm : {4, 8, 16})
      for (int tpg : {1, 4}) {
        BatchConfig c;
        c.grid = cus * gm;
        c.tiles_per_group = tpg;
        set_config(c);
        rebuild();
        upload_state(e0);
        const float ms = time_epoch();
        if (ms < best) {
          best = ms;
          best_cfg = c;
        }
      }
    for (auto &mp : members_) init_member_tau(*mp);
    set_config(best_cfg);
    rebuild();
    upload_state(e0);
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  tuned_ms = best;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune_cache[key] = best_cfg;
  return real;
}

// ------------------------------------------------------- batch ABI

constexpr int kPrepThreads = 2;

int prep_threads() {
  static const int n = [] {
    const char *v = getenv("ND_PREP_THREADS");
    const int x = v ? atoi(v) : kPrepThreads;
    return x < 1 ? 1 : x > 16 ? 16 : x;
  }();
  return n;
}

namespace {

// Prepares graphs for one kind on up to prep_threads() host threads, each
// with a stream of its own ordered after the caller's, largest graphs first
// (their sweeps are the longest, so they should start first).  Each
// prepared graph is handed to the consumer with an event recorded after its
// work, so the consumer's stream can wait for exactly that graph; the
// short, launch-bound build phases of different graphs overlap each other
// and the consumer's sweeps.
class PrepPool {
 public:
  PrepPool(nd_ctx *ctx, int32_t count, nd_graph *const *graphs, nd_kind kind,
           hipStream_t after)
      : ctx_(ctx), kind_(kind) {
    for (int i = 0; i < count; i++)
      if (!graphs[i]->ks[kind].ready &&
          std::find(todo_.begin(), todo_.end(), graphs[i]) == todo_.end())
        todo_.push_back(graphs[i]);
    std::stable_sort(todo_.begin(), todo_.end(),
                     [](const nd_graph *a, const nd_graph *b) { return a->nnz > b->nnz; });
    if (todo_.empty()) return;
    const int nt = (int)std::min<size_t>(prep_threads(), todo_.size());
    hipEvent_t start;
    ND_HIP(hipEventCreateWithFlags(&start, hipEventDisableTiming));
    ND_HIP(hipEventRecord(start, after));
    for (int t = 0; t < nt; t++) {
      hipStream_t st = nullptr;
      const hipError_t e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
      if (e != hipSuccess) {
        (void)hipEventDestroy(start);
        ND_HIP(e);
      }
      streams_.push_back(st);
      ND_HIP(hipStreamWaitEvent(st, start, 0));
    }
    (void)hipEventDestroy(start);
    for (int t = 0; t < nt; t++) threads_.emplace_back([this, t] { run(t); });
  }

  ~PrepPool() {
    {
      std::lock_guard<std::mutex> lk(mu_);
      failed_ = true;  // stop taking graphs
    }
    join();
    for (auto &d : done_) (void)hipEventDestroy(d.second);
    for (hipStream_t st : streams_) {
      ctx_->alloc.forget_stream(st);
      (void)hipStreamDestroy(st);
    }
  }

  int pending() const { return (int)todo_.size(); }

  // The next prepared graph and its event (owned by the caller).  Waits for
  // one when `block`; returns false when none is ready (not blocking), when
  // every graph has been handed out, or after a failure (see rethrow).
  bool next(bool block, nd_graph **g, hipEvent_t *ev) {
    std::unique_lock<std::mutex> lk(mu_);
    if (block)
      cv_.wait(lk, [&] { return !done_.empty() || failed_ || handed_ == todo_.size(); });
    if (done_.empty()) return false;
    *g = done_.front().first;
    *ev = done_.front().second;
    done_.pop_front();
    handed_++;
    return true;
  }

  // Every graph handed out.
  bool finished() {
    std::lock_guard<std::mutex> lk(mu_);
    return handed_ == todo_.size();
  }

  // A preparation failed (finish() throws it).
  bool failed() {
    std::lock_guard<std::mutex> lk(mu_);
    return code_ != ND_OK;
  }

  // Join the threads; make `s` wait for every preparation stream; throw the
  // first failure.
  void finish(hipStream_t s) {
    join();
    for (hipStream_t st : streams_) {
      hipEvent_t d;
      ND_HIP(hipEventCreateWithFlags(&d, hipEventDisableTiming));
      ND_HIP(hipEventRecord(d, st));
      ND_HIP(hipStreamWaitEvent(s, d, 0));
      (void)hipEventDestroy(d);
    }
    rethrow();
  }

  void rethrow() {
    std::lock_guard<std::mutex> lk(mu_);
    if (code_ != ND_OK) {
      set_error("%s", msg_.c_str());
      throw Err(code_);
    }
  }

 private:
  void join() {
    for (auto &th : threads_)
      if (th.joinable()) th.join();
  }

  void run(int t) {
    try {
      ND_HIP(hipSetDevice(ctx_->device));
      StreamScope scope(streams_[t]);
      for (;;) {
        nd_graph *g;
        {
          std::lock_guard<std::mutex> lk(mu_);
          if (failed_ || next_ == todo_.size()) return;
          g = todo_[next_++];
        }
        prepare(g, kind_, streams_[t]);
        hipEvent_t ev;
        ND_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        const hipError_t e = hipEventRecord(ev, streams_[t]);
        if (e != hipSuccess) {
          (void)hipEventDestroy(ev);
          ND_HIP(e);
        }
        std::lock_guard<std::mutex> lk(mu_);
        done_.emplace_back(g, ev);
        cv_.notify_all();
      }
    } catch (const Err &e) {
      fail(e.code, nd_last_error());
    } catch (const std::exception &e) {
      fail(ND_ERR_DEVICE, e.what());
    }
  }

  void fail(nd_status code, const std::string &msg) {
    std::lock_guard<std::mutex> lk(mu_);
    if (code_ == ND_OK) {
      code_ = code;
      msg_ = msg;
    }
    failed_ = true;
    cv_.notify_all();
  }

  nd_ctx *ctx_;
  nd_kind kind_;
  std::vector<nd_graph *> todo_;
  std::vector<hipStream_t> streams_;
  std::vector<std::thread> threads_;
  std::mutex mu_;
  std::condition_variable cv_;
  std::deque<std::pair<nd_graph *, hipEvent_t>> done_;
  size_t next_ = 0, handed_ = 0;
  bool failed_ = false;
  nd_status code_ = ND_OK;
  std::string msg_;
};

}  // namespace

void prepare_many(nd_ctx *ctx, int32_t count, nd_graph *const *graphs,
                  nd_kind kind, hipStream_t s) {
  PrepPool pool(ctx, count, graphs, kind, s);
  nd_graph *g;
  hipEvent_t ev;
  while (pool.next(true, &g, &ev)) (void)hipEventDestroy(ev);
  pool.finish(s);
}

// Incidence entries the live graphs must hold before sweeps run while
// other graphs are still being prepared.  Shorter epochs would mostly add
// launches and polls beside the preparation threads' own (whose build
// phases are launch-bound), slowing them more than the overlap gains.
constexpr int64_t kOverlapWork = (int64_t)1 << 24;

// The batched decomposition.  Graphs not yet prepared are prepared by a
// PrepPool while the graphs already prepared are being swept (once their
// sweeps are long enough, kOverlapWork): each joins the batch of its tau
// width (16 or 32 bits; two batches, on streams of their own, when the
// graphs need both) as soon as it is ready.
static nd_status batch_attempt(nd_ctx *ctx, int32_t count, nd_graph *const *graphs,
                               nd_kind kind, const nd_opts &opts,
                               int32_t *const *kappas, int on_device, hipStream_t s,
                               nd_result *res, const std::vector<bool> &ready0,
                               bool support) {
  std::vector<bool> was(count);  // prepared by now
  for (int i = 0; i < count; i++) was[i] = graphs[i]->ks[kind].ready;
  std::unique_ptr<Batch> batches[2];  // 16-bit, 32-bit tau
  bool tuned[2] = {false, false};
  std::map<nd_graph *, Member *> member;
  struct Events {  // the call's timing events, released on every exit
    hipEvent_t a = nullptr, b = nullptr;
    ~Events() {
      if (a) (void)hipEventDestroy(a);
      if (b) (void)hipEventDestroy(b);
    }
  } evs;
  ND_HIP(hipEventCreate(&evs.a));
  ND_HIP(hipEventCreate(&evs.b));
  hipEvent_t a = evs.a, b = evs.b;
  ND_HIP(hipEventRecord(a, s));
  auto join = [&](nd_graph *g, hipEvent_t ready) {
    const int w = g->ks[kind].tau16 ? 0 : 1;
    if (!batches[w])
      batches[w] = std::make_unique<Batch>(ctx, kind, opts.mode, w == 0,
                                           opts.use_frontier != 0, support, s);
    if (ready) ND_HIP(hipStreamWaitEvent(batches[w]->stream(), ready, 0));
    member[g] = batches[w]->add(g, opts.max_iters, nullptr);
  };
  {
    PrepPool pool(ctx, count, graphs, kind, s);
    Phase sweep_phase("nd.batch.sweeps");
    for (int i = 0; i < count; i++)
      if (was[i] && !member.count(graphs[i])) join(graphs[i], nullptr);
    int chunk = 2;
    while (!pool.failed()) {
      auto live_work = [&] {
        int64_t w = 0;
        for (auto &bt : batches)
          if (bt)
            for (Member *m : bt->live()) w += std::max<int64_t>(m->g->ks[kind].P, 1);
        return w;
      };
      int64_t work = live_work();
      // newcomers; wait for one while the sweeps would be too short to
      // overlap the preparations usefully
      nd_graph *g;
      hipEvent_t ev;
      while (pool.next(work < kOverlapWork && !pool.finished(), &g, &ev)) {
        try {
          join(g, ev);
        } catch (...) {
          (void)hipEventDestroy(ev);
          throw;
        }
        (void)hipEventDestroy(ev);
        work = live_work();
      }
      if (work == 0) {
        if (pool.finished()) break;
        continue;
      }
      int ran[2] = {0, 0};
      for (int w = 0; w < 2; w++) {
        if (!batches[w] || batches[w]->live().empty()) continue;
        if (!tuned[w]) {  // its first epoch, or trial epochs on scratch state
          ran[w] = batches[w]->autotune();
          tuned[w] = true;
        } else {
          batches[w]->run_epochs(chunk);
          ran[w] = chunk;
        }
      }
      for (int w = 0; w < 2; w++)
        if (ran[w]) batches[w]->poll(ran[w]);
      chunk = std::min(chunk * 2, Batch::kGraphEpochs);
    }
    pool.finish(s);
  }
  for (auto &bt : batches)
    if (bt) {
      hipEvent_t d;
      ND_HIP(hipEventCreateWithFlags(&d, hipEventDisableTiming));
      ND_HIP(hipEventRecord(d, bt->stream()));
      ND_HIP(hipStreamWaitEvent(s, d, 0));
      (void)hipEventDestroy(d);
    }
  ND_HIP(hipEventRecord(b, s));
  ND_HIP(hipEventSynchronize(b));
  float ms_total = 0;
  ND_HIP(hipEventElapsedTime(&ms_total, a, b));
  nd_status out = ND_OK;
  for (int i = 0; i < count; i++) {
    const Member &m = *member.at(graphs[i]);
    const KindState &ks = graphs[i]->ks[kind];
    const Batch &bt = *batches[ks.tau16 ? 0 : 1];
    hipStream_t bs = bt.stream();
    StreamScope scope(bs);
    if (ks.nr > 0) {
      ND_REQUIRE(kappas && kappas[i], ND_ERR_INVALID, "kappas[%d] is NULL", i);
      if (on_device) {
        to_original(ks, bt.result_tau(m), bt.tau16() ? 2 : 4, kappas[i], bs);
      } else {
        DArr<int32_t> tmp(ctx->alloc, ks.nr);
        to_original(ks, bt.result_tau(m), bt.tau16() ? 2 : 4, tmp.p, bs);
        ND_HIP(hipMemcpyAsync(kappas[i], tmp.p, sizeof(int32_t) * ks.nr,
                              hipMemcpyDeviceToHost, bs));
        ND_HIP(hipStreamSynchronize(bs));
      }
    }
    if (res) {
      nd_result &r = res[i];
      memset(&r, 0, sizeof r);
      r.sweeps = (int32_t)m.sweeps;
      r.converged = m.converged ? 1 : 0;
      r.n_rcliques = ks.nr;
      r.n_incidence = ks.P;
      r.updates = ks.bin_lo[kBinZero] * m.sweeps;
      r.ms_prep = ready0[i] ? 0.0 : ks.ms_prep;
      r.ms_iterate = ms_total;  // shared by the whole batch
      r.max_sdegree = ks.max_ds;
      r.tau_bytes = bt.tau16() ? 2 : 4;
    }
    if (!m.converged) out = ND_ERR_NOT_CONVERGED;
  }
  for (auto &bt : batches)
    if (bt) {
      ND_HIP(hipStreamSynchronize(bt->stream()));
      hipEvent_t d;  // the caller's later work follows the output kernels
      ND_HIP(hipEventCreateWithFlags(&d, hipEventDisableTiming));
      ND_HIP(hipEventRecord(d, bt->stream()));
      ND_HIP(hipStreamWaitEvent(s, d, 0));
      (void)hipEventDestroy(d);
    }
  if (out != ND_OK) set_error("a graph of the batch stopped without converging");
  return out;
}

nd_status batch_decompose(nd_ctx *ctx, int32_t count, nd_graph *const *graphs,
                          nd_kind kind, const nd_opts *opts_in,
                          int32_t *const *kappas, int on_device, hipStream_t s,
                          nd_result *res) {
  nd_opts opts;
  nd_opts_init(&opts);
  if (opts_in) opts = *opts_in;
  ND_REQUIRE(opts.mode == ND_SND || opts.mode == ND_AND, ND_ERR_INVALID,
             "unknown mode");
  ND_REQUIRE(opts.on_iter == nullptr && opts.stop_active_ratio == 0,
             ND_ERR_UNSUPPORTED,
             "batched decomposition supports mode, max_iters and use_frontier");
  std::vector<bool> ready0(count);
  for (int i = 0; i < count; i++) {
    ND_REQUIRE(graphs[i] && graphs[i]->ctx == ctx, ND_ERR_INVALID,
               "graph %d is NULL or from another context", i);
    ready0[i] = graphs[i]->ks[kind].ready;
  }
  for (int i = 0; i < count; i++)  // outputs of graphs already prepared
    ND_REQUIRE(!ready0[i] || graphs[i]->ks[kind].nr == 0 || (kappas && kappas[i]),
               ND_ERR_INVALID, "kappas[%d] is NULL", i);
  const KindRS rs = kind_rs(kind);
  const bool support = opts.use_frontier != 0 && rs.s == rs.r + 1;
  try {
    return batch_attempt(ctx, count, graphs, kind, opts, kappas, on_device, s, res,
                         ready0, support);
  } catch (const Err &e) {
    if (e.code != ND_ERR_OOM || !support) throw;
  }
  // Whatever fits with flags alone runs: once more without support counting, the
  // memory of the first attempt given back.
  clear_error();
  ND_HIP(hipStreamSynchronize(s));
  for (int i = 0; i < count; i++)
    if (!graphs[i]->ks[kind].ready) graphs[i]->ks[kind] = KindState{};
  ctx->alloc.trim();
  return batch_attempt(ctx, count, graphs, kind, opts, kappas, on_device, s, res,
                       ready0, false);
}

}  // namespace nd

using namespace nd;

extern "C" nd_status nd_batch_decompose(nd_ctx *ctx, int32_t count,
                                        nd_graph *const *graphs, nd_kind kind,
                                        const nd_opts *opts,
                                        int32_t *const *kappas, int on_device,
                                        void *stream, nd_result *res) {
  nd_status out = ND_OK;
  nd_status st = guarded([&] {
    ND_REQUIRE(ctx, ND_ERR_INVALID, "ctx is NULL");
    ND_REQUIRE(count >= 0 && (count == 0 || graphs), ND_ERR_INVALID,
               "bad graph list");
    ND_REQUIRE(kind_valid(kind),
               ND_ERR_UNSUPPORTED, "unknown kind");
    ND_HIP(hipSetDevice(ctx->device));
    StreamScope scope((hipStream_t)stream);
    if (count == 0) return;
    out = batch_decompose(ctx, count, graphs, kind, opts, kappas, on_device,
                          (hipStream_t)stream, res);
  });
  return st != ND_OK ? st : out;
}

extern "C" nd_status nd_prepare_many(nd_ctx *ctx, int32_t count,
                                     nd_graph *const *graphs, nd_kind kind,
                                     void *stream) {
  return guarded([&] {
    ND_REQUIRE(ctx, ND_ERR_INVALID, "ctx is NULL");
    ND_REQUIRE(count >= 0 && (count == 0 || graphs), ND_ERR_INVALID,
               "bad graph list");
    ND_REQUIRE(kind_valid(kind), ND_ERR_UNSUPPORTED, "unknown kind");
    for (int i = 0; i < count; i++)
      ND_REQUIRE(graphs[i] && graphs[i]->ctx == ctx, ND_ERR_INVALID,
                 "graph %d is NULL or from another context", i);
    ND_HIP(hipSetDevice(ctx->device));
    StreamScope scope((hipStream_t)stream);
    prepare_many(ctx, count, graphs, kind, (hipStream_t)stream);
  });
}
