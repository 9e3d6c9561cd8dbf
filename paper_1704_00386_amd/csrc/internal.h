// internal.h -- library-internal types: context, caching allocator, graph
// state and the host entry points of each kernel family.  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <map>
#include <mutex>
#include <vector>

#include "common.h"

namespace nd {

// ------------------------------------------------------------ allocator

// The stream that work issued by the current thread is ordered on.  Set at
// every ABI entry (StreamScope); the allocator tags blocks with it.
hipStream_t current_stream();
struct StreamScope {
  hipStream_t prev;
  explicit StreamScope(hipStream_t s);
  ~StreamScope();
};

// Device allocator with a byte budget and a cache of freed blocks, so that
// repeated decompositions do not pay hipMalloc/hipFree (which synchronises the
// device) on every call.  A freed block remembers the stream it was last used
// on: the same stream may reuse it at once (stream order protects it), any
// other stream only after synchronising that stream.  Thread-safe.
class Allocator {
 public:
  Allocator(int device, size_t budget) : device_(device), budget_(budget) {}
  ~Allocator();
  void *alloc(size_t bytes);  // throws Err(ND_ERR_OOM)
  void release(void *p);      // back to the cache, tagged current_stream()
  void trim();                // return cached blocks to the device
  // Before destroying stream s: wait for it and mark its cached blocks free
  // for any stream (no handle of a destroyed stream is ever used again).
  void forget_stream(hipStream_t s);
  size_t live_bytes() const;
  size_t cached_bytes() const;
  size_t budget() const { return budget_; }
  int device() const { return device_; }

 private:
  struct Cached {
    void *p;
    hipStream_t s;
    bool idle;  // no pending work may touch it: reusable without a wait
  };
  void trim_locked();
  int device_;
  size_t budget_;
  mutable std::mutex mu_;
  std::map<void *, size_t> live_;
  std::multimap<size_t, Cached> cache_;
  size_t live_total_ = 0, cache_total_ = 0;
};

// Owning device array of T.
template <typename T>
struct DArr {
  T *p = nullptr;
  int64_t n = 0;
  Allocator *a = nullptr;
  DArr() = default;
  DArr(Allocator &al, int64_t count) { reset(al, count); }
  DArr(const DArr &) = delete;
  DArr &operator=(const DArr &) = delete;
  DArr(DArr &&o) noexcept : p(o.p), n(o.n), a(o.a) { o.p = nullptr; o.n = 0; }
  DArr &operator=(DArr &&o) noexcept {
    if (this != &o) {
      free();
      p = o.p; n = o.n; a = o.a;
      o.p = nullptr; o.n = 0;
    }
    return *this;
  }
  ~DArr() { free(); }
  void reset(Allocator &al, int64_t count) {
    free();
    a = &al;
    n = count;
    p = (T *)al.alloc(sizeof(T) * (size_t)(count > 0 ? count : 1));
  }
  void free() {
    if (p && a) a->release(p);
    p = nullptr;
    n = 0;
  }
  size_t bytes() const { return sizeof(T) * (size_t)(n > 0 ? n : 1); }
};

// -------------------------------------------------------------- context

}  // namespace nd

// A context lives until nd_ctx_destroy has been called and every graph made
// from it has been destroyed, whatever the order of those calls.
struct nd_ctx {
  int device = 0;
  nd::Allocator alloc;
  int num_cu = 256;
  // Made once at creation, so that the sweep loop creates nothing on the
  // host (nd_decompose_noalloc relies on it): the pinned read-back ring of
  // the sweep counters (kHostStatsRing entries) and the timing events of the
  // sweep loop (whole loop, one sweep).
  void *host_stats = nullptr;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  std::atomic<int> refs{1};    // the owner's reference + one per graph
  nd_ctx(int dev, size_t budget) : device(dev), alloc(dev, budget) {}
  ~nd_ctx() {
    if (host_stats) (void)hipHostFree(host_stats);
    for (hipEvent_t e : ev)
      if (e) (void)hipEventDestroy(e);
  }
  void retain() { refs.fetch_add(1); }
  void release() {
    if (refs.fetch_sub(1) == 1) delete this;
  }
};

namespace nd {

// ---------------------------------------------------------- sweep bins

// r-cliques are numbered internally by sweep bin, within a bin by id (k-truss:
// see build_layout), so every sweep bin is a contiguous range of internal ids, r-cliques that
// share vertices stay close together (their gathers hit nearby cache lines),
// and zero-degree r-cliques (never swept) sit at the end.  Bins in internal
// order, with their d_s ranges:
enum SweepBin : int {
  kBinBlock = 0,  // d_s >= 2048:  one workgroup per r-clique, LDS histogram
  kBinWave,       // 1025..2047:   the same; where it fills the GPU, a wave with
                  //               its values in registers (swept_apart) or, in
                  //               a batch, in LDS
  kBinWave16,     // 513..1024:    one wave, values in LDS (or registers, the same)
  kBinWave8,      // 257..512:     one wave, values in LDS
  kBinG64,        // 65..256:      one wave, 4 values per lane
  kBinG16,        // 17..64:       16 lanes
  kBinG4,         // 5..16:        4 lanes
  kBinG1,         // 1..4:         one lane
  kBinZero,       // 0:            tau stays 0
  kNumBins
};

// Per-kind state of a graph: internal numbering, incidence lists, schedule.
struct KindState {
  bool ready = false;
  int r = 0, s = 0, k = 0;  // k = C(s,r) - 1
  int64_t nr = 0;           // |R|
  int64_t P = 0;            // sum_R d_s(R)
  DArr<int32_t> perm;       // internal id -> r-clique id
  DArr<int32_t> inv;        // r-clique id -> internal id
  DArr<int32_t> ds;         // d_s, internal order
  // incidence, internal order and ids: r-clique i owns the s-cliques
  // inc_off[i] .. inc_off[i+1]; s-clique j lists inc_ids[k*j .. k*j+k)
  DArr<int64_t> inc_off;
  DArr<int32_t> inc_ids;
  int64_t bin_lo[kNumBins] = {0}, bin_hi[kNumBins] = {0};
  int32_t max_ds = 0;
  bool tau16 = false;       // tau fits uint16 (max d_s < 32768)
  // bytes per tau value in the one-graph sweeps: 1 (max d_s < 256), 2 or 4
  // (batches and the server hold 2 or 4, by tau16)
  int tau_bytes = 4;
  double ms_prep = 0;
  size_t bytes() const;
};

}  // namespace nd

struct nd_graph {
  nd_ctx *ctx = nullptr;
  int32_t n = 0;
  int64_t nnz = 0;
  nd::DArr<int64_t> row_off;  // n+1
  nd::DArr<int32_t> col;      // nnz, ascending per row
  nd::DArr<int32_t> rowid;    // nnz: row of each entry
  // edge numbering (r = 2): edges u<v lexicographic
  bool edges_ready = false;
  int64_t ne = 0;
  nd::DArr<int32_t> ev;       // 2*ne: endpoints (u, v) of each edge
  nd::DArr<int32_t> nlow;     // n: neighbours below u
  nd::DArr<int64_t> eoff;     // n+1: first edge id of u
  nd::DArr<int32_t> eid;      // nnz: id of the edge of each entry
  // triangle numbering (r = 3): triangles u<v<w lexicographic
  bool tris_ready = false;
  int64_t nt = 0;
  nd::DArr<int64_t> toff;     // ne+1: first triangle id of edge (u,v)
  nd::DArr<int32_t> tri_w;    // nt: third vertex w
  nd::DArr<int32_t> tri_e;    // nt: edge id of (u,v)
  nd::KindState ks[nd::kNumKinds];
  double ms_build = 0;
  size_t bytes() const;
};

namespace nd {

// Free a graph whose last device work was ordered on stream s, returning
// its memory to the allocator tagged with s (waits for s first when `wait`;
// nd_graph_destroy waits for the device).  Without waiting this is still
// safe for the graph's own arrays: the allocator hands a block tagged with s
// to another stream only once s has drained.
void destroy_graph(nd_graph *g, hipStream_t s, bool wait = true);

// ------------------------------------------------------- primitives

// out[i] = sum_{j<i} in[j] for i <= n (out has n+1 entries).
void exclusive_scan_i32(const int32_t *in, int64_t *out, int64_t n,
                        hipStream_t s, Allocator &al);
void exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n,
                        hipStream_t s, Allocator &al);
// Stable LSD radix sort of keys by bits [lo_bit, hi_bit); returns whichever
// of keys/tmp holds the result.
uint64_t *radix_sort_u64(uint64_t *keys, uint64_t *tmp, int64_t n, int lo_bit,
                         int hi_bit, hipStream_t s, Allocator &al);
// items[] = 0..n-1 grouped by bin[i] (stable), offsets[b] = first index of
// bin b (host, nbins+1 entries).  nbins <= 5.  partition_start leaves the
// offsets in head (device memory, first kPartHeadWords of it int64) for the
// caller to post, with partition_offsets to read them.
constexpr int kPartHeadWords = 18;
void partition_start(const uint8_t *bin, int64_t n, int32_t *items,
                     int64_t *head, hipStream_t s, Allocator &al);
void partition_offsets(const int64_t *head, int64_t n, int nbins,
                       int64_t *offsets);
void partition_by_bin(const uint8_t *bin, int64_t n, int nbins, int32_t *items,
                      int64_t *offsets, hipStream_t s, Allocator &al);
void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s);
void fill_u64(uint64_t *p, uint64_t v, int64_t n, hipStream_t s);
void fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s);
void iota_i32(int32_t *p, int64_t n, hipStream_t s);  // p[i] = i
int64_t read_i64(const int64_t *dev, hipStream_t s);  // synchronous

// A 4 KiB pinned host chunk taken from a pool for the life of the object,
// for reading a few words back from the device.  A one-workgroup kernel stores
// them into the chunk (which the device sees), so the wait that follows is all
// that a read-back costs besides: an asynchronous copy of a few bytes goes
// through the runtime's copy path, which takes longer than the kernel.
// Several words can be posted before one wait.  Chunks return to the pool,
// never to the runtime.
class PinnedChunk {
 public:
  static constexpr size_t kBytes = 4096;
  PinnedChunk();
  ~PinnedChunk();
  PinnedChunk(const PinnedChunk &) = delete;
  PinnedChunk &operator=(const PinnedChunk &) = delete;
  template <class T>
  T *as() const { return static_cast<T *>(p_); }
  // Post n words of T (a multiple of 4 bytes, 8-byte aligned places); valid
  // after a wait for s.
  template <class T>
  const T *post(const T *dev, size_t n, hipStream_t s) {
    static_assert(sizeof(T) % 4 == 0, "whole words are posted");
    const size_t bytes = (n * sizeof(T) + 7) / 8 * 8;
    ND_REQUIRE(used_ + bytes <= kBytes, ND_ERR_INVALID, "read-back too large");
    T *to = reinterpret_cast<T *>(static_cast<char *>(p_) + used_);
    used_ += bytes;
    post_words(to, dev, n * sizeof(T) / 4, s);
    return to;
  }
  // Post n words of T and wait for s.  The next post after it starts over at
  // the chunk's beginning.
  template <class T>
  const T *read(const T *dev, size_t n, hipStream_t s) {
    const T *to = post(dev, n, s);
    ND_HIP(hipStreamSynchronize(s));
    used_ = 0;
    return to;
  }

 private:
  static void post_words(void *to, const void *dev, size_t words, hipStream_t s);
  void *p_ = nullptr;
  size_t used_ = 0;
};

// ------------------------------------------------------------ graph prep

// Canonical CSR from raw device pairs (validates ids; ND_ERR_INVALID).
void build_from_edges(nd_graph *g, int64_t m, const int32_t *src,
                      const int32_t *dst, hipStream_t s);
// Check a device CSR already copied into g (ND_ERR_INVALID when malformed).
void validate_csr(nd_graph *g, hipStream_t s);
void build_rowid(nd_graph *g, hipStream_t s);
void build_edges(nd_graph *g, hipStream_t s);
void build_triangles(nd_graph *g, hipStream_t s);
// Incidence lists in the internal numbering (each calls build_layout once
// the S-degrees are counted, then writes the lists in place).
void build_incidence_core(nd_graph *g, KindState &ks, hipStream_t s);
void build_incidence_truss(nd_graph *g, KindState &ks, hipStream_t s);
void build_incidence_n34(nd_graph *g, KindState &ks, hipStream_t s);
void build_incidence_n13(nd_graph *g, KindState &ks, hipStream_t s);
void build_incidence_n24(nd_graph *g, KindState &ks, hipStream_t s);
// From S-degrees in r-clique-id order: perm, inv, ds, inc_off, bins.  `order`:
// the r-cliques as they follow each other within a bin (NULL: by id).
void build_layout(nd_graph *g, KindState &ks, const int32_t *cnt,
                  hipStream_t s, const int32_t *order = nullptr);
// Re-index between internal and r-clique-id order; the internal side holds
// `bytes` (1, 2 or 4) per value.
void to_internal(const KindState &ks, const int32_t *in, void *out, int bytes,
                 hipStream_t s);
void to_original(const KindState &ks, const void *in, int bytes, int32_t *out,
                 hipStream_t s);
// Incidence lists in r-clique-id order with r-clique ids (off[nr+1]).
void incidence_original(nd_graph *g, const KindState &ks, int64_t *off,
                        int32_t *ids, hipStream_t s);
void sdegree_original(const KindState &ks, int32_t *ds, hipStream_t s);
// tau_0 = d_s in the internal numbering, `bytes` (1, 2 or 4) per value.
void init_tau(const KindState &ks, void *tau, int bytes, hipStream_t s);

// ---------------------------------------------------------------- sweeps

// Per-sweep counters.  Every wave adds its counts atomically; with one
// counter all those atomics would queue on a single L2 channel, so the counts
// are split over kStatParts parts, one 128-byte line each, and summed by the
// reader.
constexpr int kStatParts = 16;
struct alignas(128) StatPart {
  unsigned long long changed;
  unsigned long long evaluated;
  unsigned long long pad[14];
};
struct SweepStats {
  StatPart part[kStatParts];
  unsigned long long notified;  // 1: this sweep set the next sweep's flags
  unsigned long long active;    // r-cliques flagged for the next sweep
                                // (counted after the sweep when asked for)
  unsigned long long total;     // batches: changed_total(), summed once
  unsigned long long wide;      // nonzero: a value does not fit the next
                                // narrower type (asked for after a sweep)
  unsigned long long pad[12];
  __host__ __device__ unsigned long long changed_total() const {
    unsigned long long s = 0;
    for (int i = 0; i < kStatParts; i++) s += part[i].changed;
    return s;
  }
  __host__ __device__ unsigned long long evaluated_total() const {
    unsigned long long s = 0;
    for (int i = 0; i < kStatParts; i++) s += part[i].evaluated;
    return s;
  }
};

struct SweepArgs {
  const int64_t *inc_off;
  const int32_t *inc_ids;
  const void *tau_in;      // SND: tau_t; AND: the in-place array
  void *tau_out;           // SND: tau_{t+1}; AND: same as tau_in
  int tau_bytes;           // 1, 2 or 4, of both
  SweepStats *stats;       // this sweep's counters
  const SweepStats *prev;  // previous sweep's counters (skip when converged)
  int cap_by_tau;          // 1: clamp at tau_in(R) (iterates); 0: at d_s
  // Frontier (Section 4.3 notifications), both NULL when off: only
  // r-cliques with act[R] != 0 are recomputed; a changed one sets act_next
  // for every neighbour whose value is above its new value.
  const uint8_t *act;       // flags of this sweep (stamps, see sweep_dev.h)
  uint8_t *act_next;
  // one stamp per 64 r-cliques, set with any flag of the group (NULL: none)
  const uint8_t *act_sum;
  uint8_t *act_sum_next;
  uint8_t stamp;            // this sweep's stamp
  // Notifications start once a sweep changes at most this many r-cliques
  // (before that nearly everything is active and notifying costs as much as
  // the gathers it would save); from then on every sweep notifies and the
  // next one recomputes only flagged r-cliques.
  unsigned long long notify_below;
  // 1: the first sweep notifies too (notify_below only applies from the
  // second sweep on otherwise).
  int notify_first;
  // 1: flags are written and counted but never used to skip r-cliques (the
  // active-ratio indicator without the frontier).
  int flags_unused;
  // A sparse sweep after one that changed fewer r-cliques than this spreads
  // them over its waves (see sweep_sparse).
  unsigned long long spread_below;
  // Support counting with the frontier (see Support in sweep_dev.h), all NULL
  // when off: slack holds a tau-sized word per r-clique, lost / lost_next
  // counters of 1 << lost_shift bytes (this sweep's, the next sweep's), which
  // take the place of the flags (act and act_next then only say that there
  // are notifications).
  void *slack;
  void *lost;
  void *lost_next;
  int lost_shift;
  // PartialAND (Section 4.3, end): act marks a fixed set (stamp 1) that is
  // the only thing recomputed, every sweep, and nothing notifies (in place).
  int fixed_set;
  // At most this many workgroups per lanes-per-r-clique kernel (they stride
  // over the rest of the bin); 0: one pass, no cap.
  int grid_cap;
  // Nonzero: a notifying sweep whose previous sweep changed at least this
  // many r-cliques writes flags but no group summaries (many of its
  // notifications would store the same summary byte); launch_group_sums
  // rebuilds them after it from the flags.
  unsigned long long sums_after;
};

// The static device workspace of nd_decompose_noalloc: one array per device
// (api.hip), its address looked up when the first context on the device is
// created; NULL before that.
constexpr size_t kNoallocWorkspaceBytes = ND_NOALLOC_WORKSPACE_BYTES;
void *noalloc_workspace(int device);

// Entries of the pinned host ring that receives the sweep counters' totals.
constexpr int kHostStatsRing = 1024;
struct HostStats {
  unsigned long long changed, evaluated, notified, active, wide;
};

// Launch one sweep over every bin of ks (internal numbering, tau of
// a.tau_bytes per value).  `and_mode` selects in-place reads.
void launch_sweep(const KindState &ks, const SweepArgs &a, bool and_mode,
                  hipStream_t s);
// After the sweep of a (same arguments): the group summaries of the flags it
// wrote, when a.sums_after made it skip them; nothing otherwise.
void launch_group_sums(const KindState &ks, const SweepArgs &a, hipStream_t s);

// Plain SND sweeps (no notifications, no callback) of a graph that fits one
// workgroup's LDS: up to kTinySweeps per launch (tiny.hip).  The values after
// the last sweep go to tau0 and tau1.
constexpr int kTinyRcliques = 8192;   // swept ones
constexpr int kTinyIncidence = 20480;
constexpr int kTinySweeps = 32;
bool tiny_fits(const KindState &ks);
void launch_tiny(const KindState &ks, const void *tau_in, void *tau0, void *tau1,
                 SweepStats *ring, int ring_len, int64_t first, int count,
                 hipStream_t s);

// Host threads (each with a stream) that build or prepare several graphs
// at once: 2, or ND_PREP_THREADS.
int prep_threads();

// Whether frontier sweeps count support (Support in sweep_dev.h) rather than
// flag.  With s = r + 1 two r-cliques share one s-clique at most.  Two vertices
// share many triangles, two edges many 4-cliques: a hub's fall adds thousands
// of times to one counter, where flags store the same byte ((1,3), 79561
// vertices with lists of 33573: 14.6 ms counted, 3.4 flagged; 24665 vertices
// 9.1 and 1.2; (2,4), 276464 edges 4.5 and 3.8, 60 communities 20.6 and 20.0).
inline bool counts_support(const KindState &ks) { return ks.s == ks.r + 1; }

// Whether full sweeps that notify nobody give a bin a launch of its own, its
// values in registers: with k <= 2 where the bin holds at least half of the
// swept r-cliques and so fills the GPU by itself (k-core, 30000 vertices, lists
// of 700..1000: 1.34 ms a decomposition, 1.64 in the common launch through LDS;
// of 1100..1300: 1.93 and 3.76, a workgroup and a histogram each; k-truss, 2.8M
// edges, 1000..1300: four sweeps 100 and 116 ms).  With k = 5 both are alike
// (3.4 and 3.6 ms), and with k = 2 lists of 513..1024 are quicker in the common
// launch ((1,3), 8000 vertices 1.03 and 0.91); where the bins are mixed, the
// hubs' graphs among them, one launch for all wins.
inline bool swept_apart(const KindState &ks, int bin) {
  const int64_t n = ks.bin_hi[bin] - ks.bin_lo[bin];
  const bool gains = bin == kBinWave ? ks.k <= 2 : bin == kBinWave16 && ks.k == 1;
  return gains && n > 0 && 2 * n >= ks.bin_lo[kBinZero];
}

// Bytes (log2) of a lost-s-clique counter: at most k d_s are counted for one
// r-clique in one sweep.
inline int lost_shift(const KindState &ks) {
  const int64_t most = (int64_t)ks.k * ks.max_ds;
  return most <= 255 ? 0 : most <= 65535 ? 1 : 2;
}

// Frontier switch: notifications start once a sweep changes at most 1/d of the
// swept r-cliques.  d = 8 where a full sweep is bound by its gathers: 16.5M
// edges 42.6 ms at 8, 41.9 at 12, 44.6 at 40; 4e8 triangles 456 ms at 8, 484 at
// 24; 18.7M incidences of a k-core the same from 8 to 64, 3.4 against 2.6 ms at
// 8192.  Up to 2^22 gathers a sweep a full one is a launch and a chain of loads
// just as a sparse one, and the sparse one's chain is longer: d = 512 (k-truss
// of 1.2M gathers 0.46 ms at 8, 0.36 at 256 and 0.37 at 1024; (1,3) of 0.7M
// 1.11 / 0.50 / 0.38; k-core of 1.9M 0.77 / 0.69 / 0.66).  With support counts
// also up to 2^17 swept r-cliques with 128 gathers and more each: their values
// fit the caches, so a full sweep's gathers are quick, while the notifications
// of long lists meet on few counters (k-core, 30000 vertices, lists of 900:
// 1.95 ms at 8, 1.43 at 512, of 300: 0.82 and 0.65; 100000 vertices, 900: 12.1
// and 11.0; k-truss, 108000 edges, 216: 3.87 and 3.12; but 100000 vertices, 100:
// 1.21 and 1.36, 300000 vertices, 100: 2.71 and 3.22).  ND_FRONTIER_SWITCH
// overrides all (0: from the first sweep on).
// (gathers: of a sweep that may notify, of many graphs in a batch.)
inline bool notifies_late(const KindState &ks, int64_t gathers) {
  const int64_t swept = ks.bin_lo[kBinZero];
  return gathers <= (int64_t)1 << 22 ||
         (counts_support(ks) && swept <= 1 << 17 && ks.P * ks.k / 128 >= swept);
}
int frontier_switch(bool late);

}  // namespace nd
