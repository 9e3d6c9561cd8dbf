// sweep_kernels.h -- the single-graph sweep kernels (see sweep.hip for the
// method) and their launch for one k = C(s,r) - 1 and one type of tau, each
// compiled in its own translation unit (sweep_inst.hip).  Internal header.
#pragma once

#include <algorithm>

#include "sweep_dev.h"

namespace nd {

namespace {

using namespace dev;

// Frontier state of this sweep (uniform over the launch): flags are read
// only if the previous sweep wrote them (and a.flags_unused is clear); this
// sweep notifies once the previous one changed few enough r-cliques, and
// keeps notifying after; the first sweep notifies only with a.notify_first.
__device__ __forceinline__ void frontier_mode(const SweepArgs &a,
                                              unsigned long long before,
                                              const uint8_t **act,
                                              uint8_t **act_next,
                                              const uint8_t **act_sum,
                                              uint8_t **sum_next,
                                              Support *sp) {
  *act_sum = nullptr;
  *sum_next = nullptr;
  const bool flags_valid =
      !a.flags_unused && a.prev != nullptr && a.prev->notified;
  const bool notify =
      a.prev != nullptr
          ? (a.prev->notified || before <= a.notify_below)
          : a.notify_first != 0;
  *act = flags_valid ? a.act : nullptr;
  *act_next = notify ? a.act_next : nullptr;
  *act_sum = flags_valid ? a.act_sum : nullptr;
  *sum_next = notify ? a.act_sum_next : nullptr;
  if (a.sums_after != 0 && before >= a.sums_after)
    *sum_next = nullptr;  // k_group_sums writes them
  // Slack is kept from the first notifying sweep on.  (The rest without a branch,
  // which keeps it in scalar registers; none is read while slack is NULL.)
  sp->slack = notify ? a.slack : nullptr;
  sp->lost = a.lost;
  sp->lost_next = a.lost_next;
  sp->shift = a.lost_shift;
  if (notify && blockIdx.x == 0 && threadIdx.x == 0) a.stats->notified = 1;
}

// Workgroup LDS for sweep_flat: the minima of one run's incidence entries
// and the run's list offsets (relative to its first entry).
constexpr int kFlatRun = 4096;  // incidence entries per run, at most
template <typename T>
struct FlatLds {
  T rho[kFlatRun];
  int32_t off[kFlatRun / 4 + 1];
  // sweep_flat_fr: per entry, the listed members holding the minimum
  uint8_t mask[kFlatRun];
};

// A full sweep (no flags read, none written) of a bin of G lanes per
// r-clique with d_s <= 4G.  The workgroup takes one contiguous share of the
// bin in runs of kFlatRun / (4G) r-cliques (at most kFlatRun incidence
// entries).  The run's entries are gathered flat: lane t takes entries t,
// t + 256, ..., so the id stream is read in order and coalesced, and the
// values gathered by a run's r-cliques -- which share vertices -- are
// reused from the CU's cache; the minima go to LDS.  Then G lanes per
// r-clique read their values back from LDS and compute H as update_regs
// does.  Counts are added to *n_ch / *n_ev (wave totals).
template <int K, int G, typename T, bool AND>
__device__ __forceinline__ void sweep_flat(const SweepArgs &a, int64_t lo,
                                           int64_t hi, int64_t block,
                                           int64_t nblocks, FlatLds<T> *lds,
                                           unsigned long long *n_ch,
                                           unsigned long long *n_ev) {
  constexpr int M = 4;
  constexpr int kRun = kFlatRun / (G * M);  // r-cliques per run
  constexpr int kPerPass = 256 / G;         // r-cliques per h-index pass
  const T *tin = (const T *)a.tau_in;
  T *tout = (T *)a.tau_out;
  const int t = threadIdx.x;
  const int sl = lane_id() % G;
  const int64_t nruns = (hi - lo + kRun - 1) / kRun;
  const int64_t per = (nruns + nblocks - 1) / nblocks;
  const int64_t q1 = std::min<int64_t>(nruns, (block + 1) * per);
  for (int64_t q = block * per; q < q1; q++) {  // uniform over the workgroup
    const int64_t r0 = lo + q * kRun;
    const int n = (int)std::min<int64_t>(kRun, hi - r0);
    const int64_t e0 = a.inc_off[r0];
    for (int i = t; i <= n; i += blockDim.x)
      lds->off[i] = (int32_t)(a.inc_off[r0 + i] - e0);
    __syncthreads();
    const int ne = lds->off[n];
    for (int e = t; e < ne; e += blockDim.x)
      lds->rho[e] = (T)gather_rho<K, T, AND>(a.inc_ids, e0 + e, tin);
    __syncthreads();
    for (int p = 0; p < n; p += kPerPass) {  // uniform over the workgroup
      const int i = p + t / G;
      const bool active = i < n;
      int32_t told = 0, c = 0;
      int b = 0, d = 0;
      if (active) {
        told = (int32_t)tin[r0 + i];
        b = lds->off[i];
        d = lds->off[i + 1] - b;
        c = a.cap_by_tau ? told : d;
      }
      int32_t rho[M];
#pragma unroll
      for (int m = 0; m < M; m++) {
        const int j = sl + m * G;
        rho[m] = j < d ? (int32_t)lds->rho[b + j] : -1;
      }
      const int cnt = count_ge<G, M>(rho, c);
      const int32_t h = cnt >= c ? c : hindex_search<G, M>(rho, c, cnt);
      const bool lead = sl == 0;
      const bool ch = active && h != told;
      if (active && lead) store_tau<T, AND>(tout + r0 + i, h, ch);
      *n_ch += __popcll(ballot(lead && ch));
      *n_ev += __popcll(ballot(lead && active));
    }
    __syncthreads();  // the next run reuses the LDS
  }
}

// The full sweep that notifies (Section 4.3: the first sweep after the
// frontier switches on, or every SND sweep while active counts are taken),
// in the same runs as sweep_flat: the flat gather also keeps which members
// hold each minimum, and the subgroups write, self-activate on a change,
// store their slack and notify through the kept minima (notify_kept), as
// update_regs does.
template <int K, int G, typename T, bool AND>
__device__ __forceinline__ void sweep_flat_fr(const SweepArgs &a, int64_t lo,
                                              int64_t hi, int64_t block,
                                              int64_t nblocks, uint8_t *act_next,
                                              uint8_t *sum_next,
                                              const Support &sp,
                                              FlatLds<T> *lds,
                                              unsigned long long *n_ch,
                                              unsigned long long *n_ev) {
  constexpr int M = 4;
  constexpr int kRun = kFlatRun / (G * M);
  constexpr int kPerPass = 256 / G;
  constexpr int kMaskWords = (K * M + 31) / 32;
  const T *tin = (const T *)a.tau_in;
  T *tout = (T *)a.tau_out;
  const uint8_t next = a.stamp == 255 ? 1 : a.stamp + 1;
  const int t = threadIdx.x;
  const int sl = lane_id() % G;
  const int64_t nruns = (hi - lo + kRun - 1) / kRun;
  const int64_t per = (nruns + nblocks - 1) / nblocks;
  const int64_t q1 = std::min<int64_t>(nruns, (block + 1) * per);
  for (int64_t q = block * per; q < q1; q++) {  // uniform over the workgroup
    const int64_t r0 = lo + q * kRun;
    const int n = (int)std::min<int64_t>(kRun, hi - r0);
    const int64_t e0 = a.inc_off[r0];
    for (int i = t; i <= n; i += blockDim.x)
      lds->off[i] = (int32_t)(a.inc_off[r0 + i] - e0);
    __syncthreads();
    const int ne = lds->off[n];
    for (int e = t; e < ne; e += blockDim.x) {
      uint32_t arg = 1;
      int32_t r;
      if constexpr (K > 1)
        r = gather_rho_arg<K, T, AND>(a.inc_ids, e0 + e, tin, &arg);
      else
        r = gather_rho<K, T, AND>(a.inc_ids, e0 + e, tin);
      lds->rho[e] = (T)r;
      lds->mask[e] = (uint8_t)arg;
    }
    __syncthreads();
    for (int p = 0; p < n; p += kPerPass) {  // uniform over the workgroup
      const int i = p + t / G;
      const bool active = i < n;
      int32_t told = 0, c = 0;
      int b = 0, d = 0;
      if (active) {
        b = lds->off[i];
        d = lds->off[i + 1] - b;
        told = (int32_t)tin[r0 + i];
        c = a.cap_by_tau ? told : d;
      }
      int32_t rho[M];
      uint32_t amask[kMaskWords];
#pragma unroll
      for (int w = 0; w < kMaskWords; w++) amask[w] = 0;
#pragma unroll
      for (int m = 0; m < M; m++) {
        const int j = sl + m * G;
        const bool in = j < d;
        rho[m] = in ? (int32_t)lds->rho[b + j] : -1;
        if (K > 1 && in) {
          const uint32_t am = lds->mask[b + j];
#pragma unroll
          for (int x = 0; x < K; x++) {
            const int bit = m * K + x;
            amask[bit >> 5] |= ((am >> x) & 1u) << (bit & 31);
          }
        }
      }
      const int cnt = count_ge<G, M>(rho, c);
      const int32_t h = cnt >= c ? c : hindex_search<G, M>(rho, c, cnt);
      const bool lead = sl == 0;
      const bool ch = active && h != told;
      const int64_t R = r0 + i;
      if (active && lead) {
        store_tau<T, AND>(tout + R, h, ch);
        if (sp.slack) ((T *)sp.slack)[R] = slack_word<T>(ch, cnt, c);
      }
      if (ch) {
        if (lead) self_activate(R, act_next, next, sum_next, sp);
        notify_kept<K, G, M>(a.inc_ids, e0 + b, d, sl, rho, amask, told, h,
                             act_next, next, sum_next, sp);
      }
      *n_ch += __popcll(ballot(lead && ch));
      *n_ev += __popcll(ballot(lead && active));
    }
    __syncthreads();  // the next run reuses the LDS
  }
}

// One bin [lo, hi) of G lanes per r-clique with M values per lane, swept by
// the workgroups block .. of nblocks (a launch of its own, or a block range
// of k_sweep_bins).  With `flat` LDS (lists up to 256), a full sweep that
// notifies nobody runs as sweep_flat and a full SND sweep that notifies as
// sweep_flat_fr.  Sweeps that read flags find their flagged r-cliques per
// wave (sweep_sparse): run-based variants of those (marking, or compacting
// the flagged r-cliques of each run in LDS) measured no faster.
template <int K, int G, int M, typename T, bool AND, bool FR, bool SET = false>
__device__ __forceinline__ void sweep_bin(const SweepArgs &a, int64_t lo,
                                          int64_t hi, int64_t block,
                                          int64_t nblocks, const uint8_t *act,
                                          uint8_t *act_next,
                                          const uint8_t *act_sum,
                                          uint8_t *sum_next, const Support &sp,
                                          FlatLds<T> *flat, bool spread,
                                          int wave_list = kWaveList) {
  constexpr int kPerWave = kWave / G;
  // M == 0: the wave's share of the LDS for its list (update_wave)
  T *buf = M == 0 || G <= 4 ? flat->rho + threadIdx.x / kWave * wave_list : nullptr;
  const int64_t wave = (block * blockDim.x + threadIdx.x) / kWave;
  const int64_t waves = nblocks * (blockDim.x / kWave);
  const int sub = lane_id() / G;
  const T *tin = (const T *)a.tau_in;
  T *tout = (T *)a.tau_out;
  unsigned long long n_ch = 0, n_ev = 0;  // wave totals, from ballots
  constexpr bool kFlatFr = FR && M == 4;
  if (kFlatFr && act == nullptr && act_next != nullptr &&
      (!AND || sp.slack != nullptr)) {
    if constexpr (kFlatFr)
      sweep_flat_fr<K, G, T, AND>(a, lo, hi, block, nblocks, act_next, sum_next,
                                  sp, flat, &n_ch, &n_ev);
  } else if (FR && act != nullptr) {
    if constexpr (FR) {
      // Sparse, up to 16 entries: a lane per r-clique.  The flagged r-cliques
      // share few cache lines, so a step is a chain of misses (ids, values,
      // ids again to notify); with 64 r-cliques per step instead of 16 there are
      // a quarter of the chains.
      // The members of a fixed set are many at once and lie anywhere: there a
      // lane's list is a cache line of its own, and 16 r-cliques a step are quicker
      // (see k_sweep_bins).
      constexpr bool kLane = G <= 4 && M == 4 && !SET;
      uint8_t *mbuf = kLane ? flat->mask + threadIdx.x / kWave * kWaveList : nullptr;
      sweep_sparse<K, kLane ? 1 : G, kLane ? 0 : M, T, AND>(
                                    a.inc_off, a.inc_ids, tin, tout, a.cap_by_tau,
                                    lo, hi, wave, waves, act, act_next, a.stamp,
                                    &n_ch, &n_ev, act_sum, sum_next, sp, buf, mbuf,
                                    spread);
    }
  } else if (M == 4 && act == nullptr && act_next == nullptr) {
    if constexpr (M == 4)
      sweep_flat<K, G, T, AND>(a, lo, hi, block, nblocks, flat, &n_ch, &n_ev);
  } else {
    // Each workgroup takes one contiguous share of the bin (a multiple of
    // its waves' step), its waves striding inside it: the r-cliques of a
    // share have neighbouring ids and share vertices, so the values they
    // gather are reused from the CU's cache (measured against waves striding
    // over the whole bin: 11% less time per full (3,4) sweep of the
    // block-model workload, the same on the Chung-Lu ones).
    const int64_t wib = threadIdx.x / kWave;
    const int64_t step = (int64_t)(blockDim.x / kWave) * kPerWave;
    int64_t run = (hi - lo + nblocks - 1) / nblocks;
    run = (run + step - 1) / step * step;
    const int64_t c0 = lo + block * run;
    const int64_t c1 = std::min<int64_t>(hi, c0 + run);
    for (int64_t base = c0 + wib * kPerWave; base < c1; base += step) {
      const int64_t R = base + sub;
      bool ev, changed;
      if constexpr (M == 0) {  // one r-clique per wave: R is uniform
        ev = lane_id() == 0;
        const int64_t b = a.inc_off[R];
        const int d = (int)(a.inc_off[R + 1] - b);
        const int32_t told = (int32_t)tin[R];
        changed = update_wave<K, T, AND, FR>(
            a.inc_ids, tin, tout, R, b, d, told, a.cap_by_tau ? told : d, true,
            act_next, a.stamp, sum_next, sp, buf);
      } else {
        changed = update_regs<K, G, M, T, AND, FR>(
            a.inc_off, a.inc_ids, tin, tout, a.cap_by_tau, R, R < c1, act,
            act_next, a.stamp, &ev, sum_next, sp);
      }
      n_ch += __popcll(ballot(changed));
      n_ev += __popcll(ballot(ev));
    }
  }
  stat_add_counts(a.stats, n_ch, n_ev);
}

// The hubs [lo, hi) (d_s above 1024), a workgroup each.  The workgroup takes
// every nblocks-th of them, up to 256 at a time: each thread looks whether
// one must run, and those that must run one after the other.
template <int K, typename T, bool AND, bool FR>
__device__ __forceinline__ void sweep_hubs(const SweepArgs &a, int64_t lo,
                                           int64_t hi, int64_t block,
                                           int64_t nblocks, const uint8_t *act,
                                           uint8_t *act_next, uint8_t *sum_next,
                                           const Support &sp, HubLds &L) {
  const int t = threadIdx.x;
  unsigned long long n_ch = 0, n_ev = 0;  // on the first wave
  for (int64_t b0 = lo + block; b0 < hi; b0 += nblocks * kBlockThreads) {
    const int64_t R = b0 + (int64_t)t * nblocks;
    bool run = R < hi;
    if (FR && act != nullptr && run) {
      if (sp.slack != nullptr) {
        const uint32_t lost = lost_count(sp.lost, sp.shift, R);
        const uint32_t slack = (uint32_t)((const T *)sp.slack)[R];
        if (lost) support_store<T>(sp, R, slack > lost ? slack - lost : 0);
        run = slack <= lost;
      } else {
        run = act[R] == a.stamp;
      }
    }
    if (t == 0) L.nfound = 0;
    __syncthreads();
    if (run) L.found[atomicAdd(&L.nfound, 1)] = (int32_t)R;
    __syncthreads();
    const int n = L.nfound;
    for (int i = 0; i < n; i++) {  // uniform over the workgroup
      const bool ch = update_hub<K, T, AND, FR>(
          a.inc_off, a.inc_ids, (const T *)a.tau_in, (T *)a.tau_out,
          a.cap_by_tau, __builtin_amdgcn_readfirstlane(L.found[i]), L, act_next, a.stamp, sum_next, sp);
      n_ch += t < kWave ? __popcll(ballot(ch)) : 0;
    }
    n_ev += t < kWave ? n : 0;
    __syncthreads();  // the list is used up
  }
  stat_add_counts(a.stats, n_ch, n_ev);
}

// Every bin in one launch: a sparse sweep pays for one, and in a full sweep
// the bins run side by side, the hubs first, instead of each draining the
// chip before the next starts (hubs, their 1025..2047 and the rest one after
// the other took 65 + 14 + 66 us a sweep on a 1.7M-vertex k-core with 35,000
// neighbours at most).  Range 0 are the hubs (d_s > 1024), range 1 the lists
// of 257..1024, range i the bin kBinG64 + i - 2; range i has the workgroups
// [first[i], first[i+1]).  (Bins of 513..2047 that fill the GPU by themselves are
// left to k_sweep_regs in full sweeps that notify nobody.)
constexpr int kRanges = kBinZero - kBinG64 + 2;
constexpr int64_t kHubBlocks = 1024;
constexpr int kHubMin = 1025;  // smallest d_s of kBinWave
struct BinRanges {
  int64_t lo[kRanges], hi[kRanges];
  unsigned first[kRanges + 1];
};

// LONG: with the ranges of lists above 256.  8-bit values have them only where
// wider ones were narrowed (see k_narrow in driver.hip).  SET: in-place sweeps of
// a fixed set (PartialAND), its members flagged in act, without the notifying
// sweeps' registers (100,000 members of a k-core of 1,000,000 vertices: 57 us a
// sweep as a frontier's, 36 so).
template <int K, typename T, bool AND, bool FR, bool LONG, bool SET>
__global__ __launch_bounds__(256, 6) void k_sweep_bins(SweepArgs a, BinRanges sb) {
  __shared__ union {
    FlatLds<T> flat;
    HubLds hub;
  } lds;
  const unsigned long long pc = prev_changed(a);
  if (pc == 0) return;
  const uint8_t *act = nullptr, *act_sum = nullptr;
  uint8_t *act_next = nullptr, *sum_next = nullptr;
  Support sp;
  if constexpr (SET)
    act = a.act;
  else if (FR)
    frontier_mode(a, pc, &act, &act_next, &act_sum, &sum_next, &sp);
  const bool spread = FR && !SET && pc < a.spread_below;
  int i = 0;
  while (i + 1 < kRanges && blockIdx.x >= sb.first[i + 1]) i++;
  const int64_t block = blockIdx.x - sb.first[i];
  const int64_t nblocks = sb.first[i + 1] - sb.first[i];
  if constexpr (LONG) {
    if (i == 0) {
      sweep_hubs<K, T, AND, FR>(a, sb.lo[0], sb.hi[0], block, nblocks, act,
                                act_next, sum_next, sp, lds.hub);
      return;
    }
    if (i == 1) {
      sweep_bin<K, 64, 0, T, AND, FR, SET>(a, sb.lo[1], sb.hi[1], block, nblocks, act,
                                           act_next, act_sum, sum_next, sp, &lds.flat,
                                           spread);
      return;
    }
  }
  switch (kBinG64 + i - 2) {
    case kBinG64:
      sweep_bin<K, 64, 4, T, AND, FR, SET>(a, sb.lo[i], sb.hi[i], block, nblocks, act,
                                           act_next, act_sum, sum_next, sp, &lds.flat,
                                           spread);
      break;
    case kBinG16:
      sweep_bin<K, 16, 4, T, AND, FR, SET>(a, sb.lo[i], sb.hi[i], block, nblocks, act,
                                           act_next, act_sum, sum_next, sp, &lds.flat,
                                           spread);
      break;
    case kBinG4:
      sweep_bin<K, 4, 4, T, AND, FR, SET>(a, sb.lo[i], sb.hi[i], block, nblocks, act,
                                          act_next, act_sum, sum_next, sp, &lds.flat,
                                          spread);
      break;
    default:  // kBinG1
      sweep_bin<K, 1, 4, T, AND, FR, SET>(a, sb.lo[i], sb.hi[i], block, nblocks, act,
                                          act_next, act_sum, sum_next, sp, &lds.flat,
                                          spread);
      break;
  }
}

// A full sweep that notifies nobody over one bin of the longer lists, M values
// per lane in registers (see swept_apart).
template <int K, int M, typename T, bool AND>
__global__ __launch_bounds__(256) void k_sweep_regs(SweepArgs a, int64_t lo,
                                                    int64_t hi) {
  if (prev_changed(a) == 0) return;
  sweep_bin<K, 64, M, T, AND, false>(a, lo, hi, blockIdx.x, gridDim.x, nullptr,
                                     nullptr, nullptr, nullptr, Support(), nullptr,
                                     false);
}

// Blocks for a bin of n r-cliques at G lanes each, at most a.grid_cap, and
// never more than grid_stride allows (the kernels stride over the rest).
inline unsigned regs_grid(const SweepArgs &a, int64_t n, int G) {
  const int64_t blocks = grid_stride(n, G);
  return (unsigned)(a.grid_cap > 0 ? std::min<int64_t>(blocks, a.grid_cap)
                                   : blocks);
}

template <int K, typename T, bool AND, bool FR>
void launch_bins(const KindState &ks, const SweepArgs &a, hipStream_t s) {
  // lanes per r-clique of the ranges after the hubs
  constexpr int kLanes[kRanges] = {256, 64, 64, 16, 4, 1};
  static_assert(kHubMin == kWaveList + 1 && kRanges == 6, "ranges and bins agree");
  BinRanges sb{};
  int64_t total = 0;
  bool apart16 = false, apart32 = false;
  if constexpr (!FR && K <= 2) {
    apart32 = swept_apart(ks, kBinWave);
    apart16 = swept_apart(ks, kBinWave16);
    if (apart32) {
      const int64_t lo = ks.bin_lo[kBinWave], hi = ks.bin_hi[kBinWave];
      k_sweep_regs<K, 32, T, AND><<<regs_grid(a, hi - lo, 64), 256, 0, s>>>(a, lo, hi);
      ND_LAUNCHED();
    }
    if constexpr (K == 1) {
      if (apart16) {
        const int64_t lo = ks.bin_lo[kBinWave16], hi = ks.bin_hi[kBinWave16];
        k_sweep_regs<K, 16, T, AND><<<regs_grid(a, hi - lo, 64), 256, 0, s>>>(a, lo, hi);
        ND_LAUNCHED();
      }
    }
  }
  for (int i = 0; i < kRanges; i++) {
    const int first = i == 0   ? kBinBlock
                      : i == 1 ? (apart16 ? kBinWave8 : kBinWave16)
                               : kBinG64 + i - 2;
    const int last = i == 0 ? (apart32 ? kBinBlock : kBinWave) : i == 1 ? kBinWave8 : first;
    sb.lo[i] = ks.bin_lo[first];
    sb.hi[i] = ks.bin_hi[last];
    sb.first[i] = (unsigned)total;
    const int64_t n = sb.hi[i] - sb.lo[i];
    if (n > 0)
      total += i == 0 ? std::min<int64_t>(n, kHubBlocks) : regs_grid(a, n, kLanes[i]);
  }
  sb.first[kRanges] = (unsigned)total;
  if (total > 0) {
    const bool with_long = sizeof(T) > 1 || sb.hi[1] > 0;
    const unsigned grid = (unsigned)total;
    if (AND && FR && a.fixed_set) {
      constexpr bool kSet = AND && FR;
      if (with_long)
        k_sweep_bins<K, T, AND, FR, true, kSet><<<grid, 256, 0, s>>>(a, sb);
      else
        k_sweep_bins<K, T, AND, FR, false, kSet><<<grid, 256, 0, s>>>(a, sb);
    } else if (with_long) {
      k_sweep_bins<K, T, AND, FR, true, false><<<grid, 256, 0, s>>>(a, sb);
    } else {
      k_sweep_bins<K, T, AND, FR, false, false><<<grid, 256, 0, s>>>(a, sb);
    }
    ND_LAUNCHED();
  }
}

template <int K, typename T, bool AND>
void launch_fr(const KindState &ks, const SweepArgs &a, hipStream_t s) {
  if (a.act)
    launch_bins<K, T, AND, true>(ks, a, s);
  else
    launch_bins<K, T, AND, false>(ks, a, s);
}

}  // namespace

template <int K, typename T>
void sweep_kind(const KindState &ks, const SweepArgs &a, bool and_mode,
                hipStream_t s) {
  if (and_mode)
    launch_fr<K, T, true>(ks, a, s);
  else
    launch_fr<K, T, false>(ks, a, s);
}

}  // namespace nd
