// sweep_dev.h -- device routines of one h-index update, shared by the
// single-graph sweep kernels (sweep.hip) and the batched tile kernel
// (batch.hip).  See sweep.hip for the method and the exactness argument.
#pragma once

#include "internal.h"

namespace nd {
namespace dev {

constexpr int kBlockThreads = 256;
// Frontier group summaries: one stamp per 64 consecutive r-cliques, set
// whenever a flag of the group is (see sweep_sparse).
constexpr int kGroupShift = 6;
constexpr int kHubBins = 4096;  // 16 KiB of LDS (see update_hub)

// AND reads and writes tau in place.  Reads and writes are relaxed atomics
// at workgroup scope: they may be served by (and stay in) this CU's L1 and
// this XCD's L2, which hold only values of the current launch (caches are
// made coherent at every kernel boundary), so a value read may be older than
// the latest write but never older than the sweep's start.  That keeps AND
// exact: values only fall, every value read lies between kappa and the
// previous iterate, so kappa <= AND_t <= SND_t still holds (H is monotone),
// and a sweep that changes nothing read only unchanged values, i.e. it
// certifies a fixed point.  Each value has one writer (the r-clique's own
// subgroup), so no write is lost.
template <typename T, bool AND>
__device__ __forceinline__ int32_t load_tau(const T *p) {
  if constexpr (AND) {
    return (int32_t)__hip_atomic_load(p, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
  } else {
    return (int32_t)*p;
  }
}

template <typename T, bool AND>
__device__ __forceinline__ void store_tau(T *p, int32_t h, bool changed) {
  if constexpr (AND) {
    if (changed)
      __hip_atomic_store(p, (T)h, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_WORKGROUP);
  } else {
    *p = (T)h;
  }
}

// Place of r-clique id's value.  Ids are below 2^31, so up to 16 bits the
// byte offset fits 32 bits and the load takes the array's base from scalar
// registers: one address instruction per gather instead of three.
template <typename T>
__device__ __forceinline__ const T *tau_at(const T *tau, int32_t id) {
  if constexpr (sizeof(T) <= 2)
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(tau) +
                                       (uint32_t)id * (uint32_t)sizeof(T));
  else
    return tau + (uint32_t)id;
}

// The k = K ids of the s-clique j of the list at ids.
template <int K, typename J>
__device__ __forceinline__ void load_ids(const int32_t *__restrict__ ids, J j,
                                         int32_t (&id)[K]) {
  if constexpr (K == 2) {
    const int2 p = *reinterpret_cast<const int2 *>(ids + 2 * j);
    id[0] = p.x;
    id[1] = p.y;
  } else {
#pragma unroll
    for (int x = 0; x < K; x++) id[x] = ids[K * j + x];
  }
}

// rho for the s-clique j of the incidence list (k = K ids per s-clique).
template <int K, typename T, bool AND, typename J>
__device__ __forceinline__ int32_t gather_rho(const int32_t *__restrict__ ids,
                                              J j, const T *tau) {
  int32_t id[K];
  load_ids<K>(ids, j, id);
  int32_t v = load_tau<T, AND>(tau_at(tau, id[0]));
#pragma unroll
  for (int x = 1; x < K; x++) v = min(v, load_tau<T, AND>(tau_at(tau, id[x])));
  return v;
}

// gather_rho with the frontier: also the members of the s-clique that hold
// the minimum (bit x set when the x-th listed id has tau = rho).
template <int K, typename T, bool AND, typename J>
__device__ __forceinline__ int32_t gather_rho_arg(const int32_t *__restrict__ ids,
                                                  J j, const T *tau,
                                                  uint32_t *arg) {
  int32_t id[K], v[K];
  load_ids<K>(ids, j, id);
#pragma unroll
  for (int x = 0; x < K; x++) v[x] = load_tau<T, AND>(tau_at(tau, id[x]));
  int32_t r = v[0];
#pragma unroll
  for (int x = 1; x < K; x++) r = min(r, v[x]);
  uint32_t a = 0;
#pragma unroll
  for (int x = 0; x < K; x++) a |= (uint32_t)(v[x] == r) << x;
  *arg = a;
  return r;
}

// Add wave-wide totals (the same on every lane, summed from ballots) to the
// sweep's counters: one atomic per wave and counter.
__device__ __forceinline__ void stat_add_counts(SweepStats *st,
                                                unsigned long long ch,
                                                unsigned long long ev) {
  if (lane_id() == 0 && (ch | ev)) {
    StatPart &p = st->part[(blockIdx.x + threadIdx.x / kWave) % kStatParts];
    if (ch) atomicAdd(&p.changed, ch);
    if (ev) atomicAdd(&p.evaluated, ev);
  }
}

// Total changed count of a finished sweep.  Every lane reads the same 16
// words (uniform addresses: scalar or broadcast loads), which costs far less
// at every wave's start than a cross-lane reduction.
__device__ __forceinline__ unsigned long long changed_sum(const SweepStats *st) {
  unsigned long long v = 0;
#pragma unroll
  for (int q = 0; q < kStatParts; q++) v += st->part[q].changed;
  return v;
}

// The previous sweep's changed count (1 for the first sweep: not converged).
__device__ __forceinline__ unsigned long long prev_changed(const SweepArgs &a) {
  return a.prev != nullptr ? changed_sum(a.prev) : 1ull;
}

// How many lanes of this lane's G-lane subgroup have p set: one wave ballot
// and a popcount (scalar for G = 64), no cross-lane data movement.
template <int G>
__device__ __forceinline__ int subgroup_count(bool p) {
  if constexpr (G == 1) {
    return p ? 1 : 0;
  } else {
    const uint64_t b = ballot(p);
    if constexpr (G == 64) {
      return __popcll(b);
    } else {
      const int sub = lane_id() / G;
      return __popcll((b >> (sub * G)) & (((uint64_t)1 << G) - 1));
    }
  }
}

// #{rho >= x} over the subgroup (G lanes x M values each).
template <int G, int M>
__device__ __forceinline__ int count_ge(const int32_t (&rho)[M], int32_t x) {
  int n = 0;
#pragma unroll
  for (int m = 0; m < M; m++) n += subgroup_count<G>(rho[m] >= x);
  return n;
}

// The largest h in [0, c-1] with count(h) >= h, where count(x) = #{rho >= x}
// and n = count(c) < c.  Counts only grow as x falls, so count(n) >= n and h
// lies in [n, c-1]; a probe that fails with n' < mid raises the lower end to n'
// the same way.  Late sweeps, whose n is just below c, take a probe or two
// where [0, c-1] took log2(c), each M ballots or a pass over LDS (k-core of
// 48431 vertices, lists up to 940, 30 full sweeps: 545 -> 446 us; k-truss of
// 86498 edges with the frontier 622 -> 596 us).
template <typename Count>
__device__ __forceinline__ int32_t hindex_between(Count count, int32_t c, int n) {
  int32_t lo = n, hi = c - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    const int32_t m = count(mid);
    if (m >= mid) {
      lo = mid;
    } else {
      hi = mid - 1;
      lo = max(lo, m);
    }
  }
  return lo;
}

// The same for values in registers: G lanes of a subgroup each hold M of them
// (absent values are -1).
template <int G, int M>
__device__ __forceinline__ int32_t hindex_search(const int32_t (&rho)[M],
                                                 int32_t c, int n) {
  return hindex_between([&](int32_t x) { return count_ge<G, M>(rho, x); }, c, n);
}

// Support counting.  A flagged r-clique R' recomputes to the same value
// whenever #{rho >= c'} is still at least c' = tau(R'), and most flagged ones
// do (four in five of the (3,4) block model's once the frontier runs).  So
// every r-clique keeps its slack #{rho >= c'} - c' from its last
// recomputation, each notification also counts one s-clique it may have lost
// (the notification test is exactly that rho(S,R') falls from at least c' to
// below it), and a flagged R' runs only when more were lost than its slack
// covers.  Counting one s-clique twice (two of its members falling in one
// sweep) only makes R' run early; none is missed, see notify().  A changed
// R' flags itself and stores slack 0 = run in any case, since its neighbours
// tested against its old value.
//   slack[R]: 0, or 1 + the slack; lost[R]: s-cliques lost since R last
//   looked, double-buffered like the flags (a sweep counts into the next
//   one's), at most K d_s(R) in one sweep, which sets the counters' width.
// Counters are packed in 32-bit words and added to atomically.  They take
// the place of the flags: R takes part in a sweep when it lost something or
// its slack word is 0, and clears its counter then, so that counters start
// each sweep at zero.  (With flags beside them a notification stored twice,
// and the stores were what bounded the sweeps: on the block model's first
// sparse sweep 74 million r-cliques run instead of 126 million, for 217
// million notifications.)
struct Support {
  void *slack = nullptr;  // NULL: off
  void *lost = nullptr;
  void *lost_next = nullptr;
  int shift = 0;  // log2 of the bytes per counter
};

// Notify r-clique r: count a lost s-clique, or set its flag.
__device__ __forceinline__ void mark(int32_t r, uint8_t *act_next,
                                     uint8_t stamp_next, uint8_t *sum_next,
                                     const Support &sp) {
  if (sp.slack != nullptr) {
    uint32_t *w = (uint32_t *)sp.lost_next + ((uint32_t)r >> (2 - sp.shift));
    atomicAdd(w, 1u << ((r & ((4 >> sp.shift) - 1)) << (3 + sp.shift)));
  } else {
    act_next[r] = stamp_next;
  }
  if (sum_next) sum_next[r >> kGroupShift] = stamp_next;
}

// R changed and runs again in the next sweep (with support counting its
// slack word, stored before, says so).
__device__ __forceinline__ void self_activate(int64_t R, uint8_t *act_next,
                                              uint8_t stamp_next,
                                              uint8_t *sum_next,
                                              const Support &sp) {
  if (sp.slack == nullptr) act_next[R] = stamp_next;
  if (sum_next) sum_next[R >> kGroupShift] = stamp_next;
}

__device__ __forceinline__ uint32_t lost_count(const void *lost, int shift,
                                               int64_t R) {
  return shift == 0   ? ((const uint8_t *)lost)[R]
         : shift == 1 ? ((const uint16_t *)lost)[R]
                      : ((const uint32_t *)lost)[R];
}

// R lost something and looked: clears its counter and stores what slack is
// left (0: it runs, and its slack word is written then).
template <typename T>
__device__ __forceinline__ void support_store(const Support &sp, int64_t R,
                                              uint32_t left) {
  if (sp.shift == 0)
    ((uint8_t *)sp.lost)[R] = 0;
  else if (sp.shift == 1)
    ((uint16_t *)sp.lost)[R] = 0;
  else
    ((uint32_t *)sp.lost)[R] = 0;
  if (left) ((T *)sp.slack)[R] = (T)left;
}

// slack word of a recomputed r-clique that kept value c with `cnt` >= c
// s-cliques at rho >= c (0 when it changed); clamping it low is safe.
template <typename T>
__device__ __forceinline__ T slack_word(bool changed, int64_t cnt, int32_t c) {
  constexpr int64_t kTop = sizeof(T) == 1 ? 255 : sizeof(T) == 2 ? 65535 : 0x7fffffff;
  const int64_t v = cnt - c + 1;
  return changed ? (T)0 : (T)(v < kTop ? v : kTop);
}

// Notification of Section 4.3: R changed from told to h.  A neighbour R'
// (another r-clique of an s-clique S containing R) can change at the next
// sweep only if some rho(S,R') falls from at least its next cap
// c' = tau_{t+1}(R') to below it.  Through S that needs rho_t(S,R') >= c' > h,
// i.e. both
//   h < tau(R')                 (tau_t(R') >= c'), and
//   h <= tau(Q) for every other member Q of S besides R and R'
// (rho_t(S,R') is a minimum over them and R).  In place (AND) the values read
// may already be newer; of several members of S that fell in one sweep, the
// one with the lowest new value still passes the test (<= keeps ties), so the
// s-clique is never lost.  SND reads tau_t exactly and self-activates every R
// that changed, so it only has to reach the R' that keep their value through
// sweep t+1: for those c' = tau_t(R'), and rho_t(S,R') >= c' also needs
// told >= c' and tau_t(Q) >= c' for the other members.  SND marks R' when
//   h < tau_t(R') <= told  and  tau_t(Q) >= tau_t(R') for every other Q,
// which keeps every R' that can change, so the iterates are those of full
// sweeps.  AND with support counting self-activates too and uses SND's test, on
// values that R read before it wrote its own: the minima its update gathered
// (notify_kept and the like), or a second gather ahead of the write
// (update_hub).  One rule for every list length: of the members of S that fall
// in one sweep, the first to write had read all the others before any of them
// wrote, so all at or above c', and R', which keeps its value, exactly; R'
// holds the minimum it saw, which lies in (h, told], and S is counted.  (A hub
// that wrote first and then tested h <= tau(Q) would not do beside that: a Q
// that had read the hub's new value and fell below it saw its minimum at the
// hub alone, and the hub then fails on Q.)  Byte stores of the same stamp race
// harmlessly.
template <int K, typename T, bool AND>
__device__ __forceinline__ void notify(const int32_t *__restrict__ ids,
                                       int64_t b, int64_t d, int first,
                                       int stride, int32_t told, int32_t h,
                                       const T *tau, uint8_t *act_next,
                                       uint8_t stamp_next, uint8_t *sum_next,
                                       const Support &sp) {
  const bool tight = !AND || sp.slack != nullptr;
  // several s-cliques in flight: a hub's list is walked by one workgroup
  constexpr int U = K == 1 ? 8 : K == 2 ? 4 : 2;
  for (int64_t j0 = first; j0 < d; j0 += (int64_t)stride * U) {
    int32_t r[U][K], v[U][K];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int64_t j = j0 + (int64_t)u * stride;
      if (j < d) {
        load_ids<K>(ids, b + j, r[u]);
      } else {
#pragma unroll
        for (int x = 0; x < K; x++) r[u][x] = -1;
      }
    }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int x = 0; x < K; x++)
        v[u][x] = r[u][x] >= 0 ? load_tau<T, AND>(tau_at(tau, r[u][x])) : -1;
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int x = 0; x < K; x++) {
        bool others_ok = true;
#pragma unroll
        for (int y = 0; y < K; y++)
          if (y != x) others_ok &= tight ? v[u][x] <= v[u][y] : h <= v[u][y];
        if (h < v[u][x] && (!tight || v[u][x] <= told) && others_ok)
          mark(r[u][x], act_next, stamp_next, sum_next, sp);
      }
  }
}

// The SND test of notify() from the values the update already gathered: R'
// passes it exactly when it holds the minimum rho of S and h < rho <= told,
// so the members to mark are those of the slots with rho in (h, told] whose
// bit is set in the argmin mask (bit m*K + x for slot m, member x; K = 1
// needs no mask).  Only their ids are read again, no tau.
template <int K, int G, int M>
__device__ __forceinline__ void notify_kept(const int32_t *__restrict__ ids,
                                            int64_t b, int64_t d, int sl,
                                            const int32_t *rho,
                                            const uint32_t *amask, int32_t told,
                                            int32_t h, uint8_t *act_next,
                                            uint8_t stamp_next,
                                            uint8_t *sum_next,
                                            const Support &sp) {
  int32_t id[M][K];  // of the slots that qualify, all loads in flight
#pragma unroll
  for (int m = 0; m < M; m++) {
    const int64_t j = sl + (int64_t)m * G;
    if (j < d && h < rho[m] && rho[m] <= told) {
      load_ids<K>(ids, b + j, id[m]);
    } else {
#pragma unroll
      for (int x = 0; x < K; x++) id[m][x] = -1;
    }
  }
#pragma unroll
  for (int m = 0; m < M; m++) {
#pragma unroll
    for (int x = 0; x < K; x++) {
      const int bit = m * K + x;
      if (id[m][x] >= 0 && (K == 1 || ((amask[bit >> 5] >> (bit & 31)) & 1u)))
        mark(id[m][x], act_next, stamp_next, sum_next, sp);
    }
  }
}

// Bit position of the t-th set bit (t counted from 0) of m; t < popc(m).
// Binary lifting: the largest p with popc(m below bit p) <= t is that bit.
__device__ __forceinline__ int nth_set_bit(uint64_t m, int t) {
  int p = 0;
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) {
    const uint64_t below = m & ((((uint64_t)1) << (p + w)) - 1);
    if (__popcll(below) <= t) p += w;
  }
  return p;
}

// Frontier flags hold sweep stamps instead of booleans: sweep t takes part
// for r-cliques whose flag equals stamp(t) = t mod 255 + 1, and notifies by
// writing stamp(t+1) into the other array of the pair.  Old stamps never need
// clearing: a value left from sweep t' matches stamp(t) only when
// t' = t - 254k (harmless extra work; never a skipped r-clique).
__host__ __device__ __forceinline__ uint8_t sweep_stamp(int64_t t) {
  return (uint8_t)(t % 255 + 1);
}

// One r-clique per subgroup of G lanes (sl = lane within the subgroup), each
// lane holding M gathered values of its list [b, b + d), d <= G*M; told its
// value, c the cap.  `eval` false (with d = 0) for a subgroup with no
// r-clique.  SND writes only what it recomputes: a changed r-clique also
// flags itself for the next sweep (the self-activation of Alg. 3), so an
// r-clique skipped in sweep t+1 did not change in sweep t, and the output
// buffer of sweep t+1 (the input of sweep t) already holds its value.
// Returns (on the subgroup's first lane only) whether R changed.
template <int K, int G, int M, typename T, bool AND, bool FR>
__device__ __forceinline__ bool update_list(const int32_t *__restrict__ inc_ids,
                                            const T *tau_in, T *tau_out,
                                            int64_t R, int64_t b, int d,
                                            int32_t told, int32_t c, bool eval,
                                            uint8_t *act_next, uint8_t stamp,
                                            uint8_t *sum_next,
                                            const Support &sp) {
  const int sl = lane_id() % G;
  const int32_t *ids = inc_ids + K * b;
  // With the frontier, which members hold each minimum is kept, so that
  // notifying needs no second gather (notify_kept).  (AND without support
  // counting gathers again, by its own looser test.)
  static_assert(!FR || M <= 4, "lanes with more values would lose occupancy");
  constexpr bool kKeep = FR && K > 1;
  constexpr int kMaskWords = kKeep ? (K * M + 31) / 32 : 1;
  int32_t rho[M];
  uint32_t amask[kMaskWords];
#pragma unroll
  for (int w = 0; w < kMaskWords; w++) amask[w] = 0;
#pragma unroll
  for (int m = 0; m < M; m++) {
    const int j = sl + m * G;
    if (kKeep) {
      uint32_t a = 0;
      rho[m] = (j < d) ? gather_rho_arg<K, T, AND>(ids, j, tau_in, &a) : -1;
#pragma unroll
      for (int x = 0; x < K; x++) {
        const int bit = m * K + x;
        amask[bit >> 5] |= ((a >> x) & 1u) << (bit & 31);
      }
    } else {
      rho[m] = (j < d) ? gather_rho<K, T, AND>(ids, j, tau_in) : -1;
    }
  }
  const int cnt = count_ge<G, M>(rho, c);
  const int32_t h = cnt >= c ? c : hindex_search<G, M>(rho, c, cnt);
  const bool ch = eval && h != told;  // uniform within the subgroup
  const bool lead = sl == 0;
  if (eval && lead) store_tau<T, AND>(tau_out + R, h, ch);
  if (FR && sp.slack && eval && lead)
    ((T *)sp.slack)[R] = slack_word<T>(ch, cnt, c);
  if (FR && ch && act_next) {
    const uint8_t next = stamp == 255 ? 1 : stamp + 1;
    const bool self = !AND || sp.slack != nullptr;
    if (self && lead) self_activate(R, act_next, next, sum_next, sp);
    if (!self)
      notify<K, T, AND>(inc_ids, b, d, sl, G, told, h, tau_in, act_next, next,
                        sum_next, sp);
    else
      notify_kept<K, G, M>(inc_ids, b, d, sl, rho, amask, told, h, act_next,
                           next, sum_next, sp);
  }
  return lead && ch;
}

// The same for one r-clique per wave with d <= kWaveList: the rho values go
// to the wave's own LDS (each lane reads back only what it wrote), four or
// eight gathers a lane in flight, and every count reads them again.  Kept in registers, 8
// or 16 a lane, they set the occupancy of every bin that shares the launch
// (126 registers against 71 on the (3,4) sweeps with notifications).
constexpr int kWaveList = 1024;

template <int K, typename T, bool AND, bool FR>
__device__ __forceinline__ bool update_wave(const int32_t *__restrict__ inc_ids,
                                            const T *tau_in, T *tau_out,
                                            int64_t R, int64_t b, int d,
                                            int32_t told, int32_t c, bool eval,
                                            uint8_t *act_next, uint8_t stamp,
                                            uint8_t *sum_next,
                                            const Support &sp, T *buf) {
  const int lane = lane_id();
  const int32_t *ids = inc_ids + K * b;
  constexpr int kU = FR ? 4 : 8;
  for (int j0 = lane; j0 < d; j0 += kU * kWave) {
    int32_t rho[kU];
#pragma unroll
    for (int u = 0; u < kU; u++) {
      const int j = j0 + u * kWave;
      rho[u] = j < d ? gather_rho<K, T, AND>(ids, j, tau_in) : 0;
    }
#pragma unroll
    for (int u = 0; u < kU; u++) {
      const int j = j0 + u * kWave;
      if (j < d) buf[j] = (T)rho[u];
    }
  }
  auto count = [&](int32_t x) {
    int n = 0;
#pragma unroll 1
    for (int j0 = 0; j0 < d; j0 += 4 * kWave) {  // uniform over the wave
      int32_t v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int j = j0 + u * kWave + lane;
        v[u] = j < d ? (int32_t)buf[j] : -1;
      }
#pragma unroll
      for (int u = 0; u < 4; u++) n += __popcll(ballot(v[u] >= x));
    }
    return n;
  };
  const int cnt = count(c);
  const int32_t h = cnt >= c ? c : hindex_between(count, c, cnt);
  const bool ch = eval && h != told;
  const bool lead = lane == 0;
  if (eval && lead) store_tau<T, AND>(tau_out + R, h, ch);
  if (FR && sp.slack && eval && lead)
    ((T *)sp.slack)[R] = slack_word<T>(ch, cnt, c);
  if (FR && ch && act_next) {
    const uint8_t next = stamp == 255 ? 1 : stamp + 1;
    const bool self = !AND || sp.slack != nullptr;
    if (self && lead) self_activate(R, act_next, next, sum_next, sp);
    if (!self) {
      notify<K, T, AND>(inc_ids, b, d, lane, kWave, told, h, tau_in, act_next,
                        next, sum_next, sp);
    } else {
      // as notify_kept, from the minima in LDS: only the s-cliques whose minimum
      // lies in (h, told] read their members' values again (one that fell
      // meanwhile flags itself), two rows of the wave in flight
      for (int j0 = lane; j0 < d; j0 += 2 * kWave) {
        int32_t rho[2], id[2][K], v[2][K];
#pragma unroll
        for (int u = 0; u < 2; u++) {
          const int j = j0 + u * kWave;
          rho[u] = j < d ? (int32_t)buf[j] : -1;
          const bool may = h < rho[u] && rho[u] <= told;
          if (may) load_ids<K>(ids, j, id[u]);
#pragma unroll
          for (int x = 0; x < K; x++) id[u][x] = may ? id[u][x] : -1;
        }
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
          for (int x = 0; x < K; x++)
            v[u][x] = K == 1 ? rho[u]
                      : id[u][x] >= 0 ? load_tau<T, AND>(tau_at(tau_in, id[u][x]))
                                      : -1;
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
          for (int x = 0; x < K; x++)
            if (id[u][x] >= 0 && v[u][x] == rho[u])
              mark(id[u][x], act_next, next, sum_next, sp);
      }
    }
  }
  return lead && ch;
}

// The same for one r-clique per lane, d <= kLaneList (0 for a lane without):
// values (and which members hold each minimum, as K bits) in the wave's LDS,
// element m of lane l at [64 m + l].  All 64 lanes take part.
constexpr int kLaneList = 16;

template <int K, typename T, bool AND>
__device__ __forceinline__ bool update_lane(const int32_t *__restrict__ inc_ids,
                                            const T *tau_in, T *tau_out, int32_t R,
                                            int64_t b, int d, int32_t told,
                                            int32_t c, bool eval,
                                            uint8_t *act_next, uint8_t stamp,
                                            uint8_t *sum_next, const Support &sp,
                                            T *buf, uint8_t *mbuf) {
  const int lane = lane_id();
  const int32_t *ids = inc_ids + K * b;
  int most = d;  // of the wave
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, kWave));
  most = __builtin_amdgcn_readfirstlane(most);
#pragma unroll 1
  for (int m0 = 0; m0 < most; m0 += 4) {  // four s-cliques a lane in flight
    int32_t rho[4];
    uint32_t arg[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      rho[u] = 0;
      arg[u] = 1;
      if (m0 + u < d) {
        if constexpr (K > 1)
          rho[u] = gather_rho_arg<K, T, AND>(ids, m0 + u, tau_in, &arg[u]);
        else
          rho[u] = gather_rho<K, T, AND>(ids, m0 + u, tau_in);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      buf[(m0 + u) * kWave + lane] = (T)rho[u];
      if (K > 1) mbuf[(m0 + u) * kWave + lane] = (uint8_t)arg[u];
    }
  }
  auto count = [&](int32_t x) {
    int n = 0;
#pragma unroll 1
    for (int m0 = 0; m0 < most; m0 += 4) {
#pragma unroll
      for (int u = 0; u < 4; u++)
        n += m0 + u < d && (int32_t)buf[(m0 + u) * kWave + lane] >= x;
    }
    return n;
  };
  const int cnt = count(c);
  int32_t lo = cnt, hi = c - 1;  // where cnt < c, as hindex_between
  if (cnt >= c) lo = hi = c;
  while (ballot(lo < hi) != 0) {  // uniform
    const int32_t mid = (lo + hi + 1) >> 1;
    const int32_t m = count(mid);
    if (lo < hi) {
      lo = max(lo, min(m, mid));
      if (m < mid) hi = mid - 1;
    }
  }
  const int32_t h = lo;
  const bool ch = eval && h != told;
  if (eval) {
    store_tau<T, AND>(tau_out + R, h, ch);
    if (sp.slack) ((T *)sp.slack)[R] = slack_word<T>(ch, cnt, c);
  }
  if (act_next != nullptr && ballot(ch) != 0) {
    const uint8_t next = stamp == 255 ? 1 : stamp + 1;
    if (!AND || sp.slack != nullptr) {
      if (ch) self_activate(R, act_next, next, sum_next, sp);
#pragma unroll 1
      for (int m0 = 0; m0 < most; m0 += 4) {  // as notify_kept
        int32_t id[4][K];
        uint32_t arg[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          const int m = m0 + u;
          const int32_t rho = (int32_t)buf[m * kWave + lane];
          arg[u] = 0;
          if (ch && m < d && h < rho && rho <= told) {
            arg[u] = K > 1 ? mbuf[m * kWave + lane] : 1;
            load_ids<K>(ids, m, id[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; u++)
#pragma unroll
          for (int x = 0; x < K; x++)
            if ((arg[u] >> x) & 1u) mark(id[u][x], act_next, next, sum_next, sp);
      }
    } else if (ch) {
      notify<K, T, AND>(inc_ids, b, d, 0, 1, told, h, tau_in, act_next, next,
                        sum_next, sp);
    }
  }
  return ch;
}

// update_list of r-clique R, loading its list bounds and value.  `active`
// false for a subgroup with no r-clique; with a frontier (FR), an r-clique
// whose flag is clear is skipped: it cannot change.  *evald (on the
// subgroup's first lane) whether it was recomputed.
template <int K, int G, int M, typename T, bool AND, bool FR>
__device__ __forceinline__ bool update_regs(const int64_t *__restrict__ inc_off,
                                            const int32_t *__restrict__ inc_ids,
                                            const T *tau_in, T *tau_out,
                                            int cap_by_tau, int64_t R,
                                            bool active, const uint8_t *act,
                                            uint8_t *act_next, uint8_t stamp,
                                            bool *evald,
                                            uint8_t *sum_next = nullptr,
                                            const Support &sp = Support()) {
  int32_t told = 0, c = 0;
  int64_t b = 0;
  int d = 0;
  bool eval = active;
  if (active) {
    if (FR && act && act[R] != stamp) {
      eval = false;
    } else {
      told = (int32_t)tau_in[R];
      b = inc_off[R];
      d = (int)(inc_off[R + 1] - b);
      c = cap_by_tau ? told : d;
    }
  }
  *evald = lane_id() % G == 0 && eval;
  return update_list<K, G, M, T, AND, FR>(inc_ids, tau_in, tau_out, R, b, d, told,
                                          c, eval, act_next, stamp, sum_next, sp);
}

// Lane `src` of the wave's value of x: a scalar read where src is uniform.
template <bool UNIFORM>
__device__ __forceinline__ int32_t lane_value(int32_t x, int src) {
  if constexpr (UNIFORM)
    return __builtin_amdgcn_readlane(x, __builtin_amdgcn_readfirstlane(src));
  else
    return __shfl(x, src, kWave);
}
template <bool UNIFORM>
__device__ __forceinline__ int64_t lane_value(int64_t x, int src) {
  const uint32_t lo = (uint32_t)lane_value<UNIFORM>((int32_t)x, src);
  const uint32_t hi = (uint32_t)lane_value<UNIFORM>((int32_t)(x >> 32), src);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Sparse sweep of the r-cliques [lo, hi) of one bin of G lanes per
// r-clique, the frontier's flags being valid.  The calling wave (number
// `wave` of `nwaves`) runs only flagged r-cliques, 64/G at a time, found
// through ballots (nth_set_bit); skipped ones need no write (see
// update_regs).  It finds them either through the group summaries
// (act_sum: one stamp per 64 r-cliques, for the big bins, G <= 4: a step
// tests 64 groups, then loads the flags of flagged groups only, four groups
// in flight: one after the other they were a chain of dependent loads, which
// is what the sweeps of the middle of a decomposition waited on), or by
// loading the flags of kU chunks of kChunk consecutive r-cliques at once
// (one lane per flag, coalesced, the loads in flight together).  A chunk
// holds at most 8 rounds of r-cliques, so a run of flagged hubs is not
// serialised on one wave for long.  Adds the wave's changed / recomputed
// counts to *n_ch / *n_ev.  `spread`: few r-cliques are flagged, and a lane's
// r-cliques (or groups) lie nwaves apart instead of side by side, so that
// flagged ones, which come in clusters, do not queue up on a few waves; with
// many flagged, neighbours on one wave share cache lines.  M = 0: update_wave (G = 64) or update_lane
// (G = 1), in the wave's LDS at buf and mbuf.
template <int K, int G, int M, typename T, bool AND>
__device__ __forceinline__ void sweep_sparse(
    const int64_t *__restrict__ inc_off, const int32_t *__restrict__ inc_ids,
    const T *tin, T *tout, int cap_by_tau, int64_t lo, int64_t hi,
    int64_t wave, int64_t nwaves, const uint8_t *act, uint8_t *act_next,
    uint8_t stamp, unsigned long long *n_ch, unsigned long long *n_ev,
    const uint8_t *act_sum = nullptr, uint8_t *sum_next = nullptr,
    const Support &sp = Support(), T *buf = nullptr, uint8_t *mbuf = nullptr,
    bool spread = false) {
  constexpr int kPerWave = kWave / G;
  const int sub = lane_id() / G;
  const int lane = lane_id();
  // The flagged r-cliques found are queued, one per lane (lane l holds the
  // l-th), and run 64/G at a time when the queue is full or the share ends,
  // so that a group or chunk with one flagged r-clique does not take a whole
  // step of the wave.
  int32_t pend = 0;  // this lane's queued r-clique
  int np = 0;        // queued r-cliques (uniform)
  auto flush = [&]() {
    // every queued r-clique's bounds and value at once, one lane each
    int64_t qb = 0;
    int32_t qd = 0, qt = 0;
    if (lane < np) {
      qb = inc_off[pend];
      qd = (int32_t)(inc_off[pend + 1] - qb);
      qt = (int32_t)tin[pend];
    }
    constexpr bool kUni = G == kWave;
    if constexpr (G == 1 && M == 0) {  // the whole queue in one step
      const bool changed = update_lane<K, T, AND>(
          inc_ids, tin, tout, pend, qb, qd, qt, cap_by_tau ? qt : qd, lane < np,
          act_next, stamp, sum_next, sp, buf, mbuf);
      *n_ch += __popcll(ballot(changed));
      *n_ev += np;
      np = 0;
      return;
    }
#pragma unroll 1
    for (int r0 = 0; r0 < np; r0 += kPerWave) {  // uniform over the wave
      const int t = r0 + sub;
      const bool has = t < np;
      const int src = has ? t : 0;
      const int64_t R = lane_value<kUni>(pend, src);
      const int64_t b = lane_value<kUni>(qb, src);
      // (read by every lane: a lane that does not take part serves no reads)
      const int32_t dq = lane_value<kUni>(qd, src);
      const int32_t told = lane_value<kUni>(qt, src);
      const int32_t d = has ? dq : 0;
      bool changed;
      if constexpr (G == 1 && M == 0)
        changed = false;  // above
      else if constexpr (M == 0)
        changed = update_wave<K, T, AND, true>(
            inc_ids, tin, tout, R, b, d, told, cap_by_tau ? told : d, has,
            act_next, stamp, sum_next, sp, buf);
      else
        changed = update_list<K, G, M, T, AND, true>(
            inc_ids, tin, tout, R, b, d, told, cap_by_tau ? told : d, has,
            act_next, stamp, sum_next, sp);
      *n_ch += __popcll(ballot(changed));
    }
    *n_ev += np;
    np = 0;
  };
  // The words that say whether this lane's r-clique R (`on`: there is one)
  // must run: its flag, or with support counting its losses and slack ...
  auto look = [&](bool on, int64_t R) {
    uint2 w = make_uint2(0, 1);  // (losses or flag, slack)
    if (on) {
      w.x = sp.slack == nullptr ? act[R] : lost_count(sp.lost, sp.shift, R);
      w.y = sp.slack == nullptr ? 1 : (uint32_t)((const T *)sp.slack)[R];
    }
    return w;
  };
  // ... and whether it must (its slack is brought up to date when it need
  // not, its losses are cleared).
  auto must_run = [&](int64_t R, uint2 w) {
    if (sp.slack == nullptr) return w.x == stamp;
    if (w.x) support_store<T>(sp, R, w.y > w.x ? w.y - w.x : 0);
    return w.y <= w.x;
  };
  // queues the flagged r-cliques of mask m (bit i: r-clique cb + i * stride),
  // running the queue first when they would take it past `cap`
  auto queue = [&](uint64_t m, int64_t cb, int stride, int cap) {
    const int na = __popcll(m);
    if (np + na > cap) flush();
    const int slot = lane - np;  // the slot-th flagged r-clique of m
    if (slot >= 0 && slot < na) pend = (int32_t)cb + nth_set_bit(m, slot) * stride;
    np += na;
  };
  if (G <= 4 && act_sum != nullptr) {
    // Big bins: test 64 group summaries per step (one lane each), then the
    // flags of each flagged group only.  A sweep with few flagged r-cliques
    // reads 1/64 of the flags.
    // A bin with fewer groups than 64 per wave takes fewer per step, so that
    // every wave has some: a wave running hundreds of flagged r-cliques one
    // step after the other is a chain of dependent loads (0.1 ms for 9000
    // flagged of 65000, where a full sweep takes 17 us).
    const int64_t g_lo = lo >> kGroupShift;
    const int64_t g_hi = (hi + (1 << kGroupShift) - 1) >> kGroupShift;
    const int64_t share = (g_hi - g_lo + nwaves - 1) / nwaves;
    const int step = spread || share > kWave ? kWave : (int)share;
    const int64_t apart = spread ? nwaves : 1;  // between a lane's groups
    for (int64_t gb = g_lo + wave * (spread ? 1 : step); gb < g_hi;
         gb += nwaves * step) {
      const int64_t gi = gb + lane * apart;
      uint64_t gm = ballot(lane < step && gi < g_hi && act_sum[gi] == stamp);
      constexpr int kFly = 4;  // flagged groups in flight
      while (gm) {  // uniform over the wave
        uint2 w[kFly];
        int q[kFly];
#pragma unroll
        for (int u = 0; u < kFly; u++) {
          q[u] = gm ? __ffsll((unsigned long long)gm) - 1 : -1;
          gm &= gm - 1;
          const int64_t Rl = ((gb + q[u] * apart) << kGroupShift) + lane;
          w[u] = look(q[u] >= 0 && Rl >= lo && Rl < hi, Rl);
        }
        // lane u keeps group u's number and mask until it is queued
        uint32_t m_lo = 0, m_hi = 0;
        int q_at = 0;
#pragma unroll
        for (int u = 0; u < kFly; u++) {
          const int64_t Rl = ((gb + q[u] * apart) << kGroupShift) + lane;
          const uint64_t m = ballot(must_run(Rl, w[u]));
          if (lane == u) {
            m_lo = (uint32_t)m;
            m_hi = (uint32_t)(m >> 32);
            q_at = q[u];
          }
        }
#pragma unroll 1
        for (int u = 0; u < kFly; u++) {
          const uint64_t m =
              ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(m_hi, u) << 32) |
              (uint32_t)__builtin_amdgcn_readlane(m_lo, u);
          if (m)
            queue(m, (gb + __builtin_amdgcn_readlane(q_at, u) * apart) << kGroupShift,
                  1, kWave);
        }
      }
    }
    if (np > 0) flush();
    return;
  }
  if (spread) {
    for (int64_t base = lo + wave; base < hi; base += nwaves * kWave) {
      const int64_t Rl = base + lane * nwaves;
      const uint64_t m = ballot(must_run(Rl, look(Rl < hi, Rl)));
      if (m) queue(m, base, (int)nwaves, kWave);
    }
    if (np > 0) flush();
    return;
  }
  // At most 8 rounds of r-cliques per chunk and per queue, so that a run of
  // flagged hubs is not serialised on one wave for long.
  constexpr int kChunk = kPerWave * 8 < kWave ? kPerWave * 8 : kWave;
  // Several chunks per step only where a chunk is narrow work (G <= 4: the
  // big bins, where the flag scan dominates a sparse sweep); for wide
  // mappings a step of kU chunks would serialise up to 8 kU hub r-cliques
  // on one wave.
  constexpr int kU = G <= 4 ? 8 : 1;
  constexpr int64_t kStep = (int64_t)kChunk * kU;
  for (int64_t base = lo + wave * kStep; base < hi; base += nwaves * kStep) {
    uint2 w[kU];
#pragma unroll
    for (int u = 0; u < kU; u++) {
      const int64_t Rl = base + (int64_t)u * kChunk + lane;
      w[u] = look(lane < kChunk && Rl < hi, Rl);
    }
#pragma unroll
    for (int u = 0; u < kU; u++) {
      const int64_t cb = base + (int64_t)u * kChunk;
      const uint64_t m = ballot(must_run(cb + lane, w[u]));
      if (m) queue(m, cb, 1, kChunk);
    }
  }
  if (np > 0) flush();
}

// LDS of one workgroup on a hub.
struct HubLds {
  int32_t hist[kHubBins];
  int64_t part[kBlockThreads / kWave];
  int32_t best;
  int32_t found[kBlockThreads];  // the hubs of a share that must run
  int32_t nfound;
};

__device__ __forceinline__ int64_t block_sum(int64_t x, HubLds &L) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  if (lane_id() == 0) L.part[threadIdx.x / kWave] = x;
  __syncthreads();
  int64_t s = 0;
#pragma unroll
  for (int w = 0; w < kBlockThreads / kWave; w++) s += L.part[w];
  __syncthreads();
  return s;
}

// Bins hist[0..nb) count values, bin i standing for x0 + (i << shift) and up.
// Returns the largest i with base + sum_{i' >= i} hist[i'] >= x0 + (i <<
// shift), or -1 if there is none; *over: base plus the counts of the bins
// above it.  All threads of the block call it.
__device__ inline int suffix_search(HubLds &L, const int32_t *hist, int nb,
                                    int64_t base, int64_t x0, int shift,
                                    int64_t *over) {
  const int t = threadIdx.x;
  const int chunk = (nb + kBlockThreads - 1) / kBlockThreads;
  const int lo = min(nb, t * chunk), hi = min(nb, lo + chunk);
  int64_t mine = 0;
  for (int i = lo; i < hi; i++) mine += hist[i];
  // what the chunks above mine hold: lanes above in the wave, waves above
  int64_t inc = mine;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t y = __shfl_down(inc, off, kWave);
    if (lane_id() + off < kWave) inc += y;
  }
  if (lane_id() == 0) L.part[t / kWave] = inc;
  if (t == 0) L.best = -1;
  __syncthreads();
  int64_t run = base + inc - mine;
#pragma unroll
  for (int w = 1; w < kBlockThreads / kWave; w++)
    if (w > t / kWave) run += L.part[w];
  __syncthreads();
  int found = -1;
  int64_t at = 0;
  for (int i = hi - 1; i >= lo; i--) {
    if (run + hist[i] >= x0 + ((int64_t)i << shift)) {
      found = i;
      at = run;
      break;
    }
    run += hist[i];
  }
  if (found >= 0) atomicMax(&L.best, found);
  __syncthreads();
  const int r = L.best;
  if (found == r && r >= 0) L.part[0] = at;
  __syncthreads();
  *over = L.part[0];
  __syncthreads();
  return r;
}

// One r-clique per 256-thread workgroup, any d_s (the bins above 1024 use
// it).  Each thread keeps kU gathers in flight (ids, then tau values), or one
// workgroup's walk of a long list is a chain of dependent loads.  Values >= c
// are only counted; when fewer than c reach c, H comes from an LDS histogram
// of the others: one bin per value in the kHubTop values below c (H is mostly
// just below the old value), 2^shift values per bin further down, and another
// walk of the list over the coarse bin that holds H (only the first sweeps
// get there, whose caps are the degrees).  16 KiB of bins instead of one per
// value up to 64 KiB let the hubs share a launch with the other bins.
// Returns whether R changed (thread 0 only).
constexpr int kHubTop = kHubBins / 2;

template <int K, typename T, bool AND, bool FR>
__device__ bool update_hub(const int64_t *__restrict__ inc_off,
                           const int32_t *__restrict__ inc_ids,
                           const T *tau_in, T *tau_out, int cap_by_tau,
                           int64_t R, HubLds &L, uint8_t *act_next,
                           uint8_t stamp, uint8_t *sum_next,
                           const Support &sp) {
  const int t = threadIdx.x;
  const int32_t told = (int32_t)tau_in[R];
  const int64_t b = inc_off[R];
  const int64_t d = inc_off[R + 1] - b;
  const int32_t *ids = inc_ids + K * b;
  const int32_t c = cap_by_tau ? told : (int32_t)d;
  const int32_t top = max(0, c - kHubTop);  // [top, c): a bin per value
  int shift = 0;                            // [0, top): 2^shift per bin
  while ((top >> shift) >= kHubBins - kHubTop) shift++;
  for (int x = t; x < kHubBins; x += kBlockThreads) L.hist[x] = 0;
  __syncthreads();
  constexpr int kU = K == 1 ? 8 : K == 2 ? 6 : 4;
  int64_t ge = 0;
  for (int64_t j0 = t; j0 < d; j0 += (int64_t)kBlockThreads * kU) {
    int32_t rho[kU];
#pragma unroll
    for (int u = 0; u < kU; u++) {
      const int64_t j = j0 + (int64_t)u * kBlockThreads;
      rho[u] = j < d ? gather_rho<K, T, AND>(ids, j, tau_in) : -1;
    }
#pragma unroll
    for (int u = 0; u < kU; u++) {
      if (rho[u] >= c)
        ge++;
      else if (rho[u] >= top)
        atomicAdd(&L.hist[rho[u] - top], 1);
      else if (rho[u] >= 0)
        atomicAdd(&L.hist[kHubTop + (rho[u] >> shift)], 1);
    }
  }
  ge = block_sum(ge, L);  // also: the histogram is complete
  int32_t h = c;
  if (ge < c) {
    int64_t over;
    int i = suffix_search(L, L.hist, c - top, ge, top, 0, &over);
    if (i >= 0) {
      h = top + i;
    } else {
      // below the window: over counts everything from `top` up
      int64_t mine = 0;
      for (int x = t; x < c - top; x += kBlockThreads) mine += L.hist[x];
      over = ge + block_sum(mine, L);
      int64_t x0 = 0;
      int nb = (int)(((int64_t)top + ((int64_t)1 << shift) - 1) >> shift);
      i = suffix_search(L, L.hist + kHubTop, nb, over, 0, shift, &over);
      x0 = (int64_t)i << shift;
      // H lies in [x0, x0 + 2^shift); over: values at or above its end
      while (shift > 0) {
        const int64_t x1 = min((int64_t)top, x0 + ((int64_t)1 << shift));
        int s2 = 0;
        while (((x1 - x0) >> s2) >= kHubBins) s2++;
        nb = (int)((x1 - x0 + ((int64_t)1 << s2) - 1) >> s2);
        for (int x = t; x < nb; x += kBlockThreads) L.hist[x] = 0;
        __syncthreads();
        int64_t up = 0;
        for (int64_t j0 = t; j0 < d; j0 += (int64_t)kBlockThreads * kU) {
          int32_t rho[kU];
#pragma unroll
          for (int u = 0; u < kU; u++) {
            const int64_t j = j0 + (int64_t)u * kBlockThreads;
            rho[u] = j < d ? gather_rho<K, T, AND>(ids, j, tau_in) : -1;
          }
#pragma unroll
          for (int u = 0; u < kU; u++) {
            if (rho[u] >= x1)
              up++;
            else if (rho[u] >= x0)
              atomicAdd(&L.hist[(rho[u] - x0) >> s2], 1);
          }
        }
        up = block_sum(up, L);  // AND: values may have fallen since
        const int f = suffix_search(L, L.hist, nb, up, x0, s2, &over);
        if (f < 0) break;  // AND only: nothing at or above x0 is left of H
        x0 += (int64_t)f << s2;
        shift = s2;
      }
      h = (int32_t)x0;
    }
  }
  const bool ch = h != told;
  const bool notifies = FR && ch && act_next != nullptr;
  // AND with support counting notifies before R's value is written (notify; with
  // k = 1 S has no third member)
  const bool first = AND && K > 1 && sp.slack != nullptr && notifies;
  if (t == 0 && !first) store_tau<T, AND>(tau_out + R, h, ch);
  if (FR && sp.slack && t == 0)
    ((T *)sp.slack)[R] = slack_word<T>(ch, ge, c);
  if (notifies) {
    const uint8_t next = stamp == 255 ? 1 : stamp + 1;
    if ((!AND || sp.slack) && t == 0)
      self_activate(R, act_next, next, sum_next, sp);
    notify<K, T, AND>(inc_ids, b, d, t, kBlockThreads, told, h, tau_in,
                      act_next, next, sum_next, sp);
  }
  if (first) {
    __syncthreads();  // every thread has read
    if (t == 0) store_tau<T, AND>(tau_out + R, h, true);
  }
  __syncthreads();
  return t == 0 && ch;
}

}  // namespace dev
}  // namespace nd
