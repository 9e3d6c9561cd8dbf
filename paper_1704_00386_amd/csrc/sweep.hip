// sweep.hip -- one application of the update operator U to every r-clique
// (Section 3, Defn. of U; the parallel loop of Alg. 2 and Alg. 3):
//
//   rho(S,R)  = min over the k other r-cliques R' of S of tau(R')  (gather+min)
//   tau'(R)   = H({rho(S,R)} over the d_s(R) s-cliques S containing R)
//   changed  += (tau'(R) != tau(R))                         (convergence flag)
//
// r-cliques are in the internal numbering (grouped by bin), so each bin is a
// contiguous id range and the incidence lists are read in one sequential,
// coalesced stream; the tau reads are the random part.  tau is stored as
// uint16 when every d_s fits (then every tau does: tau <= d_s), halving the
// bytes of the gathered array.
//
// H is computed exactly with a cap c (Section 4.4 "can the current value be
// preserved" check, made exact):
//   * H(min(K,c)) = min(H(K), c) for any multiset K and any c >= 0, and
//     H(K) <= |K| = d_s(R), so with c = d_s(R) the cap never changes H.
//   * For the iterates of SND/AND, U tau(R) <= tau(R) (Theorem 1, and the same
//     argument for in-place sweeps, whose inputs only decrease), so c = tau(R)
//     is exact there too and keeps the work small.
//   * If #{rho >= c} >= c then H = c (the preserve check).  Otherwise H is
//     the largest x < c with #{rho >= x} >= x, found by binary search on x
//     with counts reduced across the lanes that hold the rho values.
//
// Mappings by S-degree bin:
//   d_s <= 256     G = 1/4/16/64 lanes per r-clique, 4 rho values per lane;
//                  a full sweep gathers each run of r-cliques flat first
//                  (one lane per incidence entry, minima to LDS), then
//                  computes H from LDS (sweep_flat)
//   257..1024      one wave per r-clique, its rho values in LDS (update_wave)
//   >= 1025        one 256-thread workgroup per r-clique, LDS histogram of
//                  the values below the cap (update_hub)
//                  full sweeps of 513..2047 hold their values in registers, in
//                  launches of their own, where such lists fill the GPU
//                  (swept_apart)
// SND reads tau_t and writes tau_{t+1} (double buffer, race free, so every
// iterate is deterministic).  AND reads and writes one array in place with
// relaxed workgroup-scope atomics: a value read may predate another
// workgroup's write in the same sweep but never the sweep's start, and
// writes only ever lower values (Section 4.2; see load_tau).
#include <algorithm>

#include "sweep_dev.h"

namespace nd {

// One sweep of the bins of ks for k = K and tau of type T (sweep_inst.hip).
template <int K, typename T>
void sweep_kind(const KindState &ks, const SweepArgs &a, bool and_mode,
                hipStream_t s);

namespace {

using namespace dev;

template <typename T>
__global__ void k_zero_range(T *__restrict__ tau, int64_t lo, int64_t hi) {
  const int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < hi) tau[i] = 0;
}

template <typename T>
void launch_typed(const KindState &ks, const SweepArgs &a, bool and_mode,
                  hipStream_t s) {
  if (!a.cap_by_tau) {
    // plain U on an arbitrary tau: r-cliques in no s-clique get H({}) = 0
    const int64_t lo = ks.bin_lo[kBinZero], hi = ks.bin_hi[kBinZero];
    if (hi > lo) {
      k_zero_range<T><<<grid_for(hi - lo, 256), 256, 0, s>>>((T *)a.tau_out, lo, hi);
      ND_LAUNCHED();
    }
  }
  switch (ks.k) {
    case 1: sweep_kind<1, T>(ks, a, and_mode, s); break;
    case 2: sweep_kind<2, T>(ks, a, and_mode, s); break;
    case 3: sweep_kind<3, T>(ks, a, and_mode, s); break;
    case 5: sweep_kind<5, T>(ks, a, and_mode, s); break;
    default:
      ND_REQUIRE(false, ND_ERR_UNSUPPORTED, "no sweep kernel for k=%d", ks.k);
  }
}

// The group summaries of the flags a dense notifying sweep wrote without
// them: a thread per group of 64 flags (four 16-byte loads), striding, which
// stores the next stamp into the group's summary when any of its flags holds
// it.  Runs only when the sweep it follows took that path (the same test as
// frontier_mode, on the same counters); a small grid keeps the launches that
// find nothing to do cheap.
constexpr int kGroupSumsBlocks = 1024;

// Any nonzero counter (1 << shift bytes each) among [f0, f1), at most 64 of
// them from a multiple of 64: 16 bytes at a time where the group is whole.
__device__ __forceinline__ bool any_nonzero(const void *lost, int64_t f0,
                                            int64_t f1, int shift) {
  bool any = false;
  if (f1 - f0 == (1 << kGroupShift)) {
    const uint4 *p = reinterpret_cast<const uint4 *>((const char *)lost + (f0 << shift));
    for (int v = 0; v < (4 << shift); v++) {
      const uint4 w = p[v];
      any |= (w.x | w.y | w.z | w.w) != 0;
    }
  } else {
    for (int64_t f = f0; f < f1; f++) any |= lost_count(lost, shift, f) != 0;
  }
  return any;
}

// Any zero word among [f0, f1).
template <typename T>
__device__ __forceinline__ bool any_zero(const T *w, int64_t f0, int64_t f1) {
  bool any = false;
  if (sizeof(T) == 1 && f1 - f0 == (1 << kGroupShift)) {
    const uint32_t *p = reinterpret_cast<const uint32_t *>(w + f0);
#pragma unroll
    for (int v = 0; v < 16; v++)
      any |= ((p[v] - 0x01010101u) & ~p[v] & 0x80808080u) != 0;
  } else {
    for (int64_t f = f0; f < f1; f++) any |= w[f] == 0;
  }
  return any;
}

// T: the type of tau, for the slack words of support counting.
template <typename T>
__global__ __launch_bounds__(256) void k_group_sums(SweepArgs a, int64_t nr) {
  const unsigned long long pc = prev_changed(a);
  if (pc == 0 || a.sums_after == 0 || pc < a.sums_after) return;
  const bool notify = a.prev != nullptr
                          ? (a.prev->notified || pc <= a.notify_below)
                          : a.notify_first != 0;
  if (!notify) return;
  const uint8_t next = a.stamp == 255 ? 1 : a.stamp + 1;
  const int64_t ng = (nr + (1 << kGroupShift) - 1) >> kGroupShift;
  const uint32_t pat = 0x01010101u * next;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < ng;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t f0 = g << kGroupShift;
    bool any = false;
    if (a.slack != nullptr) {
      const int64_t f1 = std::min<int64_t>(nr, f0 + (1 << kGroupShift));
      any = any_nonzero(a.lost_next, f0, f1, a.lost_shift);
      if (!any) any = any_zero<T>((const T *)a.slack, f0, f1);
    } else if (f0 + (1 << kGroupShift) <= nr) {
      const uint4 *p = reinterpret_cast<const uint4 *>(a.act_next + f0);
#pragma unroll
      for (int v = 0; v < (1 << kGroupShift) / 16; v++) {
        const uint4 w = p[v];
        const uint32_t x[4] = {w.x ^ pat, w.y ^ pat, w.z ^ pat, w.w ^ pat};
#pragma unroll
        for (int c = 0; c < 4; c++)  // a zero byte: a flag equal to next
          any |= ((x[c] - 0x01010101u) & ~x[c] & 0x80808080u) != 0;
      }
    } else {
      for (int64_t f = f0; f < nr; f++) any |= a.act_next[f] == next;
    }
    if (any) a.act_sum_next[g] = next;
  }
}

}  // namespace

void launch_group_sums(const KindState &ks, const SweepArgs &a, hipStream_t s) {
  if (a.sums_after == 0 || a.act_next == nullptr || a.act_sum_next == nullptr ||
      ks.nr == 0)
    return;
  const int64_t swept = ks.bin_lo[kBinZero];  // the others are never notified
  const int64_t ng = (swept + (1 << dev::kGroupShift) - 1) >> dev::kGroupShift;
  const unsigned grid =
      (unsigned)std::min<int64_t>(grid_for(ng, 256), kGroupSumsBlocks);
  if (a.tau_bytes == 1)
    k_group_sums<uint8_t><<<grid, 256, 0, s>>>(a, swept);
  else if (a.tau_bytes == 2)
    k_group_sums<uint16_t><<<grid, 256, 0, s>>>(a, swept);
  else
    k_group_sums<int32_t><<<grid, 256, 0, s>>>(a, swept);
  ND_LAUNCHED();
}

void launch_sweep(const KindState &ks, const SweepArgs &a, bool and_mode,
                  hipStream_t s) {
  if (a.tau_bytes == 1)
    launch_typed<uint8_t>(ks, a, and_mode, s);
  else if (a.tau_bytes == 2)
    launch_typed<uint16_t>(ks, a, and_mode, s);
  else
    launch_typed<int32_t>(ks, a, and_mode, s);
}

}  // namespace nd
