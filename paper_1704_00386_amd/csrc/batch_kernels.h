// batch_kernels.h -- the batches' tile kernel for one k = C(s,r) - 1 and one
// type of tau, compiled beside the one-graph sweeps (sweep_inst.hip).
// Internal header.
#pragma once

#include "batch.h"
#include "sweep_kernels.h"

namespace nd {

namespace {

// Lists of 1025..2047 take a workgroup each (sweep_hubs), or in a tile of this
// many, which four waves share well, a wave each, through twice the LDS that
// lists of up to 1024 take, where the hubs' LDS holds it (16-bit values): 16
// k-cores of 2500 vertices with lists of 1200, 3.01 -> 2.41 ms.
constexpr int kWaveTile = 8;

// One epoch's tiles, one workgroup per tile (the grid is the table's
// capacity, surplus workgroups exit at once).  Workgroups are short-lived, so
// the work of other streams (a server's preparations) is dispatched between
// them rather than waiting for the epoch to end.  A tile is swept as the
// one-graph sweep would sweep it (sweep_kernels.h): flat while nothing is
// flagged, then by flags or support counts.
template <int K, typename T, bool AND, bool FR>
__global__ __launch_bounds__(256, 6) void k_batch_sweep(
    const BGraph *__restrict__ gs, const BTile *__restrict__ tiles,
    const BState *__restrict__ st) {
  __shared__ union {
    FlatLds<T> flat;
    HubLds hub;
  } lds;
  const int ti = (int)blockIdx.x;
  if (ti >= st->ntiles) return;
  const BTile tile = tiles[ti];
  const BGraph &G = gs[tile.g];
  const int64_t local = st->epoch - G.t0;
  if (local < 0 || local >= G.max_local) return;
  const SweepStats *prev = local > 0 ? &G.ring[(local - 1) % kBatchRing] : nullptr;
  const unsigned long long pc = prev != nullptr ? prev->total : 1;
  if (pc == 0) return;  // converged
  SweepArgs a{};
  a.inc_off = G.inc_off;
  a.inc_ids = G.inc_ids;
  a.tau_in = G.tau[local & 1];
  a.tau_out = G.tau[AND ? (local & 1) : ((local + 1) & 1)];
  a.stats = &G.ring[local % kBatchRing];
  a.cap_by_tau = 1;
  a.stamp = sweep_stamp(local);
  // frontier state of this graph's sweep: the rule of the one-graph sweep
  const uint8_t *act = nullptr, *act_sum = nullptr;
  uint8_t *act_next = nullptr, *sum_next = nullptr;
  Support sp;
  if (FR && prev != nullptr) {
    const bool valid = prev->notified != 0;
    if (valid) {
      act = G.act[local & 1];
      act_sum = G.act_sum[local & 1];
    }
    if (valid || pc <= G.notify_below) {
      act_next = G.act[(local + 1) & 1];
      sum_next = G.act_sum[(local + 1) & 1];
      if (threadIdx.x == 0) a.stats->notified = 1;
      sp.slack = G.slack;
    }
  }
  if (FR) {  // read only while slack is kept
    sp.lost = G.act[local & 1];
    sp.lost_next = G.act[(local + 1) & 1];
    sp.shift = (int)G.lost_shift;
  }
  int type = tile.type, list = kWaveList;
  if (sizeof(T) == 2 && type == kBinWave && tile.hi - tile.lo >= kWaveTile) {
    type = kBinWave16;
    list = 2 * kWaveList;
    static_assert(sizeof(T) != 2 || sizeof(lds) >= 8 * kWaveList * sizeof(T),
                  "four lists of the bin fit");
  }
  switch (type) {
    case kBinBlock:
    case kBinWave:
      sweep_hubs<K, T, AND, FR>(a, tile.lo, tile.hi, 0, 1, act, act_next, sum_next,
                                sp, lds.hub);
      break;
    case kBinWave16:
    case kBinWave8:
      sweep_bin<K, 64, 0, T, AND, FR>(a, tile.lo, tile.hi, 0, 1, act, act_next,
                                      act_sum, sum_next, sp, &lds.flat, false, list);
      break;
    case kBinG64:
      sweep_bin<K, 64, 4, T, AND, FR>(a, tile.lo, tile.hi, 0, 1, act, act_next,
                                      act_sum, sum_next, sp, &lds.flat, false);
      break;
    case kBinG16:
      sweep_bin<K, 16, 4, T, AND, FR>(a, tile.lo, tile.hi, 0, 1, act, act_next,
                                      act_sum, sum_next, sp, &lds.flat, false);
      break;
    case kBinG4:
      sweep_bin<K, 4, 4, T, AND, FR>(a, tile.lo, tile.hi, 0, 1, act, act_next,
                                     act_sum, sum_next, sp, &lds.flat, false);
      break;
    default:  // kBinG1
      sweep_bin<K, 1, 4, T, AND, FR>(a, tile.lo, tile.hi, 0, 1, act, act_next,
                                     act_sum, sum_next, sp, &lds.flat, false);
      break;
  }
}

}  // namespace

template <int K, typename T>
const void *batch_kernel(bool and_mode, bool fr) {
  if (and_mode)
    return fr ? (const void *)k_batch_sweep<K, T, true, true>
              : (const void *)k_batch_sweep<K, T, true, false>;
  return fr ? (const void *)k_batch_sweep<K, T, false, true>
            : (const void *)k_batch_sweep<K, T, false, false>;
}

}  // namespace nd
