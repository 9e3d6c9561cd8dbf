// partition.h -- stable partition of 0..n-1 by a small key (a sweep bin, an
// intersection bin), shared by prim.hip and layout.hip.  Internal header.
//
// A wave takes kPartItems rows of 64 consecutive items.  Equal keys within a
// row are matched with four ballots (keys have four bits) and a per-wave
// counter in LDS carries each key's count on to the next row, so an item's
// rank is known after one pass and no atomics are used; its place follows
// from the scanned (bin, workgroup) counts.  Bound by the key read twice and
// the outputs written once; sorting (bin, item) keys by radix moved 24 bytes
// an item more and took five launches where this takes three, or one up to
// kPartOne items, which one workgroup counts and places by itself.  (A ballot
// per bin and row instead of four per row took 12 and 20 us for the two passes
// over a hundred thousand items.)
#pragma once

#include <algorithm>

#include "internal.h"

namespace nd {
namespace part {

constexpr int kPartItems = 16;
constexpr int kPartThreads = 256;
constexpr int kPartTile = kPartThreads * kPartItems;  // 4096
constexpr int kPartBig = 1024;
constexpr int64_t kPartOne = (int64_t)kPartBig * kPartItems;  // 16384
// Up to this many workgroups each adds up the counts before it, one thread a
// bin; the launch that would scan them takes longer.
constexpr int64_t kPartSelf = 64;

// Where the partition ends up on the host's side: the first item of every
// bin, the total, and the largest of the values that `most` gives.
constexpr int kMaxBins = 16;
struct Head {
  int64_t start[kMaxBins + 1];
  int32_t most;
};

// Ranks of this wave's items (bin[r] of row r, -1: none) among those of the
// same bin, in item order; cnt (this wave's, zeroed here) ends as the counts.
__device__ __forceinline__ void wave_ranks(const int (&bin)[kPartItems],
                                           int32_t *cnt, int32_t (&rank)[kPartItems]) {
  const int lane = lane_id();
  if (lane < kMaxBins) cnt[lane] = 0;
#pragma unroll
  for (int r = 0; r < kPartItems; r++) {
    const bool valid = bin[r] >= 0;
    uint64_t peers = ballot(valid);
#pragma unroll
    for (int b = 0; b < 4; b++) {
      const bool bit = (bin[r] >> b) & 1;
      const uint64_t m = ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int below = lanes_below(peers);
    // one wave's LDS accesses are served in order
    __builtin_amdgcn_wave_barrier();
    const int32_t before = valid ? cnt[bin[r]] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) cnt[bin[r]] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    rank[r] = before + below;
  }
}

// In: load(i, &most) returns item i's bin in [0, NB) and raises most to the
// item's value.  In and Out: local() the same with what it reads once a thread
// already read.
template <int NB, typename In>
__global__ __launch_bounds__(kPartThreads) void k_part_count(
    In in_, int64_t n, int64_t nb, int32_t *__restrict__ count,
    int32_t *__restrict__ block_most) {
  const In in = in_.local();
  __shared__ int32_t c[kPartThreads / kWave][kMaxBins];
  __shared__ int32_t cm[kPartThreads / kWave];
  const int w = threadIdx.x / kWave, lane = lane_id(), t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kPartTile + w * kWave * kPartItems + lane;
  int32_t most = 0;
  int bin[kPartItems];
  int32_t rank[kPartItems];
#pragma unroll
  for (int r = 0; r < kPartItems; r++) {
    const int64_t i = base + r * kWave;
    bin[r] = i < n ? in.load(i, &most) : -1;
  }
  wave_ranks(bin, c[w], rank);
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, kWave));
  if (lane == 0) cm[w] = most;
  __syncthreads();
  if (t < NB) count[t * nb + blockIdx.x] = c[0][t] + c[1][t] + c[2][t] + c[3][t];
  if (t == NB) block_most[blockIdx.x] = max(max(cm[0], cm[1]), max(cm[2], cm[3]));
}

// Out: put(i, place) of item i.  off: the scanned counts, or NULL: the
// workgroup adds up `count` itself (NULL too for the only workgroup, which
// counts for itself).  Workgroup 0 also writes the head.
template <int NB, int NT, typename In, typename Out>
__global__ __launch_bounds__(NT) void k_part_place(
    In in_, Out out_, int64_t n, int64_t nb, const int32_t *__restrict__ count,
    const int64_t *__restrict__ off, const int32_t *__restrict__ block_most,
    Head *__restrict__ head) {
  const In in = in_.local();
  const Out out = out_.local();
  constexpr int kWaves = NT / kWave;
  __shared__ int32_t c[kWaves][kMaxBins];
  __shared__ int32_t cm[kWaves];
  __shared__ int64_t at[NB];  // first place of this workgroup's bins
  const int w = threadIdx.x / kWave, lane = lane_id(), t = threadIdx.x;
  const int64_t base =
      (int64_t)blockIdx.x * (NT * kPartItems) + w * kWave * kPartItems + lane;
  int bin[kPartItems];
  int32_t rank[kPartItems];
  int32_t most = 0;
#pragma unroll
  for (int r = 0; r < kPartItems; r++) {
    const int64_t i = base + r * kWave;
    bin[r] = i < n ? in.load(i, &most) : -1;
  }
  wave_ranks(bin, c[w], rank);
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, kWave));
  if (lane == 0) cm[w] = most;
  __syncthreads();
  // bin t: its waves' starts within the workgroup, its start
  __shared__ int64_t first[NB];  // of the whole bins, without `off`
  int64_t before = 0;            // bin t's items of earlier workgroups
  if (t < NB) {
    int32_t run = 0;
    for (int x = 0; x < kWaves; x++) {
      const int32_t y = c[x][t];
      c[x][t] = run;
      run += y;
    }
    if (off != nullptr) {
      at[t] = off[t * nb + blockIdx.x];
    } else {
      int64_t all = run;
      if (count != nullptr) {
        all = 0;
        for (int b = 0; b < (int)nb; b++) {
          const int32_t y = count[t * nb + b];
          before += b < (int)blockIdx.x ? y : 0;
          all += y;
        }
      }
      first[t] = all;
    }
  }
  __syncthreads();
  if (off == nullptr) {  // the bins' totals to their starts
    if (t == 0) {
      int64_t run = 0;
      for (int b = 0; b < NB; b++) {
        const int64_t y = first[b];
        first[b] = run;
        run += y;
      }
    }
    __syncthreads();
    if (t < NB) at[t] = first[t] + before;
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kPartItems; r++)
    if (bin[r] >= 0)
      out.put(base + r * kWave, (int32_t)at[bin[r]] + c[w][bin[r]] + rank[r]);
  if (blockIdx.x != 0) return;
  if (t < NB) head->start[t] = off != nullptr ? off[t * nb] : first[t];
  int32_t m = 0;
  if (block_most != nullptr) {
    for (int64_t x = t; x < nb; x += NT) m = max(m, block_most[x]);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
    if (lane == 0) cm[w] = m;
    __syncthreads();
  }
  if (t == 0) {
    m = 0;
    for (int x = 0; x < kWaves; x++) m = max(m, cm[x]);
    head->start[NB] = n;
    head->most = m;
  }
}

// Partition 0..n-1, 0 < n < 2^31, into NB bins (ordered on s); head: device
// memory.
template <int NB, typename In, typename Out>
void run(const In &in, const Out &out, int64_t n, Head *head, hipStream_t s,
         Allocator &al) {
  static_assert(NB <= kMaxBins, "a bin has four bits");
  ND_REQUIRE(n < ((int64_t)1 << 31), ND_ERR_INVALID,
             "%lld items: places must fit int32", (long long)n);
  if (n <= kPartOne) {
    k_part_place<NB, kPartBig><<<1, kPartBig, 0, s>>>(in, out, n, 1, nullptr,
                                                      nullptr, nullptr, head);
    ND_LAUNCHED();
    return;
  }
  const int64_t nb = ceil_div(n, kPartTile);
  const bool self = nb <= kPartSelf;
  DArr<int32_t> count(al, NB * nb), most(al, nb);
  DArr<int64_t> off;
  k_part_count<NB><<<(unsigned)nb, kPartThreads, 0, s>>>(in, n, nb, count.p, most.p);
  ND_LAUNCHED();
  if (!self) {
    off.reset(al, NB * nb + 1);
    exclusive_scan_i32(count.p, off.p, NB * nb, s, al);
  }
  k_part_place<NB, kPartThreads><<<(unsigned)nb, kPartThreads, 0, s>>>(
      in, out, n, nb, count.p, off.p, most.p, head);
  ND_LAUNCHED();
}

}  // namespace part
}  // namespace nd
