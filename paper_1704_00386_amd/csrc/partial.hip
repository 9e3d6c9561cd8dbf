// partial.hip -- ego-network estimates by PartialAND (the set-restricted AND
// of Section 4.3, end, applied as in Section 5.3): for a
// query r-clique q, AND recomputes only the r-cliques of
//   P(q) = {q} + every r-clique sharing an s-clique with q
// (for k-core: q and its neighbours; for k-truss: q and the other edges of
// its triangles), every other r-clique keeping tau_0 = d_s, until a sweep
// changes nothing; the estimate is q's resulting value, an upper bound on
// kappa(q).
//
// The restricted operator is monotone and tau_0 lies above its image, so
// in-place sweeps in any order reach the same limit -- the largest fixed
// point below tau_0 -- and each query's result is deterministic although the
// sweeps inside a workgroup race.
//
// Many queries run in one launch, one workgroup each (the many-small-
// problems shape of serving): P(q) is sorted into LDS together with the
// members' current values, with a bitmap of hashed ids in front: most
// gathered ids lie outside P(q), and one LDS word tells so (then the value is
// d_s from global memory) where the binary search took up to twelve dependent
// reads.  One wave recomputes one member at a time, its rho values in
// registers (4, 8, 16 or 32 per lane by d_s) or re-gathered per probe of the
// h-index search (d_s > 2048).  After the first sweep only members that a
// fallen neighbour may have pulled below their value run again (a byte each).
// Queries go out heaviest first (by the query's own d_s) from one counter, so
// that no workgroup starts a long one when the others are done.  Many small
// ones have workgroups of one wave with tables of 64 members.  Queries
// whose P(q) does not fit the LDS table run one at a time through the global
// sweep kernels.
#include <limits.h>
#include <string.h>

#include <vector>

#include "api_util.h"
#include "internal.h"
#include "sweep_dev.h"

namespace nd {

nd_status decompose_impl(nd_graph *g, nd_kind kind, const nd_opts *opts_in,
                         int32_t *kappa, int on_device, hipStream_t s,
                         nd_result *res, const uint8_t *fixed_set);

namespace {

using namespace dev;

constexpr int kEgoCap = 4096;      // members of P(q) held in LDS
constexpr int kEgoThreads = 512;   // 8 waves
// Small queries, P(q) of at most 64: a workgroup of 8 waves spends its time on
// barriers and clearing tables, so from 8192 of them on (twice the one-wave
// workgroups of a GPU) each has a wave: a million k-core queries on a path 24.8
// -> 3.4 ms, on a random graph of mean degree 8 46 -> 8.9 ms, 200,000 k-truss
// queries with lists of 10 14.8 -> 3.9 ms.
constexpr int kEgoSmall = 64;
constexpr int64_t kEgoManySmall = 8192;
constexpr int kEgoClasses = 32;

struct EgoArgs {
  const int64_t *inc_off;  // internal numbering
  const int32_t *inc_ids;
  const int32_t *ds;
  const int32_t *inv;      // original id -> internal id
  const int32_t *queries;  // original ids, already range-checked
  int64_t count;
  int32_t max_iters;
  int32_t *est;            // per query; -1 when P(q) is too large
  int32_t *sweeps;         // per query
  uint8_t *big;            // per query: 1 = run it through the fallback
  int32_t *not_converged;  // set when a query stopped at max_iters
  const int64_t *order;    // queries, heaviest first (NULL: as given)
  int64_t begin, end;      // those of this launch
  unsigned long long *head;  // how many of them have been taken
  int take;                  // so many at a time
};

// Queries dealt out by class (powers of two of d_s, largest first); all zero to
// start with where there are many.
struct EgoDeal {
  unsigned long long total[kEgoClasses];   // queries per class
  unsigned long long placed[kEgoClasses];
  unsigned long long head[2];              // see EgoArgs, per launch
};

// The tables of one workgroup: P(q) ascending, the members' values, the
// bitmap (8 bits a member), and the members to recompute.
template <int CAP>
struct EgoLds {
  static constexpr int kBits = CAP * 8;
  int32_t mem[CAP];
  int32_t tl[CAP];
  uint32_t bits[kBits / 32];
  uint8_t dirty[CAP];
};

template <int CAP>
__device__ __forceinline__ uint32_t ego_hash(int32_t x) {
  constexpr int kLog = 31 - __builtin_clz(EgoLds<CAP>::kBits);
  return ((uint32_t)x * 2654435761u) >> (32 - kLog);
}

__device__ __forceinline__ int ego_find(const int32_t *mem, int np, int32_t x) {
  int lo = 0, hi = np;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (mem[mid] < x)
      lo = mid + 1;
    else
      hi = mid;
  }
  return (lo < np && mem[lo] == x) ? lo : -1;
}

// Member number of r-clique x, -1 outside P(q).
template <int CAP>
__device__ __forceinline__ int ego_member(const EgoLds<CAP> &L, int np, int32_t x) {
  const uint32_t h = ego_hash<CAP>(x);
  if (!((L.bits[h >> 5] >> (h & 31)) & 1u)) return -1;
  return ego_find(L.mem, np, x);
}

__device__ __forceinline__ int32_t ego_load(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Current value of r-clique x: its LDS slot when x is in P(q), else d_s.
template <int CAP>
__device__ __forceinline__ int32_t ego_val(const EgoLds<CAP> &L, int np,
                                           const int32_t *ds, int32_t x) {
  const int p = ego_member(L, np, x);
  return p >= 0 ? ego_load(&L.tl[p]) : ds[x];
}

template <int K, int CAP>
__device__ __forceinline__ int32_t ego_rho(const EgoArgs &a, const EgoLds<CAP> &L,
                                           int np, int64_t j) {
  const int32_t *q = a.inc_ids + (int64_t)K * j;
  int32_t v = ego_val(L, np, a.ds, q[0]);
#pragma unroll
  for (int x = 1; x < K; x++) v = min(v, ego_val(L, np, a.ds, q[x]));
  return v;
}

// H of one member with list [b, b + d), d <= 64 M, capped at its value c.
template <int K, int M, int CAP>
__device__ __forceinline__ int32_t ego_h(const EgoArgs &a, const EgoLds<CAP> &L, int np,
                                         int64_t b, int64_t d, int32_t c) {
  int32_t rho[M];
#pragma unroll
  for (int m = 0; m < M; m++) {
    const int64_t j = lane_id() + (int64_t)m * kWave;
    rho[m] = j < d ? ego_rho<K>(a, L, np, b + j) : -1;
  }
  const int cnt = count_ge<kWave, M>(rho, c);
  return cnt >= c ? c : hindex_search<kWave, M>(rho, c, cnt);
}

__device__ __forceinline__ int wave_sum(int x) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

// Ascending bitonic sort of v[0..n), n a power of two, by the whole block.
__device__ void block_bitonic(int32_t *v, int n) {
  for (int k = 2; k <= n; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int l = i ^ j;
        if (l > i) {
          const bool up = (i & k) == 0;
          const int32_t x = v[i], y = v[l];
          if ((x > y) == up) {
            v[i] = y;
            v[l] = x;
          }
        }
      }
      __syncthreads();
    }
  }
}

// Class of query i: 0..30, fewer leading zeros for larger d_s; 31 for d_s = 0
// and for ids out of range, which k_check_queries reports.
__device__ __forceinline__ int ego_class(const EgoArgs &a, int64_t nr, int64_t i) {
  const int32_t q = a.queries[i];
  const int32_t d = q >= 0 && q < nr ? a.ds[a.inv[q]] : 0;
  return d < 1 ? kEgoClasses - 1 : __clz(d);
}

// Few queries: one workgroup counts the classes and deals the queries out.
__global__ __launch_bounds__(1024) void k_ego_order(EgoArgs a, int64_t nr,
                                                    EgoDeal *__restrict__ deal,
                                                    int64_t *__restrict__ order) {
  __shared__ int32_t at[kEgoClasses];
  const int t = threadIdx.x;
  if (t < kEgoClasses) at[t] = 0;
  if (t < 2) deal->head[t] = 0;
  __syncthreads();
  for (int64_t i = t; i < a.count; i += 1024) atomicAdd(&at[ego_class(a, nr, i)], 1);
  __syncthreads();
  if (t == 0) {
    int32_t run = 0;
    for (int c = 0; c < kEgoClasses; c++) {
      const int32_t n = at[c];
      at[c] = run;
      run += n;
    }
  }
  __syncthreads();
  for (int64_t i = t; i < a.count; i += 1024)
    order[atomicAdd(&at[ego_class(a, nr, i)], 1)] = i;
}

// Many: the classes counted, then the queries dealt out.
__global__ __launch_bounds__(1024) void k_ego_count(EgoArgs a, int64_t nr,
                                                    EgoDeal *__restrict__ deal) {
  __shared__ int32_t n[kEgoClasses];
  const int t = threadIdx.x;
  if (t < kEgoClasses) n[t] = 0;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * 1024 + t; i < a.count; i += (int64_t)gridDim.x * 1024)
    atomicAdd(&n[ego_class(a, nr, i)], 1);
  __syncthreads();
  if (t < kEgoClasses && n[t]) atomicAdd(&deal->total[t], (unsigned long long)n[t]);
}

__global__ __launch_bounds__(1024) void k_ego_deal(EgoArgs a, int64_t nr,
                                                   EgoDeal *__restrict__ deal,
                                                   int64_t *__restrict__ order) {
  __shared__ int32_t n[kEgoClasses];
  __shared__ unsigned long long at[kEgoClasses];
  const int t = threadIdx.x;
  unsigned long long start = 0;  // of class t
  for (int c = 0; c < t && t < kEgoClasses; c++) start += deal->total[c];
  for (int64_t b = (int64_t)blockIdx.x * 1024; b < a.count; b += (int64_t)gridDim.x * 1024) {
    if (t < kEgoClasses) n[t] = 0;
    __syncthreads();
    const int64_t i = b + t;
    const int c = i < a.count ? ego_class(a, nr, i) : -1;
    const int r = c >= 0 ? atomicAdd(&n[c], 1) : 0;
    __syncthreads();
    if (t < kEgoClasses && n[t])
      at[t] = start + atomicAdd(&deal->placed[t], (unsigned long long)n[t]);
    __syncthreads();
    if (c >= 0) order[at[c] + r] = i;
  }
}

// One workgroup of NT threads per query at a time, P(q) of at most CAP.
template <int K, int NT, int CAP>
__global__ __launch_bounds__(NT, NT == kWave ? 4 : 1) void k_ego(EgoArgs a) {
  constexpr int kWaves = NT / kWave;
  __shared__ EgoLds<CAP> L;
  __shared__ int32_t wsum[kWaves];
  __shared__ int s_np, s_changed;
  __shared__ unsigned long long s_next;
  int32_t *mem = L.mem, *tl = L.tl;
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  int64_t nx = 0;
  int left = 0;  // queries still held
  while (true) {  // until the counter has passed the last query
    if (left == 0) {
      if (t == 0) s_next = atomicAdd(a.head, (unsigned long long)a.take);
      __syncthreads();
      nx = a.begin + (int64_t)s_next;
      left = a.take;
      __syncthreads();
    } else {
      nx++;
    }
    left--;
    if (nx >= a.end) return;  // uniform over the block
    const int64_t qi = a.order ? a.order[nx] : nx;
    const int32_t R0 = a.inv[a.queries[qi]];
    const int64_t b0 = a.inc_off[R0];
    const int64_t d0 = a.inc_off[R0 + 1] - b0;
    const int64_t nraw = 1 + (int64_t)K * d0;
    if (nraw > CAP) {  // uniform over the block
      if (t == 0) {
        a.big[qi] = 1;
        a.est[qi] = -1;
        a.sweeps[qi] = 0;
      }
      continue;
    }
    int n2 = 1;
    while (n2 < nraw) n2 <<= 1;
    for (int i = t; i < n2; i += NT)
      mem[i] = i == 0 ? R0 : (i < nraw ? a.inc_ids[(int64_t)K * b0 + i - 1]
                                       : INT_MAX);
    for (int i = t; i < EgoLds<CAP>::kBits / 32; i += NT) L.bits[i] = 0;
    __syncthreads();
    block_bitonic(mem, n2);
    // drop repeats (none arise from a simple graph, kept for safety): keep
    // the first of each run, compacted through tl
    int keep_cnt = 0;
    const int per = (n2 + NT - 1) / NT;
    const int lo = min(n2, t * per), hi = min(n2, lo + per);
    for (int i = lo; i < hi; i++)
      keep_cnt += mem[i] != INT_MAX && (i == 0 || mem[i] != mem[i - 1]);
    // block exclusive scan of keep_cnt
    int incl = keep_cnt;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int y = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int base = 0;
    for (int q = 0; q < w; q++) base += wsum[q];
    int pos = base + incl - keep_cnt;
    for (int i = lo; i < hi; i++)
      if (mem[i] != INT_MAX && (i == 0 || mem[i] != mem[i - 1])) tl[pos++] = mem[i];
    if (t == NT - 1) s_np = base + incl;
    __syncthreads();
    const int np = s_np;
    for (int i = t; i < np; i += NT) mem[i] = tl[i];
    __syncthreads();
    for (int i = t; i < np; i += NT) {
      const int32_t x = mem[i];
      const uint32_t h = ego_hash<CAP>(x);
      atomicOr(&L.bits[h >> 5], 1u << (h & 31));
      tl[i] = a.ds[x];
      L.dirty[i] = 1;
    }
    __syncthreads();

    int sweeps = 0;
    bool changed_last = true;
    while (sweeps < a.max_iters) {
      if (t == 0) s_changed = 0;
      __syncthreads();
      for (int i = w; i < np; i += kWaves) {
        // The mark is cleared before the values are read: a neighbour that
        // falls after that marks this member again (it stores its value
        // first, and one CU's LDS serves accesses in order).
        if (__hip_atomic_load(&L.dirty[i], __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_WORKGROUP) == 0)
          continue;  // uniform over the wave
        if (lane == 0)
          __hip_atomic_store(&L.dirty[i], (uint8_t)0, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        const int32_t R = mem[i];
        const int64_t b = a.inc_off[R];
        const int64_t d = a.inc_off[R + 1] - b;
        const int32_t c = ego_load(&tl[i]);
        int32_t h;
        if (d <= (int64_t)kWave * 4) {
          h = ego_h<K, 4>(a, L, np, b, d, c);
        } else if (d <= (int64_t)kWave * 8) {
          h = ego_h<K, 8>(a, L, np, b, d, c);
        } else if (d <= (int64_t)kWave * 16) {
          h = ego_h<K, 16>(a, L, np, b, d, c);
        } else if (d <= (int64_t)kWave * 32) {
          h = ego_h<K, 32>(a, L, np, b, d, c);
        } else {
          // long list: count #{rho >= x} by a fresh pass per probe
          auto count = [&](int32_t x) {
            int n = 0;
            for (int64_t j = lane; j < d; j += kWave)
              n += ego_rho<K>(a, L, np, b + j) >= x;
            return wave_sum(n);
          };
          const int cnt = count(c);
          h = cnt >= c ? c : hindex_between(count, c, cnt);
        }
        if (h != c) {  // uniform over the wave
          if (lane == 0) {
            __hip_atomic_store(&tl[i], h, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
            s_changed = 1;
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
          // members above h may have lost this s-clique (one at or below h
          // has not)
          for (int64_t j = (int64_t)K * b + lane; j < (int64_t)K * (b + d); j += kWave) {
            const int p = ego_member(L, np, a.inc_ids[j]);
            if (p >= 0 && ego_load(&tl[p]) > h)
              __hip_atomic_store(&L.dirty[p], (uint8_t)1, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
      __syncthreads();
      sweeps++;
      changed_last = s_changed != 0;
      __syncthreads();
      if (!changed_last) break;
    }
    if (t == 0) {
      a.est[qi] = tl[ego_find(mem, np, R0)];
      a.sweeps[qi] = sweeps;
      if (changed_last) *a.not_converged = 1;
    }
    __syncthreads();
  }
}

__global__ void k_check_queries(const int32_t *__restrict__ q, int64_t count,
                                int64_t nr, int32_t *__restrict__ err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count && (q[i] < 0 || q[i] >= nr)) *err = 1;
}

// mark[R0] = 1 and mark[x] = 1 for every id x in R0's incidence list.
__global__ void k_mark_ego(const int64_t *__restrict__ inc_off,
                           const int32_t *__restrict__ inc_ids, int k,
                           int32_t R0, uint8_t *__restrict__ mark) {
  const int64_t b = inc_off[R0] * k, e = inc_off[R0 + 1] * k;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) mark[R0] = 1;
  if (b + i < e) mark[inc_ids[b + i]] = 1;
}

}  // namespace

nd_status ego_estimate(nd_graph *g, nd_kind kind, const int32_t *queries,
                       int64_t count, int32_t max_iters, int32_t *est,
                       int32_t *sweeps, int on_device, hipStream_t s) {
  ND_REQUIRE(count >= 0 && (count == 0 || (queries && est)), ND_ERR_INVALID,
             "bad query list");
  prepare(g, kind, s);
  const KindState &ks = g->ks[kind];
  Allocator &al = g->ctx->alloc;
  if (count == 0) return ND_OK;
  if (max_iters < 0) max_iters = INT_MAX;
  DArr<int32_t> dq(al, count), dest(al, count), dsw(al, count), flags(al, 2);
  DArr<uint8_t> big(al, count);
  ND_HIP(hipMemcpyAsync(dq.p, queries, sizeof(int32_t) * count,
                        on_device ? hipMemcpyDeviceToDevice
                                  : hipMemcpyHostToDevice, s));
  fill_i32(flags.p, 0, 2, s);
  fill_u8(big.p, 0, count, s);
  k_check_queries<<<grid_for(count, 256), 256, 0, s>>>(dq.p, count, ks.nr,
                                                        flags.p);
  ND_LAUNCHED();
  EgoArgs a{};
  a.inc_off = ks.inc_off.p;
  a.inc_ids = ks.inc_ids.p;
  a.ds = ks.ds.p;
  a.inv = ks.inv.p;
  a.queries = dq.p;
  a.count = count;
  a.max_iters = max_iters;
  a.est = dest.p;
  a.sweeps = dsw.p;
  a.big = big.p;
  a.not_converged = flags.p + 1;
  DArr<EgoDeal> deal(al, 1);
  DArr<int64_t> order;
  try {
    order.reset(al, count);
  } catch (const Err &e) {  // short of memory: in the order given
    if (e.code != ND_ERR_OOM) throw;
    clear_error();
  }
  a.order = order.p;
  const bool many = count >= kEgoManySmall && order.p != nullptr;
  if (order.p == nullptr) {
    fill_u64((uint64_t *)deal.p, 0, sizeof(EgoDeal) / 8, s);
  } else if (many) {
    fill_u64((uint64_t *)deal.p, 0, sizeof(EgoDeal) / 8, s);
    const unsigned grid = (unsigned)std::min<int64_t>(grid_for(count, 1024), g->ctx->num_cu);
    k_ego_count<<<grid, 1024, 0, s>>>(a, ks.nr, deal.p);
    ND_LAUNCHED();
    k_ego_deal<<<grid, 1024, 0, s>>>(a, ks.nr, deal.p, order.p);
    ND_LAUNCHED();
  } else {
    k_ego_order<<<1, 1024, 0, s>>>(a, ks.nr, deal.p, order.p);
    ND_LAUNCHED();
  }
  int32_t herr[2] = {0, 0};
  int64_t big_end = count;  // queries in the classes that may exceed kEgoSmall
  {
    PinnedChunk pc;
    const unsigned long long *total =
        many ? pc.post(deal.p->total, kEgoClasses, s) : nullptr;
    const int32_t *hf = pc.read(flags.p, 1, s);
    ND_REQUIRE(*hf == 0, ND_ERR_INVALID, "a query id is outside [0, %lld)",
               (long long)ks.nr);
    int64_t n = 0;
    for (int c = 0; many && c < kEgoClasses - 1; c++)  // d_s up to 2^(32 - c) - 1
      if ((((int64_t)1 << (32 - c)) - 1) * ks.k + 1 > kEgoSmall) n += (int64_t)total[c];
    if (count - n >= kEgoManySmall) big_end = n;
  }
  // As many workgroups as stay resident: one of eight waves per CU, 16 of one wave
  // (136 and 128 registers); the counters deal out the rest.
  auto launch = [&](auto big_kernel, auto small_kernel) {
    if (big_end > 0) {
      a.begin = 0;
      a.end = big_end;
      a.head = &deal.p->head[0];
      a.take = 1;
      const int64_t grid = std::min<int64_t>(big_end, (int64_t)g->ctx->num_cu);
      big_kernel<<<(unsigned)grid, kEgoThreads, 0, s>>>(a);
      ND_LAUNCHED();
    }
    if (big_end < count) {
      a.begin = big_end;
      a.end = count;
      a.head = &deal.p->head[1];
      const int64_t n = count - big_end;
      const int64_t grid = std::min<int64_t>(n, (int64_t)g->ctx->num_cu * 16);
      // the counter gives out a query every few nanoseconds
      a.take = (int)std::min<int64_t>(16, std::max<int64_t>(1, n / (4 * grid)));
      small_kernel<<<(unsigned)grid, kWave, 0, s>>>(a);
      ND_LAUNCHED();
    }
  };
  switch (ks.k) {
    case 1: launch(k_ego<1, kEgoThreads, kEgoCap>, k_ego<1, kWave, kEgoSmall>); break;
    case 2: launch(k_ego<2, kEgoThreads, kEgoCap>, k_ego<2, kWave, kEgoSmall>); break;
    case 3: launch(k_ego<3, kEgoThreads, kEgoCap>, k_ego<3, kWave, kEgoSmall>); break;
    case 5: launch(k_ego<5, kEgoThreads, kEgoCap>, k_ego<5, kWave, kEgoSmall>); break;
    default: ND_REQUIRE(false, ND_ERR_UNSUPPORTED, "no ego kernel for k=%d", ks.k);
  }
  std::vector<int32_t> hq(count), he(count), hs(count);
  std::vector<uint8_t> hb(count);
  ND_HIP(hipMemcpyAsync(hq.data(), dq.p, sizeof(int32_t) * count,
                        hipMemcpyDeviceToHost, s));
  ND_HIP(hipMemcpyAsync(he.data(), dest.p, sizeof(int32_t) * count,
                        hipMemcpyDeviceToHost, s));
  ND_HIP(hipMemcpyAsync(hs.data(), dsw.p, sizeof(int32_t) * count,
                        hipMemcpyDeviceToHost, s));
  ND_HIP(hipMemcpyAsync(hb.data(), big.p, count, hipMemcpyDeviceToHost, s));
  ND_HIP(hipMemcpyAsync(herr, flags.p, sizeof herr, hipMemcpyDeviceToHost, s));
  ND_HIP(hipStreamSynchronize(s));
  bool not_conv = herr[1] != 0;
  // queries whose ego network does not fit one workgroup's table
  std::vector<int32_t> inv_h;
  for (int64_t i = 0; i < count; i++) {
    if (!hb[i]) continue;
    if (inv_h.empty()) {
      inv_h.resize(ks.nr);
      ND_HIP(hipMemcpyAsync(inv_h.data(), ks.inv.p, sizeof(int32_t) * ks.nr,
                            hipMemcpyDeviceToHost, s));
      ND_HIP(hipStreamSynchronize(s));
    }
    const int32_t R0 = inv_h[hq[i]];
    DArr<uint8_t> mark(al, ks.nr);
    fill_u8(mark.p, 0, ks.nr, s);
    int64_t hoff[2];
    ND_HIP(hipMemcpyAsync(hoff, ks.inc_off.p + R0, sizeof hoff,
                          hipMemcpyDeviceToHost, s));
    ND_HIP(hipStreamSynchronize(s));
    const int64_t len = (hoff[1] - hoff[0]) * ks.k;
    k_mark_ego<<<grid_for(std::max<int64_t>(len, 1), 256), 256, 0, s>>>(
        ks.inc_off.p, ks.inc_ids.p, ks.k, R0, mark.p);
    ND_LAUNCHED();
    DArr<int32_t> full(al, ks.nr);
    nd_opts o;
    nd_opts_init(&o);
    o.max_iters = max_iters;
    nd_result r{};
    const nd_status st = decompose_impl(g, kind, &o, full.p, 1, s, &r, mark.p);
    if (st == ND_ERR_NOT_CONVERGED)
      not_conv = true;
    else if (st != ND_OK)
      return st;
    ND_HIP(hipMemcpyAsync(&he[i], full.p + hq[i], sizeof(int32_t),
                          hipMemcpyDeviceToHost, s));
    ND_HIP(hipStreamSynchronize(s));
    hs[i] = r.sweeps;
  }
  if (on_device) {
    ND_HIP(hipMemcpyAsync(est, he.data(), sizeof(int32_t) * count,
                          hipMemcpyHostToDevice, s));
    if (sweeps)
      ND_HIP(hipMemcpyAsync(sweeps, hs.data(), sizeof(int32_t) * count,
                            hipMemcpyHostToDevice, s));
  } else {
    memcpy(est, he.data(), sizeof(int32_t) * count);
    if (sweeps) memcpy(sweeps, hs.data(), sizeof(int32_t) * count);
  }
  ND_HIP(hipStreamSynchronize(s));
  if (not_conv) {
    set_error("a query stopped at max_iters without converging");
    return ND_ERR_NOT_CONVERGED;
  }
  return ND_OK;
}

}  // namespace nd

using namespace nd;

extern "C" nd_status nd_ego_estimate(nd_graph *g, nd_kind kind,
                                     const int32_t *queries, int64_t count,
                                     int32_t max_iters, int32_t *est,
                                     int32_t *sweeps, int on_device,
                                     void *stream) {
  nd_status out = ND_OK;
  nd_status st = guarded([&] {
    ND_REQUIRE(g, ND_ERR_INVALID, "graph is NULL");
    ND_HIP(hipSetDevice(g->ctx->device));
    StreamScope scope((hipStream_t)stream);
    out = ego_estimate(g, kind, queries, count, max_iters, est, sweeps,
                       on_device, (hipStream_t)stream);
  });
  return st != ND_OK ? st : out;
}
