// layout.hip -- the internal numbering of r-cliques.
//
// Sweeps run over r-cliques grouped by sweep bin (the lanes per r-clique
// chosen from d_s: d_s >= 2048 first, d_s = 0 last), each group in ascending
// id order (edges: by their endpoint of lower degree, then by the other).  Both
// choices serve the memory hierarchy, not the method:
//   * each bin becomes a contiguous id range, so no per-bin index lists are
//     read and the incidence lists are one sequential stream;
//   * within a bin, ids keep the lexicographic order of the r-cliques, so
//     r-cliques swept by neighbouring lanes share vertices, and the tau
//     values they gather (r-cliques of their common s-cliques, which share
//     those vertices too) sit in nearby cache lines.  Measured on a power-law
//     k-truss workload this beats ordering by exact d_s (which packs the most
//     gathered values together but scatters each lane group's neighbours) by
//     about 30% per sweep;
//     An edge listed with its endpoint of lower degree has its triangles'
//     other edges in two short runs; listed with the lower id, a hub's edges lie
//     in as many runs as it has neighbours (power-law k-truss of 16.5M edges: a
//     full sweep 2.42 -> 2.24 ms in 16 bits, eight 18.3 -> 17.1 ms).  Ordering
//     k-core vertices by sixteenths of their bins' degrees gained 4% on 8.4M
//     vertices and lost 11-19% on graphs of 0.4-0.7M in place: not done.
//   * r-cliques with d_s = 0 (never swept) go to the end.
// Results are un-permuted on the way out; nothing observable depends on the
// internal order (SND iterates are order-independent by definition).
#include <algorithm>

#include "internal.h"
#include "partition.h"

namespace nd {

namespace {

// Every value goes through the numbering on its way in and out, also those never
// swept, and an order other than by id scatters them (8 million edges, 16
// triangles: values out 17.8 us by id, 35.7 by the order above, of a
// decomposition of 110 us).  So from 2^20 r-cliques on the swept ones are counted
// first and an order is used only if they are a quarter or more; below, the
// values sit in the L2 either way.
constexpr int64_t kCountSwept = 1 << 20;

// Without branches: the lower bounds of the bins that d reaches.
__device__ __forceinline__ int bin_of(int32_t d) {
  static_assert(kBinZero == 8 && kBinG1 == 7 && kBinBlock == 0, "bins in order");
  return kBinZero - ((d >= 1) + (d >= 5) + (d >= 17) + (d >= 65) + (d >= 257) +
                     (d >= 513) + (d >= 1025) + (d >= 2048));
}

// r-cliques grouped by sweep bin in id order (partition.h): an internal id's
// r-clique, its inverse and its S-degree are written as it is placed.
struct Order {
  const int32_t *order;             // NULL: id order
  const unsigned long long *swept;  // not NULL: so many have d_s > 0 ...
  unsigned long long least;         // ... and `order` is for as many as this
  __device__ Order local() const {
    return Order{swept == nullptr || *swept >= least ? order : nullptr, nullptr, 0};
  }
  __device__ int32_t at(int64_t i) const { return order ? order[i] : (int32_t)i; }
};
struct DegreeIn {
  const int32_t *cnt;
  Order order;
  __device__ DegreeIn local() const { return DegreeIn{cnt, order.local()}; }
  __device__ int load(int64_t i, int32_t *most) const {
    const int32_t d = cnt[order.at(i)];
    *most = max(*most, d);
    return bin_of(d);
  }
};
struct LayoutOut {
  const int32_t *cnt;
  Order order;
  int32_t *perm, *inv, *ds;
  __device__ LayoutOut local() const { return LayoutOut{cnt, order.local(), perm, inv, ds}; }
  __device__ void put(int64_t i, int64_t place) const {
    const int32_t r = order.at(i);
    perm[place] = r;
    inv[r] = (int32_t)place;
    ds[place] = cnt[r];
  }
};

__global__ __launch_bounds__(256) void k_count_swept(
    const int32_t *__restrict__ cnt, int64_t n, unsigned long long *__restrict__ out) {
  __shared__ int32_t ws[4];
  int32_t c = 0;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int4 *v = reinterpret_cast<const int4 *>(cnt);  // 256-byte aligned
  for (int64_t i = t; i < n / 4; i += (int64_t)gridDim.x * 256) {
    const int4 x = v[i];
    c += (x.x > 0) + (x.y > 0) + (x.z > 0) + (x.w > 0);
  }
  if (t < n % 4) c += cnt[n / 4 * 4 + t] > 0;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
  if (lane_id() == 0) ws[threadIdx.x / kWave] = c;
  __syncthreads();
  c = ws[0] + ws[1] + ws[2] + ws[3];
  if (threadIdx.x == 0 && c) atomicAdd(out, (unsigned long long)c);
}

template <typename T>
__global__ void k_to_internal(const int32_t *__restrict__ in,
                              const int32_t *__restrict__ perm, int64_t nr,
                              T *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nr) out[i] = (T)in[perm[i]];
}

template <typename T>
__global__ void k_to_original(const T *__restrict__ in,
                              const int32_t *__restrict__ inv, int64_t nr,
                              int32_t *__restrict__ out) {
  const int64_t R = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (R < nr) out[R] = (int32_t)in[inv[R]];
}

// List of r-clique R (original numbering) with original ids, G lanes each.
template <int G>
__global__ __launch_bounds__(256) void k_incidence_original(
    const int64_t *__restrict__ in_off, const int32_t *__restrict__ in_ids,
    const int32_t *__restrict__ inv, const int32_t *__restrict__ perm, int k,
    int64_t nr, const int64_t *__restrict__ out_off,
    int32_t *__restrict__ out_ids) {
  const int sl = lane_id() % G;
  const int64_t nsub = (int64_t)gridDim.x * blockDim.x / G;
  for (int64_t R = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
       R < nr; R += nsub) {
    const int32_t i = inv[R];
    const int64_t b = in_off[i] * k, e = in_off[i + 1] * k, o = out_off[R] * k;
    for (int64_t j = b + sl; j < e; j += G) out_ids[o + (j - b)] = perm[in_ids[j]];
  }
}

template <typename T>
__global__ void k_init_tau(const int32_t *__restrict__ ds, int64_t nr,
                           T *__restrict__ tau) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nr) tau[i] = (T)ds[i];
}

}  // namespace

void init_tau(const KindState &ks, void *tau, int bytes, hipStream_t s) {
  if (ks.nr == 0) return;
  const unsigned grid = grid_for(ks.nr, 256);
  if (bytes == 1)
    k_init_tau<uint8_t><<<grid, 256, 0, s>>>(ks.ds.p, ks.nr, (uint8_t *)tau);
  else if (bytes == 2)
    k_init_tau<uint16_t><<<grid, 256, 0, s>>>(ks.ds.p, ks.nr, (uint16_t *)tau);
  else
    k_init_tau<int32_t><<<grid, 256, 0, s>>>(ks.ds.p, ks.nr, (int32_t *)tau);
  ND_LAUNCHED();
}

void build_layout(nd_graph *g, KindState &ks, const int32_t *cnt,
                  hipStream_t s, const int32_t *order) {
  Phase phase("nd.layout");
  Allocator &al = g->ctx->alloc;
  const int64_t nr = ks.nr;
  ND_REQUIRE(nr < ((int64_t)1 << 31), ND_ERR_INVALID,
             "%lld r-cliques: ids must fit int32", (long long)nr);
  ks.perm.reset(al, nr);
  ks.inv.reset(al, nr);
  ks.ds.reset(al, nr);
  ks.inc_off.reset(al, nr + 1);
  DArr<part::Head> head(al, 1);
  DArr<unsigned long long> swept;
  Order by{order, nullptr, 0};
  if (order != nullptr && nr >= kCountSwept) {
    swept.reset(al, 1);
    fill_u64((uint64_t *)swept.p, 0, 1, s);
    k_count_swept<<<(unsigned)std::min<int64_t>(grid_for(nr, 2048), 2048), 256, 0, s>>>(
        cnt, nr, swept.p);
    ND_LAUNCHED();
    by = Order{order, swept.p, (unsigned long long)nr / 4};
  }
  if (nr > 0)
    part::run<kNumBins>(DegreeIn{cnt, by},
                        LayoutOut{cnt, by, ks.perm.p, ks.inv.p, ks.ds.p}, nr,
                        head.p, s, al);
  exclusive_scan_i32(ks.ds.p, ks.inc_off.p, nr, s, al);
  // one wait for the bins, the largest S-degree and the total
  PinnedChunk pc;
  const part::Head *h = nr > 0 ? pc.post(head.p, 1, s) : nullptr;
  const int64_t *total = pc.read(ks.inc_off.p + nr, 1, s);
  const int32_t hmax = nr > 0 ? h->most : 0;
  ks.max_ds = hmax;
  ks.tau16 = hmax < 32768;
  ks.tau_bytes = hmax < 256 ? 1 : ks.tau16 ? 2 : 4;
  for (int b = 0; b < kNumBins; b++) {
    ks.bin_lo[b] = nr > 0 ? h->start[b] : 0;
    ks.bin_hi[b] = nr > 0 ? h->start[b + 1] : 0;
  }
  ks.P = *total;
}

void to_internal(const KindState &ks, const int32_t *in, void *out, int bytes,
                 hipStream_t s) {
  if (ks.nr == 0) return;
  const unsigned grid = grid_for(ks.nr, 256);
  if (bytes == 1)
    k_to_internal<uint8_t><<<grid, 256, 0, s>>>(in, ks.perm.p, ks.nr, (uint8_t *)out);
  else if (bytes == 2)
    k_to_internal<uint16_t><<<grid, 256, 0, s>>>(in, ks.perm.p, ks.nr, (uint16_t *)out);
  else
    k_to_internal<int32_t><<<grid, 256, 0, s>>>(in, ks.perm.p, ks.nr, (int32_t *)out);
  ND_LAUNCHED();
}

void to_original(const KindState &ks, const void *in, int bytes, int32_t *out,
                 hipStream_t s) {
  if (ks.nr == 0) return;
  const unsigned grid = grid_for(ks.nr, 256);
  if (bytes == 1)
    k_to_original<uint8_t><<<grid, 256, 0, s>>>((const uint8_t *)in, ks.inv.p, ks.nr, out);
  else if (bytes == 2)
    k_to_original<uint16_t><<<grid, 256, 0, s>>>((const uint16_t *)in, ks.inv.p, ks.nr, out);
  else
    k_to_original<int32_t><<<grid, 256, 0, s>>>((const int32_t *)in, ks.inv.p, ks.nr, out);
  ND_LAUNCHED();
}

void sdegree_original(const KindState &ks, int32_t *ds, hipStream_t s) {
  to_original(ks, ks.ds.p, 4, ds, s);
}

void incidence_original(nd_graph *g, const KindState &ks, int64_t *off,
                        int32_t *ids, hipStream_t s) {
  Allocator &al = g->ctx->alloc;
  DArr<int32_t> dso(al, ks.nr);
  sdegree_original(ks, dso.p, s);
  exclusive_scan_i32(dso.p, off, ks.nr, s, al);
  if (ks.nr == 0 || ks.P == 0) return;
  k_incidence_original<16><<<grid_stride(ks.nr, 16), 256, 0, s>>>(
      ks.inc_off.p, ks.inc_ids.p, ks.inv.p, ks.perm.p, ks.k, ks.nr, off, ids);
  ND_LAUNCHED();
}

}  // namespace nd
