// prim.hip -- device primitives used by graph preparation: exclusive scan,
// stable LSD radix sort of 64-bit keys, stable partition by a small key, and
// fills.  All integer, all deterministic.
#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.h"
#include "partition.h"

namespace nd {

namespace {

// Exclusive scan.  A wave owns 1024 consecutive values as kScanVec rows of
// 256: every lane loads four consecutive values of each row (16 bytes, so a
// row is one coalesced load), rows are scanned with wave shuffles and carried
// from row to row, and one exchange of the wave totals through LDS places the
// waves.  Bound by its streams: 4 bytes read and 8 written per value, the
// reads twice above one workgroup's size; short ones by the launch.  (One
// workgroup of 4 waves looping over up to 131072 values took 31 us on average
// in a batch of 128 small graphs, most of the time their preparation had the
// GPU: with this split the batch takes 53.2 ms instead of 65.8.)
constexpr int kScanThreads = 256;
constexpr int kScanVec = 4;                               // rows per wave
constexpr int kScanTile = kScanThreads * 4 * kScanVec;    // 4096
constexpr int kScanBig = 1024;                            // one-workgroup scan
constexpr int64_t kScanOneTile = kScanBig * 4 * kScanVec; // 16384

// Inclusive scan of one value per lane across the wave.
__device__ __forceinline__ int64_t wave_inclusive_scan(int64_t x) {
  const int lane = lane_id();
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    int64_t y = __shfl_up(x, off, kWave);
    if (lane >= off) x += y;
  }
  return x;
}

__device__ __forceinline__ int64_t wave_total(int64_t x) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

// Sum over the block of one value per wave (the same on all its lanes), and
// of the waves before this one.  ws: one slot per wave.
template <int NT>
__device__ __forceinline__ int64_t block_exclusive(int64_t wave_sum,
                                                   int64_t *ws, int64_t *all) {
  const int wid = threadIdx.x / kWave;
  __syncthreads();  // ws may still be read from the call before
  if (lane_id() == 0) ws[wid] = wave_sum;
  __syncthreads();
  int64_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / kWave; w++) {
    const int64_t x = ws[w];
    before += w < wid ? x : 0;
    tot += x;
  }
  *all = tot;
  return before;
}

// Four consecutive values from i (0 past n); one 16-byte load where they are
// all inside and T is 4 bytes (in is 16-byte aligned at multiples of 4).
template <typename T>
__device__ __forceinline__ void load4(const T *__restrict__ in, int64_t i,
                                      int64_t n, int64_t *v) {
  if (sizeof(T) == 4 && i + 4 <= n) {
    const int4 q = *reinterpret_cast<const int4 *>(in + i);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else {
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = i + k < n ? (int64_t)in[i + k] : 0;
  }
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(
    const T *__restrict__ in, int64_t n, int64_t *__restrict__ partial) {
  __shared__ int64_t ws[kScanThreads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
  int64_t sum = 0;
#pragma unroll
  for (int r = 0; r < kScanVec; r++) {
    int64_t v[4];
    load4(in, base + (int64_t)r * kScanThreads * 4, n, v);
    sum += v[0] + v[1] + v[2] + v[3];
  }
  int64_t all;
  block_exclusive<kScanThreads>(wave_total(sum), ws, &all);
  if (threadIdx.x == 0) partial[blockIdx.x] = all;
}

// Scans the tile of NT * 4 * kScanVec values at `base0`, everything before it
// summing to `off`; returns off + the tile's total.  wide: out is 16-byte
// aligned.
template <int NT, typename T>
__device__ __forceinline__ int64_t scan_tile(const T *__restrict__ in, int64_t n,
                                             int64_t base0, int64_t off,
                                             int64_t *__restrict__ out,
                                             bool wide, int64_t *ws) {
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  const int64_t wbase = base0 + (int64_t)wid * kWave * 4 * kScanVec;
  int64_t v[kScanVec][4], ex[kScanVec];
  int64_t carry = 0;
#pragma unroll
  for (int r = 0; r < kScanVec; r++)
    load4(in, wbase + ((int64_t)r * kWave + lane) * 4, n, v[r]);
#pragma unroll
  for (int r = 0; r < kScanVec; r++) {
    const int64_t s4 = v[r][0] + v[r][1] + v[r][2] + v[r][3];
    const int64_t inc = wave_inclusive_scan(s4);
    ex[r] = carry + inc - s4;
    carry += __shfl(inc, kWave - 1, kWave);
  }
  int64_t all;
  const int64_t before = off + block_exclusive<NT>(carry, ws, &all);
#pragma unroll
  for (int r = 0; r < kScanVec; r++) {
    const int64_t i = wbase + ((int64_t)r * kWave + lane) * 4;
    int64_t o[4];
    o[0] = before + ex[r];
    o[1] = o[0] + v[r][0];
    o[2] = o[1] + v[r][1];
    o[3] = o[2] + v[r][2];
    if (wide && i + 4 <= n) {
      longlong2 *q = reinterpret_cast<longlong2 *>(out + i);
      q[0] = make_longlong2(o[0], o[1]);
      q[1] = make_longlong2(o[2], o[3]);
    } else {
#pragma unroll
      for (int k = 0; k < 4; k++)
        if (i + k < n) out[i + k] = o[k];
    }
  }
  return off + all;
}

__device__ __forceinline__ bool aligned16(const void *p) {
  return ((uintptr_t)p & 15) == 0;
}

// The tiles' second pass: a workgroup's offset is scanned[b] when the tile
// sums were scanned beforehand (`scanned`), else the sum of the tile sums
// before it, which it adds up itself (at most kScanSelfSum of them).  The
// last block also writes out[n] (the grand total).
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_tile(
    const T *__restrict__ in, int64_t n, const int64_t *__restrict__ partial,
    const int64_t *__restrict__ scanned, int64_t *__restrict__ out) {
  __shared__ int64_t ws[kScanThreads / kWave];
  int64_t off = 0;
  if (scanned != nullptr) {
    off = scanned[blockIdx.x];
  } else {
    int64_t sum = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kScanThreads)
      sum += partial[b];
    block_exclusive<kScanThreads>(wave_total(sum), ws, &off);
  }
  const int64_t end = scan_tile<kScanThreads>(
      in, n, (int64_t)blockIdx.x * kScanTile, off, out, aligned16(out), ws);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = end;
}

// Short inputs: one workgroup of 16 waves scans up to kScanOneMax values,
// carrying the running total from tile to tile, in one launch.
template <typename T>
__global__ __launch_bounds__(kScanBig) void k_scan_one(
    const T *__restrict__ in, int64_t n, int64_t *__restrict__ out) {
  __shared__ int64_t ws[kScanBig / kWave];
  const bool wide = aligned16(out);
  int64_t off = 0;
  for (int64_t base = 0; base < n; base += kScanOneTile)
    off = scan_tile<kScanBig>(in, n, base, off, out, wide, ws);
  if (threadIdx.x == 0) out[n] = off;
}

// Up to two tiles of the one-workgroup scan: there one launch is quicker than
// two; above, the tiles run on many CUs.  Up to kScanSelfSum tiles every
// workgroup adds up the tile sums before it (2048 words, one round of eight
// loads a thread), which saves the launch that would scan them.
constexpr int64_t kScanOneMax = 2 * kScanOneTile;
constexpr int64_t kScanSelfSum = 2048;

template <typename T>
void exclusive_scan_impl(const T *in, int64_t *out, int64_t n, hipStream_t s,
                         Allocator &al) {
  n = std::max<int64_t>(n, 0);
  if (n <= kScanOneMax) {  // n == 0 too: writes out[0] = 0
    k_scan_one<T><<<1, kScanBig, 0, s>>>(in, n, out);
    ND_LAUNCHED();
    return;
  }
  const int64_t nb = ceil_div(n, kScanTile);
  DArr<int64_t> partial(al, nb), pscan;
  k_scan_reduce<T><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, partial.p);
  ND_LAUNCHED();
  if (nb > kScanSelfSum) {
    pscan.reset(al, nb + 1);
    exclusive_scan_impl<int64_t>(partial.p, pscan.p, nb, s, al);
  }
  k_scan_tile<T><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, partial.p, pscan.p, out);
  ND_LAUNCHED();
}

// ------------------------------------------------------------ radix sort

constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;  // 4096 keys per block
constexpr int kSortWaves = kSortThreads / kWave;

__global__ __launch_bounds__(kSortThreads) void k_radix_hist(
    const uint64_t *__restrict__ keys, int64_t n, int shift,
    int32_t *__restrict__ hist, int64_t nb) {
  __shared__ int32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
#pragma unroll 4
  for (int it = 0; it < kSortItems; it++) {
    int64_t i = base + it * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of one tile by one digit.  A wave ranks its own 1024
// consecutive keys, 64 at a time: equal digits within the 64 are matched with
// 8 ballots, a per-wave counter in LDS carries each digit's count on (one
// wave's LDS accesses are served in order, so no barrier is needed).  Then
// the tile's digit starts are scanned, the keys go to LDS in digit order, and
// leave it in runs of consecutive addresses: bound by its 16 bytes a key.
// (Storing each key straight to its place took three barriers per 256 keys
// and wrote 8-byte pieces: 2.35 ms for 268 million keys, 1.8 TB/s; now 1.21
// ms, 3.6 TB/s.)  Up to kSortSelf tiles there are no scanned offsets: every
// workgroup adds up the histogram itself (thread d the row of digit d), which
// is quicker than the launch that would scan it.
constexpr int64_t kSortSelf = 64;

__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const uint64_t *__restrict__ in, uint64_t *__restrict__ out, int64_t n,
    int shift, const int32_t *__restrict__ hist,
    const int64_t *__restrict__ offs, int64_t nb) {
  __shared__ uint64_t keys[kSortTile];
  __shared__ int32_t cnt[kSortWaves][256];
  __shared__ int32_t start[256];  // first place of each digit in the tile
  __shared__ int64_t to[256];     // its global place, less that
  __shared__ int32_t ws[kSortWaves];
  const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  const int total = (int)std::min<int64_t>(kSortTile, n - base);
  int64_t goff;
  if (offs != nullptr) {
    goff = offs[(int64_t)tid * nb + blockIdx.x];
  } else {
    int32_t all = 0, before = 0;  // of digit tid
    const int32_t *row = hist + (int64_t)tid * nb;
    for (int b = 0; b < (int)nb; b++) {
      const int32_t c = row[b];
      before += b < (int)blockIdx.x ? c : 0;
      all += c;
    }
    int32_t inc = all;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int32_t y = __shfl_up(inc, off, kWave);
      if (lane >= off) inc += y;
    }
    if (lane == kWave - 1) ws[w] = inc;
    __syncthreads();
    int32_t lower = inc - all;
#pragma unroll
    for (int x = 0; x < kSortWaves; x++) lower += x < w ? ws[x] : 0;
    goff = lower + before;
    __syncthreads();  // ws is used again
  }
#pragma unroll
  for (int x = 0; x < 256 / kWave; x++) cnt[w][x * kWave + lane] = 0;
  uint64_t key[kSortItems];
  int32_t rank[kSortItems];
  const int wbase = w * kWave * kSortItems;
#pragma unroll
  for (int it = 0; it < kSortItems; it++) {
    const int i = wbase + it * kWave + lane;
    key[it] = i < total ? in[base + i] : 0;
  }
#pragma unroll
  for (int it = 0; it < kSortItems; it++) {
    const bool valid = wbase + it * kWave + lane < total;
    const int d = (int)((key[it] >> shift) & 255);
    uint64_t peers = ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; b++) {
      const bool bit = (d >> b) & 1;
      const uint64_t m = ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int below = lanes_below(peers);
    __builtin_amdgcn_wave_barrier();
    const int before = valid ? cnt[w][d] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) cnt[w][d] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    rank[it] = before + below;
  }
  __syncthreads();
  // digit tid: its count, the waves' starts within it, its start in the tile
  int32_t run = 0;
#pragma unroll
  for (int x = 0; x < kSortWaves; x++) {
    const int32_t c = cnt[x][tid];
    cnt[x][tid] = run;
    run += c;
  }
  int32_t inc = run;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t y = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += y;
  }
  if (lane == kWave - 1) ws[w] = inc;
  __syncthreads();
  int32_t st = inc - run;
#pragma unroll
  for (int x = 0; x < kSortWaves; x++) st += x < w ? ws[x] : 0;
  start[tid] = st;
  to[tid] = goff - st;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kSortItems; it++) {
    if (wbase + it * kWave + lane < total) {
      const int d = (int)((key[it] >> shift) & 255);
      keys[start[d] + cnt[w][d] + rank[it]] = key[it];
    }
  }
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < total; i += kSortThreads) {
    const uint64_t k = keys[i];
    out[to[(k >> shift) & 255] + i] = k;
  }
}

// ------------------------------------------------------------- misc

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_u8(uint8_t *p, uint8_t v, int64_t n) {
  // four bytes per thread where aligned
  int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (i + 3 < n && ((uintptr_t)(p + i) & 3) == 0) {
    const uint32_t w = 0x01010101u * v;
    *reinterpret_cast<uint32_t *>(p + i) = w;
  } else {
    for (int64_t j = i; j < i + 4 && j < n; j++) p[j] = v;
  }
}

__global__ void k_fill_u64(uint64_t *p, uint64_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Items grouped by a byte each.
struct ByteIn {
  const uint8_t *bin;
  __device__ ByteIn local() const { return *this; }
  __device__ int load(int64_t i, int32_t *) const { return bin[i]; }
};
struct ItemOut {
  int32_t *items;
  __device__ ItemOut local() const { return *this; }
  __device__ void put(int64_t i, int64_t place) const { items[place] = (int32_t)i; }
};

}  // namespace

void exclusive_scan_i32(const int32_t *in, int64_t *out, int64_t n,
                        hipStream_t s, Allocator &al) {
  exclusive_scan_impl<int32_t>(in, out, n, s, al);
}

void exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n,
                        hipStream_t s, Allocator &al) {
  exclusive_scan_impl<int64_t>(in, out, n, s, al);
}

uint64_t *radix_sort_u64(uint64_t *keys, uint64_t *tmp, int64_t n, int lo_bit,
                         int hi_bit, hipStream_t s, Allocator &al) {
  if (n <= 1 || hi_bit <= lo_bit) return keys;
  const int64_t nb = ceil_div(n, kSortTile);
  ND_REQUIRE(nb * 256 < (int64_t)1 << 31, ND_ERR_INVALID,
             "radix sort: %lld keys is too many", (long long)n);
  const bool self = nb <= kSortSelf;
  DArr<int32_t> hist(al, 256 * nb);
  DArr<int64_t> offs;
  if (!self) offs.reset(al, 256 * nb + 1);
  uint64_t *src = keys, *dst = tmp;
  for (int shift = lo_bit; shift < hi_bit; shift += 8) {
    k_radix_hist<<<(unsigned)nb, kSortThreads, 0, s>>>(src, n, shift, hist.p,
                                                        nb);
    ND_LAUNCHED();
    if (!self) exclusive_scan_i32(hist.p, offs.p, 256 * nb, s, al);
    k_radix_scatter<<<(unsigned)nb, kSortThreads, 0, s>>>(src, dst, n, shift,
                                                           hist.p, offs.p, nb);
    ND_LAUNCHED();
    uint64_t *t = src;
    src = dst;
    dst = t;
  }
  return src;
}

static_assert(sizeof(part::Head) == 8 * kPartHeadWords, "the head's words");

void partition_start(const uint8_t *bin, int64_t n, int32_t *items,
                     int64_t *head, hipStream_t s, Allocator &al) {
  if (n > 0)
    part::run<5>(ByteIn{bin}, ItemOut{items}, n, reinterpret_cast<part::Head *>(head),
                 s, al);
}

void partition_offsets(const int64_t *head, int64_t n, int nbins,
                       int64_t *offsets) {
  ND_REQUIRE(nbins >= 1 && nbins <= 5, ND_ERR_INVALID, "bad bin count");
  const part::Head *h = reinterpret_cast<const part::Head *>(head);
  for (int b = 0; b < nbins; b++) offsets[b] = n > 0 ? h->start[b] : 0;
  offsets[nbins] = n > 0 ? n : 0;
}

void partition_by_bin(const uint8_t *bin, int64_t n, int nbins, int32_t *items,
                      int64_t *offsets, hipStream_t s, Allocator &al) {
  DArr<int64_t> head(al, kPartHeadWords);
  partition_start(bin, n, items, head.p, s, al);
  PinnedChunk pc;
  const int64_t *h = n > 0 ? pc.read(head.p, kPartHeadWords, s) : head.p;
  partition_offsets(h, n, nbins, offsets);
}

void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  k_fill_i32<<<grid_for(n, 256), 256, 0, s>>>(p, v, n);
  ND_LAUNCHED();
}

namespace {
__global__ void k_iota_i32(int32_t *__restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int32_t)i;
}
}  // namespace

void iota_i32(int32_t *p, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  k_iota_i32<<<grid_for(n, 256), 256, 0, s>>>(p, n);
  ND_LAUNCHED();
}

void fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  k_fill_u8<<<grid_for(ceil_div(n, 4), 256), 256, 0, s>>>(p, v, n);
  ND_LAUNCHED();
}

void fill_u64(uint64_t *p, uint64_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  k_fill_u64<<<grid_for(n, 256), 256, 0, s>>>(p, v, n);
  ND_LAUNCHED();
}

namespace {

__global__ void k_post(uint32_t *__restrict__ to, const uint32_t *__restrict__ from,
                       int words) {
  for (int i = threadIdx.x; i < words; i += blockDim.x) to[i] = from[i];
}

std::mutex g_pinned_mu;
std::vector<void *> g_pinned_free;
}  // namespace

PinnedChunk::PinnedChunk() {
  {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    if (!g_pinned_free.empty()) {
      p_ = g_pinned_free.back();
      g_pinned_free.pop_back();
      return;
    }
  }
  ND_HIP(hipHostMalloc(&p_, kBytes, hipHostMallocDefault));
}

PinnedChunk::~PinnedChunk() {
  std::lock_guard<std::mutex> lk(g_pinned_mu);
  g_pinned_free.push_back(p_);
}

void PinnedChunk::post_words(void *to, const void *dev, size_t words,
                             hipStream_t s) {
  k_post<<<1, kWave, 0, s>>>(static_cast<uint32_t *>(to),
                             static_cast<const uint32_t *>(dev), (int)words);
  ND_LAUNCHED();
}

int64_t read_i64(const int64_t *dev, hipStream_t s) {
  PinnedChunk h;
  return *h.read(dev, 1, s);
}

}  // namespace nd
