// tiny.hip -- plain sweeps of a graph small enough for one workgroup's LDS.
//
// A sweep of a few thousand r-cliques on the whole GPU is a launch, a chain of
// about eight dependent loads and the gap to the next launch: 12-14 us,
// whatever it computes.  Here one workgroup of 16 waves runs up to kTinySweeps
// sweeps in one launch: tau, the lists' offsets and the minima stay in LDS,
// only the ids stream from the L2 each sweep, and two barriers separate
// gathering from updating.  Bound by that stream and the LDS of one CU, about
// 2 us + 0.4 ns an incidence.
//
// Whole decompositions, whole GPU -> here: k-core of 2000 vertices, 19956
// incidences, 18 sweeps 273 -> 182 us; of a path of 8190 vertices, 4095 sweeps
// 34.0 -> 19.8 ms; k-truss of 1048 edges, 16317 incidences, 10 sweeps 194 ->
// 156 us; (2,4), 615 edges, 19134 incidences 107 -> 107 us.  Beyond the limit
// it loses: k-core, 40380 incidences 281 -> 460 us; k-truss, 32262 incidences
// 211 -> 313 us; two hubs of 8000 neighbours, each a wave's serial work here,
// 378 -> 653 us: hence 20480 incidences and lists of up to 1024.
//
// SND's iterates exactly: every sweep reads the previous one's values only.
#include <algorithm>

#include "sweep_dev.h"

namespace nd {

namespace {

using namespace dev;

constexpr int kTinyThreads = 1024;
constexpr int kTinyWaves = kTinyThreads / kWave;

template <typename T>
struct TinyLds {
  T rho[kTinyIncidence];
  T tau[2][kTinyRcliques];
  int32_t off[kTinyRcliques + 1];
  int32_t changed;
};

struct TinyArgs {
  const int64_t *inc_off;
  const int32_t *inc_ids;
  const void *tau_in;  // tau of the first sweep
  void *tau_out[2];    // receive the last sweep's values (of the swept
                       // r-cliques; the others keep their zeros)
  SweepStats *ring;    // cleared
  int ring_len;
  int64_t first;       // number of the first sweep
  int count;           // sweeps, at most
  int swept, P;
  // bins by list length, longest first: [0, end[0]) lists above 256, then
  // 65..256, 17..64, 5..16, 1..4
  int end[5];
};

// H of the r-cliques [lo, hi), G lanes each, lists of at most 4 G minima.
template <int G, typename T>
__device__ __forceinline__ int tiny_bin(TinyLds<T> &L, int cur, int lo, int hi) {
  const int sl = lane_id() % G;
  int changed = 0;  // of the wave
  for (int p = lo; p < hi; p += kTinyThreads / G) {  // uniform
    const int i = p + (int)threadIdx.x / G;
    int b = 0, d = 0;
    int32_t c = 0;
    if (i < hi) {
      b = L.off[i];
      d = L.off[i + 1] - b;
      c = (int32_t)L.tau[cur][i];
    }
    int32_t rho[4];
#pragma unroll
    for (int m = 0; m < 4; m++) {
      const int j = sl + m * G;
      rho[m] = j < d ? (int32_t)L.rho[b + j] : -1;
    }
    const int cnt = count_ge<G, 4>(rho, c);
    const int32_t h = cnt >= c ? c : hindex_search<G, 4>(rho, c, cnt);
    const bool lead = i < hi && sl == 0;
    if (lead) L.tau[cur ^ 1][i] = (T)h;
    changed += __popcll(ballot(lead && h != c));
  }
  return changed;
}

// The same for longer lists, a wave each.
template <typename T>
__device__ __forceinline__ int tiny_long(TinyLds<T> &L, int cur, int hi) {
  const int lane = lane_id();
  int changed = 0;
  for (int i = threadIdx.x / kWave; i < hi; i += kTinyWaves) {
    const int b = L.off[i], d = L.off[i + 1] - b;
    const int32_t c = (int32_t)L.tau[cur][i];
    auto count = [&](int32_t x) {
      int n = 0;
      for (int j0 = 0; j0 < d; j0 += kWave)
        n += __popcll(ballot(j0 + lane < d && (int32_t)L.rho[b + j0 + lane] >= x));
      return n;
    };
    const int cnt = count(c);
    const int32_t h = cnt >= c ? c : hindex_between(count, c, cnt);
    if (lane == 0) L.tau[cur ^ 1][i] = (T)h;
    changed += h != c;
  }
  return changed;
}

template <int K, typename T>
__global__ __launch_bounds__(kTinyThreads) void k_sweep_tiny(TinyArgs a) {
  __shared__ TinyLds<T> L;
  const int t = threadIdx.x;
  const T *in = (const T *)a.tau_in;
  for (int i = t; i <= a.swept; i += kTinyThreads) L.off[i] = (int32_t)a.inc_off[i];
  for (int i = t; i < a.swept; i += kTinyThreads) L.tau[0][i] = in[i];
  int cur = 0;
  for (int s = 0; s < a.count; s++) {  // uniform
    if (t == 0) L.changed = 0;
    __syncthreads();
#pragma unroll 4
    for (int e = t; e < a.P; e += kTinyThreads) {
      int32_t id[K];
      load_ids<K>(a.inc_ids, e, id);
      int32_t v = (int32_t)L.tau[cur][id[0]];
#pragma unroll
      for (int x = 1; x < K; x++) v = min(v, (int32_t)L.tau[cur][id[x]]);
      L.rho[e] = (T)v;
    }
    __syncthreads();
    int ch = tiny_long(L, cur, a.end[0]);
    ch += tiny_bin<64>(L, cur, a.end[0], a.end[1]);
    ch += tiny_bin<16>(L, cur, a.end[1], a.end[2]);
    ch += tiny_bin<4>(L, cur, a.end[2], a.end[3]);
    ch += tiny_bin<1>(L, cur, a.end[3], a.end[4]);
    if (lane_id() == 0 && ch) atomicAdd(&L.changed, ch);
    __syncthreads();
    const int changed = L.changed;
    if (t == 0) {
      SweepStats &st = a.ring[(a.first + s) % a.ring_len];
      st.part[0].changed = (unsigned long long)changed;
      st.part[0].evaluated = (unsigned long long)a.swept;
    }
    cur ^= 1;
    if (changed == 0) break;
    __syncthreads();  // `changed` is read before it is cleared
  }
  for (int q = 0; q < 2; q++) {
    T *out = (T *)a.tau_out[q];
    for (int i = t; i < a.swept; i += kTinyThreads) out[i] = L.tau[cur][i];
  }
}

template <typename T>
void launch(const KindState &ks, const TinyArgs &a, hipStream_t s) {
  switch (ks.k) {
    case 1: k_sweep_tiny<1, T><<<1, kTinyThreads, 0, s>>>(a); break;
    case 2: k_sweep_tiny<2, T><<<1, kTinyThreads, 0, s>>>(a); break;
    case 3: k_sweep_tiny<3, T><<<1, kTinyThreads, 0, s>>>(a); break;
    case 5: k_sweep_tiny<5, T><<<1, kTinyThreads, 0, s>>>(a); break;
    default:
      ND_REQUIRE(false, ND_ERR_UNSUPPORTED, "no sweep kernel for k=%d", ks.k);
  }
  ND_LAUNCHED();
}

}  // namespace

bool tiny_fits(const KindState &ks) {
  return ks.tau_bytes <= 2 && ks.bin_lo[kBinZero] <= kTinyRcliques &&
         ks.P <= kTinyIncidence && ks.bin_hi[kBinWave] == 0;
}

void launch_tiny(const KindState &ks, const void *tau_in, void *tau0, void *tau1,
                 SweepStats *ring, int ring_len, int64_t first, int count,
                 hipStream_t s) {
  TinyArgs a{};
  a.inc_off = ks.inc_off.p;
  a.inc_ids = ks.inc_ids.p;
  a.tau_in = tau_in;
  a.tau_out[0] = tau0;
  a.tau_out[1] = tau1;
  a.ring = ring;
  a.ring_len = ring_len;
  a.first = first;
  a.count = count;
  a.swept = (int)ks.bin_lo[kBinZero];
  a.P = (int)ks.P;
  const int last[5] = {kBinWave8, kBinG64, kBinG16, kBinG4, kBinG1};
  for (int b = 0; b < 5; b++) a.end[b] = (int)ks.bin_hi[last[b]];
  if (ks.tau_bytes == 1)
    launch<uint8_t>(ks, a, s);
  else
    launch<uint16_t>(ks, a, s);
}

}  // namespace nd
