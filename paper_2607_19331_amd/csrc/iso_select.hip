// TopKMask selection (App. F, TIES "Trim"): exact k-largest-magnitude selection by
// radix select over the storage magnitude keys, ties at the threshold broken by
// flat index.  bf16 keys (15 bits) take one histogram pass; fp32 keys (31 bits)
// take three (15 + 8 + 8 bits).
//
// Per pass, every (tensor, delta) "unit" is cut into chunks; one 1024-thread
// workgroup per chunk builds a 2^bits-bin histogram in LDS (128 KB for 15 bits)
// and flushes its nonzero bins to the unit's global histogram with integer
// atomics (deterministic: counts only).  A resolve kernel (one workgroup per
// unit) then finds the digit holding the k-th largest key.  If only part of the
// threshold bucket is kept, a tie pass counts threshold keys per 64K-element
// chunk and a find kernel walks to the quota-th tie in flat order.
#include <vector>

#include "iso_device.h"
#include "iso_kernels.h"

namespace iso {

constexpr int kHistThreads = 1024;
constexpr int kMaxBins = 1 << 15;

// ---- block helpers ------------------------------------------------------------------------------

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
  return v;
}

// Inclusive prefix sum over the block (blockDim.x <= 1024, multiple of 64).
__device__ int64_t block_inclusive_scan(int64_t v, int64_t* sh /* >= 16 */) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int64_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  if (wid == 0) {
    int64_t t = (lane < nw) ? sh[lane] : 0;
    for (int o = 1; o < 16; o <<= 1) {
      int64_t y = __shfl_up(t, o, 64);
      if (lane >= o) t += y;
    }
    if (lane < nw) sh[lane] = t;
  }
  __syncthreads();
  int64_t add = (wid > 0) ? sh[wid - 1] : 0;
  __syncthreads();
  return x + add;
}

// ---- unit setup ---------------------------------------------------------------------------------

// A unit's state before the first pass; skip: finished (no key selected).
// A member of a joint selection starts with its group's count (so that it is histogrammed
// whenever the group keeps anything); k_group_assign sets its own share before the resolve.
__device__ __forceinline__ UnitState unit_start(const DevTensor& T, int64_t k, bool skip) {
  UnitState s;
  s.prefix = 0;
  s.key_max = 0;
  s.k_rem = k;
  s.n_above = 0;
  s.bucket = T.n;
  s.cutoff = 0;
  s.done = (k == 0 || T.n == 0 || skip) ? 1 : 0;
  if (s.done) s.prefix = kNoSelectKey;
  s.pad[0] = s.pad[1] = s.pad[2] = 0;
  return s;
}

__global__ void k_select_init(const DevTensor* tab, int n_t, int K, UnitState* st, const int* gid, const int64_t* gk) {
  int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n_t * K) return;
  const DevTensor& T = tab[u / K];
  const int g = (gid != nullptr) ? gid[u / K] : -1;
  st[u] = unit_start(T, (g >= 0) ? gk[g] : T.k, false);
}

// Work item -> (tensor j, delta i, chunk c), items of tensor j laid out delta-major.
__device__ __forceinline__ void item_of(const int64_t* item0, int n_t, int K, int64_t chunk, const DevTensor* tab,
                                        int64_t item, int& j, int& i, int64_t& c) {
  int lo = 0, hi = n_t - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (item0[mid] <= item) lo = mid; else hi = mid - 1;
  }
  j = lo;
  int64_t nch = (tab[j].n + chunk - 1) / chunk;
  int64_t local = item - item0[j];
  i = (int)(local / nch);
  c = local - (int64_t)i * nch;
}

// ---- histogram pass -----------------------------------------------------------------------------
// With `dump` set (last pass only), the block also stores its chunk histogram (bin 0 =
// in-bucket entries whose digit is 0) so ties can later be located without another read.
//
// One workgroup per CU (128 KB of bins), so nothing overlaps its phases: clearing, counting (the
// chunk at the CU's share of HBM, LDS atomics and the key arithmetic), and the flush of the
// nonzero bins.  The bf16 pass does only what its keys need: digit 0 (a zero) is not counted but
// follows from the chunk's size, and the largest key is the highest bin in use.  Bins are cleared and
// flushed 16 bytes at a time.

struct HistLds {
  uint32_t bins[kMaxBins];
  uint32_t wmax[16];
  uint32_t wsum[16];
};

// Block sum and maximum (1024 threads) of one value each, in every thread.
__device__ __forceinline__ void hist_reduce(uint32_t& sum, uint32_t& mx, HistLds& sm) {
  for (int o = 32; o > 0; o >>= 1) sum += (uint32_t)__shfl_xor((int)sum, o, 64);
  mx = wave_max_u32(mx);
  if ((threadIdx.x & 63) == 0) {
    sm.wsum[threadIdx.x >> 6] = sum;
    sm.wmax[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  sum = mx = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    sum += sm.wsum[w];
    mx = max(mx, sm.wmax[w]);
  }
}

// One histogram work item: chunk c of delta i of tensor j; `item` numbers its dump slot.
template <int DT>
__device__ void hist_item(const DevTensor* __restrict__ tab, int K, int j, int i, int64_t c, int64_t item,
                          int64_t chunk, UnitState* __restrict__ st, uint32_t* __restrict__ hist, int shift,
                          int bits, int first, uint32_t* status, uint32_t* __restrict__ dump, HistLds& sm) {
  using F = Fmt<DT>;
  constexpr bool kBf = DT == ISO_BF16;         // one pass over the whole key
  constexpr int U = 8;                         // 16-byte loads in flight per thread
  uint32_t* lds = sm.bins;
  const int u = j * K + i;
  const DevTensor& T = tab[j];
  const bool active = !st[u].done;             // k == 0 units only need key_max from the first pass
  if (!first && !active) return;               // uniform per block
  const uint32_t nb = 1u << bits;
  for (uint32_t v = threadIdx.x; v < nb / 4; v += blockDim.x) ((uint4*)lds)[v] = make_uint4(0, 0, 0, 0);
  __syncthreads();

  const int hs = shift + bits;                 // bits above the digit must match the prefix
  const uint32_t want = (hs >= 32) ? 0u : (st[u].prefix >> hs);
  const uint32_t dmask = nb - 1u;
  const int64_t e0 = c * chunk;
  const int64_t e1 = min(T.n, e0 + chunk);
  const typename F::bits_t* p = (const typename F::bits_t*)T.deltas[i];
  uint32_t kmax = 0, nzero = 0;

  auto count = [&](uint32_t key) {
    if constexpr (kBf) {
      if (key != 0u) atomicAdd(&lds[key], 1u);
    } else {
      if (first) kmax = max(kmax, key);
      bool match = active && (first || ((key >> hs) == want));
      uint32_t d = (key >> shift) & dmask;
      if (match && d != 0u) atomicAdd(&lds[d], 1u);
      nzero += (match && d == 0u);
    }
  };

  const int64_t v0 = e0 / F::kPerVec;
  const int64_t v1 = e1 / F::kPerVec;         // full vectors only
  const uint4* pv = (const uint4*)p;
  for (int64_t v = v0 + threadIdx.x; v < v1; v += U * blockDim.x) {
    uint4 a[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      int64_t vv = v + (int64_t)q * blockDim.x;
      a[q] = (vv < v1) ? ld_stream(pv + vv) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      int64_t vv = v + (int64_t)q * blockDim.x;
      if (!kBf && vv >= v1) break;             // bf16: the zero fill counts nothing
      uint32_t w[4] = {a[q].x, a[q].y, a[q].z, a[q].w};
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        if constexpr (kBf) {
          count(w[h] & 0x7FFFu);
          count((w[h] >> 16) & 0x7FFFu);
        } else {
          count(w[h] & 0x7FFFFFFFu);
        }
      }
    }
  }
  // scalar tail (last chunk of a tensor whose size is not a multiple of the vector width)
  for (int64_t e = v1 * F::kPerVec + threadIdx.x; e < e1; e += blockDim.x)
    count(elem_bits<DT>(p, e) & F::kKeyMask);
  __syncthreads();

  uint4* gh = (uint4*)(hist + (size_t)u * kMaxBins);
  uint4* dp = (active && dump != nullptr) ? (uint4*)(dump + (size_t)item * nb) : nullptr;
  uint32_t nz = 0;                             // bf16: entries counted in this thread's bins
  if (active || kBf) {
    for (uint32_t v = threadIdx.x; v < nb / 4; v += blockDim.x) {
      const uint4 x = ((const uint4*)lds)[v];
      if (active) {
        if (x.x) atomicAdd(&gh[v].x, x.x);
        if (x.y) atomicAdd(&gh[v].y, x.y);
        if (x.z) atomicAdd(&gh[v].z, x.z);
        if (x.w) atomicAdd(&gh[v].w, x.w);
        if (dp != nullptr && v != 0) dp[v] = x;
      }
      if constexpr (kBf) {
        nz += x.x + x.y + x.z + x.w;
        const uint32_t top = x.w ? 3u : x.z ? 2u : x.y ? 1u : 0u;
        if (x.x | x.y | x.z | x.w) kmax = 4 * v + top;
      }
    }
  }
  uint32_t sum = kBf ? nz : nzero;
  if (kBf || first || dp != nullptr) hist_reduce(sum, kmax, sm);
  if (threadIdx.x == 0) {
    if (dp != nullptr) {
      uint4 x = ((const uint4*)lds)[0];
      x.x = kBf ? (uint32_t)(e1 - e0) - sum : sum;
      dp[0] = x;
    }
    if (first) {
      atomicMax(&st[u].key_max, kmax);
      const uint32_t expfield = kBf ? 0x7F80u : 0x7F800000u;
      if (kmax >= expfield) flag_status(status, kStatusNonFinite);
    }
  }
  __syncthreads();                             // LDS is reused by the block's next item
}

template <int DT>
__global__ void __launch_bounds__(kHistThreads) k_hist(const DevTensor* __restrict__ tab, int n_t, int K,
                                                       const int64_t* __restrict__ item0, int64_t chunk,
                                                       UnitState* __restrict__ st, uint32_t* __restrict__ hist,
                                                       int shift, int bits, int first, uint32_t* status,
                                                       uint32_t* __restrict__ dump) {
  __shared__ __attribute__((aligned(16))) HistLds sm;
  int j, i;
  int64_t c;
  item_of(item0, n_t, K, chunk, tab, blockIdx.x, j, i, c);
  hist_item<DT>(tab, K, j, i, c, blockIdx.x, chunk, st, hist, shift, bits, first, status, dump, sm);
}

// Persistent form over the flagged tensors only (items numbered as in k_hist).
template <int DT>
__global__ void __launch_bounds__(kHistThreads) k_hist_flagged(const DevTensor* __restrict__ tab, int n_t, int K,
                                                               const int64_t* __restrict__ item0, int64_t chunk,
                                                               UnitState* __restrict__ st,
                                                               uint32_t* __restrict__ hist, int shift, int bits,
                                                               int first, uint32_t* status,
                                                               uint32_t* __restrict__ dump,
                                                               const int* __restrict__ filter) {
  __shared__ __attribute__((aligned(16))) HistLds sm;
  __shared__ int sflag[1024];
  for_flagged_items(
      filter, n_t, sflag, [&](int j) { return (int64_t)K * ((tab[j].n + chunk - 1) / chunk); },
      [&](int j, int64_t it) {
        const int64_t nch = (tab[j].n + chunk - 1) / chunk;
        const int i = (int)(it / nch);
        const int64_t c = it - (int64_t)i * nch;
        hist_item<DT>(tab, K, j, i, c, item0[j] + it, chunk, st, hist, shift, bits, first, status, dump, sm);
      });
}

// The start of a filtered selection: unit states (units of unflagged tensors finished, with no key
// selected), the flagged tensors' global histograms cleared, their number added to *flagged.
__global__ void __launch_bounds__(1024) k_select_init_flagged(const DevTensor* __restrict__ tab, int n_t, int K,
                                                              UnitState* __restrict__ st, uint32_t* __restrict__ hist,
                                                              const int* __restrict__ filter, uint32_t* flagged,
                                                              const int* gid, const int64_t* gk) {
  __shared__ int sflag[1024];
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < (int64_t)n_t * K; u += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(u / K);
    const bool on = filter[j] != 0;
    const int g = (gid != nullptr) ? gid[j] : -1;
    st[u] = unit_start(tab[j], (g >= 0) ? gk[g] : tab[j].k, !on);
    if (on && u % K == 0 && flagged != nullptr) atomicAdd(flagged, 1u);
  }
  for_flagged_items(
      filter, n_t, sflag, [&](int) { return (int64_t)K * (kMaxBins / 1024); },
      [&](int j, int64_t it) { hist[(size_t)j * K * kMaxBins + (size_t)it * 1024 + threadIdx.x] = 0u; });
}

// ---- resolve: pick the digit holding the k_rem-th largest key ------------------------------------

__device__ __forceinline__ void emit_desc(const UnitState& s, iso_select_desc* __restrict__ out) {
  iso_select_desc d;
  d.t_key = s.prefix;
  d.key_max = s.key_max;
  if (s.prefix == kNoSelectKey) {
    d.n_above = 0; d.tie_quota = 0; d.tie_cutoff = 0;
  } else {
    d.n_above = s.n_above; d.tie_quota = s.k_rem; d.tie_cutoff = s.cutoff;
  }
  *out = d;
}

// Bin b of the LDS copy sits at b + b / 32: a thread sums 32 consecutive bins, and without the
// pad the 64 lanes of a wave would read one bank (a stride of 32 words).  With it and 16-byte loads
// three passes over one 256 x 256 fp32 matrix take 30 us less (the whole call 97 -> 67 us).
__device__ __forceinline__ uint32_t bin_pad(uint32_t b) { return b + (b >> 5); }

// The digit that holds the k_rem-th largest key of one unit, from the unit's global histogram;
// s receives the state after it.  `clear`: the global bins are zeroed for the next pass.  Block-
// uniform.  Bound by the latency of one workgroup: 128 KB read with eight 16-byte loads in
// flight per thread, then two walks over 32 bins per thread.
__device__ void resolve_unit(UnitState& s, uint32_t* __restrict__ gh, int shift, int bits, int clear, int last,
                             int64_t n, uint32_t* sbin, int64_t* sh, int64_t* found, uint32_t* status) {
  const uint32_t nb = 1u << bits;
  uint4* gv = (uint4*)gh;
#pragma unroll 8
  for (uint32_t v = threadIdx.x; v < nb / 4; v += blockDim.x) {
    const uint4 x = gv[v];
    const uint32_t at = bin_pad(4 * v);                // the four bins share one group of 32
    sbin[at] = x.x;
    sbin[at + 1] = x.y;
    sbin[at + 2] = x.z;
    sbin[at + 3] = x.w;
  }
  if (clear)
    for (uint32_t v = threadIdx.x; v < nb / 4; v += blockDim.x) gv[v] = make_uint4(0, 0, 0, 0);
  if (threadIdx.x == 0) { found[0] = -1; found[1] = 0; }
  __syncthreads();
  const uint32_t per = (nb + blockDim.x - 1) / blockDim.x;   // consecutive bins per thread
  const uint32_t b0 = threadIdx.x * per;
  // thread sums of bins >= 1 (bin 0 is reconstructed from the bucket total)
  int64_t mine = 0;
  for (uint32_t q = 0; q < per; ++q) {
    const uint32_t b = b0 + q;
    if (b < nb && b > 0) mine += sbin[bin_pad(b)];
  }
  const int64_t incl = block_inclusive_scan(mine, sh);
  if (threadIdx.x == blockDim.x - 1) found[2] = incl;
  __syncthreads();
  const int64_t total_nonzero = found[2];
  const int64_t zeros = s.bucket - total_nonzero;
  const int64_t need = s.k_rem;                        // 1 <= need <= bucket
  int64_t run = total_nonzero - incl;                  // entries in bins above this thread's range
  if (run < need && run + mine + (b0 == 0 ? zeros : 0) >= need) {
    for (int q = (int)per - 1; q >= 0; --q) {
      const uint32_t b = b0 + (uint32_t)q;
      if (b >= nb) continue;
      const int64_t h = (b == 0) ? zeros : (int64_t)sbin[bin_pad(b)];
      if (run < need && run + h >= need) { found[0] = b; found[1] = run; }
      run += h;
    }
  }
  __syncthreads();
  // found < 0 would mean inconsistent counts (cannot happen for 1 <= k_rem <= bucket); never index with it
  const int64_t d = found[0] < 0 ? 0 : found[0];
  if (found[0] < 0 && threadIdx.x == 0) flag_status(status, kStatusInternal);
  s.prefix |= (uint32_t)d << shift;
  s.n_above += found[1];
  s.k_rem = need - found[1];
  s.bucket = (d == 0) ? zeros : (int64_t)sbin[bin_pad((uint32_t)d)];
  if (last && s.k_rem == s.bucket) {
    s.cutoff = n;
    s.done = 1;
  }
}

constexpr int kPadBins = kMaxBins + kMaxBins / 32;

__global__ void __launch_bounds__(kHistThreads) k_resolve(const DevTensor* __restrict__ tab, int K,
                                                          UnitState* __restrict__ st, uint32_t* __restrict__ hist,
                                                          int shift, int bits, int last, uint32_t* status) {
  __shared__ uint32_t sbin[kPadBins];
  __shared__ int64_t sh[16];
  __shared__ int64_t found[3];
  const int u = blockIdx.x;
  UnitState s = st[u];
  if (s.done) return;
  resolve_unit(s, hist + (size_t)u * kMaxBins, shift, bits, !last, last, tab[u / K].n, sbin, sh, found, status);
  if (threadIdx.x == 0) st[u] = s;
}

// ---- joint selection (bf16, one pass) -------------------------------------------------------------
// The group's histogram is the sum of its members'; its threshold key and the number of entries
// with that key it keeps follow from it as for one tensor.  Each member then keeps its entries
// above the threshold and the next share of the threshold entries in table order, which is
// exactly a TopKMask of the member with that count: the per-unit resolve and tie search then
// give its descriptor unchanged.

// Group bins are 64-bit: a group (a whole-model delta) can hold more than 2^32 entries even
// though each member's own counts fit 32 bits.  With a filter only flagged groups are selected (a
// group's members are flagged together).
__global__ void __launch_bounds__(256) k_group_sum(int K, const int* __restrict__ gmem, const int* __restrict__ gmem0,
                                                   const uint32_t* __restrict__ hist, uint64_t* __restrict__ ghist,
                                                   const int* __restrict__ filter) {
  const int gi = blockIdx.y, g = gi / K, i = gi % K;
  if (filter != nullptr && !filter[gmem[gmem0[g]]]) return;
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= kMaxBins) return;
  uint64_t sum = 0;
  const int m1 = gmem0[g + 1];
#pragma unroll 8
  for (int m = gmem0[g]; m < m1; ++m) sum += hist[((size_t)gmem[m] * K + i) * kMaxBins + b];
  ghist[(size_t)gi * kMaxBins + b] = sum;
}

// The group histogram (256 KB of 64-bit bins) does not fit LDS; one workgroup reads it once, 32 bins a
// thread, kept in registers: a wave holds 2048 consecutive bins, read as 32 whole lines of 64.  The wave
// the rank falls into sums its lines from the top, eight at a time, and scans the line it ends in.
// Bound by the latency of that chain.  (Each thread reading a run of 32
// bins, twice: 35 us against 16 us.)
__global__ void __launch_bounds__(kHistThreads) k_group_resolve(const DevTensor* __restrict__ tab, int K,
                                                                const int* __restrict__ gmem,
                                                                const int* __restrict__ gmem0,
                                                                const int64_t* __restrict__ gk,
                                                                const uint64_t* __restrict__ ghist,
                                                                GroupState* __restrict__ gst, uint32_t* status,
                                                                const int* __restrict__ filter) {
  constexpr int kLines = kMaxBins / kHistThreads, kWaves = kHistThreads / 64, kStep = 8;
  __shared__ int64_t sh[kWaves];
  __shared__ int64_t found_d, found_above;
  const int gi = blockIdx.x, g = gi / K;
  const int64_t need = gk[g];
  if (need == 0 || (filter != nullptr && !filter[gmem[gmem0[g]]])) {
    if (threadIdx.x == 0) gst[gi] = GroupState{kNoSelectKey, 1, 0};
    return;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint64_t* gh = ghist + (size_t)gi * kMaxBins + wid * (64 * kLines) + lane;
  int64_t v[kLines], mine = 0;
#pragma unroll
  for (int q = 0; q < kLines; ++q) v[q] = (int64_t)gh[q * 64];
  if (threadIdx.x == 0) {
    v[0] = 0;                                       // bin 0 is not counted: the zeros are what is left
    found_d = -1;
    found_above = 0;
  }
#pragma unroll
  for (int q = 0; q < kLines; ++q) mine += v[q];
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
  if (lane == 0) sh[wid] = mine;
  __syncthreads();
  int64_t run = 0, total = 0;                       // entries above this wave's bins; all nonzero entries
  for (int w = 0; w < kWaves; ++w) {
    total += sh[w];
    if (w > wid) run += sh[w];
  }
  if (run < need && run + mine >= need) {           // the same for the whole wave
    bool done = false;
#pragma unroll
    for (int q0 = kLines - kStep; q0 >= 0; q0 -= kStep) {
      int64_t line[kStep];
#pragma unroll
      for (int e = 0; e < kStep; ++e) line[e] = v[q0 + e];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int e = 0; e < kStep; ++e) line[e] += __shfl_xor(line[e], o, 64);
#pragma unroll
      for (int e = kStep - 1; e >= 0; --e) {
        if (!done && run + line[e] >= need) {
          int64_t suf = v[q0 + e];                  // entries of this line's bins from the lane's on
          for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_down(suf, o, 64);
            if (lane + o < 64) suf += y;
          }
          const int64_t above = run + suf - v[q0 + e];
          if (above < need && run + suf >= need) {
            found_d = wid * (64 * kLines) + (q0 + e) * 64 + lane;
            found_above = above;
          }
          done = true;
        }
        run += line[e];
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (found_d < 0) {                              // every nonzero entry is kept, and some of the zeros
      int64_t n_g = 0;
      for (int m = gmem0[g]; m < gmem0[g + 1]; ++m) n_g += tab[gmem[m]].n;
      if (n_g < need) flag_status(status, kStatusInternal);
      found_above = total;
    }
    gst[gi] = GroupState{(uint32_t)(found_d < 0 ? 0 : found_d), 0, need - found_above};
  }
}

// Per member unit: entries above the group's threshold key and entries equal to it.
__global__ void __launch_bounds__(1024) k_member_counts(const DevTensor* __restrict__ tab, int K,
                                                        const int* __restrict__ gid,
                                                        const GroupState* __restrict__ gst,
                                                        const uint32_t* __restrict__ hist, int64_t* __restrict__ mcnt) {
  __shared__ int64_t sh[16];
  const int u = blockIdx.x, j = u / K, i = u % K;
  const int g = gid[j];
  if (g < 0) return;
  const GroupState G = gst[g * K + i];
  if (G.none) return;
  const uint32_t* h = hist + (size_t)u * kMaxBins;
  constexpr int kVecs = kMaxBins / 4 / 1024;
  uint4 x[kVecs];
#pragma unroll
  for (int q = 0; q < kVecs; ++q) x[q] = ((const uint4*)h)[q * 1024 + threadIdx.x];
  int64_t above = 0, nonzero = 0;
#pragma unroll
  for (int q = 0; q < kVecs; ++q) {
    const uint32_t b = 4u * (uint32_t)(q * 1024 + threadIdx.x), w[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (b + e > 0u) nonzero += w[e];
      if (b + e > G.t_key) above += w[e];
    }
  }
  above = block_inclusive_scan(above, sh);
  __syncthreads();
  nonzero = block_inclusive_scan(nonzero, sh);
  if (threadIdx.x == blockDim.x - 1) {
    mcnt[2 * (size_t)u] = above;
    mcnt[2 * (size_t)u + 1] = (G.t_key == 0) ? tab[j].n - nonzero : (int64_t)h[G.t_key];
  }
}

// One workgroup per (group, delta): the threshold entries go to the members in table order, 256
// members at a time (one thread walking 56 members took 23 us, a chain of dependent loads).
__global__ void __launch_bounds__(256) k_group_assign(int K, const int* __restrict__ gmem,
                                                      const int* __restrict__ gmem0,
                                                      const GroupState* __restrict__ gst,
                                                      const int64_t* __restrict__ mcnt, UnitState* __restrict__ st) {
  __shared__ int64_t sh[16];
  __shared__ int64_t s_total;
  const int gi = blockIdx.x, g = gi / K, i = gi % K;
  const GroupState G = gst[gi];
  if (G.none) return;
  int64_t before = 0;                               // threshold entries of earlier members
  for (int mb = gmem0[g]; mb < gmem0[g + 1]; mb += blockDim.x) {
    const int m = mb + (int)threadIdx.x;
    const int u = (m < gmem0[g + 1]) ? gmem[m] * K + i : -1;
    const bool on = u >= 0 && !st[u].done;          // an empty member is done
    const int64_t ties = on ? mcnt[2 * (size_t)u + 1] : 0;
    const int64_t incl = before + block_inclusive_scan(ties, sh);
    if (threadIdx.x == blockDim.x - 1) s_total = incl;
    if (on) {
      const int64_t kk = mcnt[2 * (size_t)u] + max<int64_t>(0, min(ties, G.quota - (incl - ties)));
      st[u].k_rem = kk;
      if (kk == 0) {
        st[u].done = 1;
        st[u].prefix = kNoSelectKey;
      }
    }
    __syncthreads();
    before = s_total;
    __syncthreads();
  }
}

// ---- ties from the chunk histograms: prefix over chunks, then one walk inside a chunk -----------

struct TieLds {
  int64_t chunk, before, seg, segbefore, idx, tot;
};

// Tie cutoff of unit u whose threshold key s.prefix is only partly kept (s.k_rem of s.bucket entries).
// cnt: LDS for one count per segment of a chunk (at most 4096).
template <int DT>
__device__ int64_t tie_find_dump(const DevTensor* __restrict__ tab, int K, const int64_t* __restrict__ item0,
                                 int64_t chunk, int u, const UnitState& s, const uint32_t* __restrict__ dump,
                                 int bits, uint32_t* cnt, int64_t* sh, TieLds& tl, uint32_t* status) {
  using F = Fmt<DT>;
  const int j = u / K, i = u % K;
  const DevTensor& T = tab[j];
  const uint32_t nb = 1u << bits;
  const int64_t nch = (T.n + chunk - 1) / chunk;
  const int64_t first_item = item0[j] + (int64_t)i * nch;
  const int64_t quota = s.k_rem;
  const uint32_t tk = s.prefix;
  const uint32_t digit = tk & (nb - 1u);
  if (threadIdx.x == 0) { tl.chunk = -1; tl.before = 0; tl.seg = -1; tl.segbefore = 0; tl.idx = -1; }
  __syncthreads();
  // 1) chunk holding the quota-th tie
  int64_t base = 0;
  for (int64_t c0 = 0; c0 < nch; c0 += blockDim.x) {
    const int64_t c = c0 + threadIdx.x;
    const int64_t v = (c < nch) ? (int64_t)dump[(size_t)(first_item + c) * nb + digit] : 0;
    const int64_t incl = block_inclusive_scan(v, sh);
    if (c < nch && base + incl - v < quota && base + incl >= quota) { tl.chunk = c; tl.before = base + incl - v; }
    if (threadIdx.x == blockDim.x - 1) tl.tot = incl;
    __syncthreads();
    base += tl.tot;
    __syncthreads();
    if (tl.chunk >= 0) break;
  }
  __syncthreads();
  if (tl.chunk < 0) {                                   // inconsistent counts: never walk out of range
    if (threadIdx.x == 0) flag_status(status, kStatusInternal);
    return T.n;
  }
  const int64_t e0 = tl.chunk * chunk, e1 = min(T.n, e0 + chunk);
  const int64_t want = quota - tl.before;               // 1-based rank inside the chunk
  // 2) threshold keys per segment of 64 vectors, one wave each (contiguous 1 KB reads, eight in
  //    flight per lane), then the segment by a scan.  One CU reads the chunk, so its loads in flight
  //    set the time: a thread per run of consecutive vectors took 110 us for 2^20 bf16 entries.
  constexpr int kSeg = 64 * F::kPerVec, U = 8;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const void* p = T.deltas[i];
  const int nseg = (int)((e1 - e0 + kSeg - 1) / kSeg);
  for (int s0 = wid; s0 < nseg; s0 += U * nw) {
    uint4 q[U];
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const int64_t e = e0 + (int64_t)(s0 + x * nw) * kSeg + lane * F::kPerVec;
      q[x] = (e + F::kPerVec <= e1) ? *((const uint4*)p + e / F::kPerVec) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const int sg = s0 + x * nw;
      if (sg >= nseg) break;                             // uniform over the wave
      const int64_t e = e0 + (int64_t)sg * kSeg + lane * F::kPerVec;
      uint32_t m = 0;
      if (e + F::kPerVec <= e1) {
        const uint32_t w[4] = {q[x].x, q[x].y, q[x].z, q[x].w};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          if constexpr (DT == ISO_BF16) m += ((w[h] & 0x7FFFu) == tk) + (((w[h] >> 16) & 0x7FFFu) == tk);
          else m += ((w[h] & 0x7FFFFFFFu) == tk);
        }
      } else {
        for (int64_t r = e; r < e1; ++r) m += ((elem_bits<DT>(p, r) & F::kKeyMask) == tk);
      }
      for (int o = 32; o > 0; o >>= 1) m += (uint32_t)__shfl_xor((int)m, o, 64);
      if (lane == 0) cnt[sg] = m;
    }
  }
  __syncthreads();
  const int per = (nseg + blockDim.x - 1) / blockDim.x, g0s = threadIdx.x * per;
  int64_t mine = 0;
  for (int x = g0s; x < min(nseg, g0s + per); ++x) mine += cnt[x];
  const int64_t incl = block_inclusive_scan(mine, sh);
  if (mine > 0 && incl - mine < want && incl >= want) {
    int64_t run = incl - mine;
    int x = g0s;
    while (run + cnt[x] < want) run += cnt[x++];
    tl.seg = x;
    tl.segbefore = run;
  }
  __syncthreads();
  if (tl.seg < 0) {
    if (threadIdx.x == 0) flag_status(status, kStatusInternal);
    return T.n;
  }
  // 3) the block walks that one segment (kSeg <= 512 entries)
  const int64_t g0 = e0 + tl.seg * kSeg;
  const int64_t e = g0 + threadIdx.x;
  const int64_t tie = (threadIdx.x < kSeg && e < e1) ? ((elem_bits<DT>(p, e) & F::kKeyMask) == tk) : 0;
  const int64_t r = block_inclusive_scan(tie, sh);
  if (tie && tl.segbefore + r == want) tl.idx = e;
  __syncthreads();
  if (tl.idx < 0 && threadIdx.x == 0) flag_status(status, kStatusInternal);
  return (tl.idx < 0) ? T.n : tl.idx + 1;
}

// The last pass's resolve, the tie search (from the chunk histograms) and the descriptor of each
// unit in one launch: all three are one workgroup per unit.
template <int DT>
__global__ void __launch_bounds__(kHistThreads) k_resolve_last(const DevTensor* __restrict__ tab, int K,
                                                               const int64_t* __restrict__ item0, int64_t chunk,
                                                               UnitState* __restrict__ st,
                                                               uint32_t* __restrict__ hist,
                                                               const uint32_t* __restrict__ dump, int shift, int bits,
                                                               iso_select_desc* __restrict__ desc, uint32_t* status) {
  __shared__ uint32_t sbin[kPadBins];
  __shared__ int64_t sh[16];
  __shared__ int64_t found[3];
  __shared__ TieLds tl;
  const int u = blockIdx.x;
  UnitState s = st[u];
  if (!s.done) {
    resolve_unit(s, hist + (size_t)u * kMaxBins, shift, bits, 0, 1, tab[u / K].n, sbin, sh, found, status);
    if (!s.done) {
      s.cutoff = tie_find_dump<DT>(tab, K, item0, chunk, u, s, dump, bits, sbin, sh, tl, status);
      s.done = 1;
    }
    if (threadIdx.x == 0) st[u] = s;
  }
  if (threadIdx.x == 0) emit_desc(s, desc + u);
}

// ---- ties: count threshold keys per chunk, then walk to the quota-th one -------------------------

template <int DT>
__device__ void tie_count_item(const DevTensor* __restrict__ tab, int K, int j, int i, int64_t c, int64_t item,
                               int64_t chunk, const UnitState* __restrict__ st, int32_t* __restrict__ cnt,
                               int64_t* sh) {
  using F = Fmt<DT>;
  const int u = j * K + i;
  if (st[u].done) return;
  const uint32_t tk = st[u].prefix;
  const DevTensor& T = tab[j];
  const int64_t e0 = c * chunk, e1 = min(T.n, e0 + chunk);
  const void* p = T.deltas[i];
  int64_t m = 0;
  const int64_t v0 = e0 / F::kPerVec, v1 = e1 / F::kPerVec;
  for (int64_t v = v0 + threadIdx.x; v < v1; v += blockDim.x) {
    uint4 a = ld_stream((const uint4*)p + v);
    uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      if constexpr (DT == ISO_BF16) {
        m += ((w[h] & 0x7FFFu) == tk) + (((w[h] >> 16) & 0x7FFFu) == tk);
      } else {
        m += ((w[h] & 0x7FFFFFFFu) == tk);
      }
    }
  }
  for (int64_t e = v1 * F::kPerVec + threadIdx.x; e < e1; e += blockDim.x)
    m += ((elem_bits<DT>(p, e) & F::kKeyMask) == tk);
  m = wave_sum_i64(m);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) cnt[item] = (int32_t)(sh[0] + sh[1] + sh[2] + sh[3]);
  __syncthreads();
}

template <int DT>
__global__ void __launch_bounds__(256) k_tie_count(const DevTensor* __restrict__ tab, int n_t, int K,
                                                   const int64_t* __restrict__ item0, int64_t chunk,
                                                   const UnitState* __restrict__ st, int32_t* __restrict__ cnt) {
  __shared__ int64_t sh[4];
  int j, i;
  int64_t c;
  item_of(item0, n_t, K, chunk, tab, blockIdx.x, j, i, c);
  tie_count_item<DT>(tab, K, j, i, c, blockIdx.x, chunk, st, cnt, sh);
}

template <int DT>
__global__ void __launch_bounds__(256) k_tie_count_flagged(const DevTensor* __restrict__ tab, int n_t, int K,
                                                           const int64_t* __restrict__ item0, int64_t chunk,
                                                           const UnitState* __restrict__ st,
                                                           int32_t* __restrict__ cnt, const int* __restrict__ filter) {
  __shared__ int64_t sh[4];
  __shared__ int sflag[1024];
  for_flagged_items(
      filter, n_t, sflag, [&](int j) { return (int64_t)K * ((tab[j].n + chunk - 1) / chunk); },
      [&](int j, int64_t it) {
        const int64_t nch = (tab[j].n + chunk - 1) / chunk;
        const int i = (int)(it / nch);
        tie_count_item<DT>(tab, K, j, i, it - (int64_t)i * nch, item0[j] + it, chunk, st, cnt, sh);
      });
}

template <int DT>
__global__ void __launch_bounds__(kHistThreads) k_tie_find(const DevTensor* __restrict__ tab, int K,
                                                           const int64_t* __restrict__ item0, int64_t chunk,
                                                           UnitState* __restrict__ st,
                                                           const int32_t* __restrict__ cnt, uint32_t* cnt_status) {
  using F = Fmt<DT>;
  __shared__ int64_t sh[16];
  __shared__ int64_t s_chunk, s_before;
  __shared__ int64_t s_idx;
  const int u = blockIdx.x;
  if (st[u].done) return;
  const int j = u / K, i = u % K;
  const DevTensor& T = tab[j];
  const int64_t nch = (T.n + chunk - 1) / chunk;
  const int32_t* cu = cnt + item0[j] + (int64_t)i * nch;
  const int64_t quota = st[u].k_rem;
  const uint32_t tk = st[u].prefix;
  if (threadIdx.x == 0) { s_chunk = -1; s_before = 0; s_idx = -1; }
  __syncthreads();
  // 1) chunk that holds the quota-th tie
  int64_t base = 0;
  for (int64_t c0 = 0; c0 < nch; c0 += blockDim.x) {
    int64_t c = c0 + threadIdx.x;
    int64_t v = (c < nch) ? cu[c] : 0;
    int64_t incl = block_inclusive_scan(v, sh);
    int64_t excl = incl - v;
    if (c < nch && base + excl < quota && base + incl >= quota) { s_chunk = c; s_before = base + excl; }
    __shared__ int64_t s_tot;
    if (threadIdx.x == blockDim.x - 1) s_tot = incl;
    __syncthreads();
    base += s_tot;
    __syncthreads();
    if (s_chunk >= 0) break;
  }
  __syncthreads();
  if (s_chunk < 0) {                                  // inconsistent tie counts: never walk out of range
    if (threadIdx.x == 0) { st[u].cutoff = T.n; st[u].done = 1; flag_status(cnt_status, kStatusInternal); }
    return;
  }
  const int64_t c = s_chunk;
  int64_t want = quota - s_before;                    // 1-based rank inside the chunk
  // 2) walk the chunk in flat order
  const void* p = T.deltas[i];
  const int64_t e0 = c * chunk, e1 = min(T.n, e0 + chunk);
  int64_t seen = 0;
  for (int64_t b = e0; b < e1; b += blockDim.x) {
    int64_t e = b + threadIdx.x;
    int64_t tie = (e < e1) ? ((elem_bits<DT>(p, e) & F::kKeyMask) == tk) : 0;
    int64_t incl = block_inclusive_scan(tie, sh);
    if (tie && seen + incl == want) s_idx = e;
    __shared__ int64_t s_tot2;
    if (threadIdx.x == blockDim.x - 1) s_tot2 = incl;
    __syncthreads();
    seen += s_tot2;
    __syncthreads();
    if (s_idx >= 0) break;
  }
  if (threadIdx.x == 0) {
    if (s_idx < 0) flag_status(cnt_status, kStatusInternal);
    st[u].cutoff = (s_idx < 0) ? T.n : s_idx + 1;
    st[u].done = 1;
  }
}

__global__ void k_emit_desc(const UnitState* __restrict__ st, int n_units, iso_select_desc* __restrict__ desc) {
  int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n_units) return;
  emit_desc(st[u], desc + u);
}

// ---- optional bitset output ---------------------------------------------------------------------

// One lane per eight entries (one 16-byte load of bf16, two of fp32): its mask byte joins those of
// the three lanes beside it by DPP and every fourth lane stores a 32-bit word, four octets in flight
// per lane.  Bound by the read of the delta.  One lane per word, reading 32 entries one by one, took
// 157 us for four deltas of 16.8M bf16 entries (0.9 TB/s).
constexpr int kMaskOct = 4;                       // octets per lane and step
template <int DT>
__device__ __forceinline__ uint32_t mask_octet(const typename Fmt<DT>::bits_t* p, int64_t o, int64_t n,
                                               const uint4 (&a)[DT == ISO_BF16 ? 1 : 2], const iso_select_desc& d) {
  using F = Fmt<DT>;
  uint32_t m = 0;
  auto take = [&](int b, uint32_t bits) {
    const uint32_t key = bits & F::kKeyMask;
    const bool sel = key > d.t_key || (key == d.t_key && o * 8 + b < d.tie_cutoff);
    m |= (uint32_t)sel << b;
  };
  if (o * 8 + 8 <= n) {
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if constexpr (DT == ISO_BF16) {
        const uint32_t w = (b < 2) ? a[0].x : (b < 4) ? a[0].y : (b < 6) ? a[0].z : a[0].w;
        take(b, (b & 1) ? w >> 16 : w);
      } else {
        const uint4& v = a[b >> 2];
        take(b, (b & 3) == 0 ? v.x : (b & 3) == 1 ? v.y : (b & 3) == 2 ? v.z : v.w);
      }
    }
  } else {
    for (int b = 0; b < 8 && o * 8 + b < n; ++b) take(b, elem_bits<DT>(p, o * 8 + b));
  }
  return m;
}

template <int DT>
__global__ void __launch_bounds__(256) k_mask_bits(const DevTensor* __restrict__ tab, int K,
                                                   const iso_select_desc* __restrict__ desc,
                                                   uint32_t* const* __restrict__ bits_out) {
  constexpr int V = (DT == ISO_BF16) ? 1 : 2;
  const int u = blockIdx.y;
  const DevTensor& T = tab[u / K];
  const iso_select_desc d = desc[u];               // kNoSelectKey lies above every key
  const int64_t n = T.n, no = (n + 31) / 32 * 4;   // octets, those past the end included
  uint32_t* out = bits_out[u];
  const auto* p = (const typename Fmt<DT>::bits_t*)T.deltas[u % K];
  const int64_t step = (int64_t)gridDim.x * (256 * kMaskOct);
  for (int64_t o0 = (int64_t)blockIdx.x * (256 * kMaskOct) + threadIdx.x; o0 < no; o0 += step) {
    uint4 a[kMaskOct][V];
#pragma unroll
    for (int q = 0; q < kMaskOct; ++q) {
      const int64_t o = o0 + q * 256;
#pragma unroll
      for (int v = 0; v < V; ++v)
        a[q][v] = (o * 8 + 8 <= n) ? ld_stream((const uint4*)p + o * V + v) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < kMaskOct; ++q) {
      const int64_t o = o0 + q * 256;              // a word's four octets are four neighbouring lanes
      uint32_t m = mask_octet<DT>(p, o, n, a[q], d) << (8 * (threadIdx.x & 3));
      m |= (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xB1, 0xF, 0xF, true);   // lane ^ 1
      m |= (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4E, 0xF, 0xF, true);   // lane ^ 2
      if ((threadIdx.x & 3) == 0 && o < no) out[o >> 2] = m;
    }
  }
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ---- host-side launch sequence ------------------------------------------------------------------

// Entries per histogram work item.  At most 2048 items, in chunks of 2^16 to 2^20 entries, is the
// coarse rule (and the only one where the histogram is the single-read path's fallback).  A CU runs
// one item at a time, and an item costs about as much as 2^16 bf16 entries besides its entries (clearing,
// flush and dump of its bins; 3 * 2^13 fp32 entries, the mean of one pass over all bins and two over few), so among
// the larger chunks the one with the least waves * (entries + overhead) is taken.  The CUs do not end long fp32
// items together: c^2 / 2^22 is added for the last wave (in one wave of 655360 entries 143M fp32 entries took 464 us,
// in three of 212992 393; 32M in one wave of 147456 120 us, in two of 65536 140).  12 deltas of 4.2M to 8.4M bf16 entries: 1028 items of 2^16
// in five waves -> 252 items in one, the select and what follows it 268 -> 235 us.
int64_t hist_chunk_for(const iso_tensor* t, int n_t, int K, int dt, bool fallback) {
  int64_t total = 0;
  for (int j = 0; j < n_t; ++j) total += t[j].rows * t[j].cols * (int64_t)K;
  const int64_t most = 1 << 20;
  int64_t c0 = 1 << 16;
  while (c0 < most && total / c0 > 2048) c0 <<= 1;
  if (fallback || c0 == most) return c0;
  // A tensor of at most c0 entries is one item per delta whatever the chunk; the others, at most 2048 / K, are
  // counted for each.  (All tensors for each of up to 33 chunks: 53 us for 339 tensors, 3.6 ms for 20000, on the host.)
  std::vector<int64_t> large;
  int64_t ones = 0;
  for (int j = 0; j < n_t; ++j) {
    const int64_t n = t[j].rows * t[j].cols;
    if (n > c0) large.push_back(n);
    else if (n > 0) ++ones;
  }
  const int64_t overhead = (dt == ISO_BF16) ? 1 << 16 : 3 << 13;
  int64_t best = c0, best_cost = INT64_MAX;
  for (int64_t oct = c0; oct <= most; oct *= 2)
    for (int64_t c = oct; c < 2 * oct && c <= most; c += oct / 8) {
      int64_t items = K * ones;
      for (const int64_t n : large) items += K * ((n + c - 1) / c);
      const int64_t cost = (items + 255) / 256 * (c + overhead) + (dt == ISO_BF16 ? 0 : c * c >> 22);
      if (cost < best_cost) {
        best = c;
        best_cost = cost;
      }
      if (items <= 256) return best;             // a larger chunk only lengthens the one wave
      if (large.empty()) return best;            // nor does it save an item
    }
  return best;
}

hipError_t fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  k_fill_u32<<<(unsigned)blocks, 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

template <int DT>
static hipError_t run_select_t(const SelectPlan& pl, hipStream_t s) {
  const int nu = pl.n_t * pl.K;
  const bool flt = pl.filter != nullptr;
  constexpr unsigned kFlaggedGrid = 256;
  // the entry points reject groups of fp32 tensors
  if (pl.n_groups > 0 && DT != ISO_BF16) return hipErrorInvalidValue;
  const int* gid = pl.n_groups > 0 ? pl.gid : nullptr;
  if (flt)
    k_select_init_flagged<<<kFlaggedGrid, 1024, 0, s>>>(pl.tab, pl.n_t, pl.K, pl.states, pl.hist, pl.filter, pl.flagged,
                                                        gid, pl.gk);
  else
    k_select_init<<<(nu + 255) / 256, 256, 0, s>>>(pl.tab, pl.n_t, pl.K, pl.states, gid, pl.gk);
  struct Pass { int shift, bits; };
  const Pass bf[1] = {{0, 15}};
  const Pass f32[3] = {{16, 15}, {8, 8}, {0, 8}};
  const Pass* ps = (DT == ISO_BF16) ? bf : f32;
  const int np = (DT == ISO_BF16) ? 1 : 3;
  for (int q = 0; q < np; ++q) {
    uint32_t* dump = (q == np - 1) ? pl.chunk_hist : nullptr;
    if (pl.hist_items > 0 && flt)
      k_hist_flagged<DT><<<kFlaggedGrid, kHistThreads, 0, s>>>(pl.tab, pl.n_t, pl.K, pl.hist_item0, pl.hist_chunk,
                                                               pl.states, pl.hist, ps[q].shift, ps[q].bits, q == 0,
                                                               pl.status, dump, pl.filter);
    else if (pl.hist_items > 0)
      k_hist<DT><<<(unsigned)pl.hist_items, kHistThreads, 0, s>>>(pl.tab, pl.n_t, pl.K, pl.hist_item0, pl.hist_chunk,
                                                                  pl.states, pl.hist, ps[q].shift, ps[q].bits,
                                                                  q == 0, pl.status, dump);
    if (pl.n_groups > 0) {
      const int ngk = pl.n_groups * pl.K;
      k_group_sum<<<dim3(kMaxBins / 256, (unsigned)ngk), 256, 0, s>>>(pl.K, pl.gmem, pl.gmem0, pl.hist, pl.ghist,
                                                                    pl.filter);
      k_group_resolve<<<ngk, kHistThreads, 0, s>>>(pl.tab, pl.K, pl.gmem, pl.gmem0, pl.gk, pl.ghist, pl.gstate,
                                                   pl.status, pl.filter);
      k_member_counts<<<nu, 1024, 0, s>>>(pl.tab, pl.K, pl.gid, pl.gstate, pl.hist, pl.mcnt);
      k_group_assign<<<ngk, 256, 0, s>>>(pl.K, pl.gmem, pl.gmem0, pl.gstate, pl.mcnt, pl.states);
    }
    if (q == np - 1 && pl.chunk_hist != nullptr)
      k_resolve_last<DT><<<nu, kHistThreads, 0, s>>>(pl.tab, pl.K, pl.hist_item0, pl.hist_chunk, pl.states, pl.hist,
                                                     pl.chunk_hist, ps[q].shift, ps[q].bits, pl.desc, pl.status);
    else
      k_resolve<<<nu, kHistThreads, 0, s>>>(pl.tab, pl.K, pl.states, pl.hist, ps[q].shift, ps[q].bits, q == np - 1,
                                            pl.status);
  }
  if (pl.chunk_hist == nullptr) {
    if (pl.tie_items > 0 && flt)
      k_tie_count_flagged<DT><<<kFlaggedGrid * 4, 256, 0, s>>>(pl.tab, pl.n_t, pl.K, pl.tie_item0, pl.tie_chunk,
                                                               pl.states, pl.tie_cnt, pl.filter);
    else if (pl.tie_items > 0)
      k_tie_count<DT><<<(unsigned)pl.tie_items, 256, 0, s>>>(pl.tab, pl.n_t, pl.K, pl.tie_item0, pl.tie_chunk,
                                                             pl.states, pl.tie_cnt);
    k_tie_find<DT><<<nu, kHistThreads, 0, s>>>(pl.tab, pl.K, pl.tie_item0, pl.tie_chunk, pl.states, pl.tie_cnt,
                                                pl.status);
    k_emit_desc<<<(nu + 255) / 256, 256, 0, s>>>(pl.states, nu, pl.desc);
  }
  return hipGetLastError();
}

int select_last_bits(int dt) { return dt == ISO_BF16 ? 15 : 8; }

hipError_t run_select(const SelectPlan& pl, int dt, hipStream_t s) {
  return dt == ISO_BF16 ? run_select_t<ISO_BF16>(pl, s) : run_select_t<ISO_F32>(pl, s);
}

hipError_t run_mask_bits(const DevTensor* tab, int n_t, int K, int dt, const iso_select_desc* desc,
                         uint32_t* const* bits_dev, int64_t max_n, hipStream_t s) {
  const int nu = n_t * K;
  const int64_t no = (max_n + 7) / 8;
  dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>((no + 256 * kMaskOct - 1) / (256 * kMaskOct), 2048)), nu);
  if (dt == ISO_BF16) k_mask_bits<ISO_BF16><<<grid, 256, 0, s>>>(tab, K, desc, bits_dev);
  else k_mask_bits<ISO_F32><<<grid, 256, 0, s>>>(tab, K, desc, bits_dev);
  return hipGetLastError();
}

}  // namespace iso
