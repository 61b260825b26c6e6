// Sort and de-duplication of one step's lookups (the paper's Sec. 5.1: sort the
// row indices of the mini-batch, merge the gradients of each row).
//
//   k_expand       lookups -> (set-major row key, gradient-row index), position order
//   radix passes   stable LSD radix sort, 8-bit digits, wave-ballot ranking, one kernel
//                  per pass with decoupled look-back
//   scans          3-phase exclusive prefix sums (u32 / u64)
//   k_uniq_*       unique-row and touched-set lists (first occurrence of each row / set)
#include <algorithm>

#include "embc_device.h"
#include "embc_dispatch.h"
#include "embc_offsets.h"
#include "embc_sort.h"

namespace embc {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kRadixThreads = 256;
constexpr int kRadixItems = 16;
constexpr int kRadixTile = kRadixThreads * kRadixItems;
constexpr int kRadixWaves = kRadixThreads / 64;

size_t scan_partial_words(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile + 64); }

// ---- block-wide exclusive scan of one value per thread (256 threads) -------------------
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* lds4, T& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds4[wv] = x;
  __syncthreads();
  T pre = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) {
    const T s = lds4[w];
    if (w < wv) pre += s;
    total += s;
  }
  __syncthreads();
  return pre + x - v;
}

// ---- 3-phase exclusive scan ---------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const T* __restrict__ in, int64_t n,
                                                              const unsigned long long* dev_n, T* part) {
  __shared__ T lds4[4];
  if (dev_n) n = min(n, (int64_t)*dev_n);
  if ((int64_t)blockIdx.x * kScanTile >= n) return;  // a tile past the values (whole block)
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i < n) s += in[base + i];
  T tot;
  block_exclusive_scan<T>(s, lds4, tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Exclusive scan of in[0, nb) into out (which may be in) by one block of kScanThreads,
// kTopItems consecutive values per thread and round; *total_out = the sum.
constexpr int kTopItems = 16;
template <typename T>
__device__ __forceinline__ void scan_one_block(const T* in, T* out, int64_t nb, T* total_out) {
  __shared__ T lds4[4];
  T carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += (int64_t)kScanThreads * kTopItems) {
    const int64_t base = b0 + (int64_t)threadIdx.x * kTopItems;
    T v[kTopItems];
    T s = 0;
#pragma unroll
    for (int q = 0; q < kTopItems; ++q) {
      v[q] = base + q < nb ? in[base + q] : (T)0;
      s += v[q];
    }
    T tot;
    T run = carry + block_exclusive_scan<T>(s, lds4, tot);
#pragma unroll
    for (int q = 0; q < kTopItems; ++q) {
      if (base + q < nb) out[base + q] = run;
      run += v[q];
    }
    carry += tot;
  }
  if (threadIdx.x == 0 && total_out) *total_out = carry;
}

// The tiles past the device-side count (dev_n) hold no values: only the first
// ceil(min(n, dev_n) / kScanTile) partials are scanned.
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_top(T* part, int64_t nb, int64_t n,
                                                           const unsigned long long* dev_n, T* total_out) {
  if (dev_n) nb = min(nb, (min(n, (int64_t)*dev_n) + kScanTile - 1) / kScanTile);
  scan_one_block<T>(part, part, nb, total_out);
}

// A short array (tens of thousands of values) in one launch.
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_one(const T* in, T* out, int64_t n, T* total_out) {
  scan_one_block<T>(in, out, n, total_out);
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const T* __restrict__ in, T* __restrict__ out, int64_t n,
                                                            const unsigned long long* dev_n, const T* part) {
  __shared__ T lds4[4];
  if (dev_n) n = min(n, (int64_t)*dev_n);
  if ((int64_t)blockIdx.x * kScanTile >= n) return;  // a tile past the values (whole block)
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T v[kScanItems];
  T s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = base + i < n ? in[base + i] : (T)0;
    s += v[i];
  }
  T tot;
  T run = block_exclusive_scan<T>(s, lds4, tot) + part[blockIdx.x];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) out[base + i] = run;
    run += v[i];
  }
}

template <typename T>
hipError_t scan_exclusive(const T* in, T* out, int64_t n, const unsigned long long* dev_n, T* part, T* total,
                          hipStream_t s) {
  if (n <= 0) {
    if (total) k_scan_top<T><<<1, kScanThreads, 0, s>>>(part, 0, 0, nullptr, total);
    return hipGetLastError();
  }
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  k_scan_reduce<T><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, dev_n, part);
  k_scan_top<T><<<1, kScanThreads, 0, s>>>(part, nb, n, dev_n, total);
  k_scan_down<T><<<(unsigned)nb, kScanThreads, 0, s>>>(in, out, n, dev_n, part);
  return hipGetLastError();
}

// kScanItems consecutive values of a and b from element base (0 past n); whole runs are
// read 16 bytes at a time (the arrays are 16-byte aligned and base is a multiple of 8).
__device__ __forceinline__ void load_pair_items(const uint32_t* a, const uint32_t* b, int64_t n, int64_t base,
                                                uint32_t (&va)[kScanItems], uint32_t (&vb)[kScanItems]) {
  static_assert(kScanItems % 4 == 0, "runs of 16 bytes");
  if (base + kScanItems <= n) {
#pragma unroll
    for (int i = 0; i < kScanItems; i += 4) {
      const uint4 x = *reinterpret_cast<const uint4*>(a + base + i);
      const uint4 y = *reinterpret_cast<const uint4*>(b + base + i);
      va[i] = x.x; va[i + 1] = x.y; va[i + 2] = x.z; va[i + 3] = x.w;
      vb[i] = y.x; vb[i + 1] = y.y; vb[i + 2] = y.z; vb[i + 3] = y.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      va[i] = base + i < n ? a[base + i] : 0u;
      vb[i] = base + i < n ? b[base + i] : 0u;
    }
  }
}

// Exclusive scans of two u32 arrays at once (a + b * 2^32 as one u64 value per element:
// the prefix sums of a stay below 2^32), written to out_a and out_b (which may be a and
// b); *total = the two totals packed the same way.
__global__ __launch_bounds__(kScanThreads) void k_scan2_reduce(const uint32_t* __restrict__ a,
                                                               const uint32_t* __restrict__ b, int64_t n,
                                                               const unsigned long long* dev_n,
                                                               unsigned long long* part) {
  __shared__ unsigned long long lds4[4];
  if (dev_n) n = min(n, (int64_t)*dev_n);
  if ((int64_t)blockIdx.x * kScanTile >= n) return;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t va[kScanItems], vb[kScanItems];
  load_pair_items(a, b, n, base, va, vb);
  unsigned long long s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) s += (unsigned long long)va[i] | ((unsigned long long)vb[i] << 32);
  unsigned long long tot;
  block_exclusive_scan<unsigned long long>(s, lds4, tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kScanThreads) void k_scan2_down(const uint32_t* a, const uint32_t* b, uint32_t* out_a,
                                                             uint32_t* out_b, int64_t n,
                                                             const unsigned long long* dev_n,
                                                             const unsigned long long* part) {
  __shared__ unsigned long long lds4[4];
  if (dev_n) n = min(n, (int64_t)*dev_n);
  if ((int64_t)blockIdx.x * kScanTile >= n) return;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t va[kScanItems], vb[kScanItems];
  load_pair_items(a, b, n, base, va, vb);
  unsigned long long s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) s += (unsigned long long)va[i] | ((unsigned long long)vb[i] << 32);
  unsigned long long tot;
  unsigned long long run = block_exclusive_scan<unsigned long long>(s, lds4, tot) + part[blockIdx.x];
  // the exclusive prefixes replace the values in place (va, vb)
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const unsigned long long v = (unsigned long long)va[i] | ((unsigned long long)vb[i] << 32);
    va[i] = (uint32_t)run;
    vb[i] = (uint32_t)(run >> 32);
    run += v;
  }
  if (base + kScanItems <= n) {
#pragma unroll
    for (int i = 0; i < kScanItems; i += 4) {
      *reinterpret_cast<uint4*>(out_a + base + i) = make_uint4(va[i], va[i + 1], va[i + 2], va[i + 3]);
      *reinterpret_cast<uint4*>(out_b + base + i) = make_uint4(vb[i], vb[i + 1], vb[i + 2], vb[i + 3]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i)
      if (base + i < n) {
        out_a[base + i] = va[i];
        out_b[base + i] = vb[i];
      }
  }
}

hipError_t scan_exclusive_pair(const uint32_t* a, const uint32_t* b, uint32_t* out_a, uint32_t* out_b, int64_t n,
                               const unsigned long long* dev_n, unsigned long long* part,
                               unsigned long long* total, hipStream_t s) {
  if (n <= 0) {
    k_scan_top<unsigned long long><<<1, kScanThreads, 0, s>>>(part, 0, 0, nullptr, total);
    return hipGetLastError();
  }
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  k_scan2_reduce<<<(unsigned)nb, kScanThreads, 0, s>>>(a, b, n, dev_n, part);
  k_scan_top<unsigned long long><<<1, kScanThreads, 0, s>>>(part, nb, n, dev_n, total);
  k_scan2_down<<<(unsigned)nb, kScanThreads, 0, s>>>(a, b, out_a, out_b, n, dev_n, part);
  return hipGetLastError();
}

template hipError_t scan_exclusive<uint32_t>(const uint32_t*, uint32_t*, int64_t, const unsigned long long*,
                                             uint32_t*, uint32_t*, hipStream_t);
template hipError_t scan_exclusive<unsigned long long>(const unsigned long long*, unsigned long long*, int64_t,
                                                       const unsigned long long*, unsigned long long*,
                                                       unsigned long long*, hipStream_t);

// ---- LSD radix sort of (key, value) pairs -----------------------------------------------
// Stable LSD radix sort, one kernel per 8-bit digit pass, after the Onesweep method
// (Adinets and Merrill, "Onesweep: A Faster Least Significant Digit Radix Sort for
// GPUs", 2022): one histogram pass for every digit, then per digit pass a single
// sweep in which each tile finds its output offsets by decoupled look-back (Merrill
// and Garland, "Single-pass Parallel Prefix Scan with Decoupled Look-back", 2016):
//   k_sort_hist   global histograms of every pass's digit in one read of the keys
//   k_sort_scan   their exclusive prefix sums: where each digit's run starts
//   k_sort_pass   per tile of kRadixTile pairs (tiles taken in launch order from an
//                 atomic ticket): rank the tile's digits, publish the per-digit tile
//                 counts, find the tile's offset inside each digit's run by looking
//                 back over the published counts of the preceding tiles (decoupled
//                 look-back), then scatter through LDS in digit runs.
// A status word per (tile, digit) holds a 2-bit state and a 30-bit count: not yet
// published, the tile's own count, or the inclusive count up to and including the
// tile.  Tiles are numbered in the order their workgroups start, so every tile a
// look-back waits for is already running; the wait is bounded all the same (after
// kSortSpinLimit polls the step is flagged as failed and the tile goes on).
//
// Segmented mode.  The lookups arrive grouped by table (bag t*B + b belongs to table
// t), so the keys of table t fill the positions [P_t, P_t+1) and every valid key there
// lies in table t's key range.  Sorting each segment by the local key (key minus the
// table's key base) gives the global order in fewer passes when every table's key
// range is far smaller than the sum of them (100 tables of 5M rows: 3 passes instead
// of 4).  Tiles never straddle a segment (each segment starts a new tile), a look-back
// ends at the segment's first tile, and digit runs start at P_t.  The per-table digit
// counts are taken by the expansion (k_expand) as it forms the keys, so this mode has
// no histogram pass of its own.  A skipped lookup
// (kKeyInvalid) takes digit 255 in every pass, above every valid local key, so it ends
// its table's segment; when there is any, one more stable pass (digit 1 for a skipped
// key, 0 for the others) moves them behind every valid key, and the pairs are copied
// back so that the result stays in the same buffer.
constexpr uint32_t kStAgg = 1u << 30;
constexpr uint32_t kStPre = 2u << 30;
constexpr uint32_t kStCount = (1u << 30) - 1;
constexpr uint32_t kSortSpinLimit = 1u << 20;

size_t sort_status_words(int64_t n, int T) {
  return 256 * (size_t)((n + kRadixTile - 1) / kRadixTile + T + 1);
}
size_t sort_seg_words(int T) { return 2 * (size_t)T * kMaxPasses * 256 + 2 * (size_t)(T + 1) + 64; }

__device__ __forceinline__ uint32_t status_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Segment of tile `tile` (< tbase[T]): the largest t with tbase[t] <= tile.  Empty
// segments share their successor's first tile and are never returned.
__device__ __forceinline__ int seg_of_tile(const uint32_t* tbase, int T, uint32_t tile) {
  int lo = 0, hi = T;  // tbase[lo] <= tile < tbase[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (tbase[mid] <= tile) lo = mid; else hi = mid;
  }
  return lo;
}

// The same by a whole wave, 64 tables per round of loads.
__device__ __forceinline__ int seg_of_tile_wave(const uint32_t* tbase, int T, uint32_t tile) {
  int lo = 0;
  for (int hi = T; hi - lo > 1;) {
    const int step = (hi - lo + 63) / 64, c = lo + (int)(threadIdx.x & 63) * step;
    const uint64_t le = __ballot(c == lo || (c < hi && tbase[c] <= tile));
    lo += (63 - (int)__clzll((unsigned long long)le)) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Digit of a key in a pass of the segmented mode: the local key's, or 255 when skipped.
__device__ __forceinline__ uint32_t seg_digit(uint32_t key, uint32_t kb, int shift) {
  return key == kKeyInvalid ? 255u : ((key - kb) >> shift) & 255u;
}

// ghist [kMaxPasses][256] and the pass tickets must be zero on entry (k_sort_begin).
// Also clears the status words of the first pass.
__global__ __launch_bounds__(256) void k_sort_hist(const uint32_t* __restrict__ keys, int64_t n, int passes,
                                                   uint32_t* __restrict__ ghist, uint32_t* __restrict__ status,
                                                   int64_t status_words) {
  __shared__ uint32_t h[kRadixWaves][kMaxPasses][256];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < kRadixWaves * kMaxPasses * 256; i += 256) (&h[0][0][0])[i] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  // whole waves iterate together (the tail lanes count nothing), so that the lanes
  // sharing lane 0's digit are counted with one atomic: high digits of keys that
  // are nearly sorted would otherwise all hit one LDS word
  for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + wv * 64; i0 < n; i0 += stride) {
    const int64_t i = i0 + lane;
    const bool valid = i < n;
    const uint32_t k = valid ? keys[i] : 0u;
    for (int p = 0; p < passes; ++p) {
      const uint32_t d = (k >> (8 * p)) & 255u;
      const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);  // all lanes active: lane 0's
      const uint64_t same = __ballot(valid && d == d0);
      if (lane == 0) atomicAdd(&h[wv][p][d0], (uint32_t)__popcll(same));
      if (valid && d != d0) atomicAdd(&h[wv][p][d], 1u);
    }
  }
  __syncthreads();
  for (int p = 0; p < passes; ++p) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) c += h[w][p][threadIdx.x];
    if (c) atomicAdd(&ghist[p * 256 + threadIdx.x], c);
  }
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < status_words; i += stride) status[i] = 0;
}

__global__ void k_sort_begin(uint32_t* __restrict__ ghist, uint32_t* __restrict__ tickets) {
  for (int i = threadIdx.x; i < kMaxPasses * 256; i += blockDim.x) ghist[i] = 0;
  if (threadIdx.x < kMaxPasses) tickets[threadIdx.x] = 0;
}

// gbase[p][d] = number of keys whose pass-p digit is below d.
__global__ __launch_bounds__(256) void k_sort_scan(const uint32_t* __restrict__ ghist, uint32_t* __restrict__ gbase,
                                                   int passes) {
  __shared__ uint32_t lds4[4];
  for (int p = 0; p < passes; ++p) {
    uint32_t tot;
    gbase[p * 256 + threadIdx.x] = block_exclusive_scan<uint32_t>(ghist[p * 256 + threadIdx.x], lds4, tot);
  }
}

// Segment starts P_t (t = 0..T; P_0 = 0 and P_T = n, so positions outside every bag,
// which hold skipped keys, join the first or the last segment) and the first tile of
// each segment (tbase[T] = number of tiles), by block 0, which also zeroes the digit
// counts and tickets (as k_sort_begin does).  With malformed offsets every key is skipped
// and the whole stream is one segment.  The grid clears the per-table histograms.
__global__ __launch_bounds__(256) void k_seg_setup(const int32_t* __restrict__ off, int32_t B, int T, int64_t n,
                                                   const unsigned long long* __restrict__ ctr, SegSort sg,
                                                   uint32_t* __restrict__ ghist, uint32_t* __restrict__ tickets) {
  __shared__ uint32_t lds4[4];
  const int64_t hw = (int64_t)T * kMaxPasses * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < hw; i += (int64_t)gridDim.x * 256) sg.hist[i] = 0;
  if (blockIdx.x != 0) return;
  for (int i = threadIdx.x; i < kMaxPasses * 256; i += blockDim.x) ghist[i] = 0;
  if (threadIdx.x < kMaxPasses) tickets[threadIdx.x] = 0;
  const bool bad = ctr[kCBadOffsets] != 0;
  const auto start = [&](int t) -> int64_t {
    if (t <= 0) return 0;
    if (t >= T || bad) return n;
    return min<int64_t>(max<int64_t>(off[(int64_t)t * B], 0), n);
  };
  uint32_t run = 0;
  for (int t0 = 0; t0 <= T; t0 += 256) {
    const int t = t0 + (int)threadIdx.x;
    uint32_t tiles = 0;
    int64_t p = 0;
    if (t <= T) {
      p = start(t);
      if (t < T) tiles = (uint32_t)((start(t + 1) - p + kRadixTile - 1) / kRadixTile);
    }
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<uint32_t>(tiles, lds4, tot);
    if (t <= T) {
      sg.pos[t] = (uint32_t)p;
      sg.tbase[t] = run + ex;
    }
    run += tot;
  }
}

// base[t][p][d] = P_t + number of table t's keys whose pass-p digit is below d (one
// block per table); block 0 also writes the bases of the pass that moves skipped keys
// last: valid keys from 0, skipped ones from n - n_skipped.
__global__ __launch_bounds__(256) void k_seg_scan(SegSort sg, int passes, int64_t n,
                                                  const uint32_t* __restrict__ n_skipped,
                                                  uint32_t* __restrict__ skip_base) {
  __shared__ uint32_t lds4[4];
  const int t = blockIdx.x;
  for (int p = 0; p < passes; ++p) {
    const int64_t i = ((int64_t)t * kMaxPasses + p) * 256 + threadIdx.x;
    uint32_t tot;
    sg.base[i] = sg.pos[t] + block_exclusive_scan<uint32_t>(sg.hist[i], lds4, tot);
  }
  if (t == 0 && threadIdx.x < 2) skip_base[threadIdx.x] = threadIdx.x == 0 ? 0u : (uint32_t)(n - n_skipped[0]);
}

// One radix pass.  kModeSeg: tiles of the segmented mode (sg, pass), digits of the local
// key.  Otherwise tiles of the whole stream, with the key's digit at `shift`
// (kModeWhole) or 1 for a skipped key and 0 for the others (kModeSkipped); a non-null
// only_if skips the pass (and the copy below) unless *only_if.
// Without LOOP, a workgroup handles the one tile its ticket names (grid = tiles: a new
// workgroup's loads overlap the scatter of a finishing one).  With LOOP the grid is at
// most what the device holds at once and every workgroup takes tiles from the ticket
// until none is left (the pass that only runs when some key was skipped: when none
// was, it ends after one read of the flag per workgroup).  Either way a look-back only
// waits on tiles whose workgroups took their ticket earlier and are running.
// kModeRuns is kModeSeg for calls of moderate size: the digit runs' starts are scanned from
// the counts by every tile itself, which saves a launch, and nothing is done when the
// offsets were rejected (`only_if`, then a flag that stops the pass).
constexpr int kModeWhole = 0, kModeSeg = 1, kModeSkipped = 2, kModeRuns = 3;

template <int MODE, bool LOOP>
__global__ __launch_bounds__(kRadixThreads) void k_sort_pass(const uint32_t* __restrict__ kin,
                                                             const uint32_t* __restrict__ vin,
                                                             uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                             int64_t n, int shift, const uint32_t* __restrict__ gbase,
                                                             uint32_t* __restrict__ status, uint32_t* __restrict__ ticket,
                                                             uint32_t* __restrict__ next_status,
                                                             int64_t status_words, int32_t* __restrict__ err,
                                                             SegSort sg, const int64_t* __restrict__ key_base, int T,
                                                             int pass, const uint32_t* __restrict__ only_if) {
  __shared__ uint32_t wcnt[kRadixWaves][256];
  __shared__ uint32_t dpre[256];
  __shared__ uint32_t goff[256];
  __shared__ uint32_t skey[kRadixTile];
  __shared__ uint32_t sval[kRadixTile];
  __shared__ uint32_t lds4[4];
  __shared__ uint32_t tile_s;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  constexpr bool SEG = MODE == kModeSeg || MODE == kModeRuns;
  if (MODE == kModeRuns && *only_if != 0) return;
  const int64_t ntiles = SEG ? (int64_t)sg.tbase[T]
                             : (only_if == nullptr || *only_if != 0) ? (n + kRadixTile - 1) / kRadixTile : 0;
  for (;;) {
    for (int i = threadIdx.x; i < kRadixWaves * 256; i += kRadixThreads) (&wcnt[0][0])[i] = 0;
    if (threadIdx.x == 0) tile_s = ntiles > 0 ? atomicAdd(ticket, 1u) : 0xFFFFFFFFu;
    __syncthreads();
    const int64_t tile = tile_s;
    if (tile >= ntiles) break;  // block-uniform
    // the tile's table and position range
    int t = 0;
    int64_t tfirst = 0, lo = tile * kRadixTile, hi = min<int64_t>(n, lo + kRadixTile);
    uint32_t kb = 0;
    if (SEG) {
      t = MODE == kModeRuns ? seg_of_tile_wave(sg.tbase, T, (uint32_t)tile) : seg_of_tile(sg.tbase, T, (uint32_t)tile);
      tfirst = sg.tbase[t];
      lo = sg.pos[t] + (tile - tfirst) * kRadixTile;
      hi = min<int64_t>(sg.pos[t + 1], lo + kRadixTile);
      kb = (uint32_t)key_base[t];
    }
    const auto digit = [&](uint32_t key) -> uint32_t {
      if constexpr (SEG) return seg_digit(key, kb, shift);
      else if constexpr (MODE == kModeSkipped) return key == kKeyInvalid ? 1u : 0u;
      else return (key >> shift) & 255u;
    };
    const int64_t base = lo + (int64_t)wv * 64 * kRadixItems;
    uint32_t k[kRadixItems], v[kRadixItems], rank[kRadixItems];
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
      const int64_t p = base + i * 64 + lane;
      const bool valid = p < hi;
      k[i] = valid ? kin[p] : 0xFFFFFFFFu;
      v[i] = valid ? vin[p] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
      const int64_t p = base + i * 64 + lane;
      const bool valid = p < hi;
      const uint32_t d = digit(k[i]);
      const uint64_t peers = match_digit(d, valid);
      const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
      // the first lane of each digit adds the digit's lanes to the wave's count and
      // hands the old count to the others; a wave's LDS operations complete in issue
      // order, so each item sees the counts of the items before it, and the 16
      // atomics of a thread are in flight together
      uint32_t old = 0;
      if (valid && before == 0) old = atomicAdd(&wcnt[wv][d], (uint32_t)__popcll(peers));
      const int first = valid ? (int)__builtin_ctzll(peers) : lane;
      rank[i] = __shfl(old, first) + before;
    }
    __syncthreads();
    {
      const int d = threadIdx.x;
      uint32_t run = 0;
#pragma unroll
      for (int w = 0; w < kRadixWaves; ++w) {
        const uint32_t c = wcnt[w][d];
        wcnt[w][d] = run;
        run += c;
      }
      uint32_t* st = status + tile * 256 + d;
      uint32_t excl = 0;
      if (tile == tfirst) {
        status_store(st, kStPre | run);
      } else {
        status_store(st, kStAgg | run);
        int64_t j = tile - 1;
        uint32_t polls = 0;
        for (;;) {
          const uint32_t w = status_load(status + j * 256 + d);
          const uint32_t state = w & ~kStCount;
          if (state == 0) {
            if (++polls > kSortSpinLimit) {
              atomicOr(err, kErrSort);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
          }
          excl += w & kStCount;
          if (state == kStPre || j == tfirst) break;
          --j;
        }
        status_store(st, kStPre | (excl + run));
      }
      uint32_t tot;
      dpre[d] = block_exclusive_scan<uint32_t>(run, lds4, tot);
      if constexpr (MODE == kModeRuns) {
        const uint32_t runs = block_exclusive_scan<uint32_t>(sg.hist[((int64_t)t * kMaxPasses + pass) * 256 + d], lds4, tot);
        goff[d] = sg.pos[t] + runs + excl;
      } else {
        goff[d] = (SEG ? sg.base[((int64_t)t * kMaxPasses + pass) * 256 + d] : gbase[d]) + excl;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
      const int64_t p = base + i * 64 + lane;
      if (p < hi) {
        const uint32_t d = digit(k[i]);
        const uint32_t pos = dpre[d] + wcnt[wv][d] + rank[i];
        skey[pos] = k[i];
        sval[pos] = v[i];
      }
    }
    __syncthreads();
    const int cnt = (int)(hi - lo);
    for (int j = threadIdx.x; j < cnt; j += kRadixThreads) {
      const uint32_t key = skey[j];
      const uint32_t d = digit(key);
      const uint32_t g = goff[d] + (uint32_t)j - dpre[d];
      if ((int64_t)g < n) {  // always, unless a look-back gave up
        kout[g] = key;
        vout[g] = sval[j];
      }
    }
    if constexpr (!LOOP) break;
    __syncthreads();  // LDS is reused by the next tile
  }
  // the other status buffer (the previous pass's, finished) is cleared for the next pass
  if (next_status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < status_words; i += stride) next_status[i] = 0;
  }
}

// (src) -> (dst) pairs when *only_if is non-zero.
__global__ __launch_bounds__(256) void k_copy_pairs(const uint32_t* __restrict__ ks, const uint32_t* __restrict__ vs,
                                                    uint32_t* __restrict__ kd, uint32_t* __restrict__ vd, int64_t n,
                                                    const uint32_t* __restrict__ only_if) {
  if (*only_if == 0) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    kd[i] = ks[i];
    vd[i] = vs[i];
  }
}

// workgroups of a pass that loops over `tiles` tiles: no more than the device holds at once
template <int MODE>
unsigned pass_grid(int64_t tiles) {
  const int64_t r = resident_grid(reinterpret_cast<const void*>(k_sort_pass<MODE, true>), kRadixThreads);
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(tiles, r));
}

hipError_t sort_pairs(uint32_t* kA, uint32_t* vA, uint32_t* kB, uint32_t* vB, int64_t n, int passes,
                      const SortScratch& ss, int32_t* err, int* in_B, hipStream_t s) {
  *in_B = 0;
  if (n <= 0) return hipSuccess;
  if (passes < 1 || passes > kMaxPasses || n > (int64_t)kStCount) return hipErrorInvalidValue;
  const int64_t nb = (n + kRadixTile - 1) / kRadixTile;
  const int64_t sw = 256 * nb;
  k_sort_begin<<<1, 256, 0, s>>>(ss.ghist, ss.tickets);
  k_sort_hist<<<grid_for(n, 2048), 256, 0, s>>>(kA, n, passes, ss.ghist, ss.status[0], sw);
  k_sort_scan<<<1, 256, 0, s>>>(ss.ghist, ss.gbase, passes);
  for (int pass = 0; pass < passes; ++pass) {
    const uint32_t* ki = *in_B ? kB : kA;
    const uint32_t* vi = *in_B ? vB : vA;
    uint32_t* ko = *in_B ? kA : kB;
    uint32_t* vo = *in_B ? vA : vB;
    uint32_t* next = pass + 1 < passes ? ss.status[(pass + 1) & 1] : nullptr;
    k_sort_pass<kModeWhole, false><<<(unsigned)nb, kRadixThreads, 0, s>>>(ki, vi, ko, vo, n, 8 * pass, ss.gbase + 256 * pass,
                                                              ss.status[pass & 1], ss.tickets + pass, next, sw, err,
                                                              SegSort{}, nullptr, 0, pass, nullptr);
    *in_B = !*in_B;
  }
  return hipGetLastError();
}

hipError_t seg_begin(int64_t n, int passes, const int32_t* off, int32_t B, int T, const int64_t* key_base,
                     const unsigned long long* ctr, const SortScratch& ss, const SegSort& sg, ExpandHist* eh,
                     hipStream_t s) {
  if (n <= 0 || passes < 1 || passes >= kMaxPasses || n > (int64_t)kStCount || T < 1) return hipErrorInvalidValue;
  const int64_t hw = (int64_t)T * kMaxPasses * 256;
  k_seg_setup<<<(unsigned)std::min<int64_t>(64, (hw + 1023) / 1024), 256, 0, s>>>(off, B, T, n, ctr, sg, ss.ghist,
                                                                                 ss.tickets);
  eh->hist = sg.hist;
  eh->key_base = key_base;
  eh->n_skipped = ss.ghist;
  eh->status = ss.status[0];
  eh->status_words = 256 * ((n + kRadixTile - 1) / kRadixTile + T);
  eh->passes = passes;
  return hipGetLastError();
}

hipError_t sort_pairs_segmented(uint32_t* kA, uint32_t* vA, uint32_t* kB, uint32_t* vB, int64_t n, int passes,
                                const int32_t* off, int32_t B, int T, const int64_t* key_base,
                                const unsigned long long* ctr, const SortScratch& ss, const SegSort& sg, int32_t* err,
                                int* in_B, hipStream_t s) {
  *in_B = 0;
  if (n <= 0) return hipSuccess;
  if (passes < 1 || passes >= kMaxPasses || n > (int64_t)kStCount || T < 1) return hipErrorInvalidValue;
  const int64_t nb_max = (n + kRadixTile - 1) / kRadixTile + T;  // every segment adds at most one partial tile
  const int64_t sw = 256 * nb_max;
  uint32_t* n_skipped = ss.ghist;  // zeroed by k_seg_setup
  uint32_t* skip_base = ss.gbase;
  k_seg_scan<<<(unsigned)T, 256, 0, s>>>(sg, passes, n, n_skipped, skip_base);
  for (int pass = 0; pass < passes; ++pass) {
    const uint32_t* ki = *in_B ? kB : kA;
    const uint32_t* vi = *in_B ? vB : vA;
    uint32_t* ko = *in_B ? kA : kB;
    uint32_t* vo = *in_B ? vA : vB;
    // the last segmented pass clears the status words of the pass for skipped keys
    uint32_t* next = ss.status[(pass + 1) & 1];
    k_sort_pass<kModeSeg, false><<<(unsigned)nb_max, kRadixThreads, 0, s>>>(ki, vi, ko, vo, n, 8 * pass, nullptr,
                                                                 ss.status[pass & 1], ss.tickets + pass, next, sw,
                                                                 err, sg, key_base, T, pass, nullptr);
    *in_B = !*in_B;
  }
  // skipped keys behind every valid key, then back into the same buffer; both kernels
  // return at once when there is none
  uint32_t* kr = *in_B ? kB : kA;
  uint32_t* vr = *in_B ? vB : vA;
  uint32_t* ko = *in_B ? kA : kB;
  uint32_t* vo = *in_B ? vA : vB;
  const uint32_t* any_skipped = n_skipped;
  const int64_t nb = (n + kRadixTile - 1) / kRadixTile;
  k_sort_pass<kModeSkipped, true><<<pass_grid<kModeSkipped>(nb), kRadixThreads, 0, s>>>(kr, vr, ko, vo, n, 0, skip_base,
                                                            ss.status[passes & 1], ss.tickets + passes, nullptr,
                                                            256 * nb, err, SegSort{}, nullptr, 0, 0, any_skipped);
  k_copy_pairs<<<grid_for(n, 2048), 256, 0, s>>>(ko, vo, kr, vr, n, any_skipped);
  return hipGetLastError();
}

// ---- calls of moderate size ------------------------------------------------------------------
// The front of the step for a mid_call: the tables' segments are sorted by their local keys as
// in the segmented mode, and the unique rows, sets and jobs of a table are listed at
// offsets that follow from its first position (TabInfo), where the launches of a small call
// take them up.  Eight launches and no pass over all tables: a scan over the unique rows
// of all tables, a pass that moves skipped lookups behind every table's and the lists made from
// it cost twelve more, some 5 us each.
//   k_mid_begin    statistics, counts and tickets zeroed; offsets checked (a flag per
//                  workgroup); segments, first tiles
//   k_mid_expand   lookups -> (local key, bag), digit counts per table
//   k_sort_pass    the digit passes
//   k_mid_count    per tile of sorted keys: rows and sets that start in it
//   k_mid_write    their first occurrences, at the table's offset plus the tiles before
//   k_mid_rows     per unique row: the update's inputs, the jobs of the gradient sums
__global__ __launch_bounds__(256) void k_mid_begin(Dev dv, Work w, const int32_t* __restrict__ off, int32_t B, int64_t L,
                                                   SegSort sg, uint32_t* __restrict__ tickets,
                                                   uint32_t* __restrict__ flags) {
  __shared__ uint32_t lds4[4];
  zero_stats(dv, kStBwdLookups, kStHitEvictions);
  zero_stats(dv, kStInvalidBwd, kStInvalidBwd);
  const int T = dv.T;
  const int64_t stride = (int64_t)gridDim.x * 256, tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = tid; i < (int64_t)T * kMaxPasses * 256; i += stride) sg.hist[i] = 0;
  bool bad = false;
  for (int64_t i = tid; i < (int64_t)T * B; i += stride) {
    bad |= bad_range(off[i], off[i + 1], L);
  }
  bad = __syncthreads_or(bad) != 0;
  if (threadIdx.x == 0) {
    flags[blockIdx.x] = bad ? 1u : 0u;
    if (bad) atomicOr(dv.err, kErrOffsets);
  }
  if (blockIdx.x != 0) return;
  if (threadIdx.x < kMaxPasses) tickets[threadIdx.x] = 0;
  // (rejected offsets may give anything here; nothing uses it then)
  const auto start = [&](int t) -> int64_t { return min<int64_t>(max<int64_t>(off[(int64_t)t * B], 0), L); };
  uint32_t run = 0;
  for (int t0 = 0; t0 <= T; t0 += 256) {
    const int t = t0 + (int)threadIdx.x;
    uint32_t tiles = 0;
    int64_t p = 0;
    if (t <= T) {
      p = start(t);
      if (t < T) tiles = (uint32_t)((max<int64_t>(start(t + 1) - p, 0) + kRadixTile - 1) / kRadixTile);
    }
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<uint32_t>(tiles, lds4, tot);
    if (t <= T) {
      sg.pos[t] = (uint32_t)p;
      sg.tbase[t] = run + ex;
      if (t < T) w.tab_info[t] = TabInfo{.pos = (uint32_t)p};
    }
    run += tot;
  }
}

// WAVES waves of BPW bags each per workgroup (256 bags of one table): 64 bags per wave when
// there are many waves anyway, 16 when there are not (a wave goes through its bags' lookups
// 128 at a time).  A workgroup across a table boundary would add the second table's counts to
// memory one by one, on hot digits one after another: 42 us at 0.49M lookups instead of 14.
// A workgroup takes every per_table.d-th run of 256 bags of its table, so that a table has at
// most kMidExpand workgroups: each adds its digit counts to the table's, and with one
// workgroup per 256 bags those additions, to the same few addresses, were most of a call of
// 2M one-lookup bags (one table, 16 columns: 374 us, now 204).
constexpr int kMidExpand = 1024;
template <int WAVES, int BPW>
__global__ __launch_bounds__(WAVES * 64) void k_mid_expand(Dev dv, Work w, const int32_t* __restrict__ idx, int64_t L,
                                                           const int32_t* __restrict__ off, int32_t B,
                                                           DivConst per_table, const uint32_t* __restrict__ flags, int nflags,
                                                           uint32_t* __restrict__ bad_out, ExpandHist eh) {
  constexpr int NT = WAVES * 64;
  __shared__ uint32_t h[kMaxPasses * 256];
  __shared__ uint32_t skipped_s;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  {
    bool bad = false;
    for (int i = threadIdx.x; i < nflags; i += NT) bad |= flags[i] != 0;
    bad = __syncthreads_or(bad) != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      *bad_out = bad ? 1u : 0u;
      if (bad) w.tab_info[0].bad = 1;
    }
    if (bad) return;
  }
  const int64_t stride = (int64_t)gridDim.x * NT;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < eh.status_words; i += stride) eh.status[i] = 0;
  const int t = (int)div_by(blockIdx.x, per_table);
  const int64_t unit0 = blockIdx.x - (uint32_t)t * per_table.d;
  const TableDesc td = dv.desc[t];
  const int32_t* offt = off + (int64_t)t * B;
  for (int i = threadIdx.x; i < eh.passes * 256; i += NT) h[i] = 0;
  if (threadIdx.x == 0) skipped_s = 0;
  __syncthreads();
  uint32_t n_skip = 0;
  for (int64_t first = unit0 * 256 + wv * BPW; first < B; first += (int64_t)per_table.d * 256) {
    const int32_t bag0 = (int32_t)first;
    const int32_t lastbag = (int32_t)min<int64_t>(first + BPW, B);
    const int64_t st = lane < BPW && first + lane < B ? (int64_t)offt[bag0 + lane] : L;
    const int64_t P0 = offt[bag0], P1 = offt[lastbag];
    const auto handle = [&](int64_t p, int32_t r, int j) {
      uint32_t key = kKeyInvalid, local = kKeyInvalid;
      if (r >= 0 && (int64_t)r < td.N) {
        local = (uint32_t)r;
        if (td.n_sets > 0) {
          const uint32_t q = div_by((uint32_t)r, td.by_sets);
          local = ((uint32_t)r - q * (uint32_t)td.n_sets) * (uint32_t)td.Q + q;
        }
        key = (uint32_t)td.key_base + local;
      } else {
        ++n_skip;
      }
      w.keysA[p] = key;
      w.valsA[p] = (uint32_t)(bag0 + j);
      for (int q = 0; q < eh.passes; ++q) atomicAdd(&h[q * 256 + ((local >> (8 * q)) & 255u)], 1u);
    };
    for (int64_t pc = P0; pc < P1; pc += 128) {
      const int64_t pA = pc + lane, pB = pc + 64 + lane;
      const bool inA = pA < P1, inB = pB < P1;
      const int32_t rA = inA ? idx[pA] : 0;
      const int32_t rB = inB ? idx[pB] : 0;
      int jA = 0, jB = 0;
#pragma unroll
      for (int step = BPW / 2; step >= 1; step >>= 1) {
        const int64_t sA = __shfl(st, jA + step);
        const int64_t sB = __shfl(st, jB + step);
        if (sA <= pA) jA += step;
        if (sB <= pB) jB += step;
      }
      if (inA) handle(pA, rA, jA);
      if (inB) handle(pB, rB, jB);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) n_skip += __shfl_xor(n_skip, o);
  if (lane == 0 && n_skip) atomicAdd(&skipped_s, n_skip);
  __syncthreads();
  uint32_t* ht = eh.hist + (int64_t)t * kMaxPasses * 256;
  for (int i = threadIdx.x; i < eh.passes * 256; i += NT) {
    const uint32_t c = h[i];
    if (c) atomicAdd(&ht[i], c);
  }
  if (threadIdx.x == 0 && skipped_s) atomicAdd(&w.tab_info[t].skipped, skipped_s);
}

// The sorted keys of tile `tile`: its table, its first position and the end of its valid keys.
struct MidTile {
  int t;
  uint32_t lo, hi, tfirst, pos, nv;
};
__device__ __forceinline__ MidTile mid_tile(const Work& w, const SegSort& sg, int T, uint32_t tile) {
  MidTile m;
  m.t = seg_of_tile_wave(sg.tbase, T, tile);
  m.tfirst = sg.tbase[m.t];
  m.pos = sg.pos[m.t];
  const uint32_t n = sg.pos[m.t + 1] - m.pos;
  m.nv = n - w.tab_info[m.t].skipped;  // skipped lookups end the segment
  m.lo = min(m.pos + (tile - m.tfirst) * (uint32_t)kRadixTile, m.pos + m.nv);
  m.hi = min(m.lo + (uint32_t)kRadixTile, m.pos + m.nv);
  return m;
}

// Which of the thread's 16 keys (wave-major runs of 64) start a row or a set.
__device__ __forceinline__ void mid_starts(const Dev& dv, const TableDesc& td, const uint32_t* __restrict__ sk,
                                           const MidTile& m, uint32_t& rows, uint32_t& sets) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  rows = sets = 0;
  uint32_t k[kRadixItems], q[kRadixItems];
#pragma unroll
  for (int i = 0; i < kRadixItems; ++i) {
    const uint32_t e = m.lo + (uint32_t)(wv * 64 * kRadixItems + i * 64 + lane);
    k[i] = e < m.hi ? sk[e] : 0u;
    q[i] = e < m.hi && e > m.pos ? sk[e - 1] : kKeyInvalid;
  }
  const uint32_t kb = (uint32_t)td.key_base;
#pragma unroll
  for (int i = 0; i < kRadixItems; ++i) {
    const uint32_t e = m.lo + (uint32_t)(wv * 64 * kRadixItems + i * 64 + lane);
    const bool row = e < m.hi && k[i] != q[i];
    const bool set = row && (e == m.pos || div_by(k[i] - kb, td.by_Q) != div_by(q[i] - kb, td.by_Q));
    rows |= (row ? 1u : 0u) << i;
    sets |= (set ? 1u : 0u) << i;
  }
}

__global__ __launch_bounds__(256) void k_mid_count(Dev dv, Work w, const uint32_t* __restrict__ sk, SegSort sg,
                                                   const uint32_t* __restrict__ bad) {
  __shared__ unsigned long long lds4[4];
  if (*bad != 0 || blockIdx.x >= sg.tbase[dv.T]) return;
  const MidTile m = mid_tile(w, sg, dv.T, blockIdx.x);
  uint32_t rows, sets;
  mid_starts(dv, dv.desc[m.t], sk, m, rows, sets);
  unsigned long long tot;
  block_exclusive_scan<unsigned long long>(
      (unsigned long long)__popc(rows) | ((unsigned long long)__popc(sets) << 32), lds4, tot);
  if (threadIdx.x == 0) w.tile_cnt[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_mid_write(Dev dv, Work w, const uint32_t* __restrict__ sk, SegSort sg,
                                                   const uint32_t* __restrict__ bad, int group) {
  __shared__ unsigned long long lds4[4];
  __shared__ uint32_t run_rows[4 * kRadixItems], run_sets[4 * kRadixItems];
  if (*bad != 0 || blockIdx.x >= sg.tbase[dv.T]) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const MidTile m = mid_tile(w, sg, dv.T, blockIdx.x);
  const TableDesc td = dv.desc[m.t];
  // the rows and sets of the table's tiles before this one
  unsigned long long c = 0, before;
  for (uint32_t j = m.tfirst + threadIdx.x; j < blockIdx.x; j += 256) c += w.tile_cnt[j];
  block_exclusive_scan<unsigned long long>(c, lds4, before);
  uint32_t rows, sets;
  mid_starts(dv, td, sk, m, rows, sets);
#pragma unroll
  for (int i = 0; i < kRadixItems; ++i) {
    const uint64_t br = __ballot((rows >> i) & 1u), bs = __ballot((sets >> i) & 1u);
    if (lane == 0) {
      run_rows[wv * kRadixItems + i] = (uint32_t)__popcll(br);
      run_sets[wv * kRadixItems + i] = (uint32_t)__popcll(bs);
    }
  }
  __syncthreads();
  unsigned long long tot;
  const int r = threadIdx.x;
  const unsigned long long ex = block_exclusive_scan<unsigned long long>(
      r < 4 * kRadixItems ? (unsigned long long)run_rows[r] | ((unsigned long long)run_sets[r] << 32) : 0ull, lds4, tot);
  if (r < 4 * kRadixItems) {
    run_rows[r] = (uint32_t)(before + ex);
    run_sets[r] = (uint32_t)((before + ex) >> 32);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kRadixItems; ++i) {
    const bool row = (rows >> i) & 1u, set = (sets >> i) & 1u;
    const uint64_t br = __ballot(row), bs = __ballot(set);
    const uint32_t e = m.lo + (uint32_t)(wv * 64 * kRadixItems + i * 64 + lane);
    const uint32_t u = m.pos + run_rows[wv * kRadixItems + i] + (uint32_t)__popcll(br & lanemask_lt());
    if (row) w.seg[u] = e;
    if (set && td.n_sets > 0) {
      const uint32_t s = m.pos + run_sets[wv * kRadixItems + i] + (uint32_t)__popcll(bs & lanemask_lt());
      w.set_first[s] = u;
      w.nch[s] = div_by(sk[e] - (uint32_t)td.key_base, td.by_Q);
    }
  }
  // the table's last tile knows its totals
  if (threadIdx.x == 0 && blockIdx.x + 1 == sg.tbase[m.t + 1]) {
    const uint32_t nU = (uint32_t)(before + tot);
    TabInfo& ti = w.tab_info[m.t];
    ti.rows = nU;
    ti.sets = td.n_sets > 0 ? (uint32_t)((before + tot) >> 32) : (nU + (uint32_t)group - 1) / (uint32_t)group;
    ti.valid = m.nv;
    unsigned long long* st = dv.stats + ((int64_t)m.t << dv.stat_shift) * kStatStride;
    st[kStBwdLookups] = m.nv;
    st[kStInvalidBwd] = ti.skipped;
    st[kStUnique] = nU;
    if (td.n_sets == 0) st[kStBypasses] = nU;
    if (ti.skipped) atomicOr(dv.err, kErrIndex);
  }
}

hipError_t launch_mid_front(const Dev& d, const Work& w, const int32_t* idx, int64_t L, const int32_t* off, int32_t B,
                            int passes, int group, const uint32_t** keys, const uint32_t** sval, hipStream_t s) {
  if (L <= 0 || passes < 1 || passes > kMaxPasses || L > (int64_t)kStCount || d.T < 1 || B < 1)
    return hipErrorInvalidValue;
  const int64_t nbags = (int64_t)d.T * B;
  const SortScratch ss{w.sort_small, w.sort_small + kMaxPasses * 256, w.sort_small + 2 * kMaxPasses * 256,
                       {w.sort_status[0], w.sort_status[1]}};
  const size_t TT = (size_t)d.T * kMaxPasses * 256;
  const SegSort sg{w.sort_seg, w.sort_seg + (d.T + 1), w.sort_seg + 2 * (d.T + 1), w.sort_seg + 2 * (d.T + 1) + TT};
  uint32_t* flags = ss.ghist;        // one per workgroup of k_mid_begin
  uint32_t* bad_flag = ss.gbase;
  const unsigned nflags = grid_for(std::max<int64_t>(nbags / 4, (int64_t)TT / 4), 256);
  const int64_t tiles = (L + kRadixTile - 1) / kRadixTile + d.T;
  ExpandHist eh;
  eh.hist = sg.hist;
  eh.key_base = d.key_base;
  eh.status = ss.status[0];
  eh.status_words = 256 * tiles;
  eh.passes = passes;
  k_mid_begin<<<nflags, 256, 0, s>>>(d, w, off, B, L, sg, ss.tickets, flags);
  const DivConst per_table = div_const(
      (uint32_t)std::min<int64_t>(((int64_t)B + 255) / 256, kMidExpand));
  const unsigned wgs = per_table.d * (unsigned)d.T;
  if (nbags < (int64_t)64 * kMidWaves)
    k_mid_expand<16, 16><<<wgs, 1024, 0, s>>>(d, w, idx, L, off, B, per_table, flags, (int)nflags, bad_flag, eh);
  else
    k_mid_expand<4, 64><<<wgs, 256, 0, s>>>(d, w, idx, L, off, B, per_table, flags, (int)nflags, bad_flag, eh);
  uint32_t *ki = w.keysA, *vi = w.valsA, *ko = w.keysB, *vo = w.valsB;
  for (int p = 0; p < passes; ++p) {
    uint32_t* next = p + 1 < passes ? ss.status[(p + 1) & 1] : nullptr;
    k_sort_pass<kModeRuns, false><<<(unsigned)tiles, kRadixThreads, 0, s>>>(
        ki, vi, ko, vo, L, 8 * p, nullptr, ss.status[p & 1], ss.tickets + p, next, eh.status_words, d.err, sg, d.key_base,
        d.T, p, bad_flag);
    std::swap(ki, ko);
    std::swap(vi, vo);
  }
  k_mid_count<<<(unsigned)tiles, 256, 0, s>>>(d, w, ki, sg, bad_flag);
  k_mid_write<<<(unsigned)tiles, 256, 0, s>>>(d, w, ki, sg, bad_flag, group);
  *sval = vi;
  *keys = ki;
  return hipGetLastError();
}

// ---- lookups -> sort pairs ----------------------------------------------------------------
// One wave per 64 consecutive bags (global bag = t*B + b); each position of those
// bags finds its bag by a binary search over the 64 lane-held bag starts.
// key: set-major row key (kKeyInvalid for an out-of-range row); value: the bag b
// within its table (its gradient row in grad_out [B][T][d] is b*T + t).
// With SEG (the per-table sort mode) the expansion also does the counting of that mode,
// from the keys it forms rather than from a second read of them: per table, the digit
// counts of every pass of the local key (255 in every digit for a skipped key), the
// number of skipped keys, and the cleared status words of the first pass.  A
// workgroup gathers the counts of its first bag's table in LDS and adds them once; a
// key of another table (a workgroup across a table boundary) is added directly.
// Positions outside every bag belong to the first table's segment (before the first
// bag) or the last one's (after the last bag), as the segment starts place them.
template <bool SEG>
__global__ __launch_bounds__(256) void k_expand(Dev dv, const int32_t* __restrict__ idx, int64_t L,
                                                const int32_t* __restrict__ off, int32_t B, DivConst byB,
                                                uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                int64_t nbag_waves, int64_t bag_blocks,
                                                const unsigned long long* __restrict__ ctr, ExpandHist eh) {
  __shared__ uint32_t h[SEG ? kMaxPasses * 256 : 1];
  __shared__ uint32_t skipped_s;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t nbags = (int64_t)dv.T * B;
  if constexpr (SEG) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < eh.status_words; i += stride)
      eh.status[i] = 0;
  }
  if (ctr[kCBadOffsets]) {
    // offsets failed validation: every lookup of the step is skipped (and the whole
    // stream is the first table's segment)
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < L; p += stride)
      keys[p] = kKeyInvalid, vals[p] = 0;
    if constexpr (SEG) {
      if (blockIdx.x == 0 && threadIdx.x == 0 && L > 0) {
        for (int p = 0; p < eh.passes; ++p) atomicAdd(&eh.hist[p * 256 + 255], (uint32_t)L);
        atomicAdd(eh.n_skipped, (uint32_t)L);
      }
    }
    return;
  }
  if ((int64_t)blockIdx.x >= bag_blocks) {
    // positions outside every bag: [0, off[0]) and [off[nbags], L)
    const int64_t head = min<int64_t>(max<int64_t>(off[0], 0), L);
    const int64_t tail = min<int64_t>(max<int64_t>(off[nbags], head), L);
    const int64_t tid = ((int64_t)blockIdx.x - bag_blocks) * blockDim.x + threadIdx.x;
    const int64_t stride = ((int64_t)gridDim.x - bag_blocks) * blockDim.x;
    for (int64_t p = tid; p < head; p += stride) keys[p] = kKeyInvalid, vals[p] = 0;
    for (int64_t p = tail + tid; p < L; p += stride) keys[p] = kKeyInvalid, vals[p] = 0;
    if constexpr (SEG) {
      if (tid == 0 && head + (L - tail) > 0) {
        const int64_t last = (int64_t)(dv.T - 1) * kMaxPasses * 256;
        for (int p = 0; p < eh.passes; ++p) {
          if (head) atomicAdd(&eh.hist[p * 256 + 255], (uint32_t)head);
          if (L - tail) atomicAdd(&eh.hist[last + p * 256 + 255], (uint32_t)(L - tail));
        }
        atomicAdd(eh.n_skipped, (uint32_t)(head + (L - tail)));
      }
    }
    return;
  }
  // the table whose counts this workgroup gathers in LDS: that of its first bag
  const int t_wg = (int)div_by((uint32_t)((int64_t)blockIdx.x * 256), byB);
  uint32_t kb_wg = 0;
  if constexpr (SEG) {
    kb_wg = (uint32_t)eh.key_base[t_wg];
    for (int i = threadIdx.x; i < kMaxPasses * 256; i += 256) h[i] = 0;
    if (threadIdx.x == 0) skipped_s = 0;
    __syncthreads();
  }
  uint32_t n_skip = 0;
  const int64_t bw = (int64_t)blockIdx.x * 4 + wv;
  if (bw < nbag_waves) {
    const int64_t bag0 = bw * 64;
    const int64_t mybag = bag0 + lane;
    const int64_t lastbag = min<int64_t>(bag0 + 64, nbags);
    int64_t st = L;
    if (mybag < nbags) st = min<int64_t>(max<int64_t>(off[mybag], 0), L);
    const int64_t P0 = min<int64_t>(max<int64_t>(off[bag0], 0), L);
    const int64_t P1 = min<int64_t>(max<int64_t>(off[lastbag], P0), L);
    uint32_t n_ok = 0, n_bad = 0;
    // global bags are below 2^32 (checked when the handle is created): their table by
    // one high multiply; the descriptor of the wave's first table is loaded once
    const int t_run = (int)div_by((uint32_t)bag0, byB);
    const TableDesc td_run = dv.desc[t_run];
    const auto handle = [&](int64_t p, int32_t r, int j) {
      const uint32_t bag = (uint32_t)(bag0 + j);
      const int t = (int)div_by(bag, byB);
      const int b = (int)(bag - (uint32_t)t * (uint32_t)B);
      const TableDesc td = t == t_run ? td_run : dv.desc[t];
      uint32_t key = kKeyInvalid;
      if (r >= 0 && (int64_t)r < td.N) {
        if (td.n_sets > 0) {
          const uint32_t q = div_by((uint32_t)r, td.by_sets);
          const uint32_t set = (uint32_t)r - q * (uint32_t)td.n_sets;
          key = (uint32_t)(td.key_base + (int64_t)set * td.Q + q);
        } else {
          key = (uint32_t)(td.key_base + r);
        }
        if (t == t_run) ++n_ok; else atomicAdd(stat_of(dv, t) + kStBwdLookups, 1ull);
      } else {
        if (t == t_run) ++n_bad; else atomicAdd(stat_of(dv, t) + kStInvalidBwd, 1ull);
        atomicOr(dv.err, kErrIndex);
      }
      keys[p] = key;
      vals[p] = (uint32_t)b;
      if constexpr (SEG) {
        n_skip += key == kKeyInvalid;
        if (t == t_wg) {
          for (int q = 0; q < eh.passes; ++q) atomicAdd(&h[q * 256 + seg_digit(key, kb_wg, 8 * q)], 1u);
        } else {
          const uint32_t kb = (uint32_t)eh.key_base[t];
          uint32_t* ht = eh.hist + (int64_t)t * kMaxPasses * 256;
          for (int q = 0; q < eh.passes; ++q) atomicAdd(&ht[q * 256 + seg_digit(key, kb, 8 * q)], 1u);
        }
      }
    };
    // two runs of 64 positions at a time: their index loads and bag searches interleave
    for (int64_t pc = P0; pc < P1; pc += 128) {
      const int64_t pA = pc + lane, pB = pc + 64 + lane;
      const bool inA = pA < P1, inB = pB < P1;
      const int32_t rA = inA ? idx[pA] : 0;
      const int32_t rB = inB ? idx[pB] : 0;
      int jA = 0, jB = 0;
#pragma unroll
      for (int step = 32; step >= 1; step >>= 1) {
        const int64_t sA = __shfl(st, jA + step);
        const int64_t sB = __shfl(st, jB + step);
        if (jA + step < 64 && sA <= pA) jA += step;
        if (jB + step < 64 && sB <= pB) jB += step;
      }
      if (inA) handle(pA, rA, jA);
      if (inB) handle(pB, rB, jB);
    }
    // lookups of the wave's first table: one atomic per wave
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      n_ok += __shfl_xor(n_ok, o);
      n_bad += __shfl_xor(n_bad, o);
    }
    if (lane == 0 && n_ok) atomicAdd(stat_of(dv, t_run) + kStBwdLookups, (unsigned long long)n_ok);
    if (lane == 0 && n_bad) atomicAdd(stat_of(dv, t_run) + kStInvalidBwd, (unsigned long long)n_bad);
  }
  if constexpr (SEG) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) n_skip += __shfl_xor(n_skip, o);
    if (lane == 0 && n_skip) atomicAdd(&skipped_s, n_skip);
    __syncthreads();
    uint32_t* ht = eh.hist + (int64_t)t_wg * kMaxPasses * 256;
    for (int i = threadIdx.x; i < eh.passes * 256; i += 256) {
      const uint32_t c = h[i];
      if (c) atomicAdd(&ht[i], c);
    }
    if (threadIdx.x == 0 && skipped_s) atomicAdd(eh.n_skipped, skipped_s);
  }
}

__global__ __launch_bounds__(256) void k_check_offsets(Dev dv, const int32_t* __restrict__ off, int64_t nbags,
                                                       int64_t L, unsigned long long* __restrict__ ctr) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nbags; i += stride) {
    if (bad_range(off[i], off[i + 1], L)) {
      ctr[kCBadOffsets] = 1;
      atomicOr(dv.err, kErrOffsets);
    }
  }
}

hipError_t launch_expand(const Dev& dv, const int32_t* idx, int64_t L, const int32_t* off, int32_t B, uint32_t* keys,
                         uint32_t* vals, unsigned long long* ctr, const ExpandHist* eh, hipStream_t s) {
  const int64_t nbags = (int64_t)dv.T * B;
  const int64_t nbag_waves = (nbags + 63) / 64;
  const int64_t bag_blocks = (nbag_waves + 3) / 4;
  const int64_t tail_blocks = 16;
  const DivConst byB = div_const(B > 0 ? (uint32_t)B : 1u);  // no bag when B = 0
  const unsigned grid = (unsigned)(bag_blocks + tail_blocks);
  if (eh) {
    k_expand<true><<<grid, 256, 0, s>>>(dv, idx, L, off, B, byB, keys, vals, nbag_waves, bag_blocks, ctr, *eh);
  } else {
    k_expand<false><<<grid, 256, 0, s>>>(dv, idx, L, off, B, byB, keys, vals, nbag_waves, bag_blocks, ctr,
                                         ExpandHist{});
  }
  return hipGetLastError();
}

// ---- unique rows and touched sets ---------------------------------------------------------
// A row start is a valid key that differs from its predecessor in the sorted stream; a
// set start is a row start of a cached table whose (table, set) differs from the
// predecessor's.  Two passes over tiles of kUqTile keys: k_uniq_count writes each tile's
// counts packed as (sets << 32 | rows); after their exclusive scan, k_uniq_write writes
// every start at its tile's offset plus its rank inside the tile: the key and first
// occurrence of each unique row, and the first unique row of each touched set.  A wave takes
// runs of 64 consecutive keys, so that loads are whole lines and a start's rank is a ballot
// (16 consecutive keys per thread: 75 + 98 us on the 49M keys of the industrial workload,
// against 70 + 79; 23 -> 13 us for the write on 4.2M keys of one table).
constexpr int kUqPer = 16;
constexpr int kUqTile = 256 * kUqPer;

size_t uniq_tile_words(int64_t n) { return (size_t)((n + kUqTile - 1) / kUqTile + 1); }

// The starts among the wave's kUqPer runs of keys from e0 on: calls on_run(i, key, row, set,
// table) per run i, for every lane.  Skipped keys end the stream, and the first of them is
// its valid length.
template <typename F>
__device__ __forceinline__ void uniq_runs(const Dev& dv, const uint32_t* __restrict__ sk, int64_t n, int64_t e0,
                                          unsigned long long* valid_out, F&& on_run) {
  const int lane = threadIdx.x & 63;
  uint32_t k[kUqPer], q[kUqPer];
#pragma unroll
  for (int i = 0; i < kUqPer; ++i) {
    const int64_t e = e0 + i * 64 + lane;
    k[i] = e < n ? sk[e] : kKeyInvalid;
    q[i] = e < n && e > 0 ? sk[e - 1] : kKeyInvalid;
  }
  // the table of the run's first key (wave-uniform), its key range and set stride
  int t = -1;
  uint32_t kb = 0, kb_next = 0;
  DivConst byQ;
  bool cached = false;
#pragma unroll
  for (int i = 0; i < kUqPer; ++i) {
    const int64_t e = e0 + i * 64 + lane;
    const bool ok = k[i] != kKeyInvalid;
    if (valid_out && !ok && e < n && (e == 0 || q[i] != kKeyInvalid)) *valid_out = (unsigned long long)e;
    const uint32_t k0 = __builtin_amdgcn_readfirstlane(k[i]);
    bool row = false, set = false;
    int tl = t;
    if (k0 != kKeyInvalid) {  // whole wave (else no key of the run is valid)
      if (t < 0 || k0 >= kb_next) {
        if (t < 0) t = table_of_key(dv.key_base, dv.T, k0);
        while ((int64_t)k0 >= dv.key_base[t + 1]) ++t;
        t = __builtin_amdgcn_readfirstlane(t);
        const TableDesc& td = dv.desc[t];
        kb = (uint32_t)td.key_base;
        kb_next = (uint32_t)dv.key_base[t + 1];
        byQ = td.by_Q;
        cached = td.n_sets > 0;
      }
      tl = t;
      row = ok && (e == 0 || k[i] != q[i]);
      if (row) {
        uint32_t b = kb;
        DivConst by = byQ;
        bool c = cached;
        if (k[i] >= kb_next) {  // a later table's key in the run
          do ++tl; while ((int64_t)k[i] >= dv.key_base[tl + 1]);
          const TableDesc& td = dv.desc[tl];
          b = (uint32_t)td.key_base;
          by = td.by_Q;
          c = td.n_sets > 0;
        }
        set = c && (e == 0 || q[i] < b || div_by(k[i] - b, by) != div_by(q[i] - b, by));
      }
    }
    on_run(i, k[i], row, set, tl);
  }
}

__global__ __launch_bounds__(256) void k_uniq_count(Dev dv, const uint32_t* __restrict__ sk, int64_t n,
                                                    unsigned long long* __restrict__ tile_cnt,
                                                    unsigned long long* __restrict__ ctr) {
  __shared__ unsigned long long lds4[4];
  const int wv = threadIdx.x >> 6;
  const int64_t e0 = (int64_t)blockIdx.x * kUqTile + (int64_t)wv * 64 * kUqPer;
  uint32_t rows = 0, sets = 0;  // of the wave
  uniq_runs(dv, sk, n, e0, ctr + kCValid, [&](int, uint32_t, bool row, bool set, int) {
    rows += (uint32_t)__popcll(__ballot(row));
    sets += (uint32_t)__popcll(__ballot(set));
  });
  if ((threadIdx.x & 63) == 0) lds4[wv] = (unsigned long long)rows | ((unsigned long long)sets << 32);
  __syncthreads();
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = lds4[0] + lds4[1] + lds4[2] + lds4[3];
}

__global__ __launch_bounds__(256) void k_uniq_write(Dev dv, const uint32_t* __restrict__ sk, int64_t n,
                                                    const unsigned long long* __restrict__ tile_pre,
                                                    uint32_t* __restrict__ uk, uint32_t* __restrict__ seg,
                                                    uint32_t* __restrict__ set_first, int32_t* __restrict__ utab,
                                                    unsigned long long* __restrict__ ctr) {
  __shared__ unsigned long long lds4[4];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const unsigned long long tot = ctr[kCScanTotal];
    const uint32_t nu = (uint32_t)(tot & 0xFFFFFFFFull), ns = (uint32_t)(tot >> 32);
    ctr[kCUnique] = nu;
    ctr[kCSets] = ns;
    seg[nu] = (uint32_t)ctr[kCValid];
    set_first[ns] = nu;
  }
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t e0 = (int64_t)blockIdx.x * kUqTile + (int64_t)wv * 64 * kUqPer;
  uint64_t br[kUqPer], bs[kUqPer];
  uint32_t key[kUqPer];
  int tab[kUqPer];
  uint32_t rows = 0, sets = 0;
  uniq_runs(dv, sk, n, e0, nullptr, [&](int i, uint32_t k, bool row, bool set, int t) {
    br[i] = __ballot(row);
    bs[i] = __ballot(set);
    rows += (uint32_t)__popcll(br[i]);
    sets += (uint32_t)__popcll(bs[i]);
    key[i] = k;
    tab[i] = t;
  });
  if (lane == 0) lds4[wv] = (unsigned long long)rows | ((unsigned long long)sets << 32);
  __syncthreads();
  unsigned long long base = tile_pre[blockIdx.x];
  for (int w = 0; w < wv; ++w) base += lds4[w];
  uint32_t u0 = (uint32_t)base, s0 = (uint32_t)(base >> 32);
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int i = 0; i < kUqPer; ++i) {
    const uint32_t u = u0 + (uint32_t)__popcll(br[i] & lt);
    if ((br[i] >> lane) & 1) {
      uk[u] = key[i];
      seg[u] = (uint32_t)(e0 + i * 64 + lane);
      utab[u] = tab[i];
    }
    if ((bs[i] >> lane) & 1) set_first[s0 + (uint32_t)__popcll(bs[i] & lt)] = u;
    u0 += (uint32_t)__popcll(br[i]);
    s0 += (uint32_t)__popcll(bs[i]);
  }
}

hipError_t launch_unique(const Dev& dv, const uint32_t* sk, int64_t n, unsigned long long* tile_cnt,
                         unsigned long long* tile_pre, uint32_t* uk, uint32_t* seg,
                         uint32_t* set_first, int32_t* utab, unsigned long long* ctr,
                         hipStream_t s) {
  const int64_t tiles = (n + kUqTile - 1) / kUqTile;
  if (tiles > 0) k_uniq_count<<<(unsigned)tiles, 256, 0, s>>>(dv, sk, n, tile_cnt, ctr);
  k_scan_one<unsigned long long><<<1, kScanThreads, 0, s>>>(tile_cnt, tile_pre, tiles, ctr + kCScanTotal);
  k_uniq_write<<<(unsigned)(tiles > 0 ? tiles : 1), 256, 0, s>>>(dv, sk, n, tile_pre, uk, seg,
                                                                 set_first, utab, ctr);
  return hipGetLastError();
}

}  // namespace embc
