// Backward + sparse update of a small call in three launches instead of about 27 (and the
// launches of a mid call after its sort, k_sort.hip):
//   k_front    one workgroup per table: offsets checked, lookups expanded, sorted in LDS, the
//              unique rows, touched sets and gradient-sum jobs listed
//   k_decide   replacement decisions per touched set (the probe included) and, by other
//              workgroups of the same launch, the gradient sums of rows with many lookups
//   k_apply    per unique row: merged gradient, fetch, optimizer, write-back; an insert
//              first writes the resident it displaces back to T
// (k_fold before k_apply when a row's block sums are many; k_mid_rows in place of the last part
// of k_front in a mid call).
// A launch that waits for the one before costs about 5 us on the device whatever it does, so
// a step of a few thousand lookups is as long as its number of launches.  Tables are
// independent and a table's unique rows, sets and jobs are listed at offsets that follow
// from its first lookup's position (every list is shorter than its share of the lookups),
// so no scan over all tables is needed between the kernels.
// The results are those of the general path bit for bit: same order of sums, same decisions.
#include <algorithm>

#include "embc_device.h"
#include "embc_dispatch.h"
#include "embc_offsets.h"
#include "embc_row.h"

namespace embc {

constexpr int kFrontThreads = 1024;
constexpr int kFrontWaves = kFrontThreads / 64;
// Keys per thread of a table sorted in LDS, at most (8 bytes each with their values), and of
// a tile of a larger one, whose pairs are in memory.  (With 16 the kernel spills registers;
// scratch memory alone adds 3 to 14 us to its launch.)
constexpr int kFrontItems = 8;
constexpr int kFrontTile = kFrontThreads * kFrontItems;

// ---- block scans of k_front ------------------------------------------------------------------
template <typename T, typename Op>
__device__ __forceinline__ T front_scan_exclusive(T v, T zero, T* lds, T& total, Op op) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o);
    if (lane >= o) x = op(y, x);
  }
  if (lane == 63) lds[wv] = x;
  __syncthreads();
  T pre = zero;
  total = zero;
#pragma unroll
  for (int w = 0; w < kFrontWaves; ++w) {
    const T s = lds[w];
    if (w < wv) pre = op(pre, s);
    total = op(total, s);
  }
  __syncthreads();
  T e = __shfl_up(x, 1);
  if (lane == 0) e = zero;
  return op(pre, e);
}

struct FrontLds {
  uint32_t key[kFrontTile];
  uint32_t val[kFrontTile];
  uint32_t cnt[kFrontWaves][256];  // digit counts of each wave, then its offsets
  uint32_t dpre[256];
  uint32_t hist[kMaxPasses][256];  // a table in memory: digit counts of every pass, then the digits' ends
  unsigned long long scan[kFrontWaves];
  uint32_t rows[kFrontItems * kFrontWaves], sets[kFrontItems * kFrontWaves];  // starts per run of 64 keys
  uint32_t n_bad, n_chunk, n_big, n_window;
};

// Ranks of ITEMS keys per thread (wave-major order: item i of wave w is key w*64*ITEMS +
// i*64 + lane) among the wave's keys of the same digit; leaves the wave's digit counts in
// S.cnt.  A wave's LDS operations complete in order, so its row needs no barrier.
template <int ITEMS>
__device__ __forceinline__ void front_rank(FrontLds& S, const uint32_t (&k)[ITEMS], uint32_t n, int shift,
                                           uint32_t (&rank)[ITEMS]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = lane; i < 256; i += 64) S.cnt[wv][i] = 0;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool valid = (uint32_t)(wv * 64 * ITEMS + i * 64 + lane) < n;
    const uint32_t d = (k[i] >> shift) & 255u;
    const uint64_t peers = match_digit(d, valid);
    const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
    uint32_t old = 0;
    if (valid && before == 0) old = atomicAdd(&S.cnt[wv][d], (uint32_t)__popcll(peers));
    const int first = valid ? (int)__builtin_ctzll(peers) : lane;
    rank[i] = __shfl(old, first) + before;
  }
}

// After a barrier: the waves' digit counts become offsets inside their digit (S.cnt), and
// returns, in threads below 256, the digit's total.
__device__ __forceinline__ uint32_t front_wave_offsets(FrontLds& S) {
  uint32_t run = 0;
  if (threadIdx.x < 256) {
#pragma unroll
    for (int w = 0; w < kFrontWaves; ++w) {
      const uint32_t c = S.cnt[w][threadIdx.x];
      S.cnt[w][threadIdx.x] = run;
      run += c;
    }
  }
  return run;
}

// Stable sort of n <= 1024*ITEMS pairs (k, v) in wave-major order by `passes` 8-bit digits;
// the sorted keys are left in S.key, the values in vout.
template <int ITEMS>
__device__ __forceinline__ void front_sort(FrontLds& S, uint32_t (&k)[ITEMS], uint32_t (&v)[ITEMS], uint32_t n,
                                           int passes, uint32_t* __restrict__ vout) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int p = 0; p < passes; ++p) {
    uint32_t rank[ITEMS];
    if (p > 0) {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const uint32_t e = (uint32_t)(wv * 64 * ITEMS + i * 64 + lane);
        k[i] = e < n ? S.key[e] : 0u;
        v[i] = e < n ? S.val[e] : 0u;
      }
    }
    front_rank<ITEMS>(S, k, n, 8 * p, rank);
    __syncthreads();
    const uint32_t tot = front_wave_offsets(S);
    unsigned long long all;
    const unsigned long long pre = front_scan_exclusive<unsigned long long>(
        threadIdx.x < 256 ? tot : 0u, 0ull, S.scan, all, [](unsigned long long a, unsigned long long b) { return a + b; });
    if (threadIdx.x < 256) S.dpre[threadIdx.x] = (uint32_t)pre;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if ((uint32_t)(wv * 64 * ITEMS + i * 64 + lane) < n) {
        const uint32_t d = (k[i] >> (8 * p)) & 255u;
        const uint32_t at = S.dpre[d] + S.cnt[wv][d] + rank[i];
        S.key[at] = k[i];
        if (p + 1 < passes) S.val[at] = v[i];
        else vout[at] = v[i];
      }
    }
    __syncthreads();
  }
}

// The windows of the lanes' big rows (big: the lane has one, row h, whose lookups are [s0, s1) of
// the sorted stream; its windows go from entry `at` on), by the whole wave: one lane alone
// would write the hundreds of a hot row one after another.
__device__ __forceinline__ void put_windows(const Work& w, bool big, uint32_t at, uint32_t h, uint32_t s0, uint32_t s1,
                                            int nblk) {
  for (uint64_t m = __ballot(big); m; m &= m - 1) {
    const int src = (int)__builtin_ctzll(m);
    const uint32_t a = __builtin_amdgcn_readlane(at, src), row = __builtin_amdgcn_readlane(h, src);
    const uint32_t b0 = __builtin_amdgcn_readlane(s0, src), b1 = __builtin_amdgcn_readlane(s1, src);
    const uint32_t n = windows_of(b1 - b0, nblk);
    for (uint32_t j = threadIdx.x & 63; j < n; j += 64) w.big_window[a + j] = make_uint4(row, j, b0, b1);
  }
}

// What k_front keeps while it works on its table.
struct FrontTab {
  const int32_t* idx;   // the table's lookups
  const int32_t* offt;  // its bags' offsets
  int32_t B;
  int64_t L;
  uint32_t P0, n;
  bool bad;  // a boundary of the tables that this thread has looked at is bad
};

// The keys (k) and bags (v) of the tile of m <= 1024*ITEMS lookups from t0 on, in wave-major
// order; true if an offset is bad, or a table's boundary.  A bag that starts in the tile marks its first position
// with its number + 1 (bags without lookups mark none), and a position takes the last mark
// at or before it: by ballot inside a run of 64, then from the run before, then from the
// waves before.  `carry` is the mark before the tile, and is moved past it.  Bags
// [b0, b1) hold every bag that starts in the tile.
template <int ITEMS>
__device__ __forceinline__ bool front_expand(FrontLds& S, const FrontTab& f, const TableDesc& td, uint32_t t0,
                                             uint32_t m, int b0, int b1, uint32_t& carry, uint32_t (&k)[ITEMS],
                                             uint32_t (&v)[ITEMS]) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // the tile's indices are on their way while the bags are found
  int32_t r[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t e = (uint32_t)(wv * 64 * ITEMS + i * 64 + lane);
    r[i] = m > 0 ? f.idx[t0 + min(e, m - 1)] : 0;
  }
  for (uint32_t i = tid; i < m; i += kFrontThreads) S.val[i] = 0;
  __syncthreads();
  bool bad = f.bad;
  for (int bt = b0 + tid; bt < b1; bt += 4 * kFrontThreads) {
    int32_t x[4], y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int b = min(bt + q * kFrontThreads, b1 - 1);
      x[q] = f.offt[b];
      y[q] = f.offt[b + 1];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int b = bt + q * kFrontThreads;
      bad |= bad_range(x[q], y[q], f.L);
      // (out of range where the offsets are bad, or in another tile)
      const int64_t at = (int64_t)x[q] - f.P0 - t0;
      if (b < b1 && y[q] > x[q] && at >= 0 && at < m) S.val[at] = (uint32_t)b + 1u;
    }
  }
  if (__syncthreads_or(bad)) return true;
  uint32_t run = 0;  // the last mark of the wave so far (wave-uniform)
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t e = (uint32_t)(wv * 64 * ITEMS + i * 64 + lane);
    const uint32_t x = e < m ? S.val[e] : 0u;
    const uint64_t marks = __ballot(x != 0), at = marks & (lanemask_lt() | (1ull << lane));
    const uint32_t near = __shfl(x, at ? 63 - (int)__clzll((unsigned long long)at) : 0);
    v[i] = at ? near : run;
    if (marks) run = __shfl(x, 63 - (int)__clzll((unsigned long long)marks));
  }
  uint32_t* last = reinterpret_cast<uint32_t*>(S.scan);
  if (lane == 0) last[wv] = run;
  __syncthreads();
  uint32_t in = carry;
  for (int w = 0; w < kFrontWaves; ++w) {
    const uint32_t x = last[w];
    if (w < wv && x) in = x;
    if (x) carry = x;
  }
  uint32_t n_bad = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t e = (uint32_t)(wv * 64 * ITEMS + i * 64 + lane);
    v[i] = (v[i] ? v[i] : in) - 1u;
    k[i] = kKeyInvalid;
    if (r[i] >= 0 && (int64_t)r[i] < td.N) {
      k[i] = (uint32_t)r[i];
      if (td.n_sets > 0) {
        const uint32_t q = div_by((uint32_t)r[i], td.by_sets);
        k[i] = ((uint32_t)r[i] - q * (uint32_t)td.n_sets) * (uint32_t)td.Q + q;
      }
    } else if (e < m) {
      ++n_bad;
    }
  }
  if (n_bad) atomicAdd(&S.n_bad, n_bad);
  __syncthreads();
  return false;
}

// Unique rows and touched sets of the m sorted keys from t0 on: a key that differs from its
// predecessor starts a row (first[u]: where), one of another set starts a set.  A run of 64
// keys is one ballot, and a start's rank is its run's offset plus the starts before it in
// the run.
template <int ITEMS>
__device__ __forceinline__ void front_unique(FrontLds& S, const Work& w, const TableDesc& td, const uint32_t* sk,
                                             uint32_t P0, uint32_t t0, uint32_t m, uint32_t* first, uint32_t& nU,
                                             uint32_t& nS) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t is_row = 0, is_set = 0;  // bit i: item i starts one
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t e = (uint32_t)(wv * 64 * ITEMS + i * 64 + lane);
    bool row = false, set = false;
    if (e < m) {
      const uint32_t key = sk[t0 + e];
      const uint32_t prev = t0 + e > 0 ? sk[t0 + e - 1] : kKeyInvalid;
      row = key != prev;
      set = row && (t0 + e == 0 || div_by(key, td.by_Q) != div_by(prev, td.by_Q));
    }
    const uint64_t br = __ballot(row), bs = __ballot(set);
    if (lane == 0) {
      S.rows[wv * ITEMS + i] = (uint32_t)__popcll(br);
      S.sets[wv * ITEMS + i] = (uint32_t)__popcll(bs);
    }
    is_row |= (row ? 1u : 0u) << i;
    is_set |= (set ? 1u : 0u) << i;
  }
  __syncthreads();
  constexpr int kRuns = kFrontWaves * ITEMS;
  const unsigned long long c =
      tid < kRuns ? (unsigned long long)S.rows[tid] | ((unsigned long long)S.sets[tid] << 32) : 0ull;
  unsigned long long tot;
  const unsigned long long ex = front_scan_exclusive<unsigned long long>(
      c, 0ull, S.scan, tot, [](unsigned long long a, unsigned long long b) { return a + b; });
  if (tid < kRuns) {
    S.rows[tid] = nU + (uint32_t)ex;
    S.sets[tid] = nS + (uint32_t)(ex >> 32);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool row = (is_row >> i) & 1u, set = (is_set >> i) & 1u;
    const uint64_t br = __ballot(row), bs = __ballot(set);
    const uint32_t u = S.rows[wv * ITEMS + i] + (uint32_t)__popcll(br & lanemask_lt());
    if (row) first[u] = t0 + (uint32_t)(wv * 64 * ITEMS + i * 64 + lane);
    if (set && td.n_sets > 0) {
      const uint32_t s = S.sets[wv * ITEMS + i] + (uint32_t)__popcll(bs & lanemask_lt());
      w.set_first[P0 + s] = P0 + u;
      w.nch[P0 + s] = div_by(sk[t0 + (uint32_t)(wv * 64 * ITEMS + i * 64 + lane)], td.by_Q);
    }
  }
  nU += (uint32_t)tot;
  nS += (uint32_t)(tot >> 32);
  __syncthreads();
}

// A table whose keys fit the LDS: true if an offset is bad.
template <int ITEMS>
__device__ __forceinline__ bool front_table(FrontLds& S, const Work& w, const FrontTab& f, const TableDesc& td,
                                            int passes, uint32_t& nU, uint32_t& nS) {
  uint32_t k[ITEMS], v[ITEMS], carry = 0;
  if (front_expand<ITEMS>(S, f, td, 0, f.n, 0, f.B, carry, k, v)) return true;
  front_sort<ITEMS>(S, k, v, f.n, passes, w.valsB + f.P0);
  front_unique<ITEMS>(S, w, td, S.key, f.P0, 0, f.n - S.n_bad, S.val, nU, nS);
  return false;
}

// One radix pass of n pairs in memory, a tile of kFrontTile at a time; S.hist[pass] holds the
// digit counts.  A tile goes through the LDS in digit order, so that it is written in runs
// (scattered from the registers, one line per lane and store, a tile took 17 us).
__device__ __forceinline__ void front_pass(FrontLds& S, const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                           uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint32_t n,
                                           int pass) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, shift = 8 * pass;
  const auto add = [](unsigned long long a, unsigned long long b) { return a + b; };
  unsigned long long all;
  uint32_t base = (uint32_t)front_scan_exclusive<unsigned long long>(tid < 256 ? S.hist[pass][tid] : 0u, 0ull, S.scan,
                                                                     all, add);  // of digit tid, moved past each tile
  for (uint32_t t0 = 0; t0 < n; t0 += kFrontTile) {
    const uint32_t m = min((uint32_t)kFrontTile, n - t0);
    uint32_t k[kFrontItems], v[kFrontItems], rank[kFrontItems];
#pragma unroll
    for (int i = 0; i < kFrontItems; ++i) {
      const uint32_t e = t0 + min((uint32_t)(wv * 64 * kFrontItems + i * 64 + lane), m - 1);
      k[i] = kin[e];
      v[i] = vin[e];
    }
    front_rank<kFrontItems>(S, k, m, shift, rank);
    __syncthreads();
    const uint32_t tot = front_wave_offsets(S);
    const uint32_t pre = (uint32_t)front_scan_exclusive<unsigned long long>(tid < 256 ? tot : 0u, 0ull, S.scan, all, add);
    if (tid < 256) {
      S.dpre[tid] = pre;
      S.hist[pass][tid] = base - pre;  // where the digit's run goes, less its start in the tile
      base += tot;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kFrontItems; ++i) {
      if ((uint32_t)(wv * 64 * kFrontItems + i * 64 + lane) < m) {
        const uint32_t d = (k[i] >> shift) & 255u;
        const uint32_t at = S.dpre[d] + S.cnt[wv][d] + rank[i];
        S.key[at] = k[i];
        S.val[at] = v[i];
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kFrontItems; ++i) {
      const uint32_t j = (uint32_t)(i * kFrontThreads + tid);
      if (j < m) {
        const uint32_t key = S.key[j], g = S.hist[pass][(key >> shift) & 255u] + j;
        kout[g] = key;
        vout[g] = S.val[j];
      }
    }
    __syncthreads();
  }
}

// A table with more keys than the LDS holds: a tile at a time, the pairs in memory, where the
// passes alternate between the two buffers and end in B.
__device__ __forceinline__ bool front_large(FrontLds& S, const Work& w, const FrontTab& f, const TableDesc& td,
                                         int passes, uint32_t& nU, uint32_t& nS) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t* ka = w.keysA + f.P0;
  uint32_t* va = w.valsA + f.P0;
  uint32_t* kb = w.keysB + f.P0;
  uint32_t* vb = w.valsB + f.P0;
  uint32_t* k0 = (passes & 1) ? ka : kb;
  uint32_t* v0 = (passes & 1) ? va : vb;
  uint32_t carry = 0;
  bool bad = f.bad;  // every offset is checked before the tiles look for theirs
  for (int b0 = threadIdx.x; b0 < f.B; b0 += 8 * kFrontThreads) {
    int32_t x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int b = min(b0 + q * kFrontThreads, f.B - 1);
      const int32_t a = f.offt[b], e = f.offt[b + 1];
      x[q] = bad_range(a, e, f.L);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) bad |= x[q] != 0;
  }
  if (__syncthreads_or(bad)) return true;
  // the first bag that starts at or after position p of the table
  const auto bag_from = [&](uint32_t p) -> int {
    int a = 0, e = f.B;
    while (a < e) {
      const int step = (e - a + 63) / 64, c = a + lane * step;
      const uint64_t ge = __ballot(c >= e || (uint32_t)f.offt[c] - f.P0 >= p);
      const int q = ge ? (int)__builtin_ctzll(ge) : 64;
      if (q == 0) break;
      const int lo = a + (q - 1) * step + 1;
      if (q < 64) e = min(e, a + q * step);
      a = lo;
    }
    return a;
  };
  for (int i = threadIdx.x; i < passes * 256; i += kFrontThreads) S.hist[i >> 8][i & 255] = 0;
  for (uint32_t t0 = 0; t0 < f.n; t0 += kFrontTile) {
    const uint32_t m = min((uint32_t)kFrontTile, f.n - t0);
    uint32_t k[kFrontItems], v[kFrontItems];
    if (front_expand<kFrontItems>(S, f, td, t0, m, bag_from(t0), bag_from(t0 + m), carry, k, v)) return true;
#pragma unroll
    for (int i = 0; i < kFrontItems; ++i) {
      const uint32_t e = (uint32_t)(wv * 64 * kFrontItems + i * 64 + lane);
      if (e < m) {
        k0[t0 + e] = k[i];
        v0[t0 + e] = v[i];
        for (int p = 0; p < passes; ++p) atomicAdd(&S.hist[p][(k[i] >> (8 * p)) & 255u], 1u);
      }
    }
  }
  __syncthreads();
  for (int p = 0; p < passes; ++p) {
    const bool from_a = ((passes - p) & 1) != 0;
    if (from_a) front_pass(S, ka, va, kb, vb, f.n, p);
    else front_pass(S, kb, vb, ka, va, f.n, p);
  }
  const uint32_t nv = f.n - S.n_bad;
  for (uint32_t t0 = 0; t0 < nv; t0 += kFrontTile)
    front_unique<kFrontItems>(S, w, td, kb, f.P0, t0, min((uint32_t)kFrontTile, nv - t0), w.seg + f.P0, nU, nS);
  return false;
}

// Workgroup t handles table t alone and changes no state but the table's statistics (a bad
// offset inside another table rejects the call: the kernels after this one look at every
// table's flag).  Its time at 2048 lookups is about a chain of 12 barriers and memory
// round trips per digit pass and list, not bandwidth: one workgroup holds the keys in
// LDS and registers from the expansion to the lists.
__global__ __launch_bounds__(kFrontThreads) void k_front(Dev dv, Work w, const int32_t* __restrict__ idx, int64_t L,
                                                         const int32_t* __restrict__ off, int32_t B, int passes,
                                                         int group, int nblk) {
  __shared__ FrontLds S;
  const int t = blockIdx.x, tid = threadIdx.x;
  const TableDesc td = dv.desc[t];
  {
    // the backward statistics of the table, in every copy
    unsigned long long* st = dv.stats + ((int64_t)t << dv.stat_shift) * kStatStride;
    for (int i = tid; i < (1 << dv.stat_shift) * kStatStride; i += kFrontThreads) {
      const int f = i % kStatStride;
      if ((f >= kStBwdLookups && f <= kStHitEvictions) || f == kStInvalidBwd) st[i] = 0;
    }
  }
  const int32_t* offt = off + (int64_t)t * B;
  const int64_t p0 = B > 0 ? offt[0] : 0, p1 = B > 0 ? offt[B] : 0;
  bool bad = bad_range(p0, p1, L);  // whole workgroup, as below
  const uint32_t P0 = bad ? 0u : (uint32_t)p0, n = bad ? 0u : (uint32_t)(p1 - p0);
  // every workgroup looks at all tables' boundaries before it writes: its positions are then its
  // own.  The threads learn of each other's boundaries with the bags', which are checked as
  // they are expanded (with a barrier of its own for the check the kernel was 0.3 us longer).
  const FrontTab f{idx + P0, offt, B, L, P0, n, B > 0 && bad_boundaries(off, dv.T, B, L, tid, kFrontThreads)};
  if (tid == 0) S.n_bad = S.n_chunk = S.n_big = S.n_window = 0;
  // expanded, sorted by the local key (a skipped lookup's digits are all 255, above every
  // valid key's, so skipped lookups end the table's run), unique rows and sets listed
  const bool in_lds = n <= (uint32_t)kFrontTile;
  uint32_t* vb = w.valsB + P0;
  uint32_t nU = 0, nS = 0;
  if (!bad) {
    if (n <= 1 * kFrontThreads) bad = front_table<1>(S, w, f, td, passes, nU, nS);
    else if (n <= 2 * kFrontThreads) bad = front_table<2>(S, w, f, td, passes, nU, nS);
    else if (n <= 4 * kFrontThreads) bad = front_table<4>(S, w, f, td, passes, nU, nS);
    else if (in_lds) bad = front_table<kFrontItems>(S, w, f, td, passes, nU, nS);
    else bad = front_large(S, w, f, td, passes, nU, nS);
  }
  if (bad) {
    if (tid == 0) {
      w.tab_info[t] = TabInfo{.bad = 1};
      atomicOr(dv.err, kErrOffsets);
    }
    return;
  }
  const uint32_t nv = n - S.n_bad;
  const uint32_t* sk = in_lds ? S.key : w.keysB + P0;
  const uint32_t* first = in_lds ? S.val : w.seg + P0;
  if (td.n_sets == 0) nS = (nU + group - 1) / group;  // runs of `group` rows, no decision
  __syncthreads();

  // ---- per unique row: the update's inputs, and the jobs of the gradient sums (their order
  // inside a table does not matter).  A row of more than kSmallDirect lookups has at most one
  // chunk per 9 of them and a row of more than kBlockAbove is one per 513, with a window per
  // 32, so the jobs of a table fit the 1/8, 1/512 and 1/32 of its positions.
  const uint32_t cbase = P0 >> kSmallChunkShift, hbase = P0 >> 9;
  for (uint32_t base = 0; base < nU; base += 4 * kFrontThreads) {  // whole waves
    uint32_t s0[4], s1[4], bag[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t i = min(base + q * kFrontThreads + tid, nU - 1);
      s0[q] = first[i];
      s1[q] = i + 1 < nU ? first[i + 1] : nv;
      bag[q] = vb[s0[q]];  // used by a row with one lookup
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (base + q * kFrontThreads >= nU) break;
      const bool live = base + q * kFrontThreads + tid < nU;
      const uint32_t u = P0 + base + q * kFrontThreads + tid;
      const uint32_t c = s1[q] - s0[q], key = sk[s0[q]];
      uint32_t r = key;
      if (td.n_sets > 0) {
        const uint32_t set = div_by(key, td.by_Q);
        r = (key - set * (uint32_t)td.Q) * (uint32_t)td.n_sets + set;
      }
      const bool big = live && c > kBlockAbove;
      uint32_t aux = 0, window = 0;
      if (big) {
        aux = hbase + atomicAdd(&S.n_big, 1u);
        window = (P0 >> kWindowShift) + atomicAdd(&S.n_window, windows_of(c, nblk));
      } else if (live && c > kSmallDirect) {
        const uint32_t nc = (c + kSumChunk - 1) / kSumChunk;
        aux = cbase + atomicAdd(&S.n_chunk, nc);
        for (uint32_t j = 0; j < nc; ++j) {
          const uint32_t a = P0 + s0[q] + j * (uint32_t)kSumChunk;
          w.chunk_span[aux + j] = make_uint2(a, min(a + (uint32_t)kSumChunk, P0 + s1[q]));
        }
      }
      if (live) w.umeta[u] = make_uint4((uint32_t)td.row_base + r, aux, c == 1 ? bag[q] : P0 + s0[q], c);
      put_windows(w, big, window, aux, P0 + s0[q], P0 + s1[q], nblk);
    }
  }
  __syncthreads();
  if (tid == 0) {
    w.tab_info[t] = TabInfo{P0, nU, nS, S.n_chunk, S.n_big, S.n_window, 0, n - nv, nv};
    unsigned long long* st = dv.stats + ((int64_t)t << dv.stat_shift) * kStatStride;
    st[kStBwdLookups] = nv;
    st[kStInvalidBwd] = n - nv;
    st[kStUnique] = nU;
    if (td.n_sets == 0) st[kStBypasses] = nU;
    if (n != nv) atomicOr(dv.err, kErrIndex);
  }
}

// ---- the tables' lists as one range ----------------------------------------------------------
// Prefix sums over the tables of one count of TabInfo, in LDS (T <= kSmallTables).
struct TabPrefix {
  uint32_t pre[kSmallTables + 1];
  uint32_t part[4];
};

// By the whole workgroup (256 threads); false if a table's offsets were rejected.
template <typename F>
__device__ __forceinline__ bool tab_prefix(TabPrefix& P, const TabInfo* ti, int T, F&& count) {
  static_assert(kSmallTables == 512, "two tables per thread");
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i0 = 2 * threadIdx.x;
  uint32_t a = 0, b = 0;
  bool bad = false;
  if (i0 < T) {
    const TabInfo x = ti[i0];
    a = count(x);
    bad |= x.bad != 0;
  }
  if (i0 + 1 < T) {
    const TabInfo x = ti[i0 + 1];
    b = count(x);
    bad |= x.bad != 0;
  }
  uint32_t s = a + b;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(s, o);
    if (lane >= o) s += y;
  }
  if (lane == 63) P.part[wv] = s;
  bad = __syncthreads_or(bad) != 0;
  uint32_t pre = s - a - b;
  for (int k = 0; k < wv; ++k) pre += P.part[k];
  P.pre[i0] = pre;
  P.pre[i0 + 1] = pre + a;
  if (threadIdx.x == 255) P.pre[kSmallTables] = pre + a + b;
  __syncthreads();
  return !bad;
}

// The table of item i < pre[T] (tables without items are skipped).
__device__ __forceinline__ int tab_of(const TabPrefix& P, int T, uint32_t i) {
  int lo = 0, hi = T;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (P.pre[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// ---- unique rows of a mid call -----------------------------------------------------------------
// Per unique row: its row, lookups and first occurrence, its gradient-sum jobs, and its probe
// with the update of its priority (with one group of lanes per set doing these as in a small
// call, an LFU set of 2000 rows took 90 us of a step of 222).  A
// workgroup takes 256*PER rows (one per thread below 2^19 lookups, whose rows are few
// workgroups' worth); the jobs of the rows of one table are placed with one
// addition per workgroup to the table's count (a workgroup across a table boundary adds
// per row).
template <int MAXA, int PER>
__global__ __launch_bounds__(256) void k_mid_rows(Dev dv, Work w, const uint32_t* __restrict__ sk,
                                                  const uint32_t* __restrict__ sval, uint32_t step, int nblk) {
  __shared__ TabPrefix P;
  __shared__ unsigned long long part[4];
  __shared__ uint32_t at_s[3];
  if (!tab_prefix(P, w.tab_info, dv.T, [](const TabInfo& x) { return x.rows; })) return;
  constexpr uint32_t kRows = 256 * PER;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t nU = P.pre[dv.T];
  for (uint32_t r0 = blockIdx.x * kRows; r0 < nU; r0 += gridDim.x * kRows) {
    const uint32_t rend = min(r0 + kRows, nU);
    const int ta = tab_of(P, dv.T, r0), tb = tab_of(P, dv.T, rend - 1);  // whole workgroup
    uint32_t s0[PER], c[PER], key[PER], bag[PER];
    int tt[PER];
    unsigned long long jobs = 0;  // chunks | big rows << 20 | windows << 40 (at most 512 per row)
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t i = min(r0 + (uint32_t)(q * 256) + threadIdx.x, rend - 1);
      tt[q] = ta == tb ? ta : tab_of(P, dv.T, i);
      const TabInfo& ti = w.tab_info[tt[q]];
      const uint32_t k = i - P.pre[tt[q]];
      s0[q] = w.seg[ti.pos + k];
      c[q] = (k + 1 < ti.rows ? w.seg[ti.pos + k + 1] : ti.pos + ti.valid) - s0[q];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      key[q] = sk[s0[q]];
      bag[q] = sval[s0[q]];
      if (r0 + (uint32_t)(q * 256) + threadIdx.x >= rend) c[q] = 0;
      jobs += c[q] > kBlockAbove ? (1ull << 20) + ((unsigned long long)windows_of(c[q], nblk) << 40)
                                 : c[q] > kMidDirect ? (c[q] + kSumChunk - 1) / kSumChunk : 0u;
    }
    unsigned long long x = jobs;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    __syncthreads();  // the previous round's part and at_s have been read
    if (lane == 63) part[wv] = x;
    __syncthreads();
    unsigned long long pre = x - jobs, tot = 0;
    for (int k = 0; k < 4; ++k) {
      if (k < wv) pre += part[k];
      tot += part[k];
    }
    if (ta == tb && threadIdx.x < 3) {
      const uint32_t n = (uint32_t)(tot >> (20 * threadIdx.x)) & (threadIdx.x < 2 ? 0xFFFFFu : ~0u);
      TabInfo& ti = w.tab_info[ta];
      at_s[threadIdx.x] = n ? atomicAdd(threadIdx.x == 0 ? &ti.chunks : threadIdx.x == 1 ? &ti.big : &ti.windows, n) : 0u;
    }
    __syncthreads();
    // (where this thread's jobs go; a workgroup across a table boundary places them one by one)
    uint32_t chunk_at = at_s[0] + ((uint32_t)pre & 0xFFFFFu), big_at = at_s[1] + ((uint32_t)(pre >> 20) & 0xFFFFFu),
             window_at = at_s[2] + (uint32_t)(pre >> 40);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const bool live = c[q] != 0, big = c[q] > kBlockAbove;
      const int t = tt[q];
      const uint32_t pos = w.tab_info[t].pos;
      const TableDesc& td = dv.desc[t];
      uint32_t aux = 0, window = 0;
      if (big) {
        const uint32_t nw = windows_of(c[q], nblk);
        aux = (pos >> 9) + (ta == tb ? big_at++ : atomicAdd(&w.tab_info[t].big, 1u));
        window = (pos >> kWindowShift) + (ta == tb ? window_at : atomicAdd(&w.tab_info[t].windows, nw));
        window_at += nw;
      } else if (c[q] > kMidDirect) {
        const uint32_t nc = (c[q] + kSumChunk - 1) / kSumChunk;
        if (ta == tb) {
          aux = (pos >> kMidChunkShift) + chunk_at;
          chunk_at += nc;
        } else {
          aux = (pos >> kMidChunkShift) + atomicAdd(&w.tab_info[t].chunks, nc);
        }
        for (uint32_t j = 0; j < nc; ++j) {
          const uint32_t a = s0[q] + j * (uint32_t)kSumChunk;
          w.chunk_span[aux + j] = make_uint2(a, min(a + (uint32_t)kSumChunk, s0[q] + c[q]));
        }
      }
      if (live) {
        const uint32_t u = pos + r0 + (uint32_t)(q * 256) + threadIdx.x - P.pre[t];
        uint32_t r = key[q] - (uint32_t)td.key_base;
        if (td.n_sets > 0) {
          const uint32_t set = div_by(r, td.by_Q);
          r = (r - set * (uint32_t)td.Q) * (uint32_t)td.n_sets + set;
        }
        const uint32_t grow = (uint32_t)td.row_base + r;
        w.umeta[u] = make_uint4(grow, aux, c[q] == 1 ? bag[q] : s0[q], c[q]);
        const int32_t slot = probe_slot<MAXA>(dv, td, (int32_t)r);
        w.uslot[u] = slot;
        w.uact[u] = slot >= 0 ? kActHitStay : kActBypass;
        if (dv.policy == 0) {
          if (slot >= 0) dv.ts[slot] = (int32_t)step;
        } else {
          const int64_t cc = (int64_t)dv.cnt[grow] + c[q];
          const int32_t cn = cc > 0x7FFFFFFF ? 0x7FFFFFFF : (int32_t)cc;
          dv.cnt[grow] = cn;
          w.ukey[u] = slot >= 0 ? 0ull : ((unsigned long long)(uint32_t)cn << 32) | (uint32_t)~grow;
        }
      }
      put_windows(w, big, window, aux, s0[q], s0[q] + c[q], nblk);
    }
  }
}

// ---- decisions ---------------------------------------------------------------------------------
// One group of G lanes (G >= assoc) per touched set: the set's tags are loaded once, one per
// lane, and every row of the set is compared with all of them by a ballot, so the probe
// needs no pass of its own; then the priorities are updated and the inserts and their
// victims chosen as k_policy does.  The set's rows, tags, stamps and the counts of its rows
// are touched by this group alone.  PROBED: k_mid_rows has probed the rows and updated the
// priorities.
template <int G, bool PROBED>
__device__ __forceinline__ void decide_sets(const Dev& dv, const Work& w, TabPrefix& P, uint32_t step, int wg, int nwg) {
  __shared__ PolicyLds lds_all[4];
  __shared__ int32_t hitc_all[4][64];  // LFU: the count of the row that hit way w
  __shared__ __attribute__((aligned(16))) int32_t tags_all[4][64];
  __shared__ int32_t tab_s;
  __shared__ uint32_t sums_s[PolicyStats::kN];
  PolicyLds& L = lds_all[threadIdx.x >> 6];
  int32_t* hitc = hitc_all[threadIdx.x >> 6];
  int32_t* tags = tags_all[threadIdx.x >> 6];
  const int lane = threadIdx.x & 63;
  const int gb = lane & ~(G - 1), l = lane & (G - 1);
  const uint64_t gmask = G == 64 ? ~0ull : (((1ull << G) - 1) << gb);
  const uint64_t below = lanemask_lt() & gmask;
  const int A = dv.assoc;
  const bool lru = dv.policy == 0;
  const uint32_t nS = P.pre[dv.T];
  int64_t k0, k1;
  part_range(0, nS, wg, nwg, k0, k1);
  PolicyStats ps;
  for (int64_t k = k0 + threadIdx.x / G; k < k1; k += 256 / G) {
    const int t = tab_of(P, dv.T, (uint32_t)k);
    const TabInfo ti = w.tab_info[t];
    const TableDesc td = dv.desc[t];
    const uint32_t s = ti.pos + (uint32_t)k - P.pre[t];
    if (t != ps.t) {
      if (l == 0) ps.flush(dv);
      ps.t = t;
    }
    const uint32_t uend = ti.pos + ti.rows;
    if (td.n_sets == 0) {
      // no cache: every row is written to T (their bypasses were counted with the lists)
      const uint32_t u = ti.pos + ((uint32_t)k - P.pre[t]) * G + l;
      if (!PROBED && u < uend) {
        w.uact[u] = kActBypass;
        if (!lru) {
          const uint4 m = w.umeta[u];
          const int64_t c = (int64_t)dv.cnt[m.x] + m.w;
          dv.cnt[m.x] = c > 0x7FFFFFFF ? 0x7FFFFFFF : (int32_t)c;
        }
      }
      continue;
    }
    const uint32_t u0 = w.set_first[s], u1 = (uint32_t)k + 1 < P.pre[t + 1] ? w.set_first[s + 1] : uend;
    const int64_t sbase = td.slot_base + (int64_t)w.nch[s] * A;
    int32_t tg = -1;
    long long vpv = LLONG_MAX;
    if (l < A) {
      tg = dv.tag[sbase + l];
      if (lru) vpv = dv.ts[sbase + l];
      else if (PROBED && tg >= 0) vpv = dv.cnt[td.row_base + tg];
    }
    L.hitu[lane] = -1;
    tags[lane] = tg;
    __builtin_amdgcn_wave_barrier();
    uint32_t M = 0, H = 0;
    int64_t last_miss = -1;        // the set's last missed row
    // LFU: the lane's four best rank keys so far (count, then the lower row; 0: none), and
    // their rows; a lane that has given all four looks for the next in memory (sets of more
    // than 4G rows).  Scanning every key of the set for every candidate, a set of 2000 rows
    // took 100 us.
    unsigned long long top[4] = {0, 0, 0, 0};
    int32_t top_u[4] = {-1, -1, -1, -1};
    const auto keep = [&](unsigned long long key, int32_t u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (key > top[i]) {
          const unsigned long long k1 = top[i];
          const int32_t u1_ = top_u[i];
          top[i] = key;
          top_u[i] = u;
          key = k1;
          u = u1_;
        }
      }
    };
    // the rows are loaded two rounds ahead and their counts one (a set may have thousands)
    if constexpr (PROBED) {
      const auto slot_at = [&](uint32_t u) { return w.uslot[min(u, u1 - 1)]; };
      const auto key_at = [&](uint32_t u) { return lru ? 0ull : w.ukey[min(u, u1 - 1)]; };
      int32_t sa = slot_at(u0 + l), sb = slot_at(u0 + G + l);
      unsigned long long ka = key_at(u0 + l), kb = key_at(u0 + G + l);
      for (uint32_t c = u0; c < u1; c += G) {
        const uint32_t u = c + l;
        const int32_t sl = sa;
        const unsigned long long key = ka;
        sa = sb;
        ka = kb;
        sb = slot_at(u + 2 * G);
        kb = key_at(u + 2 * G);
        const bool hit = u < u1 && sl >= 0, miss = u < u1 && sl < 0;
        if (hit) L.hitu[gb + (int)(sl - sbase)] = (int32_t)u;
        if (!lru && miss) keep(key, (int32_t)u);
        const uint64_t mm = __ballot(miss) & gmask;
        if (lru) {
          const uint32_t rank = M + (uint32_t)__popcll(mm & below);
          if (miss && rank < (uint32_t)A) {
            L.cand_u[gb + rank] = (int32_t)u;
            L.cand_pv[gb + rank] = (long long)step;
          }
          if (mm) last_miss = (int64_t)c + (63 - __clzll((unsigned long long)mm)) - gb;
        }
        M += (uint32_t)__popcll(mm);
        H += (uint32_t)__popcll(__ballot(hit) & gmask);
      }
    } else {
      uint4 next = w.umeta[min(u0 + l, u1 - 1)], next2 = w.umeta[min(u0 + G + l, u1 - 1)];
      int32_t cnext = !lru ? dv.cnt[next.x] : 0;
      for (uint32_t c = u0; c < u1; c += G) {
        const uint32_t u = c + l;
        const bool act = u < u1;
        const uint4 meta = next;
        const int32_t cnt0 = cnext;
        next = next2;
        next2 = w.umeta[min(u + 2 * G, u1 - 1)];
        if (!lru && c + G < u1) cnext = dv.cnt[next.x];
        const int32_t r = (int32_t)(meta.x - (uint32_t)td.row_base);
        int way = -1;
        if (A >= 4) {
          for (int j = 0; j < A; j += 4) {
            const int4 tj = *reinterpret_cast<const int4*>(tags + gb + j);
            // (the last way that holds the row, as probe_set: an imported cache may hold it twice)
            way = tj.w == r ? j + 3 : tj.z == r ? j + 2 : tj.y == r ? j + 1 : tj.x == r ? j : way;
          }
        } else {
          for (int j = 0; j < A; ++j) way = tags[gb + j] == r ? j : way;
        }
        const bool hit = act && way >= 0, miss = act && way < 0;
        if (act) {
          w.uact[u] = hit ? kActHitStay : kActBypass;
          w.uslot[u] = hit ? (int32_t)(sbase + way) : -1;
          int32_t cn = 0;
          if (lru) {
            if (hit) dv.ts[sbase + way] = (int32_t)step;
          } else {
            const int64_t cc = (int64_t)cnt0 + meta.w;
            cn = cc > 0x7FFFFFFF ? 0x7FFFFFFF : (int32_t)cc;
            dv.cnt[meta.x] = cn;
            const unsigned long long key = hit ? 0ull : ((unsigned long long)(uint32_t)cn << 32) | (uint32_t)~meta.x;
            keep(key, (int32_t)u);
            if (u1 - u0 > 4 * (uint32_t)G) w.ukey[u] = key;
          }
          if (hit) {
            L.hitu[gb + way] = (int32_t)u;
            hitc[gb + way] = cn;
          }
        }
        const uint64_t mm = __ballot(miss) & gmask;
        if (lru) {
          // the candidates: the first missed rows in row order
          const uint32_t rank = M + (uint32_t)__popcll(mm & below);
          if (miss && rank < (uint32_t)A) {
            L.cand_u[gb + rank] = (int32_t)u;
            L.cand_pv[gb + rank] = (long long)step;
          }
          if (mm) last_miss = (int64_t)c + (63 - __clzll((unsigned long long)mm)) - gb;
        }
        M += (uint32_t)__popcll(mm);
        H += (uint32_t)__popcll(__ballot(hit) & gmask);
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (l == 0) ps.hits += H;
    if (M == 0) continue;

    // priorities of the ways after this step's accesses (empty = lowest)
    if (l < A) {
      const int32_t hu = L.hitu[lane];
      if (tg < 0) vpv = LLONG_MIN;
      else if (PROBED) {}  // as loaded
      else if (lru) vpv = hu >= 0 ? (long long)(int32_t)step : vpv;
      else vpv = hu >= 0 ? (long long)hitc[lane] : (long long)dv.cnt[td.row_base + tg];
    }
    int my_way = 0;
    int32_t my_u = -1, my_old = -1, my_hu = -1;
    int n_ins = 0;
    if (A == 1 && lru) {
      // direct-mapped LRU: no priority test; the largest missed row ends in the way
      n_ins = 1;
      my_u = (int32_t)last_miss;
      my_old = __shfl(tg, gb);
      my_hu = my_old >= 0 ? L.hitu[gb] : -1;
    } else {
      int vr = 0;
      for (int j = 0; j < A; ++j) {
        const long long pj = __shfl(vpv, gb + j);
        vr += (pj < vpv || (pj == vpv && j < l)) ? 1 : 0;
      }
      if (l < A) {
        L.vic_way[gb + vr] = l;
        L.vic_pv[gb + vr] = vpv;
      }
      int K = M < (uint32_t)A ? (int)M : A;
      if (!lru) {
        int given = 0, taken = 0;
        for (int r = 0; r < K; ++r) {
          unsigned long long best = top[0];
          int32_t bu = top_u[0];
#pragma unroll
          for (int o = G / 2; o >= 1; o >>= 1) {
            const unsigned long long ob = __shfl_xor(best, o, G);
            const int32_t ou = __shfl_xor(bu, o, G);
            if (ob > best) {
              best = ob;
              bu = ou;
            }
          }
          const long long cpv = (long long)(best >> 32);
          if (best == 0 || !(cpv > L.vic_pv[gb + r])) break;
          if (l == 0) {
            L.cand_u[gb + r] = bu;
            L.cand_pv[gb + r] = cpv;
          }
          if (top[0] == best) {  // the one lane that had it (keys are unique)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
              top[i] = top[i + 1];
              top_u[i] = top_u[i + 1];
            }
            top[3] = 0;
            if (++given % 4 == 0 && u1 - u0 > 4 * (uint32_t)G) {
              for (uint32_t c = u0 + l; c < u1; c += G) {  // (its own rows' keys)
                const unsigned long long key = w.ukey[c];
                if (key < best) keep(key, (int32_t)c);
              }
            }
          }
          taken = r + 1;
        }
        K = taken;
      }
      __builtin_amdgcn_wave_barrier();
      const bool ok = l < K && L.cand_pv[gb + l] > L.vic_pv[gb + l];
      const uint64_t fail = __ballot(l < K && !ok) & gmask;
      n_ins = fail ? __ffsll((unsigned long long)fail) - 1 - gb : K;
      my_way = l < n_ins ? L.vic_way[gb + l] : 0;
      my_old = __shfl(tg, gb + my_way);
      my_u = l < n_ins ? L.cand_u[gb + l] : -1;
      my_hu = (l < n_ins && my_old >= 0) ? L.hitu[gb + my_way] : -1;
      __builtin_amdgcn_wave_barrier();
    }
    if (l < n_ins) {
      w.uact[my_u] = kActInsert;
      w.uslot[my_u] = (int32_t)(sbase + my_way);
      w.uvic_row[my_u] = my_old;
      w.uvic_u[my_u] = my_hu;
      if (my_hu >= 0) w.uact[my_hu] = kActDone;
    }
    const uint32_t n_valid = (uint32_t)__popcll(__ballot(l < n_ins && my_old >= 0) & gmask);
    const uint32_t n_hitev = (uint32_t)__popcll(__ballot(l < n_ins && my_hu >= 0) & gmask);
    if (l == 0) {
      ps.ins += (uint32_t)n_ins;
      ps.byp += M - (uint32_t)n_ins;
      ps.ev += n_valid;
      ps.em += (uint32_t)n_ins - n_valid;
      ps.he += n_hitev;
    }
  }
  ps.flush_workgroup(dv, l == 0, &tab_s, sums_s);
}

// ---- gradient sums ----------------------------------------------------------------------------
// Left-to-right sum of the gradient rows of occurrences [i0, i1) of the sorted stream
// (i0 < i1) by GL = min(64, d) lanes, CL = d/GL columns per lane, from -0 (the identity of
// IEEE addition).  U rows are in flight, loaded without a branch (an index past the last
// occurrence re-reads it and adds -0): with the loads under a condition per row, one at a
// time came back, and a 64-lookup chunk took 40 us.
template <int D>
struct SumGeo {
  static constexpr int GL = D < 64 ? D : 64;
  static constexpr int CL = D / GL;
};

template <int D>
__device__ __forceinline__ void sum_span(const uint32_t* __restrict__ sval, uint32_t i0, uint32_t i1, GradRows<D> gr,
                                         int l, float (&acc)[SumGeo<D>::CL]) {
  constexpr int GL = SumGeo<D>::GL, CL = SumGeo<D>::CL, U = D == 16 || D == 256 ? 16 : 32;
#pragma unroll
  for (int c = 0; c < CL; ++c) acc[c] = -0.0f;
  uint32_t next = sval[min(i0 + l, i1 - 1)];
  for (uint32_t ic = i0; ic < i1; ic += GL) {
    const uint32_t my = next;
    next = sval[min(ic + GL + l, i1 - 1)];
    const int n = (int)min((uint32_t)GL, i1 - ic);
    for (int j = 0; j < n; j += U) {
      float x[U][CL];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        uint32_t b;
        if constexpr (GL == 64) b = __builtin_amdgcn_readlane(my, j + q);
        else b = __shfl(my, j + q, GL);
        const float* p = gr.row(b) + l * CL;
#pragma unroll
        for (int c = 0; c < CL; ++c) x[q][c] = p[c];
      }
#pragma unroll
      for (int q = 0; q < U; ++q)
#pragma unroll
        for (int c = 0; c < CL; ++c) acc[c] = acc[c] + (j + q < n ? x[q][c] : -0.0f);
    }
  }
}

// The same sum of a long span by a whole wave, for rows of up to 64 columns: 8 loads of 64
// lanes, 16 bytes each, bring 2048/d rows at once (16 lanes of 4 bytes per row would have 16
// rows in flight), which d lanes add from LDS while the next ones are loaded.  The
// occurrences may be of several bag blocks (unless `one`): put(k, sum, k') ends the sum of
// block k, which block k' follows, and the last block's sum is returned.
constexpr int kWaveLoads = 8;
typedef float f4w __attribute__((ext_vector_type(4)));

template <int D, typename Put>
__device__ __forceinline__ float wave_sum_blocks(const uint32_t* __restrict__ sval, uint32_t i0, uint32_t i1,
                                                 GradRows<D> gr, bool one, int nb_shift, f4w* lds, Put&& put) {
  static_assert(D <= 64, "one lane per column");
  constexpr int LPW = D / 4, RPI = 64 / LPW, R = RPI * kWaveLoads, NB = (R + 63) / 64;
  const int lane = threadIdx.x & 63;
  const float* lf = reinterpret_cast<const float*>(lds);
  f4w v[kWaveLoads];
  uint32_t bag[NB];
  const auto load = [&](uint32_t at) {
#pragma unroll
    for (int b = 0; b < NB; ++b) bag[b] = sval[min(at + (uint32_t)(b * 64 + lane), i1 - 1)];
#pragma unroll
    for (int q = 0; q < kWaveLoads; ++q) {
      // row q*RPI + lane/LPW of the batch
      const uint32_t b = __shfl(bag[q * RPI / 64], (q * RPI) % 64 + lane / LPW);
      v[q] = reinterpret_cast<const f4w*>(gr.row(b))[lane % LPW];
    }
  };
  load(i0);
  float acc = -0.0f;
  uint32_t cur = __builtin_amdgcn_readfirstlane(bag[0]) >> nb_shift;
  for (uint32_t ic = i0; ic < i1; ic += R) {
#pragma unroll
    for (int q = 0; q < kWaveLoads; ++q) lds[q * 64 + lane] = v[q];
    __builtin_amdgcn_wave_barrier();
    uint32_t blk[NB];
    uint64_t turn[NB];  // rows of the batch that are the first of a block
    bool any = false;
    if (!one) {  // (positions past the last occurrence repeat its bag)
      uint32_t before = cur;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        blk[b] = bag[b] >> nb_shift;
        const uint32_t p = __shfl_up(blk[b], 1);
        turn[b] = __ballot(blk[b] != (lane == 0 ? before : p));
        if (R < 64) turn[b] &= (1ull << (R & 63)) - 1;
        before = __builtin_amdgcn_readlane(blk[b], 63);
        any |= turn[b] != 0;
      }
    }
    if (ic + R < i1) load(ic + R);
    const int m = (int)min((uint32_t)R, i1 - ic);
    const auto add = [&](int r0, int r1) {
      if (lane < D) {
        int r = r0;
        for (; r + 8 <= r1; r += 8) {
          float x[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) x[q] = lf[(r + q) * D + lane];
#pragma unroll
          for (int q = 0; q < 8; ++q) acc = acc + x[q];
        }
        for (; r < r1; ++r) acc = acc + lf[r * D + lane];
      }
    };
    if (!any) {
      add(0, m);
    } else {
      int r0 = 0;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        for (uint64_t left = turn[b]; left; left &= left - 1) {  // whole wave
          const int j = (int)__builtin_ctzll(left), r1 = b * 64 + j;
          add(r0, r1);
          const uint32_t k = __builtin_amdgcn_readlane(blk[b], j);
          put(cur, acc, k);
          cur = k;
          acc = -0.0f;
          r0 = r1;
        }
      }
      add(r0, m);
    }
    __builtin_amdgcn_wave_barrier();
  }
  return acc;
}

// First occurrence in [a, b) of the sorted stream whose bag is at least `bag` (b if none), by
// a wave testing 64 points of the remaining range per round.
__device__ __forceinline__ uint32_t first_of_bag(const uint32_t* __restrict__ sval, uint32_t a, uint32_t b, uint32_t bag) {
  const uint32_t lane = threadIdx.x & 63;
  while (a < b) {
    const uint32_t step = (b - a + 63) / 64;
    const uint32_t m = a + lane * step;
    const uint64_t ge = __ballot(m >= b || sval[m] >= bag);
    const int f = ge ? (int)__builtin_ctzll(ge) : 64;
    if (f == 0) break;
    const uint32_t lo = a + (uint32_t)(f - 1) * step + 1;
    if (f < 64) b = min(b, a + (uint32_t)f * step);
    a = lo;
  }
  return a;
}

// The block sums of one window of a big row (e: the row, the window, the row's occurrences
// [z, w)), and the flags that say which blocks of the row have a sum (the fold adds those).  A
// window of one bag block searches its bounds; a window of kWindow occurrences takes the
// blocks whose first occurrence lies in it, and the flags from its first block up to the next
// window's.  With a window per block for every row, 1500 rows of 667 one-lookup bags were
// 0.73M windows of one or two occurrences (a step of 1M lookups, 16 columns: 848 us, now
// 261); with windows of occurrences for every row most windows of a row with many
// occurrences per block were empty, and held up the others (100 tables of 80,000 lookups, 16
// columns, two blocks: 873 us, now 643).
template <int D>
__device__ __forceinline__ void sum_window(const Work& w, const uint4& e, const uint32_t* __restrict__ sval,
                                           GradRows<D> gr, int nblk, int nb_shift, f4w* lds) {
  static_assert(kWindow == 64, "an occurrence per lane");
  constexpr int GL = SumGeo<D>::GL, CL = SumGeo<D>::CL;  // GL is 64 where runs are taken
  const uint32_t lane = threadIdx.x & 63, l = lane & (GL - 1);
  const uint32_t s0 = e.z, s1 = e.w;
  uint32_t* fl = w.bbound + (int64_t)e.x * bound_stride(w.max_nblk);
  float* bp = w.bpart + (int64_t)e.x * w.max_nblk * D;
  uint32_t a, b, ka, kl, k_next;  // occurrences [a, b), blocks [ka, kl]; the flags up to k_next
  if (block_windows(s1 - s0, nblk)) {
    ka = kl = e.y;
    k_next = ka + 1;
    a = first_of_bag(sval, s0, s1, ka << nb_shift);
    b = first_of_bag(sval, a, s1, k_next << nb_shift);
    if (a == b) {
      if (lane == 0) fl[ka] = 0;
      return;
    }
  } else {
    a = s0 + e.y * kWindow;
    const uint32_t wend = min(a + kWindow, s1), n = wend - a;
    // the window's blocks, one occurrence per lane, and those of the 64 after it
    const uint32_t v = sval[min(a + lane, s1 - 1)] >> nb_shift, after = sval[min(wend + lane, s1 - 1)] >> nb_shift;
    ka = __builtin_amdgcn_readfirstlane(v);
    kl = __builtin_amdgcn_readlane(v, n - 1);
    if (a > s0) {  // the block of the occurrence before belongs to an earlier window
      const uint32_t before = sval[a - 1] >> nb_shift;
      const uint64_t own = __ballot(lane < n && v != before);
      if (own == 0) return;
      const int first = (int)__builtin_ctzll(own);
      a += (uint32_t)first;
      ka = __builtin_amdgcn_readlane(v, first);
    }
    const uint64_t past = __ballot(wend + lane >= s1 || after != kl);
    if (past) {
      const int first = (int)__builtin_ctzll(past);
      b = wend + (uint32_t)first;
      k_next = b < s1 ? __builtin_amdgcn_readlane(after, first) : (uint32_t)nblk;
    } else {
      b = first_of_bag(sval, wend, s1, (kl + 1) << nb_shift);
      k_next = b < s1 ? sval[b] >> nb_shift : (uint32_t)nblk;
    }
    if (a == s0)
      for (uint32_t k = lane; k < ka; k += 64) fl[k] = 0;
  }
  float acc[CL];
  const auto put = [&](uint32_t k, uint32_t next) {  // the sum of block k; no sums up to block `next`
    if (lane < GL) {
#pragma unroll
      for (int c = 0; c < CL; ++c) bp[(int64_t)k * D + l * CL + c] = acc[c];
    }
    for (uint32_t j = k + lane; j < next; j += 64) fl[j] = j == k ? 1u : 0u;
  };
  const uint32_t bags = sval[b - 1] - sval[a] + 1;  // at most so many rows are loaded
  if constexpr (D <= 64) {
    if (D < 64 || b - a < 16 * bags) {
      acc[0] = wave_sum_blocks<D>(sval, a, b, gr, ka == kl, nb_shift, lds, [&](uint32_t k, float sum, uint32_t next) {
        acc[0] = sum;
        put(k, next);
      });
      put(kl, k_next);
      return;
    }
  } else if (ka == kl && b - a < 8 * bags) {
    sum_span<D>(sval, a, b, gr, l, acc);
    put(ka, k_next);
    return;
  }
  // else run by run of occurrences in one bag, whose row is loaded once and added as often as
  // the run is long, up to 16 runs in flight (with a load per occurrence the sum of a hot row is
  // one chain of load latencies: 1024 bags of 488 lookups, 128 columns, 1490 us a step, now 653,
  // 64 columns 1536 and 1030; the general path 960 and 1268; but at 4 occurrences of a row per
  // bag a load each is ahead, 130 and 149, and up to 32 columns the waves above always are)
#pragma unroll
  for (int c = 0; c < CL; ++c) acc[c] = -0.0f;
  uint32_t cur = ka;
  uint32_t next = sval[min(a + lane, b - 1)];
  for (uint32_t ic = a; ic < b; ic += 64) {
    const uint32_t my = next;
    next = sval[min(ic + 64 + lane, b - 1)];
    const int n = (int)min(64u, b - ic);
    const uint32_t before = __shfl_up(my, 1);
    uint64_t starts = __ballot((int)lane < n && (lane == 0 || my != before));
    const auto group = [&](auto runs) {  // the next U runs
      constexpr int U = decltype(runs)::value;
      int at[U + 1];
      uint32_t bag[U];
      float x[U][CL];
#pragma unroll
      for (int q = 0; q <= U; ++q) {
        at[q] = starts ? (int)__builtin_ctzll(starts) : n;
        if (q < U) starts &= starts - 1;  // (0 stays 0)
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        bag[q] = __builtin_amdgcn_readlane(my, min(at[q], n - 1));
        const float* p = gr.row(bag[q]) + l * CL;
#pragma unroll
        for (int c = 0; c < CL; ++c) x[q][c] = p[c];
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (at[q] >= n) break;
        const uint32_t k = bag[q] >> nb_shift;
        if (k != cur) {
          put(cur, k);
          cur = k;
#pragma unroll
          for (int c = 0; c < CL; ++c) acc[c] = -0.0f;
        }
        int r = at[q + 1] - at[q];
        for (; r >= 8; r -= 8) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int c = 0; c < CL; ++c) acc[c] = acc[c] + x[q][c];
        }
        for (; r > 0; --r)
#pragma unroll
          for (int c = 0; c < CL; ++c) acc[c] = acc[c] + x[q][c];
      }
    };
    while (starts) {  // whole wave
      if (__popcll(starts) <= 4) group(std::integral_constant<int, 4>{});
      else group(std::integral_constant<int, 16>{});
    }
  }
  put(cur, k_next);
}

template <int D>
__device__ __forceinline__ void sum_jobs(const Dev& dv, const Work& w, TabPrefix& P, const float* __restrict__ grad,
                                         const uint32_t* __restrict__ sval, int nblk, int nb_shift, int cshift, int wg,
                                         int nwg) {
  constexpr int GL = SumGeo<D>::GL, CL = SumGeo<D>::CL, GPB = 256 / GL;
  const int l = threadIdx.x & (GL - 1);
  // chunks, then (big row, bag block) pairs
  const uint32_t nC = P.pre[dv.T];
  for (uint32_t c = (uint32_t)wg * GPB + threadIdx.x / GL; c < nC; c += (uint32_t)nwg * GPB) {
    const int t = tab_of(P, dv.T, c);
    const uint32_t at = (w.tab_info[t].pos >> cshift) + c - P.pre[t];
    const uint2 sp = w.chunk_span[at];
    float acc[CL];
    sum_span<D>(sval, sp.x, sp.y, grad_rows<D>(grad, t, dv.T), l, acc);
    float* o = w.partial + (int64_t)at * D + l * CL;
#pragma unroll
    for (int q = 0; q < CL; ++q) o[q] = acc[q];
  }
  // then the windows of the big rows, a wave each
  __syncthreads();
  tab_prefix(P, w.tab_info, dv.T, [](const TabInfo& x) { return x.windows; });
  const uint32_t nW = P.pre[dv.T];
  __shared__ f4w stage[D <= 64 ? 4 * kWaveLoads * 64 : 1];
  const int wv = threadIdx.x >> 6;
  for (uint32_t i = (uint32_t)wg * 4 + wv; i < nW; i += (uint32_t)nwg * 4) {
    const int t = tab_of(P, dv.T, i);
    const uint4 e = w.big_window[(w.tab_info[t].pos >> kWindowShift) + i - P.pre[t]];
    sum_window<D>(w, e, sval, grad_rows<D>(grad, t, dv.T), nblk, nb_shift, stage + (D <= 64 ? wv * kWaveLoads * 64 : 0));
  }
}

// Workgroups below n_sum take the gradient sums (the longer chains, started first), the
// others the sets.
template <int D, int G, bool PROBED>
__global__ __launch_bounds__(256) void k_decide(Dev dv, Work w, const uint32_t* __restrict__ sval,
                                                const float* __restrict__ grad, uint32_t step, int nblk, int nb_shift,
                                                int cshift, int n_sum) {
  __shared__ TabPrefix P;
  if ((int)blockIdx.x < n_sum) {
    if (!tab_prefix(P, w.tab_info, dv.T, [](const TabInfo& x) { return x.chunks; })) {
      // rejected offsets: the backward statistics read 0
      if (blockIdx.x == 0) {
        const int64_t n = ((int64_t)dv.T << dv.stat_shift) * kStatStride;
        for (int64_t i = threadIdx.x; i < n; i += 256) {
          const int f = (int)(i % kStatStride);
          if ((f >= kStBwdLookups && f <= kStHitEvictions) || f == kStInvalidBwd) dv.stats[i] = 0;
        }
      }
      return;
    }
    sum_jobs<D>(dv, w, P, grad, sval, nblk, nb_shift, cshift, (int)blockIdx.x, n_sum);
  } else {
    if (!tab_prefix(P, w.tab_info, dv.T, [](const TabInfo& x) { return x.sets; })) return;
    decide_sets<G, PROBED>(dv, w, P, step, (int)blockIdx.x - n_sum, (int)gridDim.x - n_sum);
  }
}

// ---- update ------------------------------------------------------------------------------------
// Left-to-right fold of the block sums of big row h whose flag is set, U loaded at a time.
template <int D>
__device__ __forceinline__ void fold_flagged(const Work& w, uint32_t h, int nblk, int g, float (&acc)[8]) {
  constexpr int U = 4;
  const uint32_t* fl = w.bbound + (int64_t)h * bound_stride(w.max_nblk);
  const float* bp = w.bpart + (int64_t)h * w.max_nblk * D;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = -0.0f;
  for (int k0 = 0; k0 < nblk; k0 += U) {
    uint32_t f[U];
    float x[U][8];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int k = min(k0 + q, nblk - 1);
      f[q] = k0 + q < nblk ? fl[k] : 0u;
      load_row<D>(bp + (int64_t)k * D, g, x[q]);
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = acc[i] + (f[q] ? x[q][i] : -0.0f);
  }
}

// Up to kFoldInline blocks a row's sums are folded by the update; more, by a launch of their
// own, one workgroup per row: its waves bring kFoldRows block sums at a time to the LDS,
// where one lane per column adds them in order into the row's first slot.
constexpr int kFoldInline = 8;

template <int D>
__global__ __launch_bounds__(256) void k_fold(Dev dv, Work w, int nblk) {
  constexpr int kFoldRows = D == 256 ? 32 : 64, LPW = D / 4, PER = kFoldRows * LPW / 256;
  __shared__ TabPrefix P;
  __shared__ f4w stage[kFoldRows * LPW];
  if (!tab_prefix(P, w.tab_info, dv.T, [](const TabInfo& x) { return x.big; })) return;
  const float* sf = reinterpret_cast<const float*>(stage);
  const uint32_t n = P.pre[dv.T];
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int t = tab_of(P, dv.T, i);
    const uint32_t h = (w.tab_info[t].pos >> 9) + i - P.pre[t];
    const uint32_t* fl = w.bbound + (int64_t)h * bound_stride(w.max_nblk);
    float* bp = w.bpart + (int64_t)h * w.max_nblk * D;
    float acc = -0.0f;
    for (int k0 = 0; k0 < nblk; k0 += kFoldRows) {
      f4w v[PER];
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        // (a block without occurrences has no sum: -0, the identity of the addition)
        const int e = q * 256 + (int)threadIdx.x, k = k0 + e / LPW;
        v[q] = f4w{-0.0f, -0.0f, -0.0f, -0.0f};
        if (k < nblk && fl[k]) v[q] = reinterpret_cast<const f4w*>(bp + (int64_t)k * D)[e % LPW];
      }
      __syncthreads();  // the sums of the rows before have been read
#pragma unroll
      for (int q = 0; q < PER; ++q) stage[q * 256 + threadIdx.x] = v[q];
      __syncthreads();
      if ((int)threadIdx.x < D) {
#pragma unroll 8
        for (int r = 0; r < kFoldRows; ++r) acc = acc + sf[r * D + threadIdx.x];
      }
    }
    if ((int)threadIdx.x < D) bp[threadIdx.x] = acc;
    __syncthreads();
  }
}

// Merged gradient of a unique row (inputs m).
template <int D>
__device__ __forceinline__ void small_grad(const Work& w, const uint32_t* __restrict__ sval, uint32_t direct,
                                           const uint4& m, GradRows<D> gr, int nblk, int g, float (&acc)[8]) {
  constexpr int U = 4;
  const uint32_t n = m.w;
  if (n == 1) {
    load_row<D>(gr.row(m.z), g, acc);
  } else if (n <= direct) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = -0.0f;
    for (uint32_t j = 0; j < n; j += U) {
      uint32_t b[U];
      float x[U][8];
#pragma unroll
      for (int q = 0; q < U; ++q) b[q] = sval[m.z + min(j + q, n - 1)];
#pragma unroll
      for (int q = 0; q < U; ++q) load_row<D>(gr.row(b[q]), g, x[q]);
#pragma unroll
      for (int q = 0; q < U; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = acc[i] + (j + q < n ? x[q][i] : -0.0f);
    }
  } else if (n <= kBlockAbove) {
    fold_chunks<D>(w.partial, m.y, (n + kSumChunk - 1) / kSumChunk, g, acc);
  } else if (nblk <= kFoldInline) {
    fold_flagged<D>(w, m.y, nblk, g, acc);
  } else {
    load_row<D>(w.bpart + (int64_t)m.y * w.max_nblk * D, g, acc);
  }
}

// One row group per unique row.  An insert reads the resident of its way, applies that row's
// own update if it has one (LFU and direct-mapped caches: a row updated this step and then
// displaced), writes it back to T and takes the way; a way is touched by one row alone.
template <int D, int BITS, bool SB16>
__global__ __launch_bounds__(256) void k_apply(Dev dv, Work w, const uint32_t* __restrict__ sval,
                                               const float* __restrict__ grad, uint32_t step, int nblk, uint32_t direct) {
  __shared__ TabPrefix P;
  constexpr int LPR = Geo<D>::LPR, GPB = 256 / LPR;
  if (!tab_prefix(P, w.tab_info, dv.T, [](const TabInfo& x) { return x.rows; })) return;
  const int g = threadIdx.x & (LPR - 1);
  const bool sr = dv.rounding != 0;
  const uint32_t nU = P.pre[dv.T];
  for (uint32_t i = blockIdx.x * GPB + threadIdx.x / LPR; i < nU; i += gridDim.x * GPB) {
    const int t = tab_of(P, dv.T, i);
    const uint32_t u = w.tab_info[t].pos + i - P.pre[t];
    const int32_t act = w.uact[u];
    const uint4 m = w.umeta[u];
    const int32_t slot = w.uslot[u];
    if (act == kActDone) continue;
    const int64_t row_base = dv.desc[t].row_base;
    const GradRows gtab = grad_rows<D>(grad, t, dv.T);
    const bool hit = act == kActHitStay, insert = act == kActInsert;
    const int64_t grow = m.x;
    uint8_t* rec = rec_of<D, BITS, SB16>(dv, grow);
    float x[8], gr[8];
    CodeWords<BITS> cw;
    SbWords<SB16> sbw;
    if (hit) {
      load_row<D>(dv.crow + (int64_t)slot * D, g, x);
    } else {
      if constexpr (kSplit<D>) cw = load_split_code_words<D, BITS>(rec, g);
      else cw = load_code_words<BITS>(rec, g);
      sbw = load_sb_words<D, BITS, SB16>(rec);
    }
    float* acc_in = nullptr;
    float* acc_out = nullptr;
    if (dv.optimizer) {
      acc_in = hit ? dv.acc_slot + slot : acc_of<D, BITS, SB16>(dv, grow, rec);
      acc_out = insert ? dv.acc_slot + slot : acc_in;
    }
    const float G_old = load_G(dv, acc_in);
    if (insert) {
      const int32_t vrow = w.uvic_row[u], vu = w.uvic_u[u];
      if (vrow >= 0) {
        const int64_t vgrow = row_base + vrow;
        uint8_t* vrec = rec_of<D, BITS, SB16>(dv, vgrow);
        float xv[8];
        load_row<D>(dv.crow + (int64_t)slot * D, g, xv);
        // the displaced row's accumulator leaves the slot for its record
        float* vacc = dv.optimizer ? acc_of<D, BITS, SB16>(dv, vgrow, vrec) : nullptr;
        const float Gv = dv.optimizer ? dv.acc_slot[slot] : 0.0f;
        if (vu >= 0) {
          float gv[8];
          small_grad<D>(w, sval, direct, w.umeta[vu], gtab, nblk, g, gv);
          apply_optimizer<D>(dv, xv, gv, vacc, g, Gv);
        } else if (dv.optimizer && g == 0) {
          *vacc = Gv;
        }
        quantize_store<D, BITS, SB16>(xv, g, vrec, sr, dv.seed, step, (uint32_t)t, (uint32_t)vrow);
      }
    }
    small_grad<D>(w, sval, direct, m, gtab, nblk, g, gr);
    if (!hit) {
      float sc, bi;
      decode_sb<SB16>(sbw, sc, bi);
      dequant8<BITS>(cw, sc, bi, x);
    }
    apply_optimizer<D>(dv, x, gr, acc_out, g, G_old);
    if (hit || insert) {
      store_row<D>(dv.crow + (int64_t)slot * D, g, x);
      if (insert && g == 0) {
        dv.tag[slot] = (int32_t)(grow - row_base);
        if (dv.policy == 0) dv.ts[slot] = (int32_t)step;
      }
    } else {
      quantize_store<D, BITS, SB16>(x, g, rec, sr, dv.seed, step, (uint32_t)t, (uint32_t)(grow - row_base));
    }
  }
}

// LFU decay, unless a table's offsets were rejected.
__global__ __launch_bounds__(256) void k_decay_small(int32_t* __restrict__ cnt, int64_t n,
                                                     const TabInfo* __restrict__ ti, int T) {
  bool bad = false;
  for (int t = threadIdx.x; t < T; t += 256) bad |= ti[t].bad != 0;
  if (__syncthreads_or(bad)) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) cnt[i] >>= 1;
}

hipError_t launch_backward_small(const Dev& d, const Work& w, const int32_t* idx, int64_t L, const int32_t* off,
                                 int32_t B, const float* grad, uint64_t step64, int passes, bool decay,
                                 const hipEvent_t* update_events, hipStream_t s, bool mid) {
  const uint32_t step = (uint32_t)step64;
  const int G = d.assoc <= 16 ? 16 : d.assoc <= 32 ? 32 : 64;
  const int nb_shift = __builtin_ctz((unsigned)(kBlockFloats / d.dim));
  const int nblk = (int)(((int64_t)B + (kBlockFloats / d.dim) - 1) >> nb_shift);
  if (nblk > w.max_nblk || d.T > kSmallTables || L > (mid ? kMidLookupsMost : kSmallLookups)) return hipErrorInvalidValue;
  const uint32_t* sval = w.valsB;
  if (mid) {
    const uint32_t* sk = nullptr;
    const hipError_t e = launch_mid_front(d, w, idx, L, off, B, passes, G, &sk, &sval, s);
    if (e != hipSuccess) return e;
    if (decay && d.cnt) k_decay_small<<<grid_for(d.total_rows), 256, 0, s>>>(d.cnt, d.total_rows, w.tab_info, d.T);
    const auto rows = [&](auto kernel, int per) {
      kernel<<<(unsigned)std::min<int64_t>((L + 256 * per - 1) / (256 * per), 1024), 256, 0, s>>>(d, w, sk, sval, step, nblk);
    };
    if (L < (1 << 19)) d.assoc <= 16 ? rows(k_mid_rows<16, 1>, 1) : rows(k_mid_rows<64, 1>, 1);
    else d.assoc <= 16 ? rows(k_mid_rows<16, 4>, 4) : rows(k_mid_rows<64, 4>, 4);
  } else {
    k_front<<<(unsigned)d.T, kFrontThreads, 0, s>>>(d, w, idx, L, off, B, passes, G, nblk);
    if (decay && d.cnt) k_decay_small<<<grid_for(d.total_rows), 256, 0, s>>>(d.cnt, d.total_rows, w.tab_info, d.T);
  }
  const uint32_t direct = mid ? kMidDirect : kSmallDirect;
  const int cshift = mid ? kMidChunkShift : kSmallChunkShift;
  return dispatch_row(d.dim, d.bits, d.sb16, [&]<int D, int BITS, bool SB16>() -> hipError_t {
    // a set or a row per lookup, a chunk per direct + 1 at most
    const auto blocks = [](int64_t items, int per, int64_t cap) {
      return (int)std::max<int64_t>(1, std::min<int64_t>((items + per - 1) / per, cap));
    };
    const int n_sum = blocks(L / (direct + 1) + 1, 256 / SumGeo<D>::GL, mid ? 1536 : 512);
    const int n_set = blocks(L, 256 / G, 1024);
    const auto decide = [&](auto kernel) {
      kernel<<<(unsigned)(n_sum + n_set), 256, 0, s>>>(d, w, sval, grad, step, nblk, nb_shift, cshift, n_sum);
    };
    if (G == 16) mid ? decide(k_decide<D, 16, true>) : decide(k_decide<D, 16, false>);
    else if (G == 32) mid ? decide(k_decide<D, 32, true>) : decide(k_decide<D, 32, false>);
    else mid ? decide(k_decide<D, 64, true>) : decide(k_decide<D, 64, false>);
    if (nblk > kFoldInline && L > (int64_t)kBlockAbove)
      k_fold<D><<<(unsigned)blocks(L / kBlockAbove, 1, 1024), 256, 0, s>>>(d, w, nblk);
    if (update_events) {
      const hipError_t e = hipEventRecord(update_events[0], s);
      if (e != hipSuccess) return e;
    }
    const int64_t cap = resident_grid(reinterpret_cast<const void*>(k_apply<D, BITS, SB16>));
    k_apply<D, BITS, SB16><<<(unsigned)blocks(L, 256 / Geo<D>::LPR, cap), 256, 0, s>>>(d, w, sval, grad, step, nblk, direct);
    if (update_events) {
      const hipError_t e = hipEventRecord(update_events[1], s);
      if (e != hipSuccess) return e;
    }
    return hipGetLastError();
  });
}

}  // namespace embc
