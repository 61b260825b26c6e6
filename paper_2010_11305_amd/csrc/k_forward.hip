// State reset, uniform initialisation, and the forward pass:
// pooled[b][t] = sum over the bag of fetch(T_t, C_t, i) (Sec. 3 fetch operator).
#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>

#include "emb_cache.h"
#include "embc_device.h"
#include "embc_dispatch.h"
#include "embc_offsets.h"
#include "embc_sort.h"

namespace embc {

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill_u32<<<grid_for(n), 256, 0, s>>>(p, v, n);
  return hipGetLastError();
}

hipError_t launch_reset_state(const Dev& d, hipStream_t s) {
  hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.rec), 0u, d.total_rows * d.rec_bytes / 4, s);
  if (e == hipSuccess) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.crow), 0u, d.total_slots * d.dim, s);
  if (e == hipSuccess) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.tag), 0xFFFFFFFFu, d.total_slots, s);
  if (e == hipSuccess && d.ts) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.ts), 0xFFFFFFFFu, d.total_slots, s);
  if (e == hipSuccess && d.cnt) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.cnt), 0u, d.total_rows, s);
  if (e == hipSuccess && d.acc_slot) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.acc_slot), 0u, d.total_slots, s);
  if (e == hipSuccess && d.acc_rows) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.acc_rows), 0u, d.total_rows, s);
  if (e == hipSuccess) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.stats), 0u,
                                           ((int64_t)d.T << d.stat_shift) * kStatStride * 2, s);
  if (e == hipSuccess) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.err), 0u, 1, s);
  return e;
}

// Table owning global row `grow` (binary search over row_base).
__device__ __forceinline__ int table_of_row(const Dev& dv, int64_t grow) {
  int lo = 0, hi = dv.T;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (grow >= dv.desc[mid].row_base) lo = mid; else hi = mid;
  }
  return lo;
}

// x_j = u*(hi-lo) + lo (fused), u = Philox uniform keyed (init_seed; j/4, row, table, 0xFFFFFFFF),
// then nearest-even quantization of the row; its Adagrad accumulator (if any) to 0.
template <int D, int BITS, bool SB16>
__global__ __launch_bounds__(256) void k_init_uniform(Dev dv, float lo, float hi, uint64_t init_seed) {
  constexpr int LPR = Geo<D>::LPR;
  const int g = threadIdx.x & (LPR - 1);
  const int64_t ngroups = (int64_t)gridDim.x * blockDim.x / LPR;
  const float width = hi - lo;
  for (int64_t grow = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / LPR; grow < dv.total_rows;
       grow += ngroups) {
    const int t = table_of_row(dv, grow);
    const uint32_t r = (uint32_t)(grow - dv.desc[t].row_base);
    float u[8], x[8];
    uniforms_row<D>(init_seed, 0xFFFFFFFFu, (uint32_t)t, r, g, u);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __builtin_fmaf(u[i], width, lo);
    uint8_t* rec = rec_of<D, BITS, SB16>(dv, grow);
    quantize_store<D, BITS, SB16>(x, g, rec, false, 0, 0, 0, 0);
    if (dv.optimizer && g == 0) *acc_of<D, BITS, SB16>(dv, grow, rec) = 0.0f;
  }
}

// Row-wise Adagrad: the accumulators of the rows cached in slots [s0, s0 + n) of the table
// whose rows start at row_base, moved from the slots to the records (to_rec) or back.
__global__ __launch_bounds__(256) void k_move_acc(Dev dv, int64_t s0, int64_t n, int64_t row_base, bool to_rec) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int32_t r = dv.tag[s0 + i];
    if (r < 0) continue;
    float* a = dv.acc_rows ? dv.acc_rows + row_base + r
                           : reinterpret_cast<float*>(dv.rec + (row_base + r) * dv.rec_bytes + dv.acc_offset);
    if (to_rec) *a = dv.acc_slot[s0 + i];
    else dv.acc_slot[s0 + i] = *a;
  }
}

hipError_t launch_move_acc(const Dev& d, int64_t slot0, int64_t slots, int64_t row_base, bool to_rec, hipStream_t s) {
  if (!d.acc_slot || slots <= 0) return hipSuccess;
  k_move_acc<<<grid_for(slots), 256, 0, s>>>(d, slot0, slots, row_base, to_rec);
  return hipGetLastError();
}

hipError_t launch_init_uniform(const Dev& d, float lo, float hi, uint64_t init_seed, hipStream_t s) {
  hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.tag), 0xFFFFFFFFu, d.total_slots, s);
  if (e == hipSuccess && d.ts) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.ts), 0xFFFFFFFFu, d.total_slots, s);
  if (e == hipSuccess) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.crow), 0u, d.total_slots * d.dim, s);
  if (e == hipSuccess && d.cnt) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.cnt), 0u, d.total_rows, s);
  if (e == hipSuccess && d.acc_slot) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.acc_slot), 0u, d.total_slots, s);
  if (e == hipSuccess && d.acc_rows) e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.acc_rows), 0u, d.total_rows, s);
  if (e != hipSuccess) return e;
  return dispatch_row(d.dim, d.bits, d.sb16, [&]<int D, int BITS, bool SB16>() -> hipError_t {
    const int64_t threads = d.total_rows * Geo<D>::LPR;
    k_init_uniform<D, BITS, SB16><<<grid_for(threads, 16384), 256, 0, s>>>(d, lo, hi, init_seed);
    return hipGetLastError();
  });
}

// ---- forward --------------------------------------------------------------------------
// Two passes.  k_fwd_probe: one lane per lookup up to 8 ways, 2 lanes for 16 or 32, 4 for 64,
// checks the row, probes its set, and write a code: the cache slot (hit), -2-row (miss) or
// -1 (skipped).  k_fwd_gather: one group of LPR
// lanes per bag (64/LPR bags per wave), tables split over the XCDs; lane j reads the
// code of position j of each chunk of LPR positions, the rows are fetched FU at a time
// (all FU loads issued before any is used) and summed left to right.  A bag with no
// valid lookup gives +0.
// Both take their work flat: the positions (probe) and tiles of 256/LPR bags (gather) of all
// tables, one contiguous run per XCD, so that a call of few bags per table, or of a number of
// tables that is no multiple of 8, still fills every XCD.  With one table at a time per XCD,
// 100 tables of 512 bags (1.5M lookups) took 275 us and take 79; 10 tables of 16384 bags
// 307 and 205; full tables are as before (100 tables of 16384 bags: 1.78 ms).
constexpr int kFwdUnroll = 2;

// Lookups in flight per lane group of the probe (PU).  On a large step 6 (96 tags per
// lane, 2 waves per SIMD) is faster than 4 at 4 waves (355 -> 332 us on the industrial
// workload; 8: 334 us, 12: 531 us); a step of few lookups wants the waves instead.
constexpr int kProbeUnroll = 6, kProbeUnrollSmall = 4;
constexpr int kProbeSums = 64;  // tables of a range whose counts a workgroup gathers in LDS
constexpr int64_t kProbeSmallBelow = 1 << 21;  // lookups per call

// QL = assoc/W lanes share one lookup (W = assoc up to 8 ways, 8 at 16 ways, 16 beyond),
// each comparing W of the set's tags loaded 16 bytes at a time; every lane group keeps
// PU lookups in flight (all index loads, then all tag loads).  At 16 ways two lanes of 8
// tags are faster than one of 16 (industrial probe 331 -> 303 us: a wave's tag loads
// then touch 32 sets' lines each instead of 64), four of 4 slower (439 us); at 32 ways four
// lanes of 8 are slower than two of 16 (stress workload 86 -> 127 us).
template <int W, int PU>
__global__ __launch_bounds__(256) void k_fwd_probe(Dev dv, const int32_t* __restrict__ idx, int64_t L,
                                                   const int32_t* __restrict__ off, int32_t B,
                                                   int32_t* __restrict__ src) {
  __shared__ uint32_t sums[kProbeSums][3];  // counts of the range's first tables
  for (int i = threadIdx.x; i < 3 * kProbeSums; i += blockDim.x) sums[i / 3][i % 3] = 0;
  __syncthreads();
  const int64_t pfirst = min<int64_t>(max<int64_t>(off[0], 0), L);
  const int64_t plast = min<int64_t>(max<int64_t>(off[(int64_t)dv.T * B], pfirst), L);
  if (blockIdx.x == 0) {
    // positions outside every bag are skipped
    for (int64_t p = threadIdx.x; p < pfirst; p += blockDim.x) src[p] = -1;
    for (int64_t p = plast + threadIdx.x; p < L; p += blockDim.x) src[p] = -1;
  }
  // workgroup -> contiguous range of positions, XCD-major
  const int64_t place = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  int64_t pa, pb;
  part_range(pfirst, plast, (int)place, (int)gridDim.x, pa, pb);
  const int A = dv.assoc;
  const int QL = A / W;  // 1 up to 16 ways, 2 or 4 for 32 or 64
  const int sub = threadIdx.x % QL;
  const int64_t ptid = threadIdx.x / QL, pstride = blockDim.x / QL;
  // the range's first table: the last one that starts at or before it, searched by the
  // whole wave (64 tables per round; with malformed offsets some table, or none, is found)
  int t0 = 0;
  for (int hi = dv.T; hi - t0 > 1;) {
    const int step = (hi - t0 + 63) / 64, c = t0 + (int)(threadIdx.x & 63) * step;
    const uint64_t le = __ballot(c == t0 || (c < hi && off[(int64_t)c * B] <= pa));
    t0 += (63 - (int)__clzll((unsigned long long)le)) * step;
    hi = min(hi, t0 + step);
  }
  for (int t = t0; t < dv.T; ++t) {
    const TableDesc td = dv.desc[t];
    const int64_t a = min<int64_t>(max<int64_t>(off[(int64_t)t * B], 0), L);
    const int64_t b = min<int64_t>(max<int64_t>(off[(int64_t)(t + 1) * B], a), L);
    if (a >= pb) break;
    const int64_t lo = max<int64_t>(a, pa), hi = min<int64_t>(b, pb);
    const int32_t* tags = dv.tag + td.slot_base + sub * W;
    uint32_t ok = 0, hit = 0, bad = 0;
    // the index loads run one iteration ahead of the tag loads, and every load is
    // unconditional (a position past hi re-reads position lo, an invalid row probes
    // set 0), so an iteration's tags are waited for with the next indices in flight
    int32_t rn[PU];
    if (lo + ptid < hi) {
#pragma unroll
      for (int q = 0; q < PU; ++q) {
        const int64_t p = lo + ptid + q * pstride;
        rn[q] = idx[p < hi ? p : lo];
      }
    }
    for (int64_t p0 = lo + ptid; p0 < hi; p0 += pstride * PU) {
      int32_t r[PU], found[PU];
      bool valid[PU];
      int32_t tw[PU][W];
#pragma unroll
      for (int q = 0; q < PU; ++q) {
        r[q] = rn[q];
        valid[q] = p0 + q * pstride < hi && r[q] >= 0 && (int64_t)r[q] < td.N;
        found[q] = -1;
      }
      if (td.n_sets > 0) {
#pragma unroll
        for (int q = 0; q < PU; ++q) {
          const int64_t set = valid[q] ? (int64_t)mod_by((uint32_t)r[q], td.by_sets) : 0;
          const int32_t* tg = tags + set * A;
          if constexpr (W % 4 == 0) {
#pragma unroll
            for (int k = 0; k < W; k += 4) {
              const int4 v = *reinterpret_cast<const int4*>(tg + k);
              tw[q][k] = v.x; tw[q][k + 1] = v.y; tw[q][k + 2] = v.z; tw[q][k + 3] = v.w;
            }
          } else if constexpr (W == 2) {
            const int2 v = *reinterpret_cast<const int2*>(tg);
            tw[q][0] = v.x; tw[q][1] = v.y;
          } else {
            tw[q][0] = tg[0];
          }
        }
      }
      // the next iteration's indices
      {
        const int64_t pn = p0 + pstride * PU;
#pragma unroll
        for (int q = 0; q < PU; ++q) {
          const int64_t p = pn + q * pstride;
          rn[q] = idx[p < hi ? p : lo];
        }
      }
      if (td.n_sets > 0) {
#pragma unroll
        for (int q = 0; q < PU; ++q) {
          const int64_t set = valid[q] ? (int64_t)mod_by((uint32_t)r[q], td.by_sets) : 0;
#pragma unroll
          for (int k = 0; k < W; ++k)
            if (valid[q] && tw[q][k] == r[q]) found[q] = (int32_t)(td.slot_base + set * A + sub * W + k);
        }
      }
#pragma unroll
      for (int q = 0; q < PU; ++q) {
        for (int o = 1; o < QL; o <<= 1) found[q] = max(found[q], __shfl_xor(found[q], o, QL));
        const int64_t p = p0 + q * pstride;
        if (sub == 0 && p < hi) {
          src[p] = valid[q] ? (found[q] >= 0 ? found[q] : -2 - r[q]) : -1;
          ok += valid[q];
          hit += found[q] >= 0;
          bad += !valid[q];
        }
      }
    }
    // statistics of the table, gathered in LDS for the workgroup
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ok += __shfl_xor(ok, o);
      hit += __shfl_xor(hit, o);
      bad += __shfl_xor(bad, o);
    }
    if ((threadIdx.x & 63) == 0) {
      const int i = t - t0;
      if (i < kProbeSums) {
        if (ok) atomicAdd(&sums[i][0], ok);
        if (hit) atomicAdd(&sums[i][1], hit);
        if (bad) atomicAdd(&sums[i][2], bad);
      } else {
        unsigned long long* st = stat_of(dv, t);
        if (ok) atomicAdd(st + kStLookups, (unsigned long long)ok);
        if (hit) atomicAdd(st + kStHitLookups, (unsigned long long)hit);
        if (bad) atomicAdd(st + kStInvalidFwd, (unsigned long long)bad);
      }
      if (bad) atomicOr(dv.err, kErrIndex);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 3 * kProbeSums; i += blockDim.x) {
    const uint32_t v = sums[i / 3][i % 3];
    const int f = i % 3 == 0 ? kStLookups : i % 3 == 1 ? kStHitLookups : kStInvalidFwd;
    if (v) atomicAdd(stat_of(dv, t0 + i / 3) + f, (unsigned long long)v);
  }
}

template <int D, int BITS, bool SB16>
__global__ __launch_bounds__(256) void k_fwd_gather(Dev dv, const int32_t* __restrict__ src, int64_t L,
                                                    const int32_t* __restrict__ off, int32_t B, DivConst per_table,
                                                    int tile_bags, float* __restrict__ out) {
  constexpr int LPR = Geo<D>::LPR, FU = kFwdUnroll;
  const int64_t RB = dv.rec_bytes;
  const int g = threadIdx.x & (LPR - 1);
  // tiles of tile_bags (at most GPB) bags of one table, table-major: a contiguous run of
  // tiles per XCD, which its workgroups walk side by side
  const int xcd = blockIdx.x % kXcds, unit = blockIdx.x / kXcds, units = gridDim.x / kXcds;
  const int64_t ntiles = (int64_t)per_table.d * dv.T;
  int64_t clo, chi;
  part_range(0, ntiles, xcd, kXcds, clo, chi);
  if (clo + unit >= chi) return;
  const auto tile_bag = [&](int64_t c, int& t) -> uint32_t {
    t = (int)div_by((uint32_t)c, per_table);
    return ((uint32_t)c - (uint32_t)t * per_table.d) * (uint32_t)tile_bags + threadIdx.x / LPR;
  };
  if ((int)threadIdx.x / LPR >= tile_bags) return;  // whole row groups; no barrier below
  const uint32_t last = (uint32_t)B - 1u;
  // the offsets of the group's next bag are loaded one tile ahead, the codes of the next
  // LPR positions one chunk ahead (indices clamped so that the loads are unconditional; a
  // clamped load is not used)
  int tn;
  uint32_t bn = tile_bag(clo + unit, tn);
  int64_t o0 = off[(int64_t)tn * B + min(bn, last)], o1 = off[(int64_t)tn * B + min(bn, last) + 1];
  int t = -1;
  const uint8_t* rec0 = nullptr;
  int32_t slot_lo = 0, slot_hi = 0, nrows = 0;
  for (int64_t c = clo + unit; c < chi; c += units) {
    {
      if (tn != t) {  // whole workgroup
        t = tn;
        // codes outside this table's slots and rows are skipped (only malformed offsets
        // produce them); slots, rows and positions are below 2^31 (32-bit arithmetic)
        const TableDesc& td = dv.desc[t];
        rec0 = dv.rec + td.row_base * RB;
        slot_lo = (int32_t)td.slot_base, slot_hi = (int32_t)(td.slot_base + td.n_sets * dv.assoc);
        nrows = (int32_t)td.N;
      }
      const uint32_t b = bn;
      const int64_t p0 = o0 < 0 ? 0 : o0;
      const int64_t p1 = o1 > L ? L : o1;
      bn = tile_bag(min<int64_t>(c + units, chi - 1), tn);
      {
        const int64_t nb = (int64_t)tn * B + min(bn, last);
        o0 = off[nb];
        o1 = off[nb + 1];
      }
      if (b > last) continue;  // past the table's last bag
      // the sum starts from -0, the identity of IEEE addition (adding the first term
      // gives exactly that term, as in the seeded left-to-right sum); a bag without a
      // valid lookup gives +0
      float acc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = -0.0f;
      bool any = false;
      int32_t code_next = p0 + g < p1 ? src[p0 + g] : -1;
      for (int64_t pc = p0; pc < p1; pc += LPR) {
        const int n = (int)min<int64_t>(LPR, p1 - pc);
        const int32_t code = code_next;
        code_next = pc + LPR + g < p1 ? src[pc + LPR + g] : -1;
        for (int j = 0; j < n; j += FU) {
          float raw[FU][8];
          RecRaw<D, BITS, SB16> rr[FU];
          int kind[FU];  // 0 skip, 1 cache row, 2 low-precision row
#pragma unroll
          for (int q = 0; q < FU; ++q) {
            const int32_t cq = __shfl(code, j + q, LPR);
            kind[q] = 0;
            if (j + q < n) {
              if (cq >= slot_lo && cq < slot_hi) kind[q] = 1;
              else if (cq <= -2 && -2 - cq < nrows) kind[q] = 2;
            }
            if (kind[q] == 1) {
              load_row<D>(dv.crow + (int64_t)cq * D, g, raw[q]);
            } else if (kind[q] == 2) {
              const uint8_t* rec = static_cast<const uint8_t*>(
                  __builtin_assume_aligned(rec0 + (int64_t)(-2 - cq) * RB, Rec<D, BITS, SB16>::ALIGN));
              rr[q] = load_rec_raw<D, BITS, SB16>(rec, g);  // unpacked after the loads
            }
          }
#pragma unroll
          for (int q = 0; q < FU; ++q) {
            if (kind[q] == 0) continue;
            if (kind[q] == 2) {
              CodeWords<BITS> cw;
              SbWords<SB16> sbw;
              rec_words_unpack<D, BITS, SB16>(rr[q], cw, sbw);
              float sq, bq;
              decode_sb<SB16>(sbw, sq, bq);
              dequant8<BITS>(row_code_words<D, BITS>(cw, g), sq, bq, raw[q]);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = acc[i] + raw[q][i];
            any = true;
          }
        }
      }
      if (!any) {
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.0f;
      }
      store_row_nt<D>(out + ((int64_t)b * dv.T + t) * D, g, acc);
    }
  }
}

// Zeroes the forward statistics and checks the offsets: one launch before the kernels that
// count.
__global__ __launch_bounds__(256) void k_fwd_begin(Dev dv, const int32_t* __restrict__ off, int64_t nbags, int64_t L) {
  zero_stats(dv, kStLookups, kStHitLookups);
  zero_stats(dv, kStInvalidFwd, kStInvalidFwd);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nbags; i += stride) {
    if (bad_range(off[i], off[i + 1], L)) atomicOr(dv.err, kErrOffsets);
  }
}

// ---- forward of small calls ------------------------------------------------------------------
// One kernel probes and gathers: a row group per bag; lane j of the group probes position j
// of each run of LPR positions (all the set's tags in flight), then the rows are fetched
// FU at a time and summed left to right, as in k_fwd_gather.  Such a call waits on its
// chain of dependent loads and on launches (about 5 us each): 26 tables of 256 one-lookup
// bags take 12 us in two launches against 18 in three, 12 tables of 1000 20-lookup bags
// (0.24M lookups) 19 against 25.  From about 0.3M lookups on the chip is full and two
// passes are faster, each with more waves in flight than this kernel's registers allow
// (0.49M lookups: 33 us against 27, 1.5M: 114 against 79).
// Bags are taken flat, table-major, in one contiguous range per XCD and per workgroup, so
// that a workgroup meets few tables and every XCD has the same number of bags.
constexpr int kFusedUnroll = 4;  // rows in flight per row group

template <int D, int BITS, bool SB16, int MAXA>
__global__ __launch_bounds__(256) void k_fwd_fused(Dev dv, const int32_t* __restrict__ idx, int64_t L,
                                                   const int32_t* __restrict__ off, int32_t B, DivConst byB,
                                                   float* __restrict__ out) {
  constexpr int LPR = Geo<D>::LPR, FU = kFusedUnroll, GPB = 256 / LPR;
  __shared__ uint32_t sum_s[4][3];
  __shared__ int tab_s[4];
  const int64_t RB = dv.rec_bytes;
  const int g = threadIdx.x & (LPR - 1);
  const int64_t nbags = (int64_t)dv.T * B;
  // workgroup -> contiguous range of bags, XCD-major
  const int64_t place = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  int64_t blo, bhi;
  part_range(0, nbags, (int)place, (int)gridDim.x, blo, bhi);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int t = -1;
  TableDesc td{};
  uint32_t n_ok = 0, n_hit = 0, n_bad = 0;
  const auto flush_lane = [&]() {  // a group that goes on to another table
    unsigned long long* st = stat_of(dv, t);
    if (n_ok) atomicAdd(st + kStLookups, (unsigned long long)n_ok);
    if (n_hit) atomicAdd(st + kStHitLookups, (unsigned long long)n_hit);
    if (n_bad) {
      atomicAdd(st + kStInvalidFwd, (unsigned long long)n_bad);
      atomicOr(dv.err, kErrIndex);
    }
    n_ok = n_hit = n_bad = 0;
  };
  for (int64_t gbag = blo + threadIdx.x / LPR; gbag < bhi; gbag += GPB) {
    const int tb = (int)div_by((uint32_t)gbag, byB);
    if (tb != t) {
      if (t >= 0) flush_lane();
      t = tb;
      td = dv.desc[t];
    }
    const int64_t o0 = off[gbag], o1 = off[gbag + 1];
    const int64_t p0 = o0 < 0 ? 0 : o0;
    const int64_t p1 = o1 > L ? L : o1;
    const uint8_t* rec0 = dv.rec + td.row_base * RB;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = -0.0f;
    bool any = false;
    for (int64_t pc = p0; pc < p1; pc += LPR) {
      const int n = (int)min<int64_t>(LPR, p1 - pc);
      int32_t code = -1;
      if (g < n) {
        const int32_t r = idx[pc + g];
        if (r >= 0 && (int64_t)r < td.N) {
          const int32_t sl = probe_slot<MAXA>(dv, td, r);
          code = sl >= 0 ? sl : -2 - r;
          ++n_ok;
          n_hit += sl >= 0;
        } else {
          ++n_bad;
        }
      }
      for (int j = 0; j < n; j += FU) {
        float raw[FU][8];
        RecRaw<D, BITS, SB16> rr[FU];
        int kind[FU];  // 0 skip, 1 cache row, 2 low-precision row
#pragma unroll
        for (int q = 0; q < FU; ++q) {
          const int32_t cq = __shfl(code, j + q, LPR);
          kind[q] = j + q < n ? (cq >= 0 ? 1 : cq <= -2 ? 2 : 0) : 0;
          if (kind[q] == 1) {
            load_row<D>(dv.crow + (int64_t)cq * D, g, raw[q]);
          } else if (kind[q] == 2) {
            const uint8_t* rec = static_cast<const uint8_t*>(
                __builtin_assume_aligned(rec0 + (int64_t)(-2 - cq) * RB, Rec<D, BITS, SB16>::ALIGN));
            rr[q] = load_rec_raw<D, BITS, SB16>(rec, g);
          }
        }
#pragma unroll
        for (int q = 0; q < FU; ++q) {
          if (kind[q] == 0) continue;
          if (kind[q] == 2) {
            CodeWords<BITS> cw;
            SbWords<SB16> sbw;
            rec_words_unpack<D, BITS, SB16>(rr[q], cw, sbw);
            float sq, bq;
            decode_sb<SB16>(sbw, sq, bq);
            dequant8<BITS>(row_code_words<D, BITS>(cw, g), sq, bq, raw[q]);
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[i] = acc[i] + raw[q][i];
          any = true;
        }
      }
    }
    if (!any) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = 0.0f;
    }
    const int64_t b = gbag - (int64_t)t * B;
    store_row_nt<D>(out + (b * dv.T + t) * D, g, acc);
  }
  // the last table's counts: one atomic per workgroup and counter (waves of one table)
  const uint64_t has = __ballot(t >= 0);
  const int t0 = has ? __shfl(t, (int)__builtin_ctzll(has)) : -1;
  if (t >= 0 && t != t0) flush_lane();
  if (n_bad) atomicOr(dv.err, kErrIndex);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    n_ok += __shfl_xor(n_ok, o);
    n_hit += __shfl_xor(n_hit, o);
    n_bad += __shfl_xor(n_bad, o);
  }
  if (lane == 0) {
    tab_s[wv] = t0;
    sum_s[wv][0] = n_ok;
    sum_s[wv][1] = n_hit;
    sum_s[wv][2] = n_bad;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int f = threadIdx.x == 0 ? kStLookups : threadIdx.x == 1 ? kStHitLookups : kStInvalidFwd;
    uint32_t run = 0;
    for (int w = 0; w < 4; ++w) {
      run += sum_s[w][threadIdx.x];
      if (w == 3 || tab_s[w + 1] != tab_s[w]) {
        if (run && tab_s[w] >= 0) atomicAdd(stat_of(dv, tab_s[w]) + f, (unsigned long long)run);
        run = 0;
      }
    }
  }
}

hipError_t launch_forward(const Dev& d, const Work& w, const int32_t* idx, int64_t L, const int32_t* off, int32_t B,
                          float* out, hipStream_t s) {
  const int64_t nbags = (int64_t)d.T * B;
  k_fwd_begin<<<grid_for(nbags, 2048), 256, 0, s>>>(d, off, nbags, L);
  if (nbags == 0) return hipGetLastError();
  if (fused_call(L, nbags, d.dim, d.assoc)) {
    const DivConst byB = div_const((uint32_t)B);
    return dispatch_row(d.dim, d.bits, d.sb16, [&]<int D, int BITS, bool SB16>() -> hipError_t {
      // (few bags are spread over 512 workgroups)
      const int64_t wgs = std::max<int64_t>((nbags * Geo<D>::LPR + 255) / 256, std::min<int64_t>(nbags, 512));
      const auto run = [&](auto kernel) {
        const int64_t cap = resident_grid(reinterpret_cast<const void*>(kernel));
        const int64_t blocks = std::min<int64_t>((wgs + 7) / 8 * 8, cap);
        kernel<<<(unsigned)blocks, 256, 0, s>>>(d, idx, L, off, B, byB, out);
      };
      if (d.assoc <= 16) run(k_fwd_fused<D, BITS, SB16, 16>);
      else run(k_fwd_fused<D, BITS, SB16, 64>);
      return hipGetLastError();
    });
  }
  if (L > 0) {
    const auto probe = [&](auto kernel, int lookups) {
      // a workgroup's round of lookups each, at most the resident count
      const int64_t cap = resident_grid(reinterpret_cast<const void*>(kernel));
      const int64_t blocks = std::min<int64_t>((L + lookups - 1) / lookups / 8 * 8 + 8, cap);
      kernel<<<(unsigned)blocks, 256, 0, s>>>(d, idx, L, off, B, w.fwd_src);
    };
    const auto probe_w = [&](auto pu) {
      constexpr int PU = decltype(pu)::value;
      // tags per lane: the whole set up to 8 ways, 8 of 16 (two lanes per lookup), 16 beyond
      switch (d.assoc <= 8 ? d.assoc : d.assoc == 16 ? 8 : 16) {
        case 1: probe(k_fwd_probe<1, PU>, 256 * 1 / d.assoc * PU); return hipSuccess;
        case 2: probe(k_fwd_probe<2, PU>, 256 * 2 / d.assoc * PU); return hipSuccess;
        case 4: probe(k_fwd_probe<4, PU>, 256 * 4 / d.assoc * PU); return hipSuccess;
        case 8: probe(k_fwd_probe<8, PU>, 256 * 8 / d.assoc * PU); return hipSuccess;
        case 16: probe(k_fwd_probe<16, PU>, 256 * 16 / d.assoc * PU); return hipSuccess;
        default: return hipErrorInvalidValue;
      }
    };
    const hipError_t e = L < kProbeSmallBelow ? probe_w(std::integral_constant<int, kProbeUnrollSmall>{})
                                              : probe_w(std::integral_constant<int, kProbeUnroll>{});
    if (e != hipSuccess) return e;
  }
  return dispatch_row(d.dim, d.bits, d.sb16, [&]<int D, int BITS, bool SB16>() -> hipError_t {
    // one tile per workgroup, in whole multiples of 8 workgroups, at most the resident count;
    // few bags are spread over 512 workgroups (16 long bags in one wave take 449 us, 344 on 8
    // workgroups)
    int tile_bags = 256 / Geo<D>::LPR;
    while (tile_bags > 1 && d.T * (((int64_t)B + tile_bags - 1) / tile_bags) < 512) tile_bags /= 2;
    const DivConst per_table = div_const((uint32_t)(((int64_t)B + tile_bags - 1) / tile_bags));
    const int64_t tiles = (int64_t)per_table.d * d.T;
    const int64_t cap = resident_grid(reinterpret_cast<const void*>(k_fwd_gather<D, BITS, SB16>));
    const int64_t blocks = std::min<int64_t>((tiles + 7) / 8 * 8, cap);
    k_fwd_gather<D, BITS, SB16><<<(unsigned)blocks, 256, 0, s>>>(d, w.fwd_src, L, off, B, per_table, tile_bags, out);
    return hipGetLastError();
  });
}

// ---- forward without a workspace ---------------------------------------------------------
// For callers that cannot allocate: the forward's per-call temporaries (one code per lookup) live
// in `scratch`, a static device array that every GPU the library runs on holds until the
// process ends; its first kNoAllocHeader bytes are not used (EMB_NOALLOC_MAX_INDICES leaves
// them out).  Host code never passes the array's name to a kernel (on the host it is only a
// stand-in): it passes the device address that hipGetSymbolAddress returns for the current
// device, looked up once per device.
constexpr size_t kNoAllocHeader = 256;
static_assert(EMB_NOALLOC_MAX_INDICES == (EMB_NOALLOC_SCRATCH_BYTES - kNoAllocHeader) / 4, "scratch layout");
static __device__ __align__(256) uint8_t scratch[EMB_NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(uint8_t** out) {
  static std::mutex mu;
  static std::map<int, uint8_t*> addr;  // device -> address of its copy of `scratch`
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  const auto it = addr.find(dev);
  if (it != addr.end()) {
    *out = it->second;
    return hipSuccess;
  }
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || p == nullptr) return e != hipSuccess ? e : hipErrorInvalidSymbol;
  addr[dev] = static_cast<uint8_t*>(p);
  *out = static_cast<uint8_t*>(p);
  return hipSuccess;
}

hipError_t launch_forward_noalloc(const Dev& d, uint8_t* scratch_dev, const int32_t* idx, int64_t L,
                                  const int32_t* off, int32_t B, float* out, hipStream_t s) {
  if (scratch_dev == nullptr || L < 0 || L > EMB_NOALLOC_MAX_INDICES) return hipErrorInvalidValue;
  // the same kernels as launch_forward; nothing in the scratch is read before it is written
  // in the same call, so it needs no clearing
  Work w{};
  w.fwd_src = reinterpret_cast<int32_t*>(scratch_dev + kNoAllocHeader);
  w.max_indices = EMB_NOALLOC_MAX_INDICES;
  return launch_forward(d, w, idx, L, off, B, out, s);
}

}  // namespace embc
