// Row-level device code shared by the kernels of the training step: gradient rows and
// their sums, the optimizer, and the bookkeeping of the replacement decisions.
#pragma once

#include "embc_device.h"

namespace embc {

constexpr int32_t kActDone = 4;  // row handled by the row that displaces it

// what the update does with a row
constexpr uint32_t kKindHit = 0, kKindInsert = 1, kKindBypass = 2, kKindDone = 3;

constexpr int kUnroll = 2;  // independent row loads in flight per row group

// ---- merged gradient ----------------------------------------------------------------------
// Gradient rows of table t: grad_out is [B][T][d], so bag b's row is row b*T + t (an
// index below 2^32: B*T < 2^32 is checked when the handle is created).
template <int D>
struct GradRows {
  const float* grad;
  uint32_t T, t;
  __device__ const float* row(uint32_t b) const { return grad + (int64_t)(b * T + t) * D; }
};

template <int D>
__device__ __forceinline__ GradRows<D> grad_rows(const float* grad, int t, int T) {
  return GradRows<D>{grad, (uint32_t)T, (uint32_t)t};
}

// Left-to-right sum of the gradient rows of occurrences [i0, i1) of the sorted
// stream (i0 < i1), seeded with the first.  Lane j of the group preloads the bag of
// occurrence j of each run of LPR occurrences (for the first run the caller may pass
// them in, myv0); U rows are loaded before they are added in order.
// Rows narrower than 16 lanes (d < 128) hold kRun/LPR bags per lane, so that a run (one
// load of bags) covers kRun occurrences whatever the width, with kSmallUnroll rows in
// flight; the order of the additions is the same.
constexpr int kRun = 16;
constexpr int kSmallUnroll = 8;

template <int D>
__device__ __forceinline__ void sum_occ(const uint32_t* __restrict__ sval, int64_t i0, int64_t i1, GradRows<D> gr,
                                        int g, float (&acc)[8], uint32_t myv0 = 0u, bool have0 = false) {
  constexpr int LPR = Geo<D>::LPR, CPL = 8, U = kUnroll;
  if constexpr (LPR < kRun) {
    constexpr int BPL = kRun / LPR, US = kSmallUnroll;
    bool first = true;
    for (int64_t ic = i0; ic < i1; ic += kRun) {
      const int n = (int)min<int64_t>(kRun, i1 - ic);
      // occurrence j of the run: bag myv[j / LPR] of lane j % LPR
      uint32_t myv[BPL];
#pragma unroll
      for (int b = 0; b < BPL; ++b) {
        const int64_t i = ic + b * LPR + g;
        myv[b] = (b == 0 && have0 && ic == i0) ? myv0 : (i < i1 ? sval[i] : 0u);
      }
#pragma unroll
      for (int j0 = 0; j0 < kRun; j0 += US) {
        if (j0 >= n) break;
        float x[US][CPL];
#pragma unroll
        for (int q = 0; q < US; ++q) {
          const int j = j0 + q;
          if (j < n) load_row<D>(gr.row(__shfl(myv[j / LPR], j % LPR, LPR)), g, x[q]);
        }
#pragma unroll
        for (int q = 0; q < US; ++q) {
          if (j0 + q >= n) break;
          if (first) {
#pragma unroll
            for (int k = 0; k < CPL; ++k) acc[k] = x[q][k];
            first = false;
          } else {
#pragma unroll
            for (int k = 0; k < CPL; ++k) acc[k] = acc[k] + x[q][k];
          }
        }
      }
    }
    return;
  }
  bool first = true;
  for (int64_t ic = i0; ic < i1; ic += LPR) {
    const int n = (int)min<int64_t>(LPR, i1 - ic);
    // the first run's values may have been loaded by the caller (have0)
    const uint32_t myv = (have0 && ic == i0) ? myv0 : (g < n ? sval[ic + g] : 0u);
    int j = 0;
    if (first) {
      load_row<D>(gr.row(__shfl(myv, 0, LPR)), g, acc);
      first = false;
      j = 1;
    }
    for (; j + U <= n; j += U) {
      float x[U][CPL];
#pragma unroll
      for (int q = 0; q < U; ++q) load_row<D>(gr.row(__shfl(myv, j + q, LPR)), g, x[q]);
#pragma unroll
      for (int q = 0; q < U; ++q)
#pragma unroll
        for (int k = 0; k < CPL; ++k) acc[k] = acc[k] + x[q][k];
    }
    for (; j < n; ++j) {
      float x[CPL];
      load_row<D>(gr.row(__shfl(myv, j, LPR)), g, x);
#pragma unroll
      for (int k = 0; k < CPL; ++k) acc[k] = acc[k] + x[k];
    }
  }
}

// Left-to-right fold of the n >= 1 chunk sums of one row, rows c0 .. c0+n-1 of
// `partial` (acc = p0, then acc + p1, ...), U rows loaded before they are added.
template <int D>
__device__ __forceinline__ void fold_chunks(const float* __restrict__ partial, int64_t c0, uint32_t n, int g,
                                            float (&acc)[8]) {
  constexpr int U = kUnroll;
  load_row<D>(partial + c0 * D, g, acc);
  uint32_t j = 1;
  for (; j + U <= n; j += U) {
    float x[U][8];
#pragma unroll
    for (int q = 0; q < U; ++q) load_row<D>(partial + (c0 + j + q) * D, g, x[q]);
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = acc[k] + x[q][k];
  }
  for (; j < n; ++j) {
    float x[8];
    load_row<D>(partial + (c0 + j) * D, g, x);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = acc[k] + x[k];
  }
}

// ---- optimizer (FP32) -----------------------------------------------------------------------
// SGD: x = fma(-lr, g, x).  Row-wise Adagrad: S = halving-tree sum of g_j^2
// (a[j] += a[j + h] for h = D/2, ..., 1, the pairs of columns taken across or inside
// the lanes as the row layout places them), G += S * (1/D), r = lr / (sqrt(G) + eps),
// x = fma(-r, g, x).
template <int D>
__device__ __forceinline__ void apply_optimizer(const Dev& dv, float (&x)[8], const float (&gr)[8], float* acc,
                                                int g, float G_old) {
  constexpr int LPR = Geo<D>::LPR;
  if (dv.optimizer == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __builtin_fmaf(-dv.lr, gr[i], x[i]);
    return;
  }
  // the halving tree over the row's squares, in the lanes' column layout
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = gr[i] * gr[i];
  if constexpr (kSplit<D>) {
    // h = D/2 pairs element i with i + 4 of the same lane; h = D/4 .. 4 pairs lanes
    // g and g ^ (h/4); h = 2, 1 are inside the lane
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = a[i] + a[i + 4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = butterfly<LPR>(a[i], [](float p, float q) { return p + q; });
#pragma unroll
    for (int h = 2; h >= 1; h >>= 1)
#pragma unroll
      for (int i = 0; i < h; ++i) a[i] = a[i] + a[i + h];
  } else {
    // h = D/2 .. 8 pairs lanes g and g ^ (h/8); h = 4, 2, 1 are inside the lane
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = butterfly<LPR>(a[i], [](float p, float q) { return p + q; });
#pragma unroll
    for (int h = 4; h >= 1; h >>= 1)
#pragma unroll
      for (int i = 0; i < h; ++i) a[i] = a[i] + a[i + h];
  }
  const float Gn = G_old + a[0] * (1.0f / (float)D);
  if (g == 0) *acc = Gn;
  const float rate = dv.lr / (__builtin_sqrtf(Gn) + dv.eps);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = __builtin_fmaf(-rate, gr[i], x[i]);
}

// A row's Adagrad accumulator: in the slot array while the row is cached, in its record
// otherwise (it moves with the row on an insert and an eviction).
__device__ __forceinline__ float load_G(const Dev& dv, const float* acc) {
  return dv.optimizer ? *acc : 0.0f;
}

// ---- replacement decision -------------------------------------------------------------------
struct PolicyLds {
  int32_t hitu[64];       // unique row that hit way w this step, or -1
  int32_t cand_u[64];     // candidates by rank
  long long cand_pv[64];
  int32_t vic_way[64];    // victims by rank
  long long vic_pv[64];
};

// Statistics of the sets a row group handles, accumulated while the table does not change.
struct PolicyStats {
  static constexpr int kN = 6;
  int t = -1;
  uint32_t ins = 0, byp = 0, ev = 0, em = 0, he = 0, hits = 0;
  __device__ static int field(int i) {
    constexpr int f[kN] = {kStUniqueHits, kStInserts, kStBypasses, kStEvictions, kStEmptyFills, kStHitEvictions};
    return f[i];
  }
  __device__ void get(uint32_t (&v)[kN]) const {
    v[0] = hits; v[1] = ins; v[2] = byp; v[3] = ev; v[4] = em; v[5] = he;
  }
  __device__ void flush(const Dev& dv) {
    if (t < 0) return;
    unsigned long long* s = stat_of(dv, t);
    uint32_t v[kN];
    get(v);
    for (int i = 0; i < kN; ++i)
      if (v[i]) atomicAdd(s + field(i), (unsigned long long)v[i]);
    ins = byp = ev = em = he = hits = 0;
  }
  // At the end, by the whole workgroup: the groups (each by its leader lane) of one table as
  // the workgroup's first group are summed in LDS and added once; the others add their own.
  __device__ void flush_workgroup(const Dev& dv, bool leader, int32_t* tab_s, uint32_t* sums_s) {
    if (threadIdx.x == 0) *tab_s = t;
    if (threadIdx.x < kN) sums_s[threadIdx.x] = 0;
    __syncthreads();
    if (leader && t >= 0) {
      if (t == *tab_s) {
        uint32_t v[kN];
        get(v);
        for (int i = 0; i < kN; ++i)
          if (v[i]) atomicAdd(&sums_s[i], v[i]);
      } else {
        flush(dv);
      }
    }
    __syncthreads();
    if (threadIdx.x < kN && sums_s[threadIdx.x])
      atomicAdd(stat_of(dv, *tab_s) + field(threadIdx.x), (unsigned long long)sums_s[threadIdx.x]);
  }
};

}  // namespace embc
