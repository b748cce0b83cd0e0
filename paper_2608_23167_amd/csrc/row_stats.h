// Row statistics shared by the float32 and bfloat16 LM heads: the order of
// candidate tokens, softmax partials and the block-wide top-k of a row.
#pragma once

#include "common.h"

namespace ssm {

constexpr int STAT_K = 8;                 // longest top-k list
constexpr int STAT_NONE = 0x7fffffff;     // id of an empty list entry (value -inf)

// Candidate order: larger value first, then lower id.
__device__ __forceinline__ bool stat_better(float v, int i, float w, int j) {
  return v > w || (v == w && i < j);
}

// Inserts (v, i) into the descending list (tv, ti).
__device__ __forceinline__ void stat_insert(float (&tv)[STAT_K], int (&ti)[STAT_K], float v, int i) {
#pragma unroll
  for (int q = 0; q < STAT_K; ++q) {
    const bool gt = stat_better(v, i, tv[q], ti[q]);
    const float ov = tv[q];
    const int oi = ti[q];
    tv[q] = gt ? v : ov;
    ti[q] = gt ? i : oi;
    v = gt ? ov : v;
    i = gt ? oi : i;
  }
}

// Float bits as a signed integer in the order of the values (-0 as +0; not
// for NaN), and back.
__device__ __forceinline__ int ordered_bits(float v) {
  const int b = __float_as_int(v + 0.0f);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float ordered_float(int o) {
  return __int_as_float(o ^ ((o >> 31) & 0x7fffffff));
}

// (max, sum of exp(x - max)) pairs: s == 0 is an empty one.
__device__ __forceinline__ void stat_combine(float& m, float& s, float om, float os) {
  if (!(os > 0.f)) return;
  if (!(s > 0.f)) { m = om; s = os; return; }
  const float M = fmaxf(m, om);
  s = s * expf(m - M) + os * expf(om - M);
  m = M;
}

struct __attribute__((aligned(16))) RowStatShared {
  long long key[256];
  float m[4], s[4], cv[64], bv[STAT_K], tv;
  int ci[64], bi[STAT_K], ti;
};

// Block-wide end of a row's statistics (256 threads): thread t brings the
// (max, sum) pair of its part of the row and the best (value, id) in it, and
// fill(tv, ti, floor_v, floor_i) lists its candidates that are not worse than
// the floor, best first.  The 8 best of the row all come from the 8 threads
// whose best ranks first (any other thread has 8 values ahead of all its
// own), so only those list theirs; the ranks of the threads, and of the 64
// values they hand over, are counts over LDS instead of a chain of 8
// block-wide searches.  Every result is independent of the order of events.
template <class Fill>
__device__ __forceinline__ void row_stats_end(RowStatShared& sh, float m, float s, float v, int i,
                                              int row, int k, int32_t* argmax, float* conf,
                                              int32_t* topk_ids, float* topk_w, Fill fill) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // id STAT_NONE sorts last among -inf
  const long long key = ((long long)ordered_bits(v) << 32) | (unsigned)(STAT_NONE - i);
  sh.key[tid] = key;
  if (tid < 64) { sh.cv[tid] = -INFINITY; sh.ci[tid] = STAT_NONE; }
  if (tid < STAT_K) { sh.bv[tid] = -INFINITY; sh.bi[tid] = STAT_NONE; }
  if (tid == 0) { sh.tv = -INFINITY; sh.ti = STAT_NONE; }
  // (max, sum) pairs: a butterfly within each wave (both partners compute the
  // same sum, in either order), then the 4 waves in order
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float om = __shfl_xor(m, o, 64), os = __shfl_xor(s, o, 64);
    stat_combine(m, s, om, os);
  }
  if (lane == 0) { sh.m[wave] = m; sh.s[wave] = s; }
  __syncthreads();
  int rank = 0;
  const longlong2* keys = (const longlong2*)sh.key;
#pragma unroll 16
  for (int u = 0; u < 128; ++u) {
    const longlong2 k2 = keys[u];
    rank += (k2.x > key) + (k2.y > key);
  }
  const bool lists = rank < STAT_K && i != STAT_NONE;   // ids are unique
  if (lists && rank == STAT_K - 1) { sh.tv = v; sh.ti = i; }
  __syncthreads();
  if (lists) {
    float tv[STAT_K];
    int ti[STAT_K];
#pragma unroll
    for (int q = 0; q < STAT_K; ++q) { tv[q] = -INFINITY; ti[q] = STAT_NONE; }
    fill(tv, ti, sh.tv, sh.ti);
#pragma unroll
    for (int q = 0; q < STAT_K; ++q) {
      sh.cv[STAT_K * rank + q] = tv[q];
      sh.ci[STAT_K * rank + q] = ti[q];
    }
  }
  __syncthreads();
  if (tid < 64) {
    const float cv = sh.cv[tid];
    const int ci = sh.ci[tid];
    int r = 0;
#pragma unroll 16
    for (int u = 0; u < 64; ++u) r += stat_better(sh.cv[u], sh.ci[u], cv, ci);
    if (r < STAT_K && ci != STAT_NONE) { sh.bv[r] = cv; sh.bi[r] = ci; }
  }
  __syncthreads();
  if (tid == 0) {
    float M = sh.m[0], S = sh.s[0];
    for (int w = 1; w < 4; ++w) stat_combine(M, S, sh.m[w], sh.s[w]);
    argmax[row] = sh.bi[0];
    // exp(max - max) / sum exp(x - max): NaN for a best value of +inf, whose
    // share of the partial sums stat_combine drops (inf - inf)
    conf[row] = (sh.bv[0] == INFINITY ? __builtin_nanf("") : 1.0f) / S;
    float e[STAT_K], z = 0.f;
#pragma unroll
    for (int q = 0; q < STAT_K; ++q) {
      e[q] = expf(sh.bv[q] - sh.bv[0]);
      if (q < k) z += e[q];
    }
#pragma unroll
    for (int q = 0; q < STAT_K; ++q)
      if (q < k) {
        topk_ids[(size_t)row * k + q] = sh.bi[q];
        topk_w[(size_t)row * k + q] = e[q] / z;
      }
  }
}

}  // namespace ssm
