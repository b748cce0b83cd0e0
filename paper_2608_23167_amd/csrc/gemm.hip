// Projections of the decoder layer: C = A * W^T with A [M, K] activations
// and W [N, K] row-major weights (nn.Linear layout).
//
// bfloat16 path.  The activation operand arrives as bfloat16 (hi) or as a
// bfloat16 pair (hi, lo) with hi + lo = the float32 value to about 16
// significant bits; with the pair each product is taken twice (hi*W + lo*W),
// the weights being exact in bfloat16.  MFMA v_mfma_f32_16x16x32_bf16, fp32
// accumulation.  A workgroup of 512 threads computes a 128 x BN output tile
// with two kinds of waves (one of each per SIMD):
//   * staging waves (4-7) stream the weight tile from HBM: a ring of four
//     K-steps of 16-byte loads in flight per thread, written into a ring of
//     three or four LDS buffers two or three K-steps ahead of their use;
//   * compute waves (0-3) each own 32 rows x BN columns: they load their
//     activation fragments straight from global memory (small, shared by
//     every workgroup, L2-resident, stored in fragment order so that each
//     16-byte-per-lane load reads 1 KB contiguously) two K-steps ahead, read
//     the weight fragments from LDS and issue the MFMAs.
// Splitting the roles keeps the in-order retirement of vector loads from
// coupling the long HBM latency of the weights to the MFMA issue.  One
// barrier per K-step (64) hands the LDS buffers over.  The epilogue runs from
// registers (whole-tile statistics from LDS).
//
// Every output tile of BN columns reads its first BN/2 weight rows from one
// base pointer and its last BN/2 from another.  That is how the fused
// epilogues get the pairs they need without any weight repacking:
//   QKV    : columns (c, c + dh/2) of one head -> rotate-half RoPE, then the
//            query buffer or the KV cache slot of the row;
//   SwiGLU : gate row j and up row j -> silu(g) * u, written as the next
//            projection's activation (pair);
//   resid  : plain rows -> residual stream += value;
//   LM head: per-row softmax statistics of every 64 columns (merged later).
// Split-K writes float32 partial tiles that a second kernel sums in a fixed
// order before applying the same epilogue.
//
// gemm_bf16_kernel above serves the row counts that are bound by the weight
// stream; gemm_pp_kernel, below, the row counts that are bound by the MFMAs and
// the smaller launches whose widths leave the first one few workgroups.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "internal.h"
#include "row_stats.h"

namespace ssm {

// ---------------------------------------------------------------------------
// Epilogue policies
// ---------------------------------------------------------------------------
// Eight consecutive row-major elements (16 or 32 bytes, aligned).
__device__ __forceinline__ void store_row8(float* p, const float (&v)[8]) {
  *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
  *(float4*)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store_row8(bf16_t* p, const float (&v)[8]) {
  uint16_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = f2bf(v[e]);
  *(u32x4_t*)p = *(const u32x4_t*)h;
}
__device__ __forceinline__ void store_row8(f16_t* p, const float (&v)[8]) {
  f16x8_t h;
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = (f16_t)v[e];
  *(f16x8_t*)p = h;
}

// Four consecutive row-major elements (8 bytes, aligned).
__device__ __forceinline__ void store_row4(f16_t* p, f32x4_t v) {
  *(f16x4_t*)p = __builtin_convertvector(v, f16x4_t);
}

// Column tile t of width BN covers BN / 2 consecutive entries of the
// concatenated first halves of all heads (query heads, then key, then value)
// and the same entries of the second halves, so the pairs (i, i + d_h / 2)
// that RoPE rotates always meet in one tile, at any width whose half is a
// multiple of 8.  T: weight type; TO: type of q and of the KV cache (float16
// for bfloat16 weights: the attention operands keep three more significand
// bits than bfloat16).
template <typename T, typename TO = T>
struct PolQKV {
  static constexpr bool PAIRED = true;
  static constexpr bool ROW_MAP = true;
  const T *wq, *wk, *wv;
  int ldb, H, Hkv, dh;
  TO *q, *kc, *vc;
  int cap, n_cached, n_rows;
  const float2* rope;
  int rope_per_seq;    // 1: RoPE table [B, n_rows, d_h / 2] (padded batch), 0: [n_rows, d_h / 2]

  uintptr_t weight_bits() const { return (uintptr_t)wq | (uintptr_t)wk | (uintptr_t)wv; }
  __device__ __forceinline__ const T* head_rows(int head) const {
    if (head < H) return wq + (size_t)head * dh * ldb;
    if (head < H + Hkv) return wk + (size_t)(head - H) * dh * ldb;
    return wv + (size_t)(head - H - Hkv) * dh * ldb;
  }
  // weight row of tile row r: rows [0, BN/2) from the first halves, the rest
  // from the second
  __device__ __forceinline__ const T* b_row(int t, int BN, int r) const {
    const int half = dh / 2, second = r >= BN / 2;
    const int j = t * (BN / 2) + (second ? r - BN / 2 : r);
    const int head = j / half;
    return head_rows(head) + (size_t)(j - head * half + (second ? half : 0)) * ldb;
  }
  // both halves as row ranges; only for tiles whose half stays in one head
  // ((BN / 2) divides d_h / 2)
  __device__ __forceinline__ void b_ptrs(int t, int BN, const T*& lo, const T*& hi) const {
    lo = b_row(t, BN, 0);
    hi = lo + (size_t)(dh / 2) * ldb;
  }
  // columns c0 .. c0 + 7 of both halves (c0 a multiple of 8: one head)
  __device__ __forceinline__ void store8(int m, int t, int c0, int BN, const float (&vlo)[8],
                                         const float (&vhi)[8]) const {
    const int half = dh / 2, j = t * (BN / 2) + c0, head = j / half, i0 = j - head * half;
    const int s = m / n_rows, row = m % n_rows;
    float a[8], b[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      a[e] = vlo[e];
      b[e] = vhi[e];
    }
    if (head < H + Hkv) {
      const float2* cs = rope + ((size_t)(rope_per_seq ? s : 0) * n_rows + row) * half + i0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float2 r = cs[e];
        a[e] = vlo[e] * r.x - vhi[e] * r.y;
        b[e] = vhi[e] * r.x + vlo[e] * r.y;
      }
    }
    TO* dst;
    if (head < H) dst = q + (((size_t)s * H + head) * n_rows + row) * dh;
    else if (head < H + Hkv) dst = kc + (((size_t)s * Hkv + (head - H)) * cap + n_cached + row) * dh;
    else dst = vc + (((size_t)s * Hkv + (head - H - Hkv)) * cap + n_cached + row) * dh;
    store_row8(dst + i0, a);
    store_row8(dst + i0 + half, b);
  }
  // columns c0 .. c0 + 3 of both halves (c0 a multiple of 4: one head)
  __device__ __forceinline__ void store4(int m, int t, int c0, int BN, f32x4_t lo, f32x4_t hi) const {
    const int half = dh / 2, j = t * (BN / 2) + c0, head = j / half, i0 = j - head * half;
    const int s = m / n_rows, row = m % n_rows;
    f32x4_t a = lo, b = hi;
    if (head < H + Hkv) {
      const float4* cs = (const float4*)(rope + ((size_t)(rope_per_seq ? s : 0) * n_rows + row) * half + i0);
      const float4 r0 = cs[0], r1 = cs[1];     // two (cos, sin) pairs each
      const f32x4_t c = {r0.x, r0.z, r1.x, r1.z}, sn = {r0.y, r0.w, r1.y, r1.w};
      a = lo * c - hi * sn;
      b = hi * c + lo * sn;
    }
    TO* dst;
    if (head < H) dst = q + (((size_t)s * H + head) * n_rows + row) * dh;
    else if (head < H + Hkv) dst = kc + (((size_t)s * Hkv + (head - H)) * cap + n_cached + row) * dh;
    else dst = vc + (((size_t)s * Hkv + (head - H - Hkv)) * cap + n_cached + row) * dh;
    store_row4(dst + i0, a);
    store_row4(dst + i0 + half, b);
  }
};

template <typename T>
struct PolSwiGLU {
  static constexpr bool PAIRED = true;
  const T *wg, *wu;
  int ldb, F;
  ActOut act;
  uintptr_t weight_bits() const { return (uintptr_t)wg | (uintptr_t)wu; }
  __device__ __forceinline__ void b_ptrs(int t, int BN, const T*& lo, const T*& hi) const {
    lo = wg + (size_t)t * (BN / 2) * ldb;
    hi = wu + (size_t)t * (BN / 2) * ldb;
  }
  __device__ __forceinline__ void store8(int m, int t, int c0, int BN, const float (&g)[8],
                                         const float (&u)[8]) const {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
    act.store8<T>(m, t * (BN / 2) + c0, v);
  }
  __device__ __forceinline__ void store4(int m, int t, int c0, int BN, f32x4_t g, f32x4_t u) const {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
    act.store4(m, t * (BN / 2) + c0, v);
  }
};

template <typename T>
struct PolResid {
  static constexpr bool PAIRED = false;
  const T* w;
  int ldb, N;
  float* resid;
  uintptr_t weight_bits() const { return (uintptr_t)w; }
  __device__ __forceinline__ void b_ptrs(int t, int BN, const T*& lo, const T*& hi) const {
    lo = w + (size_t)t * BN * ldb;
    hi = lo + (size_t)(BN / 2) * ldb;
  }
  __device__ __forceinline__ void store8_1(int m, int n0, const float (&v)[8]) const {
    float4* p = (float4*)(resid + (size_t)m * N + n0);
    float4 a = p[0], b = p[1];
    a.x += v[0]; a.y += v[1]; a.z += v[2]; a.w += v[3];
    b.x += v[4]; b.y += v[5]; b.z += v[6]; b.w += v[7];
    p[0] = a;
    p[1] = b;
  }
  __device__ __forceinline__ void store4_1(int m, int n0, f32x4_t v) const {
    f32x4_t* p = (f32x4_t*)(resid + (size_t)m * N + n0);
    *p += v;
  }
};

template <typename T>
struct PolStore {
  static constexpr bool PAIRED = false;
  const T* w;
  int ldb, ldc;
  float* c;
  __device__ __forceinline__ void b_ptrs(int t, int BN, const T*& lo, const T*& hi) const {
    lo = w + (size_t)t * BN * ldb;
    hi = lo + (size_t)(BN / 2) * ldb;
  }
  __device__ __forceinline__ void store8_1(int m, int n0, const float (&v)[8]) const {
    store_row8(c + (size_t)m * ldc + n0, v);
  }
};

// LM head: per-row partial softmax statistics of every 64 vocabulary columns
// (a segment): running max, sum of exp(x - max) and the 8 largest logits with
// their ids, best first, [MASK] excluded; optionally the logits themselves.
// The part that every merge reads lies apart from the rest of the list.
struct LMHead {
  float m, s, v0;
  int id0;
};
struct LMTail {
  float v[7];
  int id[7];
};
struct LMParts {
  LMHead* head;        // [M][n_part]
  LMTail* tail;        // [M][n_part]
  int n_part;          // N / 64
};

// Compare-exchange and top-8 networks on float64 keys: v_max_f64 / v_min_f64
// move a value and its column together, with no branch.
__device__ __forceinline__ void key_ce(double& a, double& b) {
  const double x = __builtin_fmax(a, b), y = __builtin_fmin(a, b);
  a = x;
  b = y;
}
// sorts 8 keys, largest first (odd-even merge sort, 19 exchanges)
__device__ __forceinline__ void key_sort8(double (&a)[8]) {
  key_ce(a[0], a[1]); key_ce(a[2], a[3]); key_ce(a[4], a[5]); key_ce(a[6], a[7]);
  key_ce(a[0], a[2]); key_ce(a[1], a[3]); key_ce(a[4], a[6]); key_ce(a[5], a[7]);
  key_ce(a[1], a[2]); key_ce(a[5], a[6]);
  key_ce(a[0], a[4]); key_ce(a[1], a[5]); key_ce(a[2], a[6]); key_ce(a[3], a[7]);
  key_ce(a[2], a[4]); key_ce(a[3], a[5]);
  key_ce(a[1], a[2]); key_ce(a[3], a[4]); key_ce(a[5], a[6]);
}
// the 8 largest of two sorted lists, sorted (bitonic merge, 12 exchanges)
__device__ __forceinline__ void key_merge8(double (&a)[8], const double (&b)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = __builtin_fmax(a[i], b[7 - i]);
#pragma unroll
  for (int d = 4; d > 0; d >>= 1)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (!(i & d)) key_ce(a[i], a[i + d]);
}

template <typename T>
struct PolLMStats {
  static constexpr bool PAIRED = false;
  static constexpr bool TILE = true;
  const T* w;
  int ldb, N, mask_id;
  LMParts part;
  float* logits;       // optional [M][ldc]
  int ldc;
  uintptr_t weight_bits() const { return (uintptr_t)w; }
  __device__ __forceinline__ void b_ptrs(int t, int BN, const T*& lo, const T*& hi) const {
    lo = w + (size_t)t * BN * ldb;
    hi = lo + (size_t)(BN / 2) * ldb;
  }
  // One thread per (row, segment).  Per segment: the top 8 of 64 keys by sorting
  // networks over batches of 8, then the sum of exponentials against the
  // maximum just found.  A key is 64 times the ordered bits of the value plus
  // 63 - column, an integer that float64 holds exactly; NaN and [MASK] are
  // below every value.  (A sorted insertion per value runs nearly all of its 8
  // steps for some lane of the wave: the 120-row head of 126464 ids took 229 us
  // with it, 218 with the networks; at 480 rows on gemm_pp_kernel 627 and 494.)
  template <int BM, int BN, int CS>
  __device__ __forceinline__ void tile(const float* Cs, int m0, int M, int t) const {
    const int tid = threadIdx.x;
    if (logits) {
      for (int idx = tid; idx < BM * BN; idx += blockDim.x) {
        const int r = idx / BN, c = idx % BN;
        if (m0 + r < M) logits[(size_t)(m0 + r) * ldc + (size_t)t * BN + c] = Cs[r * CS + c];
      }
    }
    constexpr double NONE = -1.0e18;
    for (int idx = tid; idx < BM * (BN / 64); idx += blockDim.x) {
      const int r = idx % BM, h = idx / BM;          // rows fastest
      if (m0 + r >= M) continue;
      const float* x = Cs + r * CS + 64 * h;
      const int id_base = t * BN + 64 * h, masked = mask_id - id_base;
      double top[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) top[q] = NONE;
      for (int c0 = 0; c0 < 64; c0 += 8) {
        double b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = x[c0 + e];
          const double key = fma((double)ordered_bits(v), 64.0, (double)(63 - c0 - e));
          b[e] = (v == v && c0 + e != masked) ? key : NONE;
        }
        key_sort8(b);
        key_merge8(top, b);
      }
      float tv[8];
      int ti[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const long long kq = (long long)top[q];
        const bool none = top[q] == NONE;
        tv[q] = none ? -INFINITY : ordered_float((int)(kq >> 6));
        ti[q] = none ? STAT_NONE : id_base + 63 - (int)(kq & 63);
      }
      // the best column counts as 1 (exp(inf - inf) is not)
      const float mx = tv[0];
      const int best = ti[0] - id_base;
      float sm = 0.f;
#pragma unroll 8
      for (int c = 0; c < 64; ++c)
        if (c != masked) sm += c == best ? 1.0f : expf(x[c] - mx);
      const size_t o = (size_t)(m0 + r) * part.n_part + (BN / 64) * t + h;
      *(float4*)(part.head + o) = make_float4(mx, sm, tv[0], __int_as_float(ti[0]));
      LMTail l;
#pragma unroll
      for (int q = 1; q < 8; ++q) { l.v[q - 1] = tv[q]; l.id[q - 1] = ti[q]; }
      part.tail[o] = l;
    }
  }
};

template <class P, class = void> struct has_tile { static constexpr bool value = false; };
template <class P> struct has_tile<P, std::void_t<decltype(P::TILE)>> {
  static constexpr bool value = P::TILE;
};
template <class P, class = void> struct has_row_map { static constexpr bool value = false; };
template <class P> struct has_row_map<P, std::void_t<decltype(P::ROW_MAP)>> {
  static constexpr bool value = P::ROW_MAP;
};

// Weight row r of column tile t (lo, hi: the tile's two half ranges from
// b_ptrs, for policies whose halves are row ranges).
template <class Pol, class T>
__device__ __forceinline__ const T* weight_row(const Pol& pol, int t, int BN, int r, const T* lo,
                                               const T* hi) {
  if constexpr (has_row_map<Pol>::value) return pol.b_row(t, BN, r);
  else return r < BN / 2 ? lo + (size_t)r * pol.ldb : hi + (size_t)(r - BN / 2) * pol.ldb;
}

// Applies the epilogue to a BM x BN float tile staged in LDS (row stride CS).
template <int BM, int BN, int CS, class Pol>
__device__ __forceinline__ void tile_epilogue(const Pol& pol, const float* Cs, int m0, int M,
                                              int t, float* part, int split, int ldp) {
  const int tid = threadIdx.x;
  if (part) {
    // float32 partial tile, 8 columns per thread
    for (int idx = tid; idx < BM * (BN / 8); idx += blockDim.x) {
      const int r = idx / (BN / 8), c0 = (idx % (BN / 8)) * 8, gm = m0 + r;
      if (gm >= M) continue;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = Cs[r * CS + c0 + e];
      store_row8(part + ((size_t)split * M + gm) * ldp + (size_t)t * BN + c0, v);
    }
  } else if constexpr (Pol::PAIRED) {
    // 8 columns of each half per thread; 16 consecutive threads take the 16
    // rows of one row group, which are adjacent chunks of the fragment order
    constexpr int C8 = BN / 16;
    for (int idx = tid; idx < BM * C8; idx += blockDim.x) {
      const int rest = idx >> 4, r = (rest / C8) * 16 + (idx & 15), c0 = (rest % C8) * 8;
      const int gm = m0 + r;
      if (gm >= M) continue;
      float lo[8], hi[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        lo[e] = Cs[r * CS + c0 + e];
        hi[e] = Cs[r * CS + c0 + BN / 2 + e];
      }
      pol.store8(gm, t, c0, BN, lo, hi);
    }
  } else {
    for (int idx = tid; idx < BM * (BN / 8); idx += blockDim.x) {
      const int r = idx / (BN / 8), c0 = (idx % (BN / 8)) * 8, gm = m0 + r;
      if (gm >= M) continue;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = Cs[r * CS + c0 + e];
      pol.store8_1(gm, t * BN + c0, v);
    }
  }
}

// ---------------------------------------------------------------------------
// bfloat16 MFMA kernel
// ---------------------------------------------------------------------------
// Tile order: the grid is 1-D over (split, n-tile, m-tile) triples.
// Workgroups are dealt to the 8 XCDs round-robin by linear id, so id w runs
// on XCD w % 8; the order below gives each XCD a contiguous range of the
// triples, split-major, then n-tiles, m-tiles innermost.  The workgroups that
// share a weight tile then run on the same XCD at about the same time and
// read it once into that XCD's L2, and each XCD touches as few K-slices of
// the activations as possible, so that its slice stays resident in its L2.
__device__ __forceinline__ void tile_of(int w, int total, int ntm, int mt, int& split, int& tn,
                                        int& tm) {
  const int per = total / 8;
  const int v = w < per * 8 ? (w % 8) * per + (w / 8) : w;
  split = v / ntm;
  const int t = v % ntm;
  tn = t / mt;
  tm = t % mt;
}

// K-step handover between the two kinds of waves.  The buffer schedule below
// never lets a compute wave read an LDS buffer in the step in which it is
// rewritten, so the compute waves pass the barrier without waiting for their
// own outstanding LDS reads (the fence of __syncthreads would wait for them);
// the staging waves wait for their LDS writes to land first.  The empty asm
// statements keep the compiler from moving memory accesses across.
__device__ __forceinline__ void lds_handover_barrier() {
  asm volatile("s_barrier" ::: "memory");
}
__device__ __forceinline__ void lds_written_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Warp-specialised workgroup of 8 waves, BM rows (128 or 256; 64 and 192 in a
// tuning build) x BN columns.
//  * Waves 4-7 ("staging") stream the weight tile of each K-step (BN rows x 64
//    k, the HBM-bound stream) through a ring of 4 register stages into a ring
//    of 3 or 4 LDS buffers, 2 or 3 K-steps ahead.  A staging thread holds only BN / 32
//    x 16 bytes per stage, so the ring is deep at little register cost.
//  * Waves 0-3 ("compute") each own BM / 4 rows x all BN columns.  They load
//    their activation fragments (bfloat16 hi and optionally lo, L2-resident)
//    straight from global memory into registers in the MFMA operand layout,
//    two K-steps ahead, read the weight fragments from LDS one half-step
//    ahead of use, and run the MFMAs (v_mfma_f32_16x16x32_bf16) ordered so
//    that updates of one accumulator are FM * FN instructions apart.
// Loads retire in issue order per wave; keeping the two streams in different
// waves lets each wait only for its own data.  LDS carries only the weight
// tile (written once, read once by each compute wave).  Every K-step ends with
// one workgroup barrier on both paths.
template <int BM, int BN, int PW, bool SPLIT, class Pol>
__global__ void __launch_bounds__(512) gemm_bf16_kernel(Pol pol, const bf16_t* __restrict__ Ahi,
                                                        const bf16_t* __restrict__ Alo, int G,
                                                        int M, int k_per_split, int mt,
                                                        int n_split, float* __restrict__ part,
                                                        int ldp, int krot) {
  static_assert(BM == 64 || BM == 128 || BM == 192 || BM == 256, "4 compute waves of BM / 4 rows");
  constexpr int BK = 64, LS = BK + 8;            // LDS row stride (elements), 144 B
  constexpr int FM = BM / 64, FN = BN / 16;      // per compute wave: 16 FM rows x BN columns
  constexpr int RW = 16 * FM;
  constexpr int NA = SPLIT ? 2 : 1;
  constexpr int WR = BN / 32;                    // weight rows per staging thread per stage
  // LDS weight buffers: 4 (three K-steps ahead) for the 96-column tiles, 3
  // (two ahead) for the others, which measured 2-3% slower with 4
  constexpr int NBUF = BN == 96 ? 4 : 3;
  constexpr int AHEAD = NBUF - 1;                // K-steps the staging runs ahead
  static_assert(PW == 4 || PW == 8, "weight register ring of 4 or 8 K-steps");
  static_assert(AHEAD < PW, "the prologue refills the first AHEAD register sets");
  constexpr int BUF_ELEMS = BN * LS;
  constexpr int SMEM_W = NBUF * BUF_ELEMS * 2;
  // the epilogue runs from registers; policies that look at a whole tile get it in LDS
  constexpr bool TILE = has_tile<Pol>::value;
  constexpr int CS = BN + 4;
  constexpr int SMEM_C = TILE ? BM * CS * 4 : 0;
  constexpr int SMEM = SMEM_W > SMEM_C ? SMEM_W : SMEM_C;
  static_assert(TILE || !Pol::PAIRED || FN % 2 == 0, "halves of whole fragments");
  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  bf16_t* Ws = (bf16_t*)smem;                    // [NBUF][BN][LS]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int t, mtile, split;
  tile_of(blockIdx.x, gridDim.x, gridDim.x / n_split, mt, split, t, mtile);
  const int m0 = mtile * BM;
  const int kbeg = split * k_per_split;
  const int nk = k_per_split / BK;               // a multiple of 4 (host-checked)
  const int last = nk - 1;
  // K-step kt of this tile reads K-step kmap(kt): column tiles start at
  // different K offsets, so the weight rows read at any one time do not all
  // share their low address bits
  const int rot = krot ? (int)(((long long)t * krot) % nk) : 0;
  auto kmap = [rot, nk](int k) {
    const int x = k + rot;
    return x >= nk ? x - nk : x;
  };
  float* Cs = (float*)smem;

  if (wave < 4) {
    // ------------------------------ compute waves ------------------------------
    // activation fragment i, half kk of K-step kt: the 1 KB fragment-order
    // block of row group (m0 + 32 wave + 16 i) / 16, lane l at 8 l (groups past
    // the allocation read the last one; rows past M are computed and discarded)
    const size_t a_kstep = (size_t)G * 1024;
    size_t a_off[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i)
      a_off[i] = (size_t)(kbeg >> 6) * a_kstep +
                 (size_t)min((m0 + RW * wave + 16 * i) >> 4, G - 1) * 1024 + lane * 8;
    // weight fragment j, half kk: LDS row 16 j + lane % 16, column 32 kk + 8 (lane / 16)
    const int wfrag = (lane & 15) * LS + (lane >> 4) * 8;
    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t a0[NA][FM][2], a1[NA][FM][2];        // activation stages kt (even / odd)
    bf16x8_t wf0[FN], wf1[FN];                   // weight fragments: two halves of a K-step

#define LOAD_A(RA, KT)                                                                \
  do {                                                                                \
    _Pragma("unroll") for (int i = 0; i < FM; ++i)                                    \
    _Pragma("unroll") for (int kk = 0; kk < 2; ++kk) {                                \
      RA[0][i][kk] = *(const u32x4_t*)(Ahi + a_off[i] + kmap(KT) * a_kstep + kk * 512);  \
      if (SPLIT) RA[NA - 1][i][kk] = *(const u32x4_t*)(Alo + a_off[i] + kmap(KT) * a_kstep + kk * 512); \
    }                                                                                 \
  } while (0)
#define READ_W(F, BUF, KK)                                                            \
  do {                                                                                \
    const bf16_t* base_ = Ws + (BUF) * BUF_ELEMS + wfrag + (KK) * 32;                 \
    _Pragma("unroll") for (int j = 0; j < FN; ++j)                                    \
        F[j] = *(const bf16x8_t*)(base_ + j * 16 * LS);                               \
  } while (0)
#define MFMA_H(RA, F, KK)                                                             \
  do {                                                                                \
    _Pragma("unroll") for (int p = 0; p < NA; ++p)                                    \
    _Pragma("unroll") for (int i = 0; i < FM; ++i)                                    \
    _Pragma("unroll") for (int j = 0; j < FN; ++j)                                    \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                          \
            F[j], __builtin_bit_cast(bf16x8_t, RA[p][i][KK]), acc[i][j], 0, 0, 0);     \
  } while (0)
    // step kt: wf0 holds (kt, first half); read (kt, second half) into wf1,
    // use wf0; read (kt + 1, first half) into wf0, use wf1; fetch the
    // activations of kt + 2 into the set just used; barrier
#define CSTEP(KT, RA)                                                                 \
  do {                                                                                \
    const int kt_ = (KT);                                                             \
    READ_W(wf1, kt_ % NBUF, 1);                                                       \
    MFMA_H(RA, wf0, 0);                                                               \
    READ_W(wf0, (kt_ + 1) % NBUF, 0);                                                 \
    MFMA_H(RA, wf1, 1);                                                               \
    LOAD_A(RA, min(kt_ + 2, last));                                                   \
    lds_handover_barrier();                                                           \
  } while (0)

    if (m0 + RW * wave >= M) {
      // every row of this wave is padding (few rows, e.g. the LM head's
      // block rows): no loads or MFMAs, only the barrier schedule
      __syncthreads();
      for (int kt = 0; kt < nk; ++kt) lds_handover_barrier();
    } else {
      LOAD_A(a0, 0);
      LOAD_A(a1, min(1, last));
      __syncthreads();                             // weight stages 0 .. AHEAD - 1 are in LDS
      READ_W(wf0, 0, 0);
      for (int kt = 0; kt < nk; kt += 2) {
        CSTEP(kt, a0);
        CSTEP(kt + 1, a1);
      }
      // acc[i][j][r] = C[RW wave + 16 i + lane % 16][16 j + 4 (lane / 16) + r]: the
      // weights are the MFMA's first operand, so a lane holds 4 consecutive
      // columns of a row, and both columns of a pair (tiles' halves are whole
      // fragments)
      const int c4 = 4 * (lane >> 4);
      if constexpr (TILE) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            *(f32x4_t*)&Cs[(RW * wave + i * 16 + (lane & 15)) * CS + j * 16 + c4] = acc[i][j];
      } else {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int m = m0 + RW * wave + 16 * i + (lane & 15);
          if (m >= M) continue;
          if (part) {
            float* p = part + ((size_t)split * M + m) * ldp + (size_t)t * BN + c4;
#pragma unroll
            for (int j = 0; j < FN; ++j) *(f32x4_t*)(p + 16 * j) = acc[i][j];
          } else if constexpr (Pol::PAIRED) {
#pragma unroll
            for (int j = 0; j < FN / 2; ++j)
              pol.store4(m, t, 16 * j + c4, BN, acc[i][j], acc[i][j + FN / 2]);
          } else {
#pragma unroll
            for (int j = 0; j < FN; ++j) pol.store4_1(m, t * BN + 16 * j + c4, acc[i][j]);
          }
        }
      }
    }
#undef LOAD_A
#undef READ_W
#undef MFMA_H
#undef CSTEP
  } else {
    // ------------------------------ staging waves ------------------------------
    const bf16_t *blo, *bhi;
    pol.b_ptrs(t, BN, blo, bhi);
    const int st = tid - 256, r0 = st >> 3, col = (st & 7) * 8;
    const bf16_t* w_src[WR];
#pragma unroll
    for (int i = 0; i < WR; ++i) {
      const int r = r0 + 32 * i;   // tile rows [0, BN/2) come from lo, the rest from hi
      w_src[i] = weight_row(pol, t, BN, r, blo, bhi) + kbeg + col;
    }
    u32x4_t sr[PW][WR];                          // stage x in register set x % PW
#define LOAD_S(S, KT)                                                                 \
  do {                                                                                \
    _Pragma("unroll") for (int i = 0; i < WR; ++i) S[i] = *(const u32x4_t*)(w_src[i] + kmap(KT) * BK); \
  } while (0)
#define STORE_S(S, BUF)                                                               \
  do {                                                                                \
    _Pragma("unroll") for (int i = 0; i < WR; ++i)                                    \
        *(u32x4_t*)(Ws + (BUF) * BUF_ELEMS + (r0 + 32 * i) * LS + col) = S[i];        \
  } while (0)
    // during step kt the compute waves read buffers kt % NBUF and (kt + 1) %
    // NBUF; the staging waves fill buffer (kt + AHEAD) % NBUF with stage
    // kt + AHEAD and fetch stage kt + AHEAD + PW into the register set it
    // came from
#pragma unroll
    for (int u = 0; u < PW; ++u) LOAD_S(sr[u], min(u, last));
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      STORE_S(sr[u], u);
      LOAD_S(sr[u], min(u + PW, last));
    }
    __syncthreads();                               // weight stages 0 .. AHEAD - 1 are in LDS
    for (int kt = 0; kt < nk; kt += PW) {          // nk is a multiple of PW (host-checked)
#pragma unroll
      for (int u = 0; u < PW; ++u) {
        const int x = kt + u + AHEAD;              // the stage stored in this step
        STORE_S(sr[(u + AHEAD) % PW], x % NBUF);
        LOAD_S(sr[(u + AHEAD) % PW], min(x + PW, last));
        lds_written_barrier();
      }
    }
#undef LOAD_S
#undef STORE_S
  }
  if constexpr (TILE) {
    __syncthreads();
    pol.template tile<BM, BN, CS>(Cs, m0, M, t);
  }
}

// Waits until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// ---------------------------------------------------------------------------
// bfloat16 MFMA kernel, two wave groups in alternation
// ---------------------------------------------------------------------------
// A BM x BN output tile per workgroup of 8 waves in a WM x WN grid, K-steps of
// 64 in two halves of 32.  Waves w and w + 4 share a SIMD; the waves 4-7 run
// half a phase behind the waves 0-3, so that on every SIMD one wave issues
// MFMAs while the other reads its next operands from LDS and starts copies.
// A phase of a wave is
//   memory part:  LDS reads of one half K-step's fragments, copies of later
//                 K-steps (global_load_lds), wait for the reads, barrier;
//   MFMA part:    FM x FN MFMAs on them, barrier.
// Barriers number the slots: in slot 4t (even) the first group reads half 0
// of K-step t, in 4t + 1 the second group does while the first multiplies, and
// so on.  LDS rings: two stages of activations (BM x 64, each half separate),
// three of weights (BN x 64).  What a copy overwrites and where it is read:
//   weights t + 2        stage read last in slot 4t - 1, copied in 4t / 4t + 1,
//                        read from slot 4t + 8 on;
//   activations t + 1, half 1: read last in slot 4t - 1, copied in 4t / 4t + 1,
//                        read from slot 4t + 6 on;
//   activations t + 2, half 0: read last in slot 4t + 1, copied in 4t + 2 /
//                        4t + 3, read from slot 4t + 8 on.
// Each wave waits, before the barrier that opens a slot in which the first
// group reads, until only its copies of the last two phases are in flight.
// Copies past the last K-step repeat the last one (never read), which keeps
// the count uniform.  With SPLIT every K-step runs twice, on the hi and the lo
// part of the activations with the same weights.
//
// Activations are in fragment order: a copy of 1 KB is one MFMA operand and is
// read back at 16 bytes per lane.  A weight copy covers 8 rows of 128 bytes
// (whole cache lines); the 16-byte chunk c of row r sits at slot
// c ^ ((r / 2) % 8), so that the 16 rows of a fragment read fall on 16
// different 16-byte columns of the banks.
// The MFMA takes the weights as its first operand: a lane then holds 4
// consecutive columns of one row, and the epilogue runs from registers.
__device__ __forceinline__ void pp_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int BM, int BN, int WM, int WN, bool SPLIT, class Pol>
__global__ void __launch_bounds__(512, 2) gemm_pp_kernel(Pol pol, const bf16_t* __restrict__ Ahi,
                                                           const bf16_t* __restrict__ Alo, int G,
                                                           int M, int k_steps, int mt,
                                                           int n_split, float* __restrict__ part,
                                                           int ldp) {
  static_assert(WM * WN == 8, "8 waves");
  constexpr int RW = BM / WM, CW = BN / WN, FM = RW / 16, FN = CW / 16;
  constexpr bool PAIRED = Pol::PAIRED;
  static_assert(CW % (PAIRED ? 32 : 16) == 0 && RW % 16 == 0, "whole fragments per wave");
  constexpr int LA = BM / 128, LW = BN / 64;       // copies per wave: half K-step of A, K-step of W
  static_assert(BM % 128 == 0 && BN % 64 == 0, "whole copies per wave");
  constexpr int A_HALF = BM * 64, A_STAGE = 2 * A_HALF, W_STAGE = BN * 128;   // bytes
  constexpr int INFLIGHT = LW + 2 * LA;
  // policies that look at a whole tile get it in LDS, EB rows at a time
  constexpr bool TILE = has_tile<Pol>::value;
  constexpr int EB = 128, CS = BN + 1, SMEM_W = 2 * A_STAGE + 3 * W_STAGE, SMEM_C = TILE ? EB * CS * 4 : 0;
  static_assert(!TILE || EB % RW == 0, "a wave's rows in one chunk");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM_W > SMEM_C ? SMEM_W : SMEM_C];
  char* const Ws = smem + 2 * A_STAGE;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const bool late = wave >= 4;                     // the second group
  int t, mtile, split;
  tile_of(blockIdx.x, gridDim.x, gridDim.x / n_split, mt, split, t, mtile);
  const int m0 = mtile * BM;
  // K-steps of this split: the k_steps of the row dealt out evenly, whole steps
  const int ks0 = split * k_steps / n_split, kbeg = 64 * ks0;
  const int nk = ((split + 1) * k_steps / n_split - ks0) * (SPLIT ? 2 : 1), last = nk - 1;

  // copy sources
  const bf16_t *blo, *bhi;
  pol.b_ptrs(t, BN, blo, bhi);
  const size_t a_kstep = (size_t)G * 1024;
  const bf16_t* w_src[LW];                         // uniform: first row of each 8-row block
#pragma unroll
  for (int i = 0; i < LW; ++i)
    w_src[i] = weight_row(pol, t, BN, 8 * (wave * LW + i), blo, bhi) + kbeg;
  // byte offset of this lane's row and chunk in an even / odd block
  const uint32_t w_off0 = (uint32_t)(lane >> 3) * pol.ldb * 2 + (((lane & 7) ^ (lane >> 4)) << 4);
  const uint32_t w_off1 = (uint32_t)(lane >> 3) * pol.ldb * 2 + (((lane & 7) ^ (lane >> 4) ^ 4) << 4);
  int a_grp[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) a_grp[i] = min((m0 >> 4) + wave * LA + i, G - 1);

  // 16 bytes per lane: from a uniform address and a lane's byte offset
  auto copy = [](const bf16_t* src, uint32_t off, char* dst) {
    __builtin_amdgcn_global_load_lds((const void*)((const char*)src + off),
                                     (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
  };
  // half kk of K-step v (activations), into stage v % 2
  auto issue_a = [&](int v, int kk) {
    const int vs = min(v, last), ks = SPLIT ? vs >> 1 : vs;
    const bf16_t* base = (SPLIT && (vs & 1) ? Alo : Ahi) + (size_t)(ks0 + ks) * a_kstep + kk * 512;
    char* dst = smem + (v & 1) * A_STAGE + kk * A_HALF + wave * LA * 1024;
#pragma unroll
    for (int i = 0; i < LA; ++i) copy(base + (size_t)a_grp[i] * 1024, lane * 16, dst + i * 1024);
  };
  // K-step v (weights), into ring slot `slot`
  auto issue_w = [&](int v, int slot) {
    const int vs = min(v, last), ks = SPLIT ? vs >> 1 : vs;
    char* dst = Ws + slot * W_STAGE + wave * LW * 1024;
#pragma unroll
    for (int i = 0; i < LW; ++i)
      copy(w_src[i] + (size_t)ks * 64, ((wave * LW + i) & 1) ? w_off1 : w_off0, dst + i * 1024);
  };

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  bf16x8_t af[FM], wf[FN];

  // LDS offsets of this wave's fragments
  const int a_frag = wm * FM * 1024 + lane * 16;
  const int r16 = lane & 15, g4 = lane >> 4;
  const int w_lane = r16 * 128 + ((g4 ^ (r16 >> 1)) << 4);        // half 0; half 1: chunk ^ 4
  auto w_rows = [&](int j) {                        // first tile row of weight fragment j
    if constexpr (PAIRED) {
      constexpr int HF = FN / 2;
      return (j < HF ? wn * (CW / 2) + 16 * j : BN / 2 + wn * (CW / 2) + 16 * (j - HF));
    } else {
      return wn * CW + 16 * j;
    }
  };
  auto read = [&](int v, int slot, int kk) {
    const char* a = smem + (v & 1) * A_STAGE + kk * A_HALF + a_frag;
    const char* w = Ws + slot * W_STAGE + (w_lane ^ (kk << 6));
#pragma unroll
    for (int j = 0; j < FN; ++j) wf[j] = *(const bf16x8_t*)(w + w_rows(j) * 128);
#pragma unroll
    for (int i = 0; i < FM; ++i) af[i] = *(const bf16x8_t*)(a + i * 1024);
  };
  auto mma = [&]() {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], af[i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // end of a memory part / of an MFMA part
  auto end_mem = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
    if (late) wait_vmcnt<INFLIGHT>();
    pp_barrier();
  };
  auto end_mma = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    if (!late) wait_vmcnt<INFLIGHT>();
    pp_barrier();
  };

  issue_w(0, 0);
  issue_a(0, 0);
  issue_a(0, 1);
  issue_w(1, 1);
  issue_a(1, 0);
  wait_vmcnt<LW + LA>();
  pp_barrier();
  if (late) pp_barrier();
  int s0 = 0, s2 = 2;                               // ring slots of K-steps v and v + 2
  for (int v = 0; v < nk; ++v) {
    read(v, s0, 0);
    issue_w(v + 2, s2);
    issue_a(v + 1, 1);
    end_mem();
    mma();
    end_mma();
    read(v, s0, 1);
    issue_a(v + 2, 0);
    end_mem();
    mma();
    end_mma();
    s2 = s0;
    s0 = s0 == 2 ? 0 : s0 + 1;
  }
  if (!late) pp_barrier();
  wait_vmcnt<0>();                                  // no copy lands after the workgroup ends

  if constexpr (TILE) {
    float* Cs = (float*)smem;
#pragma unroll
    for (int h = 0; h < BM / EB; ++h) {
      __syncthreads();                              // the ring, or the chunk before, is done with
      if (RW * wm / EB == h) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              Cs[(RW * wm - EB * h + 16 * i + r16) * CS + w_rows(j) + 4 * g4 + r] = acc[i][j][r];
      }
      __syncthreads();
      pol.template tile<EB, BN, CS>(Cs, m0 + EB * h, M, t);
    }
    return;
  } else {
  // acc[i][j][r] = C[RW wm + 16 i + lane % 16][w_rows(j) + 4 (lane / 16) + r]
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + wm * RW + 16 * i + r16;
    if (m >= M) continue;
    if (part) {
      float* p = part + ((size_t)split * M + m) * ldp + (size_t)t * BN + 4 * g4;
#pragma unroll
      for (int j = 0; j < FN; ++j) *(f32x4_t*)(p + w_rows(j)) = acc[i][j];
    } else if constexpr (PAIRED) {
#pragma unroll
      for (int j = 0; j < FN / 2; ++j)
        pol.store4(m, t, w_rows(j) + 4 * g4, BN, acc[i][j], acc[i][j + FN / 2]);
    } else {
#pragma unroll
      for (int j = 0; j < FN; ++j) pol.store4_1(m, t * BN + w_rows(j) + 4 * g4, acc[i][j]);
    }
  }
  }
}

// ---------------------------------------------------------------------------
// float32 kernel (fp32 mode): 32 x 32 tiles, 256 threads, 4 outputs each
// ---------------------------------------------------------------------------
// Both operands of up to 128 K columns are in flight at once and go through
// LDS transposed (k rows of 36 floats: 16-byte aligned, so a thread reads its
// 4 columns at once).  The small model's launches are bound by the trips to
// memory: with 32 columns a trip, the 108-row projections took 5 to 11 us.
// Products are summed in chains of 32 and the chains' sums in turn: a chain of
// n products is off by about 0.31 sqrt(n) 2^-24 of its result, one of 128 by
// twice as much as this.
template <class Pol>
__global__ void __launch_bounds__(256) gemm_f32_kernel(Pol pol, const float* __restrict__ A, int lda,
                                                       int M, int k_per_split,
                                                       float* __restrict__ part, int ldp) {
  constexpr int BM = 32, BN = 32, BK = 128, LD = 36, CS = BN + 1, NQ = BK / 32;
  __shared__ __attribute__((aligned(16))) float As[BK][LD];
  __shared__ __attribute__((aligned(16))) float Bs[BK][LD];
  __shared__ float Cs[BM * CS];
  const int tid = threadIdx.x;
  const int t = blockIdx.x, m0 = blockIdx.y * BM, split = blockIdx.z;
  const int kbeg = split * k_per_split, kend = kbeg + k_per_split;
  const float *blo, *bhi;
  pol.b_ptrs(t, BN, blo, bhi);
  // copies: row tid / 8 of each operand, columns 4 (tid % 8) + 32 q (k_per_split
  // is a multiple of 32, so a 32-column group is in or out as a whole)
  const int cr = tid >> 3, cc = (tid & 7) * 4;
  const float* ap = A + (size_t)min(m0 + cr, M - 1) * lda + cc;
  const float* bp = (cr < BN / 2 ? blo + (size_t)cr * pol.ldb : bhi + (size_t)(cr - BN / 2) * pol.ldb) + cc;
  const int tr = tid / 8, tc = (tid % 8) * 4;   // output row, first of 4 columns
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    f32x4_t av[NQ], bv[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (k0 + 32 * q < kend) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {            // rows of any 4-byte alignment
          av[q][e] = ap[k0 + 32 * q + e];
          bv[q][e] = bp[k0 + 32 * q + e];
        }
      }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (k0 + 32 * q < kend) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          As[32 * q + cc + e][cr] = av[q][e];
          Bs[32 * q + cc + e][cr] = bv[q][e];
        }
      }
    __syncthreads();
    const int kn = min(BK, kend - k0);
    for (int k1 = 0; k1 < kn; k1 += 32) {          // a chain of 32, then its sum
      float sub[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
      for (int kk = k1; kk < k1 + 32; ++kk) {
        const float a = As[kk][tr];
        const f32x4_t b = *(const f32x4_t*)&Bs[kk][tc];
#pragma unroll
        for (int j = 0; j < 4; ++j) sub[j] = fmaf(a, b[j], sub[j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] += sub[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) Cs[tr * CS + tc + j] = acc[j];
  __syncthreads();
  tile_epilogue<BM, BN, CS>(pol, Cs, m0, M, t, part, split, ldp);
}

// ---------------------------------------------------------------------------
// split-K reduction: sums partial tiles in split order, then the epilogue
// ---------------------------------------------------------------------------
// Sum of the split-K partials of 8 consecutive columns, in split order.  SC
// is the split count when known at compile time (all loads in flight before
// the sum), 0 for a runtime count.
template <int SC>
__device__ __forceinline__ void sum_partials8(const float* __restrict__ p, size_t stride, int S,
                                              float (&acc)[8]) {
  if constexpr (SC > 0) {
    float4 v[SC][2];
#pragma unroll
    for (int s = 0; s < SC; ++s) {
      v[s][0] = *(const float4*)(p + s * stride);
      v[s][1] = *(const float4*)(p + s * stride + 4);
    }
#pragma unroll
    for (int s = 0; s < SC; ++s) {
      acc[0] += v[s][0].x; acc[1] += v[s][0].y; acc[2] += v[s][0].z; acc[3] += v[s][0].w;
      acc[4] += v[s][1].x; acc[5] += v[s][1].y; acc[6] += v[s][1].z; acc[7] += v[s][1].w;
    }
  } else {
    for (int s = 0; s < S; ++s) {
      const float4 a = *(const float4*)(p + s * stride), b = *(const float4*)(p + s * stride + 4);
      acc[0] += a.x; acc[1] += a.y; acc[2] += a.z; acc[3] += a.w;
      acc[4] += b.x; acc[5] += b.y; acc[6] += b.z; acc[7] += b.w;
    }
  }
}

template <int BN, class Pol, int SC>
__global__ void __launch_bounds__(256) splitk_reduce_kernel(Pol pol, const float* __restrict__ part,
                                                            int ldp, int M, int S, int ntiles) {
  // one thread per 8 consecutive output columns (of each half, when paired)
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  constexpr int C8 = Pol::PAIRED ? BN / 16 : BN / 8;
  const size_t per_row = (size_t)ntiles * C8;
  if (idx >= (size_t)M * per_row) return;
  const int m = idx / per_row, rem = idx % per_row;
  const int t = rem / C8, c0 = (rem % C8) * 8;
  float lo[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float hi[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float* p = part + (size_t)m * ldp + (size_t)t * BN + c0;
  sum_partials8<SC>(p, (size_t)M * ldp, S, lo);
  if constexpr (Pol::PAIRED) sum_partials8<SC>(p + BN / 2, (size_t)M * ldp, S, hi);
  if constexpr (Pol::PAIRED) pol.store8(m, t, c0, BN, lo, hi);
  else pol.store8_1(m, t * BN + c0, lo);
}

template <int BN, class Pol>
static void launch_reduce(const Pol& pol, const float* part, int N, int M, int S, int ntiles,
                          hipStream_t st) {
  const size_t total = (size_t)M * N / 8 / (Pol::PAIRED ? 2 : 1);
  const dim3 grid((unsigned)((total + 255) / 256)), block(256);
  if (S == 8) launch((splitk_reduce_kernel<BN, Pol, 8>), grid, block, 0, st, pol, part, N, M, S, ntiles);
  else if (S == 3) launch((splitk_reduce_kernel<BN, Pol, 3>), grid, block, 0, st, pol, part, N, M, S, ntiles);
  else if (S == 4) launch((splitk_reduce_kernel<BN, Pol, 4>), grid, block, 0, st, pol, part, N, M, S, ntiles);
  else if (S == 2) launch((splitk_reduce_kernel<BN, Pol, 2>), grid, block, 0, st, pol, part, N, M, S, ntiles);
  else launch((splitk_reduce_kernel<BN, Pol, 0>), grid, block, 0, st, pol, part, N, M, S, ntiles);
}

// ---------------------------------------------------------------------------
// host-side dispatch
// ---------------------------------------------------------------------------
// K-step rotation of the column tiles (tile t starts at K-step t * krot mod
// nk); 0 = every tile starts at K-step 0.  Measured on the 120-row steps:
// 1 spreads the concurrently read weight addresses and takes 4% off the step.
// A tuning build (SSM_TUNING defined) lets SSM_GEMM_KROT override it; the
// product build reads no environment variable.
static int gemm_krot() {
#ifdef SSM_TUNING
  static const int krot = [] {
    const char* e = getenv("SSM_GEMM_KROT");
    return e ? atoi(e) : 1;
  }();
  return krot;
#else
  return 1;
#endif
}

// Float32 partials: the workspace holds SPLIT_ROWS_MAX rows of the widest
// output (the vocabulary included).  gemm_bf16_kernel and the float32 kernel
// split K while S * M stays within SPLIT_ROWS_MAX, gemm_pp_kernel while the S * M
// rows of the projection's own width fit (O and down at 1127 rows: 2 splits).
static constexpr int SPLIT_ROWS_MAX = 1024;
size_t gemm_split_ws_floats(int M, int max_n) {
  (void)M;
  return (size_t)SPLIT_ROWS_MAX * max_n;
}

// Tiles of gemm_pp_kernel: rows, columns and the time of a K-step of 64 in a
// full round of 256 workgroups (one per CU), in us.  A round of workgroups
// takes steps * us + PP_FIXED_US (prologue, first copies, epilogue, launch).
// That holds for several rounds (gate/up of 1776 rows: 297 us, 291 in a trace);
// a launch of one round takes 18-23 us more in a stack of layers (476 rows:
// gate/up 77 and 99 us, QKV 50 and 70).
// Measured in a loop of 1024-2048 x 4096-8192 x 4096 products with random
// operands: the 256 x 256 tile takes 2415 clocks for the 2048 clocks of MFMAs
// that a K-step holds per SIMD, the smaller ones 1990 for 1536, 1600 and 1660
// for 1024, 1410 for 768: each of the 4 barriers of a K-step costs about 45
// clocks, and LDS reads outlast the MFMAs of small wave tiles.  With the
// 256 x 256 tile the clock gives way too (1.6-1.8 GHz under this load, 2.1
// with the copies left out).  A 128 x 128 tile with two workgroups per CU
// (1510 clocks for 1024) was never the cheapest.
struct PpTile {
  int bm, bn;
  float us;
};
static constexpr PpTile PP_TILES[] = {
    {256, 256, 1.42f}, {256, 192, 1.07f}, {256, 128, 0.82f}, {128, 256, 0.84f}, {128, 192, 0.66f},
};
static constexpr int N_PP_TILES = sizeof(PP_TILES) / sizeof(PP_TILES[0]);
static constexpr int PP_SLOTS = 256;
static constexpr float PP_FIXED_US = 8.0f;
// float32 partials of split-K are written once and read once
static constexpr float PP_PARTIAL_BYTES_PER_US = 5.0e6f;
static constexpr float WEIGHT_BYTES_PER_US = 5.5e6f;   // weights from HBM
static constexpr float SPLIT_SUM_US = 4.0f;            // the launch that sums partials
// (more than 4 splits pay only where their partials are small)
static int pp_max_split(int M) { return M <= 256 ? 8 : 4; }
// gemm_bf16_kernel: its K-step grows with the tile's columns and rows (us, from
// 60-240 rows of 4096-18944 columns), the fixed part as above.
static float bf16_step_us(int bn, int bm, bool pair) {
  return 0.27f + 0.0029f * bn * (bm / 128.0f) * (pair ? 2 : 1);
}

// Per-projection launch choice: tile width BN (64, 96 or 128), split-K S
// (0 = automatic) and the depth PW (4 K-steps, in a tuning build also 8) of the
// staging waves' register ring of weight loads of gemm_bf16_kernel, with its row tile bm
// (see launch_bf16_bm); or, with pp = 1 + an index into PP_TILES,
// gemm_pp_kernel (-1: the tile and split that cost least).
struct GemmCfg {
  int bn, s, pw;
  int pp = 0;
  int bm = 128;
};

// Tuning override, compiled only into a tuning build (SSM_TUNING defined):
// SSM_GEMM_CFG="kind:bn:s:pw[:pp[:bm]],..." with kind one of qkv, o, gate_up,
// down, lm (pp and bm as in GemmCfg); read at every launch.  The product build
// always takes the measured defaults.
static GemmCfg cfg_override(const char* kind, GemmCfg c) {
#ifdef SSM_TUNING
  const char* env = getenv("SSM_GEMM_CFG");
  if (!env) return c;
  const size_t kl = strlen(kind);
  for (const char* p = env; p && *p;) {
    if (strncmp(p, kind, kl) == 0 && p[kl] == ':') {
      int bn, s, pw, pp = 0, bm = 128;
      const int n = sscanf(p + kl + 1, "%d:%d:%d:%d:%d", &bn, &s, &pw, &pp, &bm);
      if (n >= 3) return GemmCfg{bn, s, pw, n >= 4 ? pp : c.pp, n == 5 ? bm : c.bm};
    }
    p = strchr(p, ',');
    if (p) ++p;
  }
  return c;
#else
  (void)kind;
  return c;
#endif
}

static int auto_split(int tiles, int M, int K, size_t ws_floats, int N) {
  int S = 1;
  while (S < 8 && tiles * S < 192 && K % (256 * S * 2) == 0 && (S * 2) * M <= SPLIT_ROWS_MAX &&
         (size_t)(S * 2) * M * N <= ws_floats)
    S *= 2;
  return S;
}

// Time of the sum of S split-K partials (0 for one), in us.
static float split_sum_us(int M, int N, int S) {
  return S > 1 ? 8.0f * S * M * N / PP_PARTIAL_BYTES_PER_US + SPLIT_SUM_US : 0.f;
}

// Time of gemm_pp_kernel with tile number `tile` (1 + its index) and split S, in
// us; never below the time the weights take from HBM.
static float pp_cost(int tile, int M, int K, int N, bool pair, int S = 1) {
  const PpTile& p = PP_TILES[tile - 1];
  const long wgs = (long)(N / p.bn) * ceil_div(M, p.bm) * S;
  const float steps = (float)ceil_div(K / 64, S) * (pair ? 2 : 1);
  const float mfma = (float)((wgs + PP_SLOTS - 1) / PP_SLOTS) * (steps * p.us + PP_FIXED_US);
  const float hbm = 2.0f * N * K / WEIGHT_BYTES_PER_US + PP_FIXED_US;
  return (mfma > hbm ? mfma : hbm) + split_sum_us(M, N, S);
}

// The tile (1 + its index) and split of gemm_pp_kernel that cost least by the
// times above, among tiles that divide N and whose weight rows the policy can
// map; 0 if there is none.  want > 0 / s > 0 fix the tile / the split.
template <class Pol>
static int pp_plan(const Pol& pol, int M, int K, int N, bool pair, size_t ws_floats,
                   int (*bn_ok)(const Pol&, int), int want, int& s) {
  int best = 0, best_s = 1;
  float best_us = 0.f;
  for (int i = 0; i < N_PP_TILES; ++i) {
    const PpTile& p = PP_TILES[i];
    if ((want > 0 && want != i + 1) || N % p.bn != 0 || !bn_ok(pol, p.bn)) continue;
    for (int S = 1; S <= pp_max_split(M); ++S) {
      if ((s > 0 && S != s) || S > K / 64 || (S > 1 && (size_t)S * M * N > ws_floats)) continue;
      const float us = pp_cost(i + 1, M, K, N, pair, S);
      if (!best || us < best_us) {
        best = i + 1;
        best_s = S;
        best_us = us;
      }
    }
  }
  s = best_s;
  return best;
}

template <int BM, int BN, int PW, bool SPLIT, class Pol>
static hipError_t launch_bf16(const Pol& pol, const ActIn& a, int M, int K, int N, int S,
                              SplitWs ws, hipStream_t st, bool reduce) {
  const int ntiles = N / BN, mt = ceil_div(M, BM);
  const dim3 grid(ntiles * mt * S);
  launch((gemm_bf16_kernel<BM, BN, PW, SPLIT, Pol>), grid, dim3(512), 0, st, pol,
                     (const bf16_t*)a.hi, a.lo, a.G, M, K / S, mt, S,
                     S > 1 ? ws.part : nullptr, N, gemm_krot());
  if constexpr (!has_tile<Pol>::value) {   // whole-tile epilogues never split K
    if (S > 1 && reduce) launch_reduce<BN>(pol, ws.part, N, M, S, ntiles, st);
  }
  return hipGetLastError();
}

template <int BM, int BN, class Pol>
static hipError_t launch_bf16_pw(const Pol& pol, const ActIn& a, int M, int K, int N, int S,
                                 int pw, SplitWs ws, hipStream_t st, bool reduce) {
  const bool split = a.lo != nullptr;
#ifdef SSM_TUNING
  // the staging loop is unrolled by the ring depth: nk = K / S / 64 must be a
  // multiple of it (of 4 always, host-checked)
  if (pw >= 8 && (K / S / 64) % 8 == 0)
    return split ? launch_bf16<BM, BN, 8, true>(pol, a, M, K, N, S, ws, st, reduce)
                 : launch_bf16<BM, BN, 8, false>(pol, a, M, K, N, S, ws, st, reduce);
#endif
  return split ? launch_bf16<BM, BN, 4, true>(pol, a, M, K, N, S, ws, st, reduce)
               : launch_bf16<BM, BN, 4, false>(pol, a, M, K, N, S, ws, st, reduce);
}

// Row tile of gemm_bf16_kernel: 128, or 256 for the one-pass gate/up on
// 96-column tiles (the register budget of a compute wave).  A tuning build has
// more: 64 (two row tiles share each weight tile through L2 on small row
// counts), and 192 and 256 for every one-pass projection on up to 96 columns.
template <int BN, class Pol>
static hipError_t launch_bf16_bm(const Pol& pol, const ActIn& a, int M, int K, int N, int S,
                                 int pw, int bm, SplitWs ws, hipStream_t st, bool reduce) {
  const bool one_pass = a.lo == nullptr;
#ifdef SSM_TUNING
  constexpr bool ROWS_256 = BN <= 96;
  if (bm == 64) return launch_bf16_pw<64, BN>(pol, a, M, K, N, S, pw, ws, st, reduce);
  if constexpr (BN <= 96)
    if (bm == 192 && one_pass) return launch_bf16<192, BN, 4, false>(pol, a, M, K, N, S, ws, st, reduce);
#else
  constexpr bool ROWS_256 = BN == 96 && std::is_same<Pol, PolSwiGLU<bf16_t>>::value;
#endif
  if constexpr (ROWS_256)
    if (bm == 256 && one_pass) return launch_bf16<256, BN, 4, false>(pol, a, M, K, N, S, ws, st, reduce);
  return launch_bf16_pw<128, BN>(pol, a, M, K, N, S, pw, ws, st, reduce);
}

// Whether gemm_pp_kernel may take these operands: its copies put 16 bytes a
// lane straight into LDS and want them aligned, as weights that are views into
// a larger buffer need not be.  gemm_bf16_kernel loads into registers, from
// any address.
template <class Pol>
static bool pp_aligned(const Pol& pol, const ActIn& a) {
  return ((pol.weight_bits() | (uintptr_t)a.hi | (uintptr_t)a.lo) & 15) == 0;
}

// Launch plan of one projection: the configuration with a valid tile width
// and the split-K factor.
template <class Pol>
static GemmCfg plan_bf16(const char* kind, const Pol& pol, const ActIn& a, int M, int K, int N,
                         GemmCfg c, const SplitWs& ws, int (*bn_ok)(const Pol&, int)) {
  const GemmCfg given = c;
  c = cfg_override(kind, c);
  const bool overridden = c.bn != given.bn || c.s != given.s || c.pp != given.pp || c.bm != given.bm || c.pw != given.pw;
  const bool pair = a.lo != nullptr, pp_ok = K % 64 == 0 && pp_aligned(pol, a);
  if (c.pp != 0 && pp_ok) {
    c.pp = pp_plan(pol, M, K, N, pair, ws.floats, bn_ok, c.pp, c.s);
    if (c.pp) return c;
  }
  c.pp = 0;
  if (c.bn > 128 || !bn_ok(pol, c.bn) || N % c.bn) c.bn = bn_ok(pol, 128) && N % 128 == 0 ? 128 : 64;
  if ((c.bm != 64 && c.bm != 192 && c.bm != 256) || ((c.bm == 192 || c.bm == 256) && c.bn > 96))
    c.bm = 128;
  const int tiles = (N / c.bn) * ceil_div(M, c.bm);
  int S = c.s > 0 ? c.s : auto_split(tiles, M, K, ws.floats, N);
  while (S > 1 && (K % (256 * S) != 0 || (size_t)S * M * N > ws.floats)) S /= 2;
  // below 512 rows gemm_pp_kernel, whose splits need not divide K, where it
  // should take less time than this kernel: in one pass from 257 rows as soon
  // as the estimates say so (8B shape, 300 rows: 234 -> 225 us a layer; at
  // d = 512, 351 rows, where they do not, it would be 182 -> 188 us for two
  // layers).  Elsewhere at less than 0.7 of it: widths that leave this kernel
  // with few workgroups or a nearly empty last round (grouped-query shape at
  // 120 rows: gate/up, 296 tiles, 84 -> 71 us; down, 28 tiles in 2 splits, 95
  // -> 48 us; QKV with the pair at 352 rows, 50 -> 43 us; 8B gate/up with the
  // pair at 440 rows, 165 -> 152 us).  At 0.8 the estimate is not safe there:
  // several workgroups of this kernel may share a CU (with the pair, 8B
  // gate/up at 330 rows, 131 us, would move to 149; QKV at 376 rows, 94 us, to
  // 100; grouped-query gate/up at 440 rows, 231 us, to 282)
  if (pp_ok && !overridden) {
    const float us = (float)ceil_div(tiles * S, 256) *
                         (K / 64 / S * bf16_step_us(c.bn, c.bm, pair) + PP_FIXED_US) +
                     split_sum_us(M, N, S);
    const float margin = !pair && M > 256 ? 1.0f : 0.7f;
    int ps = 0;
    const int tile = pp_plan(pol, M, K, N, pair, ws.floats, bn_ok, -1, ps);
    if (tile && pp_cost(tile, M, K, N, pair, ps) < margin * us) {
      c.pp = tile;
      c.s = ps;
      return c;
    }
  }
  c.s = S;
  return c;
}

template <int BM, int BN, int WM, int WN, class Pol>
static hipError_t launch_pp(const Pol& pol, const ActIn& a, int M, int K, int N, int S,
                            SplitWs ws, hipStream_t st, bool reduce) {
  const int ntiles = N / BN, mt = ceil_div(M, BM);
  const dim3 grid(ntiles * mt * S), block(512);
  float* pp = S > 1 ? ws.part : nullptr;
  if (a.lo)
    launch((gemm_pp_kernel<BM, BN, WM, WN, true, Pol>), grid, block, 0, st, pol,
           (const bf16_t*)a.hi, a.lo, a.G, M, K / 64, mt, S, pp, N);
  else
    launch((gemm_pp_kernel<BM, BN, WM, WN, false, Pol>), grid, block, 0, st, pol,
           (const bf16_t*)a.hi, a.lo, a.G, M, K / 64, mt, S, pp, N);
  if constexpr (!has_tile<Pol>::value) {   // whole-tile epilogues never split K
    if (S > 1 && reduce) launch_reduce<BN>(pol, ws.part, N, M, S, ntiles, st);
  }
  return hipGetLastError();
}

template <class Pol>
static hipError_t launch_plan(const Pol& pol, const ActIn& a, int M, int K, int N, GemmCfg c,
                              SplitWs ws, hipStream_t st, bool reduce = true) {
  switch (c.pp) {   // 1 + the index in PP_TILES
    case 1: return launch_pp<256, 256, 2, 4>(pol, a, M, K, N, c.s, ws, st, reduce);
    case 2: return launch_pp<256, 192, 4, 2>(pol, a, M, K, N, c.s, ws, st, reduce);
    case 3: return launch_pp<256, 128, 4, 2>(pol, a, M, K, N, c.s, ws, st, reduce);
    case 4: return launch_pp<128, 256, 2, 4>(pol, a, M, K, N, c.s, ws, st, reduce);
    case 5: return launch_pp<128, 192, 4, 2>(pol, a, M, K, N, c.s, ws, st, reduce);
    default: break;
  }
  if (c.bn == 96) return launch_bf16_bm<96>(pol, a, M, K, N, c.s, c.pw, c.bm, ws, st, reduce);
  if (c.bn == 64) return launch_bf16_bm<64>(pol, a, M, K, N, c.s, c.pw, c.bm, ws, st, reduce);
  return launch_bf16_bm<128>(pol, a, M, K, N, c.s, c.pw, c.bm, ws, st, reduce);
}

template <class Pol>
static hipError_t run_bf16(const char* kind, Pol pol, const ActIn& a, int M, int K, int N,
                           GemmCfg c, SplitWs ws, hipStream_t st, int (*bn_ok)(const Pol&, int)) {
  c = plan_bf16(kind, pol, a, M, K, N, c, ws, bn_ok);
  return launch_plan(pol, a, M, K, N, c, ws, st);
}

// Eight gains, 16-byte aligned.
__device__ __forceinline__ void load_gain8(const bf16_t* g, float (&v)[8]) {
  const u32x4_t w = *(const u32x4_t*)g;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(e & 1 ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
}
__device__ __forceinline__ void load_gain8(const float* g, float (&v)[8]) {
  const float4 a = ((const float4*)g)[0], b = ((const float4*)g)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Completion of a split-K residual projection fused with the RMSNorm that
// follows it: resid[m] += sum over splits of part[s][m] (split order, as the
// split-K reduction does), then y[m] = resid[m] / rms(resid[m]) * g as the next
// projection's operand.  One workgroup of 512 threads per row; thread t holds
// the 8-column chunks t + 512 q of the row (q < NC).
template <typename T, int SC, int NC>
__global__ void __launch_bounds__(512) resid_norm_kernel(const float* __restrict__ part, int S,
                                                         int M, int N, float* __restrict__ resid,
                                                         const T* __restrict__ g, float eps,
                                                         ActOut y) {
  __shared__ float red[8];
  const int m = xcd_row(blockIdx.x, gridDim.x), tid = threadIdx.x, nc8 = N >> 3;
  float v[NC][8];
  float ss = 0.f;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c8 = tid + 512 * q;
    if (c8 >= nc8) continue;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sum_partials8<SC>(part + (size_t)m * N + c8 * 8, (size_t)M * N, S, acc);
    float4* r = (float4*)(resid + (size_t)m * N + c8 * 8);
    float4 r0 = r[0], r1 = r[1];
    r0.x += acc[0]; r0.y += acc[1]; r0.z += acc[2]; r0.w += acc[3];
    r1.x += acc[4]; r1.y += acc[5]; r1.z += acc[6]; r1.w += acc[7];
    r[0] = r0;
    r[1] = r1;
    v[q][0] = r0.x; v[q][1] = r0.y; v[q][2] = r0.z; v[q][3] = r0.w;
    v[q][4] = r1.x; v[q][5] = r1.y; v[q][6] = r1.z; v[q][7] = r1.w;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[q][e] * v[q][e];
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  ss = ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
  const float inv = 1.0f / sqrtf(ss / (float)N + eps);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c8 = tid + 512 * q;
    if (c8 >= nc8) continue;
    float ge[8], o[8];
    load_gain8(g + c8 * 8, ge);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[q][e] * inv * ge[e];
    y.store8<T>(m, c8 * 8, o);
  }
}

template <typename T, int SC>
static void launch_resid_norm_s(int S, int M, int N, const float* part, float* resid,
                                const NormTo* nrm, hipStream_t st) {
  const T* g = (const T*)nrm->g;
  if (N <= 4096)
    launch(resid_norm_kernel<T, SC, 1>, dim3(M), dim3(512), 0, st, part, S, M, N, resid, g, nrm->eps, nrm->y);
  else
    launch(resid_norm_kernel<T, SC, 2>, dim3(M), dim3(512), 0, st, part, S, M, N, resid, g, nrm->eps, nrm->y);
}
template <typename T>
static void launch_resid_norm(int S, int M, int N, const float* part, float* resid,
                              const NormTo* nrm, hipStream_t st) {
  if (S == 8) launch_resid_norm_s<T, 8>(S, M, N, part, resid, nrm, st);
  else if (S == 4) launch_resid_norm_s<T, 4>(S, M, N, part, resid, nrm, st);
  else if (S == 3) launch_resid_norm_s<T, 3>(S, M, N, part, resid, nrm, st);
  else if (S == 2) launch_resid_norm_s<T, 2>(S, M, N, part, resid, nrm, st);
  else launch_resid_norm_s<T, 0>(S, M, N, part, resid, nrm, st);
}
// Whether resid_norm_kernel can take the split-K sums of this projection.
static bool resid_norm_ok(int S, int N, const NormTo* nrm) {
  return nrm && S > 1 && N % 8 == 0 && N <= 8192 && ((uintptr_t)nrm->g & 15) == 0;
}

// float32 projections: split-K while CUs are idle and every split keeps 128
// columns, one trip to memory (a shorter one costs the same and the sum a launch).
static int f32_split(int M, int K, int N, size_t ws_floats) {
  const int tiles = (N / 32) * ceil_div(M, 32);
  int S = 1;
  while (S < 8 && tiles * S < 256 && K % (32 * S * 2) == 0 && K / (S * 2) >= 128 &&
         (S * 2) * M <= SPLIT_ROWS_MAX && (size_t)(S * 2) * M * N <= ws_floats)
    S *= 2;
  return S;
}

template <class Pol>
static hipError_t run_f32(const Pol& pol, const ActIn& a, int M, int K, int N, SplitWs ws,
                          hipStream_t st, bool reduce = true) {
  constexpr int BN = 32;
  const int ntiles = N / BN, mt = ceil_div(M, 32);
  const int S = f32_split(M, K, N, ws.floats);
  dim3 grid(ntiles, mt, S);
  launch((gemm_f32_kernel<Pol>), grid, dim3(256), 0, st, pol, (const float*)a.hi,
                     a.ld, M, K / S, S > 1 ? ws.part : nullptr, N);
  if (S > 1 && reduce) launch_reduce<BN>(pol, ws.part, N, M, S, ntiles, st);
  return hipGetLastError();
}

// Default launch choices: the cached-step row counts are HBM-bound and want
// every CU streaming weights; many rows are MFMA-bound and take
// gemm_pp_kernel.  `paired`: the activations carry the lo part (twice the MFMA
// work per weight byte).  Measured choices:
//  * gemm_pp_kernel for every projection from 512 rows, below by estimate
//    (plan_bf16).  8B shape, us per layer, the four projections on
//    gemm_bf16_kernel / on gemm_pp_kernel: one pass 240 rows 173 / 197, 300
//    rows 234 / 225, 376 rows 245 / 225, 504 rows 279 / 238.  Whole layers with
//    the pair, all on gemm_bf16_kernel / gate/up alone on gemm_pp_kernel / all
//    on it: 300 rows 359 / 381 / 407, 376 rows 401 / 406 / 422, 400 rows 408 /
//    402 / 436, 440 rows 420 / 406 / 435, 511 rows 465 / 433 / 449;
//  * row tiles of gemm_bf16_kernel: 128 rows, except 256 for the one-pass
//    gate/up from 129 to 256 rows (one row tile instead of two); 64- and 192-row
//    tiles and the 256-row tiles elsewhere measured slower;
//  * QKV: 96-column tiles (128 column tiles at d = 4096 with 32 + 2 x 32 heads:
//    with the automatic split-K, 2 ways up to 128 rows, 256 workgroups where
//    128-column tiles left 64 CUs idle);
//  * gate/up: 96-column tiles (one workgroup per CU at 2F = 24576; the planner
//    falls back to 128 where 96 does not divide 2F);
//  * LM head: gemm_pp_kernel on 256-column tiles from 129 rows, where the
//    vocabulary has enough of them (lm_plan; 126464 ids: 120 rows 218 / 211, 240
//    rows 370 / 297, 480 rows 651 / 494; 152064 ids: 120 rows 249 / 268, 240 rows
//    407 / 358), which halves the activation reads per weight read; below that
//    the smaller tiles' last round is fuller;
//  * O / down (N = d): 128-column tiles with split-K; up to 128 rows O takes
//    64-column tiles and split-K 4, which halves the float32 partials of the
//    8-way split.
static GemmCfg default_cfg(const char* kind, int M, bool paired) {
  if (!strcmp(kind, "lm")) return GemmCfg{128, 1, 4, M > 128 ? -1 : 0};
  if (M > 511) return GemmCfg{128, 0, 4, -1};
  if (!strcmp(kind, "qkv")) return GemmCfg{96, 0, 4, 0};
  if (!strcmp(kind, "gate_up")) {
    GemmCfg c{96, 1, 4, 0};
    if (!paired && M > 128 && M <= 256) c.bm = 256;   // one row tile: 9% faster at 240 rows
    return c;
  }
  if (!strcmp(kind, "o") && M <= 128) return GemmCfg{64, 4, 4, 0};
  return GemmCfg{128, 0, 4, 0};
}

// tile widths: 64, 96 and 128 (gemm_bf16_kernel), 128, 192 and 256 (gemm_pp_kernel)
template <class Pol> static int any_bn(const Pol&, int bn) {
  return bn == 64 || bn == 96 || bn == 128 || bn == 192 || bn == 256;
}
// any width whose tiles divide the heads' concatenated halves (the epilogue's
// 8-column groups then never straddle a head)
static int qkv_bn(const PolQKV<bf16_t, f16_t>& p, int bn) {
  return any_bn(p, bn) && ((p.H + 2 * p.Hkv) * p.dh) % bn == 0 && (p.dh / 2) % 8 == 0;
}

hipError_t gemm_qkv(int dtype, const ActIn& a, int M, int d, const void* wq, const void* wk,
                    const void* wv, int H, int Hkv, int dh, const QKVOut& o, SplitWs ws,
                    hipStream_t st) {
  const int N = (H + 2 * Hkv) * dh;
  if (dtype == 0) {
    PolQKV<float> p{(const float*)wq, (const float*)wk, (const float*)wv, d, H, Hkv, dh,
                    (float*)o.q, (float*)o.kc, (float*)o.vc, o.cap, o.n_cached, o.n_rows, o.rope,
                    o.rope_per_seq};
    return run_f32(p, a, M, d, N, ws, st);
  }
  PolQKV<bf16_t, f16_t> p{(const bf16_t*)wq, (const bf16_t*)wk, (const bf16_t*)wv, d, H, Hkv, dh,
                          (f16_t*)o.q, (f16_t*)o.kc, (f16_t*)o.vc, o.cap, o.n_cached,
                          o.n_rows, o.rope, o.rope_per_seq};
  return run_bf16("qkv", p, a, M, d, N, default_cfg("qkv", M, a.lo != nullptr), ws, st, qkv_bn);
}

hipError_t gemm_resid(int dtype, const char* kind, const ActIn& a, int M, int K, const void* w,
                      int N, float* resid, SplitWs ws, hipStream_t st, const NormTo* nrm) {
  hipError_t e;
  bool fuse;
  if (dtype == 0) {
    PolResid<float> p{(const float*)w, K, N, resid};
    const int S = f32_split(M, K, N, ws.floats);
    fuse = resid_norm_ok(S, N, nrm);
    e = run_f32(p, a, M, K, N, ws, st, !fuse);
    if (e == hipSuccess && fuse) launch_resid_norm<float>(S, M, N, ws.part, resid, nrm, st);
  } else {
    PolResid<bf16_t> p{(const bf16_t*)w, K, N, resid};
    const GemmCfg c = plan_bf16(kind, p, a, M, K, N, default_cfg(kind, M, a.lo != nullptr), ws,
                                any_bn<PolResid<bf16_t>>);
    fuse = resid_norm_ok(c.s, N, nrm);
    e = launch_plan(p, a, M, K, N, c, ws, st, !fuse);
    if (e == hipSuccess && fuse) launch_resid_norm<bf16_t>(c.s, M, N, ws.part, resid, nrm, st);
  }
  if (e != hipSuccess || !nrm) return e;
  if (fuse) return hipGetLastError();
  return launch_norm(dtype, resid, N, nrm->g, nrm->eps, nrm->y, M, M, 0, 0, st);
}

hipError_t gemm_swiglu(int dtype, const ActIn& a, int M, int d, const void* wg, const void* wu,
                       int F, const ActOut& act, SplitWs ws, hipStream_t st) {
  if (dtype == 0) {
    PolSwiGLU<float> p{(const float*)wg, (const float*)wu, d, F, act};
    return run_f32(p, a, M, d, 2 * F, ws, st);
  }
  PolSwiGLU<bf16_t> p{(const bf16_t*)wg, (const bf16_t*)wu, d, F, act};
  return run_bf16("gate_up", p, a, M, d, 2 * F, default_cfg("gate_up", M, a.lo != nullptr), ws, st,
                  any_bn<PolSwiGLU<bf16_t>>);
}

hipError_t gemm_store_f32(const ActIn& a, int M, int K, const void* w, int N, float* c, int ldc,
                          SplitWs ws, hipStream_t st) {
  PolStore<float> p{(const float*)w, K, ldc, c};
  return run_f32(p, a, M, K, N, ws, st);
}

// Merges the partial statistics of one row (one workgroup per row), in a
// fixed order: deterministic.  120 rows of 1976 segments: 30 us with a list
// kept per thread and 8 block-wide searches, 20 us with row_stats_end.
__global__ void __launch_bounds__(256) lm_merge_kernel(LMParts part, int k,
                                                       int32_t* __restrict__ argmax,
                                                       float* __restrict__ conf,
                                                       int32_t* __restrict__ topk_ids,
                                                       float* __restrict__ topk_w) {
  __shared__ RowStatShared sh;
  const int row = blockIdx.x, tid = threadIdx.x, n = part.n_part;
  const float4* H = (const float4*)part.head + (size_t)row * n;
  const LMTail* L = part.tail + (size_t)row * n;
  float m = -INFINITY, s = 0.f, v = -INFINITY;
  int i = STAT_NONE;
  // this thread's segments j = tid + 256 c, in that order, CH loaded at a time
  constexpr int CH = 8;
  for (int j0 = tid; j0 < n; j0 += 256 * CH) {
    float4 h[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) h[c] = H[min(j0 + 256 * c, n - 1)];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      if (j0 + 256 * c >= n) break;
      if (h[c].y > 0.f) {
        if (h[c].x > m) { s = s * expf(m - h[c].x) + h[c].y; m = h[c].x; }
        else s += h[c].y * expf(h[c].x - m);
      }
      if (stat_better(h[c].z, __float_as_int(h[c].w), v, i)) { v = h[c].z; i = __float_as_int(h[c].w); }
    }
  }
  row_stats_end(sh, m, s, v, i, row, k, argmax, conf, topk_ids, topk_w,
                [&](float (&tv)[STAT_K], int (&ti)[STAT_K], float fv, int fi) {
    for (int j0 = tid; j0 < n; j0 += 256 * CH) {
      float4 h[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) h[c] = H[min(j0 + 256 * c, n - 1)];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int j = j0 + 256 * c, id0 = __float_as_int(h[c].w);
        if (j >= n || stat_better(fv, fi, h[c].z, id0)) continue;
        stat_insert(tv, ti, h[c].z, id0);
        const LMTail l = L[j];
#pragma unroll
        for (int q = 0; q < 7; ++q)
          if (!stat_better(fv, fi, l.v[q], l.id[q])) stat_insert(tv, ti, l.v[q], l.id[q]);
      }
    }
  });
}

size_t lm_stats_ws_bytes(int M, int N) {
  return (size_t)M * (N / 64) * (sizeof(LMHead) + sizeof(LMTail));
}

// Launch plan of the LM head: 256-column tiles of one or two groups of 128
// rows, whichever takes less time; a small vocabulary has too few of them
// (2048 ids, 240 rows: 50 us on 128-column tiles, 68 on these).
static GemmCfg lm_plan(const PolLMStats<bf16_t>& p, const ActIn& a, int M, int K, int N) {
  const bool pair = a.lo != nullptr;
  GemmCfg c = cfg_override("lm", default_cfg("lm", M, pair));
  const float us1 = pp_cost(1, M, K, N, pair), us4 = pp_cost(4, M, K, N, pair);
  const float us = (float)ceil_div(N / 128 * ceil_div(M, 128), 256) *
                   (K / 64 * bf16_step_us(128, 128, pair) + PP_FIXED_US);
  if (c.pp && pp_aligned(p, a) && N % 256 == 0 && (us1 < us4 ? us1 : us4) < us) c.pp = us1 < us4 ? 1 : 4;
  else c.pp = 0;
  return c;
}

hipError_t lm_head_stats(const ActIn& a, int M, int K, const void* w, int N, int mask_id, int k,
                         void* stats_ws, float* logits, int32_t* argmax, float* conf,
                         int32_t* topk_ids, float* topk_w, hipStream_t st) {
  LMParts parts{(LMHead*)stats_ws, (LMTail*)((LMHead*)stats_ws + (size_t)M * (N / 64)), N / 64};
  PolLMStats<bf16_t> p{(const bf16_t*)w, K, N, mask_id, parts, logits, N};
  const GemmCfg c = lm_plan(p, a, M, K, N);
  const SplitWs none{nullptr, 0};
  hipError_t e;
  if (c.pp == 1) e = launch_pp<256, 256, 2, 4>(p, a, M, K, N, 1, none, st, false);
  else if (c.pp == 4) e = launch_pp<128, 256, 2, 4>(p, a, M, K, N, 1, none, st, false);
  else e = launch_bf16_pw<128, 128>(p, a, M, K, N, 1, c.pw, none, st, true);
  if (e != hipSuccess) return e;
  launch(lm_merge_kernel, dim3(M), dim3(256), 0, st, parts, k, argmax, conf, topk_ids, topk_w);
  return hipGetLastError();
}

}  // namespace ssm

#ifdef SSM_DEBUG
// The launch that a projection of a bfloat16 model takes (debug library only,
// for tests of the dispatch): kind is qkv, o, gate_up, down or lm, `weights`
// stands for the address of its weights.  out: 1 for gemm_pp_kernel or 0 for
// gemm_bf16_kernel, tile rows, tile columns, K splits.
extern "C" int32_t ssm_debug_gemm_plan(const char* kind, int32_t M, int32_t d, int32_t H,
                                       int32_t Hkv, int32_t F, int32_t V, int32_t pair,
                                       uint64_t weights, int32_t* out) {
  using namespace ssm;
  const bf16_t* w = (const bf16_t*)(uintptr_t)weights;
  const ActIn a{nullptr, pair ? (const bf16_t*)256 : nullptr, d, row_groups(M)};
  const int dh = d / H, nq = (H + 2 * Hkv) * dh;
  int maxn = nq > 2 * F ? nq : 2 * F;
  if (V > maxn) maxn = V;
  const SplitWs ws{nullptr, gemm_split_ws_floats(M, maxn)};
  const GemmCfg given = default_cfg(kind, M, pair != 0);
  GemmCfg c;
  if (!strcmp(kind, "qkv")) {
    PolQKV<bf16_t, f16_t> p{};
    p.wq = p.wk = p.wv = w;
    p.H = H; p.Hkv = Hkv; p.dh = dh;
    c = plan_bf16(kind, p, a, M, d, nq, given, ws, qkv_bn);
  } else if (!strcmp(kind, "gate_up")) {
    PolSwiGLU<bf16_t> p{};
    p.wg = p.wu = w;
    c = plan_bf16(kind, p, a, M, d, 2 * F, given, ws, any_bn<PolSwiGLU<bf16_t>>);
  } else if (!strcmp(kind, "lm")) {
    PolLMStats<bf16_t> p{};
    p.w = w;
    c = lm_plan(p, a, M, d, V);
    if (!c.pp) c.bn = 128;
  } else {
    PolResid<bf16_t> p{};
    p.w = w;
    c = plan_bf16(kind, p, a, M, !strcmp(kind, "down") ? F : d, d, given, ws, any_bn<PolResid<bf16_t>>);
  }
  out[0] = c.pp != 0;
  out[1] = c.pp ? PP_TILES[c.pp - 1].bm : c.bm;
  out[2] = c.pp ? PP_TILES[c.pp - 1].bn : c.bn;
  out[3] = c.s;
  return 0;
}
#endif
