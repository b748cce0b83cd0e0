// Shared device helpers of the SSM HIP library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;
typedef _Float16 f16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

#define SSM_WAVE 64

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// float -> bfloat16, round to nearest even (v_cvt_pk_bf16_f32).
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
// Two floats -> packed bfloat16 pair, a in the low half.
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}

// Element load/store as float for the two storage types.
template <typename T> struct Elem;
template <> struct Elem<float> {
  __device__ __forceinline__ static float ld(const float* p) { return *p; }
  __device__ __forceinline__ static void st(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  __device__ __forceinline__ static float ld(const bf16_t* p) { return bf2f(*p); }
  __device__ __forceinline__ static void st(bf16_t* p, float v) { *p = f2bf(v); }
};
// float16 (round to nearest even): the attention operands q, k, v of a
// bfloat16 model (three more significand bits than bfloat16).
template <> struct Elem<f16_t> {
  __device__ __forceinline__ static float ld(const f16_t* p) { return (float)*p; }
  __device__ __forceinline__ static void st(f16_t* p, float v) { *p = (f16_t)v; }
};

template <typename T> __device__ __forceinline__ float ldf(const T* p) { return Elem<T>::ld(p); }
template <typename T> __device__ __forceinline__ void stf(T* p, float v) { Elem<T>::st(p, v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Block-wide sum for blockDim.x a multiple of 64 (<= 1024); `red` has >= 16 floats.
__device__ __forceinline__ float block_sum(float v, float* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];   // fixed order: deterministic
  return t;
}

// Row of workgroup w of a grid of one workgroup per row, for rows written in
// fragment order: workgroups are dealt to the 8 XCDs round-robin, so this
// gives each XCD a contiguous range of rows.  The 16 rows of a row group
// then share an L2, which merges their 16-byte chunks into whole lines (8 rows
// to a line of 128 bytes); rows dealt out in turn leave 8 XCDs writing parts of every line (RMSNorm of 3840
// rows of 4096: 36.3 us, 23.9 with whole lines; 1776 rows: 19.4 and 12.5).
__device__ __forceinline__ int xcd_row(int w, int total) {
  const int per = total / 8;
  return w < per * 8 ? (w % 8) * per + (w / 8) : w;
}

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
