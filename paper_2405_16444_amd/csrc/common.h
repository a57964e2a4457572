// Shared device/host helpers of the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cb {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWave = 64;

// float <-> storage type; bf16 uses round-to-nearest-even (the compiler's
// conversion, a hardware instruction on gfx950).
template <typename T> __device__ __forceinline__ float to_f32(T v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v) { return (T)v; }

// 16-byte vector of storage elements
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  float4 raw;
  __device__ __forceinline__ float get(int i) const { return ((const float *)&raw)[i]; }
  __device__ __forceinline__ void set(int i, float v) { ((float *)&raw)[i] = v; }
};
template <> struct Vec16<bf16> {
  static constexpr int N = 8;
  bf16x8 raw;
  __device__ __forceinline__ float get(int i) const { return (float)raw[i]; }
  __device__ __forceinline__ void set(int i, float v) { raw[i] = (bf16)v; }
};

// four adjacent elements
template <typename T> __device__ __forceinline__ float4 load4(const T *s);
template <> __device__ __forceinline__ float4 load4<float>(const float *s) { return *reinterpret_cast<const float4 *>(s); }
template <> __device__ __forceinline__ float4 load4<bf16>(const bf16 *s) {
  const bf16x4 v = *reinterpret_cast<const bf16x4 *>(s);
  return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}
template <typename T> __device__ __forceinline__ void store4(T *d, float a, float b, float c, float e);
template <> __device__ __forceinline__ void store4<float>(float *d, float a, float b, float c, float e) {
  *reinterpret_cast<float4 *>(d) = make_float4(a, b, c, e);
}
template <> __device__ __forceinline__ void store4<bf16>(bf16 *d, float a, float b, float c, float e) {
  bf16x4 v = {(bf16)a, (bf16)b, (bf16)c, (bf16)e};
  *reinterpret_cast<bf16x4 *>(d) = v;
}

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

// Sum over a 256-thread block; `red` is a __shared__ float[4]. Every thread gets the result.
__device__ __forceinline__ float block_sum_256(float v, float *red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = red[0] + red[1] + red[2] + red[3];
  __syncthreads();
  return r;
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace cb
