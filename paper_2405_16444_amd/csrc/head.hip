// First-token head (paper Sec. 2: the prefill phase ends when the first token is
// generated): final RMSNorm of the last query token, vocabulary projection, greedy pick.
// A matrix-vector product: every weight is read once and used once, so the bound is HBM
// (vocab * d * sizeof(T) bytes), not the matrix cores.
#include "common.h"
#include "kernels.h"
#include <algorithm>
#include <mutex>

namespace cb {

// logits[v] = sum_e xn[e] * W[v, e], xn = T(h / sqrt(mean h^2 + eps) * gain) -- rounded to the
// storage type like every other projection input.  One workgroup of 16 wavefronts per CU, all resident at once; each
// normalises the row for itself (16-32 KB of L2 hits) instead of a separate launch.  A wavefront takes one vocabulary
// row after the other, kHeadChunks KB of it per round and two rounds in flight (8 KB per wavefront, 128 KB per CU:
// what the latency of HBM asks for at full rate), across rows and across the normalisation: the first loads are on
// their way before it.  The weights are read once and by nobody else, so the loads are non-temporal.
// 32000 x 8192 bf16: 125 us (4.2 TB/s) and a launch of 12 us for the pick -> 93 us together (5.7 TB/s); 64000 x 7168:
// 6.3 TB/s, a plain read of as much memory runs at 6.5.  Measured on the way: ordinary loads 101 us; four rows at a
// time instead of 4 KB of one 106 us; four workgroups of 256 per CU 127 us, 13 us of them the 1024 arrivals at the pick.
constexpr int kHeadThreads = 1024, kHeadWaves = kHeadThreads / 64, kHeadWorkgroups = 256;
constexpr int kHeadChunks = 4;          // 16-byte chunks of a row per lane and round

// Order-preserving map of a logit and its index to one integer: a larger logit, then a lower index, is larger.
// (-0 counts as +0; NaN, whatever its sign and payload, counts as less than every number, -infinity included.)  Keys lie
// strictly between 0 and all ones, the two values the pick below uses for itself: idx < 2^31 keeps the low word above 0,
// and no number's high word exceeds that of +infinity.
__device__ __forceinline__ unsigned long long pick_key(float v, int idx) {
  const unsigned u = __float_as_uint(v + 0.f);
  const bool nan = (u & 0x7FFFFFFFu) > 0x7F800000u;
  const unsigned ord = nan ? 0u : u & 0x80000000u ? ~u : u | 0x80000000u;
  return ((unsigned long long)ord << 32) | (0xFFFFFFFFu - (unsigned)idx);
}

// The greedy pick: every workgroup contributes its best (key, as above) with one device-wide atomic maximum, the last
// one to arrive (a counter) writes the token and puts pick[0] (the maximum) and pick[1] (the counter) back to zero for the
// next call.  Maximum and counter travel through atomics alone, and the counter is added to only after the maximum
// has come back, so no cache has to be written back or invalidated.  A maximum does not depend on the order.
template <typename T>
__global__ __launch_bounds__(kHeadThreads) void lm_head_kernel(const float *__restrict__ h, const T *__restrict__ gain,
                                                               const T *__restrict__ w, int d, int vocab, float eps,
                                                               float *__restrict__ logits, int32_t *__restrict__ token,
                                                               unsigned long long *__restrict__ pick) {
  extern __shared__ __attribute__((aligned(16))) float xn[];
  __shared__ float red[kHeadWaves];
  __shared__ unsigned long long s_best[kHeadWaves];
  constexpr int N = Vec16<T>::N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chunks = d / N;                            // 16-byte chunks per row
  const int rounds = (chunks + 64 * kHeadChunks - 1) / (64 * kHeadChunks);
  const int step = (int)gridDim.x * kHeadWaves;
  f32x4 buf[2][kHeadChunks];
  int lrow = (int)blockIdx.x * kHeadWaves + wave, lk = 0;          // row and round that is loaded next
  auto load = [&](f32x4 (&dst)[kHeadChunks]) {
    if (lrow < vocab) {
      const T *row = w + (size_t)lrow * d;
#pragma unroll
      for (int a = 0; a < kHeadChunks; ++a) {
        const int c = min(lane + 64 * (kHeadChunks * lk + a), chunks - 1);   // past the row's end: its last chunk, ignored
        dst[a] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(row + c * N));
      }
      if (++lk == rounds) { lk = 0; lrow += step; }
    }
  };
  load(buf[0]);
  load(buf[1]);
  float ss = 0.f;
  for (int e = threadIdx.x; e < d; e += kHeadThreads) { const float v = h[e]; ss += v * v; }
  ss = wave_sum(ss);
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int i = 0; i < kHeadWaves; ++i) ss += red[i];
  const float inv = rsqrtf(ss / (float)d + eps);
  for (int e = threadIdx.x; e < d; e += kHeadThreads) xn[e] = to_f32(from_f32<T>(h[e] * inv * to_f32(gain[e])));
  __syncthreads();
  unsigned long long best = 0;                         // below every key
  float sum = 0.f;
  int row = (int)blockIdx.x * kHeadWaves + wave, k = 0;
  auto consume = [&](const f32x4 (&src)[kHeadChunks]) {
#pragma unroll
    for (int a = 0; a < kHeadChunks; ++a) {
      const int c = lane + 64 * (kHeadChunks * k + a);
      if (c < chunks) {
        Vec16<T> v;
        v.raw = __builtin_bit_cast(decltype(v.raw), src[a]);
#pragma unroll
        for (int i = 0; i < N; ++i) sum = fmaf(v.get(i), xn[c * N + i], sum);
      }
    }
    if (++k < rounds) return;
    const float s = wave_sum(sum);
    if (lane == 0) logits[row] = s;
    const unsigned long long key = pick_key(s, row);
    if (key > best) best = key;
    sum = 0.f;
    k = 0;
    row += step;
  };
  while (row < vocab) {
    consume(buf[0]);
    load(buf[0]);
    if (row >= vocab) break;
    consume(buf[1]);
    load(buf[1]);
  }
  if (lane == 0) s_best[wave] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kHeadWaves; ++i)
      if (s_best[i] > best) best = s_best[i];
    const unsigned long long before = __hip_atomic_fetch_max(&pick[0], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the addend depends on the maximum's answer, which orders the two
    const unsigned long long one = before == ~0ull ? 2ull : 1ull;            // no key is all ones: always 1
    const unsigned long long arrived = __hip_atomic_fetch_add(&pick[1], one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (arrived + 1 == gridDim.x) {
      const unsigned long long top = __hip_atomic_exchange(&pick[0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&pick[1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      token[0] = (int32_t)(0xFFFFFFFFu - (unsigned)top);
    }
  }
}

hipError_t launch_lm_head(int dtype, const float *h_row, const void *gain, const void *w, int d, int vocab,
                          float eps, float *logits, int32_t *token, unsigned long long *pick, hipStream_t s) {
  const dim3 grid(std::min((vocab + kHeadWaves - 1) / kHeadWaves, kHeadWorkgroups));
  const size_t smem = (size_t)d * sizeof(float);
  // d = 16384 needs 64 KB of dynamic LDS on top of the static array: above the default limit
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&lm_head_kernel<float>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 4);
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&lm_head_kernel<bf16>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 4);
  });
  if (dtype == 0)
    hipLaunchKernelGGL(lm_head_kernel<float>, grid, dim3(kHeadThreads), smem, s, h_row, (const float *)gain,
                       (const float *)w, d, vocab, eps, logits, token, pick);
  else
    hipLaunchKernelGGL(lm_head_kernel<bf16>, grid, dim3(kHeadThreads), smem, s, h_row, (const bf16 *)gain,
                       (const bf16 *)w, d, vocab, eps, logits, token, pick);
  return hipGetLastError();
}

}  // namespace cb
