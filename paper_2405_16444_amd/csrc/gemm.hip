// Projections of the selectively recomputed rows (paper Sec. 4.2: Q/K/V of the
// selected tokens, then the ordinary attention and the rest of the layer).
// C[M, N] = A[M, K] * W[N, K]^T with both operands K-contiguous.
//
// bf16 storage: matrix-core MFMAs with float accumulation.  The main kernel
// (gemm_bf16_dma_kernel, v_mfma_f32_16x16x32_bf16) streams 64 .. 384 x 128 .. 256 x 64 tiles through LDS
// rings filled by direct global->LDS loads, with an XCD-aware tile order; a simpler register-staged
// 128x128x64 kernel (v_mfma_f32_32x32x16_bf16) covers K that is not a multiple of 64.
// float storage: float MFMAs (v_mfma_f32_32x32x2_f32) on small tiles.
// The SwiGLU and float-output epilogues work straight from the accumulator registers (a lane
// holds four adjacent columns of a row); the segment epilogue parks the tile in LDS and walks it
// row-major, 4 adjacent columns per lane, which lets the two wavefront halves of an operand-pair
// tile be added and gives the half-split rotary order its partner column.  A problem with too few tiles to fill the chip is split along K: the main
// kernel then stores raw partial sums and a second kernel adds them in a fixed order
// (no atomics: bitwise reproducible) and applies the epilogue.
// Epilogues:
//   EPI_SEG    up to three column segments (Q | K | V), each with its own weight
//              matrix, destination, optional destination-row map (scatter into the
//              KV cache) and optional rotary embedding at the row's position
//   EPI_SWIGLU silu(x Wg^T) * (x Wu^T)
//   EPI_F32    float output (+ residual)
#include "common.h"
#include "kernels.h"
#include <algorithm>
#include <cstdint>
#include <mutex>

namespace cb {

struct GemmParams {
  const void *a;
  int lda;
  const int32_t *a_rows;
  int M, K, N;          // N: total output columns (EPI_SWIGLU: d_ff)
  int n_seg;
  const void *w[3];
  const float *w_scale[3];   // non-NULL (direct-to-LDS kernel only): w[i] holds int8 values and output column c of
                             // segment i is w_scale[i][c] times the sum over them
  int nb[4];            // column boundaries of the segments
  void *dst[3];
  int ld[3];
  const int32_t *row_map[3];
  int rope[3];
  const float2 *rope_tab;
  const int32_t *row_pos;
  int head_dim;
  int rope_half;        // rotary pairs (i, i + head_dim/2) instead of (2i, 2i+1)
  int raw_partial;      // the main kernel only parks its sums in `partial`; the finish launch applies the epilogue
  int a_lo_off;         // > 0: the activations are a (high, low) bf16 pair, the low parts a_lo_off elements after
                        // the high parts of the same row; both are multiplied and their products added
  int hl_cols;          // output columns that take the pair (the leading ones; the others take the high parts alone)
  int hl_tiles_m, hl_tiles_n;   // direct-to-LDS kernel: tiles of those columns
  float *out_f32;
  const float *resid;
  const int32_t *resid_rows;
  float *partial;
  // finish launch of EPI_SEG: squared distance of the stored new values of segment s from row
  // dev_row[r] of dev_cache[s] (pitch = the segment's width), summed over the segments, for rows < n_dev
  float *dev_out;
  int n_dev;
  const void *dev_cache[3];
  const int32_t *dev_row;
  // finish launch of EPI_F32: RMSNorm of the finished row (gain norm_gain, NULL: none) into norm_out
  // (pitch norm_ld); norm_lo_off > 0 also stores the rounding remainder norm_lo_off elements further on
  const void *norm_gain;
  void *norm_out;
  int norm_ld, norm_lo_off;
  float norm_eps;
  int splits, k_per_split;
  // EPI_SWIGLU: workgroup ids >= tail_first share the tiles of the last, partly filled round of
  // workgroups, tail_splits of them per tile, each over tail_k_per_split of K
  int tail_first, tail_splits, tail_k_per_split;
  // K split dealt to the XCDs (splits = 2, 4 or 8): XCD x computes split x % splits of the n-tiles
  // congruent to x / splits mod 8 / splits, so each L2 holds only its own K slice of the activations
  int xcd_split;
  int k_stagger;        // column tiles start at different k-tiles and wrap around (see pitch_is_power_of_two)
};

// weight row that feeds tile column gc (clamped into range)
// (es: elements of T per weight element, for byte-addressed callers)
template <typename T, int EPI>
__device__ __forceinline__ const T *weight_row(const GemmParams &p, int gc, int half_bn, int n0, int c, int es = 1) {
  if (EPI == EPI_SWIGLU) {
    // tile columns [0, half) come from the gate matrix, [half, 2*half) from the up matrix
    int which = c >= half_bn;
    int row = min(n0 + (which ? c - half_bn : c), p.N - 1);
    return reinterpret_cast<const T *>(p.w[which]) + (size_t)row * p.K * es;
  }
  gc = min(gc, p.N - 1);
  int s = 0;
  if (p.n_seg > 1 && gc >= p.nb[1]) s = 1;
  if (p.n_seg > 2 && gc >= p.nb[2]) s = 2;
  return reinterpret_cast<const T *>(p.w[s]) + (size_t)(gc - p.nb[s]) * p.K * es;
}

// the value a float becomes when stored in the storage type
template <typename T> __device__ __forceinline__ float as_stored(float v) { return to_f32(from_f32<T>(v)); }

// Column offset from an output column to the channel it forms a rotary pair with when heads are in
// the (i, i + head_dim/2) order.  Segments are whole heads, so gc % head_dim is the channel.
__device__ __forceinline__ int rope_partner_offset(const GemmParams &p, int gc) {
  const int half = p.head_dim / 2;
  return gc % p.head_dim < half ? half : -half;
}

// EPI_SEG: the values of output columns gc .. gc+3 of logical row gr after the rotary embedding
// (a no-op for segments without it); *seg / *lcol receive the segment and the column inside it.
// u: with p.rope_half, the values of columns gc + rope_partner_offset .. + 3.
__device__ __forceinline__ float4 seg_rotate(float4 v, float4 u, int gr, int gc, const GemmParams &p, int *seg,
                                             int *lcol) {
  int s = 0;
  if (p.n_seg > 1 && gc >= p.nb[1]) s = 1;
  if (p.n_seg > 2 && gc >= p.nb[2]) s = 2;
  const int lc = gc - p.nb[s];
  *seg = s;
  *lcol = lc;
  if (!p.rope[s]) return v;
  const int half = p.head_dim / 2;
  float4 o;
  if (p.rope_half) {
    const int ch = lc % p.head_dim;
    const bool first = ch < half;
    const float2 *t = p.rope_tab + (size_t)p.row_pos[gr] * half + (first ? ch : ch - half);
    const float2 c0 = t[0], c1 = t[1], c2 = t[2], c3 = t[3];
    if (first) {          // x0' = x0 cos - x1 sin, the partner holds x1
      o.x = v.x * c0.x - u.x * c0.y;
      o.y = v.y * c1.x - u.y * c1.y;
      o.z = v.z * c2.x - u.z * c2.y;
      o.w = v.w * c3.x - u.w * c3.y;
    } else {              // x1' = x0 sin + x1 cos, the partner holds x0
      o.x = u.x * c0.y + v.x * c0.x;
      o.y = u.y * c1.y + v.y * c1.x;
      o.z = u.z * c2.y + v.z * c2.x;
      o.w = u.w * c3.y + v.w * c3.x;
    }
  } else {
    const float2 *t = p.rope_tab + (size_t)p.row_pos[gr] * half + (lc % p.head_dim) / 2;
    const float2 c0 = t[0], c1 = t[1];
    o.x = v.x * c0.x - v.y * c0.y;
    o.y = v.x * c0.y + v.y * c0.x;
    o.z = v.z * c1.x - v.w * c1.y;
    o.w = v.z * c1.y + v.w * c1.x;
  }
  return o;
}

// One group of 4 adjacent output columns (gc .. gc+3) of logical row gr.
// v: accumulated values; u: EPI_SWIGLU: the matching "up" values; EPI_SEG with p.rope_half: the
// values of columns gc + rope_partner_offset .. + 3.  (EPI_F32 sums always go through `partial`
// and are finished by resid_norm_finish_kernel.)
template <typename T, int EPI>
__device__ __forceinline__ void apply_epilogue(float4 v, float4 u, int gr, int gc, const GemmParams &p) {
  if (EPI == EPI_SEG) {
    int s, lc;
    v = seg_rotate(v, u, gr, gc, p, &s, &lc);
    const int dr = p.row_map[s] ? p.row_map[s][gr] : gr;
    store4<T>(reinterpret_cast<T *>(p.dst[s]) + (size_t)dr * p.ld[s] + lc, v.x, v.y, v.z, v.w);
  } else if (EPI == EPI_SWIGLU) {
    float4 o;
    o.x = v.x / (1.f + expf(-v.x)) * u.x;
    o.y = v.y / (1.f + expf(-v.y)) * u.y;
    o.z = v.z / (1.f + expf(-v.z)) * u.z;
    o.w = v.w / (1.f + expf(-v.w)) * u.w;
    store4<T>(reinterpret_cast<T *>(p.dst[0]) + (size_t)gr * p.ld[0] + gc, o.x, o.y, o.z, o.w);
  }
}

// Walks `rows` x BN floats parked in LDS (pitch `pitch`); m0/n0: first logical row /
// first output column of this block of rows; z: K-split index of the workgroup.
template <typename T, int EPI, int BN>
__device__ __forceinline__ void lds_epilogue(const float *sC, int pitch, int rows, int m0, int n0, int z,
                                             const GemmParams &p) {
  constexpr int OUT_COLS = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int GROUPS = OUT_COLS / 4;
  for (int g = threadIdx.x; g < rows * GROUPS; g += (int)blockDim.x) {
    const int r = g / GROUPS, c = (g % GROUPS) * 4;
    const int gr = m0 + r, gc = n0 + c;
    if (gr >= p.M || gc >= p.N) continue;
    const float4 v = *reinterpret_cast<const float4 *>(sC + r * pitch + c);
    if (EPI != EPI_SWIGLU && (p.splits > 1 || p.raw_partial)) {
      *reinterpret_cast<float4 *>(p.partial + ((size_t)z * p.M + gr) * p.N + gc) = v;
    } else {
      float4 u = v;
      if (EPI == EPI_SWIGLU) u = *reinterpret_cast<const float4 *>(sC + r * pitch + OUT_COLS + c);
      // the tile holds whole heads (its width is a multiple of head_dim), so the partner is parked too
      if (EPI == EPI_SEG && p.rope_half)
        u = *reinterpret_cast<const float4 *>(sC + r * pitch + c + rope_partner_offset(p, gc));
      apply_epilogue<T, EPI>(v, u, gr, gc, p);
    }
  }
}

// ---------------------------------------------------------------------------
// Main bf16 kernel.
//   tile        BM = 16 RB WM rows x BN = 16 CB WN columns (kDmaTiles) x 64 k per stage (128-byte rows: every global
//               request is a whole cache line)
//   wavefronts  WM x WN, each RB x CB blocks of 16 x 16, one v_mfma_f32_16x16x32_bf16 each per 32-deep k-step: 2 x 2 (one per
//               SIMD) for the 128-column tiles of few rows, 2 x 4 for 256 columns and 4 x 2 for the widths between and the tall
//               tiles, both two per SIMD.  Operand reads are issued by hand (inline ds_read_b128 + explicit s_waitcnt
//               lgkmcnt) one half-step (half of the wavefront's row blocks of one k-step) ahead of the MFMAs that use them,
//               slotted between those MFMAs.
//   LDS rings   activation tile (BM rows x 128 bytes) and weight tile (BN rows x 128 bytes), as
//               many stages of both as fit in 160 KB, up to 6 (dma_even_stages below).
//               Both are filled by global_load_lds_dwordx4 (no register staging).  A
//               wavefront-wide load writes 1 KB contiguously (lane l -> byte 16*l),
//               i.e. 8 rows x 8 chunks; lane l fetches global chunk (l%8) ^ f(row) of
//               row l/8, f(r) = (r&7) ^ ((r>>3)&1), so that the later 16-byte operand
//               reads of 8 (and of 16) consecutive rows hit distinct bank groups
//               (XOR swizzle instead of padding).
//   pipeline    one barrier per k-tile, placed before the LAST half-step of tile t: by
//               then every wavefront holds its last fragments of stage t in
//               registers, so after "tile t+1 landed" (s_waitcnt vmcnt) + barrier the
//               stage is refilled with tile t+S and the first fragments of tile t+1
//               are requested while the last MFMAs of tile t run.  The loads of a tile
//               are spread over four half-steps (no burst on the memory pipeline).  The
//               compiler does not order LDS reads against these loads, hence the
//               explicit waits; plain s_barrier is used because __syncthreads()
//               would drain every outstanding load.
//   tile order  1-D grid; workgroup id -> (xcd = id % 8, j = id / 8); an XCD walks
//               its own n-tiles (n % 8 == xcd) in groups of 8 m-tiles (xcd_tile), so the
//               workgroups that share a weight or activation tile run together on one L2.
//               With a K split of 2, 4 or 8 the XCDs are dealt one split each (GemmParams::xcd_split),
//               so an L2 only ever fetches its own K slice of the activations.
// Requires K % 64 == 0 and k_per_split % 64 == 0.
// ---------------------------------------------------------------------------
constexpr int DMA_BK = 64;
// Stages of the two rings.  The waits count outstanding loads in issue order, so the depth that counts is that of the
// SHALLOWER ring: once a wavefront waits for its youngest needed activation tile, every weight tile requested before
// that has to be there too.  Both rings are therefore equally deep wherever 160 KB hold three stages or more of both (bf16: rows and
// columns of the tile together at most 426; int8 weights: rows and half the columns); larger tiles (bf16 192 x 256, 256 x 224, 320 x 160
// and up, 384 x 128; int8 384 x 160) keep two activation stages and three weight stages, their k-tiles last as long as a load takes.  With two activation
// stages everywhere (and 80 KB rings, two workgroups per CU, for the small tiles) a weight tile was never more than one
// k-tile ahead.  Launch with finish, bf16, before -> after: gate/up 28672 x 4096 at 64 / 128 / 256 rows 57 -> 54, 61 -> 58,
// 76 -> 67 us, at 640 rows of 57344 x 8192 603 -> 554 us; down 4096 x 14336 at 64 / 128 / 256 rows 36 -> 32, 41 -> 37, 51 -> 46 us;
// int8 gate/up 57344 x 8192 at 64 / 165 / 300 rows 146 -> 130, 192 -> 166, 356 -> 315 us.
// w8: int8 weights, 64 bytes per weight row and stage instead of 128 (the smallest tile: 80 KB, two workgroups per CU).
constexpr int dma_even_stages(int BM, int BN, bool w8) {
  const int n = 160 * 1024 / (BM * 128 + BN * (w8 ? 64 : 128)), most = w8 && BM == 64 && BN == 128 ? 5 : 6;
  return n > most ? most : n;
}
constexpr int dma_a_stages(int BM, int BN, bool w8 = false) {
  return dma_even_stages(BM, BN, w8) >= 3 ? dma_even_stages(BM, BN, w8) : 2;
}
constexpr int dma_w_stages(int BM, int BN, bool w8 = false) {
  return dma_even_stages(BM, BN, w8) >= 3 ? dma_even_stages(BM, BN, w8) : 3;
}
constexpr int dma_smem_bytes(int BM, int BN, bool w8 = false) {
  const int ring = dma_a_stages(BM, BN, w8) * BM * 128 + dma_w_stages(BM, BN, w8) * BN * (w8 ? 64 : 128);
  const int park = (BM < 128 ? BM : 128) * (BN + 4) * 4;
  return ring > park ? ring : park;
}

#define CB_GLDS16(gptr, lptr, cache)                                                       \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gptr), \
                                   (__attribute__((address_space(3))) void *)(lptr), 16, 0, cache)
constexpr int kCacheNt = 2;                            // the instruction's nt bit
// Variants of the main kernel: the start of a workgroup's k range may be staggered (a wrap test per tile, 0.7 % of a large launch)
// and the weight loads may be non-temporal as well.
enum { MODE_PLAIN, MODE_STAGGER, MODE_NT };

// LDS operand read issued by hand: the result registers are valid only after a matching
// lds_wait<N>() (N = number of younger reads that may still be in flight).
template <int OFF> __device__ __forceinline__ void lds_read16(bf16x8 &dst, unsigned addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
template <int OFF> __device__ __forceinline__ void lds_read8(u32x2 &dst, unsigned addr) {
  asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
// eight int8 weights -> the bf16 MFMA fragment (exact: |value| <= 128 needs 8 significant bits)
__device__ __forceinline__ bf16x8 int8x8_to_bf16(u32x2 q) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16)(float)(int)(signed char)(q[e >> 2] >> (8 * (e & 3)));
  return r;
}
template <int N> __device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N)); }
// ties a fragment to the preceding wait so that no use of it is scheduled before the wait
__device__ __forceinline__ void lds_pin(bf16x8 &f) { asm volatile("" : "+v"(f)); }
template <int N> __device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Tile walked by the j-th workgroup of an XCD (j < nblk * tiles_m).  The XCD owns the n-tiles
// congruent to its index mod 8 (nblk of them); row tiles are taken in groups of 8 and, inside a
// group, the row tiles of one n-tile come first.  The ~32 workgroups resident on an XCD then
// cover about 4 n-tiles x 8 m-tiles, so every weight tile and every activation tile fetched into
// its L2 serves several of them (with all row tiles innermost, a problem with many row tiles
// would share no activation tile at all).
constexpr int kGroupM = 8;
__device__ __forceinline__ void xcd_tile(int j, int xcd, int tiles_m, int nblk, int *nt, int *mt, int stride = 8) {
  const int per_group = nblk * kGroupM, full = tiles_m / kGroupM;
  int g = j / per_group, r, gm;
  if (g >= full) { g = full; r = j - full * per_group; gm = tiles_m - full * kGroupM; }
  else { r = j - g * per_group; gm = kGroupM; }
  *nt = xcd + stride * (r / gm);
  *mt = g * kGroupM + r % gm;
}

// Swaps the upper 32 lanes of x with the lower 32 lanes of y.
__device__ __forceinline__ void swap_halves(float &x, float &y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
// EPI_SWIGLU: gate and up of one output element have to end up in one lane.  A wavefront with an even number of column
// blocks holds the gate columns in the first half of them and the same up columns in the second.  With an odd number every block holds 8 gate
// columns (lanes 0 .. 31) and the same 8 up columns (lanes 32 .. 63), and pairs of blocks exchange halves (1 .. 2 % of the
// launch, so only there).
constexpr bool swiglu_mixed_blocks(int CB) { return CB % 2 != 0; }
// From the sums of two such blocks, x and y, in place: x the gate and y the up values of four adjacent output columns per
// lane -- lanes 0 .. 31 those of x's block, lanes 32 .. 63 those of y's.
__device__ __forceinline__ void pair_gate_up(f32x4 &x, f32x4 &y) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float a = x[r], b = y[r];
    swap_halves(a, b);
    x[r] = a;
    y[r] = b;
  }
}
// first of the four output columns, within the wavefront's, that a lane holds of block jb (and, mixed, of jb + 1)
template <int CB> __device__ __forceinline__ int swiglu_lane_col(int jb, int lane) {
  return swiglu_mixed_blocks(CB) ? (jb + (lane >> 5)) * 8 + ((lane >> 4) & 1) * 4 : jb * 16 + (lane >> 4) * 4;
}
// silu(g) * u = g * u / (1 + 2^(-g log2 e)) of four adjacent columns from gc on, into row orow
__device__ __forceinline__ void store_swiglu(const f32x4 &g, const f32x4 &u, bf16 *orow, int gc, int N) {
  float o[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float den = 1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g[r]);
    o[r] = g[r] * u[r] * __builtin_amdgcn_rcpf(den);
  }
  if (gc + 3 < N) {
    store4<bf16>(orow + gc, o[0], o[1], o[2], o[3]);
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (gc + r < N) orow[gc + r] = (bf16)o[r];
  }
}

// Completes the tiles that several workgroups of the SwiGLU launch shared along K.  The partial
// sums lie in register order: [slot][split][wavefront][16-row block i][16-column block jb][lane][4].
// One wavefront here owns four (wavefront, i, pair of blocks) units of a tile in turn: it adds both
// blocks over the splits in ascending K order and applies the epilogue.
template <int RB, int CB, int WM, int WN>
__global__ __launch_bounds__(256) void swiglu_tail_kernel(GemmParams p, int tiles_m, int tiles_n) {
  constexpr int BM = 16 * RB * WM, BN = 16 * CB * WN, NWV = WM * WN, HB = (CB + 1) / 2;
  constexpr bool MIXED = swiglu_mixed_blocks(CB);
  constexpr int UNITS = NWV * RB * HB;                    // per tile
  const int lane = threadIdx.x & 63;
  constexpr int PER = (UNITS + 15) / 16;                  // workgroups per tile, four wavefronts of four units
  const int slot = blockIdx.x / PER;
  const int xcd = slot & 7, j = (p.tail_first >> 3) + (slot >> 3);
  int nt, mt;
  xcd_tile(j, xcd, tiles_m, (tiles_n + 7) >> 3, &nt, &mt);
  if (nt >= tiles_n) return;
  for (int q = 0; q < 4; ++q) {
    const int u = ((blockIdx.x % PER) * 4 + (threadIdx.x >> 6)) * 4 + q;
    if (u >= UNITS) break;
    const int wave = u / (RB * HB), i = (u / HB) % RB, jb = u % HB * (MIXED ? 2 : 1);
    const bool two = jb + 1 < CB;                         // MIXED: the last block has no partner
    const int other = MIXED ? (two ? 64 * 4 : 0) : HB * 64 * 4;
    const float *pg = p.partial + (size_t)slot * p.tail_splits * (BM * BN) + (size_t)wave * (RB * CB * 4 * 64) +
                      (size_t)((i * CB + jb) * 64 + lane) * 4;
    f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = {0.f, 0.f, 0.f, 0.f};
    for (int zz = 0; zz < p.tail_splits; ++zz, pg += BM * BN) {
      x += *reinterpret_cast<const f32x4 *>(pg);
      y += *reinterpret_cast<const f32x4 *>(pg + other);
    }
    if (MIXED) pair_gate_up(x, y);
    const int wm = wave / WN, wn = wave % WN;
    const int gc = nt * (BN / 2) + wn * CB * 8 + swiglu_lane_col<CB>(jb, lane);
    const int gr = mt * BM + (WM == 4 ? i * WM + wm : wm * RB + i) * 16 + (lane & 15);
    if (gr >= p.M || (MIXED && !two && lane >= 32)) continue;
    store_swiglu(x, y, reinterpret_cast<bf16 *>(p.dst[0]) + (size_t)gr * p.ld[0], gc, p.N);
  }
}

// HL (EPI_SEG only): the leading p.hl_cols output columns take (high, low) bf16 pairs of the activations.  The
// activation tile of such a column tile holds BM/2 logical rows twice -- their high parts in its first half, their low
// parts in its second -- so the wavefronts with wm = 0 multiply the high parts and those with wm = 1 the low parts
// of the SAME output rows, and the two sets of sums are added in LDS before the epilogue.  Tiles of the
// other columns (Q beside K and V in one launch) are ordinary ones; which kind a workgroup has is uniform.
// W8: the weights are int8 (one byte per element in memory and in LDS, half the traffic of both); a fragment
// is expanded to bf16 in registers right before its k-step and the per-column scales multiply the finished sums.
// MODE: GemmPlan::mode.
template <int RB, int CB, int WM, int WN, int EPI, bool HL = false, bool W8 = false, int MODE = 0>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_dma_kernel(GemmParams p, int tiles_m, int tiles_n) {
  constexpr int NWV = WM * WN, BM = 16 * RB * WM, BN = 16 * CB * WN;
  constexpr int SA = dma_a_stages(BM, BN, W8), SW = dma_w_stages(BM, BN, W8), DMA_CP = BN + 4;
  constexpr int WE = W8 ? 1 : 2;                         // bytes per weight element
  static_assert(!HL || (EPI == EPI_SEG && WM == 2), "operand pairs are for the K/V projection only");

  constexpr int A_STAGE = BM * 128, W_STAGE = BN * 64 * WE, W_RING = SA * A_STAGE;
  constexpr int A_GROUPS = BM / 8, W_GROUPS = BN * WE / 16;   // wavefront-wide loads (1 KB each) of a tile
  constexpr int LA = A_GROUPS / NWV, LW = (W_GROUPS + NWV - 1) / NWV;   // per wavefront: 16-byte loads per lane
  static_assert(A_GROUPS % NWV == 0, "the load schedule");
  static_assert(SA >= 2 && SW >= SA, "the vmcnt bookkeeping below");
  static_assert(dma_smem_bytes(BM, BN, W8) <= 160 * 1024, "LDS of a CU");
  constexpr int IH = (RB + 1) / 2;                       // row blocks of a k-step's first half-step; the second has RB - IH
  constexpr int OUT_COLS = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  // Four wavefronts along M are dealt the row blocks in turn, so that a partly filled row tile occupies all of them alike (two that
  // share a SIMD would not gain by it: 28672 x 4096 at 500 rows 115 us with their blocks together, 119 us in turn; with
  // operand pairs wm = 0 has to be the high parts, wm = 1 the low parts).
  constexpr int RSTEP = WM == 4 ? 4 : 1;                     // tile row blocks between two blocks of a wavefront
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  // scalar, so that the LDS targets of the loads are computed on the scalar unit: a vector instruction of one
  // wavefront does not overlap the MFMAs of the other wavefront on its SIMD, it costs matrix-core time
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;              // WM x WN wavefronts
  const int row_blk0 = WM == 4 ? wm : wm * RB;                // block i of this wavefront is block row_blk0 + i * RSTEP of the tile

  // XCD-aware tile order
  int xcd = blockIdx.x & 7, j = blockIdx.x >> 3, tail_z = -1;
  if (EPI == EPI_SWIGLU && (int)blockIdx.x >= p.tail_first) {
    const int v = ((int)blockIdx.x - p.tail_first) >> 3;
    tail_z = v % p.tail_splits;
    j = (p.tail_first >> 3) + v / p.tail_splits;
  }
  int z, nt, mt;
  bool hl = false;                                       // this tile takes the pair
  int groups = 8;                                        // XCDs that share this split
  {
    // a split-dealing launch: XCDs that share one split; else all 8 share every split
    const bool dealt = EPI != EPI_SWIGLU && p.xcd_split;
    groups = dealt ? 8 / p.splits : 8;
    const int x = dealt ? xcd / p.splits : xcd;
    const int nblk = (tiles_n + groups - 1) / groups;
    const int nblk_hl = HL ? (p.hl_tiles_n + groups - 1) / groups : 0, cnt_hl = HL ? nblk_hl * p.hl_tiles_m : 0;
    const int per_z = nblk * tiles_m + cnt_hl;
    z = dealt ? xcd % p.splits : j / per_z;
    int r = dealt ? j : j - z * per_z;
    hl = HL && r < cnt_hl;                               // the pair tiles come first (they do twice the work per output)
    if (hl) {
      xcd_tile(r, x, p.hl_tiles_m, nblk_hl, &nt, &mt, groups);
      if (nt >= p.hl_tiles_n) return;
    } else {
      xcd_tile(r - cnt_hl, x, tiles_m, nblk, &nt, &mt, groups);
      if (nt >= tiles_n) return;
      if (HL) nt += p.hl_tiles_n;                        // hl_cols is a multiple of BN
    }
  }
  const int m0 = mt * (hl ? BM / 2 : BM), n0 = nt * OUT_COLS;
  const int kps = tail_z >= 0 ? p.tail_k_per_split : p.k_per_split;
  const int kb = (tail_z >= 0 ? tail_z : z) * kps;
  const int ke = min(p.K, kb + kps);
  const int nk = (ke - kb) / DMA_BK;
  const int k_first = MODE != MODE_PLAIN && p.k_stagger && nk > 0 ? (2 * (nt / groups) + nt % groups) % nk : 0;
  // first k of the t-th tile this workgroup walks (past the last: the last)
  auto k_of = [&](int t) {
    const int q = min(t, nk - 1) + k_first;
    return (MODE != MODE_PLAIN && q >= nk ? q - nk : q) * DMA_BK;
  };

  // global source of each of this lane's loads per tile (row pointer + swizzled chunk)
  const bf16 *src_a[LA];
  const char *src_w[LW];
  auto w_group = [&](int i) { return W_GROUPS % NWV == 0 ? wave + NWV * i : min(wave + NWV * i, W_GROUPS - 1); };
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (wave + NWV * i) * 8 + (lane >> 3);         // row of the activation tile
    const int chunk = (lane & 7) ^ ((r & 7) ^ ((r >> 3) & 1));
    const bool low = HL && hl && r >= BM / 2;
    int ar = min(m0 + (low ? r - BM / 2 : r), p.M - 1);
    if (p.a_rows) ar = p.a_rows[ar];
    src_a[i] = reinterpret_cast<const bf16 *>(p.a) + (size_t)ar * p.lda + chunk * 8 + kb +
               (low ? p.a_lo_off : 0);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    // a wavefront-wide load brings 1 KB: 8 rows of 128 bytes, or 16 rows of 64 bytes of int8 weights, whose four
    // 16-byte chunks are swizzled by f8(r) = (r >> 2) & 3 (the 8-byte fragment reads of 16 rows then hit 64 banks)
    // (where the tile's loads do not divide evenly the last ones are repeated: every wavefront issues the same number)
    const int r = W8 ? w_group(i) * 16 + (lane >> 2) : w_group(i) * 8 + (lane >> 3);   // row of the weight tile
    const int chunk = W8 ? (lane & 3) ^ ((r >> 2) & 3) : (lane & 7) ^ ((r & 7) ^ ((r >> 3) & 1));
    const char *wrow;
    if (EPI == EPI_SWIGLU) {
      // (swiglu_mixed_blocks)
      constexpr int WC = swiglu_mixed_blocks(CB) ? 16 : BN / WN, HC = WC / 2;   // run of gate, then of the same up columns
      const int which = (r % WC) / HC, oc = min(n0 + (r / WC) * HC + (r % HC), p.N - 1);
      wrow = reinterpret_cast<const char *>(p.w[which]) + (size_t)oc * p.K * WE;
    } else {
      wrow = reinterpret_cast<const char *>(weight_row<char, EPI>(p, n0 + r, BN / 2, n0, r, WE));
    }
    src_w[i] = wrow + chunk * 16 + kb * WE;
  }
  // load number idx of tile t: idx < LA activation, else weight; tile indices are clamped so
  // that every tile issues the same number of loads
  auto issue_one = [&](int t, int idx) {
    if (idx < LA) {
      const int k0 = k_of(t);
      CB_GLDS16(src_a[idx] + k0, smem + (t % SA) * A_STAGE + (wave + NWV * idx) * 1024, 0);
    } else {
      const int tw = t + SW - SA;                     // the weight ring runs SW - SA tiles further ahead
      const int k0 = k_of(tw);
      CB_GLDS16(src_w[idx - LA] + k0 * WE, smem + W_RING + (tw % SW) * W_STAGE + w_group(idx - LA) * 1024, MODE == MODE_NT ? kCacheNt : 0);
    }
  };
  auto issue_w = [&](int t) {
    const int k0 = k_of(t);
#pragma unroll
    for (int i = 0; i < LW; ++i)
      CB_GLDS16(src_w[i] + k0 * WE, smem + W_RING + (t % SW) * W_STAGE + w_group(i) * 1024, MODE == MODE_NT ? kCacheNt : 0);
  };

  // v_mfma_f32_16x16x32_bf16 with the WEIGHT fragment as its first operand: block (i, jb) of a wavefront is
  // 16 output rows x 16 output columns, and lane l ends up with row (l % 16), columns 4*(l/16) .. +3 of it,
  // i.e. four adjacent output columns (one 16-byte store, one rotary pair twice over).  Of the two MFMA
  // shapes this one sustains the higher rate on this chip once the operands are real data: the chip is
  // power-limited then, and the 16x16 shape moves half the accumulator registers per flop.
  f32x4 acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int jb = 0; jb < CB; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][jb][r] = 0.f;

  if (nk > 0) {
    // A fragment is 16 rows x 32 k: lane l reads the 16-byte chunk (l / 16) of the k-step's 64 bytes of row (l % 16)
    const int sw = (lane & 7) ^ ((lane >> 3) & 1);
    int rd[2];                                                    // k-step ks (32 deep) reads chunk 4*ks + l/16
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) rd[ks] = (lane & 15) * 128 + (((4 * ks + (lane >> 4)) ^ sw) << 4);
    const int a_off = row_blk0 * 16 * 128, b_off = (wn * (BN / WN)) * 128;
    int blk_ok = 0;                                    // bit i: 16-row block i of this wavefront holds a real row
#pragma unroll
    for (int i = 0; i < RB; ++i) blk_ok |= (m0 + (hl ? i : row_blk0 + i * RSTEP) * 16 < p.M) << i;
    blk_ok = __builtin_amdgcn_readfirstlane(blk_ok);
    // one scalar flag per block, re-read through an empty asm at every test: left alone the compiler hoists the
    // tests out of the loop as lane masks and rebuilds their complements with vector instructions inside it
    // (14 of the 48 vector instructions the loop had per k-tile; with these two changes it has 16)
    int row_ok[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) row_ok[i] = (blk_ok >> i) & 1;
    auto block_ok = [&](int i) {
      int v = row_ok[i];
      asm volatile("" : "+s"(v));
      return v != 0;
    };
    // A k-tile is walked in four HALF-STEPS hs = 2*ks + h: k-step ks (32 deep), row half h (IH of the wavefront's
    // 16-row blocks).  Activation fragments are double-buffered per half-step, weight fragments per k-step.
    // (int8 weights: the raw 8-byte fragments of the next k-step wait in fq and are expanded into fb[0] as the
    // k-step begins, each right before the first MFMA that uses it)
    bf16x8 fa[2][IH], fb[W8 ? 1 : 2][CB];
    u32x2 fq[W8 ? CB : 1];
    int rd8[2];                                        // int8 weights: 8 bytes of row (l % 16), k-step ks, k group l / 16
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      rd8[ks] = (lane & 15) * 64 + (((2 * ks + (lane >> 5)) ^ ((lane >> 2) & 3)) << 4) + ((lane >> 4) & 1) * 8;
    const int b_off8 = (wn * (BN / WN)) * 64;
    constexpr int NM = IH * CB;                        // MFMAs per (first) half-step per wavefront
    constexpr int NL = LA + LW;                        // loads per tile per lane
    constexpr int NSLOT = NM > IH + CB ? NM : IH + CB;
    // fragment number n (16 rows each, 2 KB apart) of the operand whose first fragment this lane reads at `base`
    auto read_wq = [&](u32x2 &dst, unsigned base, int n) {     // int8 weight fragment n (16 rows, 1 KB apart)
      switch (n) {
        case 0: lds_read8<0>(dst, base); break;
        case 1: lds_read8<1024>(dst, base); break;
        case 2: lds_read8<2048>(dst, base); break;
        case 3: lds_read8<3072>(dst, base); break;
        case 4: lds_read8<4096>(dst, base); break;
        case 5: lds_read8<5120>(dst, base); break;
        case 6: lds_read8<6144>(dst, base); break;
        default: lds_read8<7168>(dst, base); break;
      }
    };
    auto read_fa = [&](bf16x8 &dst, unsigned base, int n) {    // activation fragment: row blocks RSTEP apart
      switch (n) {
        case 0: lds_read16<0>(dst, base); break;
        case 1: lds_read16<2048 * RSTEP>(dst, base); break;
        case 2: lds_read16<4096 * RSTEP>(dst, base); break;
        default: lds_read16<6144 * RSTEP>(dst, base); break;
      }
    };
    auto read_frag = [&](bf16x8 &dst, unsigned base, int n) {
      switch (n) {
        case 0: lds_read16<0>(dst, base); break;
        case 1: lds_read16<2048>(dst, base); break;
        case 2: lds_read16<4096>(dst, base); break;
        case 3: lds_read16<6144>(dst, base); break;
        case 4: lds_read16<8192>(dst, base); break;
        case 5: lds_read16<10240>(dst, base); break;
        case 6: lds_read16<12288>(dst, base); break;
        default: lds_read16<14336>(dst, base); break;
      }
    };
    static_assert(IH <= 4 && CB <= 8, "fragment offsets above");
    const unsigned lds0 = (unsigned)(size_t)smem;
    // One half-step hs of the current tile: its MFMAs, with the operand reads of the half-step that follows
    // (half-step hsn of tile tn: its activation fragments, and the weight fragments too when it opens a
    // k-step) and the global loads q0 .. q1-1 of tile tl slotted in between them.  A wavefront issues in
    // order, so anything not placed between two MFMAs would add to the MFMA time.
    auto step = [&](int hs, bool next_reads, int tn, int hsn, int q0, int q1, int tl) {
      const int ab = hs & 1, bb = W8 ? 0 : (hs >> 1) & 1, h = hs & 1;
      const int nab = hsn & 1, nbb = W8 ? 0 : (hsn >> 1) & 1;
      const bool with_w = (hsn & 1) == 0;
      const unsigned base_a = lds0 + (tn % SA) * A_STAGE + a_off + (hsn & 1) * (IH * RSTEP * 2048) + rd[hsn >> 1];
      const unsigned base_w = lds0 + W_RING + (tn % SW) * W_STAGE + (W8 ? b_off8 + rd8[hsn >> 1] : b_off + rd[hsn >> 1]);
      const int nia = (hsn & 1) ? RB - IH : IH;        // row blocks of the next half-step
      const int n_reads = next_reads ? nia + (with_w ? CB : 0) : 0;
      // what rides along in MFMA slot j: the global loads q0 .. q1-1 of tile tl, spread evenly over the slots of
      // this half-step, and one operand read of the next half-step
      auto slot_work = [&](int j) {
#pragma unroll
        for (int q = q0 + j * (q1 - q0) / NSLOT; q < q0 + (j + 1) * (q1 - q0) / NSLOT; ++q) issue_one(tl, q);
        if (j < n_reads) {
          if (j < nia) read_fa(fa[nab][j], base_a, j);
          else if (W8) read_wq(fq[j - nia], base_w, j - nia);
          else read_frag(fb[nbb][j - nia], base_w, j - nia);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      if (W8 && h == 0) {
        // a k-step begins with int8 weights: its fragments are expanded one at a time, each while the MFMAs of
        // the fragment before it run, so this half-step walks the blocks column by column
#pragma unroll
        for (int jb = 0; jb < CB; ++jb) {
          fb[0][jb] = int8x8_to_bf16(fq[jb]);
#pragma unroll
          for (int ii = 0; ii < IH; ++ii) {
            if (block_ok(ii))
              acc[ii][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[0][jb], fa[ab][ii], acc[ii][jb], 0, 0, 0);
            slot_work(jb * IH + ii);
          }
        }
      } else {
#pragma unroll
      for (int ii = 0; ii < (h ? RB - IH : IH); ++ii) {
        // a 16-row block that lies wholly past the last row (only in the last row tile) is skipped: the
        // wavefront sharing the SIMD gets the matrix core instead.  One scalar branch per row block, not per
        // MFMA; the loads and reads of its slots follow outside the branch, so no register is written on two paths.
        if (block_ok(h * IH + ii)) {
#pragma unroll
          for (int jb = 0; jb < CB; ++jb)
            acc[h * IH + ii][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[bb][jb], fa[ab][ii], acc[h * IH + ii][jb], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jb = 0; jb < CB; ++jb) slot_work(ii * CB + jb);
      }
      }
#pragma unroll
      for (int j = h ? (RB - IH) * CB : NM; j < NSLOT; ++j) slot_work(j);
      if (next_reads) {
        lds_wait<0>();
#pragma unroll
        for (int i = 0; i < nia; ++i) lds_pin(fa[nab][i]);
        if (with_w) {
#pragma unroll
          for (int jb = 0; jb < CB; ++jb) {
            if (W8) asm volatile("" : "+v"(fq[jb]));
            else lds_pin(fb[nbb][jb]);
          }
        }
      }
    };

    // Issue order: W(0 .. SW-SA-1), then groups of one activation and one weight tile, [A(j), W(j+SW-SA)] for j = 0 ..
    // SA-1, up front; from then on the loads of a group are spread over four half-steps so that the memory pipeline never
    // sees a burst: after the barrier of tile t (its stages are free) the first half of A(t+SA); during the first three
    // half-steps of tile t+1 the second half of it, then W(t+SW) in two halves.  When tile t+1 is needed, the
    // groups of the SA-2 tiles after it may still be on their way, and of its own group the weight tile if that runs ahead.
    constexpr int QA = LA / 2, QW = LA + LW / 2, AHEAD = SA < SW ? LW : 0, YOUNGER = (SA - 2) * NL + AHEAD;
    static_assert(YOUNGER + NL < 64, "vmcnt has six bits");
#pragma unroll
    for (int s = 0; s < SW - SA; ++s) issue_w(s);
#pragma unroll
    for (int s = 0; s < SA; ++s) {
#pragma unroll
      for (int q = 0; q < NL; ++q) issue_one(s, q);
    }
    vm_wait<YOUNGER + NL>();
    wg_barrier();
#pragma unroll
    for (int q = 0; q < IH; ++q) read_fa(fa[0][q], lds0 + a_off + rd[0], q);
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      if (W8) read_wq(fq[q], lds0 + W_RING + b_off8 + rd8[0], q);
      else read_frag(fb[0][q], lds0 + W_RING + b_off + rd[0], q);
    }
    lds_wait<0>();
#pragma unroll
    for (int q = 0; q < IH; ++q) lds_pin(fa[0][q]);
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      if (W8) asm volatile("" : "+v"(fq[q]));
      else lds_pin(fb[0][q]);
    }
    if (nk > 1) {
      // tile 0: the tiles up to SA - 1 are already on their way
      step(0, true, 0, 1, 0, 0, 0);
      step(1, true, 0, 2, 0, 0, 0);
      step(2, true, 0, 3, 0, 0, 0);
      vm_wait<YOUNGER>();
      wg_barrier();
      step(3, true, 1, 0, 0, QA, SA);
    }
    for (int t = 1; t + 1 < nk; ++t) {
      step(0, true, t, 1, QA, LA, t + SA - 1);
      step(1, true, t, 2, LA, QW, t + SA - 1);
      step(2, true, t, 3, QW, NL, t + SA - 1);
      // last half-step: its fragments are in registers, so once tile t+1 has landed everywhere the
      // stages of tile t can be refilled while these MFMAs run
      vm_wait<YOUNGER>();
      wg_barrier();
      step(3, true, t + 1, 0, 0, QA, t + SA);
    }
    step(0, true, nk - 1, 1, 0, 0, 0);
    step(1, true, nk - 1, 2, 0, 0, 0);
    step(2, true, nk - 1, 3, 0, 0, 0);
    step(3, false, 0, 0, 0, 0, 0);
    vm_wait<0>();                                      // the clamped loads past the last tile
  }
  // Block (i, jb) of this wavefront, lane l: output row i*16 + l%16 and columns jb*16 + 4*(l/16) .. +3 of its sub-tile
  const int l_row = lane & 15, l_col = (lane >> 4) * 4;
  if (W8) {
    // the sums are over integer weights: scale every output column
    f32x4 scale[CB];
#pragma unroll
    for (int jb = 0; jb < CB; ++jb) {
      f32x4 sc = {0.f, 0.f, 0.f, 0.f};
      if (EPI == EPI_SWIGLU) {
        constexpr bool MIXED = swiglu_mixed_blocks(CB);
        const int gc = n0 + wn * CB * 8 + (MIXED ? jb * 8 + (l_col & 7) : jb % (CB / 2) * 16 + l_col);
        const float *ps = (MIXED ? lane < 32 : jb < CB / 2) ? p.w_scale[0] : p.w_scale[1];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (gc + r < p.N) sc[r] = ps[gc + r];
      } else {
        const int gc = n0 + wn * (BN / WN) + jb * 16 + l_col;
        int sg = 0;
        if (p.n_seg > 1 && gc >= p.nb[1]) sg = 1;
        if (p.n_seg > 2 && gc >= p.nb[2]) sg = 2;
        const float *ps = p.w_scale[sg] - p.nb[sg];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (gc + r < p.N) sc[r] = ps[gc + r];
      }
      scale[jb] = sc;
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
#pragma unroll
      for (int jb = 0; jb < CB; ++jb) acc[i][jb] *= scale[jb];
      __builtin_amdgcn_sched_barrier(0);               // in place, one row block at a time
    }
  }
  if (EPI == EPI_SWIGLU && tail_z >= 0) {
    // raw partial sums of a shared tile, in register order (each store is 1 KB contiguous)
    const int slot = (j - (p.tail_first >> 3)) * 8 + xcd;
    float *pb = p.partial + ((size_t)slot * p.tail_splits + tail_z) * (BM * BN) + (size_t)wave * (RB * CB * 4 * 64);
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int jb = 0; jb < CB; ++jb)
        *reinterpret_cast<f32x4 *>(pb + ((i * CB + jb) * 64 + lane) * 4) = acc[i][jb];
    return;
  }
  if (EPI == EPI_SWIGLU) {
    constexpr bool MIXED = swiglu_mixed_blocks(CB);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      __builtin_amdgcn_sched_barrier(0);               // one row block at a time, else the sums and results of several are live
      const int gr = m0 + (row_blk0 + i * RSTEP) * 16 + l_row;
      bf16 *orow = reinterpret_cast<bf16 *>(p.dst[0]) + (size_t)gr * p.ld[0];
#pragma unroll
      for (int jb = 0; jb < (MIXED ? CB : CB / 2); jb += MIXED ? 2 : 1) {
        const bool two = jb + 1 < CB;
        f32x4 g = acc[i][jb], u = acc[i][MIXED ? (two ? jb + 1 : jb) : jb + CB / 2];
        if (MIXED) pair_gate_up(g, u);
        if (gr < p.M && (!MIXED || two || lane < 32))
          store_swiglu(g, u, orow, n0 + wn * CB * 8 + swiglu_lane_col<CB>(jb, lane), p.N);
      }
    }
    return;
  }
  if (EPI != EPI_SEG) {
    // raw sums straight from the accumulator registers, four adjacent columns per lane
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int gr = m0 + (row_blk0 + i * RSTEP) * 16 + l_row;
      if (gr >= p.M) continue;
      float *prow = p.partial + ((size_t)z * p.M + gr) * p.N;
#pragma unroll
      for (int jb = 0; jb < CB; ++jb) {
        const int gc = n0 + wn * (BN / WN) + jb * 16 + l_col;
        if (gc + 3 < p.N) {
          *reinterpret_cast<f32x4 *>(prow + gc) = acc[i][jb];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (gc + r < p.N) prow[gc + r] = acc[i][jb][r];
        }
      }
    }
    return;
  }
  // EPI_SEG: drain the clamped tail loads, then reuse the rings as the parking area
  vm_wait<0>();
  __syncthreads();
  float *sC = reinterpret_cast<float *>(smem);
  if (HL && hl) {
    // the sums over the high parts are parked first, the sums over the low parts added to them
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      if (wm == part) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int jb = 0; jb < CB; ++jb) {
            f32x4 *dst = reinterpret_cast<f32x4 *>(sC + (i * 16 + l_row) * DMA_CP + wn * (BN / WN) + jb * 16 + l_col);
            if (part == 0) *dst = acc[i][jb];
            else *dst += acc[i][jb];
          }
      }
      __syncthreads();
    }
    lds_epilogue<bf16, EPI, BN>(sC, DMA_CP, BM / 2, m0, n0, z, p);
    return;
  }
  // park and walk the tile in passes of at most 128 rows (LDS holds 128 x 260 floats)
  constexpr int BLOCKS = BM / 16, PASSES = (BLOCKS + 7) / 8;
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    const int i0 = ps * 8;                                   // first 16-row block of the pass
    const int nb = (BLOCKS - i0) < 8 ? (BLOCKS - i0) : 8;
    if (ps > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int ib = row_blk0 + i * RSTEP;                   // this wavefront's 16-row block within the tile
      if (ib >= i0 && ib < i0 + 8) {
#pragma unroll
        for (int jb = 0; jb < CB; ++jb)
          *reinterpret_cast<f32x4 *>(sC + ((ib - i0) * 16 + l_row) * DMA_CP + wn * (BN / WN) + jb * 16 + l_col) = acc[i][jb];
      }
    }
    __syncthreads();
    lds_epilogue<bf16, EPI, BN>(sC, DMA_CP, nb * 16, m0 + i0 * 16, n0, z, p);
  }
}

// ---------------------------------------------------------------------------
// Register-staged bf16 kernel (any K % 8 == 0).  4 wavefronts as 2x2, each owning a
// 64x64 block = 2x2 MFMA tiles.  LDS rows are padded by 16 bytes so that the 16-byte
// operand reads of 8 consecutive lanes fall into 8 different bank groups.
// Operand layout of v_mfma_f32_32x32x16_bf16: lane l supplies row (l % 32) and the
// 8 consecutive k values starting at 8 * (l / 32); the result lane l holds column
// (l % 32), rows 8*(i/4) + 4*(l/32) + i%4 for i = 0..15.
// ---------------------------------------------------------------------------
constexpr int BM16 = 128, BN16 = 128, BK16 = 64, PITCH16 = BK16 + 8;
constexpr int CPITCH16 = BN16 + 4;
constexpr size_t kSmemBf16 =
    (2 * (BM16 + BN16) * PITCH16 * 2 > BM16 * CPITCH16 * 4) ? 2 * (BM16 + BN16) * PITCH16 * 2
                                                             : BM16 * CPITCH16 * 4;

template <int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  bf16 *sA = reinterpret_cast<bf16 *>(smem);               // [2][BM][PITCH]
  bf16 *sB = sA + 2 * BM16 * PITCH16;                      // [2][BN][PITCH]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int OUT_COLS = (EPI == EPI_SWIGLU) ? BN16 / 2 : BN16;
  const int m0 = blockIdx.y * BM16, n0 = blockIdx.x * OUT_COLS;
  const int kb = blockIdx.z * p.k_per_split;
  const int ke = min(p.K, kb + p.k_per_split);
  const int nk = (ke - kb + BK16 - 1) / BK16;

  // each thread moves 4 A chunks and 4 B chunks (16 bytes each) per k-tile
  const bf16 *a_ptr[4], *b_ptr[4];
  int lds_off[4], kcol[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int id = tid + i * 256, row = id >> 3, kc = id & 7;
    int ar = min(m0 + row, p.M - 1);
    if (p.a_rows) ar = p.a_rows[ar];
    a_ptr[i] = reinterpret_cast<const bf16 *>(p.a) + (size_t)ar * p.lda + kc * 8;
    b_ptr[i] = weight_row<bf16, EPI>(p, n0 + row, BN16 / 2, n0, row) + kc * 8;
    lds_off[i] = row * PITCH16 + kc * 8;
    kcol[i] = kc * 8;
  }
  bf16x8 ra[4], rb[4];
  const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  // tile t of the k loop; with a (high, low) activation pair the K range is walked twice, the
  // second time over the low parts
  const int nt_all = p.a_lo_off > 0 ? 2 * nk : nk;
  auto gload = [&](int t) {
    const int lo = t >= nk;
    const int k0 = kb + (t - lo * nk) * BK16;
    const int a_adv = k0 + lo * p.a_lo_off;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool ok = k0 + kcol[i] < ke;
      ra[i] = ok ? *reinterpret_cast<const bf16x8 *>(a_ptr[i] + a_adv) : zero;
      rb[i] = ok ? *reinterpret_cast<const bf16x8 *>(b_ptr[i] + k0) : zero;
    }
  };
  auto sstore = [&](int stage) {
    bf16 *da = sA + stage * BM16 * PITCH16, *db = sB + stage * BN16 * PITCH16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<bf16x8 *>(da + lds_off[i]) = ra[i];
      *reinterpret_cast<bf16x8 *>(db + lds_off[i]) = rb[i];
    }
  };

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  if (nk > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  const int frag_off = (lane & 31) * PITCH16 + 8 * (lane >> 5);
  for (int t = 0; t < nt_all; ++t) {
    if (t + 1 < nt_all) gload(t + 1);
    const bf16 *ca = sA + (t & 1) * BM16 * PITCH16 + (wm * 64) * PITCH16 + frag_off;
    const bf16 *cb_ = sB + (t & 1) * BN16 * PITCH16 + (wn * 64) * PITCH16 + frag_off;
#pragma unroll
    for (int ks = 0; ks < BK16 / 16; ++ks) {
      bf16x8 a0 = *reinterpret_cast<const bf16x8 *>(ca + ks * 16);
      bf16x8 a1 = *reinterpret_cast<const bf16x8 *>(ca + 32 * PITCH16 + ks * 16);
      bf16x8 b0 = *reinterpret_cast<const bf16x8 *>(cb_ + ks * 16);
      bf16x8 b1 = *reinterpret_cast<const bf16x8 *>(cb_ + 32 * PITCH16 + ks * 16);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, acc[1][1], 0, 0, 0);
    }
    if (t + 1 < nt_all) sstore((t + 1) & 1);
    __syncthreads();
  }
  // park the accumulators in LDS (the operand stages are dead after the last barrier)
  float *sC = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wm * 64 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        const int col = wn * 64 + j * 32 + (lane & 31);
        sC[row * CPITCH16 + col] = acc[i][j][r];
      }
  __syncthreads();
  lds_epilogue<bf16, EPI, BN16>(sC, CPITCH16, BM16, m0, n0, blockIdx.z, p);
}

// ---------------------------------------------------------------------------
// float kernel, v_mfma_f32_32x32x2_f32 (float products and sums).  4 wavefronts as WM x WN x WK: each owns a 32 x 32
// block of the 32 WM x 32 WN tile, and with WK = 4 the four share one block along K -- a float model is small, its
// projections have too few 64 x 64 tiles to occupy the chip, and a WK = 4 tile brings four times as many workgroups
// without parked sums or another launch.  64-deep stages, double-buffered in LDS, the next one on its way in
// registers meanwhile.
// A k-step of 8 gives lane l the four values k0 + 4 (l / 32) .. + 3 of row (l % 32): one 16-byte LDS read feeds
// four MFMAs (the two half-waves supply different k, which a sum may take in any order).  Rows are 256 bytes, the
// 16-byte chunk c of row r sits in slot c ^ (r & 15).
// Bound by latency at these sizes: 544 x 256 x 256 .. 688 took 34 us on 64 x 64 tiles of vector FMAs, 8 us here.
// ---------------------------------------------------------------------------
constexpr int BK32 = 64;
constexpr int f32_smem_bytes(int wm, int wn, int wk) {
  const int ring = 2 * 32 * (wm + wn) * BK32 * 4, park = wk * 32 * wm * (32 * wn + 4) * 4;
  return ring > park ? ring : park;
}

template <int EPI, int WM, int WN, int WK>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  static_assert(WM * WN * WK == 4, "four wavefronts");
  constexpr int BM = 32 * WM, BN = 32 * WN, CP = BN + 4;
  constexpr int OUT_COLS = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int LA = BM * BK32 / 1024, LB = BN * BK32 / 1024;      // 16-byte loads per lane per stage
  __shared__ __attribute__((aligned(16))) char smem[f32_smem_bytes(WM, WN, WK)];
  float4 *sA = reinterpret_cast<float4 *>(smem);                   // [2][BM][16]
  float4 *sB = sA + 2 * BM * 16;                                   // [2][BN][16]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / (WK * WN);
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * OUT_COLS;
  const int kb = blockIdx.z * p.k_per_split;
  const int ke = min(p.K, kb + p.k_per_split);
  const int nk = (ke - kb + BK32 - 1) / BK32;

  const int lr = tid >> 4, lc = tid & 15;                          // row (+ 16 i) and 16-byte chunk of this lane's loads
  const float *a_ptr[LA], *b_ptr[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    int ar = min(m0 + lr + 16 * i, p.M - 1);
    if (p.a_rows) ar = p.a_rows[ar];
    a_ptr[i] = reinterpret_cast<const float *>(p.a) + (size_t)ar * p.lda + lc * 4;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) b_ptr[i] = weight_row<float, EPI>(p, n0 + lr + 16 * i, BN / 2, n0, lr + 16 * i) + lc * 4;
  float4 ra[LA], rb[LB];
  auto gload = [&](int t) {
    const int k0 = kb + t * BK32;
    const bool ok = k0 + lc * 4 < ke;
#pragma unroll
    for (int i = 0; i < LA; ++i) ra[i] = ok ? *reinterpret_cast<const float4 *>(a_ptr[i] + k0) : make_float4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < LB; ++i) rb[i] = ok ? *reinterpret_cast<const float4 *>(b_ptr[i] + k0) : make_float4(0, 0, 0, 0);
  };
  auto sstore = [&](int stage) {                                   // rows lr + 16 i: r & 15 = lr
#pragma unroll
    for (int i = 0; i < LA; ++i) sA[(stage * BM + lr + 16 * i) * 16 + (lc ^ lr)] = ra[i];
#pragma unroll
    for (int i = 0; i < LB; ++i) sB[(stage * BN + lr + 16 * i) * 16 + (lc ^ lr)] = rb[i];
  };
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  if (nk > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  const int row = lane & 31, h = lane >> 5, sw = row & 15;
  constexpr int KS = BK32 / 8 / WK;                                // k-steps of 8 per stage and wavefront
  for (int t = 0; t < nk; ++t) {
    if (t + 1 < nk) gload(t + 1);
    const float4 *ca = sA + ((t & 1) * BM + wm * 32 + row) * 16, *cb_ = sB + ((t & 1) * BN + wn * 32 + row) * 16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int chunk = (2 * (wk * KS + ks) + h) ^ sw;
      const float4 av = ca[chunk], bv = cb_[chunk];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, bv.w, acc, 0, 0, 0);
    }
    if (t + 1 < nk) sstore((t + 1) & 1);
    __syncthreads();
  }
  // park the blocks; lane l holds column (l % 32), rows 8 (i / 4) + 4 (l / 32) + i % 4
  float *sC = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int i = 0; i < 16; ++i)
    sC[(wk * BM + wm * 32 + (i >> 2) * 8 + h * 4 + (i & 3)) * CP + wn * 32 + row] = acc[i];
  __syncthreads();
  if (WK > 1) {                                                    // the K shares, added in ascending order
    for (int e = tid; e < BM * BN / 4; e += 256) {
      float4 *c0 = reinterpret_cast<float4 *>(sC + (e / (BN / 4)) * CP + e % (BN / 4) * 4);
      float4 v = *c0;
#pragma unroll
      for (int z = 1; z < WK; ++z) {
        const float4 u = c0[z * BM * CP / 4];
        v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
      }
      *c0 = v;
    }
    __syncthreads();
  }
  lds_epilogue<float, EPI, BN>(sC, CP, BM, m0, n0, blockIdx.z, p);
}

// The same for launches with few 32 x 32 tiles (f32_tile): 16 x 16 tiles (v_mfma_f32_16x16x4_f32), the four wavefronts
// share K in turn, 16 deep, and read their operands straight from the cache into registers, all of up to 12 steps at once -- no
// stages, no barrier before the shares are added.  A lane's 16 bytes are four k of one row; MFMA e takes element e of both operands, so
// a wavefront's k-step is walked in an order of its own.  The weight is the first operand: lane l holds row (l % 16), columns
// 4 (l / 16) .. + 3.
constexpr int F32_STEPS = 12;
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(GemmParams p) {
  constexpr int CP = 20;
  __shared__ __attribute__((aligned(16))) float sC[4 * 16 * CP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 15, h = lane >> 4;
  const int m0 = blockIdx.y * 16, n0 = blockIdx.x * (EPI == EPI_SWIGLU ? 8 : 16);
  const int kb = blockIdx.z * p.k_per_split, ke = min(p.K, kb + p.k_per_split);
  int ar = min(m0 + ln, p.M - 1);
  if (p.a_rows) ar = p.a_rows[ar];
  const float *a = reinterpret_cast<const float *>(p.a) + (size_t)ar * p.lda;
  const float *w = weight_row<float, EPI>(p, n0 + ln, 8, n0, ln);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = kb + wave * 16 + 4 * h; k0 - 4 * h < ke; k0 += 64 * F32_STEPS) {      // uniform over the wavefront
    float4 av[F32_STEPS], wv[F32_STEPS];
#pragma unroll
    for (int i = 0; i < F32_STEPS; ++i) {
      const bool ok = k0 + 64 * i < ke;
      av[i] = ok ? *reinterpret_cast<const float4 *>(a + k0 + 64 * i) : make_float4(0, 0, 0, 0);
      wv[i] = ok ? *reinterpret_cast<const float4 *>(w + k0 + 64 * i) : make_float4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < F32_STEPS; ++i) {
      if (k0 - 4 * h + 64 * i >= ke) break;                                           // uniform over the wavefront
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i].x, av[i].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i].y, av[i].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i].z, av[i].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i].w, av[i].w, acc, 0, 0, 0);
    }
  }
  *reinterpret_cast<f32x4 *>(sC + (wave * 16 + ln) * CP + 4 * h) = acc;
  __syncthreads();
  if (tid < 64) {                                                  // the K shares, added in ascending order
    f32x4 *c0 = reinterpret_cast<f32x4 *>(sC + ln * CP + 4 * h);
    f32x4 v = *c0;
#pragma unroll
    for (int z = 1; z < 4; ++z) v += c0[z * 16 * CP / 4];
    *c0 = v;
  }
  __syncthreads();
  lds_epilogue<float, EPI, 16>(sC, CP, 16, m0, n0, blockIdx.z, p);
}

// ---------------------------------------------------------------------------
// Finish launches: one workgroup per output row adds the parked partial sums in ascending split
// order (fixed order, no atomics: bitwise reproducible) and completes the row.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float4 sum_splits(const GemmParams &p, size_t e) {
  float4 acc = make_float4(0, 0, 0, 0);
  const size_t stride = (size_t)p.M * p.N;
  for (int z = 0; z < p.splits; ++z) {
    const float4 v = *reinterpret_cast<const float4 *>(p.partial + z * stride + e);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  return acc;
}

// EPI_SEG rows: rotary embedding, conversion to the storage type, store (optionally through the
// segment's row map) and -- for rows < n_dev -- the KV deviation of the row (Sec. 4.1, Sec. 6):
// the squared distance of the values as stored from the cached row, over the segments that name a cache.
// Workgroup (r, 0) takes columns [0, first) of row r, all columns with a deviation among them; workgroup (r, y) the
// y-th run of kFinishCols columns after those.  A row alone is too little work in flight: a lane keeps two column groups
// in work and requests four splits of both before the first addition.  Bound by the parked sums it reads; on the 7B
// shape (30 .. 500 rows, K|V and Q) 9.4 us per launch where a loop of one load after the other took 13.5 us for K|V
// and 13.5 us for Q.
constexpr int kFinishCols = 2048;
template <typename T>
__global__ __launch_bounds__(256) void seg_finish_kernel(GemmParams p, int first) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  const int cb = blockIdx.y == 0 ? 0 : first + ((int)blockIdx.y - 1) * kFinishCols;
  const int ce = blockIdx.y == 0 ? first : min(p.N, cb + kFinishCols);
  const bool want_dev = p.dev_out != nullptr && blockIdx.y == 0 && r < p.n_dev;
  const int crow = want_dev ? p.dev_row[r] : 0;
  const size_t stride = (size_t)p.M * p.N;
  float dsum = 0.f;
  for (int c = cb + threadIdx.x * 4; c < ce; c += 2048) {
    const bool two = c + 1024 < ce;
    const float *src = p.partial + (size_t)r * p.N + c;
    const int off1 = two ? 1024 : 0;
    float4 a0 = make_float4(0, 0, 0, 0), a1 = a0;
    auto add = [](float4 &a, const float4 &v) { a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w; };
    int z = 0;
    for (; z + 4 <= p.splits; z += 4, src += 4 * stride) {
      float4 v0[4], v1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v0[i] = *reinterpret_cast<const float4 *>(src + i * stride);
        v1[i] = *reinterpret_cast<const float4 *>(src + i * stride + off1);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) { add(a0, v0[i]); add(a1, v1[i]); }
    }
    for (; z < p.splits; ++z, src += stride) {
      const float4 v0 = *reinterpret_cast<const float4 *>(src), v1 = *reinterpret_cast<const float4 *>(src + off1);
      add(a0, v0);
      add(a1, v1);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float4 acc = i ? a1 : a0;
      float4 partner = acc;
      if (p.rope_half) {
        // a head's other half is head_dim / 8 lanes away (heads are whole and 1024 columns hold whole heads)
        const int o = p.head_dim / 8;
        partner = make_float4(__shfl_xor(acc.x, o, 64), __shfl_xor(acc.y, o, 64), __shfl_xor(acc.z, o, 64), __shfl_xor(acc.w, o, 64));
      }
      if (i == 1 && !two) continue;
      int s, lc;
      const float4 v = seg_rotate(acc, partner, r, c + i * 1024, p, &s, &lc);
      const int dr = p.row_map[s] ? p.row_map[s][r] : r;
      store4<T>(reinterpret_cast<T *>(p.dst[s]) + (size_t)dr * p.ld[s] + lc, v.x, v.y, v.z, v.w);
      if (want_dev && p.dev_cache[s]) {
        const float4 old = load4<T>(reinterpret_cast<const T *>(p.dev_cache[s]) +
                                    (size_t)crow * (p.nb[s + 1] - p.nb[s]) + lc);
        const float d0 = as_stored<T>(v.x) - old.x, d1 = as_stored<T>(v.y) - old.y;
        const float d2 = as_stored<T>(v.z) - old.z, d3 = as_stored<T>(v.w) - old.w;
        dsum += d0 * d0 + d1 * d1 + d2 * d2 + d3 * d3;
      }
    }
  }
  if (p.dev_out != nullptr && blockIdx.y == 0) {     // uniform over the workgroup
    dsum = block_sum_256(dsum, red);
    if (want_dev && threadIdx.x == 0) p.dev_out[r] = dsum;
  }
}

// EPI_F32 rows: h = sum of the partial sums + residual, stored as float; then, when a gain is
// given, the RMSNorm of h in the storage type (the next projection's input), optionally as a
// (high, low) pair.  A lane re-reads only elements it wrote itself.
template <typename T>
__global__ __launch_bounds__(256) void resid_norm_finish_kernel(GemmParams p) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  const int rr = p.resid_rows ? p.resid_rows[r] : r;
  float *orow = p.out_f32 + (size_t)r * p.N;
  float ss = 0.f;
  for (int c = threadIdx.x * 4; c < p.N; c += 1024) {
    float4 v = sum_splits(p, (size_t)r * p.N + c);
    if (p.resid) {
      const float4 q = *reinterpret_cast<const float4 *>(p.resid + (size_t)rr * p.N + c);
      v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
    }
    *reinterpret_cast<float4 *>(orow + c) = v;
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  if (p.norm_gain == nullptr) return;      // uniform
  ss = block_sum_256(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)p.N + p.norm_eps);
  const T *gain = reinterpret_cast<const T *>(p.norm_gain);
  T *nrow = reinterpret_cast<T *>(p.norm_out) + (size_t)r * p.norm_ld;
  for (int c = threadIdx.x * 4; c < p.N; c += 1024) {
    const float4 v = *reinterpret_cast<const float4 *>(orow + c);
    const float x[4] = {v.x * inv * to_f32(gain[c]), v.y * inv * to_f32(gain[c + 1]),
                        v.z * inv * to_f32(gain[c + 2]), v.w * inv * to_f32(gain[c + 3])};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T hi = from_f32<T>(x[i]);
      nrow[c + i] = hi;
      if (p.norm_lo_off > 0) nrow[p.norm_lo_off + c + i] = from_f32<T>(x[i] - to_f32(hi));
    }
  }
}

// The same for rows of at most 1024 NC elements, with the row held in registers: a workgroup per row
// is little work in flight, so the loop above runs at the latency of one load after the other (its
// store may alias the next iteration's loads, which therefore wait for it).  Here every load of a
// split is issued before the first sum, two splits at a time, and the second pass reads no memory.
// Same order of additions per element as above.
template <typename T, int NC>
__global__ __launch_bounds__(256) void resid_norm_finish_row_kernel(GemmParams p) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  const int rr = p.resid_rows ? p.resid_rows[r] : r;
  const size_t row = (size_t)r * p.N, stride = (size_t)p.M * p.N;
  const int c0 = threadIdx.x * 4;
  float4 q[NC], acc[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = c0 + i * 1024;
    acc[i] = make_float4(0, 0, 0, 0);
    q[i] = make_float4(0, 0, 0, 0);
    if (p.resid && c < p.N) q[i] = *reinterpret_cast<const float4 *>(p.resid + (size_t)rr * p.N + c);
  }
#pragma unroll 2
  for (int z = 0; z < p.splits; ++z) {
    float4 v[NC];
    const float *src = p.partial + z * stride + row;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = c0 + i * 1024;
      v[i] = c < p.N ? *reinterpret_cast<const float4 *>(src + c) : make_float4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      acc[i].x += v[i].x; acc[i].y += v[i].y; acc[i].z += v[i].z; acc[i].w += v[i].w;
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = c0 + i * 1024;
    if (p.resid) { acc[i].x += q[i].x; acc[i].y += q[i].y; acc[i].z += q[i].z; acc[i].w += q[i].w; }
    if (c < p.N) *reinterpret_cast<float4 *>(p.out_f32 + row + c) = acc[i];
    // the expression of the stand-alone norm kernel: a layer normalised there and one normalised here agree bitwise
    ss += acc[i].x * acc[i].x + acc[i].y * acc[i].y + acc[i].z * acc[i].z + acc[i].w * acc[i].w;
  }
  if (p.norm_gain == nullptr) return;      // uniform
  ss = block_sum_256(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)p.N + p.norm_eps);
  const T *gain = reinterpret_cast<const T *>(p.norm_gain);
  T *nrow = reinterpret_cast<T *>(p.norm_out) + (size_t)r * p.norm_ld;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = c0 + i * 1024;
    if (c >= p.N) continue;
    const float4 gn = load4<T>(gain + c);
    const float x[4] = {acc[i].x * inv * gn.x, acc[i].y * inv * gn.y, acc[i].z * inv * gn.z, acc[i].w * inv * gn.w};
    float hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) hi[e] = to_f32(from_f32<T>(x[e]));
    store4<T>(nrow + c, x[0], x[1], x[2], x[3]);
    if (p.norm_lo_off > 0)
      store4<T>(nrow + p.norm_lo_off + c, x[0] - hi[0], x[1] - hi[1], x[2] - hi[2], x[3] - hi[3]);
  }
}

// ---------------------------------------------------------------------------
// Host side: choice of kernel, tile height and K split; launches.
// ---------------------------------------------------------------------------
// Tiles of the direct-to-LDS kernel: WM x WN wavefronts of RB x CB blocks of 16 x 16.
struct DmaTile {
  int RB, CB, WM, WN;
  constexpr int bm() const { return 16 * RB * WM; }
  constexpr int bn() const { return 16 * CB * WN; }
};
static constexpr DmaTile kDmaTiles[] = {
    {2, 4, 2, 2}, {4, 4, 2, 2}, {6, 4, 2, 2},                                    // 64, 128, 192 x 128: a wavefront per SIMD
    {4, 4, 2, 4}, {6, 4, 2, 4}, {8, 4, 2, 4},                                    // 128, 192, 256 x 256, two per SIMD
    {2, 5, 4, 2}, {2, 7, 4, 2},                                                  // 128 x 160, 224
    {3, 4, 4, 2}, {3, 5, 4, 2}, {3, 7, 4, 2},                                    // 192 x 128, 160, 224
    {4, 4, 4, 2}, {4, 5, 4, 2}, {4, 7, 4, 2},                                    // 256 x 128, 160, 224
    {5, 5, 4, 2}, {5, 6, 4, 2}, {6, 4, 4, 2}, {6, 5, 4, 2}};                     // 320 x 160, 192; 384 x 128, 160
// (_4x2: eight wavefronts, where the same size has four)
constexpr int kNumDmaTiles = sizeof(kDmaTiles) / sizeof(kDmaTiles[0]);
enum { T64x128, T128x128, T192x128, T128x256, T192x256, T256x256, T128x160, T128x224, T192x128_4x2, T192x160, T192x224,
       T256x128_4x2, T256x160, T256x224, T320x160, T320x192, T384x128, T384x160 };

// row blocks that a wavefront walks, summed over the row tiles: all of them but in the last tile
static long row_block_steps(const DmaTile &t, int M) {
  const int last = ceil_div(M, t.bm()) - 1;
  return (long)last * t.RB + ceil_div(ceil_div(M - last * t.bm(), 16), t.WM);
}

struct GemmPlan {
  int kind;        // 0 float, 1 register-staged bf16, 2 direct-to-LDS bf16
  int tile;        // kind 2: index into kDmaTiles
  int hl;          // output columns that take (high, low) activation pairs (bf16 EPI_SEG only)
  int bm, out_cols, bk;   // bm: output rows per tile (of the columns without pairs, kind 2)
  int hl_tiles_m, hl_tiles_n;             // kind 2: tiles of the columns with pairs; tiles_m, tiles_n: of the others
  int tiles_m, tiles_n, splits, k_per_split;
  double cost;     // estimated us of the main and the finish launch (kind 2, not EPI_SWIGLU)
  int tail_first, tail_splits, tail_k_per_split;   // EPI_SWIGLU tail sharing (tail_splits <= 1: none)
  long grid_ids;                                   // kind 2: workgroups of the main launch
  int xcd_split;                                   // kind 2: splits dealt to XCDs (see GemmParams)
  int w8;                                          // kind 2: int8 weights read by the kernel itself
  int mode;                                        // kind 2: MODE_PLAIN, MODE_STAGGER or MODE_NT (non-temporal weight loads)
  int k_stagger;                                   // kind 2: column tiles start at different k-tiles
  int raw;                                         // sums are parked in `partial` and a finish launch completes them
  size_t partial_floats;
  bool bad;                                        // needs scratch the caller did not give
};

// Weight loads are non-temporal for bf16 matrices this large that a single row tile reads: every weight is then read by one
// workgroup alone.  57344 x 8192 at 16 .. 128 rows 187 -> 165 us, 8192 x 28672 at 64 rows 100 -> 84 us, 28672 x 4096 54 -> 50 us;
// matrices of 30 .. 50 MB lost up to 10 %, several row tiles (they share weight tiles in L2) up to 20 %, int8 weights up to 20 %.
constexpr double kNtMinBytes = 128e6;

// Rows of weights whose pitch is a power of two of at least 8 KB all start at the same place of the memory channels' interleave, and
// workgroups that walk K in step ask few channels at a time.  With a single row tile (nothing then ties the column tiles
// together but the small activation slices) neighbouring column tiles of an XCD start two k-tiles apart, those of neighbouring
// XCDs one, and wrap around.  28672 x 4096 at 32 / 64 / 120 rows 47.8 -> 38.6, 48.4 -> 40.2, 52.3 -> 47.0 us; 57344 x 8192 at
// 32 rows 163 -> 153 us; 8192 x 8192 at 120 / 250 rows 46.1 -> 41.4, 59.4 -> 52.9 us.  Other pitches (7168, 14336, 20480,
// 28672 elements) gain nothing and lose up to 5 % where the activations outgrow an L2; neither do int8 rows gain.
static bool pitch_is_power_of_two(int K) { return K >= 4096 && (K & (K - 1)) == 0; }

// XCDs that share one K split (GemmParams::xcd_split): 8 / splits where the splits are dealt to them, else all 8.  One row tile
// has no activation slices worth keeping apart, and where its column tiles fill the 8 XCDs evenly anyhow the splits stay
// together: 8192 x 8192 at 64 / 128 rows in 4 splits 49 / 52 us dealt, 43 / 47 us not.
static int xcd_groups(int splits, int tiles_m, int tiles_n, int hl) {
  if (tiles_m == 1 && tiles_n % 8 == 0 && !hl) return 8;
  return splits == 2 || splits == 4 || splits == 8 ? 8 / splits : 8;
}

// Tile shape and K split of the direct-to-LDS kernel for the Q/K/V, output and down projections,
// from a cost model in microseconds fitted to sweeps of every (tile, split) pair over these
// projections of the 7B-, 34B- and 70B-shaped workloads (bf16 24 .. 1536 rows, int8 16 .. 760; over 10000 pairs) on the chip:
//   main launch   = rounds x t x k-tiles per workgroup + a fixed part (launch, pipeline fill, epilogue; bf16: 3.3 us more for every
//                   further round)
//                   at least the weights' bytes at the rate a launch reads them (few rows: no point in splitting further than
//                   that; the operand pairs of K|V are bound by the matrix cores earlier and go by the tiles alone)
//   rounds        = those of the XCD that is dealt the most workgroups, 32 at a time (one per CU; a partly filled
//                   round counts whole).  28 column tiles in 9 splits are 252 workgroups, but 36 on four of the XCDs: two
//                   rounds.  Counted over the chip instead, the model chose such splits: 7168 x 20480 at 96 / 525 rows
//                   104 / 268 us, 72 / 192 us with the pairs it chooses now.
//   t             = time of one 64-deep k-tile on every CU with no row padded; a row tile's blocks without real rows take 0.18 of
//                   it off (bf16; the int8 expansions stay).  Split shares of a multiple of 4 KB (32 k-tiles) start
//                   at the same place of the memory channels' interleave: 1.12 t (4096 x 14336 at 110 rows in 7 splits of
//                   32 k-tiles 42.5 us, in 8 of 28 36.0 us); rows of a power-of-two pitch are staggered instead.
//   finish launch = finish + park per MB of parked sums (splits x M x N floats), stores included, and 0.2 us per split where it
//                   runs anyway (it reads a few of a row's splits at a time; where it does not, an unsplit launch's own epilogue
//                   costs about as much).  Without that, small launches took twice the splits they gain by: 1024 x 2816 at 720
//                   rows 17.2 -> 18.8 us.
//                   Sums beyond 96 MB, next to the operands too much for the memory-side cache, 0.2 us per MB more: the choice is as good
//                   as without that (1000 .. 6144 rows, mean 0.1 % apart) and parks a quarter less, which is what workspaces are sized for.
// Of the pairs of a sweep over 1 .. 6144 rows (profiles/projection_tiles.tsv has a part of it) its bf16 choice is on average within 1.8 %
// (output and down; the six tiles that all three projections share come within 2.4 %) and 1.2 % (Q/K/V) of the best on the three models it was
// fitted to, and within 1.4 % and 1.2 % on eight others of 512 .. 5120 columns; int8 within 1.0 %.  (7168 x 20480 at 580
// rows 209 -> 183 us with 320 x 192; 192 x 224 tiles, tried for the same launches, take the rounds of 192 x 256 ones and 4 .. 6 % longer: 7168 x 7168
// at 285 rows 54 -> 56 us, 5120 x 5120 at 1600 rows 110 -> 117 us.)
// K and V alone, all of whose columns take operand pairs, keep constants of their own (kPairs): with those of the other bf16
// projections it chose too many splits of too wide tiles (2048 x 4096 at 64 rows in 8 splits of 64 x 128 15.7 us, in 16 of
// 128 x 128 18.6; 2600 rows of 2048 x 7168 132 -> 142 us), over 836 sizes of 11 models 0.3 % more on average, 54 of them by more than 3 %.
// t = 0: not used.
// max_splits caps the split (scratch the caller can spare); parked: a finish launch runs anyway.
constexpr int kProjectionTiles[] = {T64x128, T128x128, T192x128, T128x256, T192x256, T256x256, T256x128_4x2, T320x192};
constexpr int kSharedShapes = 6;                           // the leading ones serve the Q/K/V projections too
constexpr int kFloatOutputShapes = sizeof(kProjectionTiles) / sizeof(kProjectionTiles[0]);
struct ProjectionModel {
  double t[kFloatOutputShapes];
  double padded;         // share of t that a row tile's blocks without real rows take off
  double fixed, round;   // us; per further round
  double finish, park, split;   // us; us per MB; us per split (of launches with a finish launch anyway)
  double far;            // us per MB beyond 96 MB of a split launch
  double read;           // MB per us
  double aligned;        // factor of t where the split shares are a multiple of 4 KB apart
};
static constexpr ProjectionModel kBf16 = {{0.52, 0.61, 0.73, 0.88, 1.21, 1.38, 0.83, 1.40}, 0.18, 9.6, 3.3, 1.5, 0.342, 0.2, 0.2, 5.95, 1.12};
static constexpr ProjectionModel kPairs = {{0.58, 0.72, 0.82, 0.97, 1.28, 1.50}, 0, 9.5, 0, 2.3, 0.5, 0, 0, 5.2, 1};
static constexpr ProjectionModel kInt8 = {{0.72, 0.94, 0, 1.32, 1.53, 1.89}, 0, 9.5, 0, 2.3, 0.5, 0, 0, 5.2, 1};
constexpr int projection_shapes(int epi) { return epi == EPI_SEG ? kSharedShapes : kFloatOutputShapes; }

// Output columns [0, hl_cols) take (high, low) activation pairs, i.e. twice the tile rows per output row.
static void pick_dma_plan(const ProjectionModel &m, int epi, int M, int N, int hl_cols, int K, int max_splits, bool parked, bool w8,
                          GemmPlan *pl) {
  const int k_tiles = K / DMA_BK;
  const double mn_mb = (double)M * N * 4.0e-6, park_us = mn_mb * m.park + (parked ? m.split : 0.0);  // per split
  const double read_us = hl_cols ? 0.0 : (double)N * K * (w8 ? 1 : 2) / (m.read * 1e6);
  pl->cost = 1e30;
  for (int i = 0; i < projection_shapes(epi); ++i) {
    const DmaTile t = kDmaTiles[kProjectionTiles[i]];
    const int bm = t.bm(), bn = t.bn();
    if (m.t[i] == 0.0 || (bm == 64 && M > 64)) continue;
    if (hl_cols < N && hl_cols % bn != 0) continue;        // a tile's columns are of one kind
    const int tiles_m = ceil_div(M, bm), tiles_n = ceil_div(N - hl_cols, bn), hl_n = ceil_div(hl_cols, bn);
    const long hl_m = ceil_div(2 * M, bm);
    const double t_rows = m.t[i] * (1.0 - m.padded + m.padded * row_block_steps(t, M) / ((double)tiles_m * t.RB));
    for (int sp = 1; sp <= 16 && sp <= max_splits; ++sp) {
      if (sp > 1 && k_tiles / sp < 4) break;
      const int kt = ceil_div(k_tiles, sp);
      const double outside = m.fixed + (sp > 1 || parked ? sp * park_us + m.finish : 0.0) + (sp > 1 ? m.far * std::max(0.0, sp * mn_mb - 96.0) : 0.0);
      if (outside >= pl->cost && sp > 1) break;            // grows with the splits
      if (outside + std::max(t_rows * kt, read_us) >= pl->cost) continue;      // one round
      const int groups = xcd_groups(sp, tiles_m, tiles_n, hl_cols);
      const long per_xcd = (hl_m * ceil_div(hl_n, groups) + (long)tiles_m * ceil_div(tiles_n, groups)) * (groups < 8 ? 1 : sp);
      const long rounds = (per_xcd + 31) / 32;
      const double tk = sp > 1 && groups == 8 && kt % 32 == 0 && !pitch_is_power_of_two(K) ? m.aligned * t_rows : t_rows;
      const double cost = std::max(rounds * tk * kt, read_us) + m.round * (rounds - 1) + outside;
      if (cost < pl->cost - 1e-9) { pl->cost = cost; pl->tile = kProjectionTiles[i]; pl->splits = sp; }
    }
  }
}

// Tile of the gate/up projection, and how its last round of workgroups is shared: a cost model in microseconds fitted to sweeps of
// every tile at 1 .. 6144 rows, bf16 and int8 weights, of the 7B, 34B and 70B models and eight others of 512 .. 5120 columns
// (profiles/projection_tiles.tsv has a part of them): its choice is on average within 0.9 % (bf16) and 1.0 % (int8) of the best.
//   a round   = (idle + rows x share of the tile's row blocks that hold real rows) x k-tiles; a launch of less than one round runs
//               faster than its share of the chip (power): down to 1 - partial of that
//               at least the weights it reads, at 6.2 TB/s where every CU takes part, less where fewer do
//   launch    = 8 us + its rounds of 256 workgroups; no K split (the epilogue needs whole gate and up sums), but the workgroups
//               of a partly filled last round (or only one) can share its tiles along K, 2 .. 4 per tile: their raw sums go through memory
//               (bf16 / int8 fit: 7.1 / 6 TB/s both ways) and a second launch finishes them (2.5 / 1 us); bf16: where another
//               tile does without and the two are within 3 % that one is taken (40960 x 7168 at 430 rows: the call 2 % faster).
//               Int8 weights, 28672 x 4096 at 580 rows, 256 x 256 tiles shared by three 158 us, 192 x 256 ones 165; 22016 x 4096 at 640
//               shared by four 129, 128 x 256 ones 140; bf16, 16384 x 3072 at 128 rows, 128 tiles shared by two 34 us, alone 38;
//               1024 x 8192 at 16 rows, 16 tiles shared by four 21 us, alone 59
//   384 x 128 is for a single row tile: 28672 x 4096 at 350 rows 87 -> 82 us, but at 640 rows 147 -> 159 us
struct SwigluShape { int tile; float idle, rows; };
static constexpr SwigluShape kSwigluShapes[2][16] = {
    {{T64x128, .45f, .11f}, {T128x128, .51f, .10f}, {T128x160, .53f, .25f}, {T128x224, .65f, .33f}, {T192x128, .65f, .15f},
     {T192x160, .64f, .33f}, {T192x224, .85f, .44f}, {T192x256, 1.01f, .27f}, {T256x128_4x2, .61f, .32f}, {T256x160, .73f, .37f},
     {T256x224, .98f, .52f}, {T256x256, 1.21f, .32f}, {T320x160, .89f, .46f}, {T320x192, 1.02f, .52f}, {T384x128, .86f, .44f},
     {T384x160, 1.03f, .53f}},
    {{T64x128, .38f, .14f}, {T128x128, .64f, .19f}, {T128x256, .79f, .24f}, {T192x128_4x2, .72f, .20f}, {T192x160, .82f, .27f},
     {T192x256, .97f, .33f}, {T256x160, .95f, .34f}, {T256x256, 1.16f, .42f}, {T320x160, 1.07f, .40f}, {T384x160, 1.18f, .47f}}};
// whether a plan can ask for a tile
constexpr bool dma_tile_planned(int epi, int tile, bool w8) {
  if (epi == EPI_SWIGLU) {
    for (const SwigluShape &c : kSwigluShapes[w8])
      if (c.tile == tile && c.idle != 0.f) return true;
    return false;
  }
  for (int i = 0; i < projection_shapes(epi); ++i)
    if (kProjectionTiles[i] == tile && (w8 ? kInt8 : kBf16).t[i] != 0.0) return true;
  return false;
}
static void pick_swiglu_plan(int M, int N, int K, size_t scratch_floats, bool w8, GemmPlan *pl) {
  const int k_tiles = K / DMA_BK;
  const double partial = w8 ? 0.2 : 0.38, starve = w8 ? 0.1 : 0.3;
  double best = 1e30;
  for (const SwigluShape &c : kSwigluShapes[w8]) {
    const DmaTile t = kDmaTiles[c.tile];
    if (c.idle == 0.f || (t.bm() > 256 && M <= 256) || (c.tile == T384x128 && M > t.bm())) continue;
    const int tiles_m = ceil_div(M, t.bm());
    const long ids = 8L * ceil_div(ceil_div(N, t.bn() / 2), 8) * tiles_m, full = ids / 256, tail = ids % 256;
    const double tk = c.idle + c.rows * row_block_steps(t, M) / ((double)tiles_m * t.RB);
    auto round_us = [&](long n, int k) {
      const double share = full ? 1.0 : 1.0 - partial + partial * n / 256.0;
      const double read = (double)n / tiles_m * t.bn() * DMA_BK * (w8 ? 1 : 2) / (6.2e6 * (1.0 - starve * (1.0 - n / 256.0)));
      return k * std::max(tk * share, read);
    };
    double cost = full * round_us(256, k_tiles);
    int ts = 1;
    if (tail) {
      double last = round_us(tail, k_tiles);
      ts = (int)std::min<long>(4, 256 / tail);
      while (ts > 1 && k_tiles / ts < 8) --ts;
      if (ts > 1) {
        const int k = ceil_div(k_tiles, ts);
        const double floats = (double)tail * ts * t.bm() * t.bn();
        const double shared = round_us(tail * ts, k) + floats * 8 / (w8 ? 6.0e6 : 7.1e6) + (w8 ? 1.0 : 2.5);
        const size_t need = (size_t)tail * ceil_div(k_tiles, k) * t.bm() * t.bn();
        if (shared < last && need <= scratch_floats) last = shared;
        else ts = 1;
      }
      cost += last;
    }
    if (ts > 1 && !w8) cost *= 1.03;
    if (cost < best - 1e-9) { best = cost; pl->tile = c.tile; pl->tail_splits = ts; }
  }
}

// Tile of the float kernels: 64 x 64 when those occupy the chip twice over (a quarter of the loads per flop), else
// 32 x 32 with the wavefronts sharing K (544 rows of the 256-wide model occupy 36 CUs with 64 x 64 tiles, 136 with these),
// 16 x 16 where those leave most CUs idle too: 186 rows x 256 columns, 48 tiles of 32 x 32 against 192, 7.8 -> 4.6 us; with 136 tiles of
// 32 x 32 both take 7.5 us, with 258 / 272 the small ones, which read four times as much per flop, 8.1 / 9.8 against 6.4 / 7.7 us.
// The line lies at the same place for any K.  Time on 16 x 16 over time on 32 x 32 tiles at K = 64 / 256 / 1024 / 4096 / 16384, 64 .. 14336
// columns, 1 .. 1200 rows, on average: up to 63 tiles of 32 x 32 0.95 / 0.80 / 0.63 / 0.48 / 0.32, 64 .. 95 tiles 0.96 / 0.89 / 0.73 / 0.59 / 0.35, 128 .. 255
// tiles (256 and up) 1.05 / 0.99 / 0.79 / 0.76 with single sizes up to 1.44, beyond 1.4 .. 2.
static int f32_tile(int epi, int M, int N) {
  auto tiles = [&](int t) { return (long)ceil_div(M, t) * ceil_div(N, epi == EPI_SWIGLU ? t / 2 : t); };
  return tiles(64) >= 512 ? 64 : tiles(32) >= 96 ? 32 : 16;
}
// A float tile narrower than a head cannot pair channel i with i + head_dim/2 itself: it parks its sums and the
// finish launch rotates them.
static bool needs_raw_partial(int dtype, int epi, int M, int N, int rope_half, int head_dim) {
  return dtype == 0 && epi == EPI_SEG && rope_half && head_dim > f32_tile(epi, M, N);
}

bool gemm_int8_in_kernel(int dtype, int K) { return dtype == 1 && K % DMA_BK == 0; }

// Shape of one problem.  hl: leading output columns with (high, low) activation pairs; force_raw: the caller wants the finish
// launch (deviation, or the float output's residual + norm); scratch_floats: what `partial` holds
// (the K split is capped by it; SIZE_MAX when sizing); model: another cost model than the problem's own.
static GemmPlan make_plan(int dtype, int epi, int M, int N, int K, int hl, int force_raw, int rope_half,
                          int head_dim, size_t scratch_floats, bool w8 = false, const ProjectionModel *model = nullptr) {
  GemmPlan pl = {};
  pl.w8 = w8;
  pl.tail_splits = 1;
  if (w8 && !gemm_int8_in_kernel(dtype, K)) pl.bad = true;
  pl.splits = 1;
  pl.hl = dtype == 1 && epi == EPI_SEG ? hl : 0;
  pl.raw = force_raw || epi == EPI_F32 || needs_raw_partial(dtype, epi, M, N, rope_half, head_dim);
  const size_t mn = (size_t)M * N;
  const int max_splits = (int)std::min<size_t>(16, std::max<size_t>(1, scratch_floats / std::max<size_t>(1, mn)));
  if (pl.raw && scratch_floats < mn) pl.bad = true;
  if (dtype == 0) {
    pl.kind = 0; pl.bm = f32_tile(epi, M, N); pl.out_cols = epi == EPI_SWIGLU ? pl.bm / 2 : pl.bm; pl.bk = BK32;
  } else if (K % DMA_BK != 0) {
    pl.kind = 1; pl.bm = BM16; pl.out_cols = epi == EPI_SWIGLU ? BN16 / 2 : BN16; pl.bk = BK16;
  } else if (epi == EPI_SWIGLU) {
    pl.kind = 2; pl.bk = DMA_BK;
    pick_swiglu_plan(M, N, K, scratch_floats, w8, &pl);
  } else {
    pl.kind = 2; pl.bk = DMA_BK; pl.tile = -1;
    pick_dma_plan(model ? *model : w8 ? kInt8 : pl.hl == N ? kPairs : kBf16, epi, M, N, pl.hl, K, max_splits, pl.raw, w8, &pl);
    if (pl.tile < 0) { pl.bad = true; pl.tile = T256x256; }    // no tile width divides the columns with pairs
  }
  if (pl.kind == 2) {
    pl.bm = kDmaTiles[pl.tile].bm();
    pl.out_cols = kDmaTiles[pl.tile].bn() / (epi == EPI_SWIGLU ? 2 : 1);
  }
  pl.tiles_m = ceil_div(M, pl.bm);
  pl.tiles_n = ceil_div(pl.kind == 2 ? N - pl.hl : N, pl.out_cols);
  if (pl.kind == 2 && pl.hl) {
    pl.hl_tiles_m = ceil_div(M, pl.bm / 2);
    pl.hl_tiles_n = ceil_div(pl.hl, pl.out_cols);
  }
  const int k_tiles = ceil_div(K, pl.bk);
  const long tiles = (long)pl.tiles_m * pl.tiles_n;
  if (pl.kind == 1 && epi != EPI_SWIGLU && tiles < 256) {
    // smallest split that fills >= 90 % of a whole number of 256-workgroup rounds
    double best_eff = 0;
    for (int sp = 1; sp <= 16 && sp <= max_splits; ++sp) {
      if (sp > 1 && k_tiles / sp < 4) break;
      const long wgs = tiles * sp;
      const double eff = (double)wgs / (double)((wgs + 255) / 256 * 256);
      if (eff > best_eff + 1e-9) { best_eff = eff; pl.splits = sp; }
      if (eff >= 0.9) break;
    }
  }
  pl.k_per_split = ceil_div(k_tiles, pl.splits) * pl.bk;
  pl.splits = ceil_div(K, pl.k_per_split);
  if (pl.splits > 1) pl.raw = 1;
  pl.partial_floats = pl.raw ? (size_t)pl.splits * mn : 0;
  if (pl.kind == 2) {
    const int groups = epi == EPI_SWIGLU ? 8 : xcd_groups(pl.splits, pl.tiles_m, pl.tiles_n, pl.hl);
    pl.xcd_split = groups < 8;
    pl.k_stagger = !w8 && pl.tiles_m == 1 && pitch_is_power_of_two(K);
    const bool nt = epi != EPI_SEG && !w8 && pl.tiles_m == 1 && (epi == EPI_SWIGLU ? 4.0 : 2.0) * N * K >= kNtMinBytes;
    pl.mode = nt ? MODE_NT : pl.k_stagger ? MODE_STAGGER : MODE_PLAIN;
    const long ids = 8L * (ceil_div(pl.tiles_n, groups) * pl.tiles_m + ceil_div(pl.hl_tiles_n, groups) * pl.hl_tiles_m);
    pl.grid_ids = pl.xcd_split ? ids : ids * pl.splits;
    pl.tail_first = (int)pl.grid_ids;
    if (pl.tail_splits > 1) {
      const long tail = pl.grid_ids % 256;
      pl.tail_first = (int)(pl.grid_ids - tail);
      pl.tail_k_per_split = ceil_div(k_tiles, pl.tail_splits) * pl.bk;
      pl.tail_splits = ceil_div(K, pl.tail_k_per_split);
      pl.grid_ids = pl.tail_first + tail * pl.tail_splits;
      pl.partial_floats = (size_t)tail * pl.tail_splits * pl.bm * (2 * pl.out_cols);
    }
  }
  return pl;
}

static int problem_n(const GemmArgs &g) {
  if (g.epi == EPI_SWIGLU) return g.seg[0].n;
  int n = 0;
  for (int i = 0; i < (g.epi == EPI_SEG ? g.n_seg : 1); ++i) n += g.seg[i].n;
  return n;
}

size_t gemm_partial_floats(int dtype, int epi, int M, int N, int K, int hl, int force_raw, int rope_half,
                           int head_dim, int w8, bool split) {
  if (M <= 0) return 0;
  return make_plan(dtype, epi, M, N, K, hl, force_raw, rope_half, head_dim, split ? SIZE_MAX : 0,
                   w8 && gemm_int8_in_kernel(dtype, K)).partial_floats;
}

// For tests (no device is touched): the plan of one bf16 or float problem.  out: kind, tile rows, tile columns of the weights, K splits,
// splits of a shared last round, mode, staggered start, finish launch; returns the floats it parks.
extern "C" size_t cb_internal_projection_plan(int dtype, int epi, int M, int N, int K, int hl, int force_raw, int w8,
                                              size_t scratch_floats, int *out) {
  if (M <= 0) return 0;
  const GemmPlan pl = make_plan(dtype, epi, M, N, K, hl, force_raw, 0, 64, scratch_floats, w8 && gemm_int8_in_kernel(dtype, K));
  const int v[8] = {pl.kind, pl.bm, pl.out_cols * (epi == EPI_SWIGLU ? 2 : 1), pl.splits, pl.tail_splits, pl.mode, pl.k_stagger,
                    pl.raw || pl.tail_splits > 1};
  for (int i = 0; i < 8; ++i) out[i] = v[i];
  return pl.partial_floats;
}

static GemmPlan fill_params(const GemmArgs &g, GemmParams *pp) {
  GemmParams &p = *pp;
  p = GemmParams{};
  p.a = g.a; p.lda = g.lda; p.a_rows = g.a_rows; p.M = g.M; p.K = g.K;
  p.n_seg = g.epi == EPI_SEG ? g.n_seg : 1;
  p.nb[0] = 0;
  for (int i = 0; i < 3; ++i) {
    p.w[i] = g.seg[i].w; p.w_scale[i] = g.seg[i].w_scale; p.dst[i] = g.seg[i].dst; p.ld[i] = g.seg[i].ld_dst;
    p.row_map[i] = g.seg[i].row_map; p.rope[i] = g.seg[i].rope;
    p.nb[i + 1] = p.nb[i] + (i < p.n_seg ? g.seg[i].n : 0);
    p.dev_cache[i] = g.dev_out ? g.seg[i].dev_cache : nullptr;
  }
  p.N = problem_n(g);
  p.rope_tab = g.rope_tab; p.row_pos = g.row_pos; p.head_dim = g.head_dim;
  p.out_f32 = g.out_f32; p.resid = g.resid; p.resid_rows = g.resid_rows; p.partial = g.partial;
  p.rope_half = g.rope_half;
  p.dev_out = g.dev_out; p.n_dev = g.n_dev; p.dev_row = g.dev_row;
  p.norm_gain = g.norm_gain; p.norm_out = g.norm_out; p.norm_ld = g.norm_ld; p.norm_lo_off = g.norm_lo_off;
  p.norm_eps = g.norm_eps;
  const int hl_cols = g.a_lo_off > 0 ? p.nb[g.n_hl_seg > 0 ? std::min(g.n_hl_seg, p.n_seg) : p.n_seg] : 0;
  const size_t scratch = g.partial ? (g.split_floats ? std::min(g.split_floats, g.partial_floats) : g.partial_floats) : 0;
  GemmPlan pl = make_plan(g.dtype, g.epi, g.M, p.N, g.K, hl_cols, g.dev_out != nullptr, g.rope_half, g.head_dim, scratch,
                          g.seg[0].w_scale != nullptr);
  if (pl.kind != 2 && hl_cols != 0 && hl_cols != p.N) pl.bad = true;   // the other kernels treat all columns alike
  // every matrix of a launch is in the same format
  const int n_w = g.epi == EPI_SEG ? g.n_seg : (g.epi == EPI_SWIGLU ? 2 : 1);
  for (int i = 1; i < n_w; ++i)
    if ((g.seg[i].w_scale != nullptr) != (g.seg[0].w_scale != nullptr)) pl.bad = true;
  p.a_lo_off = pl.hl ? g.a_lo_off : 0;
  p.hl_cols = pl.hl; p.hl_tiles_m = pl.hl_tiles_m; p.hl_tiles_n = pl.hl_tiles_n;
  p.raw_partial = pl.raw;
  p.splits = pl.splits;
  p.k_per_split = pl.k_per_split;
  p.tail_first = pl.tail_first; p.tail_splits = pl.tail_splits; p.tail_k_per_split = pl.tail_k_per_split;
  p.xcd_split = pl.xcd_split;
  p.k_stagger = pl.k_stagger;
  return pl;
}

bool gemm_merge_pays(int M, int hl_cols, int M_rest, int n_rest, int K, int force_raw, int w8, size_t split_floats) {
  if (M <= 0 || M_rest <= 0 || K % DMA_BK != 0) return false;
  // one model for all three (bf16: over 7169 sizes of 11 models the calls take 0.1 % more than with the better choice each time; with a
  // model for K and V alone and another for the rest, whose errors differ, 0.4 %)
  const ProjectionModel *model = w8 ? &kInt8 : &kPairs;
  const GemmPlan one = make_plan(1, EPI_SEG, M, hl_cols + n_rest, K, hl_cols, force_raw, 0, 0, split_floats, w8, model);
  if (one.bad || one.kind != 2) return false;
  const GemmPlan kv = make_plan(1, EPI_SEG, M, hl_cols, K, hl_cols, force_raw, 0, 0, split_floats, w8, model);
  const GemmPlan q = make_plan(1, EPI_SEG, M_rest, n_rest, K, 0, 0, 0, 0, split_floats, w8, model);
  return one.cost < kv.cost + q.cost;
}

bool gemm_needs_finish(const GemmArgs &g) {
  if (g.M == 0) return false;
  GemmParams p;
  const GemmPlan pl = fill_params(g, &p);
  return pl.raw || pl.tail_splits > 1;
}

// sets a kernel's dynamic LDS limit once per process, whichever host thread launches it first
#define CB_LDS_LIMIT_ONCE(kernel_expr, bytes)                                                      \
  do {                                                                                             \
    static std::once_flag once_;                                                                   \
    std::call_once(once_, [] {                                                                     \
      (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel_expr),                       \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)(bytes));         \
    });                                                                                            \
  } while (0)

template <int T, int EPI, bool HL, bool W8, int MODE>
static void launch_dma_kernel(const GemmPlan &pl, const GemmParams &p, hipStream_t s) {
  constexpr DmaTile t = kDmaTiles[T];
  constexpr int smem = dma_smem_bytes(t.bm(), t.bn(), W8);
  CB_LDS_LIMIT_ONCE((&gemm_bf16_dma_kernel<t.RB, t.CB, t.WM, t.WN, EPI, HL, W8, MODE>), smem);
  hipLaunchKernelGGL((gemm_bf16_dma_kernel<t.RB, t.CB, t.WM, t.WN, EPI, HL, W8, MODE>), dim3((unsigned)pl.grid_ids),
                     dim3(64 * t.WM * t.WN), smem, s, p, pl.tiles_m, pl.tiles_n);
}

// Only kernels of tiles that a plan can ask for are built; false for any other.
template <int T, int EPI, bool HL>
static bool launch_dma(const GemmPlan &pl, const GemmParams &p, hipStream_t s) {
  if (pl.w8) {
    if constexpr (dma_tile_planned(EPI, T, true)) {
      launch_dma_kernel<T, EPI, HL, true, MODE_PLAIN>(pl, p, s);
      return true;
    }
  } else {
    if constexpr (dma_tile_planned(EPI, T, false)) {
      if (pl.mode == MODE_NT) launch_dma_kernel<T, EPI, HL, false, EPI == EPI_SEG ? MODE_PLAIN : MODE_NT>(pl, p, s);
      else if (pl.mode == MODE_STAGGER) launch_dma_kernel<T, EPI, HL, false, MODE_STAGGER>(pl, p, s);
      else launch_dma_kernel<T, EPI, HL, false, MODE_PLAIN>(pl, p, s);
      return true;
    }
  }
  return false;
}

template <int EPI, bool HL, int T = 0>
static bool launch_dma_shape(const GemmPlan &pl, const GemmParams &p, hipStream_t s) {
  if constexpr (T < kNumDmaTiles) return pl.tile == T ? launch_dma<T, EPI, HL>(pl, p, s) : launch_dma_shape<EPI, HL, T + 1>(pl, p, s);
  else return false;
}

template <int T = 0>
static bool launch_tail(const GemmPlan &pl, const GemmParams &p, hipStream_t s) {
  if constexpr (T < kNumDmaTiles) {
    if (pl.tile != T) return launch_tail<T + 1>(pl, p, s);
    constexpr DmaTile t = kDmaTiles[T];
    const int shared = (int)(pl.grid_ids - pl.tail_first) / pl.tail_splits;
    hipLaunchKernelGGL((swiglu_tail_kernel<t.RB, t.CB, t.WM, t.WN>), dim3((unsigned)(shared * ceil_div(t.WM * t.WN * t.RB * ((t.CB + 1) / 2), 16))),
                       dim3(256), 0, s, p, pl.tiles_m, pl.tiles_n);
    return true;
  }
  return false;
}

template <int EPI>
static bool launch_typed(const GemmPlan &pl, const GemmParams &p, hipStream_t s) {
  const dim3 grid(pl.tiles_n, pl.tiles_m, pl.splits);
  if (pl.kind == 0) {
    if (pl.bm == 16) hipLaunchKernelGGL(gemm_f32_small_kernel<EPI>, grid, dim3(256), 0, s, p);
    else if (pl.bm == 64) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, 2, 1>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, 1, 1, 4>), grid, dim3(256), 0, s, p);
    return true;
  }
  if (pl.kind == 1) {
    CB_LDS_LIMIT_ONCE((&gemm_bf16_kernel<EPI>), kSmemBf16);
    hipLaunchKernelGGL(gemm_bf16_kernel<EPI>, grid, dim3(256), kSmemBf16, s, p);
    return true;
  }
  if (EPI == EPI_SEG && pl.hl) return launch_dma_shape<EPI_SEG, true>(pl, p, s);
  return launch_dma_shape<EPI, false>(pl, p, s);
}

hipError_t launch_gemm(const GemmArgs &g, hipStream_t s) {
  if (g.M == 0) return hipSuccess;
  GemmParams p;
  const GemmPlan pl = fill_params(g, &p);
  if (pl.bad) return hipErrorInvalidValue;
  const bool built = g.epi == EPI_SEG ? launch_typed<EPI_SEG>(pl, p, s)
                     : g.epi == EPI_SWIGLU ? launch_typed<EPI_SWIGLU>(pl, p, s) : launch_typed<EPI_F32>(pl, p, s);
  return built ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_gemm_finish(const GemmArgs &g, hipStream_t s) {
  if (g.M == 0) return hipSuccess;
  GemmParams p;
  const GemmPlan pl = fill_params(g, &p);
  if (pl.bad) return hipErrorInvalidValue;
  if (pl.tail_splits > 1) {
    return launch_tail(pl, p, s) ? hipGetLastError() : hipErrorInvalidValue;
  }
  if (!pl.raw) return hipSuccess;
  const dim3 grid((unsigned)g.M);
  if (g.epi == EPI_SEG) {
    int first = std::min(p.N, kFinishCols);
    for (int i = 0; i < p.n_seg; ++i)
      if (p.dev_cache[i]) first = std::max(i == 0 ? 0 : first, p.nb[i + 1]);
    const dim3 fgrid((unsigned)g.M, 1 + ceil_div(p.N - first, kFinishCols));
    if (g.dtype == 0) hipLaunchKernelGGL(seg_finish_kernel<float>, fgrid, dim3(256), 0, s, p, first);
    else hipLaunchKernelGGL(seg_finish_kernel<bf16>, fgrid, dim3(256), 0, s, p, first);
  } else {
#define CB_ROW(NC_)                                                                                        \
  do {                                                                                                     \
    if (g.dtype == 0) hipLaunchKernelGGL((resid_norm_finish_row_kernel<float, NC_>), grid, dim3(256), 0, s, p); \
    else hipLaunchKernelGGL((resid_norm_finish_row_kernel<bf16, NC_>), grid, dim3(256), 0, s, p);          \
  } while (0)
    if (p.N <= 2048) CB_ROW(2);
    else if (p.N <= 4096) CB_ROW(4);
    else if (p.N <= 8192) CB_ROW(8);
    else if (g.dtype == 0) hipLaunchKernelGGL(resid_norm_finish_kernel<float>, grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL(resid_norm_finish_kernel<bf16>, grid, dim3(256), 0, s, p);
#undef CB_ROW
  }
  return hipGetLastError();
}

}  // namespace cb
