// Sparse-query causal attention (paper Sec. 4.2): the recomputed rows are the queries,
// the keys and values are ALL rows of the fused cache, recomputed or reused; with every
// row selected it is plain causal attention (Sec. 2).  A query at global position p
// sees cache rows 0..p.
//
// bf16 kernel (MFMA 32x32x16).  One workgroup = one kv head x a block of
// "flattened queries" m = row * g + head_in_group, so the g query heads that share
// a kv head sit side by side in the MFMA N dimension and every K/V tile staged in
// LDS is used by all of them.  Each of the 8 wavefronts owns a block of 32 queries.
// Both products are computed transposed,
//     S^T[key, query] = K Q^T            O^T[channel, query] += V^T P^T
// so that a lane always holds values of ONE query (column = lane % 32): the running
// max / sum and the rescaling of O need no cross-lane traffic except one exchange
// between the two half-waves, and the exponentiated scores are already laid out as
// the B operand of the second product (they never leave registers).  The second
// product contracts over keys; V stays row-major in LDS and its operand is fetched with
// the transposing LDS read (ds_read_b64_tr_b16).  K/V tiles are streamed through 4-stage
// LDS rings by direct global->LDS loads.
//
// float kernel: float MFMAs, 16 queries per workgroup, the wavefronts share the keys.
#include "common.h"
#include "kernels.h"
#include <algorithm>
#include <mutex>

namespace cb {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;

// ---------------------------------------------------------------------------
constexpr int BKV = 64;                 // keys per tile, walked as two sub-tiles of 32
constexpr int ATT_S = 4;                // LDS ring stages of the K ring and of the V ring
constexpr int ATT_NW = 8;               // wavefronts per workgroup: two per SIMD
constexpr int ATT_WGQ = 32 * ATT_NW;    // flattened queries per workgroup
constexpr float kLazyMax = 8.f;         // a running maximum may lag behind by a factor 2^8 (see below)

typedef __attribute__((ext_vector_type(4))) short s16x4;

// LDS reads issued by hand: the compiler waits for every outstanding global->LDS load before a transposing read
// (it cannot see that the tile being read landed long ago), which would undo the ring.  The results are valid
// only after att_wait<N>() with at most N younger reads in flight.
template <int OFF> __device__ __forceinline__ void att_read_k(bf16x8 &dst, unsigned addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
template <int OFF> __device__ __forceinline__ void att_read_v(s16x4 &dst, unsigned addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
template <int N> __device__ __forceinline__ void att_wait() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N)); }
template <int N> __device__ __forceinline__ void att_vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// maximum over the wavefront / over the two half-waves without LDS (the shuffles would count as LDS reads)
__device__ __forceinline__ float half_swap_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ int wave_max_i32(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

template <int V> struct IntC { static constexpr int value = V; };

// What bounds it and how the loop is laid out.  Per 64 keys a wavefront issues 4 DH/16 MFMAs of 32 clocks each for
// its 32 queries, and two wavefronts share a SIMD, so the matrix core needs 2048 clocks per tile at DH = 128; the
// operand reads of the 8 wavefronts take about 1340 clocks of LDS, the softmax about 110 vector and 32 transcendental
// instructions per wavefront.  All three fit side by side if the instruction streams are mixed, so the loop is
// software-pipelined by hand: a PHASE handles a sub-tile of 32 keys j and interleaves, MFMA by MFMA,
//     S(j+1) = K(j+1) Q^T        softmax of S(j)        O += V(j-1) P(j-1)
// none of which depends on another.  Operand reads run two steps ahead (a step = one MFMA of each product).
// The running maximum is updated lazily: exponents are taken relative to a reference that only moves when a score
// exceeds it by 2^8, so the accumulators are almost never rescaled (P is bf16 and the sums are float: a common factor
// costs no precision); a rescale is applied at the end of the phase, after O has taken P(j-1), which was
// computed relative to the old reference.
//   K ring, V ring: 4 stages each.  In iteration t (tile t) the phases read K(t), K(t+1) and V(t-1), V(t); the loads of
//   K(t+3) and V(t+2) are issued, and the barrier at its start waits for the loads of iteration t-2.
// Measured (32 query heads over 8 kv heads): dense 16 K x 16 K 2233 -> 1940 us (1135 TFLOP/s), 3000 rows over 20.7 K
// tokens 644 -> 537 us, 500 rows over 3136 tokens 46 -> 40 us with the merge; a tile takes 1.42 us on an otherwise idle
// chip (1.99 before) and 1.87 us with every CU busy, where power sets the clock.  The same loop on 16x16x32 MFMAs
// measured 1.59 / 1.82 us, four wavefronts of 64 queries (half the LDS reads) did not fit the register file.
template <int DH>
__global__ __launch_bounds__(64 * ATT_NW) void attn_bf16_kernel(const bf16 *__restrict__ q,
                                                        const int32_t *__restrict__ q_pos, int n_rows,
                                                        const bf16 *__restrict__ kc,
                                                        const bf16 *__restrict__ vc, bf16 *__restrict__ o,
                                                        int n_q_heads, int n_kv_heads, float scale_log2e,
                                                        int split_tiles, float *__restrict__ part_o,
                                                        float *__restrict__ part_ml,
                                                        const int32_t *__restrict__ q_rows,
                                                        int32_t *__restrict__ wg_tiles,
                                                        const int32_t *__restrict__ segs, int n_segs) {
  // K and V tiles sit row-major in LDS ([key][channel], no padding) and are filled by direct
  // global->LDS loads: one wavefront-wide 16-byte load writes 1 KB = RPI whole rows.  Instead of
  // padding, the 16-byte chunk c of row r is stored in slot c ^ f(r).
  constexpr int ROWB = DH * 2;            // bytes per row
  constexpr int CH = DH / 8;              // 16-byte chunks per row
  constexpr int RPI = 1024 / ROWB;        // rows per wavefront-wide load
  constexpr int TILEB = BKV * ROWB;       // bytes of one K (or V) tile
  constexpr int LPT = BKV / RPI / ATT_NW; // loads per lane per K tile (and per V tile)
  constexpr int NST = DH / 16;            // steps per phase: k-steps of S^T, and (16-key group, 32-channel block) pairs of O^T
  constexpr int DB = DH / 32;             // 32-channel blocks of the output
  static_assert(LPT >= 1 && NST == 2 * DB && NST % 4 == 0, "step and buffer bookkeeping");
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, h = lane >> 5;
  const int g = n_q_heads / n_kv_heads;
  const int kvh = blockIdx.x;                          // kv head varies fastest in dispatch order
  const int kv_dim = n_kv_heads * DH;
  // workgroups with the longest key range (the last rows) are dispatched first, for every kv head
  const int qwg = (int)(gridDim.y - 1 - blockIdx.y);
  // Several requests in one launch: request s owns the query workgroups [segs[s].qwg, segs[s+1].qwg),
  // the rows [row0, row0 + rows) of q_pos / q_rows / o, and the cache rows from cache0 on.
  int seg_qwg0 = 0, row0 = 0;
  if (segs) {
    int lo = 0, hi = n_segs - 1;                       // last segment whose first workgroup is <= qwg
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (segs[mid * kSegInts + kSegQwg] <= qwg) lo = mid; else hi = mid - 1;
    }
    const int32_t *sg = segs + lo * kSegInts;
    seg_qwg0 = sg[kSegQwg];
    row0 = sg[kSegOutOff];
    n_rows = sg[kSegKeep] + sg[kSegSuffix];
    const size_t cache0 = (size_t)sg[kSegCacheRow] * kv_dim;
    kc += cache0;
    vc += cache0;
    q_pos += row0;
    if (q_rows) q_rows += row0;
  }
  const int n_flat = n_rows * g;
  const int m_wg = (qwg - seg_qwg0) * ATT_WGQ;         // first flattened query of the workgroup, within its request
  const int m_pad = qwg * ATT_WGQ;                     // the same in the launch-wide numbering of the scratch
  const int n_flat_pad = (int)gridDim.y * ATT_WGQ;

  // this lane's query (the loads overlap the search for the causal bound below)
  const int m_own = m_wg + wave * 32 + ln;
  const bool valid = m_own < n_flat;
  const int r_own = (valid ? m_own : n_flat - 1) / g, j_own = (valid ? m_own : n_flat - 1) - r_own * g;
  const int my_pos = valid ? q_pos[r_own] : -1;
  const long q_off = ((long)(row0 + r_own) * n_q_heads + kvh * g + j_own) * DH;
  bf16x8 qf[NST];
  {
    const long q_src = ((long)(q_rows ? q_rows[r_own] : row0 + r_own) * n_q_heads + kvh * g + j_own) * DH;
#pragma unroll
    for (int ks = 0; ks < NST; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(q + q_src + ks * 16 + 8 * h);
  }
  // causal bound of the workgroup = largest position among its rows (they need not be sorted); every wavefront
  // looks at all of them, which needs no exchange
  int max_pos = -1;
  {
    const int last_r = (min(m_wg + ATT_WGQ, n_flat) - 1) / g;
    for (int r = m_wg / g + lane; r <= last_r; r += 64) max_pos = max(max_pos, q_pos[r]);
  }
  const int kv_len = __builtin_amdgcn_readfirstlane(wave_max_i32(max_pos)) + 1;
  const int n_tiles_all = (kv_len + BKV - 1) / BKV;
  // the merge launch needs the same bound to know which pieces of the key range ran
  if (gridDim.z > 1 && kvh == 0 && blockIdx.z == 0 && tid == 0) wg_tiles[qwg] = n_tiles_all;
  // KV split: workgroup z of gridDim.z handles tiles [t_begin, n_tiles) of the causal range and
  // leaves un-normalised partial results (flash-decoding style) for the merge kernel
  const int t_begin = blockIdx.z * split_tiles;
  if (t_begin >= n_tiles_all) return;
  const int n_tiles = min(n_tiles_all, t_begin + split_tiles);
  const int wave_max_pos = __builtin_amdgcn_readfirstlane(wave_max_i32(my_pos));
  const int wave_min_pos = -__builtin_amdgcn_readfirstlane(wave_max_i32(-my_pos));   // invalid queries (-1) force masking
  const int t_last = min(n_tiles - 1, wave_max_pos >> 6);   // last tile this wavefront computes on (may be < t_begin)

  // Swizzles f(r).  K is read 16 bytes per lane, 32 rows at a time: DH = 128 rows start at bank 0 -> f = r & 15;
  // DH = 64 rows alternate between the two bank halves -> f = (r >> 1) & 7.  V goes through the transposing
  // 8-byte read, 16 lanes of which take 32 bytes of each of 4 adjacent keys: those 4 keys have to lie in different
  // 64-byte groups (f = 4 (r & 3) + ...), else they conflict: 190 against 63 bytes per clock and CU with f = r & 15.
  auto fk = [](int r) { return DH == 128 ? (r & 15) : ((r >> 1) & 7); };
  auto fv = [](int r) { return DH == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3)); };

  // ---- global -> LDS: this lane's share of the loads of one tile ----
  const unsigned row_bytes = (unsigned)kv_dim * 2;
  int ld_row[LPT];                        // tile row of load i; K and V loads use the same rows
  unsigned ld_kcol[LPT], ld_vcol[LPT];    // byte offset of the (de-swizzled) chunk
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    ld_row[i] = (wave + ATT_NW * i) * RPI + lane / CH;
    ld_kcol[i] = (unsigned)((((lane % CH) ^ fk(ld_row[i])) * 8 + kvh * DH) * 2);
    ld_vcol[i] = (unsigned)((((lane % CH) ^ fv(ld_row[i])) * 8 + kvh * DH) * 2);
  }
  const unsigned lds0 = (unsigned)(size_t)smem;
  // one load of tile t (clamped to the last tile, rows clamped to the causal bound: every call issues its load)
  auto issue = [&](int t, int i, bool is_v) {
    const int t0 = min(t, n_tiles_all - 1) * BKV;
    const char *base = reinterpret_cast<const char *>(is_v ? vc : kc) + (size_t)t0 * row_bytes;
    const unsigned row = (unsigned)min(ld_row[i], kv_len - 1 - t0);
    const char *src = base + (size_t)(row * row_bytes + (is_v ? ld_vcol[i] : ld_kcol[i]));
    char *dst = smem + (is_v ? ATT_S * TILEB : 0) + (t & (ATT_S - 1)) * TILEB + (wave + ATT_NW * i) * 1024;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < LPT; ++i) issue(t_begin, i, false);
#pragma unroll
  for (int i = 0; i < LPT; ++i) issue(t_begin, i, true);
#pragma unroll
  for (int i = 0; i < LPT; ++i) issue(t_begin + 1, i, false);
#pragma unroll
  for (int i = 0; i < LPT; ++i) issue(t_begin + 1, i, true);
#pragma unroll
  for (int i = 0; i < LPT; ++i) issue(t_begin + 2, i, false);

  // ---- LDS read addresses of this lane, kept for the tile being read and moved from stage to stage ----
  unsigned k_addr[NST], v_addr[DB][2];
#pragma unroll
  for (int ks = 0; ks < NST; ++ks)        // K operand: row ln (+ 32 for the second sub-tile), chunk 2 ks + h
    k_addr[ks] = lds0 + (t_begin & (ATT_S - 1)) * TILEB + ln * ROWB + (((2 * ks + h) ^ fk(ln)) << 4);
  // V operand through the transposing read: lane s of a 16-lane block passes the address of
  // 4 channels (8 bytes) of key K0 + s/4 and receives, for channel C0 + s, the 4 keys K0..K0+3.
  // Starts one stage back: the first phase's read moves it to tile t_begin (there is no V(t_begin - 1) to read).
  {
    const int s16 = lane & 15, qb = lane >> 4;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int key = 8 * a + 4 * (qb >> 1) + (s16 >> 2);               // + 16 u per MFMA
        const int ch = d * 32 + 16 * (qb & 1) + 4 * (s16 & 3);
        v_addr[d][a] = lds0 + ATT_S * TILEB + (t_begin & (ATT_S - 1)) * TILEB + key * ROWB + (((ch >> 3) ^ fv(key)) << 4) + (ch & 7) * 2;
      }
  }

  f32x16 oacc[DB], sacc[2];
  union PF { unsigned w[4]; bf16x8 b; } pf[2][2];   // P of the sub-tile before and of the one in work, two 16-key groups each
  float ref = -INFINITY, thr = -INFINITY, neg_mc = 0.f, row_sum = 0.f;
  const float lazy = kLazyMax / scale_log2e;
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[d][i] = 0.f;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) pf[a][u].w[e] = 0u;

  bf16x8 kf[4];
  union VF { s16x4 s[2]; bf16x8 b; } vf[4];
  // Requests step I of a phase: the K fragment (WK) of k-step I and the V fragment (two transposing reads, WV) of
  // (16-key group I / DB, channel block I % DB).  ODD: the phase works on S of the first half of the next K
  // tile and on the first half of the V tile after the one the addresses point at, so its reads move the
  // addresses on (by dk / dv bytes; dv also serves the first phase, which rereads V(t_begin) against P = 0).
  auto read_step = [&](auto odd_, auto wk_, auto wv_, auto i_, int dk, int dv) {
    constexpr int ODD = decltype(odd_)::value, I = decltype(i_)::value, D = I % DB, U = I / DB;
    if constexpr (decltype(wk_)::value) {
      if constexpr (ODD) k_addr[I] += dk;
      att_read_k<(ODD ? 0 : 32 * ROWB)>(kf[I & 3], k_addr[I]);
    }
    if constexpr (decltype(wv_)::value) {
      if constexpr (ODD && U == 0) { v_addr[D][0] += dv; v_addr[D][1] += dv; }
      att_read_v<((ODD ? 0 : 2) + U) * 16 * ROWB>(vf[I & 3].s[0], v_addr[D][0]);
      att_read_v<((ODD ? 0 : 2) + U) * 16 * ROWB>(vf[I & 3].s[1], v_addr[D][1]);
    }
  };

  // One phase: softmax of sub-tile j = 2t + ODD (SM), S of sub-tile j+1 (WS), O += V P of sub-tile j-1.
  // NS / NX: whether the phase that follows computes S / exists (its first two steps are requested here).
  auto phase = [&](auto odd_, auto sm_, auto ws_, auto ns_, auto nx_, int t, int dk, int dv) {
    constexpr int ODD = decltype(odd_)::value, SM = decltype(sm_)::value, WS = decltype(ws_)::value;
    constexpr int NS = decltype(ns_)::value, NX = decltype(nx_)::value;
    f32x16 &sc = sacc[ODD], &sn = sacc[1 - ODD];
    PF (&pc)[2] = pf[ODD], (&pp)[2] = pf[1 - ODD];
    bool moved = false;
    float alpha = 1.f, mx = -INFINITY, psum = 0.f;
    float e[16];
    if constexpr (SM) {
      const int s0 = t * BKV + ODD * 32;
      if (s0 + 31 > wave_min_pos) {                    // wave-uniform: some key of the sub-tile is masked
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = s0 + (i >> 2) * 8 + h * 4 + (i & 3);
          sc[i] = key <= my_pos ? sc[i] : -INFINITY;
        }
      }
    }
    auto fold = [&](int i) {                           // pair i: into the sum, and to bf16
      psum += e[2 * i];
      psum += e[2 * i + 1];
      const bf16x2 w = {(bf16)e[2 * i], (bf16)e[2 * i + 1]};
      pc[i >> 2].w[i & 3] = __builtin_bit_cast(unsigned, w);
      asm volatile("" : "+v"(psum), "+v"(pc[i >> 2].w[i & 3]));
    };
    // vector work of half-step c (two per step): the maximum in the first four half-steps, then the 16
    // exponentials with their sums and conversions spread over the rest
    auto vec = [&](auto c_) {
      constexpr int C = decltype(c_)::value, C0 = 3, NC = 2 * NST - C0;
      if constexpr (SM) {
        if constexpr (C == 0) {
#pragma unroll
          for (int i = 0; i < 8; ++i) mx = fmaxf(fmaxf(mx, sc[i]), sc[i + 8]);
        } else if constexpr (C == 1) {
          mx = half_swap_max(mx);
        } else if constexpr (C == 2) {
          if (__any(mx > thr)) {
            // masked scores are -inf; a query that has seen no key yet (possible inside a later piece of
            // the key range, or for the padding lanes) keeps ref = -inf and gets p = 0 everywhere
            const float nr = fmaxf(ref, mx);
            alpha = nr > ref ? __builtin_amdgcn_exp2f((ref - nr) * scale_log2e) : 1.f;
            ref = nr;
            thr = nr + lazy;
            neg_mc = nr == -INFINITY ? 0.f : -nr * scale_log2e;
            moved = true;
          }
        } else {
          constexpr int B0 = 16 * (C - C0) / NC, B1 = 16 * (C - C0 + 1) / NC;
#pragma unroll
          for (int i = B0; i < B1; ++i) {
            e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i], scale_log2e, neg_mc));
            asm volatile("" : "+v"(e[i]));             // keeps the instruction in its slot
          }
          // conversion and sum of the pairs finished one half-step ago
          constexpr int A0 = C == C0 ? 0 : 16 * (C - C0 - 1) / NC / 2, A1 = C == C0 ? 0 : B0 / 2;
#pragma unroll
          for (int i = A0; i < A1; ++i) {
            fold(i);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&](auto i_) {
      constexpr int I = decltype(i_)::value;
      constexpr int PER = 2 + (WS ? 1 : 0), PERN = 2 + (NS ? 1 : 0);       // reads per step: this phase, the next
      constexpr int N1 = I + 1 < NST ? PER : (NX ? PERN : 0), N2 = I + 2 < NST ? PER : (NX ? PERN : 0);
      if constexpr (I + 2 < NST) read_step(odd_, ws_, IntC<1>{}, IntC<I + 2>{}, dk, dv);
      else if constexpr (NX) read_step(IntC<1 - ODD>{}, ns_, IntC<1>{}, IntC<I + 2 - NST>{}, dk, dv);
      att_wait<N1 + N2>();
      if constexpr (WS) {
        asm volatile("" : "+v"(kf[I & 3]));
        if constexpr (I == 0) {
          f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0], z, 0, 0, 0);
        } else {
          sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[I & 3], qf[I], sn, 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      vec(IntC<2 * I>{});
      asm volatile("" : "+v"(vf[I & 3].s[0]), "+v"(vf[I & 3].s[1]));
      oacc[I % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[I & 3].b, pp[I / DB].b, oacc[I % DB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      vec(IntC<2 * I + 1>{});
      // the loads of this iteration ride along in the even phase
      if constexpr (!ODD && SM && (I & 1)) {
        constexpr int L = I / 2;                       // NST / 2 = 2 LPT slots (DH = 128: 4, DH = 64: 2)
        if constexpr (L < LPT) issue(t + 3, L, false);
        else if constexpr (L < 2 * LPT) issue(t + 2, L - LPT, true);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    step(IntC<0>{}); step(IntC<1>{}); step(IntC<2>{}); step(IntC<3>{});
    if constexpr (NST == 8) { step(IntC<4>{}); step(IntC<5>{}); step(IntC<6>{}); step(IntC<7>{}); }
    if constexpr (SM) {
      constexpr int A0 = 16 * (2 * NST - 4) / (2 * NST - 3) / 2;           // pairs of the last half-step
#pragma unroll
      for (int i = A0; i < 8; ++i) {
        fold(i);
      }
      if (moved) {
        row_sum *= alpha;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[d][i] *= alpha;
      }
      row_sum += psum;
    }
  };
  // byte step from the stage of tile t to the stage of tile t + 1
  auto stage_step = [&](int t) { return (t & (ATT_S - 1)) == ATT_S - 1 ? -(ATT_S - 1) * TILEB : TILEB; };

  // ---- S of the first sub-tile ----
  att_vm_wait<4 * LPT>();                  // K(t_begin) landed
  asm volatile("s_barrier" ::: "memory");
  if (t_begin <= t_last) {
    att_read_k<0>(kf[0], k_addr[0]);
    att_read_k<0>(kf[1], k_addr[1]);
    auto sstep = [&](auto i_) {
      constexpr int I = decltype(i_)::value;
      if constexpr (I + 2 < NST) att_read_k<0>(kf[(I + 2) & 3], k_addr[I + 2]);
      att_wait<(I + 2 < NST ? 2 : I + 1 < NST ? 1 : 0)>();
      asm volatile("" : "+v"(kf[I & 3]));
      if constexpr (I == 0) {
        f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0], z, 0, 0, 0);
      } else {
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[I & 3], qf[I], sacc[0], 0, 0, 0);
      }
    };
    sstep(IntC<0>{}); sstep(IntC<1>{}); sstep(IntC<2>{}); sstep(IntC<3>{});
    if constexpr (NST == 8) { sstep(IntC<4>{}); sstep(IntC<5>{}); sstep(IntC<6>{}); sstep(IntC<7>{}); }
  }
  // iteration t begins once K(t + 1) and V(t) have landed everywhere
  att_vm_wait<2 * LPT>();
  asm volatile("s_barrier" ::: "memory");
  int t = t_begin;
  if (t_begin <= t_last) {
    // nothing was requested by a phase before; V(t_begin) stands in for V(t_begin - 1), its P is zero
    read_step(IntC<0>{}, IntC<1>{}, IntC<1>{}, IntC<0>{}, 0, 0);
    read_step(IntC<0>{}, IntC<1>{}, IntC<1>{}, IntC<1>{}, 0, 0);
    int dv = 0;
    for (; t < t_last; ++t) {
      const int dk = stage_step(t);
      phase(IntC<0>{}, IntC<1>{}, IntC<1>{}, IntC<1>{}, IntC<1>{}, t, dk, dv);
      phase(IntC<1>{}, IntC<1>{}, IntC<1>{}, IntC<1>{}, IntC<1>{}, t, dk, dv);
      dv = dk;
      att_vm_wait<2 * LPT>();
      asm volatile("s_barrier" ::: "memory");
    }
    phase(IntC<0>{}, IntC<1>{}, IntC<1>{}, IntC<0>{}, IntC<1>{}, t, 0, dv);
    phase(IntC<1>{}, IntC<1>{}, IntC<0>{}, IntC<0>{}, IntC<1>{}, t, 0, dv);
    phase(IntC<0>{}, IntC<0>{}, IntC<0>{}, IntC<0>{}, IntC<0>{}, t, 0, 0);     // O += V P of the last sub-tile
    if (++t < n_tiles) {
      att_vm_wait<2 * LPT>();
      asm volatile("s_barrier" ::: "memory");
    }
  }
  // the rest of the piece lies in this wavefront's future: it only takes part in the loads
  for (; t < n_tiles; ++t) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) issue(t + 3, i, false);
#pragma unroll
    for (int i = 0; i < LPT; ++i) issue(t + 2, i, true);
    if (t + 1 < n_tiles) {
      att_vm_wait<2 * LPT>();
      asm volatile("s_barrier" ::: "memory");
    }
  }
  att_vm_wait<0>();                        // drain the clamped tail loads before the workgroup ends
  if (gridDim.z > 1) {
    // ---- partial results: O (un-normalised), reference and sum per (kv head, query, split) ----
    const float tot = row_sum + __shfl_xor(row_sum, 32, 64);
    if (!valid) return;
    const int m = m_pad + wave * 32 + ln;
    const size_t slot = ((size_t)kvh * n_flat_pad + m) * gridDim.z + blockIdx.z;
    if (h == 0) {
      part_ml[slot * 2] = ref * scale_log2e;
      part_ml[slot * 2 + 1] = tot;
    }
    float *dst = part_o + slot * DH;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *reinterpret_cast<float4 *>(dst + d * 32 + a * 8 + h * 4) =
            make_float4(oacc[d][a * 4 + 0], oacc[d][a * 4 + 1], oacc[d][a * 4 + 2], oacc[d][a * 4 + 3]);
    return;
  }
  // ---- normalise and store ----
  const float tot = row_sum + __shfl_xor(row_sum, 32, 64);
  const float inv = 1.f / tot;
  if (!valid) return;
  bf16 *dst = o + q_off;
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      bf16x4 w = {(bf16)(oacc[d][a * 4 + 0] * inv), (bf16)(oacc[d][a * 4 + 1] * inv),
                  (bf16)(oacc[d][a * 4 + 2] * inv), (bf16)(oacc[d][a * 4 + 3] * inv)};
      *reinterpret_cast<bf16x4 *>(dst + d * 32 + a * 8 + h * 4) = w;
    }
}

// Merge of the KV-split partials: o = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s over the
// splits that ran for the query's workgroup (those below its causal bound).
template <int DH>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float *__restrict__ part_o,
                                                         const float *__restrict__ part_ml,
                                                         const int32_t *__restrict__ q_pos, int n_rows,
                                                         bf16 *__restrict__ o, int n_q_heads,
                                                         int n_kv_heads, int n_splits, int split_tiles,
                                                         int wg_queries, const int32_t *__restrict__ wg_tiles,
                                                         int n_flat_pad, const int32_t *__restrict__ segs,
                                                         int n_segs) {
  constexpr int CG = DH / 4;                           // float4 channel groups per query
  const int g = n_q_heads / n_kv_heads;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)n_kv_heads * n_flat_pad * CG) return;
  const int c = (int)(idx % CG);
  const long qh = idx / CG;                            // kvh * n_flat_pad + padded query number
  const int m_pad = (int)(qh % n_flat_pad), kvh = (int)(qh / n_flat_pad);
  const int qwg = m_pad / wg_queries;
  int seg_qwg0 = 0, row0 = 0;
  if (segs) {
    int lo = 0, hi = n_segs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (segs[mid * kSegInts + kSegQwg] <= qwg) lo = mid; else hi = mid - 1;
    }
    const int32_t *sg = segs + lo * kSegInts;
    seg_qwg0 = sg[kSegQwg];
    row0 = sg[kSegOutOff];
    n_rows = sg[kSegKeep] + sg[kSegSuffix];
  }
  const int m = m_pad - seg_qwg0 * wg_queries;        // flattened query within its request
  if (m >= n_rows * g) return;                         // padding of the request's last workgroup
  const int n_tiles = wg_tiles[qwg];                 // key tiles of the query's workgroup
  const int ns = min(n_splits, (n_tiles + split_tiles - 1) / split_tiles);
  const float *ml = part_ml + qh * n_splits * 2;
  float mx = kNegBig;
  for (int s = 0; s < ns; ++s) mx = fmaxf(mx, ml[2 * s]);
  float den = 0.f;
  float4 acc = make_float4(0, 0, 0, 0);
  for (int s = 0; s < ns; ++s) {
    const float w = exp2f(ml[2 * s] - mx);
    den += w * ml[2 * s + 1];
    const float4 v = *reinterpret_cast<const float4 *>(part_o + (qh * n_splits + s) * DH + c * 4);
    acc.x += w * v.x; acc.y += w * v.y; acc.z += w * v.z; acc.w += w * v.w;
  }
  const float inv = 1.f / den;
  const int r = m / g, j = m - r * g;
  bf16x4 w4 = {(bf16)(acc.x * inv), (bf16)(acc.y * inv), (bf16)(acc.z * inv), (bf16)(acc.w * inv)};
  *reinterpret_cast<bf16x4 *>(o + ((size_t)(row0 + r) * n_q_heads + kvh * g + j) * DH + c * 4) = w4;
}

// ---------------------------------------------------------------------------
// float kernel, v_mfma_f32_16x16x4_f32.  One workgroup = one kv head x 16 flattened queries; its 8 wavefronts take
// the 32-key tiles in turn, each with its own running maximum, and are combined in LDS at the end in a fixed order.
// Transposed products as in the bf16 kernel: lane l holds query l % 16 and, of every 16-key block, keys 4 (l / 16) .. + 3;
// the contraction index a lane supplies in MFMA s is 4 (l / 16) + s for both products, so the K operand is one
// 16-byte load per 16 channels, the exponentiated scores are the second product's operand as they are, and the V operand
// is a coalesced 4-byte load.  K and V come straight from the cache (a float model's fits L2).
// Latency-bound: 544 rows of the 4 x 64 model 145 -> 14 us against one wavefront per row with vector FMAs.
// ---------------------------------------------------------------------------
constexpr int AF_NW = 8;
template <int DH>
__global__ __launch_bounds__(64 * AF_NW) void attn_f32_kernel(const float *__restrict__ q,
                                                       const int32_t *__restrict__ q_pos, int n_rows,
                                                       const float *__restrict__ kc,
                                                       const float *__restrict__ vc, float *__restrict__ o,
                                                       int n_q_heads, int n_kv_heads, float scale_log2e,
                                                       const int32_t *__restrict__ q_rows) {
  constexpr int NC = DH / 16;                          // 16-channel blocks
  __shared__ __attribute__((aligned(16))) float s_o[AF_NW][16][DH];
  __shared__ float s_max[AF_NW][16], s_sum[AF_NW][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 15, h = lane >> 4;
  const int g = n_q_heads / n_kv_heads, kvh = blockIdx.y, kv_dim = n_kv_heads * DH;
  const int n_flat = n_rows * g, m0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * 16;   // longest key ranges first
  const int m = min(m0 + ln, n_flat - 1), r = m / g, j = m - r * g;
  const int my_pos = q_pos[r];
  const float *qrow = q + ((size_t)(q_rows ? q_rows[r] : r) * n_q_heads + kvh * g + j) * DH;
  float4 qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) qf[c] = *reinterpret_cast<const float4 *>(qrow + 16 * c + 4 * h);
  int bound = my_pos, min_pos = my_pos;                // the 16 queries sit in lanes 0..15 of every group
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) {
    bound = max(bound, __shfl_xor(bound, off, 64));
    min_pos = min(min_pos, __shfl_xor(min_pos, off, 64));
  }
  const int kv_len = bound + 1, n_tiles = (kv_len + 31) / 32;

  f32x4 oacc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) oacc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float run_max = -INFINITY, run_sum = 0.f;
  for (int t = wave; t < n_tiles; t += AF_NW) {
    const int t0 = t * 32;
    f32x4 sc[2];
    float4 kf[2][NC];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float *krow = kc + (size_t)min(t0 + 16 * b + ln, kv_len - 1) * kv_dim + kvh * DH + 4 * h;
#pragma unroll
      for (int c = 0; c < NC; ++c) kf[b][c] = *reinterpret_cast<const float4 *>(krow + 16 * c);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) sc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][c].x, qf[c].x, sc[b], 0, 0, 0);
        sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][c].y, qf[c].y, sc[b], 0, 0, 0);
        sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][c].z, qf[c].z, sc[b], 0, 0, 0);
        sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][c].w, qf[c].w, sc[b], 0, 0, 0);
      }
    float mx = -INFINITY;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[b][i] = t0 + 16 * b + 4 * h + i <= my_pos ? sc[b][i] * scale_log2e : -INFINITY;
        mx = fmaxf(mx, sc[b][i]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float new_max = fmaxf(run_max, mx);
    const float ref = new_max == -INFINITY ? 0.f : new_max;       // no key of this query seen yet: every p is 0
    const float alpha = exp2f(run_max - ref);
    float psum = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[b][i] = exp2f(sc[b][i] - ref);
        psum += sc[b][i];
      }
    run_sum = run_sum * alpha + psum;                              // this lane group's keys only; combined at the end
    run_max = new_max;
#pragma unroll
    for (int c = 0; c < NC; ++c) oacc[c] *= alpha;
    float vf[2][4][NC];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float *vrow = vc + (size_t)min(t0 + 16 * b + 4 * h + i, kv_len - 1) * kv_dim + kvh * DH + ln;
#pragma unroll
        for (int c = 0; c < NC; ++c) vf[b][i][c] = vrow[16 * c];
      }
    // A query sees cache rows 0 .. its own position, but the product below multiplies every row of the tile, by 0 where it
    // lies past the position -- and 0 times a value that is not finite is not 0.  Only tiles with such a pair are looked at.
    bool bad = false;
    if (t0 + 31 > min_pos) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < NC; ++c) bad |= !(fabsf(vf[b][i][c]) < INFINITY);
    }
    if (__any(bad)) {
      // the same sums key by key, each query up to its own position; p of key 16 b + 4 j + i is held by lane group j
#pragma unroll 1
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float pk = __shfl(sc[b][i], 16 * j + ln, 64);
            const int key = t0 + 16 * b + 4 * j + i;
            const float *vrow = vc + (size_t)min(key, kv_len - 1) * kv_dim + kvh * DH + 4 * h;
            if (key <= my_pos) {
#pragma unroll
              for (int c = 0; c < NC; ++c) oacc[c] += pk * *reinterpret_cast<const f32x4 *>(vrow + 16 * c);
            }
          }
      continue;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) oacc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[b][i][c], sc[b][i], oacc[c], 0, 0, 0);
  }
  run_sum += __shfl_xor(run_sum, 16, 64);
  run_sum += __shfl_xor(run_sum, 32, 64);
  // lane l: channels 16 c + 4 (l / 16) .. + 3 of query l % 16
#pragma unroll
  for (int c = 0; c < NC; ++c) *reinterpret_cast<f32x4 *>(&s_o[wave][ln][16 * c + 4 * h]) = oacc[c];
  if (h == 0) { s_max[wave][ln] = run_max; s_sum[wave][ln] = run_sum; }
  __syncthreads();
  for (int e = tid; e < 16 * DH / 4; e += 64 * AF_NW) {
    const int qi = e / (DH / 4), ch = e % (DH / 4) * 4;
    if (m0 + qi >= n_flat) continue;
    float top = -INFINITY;
#pragma unroll
    for (int w = 0; w < AF_NW; ++w) top = fmaxf(top, s_max[w][qi]);
    float den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < AF_NW; ++w) {
      const float wt = exp2f(s_max[w][qi] - top);                  // 0 for a wavefront that saw no key of the query
      den += wt * s_sum[w][qi];
      acc += wt * *reinterpret_cast<const f32x4 *>(&s_o[w][qi][ch]);
    }
    const int mm = m0 + qi, rr = mm / g, jj = mm - rr * g;
    *reinterpret_cast<f32x4 *>(o + ((size_t)rr * n_q_heads + kvh * g + jj) * DH + ch) = acc / den;
  }
}

// Split plan of the bf16 kernel.  Few query workgroups (the selective layers) leave most CUs idle,
// so the key range is cut into pieces of split_tiles tiles handled by separate workgroups
// (workgroup z takes tiles [z*split_tiles, (z+1)*split_tiles) and exits when its own causal
// range ends before that).  Measured on 359..986-row layers: about one round of 256 workgroups
// in total is the optimum; more pieces cost more in partial results than they gain in balance.
// n_qwg: query workgroups per kv head.
static void attn_split_plan(long n_qwg, int hkv, int n_tokens, int *n_splits, int *split_tiles) {
  const long base = n_qwg * hkv;
  const int max_tiles = (n_tokens + BKV - 1) / BKV;
  int ns = 1;
  if (base < 128) {
    ns = (int)((256 + base - 1) / base);
    ns = std::min(ns, std::max(1, max_tiles / 4));
    ns = std::min(ns, 32);
  } else if (base < 256) {
    ns = std::min(2, std::max(1, max_tiles / 4));
  }
  *split_tiles = (max_tiles + ns - 1) / ns;
  *n_splits = (max_tiles + *split_tiles - 1) / *split_tiles;
}

static long query_workgroups(int n_rows, int hq, int hkv) {
  return ((long)n_rows * (hq / hkv) + ATT_WGQ - 1) / ATT_WGQ;
}

// scratch of a launch with n_qwg query workgroups per kv head and ns key-range pieces: partial O
// and (max, sum) pairs per (kv head, padded query, piece), and one key-tile count per query workgroup
static size_t attn_scratch_floats(long n_qwg, int hkv, int dh, int ns) {
  return (size_t)hkv * n_qwg * ATT_WGQ * ns * (dh + 2) + (size_t)n_qwg;
}

size_t attention_partial_floats(int dtype, int n_rows, int hq, int hkv, int dh, int n_tokens) {
  if (dtype == 0 || n_rows == 0) return 0;
  int ns, st;
  const long n_qwg = query_workgroups(n_rows, hq, hkv);
  attn_split_plan(n_qwg, hkv, n_tokens, &ns, &st);
  if (ns <= 1) return 0;
  return attn_scratch_floats(n_qwg, hkv, dh, ns);
}

// The same for ANY cache length: the piece count never exceeds what the row count alone allows.
size_t attention_partial_floats_bound(int dtype, int n_rows, int hq, int hkv, int dh) {
  if (dtype == 0 || n_rows == 0) return 0;
  const long n_qwg = query_workgroups(n_rows, hq, hkv);
  const long base = n_qwg * hkv;
  const int ns = base < 128 ? (int)std::min<long>(32, (256 + base - 1) / base) : (base < 256 ? 2 : 1);
  if (ns <= 1) return 0;
  return attn_scratch_floats(n_qwg, hkv, dh, ns);
}

long attention_query_workgroups(int n_rows, int hq, int hkv) { return query_workgroups(n_rows, hq, hkv); }

hipError_t launch_attention(int dtype, const void *q, const int32_t *q_rows, const int32_t *q_pos, int n_rows,
                            const void *kc, const void *vc, void *o, int hq, int hkv, int dh,
                            int n_tokens, float *partial, size_t partial_floats, hipStream_t s,
                            const int32_t *segs, int n_segs, long total_qwg) {
  if (n_rows == 0) return hipSuccess;
  const float scale_log2e = kLog2e / sqrtf((float)dh);
  if (dtype == 0) {
    if (segs) return hipErrorInvalidValue;           // the float kernel takes one request per launch
    const dim3 grid((unsigned)(((long)n_rows * (hq / hkv) + 15) / 16), hkv);
    if (dh == 64)
      hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(64 * AF_NW), 0, s, (const float *)q, q_pos, n_rows,
                         (const float *)kc, (const float *)vc, (float *)o, hq, hkv, scale_log2e, q_rows);
    else
      hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(64 * AF_NW), 0, s, (const float *)q, q_pos, n_rows,
                         (const float *)kc, (const float *)vc, (float *)o, hq, hkv, scale_log2e, q_rows);
    return hipGetLastError();
  }
  const long n_qwg = segs ? total_qwg : query_workgroups(n_rows, hq, hkv);
  int n_splits, split_tiles;
  attn_split_plan(n_qwg, hkv, n_tokens, &n_splits, &split_tiles);
  while (n_splits > 1 && (!partial || partial_floats < attn_scratch_floats(n_qwg, hkv, dh, n_splits))) {
    // scratch is short: fewer, longer pieces (down to one workgroup walking all keys)
    const int max_tiles = (n_tokens + BKV - 1) / BKV;
    const int ns = n_splits - 1;
    split_tiles = (max_tiles + ns - 1) / ns;
    n_splits = (max_tiles + split_tiles - 1) / split_tiles;
  }
  const int wgq = ATT_WGQ;
  const size_t slots = (size_t)hkv * n_qwg * ATT_WGQ * n_splits;
  float *part_o = partial;
  float *part_ml = partial ? partial + slots * dh : nullptr;
  int32_t *wg_tiles = partial ? reinterpret_cast<int32_t *>(part_ml + slots * 2) : nullptr;
#define CB_ATTN(DH_)                                                                                \
  do {                                                                                              \
    constexpr int smem = 2 * ATT_S * BKV * DH_ * 2;                                                 \
    static std::once_flag once_;                                                                    \
    std::call_once(once_, [] {                                                                      \
      (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_bf16_kernel<DH_>),             \
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem);                  \
    });                                                                                             \
    hipLaunchKernelGGL((attn_bf16_kernel<DH_>), dim3(hkv, (unsigned)n_qwg, n_splits),               \
                       dim3(64 * ATT_NW), smem, s, (const bf16 *)q, q_pos, n_rows, (const bf16 *)kc, \
                       (const bf16 *)vc, (bf16 *)o, hq, hkv, scale_log2e, split_tiles, part_o,      \
                       part_ml, q_rows, wg_tiles, segs, n_segs);                                    \
  } while (0)
  if (dh == 64) CB_ATTN(64);
  else CB_ATTN(128);
#undef CB_ATTN
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || n_splits == 1) return e;
  const int n_flat_pad = (int)n_qwg * ATT_WGQ;
  const long total = (long)hkv * n_flat_pad * (dh / 4);
  const dim3 mgrid((unsigned)((total + 255) / 256));
  if (dh == 64)
    hipLaunchKernelGGL(attn_merge_kernel<64>, mgrid, dim3(256), 0, s, part_o, part_ml, q_pos, n_rows,
                       (bf16 *)o, hq, hkv, n_splits, split_tiles, wgq, wg_tiles, n_flat_pad, segs, n_segs);
  else
    hipLaunchKernelGGL(attn_merge_kernel<128>, mgrid, dim3(256), 0, s, part_o, part_ml, q_pos, n_rows,
                       (bf16 *)o, hq, hkv, n_splits, split_tiles, wgq, wg_tiles, n_flat_pad, segs, n_segs);
  return hipGetLastError();
}

}  // namespace cb
