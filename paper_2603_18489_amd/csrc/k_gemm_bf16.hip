// bf16 GEMMs on MFMA with the layer's element-wise work fused into their epilogues.
//
// C[M,N] = A[M,K] W[N,K]^T with fp32 accumulation.  Both operands arrive re-tiled into 16x32
// fragments (k_common.h), so every wave-wide operand load is one contiguous, fully coalesced KiB.
// The weight fragment is the MFMA "A" operand (16 weight rows) and the activation fragment the
// "B" operand (16 activation rows): a lane of the 16x16 result holds 4 consecutive output
// features n of one activation row m.
//
// RMSNorm is folded in: the A operand of a GEMM that follows a norm holds bf16(h * gain), NOT
// normalised, and the row's 1/rms is applied to the fp32 accumulator in the epilogue (it is a
// per-row scalar, so it commutes with the contraction).  The sum of squares of each row of h is
// accumulated by the producing epilogue with integer (44.20 fixed-point) atomics, which are
// order-independent and therefore bit-reproducible.
//
// Epilogues (template parameter EPI):
//   EPI_QKV    x 1/rms, rotary embedding on q and k (a weight tile holds 8 columns of a head
//              and their 8 partners hd/2 further on, so a rotation pair meets in lanes l and
//              l + 32), q -> query buffer, k / v -> the packed KV cache rows of the row's position
//   EPI_RESID  h += result; writes bf16(h * next gain) as the next GEMM's operand and adds the
//              row's sum of squares
//   EPI_SWIGLU x 1/rms, silu(gate) * up (8 gate rows and their 8 up rows share a tile), -> packed
//              activations
//   EPI_LOGITS x 1/rms x logit scale -> fp32 logits; the skinny kernel also reduces its block's
//              columns to one (max, argmax, sum e, sum e (z - max)) tuple per row - the
//              vocabulary reduction of Eq. 1 fused behind the LM head - and stores the logits
//              themselves only on request
//
// Kernels:
//   skinny (M <= 96): weight streaming.  A block of KS waves owns NTW weight tiles and splits K
//     across its waves; each weight byte is read from HBM exactly once while the small
//     activation fragments come from L2.  The KS partial tiles are summed in LDS in a fixed
//     order, then the epilogue runs on the sums.
//   tiled (M > 96): block tile chosen per shape so that the grid fills the 256 CUs.  4 waves
//     (residual products): LDS double buffer fed through four register sets.  8 waves (192x128 .. 192x384, 256x256): operands
//     loaded from global memory directly into an LDS ring of four k-steps.
#include "ec_internal.h"
#include "k_meet.h"
#include "k_vtuple.h"

namespace ec {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 v4_as_bf16x8(u32x4 v) {
  union { u32x4 u; bf16x8 b; } c;
  c.u = v;
  return c.b;
}
// 8 e4m3 codes (two dwords, lowest byte first) -> 8 bf16 values, exactly (every e4m3 value is a
// bf16 value): four v_cvt_scalef32_pk_bf16_fp8 with scale 1
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16x8 e4m3x8_as_bf16x8(uint32_t a, uint32_t b) {
  union { bf16x2_t h[4]; bf16x8 v; } c;
  c.h[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a, 1.0f, false);
  c.h[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a, 1.0f, true);
  c.h[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(b, 1.0f, false);
  c.h[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(b, 1.0f, true);
  return c.v;
}
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ uint32_t pack2(float a, float b) { return pack2_bf16(a, b); }
// x * sigmoid(x) with the hardware exp2 and reciprocal (about 1 ulp each; the result is rounded
// to bf16 anyway).  exp overflow gives rcp(inf) = 0, the right limit.
__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x));
}

__device__ __forceinline__ float rstd_from_sum(const GemmEpi& e, unsigned long long fx) {
  double ss = sumsq_from_fixed(fx);
  return 1.0f / sqrtf((float)(ss / (double)e.d_in) + e.eps);
}
// ---- epilogues on one lane's values -----------------------------------------------------------
// (m: activation row, < M;  vt: virtual weight tile;  q4: lane>>4, so the lane's 4 values are
// output features vt*16 + q4*4 + 0..3.)

__device__ __forceinline__ void epi_logits(const GemmEpi& e, int m, int vt, int q4, f32x4 v,
                                           float rs) {
  float s = rs * e.scale;
  float4 o = make_float4(v[0] * s, v[1] * s, v[2] * s, v[3] * s);
  *(float4*)(e.logits + (size_t)m * e.ldc + vt * 16 + q4 * 4) = o;
}

// returns the lane's contribution to the row's sum of squares
__device__ __forceinline__ float epi_resid(const GemmEpi& e, int m, int vt, int q4, f32x4 v) {
  int n = vt * 16 + q4 * 4;
  float4* hp = (float4*)(e.h + (size_t)m * e.d + n);
  float4 h = *hp;
  h.x += v[0]; h.y += v[1]; h.z += v[2]; h.w += v[3];
  *hp = h;
  const bf16_t* g = e.gain_next + n;
  u32x2 pk;
  pk[0] = pack2(h.x * bf16_to_f32(g[0]), h.y * bf16_to_f32(g[1]));
  pk[1] = pack2(h.z * bf16_to_f32(g[2]), h.w * bf16_to_f32(g[3]));
  *(u32x2*)(e.a_next + packed_act_index(m, n, e.MT)) = pk;
  return h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w;
}

// epi_resid with h and the gains already in registers (fetched at kernel start)
__device__ __forceinline__ float epi_resid_pre(const GemmEpi& e, int m, int vt, int q4, f32x4 v,
                                               float4 h, u32x2 g4) {
  int n = vt * 16 + q4 * 4;
  h.x += v[0]; h.y += v[1]; h.z += v[2]; h.w += v[3];
  *(float4*)(e.h + (size_t)m * e.d + n) = h;
  u32x2 pk;
  pk[0] = pack2(h.x * __uint_as_float(g4[0] << 16), h.y * __uint_as_float(g4[0] & 0xffff0000u));
  pk[1] = pack2(h.z * __uint_as_float(g4[1] << 16), h.w * __uint_as_float(g4[1] & 0xffff0000u));
  *(u32x2*)(e.a_next + packed_act_index(m, n, e.MT)) = pk;
  return h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w;
}

__device__ __forceinline__ void epi_add_sumsq(const GemmEpi& e, int m, bool valid, float part) {
  // the 4 lanes l, l^16, l^32, l^48 hold the same row
  part += __shfl_xor(part, 16, 64);
  part += __shfl_xor(part, 32, 64);
  if (valid && (threadIdx.x & 63) < 16) {
    unsigned long long fx = sumsq_to_fixed(part, e.sum_cap);
    const int slot = blockIdx.x & (kSumSlots - 1);
    // (the padding rows of the row list are all zeros: nothing to add)
    if (fx) atomicAdd((unsigned long long*)(e.sumsq_out + (size_t)slot * e.sum_stride + m), fx);
  }
}

// Tile p of the interleaved matrix holds gate rows 8p..8p+7 in its rows 0-7 and the matching up
// rows in rows 8-15: lanes with q4 < 2 hold gates, their partners 32 lanes up hold the ups.
// (Lanes l and l^32 share the activation row, so a row-validity condition around the call keeps
// both or neither.)
__device__ __forceinline__ void epi_swiglu(const GemmEpi& e, int m, int p, int q4, f32x4 v,
                                           float rs) {
  float o[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = other_half(v[r]);
  if (q4 < 2) {
    u32x2 pk;
    pk[0] = pack2(silu_f(v[0] * rs) * (o[0] * rs), silu_f(v[1] * rs) * (o[1] * rs));
    pk[1] = pack2(silu_f(v[2] * rs) * (o[2] * rs), silu_f(v[3] * rs) * (o[3] * rs));
    *(u32x2*)(e.act + packed_act_index(m, p * 8 + q4 * 4, e.MT)) = pk;
  }
}

// Tiles p and p+1 at once, so that every lane has an activation to compute: lanes with q4 < 2
// finish tile p (own gates, partners' ups), the others tile p+1 (partners' gates, own ups).
__device__ __forceinline__ void epi_swiglu2(const GemmEpi& e, int m, int p, int q4, f32x4 va,
                                            f32x4 vb, float rs) {
  const bool lo = q4 < 2;
  u32x2 pk;
  float a[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float got = other_half(lo ? vb[r] : va[r]);
    float g = lo ? va[r] : got, u = lo ? got : vb[r];
    a[r] = silu_f(g * rs) * (u * rs);
  }
  pk[0] = pack2(a[0], a[1]); pk[1] = pack2(a[2], a[3]);
  *(u32x2*)(e.act + packed_act_index(m, (lo ? p : p + 1) * 8 + (q4 & 1) * 4, e.MT)) = pk;
}

// Virtual tile vt of the [q | k | v] matrix.  In the q and k regions tile w of a head holds the
// head's columns 8w..8w+7 in rows 0-7 and their rotary partners (hd/2 columns later) in rows
// 8-15, so a lane and its partner 32 lanes away hold one rotation pair; in the v region the
// tiles are in natural order.
__device__ __forceinline__ void epi_qkv(const GemmEpi& e, int m, int vt, int q4, f32x4 v,
                                        float rs) {
  const int hd = e.hd, tph = hd >> 4;  // tiles per head
  const int nqt = e.Hq * tph, nkt = e.Hkv * tph;
  const int4 ri = e.rowinfo[m];  // position, -, cache offset, keys per slab
  const int pos = ri.x;
  if (vt < nqt + nkt) {
    float o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = other_half(v[r]);
    if (pos < 0) return;  // padding row (its partner lane has the same row)
    const bool is_q = vt < nqt, hi = q4 >= 2;
    const int t = is_q ? vt : vt - nqt;
    const int head = t / tph, j = (t % tph) * 8 + (q4 & 1) * 4;  // column within the half head
    const float2* cs = e.cs + (size_t)pos * (hd >> 1) + j;
    float out[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = v[r] * rs, y = o[r] * rs;
      float2 c = cs[r];
      out[r] = hi ? x * c.x + y * c.y : x * c.x - y * c.y;
    }
    u32x2 pk;
    pk[0] = pack2(out[0], out[1]); pk[1] = pack2(out[2], out[3]);
    const int col = j + (hi ? hd >> 1 : 0);
    if (is_q) {
      *(u32x2*)(e.q_out + (size_t)m * (e.Hq * hd) + head * hd + col) = pk;
    } else {
      bf16_t* slab = e.kc + ri.z + (size_t)head * ri.w * hd;
      *(u32x2*)(slab + kcache_index(pos, col, hd)) = pk;
    }
  } else if (pos >= 0) {
    const int t = vt - nqt - nkt;
    const int head = t / tph, c0 = (t % tph) * 16 + q4 * 4;
    bf16_t* slab = e.vc + ri.z + (size_t)head * ri.w * hd;
#pragma unroll
    for (int r = 0; r < 4; ++r) slab[vcache_index(pos, c0 + r, ri.w)] = f32_to_bf16(v[r] * rs);
  }
}

// ---------------------------------------------------------------------------------------------
// skinny: grid = ceil(n-tiles / NTW) blocks of KS*64 threads
// ---------------------------------------------------------------------------------------------
// W8: the weights are e4m3 codes (k_common.h: packed_w8_index), one 1 KiB fragment pair covering
// 64 k per weight tile and k-step; a lane's 16 bytes are turned into two bf16 MFMA operands in
// registers (exact), so a k-step is two MFMAs per (weight tile, m-tile) on two activation
// fragments, KB counts 64-wide steps, and the per-row scales multiply the K-reduced sums.
// The LM head of up to 32 rows keeps to 256 registers, with one k-step to a register set: two blocks to a compute unit, one
// streaming while the other is in its epilogue.  (8 tiles with two steps to a set take 264 and run alone, four rounds of
// blocks one after the other.)  us by events: 32 rows, 4096 -> 126464 186 -> 179; 3584 -> 152064 207 -> 195.
constexpr int skinny_waves(int epi, int MT) { return epi == EPI_LOGITS && MT <= 2 ? 2 : 1; }
template <int EPI, int MT, int NTW, int KS, int U, bool W8 = false>
__global__ __launch_bounds__(KS * 64, skinny_waves(EPI, MT)) void gemm_bf16_skinny_kernel(const u32x4* __restrict__ Ap,
                                                                   const u32x4* __restrict__ Wp,
                                                                   int total_nt, int KB,
                                                                   int MT_src, GemmEpi e) {
  constexpr int AW = W8 ? 2 : 1;   // activation fragments per k-step
  extern __shared__ float4 red[];  // [KS][NTW*MT][64]
  // the wave index is made a scalar so that everything derived from it (the K slice) is
  // provably wave-uniform: MFMA ignores the EXEC mask, so it must never sit under a condition
  // the compiler could treat as divergent
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt0 = blockIdx.x * NTW;
  // EPI_PARTIAL: blockIdx.y picks one of gridDim.y contiguous K ranges.  (The others are not charged the
  // division and the load of the grid's size ahead of their first operand: about 0.4 us a launch.)
  int kr_lo = 0, kr_n = KB;
  if constexpr (EPI == EPI_PARTIAL) {
    kr_lo = (int)((blockIdx.y * KB) / gridDim.y);
    kr_n = (int)(((blockIdx.y + 1) * KB) / gridDim.y) - kr_lo;
  }
  const int kb_lo = kr_lo + (wave * kr_n) / KS, kb_hi = kr_lo + ((wave + 1) * kr_n) / KS;

  // a tile past the end streams tile 0 instead (valid memory) and is dropped at the store
  const int grp = e.w_grp;
  const u32x4* wp[NTW];
#pragma unroll
  for (int i = 0; i < NTW; ++i) {
    int nt = nt0 + i < total_nt ? nt0 + i : 0;
    wp[i] = Wp + packed_w_frag(nt, kb_lo, KB, grp) * 64 + lane;
  }
  const size_t wstep = (size_t)grp * 64;  // u32x4 per k-step
  // activation rows may be gathered (LM head: only the block's masked rows)
  const u32x4* ap[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    int m = j * 16 + (lane & 15);
    int row = m < e.M ? m : 0;
    if constexpr (EPI == EPI_LOGITS) row = (m < e.M && e.row_sel) ? e.row_sel[m] : row;
    ap[j] = Ap + ((size_t)kb_lo * AW * MT_src + (row >> 4)) * 64 + (lane >> 4) * 16 + (row & 15);
  }

  constexpr bool NORMED = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LOGITS);
  float* rstd_s = (float*)(red + KS * NTW * MT * 64);  // [MT*16]: 1/rms of the block's rows

  f32x4 acc[NTW][MT];
#pragma unroll
  for (int i = 0; i < NTW; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // Two register sets of U k-steps each (U is a template parameter): while one set feeds the
  // MFMAs the other set's loads are in flight, so a wave always has up to 2*U*(NTW+MT) KiB
  // outstanding.  Every load is issued unconditionally (straight-line code lets the compiler
  // count outstanding loads exactly): k-steps past the slice re-read the slice's last fragments,
  // which are still in cache, and their activation operand is replaced by zeros, so the MFMAs,
  // which ignore EXEC and must run unconditionally anyway, add nothing.
  // The weights are loaded with the non-temporal hint: every byte of them is used once, and kept
  // out of the way they leave the L2 to the activation fragments that all blocks re-read
  // (measured: the whole partial step 3.31 -> 3.11 ms).
  const int nkb = kb_hi - kb_lo;
  const int last = nkb > 0 ? nkb - 1 : 0;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  u32x4 wa[U][NTW], aa[U][MT * AW], wb[U][NTW], ab[U][MT * AW];
#define EC_SK_LOAD(WSET, ASET, IT0)                                                        \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                          \
    const int it_ = (IT0) + u < last ? (IT0) + u : last;                                   \
    _Pragma("unroll") for (int i = 0; i < NTW; ++i) WSET[u][i] = __builtin_nontemporal_load(&wp[i][(size_t)it_ * wstep]);  \
    _Pragma("unroll") for (int j = 0; j < MT; ++j)                                         \
      _Pragma("unroll") for (int h = 0; h < AW; ++h)                                       \
        ASET[u][j * AW + h] = ap[j][((size_t)it_ * AW + h) * MT_src * 64];                 \
  }
#define EC_SK_ZERO_TAIL(ASET, IT0)                                                         \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                          \
    const bool in_ = (IT0) + u < nkb;                                                      \
    _Pragma("unroll") for (int j = 0; j < MT * AW; ++j) ASET[u][j] = in_ ? ASET[u][j] : zero4;  \
  }
#define EC_SK_MMA(WSET, ASET)                                                              \
  _Pragma("unroll") for (int u = 0; u < U; ++u)                                            \
    _Pragma("unroll") for (int i = 0; i < NTW; ++i) {                                      \
      if constexpr (W8) {                                                                  \
        const bf16x8 lo_ = e4m3x8_as_bf16x8(WSET[u][i][0], WSET[u][i][1]);                 \
        const bf16x8 hi_ = e4m3x8_as_bf16x8(WSET[u][i][2], WSET[u][i][3]);                 \
        _Pragma("unroll") for (int j = 0; j < MT; ++j) {                                   \
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                             \
              lo_, v4_as_bf16x8(ASET[u][j * AW]), acc[i][j], 0, 0, 0);                     \
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                             \
              hi_, v4_as_bf16x8(ASET[u][j * AW + AW - 1]), acc[i][j], 0, 0, 0);            \
        }                                                                                  \
      } else {                                                                             \
        _Pragma("unroll") for (int j = 0; j < MT; ++j)                                     \
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                             \
              v4_as_bf16x8(WSET[u][i]), v4_as_bf16x8(ASET[u][j]), acc[i][j], 0, 0, 0);     \
      }                                                                                    \
    }
  EC_SK_LOAD(wa, aa, 0)
  // The rows' sum-of-squares counters are fetched behind the first operand loads and turned
  // into 1/rms after the main loop, so neither the loop nor the epilogue waits on them.  All
  // threads load (those without a row of their own read row 0): no branch, so the compiler
  // still counts outstanding loads exactly.
  // Epilogue operands of the thread's first output unit are fetched here too: the residual
  // stream and gains (EPI_RESID) so that the epilogue does not start with a round trip to memory.
  constexpr int UNITS = NTW * MT * 64;  // whole waves: the wave's 64 lanes share (tile, m-tile)
  float4 pre_h = make_float4(0.f, 0.f, 0.f, 0.f);
  u32x2 pre_g = {0u, 0u};
  if constexpr (EPI == EPI_RESID) {
    const int o = threadIdx.x < UNITS ? threadIdx.x : 0;
    const int l = o & 63, unit = o >> 6, iu = unit / MT, j = unit - iu * MT;
    const int m = j * 16 + (l & 15), vt = nt0 + iu;
    const int mm = m < e.M ? m : 0, n = (vt < total_nt ? vt : 0) * 16 + (l >> 4) * 4;
    pre_h = *(const float4*)(e.h + (size_t)mm * e.d + n);
    pre_g = *(const u32x2*)(e.gain_next + n);
  }
  // W8: the block's per-row weight scales, fetched here and parked in LDS behind the main loop
  float* wsc_s = rstd_s + MT * 16 + (EPI == EPI_LOGITS ? NTW * MT * 16 * 4 : 0);  // [NTW*16]
  float wsc_reg = 1.f;
  if constexpr (W8) {
    const int n_ = nt0 * 16 + (int)threadIdx.x;
    wsc_reg = e.wscale[(threadIdx.x < NTW * 16 && n_ < total_nt * 16) ? n_ : 0];
  }
  unsigned long long ssq[kSumSlots];
  if constexpr (NORMED) {
#pragma unroll
    for (int sl = 0; sl < kSumSlots; ++sl) ssq[sl] = 0;
    __builtin_amdgcn_sched_barrier(0);
    if (threadIdx.x < MT * 16) {
      int row = (int)threadIdx.x < e.M ? (int)threadIdx.x : 0;
      if constexpr (EPI == EPI_LOGITS) row = (e.row_sel && (int)threadIdx.x < e.M) ? e.row_sel[row] : row;
#pragma unroll
      for (int sl = 0; sl < kSumSlots; ++sl) ssq[sl] = e.sumsq_in[(size_t)sl * e.sum_stride + row];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // (the scheduling barriers keep the compiler from sinking a set's loads down to their first
  // use, which would leave nothing in flight during the MFMAs)
  int it0 = 0;
  for (; it0 + 2 * U < nkb; it0 += 2 * U) {
    EC_SK_LOAD(wb, ab, it0 + U)
    __builtin_amdgcn_sched_barrier(0);
    EC_SK_MMA(wa, aa)
    __builtin_amdgcn_sched_barrier(0);
    EC_SK_LOAD(wa, aa, it0 + 2 * U)
    __builtin_amdgcn_sched_barrier(0);
    EC_SK_MMA(wb, ab)
    __builtin_amdgcn_sched_barrier(0);
  }
  // last 1 .. 2U k-steps: nothing left to prefetch; only here can a k-step lie past the slice
  EC_SK_LOAD(wb, ab, it0 + U)
  __builtin_amdgcn_sched_barrier(0);
  EC_SK_ZERO_TAIL(aa, it0)
  EC_SK_MMA(wa, aa)
  EC_SK_ZERO_TAIL(ab, it0 + U)
  EC_SK_MMA(wb, ab)
#undef EC_SK_ZERO_TAIL
#undef EC_SK_LOAD
#undef EC_SK_MMA

  // fixed-order reduction over the KS waves
#pragma unroll
  for (int i = 0; i < NTW; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      f32x4 v = acc[i][j];
      red[(wave * NTW * MT + i * MT + j) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
    }
  if constexpr (NORMED) {
    unsigned long long fx = 0;
#pragma unroll
    for (int sl = 0; sl < kSumSlots; ++sl) {
      // keeps the compiler from adding the counters up (and waiting for them) before the loop
      asm volatile("" : "+v"(ssq[sl]));
      fx = sumsq_add(fx, ssq[sl]);
    }
    if (threadIdx.x < MT * 16) rstd_s[threadIdx.x] = rstd_from_sum(e, fx);
  }
  if constexpr (W8) {
    if (threadIdx.x < NTW * 16) wsc_s[threadIdx.x] = wsc_reg;
  }
  __syncthreads();

  // sum over the KS waves of the lane's 4 output features of weight tile iu (times their scales)
  auto ksum = [&](int idx, int iu, int q4) {
    float4 s = red[idx];
#pragma unroll
    for (int w = 1; w < KS; ++w) {
      float4 v = red[w * NTW * MT * 64 + idx];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    if constexpr (W8) {
      const float4 c = *(const float4*)(wsc_s + iu * 16 + q4 * 4);
      s.x *= c.x; s.y *= c.y; s.z *= c.z; s.w *= c.w;
    }
    return (f32x4){s.x, s.y, s.z, s.w};
  };

  if constexpr (EPI == EPI_LOGITS) {
    // Logits of the block's NTW*16 columns, and their reduction.  A row's 16 columns of one tile
    // sit in the 4 lanes l, l^16, l^32, l^48 (4 columns each): maximum and lowest index holding
    // it through two lane swaps, then sum e^(z-max) and sum e^(z-max)(z-max) relative to that
    // maximum (added pairwise, the same pairs in all four lanes, so they agree bit for bit);
    // after a barrier a row's NTW tuples are merged by as many lanes into the block's.
    float4* tup = (float4*)(rstd_s + MT * 16);  // [NTW][MT*16]
    for (int o = threadIdx.x; o < UNITS; o += KS * 64) {  // (UNITS is a multiple of the wave)
      const int l = o & 63, unit = o >> 6, iu = unit / MT, j = unit - iu * MT;
      const int m = j * 16 + (l & 15), q4 = l >> 4, vt = nt0 + iu;
      const f32x4 v = ksum((iu * MT + j) * 64 + l, iu, q4);
      // (rows past M recompute row 0 and tiles past the end tile 0: finite values, dropped below)
      const float sc = rstd_s[m] * e.scale;
      const float z[4] = {v[0] * sc, v[1] * sc, v[2] * sc, v[3] * sc};
      const int n = vt * 16 + q4 * 4;
      const bool live = m < e.M && vt < total_nt;
      if (live && e.logits)
        *(float4*)(e.logits + (size_t)m * e.ldc + n) = make_float4(z[0], z[1], z[2], z[3]);
      float mx = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
      mx = fmaxf(mx, other_row(mx));
      mx = fmaxf(mx, other_half(mx));
      int idx = z[0] == mx ? n : z[1] == mx ? n + 1 : z[2] == mx ? n + 2 : z[3] == mx ? n + 3 : INT_MAX;
      idx = min(idx, __float_as_int(other_row(__int_as_float(idx))));
      idx = min(idx, __float_as_int(other_half(__int_as_float(idx))));
      float s4 = 0.f, t4 = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float d = z[r] - mx, ex = __expf(d);
        s4 += ex;
        t4 += ex * d;
      }
      s4 += other_row(s4); t4 += other_row(t4);
      s4 += other_half(s4); t4 += other_half(t4);
      if (q4 == 0)
        tup[iu * (MT * 16) + m] = vt < total_nt ? make_float4(mx, __int_as_float(idx), s4, t4)
                                                : vt_pack(vt_identity());
    }
    __syncthreads();
    // (a lane for every tuple; a row's are neighbours and NTW divides the lanes there are - a multiple of 64, or 32 with one
    // row tile and two weight tiles - so they are there together)
    for (int o = threadIdx.x; o < MT * 16 * NTW; o += KS * 64) {
      const int m = o / NTW;
      const VTuple t = vt_merge_lanes<NTW>(vt_unpack(tup[o % NTW * (MT * 16) + m]));
      if (o % NTW == 0 && m < e.M) e.vparts[(size_t)m * gridDim.x + blockIdx.x] = vt_pack(t);
    }
    return;
  }
  for (int o = threadIdx.x; o < UNITS; o += KS * 64) {
    const int l = o & 63, unit = o >> 6, iu = unit / MT, j = unit - iu * MT;
    const int m = j * 16 + (l & 15), q4 = l >> 4;
    const bool mvalid = m < e.M;
    const int vt = nt0 + iu;
    f32x4 v = ksum((iu * MT + j) * 64 + l, iu, q4);
    if constexpr (EPI == EPI_RESID) {
      float part = 0.f;
      if (mvalid && vt < total_nt)
        part = o < KS * 64 ? epi_resid_pre(e, m, vt, q4, v, pre_h, pre_g) : epi_resid(e, m, vt, q4, v);
      epi_add_sumsq(e, m, mvalid, part);
    } else if (mvalid && vt < total_nt) {
      if constexpr (EPI == EPI_PARTIAL)
        *(float4*)(e.partial + ((size_t)blockIdx.y * e.M + m) * e.d + vt * 16 + q4 * 4) =
            make_float4(v[0], v[1], v[2], v[3]);
      else if constexpr (EPI == EPI_SWIGLU) epi_swiglu(e, m, vt, q4, v, rstd_s[m]);
      else epi_qkv(e, m, vt, q4, v, rstd_s[m]);
    }
  }
}

constexpr int kSkinnySplit = 4;   // K ranges of a split few-row residual GEMM

// Second half of such a GEMM: h += sum over the ranges (fixed order), then what EPI_RESID does: next
// operand bf16(h * gain) and the row's sum of squares.  Every load is requested before the first is used.
// (Blocks that meet as those of the tiled kernels do, k_meet.h, save the launch but end later one by one: the product and
// this kernel 23.6 us, with a meeting 23.1 at 34 rows of 12288 -> 4096, and the next kernel starts slower: whole
// partial steps 0.2 % faster to 1 % slower.)
// grid (ceil(d / 1024), M), 256 threads, 4 columns per thread.
__global__ __launch_bounds__(256) void resid_finish_kernel(GemmEpi e) {
  __shared__ float red[4];
  const int m = blockIdx.y, n = (blockIdx.x * 256 + threadIdx.x) * 4;
  float part = 0.f;
  if (n < e.d) {
    f32x4 p[kSkinnySplit];
#pragma unroll
    for (int z = 0; z < kSkinnySplit; ++z)
      p[z] = *(const f32x4*)(e.partial + ((size_t)z * e.M + m) * e.d + n);
    const float4 h = *(const float4*)(e.h + (size_t)m * e.d + n);
    const u32x2 g4 = *(const u32x2*)(e.gain_next + n);
    f32x4 v = p[0];
#pragma unroll
    for (int z = 1; z < kSkinnySplit; ++z) v += p[z];
    part = epi_resid_pre(e, m, n >> 4, (n >> 2) & 3, v, h, g4);
  }
  part = block_sum<4>(part, red);
  if (threadIdx.x == 0) {
    unsigned long long fx = sumsq_to_fixed(part, e.sum_cap);
    if (fx) atomicAdd((unsigned long long*)(e.sumsq_out + (size_t)(blockIdx.x & (kSumSlots - 1)) * e.sum_stride + m), fx);
  }
}

static void launch_resid_finish(GemmEpi e, int N, hipStream_t s) {
  const dim3 grid((N + 1023) / 1024, e.M);
  e.sum_cap = sumsq_cap(grid.x);
  resid_finish_kernel<<<grid, 256, 0, s>>>(e);
}

template <int EPI, int MT, int NTW, int KS, int U = 4, bool W8 = false>
static void launch_skinny_t(const bf16_t* Ap, int MT_src, const void* Wp, int total_nt, int KB,
                            GemmEpi e, hipStream_t s, int ksplit = 1) {
  dim3 grid((total_nt + NTW - 1) / NTW, ksplit);
  if (EPI == EPI_RESID) e.sum_cap = sumsq_cap(grid.x, NTW);
  size_t smem = (size_t)KS * NTW * MT * 64 * sizeof(float4) + MT * 16 * sizeof(float);
  if (EPI == EPI_LOGITS) smem += (size_t)NTW * MT * 16 * sizeof(float4);  // per-tile row tuples
  if (W8) smem += NTW * 16 * sizeof(float);                               // weight scales
  if (smem > 48 * 1024) {
    static bool once = false;
    if (!once) {
      (void)hipFuncSetAttribute((const void*)gemm_bf16_skinny_kernel<EPI, MT, NTW, KS, U, W8>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
      once = true;
    }
  }
  gemm_bf16_skinny_kernel<EPI, MT, NTW, KS, U, W8><<<grid, KS * 64, smem, s>>>(
      (const u32x4*)Ap, (const u32x4*)Wp, total_nt, KB, MT_src, e);
}

// Tile counts per block were chosen by timing on MI355X: the kernels are bound by what the L2
// delivers (weights once + the activation fragments once per block), so more weight tiles per
// block (fewer re-reads of the activations) win as long as the grid still covers the 256 CUs.
// Weight tiles (of 16 vocabulary columns) to a block of the skinny LM head: eight, whose activations are
// then read the fewest times, where that fills the chip, fewer where it leaves compute units without a block.  us by events,
// 32 rows: vocabulary 126464, d 4096: 4 tiles 191, 8 179;  152064 of 3584: 207, 195;  4096 of 256 (32 blocks of eight):
// 8 tiles 8.5, 4 tiles 7.3, 2 tiles 6.5.
static int lm_tiles(int total_nt) { return total_nt >= 8 * 256 ? 8 : total_nt >= 4 * 256 ? 4 : 2; }
// blocks (= partial tuples per row) of the skinny LM-head GEMM over a vocabulary of V columns
int lm_head_parts(int V) { const int t = lm_tiles(V / 16); return (V / 16 + t - 1) / t; }

int skinny_tiles_per_block(int epi, int total_nt) {
  if (epi == EPI_RESID) return 1;
  if (epi == EPI_LOGITS) return lm_tiles(total_nt);
  if (total_nt >= 6 * 256) return 6;
  if (total_nt >= 3 * 256) return 3;
  return total_nt >= 2 * 256 ? 2 : 1;
}

// A residual GEMM has only d_model / 16 weight tiles, one to a block, and every block pulls the
// whole [rows, K] operand beside its 16 rows of weights: 1.2 MB beside 0.4 at 48 rows of 12288.  Four
// neighbouring tiles and a quarter of K to a block pull a quarter of that; the partial products
// are summed by resid_finish_kernel (4.8 us and the gap before it).  us on MI355X, whole K -> split
// and finish, d 4096:
//   3 row tiles  K 12288  30.5 -> 21.3 + 4.8   (e4m3 23.5 -> 15.4 + 4.0)   K 4096  11.2 ->  8.2 + 4.8
//   6 row tiles  K 12288  44.4 -> 27.0 + 5.1                               K 4096  16.6 -> 11.0 + 5.1
// which is a gain of about MT * K * 2.4e-4 - 5.5 us.  Two tiles and half of K: 23 and 33 at K 12288.
// The line holds at every width, since a block's bytes do not depend on it and the few blocks of a narrow
// matrix leave as much of the chip idle split or not.  us of a down projection with its finish, by
// events, just above the line (MT K 23808 - 24576, 2 to 6 row tiles) and at 3 row tiles of 12288:
//   d  128   17.1 -> 14.9, 22.7 -> 18.5     d 2048   20.4 -> 18.3, 28.0 -> 23.5
//   d  512   18.7 -> 15.5, 26.1 -> 19.7     d 4096   23.8 -> 21.1, 32.0 -> 26.5 (6 x 3968: 20.1 -> 20.3)
//   d 1024   19.5 -> 16.1, 26.7 -> 20.3     d 8192   38.7 -> 32.8, 56.8 -> 44.1
static bool skinny_splits(int MT, int K, const GemmEpi& e) {
  return e.partial && (size_t)kSkinnySplit * e.M * e.d <= e.partial_floats && (long)MT * K >= 23000;
}

// e4m3 weights: KB counts 64-wide k-steps; fewer steps per register set, because a step holds
// two activation fragments per m-tile
template <int EPI, int MT>
static void launch_skinny_mt_w8(const bf16_t* Ap, int MT_src, const void* Wq, int total_nt,
                                int KB, const GemmEpi& e, hipStream_t s) {
  if constexpr (EPI == EPI_LOGITS) {
    switch (lm_tiles(total_nt)) {
      case 8: launch_skinny_t<EPI, MT, 8, 4, 1, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
      case 4: launch_skinny_t<EPI, MT, 4, 4, 1, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
      default: launch_skinny_t<EPI, MT, 2, 4, 1, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
    }
  } else if constexpr (EPI == EPI_RESID) {
    if constexpr (MT > 1) {
      if (skinny_splits(MT, KB * 64, e)) {
        launch_skinny_t<EPI_PARTIAL, MT, kSkinnySplit, 4, 1, true>(Ap, MT_src, Wq, total_nt, KB, e, s, kSkinnySplit);
        launch_resid_finish(e, total_nt * 16, s);
        return;
      }
    }
    launch_skinny_t<EPI, MT, 1, 8, (MT > 3 ? 1 : 2), true>(Ap, MT_src, Wq, total_nt, KB, e, s);
  } else {
    constexpr int U6 = MT > 2 ? 1 : 2, U8 = MT > 3 ? 1 : 2;
    switch (skinny_tiles_per_block(EPI, total_nt)) {
      case 6: launch_skinny_t<EPI, MT, 6, 4, U6, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
      case 3: launch_skinny_t<EPI, MT, 3, 8, U8, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
      case 2: launch_skinny_t<EPI, MT, 2, 8, U8, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
      default: launch_skinny_t<EPI, MT, 1, 8, U8, true>(Ap, MT_src, Wq, total_nt, KB, e, s); break;
    }
  }
}

template <int EPI, int MT>
static void launch_skinny_mt(const bf16_t* Ap, int MT_src, const bf16_t* Wp, int total_nt, int KB,
                             const GemmEpi& e, hipStream_t s) {
  if constexpr (EPI == EPI_LOGITS) {
    switch (lm_tiles(total_nt)) {
      case 8: launch_skinny_t<EPI, MT, 8, 4, 1>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 4: launch_skinny_t<EPI, MT, 4, 4, 2>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      default: launch_skinny_t<EPI, MT, 2, 4, 2>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
    }
  } else if constexpr (EPI == EPI_RESID) {
    if constexpr (MT > 1) {
      if (skinny_splits(MT, KB * 32, e)) {
        // three k-steps to a register set where the two sets divide a wave's range: more in flight and no
        // step loaded twice.  us of the product and its finish, by events, two steps to a set -> three:
        //   d 4096  K  9216  3 row tiles 22.4 -> 21.5   4: 24.5 -> 23.9      K 6144  4: 20.1 -> 20.1
        //           K 12288  2: 24.2 -> 23.8   3: 26.0 -> 25.6   4: 28.5 -> 28.5
        //           K 15360  2: 28.0 -> 27.3   3: 30.1 -> 29.2   4: 32.9 -> 32.2
        //           K 18432  2: 31.8 -> 31.1   3: 33.9 -> 33.3   4: 36.9 -> 36.9
        //   d 1024  0 - 0.9 shorter at the same sizes
        // and longer where a range ends inside a set: 16 and 37 steps a wave, 17.9 -> 18.4 and 31.0 -> 31.8.
        if (MT <= 4 && KB % (6 * 4 * kSkinnySplit) == 0)
          launch_skinny_t<EPI_PARTIAL, MT, kSkinnySplit, 4, (MT > 4 ? 1 : 3)>(Ap, MT_src, Wp, total_nt, KB, e, s, kSkinnySplit);
        else
          launch_skinny_t<EPI_PARTIAL, MT, kSkinnySplit, 4, (MT > 4 ? 1 : 2)>(Ap, MT_src, Wp, total_nt, KB, e, s, kSkinnySplit);
        launch_resid_finish(e, total_nt * 16, s);
        return;
      }
    }
    launch_skinny_t<EPI, MT, 1, 8, 2>(Ap, MT_src, Wp, total_nt, KB, e, s);
  } else {
    // (five or six m-tiles: one k-step per register set where two would not fit 256 registers)
    constexpr int U8 = MT > 4 ? 1 : 2;
    switch (skinny_tiles_per_block(EPI, total_nt)) {
      case 6: launch_skinny_t<EPI, MT, 6, 4, 2>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 3: launch_skinny_t<EPI, MT, 3, 8, U8>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 2: launch_skinny_t<EPI, MT, 2, 8, U8>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      default: launch_skinny_t<EPI, MT, 1, 8, 2>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
    }
  }
}

// gate/up and LM head; rstd_s: 1/rms of the rows from row tile mt_base on, in LDS
template <int EPI, int WTM, int WTN>
__device__ __forceinline__ void tiled_epilogue(const GemmEpi& e, f32x4 (&acc)[WTN][WTM], int mt_base,
                                               int nt_base, int total_nt, int lane, const float* rstd_s) {
  const int q4 = lane >> 4;
  // every row's 1/rms first: these loads must not be strung out between the stores below
  float rsj[WTM];
#pragma unroll
  for (int j = 0; j < WTM; ++j) rsj[j] = rstd_s[j * 16 + (lane & 15)];
#pragma unroll
  for (int j = 0; j < WTM; ++j) {
    const int m = (mt_base + j) * 16 + (lane & 15);
    const bool mvalid = m < e.M;
    if constexpr (EPI == EPI_LOGITS) {
      if (mvalid) {
        const float rs = rsj[j];
#pragma unroll
        for (int i = 0; i < WTN; ++i) {
          int vt = nt_base + i;
          if (vt < total_nt) epi_logits(e, m, vt, q4, acc[i][j], rs);
        }
      }
    } else {
      if (mvalid) {
        const float rs = rsj[j];
#pragma unroll
        for (int i = 0; i < WTN; ++i) {
          int vt = nt_base + i;
          if constexpr (WTN % 2 == 0) {
            if (i & 1) continue;
            if (vt + 1 < total_nt) epi_swiglu2(e, m, vt, q4, acc[i][j], acc[i + 1][j], rs);
            else if (vt < total_nt) epi_swiglu(e, m, vt, q4, acc[i][j], rs);
          } else if (vt < total_nt) {
            epi_swiglu(e, m, vt, q4, acc[i][j], rs);
          }
        }
      }
    }
  }
}

// Where a block keeps what its epilogue needs of its rows (tiled, 8 waves): behind the operand ring, 1/rms of
// each row and, for q k v, the row's entry of the row list.  q k v also stages its rows' rotation factors in
// the ring's place once the products are done.
template <int EPI, int ROWS> constexpr int tiled_row_bytes() {
  return EPI == EPI_RESID ? 0 : ROWS * (EPI == EPI_QKV ? 20 : 4);
}

// q k v epilogue of the 8-wave kernels.  The rotation factors of the block's rows (hd / 2 pairs each, the
// same for every head) come to LDS in one go instead of 32 bytes a lane and fragment from memory, each time
// waited for.  A row's 16-byte chunks are stored at their number XOR the row's low bits: 16 rows read at the
// same column hit all banks.  Two row tiles are rotated together: after a swap of lane rows a lane
// holds 8 consecutive columns of one row, stored as 16 bytes.
//   us per launch, 4096 -> 3 x 4096, before -> after:  768 rows 192 x 192    79.3 -> 74.8
//   4096 rows 192 x 384    405 -> 360                 4096 rows 256 x 256   386 -> 328
template <int WM, int WN, int WTM, int WTN>
__device__ __forceinline__ void tiled_qkv(const GemmEpi& e, f32x4 (&acc)[WTN][WTM], int mt0, int nt0,
                                          int total_nt, int wave, int lane, u32x4* lds,
                                          const int4* row_s, const float* rstd_s) {
  static_assert(WTM % 2 == 0, "row tiles are taken in pairs");
  constexpr int ROWS = WM * WTM * 16, NW = WM * WN;
  const int wm = wave / WN, wn = wave % WN, q4 = lane >> 4, r16 = lane & 15;
  const int hd = e.hd, tph = hd >> 4, half = hd >> 1, chunks = hd >> 2;  // 16-byte chunks of a row's factors
  const int nqt = e.Hq * tph, nkt = e.Hkv * tph;
  __syncthreads();   // (the ring is no longer read, and its last loads have landed)
  for (int c = wave * 64; c < ROWS * chunks; c += NW * 64) {
    const int row = (c + lane) / chunks, at = (c + lane) % chunks;
    const int pos = max(row_s[row].x, 0);
    const char* src = (const char*)(e.cs + (size_t)pos * half) + ((at ^ (row & 15)) * 16);
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                     (void __attribute__((address_space(3)))*)(lds + c), 16, 0, 0);
  }
  wait_vmcnt<0>();
  __syncthreads();
  const bool hi = q4 >= 2;
  const unsigned sin_sign = hi ? 0u : 0x80000000u;  // first half: x cos - y sin; second: x cos + y sin
#pragma unroll
  for (int j = 0; j < WTM; j += 2) {
    const int row0 = (wm * WTM + j) * 16 + r16, row1 = row0 + 16;
    const float rs[2] = {rstd_s[row0], rstd_s[row1]};
    // the row whose 8 columns the lane stores, and the rows whose values it holds
    const int srow = (q4 & 1) ? row1 : row0;
    const int4 ri = row_s[srow];   // position (-1: padding), -, cache offset, keys per slab
    const int m = mt0 * 16 + srow, pos = max(ri.x, 0);
    const bool valid = m < e.M && ri.x >= 0;
    bf16_t* const q_row = e.q_out + (size_t)m * (e.Hq * hd) + (hi ? half : 0);
    bf16_t* const k_row = e.kc + ri.z;
    // V stays as the products left it: four columns of the lane's own two rows
    const int4 va = row_s[row0], vb = row_s[row1];
    const bool va_ok = mt0 * 16 + row0 < e.M && va.x >= 0, vb_ok = mt0 * 16 + row1 < e.M && vb.x >= 0;
#pragma unroll
    for (int i = 0; i < WTN; ++i) {
      const int vt = nt0 + wn * WTN + i;
      if (vt < nqt + nkt) {
        const bool is_q = vt < nqt;
        const int t = is_q ? vt : vt - nqt, head = t / tph, w = t - head * tph;
        unsigned pk[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 v = acc[i][j + u];
          const u32x4* cs = lds + (u ? row1 : row0) * chunks;
          union { u32x4 q[2]; float f[8]; } c;   // (cos, sin) x 4 columns
          c.q[0] = cs[(w * 4 + (q4 & 1) * 2) ^ r16];
          c.q[1] = cs[(w * 4 + (q4 & 1) * 2 + 1) ^ r16];
          float out[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float sn = __uint_as_float(__float_as_uint(c.f[2 * r + 1]) ^ sin_sign);
            out[r] = (v[r] * c.f[2 * r] + other_half(v[r]) * sn) * rs[u];
          }
          pk[u][0] = pack2(out[0], out[1]);
          pk[u][1] = pack2(out[2], out[3]);
        }
        // lanes with even q4 end with both halves of row tile j's 8 columns, the others with j + 1's
        const auto s0 = __builtin_amdgcn_permlane16_swap(pk[0][0], pk[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(pk[0][1], pk[1][1], false, false);
        const u32x4 o = {s0[0], s1[0], s0[1], s1[1]};
        if (valid) {
          if (is_q) *(u32x4*)(q_row + head * hd + w * 8) = o;
          else *(u32x4*)(k_row + (size_t)head * ri.w * hd + kcache_index(pos, w * 8 + (hi ? half : 0), hd)) = o;
        }
      } else if (vt < total_nt) {
        const int t = vt - nqt - nkt, head = t / tph, c0 = (t - head * tph) * 16 + q4 * 4;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int4 rv = u ? vb : va;
          if (u ? vb_ok : va_ok) {
            bf16_t* dst = e.vc + rv.z + (size_t)head * rv.w * hd + vcache_index(rv.x, c0, rv.w);
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[r * 8] = f32_to_bf16(acc[i][j + u][r] * rs[u]);
          }
        }
      }
    }
  }
}

// Residual epilogue of Z blocks that hold the same tile for Z ranges of K (k_meet.h).  The tile's fragments
// are shared out by their number in the wave, WTM * i + j: every wave stores those of the other blocks'
// shares (1 KiB each, as the registers hold them), and after the meeting adds the others' pieces to its
// own share in the order of the ranges and finishes it.  Rows' sums of squares go through LDS (`sums`: the
// block's WN x rows floats: added in float32, rounded to fixed point once), one addition to memory per row and
// share.
// Against partial products and a second kernel that reads them all back, in whole steps by events (768 rows,
// d 4096, 192 x 256 x 4): O 49.1 -> 44.3 us, down (K 12288) 87.6 -> 81.6; kernel trace 43.3 and 83.2.  About 14 us of
// that are the exchange and the residual stream's read and write.
template <int WM, int WN, int WTM, int WTN, int Z>
__device__ __forceinline__ void tiled_meet_resid(const GemmEpi& e, f32x4 (&acc)[WTN][WTM], int mt0,
                                                 int nt0, int total_nt, int wave, int lane, int tile,
                                                 int z, float* sums) {
  constexpr int NFR = WTN * WTM, NO = (NFR + Z - 1) / Z, ROWS = WM * WTM * 16;
  const int wm = wave / WN, wn = wave % WN, q4 = lane >> 4;
  const size_t per_range = (size_t)WM * WN * NFR * 64;
  f32x4* pieces = (f32x4*)e.partial + (size_t)tile * Z * per_range + (size_t)wave * NFR * 64 + lane;
  const int rows_j = (e.M + 15) / 16 - mt0 - wm * WTM;   // row tiles of the wave that hold rows: no exchange beyond
  // (the share's ranges are known per z at compile time: the accumulators need constant indices)
  f32x4 own[NO];
#pragma unroll
  for (int y = 0; y < Z; ++y)
    if (y == z) {
#pragma unroll
      for (int f = 0; f < NFR; ++f) {
        if (f >= y * NFR / Z && f < (y + 1) * NFR / Z) own[f - y * NFR / Z] = acc[f / WTM][f % WTM];
        else if (f % WTM < rows_j) pieces[y * per_range + f * 64] = acc[f / WTM][f % WTM];
      }
      if ((y + 1) * NFR / Z - y * NFR / Z < NO) own[NO - 1] = own[0];  // (a share one fragment short)
    }
  // The share is finished NB fragments at a time, every load of a batch ahead of its first use; the first
  // batch's residual stream and gains are on their way while the blocks meet.
  constexpr int NB = NO < 28 / Z ? NO : 28 / Z;
  float4 h[NB];
  u32x2 g[NB];
  auto row_of = [&](int f) { return (mt0 + wm * WTM + f % WTM) * 16 + (lane & 15); };
  auto tile_of = [&](int f) { return nt0 + wn * WTN + f / WTM; };
  auto fetch_h = [&](int first, int hi) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int f = min(first + k, hi - 1), m = min(row_of(f), e.M - 1), n = min(tile_of(f), total_nt - 1) * 16 + q4 * 4;
      h[k] = *(const float4*)(e.h + (size_t)m * e.d + n);
      g[k] = *(const u32x2*)(e.gain_next + n);
    }
  };
  fetch_h(z * NFR / Z, (z + 1) * NFR / Z);
  unsigned shares = meet_blocks(e.meet + tile, Z, z, e.meet_limit, e.meet_apart, [&] {
    const int lo = z * NFR / Z, n = (z + 1) * NFR / Z - lo;
#pragma unroll
    for (int k = 0; k < NO; ++k)
      if (k < n) pieces[z * per_range + (lo + k) * 64] = own[k];
  });
  float* my_sums = sums + wn * ROWS + wm * WTM * 16 + (lane & 15);
  // (its own share first, while that is in registers)
  for (int sh = z; shares; sh = __builtin_ctz(shares | 1u << Z)) {
    const int lo = sh * NFR / Z, hi = (sh + 1) * NFR / Z;
    shares &= ~(1u << sh);
    if (lane < 16) {
#pragma unroll
      for (int j = 0; j < WTM; ++j) my_sums[j * 16] = 0.f;
    }
    if (sh != z) {   // (the share of a block that has gone: this block's piece of it is in memory)
#pragma unroll
      for (int k = 0; k < NO; ++k) own[k] = pieces[z * per_range + min(lo + k, hi - 1) * 64];
    }
#pragma unroll
    for (int b0 = 0; b0 < NO; b0 += NB) {
      f32x4 p[NB][Z - 1];   // the pieces of the other ranges, in their order
#pragma unroll
      for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int y = 0; y < Z - 1; ++y)
          if ((lo + b0 + k) % WTM < rows_j) p[k][y] = pieces[(y + (y >= z)) * per_range + min(lo + b0 + k, hi - 1) * 64];
      if (sh != z || b0 > 0) fetch_h(lo + b0, hi);
#pragma unroll
      for (int k = 0; k < NB && b0 + k < NO; ++k) {
        const int f = lo + b0 + k, m = row_of(f), vt = tile_of(f);
        f32x4 v = z == 0 ? own[b0 + k] : p[k][0];
#pragma unroll
        for (int y = 1; y < Z; ++y) v += y == z ? own[b0 + k] : y < z ? p[k][y < Z - 1 ? y : 0] : p[k][y - 1];
        float part = 0.f;
        if (f < hi && m < e.M && vt < total_nt) part = epi_resid_pre(e, m, vt, q4, v, h[k], g[k]);
        part += other_row(part);
        part += other_half(part);
        if (lane < 16) my_sums[f % WTM * 16] += part;
      }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < ROWS; r += WM * WN * 64) {
      float s = sums[r];
#pragma unroll
      for (int w = 1; w < WN; ++w) s += sums[w * ROWS + r];
      const int m = mt0 * 16 + r;
      const unsigned long long fx = sumsq_to_fixed(s, e.sum_cap);
      const int slot = (nt0 / (WN * WTN) * Z + sh) & (kSumSlots - 1);
      if (fx && m < e.M) atomicAdd((unsigned long long*)(e.sumsq_out + (size_t)slot * e.sum_stride + m), fx);
    }
    if (shares) __syncthreads();
  }
}

// Residual epilogue of a whole K: D row tiles of the residual stream are on their way while one is finished
// (the epilogue of a round of 256 x 256 blocks then moves its bytes at 7 TB/s, most of them through the
// last-level cache), and a block adds each row's sum of squares once, through LDS (`sums`: WN x rows floats, added
// in float32 and rounded to fixed point once).
template <int WM, int WN, int WTM, int WTN>
__device__ __forceinline__ void tiled_resid(const GemmEpi& e, f32x4 (&acc)[WTN][WTM], int mt0, int nt0,
                                            int total_nt, int wave, int lane, float* sums) {
  constexpr int ROWS = WM * WTM * 16, D = 14 / WTN < 2 ? 2 : 14 / WTN < WTM ? 14 / WTN : WTM;
  const int wm = wave / WN, wn = wave % WN, q4 = lane >> 4;
  const int vt0 = nt0 + wn * WTN, r0 = (mt0 + wm * WTM) * 16 + (lane & 15);
  u32x2 g[WTN];
  int n[WTN];
#pragma unroll
  for (int i = 0; i < WTN; ++i) {
    n[i] = min(vt0 + i, total_nt - 1) * 16 + q4 * 4;
    g[i] = *(const u32x2*)(e.gain_next + n[i]);
  }
  float4 h[D][WTN];
  auto fetch = [&](float4 (&to)[WTN], int j) {
    const float* row = e.h + (size_t)min(r0 + j * 16, e.M - 1) * e.d;
#pragma unroll
    for (int i = 0; i < WTN; ++i) to[i] = *(const float4*)(row + n[i]);
  };
#pragma unroll
  for (int j = 0; j < D - 1; ++j) fetch(h[j], j);
  __syncthreads();   // (the LDS is no longer read)
  float* my_sums = sums + wn * ROWS + wm * WTM * 16 + (lane & 15);
#pragma unroll
  for (int j = 0; j < WTM; ++j) {
    if (j + D - 1 < WTM) fetch(h[(j + D - 1) % D], j + D - 1);
    const int m = r0 + j * 16;
    float part = 0.f;
#pragma unroll
    for (int i = 0; i < WTN; ++i)
      if (m < e.M && vt0 + i < total_nt) part += epi_resid_pre(e, m, vt0 + i, q4, acc[i][j], h[j % D][i], g[i]);
    part += other_row(part);
    part += other_half(part);
    if (lane < 16) my_sums[j * 16] = part;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < ROWS; r += WM * WN * 64) {
    float s = sums[r];
#pragma unroll
    for (int w = 1; w < WN; ++w) s += sums[w * ROWS + r];
    const int m = mt0 * 16 + r;
    const unsigned long long fx = sumsq_to_fixed(s, e.sum_cap);
    if (fx && m < e.M)
      atomicAdd((unsigned long long*)(e.sumsq_out + (size_t)((nt0 / (WN * WTN)) & (kSumSlots - 1)) * e.sum_stride + m), fx);
  }
}

// Per-row weight scales (matrices that came as e4m3 codes, expanded to bf16 for these kernels):
// the lane's 4 accumulator values of weight tile i are output features (nt_base + i)*16 + q4*4 ..
template <int WTM, int WTN>
__device__ __forceinline__ void scale_acc(const GemmEpi& e, f32x4 (&acc)[WTN][WTM], int nt_base,
                                          int total_nt, int lane) {
  const int q4 = lane >> 4;
#pragma unroll
  for (int i = 0; i < WTN; ++i) {
    const int vt = nt_base + i < total_nt ? nt_base + i : 0;
    const float4 c = *(const float4*)(e.wscale + (size_t)vt * 16 + q4 * 4);
#pragma unroll
    for (int j = 0; j < WTM; ++j) {
      f32x4 a = acc[i][j];
      a[0] *= c.x; a[1] *= c.y; a[2] *= c.z; a[3] *= c.w;
      acc[i][j] = a;
    }
  }
}

// Which (n-block, m-block) a thread block works on.  Blocks go to the 8 XCDs round-robin by
// their linear index, and each XCD has its own L2: the m-blocks that share an n-block's weight
// tiles should meet in one L2.  gridDim.x a multiple of 8 gives that by itself.  Otherwise the
// linear index is first turned into "XCD-major" order (all blocks of XCD 0, then XCD 1, ...)
// and m runs fastest in that order, so an n-block's m-blocks are neighbours on one XCD.
__device__ __forceinline__ void tiled_block_xy(int& bx, int& by) {
  const int gx = gridDim.x, gy = gridDim.y, nb = gx * gy;
  bx = blockIdx.x; by = blockIdx.y;
  if ((gx & 7) != 0) {
    const int lin = blockIdx.y * gx + blockIdx.x, xcd = lin & 7;
    // blocks before this one in XCD-major order: those of the lower XCDs, then its own earlier ones
    const int j = xcd * (nb >> 3) + min(xcd, nb & 7) + (lin >> 3);
    bx = j / gy; by = j - bx * gy;
  }
}

// Which tile and range of K a block works on where K is split over Z blocks, on a one-dimensional grid.  An XCD
// gets a run of whole tiles, the Z blocks of a tile one after the other, so that they run at the same time
// and meet in one L2.  If the XCDs' runs, up to a tile of different length, fit its 32 compute units, the
// grid has room for the longest on each (meet_grid) and the blocks it has too many find no tile: false.
// Otherwise the grid is Z blocks a tile, and what is left over on the XCDs (up to Z - 1 blocks each) makes up
// the last tiles, whose blocks have to fence.
template <int Z>
__device__ __forceinline__ bool meet_place(int tiles, int& tile, int& z) {
  const int n = gridDim.x, xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  if (n != tiles * Z) {
    tile = xcd * tiles / 8 + j / Z;
    z = j % Z;
    return tile < (xcd + 1) * tiles / 8;
  }
  const int few = n >> 3, more = n & 7;   // blocks of an XCD: few + 1 on the first `more` of them
  const int q = (few + (xcd < more)) / Z, above = min(xcd, more), below = xcd - above;
  int at = (above * ((few + 1) / Z) + below * (few / Z)) * Z + j;
  if (j >= q * Z) {
    const int whole = (more * ((few + 1) / Z) + (8 - more) * (few / Z)) * Z;
    at = whole + above * ((few + 1) % Z) + below * (few % Z) + j - q * Z;
  }
  tile = at / Z;
  z = at - tile * Z;
  return true;
}
static int meet_grid(int tiles, int Z) {
  const int longest = (tiles + 7) / 8 * Z;
  return longest <= 32 ? 8 * longest : tiles * Z;
}

// ---------------------------------------------------------------------------------------------
// tiled, 4 waves (2x2): wave tile = WTM x WTN fragments, K step 32.  Operands are double-buffered
// in LDS; global loads run through four register sets, four k-steps ahead.  For the blocks of
// residual products that are too small to keep eight waves busy (128 x 128 and 96 x 128; at 192 x 192 and 192 x 128
// eight waves take 0.53 and 0.46 us a k-step, four 0.64 and 0.55).
// grid = (ceil(n-tiles / (2*WTN)), ceil(m-tiles / (2*WTM))); K split over Z > 1 blocks: meet_grid()
// ---------------------------------------------------------------------------------------------
#define EC_TILED_GLOAD(REGS, KBV)                                                   \
  {                                                                                 \
    int kbc_ = min((KBV), KB - 1);                                                  \
    _Pragma("unroll") for (int i = 0; i < LF; ++i) REGS[i] = src[i][(size_t)kbc_ * stride[i]]; \
  }
#define EC_TILED_LSTORE(REGS, STAGE)                                                \
  {                                                                                 \
    _Pragma("unroll") for (int i = 0; i < LF; ++i) {                                \
      if (4 * i + 3 < NF || wave + 4 * i < NF) lds[STAGE][wave + 4 * i][lane] = REGS[i]; \
    }                                                                               \
  }
#define EC_TILED_COMPUTE(STAGE)                                                     \
  {                                                                                 \
    bf16x8 af_[WTM], wf_[WTN];                                                      \
    _Pragma("unroll") for (int j = 0; j < WTM; ++j)                                 \
        af_[j] = v4_as_bf16x8(lds[STAGE][wm * WTM + j][lane]);                      \
    _Pragma("unroll") for (int i = 0; i < WTN; ++i)                                 \
        wf_[i] = v4_as_bf16x8(lds[STAGE][BMT + wn * WTN + i][lane]);                \
    _Pragma("unroll") for (int i = 0; i < WTN; ++i)                                 \
      _Pragma("unroll") for (int j = 0; j < WTM; ++j)                               \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf_[i], af_[j], acc[i][j], 0, 0, 0); \
  }

template <int WTM, int WTN, bool WS, int Z>
__global__ __launch_bounds__(256) void gemm_bf16_tiled4_kernel(const u32x4* __restrict__ Ap,
                                                              const u32x4* __restrict__ Wp,
                                                              int total_nt, int KB_all, int MT,
                                                              GemmEpi e) {
  constexpr int BMT = 2 * WTM, BNT = 2 * WTN, NF = BMT + BNT;  // fragments per k-step
  constexpr int LF = (NF + 3) / 4;                             // fragments loaded per wave
  __shared__ u32x4 lds[2][NF][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int bx, by, tile = 0, z = 0;
  if constexpr (Z > 1) {
    const int gy = (e.M + 16 * BMT - 1) / (16 * BMT);   // (m fastest: the tiles that share weights meet on an XCD)
    if (!meet_place<Z>((total_nt + BNT - 1) / BNT * gy, tile, z)) return;
    bx = tile / gy; by = tile - bx * gy;
  } else {
    tiled_block_xy(bx, by);
  }
  const int mt0 = by * BMT, nt0 = bx * BNT;
  const int wm = wave >> 1, wn = wave & 1;
  // the block's range of K
  const int kb_first = z * KB_all / Z, KB = (z + 1) * KB_all / Z - kb_first;

  // Fragment f of the block (0..BMT-1 activations, BMT.. weights) is loaded by wave f % 4.
  // A fragment outside the matrix streams fragment 0 instead (valid memory); what it produces
  // lands in rows / columns that are never stored.
  const u32x4* src[LF];
  size_t stride[LF];  // u32x4 per k-step
#pragma unroll
  for (int i = 0; i < LF; ++i) {
    int f = wave + 4 * i;
    src[i] = Ap + lane;
    stride[i] = (size_t)MT * 64;
    if (f < BMT) {
      int mt = mt0 + f;
      if (mt < MT) src[i] = Ap + (size_t)mt * 64 + lane;
    } else if (f < NF) {
      int nt = nt0 + (f - BMT);
      if (nt < total_nt) {
        src[i] = Wp + packed_w_frag(nt, 0, KB_all, e.w_grp) * 64 + lane;
        stride[i] = (size_t)e.w_grp * 64;
      }
    }
    src[i] += (size_t)kb_first * stride[i];
  }

  f32x4 acc[WTN][WTM];
#pragma unroll
  for (int i = 0; i < WTN; ++i)
#pragma unroll
    for (int j = 0; j < WTM; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // prologue: k-step 0 into LDS stage 0, k-steps 1..4 in flight in four register sets (the L2
  // delivers by Little's law: bytes in flight / latency, so the sets are what buys bandwidth)
  u32x4 r0[LF], r1[LF], r2[LF], r3[LF];
  EC_TILED_GLOAD(r0, 0)
  EC_TILED_LSTORE(r0, 0)
  EC_TILED_GLOAD(r0, 1)
  EC_TILED_GLOAD(r1, 2)
  EC_TILED_GLOAD(r2, 3)
  EC_TILED_GLOAD(r3, 4)
  __syncthreads();
  // iteration kb: compute stage kb&1; the register set holding k-step kb+1 goes to stage
  // (kb+1)&1 and is reloaded with k-step kb+5
#define EC_TILED_STEP(REGS, KBV, STAGE)       \
  if ((KBV) < KB) {                           \
    EC_TILED_COMPUTE(STAGE)                   \
    EC_TILED_LSTORE(REGS, (STAGE) ^ 1)        \
    EC_TILED_GLOAD(REGS, (KBV) + 5)           \
  }                                           \
  __syncthreads();
  for (int kb = 0; kb < KB; kb += 4) {
    EC_TILED_STEP(r0, kb, 0)
    EC_TILED_STEP(r1, kb + 1, 1)
    EC_TILED_STEP(r2, kb + 2, 0)
    EC_TILED_STEP(r3, kb + 3, 1)
  }
#undef EC_TILED_STEP

  if constexpr (WS) scale_acc<WTM, WTN>(e, acc, nt0 + wn * WTN, total_nt, lane);
  if constexpr (Z > 1)
    tiled_meet_resid<2, 2, WTM, WTN, Z>(e, acc, mt0, nt0, total_nt, wave, lane, tile, z, (float*)lds);
  else
    tiled_resid<2, 2, WTM, WTN>(e, acc, mt0, nt0, total_nt, wave, lane, (float*)lds);
}
#undef EC_TILED_GLOAD
#undef EC_TILED_LSTORE
#undef EC_TILED_COMPUTE

template <bool WS, int Z, int WTM, int WTN>
static void launch_tiled4_t(const bf16_t* Ap, int MT, const bf16_t* Wp, int total_nt, int KB,
                           GemmEpi e, hipStream_t s) {
  dim3 grid((total_nt + 2 * WTN - 1) / (2 * WTN), (e.M + 32 * WTM - 1) / (32 * WTM));
  e.sum_cap = sumsq_cap((long)grid.x * Z);
  if (Z > 1) grid = dim3(meet_grid(grid.x * grid.y, Z));
  gemm_bf16_tiled4_kernel<WTM, WTN, WS, Z><<<grid, 256, 0, s>>>((const u32x4*)Ap, (const u32x4*)Wp,
                                                                 total_nt, KB, MT, e);
}

// ---------------------------------------------------------------------------------------------
// tiled, 8 waves (WM x WN): wave tile = WTM x WTN fragments of 16 rows (activations x weights),
// K step 32.  Operand fragments go from global memory straight into LDS (buffer loads of 16 bytes a lane:
// lane l's land at base + 16 l, so a 1 KiB fragment keeps its order), into a ring of four k-steps,
// no staging registers; one barrier per k-step.
// grid = (ceil(n-tiles / (WN*WTN)), ceil(m-tiles / (WM*WTM))); K split over Z > 1 blocks: meet_grid()
// ---------------------------------------------------------------------------------------------
// The fragments of k-step k+1 are read from LDS while the MFMAs of k-step k run, a few after
// each row of them: a weight fragment goes back to the registers its last MFMA has just freed, the
// activation fragments and the last weight fragment have a second set.  Reads and MFMAs of a
// k-step one after the other leave the matrix cores idle for the reads (96 KiB at 128 B a clock
// for 192 x 384) and all of a step's reads ahead of its MFMAs hold up the issue of the latter.
// What bounds the loop is power: products of random operands alone hold 1.94 GHz and 1.95 PFLOP/s, with the reads
// and loads the clock settles at 1.7 - 1.8.  So what a k-step costs in cycles matters (256 x 256: 1024 of
// MFMAs, 1160 in all) and what it moves.  Against a ring of three that the barrier drains of LDS reads, with an uneven
// number of loads a wave and their addresses in vector registers: 1252 -> 1160 cycles a k-step for 256 x 256, 1564 ->
// 1410 for 192 x 384, 1165 -> 1124 for 192 x 320.  Kernel alone, 4096 -> 2 x 12288: 4096 rows 604 -> 583 us, 24576 rows 3520 ->
// 3390; whole full steps take 2.3 - 3.8 % less.
// Measured and left out, as slower: weights straight to registers, 8 waves side by side (less LDS traffic; 5 - 15 %); 4
// waves of 128 x 128 (a third less LDS traffic, 1.90 GHz, but 1270 cycles and a longer epilogue); s_setprio around the MFMAs
// (5 % more cycles); v_mfma_f32_32x32x16 (1.78 PFLOP/s alone).
constexpr int kRing = 4;   // k-steps in LDS
// bytes of LDS: the operand ring or, if larger, the rotation factors of the rows (hd 128) in its place, and the rows
template <int EPI, int WM, int WN, int WTM, int WTN>
constexpr int tiled8_lds() {
  constexpr int ring = kRing * (WM * WTM + WN * WTN) * 1024, factors = EPI == EPI_QKV ? WM * WTM * 16 * 512 : 0;
  return (ring > factors ? ring : factors) + tiled_row_bytes<EPI, WM * WTM * 16>();
}

template <int EPI, int WM, int WN, int WTM, int WTN, bool WS, int Z>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_bf16_tiled8_kernel(
    const u32x4* __restrict__ Ap, const u32x4* __restrict__ Wp, int total_nt, int KB_all, int MT,
    GemmEpi e) {
  constexpr int NW = WM * WN, BMT = WM * WTM, BNT = WN * WTN, NF = BMT + BNT;
  // A wave loads FULL whole fragments a k-step and, where they do not divide over the waves, half of one more,
  // so that all waves have the same number of loads in flight.
  constexpr int FULL = NF / NW, LF = FULL + (NF % NW != 0);
  static_assert(NF % NW == 0 || NF % NW == NW / 2, "the fragments left over are shared by two waves each");
  static_assert(WTN > 1, "the rolling reads need two weight fragments a wave");
  extern __shared__ u32x4 lds[];  // [kRing][NF][64]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int bx, by, tile = 0, z = 0;
  if constexpr (Z > 1) {
    const int gy = (e.M + 16 * BMT - 1) / (16 * BMT);   // (m fastest: the tiles that share weights meet on an XCD)
    if (!meet_place<Z>((total_nt + BNT - 1) / BNT * gy, tile, z)) return;
    bx = tile / gy; by = tile - bx * gy;
  } else {
    tiled_block_xy(bx, by);
  }
  const int mt0 = by * BMT, nt0 = bx * BNT;
  const int wm = wave / WN, wn = wave % WN;
  // the block's range of K
  const int kb_first = z * KB_all / Z, KB = (z + 1) * KB_all / Z - kb_first;

  // Fragment f of the block: 0..BMT-1 activations, BMT.. weights.
  // A fragment outside the matrix streams fragment 0 instead (valid memory); what it produces
  // lands in rows / columns that are never stored.  The addresses are wave-uniform.
  const char* src[LF];
  unsigned step[LF];  // bytes per k-step
  int frag[LF];
#pragma unroll
  for (int l = 0; l < LF; ++l) {
    const int f = l < FULL ? wave + NW * l : NW * FULL + (wave >> 1);
    const int mt = f < BMT && mt0 + f < MT ? mt0 + f : 0;
    const int nt = f >= BMT && nt0 + f - BMT < total_nt ? nt0 + f - BMT : 0;
    frag[l] = f;
    step[l] = (unsigned)(f < BMT ? MT : e.w_grp) * 1024;
    src[l] = (f < BMT ? (const char*)Ap + (size_t)mt * 1024
                      : (const char*)Wp + packed_w_frag(nt, 0, KB_all, e.w_grp) * 1024) +
             (size_t)kb_first * step[l];
  }
  const unsigned voff = lane * 16;
  const bool my_half = (lane >> 5) == (wave & 1);
  // load L of a k-step into the slot at byte SLOT of the ring; the next one's source is STEP bytes on
#define EC_T8_LOAD(L, SLOT, STEP)                                                            \
  {                                                                                          \
    const auto rs_ = __builtin_amdgcn_make_buffer_rsrc((void*)src[L], 0, 0xffffffff, 0x00027000);  \
    const auto to_ = (void __attribute__((address_space(3)))*)((char*)lds + (SLOT) + frag[L] * 1024);  \
    if ((L) < FULL) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_, to_, 16, voff, 0, 0, 0);   \
    else if (my_half) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_, to_, 16, voff, 0, 0, 0); \
    src[L] += (STEP);                                                                        \
  }

  f32x4 acc[WTN][WTM];
#pragma unroll
  for (int i = 0; i < WTN; ++i)
#pragma unroll
    for (int j = 0; j < WTM; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  constexpr int ROWS = BMT * 16;
  static_assert(ROWS % 64 == 0, "whole waves fetch the rows' sums");
  int4* row_s = (int4*)((char*)lds + tiled8_lds<EPI, WM, WN, WTM, WTN>() - tiled_row_bytes<EPI, ROWS>());
  float* rstd_s = (float*)(row_s + (EPI == EPI_QKV ? ROWS : 0));
  {
    bf16x8 afa[WTM], afb[WTM], wf[WTN - 1], wla, wlb;
    // The rows' sums of squares are requested ahead of the first operands, by one lane a row, and turned
    // into 1/rms while those are on their way, instead of in the epilogue by every lane for each of its
    // row tiles (eight loads and a division in 64 bits): gate/up, 768 rows 126.2 -> 123.4 us, 4096 rows
    // in 256 x 256 blocks 666 -> 631.
    constexpr bool HAS_ROWS = EPI != EPI_RESID;
    unsigned long long ssq[kSumSlots];
    int4 ri = make_int4(0, 0, 0, 0);
    const int my_row = wave * 64 + lane;
    if (HAS_ROWS && wave < ROWS / 64) {
      const int m = min(mt0 * 16 + my_row, e.M - 1);
      const int src_row = (EPI == EPI_LOGITS && e.row_sel) ? e.row_sel[m] : m;
#pragma unroll
      for (int sl = 0; sl < kSumSlots; ++sl) ssq[sl] = e.sumsq_in[(size_t)sl * e.sum_stride + src_row];
      if constexpr (EPI == EPI_QKV) ri = e.rowinfo[m];
    }
    __builtin_amdgcn_sched_barrier(0);
    // k-step k sits in slot k % kRing; past the range the last one is requested again
    constexpr int SLOT = NF * 1024;
#pragma unroll
    for (int k = 0; k < kRing - 1; ++k)
#pragma unroll
      for (int l = 0; l < LF; ++l) EC_T8_LOAD(l, k * SLOT, k + 1 < KB ? step[l] : 0u)
    __builtin_amdgcn_sched_barrier(0);
    if (HAS_ROWS && wave < ROWS / 64) {
      unsigned long long fx = 0;
#pragma unroll
      for (int sl = 0; sl < kSumSlots; ++sl) fx = sumsq_add(fx, ssq[sl]);
      rstd_s[my_row] = rstd_from_sum(e, fx);
      if constexpr (EPI == EPI_QKV) row_s[my_row] = ri;
    }
    wait_vmcnt<LF * (kRing - 2)>();
    block_barrier_nofence();
    typedef const __attribute__((address_space(3))) u32x4* lds_ptr;
    const unsigned la = (unsigned)(size_t)(lds_ptr)lds + (unsigned)(wm * WTM * 1024 + lane * 16);
    const unsigned lw = (unsigned)(size_t)(lds_ptr)lds + (unsigned)((BMT + wn * WTN) * 1024 + lane * 16);
#pragma unroll
    for (int j = 0; j < WTM; ++j) afa[j] = v4_as_bf16x8(((lds_ptr)(size_t)la)[j * 64]);
#pragma unroll
    for (int i = 0; i < WTN - 1; ++i) wf[i] = v4_as_bf16x8(((lds_ptr)(size_t)lw)[i * 64]);
    wla = v4_as_bf16x8(((lds_ptr)(size_t)lw)[(WTN - 1) * 64]);
    // Step k: this wave's loads of k-step k+1 have landed; after the barrier that holds for every wave, and
    // every wave is through with the MFMAs of k-step k-1, whose slot is then refilled with k-step k+3 while slot
    // k+1 is read.  (The reads of slot k may still be under way: nothing is written there.)  Two loads
    // follow each of the first rows of MFMAs: the sooner they are out, the less the barrier two steps on
    // has to wait for them.
#define EC_T8_WF(I, WL) ((I) < WTN - 1 ? wf[(I) < WTN - 1 ? (I) : 0] : WL)
#define EC_T8_STEP(NEXT, REFILL, AF, WL, AFN, WLN, MORE)                                     \
  {                                                                                          \
    wait_vmcnt<LF>();                                                                        \
    asm volatile("s_barrier" ::: "memory");                                                  \
    unsigned va_ = la + (NEXT), vw_ = lw + (NEXT);                                           \
    asm volatile("" : "+v"(va_), "+v"(vw_)); /* (one address each, the rest are offsets) */  \
    const lds_ptr sa_ = (lds_ptr)(size_t)va_, sw_ = (lds_ptr)(size_t)vw_;                    \
    _Pragma("unroll") for (int i = 0; i < WTN; ++i) {                                        \
      _Pragma("unroll") for (int j = 0; j < WTM; ++j)                                        \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(EC_T8_WF(i, WL), AF[j],          \
                                                            acc[i][j], 0, 0, 0);             \
      __builtin_amdgcn_sched_barrier(0);                                                     \
      if (i < WTN - 1) {                                                                     \
        _Pragma("unroll")                                                                    \
        for (int j = i * WTM / (WTN - 1); j < (i + 1) * WTM / (WTN - 1); ++j)                \
          AFN[j] = v4_as_bf16x8(sa_[j * 64]);                                                \
        wf[i < WTN - 1 ? i : 0] = v4_as_bf16x8(sw_[i * 64]);                                 \
        if (i == WTN - 2) WLN = v4_as_bf16x8(sw_[(WTN - 1) * 64]);                           \
      }                                                                                      \
      _Pragma("unroll")                                                                      \
      for (int l = i * 2 < LF ? i * 2 : LF; l < (i + 1 == WTN || i * 2 + 2 > LF ? LF : i * 2 + 2); ++l)  \
        EC_T8_LOAD(l, REFILL, (MORE) ? step[l] : 0u)                                         \
      __builtin_amdgcn_sched_barrier(0);                                                     \
    }                                                                                        \
  }
    int odd = SLOT, even = 2 * SLOT;   // slots of the odd and the even k-step that follow
    for (int kb = 0; kb + 1 < KB; kb += 2) {
      EC_T8_STEP(odd, 4 * SLOT - odd, afa, wla, afb, wlb, kb + 4 < KB)
      EC_T8_STEP(even, 2 * SLOT - even, afb, wlb, afa, wla, kb + 5 < KB)
      odd = 4 * SLOT - odd;     // 1, 3, 1, ...
      even = 2 * SLOT - even;   // 2, 0, 2, ...
    }
    static_assert(kRing == 4, "the slots follow each other as above");
    if (KB & 1) {  // (an odd trip count: the last k-step's fragments are in the first set)
#pragma unroll
      for (int i = 0; i < WTN; ++i)
#pragma unroll
        for (int j = 0; j < WTM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(EC_T8_WF(i, wla), afa[j], acc[i][j], 0, 0, 0);
    }
#undef EC_T8_STEP
#undef EC_T8_WF
  }
#undef EC_T8_LOAD
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  wait_vmcnt<0>();  // drain the clamped tail loads before the LDS goes away

  if constexpr (WS) scale_acc<WTM, WTN>(e, acc, nt0 + wn * WTN, total_nt, lane);
  if constexpr (Z > 1)
    tiled_meet_resid<WM, WN, WTM, WTN, Z>(e, acc, mt0, nt0, total_nt, wave, lane, tile, z, (float*)lds);
  else if constexpr (EPI == EPI_RESID)
    tiled_resid<WM, WN, WTM, WTN>(e, acc, mt0, nt0, total_nt, wave, lane, (float*)lds);
  else if constexpr (EPI == EPI_QKV)
    tiled_qkv<WM, WN, WTM, WTN>(e, acc, mt0, nt0, total_nt, wave, lane, lds, row_s, rstd_s);
  else
    tiled_epilogue<EPI, WTM, WTN>(e, acc, mt0 + wm * WTM, nt0 + wn * WTN, total_nt, lane, rstd_s + wm * WTM * 16);
}

template <int EPI, bool WS, int Z, int WM, int WN, int WTM, int WTN>
static void launch_tiled8_t(const bf16_t* Ap, int MT, const bf16_t* Wp, int total_nt, int KB,
                            GemmEpi e, hipStream_t s) {
  const size_t smem = tiled8_lds<EPI, WM, WN, WTM, WTN>();
  auto kern = gemm_bf16_tiled8_kernel<EPI, WM, WN, WTM, WTN, WS, Z>;
  static bool attr_set = false;
  if (!attr_set && smem > 48 * 1024) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)smem);
    attr_set = true;
  }
  dim3 grid((total_nt + WN * WTN - 1) / (WN * WTN), (e.M + 16 * WM * WTM - 1) / (16 * WM * WTM));
  e.sum_cap = sumsq_cap((long)grid.x * Z);
  if (Z > 1) grid = dim3(meet_grid(grid.x * grid.y, Z));
  kern<<<grid, WM * WN * 64, smem, s>>>((const u32x4*)Ap, (const u32x4*)Wp, total_nt, KB, MT, e);
}

// Block shapes of the tiled kernels (rows x weight rows).
//   8 waves: 0: 192 x 384   1: 192 x 256   2: 192 x 192   3: 192 x 128   6: 192 x 320   7: 256 x 256
//   4 waves: 4: 128 x 128   5: 96 x 128   (residual products only: q k v and gate/up of d 512 and 1536 take 15 - 25 %
//   longer with them than with 192 x 128 at 112 - 3000 rows, and no less at any other size)
// What a whole launch loses most by is its last round: shapes 6 and 7 are there for the sizes at which
// the others leave compute units or rows idle.  Two waves per SIMD overlap one wave's LDS reads and barrier
// waits with the other's MFMAs.  The wider the block the fewer operand bytes per flop cross L2 and LDS.  A grid
// that does not fill the 256 CUs in whole rounds wastes the remainder, so narrow outputs (N = d_model) are
// also split along K over blocks that meet.
struct TilePick { int tile, ksplit; };
constexpr int kNumTiles = 8;
static const int kTileM[kNumTiles] = {12, 12, 12, 12, 8, 6, 12, 16};
static const int kTileN[kNumTiles] = {24, 16, 12, 8, 8, 8, 20, 16};
static const int kTileWaves[kNumTiles] = {8, 8, 8, 8, 4, 4, 8, 8};
// What a k-step is taken to cost with all 256 CUs busy (us): for residual products as it was measured alone with an
// earlier main loop (tile_cost), for the others as fitted in whole steps with the present one.
static const float kTileUsAlone[kNumTiles] = {0.89f, 0.66f, 0.53f, 0.46f, 0.53f, 0.45f, 0.78f, 0.80f};
static const float kTileUs[kNumTiles] = {0.762f, 0.557f, 0.470f, 0.423f, 0.f, 0.f, 0.651f, 0.656f};

// floats of the pieces that the blocks of K split ks exchange
static size_t meet_floats(const TilePick& t, int MT, int total_nt) {
  return (size_t)((MT + kTileM[t.tile] - 1) / kTileM[t.tile]) * ((total_nt + kTileN[t.tile] - 1) / kTileN[t.tile]) *
         t.ksplit * kTileM[t.tile] * kTileN[t.tile] * 256;
}

// What a launch of block shape i is expected to take beside what all shapes share (us); a K split's blocks run in
// one round.
//   Residual products: kTileUsAlone and the epilogue per 16 x 16 output fragment of a block, the residual stream's
// read and write or the exchange of a K split (the ranges are not counted, though two exchange less than four).
//   The others: kTileUs, a last round that costs the less the fewer of its compute units work, and the
// epilogue.  Fitted to every shape's time by events in whole steps (60 sizes: 112 - 24576 rows, d 512 - 4096, F 2048 - 18944).
// Against the best of all shapes and splits there, the picks take 1.6 % longer on average for residual
// products (24 % at most: O of 1536 -> 1536 at 1536 rows, where 192 x 128 x 2 beats 192 x 192 x 4), 0.0 % for q k v
// (1.3 % at most) and 0.2 % for gate/up (7 %).  With the residual products' costs the latter two took 5.7 and 6.1 % (50 %).
static float tile_cost(int epi, int i, int tiles, int KB, int ks) {
  const int frags = kTileM[i] * kTileN[i], full = tiles * ks / 256, rest = tiles * ks % 256;
  if (epi == EPI_RESID)
    return (full + (rest > 0)) * ((KB + ks - 1) / ks * kTileUsAlone[i] + 5.0f + (ks > 1 ? 0.07f : 0.008f) * frags);
  const float loop = KB * kTileUs[i], ends = epi == EPI_QKV ? 1.1f + 0.045f * frags : 0.026f * frags;
  return full * (loop + ends) + (rest ? loop * (0.76f + 0.24f / 256 * rest) + ends : 0.f);
}

static TilePick pick_tile(int epi, int MT, int total_nt, int KB, int max_ksplit, size_t piece_floats) {
  TilePick best{1, 1};
  float best_t = 1e30f;
  for (int i = 0; i < kNumTiles; ++i) {
    if (kTileWaves[i] == 4 && epi != EPI_RESID) continue;
    const int gm = (MT + kTileM[i] - 1) / kTileM[i], gn = (total_nt + kTileN[i] - 1) / kTileN[i], tiles = gm * gn;
    for (int ks = 1; ks <= max_ksplit && ks <= KB; ++ks) {
      if (ks > 1 && (tiles > kMeetSlots || meet_floats(TilePick{i, ks}, MT, total_nt) > piece_floats)) break;
      if (ks > 1 && tiles * ks > 256) break;
      const float t = tile_cost(epi, i, tiles, KB, ks);
      if (t < best_t) { best_t = t; best = TilePick{i, ks}; }
    }
  }
  return best;
}

// WS: the matrix carries per-row scales (it came as e4m3 codes): a variant of its own, so that
// the kernels of plain bf16 models are compiled exactly as they were tuned
template <int EPI, bool WS, int Z>
static void launch_tiled_pick_ws(const bf16_t* Ap, int MT, const bf16_t* Wp, int total_nt, int KB,
                                 const GemmEpi& e, hipStream_t s, int tile) {
  switch (tile) {
    case 0: launch_tiled8_t<EPI, WS, Z, 2, 4, 6, 6>(Ap, MT, Wp, total_nt, KB, e, s); break;
    case 1: launch_tiled8_t<EPI, WS, Z, 2, 4, 6, 4>(Ap, MT, Wp, total_nt, KB, e, s); break;
    case 2: launch_tiled8_t<EPI, WS, Z, 2, 4, 6, 3>(Ap, MT, Wp, total_nt, KB, e, s); break;
    case 3: launch_tiled8_t<EPI, WS, Z, 2, 4, 6, 2>(Ap, MT, Wp, total_nt, KB, e, s); break;
    case 4: if constexpr (EPI == EPI_RESID) launch_tiled4_t<WS, Z, 4, 4>(Ap, MT, Wp, total_nt, KB, e, s); break;
    case 5: if constexpr (EPI == EPI_RESID) launch_tiled4_t<WS, Z, 3, 4>(Ap, MT, Wp, total_nt, KB, e, s); break;
    case 6: launch_tiled8_t<EPI, WS, Z, 2, 4, 6, 5>(Ap, MT, Wp, total_nt, KB, e, s); break;
    default: launch_tiled8_t<EPI, WS, Z, 2, 4, 8, 4>(Ap, MT, Wp, total_nt, KB, e, s); break;
  }
}

template <int EPI, bool WS>
static void launch_tiled_pick_z(const bf16_t* Ap, int MT, const bf16_t* Wp, int total_nt, int KB,
                                const GemmEpi& e, hipStream_t s, const TilePick& tp) {
  if constexpr (EPI == EPI_RESID) {
    switch (tp.ksplit) {
      case 4: launch_tiled_pick_ws<EPI, WS, 4>(Ap, MT, Wp, total_nt, KB, e, s, tp.tile); return;
      case 3: launch_tiled_pick_ws<EPI, WS, 3>(Ap, MT, Wp, total_nt, KB, e, s, tp.tile); return;
      case 2: launch_tiled_pick_ws<EPI, WS, 2>(Ap, MT, Wp, total_nt, KB, e, s, tp.tile); return;
      default: break;
    }
  }
  launch_tiled_pick_ws<EPI, WS, 1>(Ap, MT, Wp, total_nt, KB, e, s, tp.tile);
}

// The row tiles that the shape is picked for.  Only tiles that hold rows are computed, so it is the rows' own, from
// 16 k-steps on: 368 rows, gate/up of d 4096 88 -> 72 us, of 3584 132 -> 88; 848 rows 167 -> 147 and 222 -> 185.
// Residual products, whose costs were fitted to the padded row list, and the few microseconds of a shorter K keep to
// that, unless a third of it or more is padding (272 rows in a list of 512, down projection of 4096: 192 x 256 x 4
// 65.8 us, 192 x 128 x 4 55.7).
static int pick_rows(int epi, int M_src, int M, int KB) {
  const int padded = (M_src + 15) / 16, rows = (M + 15) / 16;
  return (epi != EPI_RESID && KB >= 16) || 3 * rows <= 2 * padded ? rows : padded;
}

// row tiles up to which a product goes to the weight-streaming kernels (gathered LM-head rows: 64 at most)
static bool streams_weights(int epi, int MT) { return MT <= (epi == EPI_LOGITS ? 4 : 6); }

// K ranges that a residual product may be divided into, as far as the caller has room for it
static int max_ksplit(int epi, const GemmEpi& e) {
  return epi == EPI_RESID && e.partial && e.meet ? kMaxKSplit : 1;
}

bool gemm_bf16_block_shape(int epi, int M_src, int M, int N, int K, size_t piece_floats, int shape[3]) {
  if (streams_weights(epi, (M + 15) / 16)) return false;
  const TilePick tp = pick_tile(epi, pick_rows(epi, M_src, M, K / 32), N / 16, K / 32, epi == EPI_RESID ? kMaxKSplit : 1, piece_floats);
  shape[0] = kTileM[tp.tile] * 16; shape[1] = kTileN[tp.tile] * 16; shape[2] = tp.ksplit;
  return true;
}

template <int EPI>
static void launch_epi(const bf16_t* Ap, int M_src, const bf16_t* Wp, const void* Wq, int N, int K,
                       const GemmEpi& e, hipStream_t s) {
  const int total_nt = N / 16, KB = K / 32, MT = (e.M + 15) / 16, MT_src = (M_src + 15) / 16;
  if (Wq && streams_weights(EPI, MT)) {  // weight streaming from e4m3 codes
    switch (MT) {
      case 1: launch_skinny_mt_w8<EPI, 1>(Ap, MT_src, Wq, total_nt, K / 64, e, s); break;
      case 2: launch_skinny_mt_w8<EPI, 2>(Ap, MT_src, Wq, total_nt, K / 64, e, s); break;
      case 3: launch_skinny_mt_w8<EPI, 3>(Ap, MT_src, Wq, total_nt, K / 64, e, s); break;
      case 4: launch_skinny_mt_w8<EPI, 4>(Ap, MT_src, Wq, total_nt, K / 64, e, s); break;
      case 5: if constexpr (EPI != EPI_LOGITS) launch_skinny_mt_w8<EPI, 5>(Ap, MT_src, Wq, total_nt, K / 64, e, s); break;
      default: if constexpr (EPI != EPI_LOGITS) launch_skinny_mt_w8<EPI, 6>(Ap, MT_src, Wq, total_nt, K / 64, e, s); break;
    }
    return;
  }
  // Up to 96 rows (a block of 32 plus the paper's default budget of 64 recent tokens) the GEMMs
  // are weight-streaming: eight layers of d 4096, F 12288 take 0.93 ms a step at 64 rows and 1.10 at 96, against 1.76
  // and 1.85 through the tiled kernels.
  if (streams_weights(EPI, MT)) {
    switch (MT) {
      case 1: launch_skinny_mt<EPI, 1>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 2: launch_skinny_mt<EPI, 2>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 3: launch_skinny_mt<EPI, 3>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 4: launch_skinny_mt<EPI, 4>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      case 5: if constexpr (EPI != EPI_LOGITS) launch_skinny_mt<EPI, 5>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
      default: if constexpr (EPI != EPI_LOGITS) launch_skinny_mt<EPI, 6>(Ap, MT_src, Wp, total_nt, KB, e, s); break;
    }
  } else {
    // the tiled kernel reads its activation rows in place (no gather); only the tiles that hold rows
    // below e.M are computed (the buffer is padded to 256 rows), and rows from e.M on are dropped
    const TilePick tp = pick_tile(EPI, pick_rows(EPI, M_src, e.M, KB), total_nt, KB, max_ksplit(EPI, e), e.partial_floats);
    if (e.wscale) launch_tiled_pick_z<EPI, true>(Ap, MT_src, Wp, total_nt, KB, e, s, tp);
    else launch_tiled_pick_z<EPI, false>(Ap, MT_src, Wp, total_nt, KB, e, s, tp);
  }
}

void launch_gemm_bf16(int epi, const bf16_t* Ap, int M_src, const bf16_t* Wp, const void* Wq,
                      int N, int K, const GemmEpi& e, hipStream_t s) {
  if (e.M <= 0) return;
  switch (epi) {
    case EPI_QKV: launch_epi<EPI_QKV>(Ap, M_src, Wp, Wq, N, K, e, s); break;
    case EPI_RESID: launch_epi<EPI_RESID>(Ap, M_src, Wp, Wq, N, K, e, s); break;
    case EPI_SWIGLU: launch_epi<EPI_SWIGLU>(Ap, M_src, Wp, Wq, N, K, e, s); break;
    default:
      // Up to 64 rows the skinny kernel gathers the rows row_sel names out of Ap itself.  More
      // rows go through the tiled kernels, which read their rows in place: the caller hands
      // over the gathered rows then (row_sel still names the rows whose 1/rms applies).
      launch_epi<EPI_LOGITS>(Ap, M_src, Wp, Wq, N, K, e, s);
      break;
  }
}

}  // namespace ec
