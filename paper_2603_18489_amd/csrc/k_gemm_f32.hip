// float32 GEMMs on MFMA (v_mfma_f32_16x16x4_f32: float32 products and sums) with the layer's
// element-wise work fused in, for the float32 model path: C[M,N] = A[M,K] W[N,K]^T, both operands
// row-major and K-contiguous.
//
// These models are small: a launch has to be one short trip to memory, spread over many blocks.
// A block owns TN x TM output tiles of 16 x 16 and its KS waves split K; each wave requests four
// 16-wide k-chunks of every operand before the first product.  The weight tile is the MFMA "A"
// operand (16 weight rows), the activation tile the "B" operand: lane g*16 + r loads row r,
// k = 16 c + 4 g .. + 3 as one float4, and product s of the chunk takes element s, so both operands
// run through k in the same order.  A lane of the result holds 4 consecutive output features of
// one activation row.  The waves' tiles are summed through LDS in wave order.
//
// RMSNorm is folded in where the operand is normed: the products take h * gain, the row's sum of
// squares is gathered from the very loads that feed them (every block reads its rows whole), and
// 1/rms multiplies the sums.
//
//   F32_QKV     x 1/rms, rotary embedding on q and k, q -> query buffer, k / v -> cache rows.  A q
//               or k tile holds 8 columns of a head and their 8 partners hd/2 further on, so a
//               rotation pair meets in lanes l and l + 32; v tiles are in natural order.
//   F32_RESID   h += result
//   F32_SWIGLU  x 1/rms, silu(gate) * up (8 gate rows and their 8 up rows share a tile)
//   F32_LOGITS  x 1/rms x logit scale -> logits, and the block's columns of every row reduced to one
//               (max, argmax, sum e, sum e (z - max)) tuple for the decision kernel
//
// On MI355X the 64-step generation of the smallest model (2 layers, d 256, feed-forward 768,
// vocabulary 4096, 128 positions) takes 5.2 ms, 5 launches per layer; 40 ms with 64 x 64 tiles of
// scalar loads (8 blocks for N = 256, 30 - 43 us a launch) and norm, rotation and SwiGLU as kernels
// of their own.
#include "ec_internal.h"
#include "k_vtuple.h"

namespace ec {

template <bool VEC> __device__ __forceinline__ f32x4 load4(const float* p) {
  if constexpr (VEC) return *(const f32x4*)p;
  return (f32x4){p[0], p[1], p[2], p[3]};
}

template <int EPI, int TN, int TM, int KS, bool VEC>
__global__ __launch_bounds__(KS * 64) void gemm_f32_kernel(F32Gemm g) {
  constexpr bool NORMED = EPI != F32_RESID;
  constexpr int U = 4;
  __shared__ float4 red[KS][TN * TM][64];
  __shared__ float ssq[KS][TM * 16];
  __shared__ float4 tup[TN][TM * 16];   // F32_LOGITS
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;
  const int nt0 = blockIdx.x * TN, mt0 = blockIdx.y * TM;
  const int hd = g.hd, tph = hd >> 4, nqt = g.Hq * tph, nkt = g.Hkv * tph;

  // Rows and tiles past the end read the last ones instead (valid memory); nothing of them is stored.
  const float* wp[TN];
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    const int vt = min(nt0 + i, g.nt - 1);
    const float* W = g.W[0];
    int row;
    if constexpr (EPI == F32_QKV) {
      const int t = vt < nqt ? vt : vt < nqt + nkt ? vt - nqt : vt - nqt - nkt;
      W = vt < nqt ? g.W[0] : vt < nqt + nkt ? g.W[1] : g.W[2];
      row = vt < nqt + nkt ? t / tph * hd + t % tph * 8 + (r16 & 7) + (r16 < 8 ? 0 : hd >> 1)
                           : t * 16 + r16;
    } else if constexpr (EPI == F32_SWIGLU) {
      W = r16 < 8 ? g.W[0] : g.W[1];
      row = vt * 8 + (r16 & 7);
    } else {
      row = min(vt * 16 + r16, g.N - 1);
    }
    wp[i] = W + (size_t)row * g.K;
  }
  const float* ap[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = min((mt0 + j) * 16 + r16, g.M - 1);
    ap[j] = g.A + (size_t)(g.sel ? g.sel[m] : m) * g.K;
  }

  f32x4 acc[TN][TM];
  float ss[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    ss[j] = 0.f;
#pragma unroll
    for (int i = 0; i < TN; ++i) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const int KC = (g.K + 15) >> 4, c_lo = wave * KC / KS, c_hi = (wave + 1) * KC / KS;
  for (int c = c_lo; c < c_hi; c += U) {
    f32x4 a[U][TM], w[U][TN], gn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (K is a multiple of 8: a lane's four k are all inside or all outside; loads past the end
      // go to k = 0 and count as zeros)
      const int k = (c + u) * 16 + q4 * 4;
      const bool in = c + u < c_hi && k < g.K;
      const int kk = in ? k : 0;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < TM; ++j) { a[u][j] = load4<true>(ap[j] + kk); if (!in) a[u][j] = zero; }
#pragma unroll
      for (int i = 0; i < TN; ++i) { w[u][i] = load4<VEC>(wp[i] + kk); if (!in) w[u][i] = zero; }
      if constexpr (NORMED) { gn[u] = load4<VEC>(g.gain + kk); if (!in) gn[u] = zero; }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        f32x4 x = a[u][j];
        if constexpr (NORMED) {
          ss[j] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
          x[0] *= gn[u][0]; x[1] *= gn[u][1]; x[2] *= gn[u][2]; x[3] *= gn[u][3];
        }
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int s = 0; s < 4; ++s)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][s], x[s], acc[i][j], 0, 0, 0);
      }
  }
#pragma unroll
  for (int j = 0; j < TM; ++j) {
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const f32x4 v = acc[i][j];
      red[wave][i * TM + j][lane] = make_float4(v[0], v[1], v[2], v[3]);
    }
    if constexpr (NORMED) {
      float s = ss[j];
      s += other_row(s);
      s += other_half(s);
      if (lane < 16) ssq[wave][j * 16 + r16] = s;
    }
  }
  __syncthreads();

  for (int tile = wave; tile < TN * TM; tile += KS) {
    const int i = tile / TM, j = tile - i * TM, vt = nt0 + i, m = (mt0 + j) * 16 + r16;
    float4 v = red[0][tile][lane];
#pragma unroll
    for (int k = 1; k < KS; ++k) {
      const float4 p = red[k][tile][lane];
      v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    if constexpr (NORMED) {
      float s = ssq[0][j * 16 + r16];
#pragma unroll
      for (int k = 1; k < KS; ++k) s += ssq[k][j * 16 + r16];
      const float rs = 1.0f / sqrtf(s / (float)g.K + g.eps) * (EPI == F32_LOGITS ? g.scale : 1.f);
      v.x *= rs; v.y *= rs; v.z *= rs; v.w *= rs;
    }
    const bool valid = m < g.M && vt < g.nt;   // (lanes l and l + 32 share the row: both or neither)
    if constexpr (EPI == F32_QKV) {
      const float x[4] = {v.x, v.y, v.z, v.w};
      float y[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = other_half(x[r]);
      if (!valid) continue;
      const int pos = g.rows ? g.rows[m] : m, nkv = g.Hkv * hd;
      if (vt < nqt + nkt) {
        const bool is_q = vt < nqt, hi = q4 >= 2;
        const int t = is_q ? vt : vt - nqt, col = t % tph * 8 + (q4 & 1) * 4;
        const float2* cs = g.cs + (size_t)pos * (hd >> 1) + col;
        float4 o;
        float* op = &o.x;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          op[r] = hi ? x[r] * cs[r].x + y[r] * cs[r].y : x[r] * cs[r].x - y[r] * cs[r].y;
        float* dst = is_q ? g.C + (size_t)m * (g.Hq * hd) : g.kc + (size_t)pos * nkv;
        *(float4*)(dst + t / tph * hd + col + (hi ? hd >> 1 : 0)) = o;
      } else {
        *(float4*)(g.vc + (size_t)pos * nkv + (vt - nqt - nkt) * 16 + q4 * 4) = v;
      }
    } else if constexpr (EPI == F32_SWIGLU) {
      const float x[4] = {v.x, v.y, v.z, v.w};
      float4 o;
      float* op = &o.x;
#pragma unroll
      for (int r = 0; r < 4; ++r) op[r] = x[r] / (1.0f + expf(-x[r])) * other_half(x[r]);
      if (valid && q4 < 2) *(float4*)(g.C + (size_t)m * g.ldc + vt * 8 + q4 * 4) = o;
    } else if constexpr (EPI == F32_RESID) {
      const int n = vt * 16 + q4 * 4;
      if (valid && n < g.N) {
        float4* h = (float4*)(g.C + (size_t)m * g.ldc + n);
        float4 o = *h;
        o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
        *h = o;
      }
    } else {
      // A row's 16 columns of the tile sit in lanes l, l^16, l^32, l^48, four each; columns past the
      // vocabulary (any number; rows start anywhere) have probability 0.
      const int n = vt * 16 + q4 * 4;
      float z[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (vt >= g.nt || n + r >= g.N) z[r] = -INFINITY;
        else if (m < g.M) g.C[(size_t)m * g.ldc + n + r] = z[r];
      }
      float mx = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
      mx = fmaxf(mx, other_row(mx));
      mx = fmaxf(mx, other_half(mx));
      int idx = z[0] == mx ? n : z[1] == mx ? n + 1 : z[2] == mx ? n + 2 : z[3] == mx ? n + 3 : INT_MAX;
      idx = min(idx, __float_as_int(other_row(__int_as_float(idx))));
      idx = min(idx, __float_as_int(other_half(__int_as_float(idx))));
      float s4 = 0.f, t4 = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float d = z[r] - mx, ex = z[r] == -INFINITY ? 0.f : expf(d);
        s4 += ex;
        t4 += z[r] == -INFINITY ? 0.f : ex * d;
      }
      s4 += other_row(s4); t4 += other_row(t4);
      s4 += other_half(s4); t4 += other_half(t4);
      if (q4 == 0) tup[i][j * 16 + r16] = make_float4(mx, __int_as_float(idx), s4, t4);
    }
  }
  if constexpr (EPI == F32_LOGITS) {
    __syncthreads();
    const int m = mt0 * 16 + (int)threadIdx.x;
    if (threadIdx.x < TM * 16 && m < g.M) {
      VTuple t = vt_unpack(tup[0][threadIdx.x]);
#pragma unroll
      for (int i = 1; i < TN; ++i) t = vt_merge(t, vt_unpack(tup[i][threadIdx.x]));
      g.vparts[(size_t)m * gridDim.x + blockIdx.x] = vt_pack(t);
    }
  }
}

template <int EPI, int T, int KS, bool VEC>
static void launch_f32_t(const F32Gemm& g, hipStream_t s) {
  const dim3 grid((g.nt + T - 1) / T, ((g.M + 15) / 16 + T - 1) / T);
  gemm_f32_kernel<EPI, T, T, KS, VEC><<<grid, KS * 64, 0, s>>>(g);
}

// One 16 x 16 tile to a block spreads a small product over the chip; where there are more than two
// blocks to a compute unit, four tiles to a block halve what is read.  A wave should have all its
// k-chunks in flight at once: four waves hold K = 256, beyond that eight.  us per launch on MI355X:
//   down     K  768,   32 tiles   1x1 4 waves  9.1 (with O)   8 waves 6.8   2x2 8 waves 11.5
//   q k v    K  256,   96 tiles   1x1 4 waves  4.5            8 waves 5.6   2x2 4 waves  6.5
//   gate/up  K  256,  768 tiles   1x1 4 waves  7.2            8 waves 10.6  2x2 4 waves  6.5
//   gate/up  K  512, 3456 tiles   1x1 8 waves 33.2   2x2 4 waves 21.4       2x2 8 waves 22.0
//   O, down  K 1536,  576 tiles   1x1 8 waves 13.6   2x2 4 waves 15.8       2x2 8 waves 12.0
// Weights that are not 16-byte aligned are read by single elements and take the same two block
// shapes, eight waves each; LM head and decision at 128 rows, four tiles instead of one to a block:
// K 256, vocabulary 126464: 690 -> 404; K 512, 151936: 1230 -> 667 (half the tuples to merge, too).
template <int EPI>
static int launch_f32(const F32Gemm& g, bool vec, hipStream_t s) {
  const bool few = (long)g.nt * ((g.M + 15) / 16) <= 512, short_k = g.K <= 256;
  if (!vec) {
    if (few) launch_f32_t<EPI, 1, 8, false>(g, s);
    else launch_f32_t<EPI, 2, 8, false>(g, s);
  } else if (few && short_k) launch_f32_t<EPI, 1, 4, true>(g, s);
  else if (few) launch_f32_t<EPI, 1, 8, true>(g, s);
  else if (short_k) launch_f32_t<EPI, 2, 4, true>(g, s);
  else launch_f32_t<EPI, 2, 8, true>(g, s);
  return few ? g.nt : (g.nt + 1) / 2;
}

int launch_gemm_f32(int epi, F32Gemm g, hipStream_t s) {
  if (g.M <= 0) return 0;
  g.nt = epi == F32_QKV ? (g.Hq + 2 * g.Hkv) * (g.hd / 16)
       : epi == F32_SWIGLU ? g.N / 8 : (g.N + 15) / 16;
  // the caller's tensors may start at any element; the workspace is aligned
  const bool vec = (((uintptr_t)g.W[0] | (uintptr_t)g.W[1] | (uintptr_t)g.W[2] | (uintptr_t)g.gain) & 15) == 0;
  switch (epi) {
    case F32_QKV: return launch_f32<F32_QKV>(g, vec, s);
    case F32_RESID: return launch_f32<F32_RESID>(g, vec, s);
    case F32_SWIGLU: return launch_f32<F32_SWIGLU>(g, vec, s);
    default: return launch_f32<F32_LOGITS>(g, vec, s);
  }
}

}  // namespace ec
