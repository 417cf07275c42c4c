// Non-causal attention of the recomputed rows against the whole cached context
// ("TransformerBlock(Q_[M u R], K_[I], V_[I])" of the appendix algorithm): every query row
// attends all T cached positions, no mask.
//
// Float32 path (row-major caches [T, Hkv*hd]) on v_mfma_f32_16x16x4_f32.  A block owns 16 query
// rows of one head; its 8 waves stride over 16-key tiles with an online softmax each and are merged
// through LDS in wave order.  Per tile:
//   S^T[keys x queries] = K Q^T      lane g*16 + r loads key r, columns 16 c + 4 g .. + 3
//   O^T[hd x queries] += V^T P^T     the lane's 4 scores (keys 4 g .. + 3 of query r) ARE the second
//                                    product's operand
// 16 rows share every key and value that is read.  128 rows, 128 keys, 4 heads: 6.8 us a launch,
// 12.6 us with a block per row and head.
// The bf16 path uses the kernels of k_attn_mfma.hip.
#include "ec_internal.h"

namespace ec {

template <int HD>
__global__ __launch_bounds__(512) void attn_f32_kernel(const float* __restrict__ q,
                                                       const float* __restrict__ kc,
                                                       const float* __restrict__ vc, int M, int T,
                                                       int Hq, int Hkv, float scale,
                                                       float* __restrict__ out) {
  constexpr int NW = 8, HC = HD / 16;
  __shared__ float4 so[NW][HC][64];
  __shared__ float2 sml[NW][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4, head = blockIdx.y, kvh = head / (Hq / Hkv);
  const int nq = Hq * HD, nkv = Hkv * HD;
  const int m = blockIdx.x * 16 + r16;
  const float* qp = q + (size_t)min(m, M - 1) * nq + head * HD;   // (rows past the end: not stored)
  f32x4 qf[HC], acc[HC];
#pragma unroll
  for (int c = 0; c < HC; ++c) {
    qf[c] = *(const f32x4*)(qp + c * 16 + g * 4);
    acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  float m_run = -INFINITY, l_run = 0.f;
  const int nt = (T + 15) >> 4;
  for (int t = wave; t < nt; t += NW) {
    const float* kp = kc + (size_t)min(t * 16 + r16, T - 1) * nkv + kvh * HD;
    f32x4 kf[HC], vf[HC];
#pragma unroll
    for (int c = 0; c < HC; ++c) kf[c] = *(const f32x4*)(kp + c * 16 + g * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* vp = vc + (size_t)min(t * 16 + g * 4 + e, T - 1) * nkv + kvh * HD;
#pragma unroll
      for (int c = 0; c < HC; ++c) vf[c][e] = vp[c * 16 + r16];
    }
    f32x4 s4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < HC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        s4 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], s4, 0, 0, 0);
    float mx = m_run;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s4[e] = t * 16 + g * 4 + e < T ? s4[e] * scale : -INFINITY;
      mx = fmaxf(mx, s4[e]);
    }
    mx = fmaxf(mx, other_row(mx));
    mx = fmaxf(mx, other_half(mx));
    const float alpha = expf(m_run - mx);      // (a tile has a real key: mx is its score at least)
    float l = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s4[e] = expf(s4[e] - mx);
      l += s4[e];
    }
    l += other_row(l);
    l += other_half(l);
    l_run = l_run * alpha + l;
    m_run = mx;
#pragma unroll
    for (int c = 0; c < HC; ++c) {
      f32x4 a = acc[c];
      a[0] *= alpha; a[1] *= alpha; a[2] *= alpha; a[3] *= alpha;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        a = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][e], s4[e], a, 0, 0, 0);
      acc[c] = a;
    }
  }
#pragma unroll
  for (int c = 0; c < HC; ++c) so[wave][c][lane] = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
  sml[wave][lane] = make_float2(m_run, l_run);
  __syncthreads();
  float wgt[NW], m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, sml[w][lane].x);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wgt[w] = sml[w][lane].y > 0.f ? expf(sml[w][lane].x - m_all) : 0.f;   // (a wave without keys)
    l_all += sml[w][lane].y * wgt[w];
  }
  for (int c = wave; c < HC; c += NW) {
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 v = so[w][c][lane];
      o.x += v.x * wgt[w]; o.y += v.y * wgt[w]; o.z += v.z * wgt[w]; o.w += v.w * wgt[w];
    }
    if (m < M)
      *(float4*)(out + (size_t)m * nq + head * HD + c * 16 + g * 4) =
          make_float4(o.x / l_all, o.y / l_all, o.z / l_all, o.w / l_all);
  }
}

void launch_attention_f32(const float* q, const float* kc, const float* vc, int M, int T, int Hq,
                          int Hkv, int hd, float* out, hipStream_t s) {
  if (M <= 0) return;
  const dim3 grid((M + 15) / 16, Hq);
  const float scale = 1.0f / sqrtf((float)hd);
  if (hd == 64)
    attn_f32_kernel<64><<<grid, 512, 0, s>>>(q, kc, vc, M, T, Hq, Hkv, scale, out);
  else
    attn_f32_kernel<128><<<grid, 512, 0, s>>>(q, kc, vc, M, T, Hq, Hkv, scale, out);
}

}  // namespace ec
