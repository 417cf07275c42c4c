// (max, argmax, sum e^(z-max), sum e^(z-max) (z-max)) tuples: the one-pass form of Eq. 1.
// A row's softmax statistics follow from its tuple: confidence = 1 / S, entropy = ln S - T / S.
// Tuples of disjoint parts of the vocabulary merge associatively (re-basing both to the common
// maximum), so partial reductions can be combined in any FIXED order with bit-reproducible
// results.  Shared by the decision kernels and the LM-head epilogue.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>

#include "k_common.h"
#include "k_exp.h"

namespace ec {

struct VTuple {
  float m;   // running maximum
  int idx;   // its index (lowest index among equal maxima)
  float s;   // sum exp(z - m)
  float t;   // sum exp(z - m) * (z - m)
};

__device__ __forceinline__ VTuple vt_identity() { return {-INFINITY, INT_MAX, 0.f, 0.f}; }

// sum e^(z-m') (z-m') of a tuple for a maximum m' = m - d no smaller than its own, e = e^d.  Where e is 0 so is the sum, also when d
// times s is past the type's range (parts of a row at its lowest value, as masks leave them); -200 is past the last e that is not.
__device__ __forceinline__ float vt_rebased_t(float s, float t, float d, float e) { return e * (t + fmaxf(d, -200.f) * s); }

// Associative merge: re-base both sides to the common maximum.
__device__ __forceinline__ VTuple vt_merge(const VTuple& a, const VTuple& b) {
  if (b.s == 0.f) return a;
  if (a.s == 0.f) return b;
  VTuple r;
  bool a_wins = (a.m > b.m) || (a.m == b.m && a.idx < b.idx);
  r.m = fmaxf(a.m, b.m);
  r.idx = a_wins ? a.idx : b.idx;
  float da = a.m - r.m, db = b.m - r.m;  // <= 0
  float ea = expf(da), eb = expf(db);
  r.s = a.s * ea + b.s * eb;
  r.t = vt_rebased_t(a.s, a.t, da, ea) + vt_rebased_t(b.s, b.t, db, eb);
  return r;
}

// Tuple of NE * 64 consecutive logits held by one wave (lane l: elements first + 64 u + l, -inf for
// those past the end).  The maximum comes first, so every logit then costs one exponential and no branch.  A logit of
// -inf has probability 0 and contributes 0 (0 ln 0 := 0); a NaN makes the sums NaN.  All lanes return the same tuple.
template <int NE>
__device__ __forceinline__ VTuple vt_of_wave(const float (&z)[NE], int first) {
  static_assert(NE % 4 == 0, "taken four at a time");
  const int lane = threadIdx.x & 63;
  float four[NE / 4], m = -INFINITY;
#pragma unroll
  for (int g = 0; g < NE / 4; ++g) {
    four[g] = fmaxf(fmaxf(z[4 * g], z[4 * g + 1]), fmaxf(z[4 * g + 2], z[4 * g + 3]));
    m = fmaxf(m, four[g]);
  }
  VTuple v;
  v.m = wave_max_dpp(fmaxf(m, -INFINITY));   // (a lane of NaNs must not hand one on)
  if (!(fabsf(v.m) < INFINITY)) {
    // Nothing finite (all -inf or NaN), or a +inf: not a distribution, unless the +inf is alone.
    int n_inf = 0, n_other = 0;
    v.idx = INT_MAX;
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const bool top = z[u] == INFINITY;
      n_inf += top;
      n_other += !top && z[u] != -INFINITY;
      if (top) v.idx = min(v.idx, first + u * 64 + lane);
    }
    v.idx = wave_min_dpp(v.idx);
    n_inf = (int)wave_sum_dpp((float)n_inf);
    n_other = (int)wave_sum_dpp((float)n_other);
    v.s = n_other > 0 || n_inf > 1 ? __builtin_nanf("") : (float)n_inf;
    v.t = n_other > 0 || n_inf > 1 ? __builtin_nanf("") : 0.f;
    return v;
  }
  float s = 0.f, t = 0.f;
  unsigned long long nan = 0;
#pragma unroll
  for (int u = NE - 1; u >= 0; --u) {
    if (u & 1) nan |= __builtin_amdgcn_ballot_w64(__builtin_isunordered(z[u], z[u - 1]));
    const float d = fmaxf(z[u] - v.m, -200.f), e = exp_of_negative(d);   // (-inf: e = 0; a NaN is seen above)
    s += e;
    t = fmaf(e, d, t);
  }
  // The lowest index that holds the maximum: the lowest four of the lanes' elements that have it, then the lowest of these.
  int at = 0;
#pragma unroll
  for (int g = NE / 4 - 1; g >= 0; --g)
    if (__builtin_amdgcn_ballot_w64(four[g] == v.m)) {
#pragma unroll
      for (int u = 4 * g + 3; u >= 4 * g; --u) {
        const unsigned long long has = __builtin_amdgcn_ballot_w64(z[u] == v.m);
        at = has ? u * 64 + __builtin_ctzll(has) : at;
      }
    }
  v.idx = first + at;
  v.s = wave_sum_dpp(s);
  v.t = wave_sum_dpp(t);
  if (nan) v.s = v.t = __builtin_nanf("");
  return v;
}

__device__ __forceinline__ VTuple vt_of_lane(const VTuple& v, int l) {
  return VTuple{__shfl(v.m, l, 64), __shfl(v.idx, l, 64), __shfl(v.s, l, 64), __shfl(v.t, l, 64)};
}

// The tuples of N neighbouring lanes (2, 4, 8, 16 or 32) merged at once: every lane re-bases its own to the
// common maximum (one exponential), then the sums go through lane exchanges.  All N lanes return the result.
template <int N> __device__ __forceinline__ VTuple vt_merge_lanes(const VTuple& v) {
  VTuple r;
  float m = v.m;
  m = fmaxf(m, dpp_f<0xB1>(m));
  if (N > 2) m = fmaxf(m, dpp_f<0x4E>(m));
  if (N > 4) m = fmaxf(m, dpp_f<0x141>(m));
  if (N > 8) m = fmaxf(m, dpp_f<0x140>(m));
  if (N > 16) m = fmaxf(m, other_row(m));
  r.m = m;
  int idx = v.s != 0.f && v.m == r.m ? v.idx : INT_MAX;
  idx = min(idx, dpp_i<0xB1>(idx));
  if (N > 2) idx = min(idx, dpp_i<0x4E>(idx));
  if (N > 4) idx = min(idx, dpp_i<0x141>(idx));
  if (N > 8) idx = min(idx, dpp_i<0x140>(idx));
  if (N > 16) idx = min(idx, __float_as_int(other_row(__int_as_float(idx))));
  r.idx = idx;
  const float d = v.m - r.m, e = expf(d);
  float s = v.s != 0.f ? v.s * e : 0.f, t = v.s != 0.f ? vt_rebased_t(v.s, v.t, d, e) : 0.f;
  s += dpp_f<0xB1>(s); t += dpp_f<0xB1>(t);
  if (N > 2) { s += dpp_f<0x4E>(s); t += dpp_f<0x4E>(t); }
  if (N > 4) { s += dpp_f<0x141>(s); t += dpp_f<0x141>(t); }
  if (N > 8) { s += dpp_f<0x140>(s); t += dpp_f<0x140>(t); }
  if (N > 16) { s += other_row(s); t += other_row(t); }
  r.s = s;
  r.t = t;
  return r;
}
__device__ __forceinline__ float4 vt_pack(const VTuple& v) {
  return make_float4(v.m, __int_as_float(v.idx), v.s, v.t);
}
__device__ __forceinline__ VTuple vt_unpack(const float4& q) {
  return VTuple{q.x, __float_as_int(q.y), q.z, q.w};
}
// Eq. 1 from a row's merged tuple: confidence = max probability = e^0 / S, entropy
// H = -sum p ln p = ln S - T / S (clamped at 0 against rounding).
__device__ __forceinline__ void vt_finish(const VTuple& v, float& conf, float& H) {
  conf = 1.0f / v.s;
  H = fmaxf(logf(v.s) - v.t / v.s, 0.f);
}

}  // namespace ec
