// The O(V) decision of EntropyCache and the bookkeeping around it:
//   vocab_reduce : per logit row, partial (max, argmax, sum e^{z-max}, sum e^{z-max}(z-max))
//                  over chunks of the vocabulary, in one pass.
//   decide       : merges the partials (confidence = 1/S, entropy H = ln S - T/S; Eq. 1), picks
//                  the tokens to unmask (decode()), records the decode history (Eq. 2), selects
//                  the recent tokens (Eq. 3, tau_R, R), sets the skip flag (E <= tau) and builds
//                  the row set M u R of the next partial step.
// Every reduction runs in a fixed order, so results are bit-reproducible.
#include <limits.h>

#include "ec_internal.h"
#include "k_vtuple.h"

namespace ec {

constexpr int VR_CHUNK = 2048;  // logits per partial tuple

int vocab_reduce_parts(int V) { return (V + VR_CHUNK - 1) / VR_CHUNK; }

// One wave's part of a row: every logit is requested before the first is used (4-byte loads: rows
// may start anywhere, and 16-byte loads measured no faster).
__device__ __forceinline__ VTuple vocab_part(const float* __restrict__ z, int V, int part) {
  constexpr int NE = VR_CHUNK / 64;
  const int lo = part * VR_CHUNK, lane = threadIdx.x & 63;
  float v[NE];
  if (lo + VR_CHUNK <= V) {
#pragma unroll
    for (int u = 0; u < NE; ++u) v[u] = z[lo + u * 64 + lane];
  } else {
#pragma unroll
    for (int u = 0; u < NE; ++u) v[u] = lo + u * 64 + lane < V ? z[lo + u * 64 + lane] : -INFINITY;
  }
  return vt_of_wave<NE>(v, lo);
}

// grid (ceil(parts / 4), rows): one wave per partial tuple.  Bound by the logits' one pass from HBM and, behind it, the
// arithmetic of a logit, eleven instructions (two thirds of what a call of the C library's expf and an index carried in
// a register take): 128 rows of 126464 logits, 65 MB, 19.4 -> 16.6 us a call with the kernel below, 40 rows of 50000
// 8.9 -> 8.4, 128 of 16000 in one launch 7.6 -> 7.1.
__global__ __launch_bounds__(256) void vocab_reduce_kernel(const float* __restrict__ logits, int V,
                                                           size_t ld, int nparts,
                                                           float4* __restrict__ partials) {
  const int part = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (part >= nparts) return;
  const VTuple v = vocab_part(logits + (size_t)blockIdx.y * ld, V, part);
  if ((threadIdx.x & 63) == 0) partials[(size_t)blockIdx.y * nparts + part] = vt_pack(v);
}

void launch_vocab_reduce(const float* logits, int n_rows, int V, size_t ld, float4* partials,
                         hipStream_t s) {
  if (n_rows <= 0) return;
  const int nparts = vocab_reduce_parts(V);
  vocab_reduce_kernel<<<dim3((nparts + 3) / 4, n_rows), 256, 0, s>>>(logits, V, ld, nparts, partials);
}

// One wave per row: lane l merges parts l, l + 64, ..., then the lanes' tuples all at once, half a wave each; writes
// (token id as float, confidence, entropy, max logit).
__global__ __launch_bounds__(64) void row_stats_kernel(const float4* __restrict__ partials,
                                                       int nparts, float4* __restrict__ stats) {
  const int row = blockIdx.x;
  VTuple v = vt_identity();
  for (int p = threadIdx.x; p < nparts; p += 64)
    v = vt_merge(v, vt_unpack(partials[(size_t)row * nparts + p]));
  const unsigned long long any = __ballot(v.s != 0.f);
  if (__popcll(any) == 1) {                    // alone, whatever it is (a +inf cannot be re-based)
    v = vt_of_lane(v, __builtin_ctzll(any));
  } else {
    v = vt_merge_lanes<32>(v);
    v = vt_merge(v, vt_of_lane(v, 32));
  }
  if (threadIdx.x == 0) {
    float conf, H;
    vt_finish(v, conf, H);
    stats[row] = make_float4((float)v.idx, conf, H, v.m);
  }
}

// One block per row, the whole reduction in one launch: the waves take the row's parts in turn,
// merge their own in that order and then the waves' tuples in wave order.  A row is then one
// compute unit's to pull, so this is for short rows: per call 7.8 us against 10.4 us through the
// two kernels at up to 16384 logits (1 to 128 rows), 11.5 against 10.4 at 128 rows of 32768 and
// 36.8 against 18.3 at 128 rows of 126464.
constexpr int kDirectParts = 8;
template <int NW>
__global__ __launch_bounds__(NW * 64) void row_stats_direct_kernel(const float* __restrict__ logits,
                                                                   int V, size_t ld, int nparts,
                                                                   float4* __restrict__ stats) {
  __shared__ float4 wt[NW];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* z = logits + (size_t)blockIdx.x * ld;
  VTuple v = vt_identity();
  for (int p = wave; p < nparts; p += NW) v = vt_merge(v, vocab_part(z, V, p));
  if ((threadIdx.x & 63) == 0) wt[wave] = vt_pack(v);
  __syncthreads();
  if (threadIdx.x == 0) {
    VTuple r = vt_unpack(wt[0]);
#pragma unroll
    for (int w = 1; w < NW; ++w) r = vt_merge(r, vt_unpack(wt[w]));
    float conf, H;
    vt_finish(r, conf, H);
    stats[blockIdx.x] = make_float4((float)r.idx, conf, H, r.m);
  }
}

void launch_row_stats(const float* logits, int n_rows, int V, size_t ld, float4* partials,
                      float4* stats, hipStream_t s) {
  if (n_rows <= 0) return;
  const int nparts = vocab_reduce_parts(V);
  if (nparts <= kDirectParts) {
    row_stats_direct_kernel<4><<<n_rows, 256, 0, s>>>(logits, V, ld, nparts, stats);
  } else {
    launch_vocab_reduce(logits, n_rows, V, ld, partials, s);
    row_stats_kernel<<<n_rows, 64, 0, s>>>(partials, nparts, stats);
  }
}

// ---- block-wide integer helpers (kDecideThreads threads) --------------------------------------
constexpr int kDecideThreads = 1024, kDecideWaves = kDecideThreads / 64;

// Exclusive prefixes of up to four 0/1 flags over the block and their totals, one exchange for all
// of them (each count fits 16 bits).  `scratch` may be written again after the next barrier.  The first nw waves
// take part; the others only come to the barrier (and get no totals).
template <int NF>
__device__ __forceinline__ void block_excl_scan_flags(const bool (&flag)[NF], unsigned long long* scratch, int nw,
                                                      int (&prefix)[NF], int (&total)[NF]) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned long long mine = 0;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const unsigned long long ball = __ballot(flag[f]);
    prefix[f] = __popcll(ball & below);
    mine |= (unsigned long long)__popcll(ball) << (16 * f);
  }
  if (lane == 0) scratch[w] = mine;
  __syncthreads();
  unsigned long long off = 0, tot = 0;
  if (w < nw) {
#pragma unroll 4
    for (int i = 0; i < nw; ++i) {
      const unsigned long long c = scratch[i];
      off += i < w ? c : 0;
      tot += c;
    }
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    prefix[f] += (int)((off >> (16 * f)) & 0xffff);
    total[f] = (int)((tot >> (16 * f)) & 0xffff);
  }
}

// The quantity the threshold is applied to, accumulated over the newly decoded tokens: their
// maximum entropy (Eq. 1), the sum of their entropies, or their maximum confidence (the
// alternatives of the ablation on the thresholding variable).  Empty = the value that skips.
struct GateAcc { float v; int metric; };
__device__ __forceinline__ GateAcc gate_init(int metric) {
  return GateAcc{metric == EC_GATE_MAX_CONFIDENCE ? INFINITY : -INFINITY, metric};
}
__device__ __forceinline__ void gate_add(GateAcc& g, float H, float conf) {
  if (g.metric == EC_GATE_ENTROPY_SUM) g.v = (g.v == -INFINITY) ? H : g.v + H;
  else if (g.metric == EC_GATE_MAX_CONFIDENCE) g.v = (g.v == INFINITY) ? conf : fmaxf(g.v, conf);
  else g.v = fmaxf(g.v, H);
}
__device__ __forceinline__ bool gate_skips(float v, float tau, int metric) {
  return metric == EC_GATE_MAX_CONFIDENCE ? v >= tau : v <= tau;
}

// Lane l32 of a half wave merges parts l32, l32 + 32, ... of a row in that order, NU loads in flight.  The running
// tuple is re-based once per batch of NU parts (to the batch's maximum if that is larger), after which a part costs
// one fast exponential and a few FMAs.
template <int NU>
__device__ __forceinline__ VTuple merge_row_parts(const float4* __restrict__ pr, int l32, int nparts) {
  VTuple v = vt_identity();
  for (int p0 = l32; p0 < nparts; p0 += 32 * NU) {
    float4 q[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u)   // unconditional loads (clamped), so that all are in flight
      q[u] = pr[min(p0 + 32 * u, nparts - 1)];
    float bm = -INFINITY;
#pragma unroll
    for (int u = 0; u < NU; ++u) {   // (past the end: a maximum of -inf; an empty part has that, and sums of 0)
      q[u].x = p0 + 32 * u < nparts ? q[u].x : -INFINITY;
      bm = fmaxf(bm, q[u].x);
    }
    if (bm > v.m) {
      if (v.s != 0.f) {
        const float d = v.m - bm, e = __expf(d);
        v.t = vt_rebased_t(v.s, v.t, d, e);
        v.s *= e;
      }
      v.m = bm;
      v.idx = INT_MAX;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const float d = fmaxf(q[u].x - v.m, -200.f);            // <= 0; e^-200 is 0 in float32
      const float e = __expf(d);
      v.s += q[u].z * e;
      v.t += e * (q[u].w + d * q[u].z);
      v.idx = min(v.idx, q[u].x == v.m ? __float_as_int(q[u].y) : INT_MAX);   // lowest index among equal maxima
    }
  }
  return v;
}

// The k-th largest of the history values of a wave's copy (NU slots a lane): the largest v in [1, t] with
// count(hist >= v) >= k, by bisection; INT_MIN if fewer than k are decoded.
template <int NU>
__device__ __forceinline__ int kth_of_history(const int* s_hist, int N, int lane, int t, int k) {
  int hv[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) hv[u] = u * 64 + lane < N ? s_hist[u * 64 + lane] : INT_MIN;
  int lo = 1, hi = t, found = INT_MIN;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    int c = 0;
#pragma unroll
    for (int u = 0; u < NU; ++u) c += __popcll(__ballot(hv[u] >= mid));
    if (c >= k) { found = mid; lo = mid + 1; } else { hi = mid - 1; }
  }
  return found;
}

// ---------------------------------------------------------------------------------------------
// decide: one block of kDecideThreads threads per sequence.  A chain of latencies: the loads (state, history, mask set,
// the rows' partial tuples, the caller's forced tokens) are all on their way before the first is used, from then on the
// kernel works in LDS and registers.  Sixteen waves are four to a SIMD, so what all of them do costs four
// times: a lane merges no more parts than there are, ranks are counted by half a wave a row, the gate value
// comes from the last wave beside the others, and waves that hold no slot of the generation only come to the
// barriers.  No barrier to find the k-th largest history value (up to 512 slots) or the current block, one to compact the
// three row lists.  The forced lists are read where the host left them and the flag goes back with the result, so
// a forced step adds no copies.
// On MI355X, first instruction to the result's release: 128 slots, 4096 tokens, float32 10.1 -> 6.1 us; 32 rows of a
// small bf16 model, forced, 11.5 -> 6.4; 64 rows of 988 tuples (1 MB through one compute unit, 7 us of it) 15.4 -> 12.1; 16
// sequences of 512 slots 14.8 -> 9.7.
// dynamic LDS: int hist[N4] | uint8 masked[N4], N4 = N rounded up to 4
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kDecideThreads) void decide_kernel(DecideArgs a) {
  extern __shared__ int s_dyn[];
  {  // this block's sequence: move the pointers, take the per-sequence scalars
    const int b = blockIdx.x;
    const SeqDesc sd = a.seqs ? a.seqs[b] : a.seq0;
    if (sd.mode < 0) return;  // finished earlier: no rows in this step, nothing to decide
    a.partials += (size_t)sd.lm0 * a.nparts;
    a.n_mb = sd.n_mb; a.mode_run = sd.mode; a.n_rows_run = sd.n_rows; a.forced_n = sd.forced_n;
    a.forced_pos += b * EC_MAX_N; a.forced_tok += b * EC_MAX_N;
    a.x += sd.x_off; a.masked += sd.x_off; a.rows_partial += sd.x_off;
    a.hist += (size_t)b * a.N; a.st += b; a.out += b;
    a.mb_pos += b * a.block; a.mb_idx += b * a.block; a.row_stats += b * a.block * 4;
    a.P = sd.P; a.T = sd.T;
  }
  __shared__ int s_tok[EC_MAX_BLOCK], s_pos[EC_MAX_BLOCK];
  __shared__ float s_conf[EC_MAX_BLOCK];
  __shared__ float s_H[EC_MAX_BLOCK];
  __shared__ int s_badrow[EC_MAX_BLOCK];  // 1: the row's logits had no finite maximum / sums
  __shared__ int s_sel[EC_MAX_N];    // block rows of the step's own choice, most confident first
  __shared__ int s_fpos[EC_MAX_N], s_ftok[EC_MAX_N];   // the caller's positions and tokens
  __shared__ int s_frow[EC_MAX_N];   // block rows of the caller's positions (-1: not in the block)
  __shared__ unsigned long long scratch[2][kDecideWaves];
  __shared__ float sh_f[2];
  __shared__ int sh_bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = a.P, N = a.N;
  int* s_hist = s_dyn;
  uint8_t* s_msk = (uint8_t*)(s_dyn + ((N + 3) & ~3));
  const int nblocks = (N + a.block - 1) / a.block;

  // ---- requests: state, history, mask set, block positions, forced tokens --------------------
  // (they stay in registers until the rows' partial tuples, whose loads follow, have been merged; the forced lists
  // are in host memory and go to the last wave, whose rows wait for them, as the loads of a wave return in order:
  // as kernel arguments they measured the same)
  DevState st = *a.st;  // every thread holds a private copy; thread 0 writes it back
  int my_hist = 0, my_pos = 0, f_pos = -1, f_tok = -1;
  uint8_t my_msk = 0;
  const int f = tid - (kDecideThreads - EC_MAX_N);
  if (tid < N) { my_hist = a.hist[tid]; my_msk = a.masked[P + tid]; }
  if (!a.init_only) {
    if (tid < a.n_mb) my_pos = a.mb_pos[tid];
    if (f >= 0 && f < a.forced_n) { f_pos = a.forced_pos[f]; f_tok = a.forced_tok[f]; }
  }
  auto to_lds = [&]() {
    if (tid < N) { s_hist[tid] = my_hist; s_msk[tid] = my_msk; }
    for (int i = tid + kDecideThreads; i < N; i += kDecideThreads) {
      s_hist[i] = a.hist[i];
      s_msk[i] = a.masked[P + i];
    }
  };
  const int t = st.t;
  int n = 0;   // tokens of the step's own choice

  if (!a.init_only) {
    // ---- merge the vocabulary partials of each block row (fixed order) ----------------------
    // Half a wave per row, 32 rows at a time: each lane its parts, then the 32 tuples at once.
    for (int row0 = 0; row0 < a.n_mb; row0 += 2 * kDecideWaves) {
      const int row = row0 + wave * 2 + (lane >> 5), l32 = lane & 31;
      if (row0 + wave * 2 >= a.n_mb) break;   // (wave-uniform: nothing for either half)
      const bool live = row < a.n_mb;
      const float4* pr = a.partials + (size_t)(live ? row : 0) * a.nparts;
      VTuple v = a.nparts <= 64 ? merge_row_parts<2>(pr, l32, a.nparts)
                 : a.nparts <= 128 ? merge_row_parts<4>(pr, l32, a.nparts)
                                   : merge_row_parts<16>(pr, l32, a.nparts);
      v = vt_merge_lanes<32>(v);
      if (live && l32 == 0) {
        float conf, H;
        vt_finish(v, conf, H);
        // A row of NaNs has no maximum: its index is still the sentinel, its sums are NaN.  One of +inf has no
        // finite maximum.  The token becomes an index into the embedding table at the next step, so it must be a
        // token, 0 for both; such a row counts as least confident and of infinite entropy, and is reported.
        int tok = v.idx, bad = 0;
        if ((unsigned)tok >= (unsigned)a.vocab || !(fabsf(v.m) < INFINITY)) { tok = 0; bad = 1; }
        if (!(v.s > 0.f) || !(conf >= 0.f) || !(v.t == v.t) || !(H >= 0.f)) bad = 1;
        if (bad) { conf = 0.f; H = INFINITY; }  // (the clamp in vt_finish turns a NaN entropy into 0)
        s_badrow[row] = bad;
        s_tok[row] = tok;
        s_conf[row] = conf;
        s_H[row] = H;
        *(float4*)(a.row_stats + row * 4) = make_float4((float)tok, conf, H, v.m);
      }
    }
    to_lds();
    if (tid < a.n_mb) s_pos[tid] = my_pos;
    if (f >= 0 && f < a.forced_n) { s_fpos[f] = f_pos; s_ftok[f] = f_tok; s_frow[f] = -1; }
    __syncthreads();
    // ---- decode(): most confident rows first; ties -> lowest position (= lowest row) --------
    // A row's rank is the number of rows that go before it (counted by half a wave, as above); the
    // n lowest ranks are unmasked.
    n = min(a.n_tok, a.n_mb);
    if (a.conf_threshold > 0.f) {
      // confidence-based parallel decoding: every row above the threshold, the n most
      // confident ones in any case, no more than one result can report
      const int above = __syncthreads_count(tid < a.n_mb && s_conf[tid] > a.conf_threshold);
      n = min(min(max(n, above), EC_MAX_N), a.n_mb);
    }
    // commit, own choice or the caller's under teacher forcing (Eq. 2): to memory, and to the LDS
    // copies the rest of the kernel works on
    auto commit = [&](int pos, int tok) {
      a.x[pos] = tok;
      a.masked[pos] = 0;
      a.hist[pos - P] = t;
      s_msk[pos - P] = 0;
      s_hist[pos - P] = t;
    };
    for (int row0 = wave * 2; row0 < a.n_mb; row0 += 2 * kDecideWaves) {
      const int row = row0 + (lane >> 5), l32 = lane & 31;
      const float my_conf = s_conf[min(row, a.n_mb - 1)];
      int rank = 0;
      for (int r0 = 0; r0 < a.n_mb; r0 += 32) {
        const int r = r0 + l32;
        const float c = s_conf[min(r, a.n_mb - 1)];
        const unsigned long long before = __ballot(r < a.n_mb && (c > my_conf || (c == my_conf && r < row)));
        rank += __popc((unsigned)(lane < 32 ? before : before >> 32));
      }
      if (l32 == 0 && row < a.n_mb && rank < n) {
        s_sel[rank] = row;
        if (a.forced_n < 0) commit(s_pos[row], s_tok[row]);
      }
    }
    if (a.forced_n > 0) {
      if (tid < a.forced_n) commit(s_fpos[tid], s_ftok[tid]);
      if (tid < a.n_mb)
        for (int i = 0; i < a.forced_n; ++i)
          if (s_fpos[i] == my_pos) s_frow[i] = tid;
    }
    __syncthreads();   // the LDS copies of history and mask set are complete and committed to
    if (wave == kDecideWaves - 1) {   // beside the other waves' way to the next barrier
      const bool bad = (lane < a.n_mb && s_badrow[lane]) || (lane + 64 < a.n_mb && s_badrow[lane + 64]);
      const bool any_bad = __ballot(bad) != 0;
      if (lane == 0) {
        // gate values, accumulated in the order of the lists (the entropy sum is order-sensitive)
        GateAcc own = gate_init(a.gate_metric);
        for (int i = 0; i < n; ++i) gate_add(own, s_H[s_sel[i]], s_conf[s_sel[i]]);
        float E = own.v;
        if (a.forced_n >= 0) {
          bool all_in_block = true;
          GateAcc fa = gate_init(a.gate_metric);
          for (int i = 0; i < a.forced_n; ++i) {
            const int row = s_frow[i];
            if (row < 0) all_in_block = false; else gate_add(fa, s_H[row], s_conf[row]);
          }
          if (all_in_block) E = fa.v;                       // nothing committed: always skips
        }
        sh_f[0] = E;
        sh_f[1] = own.v;
        sh_bad = any_bad;
      }
    }
  } else {
    to_lds();
    __syncthreads();
  }

  // ---- recency threshold: tau_R = max(k-th largest history value, t - dt) --------------------
  // History values are step indices in [1, t] or "never"; fewer than k decoded -> -inf.  Up to 512 slots
  // every wave that holds some of them counts for itself, without a barrier.
  const int nw = min(kDecideWaves, (N + 63) >> 6);   // waves that hold slots
  int t_lastfull = st.t_lastfull;
  int tauR = INT_MAX;
  if (!a.init_only) {
    if (a.mode_run == EC_FULL) t_lastfull = t;
    int kth = INT_MIN;
    if (a.k_recent <= 0) {
      kth = INT_MAX;  // empty selection: nothing qualifies by rank
    } else if (N <= 512) {
      if (wave < nw)
        kth = N <= 128 ? kth_of_history<2>(s_hist, N, lane, t, a.k_recent) : kth_of_history<8>(s_hist, N, lane, t, a.k_recent);
    } else {
      int lo = 1, hi = t;
      while (lo <= hi) {  // uniform across the block
        const int mid = (lo + hi) >> 1;
        int c = 0;
        for (int base = 0; base < N; base += kDecideThreads) {  // uniform trip count
          const int i = base + tid;
          c += __syncthreads_count(i < N && s_hist[i] >= mid);
        }
        if (c >= a.k_recent) { kth = mid; lo = mid + 1; } else { hi = mid - 1; }
      }
    }
    tauR = max(kth, t_lastfull);  // t - dt == index of the last FULL step
  }

  // ---- block advance -----------------------------------------------------------------------
  const bool sliding = a.schedule == EC_SCHED_SLIDING;
  int blk = st.blk;
  if (!sliding) {
    while (wave < nw && blk < nblocks) {  // every wave with slots looks at the whole block (at most 128 slots)
      const int lo = blk * a.block + lane, hi = min(N, (blk + 1) * a.block);
      if (__ballot((lo < hi && s_msk[lo]) || (lo + 64 < hi && s_msk[lo + 64]))) break;
      ++blk;
    }
    st.blk = blk;
    st.done = (blk >= nblocks);
  }

  // ---- row lists of the next step: M and M u R, ascending ---------------------------------------
  // M = the masked rows of the current block, or (sliding window) the first `block` masked slots
  const int blo = blk * a.block, bhi = min(N, blo + a.block);   // in generation slots
  int n_rows = 0, n_mb = 0, n_recent = 0, masked_seen = 0, buf = 0;
  for (int base = 0; base < N; base += kDecideThreads, buf ^= 1) {
    const int i = base + tid, pos = P + i;
    bool inM = false, inR = false, msk = false;
    if (i < N) {
      msk = s_msk[i] != 0;
      inM = !sliding && !st.done && i >= blo && i < bhi && msk;
      const int h = s_hist[i];
      inR = !a.init_only && h != INT_MIN && h >= tauR;
    }
    if (sliding) {
      int pre[1], tot[1];
      block_excl_scan_flags<1>({msk}, scratch[buf], nw, pre, tot);
      inM = msk && masked_seen + pre[0] < a.block;
      masked_seen += tot[0];
      buf ^= 1;
    }
    int pre[3], tot[3];
    block_excl_scan_flags<3>({inM || inR, inM, inR}, scratch[buf], nw, pre, tot);
    if (inM || inR) a.rows_partial[n_rows + pre[0]] = pos;
    if (inM) {
      a.mb_pos[n_mb + pre[1]] = pos;
      a.mb_idx[n_mb + pre[1]] = n_rows + pre[0];
    }
    n_rows += tot[0];
    n_mb += tot[1];
    n_recent += tot[2];
  }
  if (sliding) st.done = (n_mb == 0);
  // The result, all of it from wave 0.  (The barriers of the lists lie between the gate values and their use here.)
  if (wave > 0) return;
  static_assert(EC_MAX_N <= kWave, "the result's lists are stored by one wave");
  if (!a.init_only && lane < EC_MAX_N) {
    ec_step_result& R = a.out->r;
    const int row = lane < n ? s_sel[lane] : 0;
    R.positions[lane] = lane < n ? s_pos[row] : -1;
    R.tokens[lane] = lane < n ? s_tok[row] : -1;
    R.entropy[lane] = lane < n ? s_H[row] : 0.f;
    R.confidence[lane] = lane < n ? s_conf[row] : 0.f;
  }
  if (lane == 0) {
    if (!a.init_only) {
      if (gate_skips(sh_f[0], a.tau, a.gate_metric)) { st.skip = 1; st.dt += 1; } else { st.skip = 0; st.dt = 0; }
      st.t_lastfull = t_lastfull;
      st.t = t + 1;
    }
    st.n_mb = n_mb;
    st.n_rows_partial = n_rows;
    st.n_recent = n_recent;
    *a.st = st;
    StepOut& o = *a.out;
    o.next_n_mb = n_mb;
    o.next_n_rows_partial = n_rows;
    if (!a.init_only) {
      o.r.n_unmasked = n;
      o.r.max_entropy = sh_f[1];
      o.r.done = st.done;
      o.r.mode_run = a.mode_run;
      o.r.next_mode = gate_skips(sh_f[1], a.tau, a.gate_metric) ? EC_PARTIAL : EC_FULL;
      o.r.n_query_rows = a.n_rows_run;
      o.r.step_index = t;
      o.r.n_block_rows = a.n_mb;
      o.r.n_recent_next = n_recent;
    }
    o.nonfinite = a.init_only ? 0 : sh_bad;
    o.skip = st.skip;
  }
  // The result sits in pinned host memory: a host that sees the serial number sees the whole of it.  Each lane's fence
  // orders what that lane stored, the wave barrier keeps all of them ahead of the number.
  __threadfence_system();
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) __hip_atomic_store(&a.out->serial, a.serial, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_decide(const DecideArgs& a, int B, hipStream_t s) {
  const size_t smem = (size_t)((a.N + 3) & ~3) * 5;   // history (int) + mask set (byte)
  static size_t attr_bytes = 48 * 1024;
  if (smem > attr_bytes) {
    (void)hipFuncSetAttribute((const void*)decide_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)smem);
    attr_bytes = smem;
  }
  decide_kernel<<<B, kDecideThreads, smem, s>>>(a);
}

// ---------------------------------------------------------------------------------------------
// init_state: x = [prompt ; mask_id ...], mask set = generation slots, history = never,
// t = 1, flag = recompute, Delta t = 0 (initialisation lines of both algorithms).
// ---------------------------------------------------------------------------------------------
__global__ void init_state_kernel(int* x, uint8_t* masked, int* hist, DevState* st,
                                  const int* prompt, int P, int N, int mask_id) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P + N) {
    x[i] = i < P ? prompt[i] : mask_id;
    masked[i] = i < P ? 0 : 1;
    if (i >= P) hist[i - P] = INT_MIN;
  }
  if (i == 0) {
    DevState z = {};
    z.t = 1;
    *st = z;
  }
}

void launch_init_state(int* x, uint8_t* masked, int* hist, DevState* st, const int* prompt_dev,
                       int P, int N, int mask_id, hipStream_t s) {
  int n = P + N;
  init_state_kernel<<<(n + 255) / 256, 256, 0, s>>>(x, masked, hist, st, prompt_dev, P, N, mask_id);
}

}  // namespace ec
