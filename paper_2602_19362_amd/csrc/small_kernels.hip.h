// The O(T) and O(N) steps of the OAPL loss head: sampled-token logit gather,
// log-sum-exp finish, per-rollout segmented sums, group value estimate and
// loss (Sec. 3.1, Eq. 2 and Eq. 3) and token coefficients.  All bandwidth-trivial next to the
// three V x d contractions; written for exactness and a fixed summation order.
#pragma once

#include <type_traits>

#include "common.hip.h"
#include "rng.hip.h"

namespace oapl {

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return (float)x; }

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void k_fill_f32(float* p, int64_t n, float v, Gate gate) {
  if (gate_closed(gate)) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// z_{t, y_t} = sum_k H[t][k] * W[y_t][k]: one wavefront per token, the gathered
// W row is read with the index exactly as given (checked against [0, V)).
// ACC is double for fp32 inputs and float for bf16 inputs (whose products are exact in fp32).  VEC elements per load: 16
// bytes, or one for fp32 rows that are not 16-byte aligned.  Reads 2 rows per token and is bound by the latency of a
// wavefront's chain of loads: element by element it took 33 us for 777 tokens at d = 4096 (64 loads in a row per lane) and
// 82 us for 32768 at d = 2048, by 16-byte loads 8.5 and 42 us.
//
// It also prepares the other per-token arrays of a loss call, where those are given: coef[t] = 0 (a token that malformed
// offsets leave out keeps it); for the single sweep the reference exponent ref2[t] of k_sweep, and "no contribution yet"
// for a row that is not swept: diff[t] = 0, nis[t] = 0.  The reference is the largest logit among a sample of the row (its
// first 256 vocabulary entries, whose running maximum `sample` carries in .x, and the sampled token's own logit) plus a
// margin, in the exp2 domain.  Some entry of the row then equals 2^-margin, so S_t >= 2^-margin, and entries down to
// 2^-(126 - margin) of the row's largest stay normal bf16 numbers.
constexpr float kSweepMargin = 40.f;
constexpr float kSweepLimit = 1.2676506e30f;   // 2^100: largest S_t the single sweep accepts
struct TokenInit {
  float* coef;            // or nullptr
  const float2* sample;   // or nullptr
  const float* sample_parts;   // or, in place of that: the sample's logits, [sample_splits][T][256] to be summed (k_ref_begin)
  int sample_splits, sample_rows;
  float* ref2;            // or nullptr: no single sweep
  double* diff;
  float* nis;
};
// What a token of a call gets with its logit z; `largest`: of the sample's logits, in the exp2 domain.
__device__ __forceinline__ void init_token(const TokenInit& init, int64_t t, float z, float largest, float* __restrict__ zy) {
  zy[t] = z;
  if (init.coef) init.coef[t] = 0.f;
  if (init.ref2) {
    init.ref2[t] = fmaxf(largest, z * kLog2e) + kSweepMargin;    // fmaxf drops a NaN (token out of range)
    init.diff[t] = 0.0;
    init.nis[t] = 0.f;
  }
}
// The largest of token t's sampled logits, in the exp2 domain, from their parts: four of 256 rows per lane.
__device__ __forceinline__ float largest_sampled(const TokenInit& init, int64_t t, int64_t T) {
  const int lane = threadIdx.x & 63;
  const f32x4* p = (const f32x4*)(init.sample_parts + t * 256) + lane;
  f32x4 z = p[0];
#pragma unroll 8
  for (int s = 1; s < init.sample_splits; ++s) z += p[(int64_t)s * T * 64];
  float largest = kNegHuge;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (4 * lane + e < init.sample_rows) largest = fmaxf(largest, z[e]);
#pragma unroll
  for (int o = 32; o > 0; o /= 2) largest = fmaxf(largest, __shfl_xor(largest, o, 64));
  return largest * kLog2e;
}
// `err` == nullptr: a token out of range is recorded by a later launch (k_lse_finish), for the status header is being cleared
// by this one.
template <class T, class ACC, int VEC>
__device__ __forceinline__ void gather_logit(int64_t t /* of this wavefront */, const T* __restrict__ H, const T* __restrict__ W,
                                             const int32_t* __restrict__ tokens, int64_t Ttok, int d, int V,
                                             float* __restrict__ zy, int* __restrict__ err, const TokenInit& init) {
  typedef T vec_t __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));   // bf16 rows may start at any element
  const int lane = threadIdx.x & 63;
  if (t >= Ttok) return;
  const int y = tokens[t];
  const float largest = init.sample_parts ? largest_sampled(init, t, Ttok) : init.sample ? init.sample[t].x : 0.f;
  auto finish = [&](float z) { init_token(init, t, z, largest, zy); };
  if (y < 0 || y >= V) {
    if (lane == 0) {
      if (err) record_token_error(err);
      finish(__builtin_nanf(""));
    }
    return;
  }
  const vec_t* h = (const vec_t*)(H + t * d);
  const vec_t* w = (const vec_t*)(W + (int64_t)y * d);
  ACC acc = 0;
#pragma unroll 4
  for (int k = lane; k < d / VEC; k += 64) {
    const vec_t a = h[k], b = w[k];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc += (ACC)to_f32((T)a[e]) * (ACC)to_f32((T)b[e]);
  }
  acc = wave_sum(acc);
  if (lane == 0) finish((float)acc);
}
template <class T, class ACC, int VEC>
__global__ void __launch_bounds__(256)
k_gather_logit(const T* __restrict__ H, const T* __restrict__ W, const int32_t* __restrict__ tokens,
               int64_t Ttok, int d, int V, float* __restrict__ zy, int* __restrict__ err, TokenInit init) {
  gather_logit<T, ACC, VEC>((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), H, W, tokens, Ttok, d, V, zy, err, init);
}

// Merges the per-split soft-max partials of each token and finishes
//   lse_t = ln sum_v exp(z_tv),   logprob_t = min(z_{t,y_t} - lse_t, 0),
// and, when asked for, the entropy of the token's distribution from the extra
// partial u = sum b^(zeta - m) * z.
// A partial is (m, s) with s = sum b^(zeta - m): LOG2 = true means zeta =
// z * log2(e), b = 2 (the MFMA kernel's epilogue); false means zeta = z, b = e.
// Everything after the fp32 partials is done in double.  A workgroup serves 256 / slices tokens; the partials of a
// token are taken by `slices` (a power of two <= 256) threads, interleaved, and combined pairwise, so the few
// tokens of a small call, which come with hundreds of partials each, are not walked by one thread each (777 tokens
// with 64 partials: 47 us with one slice, 10 us with sixteen).
struct LseFinish {
  const float2* partials;
  int n_parts;
  int64_t Ttok;
  const float *zy, *logq;
  float *logprob_out, *lse_out, *lse2_ws;
  double* diff_ws;
  float *omp_ws, *inv_omp_ws;
  const float* upart;
  float* entropy_out;
  int slices;
  const int32_t* tokens;     // to check, or nullptr
  int V;
  int* err;
};
// Tokens t0 .. end - 1, at most 256 / slices of them, by a workgroup.
template <bool LOG2>
__device__ __forceinline__ void lse_finish(const LseFinish& f, int64_t t0, int64_t end) {
  __shared__ float part_m[256];
  __shared__ double part_s[256], part_u[256];
  const float2* partials = f.partials;
  const int n_parts = f.n_parts, slices = f.slices, V = f.V;
  const int64_t Ttok = f.Ttok;
  const float *zy = f.zy, *logq = f.logq, *upart = f.upart;
  float *logprob_out = f.logprob_out, *lse_out = f.lse_out, *lse2_ws = f.lse2_ws, *omp_ws = f.omp_ws, *inv_omp_ws = f.inv_omp_ws,
        *entropy_out = f.entropy_out;
  double* diff_ws = f.diff_ws;
  const int32_t* tokens = f.tokens;
  int* err = f.err;
  const int rows = 256 / slices, col = threadIdx.x % rows, slice = threadIdx.x / rows;
  const int64_t t = t0 + col;
  float M = kNegHuge;
  if (t < end) {
#pragma unroll 8
    for (int p = slice; p < n_parts; p += slices) M = fmaxf(M, partials[(int64_t)p * Ttok + t].x);
  }
  part_m[threadIdx.x] = M;
  for (int half = slices / 2; half > 0; half /= 2) {
    __syncthreads();
    if (slice < half) part_m[threadIdx.x] = M = fmaxf(M, part_m[threadIdx.x + half * rows]);
  }
  __syncthreads();
  M = part_m[col];
  double S = 0.0, U = 0.0;
  if (t < end) {
#pragma unroll 8
    for (int p = slice; p < n_parts; p += slices) {
      const float2 a = partials[(int64_t)p * Ttok + t];
      const double e = (double)a.x - (double)M;
      const double f = LOG2 ? exp2(e) : exp(e);
      S += (double)a.y * f;
      if (entropy_out) U += (double)upart[(int64_t)p * Ttok + t] * f;
    }
  }
  part_s[threadIdx.x] = S;
  part_u[threadIdx.x] = U;
  for (int half = slices / 2; half > 0; half /= 2) {
    __syncthreads();
    if (slice < half) {
      part_s[threadIdx.x] = S += part_s[threadIdx.x + half * rows];
      part_u[threadIdx.x] = U += part_u[threadIdx.x + half * rows];
    }
  }
  if (slice != 0 || t >= end) return;
  if (tokens && (tokens[t] < 0 || tokens[t] >= V)) record_token_error(err);
  const double lse = LOG2 ? ((double)M + log2(S)) * kLn2 : (double)M + log(S);
  double lp = (double)zy[t] - lse;   // NaN if the token was out of range
  if (lp > 0.0) lp = 0.0;            // the gathered logit is rounded separately from the sum
  if (logprob_out) logprob_out[t] = (float)lp;
  if (lse_out) lse_out[t] = (float)lse;
  // policy entropy  -sum_v p_v ln p_v = lse - sum_v p_v z_v  with  sum_v p_v z_v = U / S  (>= 0 up to rounding)
  if (entropy_out) entropy_out[t] = (float)fmax(lse - U / S, 0.0);
  // the backward kernels want lse in the domain their exponentials work in
  if (lse2_ws) lse2_ws[t] = (float)(LOG2 ? lse * (double)1.4426950408889634074 : lse);
  if (diff_ws) diff_ws[t] = lp - (double)logq[t];
  // 1 - p_{t,y_t}, accurate also when the sampled token has almost all the mass;
  // its reciprocal normalises the bf16 gradient rows (0 switches a row off when
  // the soft-max is one-hot at y_t to working precision, or the token is bad)
  if (omp_ws) {
    const double omp = -expm1(lp);
    const bool ok = omp > 1e-30;
    omp_ws[t] = ok ? (float)omp : 0.f;
    inv_omp_ws[t] = ok ? (float)(1.0 / omp) : 0.f;
  }
}
template <bool LOG2>
__global__ void __launch_bounds__(256) k_lse_finish(LseFinish f, Gate gate) {
  if (gate_closed(gate)) return;
  lse_finish<LOG2>(f, (int64_t)blockIdx.x * (256 / f.slices), f.Ttok);
}

// Picks, per token, the best (score, index) pair over the vocabulary splits (ties to the smaller index); slices as
// in k_lse_finish.
__global__ void __launch_bounds__(256)
k_sample_finish(const float2* __restrict__ partials, int n_parts, int64_t Ttok, int32_t* __restrict__ tokens_out,
                float* __restrict__ score_out, int slices, int* __restrict__ status) {
  if (blockIdx.x == 0 && threadIdx.x < kStatusWords) status[threadIdx.x] = 0;   // nothing in a sampling call can set one
  __shared__ float2 part[256];
  const int rows = 256 / slices, col = threadIdx.x % rows, slice = threadIdx.x / rows;
  const int64_t t = (int64_t)blockIdx.x * rows + col;
  float best = -__builtin_inff();
  int arg = 0x7FFFFFFF;
  if (t < Ttok) {
#pragma unroll 8
    for (int p = slice; p < n_parts; p += slices) {
      const float2 a = partials[(int64_t)p * Ttok + t];
      if (better(a.x, __float_as_int(a.y), best, arg)) { best = a.x; arg = __float_as_int(a.y); }
    }
  }
  part[threadIdx.x] = make_float2(best, __int_as_float(arg));
  for (int half = slices / 2; half > 0; half /= 2) {
    __syncthreads();
    if (slice < half) {
      const float2 a = part[threadIdx.x + half * rows];
      if (better(a.x, __float_as_int(a.y), best, arg)) { best = a.x; arg = __float_as_int(a.y); }
      part[threadIdx.x] = make_float2(best, __int_as_float(arg));
    }
  }
  if (slice != 0 || t >= Ttok) return;
  tokens_out[t] = arg;
  if (score_out) score_out[t] = best;
}

// Sum over the 256 threads of a workgroup, valid in every thread: wavefront shuffles, then the 4 wave totals in order.
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double wsum[4];
  v = wave_sum(v);
  __syncthreads();      // wsum may still be read for an earlier sum
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
}

// Token range of rollout s, clamped to [0, limit] so that malformed offsets cannot reach past a buffer.
__device__ __forceinline__ void token_range(const int64_t* off, int s, int64_t limit, int64_t& a, int64_t& b) {
  a = off[s];
  b = off[s + 1];
  a = a < 0 ? 0 : (a > limit ? limit : a);
  b = b < a ? a : (b > limit ? limit : b);
}

// The last of `n` workgroups to get here returns true and sees what the others wrote before (their plain stores too).
// The counter is back at zero afterwards.
__device__ __forceinline__ bool last_workgroup(int* counter, int n) {
  __shared__ int last;
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) last = atomicInc((unsigned*)counter, (unsigned)(n - 1)) == (unsigned)(n - 1);
  __syncthreads();
  if (last) __threadfence();
  return last != 0;
}

// out[s] = sum_{t in [off[s], off[s+1])} x[t] in double: one workgroup per
// rollout, each thread a strided partial in a fixed order, then block_sum.
// Bit-reproducible.  Offsets are clamped to a >= 0, b >= a, so malformed input
// cannot read below the buffer.
template <class T>
__global__ void __launch_bounds__(256)
k_segmented_sum(const T* __restrict__ x, const int64_t* __restrict__ off, int n_seq, double* __restrict__ out) {
  const int s = blockIdx.x;
  if (s >= n_seq) return;
  int64_t a = off[s], b = off[s + 1];
  a = a < 0 ? 0 : a;
  b = b < a ? a : b;
  double acc = 0.0;
  for (int64_t t = a + threadIdx.x; t < b; t += 256) acc += (double)x[t];
  acc = block_sum(acc);
  if (threadIdx.x == 0) out[s] = acc;
}

// Butterfly reductions over a wavefront: every lane ends with the same value, combined in a
// fixed order (bit-reproducible).
__device__ __forceinline__ double wave_allsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_allmax(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_allsum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---------------------------------------------------------------------------
// What a loss call does before anything is scored.  Each step is a function of (worker, workers): one workgroup takes them
// all in one launch where rollouts and prompts are few (a launch costs a small call 2 .. 4 us), else each has a grid.
// Indices are 64 bits: rollouts and prompts may number 2^31 - 1, and a step past the last one must not wrap.
// ---------------------------------------------------------------------------

// Group value estimate, one wavefront per prompt:
//   V*_g = beta_v ln( (1/G_g) sum_{s in g} exp(r_s / beta_v) )            Eq. 2
//        = m_g + beta_v ln( (1/G_g) sum exp((r_s - m_g) / beta_v) ),  m_g = max_{s in g} r_s
// (same value; the shift keeps exp() in range for small beta and makes all-equal rewards return
// exactly r).  Group ids come in any order, so the wavefront walks the rollouts lane-strided and
// keeps those of its prompt: lane-local partial max / count / sum in rollout order, then shuffle
// butterflies.  A prompt without rollouts gets NaN and records the group error.
__device__ __forceinline__ void group_value(int64_t wave, int64_t waves, const float* __restrict__ rewards,
                                            const int32_t* __restrict__ gid, int n_seq, int n_groups, double beta_v,
                                            double* __restrict__ vstar_ws, float* __restrict__ vstar_out, int* err) {
  const int lane = threadIdx.x & 63;
  for (int64_t g = wave; g < n_groups; g += waves) {
    double m = -1.0e300;
    int cnt = 0;
    for (int64_t s = lane; s < n_seq; s += 64)
      if (gid[s] == g) { m = fmax(m, (double)rewards[s]); ++cnt; }
    m = wave_allmax(m);
    cnt = wave_allsum(cnt);
    double v;
    if (cnt == 0) {
      if (lane == 0) record_batch_error(err, kErrGroup);
      v = __builtin_nan("");
    } else {
      double sum = 0.0;
      for (int64_t s = lane; s < n_seq; s += 64)
        if (gid[s] == g) sum += exp(((double)rewards[s] - m) / beta_v);
      sum = wave_allsum(sum);
      v = m + beta_v * log(sum / (double)cnt);
    }
    if (lane == 0) {
      vstar_ws[g] = v;
      if (vstar_out) vstar_out[g] = (float)v;
    }
  }
}

// GRPO baseline (Sec. 2, the displayed GRPO objective), group step, one wavefront per prompt:
// mean and population standard deviation of the prompt's rewards and its size G_g (kept behind
// the per-rollout weights).  A prompt without rollouts gets NaN and records the group error.
__device__ __forceinline__ void grpo_group_stats(int64_t wave, int64_t waves, const float* __restrict__ rewards,
                                                 const int32_t* __restrict__ gid, int n_seq, int n_groups,
                                                 double* gmean, double* gstd, double* gsize, int* err) {
  const int lane = threadIdx.x & 63;
  for (int64_t g = wave; g < n_groups; g += waves) {
    double sum = 0.0;
    int cnt = 0;
    for (int64_t s = lane; s < n_seq; s += 64)
      if (gid[s] == g) { sum += (double)rewards[s]; ++cnt; }
    sum = wave_allsum(sum);
    cnt = wave_allsum(cnt);
    if (cnt == 0) {
      if (lane == 0) {
        record_batch_error(err, kErrGroup);
        gmean[g] = __builtin_nan("");
        gstd[g] = __builtin_nan("");
        gsize[g] = 0.0;
      }
      continue;
    }
    const double mean = sum / cnt;
    double var = 0.0;
    for (int64_t s = lane; s < n_seq; s += 64)
      if (gid[s] == g) { const double dlt = (double)rewards[s] - mean; var += dlt * dlt; }
    var = wave_allsum(var);
    if (lane == 0) {
      gmean[g] = mean;
      gstd[g] = sqrt(var / cnt);
      gsize[g] = (double)cnt;
    }
  }
}

// GRPO, rollout step: the normalised advantage
//   A_s = (r_s - mean_g r) / (std_g r + adv_eps)
// and the weight w_s = scale / (G_g |y_s|) of rollout s (0 for an empty rollout).  Validates
// offsets and group ids like the OAPL kernel and records the status.
__device__ __forceinline__ void grpo_advantage(int64_t thread, int64_t threads, const float* __restrict__ rewards,
                                               const int32_t* __restrict__ gid, const int64_t* __restrict__ off,
                                               int n_seq, int n_groups, int64_t Ttok, double adv_eps, double scale,
                                               const double* gmean, const double* gstd, const double* gsize,
                                               float* __restrict__ adv, double* __restrict__ wseq,
                                               float* __restrict__ adv_out, int* err) {
  if (thread == 0 && (off[0] != 0 || off[n_seq] != Ttok)) record_batch_error(err, kErrOffsets);
  for (int64_t s = thread; s < n_seq; s += threads) {
    if (off[s + 1] < off[s]) record_batch_error(err, kErrOffsets);
    const int g = gid[s];
    const bool ok = g >= 0 && g < n_groups;
    if (!ok) record_batch_error(err, kErrGroup);
    const double a = ok ? ((double)rewards[s] - gmean[g]) / (gstd[g] + adv_eps) : __builtin_nan("");
    const int64_t len = off[s + 1] - off[s];
    adv[s] = (float)a;
    if (adv_out) adv_out[s] = (float)a;
    wseq[s] = (ok && len > 0 && gsize[g] > 0.0) ? scale / (gsize[g] * (double)len) : 0.0;
  }
}

// The single-sweep path finishes a panel of token rows before it knows the later panels, so a
// rollout must end at most one panel after it starts: any rollout longer than `longest`
// (or malformed offsets) raises the flag that sends the call down the two-pass path instead.
// longest < 0: the call does not try the single sweep.
__device__ __forceinline__ void sweep_plan(int64_t thread, int64_t threads, const int64_t* __restrict__ off, int n_seq,
                                           int64_t Ttok, int64_t longest, int* flag) {
  if (longest < 0) return;
  bool bad = thread == 0 && (off[0] != 0 || off[n_seq] != Ttok);
  for (int64_t s = thread; s < n_seq; s += threads) {
    const int64_t len = off[s + 1] - off[s];
    bad |= len < 0 || len > longest;
  }
  if (bad) atomicCAS(flag, 0, 1);
}

// Clears the status header; every later use of it by this workgroup comes after the clear.
__device__ __forceinline__ void clear_status(int* status) {
  if (threadIdx.x < kStatusWords) __hip_atomic_store(status + threadIdx.x, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __threadfence();
  __syncthreads();
}

// Steps of a call's beginning as (block, blocks) of 256 threads.  kPlan: after a clear header, the sweep's length check and
// what prompts need; kRest: what needs the prompts' results; both: one workgroup, status header included.
enum BeginSteps { kPlan = 1, kRest = 2 };

struct OaplBegin {
  const float* rewards;
  const int32_t* gid;
  const int64_t* off;
  int n_seq, n_groups;
  int64_t Ttok, longest;
  double beta_v;
  double* vstar_ws;
  float* vstar_out;
  int* status;
  static constexpr bool kHasRest = false;
  __device__ __forceinline__ void run(int64_t block, int64_t blocks, int steps) const {
    if (steps == (kPlan | kRest)) clear_status(status);
    sweep_plan(block * 256 + threadIdx.x, blocks * 256, off, n_seq, Ttok, longest, status + kFlagWord);
    group_value(block * 4 + (threadIdx.x >> 6), blocks * 4, rewards, gid, n_seq, n_groups, beta_v, vstar_ws, vstar_out, status);
  }
};

struct GrpoBegin {
  const float* rewards;
  const int32_t* gid;
  const int64_t* off;
  int n_seq, n_groups;
  int64_t Ttok, longest;
  double adv_eps, scale;
  double *gmean, *gstd, *gsize;
  float* adv;
  double* wseq;
  float* adv_out;
  int* status;
  static constexpr bool kHasRest = true;
  __device__ __forceinline__ void run(int64_t block, int64_t blocks, int steps) const {
    if (steps == (kPlan | kRest)) clear_status(status);
    if (steps & kPlan) {
      sweep_plan(block * 256 + threadIdx.x, blocks * 256, off, n_seq, Ttok, longest, status + kFlagWord);
      grpo_group_stats(block * 4 + (threadIdx.x >> 6), blocks * 4, rewards, gid, n_seq, n_groups, gmean, gstd, gsize, status);
    }
    if (steps == (kPlan | kRest)) {
      __threadfence();
      __syncthreads();
    }
    if (steps & kRest)
      grpo_advantage(block * 256 + threadIdx.x, blocks * 256, rewards, gid, off, n_seq, n_groups, Ttok, adv_eps, scale, gmean,
                     gstd, gsize, adv, wseq, adv_out, status);
  }
};

template <class Begin>
__global__ void __launch_bounds__(256) k_begin(Begin begin, int steps) {
  begin.run(blockIdx.x, gridDim.x, steps);
}

// ---------------------------------------------------------------------------
// The objective, from diff = logprob - logq: one workgroup per rollout (at least one), the loss by the last of few to finish
// or, where rollouts are many, in a launch of its own (objective_steps in oapl_api.hip).  It may run any number of times in a
// call; rows not scored yet have diff = 0.
// ---------------------------------------------------------------------------

enum ObjectiveSteps { kRollouts = 1, kLoss = 2 };   // a launch does one of them, or both with the hand-over between them

// The factor that goes into a token's coefficient: `fast` unless the call's flag says that the two-pass schedule served
// it, then `slow`; either may be nullptr (no factor), and so may `flag` (fast).
struct TokenFactor {
  const float *fast, *slow;
  const int* flag;
};
__device__ __forceinline__ const float* token_factor(const TokenFactor f) {
  return f.flag != nullptr && *f.flag != 0 ? f.slow : f.fast;
}

// FINISH: the objective's launch makes the log-probs that it needs, each rollout's workgroup its tokens' (and the first and the
// last those that malformed offsets leave out); fp32 calls, finish_in_objective in oapl_api.hip.
__device__ __forceinline__ void finish_rollout(const LseFinish& f, const int64_t* off, int s0, int n_seq) {
  int64_t a = 0, b = f.Ttok;
  if (n_seq > 0) {
    token_range(off, s0, f.Ttok, a, b);
    if (s0 == 0) a = 0;
    if (s0 == n_seq - 1) b = f.Ttok;
  }
  const int rows = 256 / f.slices;
  for (int64_t t = a; t < b; t += rows) lse_finish<false>(f, t, b);
  __syncthreads();
}
// Only the kernels that finish log-probs take what that needs, and write what they sum up.
struct NoFinish {};
template <bool FINISH>
using FinishArg = std::conditional_t<FINISH, LseFinish, NoFinish>;
template <bool FINISH>
using DiffArg = std::conditional_t<FINISH, const double*, const double* __restrict__>;

// Steps a4, a6, a7: per rollout
//   Delta_s = sum_t diff[t]     (double, fixed order)
//   delta_s = beta_l Delta_s - (r_s - V*_{g(s)})
//   coef[t] = scale 2 beta_l delta_s (times the factor)      = d loss / d ln pi(y_t) for every token of s
// and  loss = scale sum_s delta_s^2   (Eq. 3; one workgroup walks the rollouts, fixed summation order).
// Also validates offsets and group ids; on a violation (or an empty prompt found by
// group_value, whose V* is NaN) the loss is NaN and the status word is set.
template <bool FINISH>
__global__ void __launch_bounds__(256)
k_oapl_objective(DiffArg<FINISH> diff, const float* __restrict__ rewards, const int32_t* __restrict__ gid,
                 const int64_t* __restrict__ off, int n_seq, int n_groups, int64_t Ttok, double beta_l, double scale,
                 const double* __restrict__ vstar_ws, TokenFactor factors, double* Delta, float* __restrict__ coef,
                 float* __restrict__ loss_out, float* __restrict__ seq_logratio_out, int* status, int steps, Gate gate,
                 FinishArg<FINISH> finish) {
  __shared__ int bad;
  if (gate_closed(gate)) return;
  const int tid = threadIdx.x, s0 = blockIdx.x;
  if constexpr (FINISH) {
    if (steps & kRollouts) finish_rollout(finish, off, s0, n_seq);
  }
  auto advantage = [&](int s) {      // r_s - V*
    const int g = gid[s];
    return (double)rewards[s] - (g >= 0 && g < n_groups ? vstar_ws[g] : __builtin_nan(""));
  };
  if ((steps & kRollouts) && s0 < n_seq) {
    // requested before the sum that they are combined with
    const double adv = advantage(s0);
    const float* factor = token_factor(factors);
    int64_t a, b;
    token_range(off, s0, Ttok, a, b);
    double acc = 0.0;
    for (int64_t t = a + tid; t < b; t += 256) acc += diff[t];
    acc = block_sum(acc);
    if (coef) {
      const float c = (float)(scale * 2.0 * beta_l * (beta_l * acc - adv));
      for (int64_t t = a + tid; t < b; t += 256) coef[t] = factor ? c * factor[t] : c;
    }
    if (tid == 0) {
      __hip_atomic_store(Delta + s0, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (seq_logratio_out) seq_logratio_out[s0] = (float)acc;
    }
  }
  if (!(steps & kLoss)) return;
  // the last workgroup's first 256 rollouts: requested before the hand-over, which then costs one round trip less
  const double adv0 = tid < n_seq ? advantage(tid) : 0.0;
  if ((steps & kRollouts) && !last_workgroup(status + kCounterWord, gridDim.x)) return;
  if (tid == 0) bad = (off[0] != 0 || off[n_seq] != Ttok) ? kErrOffsets : 0;
  __syncthreads();
  double acc = 0.0;
  for (int s = tid; s < n_seq; s += 256) {
    if (off[s + 1] < off[s]) atomicCAS(&bad, 0, kErrOffsets);
    if (gid[s] < 0 || gid[s] >= n_groups) atomicCAS(&bad, 0, kErrGroup);
    const double sum = __hip_atomic_load(Delta + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const double delta = beta_l * sum - (s == tid ? adv0 : advantage(s));
    acc += delta * delta;
  }
  acc = block_sum(acc);
  if (tid == 0) {
    double loss = scale * acc;
    if (bad) record_batch_error(status, bad);
    if (batch_error(status)) loss = __builtin_nan("");
    loss_out[0] = (float)loss;
  }
}

// GRPO, token step.  With r_t = pi / pi_old and IS_t = pi_old / pi_vllm,
//   term_t = IS_t min(r_t A, clip(r_t, 1 - eps, 1 + eps) A),   d term_t / d ln pi(y_t) = IS_t r_t A if unclipped else 0,
// it writes the loss gradient coefficient c_t = -w_s d term_t (times the factor) and the rollout's
// loss share -w_s sum_t term_t (double, fixed order); loss = sum of the shares, NaN if an offsets / group error was
// recorded.  lp comes as diff = lp - logq in double.
template <bool FINISH>
__global__ void __launch_bounds__(256)
k_grpo_objective(DiffArg<FINISH> diff, const float* __restrict__ logq, const float* __restrict__ logp_old,
                 const int64_t* __restrict__ off, int n_seq, int64_t Ttok, const float* __restrict__ adv,
                 const double* __restrict__ wseq, double clip_eps, TokenFactor factors, float* __restrict__ coef,
                 double* seqterm, float* __restrict__ loss_out, int* status, int steps, Gate gate, FinishArg<FINISH> finish) {
  if (gate_closed(gate)) return;
  const int tid = threadIdx.x, s0 = blockIdx.x;
  if constexpr (FINISH) {
    if (steps & kRollouts) finish_rollout(finish, off, s0, n_seq);
  }
  if ((steps & kRollouts) && s0 < n_seq) {
    int64_t a, b;
    token_range(off, s0, Ttok, a, b);
    const float* factor = token_factor(factors);
    const double A = (double)adv[s0], w = wseq[s0];
    double acc = 0.0;
    for (int64_t t = a + tid; t < b; t += 256) {
      const double q = (double)logq[t], lo = (double)logp_old[t];
      const double lp = diff[t] + q;
      const double r = exp(lp - lo), is = exp(lo - q);
      const double unclipped = r * A;
      const double rc = r < 1.0 - clip_eps ? 1.0 - clip_eps : (r > 1.0 + clip_eps ? 1.0 + clip_eps : r);
      const double clipped = rc * A;
      acc += is * (unclipped <= clipped ? unclipped : clipped);
      const double g = unclipped <= clipped ? -w * is * unclipped : 0.0;
      if (coef) coef[t] = (float)(factor ? g * (double)factor[t] : g);
    }
    acc = block_sum(acc);
    if (tid == 0) __hip_atomic_store(seqterm + s0, -w * acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!(steps & kLoss) || ((steps & kRollouts) && !last_workgroup(status + kCounterWord, gridDim.x))) return;
  double acc = 0.0;
  for (int s = tid; s < n_seq; s += 256) acc += __hip_atomic_load(seqterm + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  acc = block_sum(acc);
  if (tid == 0) loss_out[0] = batch_error(status) ? __builtin_nanf("") : (float)acc;
}

// Finishes one panel of the single sweep.  Per token row (panel-local index n, global t0 + n):
//   S = sum of the vocabulary-tile partial sums (double, fixed order),  lse = (ref2 + log2 S) ln 2,
//   logprob = min(z_y - lse, 0),  diff = logprob - logq,  nis = -1 / S  (row factor of the gradient, times the
//   correction below),
// and patches the sampled token's entry of the unnormalised soft-max panel, in both packed
// copies, to  Pt[y] - S = -S (1 - p_y)  (computed from expm1 so it is accurate when p_y -> 1).
// Rows whose sum left the accepted range raise the fallback flag.
// 32 slices, four loads each in flight: with 8 slices, one load after the other, a panel of 1003 tokens (594 tiles) took
// 36 us and one of 12288 40 us; now 9 and 13 us.
constexpr int kFinishSlices = 32;
constexpr int kFinishRows = 32;      // token rows per workgroup of kFinishSlices * kFinishRows threads
__global__ void __launch_bounds__(kFinishSlices * kFinishRows)
k_sweep_finish(const float* __restrict__ spart, int n_vt, int64_t ld_s, int64_t n_valid,
               const float* __restrict__ ref2, const float* __restrict__ zy, const float* __restrict__ logq,
               const int32_t* __restrict__ tokens, int V, float* __restrict__ logprob_out,
               double* __restrict__ diff, float* __restrict__ nis, bf16_t* __restrict__ Gp, int g_rows, int g_n_kt,
               bf16_t* __restrict__ GTp, int gt_n_kt, int* __restrict__ status, Gate gate) {
  if (gate_closed(gate)) return;
  // kFinishRows token rows per workgroup; the tile sums of a row are added in kFinishSlices interleaved slices
  // (slice s takes tiles s, s + kFinishSlices, ...), then the slices in order: a fixed order, and
  // enough workgroups to fill the chip with a panel's 12288 rows.
  __shared__ double part[kFinishSlices][kFinishRows];
  const int col = threadIdx.x % kFinishRows, slice = threadIdx.x / kFinishRows;
  const int64_t n = (int64_t)blockIdx.x * kFinishRows + col;
  double acc = 0.0;
  if (n < n_valid) {
#pragma unroll 4
    for (int mt = slice; mt < n_vt; mt += kFinishSlices) acc += (double)spart[(int64_t)mt * ld_s + n];
  }
  part[slice][col] = acc;
  __syncthreads();
  if (slice != 0 || n >= n_valid) return;
  double S = part[0][col];
#pragma unroll
  for (int s = 1; s < kFinishSlices; ++s) S += part[s][col];
  if (!(S <= (double)kSweepLimit)) atomicCAS(status + kFlagWord, 0, 1);     // also catches inf and NaN
  const double lse = ((double)ref2[n] + log2(S)) * kLn2;
  double lp = (double)zy[n] - lse;     // NaN if the token was out of range
  if (lp > 0.0) lp = 0.0;
  if (logprob_out) logprob_out[n] = (float)lp;
  diff[n] = lp - (double)logq[n];
  double row_factor = -1.0 / S;
  const int y = tokens[n];
  if (y >= 0 && y < V) {
    const double entry = S * expm1(lp);                        // -S (1 - p_y)
    const bf16_t patch = (bf16_t)(float)entry;
    // The sampled token's entry carries nearly all of the row's gradient, and bf16 keeps 8 bits of it.
    // The row factor absorbs that rounding: factor * patch is then the exact entry, and the relative
    // error (<= 2^-8) moves to the row's other entries, whose joint weight in the gradient is small.
    const double kept = (double)(float)patch;
    if (kept != 0.0 && isfinite(entry)) row_factor *= entry / kept;
    // both copies are n-side operands: blocks of g_rows tokens and of kPackRowsB vocabulary rows x 64 k
    const int64_t blk = (int64_t)kPackRowsB * kPackK;             // elements of a packed block
    // token row block / row inside it: a division by a constant for all but the few calls in narrower tiles (64 bits by a
    // variable: 165 instructions in a launch that the whole call waits for)
    const uint32_t row = (uint32_t)n, nb = g_rows == kPackRowsB ? row / kPackRowsB : row / (uint32_t)g_rows, nr = row - nb * g_rows;
    const int yb = y / kPackRowsB, yr = y - yb * kPackRowsB;      // vocabulary row block / row inside it
    Gp[(((int64_t)nb * g_n_kt + (y >> 6)) * g_rows + nr) * kPackK + (y & 63)] = patch;
    GTp[((int64_t)yb * gt_n_kt + (n >> 6)) * blk + (int64_t)yr * kPackK + (n & 63)] = patch;
  }
  if (y < 0 || y >= V) record_token_error(status);
  nis[n] = (float)row_factor;
}

}  // namespace oapl
