// fp32 contractions of the OAPL loss head on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and sums).
//
// C[m][n] = sum_k A(m, k) * B(n, k).  Each operand comes either with k contiguous in memory (H and W for the logits,
// dZ^T for dW) or with its row index contiguous (dZ^T and W for dH, H for dW); it lies in the LDS the way it lies in
// memory, so nothing is transposed on the way, and the two orders differ only in how a lane picks its fragment:
//   k contiguous:    [row][BK + 4 floats]; one 16-byte read gives a lane four k of its row (16 lanes: 16 bank groups)
//   rows contiguous: [k][rows + 8 floats]; four 4-byte reads, 32 lanes on one row of 128 bytes, the halves 32 banks apart
// A fragment's four k are 8g + 4 * (lane / 32) + 0..3; multiplication e takes element e of both operands, so the sum over
// k is taken in another order than 0, 1, 2, ...: the same multiset of products.
//
// Bound by the matrix cores (256 flop per clock and CU, 64 clocks per instruction and SIMD) as soon as a few workgroups
// sit on every CU: a 128 x 128 tile needs 8 bytes of operands per clock.  The earlier 64 x 64 tile of plain FMAs was
// bound by its 4-byte LDS reads: a loss call of 1501 tokens at d = 768, V = 8192 took 2.99 ms with it and takes 0.59 ms
// (about 95 TFLOP/s in each contraction; the matrix cores are 66 % busy at 2.4 GHz), one of 256 tokens at d = 64, V = 1024 242
// us and now 35 us.
#pragma once

#include "common.hip.h"
#include "rng.hip.h"
#include "small_kernels.hip.h"

namespace oapl {

struct F32Operand {
  const float* p;
  int64_t ld;    // elements between rows (k contiguous) or between k (rows contiguous)
  bool vec;      // 16-byte loads: p 16-byte aligned and ld a multiple of 4
};

// WM x WN wavefronts (4 in all), each TM x TN blocks of 32 x 32; BK k per LDS stage.
template <int WM_, int WN_, int TM_, int TN_, int BK_>
struct F32Cfg {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, BK = BK_;
  static constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  static_assert(WM * WN == 4 && BK % 8 == 0, "256 threads, whole groups of eight k");
  // workgroups that the registers of a shared launch must leave room for on a CU: of the large tile four, as many as the LDS
  // does (left alone it takes 130 registers and leaves room for three); the small one's 81 leave that room unasked
  static constexpr int kPerCU = BM * BN >= 128 * 128 ? 4 : 2;
};
typedef F32Cfg<2, 2, 2, 2, 16> F32Large;   // 128 x 128, 40 KB of LDS
typedef F32Cfg<2, 2, 1, 1, 32> F32Small;   // 64 x 64, 36 KB
typedef F32Cfg<1, 4, 2, 1, 32> F32Flat;    // 64 x 128, 54 KB: logits of few tokens (a wavefront still owns 64 vocabulary rows)

// One operand's ROWS x BK stage: global -> registers -> LDS.
template <int ROWS, int BK, bool KC>
struct F32Stage {
  static constexpr int PITCH = KC ? BK + 4 : ROWS + 8;
  static constexpr int FLOATS = KC ? ROWS * PITCH : BK * PITCH;
  static constexpr int N = ROWS * BK / 4 / 256;     // 4-float pieces per thread
  f32x4 v[N];

  __device__ __forceinline__ void load(const F32Operand& o, int64_t r0, int64_t R, int64_t k0, int64_t k_end) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = threadIdx.x + i * 256;
      const int64_t r = r0 + (KC ? idx / (BK / 4) : idx % (ROWS / 4) * 4);
      const int64_t k = k0 + (KC ? idx % (BK / 4) * 4 : idx / (ROWS / 4));
      const float* p = o.p + (KC ? r * o.ld + k : k * o.ld + r);
      const bool whole = KC ? r < R && k + 4 <= k_end : k < k_end && r + 4 <= R;
      if (o.vec && whole) {
        v[i] = *(const f32x4*)p;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = KC ? r < R && k + e < k_end : k < k_end && r + e < R;
          v[i][e] = ok ? p[e] : 0.f;
        }
      }
    }
  }
  __device__ __forceinline__ void store(float* s) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = threadIdx.x + i * 256;
      const int a = KC ? idx / (BK / 4) * PITCH + idx % (BK / 4) * 4 : idx / (ROWS / 4) * PITCH + idx % (ROWS / 4) * 4;
      *(f32x4*)(s + a) = v[i];
    }
  }
  // four k of row `row` (of the tile) in group g of eight, for this lane's half
  static __device__ __forceinline__ f32x4 fragment(const float* s, int row, int g, int half) {
    if (KC) return *(const f32x4*)(s + row * PITCH + g * 8 + half * 4);
    f32x4 f;
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = s[(g * 8 + half * 4 + e) * PITCH + row];
    return f;
  }
};

// Row inside a 32 x 32 block of accumulator register r, before the lane-half term 4 * (lane / 32); the column is lane % 32.
__device__ __forceinline__ constexpr int f32_acc_row(int r) { return 8 * (r >> 2) + (r & 3); }

// LDS of a tile: two stages of each operand.
template <class C, bool A_KC>
constexpr int f32_lds_a() { return 2 * F32Stage<C::BM, C::BK, A_KC>::FLOATS; }
template <class C, bool B_KC>
constexpr int f32_lds_b() { return 2 * F32Stage<C::BN, C::BK, B_KC>::FLOATS; }
constexpr int larger(int a, int b) { return a > b ? a : b; }

// Tile at block (bx, by, bz): x and y = row and column tiles in the order the epilogue names, z = one of `nz` splits of k in
// whole stages.
template <class C, bool A_KC, bool B_KC, class Epi>
__device__ __forceinline__ void gemm_f32_tile(const F32Operand& A, const F32Operand& B, int64_t M, int64_t N, int64_t K,
                                              const Epi& epi, unsigned bx, unsigned by, unsigned bz, unsigned nz,
                                              float* lds_a, float* lds_b) {
  typedef F32Stage<C::BM, C::BK, A_KC> SA;
  typedef F32Stage<C::BN, C::BK, B_KC> SB;
  float (*As)[SA::FLOATS] = (float (*)[SA::FLOATS])lds_a;
  float (*Bs)[SB::FLOATS] = (float (*)[SB::FLOATS])lds_b;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const int wm = wave / C::WN, wn = wave % C::WN;
  const int64_t m0 = (int64_t)(Epi::kRowsOnX ? bx : by) * C::BM;
  const int64_t n0 = (int64_t)(Epi::kRowsOnX ? by : bx) * C::BN;
  const int64_t stages = (K + C::BK - 1) / C::BK;
  const int64_t kb = stages * bz / nz * C::BK;
  int64_t ke = stages * (bz + 1) / nz * C::BK;
  ke = ke < K ? ke : K;

  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  SA sa;
  SB sb;
  if (kb < ke) {
    sa.load(A, m0, M, kb, ke);
    sb.load(B, n0, N, kb, ke);
    sa.store(As[0]);
    sb.store(Bs[0]);
  }
  __syncthreads();
  int cur = 0;
  for (int64_t k = kb; k < ke; k += C::BK) {
    const bool more = k + C::BK < ke;
    if (more) {     // the next stage's loads travel while this one is multiplied
      sa.load(A, m0, M, k + C::BK, ke);
      sb.load(B, n0, N, k + C::BK, ke);
    }
#pragma unroll
    for (int g = 0; g < C::BK / 8; ++g) {
      f32x4 a[C::TM], b[C::TN];
#pragma unroll
      for (int i = 0; i < C::TM; ++i) a[i] = SA::fragment(As[cur], (wm * C::TM + i) * 32 + (lane & 31), g, half);
#pragma unroll
      for (int j = 0; j < C::TN; ++j) b[j] = SB::fragment(Bs[cur], (wn * C::TN + j) * 32 + (lane & 31), g, half);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
          for (int j = 0; j < C::TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
    }
    if (more) {     // the other buffer was last read before the previous barrier
      sa.store(As[cur ^ 1]);
      sb.store(Bs[cur ^ 1]);
    }
    __syncthreads();
    cur ^= 1;
  }
  epi.template store<C::TM, C::TN>(acc, m0 + wm * C::TM * 32, n0 + wn * C::TN * 32 + (lane & 31), half, M, N, bz);
}

// Grid as gemm_f32_tile's block (y holds at most 65535).  Two workgroups per CU at least: one's products cover the other's
// stage turn.
template <class C, bool A_KC, bool B_KC, class Epi>
__global__ void __launch_bounds__(256, 2) k_gemm_f32(F32Operand A, F32Operand B, int64_t M, int64_t N, int64_t K, Epi epi) {
  __shared__ __attribute__((aligned(16))) float As[f32_lds_a<C, A_KC>()], Bs[f32_lds_b<C, B_KC>()];
  gemm_f32_tile<C, A_KC, B_KC>(A, B, M, N, K, epi, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, As, Bs);
}

// The epilogues get a wavefront's accumulators, its first row and the lane's first column.

// Logits: M = vocabulary, N = tokens.  Per token and 64 vocabulary rows (one wavefront) the pair
// (m, s) = (max_v z, sum_v exp(z - m)); parts[v / 64][t].  With `zt` the logits themselves are kept as well, for a batch
// whose gradient fits one panel: zt[v][t].
struct EpiLseF32 {
  static constexpr bool kRowsOnX = true;
  float2* parts;
  int64_t T;
  float* upart;   // optional third partial u = sum_v exp(z - m) * z (for the entropy), or nullptr
  float* zt;      // or nullptr
  int64_t ldz;
  template <int TM, int TN>
  __device__ void store(f32x16 (&acc)[TM][TN], int64_t m, int64_t n, int half, int64_t M, int64_t N, unsigned split) const {
    static_assert(TM == 2, "a partial is 64 vocabulary rows");
    if (m >= M) return;
    const int left = (int)(M - m < 64 ? M - m : 64) - 4 * half;   // this lane's rows r with row(r) >= left do not exist
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t t = n + j * 32;
      if (zt && t < N) {
        float* z0 = zt + (m + 4 * half) * ldz + t;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (i * 32 + f32_acc_row(r) < left) *z0 = acc[i][j][r];
            z0 += (r & 3) == 3 ? 5 * ldz : ldz;
          }
      }
      if (left < 64 - 4) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (i * 32 + f32_acc_row(r) >= left) acc[i][j][r] = -__builtin_inff();
      }
      float mx = -__builtin_inff();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[i][j][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float ref = fmaxf(mx, kNegHuge);
      // quads of rows in turn, then the quads pairwise: seven roundings deep with the two halves, where a walk over the
      // lane's 32 rows would be 32 (entropies of 256 x 1024 logits at d = 64: 1.7e-6 rms off that way)
      float sq[TM * 4], uq[TM * 4];
#pragma unroll
      for (int k = 0; k < TM * 4; ++k) {
        sq[k] = uq[k] = 0.f;
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const float z = acc[k / 4][j][4 * (k % 4) + e4], e = expf(z - ref);
          sq[k] += e;
          if (upart) uq[k] += e > 0.f ? e * z : 0.f;
        }
      }
#pragma unroll
      for (int step = TM * 2; step > 0; step /= 2)
#pragma unroll
        for (int k = 0; k < step; ++k) {
          sq[k] += sq[k + step];
          uq[k] += uq[k + step];
        }
      float s = sq[0], u = uq[0];
      s += __shfl_xor(s, 32, 64);
      u += __shfl_xor(u, 32, 64);
      if (half == 0 && t < N) {
        parts[(m >> 6) * T + t] = make_float2(ref, s);
        if (upart) upart[(m >> 6) * T + t] = u;
      }
    }
  }
};

// Sampling: M = vocabulary, N = tokens.  Per token and 64 vocabulary rows the best perturbed logit
// z / temperature + Gumbel(Philox(seed; v / 4, t)) and its vocabulary index; parts[v / 64][t].
struct EpiSampleF32 {
  static constexpr bool kRowsOnX = true;
  float2* parts;
  int64_t T;
  float inv_temperature;
  uint32_t seed_lo, seed_hi;
  template <int TM, int TN>
  __device__ void store(f32x16 (&acc)[TM][TN], int64_t m, int64_t n, int half, int64_t M, int64_t N, unsigned split) const {
    static_assert(TM == 2, "a partial is 64 vocabulary rows");
    if (m >= M) return;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t t = n + j * 32;
      float best = -__builtin_inff();
      int arg = 0x7FFFFFFF;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t v = m + i * 32 + 8 * q + 4 * half;      // multiple of 4: one Philox block
          uint32_t x[4];
          philox4x32_10((uint32_t)(v >> 2), (uint32_t)t, (uint32_t)(t >> 32), 0u, seed_lo, seed_hi, x);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float sc = __builtin_fmaf(acc[i][j][4 * q + e], inv_temperature, gumbel_from_bits(x[e]));
            if (v + e < M && sc > best) { best = sc; arg = (int)(v + e); }   // indices rise: strict > keeps the smallest
          }
        }
      const float so = __shfl_xor(best, 32, 64);
      const int io = __shfl_xor(arg, 32, 64);
      if (better(so, io, best, arg)) { best = so; arg = io; }
      if (half == 0 && t < N) parts[(m >> 6) * T + t] = make_float2(best, __int_as_float(arg));
    }
  }
};

// dZ^T[v][t] = c_t (1[v == y_t] - exp(z - lse_t)): from logits just computed (a batch of several panels) ...
__device__ __forceinline__ float dz_f32(float z, int v, int y, float c, float lse) {
  return c * ((v == y ? 1.f : 0.f) - expf(z - lse));
}
struct EpiDzF32 {
  static constexpr bool kRowsOnX = true;
  const int32_t* tokens;
  const float* lse;
  const float* coef;
  float* zt;
  int64_t ldz;
  template <int TM, int TN>
  __device__ void store(f32x16 (&acc)[TM][TN], int64_t m, int64_t n, int half, int64_t M, int64_t N, unsigned split) const {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t t = n + j * 32;
      if (t >= N) continue;
      const float c = coef[t], l = lse[t];
      const int left = (int)(M - m < 64 ? M - m : 64) - 4 * half, y = tokens[t] - (int)m - 4 * half;
      float* z0 = zt + (m + 4 * half) * ldz + t;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = i * 32 + f32_acc_row(r);
          if (row < left) *z0 = dz_f32(acc[i][j][r], row, y, c, l);
          z0 += (r & 3) == 3 ? 5 * ldz : ldz;
        }
    }
  }
};

// ... or in place from the logits the scoring pass kept: 256 tokens x 4 vocabulary rows per workgroup (sixteen rows took
// 8 us for 256 x 1024 logits, a chain of loads on a quarter of the chip).  Bound by memory
// (8 bytes per logit): 20 us for 1501 x 8192, a tenth of computing them again at d = 768.
constexpr int kDzRows = 4;
__global__ void __launch_bounds__(256)
k_dz_f32(float* __restrict__ zt, int64_t ldz, int V, int64_t T, const int32_t* __restrict__ tokens,
         const float* __restrict__ lse, const float* __restrict__ coef) {
  const int64_t t = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (t >= T) return;
  const float c = coef[t], l = lse[t];
  const int y = tokens[t];
  const int v0 = blockIdx.x * kDzRows;
  float z[kDzRows];
#pragma unroll
  for (int i = 0; i < kDzRows; ++i)
    if (v0 + i < V) z[i] = zt[(int64_t)(v0 + i) * ldz + t];
#pragma unroll
  for (int i = 0; i < kDzRows; ++i)
    if (v0 + i < V) zt[(int64_t)(v0 + i) * ldz + t] = dz_f32(z[i], v0 + i, y, c, l);
}

// Plain store, or read-add-store, of the tile into C[m][n]; with several splits of k each writes its own [M][N] copy.
struct EpiStoreF32 {
  static constexpr bool kRowsOnX = false;
  float* C;
  int64_t ld;
  int accumulate;
  template <int TM, int TN>
  __device__ void store(f32x16 (&acc)[TM][TN], int64_t m, int64_t n, int half, int64_t M, int64_t N, unsigned split) const {
    float* out = C + (int64_t)split * M * N;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t row = m + i * 32 + f32_acc_row(r) + 4 * half, col = n + j * 32;
          if (row < M && col < N) {
            float* p = out + row * ld + col;
            *p = accumulate ? *p + acc[i][j][r] : acc[i][j][r];
          }
        }
  }
};

// out = the splits' partial results, in order, of two contractions (n = 0: there is only one).
struct F32Reduction {
  const float* part;
  int splits;
  int64_t n;
  float* out;
};
__global__ void __launch_bounds__(256) k_reduce_f32(F32Reduction a, F32Reduction b) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n + b.n; i += (int64_t)gridDim.x * 256) {
    const bool first = i < a.n;
    const float* part = first ? a.part + i : b.part + (i - a.n);
    const int splits = first ? a.splits : b.splits;
    const int64_t n = first ? a.n : b.n;
    float sum = 0.f;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) sum += part[(int64_t)s * n];
    (first ? a.out + i : b.out + (i - a.n))[0] = sum;
  }
}

// The first launch of a loss call of few tokens: what the call begins with (workgroup 0), the sampled tokens' logits (four per
// workgroup) and the logits' tiles.  None needs the others, and a launch costs such a call 3 .. 5 us.
template <class C, class Epi, class Begin, int VEC>
__global__ void __launch_bounds__(256, 2)
k_scores_f32(Begin begin, const int32_t* __restrict__ tokens, float* __restrict__ zy, TokenInit init, F32Operand W, F32Operand H,
             int V, int64_t T, int d, Epi epi) {
  __shared__ __attribute__((aligned(16))) float As[f32_lds_a<C, true>()], Bs[f32_lds_b<C, true>()];
  int64_t b = blockIdx.x;
  if (b == 0) return begin.run(0, 1, kPlan | kRest);
  b -= 1;
  const int64_t n_gather = (T + 3) / 4, rows = (V + C::BM - 1) / C::BM;
  if (b < n_gather)
    return gather_logit<float, double, VEC>(b * 4 + (threadIdx.x >> 6), H.p, W.p, tokens, T, d, V, zy, nullptr, init);
  b -= n_gather;
  gemm_f32_tile<C, true, true>(W, H, (int64_t)V, T, (int64_t)d, epi, b % rows, b / rows, 0, 1, As, Bs);
}

// One contraction with its splits; `grid` = (columns, rows, splits) of tiles.
struct F32Contraction {
  F32Operand A, B;
  int64_t M, N, K;
  float* out;      // [splits][M][N]
  int nx, ny, splits;
};
// dH (rows of dZ^T contiguous) and dW (k contiguous) of a batch of one panel in one launch: neither fills the chip to
// the end, and they do not depend on each other.
template <class CH, class CW>
__global__ void __launch_bounds__(256, larger(CH::kPerCU, CW::kPerCU)) k_grads_f32(F32Contraction dh, F32Contraction dw) {
  __shared__ __attribute__((aligned(16))) float As[larger(f32_lds_a<CH, false>(), f32_lds_a<CW, true>())],
      Bs[larger(f32_lds_b<CH, false>(), f32_lds_b<CW, false>())];
  const int64_t n_dh = (int64_t)dh.nx * dh.ny * dh.splits;
  int64_t i = blockIdx.x;
  if (i < n_dh) {
    gemm_f32_tile<CH, false, false>(dh.A, dh.B, dh.M, dh.N, dh.K, EpiStoreF32{dh.out, dh.N, 0}, i % dh.nx, i / dh.nx % dh.ny,
                                    (unsigned)(i / ((int64_t)dh.nx * dh.ny)), dh.splits, As, Bs);
    return;
  }
  i -= n_dh;
  gemm_f32_tile<CW, true, false>(dw.A, dw.B, dw.M, dw.N, dw.K, EpiStoreF32{dw.out, dw.N, 0}, i % dw.nx, i / dw.nx % dw.ny,
                                 (unsigned)(i / ((int64_t)dw.nx * dw.ny)), dw.splits, As, Bs);
}

}  // namespace oapl
