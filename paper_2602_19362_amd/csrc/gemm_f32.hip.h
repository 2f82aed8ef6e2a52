// fp32 contractions of the OAPL loss head, on the bf16 matrix cores: C[m][n] = sum_k A(m, k) * B(n, k).
//
// An fp32 number is the sum of three bf16 numbers, each the rounding of what the ones before leave (24 bits; the signs of the
// later parts make up for the bits between): x = x0 + x1 + x2, to the bit, with |x1| <= 2^-8 |x| and |x2| <= 2^-17 |x| (Henry, Tang
// and Heinecke, 2019).  Of the nine products of two such sums eight are taken,
//     x0 y0  +  (x0 y1 + x1 y0)  +  (x1 y1 + x0 y2 + x2 y0)  +  (x1 y2 + x2 y1),
// and x2 y2, at most 2^-34 |x y|, is under half a place of the sum that it would go into.  (x1 y2 + x2 y1 reach 2^-24 |x y|, as
// much as the rounding of an fp32 product: a logit of one product 0.97 places off without them, 0.51 with.)
// A tile in which a number is past the parts' range, or a sum past that of fp32 at the parts' scale, infinite or NaN, is multiplied
// once more, as v_mfma_f32_32x32x2_f32 does it: every fp32 number is an operand, to the last bit.  (1501 tokens at d = 768, V =
// 8192 with every tile of the logits and of one gradient done twice 828 us.)
// v_mfma_f32_32x32x16_bf16 does a product exactly and sixteen times as fast as v_mfma_f32_32x32x2_f32 does an fp32 one.  The first
// products are added up apart from the others: a matrix core's addition cuts addends far below its result off downwards (-0.003
// ulp on average), which as many additions into the large sum turned into a bias of 2e-7 of a token's log-prob (with two sums
// 2e-8).  Against fp64, relative errors of log-probs fp32 multiplications / here: 256 tokens at d = 64, V = 1024 3.3e-7 / 1.6e-7,
// 1501 at d = 768, V = 8192 6.9e-7 / 2.6e-7; of dW 5.5e-6 / 3.7e-6, 1.2e-5 / 4.8e-6; over 14 shapes up to those 0.42 and 0.57
// times.
//
// Each operand comes either with k contiguous in memory (H and W for the logits, dZ^T for dW) or with its row index contiguous
// (dZ^T and W for dH, H for dW); in the LDS its parts lie with k contiguous, as the fragments want them.  A thread splits
// what it loaded before it writes it there (13 vector operations for two numbers), once for all that read it.
//
// What bounds it is the sum of things that share a SIMD and its clock, multiplications, splitting and fragments, and the waits
// between them: at 1501 x 8192 x 768 matrix cores are busy 0.40 .. 0.46 of the time (at 2.1 GHz), vector ALUs 0.22 .. 0.33, the LDS
// 0.15 .. 0.21; 116 .. 122 TFLOP/s of fp32 products.  A loss call of 1501 tokens at d = 768, V = 8192 takes 482 us; with six
// products (and less than fp32's precision) 414, with fp32 multiplications, whose matrix cores were 66 % busy, 590, with plain FMAs
// 2990.  160 calls of up to 2000 tokens at d <= 768, V <= 8192, times fp32 multiplications': losses 0.88 on average, 0.63 .. 1.02,
// scores 0.80, 0.44 .. 0.99.
#pragma once

#include "common.hip.h"
#include "rng.hip.h"
#include "small_kernels.hip.h"

namespace oapl {

struct F32Operand {
  const float* p;
  int64_t ld;    // elements between rows (k contiguous) or between k (rows contiguous)
  bool vec;      // p 16-byte aligned and ld a multiple of 4
};

// WM x WN wavefronts, each TM x TN blocks of 32 x 32; BK k per LDS stage.
template <int WM_, int WN_, int TM_, int TN_>
struct F32Cfg {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, BK = 32;
  static constexpr int BM = WM * TM * 32, BN = WN * TN * 32, NT = WM * WN * 64;
  static constexpr int STAGE_A = 3 * BM * BK * 2, STAGE_B = 3 * BN * BK * 2;   // LDS bytes of one stage
  // eight wavefronts, a CU to themselves, have two stages
  static constexpr bool TWO_STAGES = WM * WN == 8;
  static constexpr int LDS = (TWO_STAGES ? 2 : 1) * (STAGE_A + STAGE_B);
  static_assert(WM * WN == 4 || TWO_STAGES, "256 or 512 threads");
  static_assert(LDS <= 160 * 1024, "LDS of one CU");
};
typedef F32Cfg<4, 2, 2, 2> F32Wide;    // 256 x 128, 144 KB of LDS
typedef F32Cfg<2, 2, 2, 2> F32Large;   // 128 x 128, 48 KB
typedef F32Cfg<2, 2, 1, 1> F32Small;   // 64 x 64, 24 KB
typedef F32Cfg<1, 4, 2, 1> F32Flat;    // 64 x 128, 36 KB: logits of few tokens (a wavefront still owns 64 vocabulary rows)

// Numbers are multiplied by 2^24 before they are split, which makes every part of every one of them, down to the least, a normal
// bf16 number or zero.  The parts of numbers from 2^104 on are infinite, the last one NaN, and so is every sum that they go into.
constexpr float kF32Scale = 16777216.f;
constexpr float kF32Unscale = 1.f / kF32Scale / kF32Scale;     // ... of a product

// The bf16 parts of two fp32 numbers, packed: x = hi + mid + lo.
struct F32Parts {
  uint32_t hi, mid, lo;
};
__device__ __forceinline__ uint32_t f32_bf16_pair(float x0, float x1) {
  const bf16x2 v = {(bf16_t)x0, (bf16_t)x1};
  uint32_t u = __builtin_bit_cast(uint32_t, v);
  asm("" : "+v"(u));     // or the compiler converts x0 a second time, alone, for the difference
  return u;
}
__device__ __forceinline__ F32Parts f32_split(float x0, float x1) {
  F32Parts p;
  p.hi = f32_bf16_pair(x0, x1);
  const float r0 = x0 - __uint_as_float(p.hi << 16), r1 = x1 - __uint_as_float(p.hi & 0xFFFF0000u);
  p.mid = f32_bf16_pair(r0, r1);
  p.lo = f32_bf16_pair(r0 - __uint_as_float(p.mid << 16), r1 - __uint_as_float(p.mid & 0xFFFF0000u));
  return p;
}

// One operand's ROWS x 32 stage by NT threads: global -> registers -> three planes of bf16 parts in LDS, [row][k] whatever the
// order in memory.  A thread has pieces of four k of one row.  k contiguous: eight lanes load the 128 bytes of a row, a
// line, by 16 (by 32 in two loads every line is asked for twice).  Rows contiguous: 64 lanes load 64 rows of one k, and two
// pieces, eight k, are written at once.  16-byte chunk c of row r lies at chunk c ^ (r / 4 % 4): 16 lanes that read one chunk
// of consecutive rows, or write one, or write whole rows, touch all banks.  The numbers themselves (store_plain) take two
// planes, sixteen k each.
template <int ROWS, int NT, bool KC>
struct F32Stage {
  static constexpr int PITCH = 64, PLANE = ROWS * PITCH;
  static constexpr int N = ROWS * 8 / NT;     // pieces per thread
  static __device__ __forceinline__ int at(int row, int c) { return row * PITCH + ((c ^ ((row >> 2) & 3)) << 4); }
  const float* p[KC ? 1 : N / 2];   // the next stage, from the tile's first row; not KC: the wavefront's chunks of it
  f32x4 v[N];
  u32x2 hi[N], mid[N], lo[N];
  int64_t ld;
  uint32_t off[KC ? N : 1];         // KC: bytes from there to this thread's pieces (a tile has under 2^32); else the thread's row
  int wave;

  // not KC: chunk i of this wavefront
  __device__ __forceinline__ int chunk(int i) const { return wave * 64 / ROWS + i * (NT / ROWS); }
  // Rows past the matrix are its last row again: what they give is not stored.
  __device__ __forceinline__ void init(const F32Operand& o, int64_t r0, int64_t R, int64_t k0, unsigned tid) {
    ld = o.ld;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int last = (int)(R - r0 < ROWS ? R - r0 : ROWS) - 1;
    if constexpr (KC) {
      p[0] = o.p + r0 * ld + k0;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int row = (tid + i * NT) >> 3;
        off[i] = ((uint32_t)(row < last ? row : last) * (uint32_t)ld + (tid & 7) * 4) * 4;
      }
    } else {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) p[i] = o.p + (k0 + chunk(i) * 8) * ld + r0;
      const int row = tid % ROWS;
      off[0] = (uint32_t)(row < last ? row : last);
    }
  }
  // The next stage, of which `left` k exist; leaves the pointers at the one behind it.  k past the end are zeros.
  __device__ __forceinline__ void load(int64_t left) {
    if constexpr (KC) {
      auto piece = [&](int i) {
        uint32_t o = off[i];
        asm("" : "+v"(o));      // or the compiler steps N addresses of 64 bits
        return (const char*)p[0] + o;
      };
      if (left >= 32) {
        typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = *(const f32x4_any*)piece(i);
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][e] = (int)(threadIdx.x & 7) * 4 + e < left ? ((const float*)piece(i))[e] : 0.f;
      }
      p[0] += 32;
    } else {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[2 * i + e / 4][e % 4] = left >= 32 || chunk(i) * 8 + e < left ? (p[i] + e * ld)[off[0]] : 0.f;
        p[i] += 32 * ld;
      }
    }
  }
  __device__ __forceinline__ void split() {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const F32Parts x = f32_split(v[i][2 * e] * kF32Scale, v[i][2 * e + 1] * kF32Scale);
        hi[i][e] = x.hi;
        mid[i][e] = x.mid;
        lo[i][e] = x.lo;
      }
  }
  __device__ __forceinline__ void store(lds_char_ptr s) const {
    typedef __attribute__((address_space(3))) u32x2* piece;
    typedef __attribute__((address_space(3))) u32x4* pieces;
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const lds_char_ptr d = s + at((threadIdx.x + i * NT) >> 3, (threadIdx.x & 7) >> 1) + (threadIdx.x & 1) * 8;
        *(piece)d = hi[i];
        *(piece)(d + PLANE) = mid[i];
        *(piece)(d + 2 * PLANE) = lo[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const lds_char_ptr d = s + at(threadIdx.x % ROWS, chunk(i));
        *(pieces)d = __builtin_shufflevector(hi[2 * i], hi[2 * i + 1], 0, 1, 2, 3);
        *(pieces)(d + PLANE) = __builtin_shufflevector(mid[2 * i], mid[2 * i + 1], 0, 1, 2, 3);
        *(pieces)(d + 2 * PLANE) = __builtin_shufflevector(lo[2 * i], lo[2 * i + 1], 0, 1, 2, 3);
      }
    }
  }
  __device__ __forceinline__ void store_plain(lds_char_ptr s) const {
    typedef __attribute__((address_space(3))) f32x4* piece;
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        *(piece)(s + ((threadIdx.x & 7) >> 2) * PLANE + at((threadIdx.x + i * NT) >> 3, threadIdx.x & 3)) = v[i];
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int c = chunk(i / 2) * 2 + (i & 1);     // of eight
        *(piece)(s + (c >> 2) * PLANE + at(threadIdx.x % ROWS, c & 3)) = v[i];
      }
    }
  }
  // ... back: the four k 8 * g + 4 * half of a row
  static __device__ __forceinline__ f32x4 plain(lds_char_ptr s, int row, int g, int half) {
    return *(const __attribute__((address_space(3))) f32x4*)(s + (g >> 1) * PLANE + at(row, (g & 1) * 2 + half));
  }
};

// Row inside a 32 x 32 block of accumulator register r, before the lane-half term 4 * (lane / 32); the column is lane % 32.
__device__ __forceinline__ constexpr int f32_acc_row(int r) { return 8 * (r >> 2) + (r & 3); }

constexpr int larger(int a, int b) { return a > b ? a : b; }

// Tile at block (bx, by, bz): x and y = column and row of tiles, z = one of `nz` splits of k in whole stages.
template <class C, bool A_KC, bool B_KC, class Epi>
__device__ __forceinline__ void gemm_f32_tile(const F32Operand& A, const F32Operand& B, int64_t M, int64_t N, int64_t K,
                                              const Epi& epi, unsigned bx, unsigned by, unsigned bz, unsigned nz,
                                              char* lds_raw) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef F32Stage<C::BM, C::NT, A_KC> SA;
  typedef F32Stage<C::BN, C::NT, B_KC> SB;
  constexpr int STAGE = C::STAGE_A + C::STAGE_B;
  const lds_char_ptr lds = (lds_char_ptr)lds_raw;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int wm = wave / C::WN, wn = wave % C::WN;
  const int64_t m0 = (int64_t)by * C::BM, n0 = (int64_t)bx * C::BN;
  const int64_t stages = (K + C::BK - 1) / C::BK;
  const int64_t s0 = stages * bz / nz;
  const int n_stages = (int)(stages * (bz + 1) / nz - s0);
  const int64_t kb = s0 * C::BK, len = K - kb;

  // acc: the products of the first parts; small: the others, 2^-7 of those and less
  f32x16 acc[C::TM][C::TN], small[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = small[i][j][r] = 0.f;

  SA sa;
  SB sb;
  sa.init(A, m0, M, kb, threadIdx.x);
  sb.init(B, n0, N, kb, threadIdx.x);
  auto load = [&](int s) {
    sa.load(len - (int64_t)s * C::BK);
    sb.load(len - (int64_t)s * C::BK);
  };
  auto split = [&] {
    sa.split();
    sb.split();
  };
  auto store = [&](lds_char_ptr to) {
    sa.store(to);
    sb.store(to + C::STAGE_A);
  };
  const int fa = SA::at(wm * C::TM * 32 + (lane & 31), half), fb = C::STAGE_A + SB::at(wn * C::TN * 32 + (lane & 31), half);
  auto multiply = [&](const lds_char_ptr from) {
    typedef const __attribute__((address_space(3))) bf16x8* fragment;
    bf16x8 a[2][C::TM], b[2][C::TN], am[C::TM], bm[C::TN], al[C::TM], bl[C::TN];
    auto read = [&](bf16x8 (&x)[C::TM], bf16x8 (&y)[C::TN], const int ks, const int q) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i) x[i] = *(fragment)(from + (fa ^ (ks << 5)) + q * SA::PLANE + i * 32 * SA::PITCH);
#pragma unroll
      for (int j = 0; j < C::TN; ++j) y[j] = *(fragment)(from + (fb ^ (ks << 5)) + q * SB::PLANE + j * 32 * SB::PITCH);
    };
    auto products = [&](f32x16 (&to)[C::TM][C::TN], const bf16x8 (&x)[C::TM], const bf16x8 (&y)[C::TN]) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) to[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], y[j], to[i][j], 0, 0, 0);
    };
    // fragments are requested eight multiplications and more ahead, but for a stage's first
    read(a[0], b[0], 0, 0);
    read(am, bm, 0, 1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      read(al, bl, ks, 2);
      __builtin_amdgcn_sched_barrier(0);
      products(acc, a[ks], b[ks]);
      products(small, a[ks], bm);
      products(small, am, b[ks]);
      products(small, am, bm);
      products(small, am, bl);
      products(small, al, bm);
      __builtin_amdgcn_sched_barrier(0);
      if (ks == 0) {
        read(a[1], b[1], 1, 0);
        read(am, bm, 1, 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      products(small, a[ks], bl);
      products(small, al, b[ks]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  load(0);
  split();
  store(lds);
  if constexpr (C::TWO_STAGES) {
    // Two stages in LDS: s is multiplied while s + 1 is split and written, by half of the wavefronts, one per SIMD, before they
    // multiply and by the others afterwards, so that a SIMD's two wavefronts do not both multiply and then both split. The
    // barrier waits for the LDS only: loads stay in flight.
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto next = [&](int s) {
      if (s >= n_stages) return;
      split();
      store(lds + (s & 1) * STAGE);
      if (s + 1 < n_stages) load(s + 1);
    };
    if (n_stages > 1) load(1);
    barrier();
    for (int s = 0; s < n_stages; ++s) {
      if (wave >= 4) next(s + 1);
      multiply(lds + (s & 1) * STAGE);
      if (wave < 4) next(s + 1);
      barrier();
    }
  } else {
    __syncthreads();
    for (int s = 0; s < n_stages; ++s) {
      const bool more = s + 1 < n_stages;
      if (more) load(s + 1);     // the next stage's loads travel while this one is multiplied
      multiply(lds);
      if (more) {
        split();
        __syncthreads();      // everyone has read the stage
        store(lds);
        __syncthreads();
      }
    }
  }
  float finite = 0.f;     // 0 times every sum: NaN if one is not finite
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float sum = acc[i][j][r] + small[i][j][r];
        finite = __builtin_fmaf(sum, 0.f, finite);
        acc[i][j][r] = sum * kF32Unscale;
      }
  // Numbers without parts (infinities and NaN among them), or sums that the scale took out of range: once more, with fp32
  // multiplications.
  if (__builtin_expect(__syncthreads_or(!(finite == 0.f)), 0)) {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    unsigned tid = threadIdx.x;
    asm volatile("" : "+v"(tid));     // or the first pass keeps its addresses for this one
    sa.init(A, m0, M, kb, tid);
    sb.init(B, n0, N, kb, tid);
    for (int s = 0; s < n_stages; ++s) {
      load(s);
      __syncthreads();      // everyone has read the stage before
      sa.store_plain(lds);
      sb.store_plain(lds + C::STAGE_A);
      __syncthreads();
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 a[C::TM], b[C::TN];
#pragma unroll
        for (int i = 0; i < C::TM; ++i) a[i] = SA::plain(lds, (wm * C::TM + i) * 32 + (lane & 31), g, half);
#pragma unroll
        for (int j = 0; j < C::TN; ++j) b[j] = SB::plain(lds + C::STAGE_A, (wn * C::TN + j) * 32 + (lane & 31), g, half);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
      }
    }
  }
  epi.template store<C::TM, C::TN>(acc, m0 + wm * C::TM * 32, n0 + wn * C::TN * 32 + (lane & 31), half, M, N, bz);
#endif
}

// A grid for so many tiles (columns * rows * splits), with as many threads in a dimension as HIP takes (2^32 less one) at 512 a
// workgroup.  Every XCD has a range of the splits, and of the rows in them, and walks their columns first, so that few others
// read the same part of A: 1501 x 768 x 8192 in seven splits 10.6 MB per XCD in place of all 75 (logits of 1501 tokens at d = 768,
// V = 8192 133 / 127 us, with the loads by whole lines).
static inline dim3 f32_grid(int64_t tiles) {
  const int64_t x = (tiles + 7) / 8 * 8, most = 1 << 22;
  return x <= most ? dim3((unsigned)x) : dim3((unsigned)most, (unsigned)((x + most - 1) / most));
}
template <class C, bool A_KC, bool B_KC, class Epi>
__global__ void __launch_bounds__(C::NT, 2) k_gemm_f32(F32Operand A, F32Operand B, int64_t M, int64_t N, int64_t K, Epi epi,
                                                       unsigned splits) {
  extern __shared__ __attribute__((aligned(256))) char smem_raw[];     // C::LDS
  const unsigned nx = (unsigned)((N + C::BN - 1) / C::BN), ny = (unsigned)((M + C::BM - 1) / C::BM);
  const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;
  const unsigned i = (block & 7) * (gridDim.x * gridDim.y >> 3) + (block >> 3);
  if (i / nx >= ny * splits) return;
  gemm_f32_tile<C, A_KC, B_KC>(A, B, M, N, K, epi, i % nx, i / nx % ny, i / nx / ny, splits, smem_raw);
}

// The epilogues get a wavefront's accumulators, its first row and the lane's first column.

// Logits: M = vocabulary, N = tokens.  Per token and 64 vocabulary rows (one wavefront) the pair
// (m, s) = (max_v z, sum_v exp(z - m)); parts[v / 64][t].  With `zt` the logits themselves are kept as well, for a batch
// whose gradient fits one panel: zt[v][t].
// Visits column j of a wavefront's patch: f(p, value, row), p = the address of the row in a matrix of pitch `ld` whose rows
// of this lane start at p0. `rows` of the patch exist (a wavefront's, so the usual whole patch takes no test per row), `left`
// of this lane's.
template <int TM, int TN, class F>
__device__ __forceinline__ void f32_rows(float* p0, int64_t ld, int64_t rows, int left, const f32x16 (&acc)[TM][TN], int j, F f) {
  if (rows >= TM * 32) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) f(p0 + (i * 32 + f32_acc_row(r)) * ld, acc[i][j][r], i * 32 + f32_acc_row(r));
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (i * 32 + f32_acc_row(r) < left) f(p0 + (i * 32 + f32_acc_row(r)) * ld, acc[i][j][r], i * 32 + f32_acc_row(r));
}

struct EpiLseF32 {
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
        f32_rows(zt + (m + 4 * half) * ldz + t, ldz, M - m, left, acc, j, [](float* p, float z, int) { *p = z; });
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
      f32_rows(zt + (m + 4 * half) * ldz + t, ldz, M - m, left, acc, j,
               [&](float* p, float z, int row) { *p = dz_f32(z, row, y, c, l); });
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
  float* C;
  int64_t ld;
  int accumulate;
  template <int TM, int TN>
  __device__ void store(f32x16 (&acc)[TM][TN], int64_t m, int64_t n, int half, int64_t M, int64_t N, unsigned split) const {
    float* out = C + (int64_t)split * M * N;
    const int left = (int)(M - m < TM * 32 ? M - m : TM * 32) - 4 * half;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t col = n + j * 32;
      if (col >= N) continue;
      float* p0 = out + (m + 4 * half) * ld + col;
      if (accumulate) f32_rows(p0, ld, M - m, left, acc, j, [](float* p, float x, int) { *p += x; });
      else f32_rows(p0, ld, M - m, left, acc, j, [](float* p, float x, int) { *p = x; });
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
  __shared__ __attribute__((aligned(256))) char lds[C::LDS];
  int64_t b = blockIdx.x;
  if (b == 0) return begin.run(0, 1, kPlan | kRest);
  b -= 1;
  const int64_t n_gather = (T + 3) / 4, rows = (V + C::BM - 1) / C::BM;
  if (b < n_gather)
    return gather_logit<float, double, VEC>(b * 4 + (threadIdx.x >> 6), H.p, W.p, tokens, T, d, V, zy, nullptr, init);
  b -= n_gather;
  gemm_f32_tile<C, true, true>(W, H, (int64_t)V, T, (int64_t)d, epi, b / rows, b % rows, 0, 1, lds);
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
__global__ void __launch_bounds__(256, 2) k_grads_f32(F32Contraction dh, F32Contraction dw) {
  __shared__ __attribute__((aligned(256))) char lds[larger(CH::LDS, CW::LDS)];
  const int64_t n_dh = (int64_t)dh.nx * dh.ny * dh.splits;
  int64_t i = blockIdx.x;
  if (i < n_dh) {
    gemm_f32_tile<CH, false, false>(dh.A, dh.B, dh.M, dh.N, dh.K, EpiStoreF32{dh.out, dh.N, 0}, i % dh.nx, i / dh.nx % dh.ny,
                                    (unsigned)(i / ((int64_t)dh.nx * dh.ny)), dh.splits, lds);
    return;
  }
  i -= n_dh;
  gemm_f32_tile<CW, true, false>(dw.A, dw.B, dw.M, dw.N, dw.K, EpiStoreF32{dw.out, dw.N, 0}, i % dw.nx, i / dw.nx % dw.ny,
                                 (unsigned)(i / ((int64_t)dw.nx * dw.ny)), dw.splits, lds);
}

}  // namespace oapl
