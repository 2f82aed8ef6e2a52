// bf16 MFMA contractions of the OAPL loss head, hand-written for gfx950.
//
// One main loop serves all dense steps of the path.  It computes a
// 256 x 384 tile of  C[m][n] = sum_k A[m][k] * B[n][k]  with both operands
// k-contiguous, fp32 accumulation in v_mfma_f32_16x16x32_bf16, operands
// streamed L2 -> LDS by direct-to-LDS buffer loads (no VGPR staging) into a
// two-stage, XOR-swizzled LDS ring that fills the CU's 160 KB, 8 wavefronts
// (two per SIMD, so one wavefront's waits are covered by the other's MFMAs),
// each a 64 x 192 patch (192 accumulator registers per lane).  The tile is as
// large as registers and LDS allow: operand delivery from L2 is what the loop
// waits for, and 256 x 384 needs 17 % fewer operand bytes per flop than 256 x 256.
// Calls too small to fill the chip with such tiles take smaller ones of the same
// loop, and calls of few tokens read the caller's matrices in place (Mainloop's ROWS
// and ATR); oapl_api.hip has the rules.
//
// Two things bound the loop: the power the part may draw, which sets its clock, and the loads.  Multiplications alone, on
// registers, run at 1.79 GHz in the 32 x 32 x 16 shape and at 2.09 GHz in the 16 x 16 x 32 one (8.39 / 7.18 ms for 12288 x
// 4096 x 151936), which moves fewer accumulator bytes per flop. And a wave that issues its ten loads of a block in one go waits
// until the memory pipeline has taken them; given out two at a time between the multiplications they cost it nothing. dH of
// 12288 tokens at d = 4096, same box: 10.82 ms 32 x 32 with the loads in one go, 10.23 ms 16 x 16, 9.75 ms with the loads
// spread (dW 11.14 / 10.50 / 10.23, logits 11.91 / 11.41 / 10.86 ms).
//
// Operand layout in HBM ("packed"): a matrix with R rows and K columns is
// stored as blocks of RB rows x 64 columns (RB = 256 for the m-side operand,
// 384 for the n-side operand), block (rt, kt) at byte offset
// (rt * n_kt + kt) * RB * 128, row-major inside the block (128 B per row), zero
// padded to whole blocks.  One k-step of one tile is then ONE contiguous 32 / 48 KiB
// read per operand (full 128-byte lines, sequential DRAM pages), instead of
// row fragments spread over a 2 MB .. 80 MB span, and ragged edges need no
// special case in the loads: padding is zeros.  The caller's row-major H and W
// are packed once per call by k_pack_rows / k_pack_transposed; the kernels
// that produce intermediate operands write them packed directly.
//
// In the accumulator of a 16x16 MFMA block a lane owns ONE column n (lane%16)
// and 4 consecutive rows m = 4*(lane/16) + r.  Every epilogue is built around that:
//   * forward (logits^T tile, M = vocabulary, N = tokens): the soft-max
//     reduction over the vocabulary is lane-local but for its last step, across
//     the four groups of 16 lanes (reduce4);
//   * outputs with m contiguous (G[t][v], dH[t][j], dW[v][j]) get 4
//     consecutive m per lane.
//
// The bodies of the tile kernels are compiled in the device pass only (__HIP_DEVICE_COMPILE__).
// They use instructions that gfx950 alone has (16-byte direct-to-LDS loads, the 16x16x32 bf16
// MFMA, v_permlane16/32_swap).  The host pass needs nothing but the signatures, for its launch stubs;
// it checks builtins against a generic target, keeps its complaints about device code to itself,
// and has been seen to drop a kernel's launch stub, or to refuse a launch as "no matching
// function", after an unrelated edit of the main loop.
#pragma once

#include "common.hip.h"
#include "rng.hip.h"
#include "small_kernels.hip.h"

namespace oapl {


// WM x WN wavefronts, each MB x NB blocks of 16 x 16.
// PACK_B_: rows per block of the n-side operands where they are packed (0: one tile), a multiple of the tile's.
// EARLY_: a block's loads go out in one go, for walks that wait for memory rather than for the multiplications.
// ONCE_: the m-side operand is read once in the whole launch and its lines pass the caches by (non-temporal loads); a walk may
// start at any k-block.
template <int WM_, int WN_, int MB_, int NB_, int NS_, int PACK_B_ = 0, bool EARLY_ = false, bool ONCE_ = false>
struct TileCfg {
  static constexpr int WM = WM_, WN = WN_, MB = MB_, NB = NB_;
  static constexpr bool EARLY = EARLY_;
  static constexpr bool ONCE = ONCE_;
  static constexpr int NW = WM * WN;            // waves per workgroup
  static constexpr int NT = NW * 64;            // threads per workgroup
  static constexpr int WROWS = MB * 16, WCOLS = NB * 16;   // one wavefront's patch
  static constexpr int BM = WM * WROWS;
  static constexpr int BN = WN * WCOLS;
  static constexpr int BK = kPackK;             // k-extent of one LDS stage
  static constexpr int NS = NS_;                // LDS stages in the ring
  static constexpr int KSTEPS = BK / 32;        // MFMA k-steps per stage
  static constexpr int ROW_BYTES = kPackRowBytes;
  static constexpr int STAGE_A = BM * ROW_BYTES;   // one stage of the m-side operand
  static constexpr int STAGE_B = BN * ROW_BYTES;   // ... of the n-side operand
  static constexpr int PACK_A = BM > kPackRowsA ? BM : kPackRowsA;     // (taller tiles read in place only)
  static constexpr int PACK_B = PACK_B_ ? PACK_B_ : BN;
  static constexpr int PITCH_A = PACK_A * ROW_BYTES, PITCH_B = PACK_B * ROW_BYTES;   // bytes of one packed block
  static_assert(PACK_A % BM == 0 && PACK_B % BN == 0, "a tile lies in one block");
  static constexpr int SLOT = STAGE_A + STAGE_B;   // one ring slot: the m-side block, then the n-side block
  static constexpr int MAIN_BYTES = NS * (STAGE_A + STAGE_B);
  static constexpr int NI_A = BM / (8 * NW);    // direct loads per wave and stage (8 rows each), m-side operand
  static constexpr int NI_B = (BN / 8 + NW - 1) / NW;   // ... n-side operand
  static constexpr int LAST_B = BN / 8 % NW;    // waves that take part in the last of them (0: all)
  // bf16 staging tiles used by epilogues, rows padded so that a write instruction's lanes spread over the banks.  A whole
  // tile does not fit the LDS, so epilogues stage it in chunks: [n][m] by wave column (BN / WN rows of n at a
  // time), [m][n] by pairs of MFMA block rows (32 rows of every wave row at a time).
  static constexpr int PITCH_NM = BM * 2 + 16;  // tile stored [n][m]
  static constexpr int PITCH_MN = BN * 2 + 32;  // tile stored [m][n]
  static constexpr int NM_CHUNKS = WN, NM_ROWS = BN / WN;
  static constexpr int MN_CHUNKS = MB / 2, MN_ROWS = WM * 32;
  static constexpr int STAGE_NM = NM_ROWS * PITCH_NM;
  static constexpr int STAGE_MN = MN_ROWS * PITCH_MN;
  static constexpr int RED_BYTES = WM * BN * 8;
  static constexpr int LDS_BYTES =
      MAIN_BYTES > STAGE_NM ? (MAIN_BYTES > STAGE_MN ? MAIN_BYTES : STAGE_MN)
                            : (STAGE_NM > STAGE_MN ? STAGE_NM : STAGE_MN);
  static_assert(NS == 2 || NS == 4, "ring size");
  static_assert(BM % (8 * NW) == 0 && (LAST_B == 0 || NS == 2), "a ring of four counts every wave's loads");
  static_assert(RED_BYTES + RED_BYTES / 2 <= LDS_BYTES, "reduction scratch must fit");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

// s_waitcnt immediate for "at most n vector-memory operations still outstanding" (gfx9 encoding:
// vmcnt in bits [3:0] and [15:14]; expcnt and lgkmcnt fields left at their maximum = no wait).
__host__ __device__ constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// Workgroup barrier for LDS hand-offs in epilogues: waits for this wave's LDS operations only.
// __syncthreads() also waits for the wave's outstanding global stores (vmcnt(0)), i.e. for a round
// trip to memory at every hand-off; the data of a store that has been issued is already out of the
// registers, so nothing here needs that wait.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0); vmcnt and expcnt fields at their maximum = no wait
  __builtin_amdgcn_s_barrier();
}

// Transposing LDS read (see ATR below).  Without the `__restrict__` the compiler takes the read for one that may depend
// on the direct-to-LDS loads in flight (they fill the other ring slot) and waits for all of them first, which undoes
// the prefetch: 13.1 ms for a 12288-row dH contraction; the main loop waits for the slot it reads by itself.
__device__ __forceinline__ bf16x4 lds_read_transposed(const __attribute__((address_space(3))) char* __restrict__ p) {
  typedef __attribute__((address_space(3))) bf16x4* lds_bf16x4_ptr;
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)p);
}

// ROWS: both operands are read from row-major matrices as the caller holds them (rows of `ld` elements, all of
// them contracted) instead of from packed copies.  A k-step of one tile is then one 128-byte piece of every row,
// `ld` apart; rows past the matrix and columns past `ld` read as zeros because their offsets are out of the buffer's
// range, so edges still need no padding.  Packing W costs a pass over it, more than the whole contraction of a few
// hundred tokens (0.48 ms at d = 4096, V = 151936).  The loop itself is 0 .. 4 % slower in place where rows are whole 128-byte
// lines (12288 tokens: sweep 11.37 / 11.28 ms in place / packed, dH, whose operand is transposed too, 10.48 / 10.06) and 12 %
// slower where row pieces straddle lines (d = 4104); rows_pay in oapl_api.hip draws the line.
//
// ATR: the m-side operand is read from a row-major matrix whose ROWS are contracted (element (m, k) at p[k * ld + m]):
// W as the dH contraction needs it, without a transposed copy.  A k-step of one tile is a 512-byte piece of 64 rows;
// it lies in LDS as [k][m], and the fragments come out of it by the transposing read (ds_read_b64_tr_b16: of the 16
// lanes of a group, lane 4e + a points at the four m of column group a in row k + e, and lane i receives column i of
// the four rows), two reads of 8 bytes in place of one of 16.
//
// The multiplications are inline assembly because only there can an accumulator be tied to its register: given the builtin, the
// register allocator gives results new registers and spills around them (3.5 times as slow).  The price is that the compiler
// does not know what an MFMA leaves behind: a vector instruction may not read or overwrite its result for 8 wait states, nor
// an MFMA read what a vector instruction wrote less than 2 before.  The first is in the code: every step ends with settle(),
// which all accumulators pass through.  The second holds because fragments come straight from LDS reads and zero_acc comes well
// before the first multiplication; tests/test_mfma_hazards.py reads the built library for both.
template <class C, bool ROWS = false, bool ATR = false>
struct Mainloop {
  // 16-byte chunk c of LDS row `row` lives at physical chunk c ^ ((row >> 1) & 7).  The operand
  // fetch of 16 consecutive rows at one logical chunk then touches 16 distinct 16-byte bank groups:
  // two consecutive rows fill one 256-byte bank line, and the XOR walks each half's 8 slots.
  static __device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

  __amdgpu_buffer_rsrc_t ra, rb;
  int voff;                           // per-lane byte offset of this lane's chunk inside the first 8 rows a wave loads
  int vlast;                          // ROWS: ... in the last k-block (out of range where the chunk lies past the row's end)
  int istep;                          // ROWS: bytes from one load of a wave to the next (8 * NW rows)
  int first;                          // ONCE: the k-block that a walk starts with, and wraps around to behind the last
  const char* at_base;                // ATR: the tile's first column in row 0 of the matrix
  int64_t at_rows;                    // ... rows (k) from there
  int at_ld2, at_m0, at_voff;         // ... bytes per row, first column, per-lane byte offset of a wave's first load of a k-block
  // LDS byte offsets of this lane's operand fragments at k-step 0 of ring slot 0.  K-step 1 sits at the
  // same offset with address bit 6 flipped (the swizzle is an XOR on the 16-byte chunk index and
  // the k-step is bit 2 of that index).
  int rdA0, rdB0;
  int wave, lane;

  __device__ __forceinline__ void setup() {
    const int tid = threadIdx.x;
    // the wave index feeds LDS base addresses that must live in scalar registers
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    lane = tid & 63;
    const int wm = wave / C::WN, wn = wave % C::WN;
    // One wave-wide load covers 8 block rows; lane l lands at LDS byte l*16 of that 1 KiB.  Load i of
    // a wave takes rows (i * NW + wave) * 8 ..: 8 * NW rows further per i, which leaves the swizzle
    // term unchanged (8 * NW is a multiple of 16), so one lane offset serves every i and both operands;
    // the i term goes into the scalar offset.
    static_assert((8 * C::NW) % 16 == 0, "swizzle must repeat from one load of a wave to the next");
    {
      const int row = wave * 8 + (lane >> 3);
      voff = row * C::ROW_BYTES + (((lane & 7) ^ swz(row)) << 4);
    }
    const int rowA = wm * C::WROWS + (lane & 15);
    const int rowB = wn * C::WCOLS + (lane & 15);
    static_assert(C::KSTEPS == 2, "k-step index = chunk bit 2");
    const int c0 = lane >> 4;
    rdA0 = rowA * C::ROW_BYTES + ((c0 ^ swz(rowA)) << 4);
    rdB0 = C::STAGE_A + rowB * C::ROW_BYTES + ((c0 ^ swz(rowB)) << 4);
  }

  // ATR only: the m-side operand of column tile mt in a row-major matrix of R rows of `ld` elements (after setup()).
  // Chunk c (16 bytes, BM / 8 per row) of LDS row k lives at chunk c ^ at_swz(k): the eight rows of 32 lanes' transposing
  // read, 32 bytes each, then lie on 64 different banks.
  static __device__ __forceinline__ int at_swz(int k) { return ((k & 3) | ((k & 8) >> 1)) << 1; }
  __device__ __forceinline__ void set_a_transposed(const bf16_t* p, int mt, int64_t R, int ld) {
    // one wave-wide load covers RPL rows of LPR lanes; load i of a wave is NW * RPL rows further on
    constexpr int LPR = C::BM / 8, RPL = 64 / LPR;
    static_assert(!ATR || (C::NW * RPL) % 16 == 0, "swizzle must repeat from one load of a wave to the next");
    static_assert(!ATR || C::NI_A * C::NW * RPL == C::BK, "the loads cover the block");
    at_base = (const char*)(p + mt * C::BM);
    at_rows = R;
    at_ld2 = ld * 2;
    at_m0 = mt * C::BM;
    const int row = wave * RPL + lane / LPR;
    at_voff = row * at_ld2 + (((lane % LPR) ^ at_swz(row)) << 4);
    const int e = (lane >> 2) & 3, a = lane & 3, g = lane >> 4, wm = wave / C::WN;
    const int k = 8 * g + e;
    const int chunk = wm * C::MB * 2 + (a >> 1);   // m / 8 of fragment 0
    rdA0 = k * (C::BM * 2) + ((chunk ^ at_swz(k)) << 4) + ((a & 1) << 3);
  }

  // The empty asm keeps the compiler from hoisting the per-k-step addresses out of the loop (back into a table).
  static __device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
  }

  // ROWS only: the per-lane offsets for rows of `ld` elements (after setup()).
  __device__ __forceinline__ void rows_init(int ld) {
    if (!ROWS) return;
    const int row = wave * 8 + (lane >> 3), c = (lane & 7) ^ swz(row);
    voff = row * ld * 2 + (c << 4);
    vlast = ((ld - 1) & ~(C::BK - 1)) + c * 8 < ld ? voff : (int)0x80000000u;
    istep = 8 * C::NW * ld * 2;
  }
  // m-side operand from row r0 of a matrix, rows from `end` on (at most BM further) as zeros: row-major or, with r0 at a
  // multiple of BM, packed as ROWS says.
  __device__ __forceinline__ void set_a(const bf16_t* p, int64_t r0, int64_t end, int ld, int n_kt) {
    const int64_t left = end - r0;
    const int bytes = (int)(left < C::BM ? left : C::BM) * ld * 2;
    if (ROWS) ra = __builtin_amdgcn_make_buffer_rsrc((void*)(p + r0 * ld), 0, bytes, 0x00020000);
    else set_a_packed(p, r0, n_kt, 0);
  }
  // n-side operand tile `rt` (BN rows) of a matrix of R rows.
  __device__ __forceinline__ void set_b(const bf16_t* p, int64_t rt, int64_t R, int ld, int n_kt) {
    const int64_t left = R - rt * C::BN;
    const int bytes = (int)(left < C::BN ? left : C::BN) * ld * 2;
    if (ROWS) rb = __builtin_amdgcn_make_buffer_rsrc((void*)(p + rt * C::BN * ld), 0, bytes, 0x00020000);
    else set_b_packed(p, rt * C::BN, n_kt, 0);
  }

  // Operand = rows row0 .. of a packed matrix with n_kt k-blocks per strip, from k-block k0 on.
  __device__ __forceinline__ void set_a_packed(const bf16_t* p, int64_t row0, int n_kt, int k0) {
    const int in_block = (int)(row0 % C::PACK_A) * C::ROW_BYTES;
    ra = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + (row0 / C::PACK_A * n_kt + k0) * C::PITCH_A + in_block), 0,
                                           (n_kt - k0) * C::PITCH_A - in_block, 0x00020000);
  }
  __device__ __forceinline__ void set_b_packed(const bf16_t* p, int64_t row0, int n_kt, int k0) {
    const int in_block = (int)(row0 % C::PACK_B) * C::ROW_BYTES;
    rb = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + (row0 / C::PACK_B * n_kt + k0) * C::PITCH_B + in_block), 0,
                                           (n_kt - k0) * C::PITCH_B - in_block, 0x00020000);
  }

  // Per-lane offset of the loads of k-block kt: past the buffer's range, so that nothing is read and zeros are
  // written, for a block past the last.
  __device__ __forceinline__ int load_voff(int kt, int nk) const {
    const int inside = ATR ? 0 : ROWS && block(kt, nk) + 1 == nk ? vlast : voff;
    const int v = kt < nk ? inside : (int)0x80000000u;
    return ROWS ? fresh(v) : v;
  }
  // The k-block that a walk takes at its step kt.
  __device__ __forceinline__ int block(int kt, int nk) const {
    if (!C::ONCE) return kt;
    return kt + first < nk ? kt + first : kt + first - nk;
  }
  // Starts direct-to-LDS load i (of NI_A + NI_B) of k-block kt into ring slot STAGE (a literal at the call sites,
  // so the LDS addresses fold to constants once inlined), v = load_voff(kt, nk).
  // ROWS: the row term goes into the per-lane offset, because only that one is sure to be compared with the buffer's
  // range: a scalar offset past the range (rows of a matrix shorter than the tile) must not decide what is read.
  __device__ __forceinline__ void issue_one(const int STAGE, lds_char_ptr smem, int v, int kt, int nk, const int i) {
    if (i < C::NI_A) {
      const lds_void_ptr dst = (lds_void_ptr)(smem + STAGE * C::SLOT + (i * C::NW + wave) * 1024);
      if (ATR) {
        // rows past the matrix lie past its end and read as zeros; columns past `ld` are the next row's: they feed
        // output rows that are not stored
        const int kc = kt < nk ? kt : nk - 1;
        const int64_t left = at_rows - (int64_t)kc * C::BK;
        const int bytes = (int)(left < C::BK ? left : C::BK) * at_ld2 - at_m0 * 2;
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((void*)(at_base + (int64_t)kc * C::BK * at_ld2), 0, bytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, (v < 0 ? v : at_voff) + i * (C::NW * 512 / C::BM) * at_ld2, 0, 0, 0);
      } else {
        constexpr int kNonTemporal = 2;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            ra, dst, 16, ROWS ? v + i * istep : v,
            ROWS ? block(kt, nk) * C::ROW_BYTES : kt * C::PITCH_A + i * C::NW * 1024, 0, C::ONCE ? kNonTemporal : 0);
      }
    } else if (i < C::NI_A + C::NI_B) {
      const int b = i - C::NI_A;
      if (C::LAST_B != 0 && b == C::NI_B - 1 && wave >= C::LAST_B) return;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rb, (lds_void_ptr)(smem + STAGE * C::SLOT + C::STAGE_A + (b * C::NW + wave) * 1024), 16,
          ATR ? (v < 0 ? v : voff) : ROWS ? v + b * istep : v,
          ROWS ? block(kt, nk) * C::ROW_BYTES : kt * C::PITCH_B + b * C::NW * 1024, 0, 0);
    }
  }
  // ... all loads of the block.
  __device__ __forceinline__ void issue(const int STAGE, lds_char_ptr smem, int kt, int nk) {
    const int v = load_voff(kt, nk);
#pragma unroll
    for (int i = 0; i < C::NI_A + C::NI_B; ++i) issue_one(STAGE, smem, v, kt, nk, i);
  }

  // Two loads are given out per group of multiplications, from the second group on, where the patch is large enough.
  static constexpr int kLoads = C::NI_A + C::NI_B;
  static constexpr int kGroups = C::KSTEPS * ((C::NB + 1) / 2);
  static constexpr bool kSpread = C::NS == 2 && C::MB * C::NB >= 32 && !C::EARLY && 2 * (kGroups - 1) >= kLoads;

  static __device__ __forceinline__ void mfma(f32x4& c, const bf16x8 a, const bf16x8 b) {
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  }
  // The last multiplications' results are there (8 wait states) before any other instruction sees the accumulators: the wait
  // states are one statement that every accumulator goes into and comes out of, so that the order is in the data. Several
  // statements chained through an accumulator cost a wait state per link, which the compiler puts between them.
  static __device__ __forceinline__ void settle(f32x4 (&acc)[C::MB][C::NB]) {
    __builtin_amdgcn_sched_barrier(0);
#define OAPL_COLUMN(j) "+v"(acc[0][j]), "+v"(acc[1][j]), "+v"(acc[2][j]), "+v"(acc[3][j])
#define OAPL_ROW_4 "+v"(acc[4][0]), "+v"(acc[4][1]), "+v"(acc[4][2]), "+v"(acc[4][3]), "+v"(acc[4][4]), "+v"(acc[4][5]), \
                   "+v"(acc[4][6]), "+v"(acc[4][7])
#define OAPL_COLUMNS_4 OAPL_COLUMN(0), OAPL_COLUMN(1), OAPL_COLUMN(2), OAPL_COLUMN(3)
#define OAPL_COLUMNS_8 OAPL_COLUMNS_4, OAPL_COLUMN(4), OAPL_COLUMN(5), OAPL_COLUMN(6), OAPL_COLUMN(7)
#define OAPL_COLUMNS_9 OAPL_COLUMNS_8, OAPL_COLUMN(8)
#define OAPL_COLUMNS_10 OAPL_COLUMNS_9, OAPL_COLUMN(9)
#define OAPL_COLUMNS_11 OAPL_COLUMNS_10, OAPL_COLUMN(10)
#define OAPL_COLUMNS_12 OAPL_COLUMNS_11, OAPL_COLUMN(11)
    if constexpr (C::MB == 2 && C::NB == 4)
      asm volatile("s_nop 7" : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]),
                               "+v"(acc[1][0]), "+v"(acc[1][1]), "+v"(acc[1][2]), "+v"(acc[1][3]));
    else if constexpr (C::NB == 4) asm volatile("s_nop 7" : OAPL_COLUMNS_4);
    else if constexpr (C::MB == 5) asm volatile("s_nop 7" : OAPL_COLUMNS_8, OAPL_ROW_4);
    else if constexpr (C::NB == 8) asm volatile("s_nop 7" : OAPL_COLUMNS_8);
    else if constexpr (C::NB == 9) asm volatile("s_nop 7" : OAPL_COLUMNS_9);
    else if constexpr (C::NB == 10) asm volatile("s_nop 7" : OAPL_COLUMNS_10);
    else if constexpr (C::NB == 11) asm volatile("s_nop 7" : OAPL_COLUMNS_11);
    else asm volatile("s_nop 7" : OAPL_COLUMNS_12);
#undef OAPL_COLUMN
#undef OAPL_ROW_4
#undef OAPL_COLUMNS_4
#undef OAPL_COLUMNS_8
#undef OAPL_COLUMNS_9
#undef OAPL_COLUMNS_10
#undef OAPL_COLUMNS_11
#undef OAPL_COLUMNS_12
    static_assert(C::MB == 4 || (C::MB == 2 && C::NB == 4) || (C::MB == 5 && C::NB == 8), "operands of the statement above");
  }

  // Patches of up to eight blocks (64 and 128 tokens): all fragments of the block are requested before its first
  // multiplication, for eight multiplications of a k-step do not cover the next one's reads (sampling 128 tokens at d = 1024, V
  // = 8081 16.7 / 15.8 us, scoring 50 at d = 2048, V = 922 21.3 / 20.8; at V = 151936 the same; 128 x 128 tiles, sixteen
  // blocks, +1 .. +2 us).
  static constexpr bool kWhole = !ATR && C::MB * C::NB <= 8;
  static_assert(!kWhole || !kSpread, "compute_whole gives out no loads");
  __device__ __forceinline__ void compute_whole(const int STAGE, lds_char_ptr smem, f32x4 (&acc)[C::MB][C::NB]) {
    bf16x8 a[C::KSTEPS][C::MB], b[C::KSTEPS][C::NB];
#pragma unroll
    for (int ks = 0; ks < C::KSTEPS; ++ks) {
      const lds_char_ptr pa = smem + STAGE * C::SLOT + (fresh(rdA0) ^ (ks << 6));
      const lds_char_ptr pb = smem + STAGE * C::SLOT + (fresh(rdB0) ^ (ks << 6));
#pragma unroll
      for (int i = 0; i < C::MB; ++i) a[ks][i] = *(const __attribute__((address_space(3))) bf16x8*)(pa + i * 16 * C::ROW_BYTES);
#pragma unroll
      for (int j = 0; j < C::NB; ++j) b[ks][j] = *(const __attribute__((address_space(3))) bf16x8*)(pb + j * 16 * C::ROW_BYTES);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < C::KSTEPS; ++ks)
#pragma unroll
      for (int i = 0; i < C::MB; ++i)
#pragma unroll
        for (int j = 0; j < C::NB; ++j) mfma(acc[i][j], a[ks][i], b[ks][j]);
    settle(acc);
  }

  // Multiplies the block in ring slot STAGE; with LOAD also starts the loads of block kt_load into slot LSTAGE on the way.
  // A k-step's m-side fragments stay in registers, n-side fragments come two at a time, requested one group of
  // multiplications ahead (the scheduler moves a group's reads up between the previous group's multiplications, no
  // further: that is what the barriers are for).
  template <bool LOAD>
  __device__ __forceinline__ void compute(const int STAGE, lds_char_ptr smem, f32x4 (&acc)[C::MB][C::NB], const int LSTAGE = 0,
                                          int kt_load = 0, int nk = 0) {
    if constexpr (kWhole) return compute_whole(STAGE, smem, acc);
    const int v = LOAD ? load_voff(kt_load, nk) : 0;
#pragma unroll
    for (int ks = 0; ks < C::KSTEPS; ++ks) {
      bf16x8 a[C::MB];
      const int ra_ks = ATR ? fresh(rdA0) : fresh(rdA0) ^ (ks << 6), rb_ks = fresh(rdB0) ^ (ks << 6);
#pragma unroll
      for (int i = 0; i < C::MB; ++i) {
        if (ATR) {
          static_assert(!ATR || C::MB == 4, "fragment i flips chunk bits 1..2");
          const lds_char_ptr q = smem + (ra_ks ^ (i << 5)) + STAGE * C::SLOT + ks * 32 * (C::BM * 2);
          const bf16x4 lo = lds_read_transposed(q), hi = lds_read_transposed(q + 4 * (C::BM * 2));
          a[i] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
          a[i] = *(const __attribute__((address_space(3))) bf16x8*)(smem + STAGE * C::SLOT + ra_ks + i * 16 * C::ROW_BYTES);
        }
      }
#pragma unroll
      for (int j0 = 0; j0 < C::NB; j0 += 2) {
        const int w = C::NB - j0 < 2 ? 1 : 2;
        bf16x8 b[2];
#pragma unroll
        for (int j = 0; j < w; ++j)
          b[j] = *(const __attribute__((address_space(3))) bf16x8*)(smem + STAGE * C::SLOT + rb_ks +
                                                                    (j0 + j) * 16 * C::ROW_BYTES);
        const int group = ks * ((C::NB + 1) / 2) + j0 / 2;
        if (LOAD && group > 0) {
          issue_one(LSTAGE, smem, v, kt_load, nk, 2 * (group - 1));
          issue_one(LSTAGE, smem, v, kt_load, nk, 2 * (group - 1) + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < C::MB; ++i)
#pragma unroll
          for (int j = 0; j < w; ++j) mfma(acc[i][j0 + j], a[i], b[j]);
      }
    }
    settle(acc);
  }

  // Ring of four (128 x 128 tiles that have a CU to themselves, the reference pass): such a workgroup waits for the
  // latency of its loads as much as for operand bytes, so three blocks are in flight instead of one.  Loss calls of 100
  // tokens, ring of two / four: d = 4096, V = 32000 361 / 349 us, V = 8192 152 / 149, V = 151936 1168 / 1169; 1000 tokens at d
  // = 256, V = 1544 and 300 at d = 1024, V = 8192 the same.
  //
  // One k-block of the pipeline in ring slot S (a literal at the call sites): wait until the block's
  // loads have landed, barrier (which also tells that every wave is done with the other slot),
  // refill the other slot with the next block, multiply.  Branches are wave-uniform and touch no
  // accumulator.
  __device__ __forceinline__ void step(const int S, lds_char_ptr smem, int kt, int nk, f32x4 (&acc)[C::MB][C::NB]) {
    if (C::NS == 2) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __syncthreads();
      if (kSpread) {
        // past the last block the loads find nothing (load_voff); finish() waits for them all the same
        compute<true>(S, smem, acc, S ^ 1, kt + 1, nk);
        return;
      }
      if (kt + 1 < nk) issue(S ^ 1, smem, kt + 1, nk);
    } else {
      // Blocks kt + 1 and kt + 2 stay in flight (loads issued later than block kt's by someone else only make the wait
      // stricter).  __syncthreads() would wait for them, so the barrier is a bare one; this wave's LDS reads of the slot
      // that is refilled next are done (lgkmcnt), and the compiler keeps memory accesses on their side of it.
      constexpr int L = C::NI_A + C::NI_B;
      if (kt + 2 < nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * L) & ~0x0F00);
      else if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(vmcnt_imm(L) & ~0x0F00);
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & ~0x0F00);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 3 < nk) issue((S + 3) & 3, smem, kt + 3, nk);
    }
    compute<false>(S, smem, acc);
  }

  // Starts a tile: k-block 0 into slot 0 (ring of four: blocks 0 .. 2).  Every wave must be past its last LDS read of the
  // previous tile (finish() ends with a barrier).
  __device__ __forceinline__ void start(lds_char_ptr smem, int nk) {
    issue(0, smem, 0, nk);
    if (C::NS == 4 && nk > 1) issue(1, smem, 1, nk);
    if (C::NS == 4 && nk > 2) issue(2, smem, 2, nk);
  }
  // ... and block 1 into slot 1 of a ring of two, for steps<true>.
  __device__ __forceinline__ void start_preload(lds_char_ptr smem, int nk) {
    start(smem, nk);
    if (C::NS == 2 && nk > 1) issue(1, smem, 1, nk);
  }

  // k-blocks [k0, k1) of a tile with nk k-blocks in all (k0 a multiple of NS, after start() or an earlier steps()).
  // PRELOADED (ring of two, k0 = 0): k-block 1 was issued beforehand as well (start_preload()), by a caller whose work between
  // two tiles leaves the LDS alone. The first block then issues nothing. It waits for both blocks: waiting for the first alone
  // (vmcnt = the second block's loads, and a bare s_barrier, since __syncthreads() waits for every outstanding load itself)
  // measured no different.
  template <bool PRELOADED = false>
  __device__ __forceinline__ void steps(lds_char_ptr smem, int k0, int k1, int nk, f32x4 (&acc)[C::MB][C::NB]) {
    int kt = k0;
    if (C::NS == 4) {
      for (; kt + 4 <= k1; kt += 4) {
        step(0, smem, kt, nk, acc);
        step(1, smem, kt + 1, nk, acc);
        step(2, smem, kt + 2, nk, acc);
        step(3, smem, kt + 3, nk, acc);
      }
      if (kt < k1) step(0, smem, kt, nk, acc);
      if (kt + 1 < k1) step(1, smem, kt + 1, nk, acc);
      if (kt + 2 < k1) step(2, smem, kt + 2, nk, acc);
      return;
    }
    if (PRELOADED) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __syncthreads();
      compute<false>(0, smem, acc);
      kt = 1;
      if (kt < k1) {
        step(1, smem, 1, nk, acc);
        kt = 2;
      }
    }
    for (; kt + 2 <= k1; kt += 2) {
      step(0, smem, kt, nk, acc);
      step(1, smem, kt + 1, nk, acc);
    }
    if (kt < k1) step(0, smem, kt, nk, acc);
  }

  // acc += A_tile * B_tile^T over k-blocks [0, nk) after start().  Ends with a barrier: on return
  // every wave is done reading LDS and every load into it has landed, so the caller may reuse it (or start() the next
  // tile) at once.
  template <bool PRELOADED = false>
  __device__ __forceinline__ void finish(lds_char_ptr smem, int nk, f32x4 (&acc)[C::MB][C::NB]) {
    steps<PRELOADED>(smem, 0, nk, nk, acc);
    drain();
  }
  // ... the end of it, for a caller of steps().
  static __device__ __forceinline__ void drain() {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
  }
};

template <class C>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[C::MB][C::NB]) {
#pragma unroll
  for (int i = 0; i < C::MB; ++i)
#pragma unroll
    for (int j = 0; j < C::NB; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      asm volatile("" : "+v"(acc[i][j]));     // here, and not in front of the multiplication that adds to it
    }
}

// Where a lane stands in its wavefront's patch: accumulator register r of block (i, j) is row 16 i + 4 g + r, column 16 j + c.
template <class C>
struct Lane {
  int wm, wn, g, c;
  __device__ __forceinline__ Lane() {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wm = wave / C::WN;
    wn = wave % C::WN;
    g = lane >> 4;
    c = lane & 15;
  }
  __device__ __forceinline__ int row0() const { return wm * C::WROWS + 4 * g; }    // in the tile: row of (i = 0, r = 0)
  __device__ __forceinline__ int col0() const { return wn * C::WCOLS + c; }        // ... column of j = 0
};

// Rows past `rows` of a tile whose row of (i = 0, r = 0) is row0 take the value v.
template <class C>
__device__ __forceinline__ void fill_rows_past(f32x4 (&acc)[C::MB][C::NB], int row0, int rows, float v) {
#pragma unroll
  for (int i = 0; i < C::MB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (row0 + 16 * i + r >= rows) {
#pragma unroll
        for (int j = 0; j < C::NB; ++j) acc[i][j][r] = v;
      }
}

// Reduction over the four groups of 16 lanes, four columns at a time: group g ends with column g's result.  A swap hands
// one half of the lanes the other column's partial results, so three swaps and three operations serve four columns.
template <class Op>
__device__ __forceinline__ float reduce4(const float (&x)[4], Op op) {
  auto swap32 = [&](float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));    // lower half: a over both halves; upper half: b
  };
  const float p = swap32(x[0], x[2]), q = swap32(x[1], x[3]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// ... of (score, index) pairs, the better of which stays.
__device__ __forceinline__ void reduce4_better(const float (&x)[4], const int (&i)[4], float& score, int& index) {
  auto pick = [](float sa, int ia, float sb, int ib, float& so, int& io) {
    const bool first = better(sa, ia, sb, ib);
    so = first ? sa : sb;
    io = first ? ia : ib;
  };
  float p[2];
  int pi[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[k]), __float_as_uint(x[k + 2]), false, false);
    const auto ri = __builtin_amdgcn_permlane32_swap((uint32_t)i[k], (uint32_t)i[k + 2], false, false);
    pick(__uint_as_float(r[0]), (int)ri[0], __uint_as_float(r[1]), (int)ri[1], p[k], pi[k]);
  }
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p[0]), __float_as_uint(p[1]), false, false);
  const auto ri = __builtin_amdgcn_permlane16_swap((uint32_t)pi[0], (uint32_t)pi[1], false, false);
  pick(__uint_as_float(r[0]), (int)ri[0], __uint_as_float(r[1]), (int)ri[1], score, index);
}
// ... and back: x[k] = what group k holds in y.
__device__ __forceinline__ void spread4(float y, float (&x)[4]) {
  const uint32_t u = __float_as_uint(y);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);      // groups 0, 0, 2, 2 and 1, 1, 3, 3
  const auto e = __builtin_amdgcn_permlane32_swap(r[0], r[0], false, false);
  const auto o = __builtin_amdgcn_permlane32_swap(r[1], r[1], false, false);
  x[0] = __uint_as_float(e[0]);
  x[1] = __uint_as_float(o[0]);
  x[2] = __uint_as_float(e[1]);
  x[3] = __uint_as_float(o[1]);
}

// ---------------------------------------------------------------------------
// bf16 staging of an accumulator tile through LDS for 16-byte coalesced stores.
// A whole tile is larger than the LDS, so it goes in chunks (see TileCfg); every
// stage_* call must be followed by a barrier, then the matching store_*, then a
// barrier before the next chunk is staged.
// ---------------------------------------------------------------------------

// LDS chunk [n][m] (n = the BN / WN columns of wave column `chunk`): each lane of those waves
// writes 4 consecutive m (8 bytes) per step.
template <class C>
__device__ __forceinline__ void stage_nm(lds_char_ptr smem, const f32x4 (&acc)[C::MB][C::NB], int chunk) {
  const Lane<C> at;
  if (at.wn != chunk) return;
#pragma unroll
  for (int j = 0; j < C::NB; ++j)
#pragma unroll
    for (int i = 0; i < C::MB; ++i) {
      const f32x4 x = acc[i][j];
      *(__attribute__((address_space(3))) bf16x4*)(smem + (j * 16 + at.c) * C::PITCH_NM + (at.row0() + 16 * i) * 2) =
          bf16x4{(bf16_t)x[0], (bf16_t)x[1], (bf16_t)x[2], (bf16_t)x[3]};
    }
}

// Staged chunk -> out[n][m] (row pitch ldo elements, pointer at the tile origin):
// rows n < n_rows, columns m < m_cols (m_cols a multiple of 8).
template <class C>
__device__ __forceinline__ void store_nm(lds_char_ptr smem, bf16_t* out, int64_t ldo, int64_t n_rows, int64_t m_cols,
                                         int chunk) {
  constexpr int CH = C::BM / 8;
  for (int idx = threadIdx.x; idx < C::NM_ROWS * CH; idx += C::NT) {
    const int n_l = idx / CH, ch = idx % CH;
    const int n = chunk * C::NM_ROWS + n_l;
    if (n < n_rows && ch * 8 < m_cols) {
      const u32x4 v = *(const __attribute__((address_space(3))) u32x4*)(smem + n_l * C::PITCH_NM + ch * 16);
      *(u32x4*)(out + (int64_t)n * ldo + ch * 8) = v;
    }
  }
}

// ---------------------------------------------------------------------------
// Two packed copies of a tile rounded to bf16 pairs: pk[i][j][p] holds rows 2p and 2p + 1 (low / high half) of the lane's
// four in block (i, j).  Half the registers of the fp32 tile, so nothing spills around the stores.
// ---------------------------------------------------------------------------

// Copy with rows = n, k = m, straight from registers.  A lane owns 4 consecutive m (8 bytes) of its row n per block; the
// groups trade registers between two block rows (v_permlane16_swap), after which a lane holds a 16-byte piece of its row and
// the four lanes of a row 64 bytes, as much as a write request carries.  Stored in 16-byte pieces all over the lines, the
// sweep's write requests averaged 43 bytes and the kernel took 2.7 % longer.
// `dst` is the destination matrix, n_kt its strip pitch in k-blocks, n0 the tile's first row, kb0 the first
// k-block (m0 / 64).
template <class C>
__device__ __forceinline__ void store_nm_packed_direct(const uint32_t (&pk)[C::MB][C::NB][2], bf16_t* dst, int n_kt, int64_t n0,
                                                       int kb0) {
  static_assert(C::WROWS == kPackK, "a wave row spans exactly one packed k-block");
  const Lane<C> at;
  // the piece of block rows 2q, 2q + 1 sits at byte 64 q + 32 (g & 1) + 16 (g >> 1) of its row's 128-byte line
  char* base = (char*)dst + (n0 / C::PACK_B * n_kt + kb0 + at.wm) * C::PITCH_B + (n0 % C::PACK_B + at.col0()) * kPackRowBytes +
               32 * (at.g & 1) + 16 * (at.g >> 1);
#pragma unroll
  for (int j = 0; j < C::NB; ++j)
#pragma unroll
    for (int q = 0; q < C::MB / 2; ++q) {
      const auto lo = __builtin_amdgcn_permlane16_swap(pk[2 * q][j][0], pk[2 * q + 1][j][0], false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap(pk[2 * q][j][1], pk[2 * q + 1][j][1], false, false);
      *(u32x4*)(base + j * 16 * kPackRowBytes + 64 * q) = u32x4{lo[0], hi[0], lo[1], hi[1]};
    }
}

// LDS chunk [m][n] from the packed pairs: chunk q holds MFMA block rows 2q and 2q + 1 of every wave row (32 rows
// each, WM * 32 rows in all), so all waves stage at once.  Neighbouring lanes (columns n, n + 1) swap
// halves so that each lane writes 4 bytes: the even lane row m (its own low half, the neighbour's
// low half), the odd lane row m + 1 (the neighbour's high half, its own high half).
template <class C>
__device__ __forceinline__ void stage_mn_pk(lds_char_ptr smem, const uint32_t (&pk)[C::MB][C::NB][2], const int q) {
  const Lane<C> at;
  const int odd = at.c & 1;
  // v_perm_b32 picks bytes from {neighbour (4..7), own (0..3)}
  const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
  const lds_char_ptr base = smem + (at.wm * 32 + 4 * at.g + odd) * C::PITCH_MN + (at.col0() - odd) * 2;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < C::NB; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const uint32_t own = pk[2 * q + i][j][p];
        const uint32_t nbr = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1 /* quad_perm 1,0,3,2 */, 0xF, 0xF, true);
        *(__attribute__((address_space(3))) uint32_t*)(base + (16 * i + 2 * p) * C::PITCH_MN + j * 32) =
            __builtin_amdgcn_perm(nbr, own, sel);
      }
}

// Chunk q staged by stage_mn_pk -> packed n-side matrix whose rows are the m index (global row
// m0 + ..., blocks of kPackRowsB rows whatever the tile) and whose k index is n; n_kt is the destination's strip pitch in
// k-blocks, piece0 the first 16-byte piece of a row (n0 / 8: tiles of 288 and 352 columns end in the middle of a k-block).
template <class C>
__device__ __forceinline__ void store_mn_pk_packed(lds_char_ptr smem, bf16_t* base, int n_kt, int m0, int piece0, int q) {
  constexpr int CH = C::BN / 8;
  for (int idx = threadIdx.x; idx < C::MN_ROWS * CH; idx += C::NT) {
    const int m_l = idx / CH, ch = idx % CH;
    const int m = m0 + (m_l >> 5) * C::WROWS + q * 32 + (m_l & 31);
    const int blk = m / kPackRowsB, r = m - blk * kPackRowsB, piece = piece0 + ch;
    const u32x4 v = *(const __attribute__((address_space(3))) u32x4*)(smem + m_l * C::PITCH_MN + ch * 16);
    char* dst = (char*)base + ((int64_t)blk * n_kt + (piece >> 3)) * kPackBlockBytesB;
    *(u32x4*)(dst + r * kPackRowBytes + (piece & 7) * 16) = v;
  }
}

// Both packed copies of a tile: rows = vocabulary (m) with k = tokens (n), through LDS, two MFMA block rows of every wave at a
// time, then rows = tokens with k = vocabulary, whose stores drain after the workgroup has gone.
template <class C>
__device__ __forceinline__ void store_both_copies(lds_char_ptr smem, const uint32_t (&pk)[C::MB][C::NB][2], bf16_t* Gp,
                                                  int g_n_kt, bf16_t* GTp, int gt_n_kt, int m0, int64_t n0) {
  static_assert(C::STAGE_MN <= C::LDS_BYTES, "staging chunk must fit");
#pragma unroll
  for (int q = 0; q < C::MN_CHUNKS; ++q) {
    if (q > 0) lds_barrier();
    stage_mn_pk<C>(smem, pk, q);
    lds_barrier();
    store_mn_pk_packed<C>(smem, GTp, gt_n_kt, m0, (int)(n0 / 8), q);
  }
  store_nm_packed_direct<C>(pk, Gp, g_n_kt, n0, m0 / kPackK);
}

__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  const bf16x2 v = {(bf16_t)lo, (bf16_t)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// Tile coordinates for a logical workgroup id: tiles are walked in strips of
// SN tiles along n, m fastest within a strip row, so that the ~32 workgroups
// resident on one XCD form a (32 / SN) x SN patch and share operand panels.
// The kernels use SN = 4: an 8 x 4 patch of 256 x 384 tiles needs 8 x 32 KB +
// 4 x 48 KB of operands per k-step, the least for 32 tiles (sweep / dH / dW of 12288 tokens at d = 4096, V = 151936: 11.28 /
// 10.06 / 10.45 ms; SN = 8 11.31 / 10.22 / 10.57; SN = 2 11.60 / 10.10 / 10.53).
__device__ __forceinline__ void strip_tile(const int SN, int L, int MT, int NTl, int& mt, int& nt) {
  const int per_strip = SN * MT;
  const int strip = L / per_strip;
  const int rem = L - strip * per_strip;
  const int width = (NTl - strip * SN) < SN ? (NTl - strip * SN) : SN;
  mt = rem / width;
  nt = strip * SN + rem % width;
}
template <int SN>
__device__ __forceinline__ void strip_tile(int L, int MT, int NTl, int& mt, int& nt) {
  strip_tile(SN, L, MT, NTl, mt, nt);
}

// The vocabulary rows that a workgroup of the streaming kernels walks, tiles of `h` rows from r0 to r1.  Split `split` of
// n_splits: whole tiles, or (balanced, operands in place) the same number of rows to within 16 for everyone, in tiles of equal
// height.  A launch that waits for W to arrive takes as long as the workgroup with the most rows: whole tiles of 256 at V =
// 151936 are two for some CUs and three for others.  The rows that a lower tile leaves out are not read.
struct RowWalk {
  int r0, r1, h;
};
template <class C>
__host__ __device__ __forceinline__ RowWalk row_walk(int V, int split, int n_splits, int balanced) {
  const int unit = balanced ? 16 : C::BM, units = (V + unit - 1) / unit;
  const int r0 = (int)((int64_t)split * units / n_splits) * unit, end = (int)((int64_t)(split + 1) * units / n_splits) * unit;
  const int r1 = end < V ? end : V;
  if (!balanced) return RowWalk{r0, r1, C::BM};
  const int tiles = (r1 - r0 + C::BM - 1) / C::BM;
  return RowWalk{r0, r1, tiles > 0 ? ((r1 - r0 + tiles - 1) / tiles + 15) / 16 * 16 : C::BM};
}

// Where rows are a multiple of 4 KiB apart, what workgroups in step with each other request (a 128-byte piece of every row, all at
// the same k) lies on few of the memory's channels, so each starts its walk over k at another block: scoring 16 tokens at d = 2048,
// V = 151936 137 / 103 us, at d = 6144, V = 60000 169 / 129, 8192 190 / 163, at d = 4096, V = 151936 210 / 203. Other pitches
// gain nothing (d = 1024 .. 7168: -2 .. +2 %) and keep the plain order.
__device__ __forceinline__ int first_block(int split, int d, int n_kt) { return d % 2048 == 0 ? split % n_kt : 0; }

// ---------------------------------------------------------------------------
// Forward: logits^T tiles with a streaming (online) log-sum-exp over the
// vocabulary.  The T x V logits never leave registers.
//   A = packed W [V, d]  (M = vocabulary),  B = packed H [T, d]  (N = tokens),  K = d.
// One workgroup owns one token tile and walks a contiguous range ("split") of
// vocabulary tiles, carrying per token the running pair
//     m2 = max_v z * log2(e),   s = sum_v 2^(z * log2(e) - m2)
// and merging a new tile by the usual rescaling rule.  The first k-block of
// the next vocabulary tile is requested before the current tile's epilogue.
// It writes one (m2, s) pair per token and split; a later kernel merges the
// splits.  With ENT it also carries u = sum_v 2^(z * log2(e) - m2) * z, from which
// the policy entropy follows as  lse - u / s  (one more FMA per logit).
// ---------------------------------------------------------------------------
template <class C, bool ENT, bool ROWS>
__global__ void __launch_bounds__(C::NT)
k_fwd_lse(const bf16_t* __restrict__ W, const bf16_t* __restrict__ H, int V, int64_t T, int d, int n_kt,
          int n_splits, int balanced, int patch_tiles, float2* __restrict__ partials, float* __restrict__ upart,
          int* __restrict__ clear /* a status header to clear, or nullptr */, Gate gate) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;
  if (gate_closed(gate)) return;
  if (clear != nullptr && blockIdx.x == 0 && threadIdx.x < kStatusWords) clear[threadIdx.x] = 0;

  const int n_tiles = (int)((T + C::BN - 1) / C::BN);
  const int total = n_tiles * n_splits;
  const int L = xcd_logical_id(blockIdx.x, total);
  if (L >= total) return;
  // Consecutive logical ids walk `patch_tiles` token tiles first, then the vocabulary splits: the ~32
  // workgroups resident on one XCD are then patch_tiles token tiles x 32 / patch_tiles splits, which
  // walk their splits in step and share each W block patch_tiles ways (each H block is shared by the
  // splits of its token tile).
  int split, nt;
  strip_tile(patch_tiles, L, n_splits, n_tiles, split, nt);
  const RowWalk walk = row_walk<C>(V, split, n_splits, balanced);
  const int64_t n0 = (int64_t)nt * C::BN;

  Mainloop<C, ROWS> ml;
  ml.setup();
  ml.rows_init(d);
  ml.first = first_block(split, d, n_kt);
  ml.set_b(H, nt, T, d, n_kt);

  const Lane<C> at;
  // the running values of column 16 (4 q + g) + c are lane group g's: a quarter of the columns per lane
  constexpr int Q = (C::NB + 3) / 4;
  float m2[Q], s[Q], u[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) { m2[q] = kNegHuge; s[q] = 0.f; u[q] = 0.f; }

  f32x4 acc[C::MB][C::NB];
  auto set_tile = [&](int m0) { ml.set_a(W, m0, m0 + walk.h < walk.r1 ? m0 + walk.h : walk.r1, d, n_kt); };
  if (walk.r0 < walk.r1) {
    set_tile(walk.r0);
    ml.start_preload(smem, n_kt);
  }
  for (int m0 = walk.r0; m0 < walk.r1; m0 += walk.h) {
    const int end = m0 + walk.h < walk.r1 ? m0 + walk.h : walk.r1;
    zero_acc<C>(acc);
    ml.template finish<true>(smem, n_kt, acc);
    if (end < walk.r1) {  // the epilogue below works in registers only: overlap it with the next tile's first loads
      set_tile(end);
      ml.start_preload(smem, n_kt);
    }

    // a lower tile, the ragged last one among them: rows from its end on do not exist (their logits are 0, not -inf)
    if (m0 + C::BM > end) fill_rows_past<C>(acc, m0 + at.row0(), end, -__builtin_inff());
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        x[k] = -__builtin_inff();
        if (4 * q + k < C::NB) {
#pragma unroll
          for (int i = 0; i < C::MB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) x[k] = fmaxf(x[k], acc[i][4 * q + k][r]);
        }
      }
      const float mnew = fmaxf(m2[q], reduce4(x, [](float a, float b) { return fmaxf(a, b); }) * kLog2e);
      float ref[4], us[4];
      spread4(mnew, ref);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        x[k] = us[k] = 0.f;
        if (4 * q + k < C::NB) {
#pragma unroll
          for (int i = 0; i < C::MB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float z = acc[i][4 * q + k][r], e = __builtin_amdgcn_exp2f(__builtin_fmaf(z, kLog2e, -ref[k]));
              x[k] += e;
              // masked rows hold -inf with e = 0: keep their product out (0 * inf)
              if (ENT) us[k] = __builtin_fmaf(e, e > 0.f ? z : 0.f, us[k]);
            }
        }
      }
      const auto add = [](float a, float b) { return a + b; };
      const float scale = __builtin_amdgcn_exp2f(m2[q] - mnew);
      s[q] = s[q] * scale + reduce4(x, add);
      if (ENT) u[q] = u[q] * scale + reduce4(us, add);
      m2[q] = mnew;
    }
  }

  // merge the WM waves stacked along the vocabulary, through LDS.
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  __attribute__((address_space(3))) f32x2* red = (__attribute__((address_space(3))) f32x2*)smem;
  __attribute__((address_space(3))) float* red_u = (__attribute__((address_space(3))) float*)(smem + C::RED_BYTES);
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (4 * q + at.g < C::NB) {
      const int n_l = at.wm * C::BN + at.col0() + (4 * q + at.g) * 16;
      red[n_l] = f32x2{m2[q], s[q]};
      if (ENT) red_u[n_l] = u[q];
    }
  __syncthreads();
  for (int n_l = threadIdx.x; n_l < C::BN; n_l += C::NT) {
    if (n0 + n_l < T) {
      f32x2 a = red[n_l];
      float ua = ENT ? red_u[n_l] : 0.f;
#pragma unroll
      for (int w = 1; w < C::WM; ++w) {
        const f32x2 b = red[w * C::BN + n_l];
        const float M = fmaxf(a.x, b.x);
        const float fa = __builtin_amdgcn_exp2f(a.x - M), fb = __builtin_amdgcn_exp2f(b.x - M);
        a.y = a.y * fa + b.y * fb;
        if (ENT) ua = ua * fa + red_u[w * C::BN + n_l] * fb;
        a.x = M;
      }
      partials[(int64_t)split * T + n0 + n_l] = make_float2(a.x, a.y);
      if (ENT) upart[(int64_t)split * T + n0 + n_l] = ua;
    }
  }
#endif
}

// ---------------------------------------------------------------------------
// Sampling (the data-generation step of Alg. 1, as a kernel on the same fused
// head): y_t = argmax_v (z_tv / temperature + g_tv), g a standard Gumbel variate
// drawn from Philox-4x32-10 with key = seed and counter (v / 4, t, 0), which is a
// draw from softmax(z_t / temperature).  Same streaming structure as the forward
// kernel: a workgroup owns a token tile and a split of the vocabulary tiles and
// carries per token the best (score, index) so far; the 4 consecutive vocabulary
// rows a lane owns in each accumulator quad are exactly one Philox block.
// Ties go to the smaller index.  Output: one (score, index) pair per token and
// split (index bit-cast into the pair's second float).
// ---------------------------------------------------------------------------
template <class C, bool ROWS>
__global__ void __launch_bounds__(C::NT)
k_fwd_sample(const bf16_t* __restrict__ W, const bf16_t* __restrict__ H, int V, int64_t T, int d, int n_kt, int n_splits,
             int balanced, int patch_tiles, float inv_temperature, uint32_t seed_lo, uint32_t seed_hi,
             float2* __restrict__ partials) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;

  const int n_tiles = (int)((T + C::BN - 1) / C::BN);
  const int total = n_tiles * n_splits;
  const int L = xcd_logical_id(blockIdx.x, total);
  if (L >= total) return;
  int split, nt;
  strip_tile(patch_tiles, L, n_splits, n_tiles, split, nt);     // as in k_fwd_lse
  const RowWalk walk = row_walk<C>(V, split, n_splits, balanced);
  const int64_t n0 = (int64_t)nt * C::BN;

  Mainloop<C, ROWS> ml;
  ml.setup();
  ml.rows_init(d);
  ml.first = first_block(split, d, n_kt);
  ml.set_b(H, nt, T, d, n_kt);

  const Lane<C> at;
  // the running best of column 16 (4 q + g) + c is lane group g's, as in k_fwd_lse
  constexpr int Q = (C::NB + 3) / 4;
  float best[Q];
  int arg[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) { best[q] = -__builtin_inff(); arg[q] = 0x7FFFFFFF; }

  f32x4 acc[C::MB][C::NB];
  auto set_tile = [&](int m0) { ml.set_a(W, m0, m0 + walk.h < walk.r1 ? m0 + walk.h : walk.r1, d, n_kt); };
  if (walk.r0 < walk.r1) {
    set_tile(walk.r0);
    ml.start_preload(smem, n_kt);
  }
  for (int m0 = walk.r0; m0 < walk.r1; m0 += walk.h) {
    const int end = m0 + walk.h < walk.r1 ? m0 + walk.h : walk.r1;
    zero_acc<C>(acc);
    ml.template finish<true>(smem, n_kt, acc);
    if (end < walk.r1) {
      set_tile(end);
      ml.start_preload(smem, n_kt);
    }
    // a lower tile, the ragged last one among them: a logit of -inf is never drawn
    if (m0 + C::BM > end) fill_rows_past<C>(acc, m0 + at.row0(), end, -__builtin_inff());
    // Four tokens at a time, rows outside: the first two Philox rounds multiply words that depend on the row block or on the
    // token alone, and are shared over the other.  (The column made anew for every tile: what depends on the token alone would be
    // carried through the main loop otherwise, in registers that it does not have.)
    const uint32_t t0 = Mainloop<C, ROWS>::fresh((int)n0 + at.col0());     // bf16 calls have fewer than 2^32 tokens
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float top[4];
      int where[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) { top[k] = -__builtin_inff(); where[k] = 0x7FFFFFFF; }
#pragma unroll
      for (int i = 0; i < C::MB; ++i) {
        const int v0 = m0 + at.row0() + i * 16;          // multiple of 4: one Philox block
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int j = 4 * q + k;
          if (j >= C::NB) continue;
          uint32_t x[4];
          philox4x32_10((uint32_t)(v0 >> 2), t0 + j * 16, 0u, 0u, seed_lo, seed_hi, x);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float sc = __builtin_fmaf(acc[i][j][e], inv_temperature, gumbel_from_bits(x[e]));
            if (sc > top[k]) { top[k] = sc; where[k] = v0 + e; }   // indices rise: strict > keeps the smallest
          }
        }
      }
      float sc;
      int v;
      reduce4_better(top, where, sc, v);
      if (sc > best[q]) { best[q] = sc; arg[q] = v; }     // ... from tile to tile too
    }
  }

  // merge the WM waves stacked along the vocabulary, through LDS
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  __attribute__((address_space(3))) f32x2* red = (__attribute__((address_space(3))) f32x2*)smem;
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (4 * q + at.g < C::NB) red[at.wm * C::BN + at.col0() + (4 * q + at.g) * 16] = f32x2{best[q], __int_as_float(arg[q])};
  __syncthreads();
  for (int n_l = threadIdx.x; n_l < C::BN; n_l += C::NT) {
    if (n0 + n_l < T) {
      f32x2 a = red[n_l];
#pragma unroll
      for (int w = 1; w < C::WM; ++w) {
        const f32x2 b = red[w * C::BN + n_l];
        if (better(b.x, __float_as_int(b.y), a.x, __float_as_int(a.y))) a = b;
      }
      partials[(int64_t)split * T + n0 + n_l] = make_float2(a.x, a.y);
    }
  }
#endif
}

// dst = packed(S^T), an m-side operand (256-row blocks), where S [R, Ccols] is row-major (ld; Ccols and ld
// multiples of 8) and optionally row-scaled:
// dst row j (a column of S), k index r (a row of S): dst(j, r) = bf16(S[r][j] * scale[r]).
// One workgroup per destination block (jt, kt): it reads S[kt*64 .. +64][jt*256 .. +256] in 16-byte
// pieces (8 columns of one row), four consecutive rows per thread, turns each 4 x 8 patch into eight
// 8-byte column pieces (4 rows of one column) and parks them in LDS as [row quad][column]; a
// destination chunk (8 consecutive r of one j, 16 bytes) is then two 8-byte LDS reads.
// Blocks in [0, n_jt) x [0, n_kt); zero outside [0, Ccols) x [0, R).
struct PackTransposed {
  const bf16_t* src;
  int64_t R;
  int Ccols;
  int64_t ld;
  const float* scale;
  bf16_t* dst;
  int n_kt;          // strip pitch of dst
  // bytes per row quad: 256 columns x 8 bytes; +16 keeps the reads below off each other's banks
  static constexpr int kPitch = kPackRowsA * 8 + 16;
  static constexpr int kLds = (kPackK / 4) * kPitch;
};
// Block (kt, jt) by the 256 threads `tid` of a workgroup, all of whose threads come here.
__device__ __forceinline__ void pack_transposed_block(const PackTransposed& p, int kt, int jt, int tid, char* tile) {
  const bf16_t* __restrict__ src = p.src;
  const int64_t R = p.R, ld = p.ld;
  const int Ccols = p.Ccols;
  constexpr int kPitch = PackTransposed::kPitch;
  const int64_t r0 = (int64_t)kt * kPackK;
  const int j0 = jt * kPackRowsA;
  const int cc = tid & 31;                // 8-column piece of the 256 columns
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int rq = (tid >> 5) + 8 * pass;   // row quad 0 .. 15
    const int j = j0 + cc * 8;
    u32x4 row[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t r = r0 + 4 * rq + k;
      row[k] = u32x4{0u, 0u, 0u, 0u};
      if (r < R && j < Ccols) {
        row[k] = load_any16(src + r * ld + j);
        if (p.scale != nullptr) {
          const float sc = p.scale[r];
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            // a copy: a vector element is not an object whose bytes can be reinterpreted in place
            const uint32_t x = row[k][m];
            const bf16x2 v = __builtin_bit_cast(bf16x2, x);
            const bf16x2 w = {(bf16_t)((float)v[0] * sc), (bf16_t)((float)v[1] * sc)};
            row[k][m] = __builtin_bit_cast(uint32_t, w);
          }
        }
      }
    }
    // dword m of a row holds columns 2m (low half) and 2m + 1 (high half)
    char* out = tile + rq * kPitch + cc * 64;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t a0 = row[0][m], a1 = row[1][m], a2 = row[2][m], a3 = row[3][m];
      const u32x4 piece = {(a0 & 0xFFFFu) | (a1 << 16), (a2 & 0xFFFFu) | (a3 << 16),        // column 2m: rows 0..3
                           (a0 >> 16) | (a1 & 0xFFFF0000u), (a2 >> 16) | (a3 & 0xFFFF0000u)};  // column 2m + 1
      *(u32x4*)(out + m * 16) = piece;
    }
  }
  __syncthreads();
  char* outb = (char*)p.dst + ((int64_t)jt * p.n_kt + kt) * (int64_t)kPackBlockBytesA;
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int idx = it * 256 + tid;
    const int rowj = idx >> 3, c = idx & 7;                 // destination row (j), 8 consecutive k = row quads 2c, 2c + 1
    const u32x2 lo = *(const u32x2*)(tile + (2 * c) * kPitch + rowj * 8);
    const u32x2 hi = *(const u32x2*)(tile + (2 * c + 1) * kPitch + rowj * 8);
    *(u32x4*)(outb + rowj * 128 + c * 16) = u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
}
__global__ void __launch_bounds__(256) k_pack_transposed(PackTransposed p, Gate gate) {
  __shared__ __attribute__((aligned(16))) char tile[PackTransposed::kLds];
  if (gate_closed(gate)) return;
  pack_transposed_block(p, blockIdx.x, blockIdx.y, threadIdx.x, tile);
}

// ---------------------------------------------------------------------------
// Backward, step 1: recompute a logits^T tile and turn it into the gradient
// with respect to the logits.  With p = softmax(z_t) and f_t = c_t (1 - p_{t,y_t}),
//     dL/dz[t][v] = c_t (1[v == y_t] - p[t][v]) = f_t * G[t][v],
//     G[t][y_t] = 1,   G[t][v] = -p[t][v] / (1 - p[t][y_t])  otherwise.
// G is what is rounded to bf16: its one-hot entry is exact, and the remaining
// entries (tiny, with uncorrelated roundings) carry no common factor, so no
// rounding error is shared by all tokens of a rollout.  The fp32 row factor f_t
// is applied by the consumers: dH = diag(f) (G W), dW = G^T (diag(f) H).
// G is written twice, packed, for one panel of token rows:
//     Gp   rows = tokens,      k = vocabulary   -> B operand of the dH contraction
//     GTp  rows = vocabulary,  k = tokens       -> B operand of the dW contraction
// Entries outside the valid ranges are written as zeros (whole tiles are stored).
//   A = W (M = vocabulary), B = H from the panel's first token (N = tokens), packed or in place.
// ---------------------------------------------------------------------------
// In a small call the transposed rows that the next launch wants come along (`n_pack` workgroups in front, two blocks each):
// the recompute is closed in nearly every call, and a launch of its own that does nothing costs 3 us.
template <class C, bool ROWS>
__global__ void __launch_bounds__(C::NT)
k_bwd_dz(const bf16_t* __restrict__ W, const bf16_t* __restrict__ H_panel, int V, int64_t n_valid, int d, int n_kt,
         const int32_t* __restrict__ tokens, const float* __restrict__ lse2, const float* __restrict__ inv_omp,
         bf16_t* __restrict__ Gp, int g_n_kt, bf16_t* __restrict__ GTp, int gt_n_kt, Gate gate, int n_pack, PackTransposed pack,
         int pack_kt, int pack_blocks) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;
  static_assert(C::NT == 512 && 2 * PackTransposed::kLds <= C::LDS_BYTES, "two blocks per workgroup");
  if ((int)blockIdx.x < n_pack) {
    const int half = threadIdx.x >> 8, i = 2 * blockIdx.x + half;
    const int block = i < pack_blocks ? i : pack_blocks - 1;     // an odd one out is written twice, with the same values
    pack_transposed_block(pack, block % pack_kt, block / pack_kt, threadIdx.x & 255, smem_raw + half * PackTransposed::kLds);
    return;
  }
  if (gate_closed(gate)) return;

  const int MT = (V + C::BM - 1) / C::BM;
  const int NTl = (int)((n_valid + C::BN - 1) / C::BN);
  const int total = MT * NTl;
  const int L = xcd_logical_id(blockIdx.x - n_pack, total);
  if (L >= total) return;
  int mt, nt;
  strip_tile<4>(L, MT, NTl, mt, nt);
  const int m0 = mt * C::BM;
  const int64_t n0 = (int64_t)nt * C::BN;

  Mainloop<C, ROWS> ml;
  ml.setup();
  ml.rows_init(d);
  ml.set_a(W, m0, V, d, n_kt);
  ml.set_b(H_panel, nt, n_valid, d, n_kt);

  f32x4 acc[C::MB][C::NB];
  zero_acc<C>(acc);
  ml.start(smem, n_kt);
  ml.finish(smem, n_kt, acc);

  const Lane<C> at;
  const int row0 = m0 + at.row0();                 // first vocabulary row of this lane
  uint32_t pk[C::MB][C::NB][2];
#pragma unroll
  for (int j = 0; j < C::NB; ++j) {
    const int64_t n = n0 + at.col0() + j * 16;
    const bool ok = n < n_valid;
    const float ninv = ok ? -inv_omp[n] : 0.f, l2 = ok ? lse2[n] : 0.f;    // -1 / (1 - p_y), lse in the exp2 domain
    const int rel = ok ? tokens[n] - row0 : -1;                            // the one-hot term's row
#pragma unroll
    for (int i = 0; i < C::MB; ++i) {
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][r], kLog2e, -l2)) * ninv;
        if (rel == 16 * i + r) x[r] = ninv != 0.f ? 1.f : 0.f;
        if (row0 + 16 * i + r >= V) x[r] = 0.f;     // rows past the vocabulary carry exp2(0 - lse2) garbage
      }
      pk[i][j][0] = bf16_pair(x[0], x[1]);
      pk[i][j][1] = bf16_pair(x[2], x[3]);
    }
  }
  // Gp: rows = tokens (n), k = vocabulary (m);  GTp: rows = vocabulary (m), k = tokens (n)
  store_both_copies<C>(smem, pk, Gp, g_n_kt, GTp, gt_n_kt, m0, n0);
#endif
}

// The first launch of a single sweep over operands in place: what the call begins with (workgroup 0), and per 64 tokens the
// reference exponents of k_sweep (the largest logit among the first 256 vocabulary entries and the sampled token's own, which
// is gathered here) with the per-token arrays of TokenInit.  Three launches otherwise; see sweep_begins_in_one_launch in
// oapl_api.hip.
template <class C, class Begin>
__global__ void __launch_bounds__(C::NT)
k_sweep_begin(Begin begin, const bf16_t* __restrict__ W, const bf16_t* __restrict__ H, int V, int64_t T, int d, int n_kt,
              const int32_t* __restrict__ tokens, float* __restrict__ zy, TokenInit init) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;
  static_assert(C::NT == 256, "begin's steps are for 256 threads");
  if (blockIdx.x == 0) return begin.run(0, 1, kPlan | kRest);
  const int64_t nt = blockIdx.x - 1, n0 = nt * C::BN;

  Mainloop<C, true> ml;
  ml.setup();
  ml.rows_init(d);
  ml.set_b(H, nt, T, d, n_kt);
  ml.set_a(W, 0, V, d, n_kt);
  const Lane<C> at;
  constexpr int kShare = C::BN / C::NW;      // tokens per wavefront; lane i has the i-th one's
  static_assert(kShare == 16, "four rounds of four tokens");
  const int64_t t_lane = n0 + at.wm * kShare + at.c;
  const int tok = tokens[t_lane < T ? t_lane : T - 1];
  f32x4 acc[C::MB][C::NB];
  zero_acc<C>(acc);
  ml.start(smem, n_kt);
  ml.finish(smem, n_kt, acc);

  if (C::BM > V) fill_rows_past<C>(acc, at.row0(), V, -__builtin_inff());
  static_assert(C::NB == 4 && C::WN == 1, "four columns per lane");
  float x[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x[k] = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < C::MB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[k] = fmaxf(x[k], acc[i][k][r]);
  }
  __attribute__((address_space(3))) float* red = (__attribute__((address_space(3))) float*)smem;
  red[at.wm * C::BN + at.g * 16 + at.c] = reduce4(x, [](float a, float b) { return fmaxf(a, b); });
  __syncthreads();
  // each wavefront's 16 tokens, four at a time with 16 lanes each, the next four's first pieces on their way meanwhile
  const int pieces = d / 8;
  auto row = [&](int q) { return at.wm * kShare + q * 4 + at.g; };
  int y[kShare / 4];
#pragma unroll
  for (int q = 0; q < kShare / 4; ++q) y[q] = __shfl(tok, q * 4 + at.g, 64);
  auto load = [&](const int q, int e, bf16x8& h, bf16x8& w) {
    const int64_t t = n0 + row(q) < T ? n0 + row(q) : T - 1;
    const int p = e < pieces ? e : pieces - 1;
    h = *(const bf16x8*)(H + t * d + p * 8);
    w = *(const bf16x8*)(W + (int64_t)(y[q] < 0 || y[q] >= V ? 0 : y[q]) * d + p * 8);
  };
  constexpr int kAhead = 2;      // pieces per lane: rows of up to 256 elements are all under way at once
  bf16x8 h[kShare / 4][kAhead], w[kShare / 4][kAhead];
#pragma unroll
  for (int q = 0; q < kShare / 4; ++q)
#pragma unroll
    for (int k = 0; k < kAhead; ++k) load(q, at.c + 16 * k, h[q][k], w[q][k]);
  // Summed in the order of gather_logit, to the bit: lane c does the work of its lanes c, c + 16, c + 32 and c + 48, one sum
  // each. One sum of all a lane's pieces, a chain of 64 products at d = 1024, moved the last bit of the logit, with it the
  // reference exponent and the bf16 roundings of the whole panel row: gradients of 7749 tokens (V = 151936) 1e-4 from
  // gather_logit's.
#pragma unroll
  for (int q = 0; q < kShare / 4; ++q) {
    float part[4] = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](const int m, const bf16x8& x, const bf16x8& y, bool there) {
      if (!there) return;
#pragma unroll
      for (int i = 0; i < 8; ++i) part[m] += (float)x[i] * (float)y[i];
    };
#pragma unroll
    for (int k = 0; k < kAhead; ++k) add(k, h[q][k], w[q][k], at.c + 16 * k < pieces);
    for (int k0 = 16 * kAhead; k0 < pieces; k0 += 64) {
      const bool more = k0 + 32 < pieces;
      bf16x8 a[4], b[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < 2 || more) load(q, at.c + k0 + 16 * k, a[k], b[k]);     // past the row's end its last piece
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < 2 || more) add((kAhead + k) & 3, a[k], b[k], at.c + k0 + 16 * k < pieces);
    }
    float z = (part[0] + part[2]) + (part[1] + part[3]);
#pragma unroll
    for (int o = 8; o > 0; o /= 2) z += __shfl_xor(z, o, 64);
    const int64_t t = n0 + row(q);
    if (at.c != 0 || t >= T) continue;
    float largest = kNegHuge;
#pragma unroll
    for (int i = 0; i < C::WM; ++i) largest = fmaxf(largest, red[i * C::BN + row(q)] * kLog2e);
    // a token out of range is recorded by k_sweep_finish, or by the fallback where that is closed
    init_token(init, t, y[q] >= 0 && y[q] < V ? z : __builtin_nanf(""), largest, zy);
  }
#endif
}

// The first launch of a single sweep of few tokens over operands in place whose rows are long: what the call begins with
// (workgroup 0; `steps` = 0: a launch of its own has done it) and the logits of the first 256 vocabulary entries, a tile of 64
// tokens in `splits` parts over d, part[split][t][row], which the gather sums. Bound by the latency of a walk's loads, d / 64
// blocks one after the other (0.8 us each): 1003 tokens at d = 4096 49 us in one part, 14 in eight.
template <class C, class Begin>
__global__ void __launch_bounds__(C::NT)
k_ref_begin(Begin begin, int steps, const bf16_t* __restrict__ W, const bf16_t* __restrict__ H, int V, int64_t T, int d, int n_kt,
            int splits, float* __restrict__ part) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;
  static_assert(C::NT == 256 && C::BM == 256 && C::NS == 4, "begin's steps are for 256 threads; walks start at any block");
  if (blockIdx.x == 0) {
    if (steps != 0) begin.run(0, 1, steps);
    return;
  }
  const int64_t nt = (blockIdx.x - 1) / splits, n0 = nt * C::BN;
  const int split = (blockIdx.x - 1) % splits;
  const int k0 = (int)((int64_t)split * n_kt / splits), k1 = (int)((int64_t)(split + 1) * n_kt / splits);

  Mainloop<C, true> ml;
  ml.setup();
  ml.rows_init(d);
  if (k1 < n_kt) ml.vlast = ml.voff;      // this walk's last block is not the rows' last
  ml.set_a(W + k0 * C::BK, 0, V, d, n_kt);
  ml.set_b(H + k0 * C::BK, nt, T, d, n_kt);
  f32x4 acc[C::MB][C::NB];
  zero_acc<C>(acc);
  ml.start(smem, k1 - k0);
  ml.finish(smem, k1 - k0, acc);

  const Lane<C> at;
#pragma unroll
  for (int j = 0; j < C::NB; ++j) {
    const int64_t t = n0 + at.col0() + 16 * j;
    if (t >= T) continue;
#pragma unroll
    for (int i = 0; i < C::MB; ++i) *(f32x4*)(part + ((int64_t)split * T + t) * C::BM + at.row0() + 16 * i) = acc[i][j];
  }
#endif
}

// ---------------------------------------------------------------------------
// Single-sweep variant of steps a1, a2 and a8: ONE pass over the logits serves
// both the log-sum-exp and the gradient.  The soft-max is written unnormalised
// against a per-token reference exponent ref2[t] that is known before the pass
// (an upper-bound-free guess: the largest of a sample of the row's logits, see
// k_gather_logit), in the exp2 domain:
//     Pt[t][v] = 2^(z[t][v] * log2(e) - ref2[t])          (bf16, packed twice like G above)
//     spart[mt][t] = sum over the vocabulary tile mt of Pt[t][v]   (fp32, from the unrounded values)
// so that, with S_t = sum_mt spart[mt][t]:  lse_t = (ref2[t] + log2 S_t) ln 2  and
//     dL/dz[t][v] = c_t (1[v == y_t] - Pt[t][v] / S_t) = a_t * Gt[t][v],   a_t = -c_t / S_t,
//     Gt[t][v] = Pt[t][v]  (v != y_t),    Gt[t][y_t] = Pt[t][y_t] - S_t   (patched in by k_sweep_finish).
// The row factor a_t only exists once S_t and the rollout's residual are known, i.e. after the
// pass; it is applied by the same consumers as f_t above (dH epilogue, transposed H).  bf16 has
// fp32's exponent range, so the unnormalised values are as accurate as normalised ones as long
// as the row's largest logit stays within ~2^100 of the reference; k_sweep_finish checks that
// and otherwise sends the whole call down the two-pass path.
// ---------------------------------------------------------------------------
template <class C, bool ROWS>
__global__ void __launch_bounds__(C::NT)
k_sweep(const bf16_t* __restrict__ W, const bf16_t* __restrict__ H_panel, int V, int64_t n_valid, int d, int n_kt,
        const float* __restrict__ ref2 /* panel-local */, bf16_t* __restrict__ Gp, int g_n_kt,
        bf16_t* __restrict__ GTp, int gt_n_kt, float* __restrict__ spart /* [MT][ld_s], panel-local */,
        int64_t ld_s, Gate gate) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;
  if (gate_closed(gate)) return;

  const int MT = (V + C::BM - 1) / C::BM;
  const int NTl = (int)((n_valid + C::BN - 1) / C::BN);
  const int total = MT * NTl;
  const int L = xcd_logical_id(blockIdx.x, total);
  if (L >= total) return;
  int mt, nt;
  strip_tile<4>(L, MT, NTl, mt, nt);
  const int m0 = mt * C::BM;
  const int64_t n0 = (int64_t)nt * C::BN;

  Mainloop<C, ROWS> ml;
  ml.setup();
  ml.rows_init(d);
  ml.set_a(W, m0, V, d, n_kt);
  ml.set_b(H_panel, nt, n_valid, d, n_kt);

  const Lane<C> at;
  f32x4 acc[C::MB][C::NB];
  zero_acc<C>(acc);
  ml.start(smem, n_kt);
  // the epilogue's per-token references are requested two k-blocks before the end, so that their
  // latency hides behind the last multiplications instead of stalling the epilogue
  const int k_early = n_kt > C::NS ? (n_kt - 2) & ~(C::NS - 1) : 0;
  ml.steps(smem, 0, k_early, n_kt, acc);
  float r2v[C::NB];
#pragma unroll
  for (int j = 0; j < C::NB; ++j) {
    const int64_t n = n0 + at.col0() + j * 16;
    // token columns past the panel: reference +inf, every entry 2^(-inf) = 0
    r2v[j] = n < n_valid ? ref2[n] : __builtin_inff();
  }
  ml.steps(smem, k_early, n_kt, n_kt, acc);
  ml.drain();

  // ragged last vocabulary tile: rows >= V do not exist (2^(-inf) = 0 below)
  if (m0 + C::BM > V) fill_rows_past<C>(acc, m0 + at.row0(), V, -__builtin_inff());
  float csum[(C::NB + 3) / 4];    // columns 16 (4 q + g) + c, as in k_fwd_lse
  uint32_t pk[C::MB][C::NB][2];   // the tile as bf16 pairs
#pragma unroll
  for (int q = 0; q < (C::NB + 3) / 4; ++q) {
    float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = 4 * q + k;
      if (j >= C::NB) continue;
#pragma unroll
      for (int i = 0; i < C::MB; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][2 * p], kLog2e, -r2v[j]));
          const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][2 * p + 1], kLog2e, -r2v[j]));
          x[k] += e0;
          x[k] += e1;
          pk[i][j][p] = bf16_pair(e0, e1);
        }
    }
    csum[q] = reduce4(x, [](float a, float b) { return a + b; });
  }
  // row sums: the WM waves stacked along the vocabulary, through LDS, in a fixed order
  __attribute__((address_space(3))) float* red = (__attribute__((address_space(3))) float*)smem;
#pragma unroll
  for (int q = 0; q < (C::NB + 3) / 4; ++q)
    if (4 * q + at.g < C::NB) red[at.wm * C::BN + at.col0() + (4 * q + at.g) * 16] = csum[q];
  lds_barrier();
  for (int n_l = threadIdx.x; n_l < C::BN; n_l += C::NT) {
    if (n0 + n_l < n_valid) {
      float a = red[n_l];
#pragma unroll
      for (int w = 1; w < C::WM; ++w) a += red[w * C::BN + n_l];
      spart[(int64_t)mt * ld_s + n0 + n_l] = a;
    }
  }
  lds_barrier();
  store_both_copies<C>(smem, pk, Gp, g_n_kt, GTp, gt_n_kt, m0, n0);
#endif
}

// 16 bytes of the neighbouring lane (lane ^ 1, which must be active).
__device__ __forceinline__ f32x4 neighbour(const f32x4 v) {
  f32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = v[e];   // a copy: a vector element is not an object whose bytes can be reinterpreted in place
    r[e] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1 /* quad_perm 1,0,3,2 */, 0xF, 0xF, true));
  }
  return r;
}

// fp32 tile -> out[n][m] (n < n_rows, row pitch d = the m extent), overwritten or added to, straight from the
// accumulators.  A lane owns 16 bytes of its row n per block, the four groups 64 bytes; neighbouring lanes (rows n, n + 1)
// trade pieces of two block rows, so that the even lane holds block row 2q of both rows, the odd one block row 2q + 1, and
// every load and store covers whole 128-byte lines.  The old values of a block column are requested together,
// from clamped (always valid) addresses, so the read-add-write waits for memory once per column, not once per piece.
template <class C, bool ACCUMULATE>
__device__ __forceinline__ void store_f32_tile(const f32x4 (&acc)[C::MB][C::NB], float* __restrict__ out, int d, int n_rows,
                                               int m0, int n0) {
  const Lane<C> at;
  const bool odd = (at.c & 1) != 0;
  const int m = m0 + at.row0() + (odd ? 16 : 0);
#pragma unroll
  for (int j = 0; j < C::NB; ++j) {
    const int n = n0 + at.col0() + j * 16 - (odd ? 1 : 0);    // the even row; both lanes store it and the next
    f32x4 old[C::MB];
    if (ACCUMULATE) {
#pragma unroll
      for (int i = 0; i < C::MB; ++i) {
        const int mi = m + 32 * (i / 2), ni = n + (i & 1);
        old[i] = *(const f32x4*)(out + (int64_t)(ni < n_rows ? ni : n_rows - 1) * d + (mi < d ? mi : d - 4));
      }
    }
#pragma unroll
    for (int i = 0; i < C::MB; i += 2) {
      const f32x4 lo = acc[i][j], hi = acc[i + 1][j];
      const f32x4 got = neighbour(odd ? lo : hi);
      const f32x4 piece[2] = {odd ? got : lo, odd ? hi : got};
      const int mi = m + 16 * i;
#pragma unroll
      for (int r = 0; r < 2; ++r)
        if (mi < d && n + r < n_rows)
          *(f32x4*)(out + (int64_t)(n + r) * d + mi) = ACCUMULATE ? piece[r] + old[i + r] : piece[r];
    }
  }
}

// ---------------------------------------------------------------------------
// Backward, step 2: dH[t][j] = f_t * sum_v G[t][v] * W[v][j]
//   A = W^T (rows = hidden index j, k = vocabulary), read from W in place (ATR) or from a packed copy; B = Gp (rows =
//   tokens), K = V.
// A panel of few tokens has few tiles (d / 256 x tokens / 384), each a walk over the whole vocabulary: 1003 tokens at
// d = 4096 kept 48 of 256 CUs busy for 4.1 ms.  SPLIT: `splits` workgroups share a tile's k-blocks, each writing its
// fp32 partial sum (whole 128-byte lines) for k_dh_reduce; the host chooses the count (pick_dh in
// oapl_api.hip).
// ---------------------------------------------------------------------------
struct DhArgs {
  const bf16_t* W;          // or W^T, packed
  int V, wt_n_kt;
  const bf16_t* Gp;
  int g_n_kt, d;
  int64_t n_valid;
  int nk;                   // k-blocks to contract: ceil(V / 64)
  const float* row_factor;  // f_t, panel-local
  bf16_t* dH;               // panel's first row
  int splits;
  float* part;              // [splits][n_valid][d]
};
#if defined(__HIP_DEVICE_COMPILE__)
template <class C, bool SPLIT, bool ATR>
__device__ __forceinline__ void dh_tile(const DhArgs& args, int bid, lds_char_ptr smem) {
  const bf16_t* __restrict__ W = args.W;
  const bf16_t* __restrict__ Gp = args.Gp;
  const float* __restrict__ row_factor = args.row_factor;
  bf16_t* __restrict__ dH = args.dH;
  const int V = args.V, d = args.d, nk = args.nk, splits = args.splits;
  const int64_t n_valid = args.n_valid;
  const int MT = (d + C::BM - 1) / C::BM;
  const int NTl = (int)((n_valid + C::BN - 1) / C::BN);
  const int total = MT * NTl * (SPLIT ? splits : 1);
  const int L = xcd_logical_id(bid, total);
  if (L >= total) return;
  // neighbouring ids walk the tiles of one split, so the workgroups of an XCD share its operand blocks
  const int split = SPLIT ? L / (MT * NTl) : 0;
  int mt, nt;
  strip_tile<4>(L - split * (MT * NTl), MT, NTl, mt, nt);
  const int m0 = mt * C::BM;
  const int64_t n0 = (int64_t)nt * C::BN;
  const int k0 = SPLIT ? (int)((int64_t)split * nk / splits) : 0;
  const int k1 = SPLIT ? (int)((int64_t)(split + 1) * nk / splits) : nk;

  Mainloop<C, false, ATR> ml;
  ml.setup();
  if (ATR) ml.set_a_transposed(W + (int64_t)k0 * C::BK * d, mt, V - (int64_t)k0 * C::BK, d);
  else ml.set_a_packed(W, m0, args.wt_n_kt, k0);
  ml.set_b_packed(Gp, n0, args.g_n_kt, k0);

  f32x4 acc[C::MB][C::NB];
  zero_acc<C>(acc);
  ml.start(smem, k1 - k0);
  ml.finish(smem, k1 - k0, acc);

  if (SPLIT) {
    store_f32_tile<C, false>(acc, args.part + (int64_t)split * n_valid * d, d, (int)n_valid, m0, (int)n0);
    return;
  }
  const Lane<C> at;
#pragma unroll
  for (int j = 0; j < C::NB; ++j) {
    const int64_t n = n0 + at.col0() + j * 16;
    const float f = n < n_valid ? row_factor[n] : 0.f;
#pragma unroll
    for (int i = 0; i < C::MB; ++i) acc[i][j] *= f;
  }
#pragma unroll 1
  for (int c = 0; c < C::NM_CHUNKS; ++c) {
    stage_nm<C>(smem, acc, c);
    __syncthreads();
    store_nm<C>(smem, dH + n0 * d + m0, d, n_valid - n0, (int64_t)d - m0, c);
    __syncthreads();
  }
}
#endif
template <class C, bool SPLIT, bool ATR>
__global__ void __launch_bounds__(C::NT) k_bwd_dh(DhArgs args, Gate gate) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  if (gate_closed(gate)) return;
  dh_tile<C, SPLIT, ATR>(args, blockIdx.x, (lds_char_ptr)smem_raw);
#endif
}

// dH[n][j] = f_n * (sum of the splits' partial sums, in order): 8 consecutive j per thread.  Bound by memory.
__global__ void __launch_bounds__(256)
k_dh_reduce(const float* __restrict__ part, int splits, int64_t n_valid, int d, const float* __restrict__ row_factor,
            bf16_t* __restrict__ dH, Gate gate) {
  if (gate_closed(gate)) return;
  const int64_t total = n_valid * (d / 8), stride = n_valid * d;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const float* p = part + idx * 8;
    f32x4 lo = *(const f32x4*)p, hi = *(const f32x4*)(p + 4);
#pragma unroll 4
    for (int s = 1; s < splits; ++s) {
      lo += *(const f32x4*)(p + s * stride);
      hi += *(const f32x4*)(p + s * stride + 4);
    }
    const float f = row_factor[idx / (d / 8)];
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = (bf16_t)(lo[e] * f);
      v[4 + e] = (bf16_t)(hi[e] * f);
    }
    *(bf16x8*)(dH + idx * 8) = v;
  }
}

// ---------------------------------------------------------------------------
// Backward, step 3: dW[v][j] (+)= sum_t G[t][v] * (f_t H[t][j])
//   A = packed (diag(f) H)^T (rows = hidden index j, k = panel tokens), B = GTp (rows = vocabulary).
// fp32 output written straight from the accumulators: 4 consecutive j per lane.
// ---------------------------------------------------------------------------
struct DwArgs {
  const bf16_t *HTp, *GTp;
  int t_n_kt;               // strip pitch of both
  int d, V, nk;             // k-blocks to contract: ceil(panel tokens / 64)
  float* dW;
  int accumulate;
};
#if defined(__HIP_DEVICE_COMPILE__)
template <class C>
__device__ __forceinline__ void dw_tile(const DwArgs& args, int L /* tile */, lds_char_ptr smem) {
  const bf16_t* __restrict__ HTp = args.HTp;
  const bf16_t* __restrict__ GTp = args.GTp;
  float* __restrict__ dW = args.dW;
  const int d = args.d, V = args.V, nk = args.nk, t_n_kt = args.t_n_kt;
  const int MT = (d + C::BM - 1) / C::BM;
  const int NTl = (V + C::BN - 1) / C::BN;
  if (L >= MT * NTl) return;
  int mt, nt;
  strip_tile<4>(L, MT, NTl, mt, nt);
  const int m0 = mt * C::BM;
  const int n0 = nt * C::BN;

  Mainloop<C> ml;
  ml.setup();
  ml.set_a_packed(HTp, m0, t_n_kt, 0);
  ml.set_b_packed(GTp, n0, t_n_kt, 0);

  f32x4 acc[C::MB][C::NB];
  zero_acc<C>(acc);
  ml.start(smem, nk);
  ml.finish(smem, nk, acc);

  if (args.accumulate) store_f32_tile<C, true>(acc, dW, d, V, m0, n0);
  else store_f32_tile<C, false>(acc, dW, d, V, m0, n0);
}
#endif
template <class C>
__global__ void __launch_bounds__(C::NT) k_bwd_dw(DwArgs args, Gate gate) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  if (gate_closed(gate)) return;
  dw_tile<C>(args, xcd_round_major_id(blockIdx.x), (lds_char_ptr)smem_raw);   // launched in whole rounds of 256 workgroups
#endif
}

// dW's tiles (n_dw) in the launch that it shares with dH (k_bwd_grads) are spread evenly over the XCDs: in rounds of 256, 32 to
// an XCD, as a launch of its own walks them, the few tiles of such a batch all land on the first XCDs and wait there behind
// dH's workgroups (rounds / even, the launch: 4335 tokens at d = 64, V = 3951, 34 + 31 tiles, 79 / 44 us; 8000 at d = 256,
// V = 8000 152 / 94; 1000 at d = 256, V = 1544 23.2 / 21.7).
__host__ __device__ __forceinline__ int shared_dw_tile(int workgroup, int n_dw) { return xcd_logical_id(workgroup, n_dw); }

// Steps 2 and 3 of a small batch (one panel, 128 x 128 tiles, operands in place) in one launch: the first n_dh (a multiple of
// 8) workgroups are dH's, the others dW's.  Neither fills the chip and they do not depend on each other: whole calls in two
// launches / one, 1000 tokens at d = 256, V = 1544 66 / 53 us; 700 at d = 128, V = 300 48 / 39; 1000 at d = 1024, V = 8192
// 118 / 106.  256 x 384 tiles gain nothing from it (V = 151936, d = 4096, 1003 tokens: 2166 / 2185 us; with longer dH walks
// beside dW's tiles 2221, 300 tokens 1007 / 1286): the two kinds of tile share no operands in the L2.
template <class C, bool SPLIT>
__global__ void __launch_bounds__(C::NT) k_bwd_grads(DhArgs dh, int n_dh, DwArgs dw, int n_dw, Gate gate) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  lds_char_ptr smem = (lds_char_ptr)smem_raw;
  if (gate_closed(gate)) return;
  if ((int)blockIdx.x < n_dh) dh_tile<C, SPLIT, true>(dh, blockIdx.x, smem);
  else dw_tile<C>(dw, shared_dw_tile(blockIdx.x - n_dh, n_dw), smem);
#endif
}

// ---------------------------------------------------------------------------
// Packing of row-major matrices into the block layout the main loop reads.
// ---------------------------------------------------------------------------

// Aligned copy of a matrix that starts at any element: `pieces` of 16 bytes.  Bound by memory.
__global__ void __launch_bounds__(256)
k_copy_aligned(const bf16_t* __restrict__ src, int64_t pieces, bf16_t* __restrict__ dst) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pieces; i += (int64_t)gridDim.x * 256)
    ((u32x4*)dst)[i] = load_any16(src + i * 8);
}

// dst = packed(src), src [R, K] row-major with leading dimension ld (K and ld multiples of 8),
// in blocks of `rb` rows (256 for an m-side operand, 384 for an n-side operand).  One workgroup
// per block; blocks in [0, n_rt) x [0, n_kt); everything outside [0, R) x [0, K) is written as zero.
__global__ void __launch_bounds__(256)
k_pack_rows(const bf16_t* __restrict__ src, int64_t R, int K, int64_t ld, bf16_t* __restrict__ dst, int n_kt, int rb) {
  const int kt = blockIdx.x;
  const int64_t rt = blockIdx.y;
  char* out = (char*)dst + (rt * n_kt + kt) * (int64_t)rb * kPackRowBytes;
  for (int idx = threadIdx.x; idx < rb * 8; idx += 256) {   // chunks of 16 B
    const int row = idx >> 3, c = idx & 7;
    const int64_t r = rt * rb + row;
    const int k = kt * kPackK + c * 8;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (r < R && k < K) v = load_any16(src + r * ld + k);
    *(u32x4*)(out + row * 128 + c * 16) = v;
  }
}

}  // namespace oapl
