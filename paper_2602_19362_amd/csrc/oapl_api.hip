// C ABI of the OAPL loss head: argument checks, workspace plan, launch order.
// Every step of the path runs in the kernels of this directory; nothing here
// computes on the host and nothing falls back to a CPU path.
#include "oapl.h"

#include <math.h>
#include <mutex>
#include <utility>
#include <vector>

#include "gemm_bf16.hip.h"
#include "gemm_f32.hip.h"
#include "small_kernels.hip.h"

namespace oapl {

// 256 x 384 x 64 tiles, 8 wavefronts in a 4 x 2 grid, each a 64 x 192 patch
// (4 x 12 MFMA blocks, 192 accumulator registers per lane), two wavefronts per
// SIMD; operands in a ring of 2 LDS stages (160 KB, the whole LDS of a CU).
typedef TileCfg<4, 2, 4, 12, 2> Cfg;
static_assert(Cfg::BN == kPackRowsB, "n-side operands of the loss path are packed in blocks of one tile");
// ... with each block's loads in one go, for a sweep of one token tile or whose tiles are there all at once: it waits for W to
// arrive (300 tokens at d = 2048, V = 32000, 125 tiles: 84 us, 87 .. 91 spread; 380 at d = 4096, V = 151936: 464 / 469).
typedef TileCfg<4, 2, 4, 12, 2, 0, true> CfgEarly;
// Where tiles of that size are too few to fill the chip (small heads and hidden sizes): 128 x 128, two workgroups per CU,
// on the same packed blocks.
typedef TileCfg<2, 2, 4, 4, 2, kPackRowsB> CfgSmall;
// ... and, where there are no more of them than CUs, with a ring of four stages.
typedef TileCfg<2, 2, 4, 4, 4, kPackRowsB> CfgDeep;
// Tiles of the scoring and sampling kernels over row-major operands.  A call of few tokens pays for every padded
// token column and is bound by reading W once; a call of many is bound by operand delivery, which wants the largest
// tile.  128 x 64 (48 KB of LDS, three workgroups per CU to keep W streaming through each other's barriers) serves up to 64 tokens,
// 128 x 128 (two per CU) up to 128.  From there on a tile is one per CU and 256 tall, and its width follows from the token count
// (pick_tile); up to 256 tokens it may be 320 tall instead, where that divides the rows of a CU into fewer or better filled
// tiles (V = 151936, 594 rows per CU: two tiles of 297 in place of three of 198; scoring and sampling 200 tokens at d = 3000
// 249 / 271 and 266 / 286 us, at d = 512 46 / 51, 59 / 67; with loads that go out early (Cfg256Early) 254, 265).
typedef TileCfg<4, 1, 2, 4, 2> Cfg64;
typedef TileCfg<4, 2, 2, 4, 2> Cfg128;
typedef TileCfg<4, 2, 4, 8, 2> Cfg256;
typedef TileCfg<4, 2, 5, 8, 2> Cfg256Tall;
// ... up to two token tiles over a W that the memory-side cache cannot hold wait for it to arrive: their loads go out as early
// as they can. Early / spread, 200, 400 and 512 tokens: d = 4096, V = 48000 (375 MiB) sampling -5, -8, -5 %, scoring -5, -5, -4
// %; d = 2048, V = 100000 (391 MiB) -5, -5, -2 and -5, -4, -4 %; V = 151936 -4, -3, -1 and -4, -2, -2 %. Where the cache holds
// it (W the same from call to call): d = 4096, V = 3000 +8 %; d = 2048, V = 8000 +6 .. +8 %; d = 1024, V = 48000 0 .. +6 %.
typedef TileCfg<4, 2, 4, 8, 2, 0, true> Cfg256Early;
static bool early_pays(int64_t T, int V, int d) {
  return T <= 2 * Cfg256Early::BN && (int64_t)V * d * 2 > (int64_t)256 << 20;
}
// ... and one token tile reads W once: non-temporal loads, with which 16 and 64 tokens at d = 4096 and 5120 read it at 5.8 .. 6.8
// TB/s (5.5 .. 6.1 with others; of 256 tokens 3.8 .. 4.5, 3.7 .. 4.2), and, rows a multiple of 4 KiB apart, each workgroup's walk
// over k from another block on (TileCfg's ONCE).  With equally many rows for every workgroup (row_walk), scoring before / now at V
// = 151936, us: d = 4096 16 tokens 238 / 202, 64 231 / 214, 128 283 / 260, 192 340 / 286, 256 348 / 300 (sampling 227 / 197, 225 /
// 211, 283 / 264, 348 / 310, 358 / 323); d = 2048 16 tokens 153 / 107, 128 180 / 142, 256 203 / 164; d = 5120 286 / 255, 388 / 371,
// 458 / 390.  Rows that are not whole 128-byte lines would be fetched twice (d = 3000, V = 60000: +12 .. +20 %), and a W that
// mostly survives in the memory-side cache from call to call is better left there (264 MiB +3 .. +10 %, 297 MiB -4 .. -16 %, 305
// MiB -4 .. -11 %).
typedef TileCfg<4, 1, 2, 4, 2, 0, false, true> Cfg64Once;
typedef TileCfg<4, 2, 2, 4, 2, 0, false, true> Cfg128Once;
typedef TileCfg<4, 2, 4, 8, 2, 0, true, true> Cfg256Once;
typedef TileCfg<4, 2, 5, 8, 2, 0, true, true> Cfg256TallOnce;
static bool once_pays(int64_t T, int V, int d) {
  return T <= Cfg256Once::BN && d % kPackK == 0 && (int64_t)V * d * 2 > (int64_t)288 << 20;
}
// Odd widths: the n-side block is 4.5 or 5.5 loads per wave, the last of them half of the waves'.
typedef TileCfg<4, 2, 4, 9, 2> Cfg288;
typedef TileCfg<4, 2, 4, 10, 2> Cfg320;
typedef TileCfg<4, 2, 4, 11, 2> Cfg352;
// The sweep's reference exponents: the first 256 vocabulary entries of 64 tokens (a sixth of a packed block of H).
typedef TileCfg<4, 1, 4, 4, 4, kPackRowsB> CfgRef;
enum FwdTile { kTile64, kTile128, kTile256, kTile320, kTile384, kTile288, kTile352 };
struct TilePick {
  FwdTile tile = kTile384;
  int splits = 1;     // vocabulary ranges: one workgroup per (token tile, range), and the number of partials per token
  bool balanced = false;   // ranges of equally many rows instead of whole tiles (row_walk)
  bool tall = false;       // 256 columns: 320 rows in place of 256
};

// Most token rows per backward panel (bf16 path): 32 token tiles, for which the dH contraction has d / 256 x 32 tiles, whole
// rounds of 256 workgroups for d a multiple of 2048.  140897 tokens at d = 4096, V = 151936: 368.5 ms; panels of 6144 rows, which
// pay more for the read-add-write of dW, 377; of 24576 367, at twice the memory.  A smaller
// workspace makes panels smaller; a larger one buys more panel buffers (longer rollouts on the single
// sweep), never larger panels.
constexpr int64_t kPanelBf16 = 12288;
constexpr int64_t kPanelF32 = 4096;    // ... (fp32 path)
constexpr size_t kPartDhBytes = (size_t)32 << 20;    // partial sums of dH that a plan may have whatever the size of W
constexpr size_t kPartF32Bytes = (size_t)64 << 20;   // most partial results of an fp32 gradient contraction
constexpr int64_t kGroupScanLimit = (int64_t)1 << 32;   // n_seq * n_groups: every prompt's wavefront walks all rollouts
constexpr int kNumCU = 256;            // MI355X compute units (one workgroup of the dense kernels each: it fills the LDS)

static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Tile of the last panel's dH contraction, and workgroups per tile.
struct DhPick {
  bool small = false;
  int splits = 1;
};

// Tile and splits of k of an fp32 gradient contraction.
struct F32Pick {
  bool large = false;
  int splits = 1;
};

struct Plan {
  int64_t T = 0;
  int d = 0, V = 0, n_seq = 0, n_groups = 0, dtype = 0;
  bool bwd = false;
  bool rows = false;   // the kernels read W and H where they lie; else packed copies (and one of W^T) are made
  unsigned unaligned = 0;   // ... but these (Unaligned) are copied to an aligned place first
  TilePick fwd;        // tile and vocabulary splits of the scoring kernel (splits = soft-max partials per token)
  bool small_sweep = false, small_dw = false;   // 128 x 128 tiles (one panel, operands in place)
  int width = Cfg::BN;        // token columns of the large tiles of sweep, recompute and dH, and rows per block of packed G
  int n_vt = 0;        // vocabulary tiles of the sweep: row sums per token
  DhPick dh;           // the last panel's dH contraction
  bool grads_fused = false;   // ... shares its launch with dW's (bf16: both in 128 x 128 tiles; fp32: few workgroups)
  TilePick smp;        // ... of the sampling kernel (splits = (score, index) partials per token)
  int64_t Tp = 0;      // rows of one backward panel
  F32Pick f32_dh, f32_dw;   // tile and splits of the fp32 gradient contractions (of the largest panel)
  int wide_dh = 0, wide_dw = 0;   // ... or in 256 x 128 tiles with so many splits
  int64_t ldz = 0;     // fp32: row pitch of the transposed logits / dZ panel [V][ldz]
  int n_buf = 1;       // panel buffers of the single sweep (a ring; one if the batch is one panel)
  size_t size_G = 0, size_GT = 0;   // bytes of one panel buffer of each packed copy
  // packed-operand geometry (bf16 path): row tiles and k-blocks (strip pitches)
  int n_rt_v = 0, n_rt_d = 0, n_kt_d = 0, n_kt_v = 0, n_kt_g = 0, n_kt_t = 0;
  int n_rb_v = 0;      // 384-row blocks of a matrix whose rows are the vocabulary (G^T)
  int64_t n_rt_T = 0;  // 384-row token tiles of the whole batch
  size_t off_status = 0, off_partials = 0, off_fwd_partials = 0, off_upart = 0, off_zy = 0, off_lse2 = 0, off_diff = 0,
         off_coef = 0, off_delta = 0, off_cseq = 0, off_vstar = 0, off_gw = 0, off_omp = 0, off_inv = 0, off_Wp = 0,
         off_Hp = 0, off_Wc = 0, off_Hc = 0, off_WTp = 0, off_HTp = 0,
         off_part = 0, off_part_dw = 0, off_G = 0, off_GT = 0, off_ref2 = 0, off_spart = 0, total = 0;
  bool sweep = false;  // single-sweep loss path available (bf16 with backward)
};

// A call this small gains nothing from the sweep's saved pass; it takes the two-pass path, whose one-hot
// gradient entry is exact rather than exact up to the row-factor correction.
constexpr int64_t kSweepMinTokens = 64;

// Largest panel the plan may use: `max_panel_rows` <= 0 or above the library's size means that
// size; other values are rounded down to whole token tiles (bf16), with one tile as the least.
static int64_t panel_cap(int dtype, int64_t max_panel_rows) {
  const int64_t deflt = dtype == OAPL_BF16 ? kPanelBf16 : kPanelF32;
  if (max_panel_rows <= 0 || max_panel_rows > deflt) return deflt;
  if (dtype != OAPL_BF16) return max_panel_rows;
  return max_panel_rows < Cfg::BN ? Cfg::BN : max_panel_rows / Cfg::BN * Cfg::BN;
}

// Where reading W and H in place beats packing them first.  Packing moves 4 bytes per weight at ~5.3 TB/s (0.48 ms at
// d = 4096, V = 151936; with gradients there are two copies of W to save, W^T: 0.46 ms). Scoring in place / packed, ms: rows of
// whole 128-byte lines, d = 4096, 4000 tokens 3.54 / 4.03, 8000 7.15 / 7.45, 11000 9.91 / 10.13, 20000 17.93 / 17.94; others, d
// = 4104, 2000 2.15 / 2.47, 4000 4.04 / 4.09, 6000 6.23 / 5.77. Loss calls at d = 4096: 1003 tokens 3.47 / 4.42, 4000 11.86 /
// 12.70, 8000 22.4 / 23.0, 12288 32.5 / 33.0; d = 4104, 4000 12.7 / 13.1. (Between 8192 and about 20000 tokens packing costs
// whole-line rows up to 2 %: the line is older than the present main loop.)
static bool rows_pay(int64_t T, int d) {
  if (d % kPackK != 0) return T <= 4096;
  return T <= 8192;
}

// Vocabulary splits of the streaming kernels for a tile: one workgroup per (token tile, split), one workgroup per CU
// at a time.  Takes the count with the least time in the last-finishing CU: rounds of workgroups x tiles each walks,
// plus a twentieth of a tile per walk.  Short walks cost next to nothing (20000 tokens at d = 4096, patches of eight
// token tiles: 18.1 / 18.2 / 18.6 ms for walks of 3 / 2 / 1 tiles) while the long ones of neighbouring workgroups
// drift apart and share less in the L2 (18.4 / 19.0 ms for walks of 6 / 26), so the count is free to fill the last round.
template <class C>
static TilePick pick_splits(FwdTile tile, int64_t T, int V, int max_splits, double tile_cost = 1.0,
                            double* time_out = nullptr) {
  const int64_t tiles = (T + C::BN - 1) / C::BN;
  const int MT = (V + C::BM - 1) / C::BM;
  const int most = tiles <= 64 ? kNumCU : 64;   // bounds the partials: 12 bytes per token and split
  TilePick best{tile, 1};
  double best_time = 1e300;
  for (int c = 1; c <= most && c <= MT && c <= max_splits; ++c) {
    const double rounds = (double)((tiles * c + kNumCU - 1) / kNumCU);
    const double time = rounds * ((MT + c - 1) / c + 0.05) * tile_cost;
    if (time < best_time - 1e-9) { best_time = time; best.splits = c; }
  }
  if (time_out) *time_out = best_time;
  return best;
}

// Tile and splits over row-major operands.  Up to 256 tokens the call is bound by reading W, and as many workgroups as the CUs
// hold at once share its rows evenly, but for ranges in which a W that is not read once (once_pays) is read faster in whole tiles.
// Whole / even, us, scoring and sampling:
//   64 tokens: even pays only where whole tiles are 3.7 .. 4 per CU, so that their second round is a third full (even / whole over
//     d = 256 .. 4104, V = 101000 1.00 .. 1.11, 110000 0.96 .. 1.10, 122000 0.89 .. 1.00, 130000 0.90 .. 1.01, 140000 0.98 ..
//     1.06): d = 1000, V = 104857 53.4 / 54.6, 47.6 / 50.8; 125829 56.3 / 54.4, 52.2 / 52.2; 151936 75 / 78, 71 / 74.  Up to three
//     per CU there is no difference.  16 tokens: also where they are 3.1 .. 4.3 per CU (V = 101000 0.98 .. 1.02, 107000 0.92 ..
//     1.00, 122000 0.87 .. 0.93, 140000 0.96 .. 1.04, 151936 0.95 .. 1.04), unless W is small (d = 320, V = 109000 22 / 23.4; d =
//     256 to 1.09).
//   128 tokens: rows that are not whole 128-byte lines and W about as large as the memory-side cache, which then keeps more of what
//     is read in order: d = 904, V = 142671 (246 MiB) 74 / 83 on one box, 66.9 / 65.9 on another; d = 1000, V = 134217 (256) 75.6 /
//     85.2, 72.3 / 83.3; V = 140509 (268) 94.7 / 88.0, 94.6 / 87.2 (whole lines: d = 960, V = 139810 (256) 63.2 / 64.4, 65.0 /
//     64.8; d = 1088 57.8 / 56.4, 58.6 / 54.0).  And sampling on small hidden sizes, where drawing for the rows that shares leave
//     empty shows: V = 83200 (2.5 tiles per CU), d = 64 16.5 / 18.5, 272 23.0 / 24.4, 320 22.3 / 23.3, 448 28.5 / 27.2; V = 100400
//     (3.1) d = 64 22.9 / 21.1, 272 30.3 / 28.0.
//   256 tokens: W in that cache and a CU's rows two tiles that even walks leave two thirds full: d = 768, V = 84900 45.4 / 48.4,
//     54.6 / 57.3; d = 512, V = 109300 39.0 / 39.7, 48.1 / 48.7, 115400 41.5 / 40.6, 51.7 / 49.6; d = 1152, V = 97000 (213 MiB)
//     63.0 / 67.4, 71.9 / 75.3; d = 1472, V = 91000 (255) 1.02 times; rows that are not whole lines, d = 648, V = 106000 (131 MiB)
//     0.98, d = 872, V = 91000 (151) 1.00, d = 1000, V = 114000 (217) 69.8 / 69.1, d = 1480, V = 91000 (257) 1.13.
// Beyond, the wide tile is the cheapest per column and a narrower one pads fewer columns: the
// time of one 256-row tile of 256 / 288 / 320 / 352 / 384 columns is in the ratio of kScoreCost (it scales with d), in sampling,
// whose epilogue draws for every logit, of kSampleCost (8064 tokens, all rounds full, d = 4096 101 / 116 / 133 / 139 / 155 us, d =
// 2048 55 / 63 / 71 / 75 / 85; 384 columns with 32 registers in scratch). Scoring with 256, 320 and 384 alone / all five: 350
// tokens at d = 4096 433 / 403 us, 700 725 / 674, 777 825 / 779, 1003 996 / 941, 1400 1412 / 1292, 2500 and more the same.
// Sampling with 256 alone / all five, V = 151936: d = 4096, 300 tokens 563 / 396 us, 384 551 / 460, 600 775 / 656, 1003 1106 /
// 1009; d = 2048 292 / 230, 303 / 267, 421 / 364, 586 / 550.
struct TileCosts {
  double w256, w288, w320, w352, w384;
};
constexpr int64_t kFewest = 16, kWhole16 = 96;                // tokens; MiB
constexpr int kEvenFrom16 = 794, kEvenTo16 = 1100;            // tiles of 128 rows
constexpr int kEvenFrom64 = 947, kEvenTo64 = 4 * kNumCU;      // tiles of 128 rows
constexpr int64_t kWholeFrom128 = 244, kWholeTo128 = 264;     // MiB
constexpr int kWholeHidden128 = 384;
constexpr int64_t kWhole256 = 160, kWholeLines256 = 250;      // MiB
constexpr int kEvenRows256 = 448;                             // rows per CU
constexpr TileCosts kScoreCost{105.0, 115.5, 126.0, 138.0, 150.0}, kSampleCost{100.0, 115.0, 128.0, 137.0, 152.0};
static TilePick pick_tile(int64_t T, int d, int V, int max_splits, bool sampling) {
  const TileCosts& cost = sampling ? kSampleCost : kScoreCost;
  const int64_t bytes = (int64_t)V * d * 2, MiB = 1 << 20;
  const int tiles = (V + Cfg64::BM - 1) / Cfg64::BM;      // of 128 rows
  const bool once = once_pays(T, V, d), lines = d % kPackK == 0;     // rows of whole 128-byte lines
  auto even = [&](FwdTile tile, int per_cu, int rows) {   // a share per workgroup, at most one per tile of `rows` rows
    const int n = (V + rows - 1) / rows, most = per_cu * kNumCU < max_splits ? per_cu * kNumCU : max_splits;
    return TilePick{tile, n < most ? n : most, true};
  };
  auto whole = [&](FwdTile tile) { return TilePick{tile, tiles < max_splits ? tiles : max_splits}; };
  if (T <= Cfg64::BN) {
    const bool few = T <= kFewest && tiles > kEvenFrom16 && tiles < kEvenTo16 && bytes > kWhole16 * MiB;
    return once || few || (tiles > kEvenFrom64 && tiles < kEvenTo64) ? even(kTile64, 3, Cfg64::BM) : whole(kTile64);
  }
  if (T <= Cfg128::BN) {
    const bool cached = !lines && bytes > kWholeFrom128 * MiB && bytes <= kWholeTo128 * MiB;
    const bool draws = sampling && d <= kWholeHidden128 && tiles > 2 * kNumCU && tiles <= 3 * kNumCU;
    return once || !(cached || draws) ? even(kTile128, 2, Cfg128::BM) : whole(kTile128);
  }
  if (T <= Cfg256::BN) {
    // the least tile rows: of 256, or of 320 where they are fewer
    TilePick pick = even(kTile256, 1, Cfg256::BM);
    const int rows = (int)round_up((V + pick.splits - 1) / pick.splits, 16);
    const int flat = (rows + Cfg256::BM - 1) / Cfg256::BM, tall = (rows + Cfg256Tall::BM - 1) / Cfg256Tall::BM;
    pick.tall = tall * Cfg256Tall::BM < flat * Cfg256::BM;
    if (!once && !pick.tall && bytes <= (lines ? kWholeLines256 : kWhole256) * MiB && rows > Cfg256Tall::BM && rows <= kEvenRows256)
      return pick_splits<Cfg256>(kTile256, T, V, max_splits);
    return pick;
  }
  double best_time, time;
  TilePick best = pick_splits<Cfg256>(kTile256, T, V, max_splits, cost.w256, &best_time);
  auto consider = [&](const TilePick& pick) {     // ties go to the wider tile
    if (time <= best_time) { best = pick; best_time = time; }
  };
  consider(pick_splits<Cfg288>(kTile288, T, V, max_splits, cost.w288, &time));
  consider(pick_splits<Cfg320>(kTile320, T, V, max_splits, cost.w320, &time));
  consider(pick_splits<Cfg352>(kTile352, T, V, max_splits, cost.w352, &time));
  consider(pick_splits<Cfg>(kTile384, T, V, max_splits, cost.w384, &time));
  return best;
}

static TilePick pick_fwd(bool rows, int64_t T, int d, int V, int max_splits) {
  return rows ? pick_tile(T, d, V, max_splits, false) : pick_splits<Cfg>(kTile384, T, V, max_splits);
}

// ... of the sampling kernel: over packed operands 256 or 384 columns (V = 151936, 256 alone / both: 12288 tokens at d = 4096 12.7
// / 11.3 ms, 32768 35.5 / 31.9; 16384 at d = 2048 8.16 in tiles of 256, 8.54 in tiles of 384).
static TilePick pick_sample(bool rows, int64_t T, int d, int V, int max_splits) {
  if (rows) return pick_tile(T, d, V, max_splits, true);
  double narrow_time, wide_time;
  const TilePick narrow = pick_splits<Cfg256>(kTile256, T, V, max_splits, kSampleCost.w256, &narrow_time);
  const TilePick wide = pick_splits<Cfg>(kTile384, T, V, max_splits, kSampleCost.w384, &wide_time);
  return narrow_time < wide_time ? narrow : wide;
}

// Time of `tiles` tiles with nk k-blocks each, in k-blocks of a 256 x 384 tile (1.5 .. 2 us): rounds of workgroups, with
// some k-blocks each for filling the ring and the epilogue.  128 x 128 tiles run two per CU; what a pair of their k-blocks
// costs depends on how the kernel's operands reach the LDS (packed blocks least, a transposed read of W most):
//   d = 4096, small / large tiles   V = 8192, 1000 tokens   V = 32000, 1000   V = 151936, 300 / 1000
//   sweep                            67 / 138 us             304 / 294         512 / 483, 1330 / 1103
//   dH                               93 /  77                316 / 234         577 / 352, 1383 / 1034
//   dW                               77 /  97                350 / 284         877 / 694, 1710 / 1223
// and at d = 256, V = 1544, 1000 tokens 14 / 29, 12 / 22, 17 / 36 us (launches of their own; dH and dW of small tiles share
// one, 16 us). Against the best of five fixed choices over 44 shapes the chosen call is within 4 % but for four: 1000 tokens at
// d = 1024, V = 32000 (339 us, all in small tiles 294), 3000 at d = 4096, V = 1544 (240 / 223) and V = 8192 (668 / 625), 100 at
// d = 4096, V = 32000 (354 / 332): the rates do not know the launch that dH and dW of small tiles share.
struct SmallRate {
  double pair, alone;   // a k-block of two workgroups of one CU; of one that has it to itself
  int start;
};
constexpr SmallRate kSmallSweep{0.7, 0.45, 5}, kSmallDh{0.95, 0.5, 5}, kSmallDw{0.48, 0.4, 8};
static double large_time(int64_t tiles, int nk) { return (double)((tiles + kNumCU - 1) / kNumCU) * (nk + 10); }
static double small_time(const SmallRate& r, int64_t tiles, int nk) {
  const int64_t full = tiles / (2 * kNumCU), rest = tiles - full * 2 * kNumCU;
  return ((double)full * r.pair + (rest > kNumCU ? r.pair : rest > 0 ? r.alone : 0.0)) * (nk + r.start);
}
template <class C>
static int64_t tile_count(int64_t M, int64_t N) {
  return ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
}
// An M x N contraction of nk k-blocks is faster in small tiles.
static bool small_tiles_pay(const SmallRate& r, int64_t M, int64_t N, int nk) {
  return small_time(r, tile_count<CfgSmall>(M, N), nk) < large_time(tile_count<Cfg>(M, N), nk);
}

// Tile and workgroups per tile of the dH contraction of nv tokens.  Its tiles are few and long (`nk` k-blocks each): the
// pick minimises their time plus the partial sums' way through memory (8 bytes per element and split).  Whole loss calls at
// V = 151936, one workgroup per tile / the count chosen: 1003 tokens, d = 4096 3.99 / 3.47 ms (five splits);
// 6007 tokens, d = 2048 10.77 / 8.80 ms (two); 30011 tokens at d = 5120, whose last panel has 1211, 107.3 / 104.6 ms.
template <class Time>
static double pick_dh_splits(Time&& time_of, int64_t tiles, int64_t nv, int d, int nk, size_t scratch, int& splits) {
  double best = 1e300;
  for (int s = 1; s <= 64 && (s == 1 || (s * 4 <= nk && (size_t)s * nv * d * 4 <= scratch)); ++s) {
    const double time = time_of(tiles * s, (nk + s - 1) / s) + (s > 1 ? 5 + 1.2e-6 * (double)s * nv * d : 0.0);
    if (time < best - 1e-9) { best = time; splits = s; }
  }
  return best;
}
static DhPick pick_dh(int64_t nv, int d, int nk, bool allow_small, size_t scratch, double* time_out = nullptr) {
  DhPick large, small{true, 1};
  const double a = pick_dh_splits(large_time, tile_count<Cfg>(d, nv), nv, d, nk, scratch, large.splits);
  const double b = !allow_small ? 1e300 : pick_dh_splits([](int64_t tiles, int k) { return small_time(kSmallDh, tiles, k); },
                                                         tile_count<CfgSmall>(d, nv), nv, d, nk, scratch, small.splits);
  if (time_out) *time_out = a < b ? a : b;
  return b < a - 1e-9 ? small : large;
}

// Large tiles of one panel's sweep and dH (operands in place) may be narrower than 384 columns where that pads fewer tokens. A
// k-block of theirs takes kLossScale of one of 384 columns': narrow tiles read W more often and gain less than their columns.
// The ratios come from 133 shapes (T = 80 .. 3000, d = 1000 .. 5120, V = 32000 .. 151936), each timed at every width. 384 / the
// width chosen, us, V = 151936: d = 4096, 200 tokens 1481 / 1400 (256), 300 1595 / 1541 (320), 400 2152 / 1938 (256), 777 3150 /
// 2813 (288), 1003 3469 / 3379 (352); d = 2048, 800 1748 / 1535 (288).  1003 tokens at d = 1800, V = 100000, 384 / 352 / 256: 1317
// / 1298 / 1377. Where the sweep runs in small tiles all widths lose (100 tokens at d = 4096: 1175 / 1275), so those calls keep
// them. Rounds are not as sharp as the model has them (a last one of few tiles is short), so a gain of under 5 % is not taken: of
// 279 shapes with T up to 8192 and any d and V that a narrower width promises to serve better, 31 of under 5 % came out at 1.00
// times on average and up to 1.19 (d = 1624, V = 12314, 3678 tokens 493 / 588), the others at 0.95, 1.01 at the most once dH's
// small tiles, which are better than their model where there are many, are kept (d = 680, V = 21976, 3230 tokens 456 / 512; up to
// 917 tokens 0.86 .. 0.99).
constexpr double kNarrowGain = 0.95;
constexpr int64_t kNarrowSmallDh = 1024;
struct LossScale { int width; double scale; };
constexpr LossScale kLossScale[] = {{256, 0.80}, {288, 0.83}, {320, 0.86}, {352, 0.93}};
static int pick_width(int64_t T, int d, int V, double now, size_t scratch, DhPick& dh) {
  const int64_t mt_v = (V + Cfg::BM - 1) / Cfg::BM, mt_d = (d + Cfg::BM - 1) / Cfg::BM;
  const int nk_d = (d + kPackK - 1) / kPackK, nk_v = (V + kPackK - 1) / kPackK;
  int best = Cfg::BN;
  if (dh.small && T > kNarrowSmallDh) return best;
  now *= kNarrowGain;
  for (const LossScale& c : kLossScale) {
    const int64_t tiles = (T + c.width - 1) / c.width, columns = tiles * c.width;
    // fewer columns than 384 would take (which the panel has room for), and all of the token blocks that dW walks
    if (columns >= round_up(T, Cfg::BN) || columns < round_up(T, kPackK)) continue;
    DhPick pick;
    const double dh_time = pick_dh_splits(large_time, mt_d * tiles, T, d, nk_v, scratch, pick.splits);
    const double time = c.scale * (large_time(mt_v * tiles, nk_d) + dh_time);
    if (time < now - 1e-9) { now = time; best = c.width; dh = pick; }
  }
  return best;
}

// In a launch that dH shares with dW, dH's walks (nk_v k-blocks) need no split while they end with dW's (nk_t), which saves the
// partial sums and a launch. Whole calls split / not, us, d = 256 unless named: nk_v and nk_t 21, 27 63.7 / 60.4; 53, 107 131 /
// 121; 32, 32 (d = 512) 77 / 74; 25, 16 55.4 / 57.4; 29, 17 (d = 80) 51.6 / 57.4; 46, 24 63 / 76; 75, 71 111 / 110; 92, 77 128
// / 131; 126, 113 196 / 184; 144, 125 267 / 247; 166, 112 285 / 297; 235, 125 363 / 439.
static bool dh_hides_behind_dw(int nk_v, int nk_t) { return nk_v <= nk_t + nk_t / 8 + 2; }

// Tile of 128 x 128 or 64 x 64 and splits of an M x N x K fp32 contraction: the least time of the last-finishing CU in clocks, 128
// per k for a tile of 128 x 128 and 40 for one of 64 x 64 that has the CU to itself, 2000 for a workgroup to start and
// store; partial results cost 8 bytes per element and split at 1700 bytes per clock, and a launch (5000).  The figures are those
// of fp32 multiplications, in whose place whole calls from parts take 0.63 .. 1.02 times as long (gemm_f32.hip.h): what it picks
// is then no worse than it was, but not always the best.  `scratch` bounds the partial results.
static F32Pick pick_f32(int64_t M, int64_t N, int64_t K, int max_splits, size_t scratch) {
  F32Pick best;
  double best_time = 1e300;
  for (int large = 0; large < 2; ++large) {
    const int64_t tile = large ? F32Large::BM : F32Small::BM, bk = large ? F32Large::BK : F32Small::BK;
    const int64_t tiles = ((M + tile - 1) / tile) * ((N + tile - 1) / tile);
    for (int s = 1; s <= 64 && s <= max_splits && (s == 1 || (s * 2 * bk <= K && (size_t)(s * M * N) * 4 <= scratch)); ++s) {
      const double rounds = (double)((tiles * s + kNumCU - 1) / kNumCU);
      const double time = rounds * ((double)((K + s - 1) / s) * (large ? 128.0 : 40.0) + 2000.0) +
                          (s > 1 ? 5000.0 + (double)s * M * N * 8.0 / 1700.0 : 0.0);
      if (time < best_time - 1e-9) { best_time = time; best.large = large != 0; best.splits = s; }
    }
  }
  return best;
}

// ... in 256 x 128 tiles, a workgroup per CU: in how many splits, or 0 where the smaller tiles are the better. us for a CU's
// workgroups and a stage of 32 k: 256 x 128 3.1 each; 128 x 128 2.7 alone, 3.8 two; 64 x 64 1.3 alone, 0.55 each and 0.4 several.
// dH of 1501 tokens at d = 768, V = 8192 in seven splits 147 (128 x 128) / 127 us, dW 164 in two with their sum / 133; dH of 1300
// tokens at V = 8065 332 (64 x 64, one split) / 139; of 700 at d = 300, V = 8000 in 16 splits 43 (64 x 64) / 55.
static int wide_splits_f32(const F32Pick& pick, int64_t M, int64_t N, int64_t K, int max_splits, size_t scratch) {
  auto tiles = [&](int64_t bm, int64_t bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn); };
  const int64_t stages = (K + F32Wide::BK - 1) / F32Wide::BK;
  auto partials = [&](int s) { return s > 1 ? 2.5 + (double)s * M * N * 8.0 / 3.7e6 : 0.0; };
  const int64_t n = tiles(pick.large ? F32Large::BM : F32Small::BM, pick.large ? F32Large::BN : F32Small::BN) * pick.splits;
  const int64_t per_cu = (n + kNumCU - 1) / kNumCU;
  const double stage = pick.large ? 3.8 * (double)(per_cu / 2) + 2.7 * (double)(per_cu % 2)
                                  : per_cu == 1 ? 1.3 : 0.55 * (double)per_cu + 0.4;
  double now = stage * (double)stages / pick.splits + 6.0 + partials(pick.splits);
  int best = 0;
  for (int s = 1; s <= max_splits && s <= 64 && (s == 1 || (2 * s <= stages && (size_t)(s * M * N) * 4 <= scratch)); ++s) {
    const int64_t rounds = (tiles(F32Wide::BM, F32Wide::BN) * s + kNumCU - 1) / kNumCU;
    const double time = (double)rounds * (3.1 * (double)stages / s + 6.0) + partials(s);
    if (time < now - 1e-9) { now = time; best = s; }
  }
  return best;
}

static int64_t f32_groups(const F32Pick& pick, int64_t M, int64_t N) {
  const int64_t tile = pick.large ? F32Large::BM : F32Small::BM;
  return ((M + tile - 1) / tile) * ((N + tile - 1) / tile) * pick.splits;
}
// fp32 gradient contractions share a launch up to this many workgroups; beyond, each may have the tiles that suit it
// (wide_splits_f32).  Whole calls, two launches / one, us: tokens, d, V (workgroups) 256, 64, 1024 (128) 41 / 33; 939, 129, 1398
// (423) 78 / 57; 700, 300, 3000 (455) 104 / 87; 283, 714, 1376 (504) 95 / 79; 362, 752, 2503 (696) 108 / 103; 800, 768, 3000 (816)
// 159 / 164; 1501, 768, 8192 (1272) 494 / 550.  The count alone does not tell everything: between 512 and 768 calls of few tokens
// lose a seventh apart (177, 654, 2306 92 / 79), some of many gain a fifth (1959, 751, 4318 (684) 417 / 509; 1300, 600, 6000 (730)
// 344 / 392; 1047, 460, 4490 (684) 188 / 188); with the line at 512 160 calls took 1.01 times as long on average.
constexpr int64_t kSharedGroupsF32 = 3 * kNumCU;

// bf16 operands that are not 16-byte aligned.  The 16-byte direct-to-LDS loads of the in-place kernels want that; the packing
// and gathering kernels use ordinary loads, which take any address.  Such an operand is copied first and the call goes on
// as any other (W at d = 4096, V = 151936: 0.46 ms; sampling 64 tokens takes 0.69 ms, 1.68 when it packed every operand).
enum Unaligned { kUnalignedW = 1, kUnalignedH = 2, kUnalignedAny = 3 };
static unsigned unaligned_operands(int dtype, const void* H, const void* W) {
  if (dtype != OAPL_BF16) return 0;
  return (((uintptr_t)W & 15) != 0 ? kUnalignedW : 0) | (((uintptr_t)H & 15) != 0 ? kUnalignedH : 0);
}

// `unaligned`: which operands the plan has copies of (Unaligned; the workspace sizes that the library reports have both).
// `panel_buffers`: how many panels the single sweep keeps before their gradient contractions run
// (<= 0: two, the least for a batch of several panels; never more than the batch has panels).
// `max_splits`: most vocabulary splits of the streaming kernels of a call without gradients, most splits of k of the gradient
// contractions of one with gradients.  One gives the smallest workspace (see fit_splits); short of kAnySplits the fp32
// gradient contractions have one space for partial results between them, and a launch each.
constexpr int kAnySplits = 1 << 30;
static bool make_plan(Plan& p, int64_t T, int d, int V, int n_seq, int n_groups, int dtype, bool bwd, unsigned unaligned,
                      int64_t max_panel_rows = 0, int64_t panel_buffers = 0, int64_t exact_panel_rows = 0,
                      int max_splits = kAnySplits) {
  if (T < 0 || d < 1 || V < 1 || n_seq < 0 || n_groups < 1) return false;
  if (dtype != OAPL_F32 && dtype != OAPL_BF16) return false;
  if (dtype == OAPL_BF16 && (d % 8) != 0) return false;
  // a packed row-tile strip (K / 64 blocks of 32 or 48 KiB) must stay below 2 GiB for 32-bit buffer offsets,
  // and the packing kernels index token tiles with gridDim.y
  if ((int64_t)d > (1 << 21) || (int64_t)V > (1 << 21)) return false;
  if (dtype == OAPL_BF16 && T > (int64_t)65535 * 256) return false;
  // the fp32 kernels' bytes from a tile's first row to its last (255 rows of dZ^T, at most T long) and their tiles are 32-bit
  if (dtype == OAPL_F32 && T > (int64_t)65535 * 64) return false;
  if ((int64_t)n_seq * n_groups > kGroupScanLimit) return false;
  const int64_t cap = panel_cap(dtype, max_panel_rows);
  p = Plan{};
  p.T = T; p.d = d; p.V = V; p.n_seq = n_seq; p.n_groups = n_groups; p.dtype = dtype; p.bwd = bwd;
  if (dtype == OAPL_BF16) {
    const int64_t n_tiles = (T + Cfg::BN - 1) / Cfg::BN;
    const int MT = (V + Cfg::BM - 1) / Cfg::BM;
    p.rows = rows_pay(T, d);
    p.unaligned = p.rows ? unaligned : 0;
    if (!bwd) p.fwd = pick_fwd(p.rows, T, d, V, max_splits);
    p.smp = pick_sample(p.rows, T, d, V, max_splits);
    // Panel size: a multiple of the token tile, at most `cap` rows.  One panel if T fits; otherwise
    // the size (between half the cap and the cap) that costs the fewest rounds of kNumCU workgroups in
    // the dH contraction -- its tiles (d / 256 x panel rows / 384, each K = V long) are few and long, so
    // a partly filled last round is expensive -- plus a charge per panel for the fp32 read-add-write
    // pass over dW.  Ties go to the larger panel (longer rollouts fit the single sweep).
    if (T <= cap) {
      p.Tp = round_up(T > 0 ? T : 1, Cfg::BN);
    } else if (exact_panel_rows > 0) {   // a size an earlier plan for the same shapes chose
      p.Tp = exact_panel_rows;
    } else {
      const int64_t mtd = (d + Cfg::BM - 1) / Cfg::BM;
      const int64_t k_max = cap / Cfg::BN;
      double best = 1e300;
      for (int64_t k = k_max; k >= (k_max + 1) / 2; --k) {
        const int64_t rows = k * Cfg::BN;
        const int64_t full = T / rows, rest = T - full * rows;
        const int64_t rounds_full = (mtd * k + kNumCU - 1) / kNumCU;
        const int64_t rounds_rest = (mtd * ((rest + Cfg::BN - 1) / Cfg::BN) + kNumCU - 1) / kNumCU;
        const double cost = (double)(full * rounds_full + rounds_rest) + 0.35 * (double)(full + (rest > 0 ? 1 : 0));
        if (cost < best - 1e-9) { best = cost; p.Tp = rows; }
      }
    }
    p.n_rt_v = MT;
    p.n_rb_v = (int)(round_up((int64_t)MT * Cfg::BM, Cfg::BN) / Cfg::BN);
    p.n_rt_d = (d + Cfg::BM - 1) / Cfg::BM;
    p.n_rt_T = n_tiles > 0 ? n_tiles : 1;
    p.n_kt_d = (d + kPackK - 1) / kPackK;
    p.n_kt_v = (V + kPackK - 1) / kPackK;            // W^T strips: exactly the k-blocks the dH contraction walks
    p.n_kt_g = MT * (Cfg::BM / kPackK);              // G strips: whole vocabulary tiles
    p.n_kt_t = (int)(p.Tp / kPackK);                 // strips whose k index is the panel token
  } else {
    p.fwd.splits = p.smp.splits = (V + 63) / 64;
    p.Tp = T < cap ? (T > 0 ? T : 1) : cap;
  }
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += (bytes + 255) / 256 * 256; return at; };
  const size_t Tn = (size_t)(T > 0 ? T : 1);
  p.off_status = take(kStatusWords * 4);
  // (a call with gradients neither samples nor returns entropies; its bf16 scoring pass, which comes before a panel is filled
  // or after all are consumed, has its partials in the panel buffers, see below)
  p.off_partials = take(Tn * (size_t)(bwd || p.fwd.splits > p.smp.splits ? p.fwd.splits : p.smp.splits) * 8);
  p.off_fwd_partials = p.off_partials;
  p.off_upart = take(bwd ? 0 : Tn * (size_t)p.fwd.splits * 4);
  p.off_zy = take(Tn * 4);
  p.off_lse2 = take(Tn * 4);
  p.off_diff = take(Tn * 8);
  p.off_coef = take(Tn * 4);
  p.off_omp = take(Tn * 4);
  p.off_inv = take(Tn * 4);
  p.off_delta = take((size_t)(n_seq > 0 ? n_seq : 1) * 8);
  p.off_cseq = take((size_t)(n_seq > 0 ? n_seq : 1) * 4);
  p.off_vstar = take((size_t)n_groups * 16);
  p.off_gw = take((size_t)((n_seq > 0 ? n_seq : 1) + n_groups) * 8);
  if (dtype == OAPL_BF16 && !p.rows) {
    p.off_Wp = take((size_t)p.n_rt_v * p.n_kt_d * kPackBlockBytesA);
    {  // packed H: blocks of 384 rows, or of 256 for sampling in tiles of 256 columns (whichever is larger)
      const size_t a = (size_t)p.n_rt_T * p.n_kt_d * kPackBlockBytesB;
      const size_t b = (size_t)((T + Cfg256::BN - 1) / Cfg256::BN > 0 ? (T + Cfg256::BN - 1) / Cfg256::BN : 1) * p.n_kt_d *
                       Cfg256::STAGE_B;
      p.off_Hp = take(a > b ? a : b);
    }
  }
  if (p.unaligned & kUnalignedW) p.off_Wc = take((size_t)V * d * 2);
  if (p.unaligned & kUnalignedH) p.off_Hc = take(Tn * d * 2);
  if (bwd) {
    if (dtype == OAPL_BF16) {
      // the last panel's partial sums of dH: in the packed copy of W, which is dead by then, or in a space of their own
      const int64_t last = T > 0 ? T - (T - 1) / p.Tp * p.Tp : 0;
      const size_t packed_w = (size_t)p.n_rt_v * p.n_kt_d * kPackBlockBytesA;
      const bool lean = max_splits == 1;
      const size_t part_bytes = lean ? 0 : (packed_w > kPartDhBytes ? packed_w : kPartDhBytes);
      double dh_time = 0;
      if (!p.rows) p.dh = pick_dh(last, d, p.n_kt_v, false, packed_w);
      else p.dh = pick_dh(last, d, p.n_kt_v, true, part_bytes, &dh_time);
      p.small_dw = p.rows && T <= p.Tp && small_tiles_pay(kSmallDw, d, V, (int)((T + kPackK - 1) / kPackK));
      p.grads_fused = p.small_dw && p.dh.small;
      if (p.grads_fused && dh_hides_behind_dw(p.n_kt_v, (int)((T + kPackK - 1) / kPackK))) p.dh.splits = 1;
      p.small_sweep = p.rows && T <= p.Tp && !lean && small_tiles_pay(kSmallSweep, V, T, p.n_kt_d);
      if (p.rows && T > 0 && T <= p.Tp && !lean && !p.small_sweep && !p.grads_fused)
        p.width = pick_width(T, d, V, large_time(tile_count<Cfg>(V, T), p.n_kt_d) + dh_time, part_bytes, p.dh);
      p.off_part = p.rows && p.dh.splits > 1 ? take((size_t)p.dh.splits * last * d * 4) : p.off_Wp;
      p.n_vt = p.small_sweep ? (V + CfgSmall::BM - 1) / CfgSmall::BM : p.n_rt_v;
      if (!p.rows) p.off_WTp = take((size_t)p.n_rt_d * p.n_kt_v * kPackBlockBytesA);
      p.off_HTp = take((size_t)p.n_rt_d * p.n_kt_t * kPackBlockBytesA);
      // Panel buffers, both packed copies.  The single sweep keeps a ring of them: a panel's gradient
      // contractions run once every rollout that touches it is scored, i.e. n_buf - 1 panels later, so
      // rollouts of up to (n_buf - 1) panels are served (the two-pass schedule uses the first buffer only).
      const int64_t n_panels = (T + p.Tp - 1) / p.Tp;
      p.n_buf = (int)(n_panels <= 1 ? 1 : (panel_buffers < 2 ? 2 : (panel_buffers > n_panels ? n_panels : panel_buffers)));
      p.size_G = ((size_t)(p.Tp / Cfg::BN) * p.n_kt_g * kPackBlockBytesB + 255) / 256 * 256;
      p.size_GT = ((size_t)p.n_rb_v * p.n_kt_t * kPackBlockBytesB + 255) / 256 * 256;
      p.off_G = take(p.size_G * p.n_buf);
      p.off_GT = take(p.size_GT * p.n_buf);
      // as many vocabulary splits as that space takes, so small panels do not leave the scoring pass short of workgroups
      // (two passes over 16411 tokens at d = 4096 in panels of 6144, with the 32 x 32 x 16 loop: 66 ms, 113 ms with one split)
      const size_t room = (p.size_G + p.size_GT) * p.n_buf / (Tn * 8);
      p.fwd = pick_fwd(p.rows, T, d, V, room < (size_t)kAnySplits ? (room > 1 ? (int)room : 1) : kAnySplits);
      if (p.fwd.splits > 1) p.off_fwd_partials = p.off_G;
      // single-sweep path: reference exponents and per-vocabulary-tile row sums of one panel
      p.sweep = true;
      p.off_ref2 = take(Tn * 4);
      p.off_spart = take((size_t)p.n_vt * (size_t)p.Tp * 4);
    } else {
      p.ldz = max_splits > 1 ? round_up(p.Tp, 4) : p.Tp;    // a multiple of 4 floats lets the contractions load 16 bytes
      p.off_G = take((size_t)p.ldz * V * 4);
      const size_t scratch = T <= p.Tp ? kPartF32Bytes : 0;   // panels of a longer batch are rows enough for whole tiles
      p.f32_dh = pick_f32(p.Tp, d, V, max_splits, scratch);
      p.f32_dw = pick_f32(V, d, p.Tp, max_splits, scratch);
      // few workgroups share a launch, and then both have their partial results at once
      p.grads_fused = T > 0 && T <= p.Tp && max_splits == kAnySplits &&
                      f32_groups(p.f32_dh, T, d) + f32_groups(p.f32_dw, V, d) <= kSharedGroupsF32;
      if (!p.grads_fused) {
        p.wide_dh = wide_splits_f32(p.f32_dh, p.Tp, d, V, max_splits, scratch);
        p.wide_dw = wide_splits_f32(p.f32_dw, V, d, p.Tp, max_splits, scratch);
      }
      const int s_dh = p.wide_dh ? p.wide_dh : p.f32_dh.splits, s_dw = p.wide_dw ? p.wide_dw : p.f32_dw.splits;
      const size_t dh = s_dh > 1 ? (size_t)s_dh * p.Tp * d * 4 : 0, dw = s_dw > 1 ? (size_t)s_dw * V * d * 4 : 0;
      if (p.grads_fused) {
        p.off_part = take(dh);
        p.off_part_dw = take(dw);
      } else {
        p.off_part = p.off_part_dw = take(dh > dw ? dh : dw);
      }
    }
  }
  p.total = o;
  return true;
}

static inline unsigned grid1d(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// Optional per-kernel timing of the four dense kernels: when switched on, every
// launch is bracketed by a pair of events recorded on the launch stream itself.
enum DenseKernel { kFwdLse = 0, kBwdDz = 1, kBwdDh = 2, kBwdDw = 3, kFwdSample = 4, kSweep = 5, kNumDense = 6 };
struct TimingState {
  std::mutex mu;
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[kNumDense];
};
static TimingState& timing() {
  static TimingState t;
  return t;
}
struct ScopedKernelTimer {
  hipStream_t st;
  hipEvent_t stop = nullptr;
  ScopedKernelTimer(int which, hipStream_t s, bool enabled = true) : st(s) {
    if (!enabled) return;
    TimingState& t = timing();
    std::lock_guard<std::mutex> g(t.mu);
    if (!t.on) return;
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return;
    if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return; }
    (void)hipEventRecord(a, st);
    stop = b;
    t.ev[which].emplace_back(a, b);
  }
  ~ScopedKernelTimer() {
    if (stop) (void)hipEventRecord(stop, st);
  }
};

#define OAPL_LAUNCH_CHECK()                                   \
  do {                                                        \
    if (hipGetLastError() != hipSuccess) return OAPL_ERR_HIP; \
  } while (0)

template <class K>
static bool allow_big_lds(K kernel, int bytes) {
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

template <class C, bool ROWS>
static bool allow_fwd() {
  return allow_big_lds(k_fwd_lse<C, false, ROWS>, C::LDS_BYTES) && allow_big_lds(k_fwd_lse<C, true, ROWS>, C::LDS_BYTES);
}
template <class C, bool ROWS>
static bool allow_sample() {
  return allow_big_lds(k_fwd_sample<C, ROWS>, C::LDS_BYTES);
}

template <class C, bool ATR>
static bool allow_dh() {
  return allow_big_lds(k_bwd_dh<C, false, ATR>, C::LDS_BYTES) && allow_big_lds(k_bwd_dh<C, true, ATR>, C::LDS_BYTES);
}
// ... of a loss call in large tiles of C's width, operands in place
template <class C>
static bool allow_loss() {
  return allow_big_lds(k_sweep<C, true>, C::LDS_BYTES) && allow_big_lds(k_bwd_dz<C, true>, C::LDS_BYTES) && allow_dh<C, true>();
}
template <class C>
static bool allow_grads() {
  return allow_big_lds(k_bwd_dw<C>, C::LDS_BYTES) && allow_big_lds(k_bwd_grads<C, false>, C::LDS_BYTES) &&
         allow_big_lds(k_bwd_grads<C, true>, C::LDS_BYTES);
}

static bool prepare_kernels() {
  static std::once_flag once;
  static bool ok = false;
  std::call_once(once, [] {
    ok = allow_fwd<Cfg64, true>() && allow_fwd<Cfg64Once, true>() && allow_fwd<Cfg128, true>() && allow_fwd<Cfg128Once, true>() &&
         allow_fwd<Cfg256, true>() && allow_fwd<Cfg256Early, true>() && allow_fwd<Cfg256Once, true>() &&
         allow_fwd<Cfg256Tall, true>() && allow_fwd<Cfg256TallOnce, true>() && allow_fwd<Cfg288, true>() &&
         allow_fwd<Cfg320, true>() && allow_fwd<Cfg352, true>() && allow_fwd<Cfg, true>() && allow_fwd<Cfg, false>() &&
         allow_sample<Cfg64, true>() && allow_sample<Cfg64Once, true>() && allow_sample<Cfg128, true>() &&
         allow_sample<Cfg128Once, true>() && allow_sample<Cfg256, true>() && allow_sample<Cfg256Early, true>() &&
         allow_sample<Cfg256Once, true>() && allow_sample<Cfg256Tall, true>() && allow_sample<Cfg256TallOnce, true>() &&
         allow_sample<Cfg288, true>() && allow_sample<Cfg320, true>() && allow_sample<Cfg352, true>() &&
         allow_sample<Cfg, true>() && allow_sample<Cfg256, false>() && allow_sample<Cfg, false>() &&
         allow_big_lds(k_fwd_lse<CfgRef, false, true>, CfgRef::LDS_BYTES) &&
         allow_big_lds(k_fwd_lse<CfgRef, false, false>, CfgRef::LDS_BYTES) &&
         allow_big_lds(k_sweep_begin<CfgRef, OaplBegin>, CfgRef::LDS_BYTES) &&
         allow_big_lds(k_sweep_begin<CfgRef, GrpoBegin>, CfgRef::LDS_BYTES) &&
         allow_big_lds(k_ref_begin<CfgRef, OaplBegin>, CfgRef::LDS_BYTES) &&
         allow_big_lds(k_ref_begin<CfgRef, GrpoBegin>, CfgRef::LDS_BYTES) &&
         allow_big_lds(k_bwd_dz<Cfg, false>, Cfg::LDS_BYTES) && allow_big_lds(k_sweep<Cfg, false>, Cfg::LDS_BYTES) &&
         allow_loss<Cfg256>() && allow_loss<Cfg288>() && allow_loss<Cfg320>() && allow_loss<Cfg352>() && allow_loss<Cfg>() &&
         allow_big_lds(k_sweep<CfgEarly, true>, CfgEarly::LDS_BYTES) &&
         allow_big_lds(k_sweep<CfgSmall, true>, CfgSmall::LDS_BYTES) &&
         allow_big_lds(k_sweep<CfgDeep, true>, CfgDeep::LDS_BYTES) && allow_dh<Cfg, false>() &&
         allow_dh<CfgSmall, true>() && allow_dh<CfgDeep, true>() && allow_big_lds(k_bwd_dw<Cfg>, Cfg::LDS_BYTES) &&
         allow_grads<CfgSmall>() && allow_grads<CfgDeep>() &&
         allow_big_lds(k_gemm_f32<F32Wide, true, false, EpiStoreF32>, F32Wide::LDS) &&
         allow_big_lds(k_gemm_f32<F32Wide, false, false, EpiStoreF32>, F32Wide::LDS);
  });
  return ok;
}

// Steps a1-a3 of the path: partial soft-max statistics, sampled-token logit,
// finish.  Writes logprob / lse if wanted, and (for the loss) lse in the
// kernels' exponent domain plus logprob - logq in double.
constexpr Gate kNoGate{nullptr, 0};

// Slices of the finishing kernels: at least four partials per thread.
static int finish_slices(int n_parts) {
  int s = 1;
  while (s < 256 && s * 8 <= n_parts) s *= 2;
  return s;
}

struct FwdArgs {
  const bf16_t *W, *H;
  int V;
  int64_t T;
  int d, n_kt;
  TilePick pick;
};

// Token tiles per XCD patch of the streaming kernels: eight while a token tile's H strip is at most 3 MiB (384 columns: d <=
// 4096), else four. Scoring 20000 tokens at d = 4096, walks of 3 tiles: 20.2 / 18.2 / 18.1 / 18.4 ms for patches of 1 / 4 / 8 / 16;
// 30000 at d = 5120: 36.7 / 34.5 / 35.5 / 35.7; 20000 at d = 2048 10.19 / 9.15 / 9.18 / 9.28.
template <class C>
static int patch_tiles(int n_kt) { return (size_t)n_kt * C::STAGE_B <= ((size_t)3 << 20) ? 8 : 4; }

// One streaming log-sum-exp pass (the plan's tile; ENT: with the entropy's partial sums in upart).
template <class C, bool ENT, bool ROWS>
static void launch_fwd_lse_kernel(const FwdArgs& a, float2* partials, float* upart, int* clear, hipStream_t st, Gate gate) {
  const int64_t total = (a.T + C::BN - 1) / C::BN * a.pick.splits;
  const unsigned grid = (unsigned)round_up(total, 8);
  k_fwd_lse<C, ENT, ROWS><<<grid, C::NT, C::LDS_BYTES, st>>>(a.W, a.H, a.V, a.T, a.d, a.n_kt, a.pick.splits, a.pick.balanced,
                                                           patch_tiles<C>(a.n_kt), partials, upart, clear, gate);
}
template <class C, bool ROWS>
static void launch_fwd_lse(const FwdArgs& a, float2* partials, float* upart, int* clear, hipStream_t st, Gate gate) {
  if (upart) launch_fwd_lse_kernel<C, true, ROWS>(a, partials, upart, clear, st, gate);
  else launch_fwd_lse_kernel<C, false, ROWS>(a, partials, nullptr, clear, st, gate);
}
static void launch_fwd_lse(const FwdArgs& a, bool rows, float2* partials, float* upart, int* clear, hipStream_t st,
                           Gate gate) {
  if (!rows) return launch_fwd_lse<Cfg, false>(a, partials, upart, clear, st, gate);
  const bool once = once_pays(a.T, a.V, a.d);
  switch (a.pick.tile) {
    case kTile64:
      if (once) return launch_fwd_lse<Cfg64Once, true>(a, partials, upart, clear, st, gate);
      return launch_fwd_lse<Cfg64, true>(a, partials, upart, clear, st, gate);
    case kTile128:
      if (once) return launch_fwd_lse<Cfg128Once, true>(a, partials, upart, clear, st, gate);
      return launch_fwd_lse<Cfg128, true>(a, partials, upart, clear, st, gate);
    case kTile256:
      if (a.pick.tall && once) return launch_fwd_lse<Cfg256TallOnce, true>(a, partials, upart, clear, st, gate);
      if (a.pick.tall) return launch_fwd_lse<Cfg256Tall, true>(a, partials, upart, clear, st, gate);
      if (once) return launch_fwd_lse<Cfg256Once, true>(a, partials, upart, clear, st, gate);
      if (early_pays(a.T, a.V, a.d)) return launch_fwd_lse<Cfg256Early, true>(a, partials, upart, clear, st, gate);
      return launch_fwd_lse<Cfg256, true>(a, partials, upart, clear, st, gate);
    case kTile288: return launch_fwd_lse<Cfg288, true>(a, partials, upart, clear, st, gate);
    case kTile320: return launch_fwd_lse<Cfg320, true>(a, partials, upart, clear, st, gate);
    case kTile352: return launch_fwd_lse<Cfg352, true>(a, partials, upart, clear, st, gate);
    case kTile384: return launch_fwd_lse<Cfg, true>(a, partials, upart, clear, st, gate);
  }
}

// ... of the sampling kernel: patches of 1 / 4 / 8 token tiles, V = 151936, us: d = 4096, 1003 tokens 1010 / 993 / 990, 4096 3904 /
// 3835 / 3830, 6144 6170 / 5982 / 6064; d = 2048 554 / 551 / 542, 2115 / 2106 / 2086, 3339 / 3187 / 3291, 8192 4086 / 4044 / 4106.
constexpr int kSamplePatch = 4;
template <class C, bool ROWS>
static void launch_sample(const FwdArgs& a, float inv_t, uint64_t seed, float2* partials, hipStream_t st) {
  const int64_t total = (a.T + C::BN - 1) / C::BN * a.pick.splits;
  k_fwd_sample<C, ROWS><<<(unsigned)round_up(total, 8), C::NT, C::LDS_BYTES, st>>>(
      a.W, a.H, a.V, a.T, a.d, a.n_kt, a.pick.splits, a.pick.balanced, kSamplePatch, inv_t, (uint32_t)seed,
      (uint32_t)(seed >> 32), partials);
}

static void launch_sample(const FwdArgs& a, bool rows, float inv_t, uint64_t seed, float2* partials, hipStream_t st) {
  if (!rows && a.pick.tile == kTile256) return launch_sample<Cfg256, false>(a, inv_t, seed, partials, st);
  if (!rows) return launch_sample<Cfg, false>(a, inv_t, seed, partials, st);
  const bool once = once_pays(a.T, a.V, a.d);
  switch (a.pick.tile) {
    case kTile64:
      if (once) return launch_sample<Cfg64Once, true>(a, inv_t, seed, partials, st);
      return launch_sample<Cfg64, true>(a, inv_t, seed, partials, st);
    case kTile128:
      if (once) return launch_sample<Cfg128Once, true>(a, inv_t, seed, partials, st);
      return launch_sample<Cfg128, true>(a, inv_t, seed, partials, st);
    case kTile256:
      if (a.pick.tall && once) return launch_sample<Cfg256TallOnce, true>(a, inv_t, seed, partials, st);
      if (a.pick.tall) return launch_sample<Cfg256Tall, true>(a, inv_t, seed, partials, st);
      if (once) return launch_sample<Cfg256Once, true>(a, inv_t, seed, partials, st);
      if (early_pays(a.T, a.V, a.d)) return launch_sample<Cfg256Early, true>(a, inv_t, seed, partials, st);
      return launch_sample<Cfg256, true>(a, inv_t, seed, partials, st);
    case kTile288: return launch_sample<Cfg288, true>(a, inv_t, seed, partials, st);
    case kTile320: return launch_sample<Cfg320, true>(a, inv_t, seed, partials, st);
    case kTile352: return launch_sample<Cfg352, true>(a, inv_t, seed, partials, st);
    case kTile384: return launch_sample<Cfg, true>(a, inv_t, seed, partials, st);
  }
}

static F32Operand f32_operand(const void* p, int64_t ld) {
  return F32Operand{(const float*)p, ld, ld % 4 == 0 && ((uintptr_t)p & 15) == 0};
}

// 128 x 128 tiles of the logits where they give every CU one, else 64 x 128.  (From bf16 parts 64 x 128 would serve most calls
// above the line as well: 64 x 128 / 128 x 128, whole calls, us, T, d, V (tiles): 700, 300, 3000 (144) 87 / 100; 900, 400, 4000
// (256) 163 / 173; 1980, 545, 3120 (400) 254 / 244; 999, 398, 7605 (480) 243 / 235; 1300, 600, 6000 (517) 358 / 394; 1501, 768,
// 8192 (768) 475 / 492; 2000, 768, 8192 (1024) 609 / 617.)
static bool logits_large_f32(int V, int64_t T) {
  return (int64_t)grid1d(V, F32Large::BM) * grid1d(T, F32Large::BN) >= kNumCU;
}

// Logits of T token rows (transposed: M = vocabulary), in whatever form the epilogue leaves them.
template <class C, class Epi>
static void launch_logits_f32(const Plan& p, const F32Operand& A, const F32Operand& B, int64_t T, Epi epi, hipStream_t st) {
  const int64_t tiles = (int64_t)grid1d(p.V, C::BM) * grid1d(T, C::BN);
  k_gemm_f32<C, true, true><<<f32_grid(tiles), C::NT, C::LDS, st>>>(A, B, (int64_t)p.V, T, (int64_t)p.d, epi, 1);
}
template <class Epi>
static void launch_logits_f32(const Plan& p, const void* H, const void* W, int64_t T, Epi epi, hipStream_t st) {
  const F32Operand A = f32_operand(W, p.d), B = f32_operand(H, p.d);
  if (logits_large_f32(p.V, T)) launch_logits_f32<F32Large>(p, A, B, T, epi, st);
  else launch_logits_f32<F32Flat>(p, A, B, T, epi, st);
}

// ... in the launch that a loss call of few tokens starts with (k_scores_f32).
template <class C, class Begin>
static void launch_scores_f32(const Plan& p, const Begin& begin, const void* H, const void* W, const int32_t* tokens, float* zy,
                              const TokenInit& init, const EpiLseF32& epi, hipStream_t st) {
  const F32Operand A = f32_operand(W, p.d), B = f32_operand(H, p.d);
  const unsigned grid = 1 + grid1d(p.T, 4) + grid1d(p.V, C::BM) * grid1d(p.T, C::BN);
  if (A.vec && B.vec)
    k_scores_f32<C, EpiLseF32, Begin, 4><<<grid, 256, 0, st>>>(begin, tokens, zy, init, A, B, p.V, p.T, p.d, epi);
  else k_scores_f32<C, EpiLseF32, Begin, 1><<<grid, 256, 0, st>>>(begin, tokens, zy, init, A, B, p.V, p.T, p.d, epi);
}

// out[m][n] (+)= sum_k A(m, k) B(n, k), B and (unless A_KC) A with their rows contiguous.
static F32Contraction contraction_f32(const F32Pick& pick, int wide, const F32Operand& A, const F32Operand& B, int64_t M,
                                      int64_t N, int64_t K, float* out) {
  const int bm = wide ? F32Wide::BM : pick.large ? F32Large::BM : F32Small::BM;
  const int bn = wide ? F32Wide::BN : pick.large ? F32Large::BN : F32Small::BN;
  return F32Contraction{A, B, M, N, K, out, (int)grid1d(N, bn), (int)grid1d(M, bm), wide ? wide : pick.splits};
}
template <class C, bool A_KC>
static void launch_contract_f32(const F32Contraction& c, int accumulate, hipStream_t st) {
  k_gemm_f32<C, A_KC, false><<<f32_grid((int64_t)c.nx * c.ny * c.splits), C::NT, C::LDS, st>>>(
      c.A, c.B, c.M, c.N, c.K, EpiStoreF32{c.out, c.N, accumulate}, c.splits);
}
template <bool A_KC>
static void launch_contract_f32(const F32Pick& pick, int wide, const F32Contraction& c, int accumulate, hipStream_t st) {
  if (wide) launch_contract_f32<F32Wide, A_KC>(c, accumulate, st);
  else if (pick.large) launch_contract_f32<F32Large, A_KC>(c, accumulate, st);
  else launch_contract_f32<F32Small, A_KC>(c, accumulate, st);
}

// Both gradient contractions of a batch of one panel, and the sums of what was split.
static int grads_f32(const Plan& p, const void* H, const void* W, const float* zt, float* dH, float* dW, char* ws,
                     hipStream_t st) {
  float* part_dh = (p.wide_dh ? p.wide_dh : p.f32_dh.splits) > 1 ? (float*)(ws + p.off_part) : nullptr;
  float* part_dw = (p.wide_dw ? p.wide_dw : p.f32_dw.splits) > 1 ? (float*)(ws + p.off_part_dw) : nullptr;
  // dH[t][j] = sum_v dZ[t][v] W[v][j],  dW[v][j] = sum_t dZ[t][v] H[t][j]
  const F32Operand z = f32_operand(zt, p.ldz);
  const F32Contraction dh = contraction_f32(p.f32_dh, p.wide_dh, z, f32_operand(W, p.d), p.T, p.d, p.V, part_dh ? part_dh : dH);
  const F32Contraction dw = contraction_f32(p.f32_dw, p.wide_dw, z, f32_operand(H, p.d), p.V, p.d, p.T, part_dw ? part_dw : dW);
  const F32Reduction a{part_dh, dh.splits, part_dh ? dh.M * dh.N : 0, dH}, b{part_dw, dw.splits, part_dw ? dw.M * dw.N : 0, dW};
  const F32Reduction none{nullptr, 0, 0, nullptr};
  auto reduce = [&](const F32Reduction& x, const F32Reduction& y) {
    const int64_t blocks = (x.n + y.n + 255) / 256;
    if (blocks > 0) k_reduce_f32<<<(unsigned)(blocks < 8192 ? blocks : 8192), 256, 0, st>>>(x, y);
  };
  if (!p.grads_fused) {
    launch_contract_f32<false>(p.f32_dh, p.wide_dh, dh, 0, st);
    OAPL_LAUNCH_CHECK();
    reduce(a, none);      // before the other's partial results, which have the same space
    OAPL_LAUNCH_CHECK();
    launch_contract_f32<true>(p.f32_dw, p.wide_dw, dw, 0, st);
    OAPL_LAUNCH_CHECK();
    reduce(b, none);
    OAPL_LAUNCH_CHECK();
    return OAPL_OK;
  }
  const unsigned grid = (unsigned)((int64_t)dh.nx * dh.ny * dh.splits + (int64_t)dw.nx * dw.ny * dw.splits);
  if (p.f32_dh.large && p.f32_dw.large) k_grads_f32<F32Large, F32Large><<<grid, 256, 0, st>>>(dh, dw);
  else if (p.f32_dh.large) k_grads_f32<F32Large, F32Small><<<grid, 256, 0, st>>>(dh, dw);
  else if (p.f32_dw.large) k_grads_f32<F32Small, F32Large><<<grid, 256, 0, st>>>(dh, dw);
  else k_grads_f32<F32Small, F32Small><<<grid, 256, 0, st>>>(dh, dw);
  OAPL_LAUNCH_CHECK();
  reduce(a, b);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// Aligned copies of the operands that the plan has copies of, which the call uses from here on.
static int copy_unaligned(const Plan& p, const void*& H, const void*& W, char* ws, hipStream_t st) {
  auto copy = [&](const void*& m, int64_t elements, size_t off) {
    const int64_t pieces = elements / 8;
    k_copy_aligned<<<(unsigned)(pieces < 256 * 65536 ? grid1d(pieces, 256) : 65536), 256, 0, st>>>((const bf16_t*)m, pieces,
                                                                                                (bf16_t*)(ws + off));
    m = ws + off;
  };
  if (p.unaligned & kUnalignedW) copy(W, (int64_t)p.V * p.d, p.off_Wc);
  if (p.unaligned & kUnalignedH) copy(H, p.T * p.d, p.off_Hc);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// bf16: packed or aligned copies of W and H where the plan wants them.
static int pack_operands(const Plan& p, const void*& H, const void*& W, char* ws, hipStream_t st) {
  if (p.T == 0 || p.dtype != OAPL_BF16) return OAPL_OK;
  if (!prepare_kernels()) return OAPL_ERR_HIP;
  if (p.rows) return copy_unaligned(p, H, W, ws, st);
  k_pack_rows<<<dim3(p.n_kt_d, p.n_rt_v), 256, 0, st>>>((const bf16_t*)W, p.V, p.d, p.d, (bf16_t*)(ws + p.off_Wp), p.n_kt_d,
                                                        Cfg::BM);
  OAPL_LAUNCH_CHECK();
  k_pack_rows<<<dim3(p.n_kt_d, (unsigned)p.n_rt_T), 256, 0, st>>>((const bf16_t*)H, p.T, p.d, p.d, (bf16_t*)(ws + p.off_Hp),
                                                                  p.n_kt_d, Cfg::BN);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// The sampled tokens' logits, and the per-token arrays in `init`.  After the status header has been cleared.
static int gather_logits(const Plan& p, const void* H, const void* W, const int32_t* tokens, TokenInit init, char* ws,
                         hipStream_t st) {
  int* status = (int*)(ws + p.off_status);
  float* zy = (float*)(ws + p.off_zy);
  if (p.T == 0) return OAPL_OK;
  if (p.dtype == OAPL_BF16) {
    k_gather_logit<bf16_t, float, 8><<<grid1d(p.T, 4), 256, 0, st>>>((const bf16_t*)H, (const bf16_t*)W, tokens, p.T, p.d,
                                                                     p.V, zy, status, init);
  } else {
    const bool vec = p.d % 4 == 0 && (((uintptr_t)H | (uintptr_t)W) & 15) == 0;
    (vec ? k_gather_logit<float, double, 4> : k_gather_logit<float, double, 1>)<<<grid1d(p.T, 4), 256, 0, st>>>(
        (const float*)H, (const float*)W, tokens, p.T, p.d, p.V, zy, status, init);
  }
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// The operands of the contractions over d, in place or packed by pack_operands: token row t of H starts at H + t * ld
// (packed: at a multiple of the token tile).
struct ContractD {
  const bf16_t *W, *H;
  int64_t ld;
};
static ContractD contract_d(const Plan& p, const void* H, const void* W, const char* ws) {
  if (p.rows) return ContractD{(const bf16_t*)W, (const bf16_t*)H, p.d};
  return ContractD{(const bf16_t*)(ws + p.off_Wp), (const bf16_t*)(ws + p.off_Hp), (int64_t)p.n_kt_d * kPackK};
}

// The partial soft-max sums of every token (and the entropy's with `entropy`).  `clear`: a status header to clear.
static int forward_partials(const Plan& p, const void* H, const void* W, bool entropy, bool keep_logits, int* clear, char* ws,
                            hipStream_t st, Gate gate) {
  const int64_t T = p.T;
  if (T == 0) return OAPL_OK;
  float2* partials = (float2*)(ws + p.off_fwd_partials);
  float* upart = entropy ? (float*)(ws + p.off_upart) : nullptr;
  if (p.dtype == OAPL_BF16) {
    const ContractD x = contract_d(p, H, W, ws);
    const FwdArgs args{x.W, x.H, p.V, T, p.d, p.n_kt_d, p.fwd};
    ScopedKernelTimer tm(kFwdLse, st, gate.flag == nullptr);
    launch_fwd_lse(args, p.rows, partials, upart, clear, st, gate);
  } else {
    // a batch whose gradient is one panel keeps its logits for it
    float* zt = keep_logits && T <= p.Tp ? (float*)(ws + p.off_G) : nullptr;
    if (clear) k_fill_i32<<<1, 64, 0, st>>>(clear, kStatusWords, 0);
    launch_logits_f32(p, H, W, T, EpiLseF32{partials, T, upart, zt, p.ldz}, st);
  }
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// Log-probs (and lse, entropy) from the partial sums and the sampled tokens' logits; with `logq` also what the objective
// and the gradients need. `check_tokens`: the tokens, if the gather before left it to this launch to report those out of range.
static LseFinish finish_args(const Plan& p, const float* logq, float* logprob_out, float* lse_out, float* entropy_out,
                             const int32_t* check_tokens, char* ws) {
  const bool loss = logq != nullptr;
  return LseFinish{(const float2*)(ws + p.off_fwd_partials), p.fwd.splits, p.T, (const float*)(ws + p.off_zy), logq, logprob_out,
                   lse_out, loss ? (float*)(ws + p.off_lse2) : nullptr, loss ? (double*)(ws + p.off_diff) : nullptr,
                   loss ? (float*)(ws + p.off_omp) : nullptr, loss ? (float*)(ws + p.off_inv) : nullptr,
                   entropy_out ? (const float*)(ws + p.off_upart) : nullptr, entropy_out, finish_slices(p.fwd.splits),
                   check_tokens, p.V, (int*)(ws + p.off_status)};
}
static int forward_finish(const Plan& p, const LseFinish& f, hipStream_t st, Gate gate) {
  if (p.T == 0) return OAPL_OK;
  (p.dtype == OAPL_BF16 ? k_lse_finish<true> : k_lse_finish<false>)<<<grid1d(p.T, 256 / f.slices), 256, 0, st>>>(f, gate);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// An fp32 loss call's log-probs are finished by the objective's launch where that is little work for one workgroup: a dependent
// launch costs a small call 5 us whatever is in it, and a rollout's workgroup has its tokens in rounds of 256 / slices, 4 us each,
// that a launch of its own has side by side.  Up to two rounds of tokens, so that even one rollout with all of them takes no
// longer: one launch less / one more, d = 64, us: one rollout, V = 64, 512 tokens (2 rounds) 31.5 / 36.3, 1536 (6) 35.5 / 36.7,
// 2048 (8) 40.2 / 36.1, V = 1024, 128 (2) 33.2 / 35.2, 192 (3) 39.5 / 35.6, V = 8192, 16 (2) 35.9 / 36.1, 32 (4) 43.4 / 35.8.  Up
// to four rounds where rollouts of twice the mean length have one: 256 tokens of eight rollouts, V = 1024, 31.7 / 35 (all of them
// in one of the eight, which the host does not see, 39).  In bf16, where the finish is the fallback's and closed, the launch that
// it saves goes into the larger kernel (1000 tokens at d = 256, V = 1544 53.6 / 53.4).
static bool finish_in_objective(const Plan& p) {
  const int64_t round = 256 / finish_slices(p.fwd.splits);
  return p.dtype == OAPL_F32 && p.T > 0 && (p.T <= 2 * round || (p.T <= 4 * round && 2 * p.T <= round * p.n_seq));
}

// Calls f with the large tile of that many columns.
template <class F>
static void for_width(int width, F&& f) {
  if (width == Cfg256::BN) f(Cfg256{});
  else if (width == Cfg288::BN) f(Cfg288{});
  else if (width == Cfg320::BN) f(Cfg320{});
  else if (width == Cfg352::BN) f(Cfg352{});
  else f(Cfg{});
}

template <class C, bool SPLIT, bool ATR>
static void launch_dh(const DhArgs& args, hipStream_t st, Gate gate) {
  const unsigned grid = (unsigned)round_up(tile_count<C>(args.d, args.n_valid) * (SPLIT ? args.splits : 1), 8);
  k_bwd_dh<C, SPLIT, ATR><<<grid, C::NT, C::LDS_BYTES, st>>>(args, gate);
}
template <class C, bool ATR>
static void launch_dh(const DhArgs& args, bool split, hipStream_t st, Gate gate) {
  if (split) launch_dh<C, true, ATR>(args, st, gate);
  else launch_dh<C, false, ATR>(args, st, gate);
}
template <class C>
static void launch_dw(const DwArgs& args, hipStream_t st, Gate gate) {
  k_bwd_dw<C><<<(unsigned)round_up(tile_count<C>(args.d, args.V), kNumCU), C::NT, C::LDS_BYTES, st>>>(args, gate);
}
template <class C>
static void launch_grads(const DhArgs& dh, bool split, const DwArgs& dw, hipStream_t st, Gate gate) {
  const unsigned n_dh = (unsigned)round_up(tile_count<C>(dh.d, dh.n_valid) * (split ? dh.splits : 1), 8);
  const int n_dw = (int)tile_count<C>(dw.d, dw.V);
  const unsigned grid = n_dh + (unsigned)round_up(n_dw, 8);
  if (split) k_bwd_grads<C, true><<<grid, C::NT, C::LDS_BYTES, st>>>(dh, (int)n_dh, dw, n_dw, gate);
  else k_bwd_grads<C, false><<<grid, C::NT, C::LDS_BYTES, st>>>(dh, (int)n_dh, dw, n_dw, gate);
}

// One panel's dH and dW.  Only the tiles of the batch's last panel are split, and only it has a space for partial sums (no
// sweep or recompute of the call follows; the other panels of a long batch are sized to fill the chip as they are).
static int launch_gradients(const Plan& p, DhArgs dh, const DwArgs& dw, bool last, char* ws, hipStream_t st, Gate gate,
                            bool timed) {
  const bool split = last && p.dh.splits > 1, small = last && p.dh.small;
  dh.splits = split ? p.dh.splits : 1;
  dh.part = split ? (float*)(ws + p.off_part) : nullptr;
  const int64_t dh_groups = small ? tile_count<CfgDeep>(p.d, dh.n_valid) * dh.splits : 0;
  const int64_t dw_groups = p.small_dw ? tile_count<CfgDeep>(p.d, p.V) : 0;
  auto reduce = [&] {     // before anything else has pushed the partial sums out of the caches (11 us; 21 behind dW's stores)
    if (!split) return;
    const int64_t blocks = grid1d(dh.n_valid * (p.d / 8), 256);
    k_dh_reduce<<<(unsigned)(blocks < 8192 ? blocks : 8192), 256, 0, st>>>(dh.part, dh.splits, dh.n_valid, p.d, dh.row_factor,
                                                                        dh.dH, gate);
  };
  if (p.grads_fused) {
    {
      ScopedKernelTimer tm(kBwdDw, st, timed);
      if (dh_groups + dw_groups <= kNumCU) launch_grads<CfgDeep>(dh, split, dw, st, gate);
      else launch_grads<CfgSmall>(dh, split, dw, st, gate);
    }
    OAPL_LAUNCH_CHECK();
    reduce();
    OAPL_LAUNCH_CHECK();
    return OAPL_OK;
  }
  {
    ScopedKernelTimer tm(kBwdDh, st, timed);
    if (small && dh_groups <= kNumCU) launch_dh<CfgDeep, true>(dh, split, st, gate);
    else if (small) launch_dh<CfgSmall, true>(dh, split, st, gate);
    else if (p.rows) for_width(p.width, [&](auto c) { launch_dh<decltype(c), true>(dh, split, st, gate); });
    else launch_dh<Cfg, false>(dh, split, st, gate);
  }
  OAPL_LAUNCH_CHECK();
  reduce();
  OAPL_LAUNCH_CHECK();
  {
    ScopedKernelTimer tm(kBwdDw, st, timed);
    if (p.small_dw && dw_groups <= kNumCU) launch_dw<CfgDeep>(dw, st, gate);
    else if (p.small_dw) launch_dw<CfgSmall>(dw, st, gate);
    else launch_dw<Cfg>(dw, st, gate);
  }
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

template <class C, bool ROWS>
static void launch_sweep(const Plan& p, const bf16_t* W, const bf16_t* H, int64_t nv, const float* ref2, bf16_t* G, bf16_t* GT,
                         float* spart, hipStream_t st, Gate gate) {
  k_sweep<C, ROWS><<<(unsigned)round_up(tile_count<C>(p.V, nv), 8), C::NT, C::LDS_BYTES, st>>>(
      W, H, p.V, nv, p.d, p.n_kt_d, ref2, G, p.n_kt_g, GT, p.n_kt_t, spart, p.Tp, gate);
}

static int pack_wt(const Plan& p, const void* W, char* ws, hipStream_t st, Gate gate) {
  if (p.rows) return OAPL_OK;
  k_pack_transposed<<<dim3(p.n_kt_v, p.n_rt_d), 256, 0, st>>>(
      PackTransposed{(const bf16_t*)W, p.V, p.d, p.d, nullptr, (bf16_t*)(ws + p.off_WTp), p.n_kt_v}, gate);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// (diag(coef) H)^T of the panel at token t0, packed; token columns in [nv, 64 kt) come out as zeros
static PackTransposed scaled_rows(const Plan& p, const void* H, int64_t t0, char* ws) {
  const int64_t nv = (p.T - t0) < p.Tp ? (p.T - t0) : p.Tp;
  return PackTransposed{(const bf16_t*)H + t0 * p.d, nv, p.d, p.d, (const float*)(ws + p.off_coef) + t0,
                        (bf16_t*)(ws + p.off_HTp), p.n_kt_t};
}

// Step a8, two-pass form: the soft-max tiles of the panel at token t0 recomputed into G and G^T.  `pack`: the launch makes the
// panel's scaled_rows too, whatever the gate says.
static int recompute_panel(const Plan& p, const void* H, const void* W, const int32_t* tokens, int64_t t0, bf16_t* G, bf16_t* GT,
                           char* ws, hipStream_t st, Gate gate, bool pack = false) {
  const int64_t nv = (p.T - t0) < p.Tp ? (p.T - t0) : p.Tp;
  const ContractD x = contract_d(p, H, W, ws);
  const int kt = (int)((nv + kPackK - 1) / kPackK), blocks = kt * p.n_rt_d, n_pack = pack ? (blocks + 1) / 2 : 0;
  {
    ScopedKernelTimer tm(kBwdDz, st, gate.flag == nullptr);
    const PackTransposed rows = scaled_rows(p, H, t0, ws);
    auto launch = [&](auto kernel, int BN, int threads, int lds) {
      kernel<<<(unsigned)(n_pack + round_up(p.n_rt_v * ((nv + BN - 1) / BN), 8)), threads, lds, st>>>(
          x.W, x.H + t0 * x.ld, p.V, nv, p.d, p.n_kt_d, tokens + t0, (const float*)(ws + p.off_lse2) + t0,
          (const float*)(ws + p.off_inv) + t0, G, p.n_kt_g, GT, p.n_kt_t, gate, n_pack, rows, kt, blocks);
    };
    if (!p.rows) launch(k_bwd_dz<Cfg, false>, Cfg::BN, Cfg::NT, Cfg::LDS_BYTES);
    else for_width(p.width, [&](auto c) {
      typedef decltype(c) C;
      launch(k_bwd_dz<C, true>, C::BN, C::NT, C::LDS_BYTES);
    });
  }
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// Steps a9, a10: the two gradient contractions of the panel at token t0 from G and G^T, with coef[t] = the row factor
// (two-pass form: f_t = c_t (1 - p_y); single sweep: a_t).  `packed`: an earlier launch made scaled_rows.
static int panel_gradients(const Plan& p, const void* H, const void* W, int64_t t0, const bf16_t* G, const bf16_t* GT, void* dH,
                           float* dW, char* ws, hipStream_t st, Gate gate, bool timed, bool packed = false) {
  const int d = p.d;
  const int64_t nv = (p.T - t0) < p.Tp ? (p.T - t0) : p.Tp;
  const int kt = (int)((nv + kPackK - 1) / kPackK);
  const float* coef = (const float*)(ws + p.off_coef) + t0;
  bf16_t* HTp = (bf16_t*)(ws + p.off_HTp);
  if (!packed) k_pack_transposed<<<dim3(kt, p.n_rt_d), 256, 0, st>>>(scaled_rows(p, H, t0, ws), gate);
  OAPL_LAUNCH_CHECK();
  const DhArgs dh{p.rows ? (const bf16_t*)W : (const bf16_t*)(ws + p.off_WTp), p.V, p.n_kt_v, G, p.n_kt_g, d, nv, p.n_kt_v, coef,
                  (bf16_t*)dH + t0 * d, 1, nullptr};
  const DwArgs dw{HTp, GT, p.n_kt_t, d, p.V, kt, dW, t0 > 0 ? 1 : 0};
  return launch_gradients(p, dh, dw, t0 + p.Tp >= p.T, ws, st, gate, timed);
}

// Steps a8-a10, two-pass form, panel by panel, from log-sum-exps and token coefficients.  `wt_packed`: W^T has been packed
// already by this call.
static int backward_grads(const Plan& p, const void* H, const void* W, const int32_t* tokens, void* dH, float* dW,
                          char* ws, hipStream_t st, Gate gate, bool wt_packed) {
  const int64_t T = p.T;
  const int d = p.d, V = p.V;
  if (T == 0) {
    k_fill_f32<<<1024, 256, 0, st>>>(dW, (int64_t)V * d, 0.f, gate);
    OAPL_LAUNCH_CHECK();
    return OAPL_OK;
  }
  if (p.dtype == OAPL_BF16) {
    bf16_t* G = (bf16_t*)(ws + p.off_G);
    bf16_t* GT = (bf16_t*)(ws + p.off_GT);
    if (!wt_packed)
      if (int rc = pack_wt(p, W, ws, st, gate)) return rc;
    for (int64_t t0 = 0; t0 < T; t0 += p.Tp) {
      if (int rc = recompute_panel(p, H, W, tokens, t0, G, GT, ws, st, gate)) return rc;
      if (int rc = panel_gradients(p, H, W, t0, G, GT, dH, dW, ws, st, gate, gate.flag == nullptr)) return rc;
    }
    return OAPL_OK;
  }
  if ((p.wide_dh || p.wide_dw) && !prepare_kernels()) return OAPL_ERR_HIP;
  float* zt = (float*)(ws + p.off_G);   // dZ^T of a panel
  const float* lse = (const float*)(ws + p.off_lse2);
  const float* coef = (const float*)(ws + p.off_coef);
  if (T <= p.Tp) {   // the scoring pass left the logits here
    k_dz_f32<<<dim3(grid1d(V, kDzRows), grid1d(T, 256)), 256, 0, st>>>(zt, p.ldz, V, T, tokens, lse, coef);
    OAPL_LAUNCH_CHECK();
    return grads_f32(p, H, W, zt, (float*)dH, dW, ws, st);
  }
  for (int64_t t0 = 0; t0 < T; t0 += p.Tp) {
    const int64_t nv = (T - t0) < p.Tp ? (T - t0) : p.Tp;
    const float* Hp = (const float*)H + t0 * d;
    launch_logits_f32(p, Hp, W, nv, EpiDzF32{tokens + t0, lse + t0, coef + t0, zt, p.ldz}, st);
    OAPL_LAUNCH_CHECK();
    // dH[t][j] = sum_v dZ[t][v] W[v][j]
    launch_contract_f32<false>(p.f32_dh, p.wide_dh,
                               contraction_f32(p.f32_dh, p.wide_dh, f32_operand(zt, p.ldz), f32_operand(W, d), nv, d, V,
                                               (float*)dH + t0 * d), 0, st);
    OAPL_LAUNCH_CHECK();
    // dW[v][j] (+)= sum_t dZ[t][v] H[t][j]
    launch_contract_f32<true>(p.f32_dw, p.wide_dw,
                              contraction_f32(p.f32_dw, p.wide_dw, f32_operand(zt, p.ldz), f32_operand(Hp, d), V, d, nv, dW),
                              t0 > 0 ? 1 : 0, st);
    OAPL_LAUNCH_CHECK();
  }
  return OAPL_OK;
}

// A rollout may span at most n_buf - 1 panels' worth of rows on the single sweep (any length if the batch is one panel).
static int64_t sweep_longest(const Plan& p) { return p.n_buf > 1 ? (int64_t)(p.n_buf - 1) * p.Tp : p.Tp; }

// One workgroup takes a call's first steps while it has at most a few thousand (rollout, prompt) pairs to look at.
static bool begin_in_one_launch(int n_seq, int n_groups) { return (int64_t)n_seq * n_groups + n_seq + n_groups <= 8192; }
// ... else workgroups of 256 rollouts and four prompts each, at most 65536: the steps walk on from there, and thread indices
// stay far below 2^31.
static unsigned begin_grid(int n_seq, int n_groups) {
  const unsigned a = grid1d(n_groups, 4), b = grid1d(n_seq > 0 ? n_seq : 1, 256), most = 1u << 16;
  return a > most || b > most ? most : (a > b ? a : b);
}

// A call's beginning: the status header, the sweep's length check, and what needs the rewards only.
template <class Begin>
static int launch_begin(const Begin& begin, hipStream_t st) {
  if (begin_in_one_launch(begin.n_seq, begin.n_groups)) {
    k_begin<<<1, 256, 0, st>>>(begin, kPlan | kRest);
  } else {
    k_fill_i32<<<1, 64, 0, st>>>(begin.status, kStatusWords, 0);
    OAPL_LAUNCH_CHECK();
    k_begin<<<begin_grid(begin.n_seq, begin.n_groups), 256, 0, st>>>(begin, kPlan);
    if (Begin::kHasRest) {
      OAPL_LAUNCH_CHECK();
      k_begin<<<begin_grid(begin.n_seq, 1), 256, 0, st>>>(begin, kRest);
    }
  }
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

// The sweep's beginning, reference pass and gather in one launch (k_sweep_begin), whole calls in one / three, us: 1000 tokens
// at d = 256, V = 1544 53 / 59; d = 1024: 1000, V = 8000 104 / 106, 8000 463 / 466. Sixteen sampled logits per wavefront cost
// more than a launch of their own once rows are long: 1000 at d = 2048, V = 8000 168 / 165, 300 at d = 4096, V = 151936 1593 /
// 1579.
constexpr int kOneLaunchHidden = 1024;
static bool sweep_begins_in_one_launch(const Plan& p, int n_seq, int n_groups) {
  return p.rows && p.d <= kOneLaunchHidden && begin_in_one_launch(n_seq, n_groups);
}

// Otherwise: in how many parts over d the reference pass's tiles come (k_ref_begin), as many as give every CU one workgroup, of
// four k-blocks at least and eight parts at most, whose logits find room where the first panel will be; 0: it goes whole, with
// the call's beginning in front of it. Beginning, reference pass and gather of 300 and 1003 tokens at d = 4096 65 us in three
// launches, 25 in two; whole calls, us: 100 tokens, V = 8192 150 / 115, 1000 253 / 221, 300, V = 151936 1509 / 1463.
static int ref_splits(const Plan& p) {
  const int64_t tiles = grid1d(p.T, CfgRef::BN);
  for (int s = 8; s >= 2; --s)
    if (p.rows && p.d > kOneLaunchHidden && tiles * s <= kNumCU && 4 * s <= p.n_kt_d &&
        (uint64_t)s * p.T * CfgRef::BM * 4 <= p.size_G)
      return s;
  return 0;
}

// Steps a1-a3 and a8-a10 in ONE pass over the logits (bf16, T > 0).  Per panel of token rows:
// k_sweep writes the unnormalised soft-max panel and its row sums, k_sweep_finish turns the sums
// into log-probs; the objective (`objective(gate, factors)`, which must fill coef[t] = c_t * factor[t]
// for every token whose rollout is complete and may run any number of times) then gives the row
// factors, and the two gradient contractions consume the panel.  A rollout may straddle a panel
// boundary, so a panel's contractions run after the NEXT panel's sweep (two panel buffers); by
// then every rollout that touches it is complete, because no rollout is longer than a panel
// (sweep_plan raises the fallback flag otherwise).  What the sweep does runs only while the flag is 0, and the
// two-pass schedule behind it only if it is not.  A batch of one panel shares the objective and the contractions between
// the two: its fallback is the scoring pass and the recompute alone (three closed launches in place of nine).
template <class Begin, class Objective>
static int sweep_path(const Plan& p, const Begin& begin, const void* H, const void* W, const int32_t* tokens, const float* logq,
                      float* logprob_out, void* dH, float* dW, char* ws, hipStream_t st, Objective&& objective) {
  const int64_t T = p.T;
  const int d = p.d, V = p.V;
  int* flag = (int*)(ws + p.off_status) + kFlagWord;
  const Gate fast{flag, 0}, slow{flag, 1};
  const ContractD x = contract_d(p, H, W, ws);
  auto Gbuf = [&](int64_t k) { return (bf16_t*)(ws + p.off_G + (size_t)(k % p.n_buf) * p.size_G); };
  auto GTbuf = [&](int64_t k) { return (bf16_t*)(ws + p.off_GT + (size_t)(k % p.n_buf) * p.size_GT); };
  float2* sample = (float2*)(ws + p.off_partials);
  const float* zy = (const float*)(ws + p.off_zy);
  float* ref2 = (float*)(ws + p.off_ref2);
  float* spart = (float*)(ws + p.off_spart);
  double* diff = (double*)(ws + p.off_diff);
  float* nis = (float*)(ws + p.off_inv);
  const float* omp = (const float*)(ws + p.off_omp);

  TokenInit init{(float*)(ws + p.off_coef), sample, nullptr, 0, 0, ref2, diff, nis};
  const bool one = sweep_begins_in_one_launch(p, begin.n_seq, begin.n_groups);
  // k_sweep_begin leaves tokens out of range to k_sweep_finish, which is closed for the panels behind a raised flag (for all,
  // if it was raised at the beginning): the fallback, which that flag opens, then looks at every token
  const int32_t* check = one ? tokens : nullptr;
  if (one) {
    k_sweep_begin<CfgRef><<<1 + grid1d(T, CfgRef::BN), CfgRef::NT, CfgRef::LDS_BYTES, st>>>(begin, x.W, x.H, V, T, d, p.n_kt_d,
                                                                                         tokens, (float*)(ws + p.off_zy), init);
    OAPL_LAUNCH_CHECK();
  } else if (const int splits = ref_splits(p)) {
    const bool begins = begin_in_one_launch(begin.n_seq, begin.n_groups);
    if (!begins)
      if (int rc = launch_begin(begin, st)) return rc;
    init.sample_parts = (const float*)Gbuf(0);     // empty until the sweep
    init.sample_splits = splits;
    init.sample_rows = V < CfgRef::BM ? V : CfgRef::BM;
    k_ref_begin<CfgRef><<<1 + grid1d(T, CfgRef::BN) * splits, CfgRef::NT, CfgRef::LDS_BYTES, st>>>(
        begin, begins ? kPlan | kRest : 0, x.W, x.H, V, T, d, p.n_kt_d, splits, (float*)Gbuf(0));
    OAPL_LAUNCH_CHECK();
    if (int rc = gather_logits(p, H, W, tokens, init, ws, st)) return rc;
  } else {
    if (int rc = launch_begin(begin, st)) return rc;
    if (int rc = pack_wt(p, W, ws, st, kNoGate)) return rc;
    // reference exponents: running maximum over the first 256 vocabulary entries, one workgroup per 64 tokens (a walk of
    // d / 64 k-blocks each, bound by their latency)
    const FwdArgs ref{x.W, x.H, V < CfgRef::BM ? V : CfgRef::BM, T, d, p.n_kt_d, TilePick{}};
    if (p.rows) launch_fwd_lse_kernel<CfgRef, false, true>(ref, sample, nullptr, nullptr, st, fast);
    else launch_fwd_lse_kernel<CfgRef, false, false>(ref, sample, nullptr, nullptr, st, fast);
    OAPL_LAUNCH_CHECK();
    if (int rc = gather_logits(p, H, W, tokens, init, ws, st)) return rc;
  }

  auto sweep = [&](int64_t k) -> int {
    const int64_t t0 = k * p.Tp;
    const int64_t nv = (T - t0) < p.Tp ? (T - t0) : p.Tp;
    {
      ScopedKernelTimer tm(kSweep, st);
      const bf16_t* Ht = x.H + t0 * x.ld;
      if (p.small_sweep && tile_count<CfgDeep>(V, nv) <= kNumCU)
        launch_sweep<CfgDeep, true>(p, x.W, Ht, nv, ref2 + t0, Gbuf(k), GTbuf(k), spart, st, fast);
      else if (p.width != Cfg::BN)
        for_width(p.width, [&](auto c) {
          launch_sweep<decltype(c), true>(p, x.W, Ht, nv, ref2 + t0, Gbuf(k), GTbuf(k), spart, st, fast);
        });
      else if (!p.small_sweep && p.rows && (nv <= Cfg::BN || tile_count<Cfg>(V, nv) <= kNumCU))
        launch_sweep<CfgEarly, true>(p, x.W, Ht, nv, ref2 + t0, Gbuf(k), GTbuf(k), spart, st, fast);
      else if (p.small_sweep) launch_sweep<CfgSmall, true>(p, x.W, Ht, nv, ref2 + t0, Gbuf(k), GTbuf(k), spart, st, fast);
      else if (p.rows) launch_sweep<Cfg, true>(p, x.W, Ht, nv, ref2 + t0, Gbuf(k), GTbuf(k), spart, st, fast);
      else launch_sweep<Cfg, false>(p, x.W, Ht, nv, ref2 + t0, Gbuf(k), GTbuf(k), spart, st, fast);
    }
    OAPL_LAUNCH_CHECK();
    k_sweep_finish<<<grid1d(nv, kFinishRows), kFinishSlices * kFinishRows, 0, st>>>(
        spart, p.n_vt, p.Tp, nv, ref2 + t0, zy + t0, logq + t0, tokens + t0, V,
        logprob_out ? logprob_out + t0 : nullptr, diff + t0, nis + t0, Gbuf(k), p.width, p.n_kt_g, GTbuf(k), p.n_kt_t,
        (int*)(ws + p.off_status), fast);
    OAPL_LAUNCH_CHECK();
    return OAPL_OK;
  };

  const int64_t n_panels = (T + p.Tp - 1) / p.Tp;
  if (n_panels == 1) {
    if (int rc = sweep(0)) return rc;
    if (int rc = forward_partials(p, H, W, false, false, nullptr, ws, st, slow)) return rc;
    const LseFinish finish = finish_args(p, logq, logprob_out, nullptr, nullptr, check, ws);
    if (int rc = forward_finish(p, finish, st, slow)) return rc;
    if (int rc = objective(kNoGate, TokenFactor{nis, omp, flag}, nullptr)) return rc;
    if (int rc = recompute_panel(p, H, W, tokens, 0, Gbuf(0), GTbuf(0), ws, st, slow, p.grads_fused)) return rc;
    return panel_gradients(p, H, W, 0, Gbuf(0), GTbuf(0), dH, dW, ws, st, kNoGate, true, p.grads_fused);
  }

  auto gradients = [&](int64_t k) -> int {
    if (int rc = objective(fast, TokenFactor{nis, nullptr, nullptr}, nullptr)) return rc;
    return panel_gradients(p, H, W, k * p.Tp, Gbuf(k), GTbuf(k), dH, dW, ws, st, fast, true);
  };
  for (int64_t k = 0; k < n_panels; ++k) {
    if (int rc = sweep(k)) return rc;
    if (k >= p.n_buf - 1)
      if (int rc = gradients(k - (p.n_buf - 1))) return rc;
  }
  for (int64_t k = n_panels - (p.n_buf - 1); k < n_panels; ++k)
    if (int rc = gradients(k)) return rc;
  if (int rc = forward_partials(p, H, W, false, false, nullptr, ws, st, slow)) return rc;
  if (int rc = forward_finish(p, finish_args(p, logq, logprob_out, nullptr, nullptr, check, ws), st, slow)) return rc;
  if (int rc = objective(slow, TokenFactor{omp, nullptr, nullptr}, nullptr)) return rc;
  return backward_grads(p, H, W, tokens, dH, dW, ws, st, slow, true);
}

// fp32 calls whose logits do not give every CU a 128 x 128 tile start with one launch (k_scores_f32; 256 tokens at d = 64,
// V = 1024: whole call 39.4 us apart, 32.9 together; 700 at d = 300, V = 3000 91.9 / 87.0). Where they do, 128 x 128 tiles start
// apart: that launch has tiles of 64 x 128 (1501 tokens, d = 768, V = 8192 494 us apart, 478 in such tiles together; 1980, 545,
// 3120 245 / 255).
static bool scores_in_one_launch_f32(const Plan& p, int n_seq, int n_groups) {
  return p.dtype == OAPL_F32 && p.T > 0 && p.T <= kPanelF32 && !logits_large_f32(p.V, p.T) &&
         begin_in_one_launch(n_seq, n_groups);
}

// The two-pass schedule (and the scoring alone, without gradients).
template <class Begin, class Objective>
static int two_pass_path(const Plan& p, const Begin& begin, const void* H, const void* W, const int32_t* tokens,
                         const float* logq, float* logprob_out, void* dH, float* dW, char* ws, hipStream_t st,
                         Objective&& objective) {
  const int64_t T = p.T;
  const TokenInit init{p.bwd ? (float*)(ws + p.off_coef) : nullptr, nullptr, nullptr, 0, 0, nullptr, nullptr, nullptr};
  const bool one = scores_in_one_launch_f32(p, begin.n_seq, begin.n_groups);
  if (one) {
    float* zt = p.bwd && T <= p.Tp ? (float*)(ws + p.off_G) : nullptr;
    const EpiLseF32 epi{(float2*)(ws + p.off_fwd_partials), T, nullptr, zt, p.ldz};
    launch_scores_f32<F32Flat>(p, begin, H, W, tokens, (float*)(ws + p.off_zy), init, epi, st);
    OAPL_LAUNCH_CHECK();
  } else {
    if (int rc = launch_begin(begin, st)) return rc;
    if (int rc = gather_logits(p, H, W, tokens, init, ws, st)) return rc;
    if (int rc = forward_partials(p, H, W, false, p.bwd, nullptr, ws, st, kNoGate)) return rc;
  }
  const LseFinish finish = finish_args(p, logq, logprob_out, nullptr, nullptr, one ? tokens : nullptr, ws);
  const float* factor = p.bwd && p.dtype == OAPL_BF16 ? (const float*)(ws + p.off_omp) : nullptr;
  const bool together = finish_in_objective(p);
  if (!together)
    if (int rc = forward_finish(p, finish, st, kNoGate)) return rc;
  if (int rc = objective(kNoGate, TokenFactor{factor, nullptr, nullptr}, together ? &finish : nullptr)) return rc;
  if (!p.bwd) return OAPL_OK;
  return backward_grads(p, H, W, tokens, dH, dW, ws, st, kNoGate, false);
}

// A plan's partial sums (12 bytes per token and vocabulary split; partial results of the gradient contractions) may be
// most of a small head's workspace.  They only buy speed: a workspace that is too small for them is served with fewer, the
// least with none.  Returns the limit the plan was made with.
static int fit_splits(Plan& p, size_t have) {
  auto fewer = [&](int limit) {
    Plan q;
    if (!make_plan(q, p.T, p.d, p.V, p.n_seq, p.n_groups, p.dtype, p.bwd, p.unaligned, 0, 0, 0, limit)) return false;
    p = q;
    return true;
  };
  int limit = kAnySplits;
  if (p.bwd) {
    for (int next : {kAnySplits - 1, 8, 4, 2, 1}) {
      if (p.total <= have || !fewer(next)) break;
      limit = next;
    }
  } else if (p.dtype == OAPL_BF16) {
    // a split less frees 12 bytes per token at most
    while (p.total > have && limit > 1) {
      const int64_t now = p.fwd.splits > p.smp.splits ? p.fwd.splits : p.smp.splits, per = (p.T > 0 ? p.T : 1) * 12;
      const int64_t left = now - ((int64_t)(p.total - have) + per - 1) / per;
      const int next = (int)(left < 1 ? 1 : left < now ? left : now - 1);
      if (!fewer(next)) break;
      limit = next;
    }
  }
  return limit;
}

static int fit_forward_plan(Plan& p, const void* ws, size_t have) {
  fit_splits(p, have);
  if (ws == nullptr || ((uintptr_t)ws & 255) != 0 || have < p.total) return OAPL_ERR_WORKSPACE;
  return OAPL_OK;
}

// The plan of a loss call: the workspace the caller hands over is the budget.  Panel size first:
// the default panel (the fastest) if two buffers of it fit, else the largest that does.  Then as
// many panel buffers as fit (and the batch has panels): they decide how long a rollout the single
// sweep serves, not how fast it runs.
static int fit_plan(Plan& p, int64_t T, int d, int V, int n_seq, int n_groups, int dtype, bool bwd, unsigned unaligned,
                    const void* ws, size_t have) {
  if (!make_plan(p, T, d, V, n_seq, n_groups, dtype, bwd, unaligned)) return OAPL_ERR_SHAPE;
  if (!bwd) return fit_forward_plan(p, ws, have);
  if (ws == nullptr || ((uintptr_t)ws & 255) != 0) return OAPL_ERR_WORKSPACE;
  const int max_splits = fit_splits(p, have);
  if (p.total > have) {
    const int64_t step = dtype == OAPL_BF16 ? Cfg::BN : 64;
    bool found = false;
    for (int64_t rows = (p.Tp - 1) / step * step; rows >= step && !found; rows -= step) {
      Plan q;
      if (make_plan(q, T, d, V, n_seq, n_groups, dtype, bwd, unaligned, rows, 0, 0, max_splits) && q.total <= have) {
        p = q;
        found = true;
      }
    }
    if (!found) return OAPL_ERR_WORKSPACE;
  }
  if (p.sweep && p.n_buf >= 2) {
    const size_t per_buffer = p.size_G + p.size_GT;
    const int64_t extra = (int64_t)((have - p.total) / per_buffer);
    if (extra > 0) {
      Plan q;
      if (make_plan(q, T, d, V, n_seq, n_groups, dtype, bwd, unaligned, p.Tp, p.n_buf + extra, p.Tp, max_splits) &&
          q.total <= have)
        p = q;
    }
  }
  return OAPL_OK;
}

// Runs the objective's launch(grid, steps) once with both steps, or once with each.  The hand-over costs a fence and a counter
// for every rollout: whole calls in one launch / two, 1000 tokens at d = 256, V = 1544: 55.3 / 55.7 us for 8 rollouts, 55.5 /
// 54.8 for 32, 57.4 / 54.7 for 64, 69 / 55 for 256, 119 / 60 for 1024; fp32, 256 tokens, d = 64, V = 1024, where the host's
// launches are what the call waits for: 34.4 / 37.5 for 8, 36.1 / 37.6 for 64, 46 / 38 for 256.
constexpr int kOneLaunchRollouts = 32;
template <class Launch>
static int objective_steps(int n_seq, Launch&& launch) {
  const unsigned grid = n_seq > 0 ? n_seq : 1;
  const bool one = n_seq <= kOneLaunchRollouts;
  launch(grid, one ? kRollouts | kLoss : kRollouts);
  OAPL_LAUNCH_CHECK();
  if (!one) launch(1u, kLoss);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

static int loss_impl(const void* H, const void* W, const int32_t* tokens, const float* logq,
                     const int64_t* seq_offsets, const float* rewards, const int32_t* group_ids, int64_t T, int32_t d,
                     int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype, float beta_value, float beta_loss,
                     float loss_scale, uint32_t flags, float* loss_out, float* logprob_out, float* seq_logratio_out,
                     float* vstar_out, void* dH, float* dW, void* workspace, size_t workspace_bytes, void* stream,
                     bool checks_only = false) {
  if (dtype != OAPL_F32 && dtype != OAPL_BF16) return OAPL_ERR_DTYPE;
  if (flags & ~(uint32_t)OAPL_FLAG_TWO_PASS) return OAPL_ERR_SHAPE;
  const bool bwd = (dH != nullptr) || (dW != nullptr);
  Plan p;
  const unsigned unaligned = unaligned_operands(dtype, H, W);
  if (!make_plan(p, T, d, V, n_seq, n_groups, dtype, bwd, unaligned)) return OAPL_ERR_SHAPE;
  // gradients come as a pair; an empty batch has no dH rows, so its pointer may be NULL
  if (!W || !seq_offsets || !loss_out || (bwd && (!dW || (T > 0 && !dH)))) return OAPL_ERR_NULL;
  if (T > 0 && (!H || !tokens || !logq)) return OAPL_ERR_NULL;
  if (n_seq > 0 && (!rewards || !group_ids)) return OAPL_ERR_NULL;
  if (!(beta_value > 0.f) || !(beta_loss > 0.f) || !isfinite(beta_value) || !isfinite(beta_loss) ||
      !isfinite(loss_scale))
    return OAPL_ERR_BETA;
  if (int rc = fit_plan(p, T, d, V, n_seq, n_groups, dtype, bwd, unaligned, workspace, workspace_bytes)) return rc;
  if (checks_only) return OAPL_OK;

  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  int* status = (int*)(ws + p.off_status);
  double* vstar = (double*)(ws + p.off_vstar);
  const bool sweep = p.sweep && T >= kSweepMinTokens && !(flags & OAPL_FLAG_TWO_PASS);
  const int64_t longest = sweep ? sweep_longest(p) : -1;

  const OaplBegin begin{rewards, group_ids, seq_offsets, n_seq, n_groups, T,
                        longest, (double)beta_value, vstar, vstar_out, status};
  if (int rc = pack_operands(p, H, W, ws, st)) return rc;

  // Steps a4, a6, a7 from logprob - logq [T]
  auto objective = [&](Gate gate, TokenFactor factors, const LseFinish* finish) -> int {
    return objective_steps(n_seq, [&](unsigned grid, int steps) {
      auto run = [&](auto kernel, const auto& finish_arg) {
        kernel<<<grid, 256, 0, st>>>(
            (const double*)(ws + p.off_diff), rewards, group_ids, seq_offsets, n_seq, n_groups, T, (double)beta_loss,
            (double)loss_scale, vstar, factors, (double*)(ws + p.off_delta), bwd && T > 0 ? (float*)(ws + p.off_coef) : nullptr,
            loss_out, seq_logratio_out, status, steps, gate, finish_arg);
      };
      if (finish) run(k_oapl_objective<true>, *finish);
      else run(k_oapl_objective<false>, NoFinish{});
    });
  };
  // bf16 with gradients: one sweep over the logits; the two-pass schedule behind it runs only if the
  // sweep's preconditions fail on this call's data (decided on the device, in stream order)
  if (sweep) return sweep_path(p, begin, H, W, tokens, logq, logprob_out, dH, dW, ws, st, objective);
  return two_pass_path(p, begin, H, W, tokens, logq, logprob_out, dH, dW, ws, st, objective);
}

// The paper's baseline objective on the same fused head (Sec. 2): scores, group advantages,
// clipped importance-weighted token terms, then the same backward with other coefficients.
static int grpo_impl(const void* H, const void* W, const int32_t* tokens, const float* logq, const float* logp_old,
                     const int64_t* seq_offsets, const float* rewards, const int32_t* group_ids, int64_t T, int32_t d,
                     int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype, float clip_eps, float adv_eps,
                     float loss_scale, uint32_t flags, float* loss_out, float* logprob_out, float* adv_out, void* dH,
                     float* dW, void* workspace, size_t workspace_bytes, void* stream) {
  if (dtype != OAPL_F32 && dtype != OAPL_BF16) return OAPL_ERR_DTYPE;
  if (flags & ~(uint32_t)OAPL_FLAG_TWO_PASS) return OAPL_ERR_SHAPE;
  const bool bwd = (dH != nullptr) || (dW != nullptr);
  Plan p;
  const unsigned unaligned = unaligned_operands(dtype, H, W);
  if (!make_plan(p, T, d, V, n_seq, n_groups, dtype, bwd, unaligned)) return OAPL_ERR_SHAPE;
  if (!W || !seq_offsets || !loss_out || (bwd && (!dW || (T > 0 && !dH)))) return OAPL_ERR_NULL;
  if (T > 0 && (!H || !tokens || !logq || !logp_old)) return OAPL_ERR_NULL;
  if (n_seq > 0 && (!rewards || !group_ids)) return OAPL_ERR_NULL;
  if (!(clip_eps >= 0.f) || !(clip_eps < 1.f) || !(adv_eps >= 0.f) || !isfinite(adv_eps) || !isfinite(loss_scale))
    return OAPL_ERR_BETA;
  if (int rc = fit_plan(p, T, d, V, n_seq, n_groups, dtype, bwd, unaligned, workspace, workspace_bytes)) return rc;

  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  int* status = (int*)(ws + p.off_status);
  float* adv = (float*)(ws + p.off_cseq);
  double* gstat = (double*)(ws + p.off_vstar);          // [2 n_groups]: mean, std
  double* wseq = (double*)(ws + p.off_gw);              // [n_seq + n_groups]
  double* gsize = wseq + (n_seq > 0 ? n_seq : 1);
  const bool sweep = p.sweep && T >= kSweepMinTokens && !(flags & OAPL_FLAG_TWO_PASS);
  const int64_t longest = sweep ? sweep_longest(p) : -1;

  const GrpoBegin begin{rewards, group_ids, seq_offsets, n_seq, n_groups, T, longest, (double)adv_eps, (double)loss_scale, gstat,
                        gstat + n_groups, gsize, adv, wseq, adv_out, status};
  if (int rc = pack_operands(p, H, W, ws, st)) return rc;

  auto objective = [&](Gate gate, TokenFactor factors, const LseFinish* finish) -> int {
    return objective_steps(n_seq, [&](unsigned grid, int steps) {
      auto run = [&](auto kernel, const auto& finish_arg) {
        kernel<<<grid, 256, 0, st>>>(
            (const double*)(ws + p.off_diff), logq, logp_old, seq_offsets, n_seq, T, adv, wseq, (double)clip_eps, factors,
            bwd && T > 0 ? (float*)(ws + p.off_coef) : nullptr, (double*)(ws + p.off_delta), loss_out, status, steps, gate,
            finish_arg);
      };
      if (finish) run(k_grpo_objective<true>, *finish);
      else run(k_grpo_objective<false>, NoFinish{});
    });
  };
  if (sweep) return sweep_path(p, begin, H, W, tokens, logq, logprob_out, dH, dW, ws, st, objective);
  return two_pass_path(p, begin, H, W, tokens, logq, logprob_out, dH, dW, ws, st, objective);
}

// Scratch of the entry point that allocates nothing: every GPU the library runs on holds its own
// copy of this array, at its own address, until the process ends.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device (the array's name is only a host-side stand-in
// for it): resolved once per device, with that device current, and kept.
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mu;

static int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return OAPL_ERR_HIP;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return OAPL_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return OAPL_OK;
}

}  // namespace oapl

using namespace oapl;

extern "C" {

const char* oapl_status_string(int32_t status) {
  switch (status) {
    case OAPL_OK: return "ok";
    case OAPL_ERR_NULL: return "a required pointer is NULL";
    case OAPL_ERR_SHAPE: return "a size is non-positive or unsupported";
    case OAPL_ERR_DTYPE: return "unknown dtype";
    case OAPL_ERR_OFFSETS: return "seq_offsets malformed";
    case OAPL_ERR_GROUP: return "group id out of range or empty group";
    case OAPL_ERR_BETA: return "beta must be positive and finite (loss_scale finite)";
    case OAPL_ERR_WORKSPACE: return "workspace NULL, misaligned or too small";
    case OAPL_ERR_HIP: return "HIP launch or runtime call failed";
    case OAPL_ERR_TOKEN_RANGE: return "sampled token outside [0, V)";
    case OAPL_ERR_SCRATCH_LIMIT: return "sizes need more than the library's 64 MiB static scratch";
    default: return "unknown status";
  }
}

size_t oapl_workspace_bytes(int64_t T, int32_t d, int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype,
                            int32_t with_backward) {
  Plan p;
  if (!make_plan(p, T, d, V, n_seq, n_groups, dtype, with_backward != 0, kUnalignedAny)) return 0;
  return p.total;
}

size_t oapl_workspace_bytes_for(int64_t T, int32_t d, int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype,
                                int32_t with_backward, int64_t max_panel_rows, int64_t max_rollout_len,
                                int64_t* panel_rows_out, int32_t* panel_buffers_out) {
  Plan p, full;
  // fewer rows than a tile ask for the least workspace there is: no room for copies of operands that are not aligned
  const unsigned copies = max_panel_rows > 0 && max_panel_rows < Cfg::BN ? 0 : kUnalignedAny;
  if (!make_plan(p, T, d, V, n_seq, n_groups, dtype, with_backward != 0, copies, max_panel_rows)) return 0;
  if (!make_plan(full, T, d, V, n_seq, n_groups, dtype, with_backward != 0, copies)) return 0;
  // who asks for less than the library's own panels gets the least that does the work in panels of that size
  if (p.Tp < full.Tp)
    make_plan(p, T, d, V, n_seq, n_groups, dtype, with_backward != 0, copies, max_panel_rows, 0, 0, 1);
  // Buffers for the longest rollout, 1 + ceil(len / panel): only at the library's own panel size.  A
  // loss call derives its plan from the byte count alone, and k buffers of a smaller panel could not
  // be told from two buffers of a panel k / 2 times as large (which it prefers: larger panels are faster).
  if (max_rollout_len > p.Tp && p.n_buf >= 2 && p.Tp == full.Tp) {
    const int64_t want = 1 + (max_rollout_len + p.Tp - 1) / p.Tp;
    Plan q;
    if (!make_plan(q, T, d, V, n_seq, n_groups, dtype, with_backward != 0, copies, p.Tp, want, p.Tp)) return 0;
    p = q;
  }
  if (panel_rows_out) *panel_rows_out = p.Tp;
  if (panel_buffers_out) *panel_buffers_out = p.n_buf;
  return p.total;
}

int32_t oapl_logprob_fwd(const void* H, const void* W, const int32_t* tokens, int64_t T, int32_t d, int32_t V,
                         int32_t dtype, float* logprob_out, float* lse_out, float* entropy_out, void* workspace,
                         size_t workspace_bytes, void* stream) {
  if (dtype != OAPL_F32 && dtype != OAPL_BF16) return OAPL_ERR_DTYPE;
  Plan p;
  if (!make_plan(p, T, d, V, 0, 1, dtype, false, unaligned_operands(dtype, H, W))) return OAPL_ERR_SHAPE;
  if (!W) return OAPL_ERR_NULL;
  if (T > 0 && (!H || !tokens || !logprob_out)) return OAPL_ERR_NULL;
  if (int rc = fit_forward_plan(p, workspace, workspace_bytes)) return rc;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  int* status = (int*)(ws + p.off_status);
  if (T == 0) {
    k_fill_i32<<<1, 64, 0, st>>>(status, kStatusWords, 0);
    OAPL_LAUNCH_CHECK();
    return OAPL_OK;
  }
  if (int rc = pack_operands(p, H, W, ws, st)) return rc;
  if (int rc = forward_partials(p, H, W, entropy_out != nullptr, false, status, ws, st, kNoGate)) return rc;
  if (int rc = gather_logits(p, H, W, tokens, TokenInit{}, ws, st)) return rc;
  return forward_finish(p, finish_args(p, nullptr, logprob_out, lse_out, entropy_out, nullptr, ws), st, kNoGate);
}

int32_t oapl_sample_tokens(const void* H, const void* W, int64_t T, int32_t d, int32_t V, int32_t dtype,
                           float temperature, uint64_t seed, int32_t* tokens_out, float* score_out, void* workspace,
                           size_t workspace_bytes, void* stream) {
  if (dtype != OAPL_F32 && dtype != OAPL_BF16) return OAPL_ERR_DTYPE;
  Plan p;
  if (!make_plan(p, T, d, V, 0, 1, dtype, false, unaligned_operands(dtype, H, W))) return OAPL_ERR_SHAPE;
  if (!W) return OAPL_ERR_NULL;
  if (T > 0 && (!H || !tokens_out)) return OAPL_ERR_NULL;
  if (!(temperature > 0.f) || !isfinite(temperature)) return OAPL_ERR_BETA;
  if (int rc = fit_forward_plan(p, workspace, workspace_bytes)) return rc;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  int* status = (int*)(ws + p.off_status);
  if (T == 0) {
    k_fill_i32<<<1, 64, 0, st>>>(status, kStatusWords, 0);
    OAPL_LAUNCH_CHECK();
    return OAPL_OK;
  }
  float2* partials = (float2*)(ws + p.off_partials);
  const float inv_t = 1.0f / temperature;
  if (dtype == OAPL_BF16) {
    if (!prepare_kernels()) return OAPL_ERR_HIP;
    if (int rc = copy_unaligned(p, H, W, ws, st)) return rc;
    FwdArgs args{(const bf16_t*)W, (const bf16_t*)H, V, T, d, p.n_kt_d, p.smp};
    if (!p.rows) {
      bf16_t* Wp = (bf16_t*)(ws + p.off_Wp);
      bf16_t* Hp = (bf16_t*)(ws + p.off_Hp);
      k_pack_rows<<<dim3(p.n_kt_d, p.n_rt_v), 256, 0, st>>>(args.W, V, d, d, Wp, p.n_kt_d, Cfg::BM);
      OAPL_LAUNCH_CHECK();
      const int rb = p.smp.tile == kTile256 ? Cfg256::BN : Cfg::BN;
      k_pack_rows<<<dim3(p.n_kt_d, grid1d(T, rb)), 256, 0, st>>>(args.H, T, d, d, Hp, p.n_kt_d, rb);
      OAPL_LAUNCH_CHECK();
      args.W = Wp;
      args.H = Hp;
    }
    {
      ScopedKernelTimer tm(kFwdSample, st);
      launch_sample(args, p.rows, inv_t, seed, partials, st);
    }
    OAPL_LAUNCH_CHECK();
  } else {
    launch_logits_f32(p, H, W, T, EpiSampleF32{partials, T, inv_t, (uint32_t)seed, (uint32_t)(seed >> 32)}, st);
    OAPL_LAUNCH_CHECK();
  }
  const int slices = finish_slices(p.smp.splits);
  k_sample_finish<<<grid1d(T, 256 / slices), 256, 0, st>>>(partials, p.smp.splits, T, tokens_out, score_out, slices, status);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

int32_t oapl_loss_fwd_bwd(const void* H, const void* W, const int32_t* tokens, const float* logq,
                          const int64_t* seq_offsets, const float* rewards, const int32_t* group_ids, int64_t T,
                          int32_t d, int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype, float beta,
                          float loss_scale, float* loss_out, float* logprob_out, float* seq_logratio_out,
                          float* vstar_out, void* dH, float* dW, void* workspace, size_t workspace_bytes,
                          void* stream) {
  return loss_impl(H, W, tokens, logq, seq_offsets, rewards, group_ids, T, d, V, n_seq, n_groups, dtype, beta, beta,
                   loss_scale, 0u, loss_out, logprob_out, seq_logratio_out, vstar_out, dH, dW, workspace,
                   workspace_bytes, stream);
}

int32_t oapl_loss_fwd_bwd_two_beta(const void* H, const void* W, const int32_t* tokens, const float* logq,
                                   const int64_t* seq_offsets, const float* rewards, const int32_t* group_ids,
                                   int64_t T, int32_t d, int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype,
                                   float beta_value, float beta_loss, float loss_scale, uint32_t flags,
                                   float* loss_out, float* logprob_out, float* seq_logratio_out, float* vstar_out,
                                   void* dH, float* dW, void* workspace, size_t workspace_bytes, void* stream) {
  return loss_impl(H, W, tokens, logq, seq_offsets, rewards, group_ids, T, d, V, n_seq, n_groups, dtype, beta_value,
                   beta_loss, loss_scale, flags, loss_out, logprob_out, seq_logratio_out, vstar_out, dH, dW, workspace,
                   workspace_bytes, stream);
}

int32_t oapl_loss_fwd_bwd_noalloc(const void* H, const void* W, const int32_t* tokens, const float* logq,
                                  const int64_t* seq_offsets, const float* rewards, const int32_t* group_ids,
                                  int64_t T, int32_t d, int32_t V, int32_t n_seq, int32_t n_groups, int32_t dtype,
                                  float beta, float loss_scale, float* loss_out, float* logprob_out,
                                  float* seq_logratio_out, float* vstar_out, void* dH, float* dW, void* stream) {
  // every host-side check first, against an aligned stand-in of the scratch's size; nothing is launched
  int rc = loss_impl(H, W, tokens, logq, seq_offsets, rewards, group_ids, T, d, V, n_seq, n_groups, dtype, beta, beta,
                     loss_scale, 0u, loss_out, logprob_out, seq_logratio_out, vstar_out, dH, dW, (void*)(uintptr_t)256,
                     kStaticScratchBytes, stream, true);
  if (rc == OAPL_ERR_WORKSPACE) return OAPL_ERR_SCRATCH_LIMIT;
  if (rc != OAPL_OK) return rc;
  void* ws = nullptr;
  if ((rc = static_scratch(&ws)) != OAPL_OK) return rc;
  return loss_impl(H, W, tokens, logq, seq_offsets, rewards, group_ids, T, d, V, n_seq, n_groups, dtype, beta, beta,
                   loss_scale, 0u, loss_out, logprob_out, seq_logratio_out, vstar_out, dH, dW, ws, kStaticScratchBytes,
                   stream);
}

int32_t oapl_grpo_loss_fwd_bwd(const void* H, const void* W, const int32_t* tokens, const float* logq,
                               const float* logp_old, const int64_t* seq_offsets, const float* rewards,
                               const int32_t* group_ids, int64_t T, int32_t d, int32_t V, int32_t n_seq,
                               int32_t n_groups, int32_t dtype, float clip_eps, float adv_eps, float loss_scale,
                               uint32_t flags, float* loss_out, float* logprob_out, float* adv_out, void* dH,
                               float* dW, void* workspace, size_t workspace_bytes, void* stream) {
  return grpo_impl(H, W, tokens, logq, logp_old, seq_offsets, rewards, group_ids, T, d, V, n_seq, n_groups, dtype,
                   clip_eps, adv_eps, loss_scale, flags, loss_out, logprob_out, adv_out, dH, dW, workspace, workspace_bytes,
                   stream);
}

int32_t oapl_segmented_sum_f32(const float* x, const int64_t* seq_offsets, int32_t n_seq, double* out, void* stream) {
  if (n_seq < 0) return OAPL_ERR_SHAPE;
  if (n_seq == 0) return OAPL_OK;
  if (!x || !seq_offsets || !out) return OAPL_ERR_NULL;
  k_segmented_sum<float><<<n_seq, 256, 0, (hipStream_t)stream>>>(x, seq_offsets, n_seq, out);
  OAPL_LAUNCH_CHECK();
  return OAPL_OK;
}

int32_t oapl_timing_enable(int32_t enable) {
  TimingState& t = timing();
  std::lock_guard<std::mutex> g(t.mu);
  for (auto& v : t.ev) {
    for (auto& e : v) {
      (void)hipEventDestroy(e.first);
      (void)hipEventDestroy(e.second);
    }
    v.clear();
  }
  t.on = enable != 0;
  return OAPL_OK;
}

int32_t oapl_timing_read(int32_t kernel, double* total_ms, int64_t* launches) {
  if (kernel < 0 || kernel >= kNumDense) return OAPL_ERR_SHAPE;
  if (!total_ms || !launches) return OAPL_ERR_NULL;
  TimingState& t = timing();
  std::lock_guard<std::mutex> g(t.mu);
  double sum = 0.0;
  for (auto& e : t.ev[kernel]) {
    if (hipEventSynchronize(e.second) != hipSuccess) return OAPL_ERR_HIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, e.first, e.second) != hipSuccess) return OAPL_ERR_HIP;
    sum += ms;
  }
  *total_ms = sum;
  *launches = (int64_t)t.ev[kernel].size();
  return OAPL_OK;
}

int32_t oapl_read_path_taken(const void* workspace, void* stream, int32_t* two_pass_out) {
  if (!workspace || !two_pass_out) return OAPL_ERR_NULL;
  if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return OAPL_ERR_HIP;
  int32_t v = 0;
  if (hipMemcpy(&v, (const int32_t*)workspace + kFlagWord, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess)
    return OAPL_ERR_HIP;
  *two_pass_out = v != 0;
  return OAPL_OK;
}

int32_t oapl_read_device_status(const void* workspace, void* stream, int32_t* status_out) {
  if (!workspace || !status_out) return OAPL_ERR_NULL;
  if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return OAPL_ERR_HIP;
  int32_t v = 0;
  if (hipMemcpy(&v, workspace, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess) return OAPL_ERR_HIP;
  *status_out = v;
  return OAPL_OK;
}

}  // extern "C"
