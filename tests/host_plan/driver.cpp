// The library's host code (plans, launch grids) behind a line protocol: one query per line of stdin, one line of
// key=value pairs per answer.  Compiled for the host alone; nothing is launched.
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "../../paper_2602_19362_amd/csrc/oapl_api.hip"

// workgroups of a contraction with an M x N result (one split of k)
static long long groups(bool small, int64_t M, int64_t N) {
  return (long long)(small ? tile_count<CfgSmall>(M, N) : tile_count<Cfg>(M, N));
}

int main() {
  char line[256];
  while (std::fgets(line, sizeof line, stdin)) {
    int n_seq = 0, n_groups = 0, d = 0, V = 0, dtype = 0, bwd = 0;
    long long T = 0, cap = 0, have = 0;
    unsigned unaligned = 0;
    if (std::sscanf(line, "begin %d %d", &n_seq, &n_groups) == 2) {
      std::printf("one=%d grid=%u\n", begin_in_one_launch(n_seq, n_groups) ? 1 : 0, begin_grid(n_seq, n_groups));
    } else if (std::sscanf(line, "objective %d", &n_seq) == 1) {
      // the first launch of the objective: workgroups, and how many of them hand over to the last one
      unsigned first = 0, hand_over = 0;
      objective_steps(n_seq, [&](unsigned grid, int steps) {
        if (first == 0) { first = grid; hand_over = steps == (kRollouts | kLoss) ? grid : 0; }
      });
      std::printf("grid=%u hand_over=%u\n", first, hand_over);
    } else if (std::sscanf(line, "shared_dw %d %d", &d, &V) == 2) {
      // dW's workgroups in the launch that they share with dH's: tiles, tiles taken once, most tiles on one of the 8 XCDs
      const int n = (int)tile_count<CfgSmall>(d, V);
      std::vector<int> taken(n, 0);
      int on[8] = {}, once = 0, most = 0;
      for (int b = 0; b < (int)round_up(n, 8); ++b) {
        const int tile = shared_dw_tile(b, n);
        if (tile < n) { ++taken[tile]; ++on[b & 7]; }
      }
      for (int t : taken) once += t == 1;
      for (int x : on) most = x > most ? x : most;
      std::printf("tiles=%d once=%d most=%d\n", n, once, most);
    } else if (std::sscanf(line, "walks %d %d %d", &V, &n_seq, &n_groups) == 3) {
      // n_seq balanced ranges of V rows in tiles of 128, 256 or 320 rows: gaps between them, tiles that are empty or too high,
      // rows of the longest and the shortest
      int at = 0, wrong = 0, most = 0, least = V;
      for (int k = 0; k < n_seq; ++k) {
        const RowWalk w = n_groups == 128   ? row_walk<Cfg128>(V, k, n_seq, 1)
                          : n_groups == 256 ? row_walk<Cfg256>(V, k, n_seq, 1)
                                            : row_walk<Cfg256Tall>(V, k, n_seq, 1);
        wrong += w.r0 != at || w.r0 % 16 != 0 || w.h < 1 || w.h > n_groups || w.h % 16 != 0;
        wrong += w.r0 >= w.r1 || (w.r1 - w.r0 + w.h - 1) / w.h != (w.r1 - w.r0 + n_groups - 1) / n_groups;
        at = w.r1;
        most = w.r1 - w.r0 > most ? w.r1 - w.r0 : most;
        least = w.r1 - w.r0 < least ? w.r1 - w.r0 : least;
      }
      std::printf("wrong=%d end=%d most=%d least=%d\n", wrong, at, most, least);
    } else if (std::sscanf(line, "f32grid %lld", &T) == 1) {
      // the launch of T tiles: workgroups, and the most threads in a dimension
      const dim3 g = f32_grid(T);
      const long long x = (long long)g.x * F32Wide::NT, y = g.y, z = g.z;
      std::printf("tiles=%lld most=%lld rest=%d\n", (long long)g.x * y * z, x > y ? x : y, (int)(g.x % 8));
    } else if (std::sscanf(line, "finish %lld %d %d", &T, &V, &n_seq) == 3) {
      // an fp32 loss call's log-probs: in the objective's launch?
      Plan p;
      const bool ok = make_plan(p, T, 64, V, n_seq, 1, OAPL_F32, true, 0);
      std::printf("ok=%d together=%d\n", ok, finish_in_objective(p));
    } else if (std::sscanf(line, "plan %lld %d %d %d %d %lld %u %lld", &T, &d, &V, &dtype, &bwd, &cap, &unaligned, &have) == 8) {
      // the plan of a call of one rollout on `have` bytes (< 0: what the library asks for with panels of `cap` rows)
      if (have < 0) have = (long long)oapl_workspace_bytes_for(T, d, V, 1, 1, dtype, bwd, cap, 0, nullptr, nullptr);
      Plan p;
      const int rc = fit_plan(p, T, d, V, 1, 1, dtype, bwd != 0, unaligned, (void*)(uintptr_t)256, (size_t)have);
      std::printf("rc=%d have=%lld total=%lld rows=%d copies=%u panel=%lld buffers=%d fwd_tile=%d fwd_early=%d fwd_splits=%d "
                  "smp_splits=%d smp_tile=%d once=%d even=%d tall=%d smp_even=%d smp_tall=%d",
                  rc, have, (long long)p.total, p.rows ? 1 : 0, p.unaligned, (long long)p.Tp, p.n_buf, (int)p.fwd.tile,
                  p.fwd.tile == kTile256 && (once_pays(T, V, d) || (!p.fwd.tall && early_pays(T, V, d))), p.fwd.splits,
                  p.smp.splits, (int)p.smp.tile, p.rows && once_pays(T, V, d), p.fwd.balanced, p.fwd.tall, p.smp.balanced,
                  p.smp.tall);
      const int64_t last = T > 0 ? T - (T - 1) / p.Tp * p.Tp : 0;   // rows of the last panel
      if (dtype == OAPL_BF16)
        std::printf(" width=%d small_sweep=%d small_dw=%d dh_small=%d dh_splits=%d sweep_groups=%lld dw_groups=%lld "
                    "dh_groups=%lld ref_splits=%d\n",
                    p.width, p.small_sweep, p.small_dw, p.dh.small, p.dh.splits, groups(p.small_sweep, V, last),
                    groups(p.small_dw, d, V), groups(p.dh.small, d, last) * p.dh.splits, p.sweep ? ref_splits(p) : 0);
      else
        std::printf(" logits_large=%d dh_large=%d dh_splits=%d dw_large=%d dw_splits=%d wide_dh=%d wide_dw=%d\n",
                    logits_large_f32(V, T < p.Tp ? T : p.Tp), p.f32_dh.large, p.f32_dh.splits, p.f32_dw.large, p.f32_dw.splits,
                    p.wide_dh, p.wide_dw);
    } else {
      std::printf("unknown query\n");
      return 1;
    }
  }
  return 0;
}
