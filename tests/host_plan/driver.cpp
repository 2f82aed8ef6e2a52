// The library's host code (plans, launch grids) behind a line protocol: one query per line of stdin, one line of
// key=value pairs per answer.  Compiled for the host alone; nothing is launched.
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "../../paper_2602_19362_amd/csrc/oapl_api.hip"

int main() {
  char line[256];
  while (std::fgets(line, sizeof line, stdin)) {
    int n_seq = 0, n_groups = 0;
    if (std::sscanf(line, "begin %d %d", &n_seq, &n_groups) == 2) {
      std::printf("one=%d grid=%u\n", begin_in_one_launch(n_seq, n_groups) ? 1 : 0, begin_grid(n_seq, n_groups));
    } else {
      std::printf("unknown query\n");
      return 1;
    }
  }
  return 0;
}
