// Prints the runs of a camera: row_runs HEIGHT LANES M BLOCKS, one line per run
// of (row0, row1, stride) as the kernels with statistics take it, then of the
// contiguous split that the table form takes.
#include <cstdio>
#include <cstdlib>

#include "../../paper_1910_03517_amd/csrc/apply_split.h"

int main(int argc, char** argv) {
  if (argc != 5) return 1;
  const int H = std::atoi(argv[1]), lanes = std::atoi(argv[2]), m = std::atoi(argv[3]), nb = std::atoi(argv[4]);
  const int steps = (H + lanes - 1) / lanes;
  for (int form = 0; form < 2; ++form)
    for (int i = 0; i < m; ++i) {
      const rc::RowRun r = rc::row_run(H, lanes, i, m, form == 0 && rc::runs_interleave(steps, m, nb));
      std::printf("%d %d %d\n", r.row0, r.row1, r.stride);
    }
  return 0;
}
