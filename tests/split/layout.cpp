// Prints the columns and rows of a workgroup of 512 threads (lay_rows) and the
// workgroups of a rig of this one camera: layout GROUPS HEIGHT SHARE MAX_LANES.
#include <cstdio>
#include <cstdlib>

#include "../../paper_1910_03517_amd/csrc/apply_split.h"

int main(int argc, char** argv) {
  if (argc != 5) return 1;
  const int height = std::atoi(argv[2]);
  int32_t cols = 0, lanes = 0;
  rc::lay_rows(std::atoi(argv[1]), height, std::atoi(argv[3]), std::atoi(argv[4]), 512, &cols, &lanes);
  std::printf("%d %d %d\n", cols, lanes, rc::split_total((height + lanes - 1) / lanes));
  return 0;
}
