// Prints first[0 .. n] of split_shares: shares ACTIVE BYTES:STEPS ...
#include <cstdio>
#include <cstdlib>

#include "../../paper_1910_03517_amd/csrc/apply_split.h"

int main(int argc, char** argv) {
  const int n = argc - 2;
  if (n < 1 || n > 64) return 1;
  int64_t bytes[64];
  int32_t steps[64];
  for (int k = 0; k < n; ++k) {
    char* colon = nullptr;
    bytes[k] = std::strtoll(argv[2 + k], &colon, 10);
    steps[k] = std::atoi(colon + 1);
  }
  uint16_t first[65];
  const int w = rc::split_shares(n, bytes, steps, std::strtoull(argv[1], nullptr, 10), first);
  for (int k = 0; k <= n; ++k) std::printf("%d ", first[k]);
  return w == first[n] ? 0 : 2;
}
