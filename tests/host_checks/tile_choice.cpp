// Prints which tile the closed-form launcher takes (1: paired, 0: split), by
// the library's own rule (csrc/launch_rules.hpp):
//   tile_choice FUSED LINES BYTES SLOTS NY NX
#include <cstdio>
#include <cstdlib>

#include "../../paper_2510_01190_amd/csrc/launch_rules.hpp"

int main(int argc, char** argv) {
  if (argc != 7) return 2;
  long long a[6];
  for (int i = 0; i < 6; ++i) a[i] = std::atoll(argv[i + 1]);
  std::printf("%d\n", pdiv::use_paired_tile(a[0] != 0, a[1] != 0, int(a[2]), int(a[3]), a[4], a[5]));
  return 0;
}
