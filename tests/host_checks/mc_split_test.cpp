// Host check of the Monte Carlo launch's sample arithmetic
// (csrc/mc_split.hpp, the header the library compiles), up to the largest
// sample count a call accepts (2^31 - 1): every sample has its step, no step
// is empty, and a split's runs cover the steps once, in int arithmetic that
// stays in range (the kernel forms a run's end as first + per_split).
// Built with g++ under ASan/UBSan.
#include <cstdio>
#include <initializer_list>

#include "../../paper_2510_01190_amd/csrc/mc_split.hpp"

namespace {

int failures = 0;

void check(bool ok, const char* what, long long a, long long b) {
  if (!ok) {
    if (failures < 20) std::printf("FAIL %s (%lld, %lld)\n", what, a, b);
    ++failures;
  }
}

void check_samples(int n) {
  for (int per : {2, 4}) {
    const int64_t steps = per == 2 ? pdiv::mc_pairs(n) : pdiv::mc_groups(n);
    check(steps * per >= n && (steps - 1) * per < n, "steps", n, per);
    for (int64_t tiles : {1LL, 2LL, 16LL, 169LL, 1023LL, 1035LL, 5000LL, 1LL << 26}) {
      const int slots = n % 3 == 0 ? 16 : n % 3 == 1 ? 8 : 1;
      const pdiv::McSplit s = pdiv::mc_split(tiles, int(steps), slots, per == 4);
      check(s.splits >= 1 && s.splits <= 256 && s.per_split >= 1, "split range", tiles, n);
      check(int64_t(s.splits) * s.per_split >= steps, "steps covered", tiles, n);
      check(int64_t(s.splits - 1) * s.per_split < steps, "no empty run", tiles, n);
      const int last_first = (s.splits - 1) * s.per_split;  // as the last block forms it
      const int end = last_first + s.per_split;
      check(end >= last_first, "run end", tiles, n);
    }
  }
}

// Where a split lost to whole blocks (us, whole and split as noted), and where
// it must stay.
void check_choices() {
  check(pdiv::mc_split(1035, 30, 16, false).splits == 1, "201 / 237 us", 1035, 30);
  check(pdiv::mc_split(1035, 50, 16, false).splits == 1, "313 / 320 us", 1035, 50);
  check(pdiv::mc_split(1089, 30, 16, false).splits == 1, "238 / 258 us", 1089, 30);
  check(pdiv::mc_split(1035, 30, 8, false).splits <= 2, "170 / 188 us with 3", 1035, 30);
  check(pdiv::mc_split(506, 15, 16, true).splits == 1, "83 / 108 us", 506, 15);
  check(pdiv::mc_split(256, 15, 16, true).splits <= 2, "70 / 75 us with 3", 256, 15);
  check(pdiv::mc_split(16, 1000, 1, false).splits >= 48, "2215 / 71 us", 16, 1000);
  check(pdiv::mc_split(1035, 500, 8, false).splits >= 4, "2513 / 2103 us", 1035, 500);
  check(pdiv::mc_split(1035, 500, 16, false).splits >= 4, "2699 / 2374 us", 1035, 500);
  // short splits of few tiles and many isovalues
  check(pdiv::mc_split(33, 18, 9, true).splits == 4, "113 / 29 us", 33, 18);
  check(pdiv::mc_split(21, 15, 9, true).splits == 3, "110 / 37 us", 21, 15);
  check(pdiv::mc_split(57, 13, 9, false).splits == 3, "77 / 27 us", 57, 13);
  check(pdiv::mc_split(44, 13, 16, false).splits == 3, "79 / 29 us", 44, 13);
  check(pdiv::mc_split(1089, 84, 9, true).splits == 4, "640 / 549 us", 1089, 84);
  check(pdiv::mc_split(1089, 50, 9, false).splits == 3, "349 / 309 us", 1089, 50);
  check(pdiv::mc_split(16, 167, 8, false).splits >= 24, "49 / 42 us with 16", 16, 167);
}

}  // namespace

int main() {
  check_choices();
  for (int n = 1; n <= 3000; ++n) check_samples(n);
  for (int n : {65535, 65536, 1000003, 1 << 30, (1 << 30) + 1}) check_samples(n);
  for (int d = 0; d < 9; ++d) check_samples(0x7fffffff - d);
  if (failures == 0) std::printf("ALL PASS\n");
  return failures != 0;
}
