// The Monte Carlo launch's sample arithmetic, the parts that are plain C++:
// the steps a sample count takes and how they are split over blocks.
#pragma once

#include <cstdint>

namespace pdiv {

// Steps of n >= 1 samples: pairs (vector sampling) or groups of four (vertex
// sampling), the last one short or whole.  Formed without n + 1 or n + 3,
// which pass the int range at the largest counts, 2^31 - 1 and 2^31 - 3 up.
constexpr int mc_pairs(int n) { return ((n - 1) >> 1) + 1; }
constexpr int mc_groups(int n) { return ((n - 1) >> 2) + 1; }

// How the samples of a launch are split over blocks.  A block walks its
// tile's sample steps (pairs, or groups of four) one after another, so a grid
// of few tiles leaves most of the chip idle, and one of just over a multiple
// of the resident blocks runs a nearly empty last round.  `splits` blocks per
// tile share the steps; kSlots blocks run at once (4 per CU on 256 CUs) and a
// block costs some steps to start and finish, more where it adds its counts to
// the map by atomics at 8 and 16 slots (1035 tiles, 100 samples, 16 isovalues: 313,
// 320, 339, 365 us with 1 to 4 splits), so a launch takes about
// ceil(tiles * splits / kSlots) * (per_split + end) steps.  Splitting adds two
// small launches, so it has to promise a tenth.
// Measured, one block per tile against split: 128x128, 1 isovalue, 2000
// samples (16 tiles) 2215 against 71 us; 721x1440, 8 isovalues, 1000 samples
// (1035 tiles, 11 past a full round) 2513 against 2103 us.  With ends of 4 steps
// at every count and mode, 16 isovalues lost: 721x1440, 60 samples, 201 -> 278 us,
// 721x700 by vertices 83 -> 108.
struct McSplit {
  int splits, per_split;
};

inline McSplit mc_split(int64_t tiles, int steps, int slots, bool vertex) {
  constexpr int64_t kSlots = 1024, kShortest = 4, kMaxSplits = 256;
  const int whole_end = slots >= 16 ? 2 : 4;
  const int split_end = slots < 8 ? 4 : slots == 8 ? 5 : vertex ? 10 : 6;
  McSplit best{1, steps};
  const double whole = double((tiles + kSlots - 1) / kSlots) * double(steps + whole_end);
  double least = 0.9 * whole - 4.0;
  for (int64_t z = 2; z <= kMaxSplits && z * kShortest <= steps; ++z) {
    const int per = int((steps + z - 1) / z);
    const int64_t used = (steps + per - 1) / per;  // splits that have work
    const double cost = double((tiles * used + kSlots - 1) / kSlots) * double(per + split_end);
    if (cost < least) {
      least = cost;
      best = {int(used), per};
    }
  }
  return best;
}

}  // namespace pdiv
