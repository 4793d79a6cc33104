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
// block costs kSetup steps to start and finish, so a launch takes about
// ceil(tiles * splits / kSlots) * (per_split + kSetup) steps.  Splitting adds
// two small launches and the counters' atomics, so it has to promise a tenth.
// Measured, one block per tile against split: 128x128, 1 isovalue, 2000
// samples (16 tiles) 2215 against 71 us; 721x1440, 8 isovalues, 1000 samples
// (1035 tiles, 11 past a full round) 2513 against 2030 us.
struct McSplit {
  int splits, per_split;
};

inline McSplit mc_split_by_rounds(int64_t tiles, int steps) {
  constexpr int64_t kSlots = 1024, kSetup = 4, kMaxSplits = 256;
  McSplit best{1, steps};
  const double whole = double((tiles + kSlots - 1) / kSlots) * double(int64_t(steps) + kSetup);
  double least = 0.9 * whole - 4.0;
  for (int64_t z = 2; z <= kMaxSplits && z * kSetup <= steps; ++z) {
    const int per = int((steps + z - 1) / z);
    const int64_t used = (steps + per - 1) / per;  // splits that have work
    const double cost = double((tiles * used + kSlots - 1) / kSlots) * double(per + kSetup);
    if (cost < least) {
      least = cost;
      best = {int(used), per};
    }
  }
  return best;
}

// Many isovalues: the atomics are a larger part, and a lone round of blocks
// that share a CU hides more of the others' waits than it costs them, so the
// split above is taken only where it beats whole blocks by a closer count.  With
// q blocks a CU, `resident` of them at once, a launch takes (per_split + start)
// steps times 1 + share (r - 1) for each round of r blocks, plus the two launches
// and the atomics per 1000 tiles, splits and isovalues, in steps of a lone block.
// The constants decide all but 2 of 2000 random grids (33 to 1500 a side, 7 to 2000
// samples) within 3% of the better of both; without them 721x1440 at 16 isovalues,
// 60 samples, takes 237 us for 201, 721x700 by vertices 108 for 83.  Ends of more
// steps in the rounds above instead refused splits that pay: 9 isovalues by
// vertices 33 tiles of 71 samples 113 us for 29, 1040x1040 at 333 640 for 549.
struct McCosts {
  int resident;
  double share, start, atomics, launches;
};

constexpr McCosts mc_costs(int kc, bool vertex) {
  return kc <= 8  ? McCosts{4, 0.064, 1.0, 0.693, 0.95}
         : vertex ? McCosts{5, 0.479, 0.0, 0.237, 2.35}
                  : McCosts{4, 0.072, 0.0, 0.572, 3.6};
}

inline McSplit mc_split(int64_t tiles, int steps, int kc, bool vertex) {
  const McSplit split = mc_split_by_rounds(tiles, steps);
  if (split.splits == 1 || kc <= 4 || (kc <= 8 && vertex)) return split;
  constexpr int64_t kCus = 256;
  const McCosts c = mc_costs(kc, vertex);
  auto cost = [&](int64_t splits, int per) {
    const int64_t q = (tiles * splits + kCus - 1) / kCus;
    const int64_t last = q % c.resident;
    const double rounds = double(q / c.resident) * (1.0 + c.share * (c.resident - 1)) +
                          (last ? 1.0 + c.share * double(last - 1) : 0.0);
    return (double(per) + c.start) * rounds;
  };
  const double added = c.launches + c.atomics * double(tiles * split.splits) * kc / 1000.0;
  if (cost(1, steps) <= cost(split.splits, split.per_split) + added) return {1, steps};
  return split;
}

}  // namespace pdiv
