// Autotuned tile configurations of the digit form (host code).
#pragma once
#include <stdint.h>

#include <map>
#include <utility>

namespace hfe {
using TunedTiles = std::map<std::pair<int, int64_t>, int>;  // (level, column bucket) -> configuration

// Calls of up to this many columns fill one tile of the narrow configuration, whose products then hide behind the reading
// of the database; more columns are more of its tiles, at half the rows' reuse (13,097 rows, K = 13,696 in three
// primes: 16 columns 0.49 ms against 0.70 in the default's 64-column tile, 512 columns 5.95 against 5.14).  So they and
// larger calls have entries of their own.
constexpr int64_t kNarrowCols = 32;

constexpr int64_t tune_bucket(int64_t d3) {
  int64_t b = kNarrowCols;
  while (b < d3) b <<= 1;
  return b;
}

// The entry of this level with the nearest bucket on d3's side of kNarrowCols, else `untuned`.
inline int tuned_tile(const TunedTiles& tuned, int level, int64_t d3, int untuned) {
  const int64_t b = tune_bucket(d3);
  int best = untuned;
  int64_t best_dist = -1;
  for (const auto& kv : tuned) {
    const int64_t k = kv.first.second;
    if (kv.first.first != level || k <= 0 || (k <= kNarrowCols) != (b <= kNarrowCols)) continue;
    const int64_t dist = k > b ? k / b : b / k;
    if (best_dist < 0 || dist < best_dist) {
      best_dist = dist;
      best = kv.second;
    }
  }
  return best;
}
}  // namespace hfe
