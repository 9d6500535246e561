// How many parts a contraction's K-blocks are cut into (host code).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace hfe {
// What a part costs its workgroups beside its K-blocks, in K-blocks of the form's tile: the prologue, the epilogue, its
// residues written and read back by launch_add_parts, and that a chip filled with parts runs each workgroup slower than
// one that is partly empty.  The last is most of it where the products are many: few columns, which are mostly padding
// to the tile and take little power, have an edge of their own.
constexpr int edge_i8(int64_t) { return 10; }
constexpr int edge_p2(int64_t cols) { return cols <= 32 ? 17 : 35; }
constexpr int edge_rns(int64_t cols) { return cols <= 96 ? 28 : 60; }
constexpr size_t kMaxPartBytes = 256u << 20;

// Parts for `tiles` workgroups on `cus` CUs (two workgroups of a CU share its matrix cores and its path to memory, so a
// CU counts once whatever it holds) and results of `bytes` in all: each part's workgroups give residues of their own,
// and one pass adds them (launch_add_parts).  The model, rounds of the chip times K-blocks and edge of a part, ranks
// the measured times; a further part has to shorten it by 5%, about half of which is seen.  K = 8,192 (128 K-blocks):
//   digit, 52 workgroups, 48 columns: 232 us, in 4 parts 93, in 5 150 (a second round)
//   RNS, 154 workgroups, 200 columns: 105 us, in 3 parts 141; 286, 16 columns: 143, in 2 129; 256 columns: 231, in 3 300
//   RNS, 561 workgroups of 76 K-blocks, 1 column: 137 us, in 2 parts 129; 20 columns: 140 and 140; 64: 152 and 167
//   n^2, 156 workgroups, 128 columns: 180 us, in 3 parts 199; 16 columns: 157 and 151
// and K = 20,992 (328):
//   digit, 2.03 rounds: 2.25 ms, in 2 parts 2.10; 4.06 rounds: 3.98 and 3.80; 5.03 rounds: 4.87 and 4.76, in 11, where
//   the chain of K-blocks alone is shortest, 5.38 with 925 MB of parts
//   n^2, 2.46 rounds: 1.44 ms, in 2 parts 1.36; 4.78 rounds: 2.62 and 2.71; RNS, 4 rounds and more: none pays
inline int gemm_splits(int64_t tiles, int64_t cus, int64_t KB, int edge, size_t bytes) {
  if (tiles <= 0 || cus <= 0) return 1;
  auto cost = [&](int64_t s) { return (double)((tiles * s + cus - 1) / cus) * ((double)KB / (double)s + edge); };
  const int most = tiles > cus ? 4 : 16;
  int best = 1;
  for (int s = 2; s <= most && s * 16 <= KB && (size_t)s <= kMaxPartBytes / (bytes ? bytes : 1); ++s)
    if (cost(s) < 0.95 * cost(best)) best = s;
  return best;
}
}  // namespace hfe
