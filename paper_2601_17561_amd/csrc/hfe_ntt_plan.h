// The shape of the register-resident transforms (hfe_ntt_reg.h) and the order of the transform domain, for host
// and device code.
#pragma once
#include <hip/hip_runtime.h>

namespace hfe {
// Stages per round of a transform of degree 2^L with 2^e values per thread, and the exchange after it: place
// i + (i >> sh) pad of index i, chosen with a bank model (32 lanes of 8 bytes over 64 banks) so that neither
// side of an exchange meets a bank conflict.
struct NttPlan {
  int n, s[4], sh[3], pad[3];
};
constexpr NttPlan ntt_plan(int L, int e) {
  return L == 14 && e == 5   ? NttPlan{3, {5, 5, 4, 0}, {9, 5, 0}, {16, 1, 0}}
         : L == 14 && e == 4 ? NttPlan{4, {4, 4, 3, 3}, {10, 6, 3}, {0, 8, 1}}
         : L == 13 && e == 5 ? NttPlan{3, {5, 4, 4, 0}, {8, 4, 0}, {16, 1, 0}}
         : L == 13 && e == 4 ? NttPlan{4, {4, 3, 3, 3}, {9, 6, 3}, {0, 8, 1}}
         : L == 11 && e == 3 ? NttPlan{4, {3, 3, 3, 2}, {8, 5, 4}, {0, 4, 1}}
         : L == 10 && e == 3 ? NttPlan{4, {3, 3, 2, 2}, {5, 5, 2}, {4, 4, 1}}
         : L == 12           ? NttPlan{3, {4, 4, 4, 0}, {8, 4, 0}, {16, 1, 0}}
         : L == 11           ? NttPlan{3, {4, 4, 3, 0}, {7, 5, 0}, {8, 1, 0}}
         : L == 10           ? NttPlan{3, {4, 3, 3, 0}, {6, 3, 0}, {8, 1, 0}}
                             : NttPlan{3, {3, 3, 3, 0}, {6, 3, 0}, {8, 1, 0}};
}
constexpr int ntt_def_e(int L) { return L >= 13 ? 5 : L >= 10 ? 4 : 3; }
constexpr int kRegLogMin = 9, kRegLogMax = 14;

// The bit-reversed point that index i (r TH + t) of the transform domain holds, in by_ntt's order (acc = false) or
// by_ntt_acc's, and the index of a point.
__host__ __device__ constexpr int ntt_e(int logn, bool acc) {
  return acc && logn >= 13 ? 4 : acc && (logn == 10 || logn == 11) ? 3 : ntt_def_e(logn);
}
__host__ __device__ inline int ntt_point(int logn, bool acc, int i) {
  if (logn < kRegLogMin || logn > kRegLogMax) return i;
  const int e = ntt_e(logn, acc), lt = logn - e;
  const NttPlan p = ntt_plan(logn, e);
  const int s = p.s[p.n - 1], r = i >> lt, t = i & ((1 << lt) - 1);
  return ((t + ((r >> s) << lt)) << s) | (r & ((1 << s) - 1));
}
__host__ __device__ inline int ntt_index(int logn, bool acc, int point) {
  if (logn < kRegLogMin || logn > kRegLogMax) return point;
  const int e = ntt_e(logn, acc), lt = logn - e;
  const NttPlan p = ntt_plan(logn, e);
  const int s = p.s[p.n - 1], g = point >> s, r = ((g >> lt) << s) | (point & ((1 << s) - 1));
  return (r << lt) | (g & ((1 << lt) - 1));
}

}  // namespace hfe
