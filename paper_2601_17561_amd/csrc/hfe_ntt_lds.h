// LDS-resident negacyclic NTT, used for ring degrees up to 2^8 (larger ones stay in registers, hfe_ntt_reg.h): the
// merged transforms of Longa and Naehrig (2016), forward Cooley-Tukey
// with twiddles psi^brv(i) (output in bit-reversed order), inverse Gentleman-Sande with psi^-brv(i)
// and a final 1/n scale.  Residues mod a 36-bit prime are held as doubles (exact integers below 2^36)
// and multiplied with the error-free fp64 products of hfe_exact.h.
#pragma once
#include <type_traits>

#include "hfe_internal.h"

namespace hfe {
constexpr int kNttThreads = 1024;

// ------------------------------------------------------------------ fp64 residue arithmetic
// Residues mod q < 2^36 as doubles holding exact integers in [0, q); products by mulmod_d
// (hfe_exact.h).
__device__ __forceinline__ double to_d(uint64_t x) { return (double)x; }    // exact below 2^53
__device__ __forceinline__ uint64_t to_u(double x) { return (uint64_t)x; }  // x an integer in [0, q)

// Both transforms run in rounds of up to three butterfly stages: a thread loads a group of 2^S
// coefficients into registers, applies S stages there and stores them back, so a transform of
// degree 2^logn takes ceil(logn / 3) LDS passes and barriers instead of logn.
//
// Forward (Cooley-Tukey) round with first half-size t: group g holds a[base + k stride], k < 2^S,
// stride = t / 2^(S-1), base = B 2t + r (B = g / stride, r = g mod stride).  Stage s (half-size
// t / 2^s, m = n / (2t) 2^s blocks) pairs k and k + 2^(S-1-s); the pair lies in block
// B 2^s + (k >> (S - s)), whose twiddle is psi[m + block].
// The S stages of one forward round on the group held in registers x[0 .. 2^S) (first twiddle block m1 = n / (2t),
// group block B as above), on signed values (ct_butterfly_c): each stage adds at most about q/2 to the magnitude.
template <int S>
__device__ __forceinline__ void fwd_stages_c(double* x, const NttTab& T, int m1, int B) {
  constexpr int G = 1 << S;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int h = 1 << (S - 1 - s);
#pragma unroll
    for (int k = 0; k < G; ++k) {
      if (k & h) continue;
      const uint32_t w = (uint32_t)((m1 << s) + (B << s) + (k >> (S - s)));
      ct_butterfly_c(x[k], x[k + h], T.psi_d[w], T.qd, T.qinv);
    }
  }
}

template <int S>
__device__ __forceinline__ void fwd_round_c(double* a, const NttTab& T, int n, int t) {
  constexpr int G = 1 << S;
  const int ls = __builtin_ctz((unsigned)t) - (S - 1);  // stride = 2^ls (t, n powers of two)
  const int stride = 1 << ls, m1 = n / (2 * t);
  for (int g = threadIdx.x; g < (n >> S); g += blockDim.x) {
    const int B = g >> ls, r = g & (stride - 1);
    double* p0 = a + (B << (ls + S)) + r;  // base = B 2t + r
    double x[G];
#pragma unroll
    for (int k = 0; k < G; ++k) x[k] = p0[k << ls];
    fwd_stages_c<S>(x, T, m1, B);
#pragma unroll
    for (int k = 0; k < G; ++k) p0[k << ls] = x[k];
  }
  __syncthreads();
}

// Inverse (Gentleman-Sande) round with first half-size t: group g holds a[base + k t], k < 2^S,
// base = B 2^S t + r (B = g / t, r = g mod t).  Stage s (half-size 2^s t, m = n / (2^(s+1) t)
// blocks) pairs k and k + 2^s; the pair lies in block B 2^(S-1-s) + (k >> (s + 1)), twiddle
// ipsi[m + block].  On signed values: the round first takes its values (any integers below 2^47 in
// magnitude) to centered representatives (reduce_c_d, at most (1/2 + 2^-11) q), so that its S <= 3
// Gentleman-Sande stages (X + Y, and (X - Y) W centered) keep every value below 4.01q and every
// product operand below 8.02q; the last round scales by 1/n and returns residues in [0, q).
template <int S>
__device__ __forceinline__ void inv_round_c(double* a, const NttTab& T, int n, int t, bool last) {
  constexpr int G = 1 << S;
  const double q = T.qd, qinv = T.qinv;
  const int lt = __builtin_ctz((unsigned)t);
  for (int g = threadIdx.x; g < (n >> S); g += blockDim.x) {
    const int B = g >> lt, r = g & (t - 1);
    double* p0 = a + (B << (lt + S)) + r;  // base = B 2^S t + r
    double x[G];
#pragma unroll
    for (int k = 0; k < G; ++k) x[k] = reduce_c_d(p0[k << lt], q, qinv);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int h = 1 << s;
      const int m = n / (2 * h * t);
#pragma unroll
      for (int k = 0; k < G; ++k) {
        if (k & h) continue;
        const uint32_t w = (uint32_t)(m + (B << (S - 1 - s)) + (k >> (s + 1)));
        const double U = x[k], V = x[k + h];
        x[k] = U + V;
        x[k + h] = mulmod_c_d(U - V, T.ipsi_d[w], q, qinv);
      }
    }
    if (last) {
#pragma unroll
      for (int k = 0; k < G; ++k) x[k] = residue_of_c(mulmod_c_d(x[k], T.n_inv_d, q, qinv), q);
    }
#pragma unroll
    for (int k = 0; k < G; ++k) p0[k << lt] = x[k];
  }
  __syncthreads();
}

// Forward negacyclic NTT in place (output in bit-reversed order) on signed values without corrections
// (fwd_round_c): inputs in [0, q) give outputs congruent to the exact ones, each stage adding at most
// (1/2 + 2^-11) q in magnitude.
__device__ __forceinline__ void ntt_fwd_lds_c(double* a, const NttTab& T) {
  const int n = 1 << T.logn;
  int t = n >> 1, left = T.logn;
  while (left > 0) {
    if (left >= 3) {
      fwd_round_c<3>(a, T, n, t);
      t >>= 3;
      left -= 3;
    } else if (left == 2) {
      fwd_round_c<2>(a, T, n, t);
      t >>= 2;
      left -= 2;
    } else {
      fwd_round_c<1>(a, T, n, t);
      t >>= 1;
      left -= 1;
    }
  }
}

// The inverse on signed inputs (any integers below 2^47 in magnitude) through inv_round_c; outputs in
// [0, q).
__device__ __forceinline__ void ntt_inv_lds_c(double* a, const NttTab& T) {
  const int n = 1 << T.logn;
  int t = 1, left = T.logn;
  while (left > 0) {
    if (left >= 3) {
      inv_round_c<3>(a, T, n, t, left == 3);
      t <<= 3;
      left -= 3;
    } else if (left == 2) {
      inv_round_c<2>(a, T, n, t, true);
      t <<= 2;
      left -= 2;
    } else {
      inv_round_c<1>(a, T, n, t, true);
      t <<= 1;
      left -= 1;
    }
  }
}

static int ntt_block(int logn) {
  int half = 1 << (logn > 0 ? logn - 1 : 0);
  int b = half < 64 ? 64 : half;
  return b > kNttThreads ? kNttThreads : b;
}

template <class K>
static hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace hfe
