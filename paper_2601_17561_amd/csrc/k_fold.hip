// Normalise and fold (Algorithm 2, Section 4.3, Appendix C.2): the kernels of a small CKKS evaluator at
// ring degree N <= 2^14 over the slots q_0 .. q_4 and the special prime p (slot 5).
//
// Ciphertexts are kept in the NTT domain as uint64 residues, [item][part (b, a)][slot][N], in the order of the
// register transforms; every transform is one polynomial per workgroup, in registers from its loads to its stores
// (hfe_ntt_reg.h; ntt_waves names what is spilled at 2^13 and 2^14).  q_1 .. q_3 lie below 2^24, where a product of two residues is exact in a double and the
// modular product takes four instructions instead of six (the SM variants).  The operations a fold needs are
// built from a few passes:
//   k_fold_encode     the slot encoder (plaintext coefficients from integer slot values, hfe_slots.h)
//   k_fold_fwd        signed coefficients -> NTT-domain residues, for several slots
//   k_fold_inv        NTT-domain residues (or the product of two, or with a plaintext)
//                     -> coefficients (residues, centered, or the digits of a key switch)
//   k_fold_ks_mac     (k_fold_ks.hip) sum_i NTT(d_i) K_i for one slot, the products accumulated in registers;
//                     the special prime's sum is transformed back and centered
//   k_fold_lift       (k_fold_ks.hip) (x k - NTT([y]_div)) div^-1 plus addends on every kept slot: RS_div of a product, of a
//                     constant times a ciphertext (with a mod-drop and an added constant), and the end of a
//                     key switch (with the tensor terms d0, d1 of a product, or sigma(b) of a rotation), and of
//                     a plaintext product (the normalisation, the product formed on load)
//   elementwise       the automorphism of a rotation as a permutation of the NTT points,
//                     group sums, key and input draws
#include "hfe_fold_dev.h"
#include "hfe_slots.h"

namespace hfe {
namespace {

__device__ __forceinline__ double mm_d(double a, double b, int z, const FoldConsts& C) {
  return mulmod_d(a, b, C.zd[z], C.zinv[z]);
}

// ------------------------------------------------------------------ encoder
// Slot weights: w = v (mode 0, |v| <= 2^24) or round(2^30 / v) = floor((2^31 + v) / (2v)) (mode 1,
// 1 <= v <= 2^24); a value outside its range sets *bad and is replaced by 0 (mode 0) or 1 (mode 1).
__global__ void k_fold_weights(const int32_t* values, int64_t total, int mode, int64_t* w, uint32_t* bad) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t v = values[e];
    if (mode) {
      if (v < 1 || v > (1 << 24)) {
        atomicOr(bad, 1u);
        v = 1;
      }
      w[e] = ((int64_t(1) << 31) + v) / (2 * v);
    } else {
      if (v < -(1 << 24) || v > (1 << 24)) {
        atomicOr(bad, 1u);
        v = 0;
      }
      w[e] = v;
    }
  }
}

// The slot encoder (hfe_slots.h), one workgroup per item c: the M = N/2 slot values w[c][j] 2^e enter an
// inverse DFT of length M at bit-reversed positions pos[j] in LDS (real and imaginary parts, N doubles),
// log2 M radix-2 stages, then the untwist and the rounding: out[c][i], out[c][M + i].
__global__ void __launch_bounds__(kNttThreads) k_fold_encode(const int64_t* w, int logn, double scale,
                                                           const double* W, const double* Z, const int32_t* pos,
                                                           int64_t* out) {
  extern __shared__ double lds[];
  const int M = 1 << (logn - 1);
  double* xr = lds;
  double* xi = lds + M;
  const int64_t c = blockIdx.x;
  for (int j = threadIdx.x; j < M; j += blockDim.x) {
    const int p = pos[j];
    xr[p] = (double)w[c * M + j] * scale;  // exact: |w| < 2^31, scale a power of two
    xi[p] = 0.0;
  }
  __syncthreads();
  for (int half = 1, lh = 0; half < M; half *= 2, ++lh) {
    const int step = M / (2 * half);
    for (int b = threadIdx.x; b < M / 2; b += blockDim.x) {
      const int t = b & (half - 1);
      const int ia = ((b >> lh) << (lh + 1)) + t, ic = ia + half;
      slot_butterfly(xr[ia], xi[ia], xr[ic], xi[ic], W[2 * t * step], W[2 * t * step + 1]);
    }
    __syncthreads();
  }
  const double inv_m = 1.0 / (double)M;
  int64_t* o = out + c * 2 * M;
  for (int i = threadIdx.x; i < M; i += blockDim.x) {
    double ur, ui;
    slot_untwist(xr[i], xi[i], Z[2 * i], Z[2 * i + 1], inv_m, ur, ui);
    o[i] = round_half_up(ur);
    o[M + i] = round_half_up(ui);
  }
}

// ------------------------------------------------------------------ transforms
// job = item * nsl + s: src[item * si + s * ss + t] (signed, |x| < 2^63) mod z_s -> forward NTT ->
// dst[item * di + s * ds + t].
template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_fold_fwd(FoldConsts C, const int64_t* src, int64_t si, int64_t ss, uint64_t* dst, int64_t di, int64_t ds, SlotMap zm,
           int nsl) {
  extern __shared__ double lds[];
  const int n = 1 << C.logn;
  const int64_t item = blockIdx.x / nsl;
  const int s = blockIdx.x - (int)(item * nsl);
  const int z = zm.z[s];
  const double zd = C.zd[z], zi = C.zinv[z], c32 = C.c32[z];
  const int64_t* p = src + item * si + s * ss;
  uint64_t* o = dst + item * di + s * ds;
  by_size(zd, [&](auto smc) {
  constexpr bool SM = decltype(smc)::value;
  double x[X::E];
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    x[r] = X::has(r, n) ? signed64_mod(as_global(p + X::base(r))[threadIdx.x], c32, zd, zi) : 0.0;
    if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
  }
  X::template fwd<SM>(x, lds, C.tab[z]);
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    if (X::has(r, n)) (o + X::base(r))[threadIdx.x] = d2residue(x[r], zd, zi);
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  });
}

// job = item * nsl + s: inverse NTT of src[item * si + s * ss] mod z_s (times the plaintext pm at slot z_s
// when pm is given, times y at the same place when y is given); mode 0: residues (uint64), 1: centered (double),
// 2: residues times factor[s] mod z_s (the digits of a key switch).
template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_fold_inv(FoldConsts C, FoldInv a) {
  extern __shared__ double lds[];
  const int n = 1 << C.logn;
  const int64_t item = blockIdx.x / a.nsl;
  const int s = blockIdx.x - (int)(item * a.nsl);
  const int z = a.zm.z[s];
  const int64_t off = item * a.si + s * a.ss, doff = item * a.di + s * a.ds;
  const uint64_t* p = a.src + off;
  const uint64_t* y = a.pm ? a.pm + (item >> 1) * a.pmi + (int64_t)z * n : a.y ? a.y + off : nullptr;
  const double zd = C.zd[z], zi = C.zinv[z];
  by_size(zd, [&](auto smc) {
  constexpr bool SM = decltype(smc)::value;
  double x[X::E];
  if (y) {
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      x[r] = X::has(r, n) ? mulc(u2d(as_global(p + X::base(r))[threadIdx.x]),
                                 u2d(as_global(y + X::base(r))[threadIdx.x]), zd, zi)
                          : 0.0;
      if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int r = 0; r < X::E; ++r) x[r] = X::has(r, n) ? u2d(as_global(p + X::base(r))[threadIdx.x]) : 0.0;
  }
  X::template inv<SM>(x, lds, C.tab[z]);
  if (a.mode == 1) {
    double* o = static_cast<double*>(a.dst) + doff;
#pragma unroll
    for (int r = 0; r < X::E; ++r)
      if (X::has(r, n)) (o + X::base(r))[threadIdx.x] = center_exact(x[r], zd);
  } else {
    uint64_t* o = static_cast<uint64_t*>(a.dst) + doff;
    const double fz = a.f.v[s];
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      const double v = a.mode == 2 ? mulc(x[r], fz, zd, zi) : x[r];
      if (X::has(r, n)) (o + X::base(r))[threadIdx.x] = d2u(residue_of_c(v, zd));
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  });
}

// The end of a relinearised product divided by p q_l in one rounding: job = part * items + item,
// X = acc[item][part][l] + (p mod q_l) d (d the tensor's d0 or d1 at slot l, formed from tx, ty), its
// inverse transform r (mod q_l), and the value c = a + p ((r - a) p^-1 mod q_l) (a = accp, centered mod p),
// the representative of X modulo D = p q_l, centered: cen[item][part][t].  l is 1 .. 3: q_l is below 2^24.
template <class X, int PART>
__device__ __forceinline__ void relin_center(double* lds, const FoldConsts& C, int level, int64_t item,
                                             const uint64_t* acc, const double* accp, const uint64_t* tx,
                                             const uint64_t* ty, double p_l, double pinv_l, int64_t D, int64_t* cen) {
  const int n = 1 << C.logn;
  const int l = level;
  const int64_t per = (int64_t)(l + 1) * n, ip = item * 2 + PART;
  const uint64_t* xa = acc + ip * per + (int64_t)l * n;
  const uint64_t* bx = tx + item * 2 * per + (int64_t)l * n;
  const uint64_t* by = ty + item * 2 * per + (int64_t)l * n;
  const double zd = C.zd[l], zi = C.zinv[l];
  double x[X::E];
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    x[r] = 0.0;
    if (!X::has(r, n)) continue;
    const int b = X::base(r);
    const double vx = u2d((bx + b)[threadIdx.x]), vy = u2d((by + b)[threadIdx.x]);
    double d;
    if constexpr (PART == 0)
      d = mulc<true>(vx, vy, zd, zi);
    else
      d = mulc<true>(u2d((bx + per + b)[threadIdx.x]), vy, zd, zi) +
          mulc<true>(u2d((by + per + b)[threadIdx.x]), vx, zd, zi);
    x[r] = u2d((xa + b)[threadIdx.x]) + mulc<true>(d, p_l, zd, zi);
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  X::template inv<true>(x, lds, C.tab[l]);
  const int64_t p = (int64_t)C.mod[5].q;
  const double* ap = accp + ip * n;
  int64_t* o = cen + ip * n;
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    if (!X::has(r, n)) continue;
    const int b = X::base(r);
    const double a = (ap + b)[threadIdx.x];
    const double u = mulc<true>(x[r] - reduce_c_d(a, zd, zi), pinv_l, zd, zi);  // (r - a) p^-1 mod q_l
    int64_t v = d2i(a) + p * (int64_t)d2u(residue_of_c(u, zd));                 // in (-p/2, D): |v| < 2^60
    if (v > D / 2) v -= D;
    (o + b)[threadIdx.x] = v;
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
}
template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_fold_relin_center(FoldConsts C, int level, const uint64_t* acc, const double* accp, const uint64_t* tx,
                    const uint64_t* ty, double p_l, double pinv_l, int64_t D, int64_t* cen) {
  extern __shared__ double lds[];
  const int64_t items = gridDim.x / 2;
  if (blockIdx.x < items)
    relin_center<X, 0>(lds, C, level, blockIdx.x, acc, accp, tx, ty, p_l, pinv_l, D, cen);
  else
    relin_center<X, 1>(lds, C, level, blockIdx.x - items, acc, accp, tx, ty, p_l, pinv_l, D, cen);
}

// ------------------------------------------------------------------ elementwise
// Rotation's automorphism on gathered items with nsl slots: out[u][part][s][t] =
// x[src[u]][part][s][perm[amt[u]][t]] (the NTT points of every prime are ordered alike).
__global__ void k_fold_perm(FoldConsts C, const uint64_t* x, const int32_t* src, const int32_t* amt,
                            const int32_t* perm, uint64_t* out, int64_t items, int nsl) {
  const int n = 1 << C.logn;
  const int64_t per = 2 * (int64_t)nsl * n;
  const int64_t total = items * per;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(e & (n - 1));
    const int64_t u = e / per, w = e - u * per;
    out[e] = x[(int64_t)src[u] * per + (w - t) + perm[(int64_t)amt[u] * n + t]];
  }
}

// Group sums of items with nsl slots: out[g] = sum over the members of group g; members are listed in
// mem[beg[g] .. beg[g+1]) as idx * 2 + (rotated ? 1 : 0), rotated[idx] or f[idx].
__global__ void k_fold_group_sum(FoldConsts C, const uint64_t* f, const uint64_t* rotated, const int32_t* beg,
                                 const int32_t* mem, uint64_t* out, int64_t groups, int nsl) {
  const int n = 1 << C.logn;
  const int64_t per = 2 * (int64_t)nsl * n;
  const int64_t total = groups * per;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t g = e / per, w = e - g * per;
    const double zd = C.zd[(int)((w >> C.logn) % nsl)];
    double v = 0.0;
    for (int m = beg[g]; m < beg[g + 1]; ++m) {
      const int32_t code = mem[m];
      const uint64_t* b = (code & 1) ? rotated : f;
      v = addmod_d(v, to_d(b[(int64_t)(code >> 1) * per + w]), zd);
    }
    out[e] = to_u(v);
  }
}

// Scatter rotated items back: x[dst[u]] = y[u] (items with nsl slots).
__global__ void k_fold_scatter(FoldConsts C, const uint64_t* y, const int32_t* dst, uint64_t* x, int64_t items,
                               int nsl) {
  const int n = 1 << C.logn;
  const int64_t per = 2 * (int64_t)nsl * n;
  const int64_t total = items * per;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t u = e / per, w = e - u * per;
    x[(int64_t)dst[u] * per + w] = y[e];
  }
}

// ------------------------------------------------------------------ draws
// Key coefficients: for key kappa (column kappa * 8 + i), slot s of the key's slot list zm and digit
// i <= level: out[s][i][0][t] = uniform mod z (stream FKA, sub = stream id of z), out[s][i][1][t] =
// the Gaussian error (stream FKE, sub 0) as a residue mod z.
__global__ void k_fold_key_coeffs(FoldConsts C, uint64_t seed, int kappa, int level, SlotMap zm, const uint64_t* cdt,
                                  uint64_t* out) {
  const int n = 1 << C.logn;
  const int nsl = level + 2;
  const int64_t total = (int64_t)nsl * (level + 1) * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(e & (n - 1));
    const int64_t r = e >> C.logn;
    const int i = (int)(r % (level + 1));
    const int s = (int)(r / (level + 1));
    const int z = zm.z[s];
    const Mod md = C.mod[z];
    const uint64_t col = (uint64_t)kappa * 8 + (uint64_t)i;
    const uint64_t u = uniform_at(seed, stream_tag(kFKA, C.pid[z]), (uint64_t)t, col, md);
    const int32_t g = gaussian_at(seed, stream_tag(kFKE, 0), (uint64_t)t, col, cdt);
    out[(r * 2 + 0) * n + t] = u;
    out[(r * 2 + 1) * n + t] = from_signed(g, md.q, md.mu);
  }
}

// Key finish, NTT domain: beta = -k s + g_{s,i} s_from + e, stored as doubles [s][i][2][N]
// (part 0: k, part 1: beta).  s_hat, from_hat: [slot z][N] NTT residues; gk[s][i] = p (Q_l / q_i) mod z.
__global__ void k_fold_key_finish(FoldConsts C, int level, SlotMap zm, const uint64_t* coef_hat, const uint64_t* s_hat,
                                  const uint64_t* from_hat, KeyGadget gk, double* key) {
  const int n = 1 << C.logn;
  const int64_t total = (int64_t)(level + 2) * (level + 1) * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(e & (n - 1));
    const int64_t r = e >> C.logn;
    const int i = (int)(r % (level + 1));
    const int s = (int)(r / (level + 1));
    const int z = zm.z[s];
    const double zd = C.zd[z];
    const double k = to_d(coef_hat[(r * 2 + 0) * n + t]);
    const double err = to_d(coef_hat[(r * 2 + 1) * n + t]);
    double beta = submod_d(err, mm_d(k, to_d(s_hat[(int64_t)z * n + t]), z, C), zd);
    beta = addmod_d(beta, mm_d(gk.v[s][i], to_d(from_hat[(int64_t)z * n + t]), z, C), zd);
    key[(r * 2 + 0) * n + t] = k;
    key[(r * 2 + 1) * n + t] = beta;
  }
}

// Input errors: m[c][t] += the Gaussian at (t, c) of stream FXE.
__global__ void k_fold_add_errors(FoldConsts C, uint64_t seed, const uint64_t* cdt, int64_t* m, int64_t items) {
  const int n = 1 << C.logn;
  const int64_t total = items * (int64_t)n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e >> C.logn;
    const int t = (int)(e & (n - 1));
    m[e] += gaussian_at(seed, stream_tag(kFXE, 0), (uint64_t)t, (uint64_t)c, cdt);
  }
}

// Input masks and bodies, job = c * 5 + z: a (stream FXA, sub = stream id of q_z, element (t, c)) ->
// NTT -> ct[c][1][z]; ct[c][0][z] = (m + e)_hat - a_hat s_hat (the encoded inner products with their
// errors are already in ct[c][0][z]).
template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_fold_encrypt(FoldConsts C, uint64_t seed, const uint64_t* s_hat, uint64_t* ct) {
  extern __shared__ double lds[];
  const int n = 1 << C.logn;
  const int64_t c = blockIdx.x / 5;
  const int z = (int)(blockIdx.x - c * 5);
  const Mod md = C.mod[z];
  const uint64_t tag = stream_tag(kFXA, C.pid[z]);
  double x[X::E];
  X::from_quads(x, lds, n, [&](int v4, double (&o)[4]) {
    const Philox4 q = philox4x64_10(seed, tag, (uint64_t)v4, (uint64_t)c, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[j] = u2d(q.v[j] < md.bound ? barrett64(q.v[j], md.q, md.mu)
                                   : uniform_at(seed, tag, (uint64_t)(4 * v4 + j), (uint64_t)c, md));
  });
  const double zd = C.zd[z], zi = C.zinv[z];
  X::fwd(x, lds, C.tab[z]);
  uint64_t* b = ct + ((c * 2 + 0) * 5 + z) * n;
  uint64_t* a = ct + ((c * 2 + 1) * 5 + z) * n;
  const uint64_t* sh = s_hat + (int64_t)z * n;
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    if (!X::has(r, n)) continue;
    const int o = X::base(r);
    const double sv = u2d((sh + o)[threadIdx.x]);
    (a + o)[threadIdx.x] = d2residue(x[r], zd, zi);
    (b + o)[threadIdx.x] = d2residue(u2d((b + o)[threadIdx.x]) - mulc(x[r], sv, zd, zi), zd, zi);
  }
}

// Decryption at level 0 in the NTT domain: out[c][t] = b + a s mod q_0 (then an inverse transform).
__global__ void k_fold_dec_products(FoldConsts C, const uint64_t* ct, const uint64_t* s_hat, uint64_t* out,
                                    int64_t items) {
  const int n = 1 << C.logn;
  const int64_t total = items * (int64_t)n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e >> C.logn;
    const int t = (int)(e & (n - 1));
    const double b = to_d(ct[(c * 2 + 0) * n + t]), a = to_d(ct[(c * 2 + 1) * n + t]);
    out[e] = to_u(addmod_d(b, mm_d(a, to_d(s_hat[t]), 0, C), C.zd[0]));
  }
}

// Decoding (floating point), one workgroup per item: the slots m(zeta^(g_j)) of the centered coefficients
// m[c][0 .. N) as the DFT of length M of (m_i + i m_(M+i)) zeta^i (conjugate twiddles of the encoder's,
// bit-reversed input), real parts divided by the scale: v[c][j] at the transform's output k_j.
__global__ void __launch_bounds__(kNttThreads) k_fold_decode(const double* m, int logn, const double* W,
                                                           const double* Z, const int32_t* kj, double inv_scale,
                                                           double* v) {
  extern __shared__ double lds[];
  const int M = 1 << (logn - 1);
  double* xr = lds;
  double* xi = lds + M;
  const int64_t c = blockIdx.x;
  const double* mc = m + c * 2 * M;
  for (int i = threadIdx.x; i < M; i += blockDim.x) {
    const int p = (int)slot_brv((uint32_t)i, logn - 1);
    slot_twist(mc[i], mc[M + i], Z[2 * i], Z[2 * i + 1], xr[p], xi[p]);
  }
  __syncthreads();
  for (int half = 1, lh = 0; half < M; half *= 2, ++lh) {
    const int step = M / (2 * half);
    for (int b = threadIdx.x; b < M / 2; b += blockDim.x) {
      const int t = b & (half - 1);
      const int ia = ((b >> lh) << (lh + 1)) + t, ic = ia + half;
      slot_butterfly(xr[ia], xi[ia], xr[ic], xi[ic], W[2 * t * step], -W[2 * t * step + 1]);
    }
    __syncthreads();
  }
  for (int j = threadIdx.x; j < M; j += blockDim.x) v[c * M + j] = xr[kj[j]] * inv_scale;
}

unsigned ew_grid(int64_t total) {
  int64_t g = (total + 255) / 256;
  return (unsigned)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

}  // namespace

// ------------------------------------------------------------------ launchers
hipError_t launch_fold_weights(const int32_t* values, int64_t total, int mode, int64_t* w, uint32_t* bad,
                               hipStream_t s) {
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fold_weights, dim3(ew_grid(total)), dim3(256), 0, s, values, total, mode, w, bad);
  return hipGetLastError();
}

hipError_t launch_fold_encode(const int64_t* w, int64_t items, int logn, double scale, const double* W,
                              const double* Z, const int32_t* pos, int64_t* out, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  const size_t lds = sizeof(double) << logn;
  hipError_t e = allow_lds(k_fold_encode, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fold_encode, dim3((unsigned)items), dim3(ntt_block(logn)), lds, s, w, logn, scale, W, Z, pos,
                     out);
  return hipGetLastError();
}

hipError_t launch_fold_fwd(const FoldConsts& C, const int64_t* src, int64_t si, int64_t ss, uint64_t* dst, int64_t di,
                           int64_t ds, const SlotMap& zm, int nsl, int64_t items, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  return by_ntt(C.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    const size_t lds = sizeof(double) * X::LDS;
    hipError_t e = allow_lds(k_fold_fwd<X>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold_fwd<X>, dim3((unsigned)(items * nsl)), dim3(block), lds, s, C, src, si, ss, dst, di, ds,
                       zm, nsl);
    return hipGetLastError();
  });
}

hipError_t launch_fold_inv(const FoldConsts& C, const FoldInv& a, int64_t items, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  return by_ntt(C.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    const size_t lds = sizeof(double) * X::LDS;
    hipError_t e = allow_lds(k_fold_inv<X>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold_inv<X>, dim3((unsigned)(items * a.nsl)), dim3(block), lds, s, C, a);
    return hipGetLastError();
  });
}

hipError_t launch_fold_relin_center(const FoldConsts& C, int level, const uint64_t* acc, const double* accp,
                                   const uint64_t* tx, const uint64_t* ty, int64_t items, int64_t* cen, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  const uint64_t ql = C.mod[level].q, p = C.mod[5].q;
  const double p_l = (double)(p % ql), pinv_l = (double)inv_mod(p % ql, ql);
  return by_ntt(C.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    const size_t lds = sizeof(double) * X::LDS;
    hipError_t e = allow_lds(k_fold_relin_center<X>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold_relin_center<X>, dim3((unsigned)(items * 2)), dim3(block), lds, s, C, level, acc, accp, tx, ty,
                       p_l, pinv_l, (int64_t)(p * ql), cen);
    return hipGetLastError();
  });
}

hipError_t launch_fold_perm(const FoldConsts& C, const uint64_t* x, const int32_t* src, const int32_t* amt,
                            const int32_t* perm, uint64_t* out, int64_t items, int nsl, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fold_perm, dim3(ew_grid(items * 2 * nsl << C.logn)), dim3(256), 0, s, C, x, src, amt, perm,
                     out, items, nsl);
  return hipGetLastError();
}

hipError_t launch_fold_group_sum(const FoldConsts& C, const uint64_t* f, const uint64_t* rotated, const int32_t* beg,
                                 const int32_t* mem, uint64_t* out, int64_t groups, int nsl, hipStream_t s) {
  if (groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fold_group_sum, dim3(ew_grid(groups * 2 * nsl << C.logn)), dim3(256), 0, s, C, f, rotated, beg,
                     mem, out, groups, nsl);
  return hipGetLastError();
}

hipError_t launch_fold_scatter(const FoldConsts& C, const uint64_t* y, const int32_t* dst, uint64_t* x, int64_t items,
                               int nsl, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fold_scatter, dim3(ew_grid(items * 2 * nsl << C.logn)), dim3(256), 0, s, C, y, dst, x, items,
                     nsl);
  return hipGetLastError();
}

hipError_t launch_fold_key_coeffs(const FoldConsts& C, uint64_t seed, int kappa, int level, const SlotMap& zm,
                                  const uint64_t* cdt, uint64_t* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fold_key_coeffs, dim3(ew_grid((int64_t)(level + 2) * (level + 1) << C.logn)), dim3(256), 0, s,
                     C, seed, kappa, level, zm, cdt, out);
  return hipGetLastError();
}

hipError_t launch_fold_key_finish(const FoldConsts& C, int level, const SlotMap& zm, const uint64_t* coef_hat,
                                  const uint64_t* s_hat, const uint64_t* from_hat, const KeyGadget& gk, double* key,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_fold_key_finish, dim3(ew_grid((int64_t)(level + 2) * (level + 1) << C.logn)), dim3(256), 0, s,
                     C, level, zm, coef_hat, s_hat, from_hat, gk, key);
  return hipGetLastError();
}

hipError_t launch_fold_add_errors(const FoldConsts& C, uint64_t seed, const uint64_t* cdt, int64_t* m, int64_t items,
                                  hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fold_add_errors, dim3(ew_grid(items << C.logn)), dim3(256), 0, s, C, seed, cdt, m, items);
  return hipGetLastError();
}

hipError_t launch_fold_encrypt(const FoldConsts& C, uint64_t seed, const uint64_t* s_hat, uint64_t* ct, int64_t items,
                               hipStream_t s) {
  if (items <= 0) return hipSuccess;
  return by_ntt(C.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    const size_t lds = sizeof(double) * X::LDS;
    hipError_t e = allow_lds(k_fold_encrypt<X>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold_encrypt<X>, dim3((unsigned)(items * 5)), dim3(block), lds, s, C, seed, s_hat, ct);
    return hipGetLastError();
  });
}

hipError_t launch_fold_dec_products(const FoldConsts& C, const uint64_t* ct, const uint64_t* s_hat, uint64_t* out,
                                    int64_t items, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fold_dec_products, dim3(ew_grid(items << C.logn)), dim3(256), 0, s, C, ct, s_hat, out, items);
  return hipGetLastError();
}

hipError_t launch_fold_decode(const double* m, int64_t items, int logn, const double* W, const double* Z,
                              const int32_t* kj, double inv_scale, double* v, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  const size_t lds = sizeof(double) << logn;
  hipError_t e = allow_lds(k_fold_decode, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fold_decode, dim3((unsigned)items), dim3(ntt_block(logn)), lds, s, m, logn, W, Z, kj,
                     inv_scale, v);
  return hipGetLastError();
}

}  // namespace hfe
