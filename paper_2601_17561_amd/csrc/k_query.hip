// Query encryption (one workgroup per query column and modulus) and the decryption products, built on the
// register-resident transforms of hfe_ntt_reg.h; rings above 2^14 go through k_ntt_big.hip.
#include "hfe_ntt_reg.h"

namespace hfe {

// ------------------------------------------------------------------ query encryption
// Workgroup (query column c, modulus z): a_c uniform in R_{N_Q} (stream QA, element (t, c)), and
// for each chunk j of N_Q code rows b[t] = -(s_j a_c)[t - j N_Q] + Delta m[c][t] + e(t, c).
// Output row c of XT[z]: [b_c (d2) | a_c (N_Q)].  One launch covers every modulus of the level (a launch
// per modulus left the chip idle at each one's end).  ONE: workgroup (c, z, j) takes chunk j alone and makes
// NTT(a_c) itself, for calls whose workgroups would not fill the chip.

template <class X, bool CHAIN, bool ONE>
__global__ void __launch_bounds__(X::MAXT)
    __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, ONE ? 1 : 2), ntt_waves(X::E, ONE ? 1 : 2))))
k_q_encrypt(QEncArgs A, QEncModuli B, uint64_t* XT) {
  extern __shared__ double lds[];
  const int64_t c = blockIdx.x;
  const int z = blockIdx.y;
  const NttTab T = B.T[z];
  const Mod M = B.M[z];
  const int n = 1 << T.logn;
  uint64_t* row = XT + ((int64_t)z * A.d3 + c) * A.K;
  double ahat[X::E];
  draw_mask<X, CHAIN>(ahat, lds, n, A.seed, stream_tag(kQA, B.id[z]), c, M, row + A.d2);
  X::fwd(ahat, lds, T);  // signed, uncorrected: below 9.1q
  const double q = T.qd, qinv = T.qinv, delta = u2d(B.delta[z]);
  const int8_t* m = A.m_q + c * A.d2;
  const int8_t* errs = A.e + c * A.d2;
  const int j0 = ONE ? (int)blockIdx.z : 0, j1 = ONE ? j0 + 1 : A.k;
  for (int j = j0; j < j1; ++j) {
    const gptr<uint64_t> w = as_global(B.s_hat[z]) + (int64_t)j * n;
    double x[X::E];
#pragma unroll
    for (int r = 0; r < X::E; ++r)
      x[r] = X::has(r, n) ? mulc(ahat[r], u2d((w + X::base(r))[threadIdx.x]), q, qinv) : 0.0;
    X::inv(x, lds, T);  // centered
    const int64_t lo = (int64_t)j * n;
    const int left = (int)(A.d2 - lo < n ? A.d2 - lo : n);
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      const int v = X::base(r) + (int)threadIdx.x;
      if (!X::has(r, n) || v >= left) continue;
      const int64_t t = lo + v;
      const double mv = (double)(int)m[t], e = (double)(int)errs[t];
      if constexpr (CHAIN)
        row[t] = from_signed(d2i(mv * delta - x[r] + e), M.q, M.mu);
      else
        row[t] = d2residue(mv * delta - x[r] + e, q, qinv);  // |.| < 1.6q
    }
  }
}

// The Gaussians of stream key_e at elements (u, c), u < per, c < cols, as e[c][u]: |e| <= 19 fits int8; two
// positions from each Philox block.
__global__ void k_errors(uint64_t seed, uint64_t key_e, const uint64_t* cdt, int64_t cols, int64_t per, int8_t* e) {
  const int64_t half = (per + 1) / 2, n = cols * half;
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = x / half, u = x - c * half;
    int32_t e0, e1;
    gaussian_pair_at(seed, key_e, (uint64_t)u, (uint64_t)c, cdt, e0, e1);
    e[c * per + 2 * u] = (int8_t)e0;
    if (2 * u + 1 < per) e[c * per + 2 * u + 1] = (int8_t)e1;
  }
}

hipError_t launch_errors(uint64_t seed, uint64_t purpose, const uint64_t* cdt, int64_t cols, int64_t per, int8_t* e,
                         hipStream_t s) {
  const int64_t n = cols * ((per + 1) / 2);
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192;
  hipLaunchKernelGGL(k_errors, dim3((unsigned)blocks), dim3(256), 0, s, seed, stream_tag(purpose, 0), cdt, cols, per,
                     e);
  return hipGetLastError();
}

// The same Gaussians added to finished residues, less what the encryption had in their place.
__global__ void k_add_errors(uint64_t seed, uint64_t key_e, const uint64_t* cdt, int64_t cols, int64_t per,
                             const int8_t* minus, uint64_t* x, int64_t col, int64_t q) {
  const int64_t half = (per + 1) / 2, n = cols * half;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = i / half, u = i - c * half;
    int32_t e[2];
    gaussian_pair_at(seed, key_e, (uint64_t)u, (uint64_t)c, cdt, e[0], e[1]);
    for (int k = 0; k < 2 && 2 * u + k < per; ++k) {
      const int64_t at = 2 * u + k;
      int64_t v = (int64_t)x[c * col + at] + e[k] - (minus ? minus[c * per + at] : 0);  // within 20 of [0, q)
      v = v < 0 ? v + q : v >= q ? v - q : v;
      x[c * col + at] = (uint64_t)v;
    }
  }
}

hipError_t launch_add_errors(uint64_t seed, uint64_t purpose, const uint64_t* cdt, int64_t cols, int64_t per,
                             const int8_t* minus, uint64_t* x, int64_t col, uint64_t q, hipStream_t s) {
  const int64_t n = cols * ((per + 1) / 2);
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192;
  hipLaunchKernelGGL(k_add_errors, dim3((unsigned)blocks), dim3(256), 0, s, seed, stream_tag(purpose, 0), cdt, cols,
                     per, minus, x, col, (int64_t)q);
  return hipGetLastError();
}

hipError_t launch_q_encrypt(const QEncArgs& args, const QEncModuli& b, int level, uint64_t* XT, hipStream_t s) {
  QEncArgs a = args;
  if (a.d3 <= 0) return hipSuccess;
  if (level < 1 || level > HFE_MAX_QPRIMES) return hipErrorInvalidValue;
  if (b.T[0].logn > kMaxLogN) {
    for (int i = 0; i < level; ++i) {
      const hipError_t e = launch_q_encrypt_big(a, XT + (size_t)i * a.d3 * a.K, b.id[i], b.M[i], b.delta[i], b.T[i],
                                                b.s_hat[i], s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const bool after = a.e == nullptr;
  if (after) a.e = a.m_q;  // in the errors' place, of their shape; taken off again where they are added
  const bool chain = b.M[0].q != b.T[0].q;  // residues mod n^2, products through the table's prime
  // up to two workgroups per CU the chunks run side by side (each repeats the mask's draw and transform)
  const bool one = a.k == 1 || a.d3 * level * a.k <= 512;
  return by_ntt(b.T[0].logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    auto kern = chain ? (one ? k_q_encrypt<X, true, true> : k_q_encrypt<X, true, false>)
                      : (one ? k_q_encrypt<X, false, true> : k_q_encrypt<X, false, false>);
    hipError_t e = allow_lds(kern, sizeof(double) * X::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.d3, (unsigned)level, one ? (unsigned)a.k : 1u), dim3(block),
                       sizeof(double) * X::LDS, s, a, b, XT);
    e = hipGetLastError();
    for (int i = 0; after && i < level && e == hipSuccess; ++i)
      e = launch_add_errors(a.seed, kQE, a.cdt, a.d3, a.d2, a.m_q, XT + i * a.d3 * a.K, a.K, b.M[i].q, s);
    return e;
  });
}

// ------------------------------------------------------------------ decryption products
// Workgroup (c, j, z): y[z][c][r] = B_out[z][c][r] + (s'_j * A_out[z][c])[(row0 + r) - j N_DB] mod q_z for the
// selected rows r whose database row row0 + r lies in chunk j.  One launch covers the level's moduli.

template <class X, bool CHAIN>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_dec_products(const uint64_t* out, int64_t R_out, int64_t row0, int64_t rows, DecModuli B, int j0, uint64_t* y) {
  extern __shared__ double lds[];
  const int64_t c = blockIdx.x;
  const int j = j0 + (int)blockIdx.y, z = blockIdx.z;
  const NttTab T = B.T[z];
  const Mod M = B.M[z];  // the arithmetic modulus (the table's prime, or n^2 of the chain)
  const int n = 1 << T.logn;
  const int64_t zc = (int64_t)z * gridDim.x + c;
  const uint64_t* ocol = out + zc * R_out;
  uint64_t* yc = y + zc * rows;
  double x[X::E];
#pragma unroll
  for (int r = 0; r < X::E; ++r) x[r] = X::has(r, n) ? enter_ntt<CHAIN>((ocol + X::base(r))[threadIdx.x], M.q) : 0.0;
  X::fwd(x, lds, T);  // signed, uncorrected: below 9.1q
  const double q = T.qd, qinv = T.qinv;
  const gptr<uint64_t> w = as_global(B.s_hat[z]) + (int64_t)j * n;
#pragma unroll
  for (int r = 0; r < X::E; ++r)
    x[r] = X::has(r, n) ? mulc(x[r], u2d((w + X::base(r))[threadIdx.x]), q, qinv) : 0.0;
  X::inv(x, lds, T);  // centered
  const int64_t first = (int64_t)j * n - row0;  // the result row of coefficient 0
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    const int64_t t = first + X::base(r) + (int)threadIdx.x;
    if (!X::has(r, n) || t < 0 || t >= rows) continue;
    const uint64_t b = ocol[n + t];
    if constexpr (CHAIN)
      yc[t] = from_signed(d2i(x[r]) + (int64_t)b, M.q, M.mu);
    else
      yc[t] = d2residue(x[r] + u2d(b), q, qinv);
  }
}

hipError_t launch_dec_products(const uint64_t* out, int64_t d3, int64_t R_out, int64_t row0, int64_t rows,
                               int n_db_log, const DecModuli& b, int level, int k_db, uint64_t* y, hipStream_t s) {
  if (d3 <= 0 || rows <= 0) return hipSuccess;
  if (level < 1 || level > HFE_MAX_QPRIMES) return hipErrorInvalidValue;
  const int64_t n = 1ll << n_db_log;
  const int j0 = (int)(row0 / n), j1 = (int)((row0 + rows - 1) / n);
  if (j1 >= k_db) return hipErrorInvalidValue;
  if (n_db_log > kMaxLogN) {
    for (int i = 0; i < level; ++i) {
      const hipError_t e = launch_dec_products_big(out + (size_t)i * d3 * R_out, d3, R_out, row0, rows, b.T[i],
                                                   b.s_hat[i], j0, j1, b.M[i], y + (size_t)i * d3 * rows, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const bool chain = b.M[0].q != b.T[0].q;
  return by_ntt(n_db_log, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    auto kern = chain ? k_dec_products<X, true> : k_dec_products<X, false>;
    hipError_t e = allow_lds(kern, sizeof(double) * X::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)d3, (unsigned)(j1 - j0 + 1), (unsigned)level), dim3(block),
                       sizeof(double) * X::LDS, s, out, R_out, row0, rows, b, j0, y);
    return hipGetLastError();
  });
}

}  // namespace hfe
