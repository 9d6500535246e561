// The kernels built on the negacyclic NTT of one polynomial per workgroup (ring degrees up to 2^14):
// secret-key transforms, T = M_DB S_Q, database encryption (query encryption and decryption
// products: k_query.hip).
// Larger ring degrees (2^15, 2^16) go through the two-pass transforms of k_ntt_big.hip, which the
// launchers below call with the same arguments.
//
// Products in R_n = Z[X]/(X^n + 1) mod a 36-bit prime q (Section 2.2.1) are computed as
// INTT(NTT(a) . NTT(s)) with the merged negacyclic transforms of Longa and Naehrig (2016):
// forward Cooley-Tukey with twiddles psi^brv(i) (output in bit-reversed order), inverse
// Gentleman-Sande with psi^-brv(i) and a final 1/n scale.  One workgroup transforms one
// polynomial, in its registers from the load to the store (hfe_ntt_reg.h, but for what ntt_waves says is spilled at
// 2^13 and 2^14; degrees below 2^9 in LDS, LdsNtt).  Residues are held as doubles (exact signed integers) and multiplied mod q with an error-free
// fp64 product (mulmod_c_d): about a third of the integer instructions of a 64-bit Shoup product, at the
// same issue rate on this chip.  Arrays in the transform domain (the secrets) use the register order.
#include <type_traits>

#include "hfe_ntt_reg.h"

namespace hfe {

// ------------------------------------------------------------------ batch forward NTT

template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_ntt_fwd(uint64_t* a, int64_t stride, NttTab T) {
  extern __shared__ double lds[];
  const int n = 1 << T.logn;
  uint64_t* poly = a + (int64_t)blockIdx.x * stride;
  double x[X::E];
  load_poly<X>(x, poly, n);
  X::fwd(x, lds, T);
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    if (X::has(r, n)) (poly + X::base(r))[threadIdx.x] = d2residue(x[r], T.qd, T.qinv);
  }
}

hipError_t launch_ntt_fwd(uint64_t* a, int64_t count, int64_t stride, NttTab tab, hipStream_t s, bool acc_order) {
  if (count <= 0) return hipSuccess;
  if (tab.logn > kMaxLogN) return launch_ntt_fwd_big(a, count, stride, tab, s);
  auto go = [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    hipError_t e = allow_lds(k_ntt_fwd<X>, sizeof(double) * X::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ntt_fwd<X>, dim3((unsigned)count), dim3(block), sizeof(double) * X::LDS, s, a, stride, tab);
    return hipGetLastError();
  };
  return acc_order ? by_ntt_acc(tab.logn, go) : by_ntt(tab.logn, go);
}

// ------------------------------------------------------------------ T = M_DB S_Q
// Row i of T is sum_j s~_j * m_i^(j) in R_{N_Q} (s~_j(X) = s_j(1/X), m_i^(j) = chunk j of
// row i).  Exact integers with |T| <= d2 < q_0 / 2, so one prime suffices; the sum is
// accumulated in the NTT domain in registers.  Output row-major T[i][v] (int32).

template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 2), ntt_waves(X::E, 2))))
k_db_T(const int8_t* m_db, int32_t d2, const uint64_t* sconj_hat, int k, NttTab T, int32_t* Trow) {
  extern __shared__ double lds[];
  const int n = 1 << T.logn;
  const int64_t i = blockIdx.x;
  const double q = T.qd, qinv = T.qinv;
  double acc[X::E], x[X::E];
#pragma unroll
  for (int r = 0; r < X::E; ++r) acc[r] = 0.0;
  for (int j = 0; j < k; ++j) {
    const int8_t* m = m_db + i * d2 + (int64_t)j * n;
    const int left = (int)(d2 - (int64_t)j * n);
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      const int v = X::base(r) + (int)threadIdx.x;
      x[r] = X::has(r, n) && v < left ? (double)(int)(m + X::base(r))[threadIdx.x] : 0.0;
    }
    X::fwd(x, lds, T);
    const uint64_t* w = sconj_hat + (int64_t)j * n;
#pragma unroll
    for (int r = 0; r < X::E; ++r)
      if (X::has(r, n))
        acc[r] = reduce_c_d(acc[r] + mulc(x[r], u2d((w + X::base(r))[threadIdx.x]), q, qinv), q, qinv);
  }
  X::inv(acc, lds, T);
#pragma unroll
  for (int r = 0; r < X::E; ++r)
    if (X::has(r, n)) (Trow + i * n + X::base(r))[threadIdx.x] = (int32_t)d2i(acc[r]);
}

__global__ void k_transpose_i32(const int32_t* in, int64_t rows, int64_t cols, int32_t* out) {
  __shared__ int32_t tile[32][33];
  const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
  for (int y = threadIdx.y; y < 32; y += blockDim.y) {
    const int64_t r = r0 + y, c = c0 + threadIdx.x;
    if (r < rows && c < cols) tile[y][threadIdx.x] = in[r * cols + c];
  }
  __syncthreads();
  for (int y = threadIdx.y; y < 32; y += blockDim.y) {
    const int64_t c = c0 + y, r = r0 + threadIdx.x;
    if (r < rows && c < cols) out[c * rows + r] = tile[threadIdx.x][y];
  }
}

hipError_t launch_db_T(const int8_t* m_db, int64_t d1, int32_t d2, const uint64_t* sconj_hat, int k,
                       NttTab tab_q0, int32_t* Trow, int32_t* Tt, hipStream_t s) {
  if (d1 <= 0) return hipSuccess;
  const int n = 1 << tab_q0.logn;
  hipError_t e = tab_q0.logn > kMaxLogN ? launch_db_T_big(m_db, d1, d2, sconj_hat, k, tab_q0, Trow, s)
                                        : by_ntt(tab_q0.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    hipError_t e2 = allow_lds(k_db_T<X>, sizeof(double) * X::LDS);
    if (e2 != hipSuccess) return e2;
    hipLaunchKernelGGL(k_db_T<X>, dim3((unsigned)d1), dim3(block), sizeof(double) * X::LDS, s, m_db, d2, sconj_hat,
                       k, tab_q0, Trow);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)((n + 31) / 32), (unsigned)((d1 + 31) / 32));
  hipLaunchKernelGGL(k_transpose_i32, grid, dim3(32, 8), 0, s, Trow, d1, (int64_t)n, Tt);
  return hipGetLastError();
}

// ------------------------------------------------------------------ database encryption
// One workgroup per column c of D (one a-polynomial): a_c uniform (stream DBA, element
// (v, c)), then for each database chunk j the product s'_j * a_c, and for database rows i of
// chunk j: B[i][c] = -(s'_j a_c)[i - j N_DB] + p * plain[i][c] + e(i, c) (stream DBE).
// plain = M_DB for c < d2, T for c >= d2.  Column c of D is stored contiguously: Dt[c][row].
// ONE: the database has one chunk, so NTT(a_c) need not outlive its product (one polynomial in registers).

template <class X, bool CHAIN, bool ONE>
__global__ void __launch_bounds__(X::MAXT)
    __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, ONE ? 1 : 2), ntt_waves(X::E, ONE ? 1 : 2))))
k_db_encrypt(DbEncArgs A, uint64_t* Dt, uint32_t prime_id, Mod M, NttTab T, const uint64_t* sdb_hat) {
  extern __shared__ double lds[];
  const int n = 1 << T.logn;
  const int64_t c = blockIdx.x;
  uint64_t* col = Dt + c * A.R;
  double ahat[X::E];
  draw_mask<X, CHAIN>(ahat, lds, n, A.seed, stream_tag(kDbA, prime_id), c, M, col);
  X::fwd(ahat, lds, T);  // signed, uncorrected: below 9.1q
  const double q = T.qd, qinv = T.qinv;
  const uint64_t pm = barrett64(A.p, M.q, M.mu);
  const int8_t* errs = A.e + c * A.e_col;
  const int chunks = ONE ? 1 : (int)((A.d1 + n - 1) / n);
  for (int j = 0; j < chunks; ++j) {
    const uint64_t* w = sdb_hat + (int64_t)j * n;
    double x[X::E];
#pragma unroll
    for (int r = 0; r < X::E; ++r)
      x[r] = X::has(r, n) ? mulc(ahat[r], u2d((w + X::base(r))[threadIdx.x]), q, qinv) : 0.0;
    X::inv(x, lds, T);  // centered
    const int64_t lo = (int64_t)j * n;
    const int left = (int)(A.d1 - lo < n ? A.d1 - lo : n);
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      const int v = X::base(r) + (int)threadIdx.x;
      if (!X::has(r, n) || v >= left) continue;
      const int64_t i = lo + v;
      const int32_t pl = c < A.d2 ? (int32_t)A.MT[c * A.d1 + i] : A.Tt[(c - A.d2) * A.d1 + i];
      const int32_t e = errs[i];
      if constexpr (CHAIN)  // |p pl| < 2^16 2^31
        col[n + i] = from_signed((int64_t)pm * pl - d2i(x[r]) + e, M.q, M.mu);
      else
        col[n + i] = d2residue(mulc((double)pl, u2d(pm), q, qinv) - x[r] + (double)e, q, qinv);
    }
  }
}

hipError_t launch_db_encrypt(const DbEncArgs& a, uint64_t* Dt_prime, uint32_t prime_id, const Mod& m,
                             NttTab tab_db, const uint64_t* sdb_hat_prime, hipStream_t s) {
  if (a.K <= 0) return hipSuccess;
  if (tab_db.logn > kMaxLogN) return launch_db_encrypt_big(a, Dt_prime, prime_id, m, tab_db, sdb_hat_prime, s);
  if (!a.e) return hipErrorInvalidValue;
  const bool chain = m.q != tab_db.q;  // residues mod n^2, products through the table's prime
  const bool one = a.d1 <= (1ll << tab_db.logn);
  return by_ntt(tab_db.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    auto kern = chain ? (one ? k_db_encrypt<X, true, true> : k_db_encrypt<X, true, false>)
                      : (one ? k_db_encrypt<X, false, true> : k_db_encrypt<X, false, false>);
    hipError_t e = allow_lds(kern, sizeof(double) * X::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.K), dim3(block), sizeof(double) * X::LDS, s, a, Dt_prime, prime_id, m,
                       tab_db, sdb_hat_prime);
    e = hipGetLastError();
    if (e != hipSuccess || a.e_col) return e;
    return launch_add_errors(a.seed, kDbE, a.cdt, a.K, a.d1, nullptr, Dt_prime + (1ll << tab_db.logn), a.R, m.q, s);
  });
}

}  // namespace hfe
