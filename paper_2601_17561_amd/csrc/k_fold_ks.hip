// The fold's key-switching sums and lifts (see k_fold.hip for the evaluator they belong to).
#include "hfe_fold_dev.h"

namespace hfe {
namespace {

// ------------------------------------------------------------------ key switching
// job = s * items + item (slot-major: the blocks that run together share the slot's keys, (level + 1) pairs of
// N doubles, which stay in each XCD's L2), slot z = s (s <= level) or p (s = level + 1).  For each digit i <= level
// (dig[item][i][N], residues mod q_i): reduce mod z, forward NTT, multiply by the key's two parts for (z, i) and
// accumulate (KeyMac: keys and the next digit are loaded ahead of their use).  At z = q_i the
// digit's transform is the NTT-domain value it came from times its factor (src [times y] at slot i, times
// dg.f[i], as the digit pass k_fold_inv with mode 2 describes it), taken directly.  The key of the
// item is keys + kidx[item] * kstride (kidx NULL: key 0), laid out [s][i][2][N] doubles.  Slots of Q_l
// store the NTT-domain sums to acc[item][part][s][N]; the special prime's sums are transformed back,
// centered and stored to accp[item][part][N].
// Signed transforms: each digit's transform is below 9.1z in magnitude, each product centered within
// (1/2 + 2^-11) z, so the sums over at most 4 digits stay below 2.1z.
template <class X>
constexpr int mac_waves() {
  return X::MAXT >= 512 ? 2 : ntt_waves(X::E, 3);
}
template <class X>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(mac_waves<X>(), mac_waves<X>())))
k_fold_ks_mac(FoldConsts C, int level, FoldInv dg, const uint64_t* dig, const double* keys, int64_t kstride,
              const int32_t* kidx, uint64_t* acc_out, double* accp) {
  extern __shared__ double lds[];
  const int n = 1 << C.logn;
  const int nsl = level + 2;
  const int64_t items = gridDim.x / nsl;
  const int s = (int)(blockIdx.x / items);
  const int64_t item = blockIdx.x - s * items;
  const bool special = s == level + 1;
  const int z = special ? 5 : s;
  const double* key = keys + (kidx ? (int64_t)kidx[item] : 0) * kstride + (int64_t)s * (level + 1) * 2 * n;
  const double zd = C.zd[z], zi = C.zinv[z];
  const int64_t off = item * dg.si + s * dg.ss;
  const uint64_t* own = special ? nullptr : dg.src + off;
  const uint64_t* d0 = dig + item * (level + 1) * n;
  by_size(zd, [&](auto smc) {
  constexpr bool SM = decltype(smc)::value;
  double acc[2][X::E], x[X::E];
  if (own) {  // the digit of the slot's own prime
    const double f = dg.f.v[s];
    const uint64_t* y = dg.y ? dg.y + off : nullptr;
    const double* ka = key + (int64_t)s * 2 * n;
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      acc[0][r] = acc[1][r] = 0.0;
      if (!X::has(r, n)) continue;
      double v = u2d(as_global(own + X::base(r))[threadIdx.x]);
      if (y) v = mulc<SM>(v, u2d(as_global(y + X::base(r))[threadIdx.x]), zd, zi);
      v = mulc<SM>(v, f, zd, zi);
      acc[0][r] = mulc<SM>(v, (ka + X::base(r))[threadIdx.x], zd, zi);
      acc[1][r] = mulc<SM>(v, (ka + n + X::base(r))[threadIdx.x], zd, zi);
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int r = 0; r < X::E; ++r) acc[0][r] = acc[1][r] = 0.0;
  }
  // the other digits; x: the bits of the next one's residues
  int i = s == 0 ? 1 : 0;
#pragma unroll
  for (int r = 0; r < X::E; ++r)
    x[r] = X::has(r, n) ? __longlong_as_double((long long)as_global(d0 + (int64_t)i * n + X::base(r))[threadIdx.x]) : 0.0;
  for (;;) {
    const int j = i + 1 == s ? i + 2 : i + 1;
    KeyMac<X, 2> mac;
    mac.n = n;
    mac.key[0] = key + (int64_t)i * 2 * n;  // part 1 of the sums: the mask k_i
    mac.key[1] = mac.key[0] + n;            // part 0: beta_i
    mac.keys_begin();
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      const double v = u2d((uint64_t)__double_as_longlong(x[r]));  // below 2^36: below 2z unless z is small
      x[r] = SM ? reduce_c_d(v, zd, zi) : v;
    }
    X::template fwd<SM>(x, lds, C.tab[z]);
    mac.template run<SM>(x, acc, reinterpret_cast<const double*>(d0 + (int64_t)(j <= level ? j : i) * n), zd, zi);
    if (j > level) break;
    i = j;
  }
  if (!special) {
    uint64_t* ob = acc_out + ((item * 2 + 0) * (level + 1) + s) * n;
    uint64_t* oa = acc_out + ((item * 2 + 1) * (level + 1) + s) * n;
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      if (!X::has(r, n)) continue;
      (ob + X::base(r))[threadIdx.x] = d2residue(acc[1][r], zd, zi);
      (oa + X::base(r))[threadIdx.x] = d2residue(acc[0][r], zd, zi);
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    return;
  }
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    double (&v)[X::E] = acc[1 - part];
    X::inv(v, lds, C.tab[z]);
    double* o = accp + (item * 2 + part) * n;
#pragma unroll
    for (int r = 0; r < X::E; ++r)
      if (X::has(r, n)) (o + X::base(r))[threadIdx.x] = center_exact(v[r], zd);
  }
  });
}

// job = (item * 2 + part) * nsl + s, slot z = zm.z[s]:
// out = (x pm xmul[s] - NTT_z(cen mod z)) inv[s] + addends mod z (pm the plaintext at slot z when given), with
// cen = cen[(item * 2 + part) * N + t] (cen64: the same, 64-bit integers below 2^60), or
// cen = the centered k u mod q_cl from the residues u = ures[(item * 2 + part) * N + t] when ures is given.
// Addends: add (on part 0 only with add_b), the tensor terms of tx and ty (part 0: b_x b_y, part 1: a_x b_y + a_y b_x,
// times tscale[s] with cen64) and, with ures, the constant cres on part 0.  F: which of them the call has, fixed at
// compile time so that no branch separates the loads of a chunk of coefficients.
enum : int { kLiftPm = 1, kLiftAdd = 2, kLiftTensor = 4, kLift64 = 8, kLiftU = 16 };
// PART: the part, fixed where the tensor terms depend on it (-1: any).
template <class X, int F, int PART, bool SM>
__device__ __forceinline__ void lift_body(double* lds, const FoldConsts& C, const FoldLift& a, int64_t item, int part,
                                          int s) {
  const int n = 1 << C.logn;
  const int z = a.zm.z[s];
  const int64_t ip = item * 2 + part;
  const double zd = C.zd[z], zi = C.zinv[z];
  double y[X::E];
  if constexpr (F & kLiftU) {  // a constant's rescale: the centered value of k u mod q_cl, below z
    const gptr<uint64_t> u = as_global(a.ures + ip * n);
    const double qc = C.zd[a.cl], qi = C.zinv[a.cl], ku = a.ku;
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      y[r] = X::has(r, n) ? center_exact(mulc(u2d((u + X::base(r))[threadIdx.x]), ku, qc, qi), qc) : 0.0;
      if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  } else if constexpr (F & kLift64) {
    const gptr<int64_t> c = as_global(a.cen64 + ip * n);
    const double c32 = C.c32[z];
#pragma unroll
    for (int r = 0; r < X::E; ++r) {
      y[r] = X::has(r, n) ? signed64_mod((c + X::base(r))[threadIdx.x], c32, zd, zi) : 0.0;
      if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    const gptr<double> c = as_global(a.cen + ip * n);
#pragma unroll
    for (int r = 0; r < X::E; ++r) y[r] = X::has(r, n) ? reduce_c_d((c + X::base(r))[threadIdx.x], zd, zi) : 0.0;
  }
  X::template fwd<SM>(y, lds, C.tab[z]);  // below 9.1z
  const int64_t so = (int64_t)s * n;
  const gptr<uint64_t> xx = as_global(a.x + item * a.xi + part * a.xp + so);
  const gptr<uint64_t> aa = as_global(a.add + item * a.ai + part * a.ap + so);
  const gptr<uint64_t> tx = as_global(a.tx + item * a.ti + so), ty = as_global(a.ty + item * a.ti + so);
  const gptr<uint64_t> pm = as_global(a.pm + item * a.pmi + (int64_t)z * n);
  const int64_t tp = a.tp;
  uint64_t* o = a.out + item * a.oi + part * a.op + so;
  const double w = a.inv.v[s], km = a.xmul.v[s], kc = part == 0 ? a.cres.v[s] : 0.0, ts = a.tscale.v[s];
  // every term is centered or a residue, so the sum of all stays below 8z: one reduction at the end
  constexpr int CH = X::E < 4 ? X::E : 4;
#pragma unroll
  for (int r = 0; r < X::E; ++r) {
    if (X::has(r, n)) {
      const int b = X::base(r);
      double xv = u2d((xx + b)[threadIdx.x]);
      if constexpr (F & kLiftPm) xv = mulc<SM>(xv, u2d((pm + b)[threadIdx.x]), zd, zi);
      if constexpr (F & kLiftU) xv = mulc<SM>(xv, km, zd, zi);
      double v = mulc<SM>(xv - y[r], w, zd, zi);  // |x - NTT| < 10.1z
      if constexpr (F & kLiftU) v += kc;
      if constexpr (F & kLiftAdd) v += u2d((aa + b)[threadIdx.x]);
      if constexpr (F & kLiftTensor) {
        const double bx = u2d((tx + b)[threadIdx.x]), by = u2d((ty + b)[threadIdx.x]);
        double d;
        if constexpr (PART == 0)
          d = mulc<SM>(bx, by, zd, zi);
        else
          d = mulc<SM>(u2d((tx + tp + b)[threadIdx.x]), by, zd, zi) +
              mulc<SM>(u2d((ty + tp + b)[threadIdx.x]), bx, zd, zi);
        if constexpr (F & kLift64) d = mulc<SM>(d, ts, zd, zi);
        v += d;
      }
      (o + b)[threadIdx.x] = d2residue(v, zd, zi);
    }
    if (r % CH == CH - 1) __builtin_amdgcn_sched_barrier(0);  // no more loads in flight than registers hold
  }
}
template <class X, int F>
__global__ void __launch_bounds__(X::MAXT) __attribute__((amdgpu_waves_per_eu(ntt_waves(X::E, 1), ntt_waves(X::E, 1))))
k_fold_lift(FoldConsts C, FoldLift a) {
  extern __shared__ double lds[];
  const int64_t ip = blockIdx.x / a.nsl;
  const int s = blockIdx.x - (int)(ip * a.nsl);
  const int64_t item = ip >> 1;
  by_size(C.zd[a.zm.z[s]], [&](auto smc) {
    constexpr bool SM = decltype(smc)::value;
    const int part = (int)(ip & 1);
    if constexpr (F & kLiftTensor) {
      if (part == 0)
        lift_body<X, F, 0, SM>(lds, C, a, item, 0, s);
      else
        lift_body<X, F, 1, SM>(lds, C, a, item, 1, s);
    } else if constexpr (F == kLiftAdd) {
      if (part && a.add_b)
        lift_body<X, 0, -1, SM>(lds, C, a, item, part, s);
      else
        lift_body<X, F, -1, SM>(lds, C, a, item, part, s);
    } else {
      lift_body<X, F, -1, SM>(lds, C, a, item, part, s);
    }
  });
}

}  // namespace

hipError_t launch_fold_ks_mac(const FoldConsts& C, int level, const FoldInv& dg, const uint64_t* dig, const double* keys,
                              int64_t kstride, const int32_t* kidx, uint64_t* acc, double* accp, int64_t items,
                              hipStream_t s) {
  if (items <= 0) return hipSuccess;
  return by_ntt(C.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    const size_t lds = sizeof(double) * X::LDS;
    hipError_t e = allow_lds(k_fold_ks_mac<X>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold_ks_mac<X>, dim3((unsigned)(items * (level + 2))), dim3(block), lds, s, C, level, dg,
                       dig, keys, kstride, kidx, acc, accp);
    return hipGetLastError();
  });
}

hipError_t launch_fold_lift(const FoldConsts& C, const FoldLift& a, int64_t items, hipStream_t s) {
  if (items <= 0 || a.nsl <= 0) return hipSuccess;
  const int f = (a.pm ? kLiftPm : 0) | (a.add ? kLiftAdd : 0) | (a.tx ? kLiftTensor : 0) | (a.cen64 ? kLift64 : 0) |
                (a.ures ? kLiftU : 0);
  return by_ntt(C.logn, [&](auto xc, int block) -> hipError_t {
    using X = decltype(xc);
    const size_t lds = sizeof(double) * X::LDS;
    auto go = [&](auto fc) -> hipError_t {
      constexpr int F = decltype(fc)::value;
      hipError_t e = allow_lds(k_fold_lift<X, F>, lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((k_fold_lift<X, F>), dim3((unsigned)(items * 2 * a.nsl)), dim3(block), lds, s, C, a);
      return hipGetLastError();
    };
    switch (f) {
      case 0: return go(std::integral_constant<int, 0>{});
      case kLiftPm: return go(std::integral_constant<int, kLiftPm>{});
      case kLiftAdd: return go(std::integral_constant<int, kLiftAdd>{});
      case kLiftTensor | kLiftAdd: return go(std::integral_constant<int, kLiftTensor | kLiftAdd>{});
      case kLiftTensor | kLift64: return go(std::integral_constant<int, kLiftTensor | kLift64>{});
      case kLiftTensor | kLift64 | kLiftAdd: return go(std::integral_constant<int, kLiftTensor | kLift64 | kLiftAdd>{});
      case kLiftU: return go(std::integral_constant<int, kLiftU>{});
      default: return hipErrorInvalidValue;
    }
  });
}

}  // namespace hfe
