// Negacyclic NTT of degree 2^9 .. 2^14 with the polynomial in registers: one workgroup per polynomial, E = 8,
// 16 or 32 coefficients per thread, three or four rounds of up to five butterfly stages each, and LDS only to
// exchange the values between two rounds.
//
// What bounds it: with the polynomial resident in LDS (hfe_ntt_lds.h) a transform of 2^14 read and wrote all of
// it five times between barriers, computed every LDS and twiddle address, and its 128 KiB left one workgroup per
// CU, so nothing ran under its memory phases.  Here two exchanges remain, all addresses are a thread's base plus
// an immediate, half of the polynomial at a time passes through LDS (HALF: 67 KiB at 2^14, two workgroups per
// CU), and values are loaded and stored once, coalesced, straight from and to registers.  Measured per transform
// on a full chip (load, forward transform, store; 2^26 coefficients): degree 2^14 410 -> 272 us, 2^13 340 -> 220,
// 2^12 345 -> 193 (5.6 TB/s); inverse 490 -> 318, 455 -> 255, 427 -> 222.
//
// Values are signed integers held in doubles, as in the LDS transforms on signed values: a forward transform of
// values below 2q stays below 9.1q (each stage adds at most (1/2 + 2^-11) q); an inverse round starts from
// centered representatives, so its S <= 5 stages keep sums below 2^S (1/2 + 2^-11) q <= 16.1q, the range the
// centered product takes (mulmod_c_d, hfe_exact.h).
//
// Order: register r of thread t holds coefficient r TH + t, and on the transformed side the value kept at
// r TH + t of an array (ntt_point gives the transform's point).  Every array in the transform domain uses
// that order, so that its loads and stores are coalesced without a pass through LDS.
#pragma once
#include <utility>

#include "hfe_ntt_lds.h"
#include "hfe_ntt_plan.h"

namespace hfe {

// waits for this wave's LDS operations and then for the workgroup; loads from memory stay in flight
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A pointer to device memory as such: one that reaches the kernel inside a struct would be read with flat loads,
// which wait on LDS and memory counters together.
template <class T>
using gptr = const __attribute__((address_space(1))) T*;
template <class T>
__device__ __forceinline__ gptr<T> as_global(const T* p) {
  return (gptr<T>)(p);
}

// the residue in [0, q) of an integer below 2^47 in magnitude
__device__ __forceinline__ uint64_t d2residue(double x, double q, double qinv) {
  return d2u(residue_of_c(reduce_c_d(x, q, qinv), q));
}

// a w mod q centered; SMALL: q < 2^24 and |a| <= 16q, so the product is exact in a double
template <bool SMALL = false>
__device__ __forceinline__ double mulc(double a, double w, double q, double qinv) {
  if constexpr (SMALL) {
#pragma clang fp contract(off)
    const double p = a * w;
    return __builtin_fma(-__builtin_rint(p * qinv), q, p);
  } else {
    return mulmod_c_d(a, w, q, qinv);
  }
}

typedef double v2d __attribute__((ext_vector_type(2)));

template <class F, int... I>
__device__ __forceinline__ void static_for_(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_(f, std::make_integer_sequence<int, N>{});
}

// doubles of LDS (half: half of the values at a time)
constexpr int ntt_lds(int L, int e, bool half) {
  const NttPlan p = ntt_plan(L, e);
  const int n = half ? 1 << (L - 1) : 1 << L;
  int most = 0;
  for (int x = 0; x + 1 < p.n; ++x) {
    const int z = n + (n >> p.sh[x]) * p.pad[x];
    most = z > most ? z : most;
  }
  return most;
}

template <int L, int e = ntt_def_e(L), bool HALF_ = (L >= 12)>
struct RegNtt {
  static constexpr NttPlan P = ntt_plan(L, e);
  static constexpr int E = 1 << e, LT = L - e, TH = 1 << LT, NR = P.n, MAXT = TH;
  static constexpr bool HALF = HALF_;
  static constexpr int LDS = ntt_lds(L, e, HALF);

  // S of round r and its low bit
  static constexpr int S(int r) { return P.s[r]; }
  static constexpr int LO(int r) {
    int lo = L;
    for (int i = 0; i <= r; ++i) lo -= P.s[i];
    return lo;
  }
  // index of register m of thread t in round r: the thread's part and the register's part (disjoint bits)
  template <int R>
  __device__ __forceinline__ static int tpart(int t) {
    if constexpr (R == 0) return t;
    constexpr int lo = LO(R), hi = lo + S(R);
    return ((t >> lo) << hi) | (t & ((1 << lo) - 1));
  }
  template <int R>
  static constexpr int mpart(int m) {
    constexpr int s = S(R), lo = LO(R), hi = lo + s;
    const int j = m >> s, k = m & ((1 << s) - 1);
    const int g = j << LT;  // lies above the thread's bits
    return ((g >> lo) << hi) | (k << lo);
  }
  template <int X>
  __device__ __host__ static constexpr int place(int i) {
    return i + (i >> P.sh[X]) * P.pad[X];
  }
  // exchange X: values held in round FROM's order to round TO's
  template <int X, int FROM, int TO>
  __device__ __forceinline__ static void exchange(double (&x)[E], double* lds) {
    const int t = threadIdx.x;
    if constexpr (!HALF) {
      const int pw = place<X>(tpart<FROM>(t)), pr = place<X>(tpart<TO>(t));
      lds_barrier();
#pragma unroll
      for (int m = 0; m < E; ++m) lds[pw + place<X>(mpart<FROM>(m))] = x[m];
      lds_barrier();
#pragma unroll
      for (int m = 0; m < E; ++m) x[m] = lds[pr + place<X>(mpart<TO>(m))];
    } else {
      constexpr int H = 1 << (L - 1);
      const int pw = place<X>(tpart<FROM>(t) & (H - 1)), pr = place<X>(tpart<TO>(t) & (H - 1));
      constexpr bool wt = (E >> S(FROM)) == 1 && FROM != 0;  // the top index bit is the thread's
      constexpr bool rt = (E >> S(TO)) == 1 && TO != 0;
      const bool thi = __builtin_amdgcn_readfirstlane(t) >= TH / 2;
      // the values are formed here: the compiler would sink the last stage's additions past the branches and
      // keep both operands of each
#pragma unroll
      for (int m = 0; m < E; ++m) asm volatile("" : "+v"(x[m]));
      double y[E];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        lds_barrier();
        if (!wt || thi == (p == 1)) {
#pragma unroll
          for (int m = 0; m < E; ++m)
            if (wt || (mpart<FROM>(m) >= H) == (p == 1)) lds[pw + place<X>(mpart<FROM>(m) & (H - 1))] = x[m];
        }
        lds_barrier();
        if (!rt || thi == (p == 1)) {
#pragma unroll
          for (int m = 0; m < E; ++m)
            if (rt || (mpart<TO>(m) >= H) == (p == 1)) y[m] = lds[pr + place<X>(mpart<TO>(m) & (H - 1))];
        }
      }
#pragma unroll
      for (int m = 0; m < E; ++m) x[m] = y[m];
    }
  }
  // A round runs its stages in steps of at most CW twiddles: step (stage s, part c) covers the butterflies of
  // twiddles c CW .. of that stage (group j's 2^b consecutive table entries, b = s forward, S - 1 - s inverse,
  // at j 2^b).  Each step's twiddles are loaded while the step before it computes; the scheduling barriers keep
  // the compiler from hoisting more of them, which spills.
  static constexpr int CW = L <= 12 && E == 16 ? 8 : 4;
  static constexpr int n_tw(int r, int b) { return (E >> S(r)) << b; }
  static constexpr int n_steps(int r, bool inv) {
    int n = 0;
    for (int s = 0; s < S(r); ++s) n += (n_tw(r, inv ? S(r) - 1 - s : s) + CW - 1) / CW;
    return n;
  }
  static constexpr int step_stage(int r, bool inv, int i) {
    for (int s = 0; s < S(r); ++s) {
      const int c = (n_tw(r, inv ? S(r) - 1 - s : s) + CW - 1) / CW;
      if (i < c) return s;
      i -= c;
    }
    return -1;
  }
  static constexpr int step_part(int r, bool inv, int i) {
    for (int s = 0; s < S(r); ++s) {
      const int c = (n_tw(r, inv ? S(r) - 1 - s : s) + CW - 1) / CW;
      if (i < c) return i;
      i -= c;
    }
    return 0;
  }
  // the twiddles of step I of round R
  template <int R, bool INV, int I>
  __device__ __forceinline__ static void load_step(double (&w)[CW], const NttTab& T) {
    constexpr int s_ = S(R), lo = LO(R), s = step_stage(R, INV, I), b = INV ? s_ - 1 - s : s;
    constexpr int t0 = step_part(R, INV, I) * CW, cnt = n_tw(R, b) - t0 < CW ? n_tw(R, b) - t0 : CW;
    const double* tab = INV ? T.ipsi_d : T.psi_d;
    if constexpr (R == 0) {
      const auto* p = (const __attribute__((address_space(4))) double*)(tab + (1 << b) + t0);
      static_for<cnt>([&](auto ic) { w[decltype(ic)::value] = p[decltype(ic)::value]; });
    } else {
      constexpr int run = cnt < (1 << b) ? cnt : 1 << b;  // consecutive entries of one group
      static_for<cnt / run>([&](auto jc) {
        constexpr int c0 = decltype(jc)::value * run, j = (t0 + c0) >> b, o = (t0 + c0) & ((1 << b) - 1);
        const int B = (threadIdx.x + (j << LT)) >> lo;
        const gptr<double> p = as_global(tab) + ((((1 << (L - lo - s_)) + B) << b) + o);
        if constexpr (run == 1) {
          w[c0] = p[0];
        } else {
          static_for<run / 2>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const v2d v = ((const __attribute__((address_space(1))) v2d*)p)[i];
            w[c0 + 2 * i] = v[0];
            w[c0 + 2 * i + 1] = v[1];
          });
        }
      });
    }
  }
  template <int R, bool SM, bool INV, int I>
  __device__ __forceinline__ static void run_step(double (&x)[E], const double (&w)[CW], const NttTab& T) {
    constexpr int s_ = S(R), s = step_stage(R, INV, I), b = INV ? s_ - 1 - s : s;
    constexpr int t0 = step_part(R, INV, I) * CW, cnt = n_tw(R, b) - t0 < CW ? n_tw(R, b) - t0 : CW;
    constexpr int h = 1 << (s_ - 1 - b);  // half-size in registers
#pragma unroll
    for (int c = 0; c < cnt; ++c)
#pragma unroll
      for (int u = 0; u < h; ++u) {
        const int k = (t0 + c) * 2 * h + u;  // twiddle t serves registers t 2h .. (t + 1) 2h - 1
        double& X = x[k];
        double& Y = x[k + h];
        if constexpr (INV) {
          const double d = X - Y;
          X = X + Y;
          Y = mulc<SM>(d, w[c], T.qd, T.qinv);
        } else {
          const double v = mulc<SM>(Y, w[c], T.qd, T.qinv);
          Y = X - v;
          X = X + v;
        }
        if ((c * h + u) % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
  }
  template <int R, bool SM, bool INV, int I>
  __device__ __forceinline__ static void steps(double (&x)[E], const double (&w)[CW], const NttTab& T) {
    constexpr int n = n_steps(R, INV);
    double w2[CW];
    if constexpr (I + 1 < n) load_step<R, INV, I + 1>(w2, T);
    run_step<R, SM, INV, I>(x, w, T);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (I + 1 < n) steps<R, SM, INV, I + 1>(x, w2, T);
  }
  template <int R, bool SM, bool INV>
  __device__ __forceinline__ static void round(double (&x)[E], const double (&w)[CW], const NttTab& T) {
    if constexpr (INV) {
#pragma unroll
      for (int m = 0; m < E; ++m) x[m] = reduce_c_d(x[m], T.qd, T.qinv);
    }
    steps<R, SM, INV, 0>(x, w, T);
  }
  template <int R, bool SM>
  __device__ __forceinline__ static void fwd_from(double (&x)[E], const double (&w)[CW], double* lds, const NttTab& T) {
    round<R, SM, false>(x, w, T);
    if constexpr (R + 1 < NR) {
      double w2[CW];
      load_step<R + 1, false, 0>(w2, T);
      exchange<R, R, R + 1>(x, lds);
      fwd_from<R + 1, SM>(x, w2, lds, T);
    }
  }
  template <int R, bool SM>
  __device__ __forceinline__ static void inv_from(double (&x)[E], const double (&w)[CW], double* lds, const NttTab& T) {
    round<R, SM, true>(x, w, T);
    if constexpr (R > 0) {
      double w2[CW];
      exchange<R - 1, R, R - 1>(x, lds);
      load_step<R - 1, true, 0>(w2, T);
      inv_from<R - 1, SM>(x, w2, lds, T);
    }
  }
  // The tables behind pointers the compiler cannot see through: in a loop over transforms it would otherwise keep
  // every twiddle it can across the iterations, and spill.
  __device__ __forceinline__ static NttTab opaque(NttTab T) {
    asm volatile("" : "+s"(T.psi_d), "+s"(T.ipsi_d));
    return T;
  }
  // Forward transform of x (signed, below 2q): below 9.1q.  Inverse of x (signed, below 2^47): centered.
  template <bool SM = false>
  __device__ __forceinline__ static void fwd(double (&x)[E], double* lds, const NttTab& tab) {
    const NttTab T = opaque(tab);
    double w[CW];
    load_step<0, false, 0>(w, T);
    fwd_from<0, SM>(x, w, lds, T);
  }
  template <bool SM = false>
  __device__ __forceinline__ static void inv(double (&x)[E], double* lds, const NttTab& tab) {
    const NttTab T = opaque(tab);
    double w[CW];
    load_step<NR - 1, true, 0>(w, T);
    inv_from<NR - 1, SM>(x, w, lds, T);
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = mulc<SM>(x[m], T.n_inv_d, T.qd, T.qinv);
  }

  // ---- the interface shared with LdsNtt
  // whether register r of this thread holds a value, and the offset of register 0 .. E - 1's values from the
  // thread's first
  __device__ __forceinline__ static constexpr bool has(int, int) { return true; }
  __device__ __forceinline__ static int base(int r) { return r * TH; }
  // x[r] = the value of index base(r) + t, with gen(v, o) giving those of indices 4 v .. 4 v + 3 (a thread
  // makes E / 4 quads, which change threads through LDS)
  template <class Gen>
  __device__ __forceinline__ static void from_quads(double (&x)[E], double* lds, int, Gen gen) {
    static_for<E / 4>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      double o[4];
      gen(i * TH + (int)threadIdx.x, o);
      for (int j = 0; j < 4; ++j) x[4 * i + j] = o[j];
    });
    constexpr int PH = HALF ? 2 : 1, C = E / PH;
    double y[E];
#pragma unroll
    for (int p = 0; p < PH; ++p) {
      lds_barrier();
#pragma unroll
      for (int i = 0; i < C / 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) lds[4 * (i * TH + (int)threadIdx.x) + j] = x[p * C + 4 * i + j];
      lds_barrier();
#pragma unroll
      for (int r = 0; r < C; ++r) y[p * C + r] = (lds + r * TH)[threadIdx.x];
    }
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = y[r];
  }
};

// The same interface over the LDS-resident transforms, for degrees up to 2^8 (workgroups of 64 or 128 threads,
// natural order on both sides; a value is present where its index lies below n).
struct LdsNtt {
  static constexpr int E = 2, LDS = 256, MAXT = 128;
  __device__ __forceinline__ static bool has(int r, int n) { return (int)(threadIdx.x + r * blockDim.x) < n; }
  __device__ __forceinline__ static int base(int r) { return r * blockDim.x; }
  template <bool SM = false>
  __device__ __forceinline__ static void fwd(double (&x)[E], double* lds, const NttTab& T) {
    put(x, lds, 1 << T.logn);
    ntt_fwd_lds_c(lds, T);
    get(x, lds, 1 << T.logn);
  }
  template <bool SM = false>
  __device__ __forceinline__ static void inv(double (&x)[E], double* lds, const NttTab& T) {
    put(x, lds, 1 << T.logn);
    ntt_inv_lds_c(lds, T);
    get(x, lds, 1 << T.logn);
    // the LDS transform returns residues: centered here, as the register transform's results are
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = x[r] > 0.5 * T.qd ? x[r] - T.qd : x[r];
  }
  template <class Gen>
  __device__ __forceinline__ static void from_quads(double (&x)[E], double* lds, int n, Gen gen) {
    for (int v = threadIdx.x; v < (n + 3) / 4; v += blockDim.x) {
      double o[4];
      gen(v, o);
      for (int j = 0; j < 4; ++j)
        if (4 * v + j < n) lds[4 * v + j] = o[j];
    }
    __syncthreads();
    get(x, lds, n);
  }
  __device__ __forceinline__ static void put(const double (&x)[E], double* lds, int n) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r)
      if (has(r, n)) lds[threadIdx.x + r * blockDim.x] = x[r];
    __syncthreads();
  }
  __device__ __forceinline__ static void get(double (&x)[E], const double* lds, int n) {
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = has(r, n) ? lds[threadIdx.x + r * blockDim.x] : 0.0;
  }
};

// Waves per SIMD that a kernel with `polys` polynomials in registers is built for (512 registers per lane,
// about 60 beside the polynomials).  With 32 values a thread (2^13, 2^14) that is 4 waves of 128 registers for one
// polynomial, and the exchange in halves alone keeps 1.5 of it live, so those kernels spill registers at its ends: the
// fold's lifts 44 to 104, k_q_encrypt 48 to 52 and k_db_encrypt 18 to 20 with one chunk, k_ntt_fwd 8 and 40,
// k_dec_products 10 to 12.  The kernels with sums beside the transform spill 77 or 78 (k_fold_ks_mac at 2^13 and 2^14),
// 86 and 116 (k_fs_ring and k_fs_conv at 2^14); all others at most 8.
constexpr int ntt_waves(int E, int polys) {
  const int w = 512 / (2 * E * polys + 60);
  return w > 4 ? 4 : w < 1 ? 1 : w;
}

// f(X{}, block size) with the transform of degree 2^logn (logn <= kRegLogMax).  by_ntt_acc: at most 16 values per
// thread (four rounds at 2^13 and 2^14), for the kernels that keep sums of two or more polynomials in registers
// beside the transform, and 8 at 2^10 and 2^11 (four rounds), where 16 left 64 and 128 threads to a polynomial and the
// chip short of waves: ring switch of 151 columns at 2^11, 64 terms 336 and 253 us, conversion of 113 columns 88 and 54;
// of 56 columns at 2^10 50 and 36, 32 and 17 (402 columns: 1,007 and 1,059, 62 and 45).  At 2^12 8 values lose (ring
// switch 96 and 134 us).  The two differ in the order of the transform domain at 2^10, 2^11, 2^13 and 2^14.
template <class F>
static hipError_t by_ntt_common(int logn, F f) {
  switch (logn) {
    case 9: return f(RegNtt<9>{}, RegNtt<9>::TH);
    case 12: return f(RegNtt<12>{}, RegNtt<12>::TH);
    default: return logn < kRegLogMin ? f(LdsNtt{}, ntt_block(logn)) : hipErrorInvalidValue;
  }
}

template <class F>
static hipError_t by_ntt(int logn, F f) {
  switch (logn) {
    case 10: return f(RegNtt<10>{}, RegNtt<10>::TH);
    case 11: return f(RegNtt<11>{}, RegNtt<11>::TH);
    case 13: return f(RegNtt<13>{}, RegNtt<13>::TH);
    case 14: return f(RegNtt<14>{}, RegNtt<14>::TH);
    default: return by_ntt_common(logn, f);
  }
}
template <class F>
static hipError_t by_ntt_acc(int logn, F f) {
  switch (logn) {
    case 10: return f(RegNtt<10, 3>{}, RegNtt<10, 3>::TH);
    case 11: return f(RegNtt<11, 3>{}, RegNtt<11, 3>::TH);
    case 13: return f(RegNtt<13, 4>{}, RegNtt<13, 4>::TH);
    case 14: return f(RegNtt<14, 4>{}, RegNtt<14, 4>::TH);
    default: return by_ntt_common(logn, f);
  }
}

// ------------------------------------------------------------------ shared by the kernels of both rings
// The n^2 modulus chain multiplies by the ternary secrets through the NTT prime q of the tables: a
// residue x mod m (m = n^2 < 2^16) enters as its centered integer, and every product coefficient is an
// integer of magnitude at most N m / 2 <= 2^31 < q / 2, so the centered result mod q is that integer,
// which is then reduced mod m.  (For the 36-bit primes m = q: a residue enters as it is, and the
// result is reduced mod q.)
template <bool CHAIN>
__device__ __forceinline__ double enter_ntt(uint64_t x, uint64_t m) {
  return CHAIN ? (double)(int32_t)centered(x, m) : u2d(x);
}

template <class X>
__device__ __forceinline__ void load_poly(double (&x)[X::E], const uint64_t* p, int n) {
#pragma unroll
  for (int r = 0; r < X::E; ++r) x[r] = X::has(r, n) ? u2d((p + X::base(r))[threadIdx.x]) : 0.0;
}

// Multiply-accumulate of a transformed polynomial with NK key polynomials, acc[p] += x k[p] (centered products,
// exact integers: mulmod_c_d), in groups of G registers.  The keys of a group are loaded D groups ahead, the first
// D groups' (keys_begin) before the transform whose output they multiply, and x takes the next polynomial's values
// as its registers fall free, so that neither waits for memory where its values are used.  (All of a
// polynomial's keys in flight at once spill; loaded where they are used they cost four L2 latencies per
// polynomial.)
template <class X, int NK>
struct KeyMac {
  static constexpr int E = X::E, G = 2, NG = E / G, D = NG < 2 ? NG : 2;
  double kb[D + 1][NK][G];
  const double* key[NK];
  int n;
  template <int g>
  __device__ __forceinline__ void load() {
    static_for<NK>([&](auto pc) {
      constexpr int p = decltype(pc)::value;
      static_for<G>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        kb[g % (D + 1)][p][i] = X::has(g * G + i, n) ? (as_global(key[p]) + X::base(g * G + i))[threadIdx.x] : 0.0;
      });
    });
  }
  __device__ __forceinline__ void keys_begin() {
    static_for<D>([&](auto gc) { load<decltype(gc)::value>(); });
  }
  // next: the polynomial that x holds afterwards (SM: for a prime below 2^24)
  template <bool SM = false>
  __device__ __forceinline__ void run(double (&x)[E], double (&acc)[NK][E], const double* next, double q, double qinv) {
    static_for<NG>([&](auto gc) {
      constexpr int g = decltype(gc)::value;
      if constexpr (g + D < NG) load<g + D>();
      static_for<G>([&](auto ic) {
        constexpr int i = decltype(ic)::value, r = g * G + i;
        static_for<NK>([&](auto pc) {
          constexpr int p = decltype(pc)::value;
          acc[p][r] += mulc<SM>(x[r], kb[g % (D + 1)][p][i], q, qinv);
        });
        x[r] = X::has(r, n) ? (as_global(next) + X::base(r))[threadIdx.x] : 0.0;
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  }
};

// The uniform polynomial of stream key_a, column c (four coefficients from each Philox block), stored to row
// as residues mod M.q and returned as the transform takes it.
template <class X, bool CHAIN>
__device__ __forceinline__ void draw_mask(double (&x)[X::E], double* lds, int n, uint64_t seed, uint64_t key_a,
                                          int64_t c, const Mod& M, uint64_t* row) {
  X::from_quads(x, lds, n, [&](int v4, double (&o)[4]) {
    const Philox4 b = philox4x64_10(seed, key_a, (uint64_t)v4, (uint64_t)c, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = 4 * v4 + j;
      const uint64_t w = b.v[j];
      const uint64_t u = w < M.bound ? barrett64(w, M.q, M.mu) : uniform_at(seed, key_a, (uint64_t)v, (uint64_t)c, M);
      if (v < n) row[v] = u;
      o[j] = enter_ntt<CHAIN>(u, M.q);
    }
  });
}

}  // namespace hfe
