// Elementwise and layout kernels around the contraction: masked ternary encoding, int8
// transpose, digit split of the database, centered CRT lift of the query with its digit
// split, rescale by the special prime, CRT decode, and the plaintext match decision.
#include "hfe_device.h"

namespace hfe {

constexpr int kMaxShifts = 64;
struct Shifts {
  int32_t r[kMaxShifts];
};

// ------------------------------------------------------------------ encode (Section 2.1.3)
// out[(e * S + s) * d2 + t] = m' - 2 (c' AND m'), c' and m' = row e rolled by shifts[s].
__global__ void k_encode(const uint8_t* codes, const uint8_t* masks, int64_t n, int32_t d2,
                         Shifts sh, int32_t n_shifts, int8_t* out) {
  const int64_t row = blockIdx.y;               // e * S + s
  const int64_t e = row / n_shifts;
  const int32_t r = sh.r[row % n_shifts];
  const uint8_t* c = codes + e * d2;
  const uint8_t* m = masks + e * d2;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < d2;
       t += (int64_t)gridDim.x * blockDim.x) {
    int64_t src = (t - r) % d2;
    if (src < 0) src += d2;
    const int cm = c[src] & m[src] & 1;
    out[row * d2 + t] = (int8_t)((m[src] & 1) - 2 * cm);
  }
}

// Input check of a ternary matrix: flag[0] |= 1 if any of its n entries lies outside {-1, 0, 1}.
// Thread: 16 entries (one 16-byte load when m is 16-byte aligned), grid-stride.
__global__ void __launch_bounds__(256) k_check_ternary(const int8_t* m, int64_t n, uint32_t* flag) {
  const bool vec = (reinterpret_cast<uintptr_t>(m) & 15) == 0;
  uint32_t bad = 0;
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 16; i < n;
       i += (int64_t)gridDim.x * blockDim.x * 16) {
    if (vec && i + 16 <= n) {
      const uint4 w = *reinterpret_cast<const uint4*>(m + i);
      const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // byte b is in {-1, 0, 1} iff u = b + 1 (mod 256) is in {0, 1, 2}: no bit above bit 1, and
        // not bits 0 and 1 together (u = 3); the per-byte increment carries into bit 7 at most
        const uint32_t u = ((v[k] & 0x7f7f7f7fu) + 0x01010101u) ^ (v[k] & 0x80808080u);
        bad |= (u & 0xfcfcfcfcu) | (u & (u >> 1) & 0x01010101u);
      }
    } else {
      for (int64_t j = i; j < n && j < i + 16; ++j) bad |= (uint32_t)(m[j] < -1 || m[j] > 1);
    }
  }
  if (bad) atomicOr(flag, 1u);
}

hipError_t launch_check_ternary(const int8_t* m, int64_t n, uint32_t* flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 16 * 256 - 1) / (16 * 256), 4096);
  hipLaunchKernelGGL(k_check_ternary, dim3((unsigned)blocks), dim3(256), 0, s, m, n, flag);
  return hipGetLastError();
}

hipError_t launch_encode(const uint8_t* codes, const uint8_t* masks, int64_t n, int32_t d2,
                         const int32_t* shifts, int32_t n_shifts, int8_t* out, hipStream_t s) {
  if (n <= 0 || d2 <= 0) return hipSuccess;
  if (n_shifts < 1 || n_shifts > kMaxShifts) return hipErrorInvalidValue;
  Shifts sh{};
  for (int i = 0; i < n_shifts; ++i) sh.r[i] = shifts[i];
  dim3 grid((unsigned)((d2 + 255) / 256), (unsigned)(n * n_shifts));
  hipLaunchKernelGGL(k_encode, grid, dim3(256), 0, s, codes, masks, n, d2, sh, n_shifts, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ int8 transpose
__global__ void k_transpose_i8(const int8_t* in, int64_t rows, int64_t cols, int8_t* out) {
  __shared__ int8_t tile[64][65];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  for (int y = threadIdx.y; y < 64; y += blockDim.y) {
    const int64_t r = r0 + y, c = c0 + threadIdx.x;
    if (r < rows && c < cols) tile[y][threadIdx.x] = in[r * cols + c];
  }
  __syncthreads();
  for (int y = threadIdx.y; y < 64; y += blockDim.y) {
    const int64_t c = c0 + y, r = r0 + threadIdx.x;
    if (r < rows && c < cols) out[c * rows + r] = tile[threadIdx.x][y];
  }
}

hipError_t launch_transpose_i8(const int8_t* in, int64_t rows, int64_t cols, int8_t* out,
                               hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64));
  hipLaunchKernelGGL(k_transpose_i8, grid, dim3(64, 4), 0, s, in, rows, cols, out);
  return hipGetLastError();
}

// The five digits of each residue, one plane each.
__global__ void __launch_bounds__(256) k_split_db(const uint64_t* Dt, int64_t K, int64_t R, int64_t KB,
                                                  int64_t R_pad, uint64_t q, int8_t* dig) {
  const SplitAt at = split_at();
  if (at.r >= R_pad) return;
  double x[16];
  split_load(at, Dt, K, R, q, x);
  uint32_t w[kDigits][4] = {};
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    int32_t d[kDigits];
    split5(d2i(x[i]), d);
#pragma unroll
    for (int t = 0; t < kDigits; ++t) w[t][i >> 2] |= ((uint32_t)(d[t] & 255)) << (8 * (i & 3));
  }
#pragma unroll
  for (int t = 0; t < kDigits; ++t) split_store(at, dig, t, KB, R_pad, w[t]);
}

hipError_t launch_split_db(const uint64_t* Dt_prime, int64_t K, int64_t R, int64_t KB, int64_t R_pad,
                           uint64_t q, int8_t* dig_prime, hipStream_t s) {
  hipLaunchKernelGGL(k_split_db, split_grid(R_pad, KB), dim3(256), 0, s, Dt_prime, K, R, KB, R_pad, q, dig_prime);
  return hipGetLastError();
}

// ------------------------------------------------------------------ query lift + digit split
// Element (c, k): residues XT[i][c][k] of L(x) mod q_i, where the lift L(x) is the centered CRT
// value in (-Q/2, Q/2).  Writes Xp[c][k] = L mod p (plain form) and, for every prime of the level
// and p, the 5 digit planes of the centered residue (i8 form), zero in the padding.  The K-range
// KB * 64 is a multiple of the block, so lane quads are whole.
__global__ void __launch_bounds__(256) k_lift(const uint64_t* XT, int64_t d3, int64_t K, int64_t KB,
                                              int64_t d3_pad, LiftArgs la, uint64_t* Xp, int8_t* Xd) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= KB * kKB) return;
  lift_lane(XT, d3, K, KB, d3_pad, la, 0, Xp, Xd, blockIdx.y, k);
}

hipError_t launch_lift(const uint64_t* XT, int64_t d3, int64_t K, int64_t KB, int64_t d3_pad,
                       const LiftArgs& la, uint64_t* Xp, int8_t* Xd, hipStream_t s) {
  const int64_t kpad = KB * kKB;
  const int64_t cols = Xd ? d3_pad : d3;
  dim3 grid((unsigned)((kpad + 255) / 256), (unsigned)cols);
  hipLaunchKernelGGL(k_lift, grid, dim3(256), 0, s, XT, d3, K, KB, d3_pad, la, Xp, Xd);
  return hipGetLastError();
}

// ------------------------------------------------------------------ rescale by p
// out[i][e] = (C[i][e] - centered(Cp[e]) mod q_i) * p^-1 mod q_i = RS_p of the CRT value.
__global__ void k_rescale(const uint64_t* C, const uint64_t* Cp, int64_t n, RescaleArgs ra,
                          uint64_t* out) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    rescale_element(C, Cp, n, ra, out, e, n);
}

hipError_t launch_rescale(const uint64_t* C, const uint64_t* Cp, int64_t n, const RescaleArgs& ra,
                          uint64_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_rescale, dim3((unsigned)blocks), dim3(256), 0, s, C, Cp, n, ra, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ CRT decode
// y residues [level][n] -> Y centered in (-Q/2, Q/2) as a 320-bit two's complement integer,
// ip = floor(Y / 2^s + 1/2) and v = Y / 2^s.
__global__ void k_decode(const uint64_t* y, int64_t n, DecodeArgs da, double* v, int32_t* ip) {
  // every array below is indexed by compile-time constants (loops unrolled to the maximum level,
  // guarded by the actual one), so it stays in registers
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    uint64_t r[HFE_MAX_QPRIMES] = {}, g[HFE_MAX_QPRIMES] = {};
#pragma unroll
    for (int i = 0; i < HFE_MAX_QPRIMES; ++i)
      if (i < da.level) r[i] = y[(int64_t)i * n + e];
    if (da.small)
      garner_digits_u16(r, da.level, da.garner, da.q, da.magic, g);
    else
      garner_digits(r, da.level, da.garner, da.q, da.mu, g);
    // Horner: Y = g_{l-1}; Y = Y * q_i + g_i for i = l-2 .. 0 (5 words, little endian)
    uint64_t w[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < HFE_MAX_QPRIMES; ++i)
      if (i == da.level - 1) w[0] = g[i];
#pragma unroll
    for (int i = HFE_MAX_QPRIMES - 2; i >= 0; --i) {
      if (i > da.level - 2) continue;
      uint64_t carry = g[i];
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const uint64_t lo = w[j] * da.q[i];
        const uint64_t hi = mulhi64(w[j], da.q[i]);
        const uint64_t sm = lo + carry;
        carry = hi + (sm < lo ? 1 : 0);
        w[j] = sm;
      }
    }
    if (above_half(g, da.half_digits, da.level)) {  // Y -= Q
      uint64_t borrow = 0;
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const uint64_t x = w[j], q = da.Qw[j];
        const uint64_t d = x - q - borrow;
        borrow = (x < q || (x == q && borrow)) ? 1 : 0;
        w[j] = d;
      }
    }
    const bool neg = (int64_t)w[4] < 0;
    // v = Y / 2^s
    uint64_t m[5];
    if (neg) {
      uint64_t carry = 1;
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        m[j] = ~w[j] + carry;
        carry = (carry && m[j] == 0) ? 1 : 0;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 5; ++j) m[j] = w[j];
    }
    double mag = 0.0;
#pragma unroll
    for (int j = 4; j >= 0; --j) mag = mag * 18446744073709551616.0 + (double)m[j];
    if (v) v[e] = ldexp(neg ? -mag : mag, -da.delta_log);
    // ip = (Y + 2^(s-1)) >> s, arithmetic
    const int s = da.delta_log;
    const int aw = (s - 1) >> 6;
    uint64_t carry = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const uint64_t add = (s > 0 && j == aw) ? 1ull << ((s - 1) & 63) : 0;
      const uint64_t x = w[j] + add;
      const uint64_t c1 = x < w[j] ? 1 : 0;
      const uint64_t b2 = x + carry;
      const uint64_t c2 = b2 < x ? 1 : 0;
      w[j] = b2;
      carry = c1 | c2;
    }
    const int wi = s >> 6, bi = s & 63;
    uint64_t lo = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      if (j == wi) lo |= w[j] >> bi;
      if (bi && j == wi + 1) lo |= w[j] << (64 - bi);
    }
    ip[e] = (int32_t)(uint32_t)lo;
  }
}

hipError_t launch_decode(const uint64_t* y, int64_t n, const DecodeArgs& da, double* v, int32_t* ip,
                         hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_decode, dim3((unsigned)blocks), dim3(256), 0, s, y, n, da, v, ip);
  return hipGetLastError();
}

// ------------------------------------------------------------------ match decision
// Masks packed into 64-bit words, words-major ([word][row]) so that a row block reads
// contiguous words.  Query masks are rolled by their shifts while packing.
// The bits of four mask bytes, byte k's lowest bit at bit k (the product's partial sums never meet).
__device__ __forceinline__ uint32_t pack4(uint32_t v) { return ((v & 0x01010101u) * 0x01020408u) >> 24 & 15u; }

// 16 mask bytes at any alignment, and their bits.
struct Mask16 {
  uint32_t v[4];
};
__device__ __forceinline__ Mask16 load16(const uint8_t* p) {
  Mask16 x;
  __builtin_memcpy(x.v, p, 16);
  return x;
}
__device__ __forceinline__ uint64_t pack16(const Mask16& x) {
  return pack4(x.v[0]) | pack4(x.v[1]) << 4 | pack4(x.v[2]) << 8 | pack4(x.v[3]) << 12;
}

// Bits t0 .. t0 + 63 of a mask row rolled by r, 0 <= r < d2 (bit b = mask[(t - r) mod d2] & 1, zero beyond d2): four 16-byte
// loads in flight together where the word neither wraps nor ends inside (a branch to each piece makes them wait for
// one another: 30,720 rows of 12,800 157 us, so 98), else in pieces of 16, byte by byte where a piece does.
__device__ __forceinline__ uint64_t pack_word(const uint8_t* m, int32_t d2, int32_t t0, int32_t r) {
  int32_t s0 = t0 - r;
  if (s0 < 0) s0 += d2;
  if (t0 + 64 <= d2 && s0 + 64 <= d2) {
    const Mask16 a = load16(m + s0), b = load16(m + s0 + 16), c = load16(m + s0 + 32), d = load16(m + s0 + 48);
    return pack16(a) | pack16(b) << 16 | pack16(c) << 32 | pack16(d) << 48;
  }
  uint64_t word = 0;
  for (int p = 0; p < 4; ++p) {
    const int32_t t = t0 + 16 * p;
    if (t >= d2) break;
    int32_t src = t - r;
    if (src < 0) src += d2;
    if (t + 16 <= d2 && src + 16 <= d2) {
      word |= pack16(load16(m + src)) << (16 * p);
    } else {
      const int n = d2 - t < 16 ? d2 - t : 16;
      for (int b = 0; b < n; ++b) {
        word |= (uint64_t)(m[src] & 1) << (16 * p + b);
        src = src + 1 == d2 ? 0 : src + 1;
      }
    }
  }
  return word;
}

// Thread (word, row), lanes on consecutive rows of one word (coalesced writes): the first q_items threads pack the
// query masks (columns d3 .. d3p - 1 are zero), the others the database's.  Thread 0 .. n_eyes - 1 also clear
// the eyes' answers, which k_match sets.
__global__ void __launch_bounds__(256)
k_pack_masks(const uint8_t* q_masks, int64_t d3, int64_t d3p, Shifts sh, int32_t n_shifts, const uint8_t* db_masks,
             int64_t rows, int32_t d2, int32_t W, uint64_t* qwords, uint64_t* dbwords, int64_t n_eyes, uint8_t* eye) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_eyes) eye[i] = 0;
  const int64_t q_items = d3p * W;
  if (i < q_items) {
    const int32_t w = (int32_t)(i / d3p);
    const int64_t c = i - (int64_t)w * d3p;  // e * S + s
    qwords[i] = c < d3 ? pack_word(q_masks + c / n_shifts * d2, d2, w * 64, sh.r[c % n_shifts]) : 0;
    return;
  }
  const int64_t j = i - q_items;
  if (j >= rows * W) return;
  const int32_t w = (int32_t)(j / rows);
  const int64_t row = j - (int64_t)w * rows;
  dbwords[j] = pack_word(db_masks + row * d2, d2, w * 64, 0);
}

// Block (row block, column group): thread = one database row, COLS query columns, whose words are the same for every
// thread (scalar loads, four vector instructions per word and column: two ANDs, two counting adds).  U words of the
// row are loaded before the first is used: a thread waits for memory W / U times.
template <int COLS, int U>
__global__ void __launch_bounds__(256)
k_match(const int32_t* ip, const uint64_t* qwords, const uint64_t* dbwords, int64_t d3, int64_t d3p, int64_t rows,
        int32_t W, uint32_t t_num, uint32_t t_den, int32_t n_shifts, uint8_t* decision, uint8_t* eye) {
  const int64_t c0 = (int64_t)blockIdx.y * COLS;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = r < rows;
  const uint64_t* dp = dbwords + (live ? r : 0);
  const auto* qp = (const __attribute__((address_space(4))) uint64_t*)(qwords + c0);
  uint32_t ov[COLS];
#pragma unroll
  for (int cc = 0; cc < COLS; ++cc) ov[cc] = 0;
  for (int w0 = 0; w0 < W; w0 += U) {
    uint64_t dw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) dw[u] = w0 + u < W ? dp[(int64_t)(w0 + u) * rows] : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (w0 + u >= W) break;
      const auto* qw = qp + (int64_t)(w0 + u) * d3p;
#pragma unroll
      for (int cc = 0; cc < COLS; ++cc) {
        const uint64_t q = qw[cc];
        ov[cc] += __popc((uint32_t)q & (uint32_t)dw[u]);
        ov[cc] += __popc((uint32_t)(q >> 32) & (uint32_t)(dw[u] >> 32));
      }
    }
  }
  if (!live) return;
  const int64_t lhs_scale = t_den, rhs_scale = (int64_t)t_den - 2 * (int64_t)t_num;
  int64_t eye_i = c0 / n_shifts;
  int left = n_shifts - (int)(c0 - eye_i * n_shifts);  // columns of this eye still to come
#pragma unroll
  for (int cc = 0; cc < COLS; ++cc) {
    const int64_t c = c0 + cc;
    if (c >= d3) break;
    if (left-- == 0) {
      ++eye_i;
      left = n_shifts - 1;
    }
    const int64_t x = ip[c * rows + r];
    const bool dec = ov[cc] > 0 && x * lhs_scale > rhs_scale * (int64_t)ov[cc];
    if (decision) decision[c * rows + r] = dec ? 1 : 0;
    if (dec) eye[eye_i] = 1;  // benign race: every writer stores 1
  }
}

int64_t match_cols(int64_t d3) { return (d3 + 15) / 16 * 16; }

hipError_t launch_match(const int32_t* ip, const uint8_t* q_masks, int64_t n_eyes,
                        const int32_t* shifts, int32_t n_shifts, const uint8_t* db_masks,
                        int64_t rows, int32_t d2, uint32_t t_num, uint32_t t_den, uint64_t* qwords,
                        uint64_t* dbwords, uint8_t* decision, uint8_t* eye_match, hipStream_t s) {
  if (n_shifts < 1 || n_shifts > kMaxShifts) return hipErrorInvalidValue;
  const int32_t W = (d2 + 63) / 64;
  const int64_t d3 = n_eyes * n_shifts, d3p = match_cols(d3);
  Shifts sh{};
  for (int i = 0; i < n_shifts; ++i) {
    const int64_t r = shifts[i] % (int64_t)d2;
    sh.r[i] = (int32_t)(r < 0 ? r + d2 : r);
  }
  const int64_t items = (d3p + rows) * W;  // at least n_eyes
  hipLaunchKernelGGL(k_pack_masks, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, q_masks, d3, d3p, sh,
                     n_shifts, db_masks, rows, d2, W, qwords, dbwords, n_eyes, eye_match);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // 16 columns per thread where that fills the chip (a word of the row is read once per 16 columns), else 4 columns
  // and blocks of one wavefront
  const int64_t nb = (rows + 255) / 256;
  if (nb * (d3p / 16) >= 512)
    hipLaunchKernelGGL((k_match<16, 4>), dim3((unsigned)nb, (unsigned)(d3p / 16)), dim3(256), 0, s, ip, qwords, dbwords,
                       d3, d3p, rows, W, t_num, t_den, n_shifts, decision, eye_match);
  else
    hipLaunchKernelGGL((k_match<4, 8>), dim3((unsigned)((rows + 63) / 64), (unsigned)((d3 + 3) / 4)), dim3(64), 0, s,
                       ip, qwords, dbwords, d3, d3p, rows, W, t_num, t_den, n_shifts, decision, eye_match);
  return hipGetLastError();
}

}  // namespace hfe
