// Small-modulus (RNS) int8 form of the modular contraction (Section 6.3: matrix products modulo a
// large modulus reduced to int8 products through RNS over small moduli).  For a prime q of the
// basis, C = D X mod q is recovered from the exact integer sum S = sum_k d_k x_k of centered
// residues: S mod m_j for n small pairwise coprime moduli m_j <= 256 (one int8 product each,
// int32 accumulation), then the CRT of those residues to S (the moduli's product exceeds 2 |S|),
// then S mod q.  One int8 product per modulus instead of 25 digit-pair products per prime.
#include "hfe_device.h"

namespace hfe {

// ------------------------------------------------------------------ database split
// The balanced residues of each centered residue modulo the small moduli, one plane each.
__global__ void __launch_bounds__(256) k_split_db_rns(const uint64_t* Dt, int64_t K, int64_t R, int64_t KB,
                                                      int64_t R_pad, uint64_t q, int n_mod, int8_t* dig) {
  const SplitAt at = split_at();
  if (at.r >= R_pad) return;
  double x[16];
  split_load(at, Dt, K, R, q, x);
  for (int j = 0; j < n_mod; ++j) {
    uint32_t w[4] = {};
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i >> 2] |= balanced_byte(x[i], j) << (8 * (i & 3));
    split_store(at, dig, j, KB, R_pad, w);
  }
}

hipError_t launch_split_db_rns(const uint64_t* Dt_prime, int64_t K, int64_t R, int64_t KB, int64_t R_pad,
                               uint64_t q, int n_mod, int8_t* dig_prime, hipStream_t s) {
  hipLaunchKernelGGL(k_split_db_rns, split_grid(R_pad, KB), dim3(256), 0, s, Dt_prime, K, R, KB, R_pad, q, n_mod, dig_prime);
  return hipGetLastError();
}

// ------------------------------------------------------------------ query lift
// Element (c, k): the lift of the query residues (as for the digit form), then for every prime of
// the level and p the balanced residues of the centered value modulo each small modulus:
// Xr[z][j][kb][c][kk], zero in the padding.
template <bool QUAD>
__global__ void __launch_bounds__(256) k_lift_rns(const uint64_t* XT, int64_t d3, int64_t K, int64_t KB,
                                                  int64_t d3_pad, LiftArgs la, int n_mod, int8_t* Xr) {
  const int64_t k = (QUAD ? 4 : 1) * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (k >= KB * kKB) return;
  if constexpr (QUAD)
    lift_quad(XT, d3, K, KB, d3_pad, la, n_mod, nullptr, Xr, blockIdx.y, k);
  else
    lift_lane(XT, d3, K, KB, d3_pad, la, n_mod, nullptr, Xr, blockIdx.y, k);
}

hipError_t launch_lift_rns(const uint64_t* XT, int64_t d3, int64_t K, int64_t KB, int64_t d3_pad,
                           const LiftArgs& la, int n_mod, int8_t* Xr, hipStream_t s) {
  const bool quad = KB * kKB * d3_pad >= kLiftQuadFrom;
  const int64_t per_block = quad ? 1024 : 256;
  dim3 grid((unsigned)((KB * kKB + per_block - 1) / per_block), (unsigned)d3_pad);
  hipLaunchKernelGGL(quad ? k_lift_rns<true> : k_lift_rns<false>, grid, dim3(256), 0, s, XT, d3, K, KB, d3_pad, la, n_mod, Xr);
  return hipGetLastError();
}

// ------------------------------------------------------------------ contraction per modulus
// Workgroup tile: 256 database rows x TQ query columns of one (prime, modulus).  Each wave owns 64
// query columns x 128 rows as 2 x 4 blocks of 32 x 32 with one int32 accumulator each
// (v_mfma_i32_32x32x32_i8), so each fragment read from LDS feeds 2 or 4 MFMAs.  One 64-byte K-block
// of both operands per LDS stage, fed by direct global-to-LDS loads (same row swizzle as the digit
// form's DMA tiles).
//   TQ = 256: 4 x 2 waves (two per SIMD), four stages of 32 KiB, one workgroup per CU; up to three
//     K-blocks are in flight while one is multiplied (three stages measured 6% slower, five no faster).
//   TQ = 128: 2 x 2 waves, three stages of 24 KiB, two workgroups per CU.  About 9% slower per
//     column than TQ = 256, but it pads query columns to 128 instead of 256; the host picks the
//     width per call by padded work.
//   TQ = 64, 32: 1 x 4 waves of 2 x 2 and 1 x 2 blocks, three and four stages of 20 and 18 KiB, two workgroups per CU:
//     for calls that only stream the database.
// Exactness: |S| over the K-range <= K * 128 * 128 < 2^31 for K < 2^17 (checked by the host).
template <int TQ>
struct RnsCfg {
  static_assert(TQ == 32 || TQ == 64 || TQ == 128 || TQ == 256, "no such query tile");
  static constexpr int WQB = TQ == 32 ? 1 : 2, WRB = TQ < 128 ? 2 : 4, WPE = 2;  // 32 x 32 blocks per wave; waves per SIMD
  static constexpr int TR = kRnsTileR;
  static constexpr int NQ = TQ / (32 * WQB), NR = TR / (32 * WRB), NW = NQ * NR;
  static constexpr int STAGES = TQ == 256 || TQ == 32 ? 4 : 3;
  static constexpr int PA = TQ * kKB, PB = TR * kKB, STAGE = PA + PB;
  // 16-row loads of a stage, dealt to the waves by index: EVERY of each wave, and one more of the first waves
  static constexpr int LOADS_A = TQ / 16, LOADS = LOADS_A + TR / 16, EVERY = LOADS / NW, NL = (LOADS + NW - 1) / NW;
  static constexpr int VM = EVERY * (STAGES - 2);  // loads a wave may leave in flight at a wait
  static constexpr int LDS = STAGES * STAGE;
  static_assert(STAGES >= 3, "the K-block wait leaves STAGES - 2 blocks in flight");
  static_assert(NW == (TQ == 256 ? 8 : 4), "the launch's block size");
};

// One output tile (rows r0.., query columns c0..) of one (prime, modulus) product: X and D are that
// modulus' query and database planes, res its residue plane [d3][R_out].
struct RnsTile {
  const int8_t* X;
  const int8_t* D;
  uint8_t* res;
  int32_t m;
  uint32_t magic;
  int64_t nk, R_pad, d3_pad, n_db, row0, R_out, d3, r0, c0;  // nk: K-blocks from the first of X and D
};

// this wave's loads of the oldest outstanding K-block have landed (the younger ones may still fly)
// and its LDS reads are done; then the same for every wave
template <int VM>
__device__ __forceinline__ void rns_wait_block() {
  static_assert(VM == 5 || VM == 6 || VM == 8, "no K-block wait for this tile shape");
  if constexpr (VM == 5)
    asm volatile("s_waitcnt vmcnt(5) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else if constexpr (VM == 6)
    asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A query column of a job's tile: its planes, its results' entry of the job's row 0, and the rows that are its own.
struct RnsCol {
  const int8_t* X;
  uint8_t* res;
  int32_t lo, hi;
  int64_t step;  // bytes between its K-blocks
};

// JOB: the tile is of a job's rows (g.D and g.r0, g.R_out) and its columns are `col`; otherwise of one problem.
template <int TQ, bool JOB>
__device__ __forceinline__ void rns_tile(const RnsTile& g, int8_t* lds, const RnsCol* col) {
  using C = RnsCfg<TQ>;
  const int64_t r0 = g.r0, c0 = g.c0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wq = wave % C::NQ, wr = wave / C::NQ;
  const int8_t* X = g.X;
  const int8_t* D = g.D;
  const size_t stepA = (size_t)g.d3_pad * kKB, stepB = (size_t)g.R_pad * kKB;
  // load L fills stage rows 16 L .. 16 L + 15, the query's and then the database's (lane l: row + l / 4, stored chunk
  // l % 4 holding logical chunk (l % 4) ^ ((row >> 2) & 3)); wave w issues loads w, w + NW, ..
  const int ld_chunk = ((lane & 3) ^ ((lane >> 4) & 3)) * 16;
  const int8_t* gp[C::NL];
  size_t colstep[JOB ? C::NL : 1];  // columns of several problems: each its own stride
#pragma unroll
  for (int i = 0; i < C::NL; ++i) {
    const int L = wave + C::NW * i < C::LOADS ? wave + C::NW * i : C::LOADS - 1;
    if (L < C::LOADS_A) {
      const int c = 16 * L + (lane >> 2);
      gp[i] = (JOB ? col[c].X : X + (size_t)(c0 + c) * kKB) + ld_chunk;
      if constexpr (JOB) colstep[i] = col[c].step;
    } else {
      const int64_t r = r0 + 16 * (L - C::LOADS_A) + (lane >> 2);
      gp[i] = D + (size_t)(JOB ? r : src_row(r, g.n_db, g.row0)) * kKB + ld_chunk;
      if constexpr (JOB) colstep[i] = stepB;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds + wave * 16 * kKB;
  auto issue = [&](int stage) {
    const uint32_t base = lds0 + stage * C::STAGE;
#pragma unroll
    for (int i = 0; i < C::NL; ++i)
      if (C::NW * (i + 1) <= C::LOADS || wave + C::NW * i < C::LOADS) dma16(gp[i], base + 16 * C::NW * i * kKB);
  };
  // The load addresses move on to the next K-block; past the last one the loads repeat it.  One 64-bit addition each,
  // issued among the matrix instructions: the products of block index and stride that stood at the barrier instead
  // kept the matrix cores of all its waves waiting: 512 columns, 30,720
  // rows, K = 20,992 in four primes 15.8 ms, now 14.2.
  int32_t left = (int32_t)g.nk - 1;
  auto advance = [&]() {
    const size_t dA = left > 0 ? stepA : 0, dB = left > 0 ? stepB : 0;
    --left;
#pragma unroll
    for (int i = 0; i < C::NL; ++i)
      gp[i] += JOB ? (left >= 0 ? colstep[i] : 0) : wave + C::NW * i < C::LOADS_A ? dA : dB;
  };
  const int sw = ((lane & 31) >> 2) & 3, cl = lane >> 5;
  const int offA = (wq * 32 * C::WQB + (lane & 31)) * kKB;
  const int offB = C::PA + (wr * 32 * C::WRB + (lane & 31)) * kKB;
  v16i acc[C::WQB][C::WRB];
#pragma unroll
  for (int a = 0; a < C::WQB; ++a)
#pragma unroll
    for (int b = 0; b < C::WRB; ++b) acc[a][b] = (v16i){0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const int32_t KB = (int32_t)g.nk;
  // fragments of one half (32 bytes of K) of the K-block in stage st
  auto read_half = [&](int st, int h, v4i (&fa)[C::WQB], v4i (&fb)[C::WRB]) {
    const int8_t* S = lds + st * C::STAGE;
    const int chunk = ((cl + 2 * h) ^ sw) << 4;
#pragma unroll
    for (int a = 0; a < C::WQB; ++a) fa[a] = *reinterpret_cast<const v4i*>(S + offA + a * 32 * kKB + chunk);
#pragma unroll
    for (int b = 0; b < C::WRB; ++b) fb[b] = *reinterpret_cast<const v4i*>(S + offB + b * 32 * kKB + chunk);
  };
  auto mma = [&](const v4i (&fa)[C::WQB], const v4i (&fb)[C::WRB]) {
#pragma unroll
    for (int a = 0; a < C::WQB; ++a)
#pragma unroll
      for (int b = 0; b < C::WRB; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[a], fb[b], acc[a][b], 0, 0, 0);
  };
  // Software pipeline: the fragments of half 0 of block i are in registers when iteration i
  // starts; half 1 is read while half 0 multiplies, and half 0 of block i + 1 while half 1
  // multiplies, so LDS latency hides behind the MFMAs.  The barrier sits between the halves:
  // after it block i + 1 is in LDS and no wave reads block i's stage any more, which then
  // receives block i + STAGES.
#pragma unroll
  for (int st = 0; st < C::STAGES - 1; ++st) {
    issue(st);
    advance();
  }
  rns_wait_block<C::VM>();
  issue(C::STAGES - 1);
  advance();
  v4i f0a[C::WQB], f0b[C::WRB], f1a[C::WQB], f1b[C::WRB];
  read_half(0, 0, f0a, f0b);
  // settle every outstanding LDS and scalar load here, so that the compiler's wait analysis
  // enters the loop with LDS reads only and waits for the older half alone inside it
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt, expcnt untouched
  int cur = 0;
  for (int32_t i = 0; i < KB; ++i) {
    read_half(cur, 1, f1a, f1b);
    __builtin_amdgcn_sched_barrier(0);
    mma(f0a, f0b);
    __builtin_amdgcn_sched_barrier(0);
    rns_wait_block<C::VM>();
    issue(cur);
    cur = cur + 1 == C::STAGES ? 0 : cur + 1;
    read_half(cur, 0, f0a, f0b);  // block i + 1 (a landed duplicate of the last block at the end)
    __builtin_amdgcn_sched_barrier(0);
    advance();
    mma(f1a, f1b);
    __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  // epilogue: S mod m_j in [0, m_j) -> res[z][j][c][r]; 32 x 32 result layout as in the digit
  // form (lane l, element e: query column 8 (e / 4) + 4 (l / 32) + e % 4, row l % 32)
  const uint32_t m = (uint32_t)g.m;
  const uint32_t magic = g.magic;
  const RnsAccConsts ac = rns_acc_consts(m, magic);  // |acc| < 2^31 -> acc mod m (hfe_exact.h)
  if constexpr (JOB) {
#pragma unroll
    for (int a = 0; a < C::WQB; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const RnsCol& cc = col[wq * 32 * C::WQB + a * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)];
        uint8_t* out = cc.res;
        const int32_t lo = cc.lo, hi = cc.hi;
#pragma unroll
        for (int b = 0; b < C::WRB; ++b) {
          const int64_t r = r0 + wr * 32 * C::WRB + b * 32 + (lane & 31);
          if (r >= lo && r < hi) out[r] = (uint8_t)rns_acc_mod(acc[a][b][e], m, magic, ac);
        }
      }
    return;
  }
  uint8_t* res = g.res;
#pragma unroll
  for (int b = 0; b < C::WRB; ++b) {
    const int64_t r = r0 + wr * 32 * C::WRB + b * 32 + (lane & 31);
    if (r >= g.R_out) continue;
#pragma unroll
    for (int a = 0; a < C::WQB; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int64_t c = c0 + wq * 32 * C::WQB + a * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (c >= g.d3) continue;
        res[c * g.R_out + r] = (uint8_t)rns_acc_mod(acc[a][b][e], m, magic, ac);
      }
  }
}

template <int TQ>
__global__ void __launch_bounds__(64 * RnsCfg<TQ>::NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_gemm_rns(RnsGemmArgs g) {
  using C = RnsCfg<TQ>;
  __shared__ __attribute__((aligned(16))) int8_t lds[C::LDS];
  const int64_t n_ct = (g.d3 + TQ - 1) / TQ, n_rt = (g.R_out + C::TR - 1) / C::TR;
  const int ns = g.splits;
  TileAt at;
  if (!xcd_tile(g.n_mod * ns * g.nz, n_rt, n_ct, at)) return;
  const int64_t ct = at.ct, rt = at.rt;
  const int zs = uniform(at.plane / g.n_mod), j = at.plane - zs * g.n_mod, z = uniform((uint32_t)zs / ns), sp = zs - z * ns;
  const int64_t k0 = g.KB * sp / ns, k1 = g.KB * (sp + 1) / ns;  // part sp of the K-blocks
  RnsTile t{g.Xr[z] + ((size_t)j * g.KB + k0) * g.d3_pad * kKB, g.Dr[z] + ((size_t)j * g.KB + k0) * g.R_pad * kKB,
            g.res + (((size_t)sp * g.nz + z) * g.n_mod + j) * g.d3 * g.R_out, g.m[j], g.magic[j], k1 - k0, g.R_pad, g.d3_pad, g.n_db,
            g.row0, g.R_out, g.d3, rt * C::TR, ct * TQ};
  rns_tile<TQ, false>(t, lds, nullptr);
}

// Persistent batched form: workgroups claim the jobs' tiles in order from one counter per XCD, slot t from XCD t mod
// 8's, as the digit form's batched kernel.  What bounds it is reading the database planes, which is why requests on the
// same rows share a job: twelve requests of 16 .. 128 columns on shards of 30,720 rows, K = 20,992 read 133 GB request
// by request (20.2 + 6.3 ms), 71 GB in shared jobs (14.0 + 3.9 ms).
template <int TQ>
__global__ void __launch_bounds__(64 * RnsCfg<TQ>::NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_gemm_rns_batched(RnsBatchArgs a) {
  using C = RnsCfg<TQ>;
  __shared__ __attribute__((aligned(16))) int8_t lds[C::LDS];
  __shared__ RnsCol col[TQ];
  // this launch's jobs and tiles (read on the device, so that a captured graph serves any batch)
  constexpr bool narrow = TQ == 128;
  const int p_lo = narrow ? a.hdr->n_wide : 0, p_hi = narrow ? a.hdr->n : a.hdr->n_wide;
  const int64_t t_lo = narrow ? a.hdr->tiles_wide : 0, t_hi = narrow ? a.hdr->total_tiles : a.hdr->tiles_wide;
  uint32_t* next = narrow ? a.next_narrow : a.next;
  const int xcd = blockIdx.x % kXcds;
  const int64_t per_xcd = (t_hi - t_lo) / kXcds;
  for (;;) {
    __syncthreads();  // the previous tile is done with LDS
    if (threadIdx.x == 0) *reinterpret_cast<uint32_t*>(lds) = atomicAdd(next + xcd, 1u);
    __syncthreads();
    const int64_t jc = (uint32_t)__builtin_amdgcn_readfirstlane(*reinterpret_cast<const uint32_t*>(lds));
    __syncthreads();  // every thread has read the claim before the tile overwrites LDS
    if (jc >= per_xcd) break;
    const int64_t t = t_lo + jc * kXcds + xcd;
    int lo = p_lo, hi = p_hi - 1;  // last problem of this launch whose first tile is <= t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.job[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
    }
    const RnsJob& d = a.job[lo];
    const int64_t n_ct = (d.cols + TQ - 1) / TQ, n_rt = (d.rows + C::TR - 1) / C::TR;
    TileAt at;
    if (!batch_tile(t - d.tile_begin, a.n_mod, n_rt, n_ct, d.rot, at)) continue;
    const int64_t ct = at.ct, rt = at.rt;
    const int j = at.plane;
    if (threadIdx.x < TQ) {  // the column's segment; padding columns read the last column and keep nothing
      const int64_t want = ct * TQ + threadIdx.x;
      const int64_t c = d.col0 + (want < d.cols ? want : d.cols - 1);
      int64_t first = 0, at0 = 0;
      int sel = 0;
      for (int i = 0; i < d.n_seg; ++i) {
        if (c >= first) {
          sel = i;
          at0 = first;
        }
        first += a.seg[d.seg + i].cols;
      }
      const RnsSeg g = a.seg[d.seg + sel];
      const int64_t k = c - at0, zj = (int64_t)(d.n_slot_p ? g.level : d.slot) * a.n_mod + j;
      col[threadIdx.x] = RnsCol{g.X + (zj * a.KB * g.d3_pad + k) * kKB, g.res + (zj * g.cols + k) * g.R_out,
                                want < d.cols ? g.lo : 0, want < d.cols ? g.hi : 0, g.d3_pad * kKB};
    }
    __syncthreads();
    RnsTile tl{nullptr, a.Dr + (((size_t)d.slot * a.n_mod + j) * a.KB * a.R_pad + d.db_row) * kKB, nullptr, a.m[j],
               a.magic[j], a.KB, a.R_pad, 0, 0, 0, d.rows, d.cols, rt * C::TR, ct * TQ};
    rns_tile<TQ, true>(tl, lds, col);
  }
}

int64_t rns_batched_tiles(int64_t cols, int64_t rows, int n_mod, int tq, int64_t* groups) {
  *groups = (rows + kRnsTileR - 1) / kRnsTileR * n_mod;
  return batch_slots(*groups, (cols + tq - 1) / tq);
}

hipError_t launch_gemm_rns_batched(const RnsBatchArgs& a, int grid, int tq, hipStream_t s) {
  if (tq == 128)
    hipLaunchKernelGGL(k_gemm_rns_batched<128>, dim3((unsigned)grid), dim3(64 * RnsCfg<128>::NW), 0, s, a);
  else if (tq == 256)
    hipLaunchKernelGGL(k_gemm_rns_batched<256>, dim3((unsigned)grid), dim3(64 * RnsCfg<256>::NW), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

int64_t rns_tiles(int64_t d3, int64_t R_out, int tq) {
  return ((d3 + tq - 1) / tq) * ((R_out + kRnsTileR - 1) / kRnsTileR);
}

// resident workgroups per CU: as many as the 160 KiB of LDS hold, at most two waves per SIMD
template <int TQ>
static int wgs_per_cu() {
  using C = RnsCfg<TQ>;
  const int by_lds = 160 * 1024 / C::LDS, by_waves = C::WPE * 4 / C::NW;
  const int w = by_lds < by_waves ? by_lds : by_waves;
  return w > 0 ? w : 1;
}
int rns_wgs_per_cu(int tq) {
  return tq == 32 ? wgs_per_cu<32>() : tq == 64 ? wgs_per_cu<64>() : tq == 128 ? wgs_per_cu<128>() : wgs_per_cu<256>();
}

// Query tile of the RNS contraction of d3 columns: 32 or 64 if that holds them all (16 columns, 30,720 rows, K = 20,992
// in four primes 4.56 ms, 6.2 TB/s, against 4.93 in the 128-column tile, whose products for padding cost power that
// the loads need; 32 columns, 644 rows 25 us against 37; 48 columns, 4,878 rows 96 against 106); else of 128 and 256
// the width whose padded work, weighted by its measured time per column, is smaller (ties: 256).
int rns_tile_q(int64_t d3) {
  if (d3 <= 64) return d3 <= 32 ? 32 : 64;
  return (d3 + 127) / 128 * 128 * 1.09 < (d3 + 255) / 256 * 256 ? 128 : 256;
}

hipError_t launch_gemm_rns(const RnsGemmArgs& g, int tq, hipStream_t s) {
  if (g.R_out <= 0 || g.d3 <= 0) return hipSuccess;
  if ((tq != 32 && tq != 64 && tq != 128 && tq != 256) || g.d3_pad % tq != 0) return hipErrorInvalidValue;
  const int64_t n_ct = (g.d3 + tq - 1) / tq, n_rt = (g.R_out + kRnsTileR - 1) / kRnsTileR;
  if (g.splits < 1 || g.splits > g.KB) return hipErrorInvalidValue;
  const dim3 grid = xcd_grid(n_rt * g.n_mod * g.splits * g.nz, n_ct);
  auto kern = tq == 32 ? k_gemm_rns<32> : tq == 64 ? k_gemm_rns<64> : tq == 128 ? k_gemm_rns<128> : k_gemm_rns<256>;
  hipLaunchKernelGGL(kern, grid, dim3(tq == 256 ? 64 * RnsCfg<256>::NW : 64 * RnsCfg<128>::NW), 0, s, g);
  return hipGetLastError();
}

// ------------------------------------------------------------------ CRT back to the prime
// Entry e of prime slot z: residues s_j = S mod m_j.  With y_j = s_j (M/m_j)^-1 mod m_j,
// S = sum_j y_j (M/m_j) - a M with a = round(sum_j y_j / m_j), since sum_j y_j (M/m_j) = S
// (mod M) and |S| <= M / 4 (the host chooses M >= 4 max |S|), so the fraction sum_j y_j / m_j
// - floor(...) = (S mod M) / M lies at least 1/4 away from 1/2 and single precision (error
// below 2^-19 over 16 terms) decides a exactly; then
// C = sum_j y_j ((M/m_j) mod q) - a (M mod q) mod q.
// Thread: 4 consecutive entries of one prime slot (blockIdx.y).
__global__ void __launch_bounds__(256) k_crt_rns(const uint8_t* res, int64_t n, RnsCrtArgs ra, uint64_t* C) {
  const int z = blockIdx.y;
  const int64_t e0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (e0 >= n) return;
  crt_quad(res + (size_t)z * ra.n * n, n, ra, z, C + (size_t)z * n, e0);
}

// CRT and rescale by p in one pass (single calls): per entry the residues of the special prime's
// slot (z = level) give cp, then each query prime's residue is reconstructed and rescaled,
// out[i][e] = (C_i - [cp] mod q_i) p^-1 mod q_i, so the contraction output C is never written.
// Thread: 4 consecutive entries (n a multiple of 4) or, otherwise, one entry.
__global__ void __launch_bounds__(256) k_crt_rescale_rns(const uint8_t* res, int64_t n, RnsCrtArgs ra,
                                                         RescaleArgs rs, uint64_t* out) {
  const int level = rs.level;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if ((n & 3) == 0) {
    const int64_t e0 = 4 * t;
    if (e0 >= n) return;
    uint64_t v[4];
    int64_t cp[4];
    crt_quad_vals(res + (size_t)level * ra.n * n, n, ra, level, e0, v);
#pragma unroll
    for (int b = 0; b < 4; ++b) cp[b] = centered(v[b], rs.p);
    for (int i = 0; i < level; ++i) {
      crt_quad_vals(res + (size_t)i * ra.n * n, n, ra, i, e0, v);
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = rescale_value(v[b], cp[b], rs, i);
      reinterpret_cast<ulonglong2*>(out + (size_t)i * n + e0)[0] = make_ulonglong2(v[0], v[1]);
      reinterpret_cast<ulonglong2*>(out + (size_t)i * n + e0)[1] = make_ulonglong2(v[2], v[3]);
    }
  } else {
    const int64_t e = t;
    if (e >= n) return;
    const int64_t cp = centered(crt_entry(res + (size_t)level * ra.n * n + e, n, ra, level), rs.p);
    for (int i = 0; i < level; ++i)
      out[(size_t)i * n + e] = rescale_value(crt_entry(res + (size_t)i * ra.n * n + e, n, ra, i), cp, rs, i);
  }
}

hipError_t launch_crt_rescale_rns(const uint8_t* res, int64_t n, const RnsCrtArgs& ra, const RescaleArgs& rs,
                                  uint64_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t per = (n & 3) == 0 ? 4 : 1;
  const int64_t blocks = (n / per + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_crt_rescale_rns, dim3((unsigned)blocks), dim3(256), 0, s, res, n, ra, rs, out);
  return hipGetLastError();
}

hipError_t launch_crt_rns(const uint8_t* res, int nz, int64_t n, const RnsCrtArgs& ra, uint64_t* C,
                          hipStream_t s) {
  if (nz <= 0 || n <= 0) return hipSuccess;
  const int64_t blocks = (n + 4 * 256 - 1) / (4 * 256);
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_crt_rns, dim3((unsigned)blocks, (unsigned)nz), dim3(256), 0, s, res, n, ra, C);
  return hipGetLastError();
}

}  // namespace hfe
