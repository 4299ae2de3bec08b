// bf16 MFMA GEMM core for gfx950:  C[M][N] = sum_k A[row(m)][k] * B[n][k]   (both operands K-contiguous).
//
// It serves both contractions of Eq. 5:
//   dX_q = dY . W_q        A = dY [T][C_out],               B = W_q^T [C_in][C_out]
//   dW_q[id] = dY[:,id]^T X_q   A = rows id of dY^T [C_out][T] (gather fused into the A-tile loads),
//                               B = (codes - Z_x)^T [C_in][T]
// 256 threads = 4 wavefronts in a 2x2 grid, v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  Operand tiles
// go global -> LDS directly (global_load_lds_dwordx4, 128-byte row segments = whole cache lines per request)
// into two LDS stages of K = 64 with an XOR swizzle that makes the ds_read_b128 fragment reads conflict free;
// fragments are double-buffered in registers and the loads of the stage after next are spread over three of the
// four MFMA sub-steps.  Split-K writes raw fp32 partial tiles (deterministic second-pass reduction).
#pragma once
#include "common.hpp"

#include <type_traits>

#include "gemm_epilogue.hpp"
#include "lds_copy.hpp"

namespace efqat {

typedef int intx4_t __attribute__((ext_vector_type(4)));
typedef int intx16_t __attribute__((ext_vector_type(16)));

#ifndef EFQAT_GEMM_GM
#define EFQAT_GEMM_GM 8   // row tiles per group of the block -> tile walk
#endif
constexpr int KALIGN = 64;  // split-K slices start on multiples of this many K elements



// BM x BN output tile per 256-thread block; one LDS stage holds 128 bytes of K per tile row (64 bf16 or 128 int8),
// S stages.
template <int BM_, int BN_, int S>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_;
  static constexpr int BKT = 64;                        // K in units of 2 bytes
  static constexpr int WM = BM / 2, WN = BN / 2;        // per-wave tile (2 x 2 wavefronts)
  static constexpr int TM = WM / 32, TN = WN / 32;      // MFMA tiles per wave
  static constexpr int PITCH_B = BKT * 2;               // bytes per tile row in LDS
  static constexpr int CPRW = BKT / 8;                  // 16-byte chunks per row
  static constexpr int RPI = 1024 / PITCH_B;            // rows covered by one 1-KiB wave load
  static constexpr int R256 = 256 / PITCH_B;            // rows per 256 bytes (LDS bank period for b128)
  static constexpr int A_G = BM / RPI / 4, B_G = BN / RPI / 4;  // 1-KiB row groups per wave and stage
  static constexpr int NS = BKT / 16;                   // MFMA sub-steps per stage
  static constexpr int LDS_A = BM * PITCH_B, LDS_B = BN * PITCH_B;
  static constexpr int LDS_STAGE = LDS_A + LDS_B;
  static constexpr int LDS_LOOP = S * LDS_STAGE;
  static constexpr int LDS_EPI = 4 * 32 * (WN + 8) * 4;  // staging of the fused dX epilogue
  template <int EPI>
  static constexpr int lds_bytes() {
    constexpr int e = EPI == EPI_DX ? EpiDxAny<TileCfg, float>::LDS : LDS_EPI;
    return LDS_LOOP > e ? LDS_LOOP : e;
  }
  // XOR swizzle: 16 consecutive rows read the same logical chunk in one ds_read_b128 quarter-wave; with
  // f(row) = (row / R256) mod CPRW the 16 physical chunks are distinct modulo 256 bytes (64 banks).
  __device__ static __forceinline__ int swz(int row, int chunk) {
    return row * PITCH_B + ((chunk ^ ((row / R256) & (CPRW - 1))) << 4);
  }
};

struct True { static constexpr bool value = true; };
struct False { static constexpr bool value = false; };

// Scheduling hint for one MFMA sub-step: NR groups of (a share of the MF MFMAs, one LDS fragment read), the
// first NL groups followed by one global->LDS load.  The group sizes must be compile-time constants.
template <int MF, int NR, int NL, int Q>
struct SchedPattern {
  static __device__ __forceinline__ void run() {
    if constexpr (Q < NR) {
      __builtin_amdgcn_sched_group_barrier(0x008, ((Q + 1) * MF) / NR - (Q * MF) / NR, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if constexpr (Q < NL) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      SchedPattern<MF, NR, NL, Q + 1>::run();
    }
  }
};

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// EPI: EPI_RAW fp32 partial tiles (split-K), EPI_DX fused dX epilogue, EPI_FWD forward epilogue.
// I8: operands are int8 codes (A unsigned, re-biased by 128 in registers) on v_mfma_i32_32x32x32_i8; else bf16.
// CONV = 1: the A operand is gathered from a token-major dY with the im2col map of a stride-1 convolution (see GemmArgs);
// CONV = 2: of a convolution with a stride, rows sorted by phase (see ConvPhase).
template <int BM, int BN, int EPI, bool I8, int CONV = 0>
__device__ __forceinline__ void gemm_nt_block(const typename ConvArgs<CONV>::type& g, char* smem, int bid, int nblk) {
#if defined(__HIP_DEVICE_COMPILE__)   // the body uses gfx950-only builtins; the host pass needs only the launch stub
  constexpr int S = 2;
  constexpr int ESZ = I8 ? 1 : 2;                       // bytes per K element
  constexpr int BKT = 128 / ESZ;                        // K elements per LDS stage
  static_assert(I8 == (EPI == EPI_FWD), "the int8 product is the forward pass");
  using C = TileCfg<BM, BN, S>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS bases stay scalar
  const int wm = wave >> 1, wn = wave & 1;

  // ---- block -> tile: spread contiguous tile ranges over the 8 XCDs (one L2 each), then walk the
  // range in groups of 8 row-tiles so that concurrently resident blocks share operand panels.
  const int ntile = g.tiles_m * g.tiles_n;
  const int logical = xcd_contiguous_index(bid, nblk);
  const int split = logical / ntile;                   // split-K slice (0 when there is one)
  const int pid = logical - split * ntile;
  const int GM = EFQAT_GEMM_GM;
  const int per_group = GM * g.tiles_n;
  const int group = pid / per_group;
  const int first_m = group * GM;
  const int gsize = (g.tiles_m - first_m) < GM ? (g.tiles_m - first_m) : GM;
  int tm = first_m + (pid % per_group) % gsize;
  int tn = (pid % per_group) / gsize;
  ConvPhase ph;
  if constexpr (CONV == 2) strided_tile(g, bid, &ph, &tm, &tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int lm0 = m0, ln0 = n0;

  const int k_begin = split * g.k_per_split;
  const int k_end = (k_begin + g.k_per_split) < g.K ? (k_begin + g.k_per_split) : g.K;

  // ---- operand staging.  One wave instruction of the direct global->LDS load (global_load_lds_dwordx4)
  // fills 1 KiB of contiguous LDS = RPI tile rows: lane l lands in row RPI*grp + l / CPRW, slot l % CPRW, so
  // it must fetch the logical chunk slot ^ f(row) of that row (f is the same for every group of a wave).
  const int lrow = lane / C::CPRW, slot = lane % C::CPRW;
  const int lch = slot ^ (((wave * C::RPI + lrow) / C::R256) & (C::CPRW - 1));
  const char* a_ptr[C::A_G];
  const char* b_ptr[C::B_G];
  int cv_q0[CONV ? C::A_G : 1], cv_hw[CONV ? C::A_G : 1];   // CONV: n * Ho * Wo and (h << 16 | w) of the slot's pixel
#pragma unroll
  for (int j = 0; j < C::A_G; ++j) {
    int gm = lm0 + (wave + 4 * j) * C::RPI + lrow;
    const int rows = CONV == 2 ? ph.rows : g.M;
    gm = gm < rows ? gm : rows - 1;                     // rows past the edge re-read a valid row
    if constexpr (CONV == 2) {
      strided_pixel(g, ph, gm, &cv_q0[j], &cv_hw[j]);
      a_ptr[j] = nullptr;
    } else if constexpr (CONV) {
      const int hw = g.cv_H * g.cv_W;
      const int n = gm / hw, rem = gm - n * hw;
      const int h = rem / g.cv_W, w = rem - h * g.cv_W;
      cv_q0[j] = n * g.cv_Ho * g.cv_Wo;
      cv_hw[j] = (h << 16) | w;
      a_ptr[j] = nullptr;
    } else {
      const int64_t src = g.a_rows ? (int64_t)g.a_rows[gm] : (int64_t)gm;
      a_ptr[j] = (const char*)g.A + (src * g.lda + k_begin) * ESZ + lch * 16;
    }
  }
  // source of this lane's 16 bytes of A-slot j in stage kt
  auto a_src = [&](int j, int kt) -> const char* {
    if constexpr (CONV == 2) {
      int a, b, cst;
      strided_stage(g, ph, kt, &a, &b, &cst);
      const int ho = (cv_hw[j] >> 16) + ph.dh0 - a, wo = (cv_hw[j] & 0xFFFF) + ph.dw0 - b;
      const bool ok = (unsigned)ho < (unsigned)g.cv_Ho && (unsigned)wo < (unsigned)g.cv_Wo;
      const int64_t pix = (int64_t)cv_q0[j] + ho * g.cv_Wo + wo;
      return ok ? (const char*)g.A + (pix * g.lda + cst * 64) * 2 + lch * 16 : zero_page();
    } else if constexpr (CONV) {
      const int sidx = k_begin / 64 + kt;              // 64-channel stage index along K = (tap, channel)
      const int tap = (int)(((uint64_t)(uint32_t)sidx * g.cv_m_spt) >> 32), cst = sidx - tap * g.cv_spt;
      const int kh = (int)(((uint64_t)(uint32_t)tap * g.cv_m_kw) >> 32), kw = tap - kh * g.cv_KW;
      const int ho = (cv_hw[j] >> 16) + g.cv_pad - kh, wo = (cv_hw[j] & 0xFFFF) + g.cv_pad - kw;
      const bool ok = (unsigned)ho < (unsigned)g.cv_Ho && (unsigned)wo < (unsigned)g.cv_Wo;
      const int64_t pix = (int64_t)cv_q0[j] + ho * g.cv_Wo + wo;
      return ok ? (const char*)g.A + (pix * g.lda + cst * 64) * 2 + lch * 16 : zero_page();
    } else {
      return a_ptr[j] + kt * 128;
    }
  };
#pragma unroll
  for (int j = 0; j < C::B_G; ++j) {
    int gn = ln0 + (wave + 4 * j) * C::RPI + lrow;
    gn = gn < g.N ? gn : g.N - 1;
    b_ptr[j] = (const char*)g.B + ((int64_t)gn * g.ldb + k_begin) * ESZ + lch * 16;
  }
  // byte offset of stage kt in a B row: the stages of a strided convolution's phase skip the other phases' taps
  auto b_off = [&](int kt) -> int64_t {
    if constexpr (CONV == 2) {
      int a, b, cst;
      strided_stage(g, ph, kt, &a, &b, &cst);
      const int tap = (ph.kh0 + g.cv_stride * a) * g.cv_KW + ph.kw0 + g.cv_stride * b;
      return (int64_t)(tap * g.cv_spt + cst) * 128;
    } else {
      return kt * 128;
    }
  };
  const int span = CONV == 2 ? ph.ntap * g.cv_spt * 64 : k_end - k_begin;
  const int nfull = span > 0 ? span / BKT : 0;         // stages that need no predicate
  const int nk = span > 0 ? (span + BKT - 1) / BKT : 0;

  constexpr int LPS = C::A_G + C::B_G;                 // wave-level 1-KiB loads per stage
  auto issue_direct = [&](int kt, int buf) {           // a full, unpredicated stage
    char* sa = smem + buf * C::LDS_STAGE;
    char* sb = sa + C::LDS_A;
#pragma unroll
    for (int j = 0; j < C::A_G; ++j)
      __builtin_amdgcn_global_load_lds(a_src(j, kt), (lds_ptr_t)(sa + (wave + 4 * j) * 1024), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < C::B_G; ++j)
      __builtin_amdgcn_global_load_lds(b_ptr[j] + b_off(kt), (lds_ptr_t)(sb + (wave + 4 * j) * 1024), 16, 0, 0);
  };
  // any stage: a ragged last stage goes through registers.  K is a multiple of 8, so a 16-byte chunk is
  // all in or all out; missing chunks are written as zeros.
  auto issue = [&](int kt, int buf) {
    if (kt < nfull) {
      issue_direct(kt, buf);
    } else {
      char* sa = smem + buf * C::LDS_STAGE;
      char* sb = sa + C::LDS_A;
      const int koff = kt * 128;                          // bytes
      const bool ok = (koff + lch * 16) < span * ESZ;
#pragma unroll
      for (int j = 0; j < C::A_G; ++j) {
        const uint4 v = ok ? *reinterpret_cast<const uint4*>(a_src(j, kt)) : make_uint4(0, 0, 0, 0);
        *reinterpret_cast<uint4*>(sa + (wave + 4 * j) * 1024 + lane * 16) = v;
      }
#pragma unroll
      for (int j = 0; j < C::B_G; ++j) {
        const uint4 v = ok ? *reinterpret_cast<const uint4*>(b_ptr[j] + b_off(kt)) : make_uint4(0, 0, 0, 0);
        *reinterpret_cast<uint4*>(sb + (wave + 4 * j) * 1024 + lane * 16) = v;
      }
    }
  };

  typename std::conditional<I8, intx16_t, floatx16_t>::type acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
  int wsum[C::TN] = {};                                 // I8: this lane's share of sum_k w of its columns

  const int fr = lane & 31, fh = lane >> 5;
  const int a_row0 = wm * C::WM + fr, b_row0 = wn * C::WN + fr;
  intx4_t af[2][C::TM], bfr[2][C::TN];                  // 16-byte fragments: 8 bf16 or 16 int8 along K
  auto load_frags = [&](int buf, int s, int rb) {
    const char* sa = smem + buf * C::LDS_STAGE;
    const char* sb = sa + C::LDS_A;
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
      af[rb][i] = *reinterpret_cast<const intx4_t*>(sa + C::swz(a_row0 + i * 32, 2 * s + fh));
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
      bfr[rb][j] = *reinterpret_cast<const intx4_t*>(sb + C::swz(b_row0 + j * 32, 2 * s + fh));
  };
  auto mfma_all = [&](int rb) {
    if constexpr (I8) {
      // activation codes are unsigned: x - 128 fits int8 (flip the top bit of every byte); the epilogue adds
      // 128 * sum_k w back
#pragma unroll
      for (int i = 0; i < C::TM; ++i) af[rb][i] ^= (int)0x80808080;
      // ... for which the weight rows are summed here, from the fragments, instead of by a pass over W of its own
#pragma unroll
      for (int j = 0; j < C::TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) wsum[j] = __builtin_amdgcn_sdot4(bfr[rb][j][q], 0x01010101, wsum[j], false);
    }
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) {
        if constexpr (I8)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[rb][i], bfr[rb][j], acc[i][j], 0, 0, 0);
        else
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[rb][i]),
                                                              __builtin_bit_cast(bf16x8_t, bfr[rb][j]), acc[i][j],
                                                              0, 0, 0);
      }
  };

  // ---- main loop, two LDS stages.  Stage kt computes from buffer kt & 1 in NS = 4 sub-steps of K = 16:
  //   sub-step s < 3: read the fragments of sub-step s+1 while the MFMAs of sub-step s run; sub-steps 0 and 1
  //     also issue the 2nd and 3rd thirds of the loads of stage kt+1 into the other buffer;
  //   then wait for this wave's LDS reads and global->LDS loads, and barrier: stage kt+1 is complete for
  //     everybody and nobody reads this stage's buffer any more;
  //   sub-step 3: read the first fragments of stage kt+1 and issue the 1st third of the loads of stage kt+2
  //     into this stage's (now free) buffer, under the MFMAs of sub-step 3.
  // Every load thus has at least one full sub-step (16 MFMAs per wave) to land, and the texture addresser never
  // sees more than a third of a stage at once.
  static_assert(S == 2 && C::NS == 4, "two-stage schedule");
  constexpr int MF = C::TM * C::TN, NR = C::TM + C::TN;
  constexpr int P0 = (LPS + 2) / 3, P1 = (LPS - P0 + 1) / 2, P2 = LPS - P0 - P1;   // loads per third
  auto issue_range = [&](int kt, int buf, int t0, int t1) {
    char* sa = smem + buf * C::LDS_STAGE;
    char* sb = sa + C::LDS_A;
#pragma unroll
    for (int t = t0; t < t1; ++t) {
      if (t < C::A_G)
        __builtin_amdgcn_global_load_lds(a_src(t, kt), (lds_ptr_t)(sa + (wave + 4 * t) * 1024), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds(b_ptr[t - C::A_G] + b_off(kt),
                                         (lds_ptr_t)(sb + (wave + 4 * (t - C::A_G)) * 1024), 16, 0, 0);
    }
  };
  auto stage_sync = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // CONV = 2: the matrix row of every tile row, behind the stages in LDS
  int* rowmap = reinterpret_cast<int*>(smem + C::template lds_bytes<EPI>());
  if constexpr (CONV == 2) {
    if (tid < BM) {
      int q0, hw;
      rowmap[tid] = m0 + tid < ph.rows ? strided_pixel(g, ph, m0 + tid, &q0, &hw) : -1;
    }
  }

  if (nk > 0) issue(0, 0);
  wait_vmcnt<0>();
  __syncthreads();
  if (1 < nfull) issue_range(1, 1, 0, P0);
  if (nk > 0) load_frags(0, 0, 0);
  int kt = 0;
  // steady state: stages kt+1 and kt+2 are full stages -> branch-free body, one scheduling region per sub-step
  for (; kt + 2 < nfull; ++kt) {
    const int cur = kt & 1;
    __builtin_amdgcn_sched_barrier(0);
    load_frags(cur, 1, 1);
    issue_range(kt + 1, cur ^ 1, P0, P0 + P1);
    mfma_all(0);
    SchedPattern<MF, NR, P1, 0>::run();
    __builtin_amdgcn_sched_barrier(0);
    load_frags(cur, 2, 0);
    issue_range(kt + 1, cur ^ 1, P0 + P1, LPS);
    mfma_all(1);
    SchedPattern<MF, NR, P2, 0>::run();
    __builtin_amdgcn_sched_barrier(0);
    load_frags(cur, 3, 1);
    mfma_all(0);
    SchedPattern<MF, NR, 0, 0>::run();
    stage_sync();
    load_frags(cur ^ 1, 0, 0);
    issue_range(kt + 2, cur, 0, P0);
    mfma_all(1);
    SchedPattern<MF, NR, P0, 0>::run();
    __builtin_amdgcn_sched_barrier(0);
  }
  // drain: the last stages, including a ragged one
  for (; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nfull) issue_range(kt + 1, cur ^ 1, P0, LPS);   // its first third is already in flight
    else if (kt + 1 < nk) issue(kt + 1, cur ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    load_frags(cur, 1, 1);
    mfma_all(0);
    SchedPattern<MF, NR, 0, 0>::run();
    __builtin_amdgcn_sched_barrier(0);
    load_frags(cur, 2, 0);
    mfma_all(1);
    SchedPattern<MF, NR, 0, 0>::run();
    __builtin_amdgcn_sched_barrier(0);
    load_frags(cur, 3, 1);
    mfma_all(0);
    SchedPattern<MF, NR, 0, 0>::run();
    stage_sync();
    if (kt + 1 < nk) load_frags(cur ^ 1, 0, 0);
    mfma_all(1);
  }
  __syncthreads();

  // ---- epilogue.  MFMA 32x32 accumulator layout: lane holds column (lane & 31) and rows
  // 8*(r/4) + 4*(lane >> 5) + (r % 4), r = 0..15.
  if constexpr (EPI == EPI_RAW) {
    float* out = g.out + (int64_t)split * g.M * g.N;
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) {
        const int col = n0 + wn * C::WN + j * 32 + fr;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + wm * C::WM + i * 32 + 8 * (r >> 2) + 4 * fh + (r & 3);
          if (row < g.M && col < g.N) out[(int64_t)row * g.N + col] = acc[i][j][r];
        }
      }
  } else if constexpr (EPI == EPI_DX) {
    epilogue_dx<C, CONV == 2>(g, acc, smem, m0, n0, wm, wn, CONV == 2 ? ph.rows : g.M, bid, rowmap);
  } else if constexpr (EPI == EPI_DXF) {
    epilogue_dx_fast<C>(g, acc, smem, m0, n0, wm, wn, bid);
  } else {
    // Forward epilogue: the int32 sums are over (code - 128) * w, so
    //   y[m][n] = S_x * S_w[n] * (acc + (128 - round(Z_x)) * sum_k w[n][k]).
    // A lane's accumulators belong to TN columns, whose weight sums and scales it holds itself; the products then go
    // through the wavefront's own LDS slab, 32 rows at a time, so that a lane stores 8 consecutive columns of a row.
    constexpr int PITCH = C::WN + 8;
    constexpr int CPR = C::WN / 8;
    constexpr int RPP = 64 / CPR;
    constexpr int NPASS = (32 + RPP - 1) / RPP;
    float* stage = reinterpret_cast<float*>(smem) + wave * 32 * PITCH;
    const float sx = g.s_x[0];
    const long long zr = (long long)rintf(g.z_x[0]);
    // |sum_k (code - Z) w| <= 128 K max(|Z|, |255 - Z|): below 2^31 the result needs 32 bits only, and arithmetic modulo
    // 2^32 forms it whatever the terms were.  A zero point far outside the codes' range takes the 64-bit sum.
    const bool narrow = 128.0 * (double)g.K * (double)(zr >= 128 ? zr : 255 - zr) < 2147483648.0;
    float scl[C::TN];
    long long corr[C::TN];
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
      const int col = n0 + wn * C::WN + j * 32 + fr;
      scl[j] = col < g.N ? sx * g.s_w[col] : 0.0f;
      corr[j] = (128 - zr) * (long long)(wsum[j] + __shfl_xor(wsum[j], 32, kWave));
    }
    const int row_l0 = lane / CPR, ch = lane % CPR;
    const int gcol = n0 + wn * C::WN + ch * 8;
    const bool lane_on = row_l0 < RPP && gcol < g.N;
    auto wave_fence = []() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
      wave_fence();
      if (narrow) {
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            stage[(8 * (r >> 2) + 4 * fh + (r & 3)) * PITCH + j * 32 + fr] =
                scl[j] * (float)(int)((uint32_t)acc[i][j][r] + (uint32_t)corr[j]);
      } else {
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            stage[(8 * (r >> 2) + 4 * fh + (r & 3)) * PITCH + j * 32 + fr] = scl[j] * (float)((long long)acc[i][j][r] + corr[j]);
      }
      wave_fence();
#pragma unroll
      for (int p = 0; p < NPASS; ++p) {
        const int row_l = p * RPP + row_l0;
        const int grow = m0 + wm * C::WM + i * 32 + row_l;
        if (lane_on && row_l < 32 && grow < g.M) {
          const float4 o0 = *reinterpret_cast<const float4*>(stage + row_l * PITCH + ch * 8);
          const float4 o1 = *reinterpret_cast<const float4*>(stage + row_l * PITCH + ch * 8 + 4);
          const int64_t e = (int64_t)grow * g.N + gcol;
          if (g.epi_vec && gcol + 8 <= g.N) {
            if (g.y_dtype == EFQAT_F32) {
              *reinterpret_cast<float4*>((float*)g.y + e) = o0;
              *reinterpret_cast<float4*>((float*)g.y + e + 4) = o1;
            } else {
              *reinterpret_cast<uint4*>((bf16_t*)g.y + e) = make_uint4(pack_bf16x2(o0.x, o0.y), pack_bf16x2(o0.z, o0.w),
                                                                       pack_bf16x2(o1.x, o1.y), pack_bf16x2(o1.z, o1.w));
            }
          } else {
            const float o[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
#pragma unroll
            for (int t = 0; t < 8; ++t)
              if (gcol + t < g.N) {
                if (g.y_dtype == EFQAT_F32) ((float*)g.y)[e + t] = o[t];
                else ((bf16_t*)g.y)[e + t] = f32_to_bf16(o[t]);
              }
          }
        }
      }
    }
  }
#endif
}

// two blocks of up to 128 x 128, or four of 64 x 64, share a CU (by LDS): the epilogue must leave them the registers
template <int BM, int BN, int EPI, bool I8, int CONV = 0>
__global__ __launch_bounds__(256, BM * BN <= 64 * 64 ? 4 : BM * BN <= 128 * 128 ? 2 : 1) void k_gemm_nt(
    const typename ConvArgs<CONV>::type g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_nt_block<BM, BN, EPI, I8, CONV>(g, smem, blockIdx.x, gridDim.x);
}

}  // namespace efqat
