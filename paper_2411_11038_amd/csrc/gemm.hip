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
#include "common.hpp"

#include <algorithm>
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
// two blocks of up to 128 x 128, or four of 64 x 64, share a CU (by LDS): the epilogue must leave them the registers
template <int BM, int BN, int EPI, bool I8, int CONV = 0>
__global__ __launch_bounds__(256, BM * BN <= 64 * 64 ? 4 : BM * BN <= 128 * 128 ? 2 : 1) void k_gemm_nt(const typename ConvArgs<CONV>::type g) {
#if defined(__HIP_DEVICE_COMPILE__)   // the body uses gfx950-only builtins; the host pass needs only the launch stub
  constexpr int S = 2;
  constexpr int ESZ = I8 ? 1 : 2;                       // bytes per K element
  constexpr int BKT = 128 / ESZ;                        // K elements per LDS stage
  static_assert(I8 == (EPI == EPI_FWD), "the int8 product is the forward pass");
  using C = TileCfg<BM, BN, S>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS bases stay scalar
  const int wm = wave >> 1, wn = wave & 1;

  // ---- block -> tile: spread contiguous tile ranges over the 8 XCDs (one L2 each), then walk the
  // range in groups of 8 row-tiles so that concurrently resident blocks share operand panels.
  const int ntile = gridDim.x;
  const int logical = xcd_contiguous_index(blockIdx.y * ntile + blockIdx.x, ntile * gridDim.y);
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
  if constexpr (CONV == 2) strided_tile(g, blockIdx.x, &ph, &tm, &tn);
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
    epilogue_dx<C, CONV == 2>(g, acc, smem, m0, n0, wm, wn, CONV == 2 ? ph.rows : g.M, rowmap);
  } else if constexpr (EPI == EPI_DXF) {
    epilogue_dx_fast<C>(g, acc, smem, m0, n0, wm, wn);
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

// ---------------------------------------------------------------------------------------------- host
// Tile / split-K choice: a small cost model in CU clock cycles, evaluated on the host and calibrated on
// measured runs of this kernel (rates in flop per clock per block):
//   - a T x T block runs its K loop at `rate`: 256 -> 2500, 192 -> 2100, 128 -> 1000 with two blocks resident
//     per CU.  The big tiles are bounded by what one CU's vector L1 pulls from L2 (about 19 B/clk) times their
//     flop per byte, the small one additionally by its doubled L2 traffic;
//   - per block: launch/prologue 4000 cycles plus the epilogue, 0.75 cycles per output element for the fused
//     dX epilogue (it streams x, codes, mask and dX through HBM), 0.6 when a second resident block overlaps it,
//     0.3 for the raw fp32 store;
//   - blocks run in rounds of 256 CUs x blocks-per-CU;  split-K adds its fp32 partial tiles, written and read once.
struct TileModel { int t; int bpc; double rate; double epi_dx; };
static const TileModel kTiles[3] = {{256, 1, 2500.0, 0.75}, {192, 1, 2100.0, 0.75}, {128, 2, 1000.0, 0.6}};

GemmPlan gemm_plan(int64_t M, int64_t N, int64_t K, bool allow_split, bool allow_192, bool allow_256) {
  GemmPlan best{};
  double best_t = 1e300;
  const int64_t ksteps = ceil_div(K, KALIGN);
  for (const TileModel& tm : kTiles) {
    if (tm.t == 192 && !allow_192) continue;
    if (tm.t == 256 && !allow_256) continue;
    const int64_t tiles = ceil_div(M, tm.t) * ceil_div(N, tm.t);
    int64_t max_s = allow_split ? ksteps / 8 : 1;
    if (max_s < 1) max_s = 1;
    if (max_s > 32) max_s = 32;
    for (int64_t s = 1; s <= max_s; ++s) {
      const int64_t kslice = ceil_div(ksteps, s) * KALIGN;
      const double per_elem = allow_split ? 0.3 : tm.epi_dx;
      const double block = 2.0 * tm.t * tm.t * (double)kslice / tm.rate + 4000.0 + per_elem * tm.t * tm.t;
      const double rounds = (double)ceil_div(tiles * s, 256 * tm.bpc);
      double t = rounds * block;
      if (allow_split) t += (double)s * (double)M * (double)N * 8.0 / 2400.0;   // partial tiles at ~5 TB/s
      if (t < best_t) {
        best_t = t;
        best.tile = tm.t; best.split_k = (int)s;
        best.tiles_m = (int)ceil_div(M, tm.t); best.tiles_n = (int)ceil_div(N, tm.t);
      }
    }
  }
  return best;
}

// Kernel and tile of a dX product.  Microseconds per K stage of 64 and per block (launch, first loads, epilogue) with one
// block on a CU (lone; of a tile that fits once: on few of the CUs, where clock and memory are its own) and with all `bpc`
// that fit by LDS and registers (full), between the two by the number resident; what
// x and dX in fp32 add and what the straight-line epilogue of whole bf16 tiles saves.  A product is its whole rounds of
// 256 * bpc blocks plus what is left.  Fitted to measured launches of 300 linear layers (each dimension 64 .. 16384) and 28
// convolutions; the choice is 0.9 % from the fastest of the six in the mean, the linear layers 1.33 x and the convolutions
// 1.6 x as fast as with tiles of 128 and more only.  T x C_out -> C_in in us by k_gemm_kk 64 / nt 64 / kk 128 / nt 128 / kk 192 /
// dx8 256, bf16:
//   256 x 256 -> 256         6.6 / 5.8 / 8.4 /  - /  18 / -      few tiles: the smallest, with the shortest epilogue
//   64 x 4096 -> 4096         21 /  33 /  30 /  46 /  51 /  -    ... and the ring, where K is long
//   2048 x 768 -> 3072        28 /  28 /  26 /  26 /  30 /  30   (C_out 320)
//   4224 x 112 -> 6144        46 /  37 /  46 /  34 /  38 /  44   two blocks a CU hide each other's epilogues
//   12288 x 3072 -> 768       89 /  99 /  87 /  85 /  54 /  -    one round of 192 x 192
//   13824 x 2504 -> 768      135 / 132 /  93 /  93 /  95 /  65   long K and whole rounds: 256 x 256 (without int8 operand:
//                                                               k_gemm_nt, priced the same)
// Convolutions pay for the gather in every stage.
struct DxTile { int t; bool ring; int bpc; double lone[2], full[2], f32[2], fast[2]; };
static const DxTile kDxTiles[] = {{64, true, 3, {0.28, 5.6}, {0.73, 4.5}, {0.1, 1.0}, {0.0, 0.0}},
                                  {64, false, 4, {0.465, 4.4}, {0.965, 4.4}, {0.1, 1.6}, {0.0, 0.0}},
                                  {128, true, 1, {0.495, 9.2}, {0.587, 7.9}, {0.0, 1.4}, {-1.7, -1.7}},
                                  {128, false, 2, {0.74, 8.0}, {1.075, 9.7}, {0.7, 3.5}, {-1.7, -2.0}},
                                  {192, true, 1, {0.695, 15.6}, {0.98, 15.6}, {0.0, 4.8}, {-4.2, -4.2}},
                                  {256, false, 1, {0.92, 23.3}, {1.61, 23.3}, {1.9, 12.0}, {-6.7, -6.7}}};
static const DxTile kDxConvTiles[] = {{64, true, 3, {0.30, 6.3}, {0.575, 6.6}, {0.0, 0.0}, {0.0, 0.0}},
                                      {64, false, 4, {0.54, 5.2}, {0.71, 5.4}, {0.0, 0.1}, {0.0, 0.0}},
                                      {128, true, 1, {0.56, 10.0}, {0.56, 10.0}, {0.5, 0.5}, {-1.0, -1.0}},
                                      {128, false, 2, {0.79, 9.4}, {0.94, 11.2}, {0.0, 0.6}, {-1.0, -1.0}},
                                      {192, false, 1, {1.12, 15.6}, {1.12, 15.6}, {0.2, 0.2}, {-1.0, -1.0}}};
static int64_t conv_phases(const ConvDxStridedMap& cm, int tile, ConvPhase* out, int* nphase);

GemmPlan dx_plan(int64_t M, int64_t N, int64_t K, bool f32, bool conv, const ConvDxStridedMap* strided, bool int8_ok) {
  GemmPlan best{};
  double best_t = 0.0;
  auto price = [&](const DxTile& c) {
    if (c.t == 192 && strided) return;
    int64_t tm = ceil_div(M, c.t);
    double stages = (double)ceil_div(K, KALIGN);
    if (strided) {                                     // mean stages of a tile
      ConvPhase ph[kMaxConvStride * kMaxConvStride];
      int n = 0;
      tm = conv_phases(*strided, c.t, ph, &n);
      double sum = 0.0;
      for (int i = 0; i < n; ++i) sum += (double)ph[i].tiles * ph[i].ntap;
      stages *= sum / ((double)tm * strided->KH * strided->KW);
    }
    const int64_t tn = ceil_div(N, c.t), tiles = tm * tn, round = 256 * c.bpc;
    if (tiles >= (1 << 24) && c.t < 128) return;        // a grid dimension holds less than 2^32 work items
    const bool fast = !f32 && !strided && (M % c.t) == 0 && (N % c.t) == 0;
    const double add[2] = {(f32 ? c.f32[0] : 0.0) + (fast ? c.fast[0] : 0.0), (f32 ? c.f32[1] : 0.0) + (fast ? c.fast[1] : 0.0)};
    const double lone = c.lone[0] * stages + c.lone[1] + add[0], full = c.full[0] * stages + c.full[1] + add[1];
    double t = (double)(tiles / round) * full;
    if (const int64_t rest = tiles % round)
      t += lone + (full - lone) * (c.bpc > 1 ? (double)(ceil_div(rest, 256) - 1) / (c.bpc - 1) : (double)rest / 256.0);
    // the others need W_q^T in bf16: the codes read, twice as many bytes written, at 4 TB/s
    if (int8_ok && c.t != 256) t += 3.0 * (double)N * (double)K / 4e6;
    if (best.tile == 0 || t < best_t) { best_t = t; best = GemmPlan{c.t, 1, (int)tm, (int)tn, c.ring}; }
  };
  if (conv) for (const DxTile& c : kDxConvTiles) price(c);
  else for (const DxTile& c : kDxTiles) price(c);
  return best;
}

// Tile and split-K of a dW product.  Costs as in kDxTiles; to them comes the second pass (k_dw_finish), which reads every
// slice: 3.7 us, 0.07 us a slice, and 0.119 us per 2^20 values and 4 bytes.  Slices of two K stages and more, where
// eight stages and fewer, larger tiles were the rule before.  Fitted to 100 layers and convolutions by k_gemm_tn and 55 from
// staged operands, dW product and second pass together: 1.02 x (staged 1.06 x) the fastest of all tiles and splits, 1.21 x
// (convolutions 1.25 x, staged 1.29 x) as fast as before.  T x C_in, k rows, us with the best split on 64 / 128 rows (slices):
//   480 x 512, 172        7.8 (4) / 10.1 (4), before 13.4 (1)     few tiles: as many short slices as fill the chip
//   12144 x 688, 40      13.9 (32) / 15.5 (32), before 16.7 (22)  half of a 128-row tile would be padding
//   6848 x 1776, 1500    63 (3) / 54 (3)                          many tiles: fewer LDS bytes per product
// The 256 x 256 and 192 x 192 tiles stay where gemm_plan prices them lowest: large products.
struct DwTile { int bm, bn, bpc; double lone[2], full[2]; };
static const DwTile kDwTiles[3][2] = {{{64, 128, 4, {0.515, 4.4}, {1.10, 6.2}}, {128, 128, 3, {0.575, 5.8}, {1.305, 8.3}}},
                                      {{64, 128, 4, {0.785, 5.0}, {1.51, 7.6}}, {128, 128, 3, {0.955, 6.6}, {1.68, 11.2}}},
                                      {{64, 64, 4, {0.453, 3.0}, {0.95, 3.5}}, {128, 128, 2, {0.71, 4.5}, {0.88, 7.0}}}};
GemmPlan dw_plan(DwKind kind, int64_t M, int64_t N, int64_t K) {
  GemmPlan best = gemm_plan(M, N, K, true, kind == DW_STAGED, kind != DW_CONV);
  if (best.tile > 128) return best;
  const int64_t stages = ceil_div(K, KALIGN);
  double best_t = 0.0;
  bool have = false;
  for (const DwTile& c : kDwTiles[kind]) {
    const int64_t tm = ceil_div(M, c.bm), tn = ceil_div(N, c.bn), round = 256 * c.bpc;
    if (tm * tn >= (1 << 24)) continue;                 // a grid dimension holds less than 2^32 work items
    for (int64_t s = 1; s <= 64 && (s == 1 || 2 * s <= stages); ++s) {
      const int64_t per = ceil_div(stages, s);
      if (ceil_div(stages, per) != s) continue;         // slices without a stage
      const double lone = c.lone[0] * (double)per + c.lone[1], full = c.full[0] * (double)per + c.full[1];
      double t = (double)(tm * tn * s / round) * full + 3.7 + 0.07 * (double)s + 0.119e-6 * (double)M * (double)N * (double)(4 * s + 9);
      if (const int64_t rest = tm * tn * s % round)
        t += lone + (full - lone) * (double)(ceil_div(rest, 256) - 1) / (double)(c.bpc - 1);
      if (!have || t < best_t) { best_t = t; best = GemmPlan{c.bm, (int)s, (int)tm, (int)tn, false}; have = true; }
    }
  }
  return best;
}

bool gemm_epilogue_vec_ok(const GemmEpilogueDx& e, int64_t N) {
  return (N % 8) == 0 && ((uintptr_t)e.x_codes % 8) == 0 && ((uintptr_t)e.x % 16) == 0 && ((uintptr_t)e.dx % 16) == 0;
}

template <int BM, int BN, int EPI, bool I8, int CONV = 0>
static int launch_cfg(const typename ConvArgs<CONV>::type& a, int split_k, hipStream_t st) {
  using C = TileCfg<BM, BN, 2>;
  constexpr int kLds = C::template lds_bytes<EPI>() + (CONV == 2 ? BM * (int)sizeof(int) : 0);
  // set once per process (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_gemm_nt<BM, BN, EPI, I8, CONV>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  dim3 grid((unsigned)(a.tiles_m * a.tiles_n), (unsigned)split_k);
  constexpr int kProf = (EPI == EPI_DX || EPI == EPI_DXF) ? PROF_DX : (EPI == EPI_RAW ? PROF_DW : PROF_FWD);
  {
    ProfScope prof(kProf, st);
    hipLaunchKernelGGL((k_gemm_nt<BM, BN, EPI, I8, CONV>), grid, dim3(256), kLds, st, a);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

// nothing left to decide in the dX epilogue: bf16 in and out, whole tiles, 32-bit element offsets, aligned pointers
static bool nt_epilogue_fast(const GemmArgs& g, const GemmEpilogueDx& epi, int tile) {
  return g.epi_vec && epi.x_dtype == EFQAT_BF16 && epi.dx_dtype == EFQAT_BF16 && (g.M % tile) == 0 &&
         (g.N % tile) == 0 && (int64_t)g.M * g.N <= (int64_t)INT32_MAX;
}

int launch_gemm_nt(const bf16_t* A, int64_t lda, const int32_t* a_rows, const bf16_t* B, int64_t ldb, int64_t M,
                   int64_t N, int64_t K, const GemmPlan& plan, float* out_partial, const GemmEpilogueDx* epi,
                   hipStream_t stream) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 8) || (lda % 8) || (ldb % 8)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return EFQAT_ERR_BAD_SHAPE;
  const int split_k = plan.split_k;
  if (epi && split_k != 1) return EFQAT_ERR_BAD_SHAPE;
  GemmArgs a{};
  a.A = A; a.lda = lda; a.a_rows = a_rows; a.B = B; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(ceil_div(K, KALIGN), split_k) * KALIGN);
  a.out = out_partial;
  if (epi) {
    a.x_codes = epi->x_codes; a.x_clip = epi->x_clip; a.x = epi->x; a.x_dtype = epi->x_dtype;
    a.s_x = epi->s_x; a.z_x = epi->z_x; a.dx = epi->dx; a.dx_dtype = epi->dx_dtype; a.partial = epi->partial;
    a.epi_vec = gemm_epilogue_vec_ok(*epi, N) ? 1 : 0;
  }
  a.tiles_m = plan.tiles_m;
  a.tiles_n = plan.tiles_n;
  switch (plan.tile) {
    case 256:
      return epi ? launch_cfg<256, 256, EPI_DX, false>(a, 1, stream)
                 : launch_cfg<256, 256, EPI_RAW, false>(a, split_k, stream);
    case 192:
      return epi ? launch_cfg<192, 192, EPI_DX, false>(a, 1, stream)
                 : launch_cfg<192, 192, EPI_RAW, false>(a, split_k, stream);
    case 64:
      return epi ? launch_cfg<64, 64, EPI_DX, false>(a, 1, stream) : launch_cfg<64, 64, EPI_RAW, false>(a, split_k, stream);
    case 128:
      if (epi && nt_epilogue_fast(a, *epi, 128)) return launch_cfg<128, 128, EPI_DXF, false>(a, 1, stream);
      return epi ? launch_cfg<128, 128, EPI_DX, false>(a, 1, stream)
                 : launch_cfg<128, 128, EPI_RAW, false>(a, split_k, stream);
    default:
      return EFQAT_ERR_BAD_SHAPE;
  }
}

int launch_gemm_nt_conv_dx(const bf16_t* dy_tok, int64_t ldc, const bf16_t* wqT, int64_t ldb, int64_t M, int64_t N,
                           int64_t K, const ConvDxMap& cm, const GemmPlan& plan, const GemmEpilogueDx& epi,
                           hipStream_t stream) {
  if (M <= 0 || N <= 0 || K <= 0 || (ldc % 64) || (K % 64) || (ldb % 8) || cm.H > 65535 || cm.W > 65535)
    return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || plan.split_k != 1) return EFQAT_ERR_BAD_SHAPE;
  GemmArgs a{};
  a.A = dy_tok; a.lda = ldc; a.a_rows = nullptr; a.B = wqT; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(K, KALIGN) * KALIGN);
  a.x_codes = epi.x_codes; a.x_clip = epi.x_clip; a.x = epi.x; a.x_dtype = epi.x_dtype;
  a.s_x = epi.s_x; a.z_x = epi.z_x; a.dx = epi.dx; a.dx_dtype = epi.dx_dtype; a.partial = epi.partial;
  a.epi_vec = gemm_epilogue_vec_ok(epi, N) ? 1 : 0;
  a.tiles_m = plan.tiles_m; a.tiles_n = plan.tiles_n;
  a.cv_H = cm.H; a.cv_W = cm.W; a.cv_Ho = cm.Ho; a.cv_Wo = cm.Wo; a.cv_KW = cm.KW; a.cv_pad = cm.pad;
  a.cv_spt = (int)(ldc / 64);
  a.cv_m_spt = (1ull << 32) / (uint64_t)a.cv_spt + 1; a.cv_m_kw = (1ull << 32) / (uint64_t)cm.KW + 1;
  switch (plan.tile) {
    case 192: return nt_epilogue_fast(a, epi, 192) ? launch_cfg<192, 192, EPI_DXF, false, 1>(a, 1, stream)
                                                   : launch_cfg<192, 192, EPI_DX, false, 1>(a, 1, stream);
    case 64:
      if (plan.ring) return launch_gemm_kk_conv(a, 64, false, stream);
      return launch_cfg<64, 64, EPI_DX, false, 1>(a, 1, stream);
    case 128:
      if (plan.ring) return launch_gemm_kk_conv(a, 128, nt_epilogue_fast(a, epi, 128), stream);
      return nt_epilogue_fast(a, epi, 128) ? launch_cfg<128, 128, EPI_DXF, false, 1>(a, 1, stream)
                                           : launch_cfg<128, 128, EPI_DX, false, 1>(a, 1, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}

// Phases of a convolution with stride s <= kMaxConvStride, most taps first; returns the row tiles in all.
static int64_t conv_phases(const ConvDxStridedMap& cm, int tile, ConvPhase* out, int* nphase) {
  ConvPhase p[kMaxConvStride * kMaxConvStride];
  int n = 0;
  const int s = cm.stride;
  // taps kh with (ph + pad - kh) % s == 0: kh0 = (ph + pad) % s, kh0 + s, ...; the first reaches output row hi + dh0
  auto taps = [s](int K, int first) { return first < K ? (K - first + s - 1) / s : 0; };
  for (int ph = 0; ph < s; ++ph)
    for (int pw = 0; pw < s; ++pw) {
      ConvPhase c{};
      c.ph = ph; c.pw = pw;
      c.Hp = cm.H > ph ? (cm.H - ph + s - 1) / s : 0;
      c.Wp = cm.W > pw ? (cm.W - pw + s - 1) / s : 0;
      c.rows = cm.N * c.Hp * c.Wp;
      c.kh0 = (ph + cm.pad) % s; c.kw0 = (pw + cm.pad) % s;
      c.dh0 = (ph + cm.pad) / s; c.dw0 = (pw + cm.pad) / s;
      const int nkh = taps(cm.KH, c.kh0);
      c.nkw = taps(cm.KW, c.kw0);
      c.ntap = nkh * c.nkw;
      if (c.nkw == 0) c.nkw = 1;                        // never divided by
      c.tiles = (int)ceil_div(c.rows, tile);
      if (c.rows > 0) p[n++] = c;
    }
  int64_t total = 0;
  for (int i = 0; i < n; ++i) {                         // selection by taps, stable
    int best = -1;
    for (int j = 0; j < n; ++j)
      if (p[j].tiles >= 0 && (best < 0 || p[j].ntap > p[best].ntap)) best = j;
    ConvPhase c = p[best];
    p[best].tiles = -1;
    c.tile0 = (int)total;
    total += c.tiles;
    if (out) out[i] = c;
  }
  if (nphase) *nphase = n;
  return total;
}

int64_t conv_dx_strided_row_tiles(const ConvDxStridedMap& cm, int tile) { return conv_phases(cm, tile, nullptr, nullptr); }

int launch_gemm_conv_dx_strided(const bf16_t* dy_tok, int64_t ldc, const bf16_t* wqT, int64_t ldb, int64_t M, int64_t N,
                                const ConvDxStridedMap& cm, const GemmPlan& plan, const GemmEpilogueDx& epi,
                                hipStream_t stream) {
  if (M <= 0 || N <= 0 || (ldc % 64) || (ldb % 8) || cm.H > 65535 || cm.W > 65535 || cm.stride < 2 ||
      cm.stride > kMaxConvStride || (plan.tile != 128 && plan.tile != 64) || plan.split_k != 1 || M > INT32_MAX || N > INT32_MAX)
    return EFQAT_ERR_BAD_SHAPE;
  GemmStridedArgs a{};
  a.A = dy_tok; a.lda = ldc; a.B = wqT; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N;
  a.x_codes = epi.x_codes; a.x_clip = epi.x_clip; a.x = epi.x; a.x_dtype = epi.x_dtype;
  a.s_x = epi.s_x; a.z_x = epi.z_x; a.dx = epi.dx; a.dx_dtype = epi.dx_dtype; a.partial = epi.partial;
  a.epi_vec = gemm_epilogue_vec_ok(epi, N) ? 1 : 0;
  a.cv_H = cm.H; a.cv_W = cm.W; a.cv_Ho = cm.Ho; a.cv_Wo = cm.Wo; a.cv_KW = cm.KW; a.cv_pad = cm.pad;
  a.cv_stride = cm.stride;
  a.cv_spt = (int)(ldc / 64);
  a.cv_m_spt = (1ull << 32) / (uint64_t)a.cv_spt + 1;
  a.tiles_n = plan.tiles_n;
  a.tiles_m = (int)conv_phases(cm, plan.tile, a.phase, &a.nphase);
  if (a.tiles_m != plan.tiles_m) return EFQAT_ERR_BAD_SHAPE;
  if (plan.ring) return launch_gemm_kk_conv_strided(a, plan.tile, stream);
  if (plan.tile == 64) return launch_cfg<64, 64, EPI_DX, false, 2>(a, 1, stream);
  return launch_cfg<128, 128, EPI_DX, false, 2>(a, 1, stream);
}

// Tile of the int8 forward product.  `lone` / `full`: microseconds per K stage of 128 codes and per block (launch, first
// loads, epilogue) with one block on a CU and with all `bpc` that fit (LDS); between the two by the number resident.  A
// product is its whole rounds of 256 * bpc blocks plus what is left.  Fitted to measured launches; against the tile that
// is fastest by measurement at 12 sizes of 128 .. 16384 tokens the choice loses 5 % at most.  T x C_in -> C_out, us with
// tiles of 256x256 / 192x128 / 128x128 / 64x64:
//   8192 x 4096 -> 4096    136 / 146 / 151 / 229    whole rounds of large tiles: fewest LDS bytes per operation
//   2048 x 4096 -> 11008   138 / 105 / 120 / 161    two 192x128 blocks fill the 160 KB of LDS and overlap their epilogues
//   12288 x 768 -> 3072     67 /  43 /  50 /  66
//   2048 x 4096 -> 4096    few tiles: 128x128 is one round of two blocks a CU
//   512 x 4096 -> 4096      57 /  31 /  26 /  21    less than one tile per CU: latency, the smallest tile
struct FwdTile { int bm, bn, bpc; double lone[2], full[2]; };
static const FwdTile kFwdTiles[] = {{256, 256, 1, {1.75, 13.5}, {1.75, 13.5}},
                                    {192, 128, 2, {0.77, 5.9}, {1.30, 7.0}},
                                    {128, 128, 2, {0.67, 4.3}, {1.06, 5.0}},
                                    {64, 64, 5, {0.53, 2.4}, {1.00, 3.0}}};
static FwdTile fwd_tile(int64_t M, int64_t N, int64_t K) {
  const double stages = (double)ceil_div(K, 128);
  const FwdTile* best = nullptr;
  double best_t = 0.0;
  for (const FwdTile& c : kFwdTiles) {
    const int64_t tiles = ceil_div(M, c.bm) * ceil_div(N, c.bn), round = 256 * c.bpc;
    if (tiles >= (1 << 24) && c.bm < 256) continue;     // a grid dimension holds less than 2^32 work items
    const double lone = c.lone[0] * stages + c.lone[1], full = c.full[0] * stages + c.full[1];
    double t = (double)(tiles / round) * full;
    if (const int64_t rest = tiles % round) {
      const int64_t resident = ceil_div(rest, 256);
      t += lone + (full - lone) * (double)(resident - 1) / (double)std::max(1, c.bpc - 1);
    }
    if (!best || t < best_t) { best = &c; best_t = t; }
  }
  return *best;
}

int launch_gemm_fwd_i8(const uint8_t* x_codes, int64_t lda, const int8_t* w_codes, int64_t ldb, int64_t M, int64_t N,
                       int64_t K, const float* s_x, const float* z_x, const float* s_w, void* y, int y_dtype,
                       hipStream_t stream) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 16) || (lda % 16) || (ldb % 16)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return EFQAT_ERR_BAD_SHAPE;
  GemmArgs a{};
  a.A = x_codes; a.lda = lda; a.a_rows = nullptr; a.B = w_codes; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(K, 2 * KALIGN) * 2 * KALIGN);
  a.s_x = s_x; a.z_x = z_x; a.s_w = s_w; a.y = y; a.y_dtype = y_dtype;
  a.epi_vec = ((N % 8) == 0 && ((uintptr_t)y % 16) == 0) ? 1 : 0;
  const FwdTile t = fwd_tile(M, N, K);
  a.tiles_m = (int)ceil_div(M, t.bm);
  a.tiles_n = (int)ceil_div(N, t.bn);
  switch (t.bm) {
    case 256: return launch_cfg<256, 256, EPI_FWD, true>(a, 1, stream);
    case 192: return launch_cfg<192, 128, EPI_FWD, true>(a, 1, stream);
    case 128: return launch_cfg<128, 128, EPI_FWD, true>(a, 1, stream);
    default: return launch_cfg<64, 64, EPI_FWD, true>(a, 1, stream);
  }
}

}  // namespace efqat
