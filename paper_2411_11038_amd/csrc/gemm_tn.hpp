// Weight-gradient product straight from token-major operands (Eq. 5 right, restricted as in Alg. 1):
//
//   C[m][n] = sum_t A[t][m] * (B[t][n] - z),   A = selected columns of dY, bf16 [T][lda];  B = activation codes, u8 [T][ldb]
//
// Both operands have the contraction index t as their row index, i.e. they are "transposed" for the matrix
// cores, which want K contiguous per lane.  Instead of transposing them through HBM, tiles are copied as they
// are (global -> LDS, global_load_lds_dwordx4) and the MFMA fragments are read with the gfx950 LDS transpose
// loads: ds_read_b64_tr_b16 for A (4 consecutive t of one m per lane), ds_read_b64_tr_b8 for B (8 consecutive
// t of one n), whose bytes are turned into bf16 (code - z, exact) in registers.  The activation operand thus
// costs one byte per element in HBM, L2 and LDS.
//
// 256 threads = 1 x 4 wavefronts, v_mfma_f32_32x32x16_bf16, K-stage of 64 tokens, two LDS stages, the same
// software pipeline as the K-contiguous kernel.  Rows beyond K / columns beyond the operand widths are read
// from a zero page, so no load needs a predicate.  Output: raw fp32 partial tiles (split-K).
#pragma once
#include "common.hpp"

#include <type_traits>

#include "gemm_epilogue.hpp"
#include "lds_copy.hpp"

namespace efqat {

template <int BM_, int BN_>
struct TnCfg {
  static constexpr int BM = BM_, BN = BN_;
  // wavefront grid 1 x 4: every wavefront spans all rows of the tile, so each uint8 fragment of B is converted to
  // bf16 by exactly one wavefront
  static constexpr int WGM = 1, WGN = 4;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int RA = 2 * BM, RB = BN;                 // bytes per LDS row (one token)
  static constexpr int CA = RA / 16, CB = RB / 16;           // 16-byte chunks per row
  static constexpr int A_G = 64 * RA / 1024 / 4, B_G = 64 * RB / 1024 / 4;   // 1-KiB loads per wave and stage
  static constexpr int LDS_A = 64 * RA, LDS_B = 64 * RB;
  static constexpr int LDS_STAGE = LDS_A + LDS_B;
  static constexpr int LDS_BYTES = 2 * LDS_STAGE;
  static constexpr int KSH = RB == 256 ? 0 : 1;              // B swizzle: rows per 256 bytes = 1 << KSH
  // physical 16-byte chunk of logical chunk c in token row k.  A: a 16-lane transpose read touches 4 rows x 32
  // bytes, B: 8 rows x 16 bytes; these XORs spread each half-wave's 256 bytes over all 64 banks (A rows of 128 bytes: two
  // rows lie beside each other in the banks already).
  __device__ static __forceinline__ int swz_a_row(int k) { return BM == 64 ? (k >> 1) & 1 : k & 3; }
  __device__ static __forceinline__ int swz_a(int c, int k) { return c ^ (4 * swz_a_row(k)); }
  __device__ static __forceinline__ int swz_b(int c, int k) { return c ^ (2 * ((k >> KSH) & (CB / 2 - 1))); }
};

template <int BM, int BN, bool CONV = false>
__device__ __forceinline__ void gemm_tn_block(const GemmTnArgs& g, char* smem, int bid, int nblk) {
#if defined(__HIP_DEVICE_COMPILE__)
  using C = TnCfg<BM, BN>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave;

  // (tile, split-K slice) of this block: slice-major logical order, one contiguous range per XCD
  const int ntile = g.tiles_m * g.tiles_n;
  const int logical = xcd_contiguous_index(bid, nblk);
  const int split = logical / ntile;
  const int pid = logical - split * ntile;
  const int GM = g.group_m;
  const int per_group = GM * g.tiles_n;
  const int group = pid / per_group;
  const int first_m = group * GM;
  const int gsize = (g.tiles_m - first_m) < GM ? (g.tiles_m - first_m) : GM;
  const int tm = first_m + (pid % per_group) % gsize;
  const int tn = (pid % per_group) / gsize;
  const int m0 = tm * C::BM, n0 = tn * C::BN;

  const int k_begin = split * g.k_per_split;
  const int k_end = (k_begin + g.k_per_split) < g.K ? (k_begin + g.k_per_split) : g.K;
  const int span = k_end - k_begin;
  const int nk = span > 0 ? (span + 63) / 64 : 0;

  const int nfull = span > 0 ? span / 64 : 0;          // stages whose 64 token rows all exist

  // ---- global -> LDS copies.  Load slot j of this wave covers the token rows (wave + 4 j) * RPI .. + RPI - 1 of
  // a stage; lane l lands in row l / chunks-per-row, physical chunk l % chunks-per-row, and therefore fetches the
  // logical chunk that the swizzle maps there.  Every slot keeps a running source pointer that moves on by one
  // stage (64 token rows) after each use; slots whose columns lie outside the operand sit on the zero page with
  // stride 0, so the steady-state loads need no predicate and no multiply.
  constexpr int RPIA = 1024 / C::RA, RPIB = 1024 / C::RB;
  const char* zero = zero_page();
  const int a_r0 = lane / C::CA, b_r0 = lane / C::CB;
  const char* a_ptr[C::A_G];
  const char* b_ptr[C::B_G];
  uint32_t a_st[C::A_G], b_st[C::B_G];
#pragma unroll
  for (int j = 0; j < C::A_G; ++j) {
    const int kr = (wave + 4 * j) * RPIA + a_r0;
    const int col = m0 + C::swz_a(lane % C::CA, kr) * 8;
    const bool on = col < g.a_cols;
    a_ptr[j] = on ? (const char*)g.A + ((int64_t)(k_begin + kr) * g.lda + col) * 2 : zero;
    a_st[j] = on ? (uint32_t)(g.lda * 128) : 0u;
  }
#pragma unroll
  for (int j = 0; j < C::B_G; ++j) {
    const int kr = (wave + 4 * j) * RPIB + b_r0;
    const int col = n0 + C::swz_b(lane % C::CB, kr) * 16;
    const bool on = col < g.b_cols;
    b_ptr[j] = on ? (const char*)g.B + (int64_t)(k_begin + kr) * g.ldb + col : zero;
    b_st[j] = on ? (uint32_t)(g.ldb * 64) : 0u;
  }
  constexpr int LPS = C::A_G + C::B_G;
  // CONV: output-pixel coordinates of every slot's token row (slots 0 .. A_G-1: A, then B), advanced by 64 tokens
  // after each use; the block's tap; per-lane byte offset of the B column inside a pixel
  int cv_n[CONV ? LPS : 1], cv_ho[CONV ? LPS : 1], cv_wo[CONV ? LPS : 1];
  int cv_kh = 0, cv_kw = 0;
  int64_t cv_bcol[CONV ? C::B_G : 1];
  if constexpr (CONV) {
    const int tap = n0 / g.cv_cin;
    cv_kh = tap / g.cv_KW; cv_kw = tap - cv_kh * g.cv_KW;
    const int hw = g.cv_Ho * g.cv_Wo;
#pragma unroll
    for (int t = 0; t < LPS; ++t) {
      const int kr = t < C::A_G ? (wave + 4 * t) * RPIA + a_r0 : (wave + 4 * (t - C::A_G)) * RPIB + b_r0;
      const int tok = k_begin + kr;
      const int n = tok / hw, rem = tok - n * hw;
      cv_n[t] = n; cv_ho[t] = rem / g.cv_Wo; cv_wo[t] = rem - cv_ho[t] * g.cv_Wo;
    }
#pragma unroll
    for (int j = 0; j < C::B_G; ++j) {
      const int kr = (wave + 4 * j) * RPIB + b_r0;
      const int col = (n0 - tap * g.cv_cin) + C::swz_b(lane % C::CB, kr) * 16;
      cv_bcol[j] = col < g.cv_cin ? (int64_t)col : -1;
    }
  }
  // input pixel of slot t's token under the block's tap, or -1 when it lies outside the image; then step the token
  auto cv_pixel = [&](int t) -> int64_t {
    const int hi = cv_ho[t] * g.cv_stride + cv_kh - g.cv_pad, wi = cv_wo[t] * g.cv_stride + cv_kw - g.cv_pad;
    const bool ok = (unsigned)hi < (unsigned)g.cv_H && (unsigned)wi < (unsigned)g.cv_W;
    const int64_t pix = ((int64_t)cv_n[t] * g.cv_H + hi) * g.cv_W + wi;
    int wo = cv_wo[t] + g.cv_dw;
    const int c1 = wo >= g.cv_Wo ? 1 : 0;
    wo -= c1 * g.cv_Wo;
    int ho = cv_ho[t] + g.cv_dh + c1;
    const int c2 = ho >= g.cv_Ho ? 1 : 0;
    ho -= c2 * g.cv_Ho;
    cv_wo[t] = wo; cv_ho[t] = ho; cv_n[t] += g.cv_dn + c2;
    return ok ? pix : -1;
  };
  using Checked = std::integral_constant<bool, true>;
  using Unchecked = std::integral_constant<bool, false>;
  // issues load slots t0 .. t1-1 of stage kt; every slot must be issued exactly once per stage, in stage order
  auto issue_range = [&](auto checked, int kt, int buf, int t0, int t1) {
    char* sa = smem + buf * C::LDS_STAGE;
    char* sb = sa + C::LDS_A;
    const int kb = kt * 64;
#pragma unroll
    for (int t = t0; t < t1; ++t) {
      if (t < C::A_G) {
        const char* src = a_ptr[t];
        if constexpr (CONV) {
          if (cv_pixel(t) < 0) src = zero;              // this token's tap falls into the padding: drop its term
        }
        if constexpr (decltype(checked)::value) {
          if (kb + (wave + 4 * t) * RPIA + a_r0 >= span) src = zero;
        }
        dma16(src, sa + (wave + 4 * t) * 1024);
        a_ptr[t] += a_st[t];
      } else {
        const int u = t - C::A_G;
        const char* src = b_ptr[u];
        if constexpr (CONV) {
          const int64_t pix = cv_pixel(t);
          src = (pix >= 0 && cv_bcol[u] >= 0) ? (const char*)g.B + pix * g.cv_cin + cv_bcol[u] : zero;
        }
        if constexpr (decltype(checked)::value) {
          if (kb + (wave + 4 * u) * RPIB + b_r0 >= span) src = zero;
        }
        dma16(src, sb + (wave + 4 * u) * 1024);
        b_ptr[u] += b_st[u];
      }
    }
  };

  floatx16_t acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // ---- fragment reads.  16-lane group q = lane / 16: m (n) half mb = 16 (q & 1), K half h = q >> 1; s = lane % 16.
  //   A, transpose read r in {0,1}: lane addresses 8 bytes = 4 m at token 16*sub + 8h + 4r + s/4,
  //      m = 32 i + mb + 4 (s % 4);  result: lane owns m = 32 i + mb + s, tokens 8h + 4r + 0..3.
  //      Its 16-byte chunk is 4 i + c0 (c0 < 4), which the swizzle moves to 4 (i ^ (s/4)) + c0: four base
  //      addresses per LDS buffer (one per i % 4; a 64-row tile has two) and compile-time offsets for i / 4, r and the sub-step.
  //   B: lane addresses 8 bytes = 8 n at token 16*sub + 8h + s/2, n = wave_n + 32 j + mb + 8 (s % 2);
  //      result: lane owns n = ... + mb + s, tokens 8h + 0..7.
  static_assert(C::WGM == 1, "A fragment addressing");
  constexpr int UA = C::TM < 4 ? C::TM : 4;
  const int s16 = lane & 15, q = lane >> 4;
  const int mb = 16 * (q & 1), h = q >> 1;
  int a_base[2][UA], b_base[2][C::TN];          // LDS byte offsets of sub-step 0, per buffer
  {
    const int k = 8 * h + (s16 >> 2), kk = C::swz_a_row(s16 >> 2);
    const int c0 = (mb >> 3) + ((s16 & 3) >> 1);
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      a_base[0][u] = k * C::RA + ((4 * (u ^ kk) + c0) << 4) + 8 * (s16 & 1);
      a_base[1][u] = a_base[0][u] + C::LDS_STAGE;
    }
  }
#pragma unroll
  for (int j = 0; j < C::TN; ++j) {
    const int k = 8 * h + (s16 >> 1);
    const int nbyte = wn * C::WN + 32 * j + mb + 8 * (s16 & 1);
    b_base[0][j] = C::LDS_A + k * C::RB + (C::swz_b(nbyte >> 4, k) << 4) + (nbyte & 15);
    b_base[1][j] = b_base[0][j] + C::LDS_STAGE;
  }
  const float z = rintf(g.z_x[0]);
  shortx4_t af[2][C::TM][2];
  intx2_t braw[2][C::TN];
  uint32_t bw[2][C::TN][4];                         // converted B fragments: 4 words of two bf16 each
  // LDS read number r of a sub-step: the B codes, then the two halves of every A fragment
  constexpr int NRD = C::TN + 2 * C::TM;
  auto lds_read = [&](auto bufc, int sub, int rb, int r) {
    constexpr int buf = decltype(bufc)::value;
    if (r < C::TN) {
      braw[rb][r] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
          (__attribute__((address_space(3))) intx2_t*)(smem + b_base[buf][r] + sub * 16 * C::RB));
    } else {
      const int i = (r - C::TN) >> 1, hh = (r - C::TN) & 1;
      af[rb][i][hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4_t*)(
          smem + a_base[buf][i % UA] + (i / UA) * 256 + hh * 4 * C::RA + sub * 16 * C::RA));
    }
  };
  auto load_frags = [&](auto bufc, int sub, int rb) {
#pragma unroll
    for (int r = 0; r < NRD; ++r) lds_read(bufc, sub, rb, r);
  };
  // Activation codes -> (code - z) as bf16: integers of magnitude <= 255 are exact.  Piece p of fragment j makes
  // elements 2p and 2p + 1 (5 VALU operations).
  constexpr int NPIECE = 4 * C::TN;
  auto conv_piece = [&](int rb, int piece) {
    const int j = piece >> 2, pp = piece & 3;
    const uint32_t w = (uint32_t)braw[rb][j][pp >> 1];
    const int sh = 16 * (pp & 1);
    const float f0 = (float)((w >> sh) & 0xFFu) - z;
    const float f1 = (float)((w >> (sh + 8)) & 0xFFu) - z;
    bw[rb][j][pp] = pack_bf16x2(f0, f1);
  };
  auto convert = [&](int rb) {
#pragma unroll
    for (int piece = 0; piece < NPIECE; ++piece) conv_piece(rb, piece);
  };
  auto mfma_one = [&](int rb, int i, int j) {
    struct { shortx4_t lo, hi; } a2 = {af[rb][i][0], af[rb][i][1]};
    const uint4 pk = make_uint4(bw[rb][j][0], bw[rb][j][1], bw[rb][j][2], bw[rb][j][3]);
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a2),
                                                        __builtin_bit_cast(bf16x8_t, pk), acc[i][j], 0, 0, 0);
  };
  auto mfma_all = [&](int rb) {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) mfma_one(rb, i, j);
  };

  constexpr int P0 = (LPS + 2) / 3, P1 = (LPS - P0 + 1) / 2, P2 = LPS - P0 - P1;
  auto stage_sync = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- main loop, two LDS stages of 64 tokens, four sub-steps of 16 tokens each.  During the MFMAs of sub-step s
  // the fragments of sub-step s+1 are read and its activation bytes converted; sub-steps 0 and 1 also issue the
  // 2nd and 3rd thirds of the loads of stage kt+1; after sub-step 2 everybody synchronises (stage kt+1 complete,
  // buffer kt free); sub-step 3 reads the first fragments of stage kt+1 and issues the first third of stage kt+2.
  // Invariant: when stage kt starts, the first third of stage kt+1 is in flight iff kt+1 < nfull.
  //
  // A steady-state sub-step has its instruction order pinned, one group per MFMA (the compiler's own interleaving
  // left the conversions of some sub-steps in one clump behind the last MFMA): the MFMAs of fragment set rb; in the
  // first half the LDS reads of the next sub-step (set rb ^ 1), in the second half the conversion of what they
  // returned; the first t1 - t0 groups also issue one global->LDS copy each (stage kt_i into buffer buf_i).
  constexpr int MF = C::TM * C::TN, HF = MF / 2;
  static_assert(HF >= 1 && P0 <= MF && P1 <= MF && P2 <= MF, "copies per sub-step must not exceed its MFMAs");
  auto substep = [&](auto bufn, int sub_next, int rb, int kt_i, int buf_i, int t0, int t1) {
#pragma unroll
    for (int qq = 0; qq < MF; ++qq) {
      mfma_one(rb, qq / C::TN, qq % C::TN);
      if (qq < HF) {
#pragma unroll
        for (int r = (qq * NRD) / HF; r < ((qq + 1) * NRD) / HF; ++r) lds_read(bufn, sub_next, rb ^ 1, r);
      }
      if (qq < t1 - t0) issue_range(Unchecked{}, kt_i, buf_i, t0 + qq, t0 + qq + 1);
      if (qq >= MF - HF) {
        const int q2 = qq - (MF - HF);
#pragma unroll
        for (int piece = (q2 * NPIECE) / HF; piece < ((q2 + 1) * NPIECE) / HF; ++piece) conv_piece(rb ^ 1, piece);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto stage = [&](auto bufc, auto steadyc, int kt) {
    constexpr int cur = decltype(bufc)::value;
    constexpr bool ST = decltype(steadyc)::value;
    using Other = std::integral_constant<int, cur ^ 1>;
    if constexpr (ST) {
      __builtin_amdgcn_sched_barrier(0);
      substep(bufc, 1, 0, kt + 1, cur ^ 1, P0, P0 + P1);
      substep(bufc, 2, 1, kt + 1, cur ^ 1, P0 + P1, LPS);
      substep(bufc, 3, 0, 0, 0, 0, 0);
      stage_sync();
      substep(Other{}, 0, 1, kt + 2, cur, 0, P0);
    } else {
      const bool more1 = kt + 1 < nk;
      if (kt + 1 < nfull) issue_range(Unchecked{}, kt + 1, cur ^ 1, P0, LPS);
      else if (more1) issue_range(Checked{}, kt + 1, cur ^ 1, 0, LPS);
      __builtin_amdgcn_sched_barrier(0);
      load_frags(bufc, 1, 1);
      mfma_all(0);
      convert(1);
      __builtin_amdgcn_sched_barrier(0);
      load_frags(bufc, 2, 0);
      mfma_all(1);
      convert(0);
      __builtin_amdgcn_sched_barrier(0);
      load_frags(bufc, 3, 1);
      mfma_all(0);
      convert(1);
      stage_sync();
      if (more1) load_frags(Other{}, 0, 0);
      if (kt + 2 < nfull) issue_range(Unchecked{}, kt + 2, cur, 0, P0);
      mfma_all(1);
      if (more1) convert(0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  using Steady = std::integral_constant<bool, true>;
  using Drain = std::integral_constant<bool, false>;

  if (nk > 0) issue_range(Checked{}, 0, 0, 0, LPS);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (1 < nfull) issue_range(Unchecked{}, 1, 1, 0, P0);
  if (nk > 0) {
    load_frags(B0{}, 0, 0);
    convert(0);
  }
  int kt = 0;
  for (; kt + 3 < nfull; kt += 2) {                    // stages kt+1 .. kt+3 are full: branch-free pair of stages
    stage(B0{}, Steady{}, kt);
    stage(B1{}, Steady{}, kt + 1);
  }
  for (; kt < nk; kt += 2) {                           // the last (up to four) stages, including a ragged one
    stage(B0{}, Drain{}, kt);
    if (kt + 1 < nk) stage(B1{}, Drain{}, kt + 1);
  }

  // ---- raw fp32 partial tile.  Accumulator layout of the 32x32 MFMA: column lane & 31, rows 8 (r/4) + 4 (lane/32) + r%4.
  const int fr = lane & 31, fh = lane >> 5;
  float* out = g.out + (int64_t)split * g.M * g.N;
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
      const int col = n0 + wn * C::WN + j * 32 + fr;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + i * 32 + 8 * (r >> 2) + 4 * fh + (r & 3);
        if (row < g.M && col < g.N) out[(int64_t)row * g.N + col] = acc[i][j][r];
      }
    }
#endif
}

template <int BM, int BN, bool CONV = false>
__global__ __launch_bounds__(256) void k_gemm_tn(const GemmTnArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_tn_block<BM, BN, CONV>(g, smem, blockIdx.x, gridDim.x);
}

}  // namespace efqat
