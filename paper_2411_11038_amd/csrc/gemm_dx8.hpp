// Input-gradient product with the weight operand taken straight from the int8 codes (Eq. 5 left):
//
//   dX_q[t][i] = sum_c dY[t][c] * (S_w[c] * code[c][i]),   A = dY bf16 [T][lda] (K = c contiguous),
//                                                          B = weight codes int8 [C_out][ldb] (K = c is the row)
//
// A tiles are staged and read like any K-contiguous operand (128-byte rows, 16-byte fragment reads); B tiles are
// copied as they lie and read with ds_read_b64_tr_b8, then turned into bf16(S_w[c] * code) in registers with the
// 64 scales of the stage, which travel through LDS as well.  bf16(S_w * code) is the same rounding a materialised
// bf16 copy of W_q would apply, so results do not depend on which kernel runs.  Compared with that copy the
// weight operand costs half the bytes in L2, L1 and LDS (a 256 x 256 stage is 48 KB instead of 64 KB), and the
// transposed bf16 matrix is never written.  Same wavefront grid (1 x 4), pipeline and load discipline as k_gemm_tn;
// the epilogue is the fused straight-through / dS_x / dZ_x epilogue shared with the K-contiguous kernel.
//
// The same kernel in DW mode is the weight-gradient product for a channel-major dY [C_out][T] (Eq. 5 right,
// restricted):  dW_q[m][i] = sum_t dY[idx[m]][t] * (code[t][i] - Z_x).  The A rows are the selected channels, read
// through the index list in the tile loads (frozen channels are never touched), B = the uint8 activation codes as
// they lie ([T][C_in]; the contraction index is the row), converted as in k_gemm_tn; split-K, raw fp32 partial tiles.
// ATN: the A operand has the contraction index as its row ([K][lda], K-major like B) and is read with
// ds_read_b64_tr_b16 as in k_gemm_tn; otherwise it is K-contiguous ([M][lda]).
#pragma once
#include "common.hpp"

#include <type_traits>

#include "gemm_epilogue.hpp"
#include "lds_copy.hpp"

namespace efqat {

template <int BM_, int BN_, bool ATN = false>
struct Dx8Cfg {
  static constexpr int BM = BM_, BN = BN_;
  static constexpr int WGM = 1, WGN = 4;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int RB = BN;                              // bytes per LDS row of B (one channel c)
  static constexpr int CB = RB / 16;
  static constexpr int RA = 2 * BM, CA = RA / 16;            // ATN: bytes / chunks per LDS row of A (one K index)
  static constexpr int A_G = BM / 8 / 4, B_G = 64 * RB / 1024 / 4;   // 1-KiB loads per wave and stage
  static constexpr int LDS_A = BM * 128, LDS_B = 64 * RB, LDS_S = 4 * 256;   // scales: one copy per wavefront
  static constexpr int LDS_STAGE = LDS_A + LDS_B + LDS_S;
  static constexpr int LDS_LOOP = 2 * LDS_STAGE;
  static constexpr int LDS_EPI = 4 * 32 * (WN + 8) * 4;
  template <bool ANY>                                        // with EpiDxAny
  static constexpr int lds_bytes() {
    constexpr int e = ANY ? EpiDxAny<Dx8Cfg, float>::LDS : LDS_EPI;
    return LDS_LOOP > e ? LDS_LOOP : e;
  }
  static constexpr int KSH = RB == 256 ? 0 : 1;
  __device__ static __forceinline__ int swz_a(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }
  __device__ static __forceinline__ int swz_atn_row(int k) { return BM == 64 ? (k >> 1) & 1 : k & 3; }   // as in TnCfg
  __device__ static __forceinline__ int swz_atn(int c, int k) { return c ^ (4 * swz_atn_row(k)); }
  __device__ static __forceinline__ int swz_b(int c, int k) { return c ^ (2 * ((k >> KSH) & (CB / 2 - 1))); }
};

// FAST (dX only): the straight-line epilogue for bf16 x / dX and whole tiles (epilogue_dx_fast).
// MASK: the general epilogue keeps the mask in every chunk (see epi_chunk).
template <int BM, int BN, bool DW = false, bool ATN = false, bool FAST = false, bool MASK = false>
__device__ __forceinline__ void gemm_dx8_block(const GemmDx8Args& ga, char* smem, int bid, int nblk) {
#if defined(__HIP_DEVICE_COMPILE__)
  using C = Dx8Cfg<BM, BN, ATN>;
  const GemmArgs& g = ga.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = 0, wn = wave;

  const int ntile = g.tiles_m * g.tiles_n;
  const int logical = xcd_contiguous_index(bid, nblk);
  const int split = logical / ntile;                   // split-K slice (0 when there is one)
  const int pid = logical - split * ntile;
  const int GM = g.group_m;
  const int per_group = GM * g.tiles_n;
  const int group = pid / per_group;
  const int first_m = group * GM;
  const int gsize = (g.tiles_m - first_m) < GM ? (g.tiles_m - first_m) : GM;
  const int tm = first_m + (pid % per_group) % gsize;
  const int tn = (pid % per_group) / gsize;
  const int m0 = tm * C::BM, n0 = tn * C::BN;

  // K range of this block: everything for dX, one split-K slice for dW (K below is the length of the slice)
  const int k_begin = DW ? split * g.k_per_split : 0;
  const int k_end_ = DW ? ((k_begin + g.k_per_split) < g.K ? (k_begin + g.k_per_split) : g.K) : g.K;
  const int K = k_end_ > k_begin ? k_end_ - k_begin : 0;
  const int nk = (K + 63) / 64;
  const int nfull = K / 64;
  const char* zero = zero_page();

  // ---- global -> LDS copies with running pointers (one 64-bit add per copy; slots outside the operands rest on
  // the zero page with stride 0).  A: slot j covers tile rows (wave + 4 j) * 8 .. + 7, lane l lands in row l / 8,
  // physical chunk l % 8.  B: slot j covers channel rows (wave + 4 j) * RPIB .. of the stage.
  constexpr int RPIB = 1024 / C::RB;
  const int a_lrow = lane >> 3;
  const int a_lch = (lane & 7) ^ (((wave * 8 + a_lrow) >> 1) & 7);   // logical chunk fetched by this lane (same for all j)
  const int b_r0 = lane / C::CB;
  const char* a_ptr[C::A_G];
  const char* b_ptr[C::B_G];
  uint32_t b_st[C::B_G];
  uint32_t a_st[C::A_G];                                // per-stage pointer step of the A slots
  constexpr int RPIA = 1024 / C::RA;                    // ATN: K rows per 1-KiB load
  const int atn_r0 = lane / C::CA;
#pragma unroll
  for (int j = 0; j < C::A_G; ++j) {
    if constexpr (ATN) {
      // slot j covers the K rows (wave + 4 j) * RPIA .. of a stage; lane l lands in row l / CA, physical chunk l % CA
      const int kr = (wave + 4 * j) * RPIA + atn_r0;
      const int col = m0 + C::swz_atn(lane % C::CA, kr) * 8;
      const bool on = col < ga.a_cols;
      a_ptr[j] = on ? (const char*)g.A + ((int64_t)(k_begin + kr) * g.lda + col) * 2 : zero;
      a_st[j] = on ? (uint32_t)(g.lda * 128) : 0u;
    } else {
      int gm = m0 + (wave + 4 * j) * 8 + a_lrow;
      gm = gm < g.M ? gm : g.M - 1;                     // rows past the edge re-read a valid row (outputs discarded)
      const int64_t src_row = (DW && g.a_rows) ? (int64_t)g.a_rows[gm] : (int64_t)gm;
      a_ptr[j] = (const char*)g.A + (src_row * g.lda + k_begin) * 2 + a_lch * 16;
      a_st[j] = 128u;
    }
  }
#pragma unroll
  for (int j = 0; j < C::B_G; ++j) {
    const int kr = (wave + 4 * j) * RPIB + b_r0;
    const int col = n0 + C::swz_b(lane % C::CB, kr) * 16;
    const bool on = col < ga.b_cols;
    b_ptr[j] = on ? (const char*)g.B + (int64_t)(k_begin + kr) * g.ldb + col : zero;
    b_st[j] = on ? (uint32_t)(g.ldb * 64) : 0u;
  }
  const char* s_ptr = DW ? zero : (const char*)g.s_w + lane * 4;   // dX: the scale of channel kt * 64 + lane
  constexpr int LPS = C::A_G + C::B_G + (DW ? 0 : 1);
  using Checked = std::integral_constant<bool, true>;
  using Unchecked = std::integral_constant<bool, false>;
  auto issue_range = [&](auto checked, int kt, int buf, int t0, int t1) {
    char* sa = smem + buf * C::LDS_STAGE;
    char* sb = sa + C::LDS_A;
    char* ss = sb + C::LDS_B;
    const int kb = kt * 64;
#pragma unroll
    for (int t = t0; t < t1; ++t) {
      if (t < C::A_G) {
        const char* src = a_ptr[t];
        if constexpr (decltype(checked)::value) {
          if constexpr (ATN) {
            if (kb + (wave + 4 * t) * RPIA + atn_r0 >= K) src = zero;
          } else {
            if (kb + a_lch * 8 >= K) src = zero;        // K is a multiple of 8: a chunk is all in or all out
          }
        }
        dma16(src, sa + (wave + 4 * t) * 1024);
        a_ptr[t] += a_st[t];
      } else if (t < C::A_G + C::B_G) {
        const int u = t - C::A_G;
        const char* src = b_ptr[u];
        if constexpr (decltype(checked)::value) {
          if (kb + (wave + 4 * u) * RPIB + b_r0 >= K) src = zero;
        }
        dma16(src, sb + (wave + 4 * u) * 1024);
        b_ptr[u] += b_st[u];
      } else {
        // every wavefront fetches its own copy of the stage's 64 scales: no branch in the loop body
        const char* src = s_ptr;
        if constexpr (decltype(checked)::value) {
          if (kb + lane >= K) src = zero;
        }
        dma4(src, ss + wave * 256);
        s_ptr += 256;
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

  // ---- fragment reads.  A (rows = tokens, 16 bytes = 8 channels): lane owns row 32 i + lane % 32, channels
  // 16 sub + 8 (lane / 32) + 0..7.  B (transpose read): lane addresses 8 columns of channel 16 sub + 8 h + s / 2 and
  // ends up with column 32 j + lane % 32, channels 16 sub + 8 h + 0..7, h = lane / 32.
  const int fr = lane & 31, fh = lane >> 5;
  const int s16 = lane & 15, q = lane >> 4;
  const int mb = 16 * (q & 1);
  int b_base[2][C::TN];
#pragma unroll
  for (int j = 0; j < C::TN; ++j) {
    const int k = 8 * fh + (s16 >> 1);
    const int nbyte = wn * C::WN + 32 * j + mb + 8 * (s16 & 1);
    b_base[0][j] = C::LDS_A + k * C::RB + (C::swz_b(nbyte >> 4, k) << 4) + (nbyte & 15);
    b_base[1][j] = b_base[0][j] + C::LDS_STAGE;
  }
  typedef int intx4_t __attribute__((ext_vector_type(4)));
  intx4_t af[2][C::TM];
  // ATN: four base addresses per LDS buffer for the transpose reads of A (see k_gemm_tn)
  constexpr int UA = C::TM < 4 ? C::TM : 4;
  int atn_base[2][UA];
  if constexpr (ATN) {
    const int h = q >> 1;
    const int k = 8 * h + (s16 >> 2), kk = C::swz_atn_row(s16 >> 2);
    const int c0 = (mb >> 3) + ((s16 & 3) >> 1);
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      atn_base[0][u] = k * C::RA + ((4 * (u ^ kk) + c0) << 4) + 8 * (s16 & 1);
      atn_base[1][u] = atn_base[0][u] + C::LDS_STAGE;
    }
  }
  intx2_t braw[2][C::TN];
  float scf[2][8];                                  // the 8 scales of a lane's K positions
  uint32_t bw[2][C::TN][4];                         // converted B fragments: 4 words of two bf16 each
  // LDS read number r of a sub-step: B codes, the scales, then the A fragments
  constexpr int NSC = DW ? 0 : 2;                   // LDS reads of scales per sub-step
  constexpr int NRD = C::TN + NSC + (ATN ? 2 : 1) * C::TM;
  auto lds_read = [&](auto bufc, int sub, int rb, int r) {
    constexpr int buf = decltype(bufc)::value;
    const char* st = smem + buf * C::LDS_STAGE;
    if (r < C::TN) {
      braw[rb][r] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
          (__attribute__((address_space(3))) intx2_t*)(smem + b_base[buf][r] + sub * 16 * C::RB));
    } else if (r < C::TN + NSC) {
      const int hlf = r - C::TN;
      const float4 v = *reinterpret_cast<const float4*>(st + C::LDS_A + C::LDS_B + wave * 256 +
                                                        (16 * sub + 8 * fh + 4 * hlf) * 4);
      scf[rb][4 * hlf] = v.x; scf[rb][4 * hlf + 1] = v.y; scf[rb][4 * hlf + 2] = v.z; scf[rb][4 * hlf + 3] = v.w;
    } else if constexpr (ATN) {
      const int i = (r - C::TN - NSC) >> 1, hh = (r - C::TN - NSC) & 1;
      const shortx4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4_t*)(
          smem + atn_base[buf][i % UA] + (i / UA) * 256 + hh * 4 * C::RA + sub * 16 * C::RA));
      const intx2_t v2 = __builtin_bit_cast(intx2_t, v);
      af[rb][i][2 * hh] = v2[0]; af[rb][i][2 * hh + 1] = v2[1];
    } else {
      const int i = r - C::TN - NSC;
      af[rb][i] = *reinterpret_cast<const intx4_t*>(st + C::swz_a(32 * i + fr, 2 * sub + fh));
    }
  };
  const float zq = DW ? rintf(g.z_x[0]) : 0.0f;
  auto load_frags = [&](auto bufc, int sub, int rb) {
#pragma unroll
    for (int r = 0; r < NRD; ++r) lds_read(bufc, sub, rb, r);
  };
  // Weight codes -> bf16(S_w[c] * code): the signed byte is converted in one operation (the conversion selects and
  // sign-extends the byte of its source) and multiplied by its scale in fp32, then rounded once like the product
  // itself.  Piece p of fragment j makes elements 2p and 2p + 1 (5 VALU operations).
  constexpr int NPIECE = 4 * C::TN;
  auto conv_piece = [&](int rb, int piece) {
    const int j = piece >> 2, pp = piece & 3;
    const int sh = 16 * (pp & 1);
    if constexpr (DW) {                                // activation codes: (code - Z_x), exact in bf16
      const uint32_t w = (uint32_t)braw[rb][j][pp >> 1];
      bw[rb][j][pp] = pack_bf16x2((float)((w >> sh) & 0xFFu) - zq, (float)((w >> (sh + 8)) & 0xFFu) - zq);
    } else {
      const uint32_t w = (uint32_t)braw[rb][j][pp >> 1];
      const float f0 = (float)(int8_t)((w >> sh) & 0xFFu) * scf[rb][2 * pp];
      const float f1 = (float)(int8_t)((w >> (sh + 8)) & 0xFFu) * scf[rb][2 * pp + 1];
      bw[rb][j][pp] = pack_bf16x2(f0, f1);
    }
  };
  auto convert = [&](int rb) {
#pragma unroll
    for (int piece = 0; piece < NPIECE; ++piece) conv_piece(rb, piece);
  };
  auto mfma_one = [&](int rb, int i, int j) {
    const uint4 pk = make_uint4(bw[rb][j][0], bw[rb][j][1], bw[rb][j][2], bw[rb][j][3]);
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[rb][i]),
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

  // One steady-state sub-step with its instruction order pinned, one group per MFMA: the MFMAs of fragment set rb;
  // in the first half the LDS reads of the next sub-step (set rb ^ 1), in the second half the conversion of what
  // they returned; the first t1 - t0 groups also issue one global->LDS copy each (stage kt_i into buffer buf_i).
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

  // ---- main loop: the schedule of k_gemm_tn (two LDS stages, four sub-steps, loads of the next stage in thirds)
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
  for (; kt + 3 < nfull; kt += 2) {
    stage(B0{}, Steady{}, kt);
    stage(B1{}, Steady{}, kt + 1);
  }
  for (; kt < nk; kt += 2) {
    stage(B0{}, Drain{}, kt);
    if (kt + 1 < nk) stage(B1{}, Drain{}, kt + 1);
  }
  __syncthreads();

  if constexpr (DW) {
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
  } else if constexpr (FAST) {
    epilogue_dx_fast<C>(g, acc, smem, m0, n0, wm, wn, bid);
  } else {
    epilogue_dx<C, false, MASK>(g, acc, smem, m0, n0, wm, wn, g.M, bid);
  }
#endif
}

template <int BM, int BN, bool DW = false, bool ATN = false, bool FAST = false, bool MASK = false>
__global__ __launch_bounds__(256, BM == 64 ? 3 : BM == 128 ? 2 : 1) void k_gemm_dx8(const GemmDx8Args ga) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_dx8_block<BM, BN, DW, ATN, FAST, MASK>(ga, smem, blockIdx.x, gridDim.x);
}

}  // namespace efqat
