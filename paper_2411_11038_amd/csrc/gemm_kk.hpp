// Input-gradient product from two K-contiguous bf16 operands with a hand-pinned instruction order (Eq. 5 left):
//
//   C[m][n] = sum_k A[m][k] * B[n][k],   A = dY bf16 [M][lda],  B = de-quantised W_q^T bf16 [N][ldb]
//
// Same arithmetic as k_gemm_nt; what differs is how the loop is laid out.  Tiles are copied global -> LDS as they
// lie (128-byte rows of 64 K-values, 16-byte chunks XOR-swizzled by the row so that fragment reads are free of bank
// conflicts), fragments are plain 16-byte LDS reads, and every sub-step (one K-slice of 16) is written out as one
// group per MFMA: the MFMA, at most two LDS reads of the next sub-step's fragments, and at most one global -> LDS
// copy of the next stage.  With a single block of four wavefronts per CU there is no second wavefront on a SIMD to
// cover a stall, so the order of these three instruction streams decides the speed; left to the compiler's
// scheduler the reads and copies clump and the matrix cores idle for more than half of the loop.
//
// 256 threads; square tiles of 192 (96 x 96 per wavefront, 9 accumulators), 128 or 64, wavefront grid 2 x 2;
// v_mfma_f32_32x32x16_bf16; K-stage of 64; a ring of NST LDS stages: three (144, 96 or 48 KB; one block a CU, of the 64 x 64 tile
// three, which serves products of too few larger tiles), or eight (see kk_ring_stages).  The copies of stage kt + NST - 1 are issued
// while stage kt is multiplied and are only waited for at the end of stage kt + NST - 2, so with three a copy may take more than a
// whole stage (about 1200 cycles of MFMA work at 192 x 192) before it stalls anything - with two stages the memory latency under
// load did not fit.  Rows past M / N re-read the last valid row (their outputs are discarded), chunks past K come
// from a zero page, so no copy needs a predicate.
#pragma once
#include "common.hpp"

#include <type_traits>
#include <utility>

#include "gemm_epilogue.hpp"
#include "lds_copy.hpp"

namespace efqat {

template <int BM_, int BN_, int NST_ = 3>
struct KkCfg {
  static constexpr int BM = BM_, BN = BN_;
  static constexpr int WGM = 2, WGN = 2;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int A_G = BM / 8 / 4, B_G = BN / 8 / 4;       // 1-KiB copies (8 rows) per wavefront and stage
  static constexpr int LDS_A = BM * 128, LDS_B = BN * 128;
  static constexpr int LDS_STAGE = LDS_A + LDS_B;
  static constexpr int NST = NST_;                               // LDS stages in the ring
  static constexpr int LDS_LOOP = NST * LDS_STAGE;
  static constexpr int LDS_EPI = 4 * 32 * (WN + 8) * 4;
  template <int EPI>
  static constexpr int lds_bytes() {
    constexpr int e = EPI == EPI_DX || EPI == EPI_DXS ? EpiDxAny<KkCfg, float>::LDS : LDS_EPI;
    return LDS_LOOP > e ? LDS_LOOP : e;
  }
  static_assert(WGM * WGN == 4 && WM % 32 == 0 && WN % 32 == 0 && BM % 32 == 0, "tile / wavefront grid");
};

// f(0), f(1), .. with compile-time numbers
template <class F, int... B>
__device__ __forceinline__ void kk_round(F f, std::integer_sequence<int, B...>) { (f(std::integral_constant<int, B>{}), ...); }

// CONV = 1: the A operand is gathered from a token-major dY with the im2col map of a stride-1 convolution, as in
// k_gemm_nt (see GemmArgs): every copy slot keeps (n, h, w) of its input pixel and forms its source address per stage
// from the stage's tap; K = taps * ldc is a whole number of stages.  CONV = 2: a convolution with a stride, rows sorted
// by phase (see ConvPhase); W_q^T is read at the stage's tap as well.
//
// AHEAD (EPI_DXF): the first two rounds of the ring request the epilogue's inputs behind their copies (kk_inputs_ahead); K is at
// least kKkAheadStages whole stages.
constexpr int kKkAheadStages = 9;                     // two rounds of three stages, and the copies in flight behind them
template <int BM, int BN, int EPI, int CONV = 0, int NST = 3, bool AHEAD = false>
__device__ __forceinline__ void gemm_kk_block(const typename ConvArgs<CONV>::type& g, char* smem, int bid, int ntile) {
#if defined(__HIP_DEVICE_COMPILE__)
  using C = KkCfg<BM, BN, NST>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WGN, wn = wave % C::WGN;

  // consecutive block ids land on different XCDs: give each XCD a contiguous range of tiles, then walk the tiles
  // in groups of GM tile rows so that the blocks running together share operand rows in L2
  const int pid = xcd_contiguous_index(bid, ntile);
  const int GM = 8;
  const int per_group = GM * g.tiles_n;
  const int group = pid / per_group;
  const int first_m = group * GM;
  const int gsize = (g.tiles_m - first_m) < GM ? (g.tiles_m - first_m) : GM;
  int tm = first_m + (pid % per_group) % gsize;
  int tn = (pid % per_group) / gsize;
  ConvPhase ph;
  if constexpr (CONV == 2) strided_tile(g, bid, &ph, &tm, &tn);
  const int m0 = tm * C::BM, n0 = tn * C::BN;

  const int K = CONV == 2 ? ph.ntap * g.cv_spt * 64 : g.K;
  const int nk = (K + 63) / 64;
  const int nfull = K / 64;
  const char* zero = zero_page();

  // ---- global -> LDS copies with running pointers.  Slot j of an operand covers tile rows (wave + 4 j) * 8 .. + 7;
  // lane l lands in row l / 8, physical chunk l % 8, and fetches the logical chunk that the swizzle puts there.
  const int c_lrow = lane >> 3;
  const int c_lch = (lane & 7) ^ (((wave * 8 + c_lrow) >> 1) & 7);   // same for every slot: 32 j = 0 (mod 16)
  const char* a_ptr[C::A_G];
  const char* b_ptr[C::B_G];
  int cv_q0[CONV ? C::A_G : 1], cv_hw[CONV ? C::A_G : 1];   // CONV: n * Ho * Wo and (h << 16 | w) of the slot's pixel
#pragma unroll
  for (int j = 0; j < C::A_G; ++j) {
    int gm = m0 + (wave + 4 * j) * 8 + c_lrow;
    const int rows = CONV == 2 ? ph.rows : g.M;
    gm = gm < rows ? gm : rows - 1;
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
      a_ptr[j] = (const char*)g.A + (int64_t)gm * g.lda * 2 + c_lch * 16;
    }
  }
  // CONV: source of this lane's 16 bytes of A slot j in stage kt (the zero page when the tap falls outside the image)
  auto a_src_conv = [&](int j, int kt) -> const char* {
    if constexpr (CONV == 2) {
      int a, b, cst;
      strided_stage(g, ph, kt, &a, &b, &cst);
      const int ho = (cv_hw[j] >> 16) + ph.dh0 - a, wo = (cv_hw[j] & 0xFFFF) + ph.dw0 - b;
      const bool ok = (unsigned)ho < (unsigned)g.cv_Ho && (unsigned)wo < (unsigned)g.cv_Wo;
      const int64_t pix = (int64_t)cv_q0[j] + ho * g.cv_Wo + wo;
      return ok ? (const char*)g.A + (pix * g.lda + cst * 64) * 2 + c_lch * 16 : zero;
    } else {
      // stage kt = (tap, 64-channel stage) along K
      const int tap = (int)(((uint64_t)(uint32_t)kt * g.cv_m_spt) >> 32), cst = kt - tap * g.cv_spt;
      const int kh = (int)(((uint64_t)(uint32_t)tap * g.cv_m_kw) >> 32), kw = tap - kh * g.cv_KW;
      const int ho = (cv_hw[j] >> 16) + g.cv_pad - kh, wo = (cv_hw[j] & 0xFFFF) + g.cv_pad - kw;
      const bool ok = (unsigned)ho < (unsigned)g.cv_Ho && (unsigned)wo < (unsigned)g.cv_Wo;
      const int64_t pix = (int64_t)cv_q0[j] + ho * g.cv_Wo + wo;
      return ok ? (const char*)g.A + (pix * g.lda + cst * 64) * 2 + c_lch * 16 : zero;
    }
  };
#pragma unroll
  for (int j = 0; j < C::B_G; ++j) {
    int gn = n0 + (wave + 4 * j) * 8 + c_lrow;
    gn = gn < g.N ? gn : g.N - 1;
    b_ptr[j] = (const char*)g.B + (int64_t)gn * g.ldb * 2 + c_lch * 16;
  }
  constexpr int LPS = C::A_G + C::B_G;
  using Checked = std::integral_constant<bool, true>;
  using Unchecked = std::integral_constant<bool, false>;
  auto issue_range = [&](auto checked, int kt, int buf, int t0, int t1) {
    char* sa = smem + buf * C::LDS_STAGE;
    char* sb = sa + C::LDS_A;
    const bool off = decltype(checked)::value && (kt * 64 + c_lch * 8 >= K);   // K % 8 == 0: a chunk is all in or out
#pragma unroll
    for (int t = t0; t < t1; ++t) {
      if (t < C::A_G) {
        if constexpr (CONV) {
          dma16(a_src_conv(t, kt), sa + (wave + 4 * t) * 1024);
        } else {
          dma16(off ? zero : a_ptr[t], sa + (wave + 4 * t) * 1024);
          a_ptr[t] += 128;
        }
      } else {
        const int u = t - C::A_G;
        if constexpr (CONV == 2) {
          int a, b, cst;
          strided_stage(g, ph, kt, &a, &b, &cst);
          const int tap = (ph.kh0 + g.cv_stride * a) * g.cv_KW + ph.kw0 + g.cv_stride * b;
          dma16(b_ptr[u] + (int64_t)(tap * g.cv_spt + cst) * 128, sb + (wave + 4 * u) * 1024);
        } else {
          dma16(off ? zero : b_ptr[u], sb + (wave + 4 * u) * 1024);
          b_ptr[u] += 128;
        }
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

  // ---- fragment reads: lane owns row 32 i + lane % 32 of its wavefront's rows, K-values 16 sub + 8 (lane / 32) + 0..7,
  // i.e. logical chunk 2 sub + lane / 32.  Rows 32 i + r share their swizzle term, so one address per (buffer, sub)
  // and operand serves every fragment through the instruction's immediate offset.
  const int fr = lane & 31, fh = lane >> 5;
  int a_addr[C::NST][4], b_addr[C::NST][4];
#pragma unroll
  for (int sub = 0; sub < 4; ++sub) {
    const int ch = ((2 * sub + fh) ^ ((fr >> 1) & 7)) << 4;
    a_addr[0][sub] = (wm * C::WM + fr) * 128 + ch;
    b_addr[0][sub] = C::LDS_A + (wn * C::WN + fr) * 128 + ch;
#pragma unroll
    for (int b = 1; b < C::NST; ++b) {
      a_addr[b][sub] = a_addr[0][sub] + b * C::LDS_STAGE;
      b_addr[b][sub] = b_addr[0][sub] + b * C::LDS_STAGE;
    }
  }
  static_assert((C::WM % 16) == 0 && (C::WN % 16) == 0, "the swizzle term must not depend on the wavefront's origin");
  typedef int intx4_t __attribute__((ext_vector_type(4)));
  intx4_t af[2][C::TM], bf[2][C::TN];
  // LDS read number r of a sub-step, in the order the MFMAs first need them: A0, all of B, then the other A
  constexpr int NRD = C::TM + C::TN;
  auto lds_read = [&](auto bufc, int sub, int rb, int r) {
    constexpr int buf = decltype(bufc)::value;
    if (r == 0) {
      af[rb][0] = *reinterpret_cast<const intx4_t*>(smem + a_addr[buf][sub]);
    } else if (r <= C::TN) {
      bf[rb][r - 1] = *reinterpret_cast<const intx4_t*>(smem + b_addr[buf][sub] + (r - 1) * 4096);
    } else {
      af[rb][r - C::TN] = *reinterpret_cast<const intx4_t*>(smem + a_addr[buf][sub] + (r - C::TN) * 4096);
    }
  };
  auto load_frags = [&](auto bufc, int sub, int rb) {
#pragma unroll
    for (int r = 0; r < NRD; ++r) lds_read(bufc, sub, rb, r);
  };
  auto mfma_one = [&](int rb, int i, int j) {
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[rb][i]),
                                                        __builtin_bit_cast(bf16x8_t, bf[rb][j]), acc[i][j], 0, 0, 0);
  };
  auto mfma_all = [&](int rb) {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) mfma_one(rb, i, j);
  };

  // copies of one stage, by the sub-step that issues them: the first P0 go out one stage early (last sub-step of the
  // stage before, right after the barrier that frees their buffer), the rest in sub-steps 0, 1, 2
  constexpr int P0 = LPS / 4, P1 = (LPS - P0 + 2) / 3, P2 = (LPS - P0 - P1 + 1) / 2, P3 = LPS - P0 - P1 - P2;
  // end of a stage: the copies of the next stage have landed, every wavefront is done reading this stage's buffer.
  // steady: the copies of the NST - 2 stages behind the next, and `more` other loads issued since its last copy, stay in
  // flight.  Otherwise the copies of `ahead` stages do; ahead < 0: one of the last two stages - every copy landed before it
  // began and none is issued any more.
  auto stage_sync = [&](auto steadyc, auto morec, int ahead) {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(steadyc)::value) {
      constexpr int N = (NST - 2) * LPS + decltype(morec)::value;
      static_assert(N < 64, "the counter has six bits");
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
    } else if (ahead < 0) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    } else if (ahead >= 4) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * LPS < 64 ? 4 * LPS : 0) : "memory");
    } else if (ahead >= 2) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * LPS) : "memory");
    } else if (ahead == 1) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPS) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // One steady-state sub-step, one group per MFMA: the MFMAs of fragment set rb; spread over the first RG groups
  // the LDS reads of the next sub-step (into set rb ^ 1); the first t1 - t0 groups also issue one global -> LDS copy
  // each (stage kt_i into buffer buf_i).
  constexpr int MF = C::TM * C::TN;
  constexpr int RG = (2 * MF + 2) / 3;
  static_assert(P0 <= MF && P1 <= MF && P2 <= MF && P3 <= MF, "copies per sub-step must not exceed its MFMAs");
  auto substep = [&](auto bufn, int sub_next, int rb, int kt_i, int buf_i, int t0, int t1) {
#pragma unroll
    for (int qq = 0; qq < MF; ++qq) {
      mfma_one(rb, qq / C::TN, qq % C::TN);
      if (qq < RG) {
#pragma unroll
        for (int r = (qq * NRD) / RG; r < ((qq + 1) * NRD) / RG; ++r) lds_read(bufn, sub_next, rb ^ 1, r);
      }
      if (qq < t1 - t0) issue_range(Unchecked{}, kt_i, buf_i, t0 + qq, t0 + qq + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // the fused dX epilogue
  static_assert(!AHEAD || (EPI == EPI_DXF && 3 * NST == kKkAheadStages), "inputs ahead: straight-line epilogue, ring of three");
  typename std::conditional<EPI == EPI_DXF, EpiDxFast<C, AHEAD>,
                            EpiDxAny<C, typename std::conditional<EPI == EPI_DXS, float, bf16_t>::type, CONV == 2>>::type epi;
  const int m_end = CONV == 2 ? ph.rows : g.M;
  const bool edge = m0 + C::BM > m_end || n0 + C::BN > g.N;
  int* rowmap = reinterpret_cast<int*>(smem + C::template lds_bytes<EPI>());   // CONV = 2: the matrix row of every tile row
  constexpr int PEEL = 2 * NST;                       // two rounds of the ring
  const int kt_epi = nk >= 2 ? nk - 2 : 0;            // the first of the last two stages
  if constexpr (EPI == EPI_DXF) epi.begin(g, m0, n0, wm, wn);

  // ---- main loop.  Stage kt lives in buffer kt % NST.  On entry to stage kt the first P0 copies of stage kt + NST - 1 have
  // been issued if and only if that stage is a full one; both variants keep this true for kt + 1.
  //
  // AHEAD: the first PEEL stages, steady ones (kt + NST < nfull), also request the epilogue's inputs, some groups of rows each, behind
  // the stage's copies.  They come out of HBM while the matrix cores work and are waited for one stage later than the copies before
  // them.
  // the requests of peeled stage ps, then its end
  auto request_and_sync = [&](auto& e, auto psc) {
    using E = typename std::remove_reference<decltype(e)>::type;
    constexpr int PS = decltype(psc)::value;
    constexpr int G0 = PS >= NST - 2 ? (PS - NST + 2) * E::GROUPS / PEEL : 0, G1 = PS * E::GROUPS / PEEL, G2 = (PS + 1) * E::GROUPS / PEEL;
    asm volatile("" ::: "memory");                    // behind the copies: stage_sync counts on this order
#pragma unroll
    for (int q = G1; q < G2; ++q) e.fetch(q / E::HP, q % E::HP);
    stage_sync(std::integral_constant<bool, true>{}, std::integral_constant<int, E::LOADS * (G2 - G0)>{}, 0);
  };
  auto stage = [&](auto bufc, auto steadyc, int kt, auto peelc) {
    constexpr int cur = decltype(bufc)::value;
    constexpr bool ST = decltype(steadyc)::value;
    constexpr int PS = decltype(peelc)::value;        // peeled stage, -1: none
    constexpr int nxt = (cur + 1) % NST, nn = (cur + NST - 1) % NST;
    using Next = std::integral_constant<int, nxt>;
    const int ki = kt + NST - 1;     // the stage whose copies are issued
    if constexpr (ST) {              // kt + NST < nfull
      __builtin_amdgcn_sched_barrier(0);
      substep(bufc, 1, 0, ki, nn, P0, P0 + P1);
      substep(bufc, 2, 1, ki, nn, P0 + P1, P0 + P1 + P2);
      substep(bufc, 3, 0, ki, nn, P0 + P1 + P2, LPS);
      if constexpr (PS >= 0) request_and_sync(epi, peelc);
      else stage_sync(steadyc, std::integral_constant<int, 0>{}, 0);
      substep(Next{}, 0, 1, ki + 1, cur, 0, P0);
    } else {
      const bool more1 = kt + 1 < nk;
      // the last two stages: the preceding barrier was passed with every copy landed, and nothing more is issued - the
      // moment to request the epilogue's first inputs
      const int ahead = kt + 2 >= nk ? -1 : kt + 3 >= nk ? 0 : (ki < nk - 1 ? ki : nk - 1) - (kt + 1);
      if (ki < nfull) issue_range(Unchecked{}, ki, nn, P0, LPS);
      else if (ki < nk) issue_range(Checked{}, ki, nn, 0, LPS);
      if (kt == kt_epi) {
        if constexpr (EPI == EPI_DXF) { if (!AHEAD) epi.prefetch(); }
        else epi.prefetch(g, m0, n0, wm, wn, m_end, edge, rowmap);
      }
      __builtin_amdgcn_sched_barrier(0);
      load_frags(bufc, 1, 1);
      mfma_all(0);
      __builtin_amdgcn_sched_barrier(0);
      load_frags(bufc, 2, 0);
      mfma_all(1);
      __builtin_amdgcn_sched_barrier(0);
      load_frags(bufc, 3, 1);
      mfma_all(0);
      stage_sync(steadyc, std::integral_constant<int, 0>{}, ahead);
      if (more1) load_frags(Next{}, 0, 0);
      if (ki + 1 < nfull) issue_range(Unchecked{}, ki + 1, cur, 0, P0);
      mfma_all(1);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using Steady = std::integral_constant<bool, true>;
  using Drain = std::integral_constant<bool, false>;

  if constexpr (CONV == 2) {
    if (tid < C::BM) {
      int q0, hw;
      rowmap[tid] = m0 + tid < ph.rows ? strided_pixel(g, ph, m0 + tid, &q0, &hw) : -1;
    }
  }

#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nk) issue_range(Checked{}, s, s, 0, LPS);
  // stage 0 has to be there; the last stages (see stage_sync) count on everything having landed
  if (nk >= NST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * LPS) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (NST - 1 < nfull) issue_range(Unchecked{}, NST - 1, NST - 1, 0, P0);
  if (nk > 0) load_frags(std::integral_constant<int, 0>{}, 0, 0);
  int kt = 0;
  using No = std::integral_constant<int, -1>;
  // f(stage of the round) for a round of the ring
  auto round = [&](auto f) { kk_round(f, std::make_integer_sequence<int, NST>{}); };
  if constexpr (AHEAD) {
    round([&](auto b) { stage(b, Steady{}, decltype(b)::value, b); });
    round([&](auto b) { stage(b, Steady{}, NST + decltype(b)::value, std::integral_constant<int, NST + decltype(b)::value>{}); });
    kt = PEEL;
  }
  for (; kt + 2 * NST - 1 < nfull; kt += NST) round([&](auto b) { stage(b, Steady{}, kt + decltype(b)::value, No{}); });
  for (; kt < nk; kt += NST)
    round([&](auto b) {
      if (kt + decltype(b)::value < nk) stage(b, Drain{}, kt + decltype(b)::value, No{});
    });
  __syncthreads();

  if constexpr (EPI == EPI_DXF) {
    epi.run(g, acc, smem, bid);
  } else {
    if (CONV == 2 && nk == 0) epi.prefetch(g, m0, n0, wm, wn, m_end, edge, rowmap);   // a phase without taps
    epi.run(g, acc, smem, edge, bid);
  }
#endif
}

template <int BM, int BN, int EPI, int CONV = 0, int NST = 3, bool AHEAD = false>
__global__ __launch_bounds__(256) void k_gemm_kk(const typename ConvArgs<CONV>::type g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_kk_block<BM, BN, EPI, CONV, NST, AHEAD>(g, smem, blockIdx.x, gridDim.x);
}

}  // namespace efqat
