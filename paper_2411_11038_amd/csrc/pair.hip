// The two products of Eq. 5 in one grid: dX on tiles of 64 x 64 (k_gemm_kk's or k_gemm_nt's loop) and dW on 64-row tiles
// (k_gemm_tn's, or k_gemm_nt's from staged operands).  They do not depend on each other, and where neither fills the chip
// one behind the other costs the sum of two latencies: launch, first loads, K loop, drain.  pair_plan decides by the measured
// costs of both; backward calls in one grid / one after the other, us: 192 x 640 -> 128, k = 6: 12.2 / 16.4; 64 x 7 x 7, 128 -> 256,
// 1 x 1: 13.6 / 18.5; 792 x 256 -> 1464, k = 366: 21.7 / 27.4; 16 x 24 x 24, 120 -> 320, 3 x 3: 56.6 / 71.0; 100 drawn layers and
// convolutions 1.125 x, none slower by 2 %.  64-row tiles only: four (two stages) or three (ring) blocks of either
// share a CU.
#include "gemm_dx8.hpp"
#include "gemm_kk.hpp"
#include "gemm_nt.hpp"
#include "gemm_tn.hpp"

#include <algorithm>

namespace efqat {

template <bool RING, int EPI, int CONV, bool STAGED>
struct PairCfg {
  static constexpr int kDx = (RING ? KkCfg<64, 64>::template lds_bytes<EPI>() : TileCfg<64, 64, 2>::template lds_bytes<EPI>()) +
                             (CONV == 2 ? 64 * (int)sizeof(int) : 0);
  static constexpr int kDw = STAGED ? TileCfg<64, 64, 2>::template lds_bytes<EPI_RAW>() : TnCfg<64, 128>::LDS_BYTES;
  static constexpr int kLds = kDx > kDw ? kDx : kDw;
  struct Args {
    typename ConvArgs<CONV>::type dx;
    typename std::conditional<STAGED, GemmArgs, GemmTnArgs>::type dw;
    int n_dx;
  };
};

// blocks 0 .. n_dx - 1: tiles of dX, then the tiles and slices of dW
template <bool RING, int EPI, int CONV, bool STAGED>
__global__ __launch_bounds__(256, RING ? 3 : 4) void k_pair(const typename PairCfg<RING, EPI, CONV, STAGED>::Args p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x;
  if (b < p.n_dx) {
    if constexpr (RING) gemm_kk_block<64, 64, EPI, CONV>(p.dx, smem, b, p.n_dx);
    else gemm_nt_block<64, 64, EPI, false, CONV>(p.dx, smem, b, p.n_dx);
  } else {
    if constexpr (STAGED) gemm_nt_block<64, 64, EPI_RAW, false>(p.dw, smem, b - p.n_dx, gridDim.x - p.n_dx);
    else gemm_tn_block<64, 128, CONV != 0>(p.dw, smem, b - p.n_dx, gridDim.x - p.n_dx);
  }
}

template <bool RING, int EPI, int CONV, bool STAGED>
static int launch_cfg(const GemmStridedArgs& dx, const GemmTnArgs* tn, const GemmArgs* staged, int split_k, hipStream_t st) {
  using P = PairCfg<RING, EPI, CONV, STAGED>;
  // set once per process (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_pair<RING, EPI, CONV, STAGED>, hipFuncAttributeMaxDynamicSharedMemorySize, P::kLds);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  typename P::Args p;
  p.dx = dx;
  if constexpr (STAGED) p.dw = *staged; else p.dw = *tn;
  p.n_dx = dx.tiles_m * dx.tiles_n;
  const dim3 grid((unsigned)(p.n_dx + p.dw.tiles_m * p.dw.tiles_n * split_k));
  hipLaunchKernelGGL((k_pair<RING, EPI, CONV, STAGED>), grid, dim3(256), P::kLds, st, p);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

template <int CONV, bool STAGED>
static int launch_conv(const GemmStridedArgs& dx, bool ring, const GemmTnArgs* tn, const GemmArgs* staged, int split_k, hipStream_t st) {
  if (!ring) return launch_cfg<false, EPI_DX, CONV, STAGED>(dx, tn, staged, split_k, st);
  if (dx.x_dtype == EFQAT_F32) return launch_cfg<true, EPI_DXS, CONV, STAGED>(dx, tn, staged, split_k, st);
  return launch_cfg<true, EPI_DX, CONV, STAGED>(dx, tn, staged, split_k, st);
}

// The same for a channel-major dY, both products by k_gemm_dx8's loop on tiles of 64 x 128: 160 drawn bf16 layers 1.38 x as fast
// as on 128 x 128 tiles in two launches (12288 x 768 -> 768, k = 192, training step 68.5 -> 58.2 us).
struct PairCmArgs { GemmDx8Args dx, dw; int n_dx; };
__global__ __launch_bounds__(256, 3) void k_pair_cm(const PairCmArgs p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x;
  if (b < p.n_dx) gemm_dx8_block<64, 128, false, true>(p.dx, smem, b, p.n_dx);
  else gemm_dx8_block<64, 128, true>(p.dw, smem, b - p.n_dx, gridDim.x - p.n_dx);
}

int launch_pair_cm(const GemmDx8Args& dx, const GemmDx8Args& dw, int split_k, hipStream_t st) {
  constexpr int kLds = std::max(Dx8Cfg<64, 128, true>::lds_bytes<true>(), Dx8Cfg<64, 128>::lds_bytes<false>());
  // set once per process (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_pair_cm, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  PairCmArgs p{dx, dw, dx.g.tiles_m * dx.g.tiles_n};
  const dim3 grid((unsigned)(p.n_dx + dw.g.tiles_m * dw.g.tiles_n * split_k));
  hipLaunchKernelGGL(k_pair_cm, grid, dim3(256), kLds, st, p);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

int launch_pair(const GemmStridedArgs& dx, int conv, const GemmPlan& plan_dx, const GemmTnArgs* tn, const GemmArgs* staged,
                const GemmPlan& plan_dw, hipStream_t stream) {
  if (plan_dx.tile != 64 || plan_dw.tile != 64 || (tn && (tn->cv_cin > 0) != (conv != 0))) return EFQAT_ERR_BAD_SHAPE;
  const bool ring = plan_dx.ring;
  const int s = plan_dw.split_k;
  switch (conv) {
    case 0: return staged ? launch_conv<0, true>(dx, ring, tn, staged, s, stream) : launch_conv<0, false>(dx, ring, tn, staged, s, stream);
    case 1: return staged ? launch_conv<1, true>(dx, ring, tn, staged, s, stream) : launch_conv<1, false>(dx, ring, tn, staged, s, stream);
    default: return staged ? launch_conv<2, true>(dx, ring, tn, staged, s, stream) : launch_conv<2, false>(dx, ring, tn, staged, s, stream);
  }
}

}  // namespace efqat
