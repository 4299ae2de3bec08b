// Launches of the dX kernels with the ring of LDS stages (gemm_kk.hpp).
#include "gemm_kk.hpp"

namespace efqat {

// LDS stages of the ring.  64 x 64 tiles of a linear layer that have a CU for themselves take eight, 128 KB, where the contraction is
// long; before, the deeper prologue and drain of a block cost more than they hide.  Rows that are no whole number of 128-byte lines
// are bound by their copies, each of which touches two lines; there eight stages lose on whole tiles of C_in.  Backward call
// without selected channels, three / eight, us:
//   512 x 512  -> 768    12.6 / 13.5     512 x 1792 -> 768    17.6 / 17.8     512 x 2048 -> 768    18.2 / 17.7
//   64 x 4096  -> 1024   26.0 / 23.4     200 x 8000 -> 100    38.0 / 32.5    1000 x 8192 -> 777    56.7 / 42.8
//   512 x 3000 -> 1024   29.6 / 30.8     512 x 8008 -> 1024   71.9 / 72.6    1000 x 6008 -> 777    48.1 / 43.2
//   64 x 4816  -> 1024   38.1 / 39.0     256 x 8008 -> 200    45.6 / 47.1    2000 x 4104 -> 333    35.5 / 31.8
// With the dW product on a second stream its blocks need room beside them:
//   153 x 4608 -> 640, k = 2304, 30 tiles, 41.6 / 39.9; 512 x 4608 -> 1024, k = 2304, 128 tiles, 47.7 / 50.1
//   512 x 8192 -> 1024, k = 4096, 128 tiles, 64.0 / 58.8; 1024 x 8000 -> 1024, k = 2000, 256 tiles, 64.0 / 72.1
//   153 x 8008 -> 640, k = 8008, 66.6 / 67.3
// Convolutions form an address for every copy, and eight stages of that code cost them 1 to 19 % at 1 to 196 tiles and 9 to 400 K stages.
// Four stages of the 128 x 128 tile gain nothing.
constexpr int kKkDeep = 8;
int kk_ring_stages(int tile, int64_t tiles, int64_t N, int64_t K, bool beside) {
  if (tile != 64 || tiles > 256) return 3;
  const int64_t stages = ceil_div(K, 64);
  if (beside) return K % 64 == 0 && ((tiles <= 64 && stages >= 64) || (tiles <= 128 && stages >= 112)) ? kKkDeep : 3;
  if (K % 64) return N % 64 && tiles >= 64 && stages >= 64 ? kKkDeep : 3;
  return stages >= 32 ? kKkDeep : 3;
}

// Should the straight-line epilogue's inputs be requested during the first stages?  On 192 x 192 tiles, whose epilogues are the longest,
// and where every CU has one: blocks that follow one another win back what the requests cost the stages, a full round of long
// contractions does where the caches do not hold the buffers, as in a training step.  Backward call without selected channels,
// without / with, us, buffers not in the caches | in them:
//   6144 x 768  -> 3072 (2 rounds)  53.7 / 49.9 | 46.3 / 47.3     12288 x 1536 -> 768  (256 tiles)  40.5 / 38.8 | 37.0 / 38.2
//  12288 x 1536 -> 1536 (2)         76.2 / 72.8 | 68.2 / 67.3      3072 x 3072 -> 3072 (256)        67.5 / 64.9 | 62.1 / 63.2
//  12288 x 3072 -> 3072 (4)        226   / 225  | 220  / 219       3072 x 768  -> 3072 (256)        27.4 / 27.7 | 27.8 / 29.2
//  12288 x 256  -> 1536 (2)         39.6 / 40.2 | 33.8 / 37.1      4608 x 3072 -> 1536 (192)        50.6 / 52.7 | 51.2 / 52.7
// With 128 x 128 tiles it costs 2 %.
static bool kk_inputs_ahead(const GemmArgs& a, int tile) {
  const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
  return tile == 192 && tiles >= 256 && a.K / 64 >= (tiles > 256 ? kKkAheadStages : 24);
}

template <int BM, int BN, int EPI, int CONV = 0, int NST = 3, bool AHEAD = false>
static int launch_kk_cfg(const typename ConvArgs<CONV>::type& a, hipStream_t st) {
  using C = KkCfg<BM, BN, NST>;
  // set once per process (initialisation of a function-local static is thread-safe)
  constexpr int kLds = C::template lds_bytes<EPI>() + (CONV == 2 ? C::BM * (int)sizeof(int) : 0);
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_gemm_kk<BM, BN, EPI, CONV, NST, AHEAD>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  const dim3 grid((unsigned)(a.tiles_m * a.tiles_n));
  {
    ProfScope prof(PROF_DX, st);
    hipLaunchKernelGGL((k_gemm_kk<BM, BN, EPI, CONV, NST, AHEAD>), grid, dim3(256), kLds, st, a);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

int launch_gemm_kk(const GemmArgs& a, int tile, bool beside, hipStream_t stream) {
  // bf16 in and out, whole tiles, 32-bit element offsets: nothing to decide at run time, the straight-line epilogue
  const bool fast = dx_epilogue_fast(a, tile, tile);
  const bool deep = kk_ring_stages(tile, (int64_t)a.tiles_m * a.tiles_n, a.N, a.K, beside) == kKkDeep;
  switch (tile) {
    case 192:
      if (fast && kk_inputs_ahead(a, tile)) return launch_kk_cfg<192, 192, EPI_DXF, 0, 3, true>(a, stream);
      if (fast) return launch_kk_cfg<192, 192, EPI_DXF>(a, stream);
      return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<192, 192, EPI_DXS>(a, stream) : launch_kk_cfg<192, 192, EPI_DX>(a, stream);
    case 128:
      if (fast) return launch_kk_cfg<128, 128, EPI_DXF>(a, stream);
      return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<128, 128, EPI_DXS>(a, stream) : launch_kk_cfg<128, 128, EPI_DX>(a, stream);
    case 64:
      if (deep) return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<64, 64, EPI_DXS, 0, kKkDeep>(a, stream) : launch_kk_cfg<64, 64, EPI_DX, 0, kKkDeep>(a, stream);
      return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<64, 64, EPI_DXS>(a, stream) : launch_kk_cfg<64, 64, EPI_DX>(a, stream);
    default:
      return EFQAT_ERR_BAD_SHAPE;
  }
}

// dX product of a stride-1 convolution; `a` by dx_args_conv
int launch_gemm_kk_conv(const GemmArgs& a, int tile, hipStream_t stream) {
  if (tile == 64)
    return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<64, 64, EPI_DXS, 1>(a, stream) : launch_kk_cfg<64, 64, EPI_DX, 1>(a, stream);
  if (dx_epilogue_fast(a, 128, 128)) return launch_kk_cfg<128, 128, EPI_DXF, 1>(a, stream);
  return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<128, 128, EPI_DXS, 1>(a, stream) : launch_kk_cfg<128, 128, EPI_DX, 1>(a, stream);
}

int launch_gemm_kk_conv_strided(const GemmStridedArgs& a, int tile, hipStream_t stream) {
  if (tile == 64)
    return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<64, 64, EPI_DXS, 2>(a, stream) : launch_kk_cfg<64, 64, EPI_DX, 2>(a, stream);
  return a.x_dtype == EFQAT_F32 ? launch_kk_cfg<128, 128, EPI_DXS, 2>(a, stream) : launch_kk_cfg<128, 128, EPI_DX, 2>(a, stream);
}

}  // namespace efqat
