// Products that read an int8 or uint8 operand as it lies: launches of k_gemm_tn (gemm_tn.hpp), and k_gemm_dx8.
#include "gemm_dx8.hpp"
#include "gemm_tn.hpp"

namespace efqat {

// Row tiles per group of the tile order (a group's tiles are walked row-fastest, so the 32 tiles that run on an XCD at
// one time are group_m rows by 32 / group_m columns of tiles and share that many operand panels in its L2).  Measured
// on the LLM-sized products: 2 or 3 for 256 x 256 tiles (dX -1.6 %, dW -3 % against 8); no difference for the
// smaller tiles, which stay at 8.
static int tile_group_m(int tile) { return tile == 256 ? 2 : 8; }

template <int BM, int BN, bool CONV = false>
static int launch_tn_cfg(const GemmTnArgs& a, int split_k, hipStream_t st) {
  using C = TnCfg<BM, BN>;
  // set once per process (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_gemm_tn<BM, BN, CONV>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  const dim3 grid((unsigned)(a.tiles_m * a.tiles_n * split_k));
  {
    ProfScope prof(PROF_DW, st);
    hipLaunchKernelGGL((k_gemm_tn<BM, BN, CONV>), grid, dim3(256), C::LDS_BYTES, st, a);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

int dw_args_tn(GemmTnArgs* out, const bf16_t* A, int64_t lda, int64_t a_cols, const uint8_t* B, int64_t ldb, int64_t b_cols,
               const float* z_x, int64_t M, int64_t N, int64_t K, const GemmPlan& plan, float* out_partial) {
  if (M <= 0 || N <= 0 || K <= 0 || (lda % 8) || (ldb % 16) || (a_cols % 8) || (b_cols % 16)) return EFQAT_ERR_BAD_SHAPE;
  if (lda >= (1 << 24) || ldb >= (1 << 24)) return EFQAT_ERR_BAD_SHAPE;   // 32-bit per-stage pointer strides
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || a_cols > lda || b_cols > ldb) return EFQAT_ERR_BAD_SHAPE;
  if (((uintptr_t)A % 16) || ((uintptr_t)B % 16)) return EFQAT_ERR_ALIGNMENT;
  GemmTnArgs a{};
  a.A = A; a.lda = lda; a.B = B; a.ldb = ldb; a.a_cols = (int)a_cols; a.b_cols = (int)b_cols;
  a.z_x = z_x;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(ceil_div(K, 64), plan.split_k) * 64);
  a.tiles_m = plan.tiles_m; a.tiles_n = plan.tiles_n; a.group_m = tile_group_m(plan.tile);
  a.out = out_partial;
  *out = a;
  return EFQAT_OK;
}

int dw_args_tn_conv(GemmTnArgs* out, const bf16_t* A, int64_t lda, int64_t a_cols, const uint8_t* x_codes, const ConvDwMap& cm,
                    const float* z_x, int64_t M, int64_t N, int64_t K, const GemmPlan& plan, float* out_partial) {
  if (M <= 0 || N <= 0 || K <= 0 || (lda % 8) || (a_cols % 8) || a_cols > lda || lda >= (1 << 24)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || (plan.tile != 128 && plan.tile != 64) || (cm.c_in % 128) != 0)
    return EFQAT_ERR_BAD_SHAPE;
  if (((uintptr_t)A % 16) || ((uintptr_t)x_codes % 16)) return EFQAT_ERR_ALIGNMENT;
  GemmTnArgs a{};
  a.A = A; a.lda = lda; a.B = x_codes; a.ldb = 0; a.a_cols = (int)a_cols; a.b_cols = INT32_MAX;
  a.z_x = z_x;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(ceil_div(K, 64), plan.split_k) * 64);
  a.tiles_m = plan.tiles_m; a.tiles_n = plan.tiles_n; a.group_m = tile_group_m(plan.tile);
  a.out = out_partial;
  a.cv_H = cm.H; a.cv_W = cm.W; a.cv_Ho = cm.Ho; a.cv_Wo = cm.Wo; a.cv_KW = cm.KW; a.cv_stride = cm.stride;
  a.cv_pad = cm.pad; a.cv_cin = cm.c_in;
  const int hw = cm.Ho * cm.Wo, rem = 64 % hw;
  a.cv_dn = 64 / hw; a.cv_dh = rem / cm.Wo; a.cv_dw = rem % cm.Wo;
  *out = a;
  return EFQAT_OK;
}

int launch_gemm_tn(const GemmTnArgs& a, const GemmPlan& plan, hipStream_t stream) {
  if (a.cv_cin) return plan.tile == 64 ? launch_tn_cfg<64, 128, true>(a, plan.split_k, stream) : launch_tn_cfg<128, 128, true>(a, plan.split_k, stream);
  switch (plan.tile) {
    case 256: return launch_tn_cfg<256, 256>(a, plan.split_k, stream);
    case 128: return launch_tn_cfg<128, 128>(a, plan.split_k, stream);
    case 64: return launch_tn_cfg<64, 128>(a, plan.split_k, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}


template <int BM, int BN, bool DW = false, bool ATN = false, bool FAST = false, bool MASK = false>
static int launch_dx8_cfg(const GemmDx8Args& a, int split_k, hipStream_t st) {
  constexpr int kLds = Dx8Cfg<BM, BN, ATN>::template lds_bytes<!DW && !FAST>();
  // set once per process (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_gemm_dx8<BM, BN, DW, ATN, FAST, MASK>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  const dim3 grid((unsigned)(a.g.tiles_m * a.g.tiles_n * split_k));
  {
    ProfScope prof(DW ? PROF_DW : PROF_DX, st);
    hipLaunchKernelGGL((k_gemm_dx8<BM, BN, DW, ATN, FAST, MASK>), grid, dim3(256), kLds, st, a);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

int dx_args_cm(GemmDx8Args* out, const bf16_t* dy_cm, int64_t lda, const int8_t* w_codes, int64_t ldb, const float* s_w, int64_t M,
               int64_t N, int64_t K, const GemmPlan& plan, const GemmEpilogueDx& epi) {
  if (M <= 0 || N <= 0 || K <= 0 || (M % 8) || (lda % 8) || (ldb % 16) || (N % 16)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || ldb >= (1 << 24) || lda >= (1 << 24)) return EFQAT_ERR_BAD_SHAPE;
  if (((uintptr_t)dy_cm % 16) || ((uintptr_t)w_codes % 16) || ((uintptr_t)s_w % 4))
    return EFQAT_ERR_ALIGNMENT;
  GemmDx8Args a{};
  a.g.A = dy_cm; a.g.lda = lda; a.g.B = w_codes; a.g.ldb = ldb;
  a.g.M = (int)M; a.g.N = (int)N; a.g.K = (int)K;
  a.g.s_w = s_w;
  a.g.x_codes = epi.x_codes; a.g.x_clip = epi.x_clip; a.g.x = epi.x; a.g.x_dtype = epi.x_dtype;
  a.g.s_x = epi.s_x; a.g.z_x = epi.z_x; a.g.dx = epi.dx; a.g.dx_dtype = epi.dx_dtype; a.g.partial = epi.partial;
  a.g.epi_vec = gemm_epilogue_vec_ok(epi, N) ? 1 : 0;
  a.g.tiles_m = plan.tiles_m; a.g.tiles_n = plan.tiles_n; a.g.group_m = tile_group_m(plan.tile);
  a.a_cols = (int)M; a.b_cols = (int)N;
  *out = a;
  return EFQAT_OK;
}

int launch_gemm_dx8_cm(const GemmDx8Args& a, const GemmPlan& plan, hipStream_t stream) {
  if (plan.wide)
    return dx_epilogue_fast(a.g, 128, 256) ? launch_dx8_cfg<128, 256, false, true, true>(a, 1, stream)
                                           : launch_dx8_cfg<128, 256, false, true>(a, 1, stream);
  // a block on a CU: the branch around the mask costs it 1 % (80 sizes; 1600 x 797 -> 1584 18.6 -> 19.4 us, without it 18.5), which two of
  // them hide: more tiles gain 1 % (60 sizes) by it
  const bool alone = (int64_t)plan.tiles_m * plan.tiles_n <= 256;
  switch (plan.tile) {
    case 64: return launch_dx8_cfg<64, 128, false, true>(a, 1, stream);
    case 256: return dx_epilogue_fast(a.g, 256, 256) ? launch_dx8_cfg<256, 256, false, true, true>(a, 1, stream)
                                                      : launch_dx8_cfg<256, 256, false, true>(a, 1, stream);
    case 128:
      if (dx_epilogue_fast(a.g, 128, 128)) return launch_dx8_cfg<128, 128, false, true, true>(a, 1, stream);
      return alone ? launch_dx8_cfg<128, 128, false, true, false, true>(a, 1, stream) : launch_dx8_cfg<128, 128, false, true>(a, 1, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}

int dw_args_rows(GemmDx8Args* out, const bf16_t* dy_cm, int64_t lda, const int32_t* idx, const uint8_t* x_codes, int64_t ldb,
                 const float* z_x, int64_t M, int64_t N, int64_t K, const GemmPlan& plan, float* out_partial) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 8) || (lda % 8) || (ldb % 16) || (N % 16)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || ldb >= (1 << 24)) return EFQAT_ERR_BAD_SHAPE;
  if (((uintptr_t)dy_cm % 16) || ((uintptr_t)x_codes % 16)) return EFQAT_ERR_ALIGNMENT;
  GemmDx8Args a{};
  a.g.A = dy_cm; a.g.lda = lda; a.g.a_rows = idx; a.g.B = x_codes; a.g.ldb = ldb;
  a.g.M = (int)M; a.g.N = (int)N; a.g.K = (int)K;
  a.g.k_per_split = (int)(ceil_div(ceil_div(K, 64), plan.split_k) * 64);
  a.g.z_x = z_x; a.g.out = out_partial;
  a.g.tiles_m = plan.tiles_m; a.g.tiles_n = plan.tiles_n; a.g.group_m = tile_group_m(plan.tile);
  a.b_cols = (int)N;
  *out = a;
  return EFQAT_OK;
}

int launch_gemm_dw_rows(const GemmDx8Args& a, const GemmPlan& plan, hipStream_t stream) {
  switch (plan.tile) {
    case 64: return launch_dx8_cfg<64, 128, true>(a, plan.split_k, stream);
    case 256: return launch_dx8_cfg<256, 256, true>(a, plan.split_k, stream);
    case 128: return launch_dx8_cfg<128, 128, true>(a, plan.split_k, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}

int launch_gemm_dx8(const bf16_t* dy, int64_t lda, const int8_t* w_codes, int64_t ldb, const float* s_w, int64_t M,
                    int64_t N, int64_t K, int tile, const GemmEpilogueDx& epi, hipStream_t stream) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 8) || (lda % 8) || (ldb % 16) || (N % 16)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || ldb >= (1 << 24)) return EFQAT_ERR_BAD_SHAPE;
  if (((uintptr_t)dy % 16) || ((uintptr_t)w_codes % 16) || ((uintptr_t)s_w % 4))
    return EFQAT_ERR_ALIGNMENT;
  GemmDx8Args a{};
  a.g.A = dy; a.g.lda = lda; a.g.B = w_codes; a.g.ldb = ldb;
  a.g.M = (int)M; a.g.N = (int)N; a.g.K = (int)K;
  a.g.s_w = s_w;
  a.g.x_codes = epi.x_codes; a.g.x_clip = epi.x_clip; a.g.x = epi.x; a.g.x_dtype = epi.x_dtype;
  a.g.s_x = epi.s_x; a.g.z_x = epi.z_x; a.g.dx = epi.dx; a.g.dx_dtype = epi.dx_dtype; a.g.partial = epi.partial;
  a.g.epi_vec = gemm_epilogue_vec_ok(epi, N) ? 1 : 0;
  a.g.tiles_m = (int)ceil_div(M, tile); a.g.tiles_n = (int)ceil_div(N, tile); a.g.group_m = tile_group_m(tile);
  a.b_cols = (int)N;
  switch (tile) {
    case 256: return dx_epilogue_fast(a.g, 256, 256) ? launch_dx8_cfg<256, 256, false, false, true>(a, 1, stream)
                                                      : launch_dx8_cfg<256, 256>(a, 1, stream);
    case 128: return dx_epilogue_fast(a.g, 128, 128) ? launch_dx8_cfg<128, 128, false, false, true>(a, 1, stream)
                                                      : launch_dx8_cfg<128, 128>(a, 1, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}

}  // namespace efqat
