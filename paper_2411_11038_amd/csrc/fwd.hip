// Low-precision forward product of a quantized linear layer (Sec. 3.1: Y = X_q W_q^T computed on integer codes):
// the 8-bit codes go straight to the int8 matrix cores, the quantizer scales and the zero point are applied
// once per output element in the epilogue.
#include "common.hpp"

#include <algorithm>
#include <type_traits>

namespace efqat {

typedef int intx4_t __attribute__((ext_vector_type(4)));

// The product for few tokens (decoding, short batches): a pass over the weight codes, HBM bound.  No tile of 64 or more
// columns fills the chip at such sizes, and every byte of W is used once, so nothing is staged: a block takes 16 NT
// weight rows, its 8 wavefronts split K, every lane loads its 16-byte MFMA fragments straight from memory (16 rows x 64
// contiguous bytes per load, v_mfma_i32_16x16x64_i8) with a batch of loads in flight, and the int32 sums meet in LDS.
// sum_k w, which the zero point needs, is taken from the same fragments.  Rows of any length and alignment.
// One launch of 1 / 16 / 32 / 64 tokens, 4096 -> 11008 (45 MB of weight codes): 12 / 16 / 18 / 23 us; with 128 x 128
// tiles on 86 CUs after a pass for the row sums it was 40 - 42 us.  NT: see skinny_columns.
constexpr int kSkinnyWaves = 8;
template <int MT, int NT, int BATCH>
__global__ __launch_bounds__(64 * kSkinnyWaves) void k_fwd_skinny(
    const uint8_t* __restrict__ x, const int8_t* __restrict__ w, int T, int c_out, int K, const float* __restrict__ s_x,
    const float* __restrict__ z_x, const float* __restrict__ s_w, void* __restrict__ y, int y_dtype) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NW = kSkinnyWaves, COLS = 16 * NT;
  __shared__ int red[NW][MT * NT * 4][64];
  __shared__ int red_w[NW][COLS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kg = lane >> 4;
  const int n0 = (int)(blockIdx.y * gridDim.x + blockIdx.x) * COLS;
  if (n0 >= c_out) return;                              // the last row of the grid
  const int steps = (K + 63) / 64, per = (steps + NW - 1) / NW;
  const int s_end = (wave + 1) * per < steps ? (wave + 1) * per : steps;
  const uint8_t* xp[MT];
  const uint8_t* wp[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) xp[i] = x + (int64_t)(16 * i + l16 < T ? 16 * i + l16 : T - 1) * K;
#pragma unroll
  for (int j = 0; j < NT; ++j)
    wp[j] = (const uint8_t*)w + (int64_t)(n0 + 16 * j + l16 < c_out ? n0 + 16 * j + l16 : c_out - 1) * K;
  // 16 bytes of a row from column k on, zeros past the end of the row
  auto load16 = [&](const uint8_t* row, int k) {
    intx4_t v = {0, 0, 0, 0};
    if (k + 16 <= K) __builtin_memcpy(&v, row + k, 16);
    else if (k < K) {
#pragma unroll
      for (int b = 0; b < 15; ++b)
        if (k + b < K) v[b >> 2] |= (int)((unsigned)row[k + b] << (8 * (b & 3)));
    }
    return v;
  };
  intx4_t acc[MT][NT];
  int wsum[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    wsum[j] = 0;
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i][j] = (intx4_t){0, 0, 0, 0};
  }
  for (int s0 = wave * per; s0 < s_end; s0 += BATCH) {
    intx4_t a[BATCH][MT], b[BATCH][NT];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int k = s0 + u < s_end ? (s0 + u) * 64 + kg * 16 : K;   // past the slice: zeros
#pragma unroll
      for (int j = 0; j < NT; ++j) b[u][j] = load16(wp[j], k);
#pragma unroll
      for (int i = 0; i < MT; ++i) a[u][i] = load16(xp[i], k);
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
#pragma unroll
      for (int i = 0; i < MT; ++i) a[u][i] ^= (int)0x80808080;      // unsigned codes - 128
#pragma unroll
      for (int j = 0; j < NT; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) wsum[j] = __builtin_amdgcn_sdot4(b[u][j][q], 0x01010101, wsum[j], false);
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    wsum[j] += __shfl_xor(wsum[j], 16, kWave);
    wsum[j] += __shfl_xor(wsum[j], 32, kWave);
    if (kg == 0) red_w[wave][16 * j + l16] = wsum[j];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(i * NT + j) * 4 + r][lane] = acc[i][j][r];
  }
  __syncthreads();
  const float sx = s_x[0];
  const long long zc = 128 - (long long)rintf(z_x[0]);
  // accumulator layout: column lane & 15, rows 4 (lane / 16) + r
  for (int o = tid; o < MT * NT * 4 * 64; o += 64 * NW) {
    const int ln = o & 63, q = o >> 6, r = q & 3, j = (q >> 2) % NT, i = (q >> 2) / NT;
    const int col = 16 * j + (ln & 15), m = 16 * i + 4 * (ln >> 4) + r;
    long long sum = 0, ws = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) { sum += red[v][q][ln]; ws += red_w[v][col]; }
    if (m < T && n0 + col < c_out) {
      const float out = sx * s_w[n0 + col] * (float)(sum + zc * ws);
      const int64_t e = (int64_t)m * c_out + n0 + col;
      if (y_dtype == EFQAT_F32) ((float*)y)[e] = out;
      else ((bf16_t*)y)[e] = f32_to_bf16(out);
    }
  }
#endif
}

// out[r][0..ldo) = in[r][0..cols) followed by zeros (byte rows; makes K a multiple of 16 for ragged widths)
__global__ __launch_bounds__(256) void k_pad_rows_u8(const uint8_t* __restrict__ in, int64_t rows, int64_t cols,
                                                     uint8_t* __restrict__ out, int64_t ldo) {
  const int64_t total = rows * ldo;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / ldo, j = e - r * ldo;
    out[e] = j < cols ? in[r * cols + j] : (uint8_t)0;
  }
}

constexpr int64_t kSkinnyTokens = 64;

// Groups of 16 weight rows of a block (NT of k_fwd_skinny).  The fragments of the tokens are read from L2 by every block and cost as
// much of the loads as T rows of weights, so a wide block saves loads; but what takes the time is the busiest CU, and a block that
// leaves CUs idle, or a second one for a few of them, costs more.  In units of 16 bytes and column of C_in: the loads and the
// reductions of the busiest CU's blocks, and per group the latency that a wide block hides worse.  Under a floor the loads are free:
// several blocks of one group share a CU, and what is left of a wide block is its longer reduction.  Rows that are not aligned take
// more loads a fragment, each with its own wait: where they are short, wide blocks pay late.  Fitted to 1398 sizes (1 to 64 tokens,
// C_in 64 to 11008, C_out 4096 to 32768): 1.2 % from the fastest in the mean; 0.91 of the time of one group (four from 33 tokens and
// 8192 columns on), the first rule, and 0.98 of the second, the loads alone, which was up to 1.4 x as slow as the first where rows
// are short.  With up to 16 tokens three groups pay later than that (95 of 581 sizes of 5 to 16 tokens took them and lost 1 %): 0.950 of
// the time of one group, 5 % of the sizes 3 to 19 % slower than it.  NT = 1 / 2 / 3 / 4, us (* chosen):
//   tokens  C_in  -> C_out
//    1      4096     11008    11.9* / 14.7  / 14.1  / 16.0
//   16      4096      6000    11.6  / 10.6* / 13.2  / 15.7
//   16      4096     11008    17.1  / 18.3  / 15.8* / 17.7
//    9      1136     11251     4.7* /  5.3  /  5.2  /  5.8
//    5      2980      8309    10.1* / 12.0  / 11.6  / 12.7
//   16     11008      4096    16.1* / 23.5  / 30.4  / 35.9
//   16      8192     28672    70.4  / 66.2  / 66.6  / 60.1*
//   32      4096     11008    22.9  / 22.9  / 18.1* / 21.1
//   64      4096      6000    24.2  / 18.2* / 20.6  / 23.8
//   64      4096     11008    35.2  / 30.6  / 23.1* / 26.1
//   16        96     11008     3.7* /  4.2  /  4.7  /  4.4
//   16        96     28672     6.4  /  6.5  /  7.8  /  4.9*
//   64       256      4112     4.4* /  5.4  /  6.2  /  7.1
//   64       192      8192     4.5* /  5.1  /  6.0  /  6.8
//   16      1024      4112     4.5* /  4.8  /  5.8  /  5.8
//   32      1024     32768    18.2  / 15.6  / 14.6  / 12.8*
//   16       333     11008     6.7* /  8.0  /  8.8  /  9.4
//   20      1500      8192    10.2* / 10.9  / 13.3  / 15.6
//   16      3001     28672    58.2  / 51.0  / 53.5  / 43.9*
static int skinny_columns(int64_t T, int64_t c_in, int64_t c_out) {
  if (T <= 4) return 1;                                 // next to no loads to save
  if (c_in < 640 && c_out < 5120) return 1;             // a second block on some CUs runs beside the first
  if (c_in % 16 && c_in < 2048 &&
      (T <= 16 ? c_out < 16384 || c_in % 4 == 0 : T <= 32 ? c_in >= 1024 && c_out < 12288 : c_out < (c_in < 640 ? 8192 : 4608)))
    return 1;
  const double mt = T <= 16 ? 1.0 : T <= 32 ? 2.0 : 4.0, k = (double)c_in;
  int best = 1;
  double best_t = 0.0;
  for (int nt = 1; nt <= 4; ++nt) {
    const double rounds = (double)ceil_div(ceil_div(c_out, 16 * nt), 256);
    const double loads = rounds * (k * (nt + 1.2 * (double)T / 16.0) + 600.0 * mt * nt + 1000.0);
    const double t = (std::max(loads, 8000.0) + nt * (0.55 * k + 450.0 * mt)) * (nt == 3 && T <= 16 ? 1.08 : 1.0);
    if (nt == 1 || t < best_t) { best = nt; best_t = t; }
  }
  return best;
}

struct FwdPlan {
  int64_t ldk;       // C_in rounded up to 16
  bool pad;          // operands copied into zero-padded rows
  size_t b_xpad, b_wpad, total;
};

static FwdPlan make_fwd_plan(int64_t T, int64_t c_in, int64_t c_out) {
  FwdPlan p{};
  p.ldk = round_up(c_in, 16);
  p.pad = p.ldk != c_in && T > kSkinnyTokens;         // k_fwd_skinny reads rows of any length
  WsCarver cv(nullptr);
  p.b_xpad = p.pad ? (size_t)T * p.ldk : 0; cv.take(p.b_xpad);
  p.b_wpad = p.pad ? (size_t)c_out * p.ldk : 0; cv.take(p.b_wpad);
  p.total = cv.off ? cv.off : 256;                     // 0 bytes stand for a bad shape in the size query
  return p;
}

}  // namespace efqat

using namespace efqat;

extern "C" size_t efqat_linear_fwd_workspace_bytes(int64_t T, int64_t c_in, int64_t c_out) {
  if (T <= 0 || c_in <= 0 || c_out <= 0) return 0;
  return make_fwd_plan(T, c_in, c_out).total;
}

extern "C" int efqat_linear_fwd(const uint8_t* x_codes, const float* s_x, const float* z_x, const int8_t* w_codes,
                                const float* s_w, int64_t T, int64_t c_in, int64_t c_out, void* y, int y_dtype,
                                void* ws, size_t ws_bytes, void* stream) {
  if (T <= 0 || c_in <= 0 || c_out <= 0 || T > (1 << 30) || c_out > (1 << 30)) return EFQAT_ERR_BAD_SHAPE;
  // (128 - Z_x) * sum_k w must fit the exact 64-bit correction and the int32 accumulators: K <= 2^17 is ample
  if (c_in > (1 << 17)) return EFQAT_ERR_BAD_SHAPE;
  if (y_dtype != EFQAT_F32 && y_dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (!x_codes || !s_x || !z_x || !w_codes || !s_w || !y || !ws) return EFQAT_ERR_NULL_PTR;
  if (((uintptr_t)ws % 256) != 0 || ((uintptr_t)y % (y_dtype == EFQAT_F32 ? 4 : 2)) != 0) return EFQAT_ERR_ALIGNMENT;
  const FwdPlan p = make_fwd_plan(T, c_in, c_out);
  if (ws_bytes < p.total) return EFQAT_ERR_WORKSPACE;
  // the tile loads are 16-byte vectors when the codes are used in place
  if (p.ldk == c_in && ((((uintptr_t)x_codes) % 16) != 0 || (((uintptr_t)w_codes) % 16) != 0)) return EFQAT_ERR_ALIGNMENT;
  hipStream_t st = (hipStream_t)stream;
  if (T <= kSkinnyTokens) {
    ProfScope prof(PROF_FWD, st);
    // a grid dimension holds less than 2^32 work items
    auto grid = [&](int cols) {
      const int64_t blocks = ceil_div(c_out, cols), bx = std::min<int64_t>(blocks, 1 << 22);
      return dim3((unsigned)bx, (unsigned)ceil_div(blocks, bx));
    };
#define EFQAT_SKINNY(MT, NT, BATCH)                                                                                      \
  hipLaunchKernelGGL((k_fwd_skinny<MT, NT, BATCH>), grid(16 * NT), dim3(64 * kSkinnyWaves), 0, st, x_codes, w_codes, (int)T, \
                     (int)c_out, (int)c_in, s_x, z_x, s_w, y, y_dtype)
    // steps of 64 columns whose loads are in flight together: what the registers allow, more measured the same
#define EFQAT_SKINNY_NT(MT, B1, B2, B3, B4)                                                                              \
  switch (skinny_columns(T, c_in, c_out)) {                                                                                    \
    case 1: EFQAT_SKINNY(MT, 1, B1); break;                                                                              \
    case 2: EFQAT_SKINNY(MT, 2, B2); break;                                                                              \
    case 3: EFQAT_SKINNY(MT, 3, B3); break;                                                                              \
    default: EFQAT_SKINNY(MT, 4, B4);                                                                                    \
  }
    if (T <= 16) { EFQAT_SKINNY_NT(1, 4, 4, 4, 2) }
    else if (T <= 32) { EFQAT_SKINNY_NT(2, 4, 4, 2, 2) }
    else { EFQAT_SKINNY_NT(4, 2, 2, 1, 1) }
#undef EFQAT_SKINNY_NT
#undef EFQAT_SKINNY
    EFQAT_LAUNCH_CHECK();
    return EFQAT_OK;
  }
  WsCarver cv(ws);
  uint8_t* xpad = (uint8_t*)cv.take(p.b_xpad);
  uint8_t* wpad = (uint8_t*)cv.take(p.b_wpad);
  const uint8_t* xa = x_codes;
  const int8_t* wb = w_codes;
  if (p.pad) {
    auto grid = [](int64_t n) { int64_t b = ceil_div(n, 256); return (unsigned)(b > 16384 ? 16384 : b); };
    hipLaunchKernelGGL(k_pad_rows_u8, dim3(grid(T * p.ldk)), dim3(256), 0, st, x_codes, T, c_in, xpad, p.ldk);
    EFQAT_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_pad_rows_u8, dim3(grid(c_out * p.ldk)), dim3(256), 0, st, (const uint8_t*)w_codes, c_out,
                       c_in, wpad, p.ldk);
    EFQAT_LAUNCH_CHECK();
    xa = xpad; wb = (const int8_t*)wpad;
  }
  return launch_gemm_fwd_i8(xa, p.ldk, wb, p.ldk, T, c_out, p.ldk, s_x, z_x, s_w, y, y_dtype, st);
}

extern "C" int efqat_linear_fwd_plan(int64_t T, int64_t c_in, int64_t c_out, int32_t* plan) {
  if (!plan) return EFQAT_ERR_NULL_PTR;
  if (T <= 0 || c_in <= 0 || c_out <= 0 || T > (1 << 30) || c_out > (1 << 30) || c_in > (1 << 17)) return EFQAT_ERR_BAD_SHAPE;
  const bool few = T <= kSkinnyTokens;
  plan[EFQAT_FWD_PLAN_FEW_TOKENS] = few;
  plan[EFQAT_FWD_PLAN_COLUMNS] = few ? 16 * skinny_columns(T, c_in, c_out) : fwd_tile_columns(T, c_out, make_fwd_plan(T, c_in, c_out).ldk);
  return EFQAT_OK;
}
