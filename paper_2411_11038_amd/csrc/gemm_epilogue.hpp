// Pieces shared by the product kernels: the argument block and the fused epilogue of the dX product.
#pragma once
#include "common.hpp"

#include <type_traits>

namespace efqat {

typedef float floatx16_t __attribute__((ext_vector_type(16)));

// the dX epilogue for any matrix with x in bf16 (DX) or fp32 (DXS), and for whole bf16 tiles (DXF)
enum { EPI_RAW = 0, EPI_DX = 1, EPI_FWD = 2, EPI_DXF = 3, EPI_DXS = 4 };

struct GemmArgs {
  const void* A; int64_t lda; const int32_t* a_rows;   // lda / ldb / K in elements (bf16 or int8)
  const void* B; int64_t ldb;
  int M, N, K;
  int k_per_split;        // multiple of 64
  int tiles_m, tiles_n;
  int group_m;                        // row tiles per group of the tile order (the kernels of gemm_tn.hip)
  float* out;             // raw fp32 [split][M][N]
  // fused dX epilogue
  const uint8_t* x_codes; const uint32_t* x_clip; const void* x; int x_dtype;
  const float* s_x; const float* z_x; void* dx; int dx_dtype; float* partial;
  int epi_vec;            // 8-wide vector accesses allowed in the fused epilogue
  // forward epilogue (int8 product): y = s_x * s_w[n] * (acc + (128 - round(z_x)) * sum_k w[n][k])
  const float* s_w; void* y; int y_dtype;
  // implicit im2col of the A operand (dX product of a stride-1 convolution): row m is the input pixel (n, h, w),
  // K runs over (tap, c_out) with cv_spt 64-channel stages per tap, and the operand element is
  // dY[n][h + pad - kh][w + pad - kw][c_out] or zero outside the output image
  int cv_H, cv_W, cv_Ho, cv_Wo, cv_KW, cv_pad, cv_spt;
  uint64_t cv_m_spt, cv_m_kw;   // floor(2^32 / d) + 1 for d = cv_spt, cv_KW: n / d = (n * m) >> 32 for n * d < 2^32
};

// dX product of a convolution with a stride: the input pixels are sorted into stride x stride phases (h mod s, w mod s),
// and a row tile lies inside one phase, whose pixels all receive the same taps kh = kh0 + s a, kw = kw0 + s b from the
// output pixel (hi + dh0 - a, wi + dw0 - b), hi = h / s, wi = w / s.  K of a tile = the taps of its phase, so no products
// with the zeros between the strides are formed (3 of 4 at stride 2); a phase without taps has K = 0 and dX = 0.
struct ConvPhase { int tile0, tiles, rows, Hp, Wp, ph, pw, ntap, nkw, kh0, kw0, dh0, dw0; };
struct GemmStridedArgs : GemmArgs {
  int cv_stride, nphase;
  ConvPhase phase[kMaxConvStride * kMaxConvStride];    // most taps first: the longest tiles start first
};
template <int CONV> struct ConvArgs { typedef GemmArgs type; };
template <> struct ConvArgs<2> { typedef GemmStridedArgs type; };

struct GemmTnArgs {
  const bf16_t* A; int64_t lda;       // [K][lda], lda multiple of 8; columns >= a_cols are not read
  const uint8_t* B; int64_t ldb;      // [K][ldb], ldb multiple of 16
  int a_cols, b_cols;                 // readable widths (multiples of 8 / 16): beyond them the zero page is read
  const float* z_x;
  int M, N, K;
  int k_per_split;                    // multiple of 64
  int tiles_m, tiles_n;
  int group_m;                        // row tiles per group of the tile order (the kernels of gemm_tn.hip)
  float* out;                         // raw fp32 [split][M][N]
  // implicit im2col of the B operand (dW product of a convolution): row t is the output pixel (n, ho, wo), the
  // N-tile at n0 belongs to tap n0 / cv_cin = (kh, kw), and the operand is the code of input pixel
  // (n, ho*s + kh - p, wo*s + kw - p), channel n0 % cv_cin + column.  Outside the image the term is dropped by
  // zeroing the A row of that token in this block (a padded activation is 0 after de-quantisation, which need not
  // be a representable code).  cv_dn / cv_dh / cv_dw: how (n, ho, wo) moves when t advances by 64.
  int cv_H, cv_W, cv_Ho, cv_Wo, cv_KW, cv_stride, cv_pad, cv_cin, cv_dn, cv_dh, cv_dw;
};

struct GemmDx8Args {
  int a_cols;              // ATN: readable width of A (multiple of 8)
  GemmArgs g;              // dX: A = dY, B = weight codes, M = T, N = C_in, K = C_out, fused dX epilogue fields
                           // dW: A = dY channel-major with a_rows = idx, B = activation codes, M = k, N = C_in, K = T
  int b_cols;              // readable width of B (multiple of 16)
};

// ---- host side: argument blocks of the products (checked, nothing launched) and their launches
// dX: A, B, epilogue as launch_dx takes them; linear, stride-1 convolution (K = KH*KW*ldc), strided convolution
int dx_args_linear(GemmArgs* out, const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                   const GemmPlan& plan, const GemmEpilogueDx& epi);
int dx_args_conv(GemmArgs* out, const bf16_t* dy_tok, int64_t ldc, const bf16_t* wqT, int64_t ldb, int64_t M, int64_t N, int64_t K,
                 const ConvDxMap& cm, const GemmPlan& plan, const GemmEpilogueDx& epi);
int dx_args_strided(GemmStridedArgs* out, const bf16_t* dy_tok, int64_t ldc, const bf16_t* wqT, int64_t ldb, int64_t M, int64_t N,
                    const ConvDxStridedMap& cm, const GemmPlan& plan, const GemmEpilogueDx& epi);
// conv: 0 linear, 1 stride 1, 2 strided (only then the phases of `a` are read)
// beside: the dW product runs at the same time, on another stream
int launch_dx(const GemmStridedArgs& a, int conv, const GemmPlan& plan, bool beside, hipStream_t stream);
int launch_gemm_kk(const GemmArgs& a, int tile, bool beside, hipStream_t stream);
int kk_ring_stages(int tile, int64_t tiles, int64_t N, int64_t K, bool beside);   // LDS stages that it takes
int launch_gemm_kk_conv(const GemmArgs& a, int tile, hipStream_t stream);
int launch_gemm_kk_conv_strided(const GemmStridedArgs& a, int tile, hipStream_t stream);
// dW from token-major operands (k_gemm_tn), linear or convolution (cv_cin > 0), or from staged ones (k_gemm_nt)
int dw_args_tn(GemmTnArgs* out, const bf16_t* A, int64_t lda, int64_t a_cols, const uint8_t* B, int64_t ldb, int64_t b_cols,
               const float* z_x, int64_t M, int64_t N, int64_t K, const GemmPlan& plan, float* out_partial);
int dw_args_tn_conv(GemmTnArgs* out, const bf16_t* A, int64_t lda, int64_t a_cols, const uint8_t* x_codes, const ConvDwMap& cm,
                    const float* z_x, int64_t M, int64_t N, int64_t K, const GemmPlan& plan, float* out_partial);
int dw_args_staged(GemmArgs* out, const bf16_t* A, int64_t lda, const int32_t* a_rows, const bf16_t* B, int64_t ldb, int64_t M,
                   int64_t N, int64_t K, const GemmPlan& plan, float* out_partial);
int launch_gemm_tn(const GemmTnArgs& a, const GemmPlan& plan, hipStream_t stream);
int launch_gemm_nt_raw(const GemmArgs& a, const GemmPlan& plan, hipStream_t stream);
// channel-major dY: dX by k_gemm_dx8 from dY [C_out][lda] (lda >= M = T, T % 8 == 0) and the int8 weight codes, both with the
// contraction index as their row; dW from the rows idx of dY [C_out][lda] (lda >= K = T, K % 8 == 0) and the uint8 codes:
//   out[s][m][n] = sum over the K-slice s of dY[idx[m]][t] * (codes[t][n] - round(z_x)).  Tiles 256, 128 (dX also 128 x 256), 64 (64 x 128).
int dx_args_cm(GemmDx8Args* out, const bf16_t* dy_cm, int64_t lda, const int8_t* w_codes, int64_t ldb, const float* s_w, int64_t M,
               int64_t N, int64_t K, const GemmPlan& plan, const GemmEpilogueDx& epi);
int dw_args_rows(GemmDx8Args* out, const bf16_t* dy_cm, int64_t lda, const int32_t* idx, const uint8_t* x_codes, int64_t ldb,
                 const float* z_x, int64_t M, int64_t N, int64_t K, const GemmPlan& plan, float* out_partial);
int launch_gemm_dx8_cm(const GemmDx8Args& a, const GemmPlan& plan, hipStream_t stream);
int launch_gemm_dw_rows(const GemmDx8Args& a, const GemmPlan& plan, hipStream_t stream);
int launch_pair_cm(const GemmDx8Args& dx, const GemmDx8Args& dw, int split_k, hipStream_t stream);
// both products of one layer in one grid (pair.hip): tn or staged, the other one null
int launch_pair(const GemmStridedArgs& dx, int conv, const GemmPlan& plan_dx, const GemmTnArgs* tn, const GemmArgs* staged,
                const GemmPlan& plan_dw, hipStream_t stream);
// nothing left to decide in the dX epilogue: bf16 in and out, whole tiles, 32-bit element offsets, aligned pointers
inline bool dx_epilogue_fast(const GemmArgs& g, int bm, int bn) {
  return g.epi_vec && g.x_dtype == EFQAT_BF16 && g.dx_dtype == EFQAT_BF16 && (g.M % bm) == 0 && (g.N % bn) == 0 &&
         (int64_t)g.M * g.N <= (int64_t)INT32_MAX;
}

// phase and phase-local row tile / column tile of a block: each XCD gets a contiguous range of every phase's tiles
__device__ __forceinline__ void strided_tile(const GemmStridedArgs& g, int block, ConvPhase* ph, int* tm, int* tn) {
  int f = 0;
  while (f + 1 < g.nphase && block >= g.phase[f + 1].tile0 * g.tiles_n) ++f;
  *ph = g.phase[f];
  const int pid = xcd_contiguous_index(block - ph->tile0 * g.tiles_n, ph->tiles * g.tiles_n);
  *tm = pid / g.tiles_n;
  *tn = pid - *tm * g.tiles_n;
}
// (n * Ho * Wo) and (hi << 16 | wi) of phase-local row r; its input pixel
__device__ __forceinline__ int strided_pixel(const GemmStridedArgs& g, const ConvPhase& ph, int r, int* q0, int* hw) {
  const int per = ph.Hp * ph.Wp;
  const int n = r / per, rem = r - n * per;
  const int hi = rem / ph.Wp, wi = rem - hi * ph.Wp;
  *q0 = n * g.cv_Ho * g.cv_Wo;
  *hw = (hi << 16) | wi;
  return (n * g.cv_H + hi * g.cv_stride + ph.ph) * g.cv_W + wi * g.cv_stride + ph.pw;
}
// (a, b) of the phase's tap and the channel stage of K stage sidx
__device__ __forceinline__ void strided_stage(const GemmStridedArgs& g, const ConvPhase& ph, int sidx, int* a, int* b,
                                              int* cst) {
  const int t = (int)(((uint64_t)(uint32_t)sidx * g.cv_m_spt) >> 32);
  *cst = sidx - t * g.cv_spt;
  *a = t / ph.nkw;
  *b = t - *a * ph.nkw;
}

// Block barrier that orders LDS traffic only.  __syncthreads() also fences global memory, i.e. waits for every
// outstanding global load and store of the wavefront; between the staging writes and reads of an epilogue that
// would expose a memory round trip per barrier.  Global accesses keep their own dependency tracking.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Eight columns of one row in the dX epilogue.  a: the product; becomes dX.  xf, cw, mb: x, codes and mask bits (1 = in range).
// s1 += a gs with gs = in range ? (code - Z) - x / S : code - Z, term by term (in range |gs| <= 1/2); sd += a where clipped, and
// a - a where not: nothing, but undefined for an infinite or undefined a.
// What this costs is the number of operations, each of which takes four cycles of a SIMD that few wavefronts share.  Nearly all
// values are in range (a per-tensor scale clips some in 10^4 or none), so a chunk in which no lane of the wavefront has a clipped one
// leaves the mask and sd out: 5 operations an element, 12 with them.  The sums are the same bit for bit where every a is finite; where
// one is not, s1 is not either, and the epilogue adds the a - a of its rows behind the chunks (half an operation an element to keep
// the largest |a| for that cost the dX products 1 %).
// SKIP: off for wavefronts of one 32 x 32 accumulator (tiles of 64 x 64), up to four blocks of which share a CU and hide the operations,
// not the branch (37.3 us of both products of a convolution so, 37.7 with it); and in EpiDxAny for wavefronts of 256 rows (256 x 256 by
// k_gemm_dx8; 2376 x 352 -> 6000 34.1 us before, 37.1 with it, 35.1 so; 40 such layers 1.005 of the time before, 1.03 with it), whereas
// the straight-line epilogue of these tiles gains 3.5 %.  MASK: off for 128 x 128 tiles of k_gemm_dx8 that have a CU for themselves (see
// launch_gemm_dx8_cm).
template <bool SKIP>
__device__ __forceinline__ void epi_chunk(float (&a)[8], const float (&xf)[8], const uint2& cw, uint32_t mb, float z,
                                          float ninv_s, float& s1, float& sd) {
  auto code = [&](int t) { return (float)(((t < 4 ? cw.x : cw.y) >> (8 * (t & 3))) & 0xFFu) - z; };
  if (SKIP && __ballot((mb & 0xFFu) != 0xFFu) == 0ull) {
#pragma unroll
    for (int t = 0; t < 8; ++t) s1 = fmaf(a[t], fmaf(xf[t], ninv_s, code(t)), s1);
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool inr = (mb >> t) & 1u;
      const float q = code(t);
      const float gs = inr ? fmaf(xf[t], ninv_s, q) : q;
      s1 = fmaf(a[t], gs, s1);
      const float o = inr ? a[t] : 0.0f;
      sd += a[t] - o;
      a[t] = o;
    }
  }
}
// a product may have been infinite or undefined
__device__ __forceinline__ bool epi_undefined(float s1) { return __ballot(!(fabsf(s1) < __builtin_inff())) != 0ull; }
// the a - a of a chunk in range
__device__ __forceinline__ void epi_undefined_chunk(const float* a, uint32_t mb, float& sd) {
#pragma unroll 1
  for (int t = 0; t < 8; ++t)
    if ((mb >> t) & 1u) sd += a[t] - a[t];
}

// Fused epilogue of the dX product for a 256-thread block whose wavefront (wm, wn) holds the C::WM x C::WN
// sub-tile at (m0 + wm * C::WM, n0 + wn * C::WN) of an M x N output in C::TM x C::TN 32x32 MFMA accumulators.
//   dX = dX_q where the activation was not clipped (straight-through), 0 elsewhere; block partial sums of
//   dS_x = sum dX_q * (in range ? (code - Z) - x/S : code - Z) and dZ_x = sum dX_q * (in range ? 0 : -S).
// Any M, N, type and alignment of x (XT) and dX; EpiDxFast below is the case without edges.  The accumulators go to the
// wavefront's own part of LDS, GS slabs of 32 rows at a time, so that a lane then owns chunks of 8 consecutive columns of a
// row: LPR lanes share a row, a pass covers 64 / LPR rows.  Rows of any width and alignment are read and written in whole
// chunks (the hardware takes vector accesses at element alignment; a chunk that runs over the end of its row reads into the
// next one, the last ones of the matrix start earlier and are shifted), so every lane has one load of codes and one or two
// of x per chunk, and U passes of them are in flight: what bounds it is the chain of these loads behind the main loop, a
// lone block has nothing else to run meanwhile.  On 128 x 128 fp32 tiles of a lone block it takes 3.6 us, 4.2 us where the
// width is odd; with branches on type and edge around each element and one 32-row slab of loads in flight (one column a
// lane for odd widths) it took 6.5 and 12.6 us.
template <class C, typename XT, bool MAP = false, bool MASK = false>
struct EpiDxAny {
  static constexpr int PITCH = C::WN + 8;            // floats; 4*PITCH = 32 (mod 64) banks
  static constexpr int CPR = C::WN / 8;              // 8-column chunks per row
  static constexpr int LPR = (CPR % 8 == 0) ? 8 : 4;
  static_assert(CPR % LPR == 0, "chunks per row");
  static constexpr int KC = CPR / LPR, RP = 64 / LPR, NP = 32 / RP * KC;   // NP: passes per slab
  // half of them where that lets two blocks of 128 x 256 share a CU
  static constexpr int GS = C::TM * 512 * PITCH <= (C::BM == 128 && C::BN == 256 ? 80 : 160) * 1024 ? C::TM : C::TM / 2;
  static constexpr int LDS = GS * 512 * PITCH;       // 4 wavefronts x 32 rows x 4 bytes
  static_assert(LDS <= 160 * 1024 && C::TM % GS == 0, "staging");
  static constexpr int U = KC == 1 ? (NP * GS < 4 ? NP * GS : 4) : 2 * KC;
  static_assert(NP * GS % U == 0 && U % KC == 0, "passes");
  static constexpr int XW = sizeof(XT) / 2;          // 16-byte words of x per chunk
  static constexpr bool kSkip = !MASK && C::TM * C::TN > 1 && C::WM < 256;   // see epi_chunk
  struct Inputs { uint2 cw; uint4 xa[XW]; uint32_t mb; };
  Inputs in[U];
  int row_b, col_b, first_row, rows;                 // rows: of this wavefront's sub-tile that lie inside the matrix
  const int* rowmap;
  int64_t last;                                      // the last element a chunk may start at

  // matrix row of the lane's row in the pass from row r of the sub-tile on, -1 past the end; first column of its chunk
  template <bool EDGE>
  __device__ __forceinline__ int row_of(int r) const {
    if (EDGE && r + (int)(threadIdx.x & 63) / LPR >= rows) return -1;
    if constexpr (MAP) return rowmap[row_b + r];
    else return first_row + row_b + r;
  }
  __device__ __forceinline__ int col_of(int u) const { return col_b + 8 * LPR * (u % KC); }
  // EDGE: the tile reaches over the end of the rows or columns.  Chunks outside the matrix stand at its first row or column.
  template <bool EDGE>
  __device__ __forceinline__ int64_t elem(const GemmArgs& g, int row, int col) const {
    if constexpr (EDGE) return (int64_t)(row < 0 ? 0 : row) * g.N + (col < g.N ? col : 0);
    else return (int64_t)row * g.N + col;
  }
  // requests the inputs of the pass from row r of the sub-tile on, set u
  template <bool EDGE>
  __device__ __forceinline__ void fetch(const GemmArgs& g, int r, int u) {
    const int row = row_of<EDGE>(r), col = col_of(u);
    const int64_t e = elem<EDGE>(g, row, col), a = EDGE && e > last ? last : e;
    const int64_t wpr = (g.N + 31) >> 5;
    in[u].mb = g.x_clip[(EDGE && row < 0 ? 0 : row) * wpr + ((EDGE && col >= g.N ? 0 : col) >> 5)];
    if (!EDGE || last >= 0) {
      __builtin_memcpy(&in[u].cw, g.x_codes + a, 8);
      __builtin_memcpy(in[u].xa, (const XT*)g.x + a, 8 * sizeof(XT));
    } else {                                         // a matrix of fewer than 8 elements, from its last one downwards
#pragma unroll 1
      for (int64_t t = (int64_t)g.M * g.N - 1; t >= e; --t) {
        in[u].cw.y = (in[u].cw.y << 8) | (in[u].cw.x >> 24); in[u].cw.x = (in[u].cw.x << 8) | g.x_codes[t];
        uint4& x0 = in[u].xa[0];
        uint4& x1 = in[u].xa[XW - 1];
        if constexpr (XW == 1) {
          x0.w = (x0.w << 16) | (x0.z >> 16); x0.z = (x0.z << 16) | (x0.y >> 16); x0.y = (x0.y << 16) | (x0.x >> 16);
          x0.x = (x0.x << 16) | ((const bf16_t*)g.x)[t];
        } else {
          x1.w = x1.z; x1.z = x1.y; x1.y = x1.x; x1.x = x0.w; x0.w = x0.z; x0.z = x0.y; x0.y = x0.x;
          x0.x = ((const uint32_t*)g.x)[t];
        }
      }
    }
  }
  // Addresses of this wavefront's sub-tile, and the requests for its first U passes.  A kernel may call this
  // before its main loop has ended, provided none of its own global -> LDS copies is still outstanding or issued later
  // (a wavefront's loads complete in order).  m_end: end of the rows that m0 counts in.  map: the matrix row of every row
  // of the tile (MAP).
  template <bool EDGE>
  __device__ __forceinline__ void prefetch_tile(const GemmArgs& g, int m0, int n0, int wm, int wn, int m_end,
                                                const int* map) {
    const int lane = threadIdx.x & 63;
    row_b = wm * C::WM + lane / LPR;
    col_b = n0 + wn * C::WN + (lane % LPR) * 8;
    first_row = m0; rowmap = map;
    rows = n0 + wn * C::WN >= g.N ? 0 : m_end - m0 - wm * C::WM < C::WM ? m_end - m0 - wm * C::WM : C::WM;
    last = (int64_t)g.M * g.N - 8;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (EDGE) in[u] = Inputs{};
      if (!EDGE || RP * (u / KC) < rows) fetch<EDGE>(g, RP * (u / KC), u);
    }
  }
  __device__ __forceinline__ void prefetch(const GemmArgs& g, int m0, int n0, int wm, int wn, int m_end, bool edge,
                                           const int* map) {
    if (edge) prefetch_tile<true>(g, m0, n0, wm, wn, m_end, map);
    else prefetch_tile<false>(g, m0, n0, wm, wn, m_end, map);
  }
  // The epilogue proper; prefetch() has been called with the same `edge`.  smem: LDS bytes, no longer used by the main loop
  // (the caller has synchronised).  part_idx: the tile's slot in g.partial.
  __device__ __forceinline__ void run(const GemmArgs& g, floatx16_t (&acc)[C::TM][C::TN], char* smem, bool edge,
                                      int part_idx) {
    float s1 = 0.0f, sd = 0.0f;
    if (edge) sum_tile<true>(g, acc, smem, s1, sd);
    else sum_tile<false>(g, acc, smem, s1, sd);
    finish(g, smem, s1, sd, part_idx);
  }
  __device__ __forceinline__ void finish(const GemmArgs& g, char* smem, float s1, float sd, int part_idx) {
    const float ps = wave_sum(s1);
    const float pz = wave_sum(sd);
    lds_barrier();                                   // staging area is dead: reuse for the block sum
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float* red = reinterpret_cast<float*>(smem);
    if ((threadIdx.x & 63) == 0) { red[2 * wave] = ps; red[2 * wave + 1] = pz; }
    lds_barrier();
    if (threadIdx.x == 0) {
      g.partial[2 * part_idx] = (red[0] + red[2]) + (red[4] + red[6]);
      g.partial[2 * part_idx + 1] = -g.s_x[0] * ((red[1] + red[3]) + (red[5] + red[7]));
    }
  }
  // the tile's dX; s1, sd: this lane's share of the sums (see epi_chunk)
  template <bool EDGE>
  __device__ __forceinline__ void sum_tile(const GemmArgs& g, floatx16_t (&acc)[C::TM][C::TN], char* smem, float& s1,
                                           float& sd) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    float* stage = reinterpret_cast<float*>(smem) + wave * GS * 32 * PITCH;
    const float z = rintf(g.z_x[0]);
    const float ninv_s = -1.0f / g.s_x[0];
    const float* st_b = stage + (lane / LPR) * PITCH + (lane % LPR) * 8;
#pragma unroll
    for (int i0 = 0; i0 < C::TM; i0 += GS) {
      // a wavefront reads what it wrote itself: no barrier, its own LDS accesses have to be done
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < GS; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            stage[(32 * i + 8 * (r >> 2) + 4 * fh + (r & 3)) * PITCH + j * 32 + fr] = acc[i0 + i][j][r];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll 1
      for (int r0 = 0; r0 < 32 * GS; r0 += RP * U / KC) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int r = r0 + RP * (u / KC);
          if (EDGE && 32 * i0 + r >= rows) continue;
          const float4 n0v = *reinterpret_cast<const float4*>(st_b + r * PITCH + 8 * LPR * (u % KC));
          const float4 n1v = *reinterpret_cast<const float4*>(st_b + r * PITCH + 8 * LPR * (u % KC) + 4);
          float a[8] = {n0v.x, n0v.y, n0v.z, n0v.w, n1v.x, n1v.y, n1v.z, n1v.w};
          Inputs q8 = in[u];
          if (32 * i0 + r + RP * U / KC < (EDGE ? rows : C::WM)) fetch<EDGE>(g, 32 * i0 + r + RP * U / KC, u);
          const int row = row_of<EDGE>(32 * i0 + r), col = col_of(u);
          const int64_t e = elem<EDGE>(g, row, col);
          uint32_t mb = q8.mb >> (col & 31);          // mask bits of the chunk
          int n = 8;                                  // its elements inside the matrix
          if constexpr (EDGE) {
            n = row < 0 ? 0 : g.N - col;
            mb &= n >= 8 ? 0xFFu : n > 0 ? (1u << n) - 1u : 0u;
#pragma unroll
            for (int t = 0; t < 8; ++t) a[t] = t < n ? a[t] : 0.0f;
            if (last >= 0)
#pragma unroll 1
              for (int64_t sh = e - last; sh > 0; --sh) {  // the chunk was read from `last` on: move it down
                q8.cw.x = (q8.cw.x >> 8) | (q8.cw.y << 24); q8.cw.y >>= 8;
                uint4& x0 = q8.xa[0];
                uint4& x1 = q8.xa[XW - 1];
                if constexpr (XW == 1) {
                  x0.x = (x0.x >> 16) | (x0.y << 16); x0.y = (x0.y >> 16) | (x0.z << 16);
                  x0.z = (x0.z >> 16) | (x0.w << 16); x0.w >>= 16;
                } else {
                  x0.x = x0.y; x0.y = x0.z; x0.z = x0.w; x0.w = x1.x; x1.x = x1.y; x1.y = x1.z; x1.z = x1.w;
                }
              }
          }
          const uint32_t xw[8] = {q8.xa[0].x,      q8.xa[0].y,      q8.xa[0].z,      q8.xa[0].w,
                                  q8.xa[XW - 1].x, q8.xa[XW - 1].y, q8.xa[XW - 1].z, q8.xa[XW - 1].w};
          float xf[8];
#pragma unroll
          for (int t = 0; t < 8; ++t)
            xf[t] = XW == 2 ? __uint_as_float(xw[t])
                            : __uint_as_float((t & 1) ? xw[t >> 1] & 0xFFFF0000u : xw[t >> 1] << 16);
          epi_chunk<kSkip>(a, xf, q8.cw, mb, z, ninv_s, s1, sd);
          if (g.dx_dtype == EFQAT_F32) {
            float* d = (float*)g.dx + e;
            if (!EDGE || n >= 8) __builtin_memcpy(d, a, 32);
            else
#pragma unroll 1
              for (int t = 0; t < n; ++t) {
                d[t] = a[0];
#pragma unroll
                for (int v = 0; v < 6; ++v) a[v] = a[v + 1];
              }
          } else {
            bf16_t* d = (bf16_t*)g.dx + e;
            uint32_t w[4] = {pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]),
                             pack_bf16x2(a[6], a[7])};
            if (!EDGE || n >= 8) __builtin_memcpy(d, w, 16);
            else
#pragma unroll 1
              for (int t = 0; t < n; ++t) {
                d[t] = (bf16_t)w[0];
#pragma unroll
                for (int v = 0; v < 3; ++v) w[v] = (w[v] >> 16) | (w[v + 1] << 16);
                w[3] >>= 16;
              }
          }
          __builtin_amdgcn_sched_barrier(0);          // keeps the passes from piling up in registers
        }
      }
      if (kSkip && epi_undefined(s1)) {
#pragma unroll 1
        for (int r = 0; r < 32 * GS; r += RP)
#pragma unroll 1
          for (int k = 0; k < KC; ++k) {
            const int row = 32 * i0 + r < rows ? row_of<EDGE>(32 * i0 + r) : -1, col = col_of(k), n = g.N - col;
            if (row < 0 || n <= 0) continue;
            const uint32_t mb = g.x_clip[row * (((int64_t)g.N + 31) >> 5) + (col >> 5)] >> (col & 31);
            epi_undefined_chunk(st_b + r * PITCH + 8 * LPR * k, n < 8 ? mb & ((1u << n) - 1u) : mb, sd);
          }
      }
    }
  }
};

// ... with the type of x decided at run time, all requests behind the main loop
template <class C, bool MAP = false, bool MASK = false>
__device__ __forceinline__ void epilogue_dx(const GemmArgs& g, floatx16_t (&acc)[C::TM][C::TN], char* smem, int m0,
                                            int n0, int wm, int wn, int m_end, int part_idx,
                                            const int* rowmap = nullptr) {
  const bool edge = m0 + C::BM > m_end || n0 + C::BN > g.N;
  auto all = [&](auto e, auto edgec) {
    constexpr bool EDGE = decltype(edgec)::value;
    e.template prefetch_tile<EDGE>(g, m0, n0, wm, wn, m_end, rowmap);
    float s1 = 0.0f, sd = 0.0f;
    e.template sum_tile<EDGE>(g, acc, smem, s1, sd);
    e.finish(g, smem, s1, sd, part_idx);
  };
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;
  if (g.x_dtype == EFQAT_F32) {
    if (edge) all(EpiDxAny<C, float, MAP, MASK>(), Yes{});
    else all(EpiDxAny<C, float, MAP, MASK>(), No{});
  } else {
    if (edge) all(EpiDxAny<C, bf16_t, MAP, MASK>(), Yes{});
    else all(EpiDxAny<C, bf16_t, MAP, MASK>(), No{});
  }
}

// The same epilogue for the case that needs no decision about type or edge at run time: bf16 x, bf16 dX, every tile of the block grid
// entirely inside the matrix (M % BM == 0, N % BN == 0), M * N < 2^31 so that element offsets fit 32 bits, 16-byte aligned x / dX and
// 8-byte aligned codes.  LPR lanes share a row of the 32 x WN slab, each taking KC of its 8-column chunks (chunk LPR k + lane % LPR), so
// a pass covers 64 / LPR rows with all 64 lanes busy and every address is one per-lane base plus compile-time offsets.  The only branch
// of a pass is epi_chunk's, one for the wavefront; the LDS reads of the next pass are issued before the arithmetic of the current one,
// and the global inputs of a group of rows (KC passes) of the next slab are requested as soon as this slab's group is done (one
// register set, a whole slab of prefetch distance).  With a single resident block per CU the predicated formulation above runs at
// about half this speed.
// ALL: the inputs of the whole sub-tile are held in registers, requested a group of rows at a time while the main loop runs
// (k_gemm_kk); else one slab of them.
template <class C, bool ALL = false>
struct EpiDxFast {
  static constexpr int PITCH = C::WN + 8;            // floats; 4*PITCH = 32 (mod 64) banks
  static constexpr int CPR = C::WN / 8;              // 8-column chunks per row
  static constexpr int LPR = (CPR % 8 == 0) ? 8 : 4;
  static_assert(CPR % LPR == 0, "chunks per row");
  static constexpr int KC = CPR / LPR, RP = 64 / LPR, HP = 32 / RP, NP = HP * KC;
  static constexpr int GROUPS = HP * C::TM;          // groups of RP rows in the sub-tile
  // a group's loads: the mask words of a row, KC chunks of codes and of x.  No two of them have neighbouring addresses, so they
  // stay as many instructions as they are here: the waits of a kernel that requests them in its main loop count them.
  static constexpr int LOADS = LPR == 4 ? 1 + 2 * KC : 3 * KC;
  struct Inputs { uint32_t mb[KC]; uint2 cw[KC]; uint4 xa[KC]; };
  Inputs in[ALL ? GROUPS : HP];
  uint32_t un, uwpr, row_b, col_b;
  const uint8_t* codes; const uint32_t* clip; const bf16_t* xp; bf16_t* dxp;
  float s, zp;

  // element offset of chunk k of the lane's row in group h of slab i
  __device__ __forceinline__ uint32_t elem(int i, int h, int k) const {
    return (row_b + (uint32_t)(32 * i + RP * h)) * un + col_b + (uint32_t)(8 * LPR * k);
  }
  __device__ __forceinline__ Inputs& inputs(int i, int h) { return in[ALL ? HP * i + h : h]; }
  __device__ __forceinline__ void fetch(int i, int h) {
    const uint32_t row = row_b + (uint32_t)(32 * i + RP * h);
    Inputs& q = inputs(i, h);
    // shifted at use: no arithmetic on a value still in flight
    if constexpr (LPR == 4) {                         // chunks 32 columns apart: consecutive words
      __builtin_memcpy(q.mb, clip + row * uwpr + (col_b >> 5), 4 * KC);
    } else {
#pragma unroll
      for (int k = 0; k < KC; ++k) q.mb[k] = clip[row * uwpr + (col_b >> 5) + (uint32_t)(LPR / 4 * k)];
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const uint32_t e = elem(i, h, k);
      q.cw[k] = *reinterpret_cast<const uint2*>(codes + e);
      q.xa[k] = *reinterpret_cast<const uint4*>(xp + e);
    }
  }
  // Addresses of this wavefront's sub-tile, scale and zero point.
  __device__ __forceinline__ void begin(const GemmArgs& g, int m0, int n0, int wm, int wn) {
    const int lane = threadIdx.x & 63;
    un = (uint32_t)g.N; uwpr = (uint32_t)((g.N + 31) >> 5);
    row_b = (uint32_t)(m0 + wm * C::WM) + (uint32_t)lane / LPR;
    col_b = (uint32_t)(n0 + wn * C::WN) + ((uint32_t)lane % LPR) * 8u;
    codes = g.x_codes; clip = g.x_clip; xp = (const bf16_t*)g.x; dxp = (bf16_t*)g.dx;
    s = g.s_x[0]; zp = g.z_x[0];
  }
  // Requests the inputs of the first slab (ALL: of all slabs).  A kernel may call
  // this before its main loop has ended, provided none of its own global -> LDS copies is still outstanding or
  // issued later (a wavefront's loads complete in order).
  __device__ __forceinline__ void prefetch() {
#pragma unroll
    for (int h = 0; h < (ALL ? GROUPS : HP); ++h) fetch(h / HP, h % HP);
  }
  // The epilogue proper; prefetch() has been called.  smem: at least 4 * 32 * (C::WN + 8) floats, no longer used by
  // the main loop (the caller has synchronised).  part_idx: the tile's slot in g.partial.
  __device__ __forceinline__ void run(const GemmArgs& g, floatx16_t (&acc)[C::TM][C::TN], char* smem, int part_idx) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    float* stage = reinterpret_cast<float*>(smem) + wave * 32 * PITCH;
    const float z = rintf(zp);
    const float ninv_s = -1.0f / s;
    const float* st_b = stage + ((uint32_t)lane / LPR) * PITCH + ((uint32_t)lane % LPR) * 8;
    auto lds_chunk = [&](int p, float4& a0, float4& a1) {   // pass p: chunk p % KC of group p / KC
      a0 = *reinterpret_cast<const float4*>(st_b + RP * (p / KC) * PITCH + 8 * LPR * (p % KC));
      a1 = *reinterpret_cast<const float4*>(st_b + RP * (p / KC) * PITCH + 8 * LPR * (p % KC) + 4);
    };
    const uint32_t msh = col_b & 31u;                 // a pass moves by a multiple of 32 columns
    static_assert((8 * LPR) % 32 == 0, "mask bit offset is the same in every pass");
    float s1 = 0.0f, sd = 0.0f;
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
      // a wavefront reads what it wrote itself: no barrier, its own LDS accesses have to be done
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int j = 0; j < C::TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          stage[(8 * (r >> 2) + 4 * fh + (r & 3)) * PITCH + j * 32 + fr] = acc[i][j][r];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      float4 n0v, n1v;
      lds_chunk(0, n0v, n1v);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        float a[8] = {n0v.x, n0v.y, n0v.z, n0v.w, n1v.x, n1v.y, n1v.z, n1v.w};
        if (p + 1 < NP) lds_chunk(p + 1, n0v, n1v);
        const int h = p / KC, k = p % KC;
        const Inputs& q8 = inputs(i, h);
        const uint32_t xw[4] = {q8.xa[k].x, q8.xa[k].y, q8.xa[k].z, q8.xa[k].w};
        const uint2 cw = q8.cw[k];
        const uint32_t mb = q8.mb[k] >> msh;
        float xf[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) xf[t] = __uint_as_float((t & 1) ? xw[t >> 1] & 0xFFFF0000u : xw[t >> 1] << 16);
        epi_chunk<true>(a, xf, cw, mb, z, ninv_s, s1, sd);
        *reinterpret_cast<uint4*>(dxp + elem(i, h, k)) =
            make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]),
                       pack_bf16x2(a[6], a[7]));
        if (!ALL && k == KC - 1 && i + 1 < C::TM) fetch(i + 1, h);   // this group's registers are free
        __builtin_amdgcn_sched_barrier(0);            // keeps the passes from piling up in registers
      }
      if (epi_undefined(s1)) {
#pragma unroll 1
        for (int h = 0; h < HP; ++h)
#pragma unroll 1
          for (int k = 0; k < KC; ++k) {
            const uint32_t row = row_b + (uint32_t)(32 * i + RP * h), col = col_b + (uint32_t)(8 * LPR * k);
            epi_undefined_chunk(st_b + RP * h * PITCH + 8 * LPR * k, clip[row * uwpr + (col >> 5)] >> msh, sd);
          }
      }
    }
    const float ps = wave_sum(s1);
    const float pz = wave_sum(sd);
    lds_barrier();                                   // staging area is dead: reuse for the block sum
    float* red = reinterpret_cast<float*>(smem);
    if (lane == 0) { red[2 * wave] = ps; red[2 * wave + 1] = pz; }
    lds_barrier();
    if (tid == 0) {
      g.partial[2 * part_idx] = (red[0] + red[2]) + (red[4] + red[6]);
      g.partial[2 * part_idx + 1] = -s * ((red[1] + red[3]) + (red[5] + red[7]));
    }
  }
};

template <class C>
__device__ __forceinline__ void epilogue_dx_fast(const GemmArgs& g, floatx16_t (&acc)[C::TM][C::TN], char* smem,
                                                 int m0, int n0, int wm, int wn, int part_idx) {
  EpiDxFast<C> e;
  e.begin(g, m0, n0, wm, wn);
  e.prefetch();
  e.run(g, acc, smem, part_idx);
}

}  // namespace efqat
