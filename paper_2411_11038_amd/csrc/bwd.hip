// EfQAT backward of one quantized layer (Alg. 1 backward step, Eq. 5): operand preparation,
// the two MFMA contractions, and the fused / second-pass epilogues that apply the straight-through
// clip masks and reduce the quantizer-parameter gradients.
#include "gemm_epilogue.hpp"

#include <algorithm>
#include <type_traits>

namespace efqat {

// ------------------------------------------------------------------------------------------------
// element readers
template <typename T> __device__ __forceinline__ float rd(const T* p, int64_t i);
template <> __device__ __forceinline__ float rd<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ float rd<bf16_t>(const bf16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
template <> __device__ __forceinline__ float rd<int8_t>(const int8_t* p, int64_t i) { return (float)p[i]; }
template <> __device__ __forceinline__ float rd<uint8_t>(const uint8_t* p, int64_t i) { return (float)p[i]; }

// Tiled transpose with conversion to bf16:
//   out[j][i] = bf16( (in[i][cm(j)] - sub) * rs(i) ),  i < R, j < Cn;  out[j][i] = 0 for R <= i < i_pad.
//   cm(j) = colmap ? colmap[j] : j     (gather of selected channels when dY is token major)
//   rs(i) = rowscale ? rowscale[i] : 1 (per-output-channel weight scale)
//   sub   = subz ? round(subz[0]) : 0  (activation zero point)
// `out` row j starts at out + j*ldo + out_off (ldo = pitch in elements).
template <typename T> struct Vec4 { };
template <> struct Vec4<float> { typedef float4 type; };
template <> struct Vec4<bf16_t> { typedef uint2 type; };
template <> struct Vec4<int8_t> { typedef uint32_t type; };
template <> struct Vec4<uint8_t> { typedef uint32_t type; };
__device__ __forceinline__ void unpack4(const float4& v, float (&o)[4]) { o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
__device__ __forceinline__ void unpack4(const uint2& v, float (&o)[4]) {
  o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
  o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
}
template <typename T>
__device__ __forceinline__ void unpack4b(uint32_t v, float (&o)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) o[t] = (float)(T)((v >> (8 * t)) & 0xFFu);
}

struct ConvGeom {
  int N, H, W, c_in, c_out, KH, KW, stride, pad, Ho, Wo;
};

// Extras of the transposing copy, all zero / off for a plain 2-D transpose.  blockIdx.z = tap of a convolution:
//   weights:      tap t reads in + t * z_in and writes at column offset out_off + t * z_out;
//   activations:  (conv = 1) source row i is an output pixel (n, ho, wo); tap t reads the input pixel
//                 (n, ho*s + kh - p, wo*s + kw - p), or contributes 0 when that lies outside the image (the
//                 padding is zero in the de-quantised domain), and writes output rows t * z_orow + j.
struct TransposeExtra {
  int64_t z_in, z_out, z_orow;
  int conv;
  ConvGeom g;
};

typedef bf16_t TransposeTile[64][66];                  // tile[i][j] of a block

// tile (bx, by) of tap `tap`; colmap without rowscale and subz
template <typename T>
__device__ __forceinline__ void transpose_block(TransposeTile& tile, int bx, int by, int tap, const T* __restrict__ in,
                                                int64_t ld_in, int64_t R, int64_t Cn, const int32_t* __restrict__ colmap,
                                                const float* __restrict__ rowscale, const float* __restrict__ subz,
                                                bf16_t* __restrict__ out, int64_t ldo, int64_t out_off, int64_t i_pad,
                                                const TransposeExtra& ex) {
  const int64_t i0 = (int64_t)bx * 64, j0 = (int64_t)by * 64;
  const float sub = subz ? rintf(subz[0]) : 0.0f;
  in += (int64_t)tap * ex.z_in;
  out += (int64_t)tap * ex.z_out + (int64_t)tap * ex.z_orow * ldo;
  const int tap_h = ex.conv ? tap / ex.g.KW : 0, tap_w = ex.conv ? tap - tap_h * ex.g.KW : 0;
  // source row of logical row i, or -1: contributes zeros
  auto src_row = [&](int64_t i) -> int64_t {
    if (i >= R) return -1;
    if (!ex.conv) return i;
    const ConvGeom& g = ex.g;                         // pixel numbers are below 2^30 (conv_geom): 32-bit divisions.  64-bit
    // ones also made k_prep spill; 64 x 34 x 34, 232 -> 16 channels, 3 x 3, all selected, fp32 / bf16: backward call 336 / 316 us,
    // with them 387 / 366
    const uint32_t r = (uint32_t)i / (uint32_t)g.Wo, n = r / (uint32_t)g.Ho;
    const int wo = (int)((uint32_t)i - r * (uint32_t)g.Wo), ho = (int)(r - n * (uint32_t)g.Ho);
    const int h = ho * g.stride + tap_h - g.pad, w = wo * g.stride + tap_w - g.pad;
    if (h < 0 || h >= g.H || w < 0 || w >= g.W) return -1;
    return ((int64_t)n * g.H + h) * g.W + w;
  };
  if (!colmap) {
    // dense source, 4 consecutive columns per lane: one load of 4 to 16 bytes at any alignment, but for the chunk that ends a row
    const int jq = (threadIdx.x & 15) * 4, ib = threadIdx.x >> 4;
    const int64_t left = Cn - j0 - jq;
    float v[4][4], sb[4], rs[4];
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int64_t i = i0 + ib + 16 * rr, si = src_row(i);
      sb[rr] = si >= 0 ? sub : 0.0f;                   // padding is zero beside an infinite Z_x or S_w too
      rs[rr] = rowscale && i < R ? rowscale[i] : 1.0f;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[rr][t] = 0.0f;
      if (si >= 0 && left >= 4) {
        typename Vec4<T>::type raw;
        __builtin_memcpy(&raw, in + si * ld_in + j0 + jq, 4 * sizeof(T));
        if constexpr (sizeof(T) == 1) unpack4b<T>(raw, v[rr]); else unpack4(raw, v[rr]);
      } else if (si >= 0) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
          if (t < left) v[rr][t] = rd<T>(in, si * ld_in + j0 + jq + t);
      }
    }
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int li = ib + 16 * rr;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[rr][t] = (v[rr][t] - sb[rr]) * rs[rr];
      *reinterpret_cast<uint32_t*>(&tile[li][jq]) = pack_bf16x2(v[rr][0], v[rr][1]);
      *reinterpret_cast<uint32_t*>(&tile[li][jq + 2]) = pack_bf16x2(v[rr][2], v[rr][3]);
    }
  } else {
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t j = j0 + tx;
    const int64_t jc = j < Cn ? (int64_t)colmap[j] : 0;
    float v[16];                                       // all in flight
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) {
      const int64_t si = src_row(i0 + ty + 4 * rr);
      v[rr] = si >= 0 && j < Cn ? rd<T>(in, si * ld_in + jc) : 0.0f;
    }
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) tile[ty + 4 * rr][tx] = f32_to_bf16(v[rr]);
  }
  __syncthreads();
  // out[j][i0 + 8a .. 8a+7]: one 16-byte store per lane, 8 lanes cover the 128 bytes of one output row
  const int a8 = (threadIdx.x & 7) * 8, jb = threadIdx.x >> 3;
#pragma unroll
  for (int ww = 0; ww < 2; ++ww) {
    const int lj = jb + 32 * ww;
    const int64_t jo = j0 + lj, io = i0 + a8;
    if (jo < Cn && io < i_pad) {
      uint32_t w[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) w[t] = (uint32_t)tile[a8 + 2 * t][lj] | ((uint32_t)tile[a8 + 2 * t + 1][lj] << 16);
      *reinterpret_cast<uint4*>(out + jo * ldo + out_off + io) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// A row in segments, one wavefront each: of 2048 columns, or of 512 where that leaves few wavefronts (the selected rows of
// a channel-major dY are few and long).  2 of 40 channels, 25088 tokens, fp32: backward call 73 us, with a wavefront per
// row 124 us; 2049 x 1001, 1001 rows: segments of 512 are 1 us slower than of 2048.
struct RowCut { uint32_t segs, cols; };

// Row-wise cast/copy to bf16 with zero-padded pitch: out[m][j] = bf16(in[rm(m)][j]), j < Cn; 0 up to ldo (a multiple of
// 8), a chunk of 8 a lane: one or two 16-byte loads at any alignment, but for the chunk that ends a long row.  flat == 1: no
// padding and no row map, i.e. one run of chunks; flat = 2 .. 64, a power of two: that many lanes to a row; 0: a wavefront
// per row segment.  block b of nb.
template <typename T>
__device__ __forceinline__ void rows_block(int64_t b, int64_t nb, const T* __restrict__ in, int64_t ld_in, int64_t R,
                                           int64_t Cn, const int32_t* __restrict__ rowmap, bf16_t* __restrict__ out,
                                           int64_t ldo, int flat, const RowCut& cut) {
  auto load8 = [](const T* src, uint32_t (&w)[4]) {
    if constexpr (sizeof(T) == 4) {
      float f[8];
      __builtin_memcpy(f, src, 32);
#pragma unroll
      for (int t = 0; t < 4; ++t) w[t] = pack_bf16x2(f[2 * t], f[2 * t + 1]);
    } else {
      __builtin_memcpy(w, src, 16);
    }
  };
  auto store8 = [](bf16_t* dst, const uint32_t (&w)[4]) { *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]); };
  auto chunk = [&](const T* src, bf16_t* dst) {
    uint32_t w[4];
    load8(src, w);
    store8(dst, w);
  };
  auto chunk_end = [](const T* src, int64_t n, bf16_t* dst) {   // of n < 8 values, then zeros
    float f[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) f[t] = t < n ? rd<T>(src, t) : 0.0f;
    *reinterpret_cast<uint4*>(dst) =
        make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
  };
  // columns j .. j + 7 of a row; its end is its last eight values moved down, so that no lane reads value by value while its neighbours
  // wait.  Long rows, few of whose chunks end one, are the faster without (2049 x 1001 fp32: 0.1 us of 8.3).
  auto chunk_of_row = [&](const T* row, int64_t j, bf16_t* dst) {
    const int64_t over = j + 8 - Cn;
    if (Cn < 8) return chunk_end(row + j, Cn - j, dst);
    uint32_t w[4];
    load8(row + (over > 0 ? Cn - 8 : j), w);
    if (over > 0) {
      if (over & 4) { w[0] = w[2]; w[1] = w[3]; w[2] = w[3] = 0; }
      if (over & 2) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = 0; }
      if (over & 1) { w[0] = w[0] >> 16 | w[1] << 16; w[1] = w[1] >> 16 | w[2] << 16; w[2] = w[2] >> 16 | w[3] << 16; w[3] >>= 16; }
      if (over >= 8) w[0] = w[1] = w[2] = w[3] = 0;
    }
    store8(dst, w);
  };
  if (flat > 1) {
    const int lg = 31 - __builtin_clz(flat), sub = threadIdx.x & (flat - 1), per = 256 >> lg;
    for (int64_t m = b * per + (threadIdx.x >> lg); m < R; m += nb * per)
      for (int64_t j = 8 * sub; j < ldo; j += 8 * flat) chunk_of_row(in + m * ld_in, j, out + m * ldo + j);
    return;
  }
  if (flat) {
    const int64_t n8 = R * (ldo >> 3);
    for (int64_t e = b * 256 + threadIdx.x; e < n8; e += nb * 256) chunk(in + e * 8, out + e * 8);
    return;
  }
  const int lane = threadIdx.x & 63;
  for (int64_t u = b * 4 + (threadIdx.x >> 6); u < R * cut.segs; u += nb * 4) {
    // several segments a row: fewer than 2^32 in all (each is 512 or more elements in memory)
    const int64_t m = cut.segs == 1 ? u : (int64_t)((uint32_t)u / cut.segs), s0 = (u - m * cut.segs) * cut.cols;
    const int64_t s1 = s0 + cut.cols < ldo ? s0 + cut.cols : ldo;
    const T* src = in + (rowmap ? (int64_t)rowmap[m] : m) * ld_in;
#pragma unroll 4
    for (int64_t j = s0 + 8 * lane; j < s1; j += 512) {
      if (j + 8 <= Cn) chunk(src + j, out + m * ldo + j);
      else chunk_end(src + j, Cn - j, out + m * ldo + j);
    }
  }
}

// Compaction of the selected output channels of a token-major dY (the channel extraction step of Alg. 1, done
// once per call):  out[t][m] = bf16(dY[t][idx[m]]), m < k;  0 for k <= m < kp.
// A lane owns two neighbouring compacted channels (their source columns stay in registers); a wavefront thus
// reads 128 selected channels of one token - a span of a few cache lines, since idx ascends - and writes 256
// contiguous bytes.  The four wavefronts of a block take every fourth token row of the block's row range.
constexpr int kGatherRows = 32;                       // token rows per block
template <typename T>
__device__ __forceinline__ void gather_block(int bx, int by, int nby, const T* __restrict__ dy, int64_t ld, int64_t rows,
                                             const int32_t* __restrict__ idx, int64_t k, bf16_t* __restrict__ out,
                                             int64_t kp) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t m0 = 2 * ((int64_t)bx * 64 + lane);
  if (m0 >= kp) return;
  const int64_t c0 = m0 < k ? (int64_t)idx[m0] : -1, c1 = m0 + 1 < k ? (int64_t)idx[m0 + 1] : -1;
  for (int64_t t0 = (int64_t)by * kGatherRows; t0 < rows; t0 += (int64_t)nby * kGatherRows) {
    float a[kGatherRows / 4], b[kGatherRows / 4];
#pragma unroll
    for (int r = 0; r < kGatherRows / 4; ++r) {
      const int64_t t = t0 + wave + 4 * r;
      a[r] = (c0 >= 0 && t < rows) ? rd<T>(dy, t * ld + c0) : 0.0f;
      b[r] = (c1 >= 0 && t < rows) ? rd<T>(dy, t * ld + c1) : 0.0f;
    }
#pragma unroll
    for (int r = 0; r < kGatherRows / 4; ++r) {
      const int64_t t = t0 + wave + 4 * r;
      if (t < rows) *reinterpret_cast<uint32_t*>(out + t * kp + m0) = pack_bf16x2(a[r], b[r]);
    }
  }
}
template <typename T>
__global__ __launch_bounds__(256) void k_gather_cols(const T* __restrict__ dy, int64_t ld, int64_t rows,
                                                     const int32_t* __restrict__ idx, int64_t k,
                                                     bf16_t* __restrict__ out, int64_t kp) {
  gather_block<T>(blockIdx.x, blockIdx.y, gridDim.y, dy, ld, rows, idx, k, out, kp);
}

// Everything that has to be laid out ahead of the two products, in one launch: the compaction of the selected dY columns,
// the bf16 copy of a token-major dY that cannot be used in place, the bf16 W_q^T, and for the shapes that the products
// cannot read as they lie (ragged or few input channels, fp32 or unaligned channel-major dY) the transposed codes and
// the selected rows of dY.  They do not depend on each other, and each alone is at most some microseconds that end with
// the chip draining (about 4.5 us a launch, whatever it does).  2049 x 777 -> 1001, fp32: copies of
// 12.9, 9.0 and 9.2 us in three launches, training step 107.8 us; in one launch 91.6 us.
// The blocks of the parts follow each other; a part that is not needed has no blocks.
struct PrepArgs {
  const void* dy; int64_t c_out, t_out, ldc;
  const int32_t* idx; int64_t k; bf16_t* sel; int64_t kp;          // compaction
  bf16_t* dyn; int rows_flat;                                       // copy of a token-major dY
  RowCut rows_cut, sel_cut;                                         // of that copy, and of the selected rows
  int64_t c_in, w_ld, w_ldo;                                        // W_q^T
  const int8_t* w_codes; const float* s_w; bf16_t* wqT;
  TransposeExtra w_ex;
  uint32_t* zero_page;                                              // optional: the 256 zero bytes a made operand ends in
  const uint8_t* x_codes; const float* z_x; bf16_t* xcT;            // (codes - Z_x)^T
  int64_t ldt;
  TransposeExtra x_ex;
  int chan;                                                         // dY is channel major; transposed to dyn
  uint32_t gather_x, w_x, w_y, x_x, x_y, sel_x, dyn_x;             // blocks along the first axes of a part
  uint32_t n_gather, n_rows, n_w, n_x, n_sel, n_dyn;
};
template <typename T>
__global__ __launch_bounds__(256) void k_prep(const PrepArgs p) {
  __shared__ TransposeTile tile;
  const T* dy = (const T*)p.dy;
  uint32_t b = blockIdx.x + blockIdx.y * gridDim.x;
  if (b < p.n_gather) {
    gather_block<T>(b % p.gather_x, b / p.gather_x, p.n_gather / p.gather_x, dy, p.c_out, p.t_out, p.idx, p.k, p.sel, p.kp);
    return;
  }
  b -= p.n_gather;
  if (b < p.n_rows) {
    rows_block<T>(b, p.n_rows, dy, p.c_out, p.t_out, p.c_out, nullptr, p.dyn, p.ldc, p.rows_flat, p.rows_cut);
    return;
  }
  b -= p.n_rows;
  if (b < p.n_w) {
    if (p.zero_page && b == 0 && threadIdx.x < 64) p.zero_page[threadIdx.x] = 0u;
    // wqT[ci][tap ldc + co] = S_w[co] code[co][tap][ci]
    transpose_block<int8_t>(tile, b % p.w_x, (b / p.w_x) % p.w_y, b / (p.w_x * p.w_y), p.w_codes, p.w_ld, p.c_out, p.c_in,
                            nullptr, p.s_w, nullptr, p.wqT, p.w_ldo, 0, p.ldc, p.w_ex);
    return;
  }
  b -= p.n_w;
  if (b < p.n_x) {                                     // xcT[(tap, ci)][t] = code - Z_x of the input pixel
    transpose_block<uint8_t>(tile, b % p.x_x, (b / p.x_x) % p.x_y, b / (p.x_x * p.x_y), p.x_codes, p.c_in, p.t_out, p.c_in,
                             nullptr, nullptr, p.z_x, p.xcT, p.ldt, 0, p.ldt, p.x_ex);
    return;
  }
  b -= p.n_x;
  const TransposeExtra none{};
  if (b < p.n_sel) {                                   // sel[m][t] = dY of channel idx[m]
    if (p.chan) rows_block<T>(b, p.n_sel, dy, p.t_out, p.k, p.t_out, p.idx, p.sel, p.ldt, 0, p.sel_cut);
    else
      transpose_block<T>(tile, b % p.sel_x, b / p.sel_x, 0, dy, p.c_out, p.t_out, p.k, p.idx, nullptr, nullptr, p.sel,
                         p.ldt, 0, p.ldt, none);
    return;
  }
  b -= p.n_sel;
  if (b < p.n_dyn)                                     // channel-major [c_out][t_out] -> [t_out][ldc]
    transpose_block<T>(tile, b % p.dyn_x, b / p.dyn_x, 0, dy, p.t_out, p.c_out, p.t_out, nullptr, nullptr, nullptr, p.dyn,
                       p.ldc, 0, p.ldc, none);
}

// ------------------------------------------------------------------------------------------------
// conv helpers (explicit im2col into workspace; the contractions then run on the same GEMM core)
// dX operand: colA[(n,h,w)][tap*ldc + co] = dYn[(n,ho,wo)][co] with ho*stride + kh - pad = h (else 0).
// dYn is the token-major bf16 copy of dY with pitch ldc (multiple of 8).
__global__ __launch_bounds__(256) void k_im2col_dy(const bf16_t* __restrict__ dyn, int64_t ldc, ConvGeom g,
                                                   bf16_t* __restrict__ col) {
  const int64_t ch = ldc >> 3;                        // 16-byte chunks per tap
  const int taps = g.KH * g.KW;
  const int64_t total = (int64_t)g.N * g.H * g.W * taps * ch;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c8 = e % ch;
    int64_t r = e / ch;
    const int tap = (int)(r % taps);
    r /= taps;                                        // pixel index (n,h,w)
    const int w = (int)(r % g.W);
    const int h = (int)((r / g.W) % g.H);
    const int n = (int)(r / ((int64_t)g.W * g.H));
    const int kh = tap / g.KW, kw = tap % g.KW;
    const int hn = h + g.pad - kh, wn = w + g.pad - kw;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (hn >= 0 && wn >= 0 && hn % g.stride == 0 && wn % g.stride == 0) {
      const int ho = hn / g.stride, wo = wn / g.stride;
      if (ho < g.Ho && wo < g.Wo)
        v = *reinterpret_cast<const uint4*>(dyn + (((int64_t)n * g.Ho + ho) * g.Wo + wo) * ldc + c8 * 8);
    }
    *reinterpret_cast<uint4*>(col + (r * taps + tap) * ldc + c8 * 8) = v;
  }
}

// ------------------------------------------------------------------------------------------------
// dS_x, dZ_x: ordered sum of the per-block partials written by the dX epilogue.
template <int NTH>
__device__ __forceinline__ void sum_partials_block(const float* __restrict__ part, int64_t n,
                                                   float* __restrict__ ds_x, float* __restrict__ dz_x) {
  constexpr int NW = NTH / 64;
  double a = 0.0, b = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += NTH) { a += (double)part[2 * i]; b += (double)part[2 * i + 1]; }
  a = wave_sum(a); b = wave_sum(b);
  __shared__ double sa[NW], sb[NW];
  if ((threadIdx.x & 63) == 0) { sa[threadIdx.x >> 6] = a; sb[threadIdx.x >> 6] = b; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double ta = 0.0, tb = 0.0;
#pragma unroll
    for (int w = 0; w < NW; w += 4) {                  // fixed order
      ta += (sa[w] + sa[w + 1]) + (sa[w + 2] + sa[w + 3]);
      tb += (sb[w] + sb[w + 1]) + (sb[w + 2] + sb[w + 3]);
    }
    ds_x[0] = (float)ta;
    dz_x[0] = (float)tb;
  }
}

__global__ __launch_bounds__(256) void k_sum_partials(const float* __restrict__ part, int64_t n,
                                                      float* __restrict__ ds_x, float* __restrict__ dz_x) {
  sum_partials_block<256>(part, n, ds_x, dz_x);
}

// Optional optimizer step fused into the second pass (off when w == nullptr), the rule of Alg. 1's optimizer step for
// unfrozen channels.  Weight rows idx: SGD with momentum and weight decay, the optimizer the network parameters keep from
// the full-precision run:  g = dW + wd * W;  buf = mu * buf + g;  W -= lr_w * buf  (buf is skipped when mu == 0).
// Their scales S_w[idx]: Adam, which the quantization parameters are always trained with (Sec. 4 "Setup"), one state
// and step count per channel:  t += 1;  m = b1 m + (1 - b1) g;  v = b2 v + (1 - b2) g^2;
// S_w -= lr_s * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
struct StepArgs {
  float* w; float* mom_w;
  float lr_w, mu, wd;
  float* s_w; float* adam_m; float* adam_v; int32_t* adam_t;
  float lr_s, b1, b2, eps;
};

// Second pass of the restricted weight gradient: ordered split-K sum, S_x scaling, straight-through mask
// of the weight quantizer and the per-row scale gradient
//   dW[c][j] = in range ? dW_q : 0,  dS_w[c] = sum_j dW_q * (in range ? code - w/S_w : code),  c = idx[m].
// One block of NTH threads per row.  What bounds it is memory for large layers, else the chain of loads of a trip through the row.
// ANY: rows of any width and alignment; a lane owns four neighbouring columns and reads them in vector accesses, the last lane of
// a row that is no multiple of four starts earlier and leaves out the d columns that its neighbour has; everything but the slices
// past the first is requested at once.  That holds 92 registers a lane; without ANY, 48, and twice the wavefronts, for
// aligned rows of four where there are many rows or long ones (2752 x 4096: 26.8 us, with ANY 29 to 32).
// 2049 x 777 -> 1001, k = 250, 3 slices: 4.1 us; by single columns, slices and weights behind one another, 7.3.
template <int NTH, bool ANY>
__global__ __launch_bounds__(NTH) void k_dw_finish(const float* __restrict__ part, int S, int64_t k, int64_t ncols,
                                                   const float* __restrict__ s_x, const int8_t* __restrict__ w_codes,
                                                   const uint32_t* __restrict__ w_clip, const float* __restrict__ w,
                                                   const float* __restrict__ s_w, const int32_t* __restrict__ idx,
                                                   float* __restrict__ dw, int scatter, float* __restrict__ ds_w,
                                                   const float* __restrict__ part_dx, int64_t n_part_dx,
                                                   float* __restrict__ ds_x, float* __restrict__ dz_x,
                                                   const StepArgs sgd) {
  // the arguments in one batch: left to the compiler, some are requested where they are used, behind one another's waits (4384 x 1088 ->
  // 6960, k = 54: 7.8 us, so 7.1; 2020 x 352 -> 6784, all selected, 12.5, 11.9)
  asm volatile("" ::"s"(part), "s"(S), "s"(s_x), "s"(w_codes), "s"(w_clip), "s"(w), "s"(s_w), "s"(idx), "s"(dw), "s"(ds_w), "s"(scatter),
               "s"(sgd.w), "s"(sgd.mom_w));
  if ((int64_t)blockIdx.x == k) {                     // one extra block: dS_x, dZ_x from the dX epilogue's partials
    sum_partials_block<NTH>(part_dx, n_part_dx, ds_x, dz_x);
    return;
  }
  const int64_t m = blockIdx.x;
  const int64_t c = idx[m];
  const int64_t wpr = (ncols + 31) >> 5;
  const float sx = s_x[0];
  const float sw = s_w[c];
  const int64_t orow = scatter ? c : m;
  const int64_t slice = k * ncols;
  float acc = 0.0f;
  if constexpr (!ANY) {
    for (int64_t j = (int64_t)threadIdx.x * 4; j < ncols; j += 4 * NTH) {
      const float* p = part + m * ncols + j;
      float4 a = *reinterpret_cast<const float4*>(p);
      int s = 1;
      for (; s + 7 < S; s += 8) {                     // eight slices in flight; summed in slice order as below
        float4 b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = *reinterpret_cast<const float4*>(p + (int64_t)(s + u) * slice);
#pragma unroll
        for (int u = 0; u < 8; ++u) { a.x += b[u].x; a.y += b[u].y; a.z += b[u].z; a.w += b[u].w; }
      }
      for (; s + 3 < S; s += 4) {
        float4 b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = *reinterpret_cast<const float4*>(p + (int64_t)(s + u) * slice);
#pragma unroll
        for (int u = 0; u < 4; ++u) { a.x += b[u].x; a.y += b[u].y; a.z += b[u].z; a.w += b[u].w; }
      }
      for (; s < S; ++s) {
        const float4 b = *reinterpret_cast<const float4*>(p + (int64_t)s * slice);
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
      }
      const float dwq[4] = {sx * a.x, sx * a.y, sx * a.z, sx * a.w};
      const uint32_t bits = w_clip[c * wpr + (j >> 5)] >> (j & 31);
      const uint32_t cw = *reinterpret_cast<const uint32_t*>(w_codes + c * ncols + j);
      const float4 wv = *reinterpret_cast<const float4*>(w + c * ncols + j);
      const float wf[4] = {wv.x, wv.y, wv.z, wv.w};
      float o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bool inr = (bits >> t) & 1u;
        const float code = (float)(int8_t)((cw >> (8 * t)) & 0xFFu);
        const float gs = inr ? (code - wf[t] / sw) : code;
        acc += dwq[t] * gs;
        o[t] = inr ? dwq[t] : 0.0f;
      }
      if (dw) *reinterpret_cast<float4*>(dw + orow * ncols + j) = make_float4(o[0], o[1], o[2], o[3]);
      if (sgd.w) {
        float gq[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) gq[t] = fmaf(sgd.wd, wf[t], o[t]);
        if (sgd.mom_w) {
          float4 mb = *reinterpret_cast<const float4*>(sgd.mom_w + c * ncols + j);
          mb.x = fmaf(sgd.mu, mb.x, gq[0]); mb.y = fmaf(sgd.mu, mb.y, gq[1]);
          mb.z = fmaf(sgd.mu, mb.z, gq[2]); mb.w = fmaf(sgd.mu, mb.w, gq[3]);
          *reinterpret_cast<float4*>(sgd.mom_w + c * ncols + j) = mb;
          gq[0] = mb.x; gq[1] = mb.y; gq[2] = mb.z; gq[3] = mb.w;
        }
        *reinterpret_cast<float4*>(sgd.w + c * ncols + j) =
            make_float4(fmaf(-sgd.lr_w, gq[0], wf[0]), fmaf(-sgd.lr_w, gq[1], wf[1]), fmaf(-sgd.lr_w, gq[2], wf[2]),
                        fmaf(-sgd.lr_w, gq[3], wf[3]));
      }
    }
  } else {
    // columns j .. j + n - 1 of the row, n <= 4 (a row of fewer than four columns: one at a time)
    auto columns = [&](int64_t j, auto width) {
      constexpr int V = decltype(width)::value;
      const int d = j + V > ncols ? (int)(j + V - ncols) : 0;
      const int64_t e = c * ncols + j - d;
      const float* p = part + m * ncols + j - d;
      float a[V], wf[V], mb[V];
      uint32_t cw = 0;
      __builtin_memcpy(a, p, 4 * V);
      __builtin_memcpy(wf, w + e, 4 * V);
      __builtin_memcpy(&cw, w_codes + e, V);
      const uint32_t bits = (w_clip[c * wpr + (j >> 5)] >> (j & 31)) << d;
      if (sgd.w && sgd.mom_w) __builtin_memcpy(mb, sgd.mom_w + e, 4 * V);
      int s = 1;
      auto slices = [&](auto count) {                   // in flight together, added in slice order
        constexpr int N = decltype(count)::value;
        float b[N][V];
#pragma unroll
        for (int u = 0; u < N; ++u) __builtin_memcpy(b[u], p + (int64_t)(s + u) * slice, 4 * V);
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
          for (int t = 0; t < V; ++t) a[t] += b[u][t];
        s += N;
      };
      while (s + 7 < S) slices(std::integral_constant<int, 8>{});
      if (s + 3 < S) slices(std::integral_constant<int, 4>{});
      if (s + 2 < S) slices(std::integral_constant<int, 3>{});
      else if (s + 1 < S) slices(std::integral_constant<int, 2>{});
      else if (s < S) slices(std::integral_constant<int, 1>{});
      float o[V];
#pragma unroll
      for (int t = 0; t < V; ++t) {
        const float dwq = sx * a[t];
        const bool inr = (bits >> t) & 1u;
        const float code = (float)(int8_t)((cw >> (8 * t)) & 0xFFu);
        const float gs = inr ? (code - wf[t] / sw) : code;
        acc = t >= d ? acc + dwq * gs : acc;
        o[t] = inr ? dwq : 0.0f;
      }
      auto store = [&](float* dst, const float (&v)[V]) {
        if (d == 0) __builtin_memcpy(dst, v, 4 * V);
        else {
#pragma unroll
          for (int t = 1; t < V; ++t)
            if (t >= d) dst[t] = v[t];
        }
      };
      if (dw) store(dw + orow * ncols + j - d, o);
      if (sgd.w) {
        float gq[V];
#pragma unroll
        for (int t = 0; t < V; ++t) gq[t] = fmaf(sgd.wd, wf[t], o[t]);
        if (sgd.mom_w) {
#pragma unroll
          for (int t = 0; t < V; ++t) gq[t] = fmaf(sgd.mu, mb[t], gq[t]);
          store(sgd.mom_w + e, gq);
        }
#pragma unroll
        for (int t = 0; t < V; ++t) gq[t] = fmaf(-sgd.lr_w, gq[t], wf[t]);
        store(sgd.w + e, gq);
      }
    };
    if (ncols >= 4)
      for (int64_t j = (int64_t)threadIdx.x * 4; j < ncols; j += 4 * NTH) columns(j, std::integral_constant<int, 4>{});
    else if ((int64_t)threadIdx.x < ncols)
      columns(threadIdx.x, std::integral_constant<int, 1>{});
  }
  acc = wave_sum(acc);
  __shared__ float red[NTH / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float ds = 0.0f;
#pragma unroll
    for (int w = 0; w < NTH / 64; w += 4) ds += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);   // fixed order
    if (ds_w) ds_w[orow] = ds;
    if (sgd.s_w) {
      // one scalar per row: double precision costs nothing here and leaves only the fp32 storage rounding
      const int t = sgd.adam_t[c] + 1;
      const double g = (double)ds, b1 = (double)sgd.b1, b2 = (double)sgd.b2;
      const double m = b1 * (double)sgd.adam_m[c] + (1.0 - b1) * g;
      const double v = b2 * (double)sgd.adam_v[c] + (1.0 - b2) * g * g;
      const double m_hat = m / (1.0 - pow(b1, (double)t)), v_hat = v / (1.0 - pow(b2, (double)t));
      sgd.adam_t[c] = t;
      sgd.adam_m[c] = (float)m;
      sgd.adam_v[c] = (float)v;
      sgd.s_w[c] = (float)((double)sw - (double)sgd.lr_s * m_hat / (sqrt(v_hat) + (double)sgd.eps));
    }
  }
}

// ------------------------------------------------------------------------------------------------
static inline unsigned grid1d(int64_t total) {
  int64_t b = ceil_div(total, 256);
  if (b > 256 * 64) b = 256 * 64;
  if (b < 1) b = 1;
  return (unsigned)b;
}

// W_q^T alone (dY is used in place and no column of it is compacted), one block per tile and tap.  With the other parts'
// code and arguments around it the launch is up to 1 us longer: 3 x 3 convolution of 8 x 14 x 14, 128 -> 64 channels, bf16,
// all selected: backward call 34.8 us, by k_prep 35.9 us; 4096 x 1024 -> 1024, nothing selected: 20.6, 21.3 us.
__global__ __launch_bounds__(256) void k_prep_w(const int8_t* __restrict__ w_codes, int64_t w_ld, int64_t c_out, int64_t c_in,
                                                const float* __restrict__ s_w, bf16_t* __restrict__ wqT, int64_t w_ldo,
                                                int64_t ldc, uint32_t* __restrict__ zero_page) {
  __shared__ TransposeTile tile;
  if (zero_page && (blockIdx.x | blockIdx.y | blockIdx.z) == 0 && threadIdx.x < 64) zero_page[threadIdx.x] = 0u;
  TransposeExtra ex{};
  ex.z_in = c_in; ex.z_out = ldc;
  transpose_block<int8_t>(tile, blockIdx.x, blockIdx.y, blockIdx.z, w_codes, w_ld, c_out, c_in, nullptr, s_w, nullptr, wqT,
                          w_ldo, 0, ldc, ex);
}

static uint32_t cut_rows(int64_t rows, int64_t ldo, RowCut* cut) {   // returns the blocks
  cut->cols = rows * ceil_div(ldo, 512) > 4096 ? 2048 : 512;
  cut->segs = (uint32_t)ceil_div(ldo, cut->cols);
  return (uint32_t)std::min<int64_t>(ceil_div(rows * cut->segs, 4), 16384);
}

static int launch_prep(const PrepArgs& a, int dy_dtype, hipStream_t st) {
  // a grid dimension holds less than 2^32 work items
  const int64_t blocks = (int64_t)a.n_gather + a.n_rows + a.n_w + a.n_x + a.n_sel + a.n_dyn;
  if (blocks == 0) return EFQAT_OK;
  if (blocks == a.n_w && a.w_y <= 65535) {
    hipLaunchKernelGGL(k_prep_w, dim3(a.w_x, a.w_y, a.n_w / (a.w_x * a.w_y)), dim3(256), 0, st, a.w_codes, a.w_ld, a.c_out,
                       a.c_in, a.s_w, a.wqT, a.w_ldo, a.ldc, a.zero_page);
    EFQAT_LAUNCH_CHECK();
    return EFQAT_OK;
  }
  const int64_t bx = std::min<int64_t>(blocks, 1 << 22);
  const dim3 grid((unsigned)bx, (unsigned)ceil_div(blocks, bx));
  if (dy_dtype == EFQAT_F32) hipLaunchKernelGGL((k_prep<float>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((k_prep<bf16_t>), grid, dim3(256), 0, st, a);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

// the W_q^T part: w codes [c_out][taps][c_in], rows of the result hold taps spans of ldc
static void prep_w_operand(PrepArgs& a, const int8_t* w_codes, const float* s_w, int64_t c_in, int64_t c_out, int taps,
                           int64_t ldc, bf16_t* wqT) {
  a.w_codes = w_codes; a.s_w = s_w; a.wqT = wqT; a.c_in = c_in; a.c_out = c_out; a.ldc = ldc;
  a.w_ld = (int64_t)taps * c_in; a.w_ldo = (int64_t)taps * ldc;
  a.w_ex.z_in = c_in; a.w_ex.z_out = ldc;
  a.w_x = (uint32_t)ceil_div(ldc, 64); a.w_y = (uint32_t)ceil_div(c_in, 64);
  a.n_w = a.w_x * a.w_y * (uint32_t)taps;
}

// widest staged copy, 65535 tiles of 64 columns: a limit of the interface, no longer of a grid
constexpr int64_t kMaxStagedColumns = 65535 * (int64_t)64;

// Plan of one backward call: sizes of every workspace slice (shared by the size query and the call).
struct BwdPlan {
  int64_t Mx;      // rows of dX as a matrix (T, or N*H*W)
  int64_t Kx;      // contraction length of the dX product (padded C_out, times taps for conv)
  int64_t Nw;      // columns of dW as a matrix (C_in, or KH*KW*C_in)
  int64_t Tw;      // contraction length of the dW product (T, or N*Ho*Wo)
  int64_t ldc;     // C_out rounded up to 8
  int64_t ldt;     // Tw rounded up to 8
  bool need_dyn;   // token-major bf16 copy of dY needed
  bool need_sel;   // gathered dY^T rows materialised (token-major dY, or fp32 / unaligned channel-major)
  bool tn;         // dW product straight from token-major dY columns and the uint8 codes (no transposed copies)
  bool tn_direct;  // ... with dY itself as the A operand (all channels selected)
  bool cmx;        // channel-major dY: dX product straight from dY [C_out][T] and the int8 weight codes
  bool rdw;        // channel-major dY: dW product from the selected rows of dY and the uint8 codes, nothing staged
  bool cdw;        // convolution dW product with the im2col gather of the codes inside the tile loads
  bool cdx;        // convolution dX product with the im2col gather inside the tile loads (no im2col matrix)
  bool cdxs;       // ... of a convolution with a stride: rows sorted by (h mod stride, w mod stride)
  bool dx8;        // dX product with the weight operand read from the int8 codes (no bf16 W_q^T copy)
  bool pair;       // both products in one grid of 64-row tiles
  int dx8_tile;
  int64_t kp;      // k rounded up to 8 (pitch of the compacted dY columns)
  GemmPlan plan_dx, plan_dw;
  size_t b_wqT, b_dyn, b_colA, b_part_dx, b_xcT, b_sel, b_part_dw, total;
};

static ConvDxStridedMap strided_map(const ConvGeom& g) {
  return ConvDxStridedMap{g.N, g.H, g.W, g.Ho, g.Wo, g.KH, g.KW, g.stride, g.pad};
}

// Can the dX product gather dY in its tile loads?  The pitch holds whole 64-channel K stages, and the multiplication that
// takes a stage apart into tap and channel stage is exact: stages of a tile times stages of a tap below 2^32 (a million
// channels and 16 taps are the first beyond).  Pixel coordinates take 16 bits each; conv_geom allows images to 2^15.
static bool conv_stages_ok(const ConvGeom& g, int64_t ldc) {
  const int64_t taps = ceil_div(g.KH, g.stride) * ceil_div(g.KW, g.stride), spt = ldc / 64;
  return (ldc % 64) == 0 && taps * spt * spt < ((int64_t)1 << 32);
}

// dxk: the caller's choice of the dX kernel (EFQAT_DX_KERNEL_*); it changes workspace sizes, so the size query takes
// it as well.  wide: tiles of 128 and more by gemm_plan's rule, for callers whose workspace or weight codes do not fit the
// plan by kDxTiles, kDwTiles and pair_plan (see choose_plan).
static BwdPlan make_plan(int64_t T_in, int64_t T_out, int64_t c_in, int64_t c_out, int taps, int64_t k,
                         int dy_dtype, int dy_layout, bool im2col, int dxk, const ConvGeom* cg, bool wide) {
  BwdPlan p{};
  p.Mx = T_in; p.Tw = T_out; p.Nw = (int64_t)taps * c_in;
  p.ldc = round_up(c_out, 8); p.ldt = round_up(T_out, 8);
  // A convolution whose channel count is no whole number of 64-channel K stages gets them by zero channels in the bf16
  // copy of dY (one copy instead of an im2col matrix of KH KW copies), unless that would more than double the product.
  // 3 x 3, c_in 128, bf16 token-major, r = 5 %, backward call padded / by im2col, us: 32 images of 28 x 28 at stride 1 with
  // 40, 72, 136, 520 channels: 52 / 67, 61 / 73, 67 / 88, 104 / 188; at stride 2: 39 / 57, 45 / 64, 50 / 76, 66 / 162; 8 of
  // 14 x 14 at stride 1: 36 / 37, 41 / 40, 46 / 47, 78 / 90 (72 channels, all selected: 41.3 / 39.9, the worst found).
  if (im2col && cg && cg->stride <= kMaxConvStride && dxk != EFQAT_DX_KERNEL_BF16_PINNED && round_up(c_out, 64) <= 2 * c_out &&
      conv_stages_ok(*cg, round_up(c_out, 64)))
    p.ldc = round_up(c_out, 64);
  p.Kx = (int64_t)taps * p.ldc;
  const bool direct_tok = dy_layout == EFQAT_DY_TOKEN_MAJOR && dy_dtype == EFQAT_BF16 && p.ldc == c_out;
  p.need_dyn = !direct_tok;
  const bool direct_rows = dy_layout == EFQAT_DY_CHANNEL_MAJOR && dy_dtype == EFQAT_BF16 && (T_out % 8) == 0;
  p.cdw = k > 0 && dy_layout == EFQAT_DY_TOKEN_MAJOR && im2col && cg && (c_in % 128) == 0;
  p.tn = k > 0 && dy_layout == EFQAT_DY_TOKEN_MAJOR && ((!im2col && (c_in % 16) == 0) || p.cdw);
  p.tn_direct = p.tn && direct_tok && k == c_out;
  p.rdw = k > 0 && direct_rows && !im2col && (c_in % 16) == 0;
  p.cmx = direct_rows && !im2col && taps == 1 && (c_in % 16) == 0 && dxk != EFQAT_DX_KERNEL_BF16_PINNED;
  if (p.cmx) p.need_dyn = false;
  p.kp = round_up(k, 8);
  p.need_sel = k > 0 && !direct_rows && !p.tn_direct;
  // stride-1 convolutions whose channel pitch is a multiple of the 64-element K stage gather dY in the tile loads
  p.cdx = im2col && cg && cg->stride == 1 && conv_stages_ok(*cg, p.ldc);
  // Strides 2 to 4 (a 3 x 3 kernel at stride 2 forms 9 products per 4 pixels instead of 36, and no im2col matrix of 9
  // copies of dY: 32 x 28 x 28, 128 -> 256 channels, fp32: the im2col pass took 42 us, the backward call 108 -> 51 us); larger
  // strides have too many phases to sort the rows for.
  p.cdxs = im2col && cg && cg->stride > 1 && cg->stride <= kMaxConvStride && conv_stages_ok(*cg, p.ldc) &&
           dxk != EFQAT_DX_KERNEL_BF16_PINNED;
  double price_dx = 0.0, price_dw = 0.0;
  const ConvDxStridedMap sm = p.cdxs ? strided_map(*cg) : ConvDxStridedMap{};
  const bool int8_ok = taps == 1 && !im2col && direct_tok && (c_in % 16) == 0 && dxk != EFQAT_DX_KERNEL_BF16;
  if (wide) {
    p.plan_dx = gemm_plan(p.Mx, c_in, p.Kx, false, true, !p.cdx);
    if (p.cdxs) p.plan_dx = GemmPlan{128, 1, (int)conv_dx_strided_row_tiles(sm, 128), (int)ceil_div(c_in, 128)};
    p.plan_dx.ring = (p.plan_dx.tile == 192 && !p.cdx) ||
                     (p.plan_dx.tile == 128 && (int64_t)p.plan_dx.tiles_m * p.plan_dx.tiles_n <= 256);
  } else {
    p.plan_dx = dx_plan(p.Mx, c_in, p.Kx, dy_dtype == EFQAT_F32, p.cdx || p.cdxs, p.cdxs ? &sm : nullptr, int8_ok, &price_dx);
  }
  if (p.cdxs) p.cdx = true;
  p.dx8 = false; p.dx8_tile = 0;
  // Products on 256 x 256 tiles with a bf16 token-major dY read the weight operand straight from the int8 codes: same speed
  // as the bf16 kernel on these shapes, and no transposed bf16 copy of W_q.
  if (p.cmx) {
    p.plan_dx = wide ? gemm_plan(p.Mx, c_in, p.Kx, false, false) : dx_cm_plan(p.Mx, c_in, p.Kx, &price_dx);
    p.dx8 = true; p.dx8_tile = p.plan_dx.tile;
  } else if (dxk == EFQAT_DX_KERNEL_BF16_PINNED) {
    if (!p.cdx) p.plan_dx = GemmPlan{192, 1, (int)ceil_div(p.Mx, 192), (int)ceil_div(c_in, 192), true};
  } else if (int8_ok && (p.plan_dx.tile == 256 || dxk == EFQAT_DX_KERNEL_INT8)) {
    p.dx8 = true; p.dx8_tile = (p.plan_dx.tile == 256 || (p.Mx >= 1024 && c_in >= 512)) ? 256 : 128;
    p.plan_dx.tiles_m = (int)ceil_div(p.Mx, p.dx8_tile); p.plan_dx.tiles_n = (int)ceil_div(c_in, p.dx8_tile);
  }
  if (k == 0) p.plan_dw = GemmPlan{128, 1, 0, 0, false};
  else if (wide) p.plan_dw = gemm_plan(k, p.Nw, p.ldt, true, !(p.tn || p.rdw), !p.cdw);
  else {
    const DwKind kind = p.rdw ? DW_ROWS : p.cdw ? DW_CONV : p.tn ? DW_TOKENS : DW_STAGED;
    p.plan_dw = dw_plan(kind, k, p.Nw, p.ldt, &price_dw);
    if (p.cmx && p.rdw && price_dw > 0.0) {
      p.pair = pair_cm_plan(p.Mx, c_in, p.Kx, k, p.Nw, p.ldt, price_dx + price_dw, &p.plan_dx, &p.plan_dw);
      p.dx8_tile = p.plan_dx.tile;
    }
    if (price_dw > 0.0 && !p.dx8 && dxk == EFQAT_DX_KERNEL_AUTO && (!im2col || p.cdx)) {
      if (int8_ok) price_dx -= 3.0 * (double)c_in * (double)p.Kx / 4e6;   // W_q^T in bf16 (dx_plan): the pair needs it as well
      p.pair = pair_plan(p.Mx, c_in, p.Kx, dy_dtype == EFQAT_F32, p.cdx, p.cdxs ? &sm : nullptr, kind, k, p.Nw, p.ldt,
                         price_dx + price_dw, &p.plan_dx, &p.plan_dw);
    }
  }
  WsCarver cv(nullptr);
  p.b_wqT = p.dx8 ? 0 : (size_t)c_in * p.Kx * 2; cv.take(p.b_wqT);
  p.b_dyn = p.need_dyn ? (size_t)T_out * p.ldc * 2 : 0; cv.take(p.b_dyn);
  p.b_colA = (im2col && !p.cdx) ? (size_t)T_in * p.Kx * 2 : 0; cv.take(p.b_colA);
  // one (dS_x, dZ_x) pair per tile: sized for the smallest tile, whichever kernel runs
  p.b_part_dx = (size_t)std::max<int64_t>(ceil_div(p.Mx, 128) * ceil_div(c_in, 128),
                                          (int64_t)p.plan_dx.tiles_m * p.plan_dx.tiles_n) * 2 * sizeof(float);
  cv.take(p.b_part_dx);
  p.b_xcT = (k > 0 && !p.tn && !p.rdw) ? (size_t)p.Nw * p.ldt * 2 : 0; cv.take(p.b_xcT);
  p.b_sel = p.need_sel ? (p.tn ? (size_t)T_out * p.kp * 2 : (size_t)k * p.ldt * 2) : 0; cv.take(p.b_sel);
  p.b_part_dw = k > 0 ? (size_t)p.plan_dw.split_k * k * p.Nw * sizeof(float) : 0; cv.take(p.b_part_dw);
  p.total = cv.off;
  return p;
}

static bool takes_side_stream(const BwdPlan& p) { return (p.tn || p.rdw) && !p.pair; }   // tn, rdw: only where k > 0

static int plan_info(const BwdPlan& p, bool im2col, int64_t k, int32_t* out) {
  out[EFQAT_PLAN_ONE_GRID] = p.pair; out[EFQAT_PLAN_SIDE_STREAM] = takes_side_stream(p);
  out[EFQAT_PLAN_DX_KERNEL] = p.dx8 ? 2 : p.plan_dx.ring ? 1 : 0;
  out[EFQAT_PLAN_DX_TILE] = p.dx8 ? p.dx8_tile : p.plan_dx.tile;
  out[EFQAT_PLAN_DX_ROWS] = p.cdxs ? 2 : p.cdx ? 1 : im2col ? 3 : 0;
  out[EFQAT_PLAN_DW_OPERANDS] = k == 0 ? 0 : p.cdw ? 2 : p.tn ? 1 : p.rdw ? 4 : 3;
  out[EFQAT_PLAN_DW_TILE] = k == 0 ? 0 : p.plan_dw.tile;
  out[EFQAT_PLAN_DW_SLICES] = k == 0 ? 0 : p.plan_dw.split_k;
  return EFQAT_OK;
}

template <class Plan>
static size_t query_plan(const Plan& plan) { return std::max(plan(false).total, plan(true).total); }

struct BwdIo {
  const void* dy; int dy_dtype; int dy_layout;
  const uint8_t* x_codes; const uint32_t* x_clip; const void* x; int x_dtype; const float* s_x; const float* z_x;
  const int8_t* w_codes; const uint32_t* w_clip; const float* w; const float* s_w; const int32_t* idx; int64_t k;
  void* dx; int dx_dtype; float* dw; int scatter; float* ds_w; float* ds_x; float* dz_x;
  StepArgs sgd;    // fused optimizer step (sgd.w == nullptr: none)
  const void* w_operand = nullptr;   // optional: the bf16 W_q^T matrix made beforehand
  hipStream_t side = nullptr;        // optional: second stream for the weight-gradient branch
};

// The plan of a call, or the wide one where that needs less workspace than the call brings, or 16-byte aligned weight codes
// that it does not.  A workspace of either size is taken, and the query returns the larger.  c_in beyond what the bf16
// W_q^T may have (check_plan) leaves the choice to gemm_plan's rule as well.  No operand is made beforehand for a layer whose
// first plan reads the weight codes themselves (efqat_linear_bwd_weight_operand): what the call brings is ignored, and the
// wide plan makes its own in the workspace.
template <class Plan>
static BwdPlan choose_plan(const Plan& plan, int64_t c_in, BwdIo& io, size_t ws_bytes) {
  const BwdPlan p = plan(c_in > kMaxStagedColumns);
  if (p.dx8) io.w_operand = nullptr;
  if (ws_bytes < p.total || (p.dx8 && ((uintptr_t)io.w_codes % 16) != 0)) {
    const BwdPlan w = plan(true);
    if (ws_bytes >= w.total) return w;
  }
  return p;
}

// Fork / join events of the optional second stream: one pair per host thread and device, made at first use and kept
// (recording an event again while an earlier wait on it is still queued is well defined: a wait refers to the
// record that preceded it).
struct SideEvents { hipEvent_t fork, join; };
static int side_events(SideEvents* out) {
  constexpr int kMaxDev = 64;
  thread_local SideEvents ev[kMaxDev];
  thread_local bool have[kMaxDev] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) return EFQAT_ERR_HIP;
  if (!have[dev]) {
    if (hipEventCreateWithFlags(&ev[dev].fork, hipEventDisableTiming) != hipSuccess) return EFQAT_ERR_HIP;
    if (hipEventCreateWithFlags(&ev[dev].join, hipEventDisableTiming) != hipSuccess) return EFQAT_ERR_HIP;
    have[dev] = true;
  }
  *out = ev[dev];
  return EFQAT_OK;
}

// Everything that can still fail once the plan is known, checked before the first launch: pointer alignment of the
// operands that the chosen kernels copy 16 bytes at a time, and the size limits of the staged copies.
static int check_plan(const BwdPlan& p, const BwdIo& io, int64_t T_out, int64_t c_in, int64_t c_out) {
  if (p.dx8 && ((uintptr_t)io.w_codes % 16) != 0) return EFQAT_ERR_ALIGNMENT;
  if ((p.tn || p.rdw) && ((uintptr_t)io.x_codes % 16) != 0) return EFQAT_ERR_ALIGNMENT;
  if (!p.dx8 && !io.w_operand && c_in > kMaxStagedColumns) return EFQAT_ERR_BAD_SHAPE;
  if (p.need_dyn && io.dy_layout == EFQAT_DY_CHANNEL_MAJOR && T_out > kMaxStagedColumns) return EFQAT_ERR_BAD_SHAPE;
  if (io.k > 0 && !p.tn && !p.rdw && (c_in > kMaxStagedColumns || io.k > kMaxStagedColumns)) return EFQAT_ERR_BAD_SHAPE;
  // 32-bit per-stage pointer steps of the kernels that read operands as they lie
  if ((p.dx8 || p.tn || p.rdw) && (c_in >= (1 << 24) || c_out >= (1 << 24))) return EFQAT_ERR_BAD_SHAPE;
  if ((p.cmx || p.rdw) && T_out >= (1 << 24)) return EFQAT_ERR_BAD_SHAPE;
  return EFQAT_OK;
}

// Shared driver.  For conv, T_in = N*H*W input pixels, T_out = N*Ho*Wo output pixels; for linear both are T.
static int run_bwd(const BwdIo& io, const BwdPlan& p, int64_t T_in, int64_t T_out, int64_t c_in, int64_t c_out,
                   const ConvGeom* cg, void* ws, hipStream_t st) {
  const int taps = cg ? cg->KH * cg->KW : 1;
  // a 1x1 / stride 1 / no-padding convolution is a linear layer over pixels: no im2col needed
  const bool im2col = cg != nullptr && !(taps == 1 && cg->stride == 1 && cg->pad == 0);
  WsCarver cv(ws);
  bf16_t* wqT = (bf16_t*)cv.take(p.b_wqT);
  bf16_t* dyn = (bf16_t*)cv.take(p.b_dyn);
  bf16_t* colA = (bf16_t*)cv.take(p.b_colA);
  float* part_dx = (float*)cv.take(p.b_part_dx);
  bf16_t* xcT = (bf16_t*)cv.take(p.b_xcT);
  bf16_t* sel = (bf16_t*)cv.take(p.b_sel);
  float* part_dw = (float*)cv.take(p.b_part_dw);
  int rc = EFQAT_OK;

  // ---- optional second stream.  The weight-gradient branch (compaction of the selected columns of dY, dW product)
  // reads the call's inputs only, so it may run beside the dX product: blocks of the two products then share the compute
  // units, and neither leaves a partly filled last round behind.  It is forked here, behind everything the caller's
  // stream held before the call, and joined before the second pass of the weight gradient.
  // Products that share a grid run beside each other already, at no cost of events; with both products on one stream the
  // result is the same bit for bit.  Launches that are timed by class are kept apart.
  const bool pair = p.pair && !prof_enabled();
  const bool use_side = io.side && io.side != st && takes_side_stream(p);
  hipStream_t st2 = st;
  SideEvents ev{};
  if (use_side) {
    rc = side_events(&ev);
    if (rc) return rc;
    if (hipEventRecord(ev.fork, st) != hipSuccess || hipStreamWaitEvent(io.side, ev.fork, 0) != hipSuccess)
      return EFQAT_ERR_HIP;
    st2 = io.side;
  }

  ProfScope prep(PROF_PREP, st);                       // operand preparation ahead of the dX product
  const bool own_wqT = !p.dx8 && !io.w_operand;
  // made beforehand by efqat_linear_bwd_weight_operand (same kernel, same bits)
  if (!p.dx8 && io.w_operand) wqT = (bf16_t*)const_cast<void*>(io.w_operand);
  const bool gather = p.tn && !p.tn_direct;
  const bool copy_dy = p.need_dyn && io.dy_layout == EFQAT_DY_TOKEN_MAJOR;
  const int64_t gx = std::max<int64_t>(1, ceil_div(p.kp, 128));
  const int64_t gy = std::max<int64_t>(1, std::min<int64_t>(65535, (1 << 24) / gx));
  const dim3 ggrid((unsigned)gx, (unsigned)std::min(ceil_div(T_out, kGatherRows), gy));
  const bool stage_dw = io.k > 0 && !p.tn && !p.rdw;   // staged bf16 operands of the fall-back dW product
  PrepArgs a{};
  a.dy = io.dy; a.c_in = c_in; a.c_out = c_out; a.t_out = T_out; a.ldc = p.ldc; a.ldt = p.ldt;
  a.idx = io.idx; a.k = io.k; a.sel = sel; a.kp = p.kp; a.dyn = dyn;
  a.chan = io.dy_layout == EFQAT_DY_CHANNEL_MAJOR ? 1 : 0;
  if (gather && !use_side) { a.gather_x = ggrid.x; a.n_gather = ggrid.x * ggrid.y; }
  if (copy_dy) {
    // dY as a token-major bf16 matrix [T_out][ldc] (A operand of the dX product)
    a.rows_flat = p.ldc == c_out ? 1 : 0;
    // lanes to a row: as many as it has chunks, or more of them idle while that makes 512 wavefronts or fewer, one trip each: with few
    // tokens the call waits for the slowest wavefront.  Backward call, us, as many lanes as chunks in as few blocks as make two chunks
    // a thread / so / a wavefront a row: 337 x 64, 19 channels, k = 3 fp32 11.7 / 11.0 / 10.9; 1635 x 128, 13 channels, k = 2 12.5 /
    // 12.1 / 12.1; 14392 x 64, 39 channels fp32 10.3 / 10.1 / 13.0; 19932 x 333, 93 channels 23.5 / 23.1 / 27.0
    if (!a.rows_flat && ((c_out % 8) == 0 || p.ldc <= 512))
      for (a.rows_flat = 2; a.rows_flat < 64 && (a.rows_flat < p.ldc / 8 || T_out * a.rows_flat <= 32 * 512);) a.rows_flat *= 2;
    int64_t nb = a.rows_flat ? ceil_div(T_out * p.ldc, 256 * 16) : cut_rows(T_out, p.ldc, &a.rows_cut);
    if (a.rows_flat > 1) nb = std::max(nb, std::min<int64_t>(ceil_div(T_out * a.rows_flat, 256), 1024));
    a.n_rows = (uint32_t)std::min<int64_t>(nb, 4096);
  } else if (p.need_dyn) {
    a.dyn_x = (uint32_t)ceil_div(p.ldc, 64);
    a.n_dyn = a.dyn_x * (uint32_t)ceil_div(T_out, 64);
  }
  if (own_wqT) prep_w_operand(a, io.w_codes, io.s_w, c_in, c_out, taps, p.ldc, wqT);
  if (stage_dw) {
    a.x_codes = io.x_codes; a.z_x = io.z_x; a.xcT = xcT;
    if (im2col) { a.x_ex.z_orow = c_in; a.x_ex.conv = 1; a.x_ex.g = *cg; }
    a.x_x = (uint32_t)ceil_div(p.ldt, 64); a.x_y = (uint32_t)ceil_div(c_in, 64);
    a.n_x = a.x_x * a.x_y * (uint32_t)(im2col ? taps : 1);
    if (p.need_sel) {
      a.sel_x = (uint32_t)ceil_div(p.ldt, 64);
      a.n_sel = a.chan ? cut_rows(io.k, p.ldt, &a.sel_cut) : a.sel_x * (uint32_t)ceil_div(io.k, 64);
    }
  }
  rc = launch_prep(a, io.dy_dtype, st);
  if (rc) return rc;
  const bf16_t* dy_tok = p.need_dyn ? dyn : (const bf16_t*)io.dy;

  // ---- operands of the dX product with the fused straight-through / qparam epilogue
  const bf16_t* A = dy_tok;
  int64_t lda = p.ldc;
  if (im2col && !p.cdx) {
    hipLaunchKernelGGL(k_im2col_dy, dim3(grid1d(T_in * taps * (p.ldc / 8))), dim3(256), 0, st, dy_tok, p.ldc, *cg,
                       colA);
    EFQAT_LAUNCH_CHECK();
    A = colA; lda = p.Kx;
  }
  prep.close();
  GemmEpilogueDx epi{io.x_codes, io.x_clip, io.x, io.x_dtype, io.s_x, io.z_x, io.dx, io.dx_dtype, part_dx};
  GemmStridedArgs dxa{};
  GemmDx8Args cma{}, rwa{};
  const int conv = p.cdxs ? 2 : p.cdx ? 1 : 0;
  if (p.cmx) {
    rc = dx_args_cm(&cma, (const bf16_t*)io.dy, T_out, io.w_codes, c_in, io.s_w, p.Mx, c_in, c_out, p.plan_dx, epi);
  } else if (p.cdxs) {
    rc = dx_args_strided(&dxa, dy_tok, p.ldc, wqT, p.Kx, p.Mx, c_in, strided_map(*cg), p.plan_dx, epi);
  } else if (p.cdx) {
    const ConvDxMap cm{cg->H, cg->W, cg->Ho, cg->Wo, cg->KW, cg->pad};
    rc = dx_args_conv(&dxa, dy_tok, p.ldc, wqT, p.Kx, p.Mx, c_in, p.Kx, cm, p.plan_dx, epi);
  } else if (!p.dx8) {
    rc = dx_args_linear(&dxa, A, lda, wqT, p.Kx, p.Mx, c_in, p.Kx, p.plan_dx, epi);
  }
  if (rc) return rc;

  // ---- operands of the dW product
  GemmTnArgs tna{};
  GemmArgs nta{};
  if (p.tn) {
    // straight from token-major operands: A = the selected columns of dY (compacted once, or dY itself when every channel is
    // selected), B = the uint8 codes; transposition happens in the LDS reads
    const bf16_t* At = gather ? sel : (const bf16_t*)io.dy;
    const int64_t ldat = gather ? p.kp : c_out, acols = ldat;
    if (p.cdw) {
      const ConvDwMap cm{cg->H, cg->W, cg->Ho, cg->Wo, cg->KW, cg->stride, cg->pad, (int)c_in};
      rc = dw_args_tn_conv(&tna, At, ldat, acols, io.x_codes, cm, io.z_x, io.k, p.Nw, T_out, p.plan_dw, part_dw);
    } else {
      rc = dw_args_tn(&tna, At, ldat, acols, io.x_codes, c_in, c_in, io.z_x, io.k, p.Nw, T_out, p.plan_dw, part_dw);
    }
  } else if (p.rdw) {                                  // channel-major dY: the selected rows are gathered by the tile loads
    rc = dw_args_rows(&rwa, (const bf16_t*)io.dy, T_out, io.idx, io.x_codes, c_in, io.z_x, io.k, p.Nw, T_out, p.plan_dw, part_dw);
  } else if (io.k > 0) {
    // staged operands; channel-major bf16 dY that is not staged: the gather is fused into the tile loads
    const bf16_t* Aw = p.need_sel ? sel : (const bf16_t*)io.dy;
    const int64_t ldaw = p.need_sel ? p.ldt : T_out;
    rc = dw_args_staged(&nta, Aw, ldaw, p.need_sel ? nullptr : io.idx, xcT, p.ldt, io.k, p.Nw, ldaw, p.plan_dw, part_dw);
  }
  if (rc) return rc;

  // ---- the products
  if (pair && p.cmx) {
    rc = launch_pair_cm(cma, rwa, p.plan_dw.split_k, st);
  } else if (pair) {
    rc = launch_pair(dxa, conv, p.plan_dx, p.tn ? &tna : nullptr, p.tn ? nullptr : &nta, p.plan_dw, st);
  } else if (p.cmx) {
    rc = launch_gemm_dx8_cm(cma, p.plan_dx, st);
  } else if (p.dx8) {
    rc = launch_gemm_dx8(dy_tok, c_out, io.w_codes, c_in, io.s_w, p.Mx, c_in, c_out, p.dx8_tile, epi, st);
  } else {
    rc = launch_dx(dxa, conv, p.plan_dx, use_side, st);
  }
  if (rc) return rc;
  const int64_t n_part_dx = (int64_t)p.plan_dx.tiles_m * p.plan_dx.tiles_n;
  if (io.k == 0) {
    ProfScope fin(PROF_FINISH, st);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, part_dx, n_part_dx, io.ds_x, io.dz_x);
    EFQAT_LAUNCH_CHECK();
    return EFQAT_OK;
  }
  if (gather && use_side) {
    ProfScope gat(PROF_PREP, st2);
    if (io.dy_dtype == EFQAT_F32)
      hipLaunchKernelGGL((k_gather_cols<float>), ggrid, dim3(256), 0, st2, (const float*)io.dy, c_out, T_out, io.idx, io.k, sel,
                         p.kp);
    else
      hipLaunchKernelGGL((k_gather_cols<bf16_t>), ggrid, dim3(256), 0, st2, (const bf16_t*)io.dy, c_out, T_out, io.idx, io.k,
                         sel, p.kp);
    EFQAT_LAUNCH_CHECK();
  }
  if (pair) rc = EFQAT_OK;
  else if (p.tn) rc = launch_gemm_tn(tna, p.plan_dw, st2);
  else if (p.rdw) rc = launch_gemm_dw_rows(rwa, p.plan_dw, st2);
  else rc = launch_gemm_nt_raw(nta, p.plan_dw, st);
  if (rc) return rc;
  if (use_side && (hipEventRecord(ev.join, st2) != hipSuccess || hipStreamWaitEvent(st, ev.join, 0) != hipSuccess))
    return EFQAT_ERR_HIP;
  ProfScope fin(PROF_FINISH, st);
  // k blocks for the rows of dW plus one that finishes dS_x, dZ_x
  // few rows: the chain of dependent loads of a trip, not bandwidth, sets the time, and a row is one trip where that can be (k = 64
  // rows of 1152, 25 slices, two trips of 256 threads 6.3 us, one of 512 4.8).  One or two slices leave nothing behind the first to
  // request together (256 x 768 -> 1000, k = 64, the call 19.6 us, with ANY 20.0; three slices and more gain 1 to 5 %).
  const bool few = io.k < 512;
  const bool vec = p.Nw % 4 == 0 && ((uintptr_t)io.w % 16) == 0 && ((uintptr_t)io.dw % 16) == 0 && ((uintptr_t)io.w_codes % 4) == 0 &&
                   ((uintptr_t)io.sgd.mom_w % 16) == 0;
  auto finish = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)io.k + 1), dim3(threads), 0, st, part_dw, p.plan_dw.split_k, io.k, p.Nw, io.s_x, io.w_codes,
                       io.w_clip, io.w, io.s_w, io.idx, io.dw, io.scatter, io.ds_w, part_dx, n_part_dx, io.ds_x, io.dz_x, io.sgd);
  };
  if (few && p.Nw > 1024 && p.Nw < 2048) finish(k_dw_finish<512, true>, 512);
  else if (few && p.Nw >= 2048) { if (vec) finish(k_dw_finish<1024, false>, 1024); else finish(k_dw_finish<1024, true>, 1024); }
  else if (vec && (!few || p.plan_dw.split_k <= 2)) finish(k_dw_finish<256, false>, 256);
  else finish(k_dw_finish<256, true>, 256);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

static int check_common(const BwdIo& io, int64_t c_out, const void* ws, int dxk) {
  if (io.dy_dtype != EFQAT_F32 && io.dy_dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (io.x_dtype != EFQAT_F32 && io.x_dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (io.dx_dtype != EFQAT_F32 && io.dx_dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (io.dy_layout != EFQAT_DY_TOKEN_MAJOR && io.dy_layout != EFQAT_DY_CHANNEL_MAJOR) return EFQAT_ERR_BAD_LAYOUT;
  if (dxk < EFQAT_DX_KERNEL_AUTO || dxk > EFQAT_DX_KERNEL_BF16_PINNED) return EFQAT_ERR_BAD_LAYOUT;
  if (io.k < 0 || io.k > c_out) return EFQAT_ERR_BAD_K;
  if (io.scatter != 0 && io.scatter != 1) return EFQAT_ERR_BAD_LAYOUT;
  if (!io.dy || !io.x_codes || !io.x_clip || !io.x || !io.s_x || !io.z_x || !io.w_codes || !io.s_w || !io.dx ||
      !io.ds_x || !io.dz_x || !ws)
    return EFQAT_ERR_NULL_PTR;
  if (io.k > 0 && (!io.idx || !io.w_clip || !io.w)) return EFQAT_ERR_NULL_PTR;
  if (io.k > 0 && !io.sgd.w && (!io.dw || !io.ds_w)) return EFQAT_ERR_NULL_PTR;   // gradients may stay unwritten only with the fused step
  if (((uintptr_t)ws % 256) != 0) return EFQAT_ERR_ALIGNMENT;
  const size_t dysz = io.dy_dtype == EFQAT_F32 ? 4 : 2;
  // the dY tile loads are 16-byte vectors when dY is used in place
  if (((uintptr_t)io.dy % 16) != 0 || ((uintptr_t)io.dy % dysz) != 0) return EFQAT_ERR_ALIGNMENT;
  if (((uintptr_t)io.x % (io.x_dtype == EFQAT_F32 ? 4 : 2)) != 0) return EFQAT_ERR_ALIGNMENT;
  if (((uintptr_t)io.dx % (io.dx_dtype == EFQAT_F32 ? 4 : 2)) != 0) return EFQAT_ERR_ALIGNMENT;
  if (((uintptr_t)io.w % 4) != 0 || ((uintptr_t)io.s_w % 4) != 0 || ((uintptr_t)io.dw % 4) != 0 ||
      ((uintptr_t)io.ds_w % 4) != 0 || ((uintptr_t)io.idx % 4) != 0 || ((uintptr_t)io.x_clip % 4) != 0 ||
      ((uintptr_t)io.w_clip % 4) != 0)
    return EFQAT_ERR_ALIGNMENT;
  return EFQAT_OK;
}

static int fill_step(const efqat_opt_step* step, float* w, float* s_w, StepArgs* out) {
  if (!step || !w || !s_w) return EFQAT_ERR_NULL_PTR;
  if (step->momentum != 0.0f && !step->mom_w) return EFQAT_ERR_NULL_PTR;
  if (!step->adam_m || !step->adam_v || !step->adam_t) return EFQAT_ERR_NULL_PTR;
  if (((uintptr_t)step->mom_w % 4) != 0 || ((uintptr_t)step->adam_m % 4) != 0 || ((uintptr_t)step->adam_v % 4) != 0 ||
      ((uintptr_t)step->adam_t % 4) != 0)
    return EFQAT_ERR_ALIGNMENT;
  // 0 <= beta < 1 (the bias correction divides by 1 - beta^t), eps >= 0
  if (!(step->beta1 >= 0.0f && step->beta1 < 1.0f) || !(step->beta2 >= 0.0f && step->beta2 < 1.0f) ||
      !(step->eps >= 0.0f))
    return EFQAT_ERR_BAD_LAYOUT;
  out->w = w; out->s_w = s_w;
  out->mom_w = step->momentum != 0.0f ? step->mom_w : nullptr;
  out->lr_w = step->lr_w; out->mu = step->momentum; out->wd = step->weight_decay;
  out->adam_m = step->adam_m; out->adam_v = step->adam_v; out->adam_t = step->adam_t;
  out->lr_s = step->lr_s; out->b1 = step->beta1; out->b2 = step->beta2; out->eps = step->eps;
  return EFQAT_OK;
}

// Upper limits of the linear entry points: tokens up to 2^30, channel counts below 2^24 (32-bit pointer steps)
static bool linear_shape_ok(int64_t T, int64_t c_in, int64_t c_out) {
  return T > 0 && c_in > 0 && c_out > 0 && T <= (1 << 30) && c_in < (1 << 24) && c_out < (1 << 24);
}

// All linear entry points end here: every check first, then the launches.
static int linear_bwd_entry(BwdIo& io, int64_t T, int64_t c_in, int64_t c_out, const efqat_opt_step* step, float* w_rw,
                            float* s_w_rw, int dxk, void* ws, size_t ws_bytes, void* stream) {
  if (!linear_shape_ok(T, c_in, c_out)) return EFQAT_ERR_BAD_SHAPE;
  int rc;
  if (step) {
    rc = fill_step(step, w_rw, s_w_rw, &io.sgd);
    if (rc) return rc;
  }
  rc = check_common(io, c_out, ws, dxk);
  if (rc) return rc;
  if (io.w_operand && dxk != EFQAT_DX_KERNEL_AUTO) return EFQAT_ERR_BAD_LAYOUT;   // the operand belongs to the default plan
  if (io.w_operand && ((uintptr_t)io.w_operand % 256) != 0) return EFQAT_ERR_ALIGNMENT;
  const BwdPlan p = choose_plan([&](bool wide) {
    return make_plan(T, T, c_in, c_out, 1, io.k, io.dy_dtype, io.dy_layout, false, dxk, nullptr, wide);
  }, c_in, io, ws_bytes);
  if (ws_bytes < p.total) return EFQAT_ERR_WORKSPACE;
  rc = check_plan(p, io, T, c_in, c_out);
  if (rc) return rc;
  return run_bwd(io, p, T, T, c_in, c_out, nullptr, ws, (hipStream_t)stream);
}

}  // namespace efqat

using namespace efqat;

extern "C" size_t efqat_linear_bwd_workspace_bytes_ex(int64_t T, int64_t c_in, int64_t c_out, int64_t k, int dy_dtype,
                                                      int dy_layout, int dx_kernel) {
  if (!linear_shape_ok(T, c_in, c_out) || k < 0 || k > c_out) return 0;
  if (dx_kernel < EFQAT_DX_KERNEL_AUTO || dx_kernel > EFQAT_DX_KERNEL_BF16_PINNED) return 0;
  return query_plan([&](bool wide) {
    return make_plan(T, T, c_in, c_out, 1, k, dy_dtype, dy_layout, false, dx_kernel, nullptr, wide);
  });
}

extern "C" size_t efqat_linear_bwd_workspace_bytes(int64_t T, int64_t c_in, int64_t c_out, int64_t k, int dy_dtype,
                                                   int dy_layout) {
  return efqat_linear_bwd_workspace_bytes_ex(T, c_in, c_out, k, dy_dtype, dy_layout, EFQAT_DX_KERNEL_AUTO);
}

extern "C" int efqat_linear_bwd(const void* dy, int dy_dtype, int dy_layout, int64_t T, int64_t c_in, int64_t c_out,
                                const uint8_t* x_codes, const uint32_t* x_clip, const void* x, int x_dtype,
                                const float* s_x, const float* z_x, const int8_t* w_codes, const uint32_t* w_clip,
                                const float* w, const float* s_w, const int32_t* idx, int64_t k, void* dx,
                                int dx_dtype, float* dw, int scatter, float* ds_w, float* ds_x, float* dz_x,
                                void* ws, size_t ws_bytes, void* stream) {
  BwdIo io{dy, dy_dtype, dy_layout, x_codes, x_clip, x, x_dtype, s_x, z_x, w_codes, w_clip, w, s_w, idx, k,
           dx, dx_dtype, dw, scatter, ds_w, ds_x, dz_x};
  return linear_bwd_entry(io, T, c_in, c_out, nullptr, nullptr, nullptr, EFQAT_DX_KERNEL_AUTO, ws, ws_bytes, stream);
}

extern "C" int efqat_linear_bwd_ex(const void* dy, int dy_dtype, int dy_layout, int64_t T, int64_t c_in, int64_t c_out,
                                   const uint8_t* x_codes, const uint32_t* x_clip, const void* x, int x_dtype,
                                   const float* s_x, const float* z_x, const int8_t* w_codes, const uint32_t* w_clip,
                                   float* w, float* s_w, const int32_t* idx, int64_t k, void* dx, int dx_dtype,
                                   float* dw, int scatter, float* ds_w, float* ds_x, float* dz_x,
                                   const void* w_operand, const efqat_opt_step* step, int dx_kernel, void* ws,
                                   size_t ws_bytes, void* stream, void* side_stream) {
  BwdIo io{dy, dy_dtype, dy_layout, x_codes, x_clip, x, x_dtype, s_x, z_x, w_codes, w_clip, w, s_w, idx, k,
           dx, dx_dtype, dw, scatter, ds_w, ds_x, dz_x};
  io.w_operand = w_operand;
  io.side = (hipStream_t)side_stream;
  return linear_bwd_entry(io, T, c_in, c_out, step, w, s_w, dx_kernel, ws, ws_bytes, stream);
}

static int plan_args(int64_t c_out, int64_t k, int dy_dtype, int dy_layout, int dxk, const int32_t* plan) {
  if (!plan) return EFQAT_ERR_NULL_PTR;
  if (k < 0 || k > c_out) return EFQAT_ERR_BAD_K;
  if (dy_dtype != EFQAT_F32 && dy_dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (dy_layout != EFQAT_DY_TOKEN_MAJOR && dy_layout != EFQAT_DY_CHANNEL_MAJOR) return EFQAT_ERR_BAD_LAYOUT;
  return dxk < EFQAT_DX_KERNEL_AUTO || dxk > EFQAT_DX_KERNEL_BF16_PINNED ? EFQAT_ERR_BAD_LAYOUT : EFQAT_OK;
}

extern "C" int efqat_linear_bwd_plan(int64_t T, int64_t c_in, int64_t c_out, int64_t k, int dy_dtype, int dy_layout,
                                     int dx_kernel, int32_t* plan) {
  if (!linear_shape_ok(T, c_in, c_out)) return EFQAT_ERR_BAD_SHAPE;
  const int rc = plan_args(c_out, k, dy_dtype, dy_layout, dx_kernel, plan);
  if (rc) return rc;
  return plan_info(make_plan(T, T, c_in, c_out, 1, k, dy_dtype, dy_layout, false, dx_kernel, nullptr, c_in > kMaxStagedColumns), false,
                   k, plan);
}

extern "C" int efqat_linear_bwd_dx_tile(int64_t T, int64_t c_in, int64_t c_out, int64_t k, int dy_dtype, int dy_layout, int dx_kernel,
                                        int side_stream, int32_t* tile) {
  if (!linear_shape_ok(T, c_in, c_out)) return EFQAT_ERR_BAD_SHAPE;
  const int rc = plan_args(c_out, k, dy_dtype, dy_layout, dx_kernel, tile);
  if (rc) return rc;
  const BwdPlan p = make_plan(T, T, c_in, c_out, 1, k, dy_dtype, dy_layout, false, dx_kernel, nullptr, c_in > kMaxStagedColumns);
  const int rows = p.dx8 ? p.dx8_tile : p.plan_dx.tile;
  tile[EFQAT_DX_TILE_ROWS] = rows;
  tile[EFQAT_DX_TILE_COLUMNS] = !p.dx8 ? rows : rows == 256 || (p.cmx && p.plan_dx.wide) ? 256 : 128;
  tile[EFQAT_DX_TILE_STAGES] = p.dx8 || !p.plan_dx.ring ? 2
                               : p.pair ? 3
                                        : kk_ring_stages(rows, (int64_t)p.plan_dx.tiles_m * p.plan_dx.tiles_n, c_in, p.Kx,
                                                         side_stream && takes_side_stream(p));
  return EFQAT_OK;
}

extern "C" size_t efqat_linear_bwd_weight_operand_bytes(int64_t T, int64_t c_in, int64_t c_out, int dy_dtype,
                                                        int dy_layout) {
  if (!linear_shape_ok(T, c_in, c_out)) return 0;
  const BwdPlan p = make_plan(T, T, c_in, c_out, 1, 0, dy_dtype, dy_layout, false, EFQAT_DX_KERNEL_AUTO, nullptr,
                              c_in > kMaxStagedColumns);
  return p.dx8 ? 0 : (size_t)round_up((int64_t)p.b_wqT, 256) + 256;   // W_q^T and 256 zero bytes (part of its format)
}

extern "C" int efqat_linear_bwd_weight_operand(const int8_t* w_codes, const float* s_w, int64_t T, int64_t c_in,
                                               int64_t c_out, int dy_dtype, int dy_layout, void* operand,
                                               size_t operand_bytes, void* stream) {
  if (!linear_shape_ok(T, c_in, c_out)) return EFQAT_ERR_BAD_SHAPE;
  if (dy_dtype != EFQAT_F32 && dy_dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (dy_layout != EFQAT_DY_TOKEN_MAJOR && dy_layout != EFQAT_DY_CHANNEL_MAJOR) return EFQAT_ERR_BAD_LAYOUT;
  const size_t need = efqat_linear_bwd_weight_operand_bytes(T, c_in, c_out, dy_dtype, dy_layout);
  if (need == 0) return EFQAT_OK;                      // this layer's dX product reads the int8 codes themselves
  if (!w_codes || !s_w || !operand) return EFQAT_ERR_NULL_PTR;
  if (operand_bytes < need) return EFQAT_ERR_WORKSPACE;
  if (((uintptr_t)operand % 256) != 0) return EFQAT_ERR_ALIGNMENT;
  if (c_in > kMaxStagedColumns) return EFQAT_ERR_BAD_SHAPE;
  const BwdPlan p = make_plan(T, T, c_in, c_out, 1, 0, dy_dtype, dy_layout, false, EFQAT_DX_KERNEL_AUTO, nullptr,
                              c_in > kMaxStagedColumns);
  PrepArgs a{};
  prep_w_operand(a, w_codes, s_w, c_in, c_out, 1, p.ldc, (bf16_t*)operand);
  a.zero_page = (uint32_t*)((char*)operand + round_up((int64_t)p.b_wqT, 256));
  hipStream_t st = (hipStream_t)stream;
  ProfScope prep(PROF_PREP, st);
  return launch_prep(a, EFQAT_BF16, st);
}

static int conv_geom(int64_t N, int64_t H, int64_t W, int64_t c_in, int64_t c_out, int64_t KH, int64_t KW,
                     int64_t stride, int64_t pad, ConvGeom* g) {
  if (N <= 0 || H <= 0 || W <= 0 || c_in <= 0 || c_out <= 0 || KH <= 0 || KW <= 0 || stride <= 0 || pad < 0)
    return EFQAT_ERR_BAD_SHAPE;
  if (N > (1 << 24) || H > (1 << 15) || W > (1 << 15) || c_in > (1 << 20) || c_out > (1 << 20) || KH > 64 || KW > 64 ||
      stride > 64 || pad > 64)
    return EFQAT_ERR_BAD_SHAPE;
  if (H + 2 * pad < KH || W + 2 * pad < KW) return EFQAT_ERR_BAD_SHAPE;
  g->N = (int)N; g->H = (int)H; g->W = (int)W; g->c_in = (int)c_in; g->c_out = (int)c_out;
  g->KH = (int)KH; g->KW = (int)KW; g->stride = (int)stride; g->pad = (int)pad;
  g->Ho = (int)((H + 2 * pad - KH) / stride + 1);
  g->Wo = (int)((W + 2 * pad - KW) / stride + 1);
  if ((int64_t)N * H * W > (1 << 30) || (int64_t)N * g->Ho * g->Wo > (1 << 30)) return EFQAT_ERR_BAD_SHAPE;
  return EFQAT_OK;
}

static bool conv_im2col(const ConvGeom& g) { return !(g.KH * g.KW == 1 && g.stride == 1 && g.pad == 0); }
static BwdPlan conv_plan(const ConvGeom& g, int64_t k, int dy_dtype, int dy_layout, int dxk, bool wide) {
  return make_plan((int64_t)g.N * g.H * g.W, (int64_t)g.N * g.Ho * g.Wo, g.c_in, g.c_out, g.KH * g.KW, k, dy_dtype,
                   dy_layout, conv_im2col(g), dxk, &g, wide);
}

extern "C" int efqat_conv_bwd_plan(int64_t N, int64_t H, int64_t W, int64_t c_in, int64_t c_out, int64_t KH, int64_t KW,
                                   int64_t stride, int64_t pad, int64_t k, int dy_dtype, int dy_layout, int dx_kernel,
                                   int32_t* plan) {
  ConvGeom g;
  int rc = conv_geom(N, H, W, c_in, c_out, KH, KW, stride, pad, &g);
  if (!rc) rc = plan_args(c_out, k, dy_dtype, dy_layout, dx_kernel, plan);
  if (rc) return rc;
  return plan_info(conv_plan(g, k, dy_dtype, dy_layout, dx_kernel, c_in > kMaxStagedColumns), conv_im2col(g), k, plan);
}

extern "C" size_t efqat_conv_bwd_workspace_bytes_ex(int64_t N, int64_t H, int64_t W, int64_t c_in, int64_t c_out,
                                                    int64_t KH, int64_t KW, int64_t stride, int64_t pad, int64_t k,
                                                    int dy_dtype, int dy_layout, int dx_kernel) {
  ConvGeom g;
  if (conv_geom(N, H, W, c_in, c_out, KH, KW, stride, pad, &g) || k < 0 || k > c_out) return 0;
  if (dx_kernel < EFQAT_DX_KERNEL_AUTO || dx_kernel > EFQAT_DX_KERNEL_BF16_PINNED) return 0;
  return query_plan([&](bool wide) { return conv_plan(g, k, dy_dtype, dy_layout, dx_kernel, wide); });
}

extern "C" size_t efqat_conv_bwd_workspace_bytes(int64_t N, int64_t H, int64_t W, int64_t c_in, int64_t c_out,
                                                 int64_t KH, int64_t KW, int64_t stride, int64_t pad, int64_t k,
                                                 int dy_dtype, int dy_layout) {
  return efqat_conv_bwd_workspace_bytes_ex(N, H, W, c_in, c_out, KH, KW, stride, pad, k, dy_dtype, dy_layout,
                                           EFQAT_DX_KERNEL_AUTO);
}

static int conv_bwd_entry(BwdIo& io, int64_t N, int64_t H, int64_t W, int64_t c_in, int64_t c_out, int64_t KH,
                          int64_t KW, int64_t stride, int64_t pad, const efqat_opt_step* step, float* w_rw,
                          float* s_w_rw, int dxk, void* ws, size_t ws_bytes, void* stream) {
  ConvGeom g;
  int rc = conv_geom(N, H, W, c_in, c_out, KH, KW, stride, pad, &g);
  if (rc) return rc;
  if (step) {
    rc = fill_step(step, w_rw, s_w_rw, &io.sgd);
    if (rc) return rc;
  }
  rc = check_common(io, c_out, ws, dxk);
  if (rc) return rc;
  const BwdPlan p = choose_plan([&](bool wide) {
    return conv_plan(g, io.k, io.dy_dtype, io.dy_layout, dxk, wide);
  }, c_in, io, ws_bytes);
  if (ws_bytes < p.total) return EFQAT_ERR_WORKSPACE;
  const int64_t T_in = (int64_t)N * H * W, T_out = (int64_t)N * g.Ho * g.Wo;
  rc = check_plan(p, io, T_out, c_in, c_out);
  if (rc) return rc;
  return run_bwd(io, p, T_in, T_out, c_in, c_out, &g, ws, (hipStream_t)stream);
}

extern "C" int efqat_conv_bwd(const void* dy, int dy_dtype, int dy_layout, int64_t N, int64_t H, int64_t W,
                              int64_t c_in, int64_t c_out, int64_t KH, int64_t KW, int64_t stride, int64_t pad,
                              const uint8_t* x_codes, const uint32_t* x_clip, const void* x, int x_dtype,
                              const float* s_x, const float* z_x, const int8_t* w_codes, const uint32_t* w_clip,
                              const float* w, const float* s_w, const int32_t* idx, int64_t k, void* dx,
                              int dx_dtype, float* dw, int scatter, float* ds_w, float* ds_x, float* dz_x, void* ws,
                              size_t ws_bytes, void* stream) {
  BwdIo io{dy, dy_dtype, dy_layout, x_codes, x_clip, x, x_dtype, s_x, z_x, w_codes, w_clip, w, s_w, idx, k,
           dx, dx_dtype, dw, scatter, ds_w, ds_x, dz_x};
  return conv_bwd_entry(io, N, H, W, c_in, c_out, KH, KW, stride, pad, nullptr, nullptr, nullptr,
                        EFQAT_DX_KERNEL_AUTO, ws, ws_bytes, stream);
}

extern "C" int efqat_conv_bwd_ex(const void* dy, int dy_dtype, int dy_layout, int64_t N, int64_t H, int64_t W,
                                 int64_t c_in, int64_t c_out, int64_t KH, int64_t KW, int64_t stride, int64_t pad,
                                 const uint8_t* x_codes, const uint32_t* x_clip, const void* x, int x_dtype,
                                 const float* s_x, const float* z_x, const int8_t* w_codes, const uint32_t* w_clip,
                                 float* w, float* s_w, const int32_t* idx, int64_t k, void* dx, int dx_dtype,
                                 float* dw, int scatter, float* ds_w, float* ds_x, float* dz_x,
                                 const efqat_opt_step* step, int dx_kernel, void* ws, size_t ws_bytes, void* stream,
                                 void* side_stream) {
  BwdIo io{dy, dy_dtype, dy_layout, x_codes, x_clip, x, x_dtype, s_x, z_x, w_codes, w_clip, w, s_w, idx, k,
           dx, dx_dtype, dw, scatter, ds_w, ds_x, dz_x};
  io.side = (hipStream_t)side_stream;
  return conv_bwd_entry(io, N, H, W, c_in, c_out, KH, KW, stride, pad, step, w, s_w, dx_kernel, ws, ws_bytes, stream);
}
