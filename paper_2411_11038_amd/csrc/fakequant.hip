// Fake-quant forward (Eq. 1-4): quantizer statistics, integer codes, straight-through clip masks.
// All kernels are HBM-bound streaming passes built on 64-wide wavefront reductions.
#include "common.hpp"

#include <algorithm>
#include <type_traits>

namespace efqat {

// ----------------------------------------------------------------------------------------------
// 8 consecutive elements as fp32 (vector path: one 16-byte load for bf16, two for fp32)
template <typename T>
__device__ __forceinline__ void load8(const T* p, float (&v)[8]);
template <>
__device__ __forceinline__ void load8<float>(const float* p, float (&v)[8]) {
  float4 a = *reinterpret_cast<const float4*>(p);
  float4 b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
__device__ __forceinline__ void load8<bf16_t>(const bf16_t* p, float (&v)[8]) {
  uint4 a = *reinterpret_cast<const uint4*>(p);
  uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}

// the same at any element alignment, which the hardware takes for vector accesses.  Loaded as vectors: of a copy to an array the compiler
// takes an element away to share its load with the branch that reads by elements, and another load is issued (60000 x 1000 fp32
// codes 55.8 us so, 49.1).
template <typename T>
__device__ __forceinline__ void load8_any(const T* p, float (&v)[8]) {
  if constexpr (sizeof(T) == 4) {
    typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
    const vec a = *reinterpret_cast<const vec*>(p), b = *reinterpret_cast<const vec*>(p + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
  } else {
    typedef uint32_t vec __attribute__((ext_vector_type(4), aligned(2)));
    const vec w = *reinterpret_cast<const vec*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
}

// ----------------------------------------------------------------------------------------------
// Eq. 2 range: alpha = min x, beta = max x over the whole tensor (MinMax observer).
constexpr int kMaxParts = 1024;
template <typename T>
__global__ __launch_bounds__(256) void k_minmax_partial(const T* __restrict__ x, int64_t n, int vec,
                                                        float* __restrict__ part) {
  float lo = INFINITY, hi = -INFINITY;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
  if (vec) {
    const int64_t n8 = n >> 3;
    int64_t i = tid;
    // four 16-byte (bf16) / 32-byte (fp32) loads in flight per lane: with one, a CU has too few bytes outstanding to
    // cover the memory latency at the HBM rate
    for (; i + 3 * nthreads < n8; i += 4 * nthreads) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) load8<T>(x + (i + u * nthreads) * 8, v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) { lo = fminf(lo, v[u][j]); hi = fmaxf(hi, v[u][j]); }
    }
    for (; i < n8; i += nthreads) {
      float v[8];
      load8<T>(x + i * 8, v);
#pragma unroll
      for (int j = 0; j < 8; ++j) { lo = fminf(lo, v[j]); hi = fmaxf(hi, v[j]); }
    }
    for (i = (n8 << 3) + tid; i < n; i += nthreads) {
      float v = load_as_f32<T>(x, i);
      lo = fminf(lo, v); hi = fmaxf(hi, v);
    }
  } else {
    for (int64_t i = tid; i < n; i += nthreads) {
      float v = load_as_f32<T>(x, i);
      lo = fminf(lo, v); hi = fmaxf(hi, v);
    }
  }
  lo = wave_min(lo); hi = wave_max(hi);
  __shared__ float s_lo[4], s_hi[4];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { s_lo[w] = lo; s_hi[w] = hi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = fminf(fminf(s_lo[0], s_lo[1]), fminf(s_lo[2], s_lo[3]));
    part[2 * blockIdx.x + 1] = fmaxf(fmaxf(s_hi[0], s_hi[1]), fmaxf(s_hi[2], s_hi[3]));
  }
}

// Eq. 2: S_x = (beta - alpha) / (2^b - 1), Z_x = -round(alpha / S_x), each a single-precision op, from the partial ranges:
// by every block of the kernel that makes the codes, for itself (minima and maxima do not depend on an order), and written
// once.  The partials are at most 8 KiB, in L2; in k_quantize_act_flat the first loads of x are in flight meanwhile.  A launch of
// one block in between was 2 to 4.5 us, this is 0.6 to 2.5: 65536 fp32 values 7.6 -> 6.2 us in all, 3.2 M bf16 9.8 -> 8.6,
// 9.4 M 12.7 -> 12.1, 33.5 M 33.5 -> 32.4, 33.5 M fp32 51.4 -> 49.4.  Ragged rows: see run_fakequant.
__device__ __forceinline__ void act_qparams_block(const float* __restrict__ part, int nparts, int bits, float* s_out,
                                                  float* z_out, float* __restrict__ scale, float* __restrict__ zp) {
  float lo = INFINITY, hi = -INFINITY;
  float2 p[kMaxParts / 256];
#pragma unroll
  for (int u = 0; u < kMaxParts / 256; ++u) {
    const int i = threadIdx.x + 256 * u;
    p[u] = i < nparts ? *reinterpret_cast<const float2*>(part + 2 * i) : make_float2(INFINITY, -INFINITY);
  }
#pragma unroll
  for (int u = 0; u < kMaxParts / 256; ++u) { lo = fminf(lo, p[u].x); hi = fmaxf(hi, p[u].y); }
  lo = wave_min(lo); hi = wave_max(hi);
  __shared__ float s_lo[4], s_hi[4];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { s_lo[w] = lo; s_hi[w] = hi; }
  __syncthreads();
  const float alpha = fminf(fminf(s_lo[0], s_lo[1]), fminf(s_lo[2], s_lo[3]));
  const float beta = fmaxf(fmaxf(s_hi[0], s_hi[1]), fmaxf(s_hi[2], s_hi[3]));
  const float qmax = (float)((1 << bits) - 1);
  float s = __fdiv_rn(__fsub_rn(beta, alpha), qmax);
  if (!(s > 0.0f)) s = 1.0f;                         // zero range
  const float z = 0.0f - rintf(__fdiv_rn(alpha, s));
  if (blockIdx.x == 0 && threadIdx.x == 0) { scale[0] = s; zp[0] = z; }
  *s_out = s; *z_out = rintf(z);
}
__global__ __launch_bounds__(256) void k_act_qparams(const float* __restrict__ part, int nparts, int bits,
                                                     float* __restrict__ scale, float* __restrict__ zp) {
  float s, z;
  act_qparams_block(part, nparts, bits, &s, &z, scale, zp);
}

// ----------------------------------------------------------------------------------------------
// round(x / s) as the round-to-nearest-even integer of the correctly rounded quotient.  x * (1/s) is within
// 1.5 ulp of it, so the two round to the same integer unless x/s sits that close to a half-way point; only
// then is the exact (slow) division needed (always for huge quotients, where the tolerance exceeds one half,
// and for a scale so small that its reciprocal overflows).
__device__ __forceinline__ float round_quotient(float x, float s, float inv_s) {
  const float qf = x * inv_s;
  float r = rintf(qf);
  const float tol = 2.5e-7f * fabsf(qf);
  if (!(0.5f - fabsf(qf - r) > tol) || !(inv_s < 3.0e38f)) r = rintf(__fdiv_rn(x, s));
  return r;
}

// ----------------------------------------------------------------------------------------------
// Eq. 1 / Eq. 3: codes + clip-mask bits (+ optional de-quantised bf16 values).
// One wavefront handles one 512-element segment of one row per iteration; a lane owns 8
// consecutive elements, four neighbouring lanes assemble one 32-bit mask word.  Rows of any length and alignment: whole chunks are
// one vector access, only the one that ends a row is read and written by elements.  With an access per element unless rows were
// aligned and of whole chunks it took, codes alone / with the range, us: 12000 x 7777 fp32 215 / 282 (now 97 / 161), bf16 161 / 152
// (68 / 96), 3000 x 12001 fp32 76 / 101 (29 / 54), 2049 x 777 fp32 6.3 / 10.0 (4.5 / 8.4), 20000 x 7 the same; rows of
// 31 to 127 fp32 values, whose one wavefront takes both ways, up to 6 % slower (952380 x 63 326 / 365, now 348 / 369), of 100 bf16 16 % faster.
// Activations: part, when given, are the partial ranges that scale and zero point are made from here.
// INIT (weights only): the wavefront first takes the row's abs-max and writes its Eq. 4 scale
// S_w[c] = max_j |w[c][j]| / (2^(b-1) - 1), then quantizes the row it has just pulled through the caches.
template <typename T, int MODE, bool INIT>
__global__ __launch_bounds__(256) void k_quantize(const T* __restrict__ x, int64_t rows, int64_t cols, int bits, float* __restrict__ scale,
                                                  float* __restrict__ zp, uint8_t* __restrict__ codes,
                                                  uint32_t* __restrict__ clip, bf16_t* __restrict__ xq,
                                                  const float* __restrict__ part, int nparts) {
  const int lane = threadIdx.x & 63;
  const int64_t segs = ceil_div(cols, 512);
  const int64_t total = rows * segs;
  const int64_t wpr = ceil_div(cols, 32);
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  float lo, hi, z = 0.0f, s_act = 1.0f;
  if (MODE == EFQAT_QUANT_ACT_PER_TENSOR_ASYM) {
    lo = 0.0f; hi = (float)((1 << bits) - 1);
    if (part) {
      act_qparams_block(part, nparts, bits, &s_act, &z, scale, zp);
    } else {
      s_act = scale[0];
      z = rintf(zp[0]);
    }
  } else {
    hi = (float)((1 << (bits - 1)) - 1); lo = -hi;
  }
  // work item = (row, 512-element segment); with INIT a wavefront keeps the whole row (one abs-max scan, then
  // all its segments) so the row is read from HBM once
  const int64_t nitems = INIT ? rows : total;
  for (int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); item < nitems; item += nwaves) {
   const int64_t row = INIT ? item : item / segs;
   float s_row = 1.0f;
   if (INIT) {
     const T* p = x + row * cols;
     float m = 0.0f;
     const int64_t n8 = cols >> 3;
     for (int64_t i = lane; i < n8; i += 64) {
       float t8[8];
       load8_any<T>(p + i * 8, t8);
#pragma unroll
       for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(t8[j]));
     }
     for (int64_t i = n8 * 8 + lane; i < cols; i += 64) m = fmaxf(m, fabsf(load_as_f32<T>(p, i)));
     m = wave_max(m);
     s_row = __fdiv_rn(m, hi);
     if (!(s_row > 0.0f)) s_row = 1.0f;             // all-zero row
     if (lane == 0) scale[row] = s_row;
   }
   for (int64_t seg = INIT ? 0 : item - row * segs; seg < (INIT ? segs : item - row * segs + 1); ++seg) {
    const int64_t col0 = seg * 512 + (int64_t)lane * 8;
    float s;
    if (MODE == EFQAT_QUANT_ACT_PER_TENSOR_ASYM) s = s_act;
    else if (INIT) s = s_row;
    else s = scale[row];
    const float inv_s = __fdiv_rn(1.0f, s);
    const int64_t base = row * cols + col0;
    float v[8];
    const bool full = col0 + 8 <= cols;
    if (full) {
      load8_any<T>(x + base, v);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (col0 + j < cols) ? load_as_f32<T>(x, base + j) : 0.0f;
    }
    uint32_t bits8 = 0;
    uint32_t cw[2] = {0u, 0u};
    float dq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float c = round_quotient(v[j], s, inv_s) + z;   // un-clamped code
      const float cc = __builtin_amdgcn_fmed3f(c, lo, hi);
      const bool inr = (c == cc);                  // closed interval: a code on the bound is not clipped
      if (inr && (col0 + j < cols)) bits8 |= (1u << j);
      if (MODE == EFQAT_QUANT_ACT_PER_TENSOR_ASYM)
        cw[j >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(cc, j & 3, cw[j >> 2]);   // cc is an integer in [0, 255]
      else
        cw[j >> 2] |= ((uint32_t)((int)cc & 0xFF)) << (8 * (j & 3));
      dq[j] = s * (cc - z);
    }
    if (full) {
      __builtin_memcpy(codes + base, cw, 8);
      if (xq) {
        const uint32_t o[4] = {pack_bf16x2(dq[0], dq[1]), pack_bf16x2(dq[2], dq[3]), pack_bf16x2(dq[4], dq[5]),
                               pack_bf16x2(dq[6], dq[7])};
        __builtin_memcpy(xq + base, o, 16);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (col0 + j < cols) {
          codes[base + j] = (uint8_t)((cw[j >> 2] >> (8 * (j & 3))) & 0xFF);
          if (xq) xq[base + j] = f32_to_bf16(dq[j]);
        }
      }
    }
    uint32_t word = bits8 << (8 * (lane & 3));
    word |= __shfl_xor(word, 1, kWave);
    word |= __shfl_xor(word, 2, kWave);
    const int64_t widx = col0 >> 5;
    if ((lane & 3) == 0 && widx < wpr) clip[row * wpr + widx] = word;
   }
  }
}

// Eq. 1 for a per-tensor quantizer whose rows are a whole number of 32-element mask words (cols % 32 == 0, aligned
// pointers): the tensor is one flat run of 8-element chunks, codes and mask words are flat as well, so no lane idles
// on a ragged segment and nothing is divided.  Each lane handles two chunks a grid-stride apart per iteration, both
// loads issued before either is used.
// RANGE: scale and zero point are made here, from the partial ranges.
template <typename T, bool RANGE>
__global__ __launch_bounds__(256) void k_quantize_act_flat(const T* __restrict__ x, int64_t nchunks, int bits,
                                                           float* __restrict__ scale, float* __restrict__ zp,
                                                           uint8_t* __restrict__ codes, uint32_t* __restrict__ clip,
                                                           bf16_t* __restrict__ xq, const float* __restrict__ part,
                                                           int nparts) {
  const int lane = threadIdx.x & 63;
  const float hi = (float)((1 << bits) - 1);
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t c0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int64_t c = c0;
  float v0[8], v1[8];                                  // RANGE: the first two chunks, requested ahead of the range
  float s, z;
  if constexpr (RANGE) {
    if (c0 < nchunks) load8<T>(x + c0 * 8, v0);
    if (c0 + stride < nchunks) load8<T>(x + (c0 + stride) * 8, v1);
    act_qparams_block(part, nparts, bits, &s, &z, scale, zp);
  } else {
    s = scale[0];
    z = rintf(zp[0]);
  }
  const float inv_s = __fdiv_rn(1.0f, s);
  auto finish = [&](int64_t c, const float (&v)[8]) {
    uint32_t bits8 = 0;
    uint32_t cw[2] = {0u, 0u};
    float dq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float cu = round_quotient(v[j], s, inv_s) + z;
      const float cc = __builtin_amdgcn_fmed3f(cu, 0.0f, hi);
      if (cu == cc) bits8 |= (1u << j);
      cw[j >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(cc, j & 3, cw[j >> 2]);
      dq[j] = s * (cc - z);
    }
    *reinterpret_cast<uint2*>(codes + c * 8) = make_uint2(cw[0], cw[1]);
    if (xq)
      *reinterpret_cast<uint4*>(xq + c * 8) = make_uint4(pack_bf16x2(dq[0], dq[1]), pack_bf16x2(dq[2], dq[3]),
                                                         pack_bf16x2(dq[4], dq[5]), pack_bf16x2(dq[6], dq[7]));
    // chunks c .. c+3 of lanes 4m .. 4m+3 make one mask word (c of lane 4m is a multiple of 4: see the launch)
    uint32_t word = bits8 << (8 * (lane & 3));
    word |= __shfl_xor(word, 1, kWave);
    word |= __shfl_xor(word, 2, kWave);
    if ((lane & 3) == 0) clip[c >> 2] = word;
  };
  // the grid covers whole groups of four chunks: nchunks % 4 == 0 and the stride is a multiple of 4, so the four
  // lanes of a mask word are in range together
  if constexpr (RANGE) {
    if (c + stride < nchunks) {
      finish(c, v0);
      finish(c + stride, v1);
      c += 2 * stride;
    } else if (c < nchunks) {
      finish(c, v0);
      return;
    }
  }
  for (; c + stride < nchunks; c += 2 * stride) {
    load8<T>(x + c * 8, v0);
    load8<T>(x + (c + stride) * 8, v1);
    finish(c, v0);
    finish(c + stride, v1);
  }
  if (c < nchunks) {
    load8<T>(x + c * 8, v0);
    finish(c, v0);
  }
}

// Eq. 3 (and Eq. 4 with INIT) with the row held in registers (weights, cols <= 8 * 64 * WPR * NIT <= 16384): WPR wavefronts
// per row (1, or the 4 of a block when there are few rows) issue all loads of the row at once, take the abs-max and write
// S_w[c] (INIT), sum |w| in double precision for Eq. 6, and quantize from the registers, so the row is read once and the
// reads are not a chain of dependent round trips.  RAG: rows of any length and alignment; a lane's 8 values are one vector
// access all the same (the hardware takes them at element alignment), except in the chunk that ends a row.
// 1001 x 777 with scales from the data 5.0 us, 768 x 768 and 11008 x 4096 with given scales 3.8 and 40 us; a wavefront that
// walked the row twice, or a kernel over 512-element segments, and a second kernel for the sums took 11.2, 6.6 and 62 us.  Long
// ragged rows hold up to 134 registers a lane (three wavefronts a SIMD) and gain all the same, with the selection behind it:
// 1664 x 8250 27 us (119), 5552 x 13219 108 (387).
template <int NIT, int WPR, bool INIT, bool RAG>
__global__ __launch_bounds__(256) void k_quantize_w_row(const float* __restrict__ w, int64_t rows, int64_t cols, int bits,
                                                        float* __restrict__ scale, int8_t* __restrict__ codes,
                                                        uint32_t* __restrict__ clip, double* __restrict__ scores) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = WPR == 4 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wave;
  const int part = WPR == 4 ? wave : 0;               // which quarter of the row's chunks (interleaved by 64)
  const bool on = row < rows;                         // WPR == 1: whole wavefronts beyond the last row idle
  const float hi = (float)((1 << (bits - 1)) - 1), lo = -hi;
  const int n8 = on ? (int)((cols + 7) >> 3) : 0;     // chunks, the last one possibly shorter (RAG)
  const float* p = w + (on ? row : 0) * cols;
  float v[NIT][8];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = (it * WPR + part) * 64 + lane;
    if constexpr (RAG) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[it][j] = 0.0f;
      if ((int64_t)i * 8 + 8 <= cols && i < n8) __builtin_memcpy(v[it], p + (int64_t)i * 8, 32);
      else if (i < n8) {
#pragma unroll
        for (int j = 0; j < 7; ++j)
          if ((int64_t)i * 8 + j < cols) v[it][j] = p[(int64_t)i * 8 + j];
      }
    } else {
      if (i < n8) load8<float>(p + (int64_t)i * 8, v[it]);
    }
  }
  float s;
  if constexpr (!INIT) s = on ? scale[row] : 1.0f;
  float m = 0.0f;
  if constexpr (INIT) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (RAG || (it * WPR + part) * 64 + lane < n8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(v[it][j]));
      }
    }
    m = wave_max(m);
  }
  // optional by-product (Eq. 6): the row's mean |w| in double precision, fixed summation order, from the registers
  double asum = 0.0;
  if (scores) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (RAG || (it * WPR + part) * 64 + lane < n8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) asum += (double)fabsf(v[it][j]);
      }
    }
    asum = wave_sum(asum);
  }
  if (WPR == 4 && (INIT || scores)) {
    __shared__ float s_m[4];
    __shared__ double s_a[4];
    if (lane == 0) { s_m[wave] = m; s_a[wave] = asum; }
    __syncthreads();
    m = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
    asum = (s_a[0] + s_a[1]) + (s_a[2] + s_a[3]);
  }
  if (scores && on && lane == 0 && part == 0) scores[row] = asum / (double)cols;
  if constexpr (INIT) {
    s = __fdiv_rn(m, hi);
    if (!(s > 0.0f)) s = 1.0f;                        // all-zero row
    if (on && lane == 0 && part == 0) scale[row] = s;
  }
  const float inv_s = __fdiv_rn(1.0f, s);
  const int64_t wpr = (cols + 31) >> 5;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = (it * WPR + part) * 64 + lane;
    uint32_t bits8 = 0;
    uint32_t cw[2] = {0u, 0u};
    // n8 % 4 == 0 without RAG: the four lanes of a mask word are in range together
    if (RAG || i < n8) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float cu = round_quotient(v[it][j], s, inv_s);
        const float cc = __builtin_amdgcn_fmed3f(cu, lo, hi);
        if (cu == cc && (!RAG || (int64_t)i * 8 + j < cols)) bits8 |= (1u << j);
        cw[j >> 2] |= ((uint32_t)((int)cc & 0xFF)) << (8 * (j & 3));
      }
      int8_t* c = codes + row * cols + (int64_t)i * 8;
      if (!RAG) *reinterpret_cast<uint2*>(c) = make_uint2(cw[0], cw[1]);
      else if (i < n8) {
        if ((int64_t)i * 8 + 8 <= cols) __builtin_memcpy(c, cw, 8);
        else {
#pragma unroll
          for (int j = 0; j < 7; ++j)
            if ((int64_t)i * 8 + j < cols) c[j] = (int8_t)(cw[j >> 2] >> (8 * (j & 3)));
        }
      }
      uint32_t word = i < n8 ? bits8 << (8 * (lane & 3)) : 0u;
      word |= __shfl_xor(word, 1, kWave);
      word |= __shfl_xor(word, 2, kWave);
      if ((lane & 3) == 0 && i < n8) clip[row * wpr + (i >> 2)] = word;
    }
  }
}

// ----------------------------------------------------------------------------------------------
static inline bool aligned_to(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// scores (weights only): where the row-in-registers kernel runs, it also writes the Eq. 6 importance of every row and
// *scores_done is set; otherwise the caller computes them in a pass of its own.
template <typename T>
static int run_fakequant(const T* x, int64_t rows, int64_t cols, int mode, int bits, int init_minmax,
                         float* scale, float* zp, void* codes, uint32_t* clip, bf16_t* xq, void* ws,
                         hipStream_t st, double* scores = nullptr, bool* scores_done = nullptr) {
  const int64_t n = rows * cols;
  ProfScope prof(mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM ? PROF_QACT : PROF_QW, st);
  const int vec_flat = aligned_to(x, 16) ? 1 : 0;
  const int vec_row = (vec_flat && cols % 8 == 0 && aligned_to(codes, 8) && (!xq || aligned_to(xq, 16))) ? 1 : 0;
  float* part = nullptr;                               // partial ranges of an activation tensor
  int nparts = 0;
  if (init_minmax && mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM) {
    const int64_t np64 = ceil_div(n, 256 * 16);
    nparts = (int)(np64 < kMaxParts ? np64 : kMaxParts);
    part = (float*)ws;
    hipLaunchKernelGGL((k_minmax_partial<T>), dim3(nparts), dim3(256), 0, st, x, n, vec_flat, part);
    EFQAT_LAUNCH_CHECK();
  }
  const bool row_items = init_minmax && mode == EFQAT_QUANT_W_PER_ROW_SYM;   // one wavefront per row
  const int64_t items = row_items ? rows : rows * ceil_div(cols, 512);
  int64_t blocks = ceil_div(items, 4);
  const bool flat = mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM && vec_row && (cols % 32) == 0;
  // Ragged rows with the range to make: every block makes scale and zero point, in two rounds of the blocks that are resident at a time;
  // or, where there are many segments and too little work behind the range in a block to repay it, a launch of its own does, and
  // more blocks balance better.  us so / in every block: fp32 100000 x 100 46.2 / 48.4, 12000 x 400 14.0 / 14.7, 30000 x 700 (350 of 512
  // values a segment) 38.9 / 39.9, but 50000 x 511 46.5 / 45.5, 16384 x 1000 30.2 / 29.5; bf16 12000 x 400 13.0 / 13.8, 19584 x 1496
  // 35.6 / 36.4, 12000 x 7777 101 / 105; 10000 x 63 (2500 blocks) the same.
  if (part && !flat && blocks > 256 * 10 && (sizeof(T) == 2 || n < 450 * items)) {
    hipLaunchKernelGGL(k_act_qparams, dim3(1), dim3(256), 0, st, part, nparts, bits, scale, zp);
    EFQAT_LAUNCH_CHECK();
    part = nullptr;
  }
  const int64_t most_rows = part ? 256 * 16 : 256 * 32;
  if (blocks > most_rows) blocks = most_rows;
  // weights, few rows or long rows: a block per row, so that the chip still holds enough wavefronts to cover the memory
  // latency and a lane holds at most 64 values
  const bool wide = (rows < 4096 && cols > 8 * 64) || cols > 8 * 64 * 8;
  if (flat) {
    const int64_t nchunks = n / 8;
    int64_t fb = ceil_div(nchunks, 512);             // two chunks per lane and iteration
    // with the range to make, blocks that are all resident at a time (8192 x 4096 bf16 32.4 us; four blocks a CU 35.1, eight 33.0,
    // sixteen 33.8, and 33.5 with a launch for the range between)
    const int64_t most = part ? 256 * 6 : 256 * 16;
    if (fb > most) fb = most;
    if (part)
      hipLaunchKernelGGL((k_quantize_act_flat<T, true>), dim3((unsigned)fb), dim3(256), 0, st, x, nchunks, bits, scale, zp,
                         (uint8_t*)codes, clip, xq, part, nparts);
    else
      hipLaunchKernelGGL((k_quantize_act_flat<T, false>), dim3((unsigned)fb), dim3(256), 0, st, x, nchunks, bits, scale, zp,
                         (uint8_t*)codes, clip, xq, part, nparts);
  } else if (mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM)
    hipLaunchKernelGGL((k_quantize<T, EFQAT_QUANT_ACT_PER_TENSOR_ASYM, false>), dim3((unsigned)blocks), dim3(256), 0,
                       st, x, rows, cols, bits, scale, zp, (uint8_t*)codes, clip, xq, part, nparts);
  // (a grid dimension holds less than 2^32 work items)
  else if ((init_minmax || scores) && std::is_same<T, float>::value && cols <= 8 * 64 * 4 * 8 && !xq &&
           rows < (wide ? 1 << 24 : 1 << 26)) {
    const bool rag = !vec_row || (cols % 32) != 0;
    const float* wf = (const float*)x;
    int8_t* cd = (int8_t*)codes;
    const int per_wave = (int)ceil_div(cols, 8 * 64 * (wide ? 4 : 1));     // 8-element chunks per lane
    const dim3 grid((unsigned)(wide ? rows : ceil_div(rows, 4)));
    auto row_kernel = [&](auto nit, auto wpr) {
      constexpr int NIT = decltype(nit)::value, WPR = decltype(wpr)::value;
      auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, wf, rows, cols, bits, scale, cd, clip, scores); };
      if (init_minmax) { if (rag) go(k_quantize_w_row<NIT, WPR, true, true>); else go(k_quantize_w_row<NIT, WPR, true, false>); }
      else { if (rag) go(k_quantize_w_row<NIT, WPR, false, true>); else go(k_quantize_w_row<NIT, WPR, false, false>); }
    };
    using W1 = std::integral_constant<int, 1>;
    using W2 = std::integral_constant<int, 2>;
    using W4 = std::integral_constant<int, 4>;
    using W6 = std::integral_constant<int, 6>;
    using W8 = std::integral_constant<int, 8>;
    if (wide) {
      if (per_wave <= 1) row_kernel(W1{}, W4{}); else if (per_wave <= 2) row_kernel(W2{}, W4{});
      else if (per_wave <= 4) row_kernel(W4{}, W4{}); else if (per_wave <= 6) row_kernel(W6{}, W4{}); else row_kernel(W8{}, W4{});
    } else {
      if (per_wave <= 2) row_kernel(W2{}, W1{}); else if (per_wave <= 4) row_kernel(W4{}, W1{}); else row_kernel(W8{}, W1{});
    }
    if (scores && scores_done) *scores_done = true;
  } else if (init_minmax)
    hipLaunchKernelGGL((k_quantize<T, EFQAT_QUANT_W_PER_ROW_SYM, true>), dim3((unsigned)blocks), dim3(256), 0, st, x,
                       rows, cols, bits, scale, zp, (uint8_t*)codes, clip, xq, nullptr, 0);
  else
    hipLaunchKernelGGL((k_quantize<T, EFQAT_QUANT_W_PER_ROW_SYM, false>), dim3((unsigned)blocks), dim3(256), 0, st, x,
                       rows, cols, bits, scale, zp, (uint8_t*)codes, clip, xq, nullptr, 0);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

}  // namespace efqat

using namespace efqat;

extern "C" size_t efqat_fakequant_fwd_workspace_bytes(int64_t rows, int64_t cols, int mode) {
  (void)rows; (void)cols;
  return mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM ? (size_t)(kMaxParts * 2 * sizeof(float)) : (size_t)256;
}

extern "C" int efqat_fakequant_fwd(const void* x, int dtype, int64_t rows, int64_t cols, int mode, int bits,
                                   int init_minmax, float* scale, float* zero_point, void* codes,
                                   uint32_t* clip_bits, void* xq, void* ws, size_t ws_bytes, void* stream) {
  if (mode != EFQAT_QUANT_ACT_PER_TENSOR_ASYM && mode != EFQAT_QUANT_W_PER_ROW_SYM) return EFQAT_ERR_BAD_LAYOUT;
  if (dtype != EFQAT_F32 && dtype != EFQAT_BF16) return EFQAT_ERR_BAD_DTYPE;
  if (rows <= 0 || cols <= 0 || rows > (INT64_MAX / cols)) return EFQAT_ERR_BAD_SHAPE;
  if (bits < 2 || bits > 8) return EFQAT_ERR_BAD_BITS;
  if (!x || !scale || !codes || !clip_bits) return EFQAT_ERR_NULL_PTR;
  if (mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM && !zero_point) return EFQAT_ERR_NULL_PTR;
  if (init_minmax && mode == EFQAT_QUANT_ACT_PER_TENSOR_ASYM) {
    if (!ws) return EFQAT_ERR_NULL_PTR;
    if (ws_bytes < efqat_fakequant_fwd_workspace_bytes(rows, cols, mode)) return EFQAT_ERR_WORKSPACE;
    if (((uintptr_t)ws % 256) != 0) return EFQAT_ERR_ALIGNMENT;
  }
  const size_t esz = dtype == EFQAT_F32 ? 4 : 2;
  if (((uintptr_t)x % esz) != 0 || ((uintptr_t)clip_bits % 4) != 0 || (xq && ((uintptr_t)xq % 2) != 0))
    return EFQAT_ERR_ALIGNMENT;
  hipStream_t st = (hipStream_t)stream;
  if (dtype == EFQAT_F32)
    return run_fakequant<float>((const float*)x, rows, cols, mode, bits, init_minmax, scale, zero_point, codes,
                                clip_bits, (bf16_t*)xq, ws, st);
  return run_fakequant<bf16_t>((const bf16_t*)x, rows, cols, mode, bits, init_minmax, scale, zero_point, codes,
                               clip_bits, (bf16_t*)xq, ws, st);
}

// Weight side of one step in a single call: Eq. 4 + Eq. 3 (codes, clip mask, scales), Eq. 6 and the Top-K.
extern "C" size_t efqat_weight_quant_select_workspace_bytes(int64_t c_out) {
  return efqat_channel_select_workspace_bytes(c_out);
}

extern "C" int efqat_weight_quant_select(const float* w, int64_t c_out, int64_t block, int bits, int init_minmax,
                                         float* scale, int8_t* codes, uint32_t* clip_bits, int64_t k, double* scores,
                                         int32_t* idx, void* ws, size_t ws_bytes, void* stream) {
  if (c_out <= 0 || block <= 0 || c_out > INT32_MAX || c_out > INT64_MAX / block) return EFQAT_ERR_BAD_SHAPE;
  if (bits < 2 || bits > 8) return EFQAT_ERR_BAD_BITS;
  if (k < 0 || k > c_out) return EFQAT_ERR_BAD_K;
  if (!w || !scale || !codes || !clip_bits || !ws || (k > 0 && !idx)) return EFQAT_ERR_NULL_PTR;
  if (ws_bytes < scores_ws_bytes(c_out)) return EFQAT_ERR_WORKSPACE;
  if (((uintptr_t)ws % 256) != 0 || ((uintptr_t)w % 4) != 0 || ((uintptr_t)clip_bits % 4) != 0 ||
      ((uintptr_t)scale % 4) != 0 || ((uintptr_t)idx % 4) != 0 || ((uintptr_t)scores % 8) != 0)
    return EFQAT_ERR_ALIGNMENT;
  hipStream_t st = (hipStream_t)stream;
  WsCarver carve(ws);
  double* own = (double*)carve.take((size_t)c_out * sizeof(double));
  void* sel_ws = take_topk_ws(carve, ws_bytes, c_out);
  double* sc = scores ? scores : own;
  bool scores_done = false;
  int rc = run_fakequant<float>(w, c_out, block, EFQAT_QUANT_W_PER_ROW_SYM, bits, init_minmax, scale, nullptr, codes,
                                clip_bits, nullptr, nullptr, st, sc, &scores_done);
  if (rc) return rc;
  if (!scores_done) {                                  // rows too long for the register kernel
    rc = launch_row_importance(w, c_out, block, sc, st);
    if (rc) return rc;
  }
  if (k == 0) return EFQAT_OK;
  return launch_topk_profiled(sc, c_out, k, idx, sel_ws, st);
}
