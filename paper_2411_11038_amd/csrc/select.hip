// Channel importance (Eq. 6) and deterministic Top-K (Sec. 3.2): scores in fp64, exact selection under the
// key (score descending, index ascending) by radix select, output compacted in ascending index order.
#include "common.hpp"

#include <algorithm>
#include <atomic>

namespace efqat {

// I[c] = (1/n) sum_j |w[c][j]|, fp64 accumulation, one wavefront per channel, fixed reduction order.
__global__ __launch_bounds__(256) void k_row_importance(const float* __restrict__ w, int64_t c_out, int64_t n,
                                                        int vec, double* __restrict__ scores) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= c_out) return;
  const float* p = w + row * n;
  double acc = 0.0;
  if (vec) {
    const int64_t n4 = n >> 2;
    for (int64_t i = lane; i < n4; i += 64) {
      const float4 v = *reinterpret_cast<const float4*>(p + i * 4);
      acc += (double)fabsf(v.x) + (double)fabsf(v.y) + (double)fabsf(v.z) + (double)fabsf(v.w);
    }
  } else {
    for (int64_t i = lane; i < n; i += 64) acc += (double)fabsf(p[i]);
  }
  acc = wave_sum(acc);
  if (lane == 0) scores[row] = acc / (double)n;
}

// ------------------------------------------------------------------------------------------------
// Exact Top-K.  Scores are non-negative doubles, so their bit patterns order like the values (whatever else a caller
// passes is ordered by its bit pattern as an unsigned number); keys are taken relative
// to the smallest one (order and equality unchanged), which puts the first digit window right below the top bit of
// (largest - smallest): the scores of a layer lie in a narrow band, and the first window of 12 bits already leaves a
// handful of them around the threshold.  The selection under (score descending, index ascending) is a threshold pair
// (T, I): element i belongs to it iff key > T or (key == T and i <= I).  Integer counting only, so the result does not
// depend on thread scheduling.
typedef unsigned long long u64;
constexpr int kSelBits = 12, kSelBins = 1 << kSelBits;   // digit windows (10 bits where at most 256 keys are looked at)
constexpr int64_t kTopkBlockKeys = 16384;             // one block selects from up to this many
constexpr int kSelRank = 64;                          // this few candidates are ranked directly by one wavefront

__device__ __forceinline__ u64 score_key(double s) { return (u64)__double_as_longlong(s); }
// v >> top == prefix; keys that differ in the sign bit need all 64 bits, and a shift by 64 is none
__device__ __forceinline__ bool has_prefix(u64 v, int top, u64 prefix) { return top >= 64 || (v >> top) == prefix; }

// Where a selected index goes.
//   plain:      idx[pos] = c                          (pos < k: never behind the caller's k entries)
//   layer_off:  one Top-K over the channels of several layers: idx[pos] = c - first channel of its layer, and
//               per_layer[layer] counts (zeroed by an earlier phase);  flags (blocks are whole layers): per_layer[c] =
//               channels of layer c if it is selected, else 0
struct SelectOut {
  int32_t* idx;
  int64_t k;
  const int64_t* layer_off;
  int64_t n_layers;
  int32_t* per_layer;
  int flags;
};

// wavefront-wide reductions in registers (DPP): a shuffle through the LDS unit costs several times the latency
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned int dpp(unsigned int old, unsigned int v) {
  return (unsigned int)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
template <class F>
__device__ __forceinline__ unsigned int wave_scan(unsigned int v, unsigned int id, F f) {   // inclusive, lane 63: total
  v = f(v, dpp<0x111, 0xf>(id, v));                   // row_shr:1, 2, 4, 8: within rows of 16
  v = f(v, dpp<0x112, 0xf>(id, v));
  v = f(v, dpp<0x114, 0xf>(id, v));
  v = f(v, dpp<0x118, 0xf>(id, v));
  v = f(v, dpp<0x142, 0xa>(id, v));                   // row_bcast:15 into rows 1 and 3
  return f(v, dpp<0x143, 0xc>(id, v));                // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ unsigned int wave_scan_add(unsigned int v) {
  return wave_scan(v, 0u, [](unsigned int a, unsigned int b) { return a + b; });
}

template <int NTH, int BITS = kSelBits>
struct SelShared {
  static constexpr int kBits = BITS, kBins = 1 << BITS, kBpt = kBins / NTH;
  unsigned int hist[kBins];
  unsigned int wave_tot[NTH / 64];
  unsigned int lo[NTH / 64], hi[NTH / 64];
  u64 cand_key[kSelRank];
  int cand_idx[kSelRank];
  unsigned int rank[kSelRank];
  int ncand, bin, need, count;
  u64 any[NTH / 64], all[NTH / 64];
  u64 T;
  int I;
};

// What is taken off every key: the upper half of the smallest one, and in *top how many bits the differences need.
// (Halves are enough: the window loses at most a bit.)  lo, hi: smallest and largest upper half of this thread's keys.
template <class SH>
__device__ __forceinline__ u64 block_base(SH& sh, unsigned int lo, unsigned int hi, int* top) {
  constexpr int NW = sizeof(sh.lo) / sizeof(sh.lo[0]);
  lo = wave_scan(lo, ~0u, [](unsigned int a, unsigned int b) { return a < b ? a : b; });
  hi = wave_scan(hi, 0u, [](unsigned int a, unsigned int b) { return a > b ? a : b; });
  if ((threadIdx.x & 63) == 63) { sh.lo[threadIdx.x >> 6] = lo; sh.hi[threadIdx.x >> 6] = hi; }
  __syncthreads();
  lo = ~0u; hi = 0u;
#pragma unroll
  for (int w = 0; w < NW; ++w) { lo = sh.lo[w] < lo ? sh.lo[w] : lo; hi = sh.hi[w] > hi ? sh.hi[w] : hi; }
  *top = 32 + (hi > lo ? 32 - __clz((int)(hi - lo)) : 0);
  return (u64)lo << 32;
}

// Finds the bin in which the need-th largest element lies: sh.bin, sh.need (still to take inside it), sh.count (its
// size).  bins[]: this thread's kBpt consecutive bins.  Ends with a barrier.
template <class SH>
__device__ __forceinline__ void search_bins(SH& sh, const unsigned int (&bins)[SH::kBpt], int need) {
  constexpr int BPT = SH::kBpt, NW = sizeof(sh.wave_tot) / sizeof(sh.wave_tot[0]);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  unsigned int tot = 0;
#pragma unroll
  for (int u = 0; u < BPT; ++u) tot += bins[u];
  const unsigned int inc = wave_scan_add(tot);
  if (lane == 63) sh.wave_tot[wv] = inc;
  __syncthreads();
  int above = -(int)inc;                              // elements in higher bins
#pragma unroll
  for (int w = 0; w < NW; ++w) above += w >= wv ? (int)sh.wave_tot[w] : 0;
  if (above < need && need <= above + (int)tot) {     // exactly one thread holds the crossing
#pragma unroll
    for (int u = BPT - 1; u >= 0; --u) {
      const int h = (int)bins[u];
      if (above < need && need <= above + h) {
        sh.bin = (int)threadIdx.x * BPT + u; sh.need = need - above; sh.count = h;
      }
      above += h;
    }
  }
  __syncthreads();
}

// Threshold pair of element number `need` (from 1) under (key descending, index ascending) among the `count` elements
// with key >> top == prefix; each(f) calls f(key, index) for every element this thread holds, at least those elements;
// indices are below n.  Windows of BITS bits from `top` downwards until few elements are left; equal keys are told apart by
// their index, the last windows.  A window that leaves every element where it was (`stuck`: so did an earlier one) is
// followed by a look at the bits in which they differ at all: none, where scores are equal.
template <int NTH, int BITS, class Each>
__device__ __forceinline__ void find_threshold(SelShared<NTH, BITS>& sh, Each each, u64 prefix, int top, int need,
                                               int count, int64_t n, bool stuck) {
  constexpr int BINS = 1 << BITS, BPT = BINS / NTH, NW = NTH / 64;
  const int tid = threadIdx.x;
  bool on_index = false;                              // all remaining elements have key T: the windows run over n - 1 - index
  u64 T = 0;
  if (tid == 0) { sh.ncand = 0; sh.T = ~0ull; sh.I = -1; }
  if (tid < kSelRank) sh.rank[tid] = 0u;
  while (count > kSelRank) {
    if (stuck) {
      stuck = false;
      u64 any = 0ull, all = ~0ull;
      each([&](u64 key, int) {
        if (has_prefix(key, top, prefix)) { any |= key; all &= key; }
      });
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) { any |= __shfl_xor(any, o, kWave); all &= __shfl_xor(all, o, kWave); }
      if ((tid & 63) == 0) { sh.any[tid >> 6] = any; sh.all[tid >> 6] = all; }
      __syncthreads();
      for (int w = 0; w < NW; ++w) { any |= sh.any[w]; all &= sh.all[w]; }
      const u64 diff = any & ~all;                    // below top
      if (top > 0) top = diff ? 64 - __clzll((long long)diff) : 0;
      prefix = top >= 64 ? 0ull : any >> top;
    }
    if (top == 0) {                                   // equal keys, more of them than are ranked directly
      T = prefix; on_index = true; prefix = 0; top = 64 - __clzll(n - 1);
    }
    const int width = top < BITS ? top : BITS, shift = top - width;
    const u64 mask = (1ull << width) - 1ull;
    for (int b = tid; b < BINS; b += NTH) sh.hist[b] = 0u;
    __syncthreads();
    if (prefix == 0 && !on_index) {                   // nothing above the window: no element to leave out but larger ones
      each([&](u64 key, int) {
        const u64 b = key >> shift;
        if (b <= mask) atomicAdd(&sh.hist[b], 1u);
      });
    } else {
      each([&](u64 key, int i) {
        const u64 v = on_index ? (u64)(n - 1 - i) : key;
        if ((!on_index || key == T) && has_prefix(v, top, prefix)) atomicAdd(&sh.hist[(v >> shift) & mask], 1u);
      });
    }
    __syncthreads();
    unsigned int bins[BPT];
#pragma unroll
    for (int u = 0; u < BPT; ++u) bins[u] = sh.hist[tid * BPT + u];
    search_bins(sh, bins, need);
    prefix = (prefix << width) | (u64)sh.bin;
    need = sh.need;
    top = shift;
    stuck = count == sh.count && !on_index;
    count = sh.count;
  }
  __syncthreads();
  each([&](u64 key, int i) {
    const u64 v = on_index ? (u64)(n - 1 - i) : key;
    if (has_prefix(v, top, prefix) && (!on_index || key == T)) {
      const int slot = atomicAdd(&sh.ncand, 1);
      sh.cand_key[slot] = key; sh.cand_idx[slot] = i;
    }
  });
  __syncthreads();
  {
    // ranks: NTH / 64 threads share a candidate, each compares it with a few of the others
    constexpr int PER = kSelRank / (NTH / 64);
    const int c = tid & 63, j0 = (tid >> 6) * PER;
    const u64 mk = sh.cand_key[c];
    const int mi = sh.cand_idx[c];
    unsigned int r = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const u64 kj = sh.cand_key[j0 + u];
      const int ij = sh.cand_idx[j0 + u];
      r += (j0 + u < count && (kj > mk || (kj == mk && ij < mi))) ? 1u : 0u;
    }
    if (c < count && r) atomicAdd(&sh.rank[c], r);
    __syncthreads();
    if (tid < count && sh.rank[tid] == (unsigned int)(need - 1)) { sh.T = mk; sh.I = mi; }
  }
  __syncthreads();
}

__device__ __forceinline__ int64_t layer_of(const int64_t* layer_off, int64_t n_layers, int64_t c) {
  int64_t lo = 0, hi = n_layers;                      // the last layer that starts at or before c
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (layer_off[mid] <= c) lo = mid; else hi = mid;
  }
  return lo;
}

// writes element c of the input: selected elements at output position pos.  Called by whole wavefronts.
__device__ __forceinline__ void emit(const SelectOut& o, bool sel, int64_t pos, int64_t c, bool in_range) {
  sel = sel && pos < o.k;
  if (!o.layer_off) {
    if (sel) o.idx[pos] = (int32_t)c;
    return;
  }
  if (o.flags) {
    if (in_range) o.per_layer[c] = sel ? (int32_t)(o.layer_off[c + 1] - o.layer_off[c]) : 0;
    if (sel) o.idx[pos] = (int32_t)c;
    return;
  }
  int64_t l = -1;
  if (sel) {
    l = layer_of(o.layer_off, o.n_layers, c);
    o.idx[pos] = (int32_t)(c - o.layer_off[l]);
  }
  // neighbouring elements mostly lie in one layer: one atomic per wavefront and layer
  u64 left = __ballot(sel);
  while (left) {
    const int src = __ffsll((long long)left) - 1;
    const int64_t l0 = __shfl(l, src, kWave);
    const u64 same = __ballot(sel && l == l0);
    if ((int)(threadIdx.x & 63) == src) atomicAdd(&o.per_layer[l0], (int32_t)__popcll(same));
    left &= ~same;
  }
}

// One block for up to 16384 keys, which stay on the CU from the one read of the scores to the ordered output: KPT per
// thread in registers, or (KPT == 0) in dynamic LDS (12 or 16 64-bit keys per thread of a 1024-thread block spill).
// What bounds it is a chain of about ten block barriers and the load latency, not work, hence many threads with few
// keys each and few, wide digit windows.  256 / 768 / 3072 / 11008 keys: 3.5 / 4.0 / 6.6 / 14.6 us; with four
// wavefronts, 8-bit windows and one-wavefront ranking through LDS it was 4.7 / 7.6 / 13.5 / 29 us.
// Equal scores, 1000 / 4000 / 16384 of them (whole call): 8 / 10 / 24 us; with windows over all the bits below the first one
// and over 32 bits of the index 15 / 29 / 93 us.
template <int NTH, int KPT, int BITS = kSelBits>
__global__ __launch_bounds__(NTH) void k_topk_block(const double* __restrict__ scores, int n, int k,
                                                    const SelectOut out) {
  constexpr int NW = NTH / 64, MAXQ = KPT ? KPT : (int)(kTopkBlockKeys / NTH);
  extern __shared__ __attribute__((aligned(16))) u64 lkeys[];
  __shared__ SelShared<NTH, BITS> sh;
  __shared__ int wave_sel[MAXQ * NW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  u64 keys[KPT ? KPT : 1];
  const int nq = (n + NTH - 1) / NTH;
  // f(q, i) for the keys of this thread: key q is element i = NTH q + tid
  auto slots = [&](auto f) {
    if constexpr (KPT > 0) {
#pragma unroll
      for (int q = 0; q < KPT; ++q) f(q, q * NTH + tid);
    } else {
#pragma unroll 4
      for (int q = 0; q < nq; ++q) f(q, q * NTH + tid);
    }
  };
  auto key_ref = [&](int q, int i) -> u64& {
    if constexpr (KPT > 0) return keys[q];
    else return lkeys[i];
  };
  unsigned int lo = ~0u, hi = 0u;
  slots([&](int q, int i) {
    if constexpr (KPT > 0) keys[q] = 0ull;
    if (i < n) {
      const u64 v = score_key(scores[i]);
      key_ref(q, i) = v;
      const unsigned int h = (unsigned int)(v >> 32);
      lo = h < lo ? h : lo; hi = h > hi ? h : hi;
    }
  });
  if (out.layer_off && !out.flags) {
    for (int64_t l = tid; l < out.n_layers; l += NTH) out.per_layer[l] = 0;
    __threadfence();
  }
  u64 T = 0;
  int I = -1;
  if (k < n) {
    int top;
    const u64 base = block_base(sh, lo, hi, &top);
    if constexpr (KPT > 0) {
#pragma unroll
      for (int q = 0; q < KPT; ++q) keys[q] -= base;
    }
    const u64 sub = KPT > 0 ? 0ull : base;
    find_threshold(sh, [&](auto f) {
      slots([&](int q, int i) {
        if (i < n) f(key_ref(q, i) - sub, i);
      });
    }, 0ull, top, k, n, n, top == 32);                // 32: no key differs in its upper half
    T = sh.T + sub; I = sh.I;
  }
  // ordered output: one wavefront turns the counts of every (q, wavefront) into prefixes in index order
  unsigned int mine = 0;                              // bit q: key q of this thread is selected
  slots([&](int q, int i) {
    bool sel = false;
    if (i < n) {
      const u64 key = key_ref(q, i);
      sel = k == n || key > T || (key == T && i <= I);
    }
    mine |= sel ? 1u << q : 0u;
    const u64 b = __ballot(sel);
    if (lane == 0) wave_sel[q * NW + wv] = __popcll(b);
  });
  __syncthreads();
  if (wv == 0) {
    constexpr int EPL = (MAXQ * NW + 63) / 64;
    const int entries = nq * NW;
    int g[EPL], gs = 0;
#pragma unroll
    for (int u = 0; u < EPL; ++u) {
      g[u] = EPL * lane + u < entries ? wave_sel[EPL * lane + u] : 0;
      gs += g[u];
    }
    int gx = (int)wave_scan_add((unsigned int)gs) - gs;
#pragma unroll
    for (int u = 0; u < EPL; ++u) {
      if (EPL * lane + u < entries) wave_sel[EPL * lane + u] = gx;
      gx += g[u];
    }
  }
  __syncthreads();
  const u64 below = (1ull << lane) - 1ull;
  slots([&](int q, int i) {
    const bool sel = (mine >> q) & 1u;
    const u64 b = __ballot(sel);
    emit(out, sel, (int64_t)(wave_sel[q * NW + wv] + __popcll(b & below)), i, i < n);
  });
}

// ---- longer inputs: four launches of up to 256 blocks, block b owns the contiguous range of sel_per_block(n) keys.
// Each launch is a read of the keys out of the L2s and costs 3 to 10 us, mostly its start: 82944 keys 22 us, where one
// block that re-read them took 186 us.  Inputs that one block can keep in LDS (16384 keys, 20 us) are not worth it.
constexpr int kSelBlocks = 256;
constexpr int kSelLayers = 1024;                      // layer tables up to this size are kept in LDS
constexpr int kSelCand = 4096;                        // candidates around the threshold kept in the workspace
struct SelWs {
  unsigned int part[2 * kSelBlocks];                  // smallest, largest upper half of every block's keys
  unsigned int hist[kSelBins];                        // all keys, first window
  int above[kSelBlocks];                              // keys of every block in bins above the threshold's
  int tie[kSelBlocks];                                // too many candidates: selected ones of every block, and
  u64 T;                                              // the threshold pair
  int I, ncand, pad[60];
  u64 cand_key[kSelCand];
  int cand_idx[kSelCand];
};
static int64_t sel_per_block(int64_t n) { return std::max<int64_t>(1024, round_up(ceil_div(n, kSelBlocks), 1024)); }

// keys b0 .. b1 - 1 by a block of NTH threads, U loads in flight per thread: f(key, index)
template <int NTH, int U, class F>
__device__ __forceinline__ void sel_keys(const double* scores, int64_t b0, int64_t b1, F f) {
  for (int64_t i0 = b0 + threadIdx.x; i0 < b1; i0 += U * NTH) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i0 + NTH * u < b1 ? scores[i0 + NTH * u] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + NTH * u < b1) f(score_key(v[u]), i0 + NTH * u);
  }
}
// keys of the block's range
template <int NTH, class F>
__device__ __forceinline__ void sel_range(const double* scores, int64_t n, int64_t per, F f) {
  const int64_t b0 = (int64_t)blockIdx.x * per;
  sel_keys<NTH, 4>(scores, b0, b0 + per < n ? b0 + per : n, f);
}

__global__ __launch_bounds__(256) void k_sel_range(const double* __restrict__ scores, int64_t n, int64_t per,
                                                   SelWs* __restrict__ ws, const SelectOut out) {
  __shared__ unsigned int s_lo[4], s_hi[4];
  unsigned int lo = ~0u, hi = 0u;
  sel_range<256>(scores, n, per, [&](u64 key, int64_t) {
    const unsigned int h = (unsigned int)(key >> 32);
    lo = h < lo ? h : lo; hi = h > hi ? h : hi;
  });
  lo = wave_scan(lo, ~0u, [](unsigned int a, unsigned int b) { return a < b ? a : b; });
  hi = wave_scan(hi, 0u, [](unsigned int a, unsigned int b) { return a > b ? a : b; });
  if ((threadIdx.x & 63) == 63) { s_lo[threadIdx.x >> 6] = lo; s_hi[threadIdx.x >> 6] = hi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < 4; ++w) { lo = s_lo[w] < lo ? s_lo[w] : lo; hi = s_hi[w] > hi ? s_hi[w] : hi; }
    ws->part[2 * blockIdx.x] = lo; ws->part[2 * blockIdx.x + 1] = hi;
  }
  // clear what the next launches add to
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
  for (int64_t b = t; b < kSelBins; b += nt) ws->hist[b] = 0u;
  if (t == 0) ws->ncand = 0;
  if (out.layer_off && !out.flags)
    for (int64_t l = t; l < out.n_layers; l += nt) out.per_layer[l] = 0;
}

// base of all keys from the parts of the nb blocks; the first window is the kSelBits below the top bit of the differences
template <class SH>
__device__ __forceinline__ u64 sel_window(SH& sh, const SelWs* ws, int nb, int* shift) {
  unsigned int lo = ~0u, hi = 0u;
  if ((int)threadIdx.x < nb) { lo = ws->part[2 * threadIdx.x]; hi = ws->part[2 * threadIdx.x + 1]; }
  int top;
  const u64 base = block_base(sh, lo, hi, &top);
  *shift = top - kSelBits;
  return base;
}

__global__ __launch_bounds__(256) void k_sel_hist(const double* __restrict__ scores, int64_t n, int64_t per,
                                                  SelWs* __restrict__ ws) {
  __shared__ SelShared<256> sh;
  int shift;
  for (int b = threadIdx.x; b < kSelBins; b += 256) sh.hist[b] = 0u;
  const u64 kmin = sel_window(sh, ws, (int)gridDim.x, &shift);   // its barrier also orders the clearing
  sel_range<256>(scores, n, per, [&](u64 key, int64_t) { atomicAdd(&sh.hist[(key - kmin) >> shift], 1u); });
  __syncthreads();
  for (int b = threadIdx.x; b < kSelBins; b += 256)
    if (sh.hist[b]) atomicAdd(&ws->hist[b], sh.hist[b]);
}

// the threshold's bin, from the histogram of all keys
template <class SH>
__device__ __forceinline__ void sel_bin(SH& sh, const SelWs* ws, int64_t k) {
  constexpr int BPT = SH::kBpt;
  unsigned int bins[BPT];
#pragma unroll
  for (int u = 0; u < BPT; u += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(&ws->hist[threadIdx.x * BPT + u]);
    bins[u] = v.x; bins[u + 1] = v.y; bins[u + 2] = v.z; bins[u + 3] = v.w;
  }
  search_bins(sh, bins, (int)k);
}

// Block b of nb collects the candidates (the keys in the threshold's bin) of its range and counts its keys above them.
// A bin may hold more candidates than are kept: most scores equal, or a few far from the rest (one channel of zeros puts
// all live channels of an octave fraction into one bin).  The additional block nb then finds the threshold pair from all
// keys by itself, beside the others and in no launch of its own, and counts what it selects of every range.  1024 threads
// for the sake of this block.  Whole call on 82944 keys, distinct / with one zero / all equal: 34 / 82 / 132 us; when every
// block of k_sel_write went through all keys instead, 35 / 195 / 469 us.
constexpr int kSelCollect = 1024;
__global__ __launch_bounds__(kSelCollect) void k_sel_collect(const double* __restrict__ scores, int64_t n, int64_t per,
                                                             int nb, int64_t k, SelWs* __restrict__ ws) {
  constexpr int NTH = kSelCollect, NW = NTH / 64;
  __shared__ SelShared<NTH> sh;
  __shared__ int red[NW];
  __shared__ int tie[kSelBlocks];
  const int tid = threadIdx.x;
  int shift;
  const u64 kmin = sel_window(sh, ws, nb, &shift);
  sel_bin(sh, ws, k);
  const u64 bin = (u64)sh.bin;
  const int need = sh.need, count = sh.count;
  const bool keep = count <= kSelCand;
  if ((int)blockIdx.x == nb) {
    if (keep) return;
    if (tid < kSelBlocks) tie[tid] = 0;
    __syncthreads();                                  // everybody has read sh.need / sh.count
    auto each = [&](auto f) {
      sel_keys<NTH, 8>(scores, 0, n, [&](u64 key, int64_t i) { f(key - kmin, (int)i); });
    };
    find_threshold(sh, each, bin, shift, need, count, n, count == n);
    const u64 T = sh.T;
    const int I = sh.I;
    each([&](u64 key, int i) {
      // a wavefront's 64 neighbours lie in one range
      const u64 sel = __ballot((key >> shift) == bin && (key > T || (key == T && i <= I)));
      if ((tid & 63) == 0 && sel) atomicAdd(&tie[(unsigned int)i / (unsigned int)per], (int)__popcll(sel));
    });
    __syncthreads();
    if (tid < nb) ws->tie[tid] = tie[tid];
    if (tid == 0) { ws->T = T; ws->I = I; }
    return;
  }
  int above = 0;
  sel_range<NTH>(scores, n, per, [&](u64 key, int64_t i) {
    const u64 b = (key - kmin) >> shift;
    above += b > bin ? 1 : 0;
    if (keep && b == bin) {
      const int slot = atomicAdd(&ws->ncand, 1);
      ws->cand_key[slot] = key - kmin; ws->cand_idx[slot] = (int)i;
    }
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) above += __shfl_xor(above, o, kWave);
  if ((tid & 63) == 0) red[tid >> 6] = above;
  __syncthreads();
  if (tid == 0) {
    above = 0;
    for (int w = 0; w < NW; ++w) above += red[w];
    ws->above[blockIdx.x] = above;
  }
}

// Writes the selected keys of b0 .. b1 - 1 in index order from output position `base` on; v: this thread's first four keys.
template <int NTH>
__device__ __forceinline__ void write_range(const double* scores, int64_t b0, int64_t b1, int64_t base, double (&v)[4],
                                            u64 kmin, u64 T, int I, int (&wave_sel)[4][NTH / 64], const SelectOut& out) {
  constexpr int NW = NTH / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const u64 below = (1ull << lane) - 1ull;
  for (int64_t i0 = b0; i0 < b1; i0 += 4 * NTH) {
    bool sel[4];
    if (i0 > b0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) { const int64_t i = i0 + NTH * u + tid; v[u] = i < b1 ? scores[i] : 0.0; }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + NTH * u + tid;
      const u64 key = score_key(v[u]) - kmin;
      sel[u] = i < b1 && (key > T || (key == T && (int)i <= I));
      const u64 b = __ballot(sel[u]);
      if (lane == 0) wave_sel[u][wv] = __popcll(b);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + NTH * u + tid;
      int64_t pos = base + __popcll(__ballot(sel[u]) & below);
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        pos += w < wv ? wave_sel[u][w] : 0;
        base += wave_sel[u][w];
      }
      emit(out, sel[u], pos, i, i < b1);
    }
    __syncthreads();
  }
}

// Every block finds the threshold pair from the candidates (or has it from k_sel_collect), counts what the blocks before it
// select, and writes its own range.
__global__ __launch_bounds__(256) void k_sel_write(const double* __restrict__ scores, int64_t n, int64_t per, int64_t k,
                                                   const SelWs* __restrict__ ws, const SelectOut out_) {
  __shared__ SelShared<256> sh;
  __shared__ int red[4], wave_sel[4][4];
  __shared__ int64_t s_off[kSelLayers + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // requested ahead of the search for the threshold: the layer table and the first 1024 keys of the range
  SelectOut out = out_;
  const bool table = out.layer_off && !out.flags && out.n_layers <= kSelLayers;
  if (table)
    for (int l = tid; l <= (int)out.n_layers; l += 256) s_off[l] = out.layer_off[l];
  const int64_t b0 = (int64_t)blockIdx.x * per;
  const int64_t b1 = b0 + per < n ? b0 + per : n;
  double v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) { const int64_t i = b0 + 256 * u + tid; v[u] = i < b1 ? scores[i] : 0.0; }
  int before = 0;                                     // selected elements ahead of this block's range: whole bins ...
  for (int b = tid; b < (int)blockIdx.x; b += 256) before += ws->above[b];
  int shift;
  const u64 kmin = sel_window(sh, ws, (int)gridDim.x, &shift);
  sel_bin(sh, ws, k);
  const u64 bin = (u64)sh.bin;
  const int need = sh.need, count = sh.count;
  __syncthreads();                                    // everybody has read sh.need / sh.count
  if (table) out.layer_off = s_off;
  u64 T;
  int I;
  if (count <= kSelCand) {
    auto each = [&](auto f) {
      for (int i = tid; i < count; i += 256) f(ws->cand_key[i], ws->cand_idx[i]);
    };
    find_threshold(sh, each, bin, shift, need, count, n, false);
    T = sh.T; I = sh.I;
    // ... and candidates
    each([&](u64 key, int i) { before += (i < b0 && (key > T || (key == T && i <= I))) ? 1 : 0; });
  } else {
    T = ws->T; I = ws->I;
    for (int b = tid; b < (int)blockIdx.x; b += 256) before += ws->tie[b];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, kWave);
  if (lane == 0) red[wv] = before;
  __syncthreads();
  write_range<256>(scores, b0, b1, (red[0] + red[1]) + (red[2] + red[3]), v, kmin, T, I, wave_sel, out);
}

// Beyond kTopkBlockKeys without a workspace (a caller that hands over no more than the scores need): one block goes through
// all keys once per window, and once more to write.  Whole call on 82944 keys, distinct / all
// equal: 155 / 188 us (the chain: 32 / 130 us).
__global__ __launch_bounds__(kSelCollect) void k_sel_one(const double* __restrict__ scores, int64_t n, int64_t k,
                                                         const SelectOut out) {
  constexpr int NTH = kSelCollect;
  __shared__ SelShared<NTH> sh;
  __shared__ int wave_sel[4][NTH / 64];
  const int tid = threadIdx.x;
  if (out.layer_off && !out.flags) {
    for (int64_t l = tid; l < out.n_layers; l += NTH) out.per_layer[l] = 0;
    __threadfence();
  }
  unsigned int lo = ~0u, hi = 0u;
  sel_keys<NTH, 8>(scores, 0, n, [&](u64 key, int64_t) {
    const unsigned int h = (unsigned int)(key >> 32);
    lo = h < lo ? h : lo; hi = h > hi ? h : hi;
  });
  int top;
  const u64 kmin = block_base(sh, lo, hi, &top);      // its barrier also orders the clearing of per_layer
  u64 T = 0;
  int I = INT32_MAX;                                  // k == n: every key
  if (k < n) {
    auto each = [&](auto f) {
      sel_keys<NTH, 8>(scores, 0, n, [&](u64 key, int64_t i) { f(key - kmin, (int)i); });
    };
    find_threshold(sh, each, 0ull, top, (int)k, (int)n, n, top == 32);
    T = sh.T; I = sh.I;
  }
  double v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) { const int64_t i = NTH * u + tid; v[u] = i < n ? scores[i] : 0.0; }
  write_range<NTH>(scores, 0, n, 0, v, kmin, T, I, wave_sel, out);
}

// One block up to kTopkBlockKeys; the four-launch chain beyond, whose workspace is topk_ws_bytes(n) (k_sel_one without it).
size_t topk_ws_bytes(int64_t n) { return n > kTopkBlockKeys ? (size_t)round_up((int64_t)sizeof(SelWs), 256) : 0; }

void* take_topk_ws(WsCarver& carve, size_t ws_bytes, int64_t n) {
  const size_t need = topk_ws_bytes(n);
  return need > 0 && carve.off + need <= ws_bytes ? carve.take(need) : nullptr;
}

// no channel selected anywhere: all counts are 0
__global__ __launch_bounds__(256) void k_zero_counts(int32_t* __restrict__ per_layer, int64_t n_layers) {
  const int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (l < n_layers) per_layer[l] = 0;
}

static void launch_select(const double* scores, int64_t n, int64_t k, const SelectOut& out, void* ws, hipStream_t st) {
  if (k == 0) {
    if (out.per_layer)
      hipLaunchKernelGGL(k_zero_counts, dim3((unsigned)ceil_div(out.n_layers, 256)), dim3(256), 0, st, out.per_layer, out.n_layers);
    return;
  }
#define EFQAT_TOPK(NTH, KPT, LDS) \
  hipLaunchKernelGGL((k_topk_block<NTH, KPT>), dim3(1), dim3(NTH), LDS, st, scores, (int)n, (int)k, out)
  if (n <= 256)
    hipLaunchKernelGGL((k_topk_block<256, 1, 10>), dim3(1), dim3(256), 0, st, scores, (int)n, (int)k, out);
  else if (n <= 1024) EFQAT_TOPK(1024, 1, 0);
  else if (n <= 2048) EFQAT_TOPK(1024, 2, 0);
  else if (n <= 4096) EFQAT_TOPK(1024, 4, 0);
  else if (n <= kTopkBlockKeys) {
    // set once per process (initialisation of a function-local static is thread-safe); a failure leaves the default
    // LDS limit in place and the launch below then reports it
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_topk_block<1024, 0>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       (int)(kTopkBlockKeys * sizeof(u64)));
    (void)attr;
    EFQAT_TOPK(1024, 0, (size_t)n * sizeof(u64));
  }
#undef EFQAT_TOPK
  else if (!ws)
    hipLaunchKernelGGL(k_sel_one, dim3(1), dim3(kSelCollect), 0, st, scores, n, k, out);
  else {
    SelWs* w = (SelWs*)ws;
    const int64_t per = sel_per_block(n);
    const dim3 grid((unsigned)ceil_div(n, per));
    hipLaunchKernelGGL(k_sel_range, grid, dim3(256), 0, st, scores, n, per, w, out);
    hipLaunchKernelGGL(k_sel_hist, grid, dim3(256), 0, st, scores, n, per, w);
    hipLaunchKernelGGL(k_sel_collect, dim3(grid.x + 1), dim3(kSelCollect), 0, st, scores, n, per, (int)grid.x, k, w);
    hipLaunchKernelGGL(k_sel_write, grid, dim3(256), 0, st, scores, n, per, k, w, out);
  }
}

void launch_topk(const double* scores, int64_t n, int64_t k, int32_t* idx, void* ws, hipStream_t st) {
  launch_select(scores, n, k, SelectOut{idx, k, nullptr, 0, nullptr, 0}, ws, st);
}

int launch_topk_profiled(const double* scores, int64_t n, int64_t k, int32_t* idx, void* ws, hipStream_t st) {
  {
    ProfScope prof(PROF_TOPK, st);
    launch_topk(scores, n, k, idx, ws, st);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

int launch_row_importance(const float* w, int64_t c_out, int64_t block, double* scores, hipStream_t st) {
  const int vec = (((uintptr_t)w % 16) == 0 && block % 4 == 0) ? 1 : 0;
  {
    ProfScope prof(PROF_IMPORTANCE, st);
    hipLaunchKernelGGL(k_row_importance, dim3((unsigned)ceil_div(c_out, 4)), dim3(256), 0, st, w, c_out, block, vec,
                       scores);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

}  // namespace efqat

using namespace efqat;

extern "C" int64_t efqat_k_from_ratio(int64_t c_out, int64_t num, int64_t den) {
  if (c_out < 0 || num < 0 || den <= 0 || num > den) return -1;
  return (int64_t)(((__int128)c_out * (__int128)num) / (__int128)den);
}

extern "C" size_t efqat_channel_select_workspace_bytes(int64_t c_out) {
  if (c_out <= 0) return 0;
  return scores_ws_bytes(c_out) + topk_ws_bytes(c_out);
}

extern "C" int efqat_channel_select(const float* w, int64_t c_out, int64_t block, int64_t k, double* scores,
                                    int32_t* idx, void* ws, size_t ws_bytes, void* stream) {
  if (c_out <= 0 || block <= 0 || c_out > INT32_MAX || c_out > INT64_MAX / block) return EFQAT_ERR_BAD_SHAPE;
  if (k < 0 || k > c_out) return EFQAT_ERR_BAD_K;
  if (!w || !ws || (k > 0 && !idx)) return EFQAT_ERR_NULL_PTR;
  if (ws_bytes < scores_ws_bytes(c_out)) return EFQAT_ERR_WORKSPACE;
  if (((uintptr_t)ws % 256) != 0 || ((uintptr_t)w % 4) != 0) return EFQAT_ERR_ALIGNMENT;
  hipStream_t st = (hipStream_t)stream;
  WsCarver carve(ws);
  double* sc = (double*)carve.take((size_t)c_out * sizeof(double));
  void* sel_ws = take_topk_ws(carve, ws_bytes, c_out);
  double* sc_out = scores ? scores : sc;
  const int vec = (((uintptr_t)w % 16) == 0 && block % 4 == 0) ? 1 : 0;
  {
    ProfScope prof(PROF_IMPORTANCE, st);
    hipLaunchKernelGGL(k_row_importance, dim3((unsigned)ceil_div(c_out, 4)), dim3(256), 0, st, w, c_out, block, vec,
                       sc_out);
  }
  EFQAT_LAUNCH_CHECK();
  if (k == 0) return EFQAT_OK;
  {
    ProfScope prof(PROF_TOPK, st);
    launch_topk(sc_out, c_out, k, idx, sel_ws, st);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

// ------------------------------------------------------------------------------------------------
// efqat_channel_select for callers that cannot allocate device memory: the per-channel scores, which the plain entry
// point keeps in the caller's workspace, live in a file-scope device array of the library instead.
namespace efqat {

constexpr int64_t kStaticSelectMaxChannels = EFQAT_STATIC_SELECT_MAX_CHANNELS;
struct StaticScratch {
  SelWs select;                                       // the Top-K of many channels
  double scores[kStaticSelectMaxChannels];
};
static_assert(sizeof(StaticScratch) <= 581 * 1024, "the size that efqat.h states, per GPU and for the process' life");
static __device__ __align__(256) StaticScratch scratch;

// Host code must not pass `scratch` itself to a kernel: here that name is only a handle for the symbol.  The
// object's device address differs per GPU (each holds its own copy) and is looked up once per device, with that
// device current.  One pointer for both parts, so that a thread that finds it finds all of it.
constexpr int kMaxDevices = 64;
static std::atomic<StaticScratch*> g_scratch_ptr[kMaxDevices];

static int static_scratch(StaticScratch** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return EFQAT_ERR_HIP;
  StaticScratch* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return EFQAT_ERR_HIP;
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return EFQAT_OK;
}

}  // namespace efqat

extern "C" int efqat_channel_select_static(const float* w, int64_t c_out, int64_t block, int64_t k, int32_t* idx,
                                           void* stream) {
  if (c_out <= 0 || block <= 0 || c_out > INT64_MAX / block) return EFQAT_ERR_BAD_SHAPE;
  if (c_out > kStaticSelectMaxChannels) return EFQAT_ERR_WORKSPACE;   // more channels than the built-in scratch holds
  if (k < 0 || k > c_out) return EFQAT_ERR_BAD_K;
  if (!w || (k > 0 && !idx)) return EFQAT_ERR_NULL_PTR;
  if (((uintptr_t)w % 4) != 0 || ((uintptr_t)idx % 4) != 0) return EFQAT_ERR_ALIGNMENT;
  StaticScratch* own = nullptr;
  const int rc = static_scratch(&own);
  if (rc) return rc;
  double* sc = own->scores;
  hipStream_t st = (hipStream_t)stream;
  const int vec = (((uintptr_t)w % 16) == 0 && block % 4 == 0) ? 1 : 0;
  // every score that Top-K reads is written by this launch first: nothing in the scratch has to start at zero
  hipLaunchKernelGGL(k_row_importance, dim3((unsigned)ceil_div(c_out, 4)), dim3(256), 0, st, w, c_out, block, vec, sc);
  EFQAT_LAUNCH_CHECK();
  if (k == 0) return EFQAT_OK;
  launch_topk(sc, c_out, k, idx, &own->select, st);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

extern "C" size_t efqat_network_select_workspace_bytes(int64_t total) {
  return 256 + (total > 0 ? topk_ws_bytes(total) : 0);   // short inputs need no scratch; callers treat every entry point alike
}

extern "C" int efqat_network_select(const double* scores, const int64_t* layer_off, int64_t n_layers,
                                    int64_t total, int64_t k_total, int32_t* idx, int32_t* k_per_layer, void* ws,
                                    size_t ws_bytes, void* stream) {
  if (n_layers <= 0 || total <= 0 || total > INT32_MAX) return EFQAT_ERR_BAD_SHAPE;
  if (k_total < 0 || k_total > total) return EFQAT_ERR_BAD_K;
  if (!scores || !layer_off || !k_per_layer || !ws || (k_total > 0 && !idx)) return EFQAT_ERR_NULL_PTR;
  if (ws_bytes < 256) return EFQAT_ERR_WORKSPACE;
  if (((uintptr_t)ws % 256) != 0) return EFQAT_ERR_ALIGNMENT;
  hipStream_t st = (hipStream_t)stream;
  WsCarver carve(ws);
  launch_select(scores, total, k_total, SelectOut{idx, k_total, layer_off, n_layers, k_per_layer, 0},
                take_topk_ws(carve, ws_bytes, total), st);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

// ------------------------------------------------------------------------------------------------
// EfQAT-LWPN (Table 2): blocks are whole layers.  Every channel of a layer has the same number of weights, so the
// layer's mean |w| is the mean of its channel means: one block per layer reduces them in double precision in a
// fixed order.
namespace efqat {

__global__ __launch_bounds__(256) void k_layer_means(const double* __restrict__ scores,
                                                     const int64_t* __restrict__ layer_off,
                                                     double* __restrict__ layer_scores) {
  __shared__ double red[256];
  const int64_t b = layer_off[blockIdx.x], e = layer_off[blockIdx.x + 1];
  double s = 0.0;
  for (int64_t i = b + threadIdx.x; i < e; i += 256) s += scores[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) layer_scores[blockIdx.x] = e > b ? red[0] / (double)(e - b) : 0.0;
}

}  // namespace efqat

using namespace efqat;

extern "C" size_t efqat_layer_select_workspace_bytes(int64_t n_layers) {
  const int64_t n = n_layers > 0 ? n_layers : 1;
  return scores_ws_bytes(n) + topk_ws_bytes(n);
}

extern "C" int efqat_layer_select(const double* scores, const int64_t* layer_off, int64_t n_layers,
                                  int64_t k_layers, double* layer_scores, int32_t* layer_idx,
                                  int32_t* k_per_layer, void* ws, size_t ws_bytes, void* stream) {
  if (n_layers <= 0 || n_layers > INT32_MAX) return EFQAT_ERR_BAD_SHAPE;
  if (k_layers < 0 || k_layers > n_layers) return EFQAT_ERR_BAD_K;
  if (!scores || !layer_off || !k_per_layer || !ws || (k_layers > 0 && !layer_idx)) return EFQAT_ERR_NULL_PTR;
  if (ws_bytes < scores_ws_bytes(n_layers)) return EFQAT_ERR_WORKSPACE;
  if (((uintptr_t)ws % 256) != 0) return EFQAT_ERR_ALIGNMENT;
  hipStream_t st = (hipStream_t)stream;
  WsCarver carve(ws);
  double* own = (double*)carve.take((size_t)n_layers * sizeof(double));
  void* sel_ws = take_topk_ws(carve, ws_bytes, n_layers);
  double* ls = layer_scores ? layer_scores : own;
  hipLaunchKernelGGL(k_layer_means, dim3((unsigned)n_layers), dim3(256), 0, st, scores, layer_off, ls);
  EFQAT_LAUNCH_CHECK();
  launch_select(ls, n_layers, k_layers, SelectOut{layer_idx, k_layers, layer_off, n_layers, k_per_layer, 1}, sel_ws, st);
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}
