// Choice of tile and split of the products, and launches of k_gemm_nt (gemm_nt.hpp).
#include "gemm_nt.hpp"

#include <algorithm>

namespace efqat {

// ---------------------------------------------------------------------------------------------- host
// Tile / split-K choice of the large products (dw_plan asks it first and keeps its 256 and 192 row tiles) and of the plans
// that fit a workspace without the smaller tiles' slices: a cost model in CU clock cycles, evaluated on the host and
// calibrated on measured runs (rates in flop per clock per block):
//   - a T x T block runs its K loop at `rate`: 256 -> 2500, 192 -> 2100, 128 -> 1000 with two blocks resident
//     per CU.  The big tiles are bounded by what one CU's vector L1 pulls from L2 (about 19 B/clk) times their
//     flop per byte, the small one additionally by its doubled L2 traffic;
//   - per block: launch/prologue 4000 cycles plus the epilogue, 0.75 cycles per output element for the fused
//     dX epilogue (it streams x, codes, mask and dX through HBM), 0.6 when a second resident block overlaps it,
//     0.3 for the raw fp32 store;
//   - blocks run in rounds of 256 CUs x blocks-per-CU;  split-K adds its fp32 partial tiles, written and read once.
struct TileModel { int t; int bpc; double rate; double epi_dx; };
static const TileModel kTiles[3] = {{256, 1, 2500.0, 0.75}, {192, 1, 2100.0, 0.75}, {128, 2, 1000.0, 0.6}};

GemmPlan gemm_plan(int64_t M, int64_t N, int64_t K, bool allow_split, bool allow_192, bool allow_256) {
  GemmPlan best{};
  double best_t = 1e300;
  const int64_t ksteps = ceil_div(K, KALIGN);
  for (const TileModel& tm : kTiles) {
    if (tm.t == 192 && !allow_192) continue;
    if (tm.t == 256 && !allow_256) continue;
    const int64_t tiles = ceil_div(M, tm.t) * ceil_div(N, tm.t);
    int64_t max_s = allow_split ? ksteps / 8 : 1;
    if (max_s < 1) max_s = 1;
    if (max_s > 32) max_s = 32;
    for (int64_t s = 1; s <= max_s; ++s) {
      const int64_t kslice = ceil_div(ksteps, s) * KALIGN;
      const double per_elem = allow_split ? 0.3 : tm.epi_dx;
      const double block = 2.0 * tm.t * tm.t * (double)kslice / tm.rate + 4000.0 + per_elem * tm.t * tm.t;
      const double rounds = (double)ceil_div(tiles * s, 256 * tm.bpc);
      double t = rounds * block;
      if (allow_split) t += (double)s * (double)M * (double)N * 8.0 / 2400.0;   // partial tiles at ~5 TB/s
      if (t < best_t) {
        best_t = t;
        best.tile = tm.t; best.split_k = (int)s;
        best.tiles_m = (int)ceil_div(M, tm.t); best.tiles_n = (int)ceil_div(N, tm.t);
      }
    }
  }
  return best;
}

// Kernel and tile of a dX product.  Microseconds per K stage of 64 and per block (launch, first loads, epilogue) with one
// block on a CU (lone; of a tile that fits once: on few of the CUs, where clock and memory are its own) and with all `bpc`
// that fit by LDS and registers (full), between the two by the number resident; what x and dX in fp32 add and what the
// straight-line epilogue of whole bf16 tiles saves.  A product is its whole rounds of 256 * bpc blocks plus what is left.
// Fitted to measured launches of 300 linear layers (each dimension 64 .. 16384) and 28 convolutions; the choice is 0.9 %
// from the fastest of the six in the mean, the linear layers 1.33 x and the convolutions 1.6 x as fast as with tiles of
// 128 and more only.  T x C_out -> C_in in us by k_gemm_kk 64 / nt 64 / kk 128 / nt 128 / kk 192 / dx8 256, bf16:
//   256 x 256 -> 256         6.6 / 5.8 / 8.4 /  - /  18 / -      few tiles: the smallest, with the shortest epilogue
//   64 x 4096 -> 4096         21 /  33 /  30 /  46 /  51 /  -    ... and the ring, where K is long
//   2048 x 768 -> 3072        28 /  28 /  26 /  26 /  30 /  30   (C_out 320)
//   4224 x 112 -> 6144        46 /  37 /  46 /  34 /  38 /  44   two blocks a CU hide each other's epilogues
//   12288 x 3072 -> 768       89 /  99 /  87 /  85 /  54 /  -    one round of 192 x 192
//   13824 x 2504 -> 768      135 / 132 /  93 /  93 /  95 /  65   long K and whole rounds: 256 x 256
// Without int8 operand the 256 x 256 tiles are k_gemm_nt's, which has no straight-line epilogue: a row of its own, fitted to 154
// more calls (0.4 % from the fastest in the mean; with the row of dx8 0.6 %, and whole bf16 tiles were taken where they lose:
// 5888 x 1716 -> 5888 205 us, now 175 on 192 x 192; 16384 x 1020 -> 2048 118, now 105 on 128 x 128).
// Convolutions pay for the gather in every stage.
struct DxTile { int t; bool ring; int bpc; double lone[2], full[2], f32[2], fast[2]; int bn; };   // bn: columns, 0: as many as rows
static const DxTile kDxTiles[] = {{64, true, 3, {0.28, 5.6}, {0.73, 4.5}, {0.1, 1.0}, {0.0, 0.0}},
                                  {64, false, 4, {0.465, 4.4}, {0.965, 4.4}, {0.1, 1.6}, {0.0, 0.0}},
                                  {128, true, 1, {0.495, 9.2}, {0.587, 7.9}, {0.0, 1.4}, {-1.7, -1.7}},
                                  {128, false, 2, {0.74, 8.0}, {1.075, 9.7}, {0.7, 3.5}, {-1.7, -2.0}},
                                  {192, true, 1, {0.695, 15.6}, {0.98, 15.6}, {0.0, 4.8}, {-4.2, -4.2}},
                                  {256, false, 1, {0.92, 23.3}, {1.61, 23.3}, {1.9, 12.0}, {-6.7, -6.7}}};   // k_gemm_dx8
static const DxTile kDxNt256 = {256, false, 1, {0.97, 17.7}, {1.71, 26.1}, {1.7, 7.4}, {0.0, 0.0}};
static const DxTile kDxConvTiles[] = {{64, true, 3, {0.30, 6.3}, {0.575, 6.6}, {0.0, 0.0}, {0.0, 0.0}},
                                      {64, false, 4, {0.54, 5.2}, {0.71, 5.4}, {0.0, 0.1}, {0.0, 0.0}},
                                      {128, true, 1, {0.56, 10.0}, {0.56, 10.0}, {0.5, 0.5}, {-1.0, -1.0}},
                                      {128, false, 2, {0.79, 9.4}, {0.94, 11.2}, {0.0, 0.6}, {-1.0, -1.0}},
                                      {192, false, 1, {1.12, 15.6}, {1.12, 15.6}, {0.2, 0.2}, {-1.0, -1.0}}};
static int64_t conv_phases(const ConvDxStridedMap& cm, int tile, ConvPhase* out, int* nphase);

// MB of x, its codes and masks and dX of a linear layer
static double dx_traffic_mb(int64_t M, int64_t N, bool f32) { return (double)M * (double)N * (f32 ? 9.125 : 5.125) / 1e6; }
// What they take to move, beyond what the caches hold: products of few K stages under a large dX are bound by that, and narrow
// tiles and lone blocks move it more slowly.  T x C_out -> C_in, k = 0, the call on 64 / 128 wide tiles, us: 11474 x 128 -> 7176
// bf16 177 / 142, 16384 x 16 -> 5872 fp32 271 / 230 (256: 264), 13840 x 96 -> 7232 fp32 273 / 236, 15872 x 17 -> 8704 bf16, k = 17,
// 256 / 207 (ring of 128: 245); but 5248 x 64 -> 5114 fp32 (245 MB) 62.6 / 63.6.  Of 524 layers the choice is 0.7 % from the
// fastest with it and 0.9 % without; where it changes the choice the calls are up to 1.23 x as fast, the worst found 0.975 x.
static double dx_memory_price(int64_t M, int64_t N, const DxTile& c, bool f32) {
  const double mb = dx_traffic_mb(M, N, f32);
  if (c.bpc == 1) return f32 ? (mb - 50.0) / 3.3 : (mb - 60.0) / 2.5;
  if (c.t == 64) return f32 ? (mb - 100.0) / 2.9 : (mb - 80.0) / 2.0;
  return f32 ? (mb - 50.0) / 3.95 : (mb - 60.0) / 2.8;
}

// K stages of a row tile of t rows (strided: in the mean) and the number of row tiles
static double dx_stages(int64_t M, int64_t K, int t, const ConvDxStridedMap* strided, int64_t* tiles_m) {
  double stages = (double)ceil_div(K, KALIGN);
  *tiles_m = ceil_div(M, t);
  if (strided) {
    ConvPhase ph[kMaxConvStride * kMaxConvStride];
    int n = 0;
    *tiles_m = conv_phases(*strided, t, ph, &n);
    double sum = 0.0;
    for (int i = 0; i < n; ++i) sum += (double)ph[i].tiles * ph[i].ntap;
    stages *= sum / ((double)*tiles_m * strided->KH * strided->KW);
  }
  return stages;
}

GemmPlan dx_plan(int64_t M, int64_t N, int64_t K, bool f32, bool conv, const ConvDxStridedMap* strided, bool int8_ok,
                 double* price_out) {
  GemmPlan best{};
  double best_t = 0.0;
  auto price = [&](const DxTile& c) {
    if (c.t == 192 && strided) return;
    int64_t tm = 0;
    const double stages = dx_stages(M, K, c.t, strided, &tm);
    const int64_t tn = ceil_div(N, c.t), tiles = tm * tn, round = 256 * c.bpc;
    if (tiles >= (1 << 24) && c.t < 128) return;        // a grid dimension holds less than 2^32 work items
    const bool fast = !f32 && !strided && (M % c.t) == 0 && (N % c.t) == 0;
    const double add[2] = {(f32 ? c.f32[0] : 0.0) + (fast ? c.fast[0] : 0.0), (f32 ? c.f32[1] : 0.0) + (fast ? c.fast[1] : 0.0)};
    const double lone = c.lone[0] * stages + c.lone[1] + add[0], full = c.full[0] * stages + c.full[1] + add[1];
    double t = (double)(tiles / round) * full;
    if (const int64_t rest = tiles % round)
      t += lone + (full - lone) * (c.bpc > 1 ? (double)(ceil_div(rest, 256) - 1) / (c.bpc - 1) : (double)rest / 256.0);
    // the others need W_q^T in bf16: the codes read, twice as many bytes written, at 4 TB/s
    const double wqt = int8_ok && c.t != 256 ? 3.0 * (double)N * (double)K / 4e6 : 0.0;
    if (price_out && (best.tile == 0 || t + wqt < *price_out)) *price_out = t + wqt;
    t = (conv ? t : std::max(t, dx_memory_price(M, N, c, f32))) + wqt;
    if (best.tile == 0 || t < best_t) { best_t = t; best = GemmPlan{c.t, 1, (int)tm, (int)tn, c.ring}; }
  };
  if (conv) for (const DxTile& c : kDxConvTiles) price(c);
  else for (const DxTile& c : kDxTiles) price(c.t == 256 && !int8_ok ? kDxNt256 : c);
  return best;
}

// Tile and split-K of a dW product.  Costs as in kDxTiles; to them comes the second pass (k_dw_finish), which reads every
// slice: 3.7 us, 0.07 us a slice, and 0.119 us per 2^20 values and 4 bytes.  Slices of two K stages and more, where
// eight stages and fewer, larger tiles were the rule before.  Fitted to 100 layers and convolutions by k_gemm_tn and 55 from
// staged operands, dW product and second pass together: 1.02 x (staged 1.06 x) the fastest of all tiles and splits, 1.21 x
// (convolutions 1.25 x, staged 1.29 x) as fast as before.  T x C_in, k rows, us with the best split on 64 / 128 rows (slices):
//   480 x 512, 172        7.8 (4) / 10.1 (4), before 13.4 (1)     few tiles: as many short slices as fill the chip
//   12144 x 688, 40      13.9 (32) / 15.5 (32), before 16.7 (22)  half of a 128-row tile would be padding
//   6848 x 1776, 1500    63 (3) / 54 (3)                          many tiles: fewer LDS bytes per product
// The 256 x 256 and 192 x 192 tiles stay where gemm_plan prices them lowest: large products.
// Gathered codes on 128-row tiles: two blocks a CU, by the registers of the pixel coordinates; priced as three before, 64 x 47 x 47,
// 512 -> 384, 2 x 2, k = 192 took 24 slices of them: 616 us, now 21 of 64-row tiles 582.  Fitted to 50 convolutions, 0.46 % from the
// fastest in the mean (0.53 %).
struct DwTile { int bm, bn, bpc; double lone[2], full[2]; };
static const DwTile kDwTiles[4][2] = {{{64, 128, 4, {0.515, 4.4}, {1.10, 6.2}}, {128, 128, 3, {0.575, 5.8}, {1.305, 8.3}}},
                                      {{64, 128, 4, {0.785, 5.0}, {1.51, 7.6}}, {128, 128, 2, {1.007, 5.9}, {1.303, 7.0}}},
                                      {{64, 64, 4, {0.453, 3.0}, {0.95, 3.5}}, {128, 128, 2, {0.71, 4.5}, {0.88, 7.0}}},
                                      {{64, 128, 4, {0.485, 3.4}, {0.89, 7.7}}, {128, 128, 3, {0.547, 4.6}, {0.917, 9.7}}}};
// the second pass over S slices of M x N values
static double finish_price(int64_t M, int64_t N, int64_t S) {
  return 3.7 + 0.07 * (double)S + 0.119e-6 * (double)M * (double)N * (double)(4 * S + 9);
}
GemmPlan dw_plan(DwKind kind, int64_t M, int64_t N, int64_t K, double* price_out) {
  if (price_out) *price_out = 0.0;
  GemmPlan best = gemm_plan(M, N, K, true, kind == DW_STAGED, kind != DW_CONV);
  if (best.tile > 128) return best;
  const int64_t stages = ceil_div(K, KALIGN);
  double best_t = 0.0;
  bool have = false;
  for (const DwTile& c : kDwTiles[kind]) {
    const int64_t tm = ceil_div(M, c.bm), tn = ceil_div(N, c.bn), round = 256 * c.bpc;
    if (tm * tn >= (1 << 24)) continue;                 // a grid dimension holds less than 2^32 work items
    for (int64_t s = 1; s <= 64 && (s == 1 || 2 * s <= stages); ++s) {
      const int64_t per = ceil_div(stages, s);
      if (ceil_div(stages, per) != s) continue;         // slices without a stage
      const double lone = c.lone[0] * (double)per + c.lone[1], full = c.full[0] * (double)per + c.full[1];
      double t = (double)(tm * tn * s / round) * full + finish_price(M, N, s);
      if (const int64_t rest = tm * tn * s % round)
        t += lone + (full - lone) * (double)(ceil_div(rest, 256) - 1) / (double)(c.bpc - 1);
      if (!have || t < best_t) { best_t = t; best = GemmPlan{c.bm, (int)s, (int)tm, (int)tn, false}; have = true; }
    }
  }
  if (price_out) *price_out = best_t;
  return best;
}

// dX of a channel-major dY by k_gemm_dx8, 64 x 128, 128 x 128, 128 x 256 and 256 x 256; fitted to 90 layers (0.2 % from the fastest in the
// mean), the row of 128 x 256 to 258 others, of which 198 have it: 0.85 % from the fastest, 5.8 % without that tile.  A tile of 128 x 256
// moves half of the bytes from L2 to LDS that the four of 64 x 128 on its area do, which is what the smaller tiles are bound by, and
// two of them on a CU hide each other's epilogues.
// T x C_out -> C_in, backward call without selected channels, us on 64 / 128 / 128 x 256 / 256, in turn on two sets of buffers:
//    2048 x 1536 -> 3072   34.0 / 32.0 / 29.4 / 39.6
//    4096 x 4096 -> 2048   94.9 / 78.2 / 70.9 / 81.0
//   12288 x 768  -> 3072  108   / 100  / 85.5 / 102
//   12288 x 768  -> 768    32.1 / 32.6 / 31.4 / 29.5
//   16384 x 64   -> 4096  105   / 117  / 92.9 / 89.5
//   16384 x 512  -> 512    22.4 / 19.9 / 19.8 / 25.5
//    8192 x 4096 -> 4096  360   / 316  / 250  / 229
// on one set:
//   14248 x 1122 -> 176    22.4 / 23.2 /  -   / 45
//    9696 x 27   -> 5696   70   / 74   /  -   / 92
//    8192 x 4096 -> 11008  -    /  -   / 4 % more than 256 / 643
static const DxTile kDxCmTiles[] = {{64, false, 3, {0.45, 6.2}, {0.935, 7.4}, {0.0, 0.0}, {0.0, 0.0}, 128},
                                    {128, false, 2, {0.55, 8.4}, {0.95, 9.1}, {0.0, 0.0}, {0.0, 0.0}, 128},
                                    {128, false, 2, {0.60, 12.0}, {1.70, 12.4}, {0.0, 0.0}, {0.0, 0.0}, 256},
                                    {256, false, 1, {1.0, 21.6}, {1.34, 24.9}, {0.0, 0.0}, {0.0, 0.0}, 256}};
GemmPlan dx_cm_plan(int64_t M, int64_t N, int64_t K, double* price) {
  GemmPlan best{};
  const double stages = (double)ceil_div(K, KALIGN);
  for (const DxTile& c : kDxCmTiles) {
    const bool wide = c.t == 128 && c.bn == 256;
    if (wide && (M % 128 || N % 256)) continue;         // whole tiles only: what was measured
    const int64_t tm = ceil_div(M, c.t), tn = ceil_div(N, c.bn), tiles = tm * tn, round = 256 * c.bpc;
    if (tiles >= (1 << 24) && c.t < 256) continue;      // a grid dimension holds less than 2^32 work items
    const double lone = c.lone[0] * stages + c.lone[1], full = c.full[0] * stages + c.full[1];
    double t = (double)(tiles / round) * full;
    if (const int64_t rest = tiles % round)
      t += lone + (full - lone) * (c.bpc > 1 ? (double)(ceil_div(rest, 256) - 1) / (c.bpc - 1) : (double)rest / 256.0);
    if (best.tile == 0 || t < *price) { *price = t; best = GemmPlan{c.t, 1, (int)tm, (int)tn, false, wide}; }
  }
  return best;
}

// Both products in one grid of 64-row tiles.  Neither fills the chip by itself where this is taken, and the shorter one, its
// launch and its drain disappear beside the other.  By the tables above, the blocks of both share the places on the CUs;
// more blocks than places are priced by the work in them, and a quarter of the longest block at the end.
static bool pair_search(double stages, int64_t tm, int64_t tn, const DxTile& c, bool f32, double places, DwKind kind, int64_t dw_m,
                        int64_t dw_n, int64_t dw_k, double* apart, GemmPlan* dx, GemmPlan* dw) {
  const DwTile& w = kDwTiles[kind][0];
  const int64_t wm = ceil_div(dw_m, w.bm), wn = ceil_div(dw_n, w.bn), wstages = ceil_div(dw_k, KALIGN);
  bool found = false;
  if (tm * tn + wm * wn * 64 >= (1 << 24)) return false;
  const double xl = c.lone[0] * stages + c.lone[1] + (f32 ? c.f32[0] : 0.0), xf = c.full[0] * stages + c.full[1] + (f32 ? c.f32[1] : 0.0);
  for (int64_t s = 1; s <= 64 && (s == 1 || 2 * s <= wstages); ++s) {
    const int64_t per = ceil_div(wstages, s);
    if (ceil_div(wstages, per) != s) continue;
    const double wl = w.lone[0] * (double)per + w.lone[1], wf = w.full[0] * (double)per + w.full[1];
    const double fx = (double)(tm * tn) / places, fw = (double)(wm * wn * s) / places, f = fx + fw;
    const double load = f < 1.0 ? f : 1.0;
    const double bx = xl + (xf - xl) * load, bw = wl + (wf - wl) * load;
    const double t = (f <= 1.0 ? std::max(bx, bw) : fx * xf + fw * wf + 0.25 * std::max(xf, wf)) + finish_price(dw_m, dw_n, s);
    if (t < *apart) {
      *apart = t; found = true;
      *dx = GemmPlan{64, 1, (int)tm, (int)tn, c.ring};
      *dw = GemmPlan{64, (int)s, (int)wm, (int)wn, false};
    }
  }
  return found;
}
bool pair_plan(int64_t M, int64_t N, int64_t K, bool f32, bool conv, const ConvDxStridedMap* strided, DwKind kind, int64_t dw_m,
               int64_t dw_n, int64_t dw_k, double apart, GemmPlan* dx, GemmPlan* dw) {
  // A dX that is bound by memory takes the wider tiles of a launch of its own.  One grid / two launches, us: fp32 13888 x 128 -> 3248,
  // k = 32 (412 MB) 158 / 140, 13184 x 64 -> 2616 (315 MB) 162 / 146, but 7776 x 24 -> 4234 (300 MB) 187 / 197; bf16 5824 x 64 -> 9856
  // (294 MB) 125 / 105, 9984 x 75 -> 4672 (239 MB) 82 / 86.
  if (!conv && dx_traffic_mb(M, N, f32) > (f32 ? 312.0 : 270.0)) return false;
  bool found = false;
  for (int ring = 0; ring < 2; ++ring) {
    const DxTile& c = conv ? kDxConvTiles[1 - ring] : kDxTiles[1 - ring];
    int64_t tm = 0;
    const double stages = dx_stages(M, K, c.t, strided, &tm);
    found |= pair_search(stages, tm, ceil_div(N, c.t), c, f32, 256.0 * (ring ? 3 : 4), kind, dw_m, dw_n, dw_k, &apart, dx, dw);
  }
  return found;
}
// The same for a channel-major bf16 dY (k_pair_cm): dX on 64 x 128 tiles of k_gemm_dx8, dW on those of its DW form, three
// blocks a CU.
bool pair_cm_plan(int64_t M, int64_t N, int64_t K, int64_t dw_m, int64_t dw_n, int64_t dw_k, double apart, GemmPlan* dx, GemmPlan* dw) {
  return pair_search((double)ceil_div(K, KALIGN), ceil_div(M, 64), ceil_div(N, kDxCmTiles[0].bn), kDxCmTiles[0], false, 256.0 * 3, DW_ROWS, dw_m,
                     dw_n, dw_k, &apart, dx, dw);
}

bool gemm_epilogue_vec_ok(const GemmEpilogueDx& e, int64_t N) {
  return (N % 8) == 0 && ((uintptr_t)e.x_codes % 8) == 0 && ((uintptr_t)e.x % 16) == 0 && ((uintptr_t)e.dx % 16) == 0;
}

template <int BM, int BN, int EPI, bool I8, int CONV = 0>
static int launch_cfg(const typename ConvArgs<CONV>::type& a, int split_k, hipStream_t st) {
  using C = TileCfg<BM, BN, 2>;
  constexpr int kLds = C::template lds_bytes<EPI>() + (CONV == 2 ? BM * (int)sizeof(int) : 0);
  // set once per process (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_gemm_nt<BM, BN, EPI, I8, CONV>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return EFQAT_ERR_HIP;
  const dim3 grid((unsigned)(a.tiles_m * a.tiles_n * split_k));
  constexpr int kProf = (EPI == EPI_DX || EPI == EPI_DXF) ? PROF_DX : (EPI == EPI_RAW ? PROF_DW : PROF_FWD);
  {
    ProfScope prof(kProf, st);
    hipLaunchKernelGGL((k_gemm_nt<BM, BN, EPI, I8, CONV>), grid, dim3(256), kLds, st, a);
  }
  EFQAT_LAUNCH_CHECK();
  return EFQAT_OK;
}

static void fill_epilogue(GemmArgs& a, const GemmEpilogueDx& epi) {
  a.x_codes = epi.x_codes; a.x_clip = epi.x_clip; a.x = epi.x; a.x_dtype = epi.x_dtype;
  a.s_x = epi.s_x; a.z_x = epi.z_x; a.dx = epi.dx; a.dx_dtype = epi.dx_dtype; a.partial = epi.partial;
  a.epi_vec = gemm_epilogue_vec_ok(epi, a.N) ? 1 : 0;
}

int dw_args_staged(GemmArgs* out, const bf16_t* A, int64_t lda, const int32_t* a_rows, const bf16_t* B, int64_t ldb, int64_t M,
                   int64_t N, int64_t K, const GemmPlan& plan, float* out_partial) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 8) || (lda % 8) || (ldb % 8)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return EFQAT_ERR_BAD_SHAPE;
  GemmArgs a{};
  a.A = A; a.lda = lda; a.a_rows = a_rows; a.B = B; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(ceil_div(K, KALIGN), plan.split_k) * KALIGN);
  a.out = out_partial;
  a.tiles_m = plan.tiles_m; a.tiles_n = plan.tiles_n;
  *out = a;
  return EFQAT_OK;
}

int dx_args_linear(GemmArgs* out, const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                   const GemmPlan& plan, const GemmEpilogueDx& epi) {
  if (plan.split_k != 1) return EFQAT_ERR_BAD_SHAPE;
  if (((uintptr_t)A % 16) || ((uintptr_t)B % 16)) return EFQAT_ERR_ALIGNMENT;
  const int rc = dw_args_staged(out, A, lda, nullptr, B, ldb, M, N, K, plan, nullptr);
  if (rc == EFQAT_OK) fill_epilogue(*out, epi);
  return rc;
}

int dx_args_conv(GemmArgs* out, const bf16_t* dy_tok, int64_t ldc, const bf16_t* wqT, int64_t ldb, int64_t M, int64_t N, int64_t K,
                 const ConvDxMap& cm, const GemmPlan& plan, const GemmEpilogueDx& epi) {
  if ((ldc % 64) || (K % 64) || cm.H > 65535 || cm.W > 65535) return EFQAT_ERR_BAD_SHAPE;
  const int rc = dx_args_linear(out, dy_tok, ldc, wqT, ldb, M, N, K, plan, epi);
  if (rc) return rc;
  GemmArgs& a = *out;
  a.cv_H = cm.H; a.cv_W = cm.W; a.cv_Ho = cm.Ho; a.cv_Wo = cm.Wo; a.cv_KW = cm.KW; a.cv_pad = cm.pad;
  a.cv_spt = (int)(ldc / 64);
  a.cv_m_spt = (1ull << 32) / (uint64_t)a.cv_spt + 1; a.cv_m_kw = (1ull << 32) / (uint64_t)cm.KW + 1;
  return EFQAT_OK;
}

int launch_gemm_nt_raw(const GemmArgs& a, const GemmPlan& plan, hipStream_t stream) {
  switch (plan.tile) {
    case 256: return launch_cfg<256, 256, EPI_RAW, false>(a, plan.split_k, stream);
    case 192: return launch_cfg<192, 192, EPI_RAW, false>(a, plan.split_k, stream);
    case 128: return launch_cfg<128, 128, EPI_RAW, false>(a, plan.split_k, stream);
    case 64: return launch_cfg<64, 64, EPI_RAW, false>(a, plan.split_k, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}

int launch_dx(const GemmStridedArgs& a, int conv, const GemmPlan& plan, bool beside, hipStream_t stream) {
  const bool fast = dx_epilogue_fast(a, plan.tile, plan.tile);
  if (plan.ring)
    return conv == 2 ? launch_gemm_kk_conv_strided(a, plan.tile, stream)
                     : conv == 1 ? launch_gemm_kk_conv(a, plan.tile, stream) : launch_gemm_kk(a, plan.tile, beside, stream);
  if (conv == 2)
    return plan.tile == 64 ? launch_cfg<64, 64, EPI_DX, false, 2>(a, 1, stream) : launch_cfg<128, 128, EPI_DX, false, 2>(a, 1, stream);
  if (conv == 1) {
    switch (plan.tile) {
      case 192: return fast ? launch_cfg<192, 192, EPI_DXF, false, 1>(a, 1, stream) : launch_cfg<192, 192, EPI_DX, false, 1>(a, 1, stream);
      case 128: return fast ? launch_cfg<128, 128, EPI_DXF, false, 1>(a, 1, stream) : launch_cfg<128, 128, EPI_DX, false, 1>(a, 1, stream);
      case 64: return launch_cfg<64, 64, EPI_DX, false, 1>(a, 1, stream);
      default: return EFQAT_ERR_BAD_SHAPE;
    }
  }
  switch (plan.tile) {                                  // tiles of 192 always take the ring
    case 256: return launch_cfg<256, 256, EPI_DX, false>(a, 1, stream);
    case 128: return fast ? launch_cfg<128, 128, EPI_DXF, false>(a, 1, stream) : launch_cfg<128, 128, EPI_DX, false>(a, 1, stream);
    case 64: return launch_cfg<64, 64, EPI_DX, false>(a, 1, stream);
    default: return EFQAT_ERR_BAD_SHAPE;
  }
}

// Phases of a convolution with stride s <= kMaxConvStride, most taps first; returns the row tiles in all.
static int64_t conv_phases(const ConvDxStridedMap& cm, int tile, ConvPhase* out, int* nphase) {
  ConvPhase p[kMaxConvStride * kMaxConvStride];
  int n = 0;
  const int s = cm.stride;
  // taps kh with (ph + pad - kh) % s == 0: kh0 = (ph + pad) % s, kh0 + s, ...; the first reaches output row hi + dh0
  auto taps = [s](int K, int first) { return first < K ? (K - first + s - 1) / s : 0; };
  for (int ph = 0; ph < s; ++ph)
    for (int pw = 0; pw < s; ++pw) {
      ConvPhase c{};
      c.ph = ph; c.pw = pw;
      c.Hp = cm.H > ph ? (cm.H - ph + s - 1) / s : 0;
      c.Wp = cm.W > pw ? (cm.W - pw + s - 1) / s : 0;
      c.rows = cm.N * c.Hp * c.Wp;
      c.kh0 = (ph + cm.pad) % s; c.kw0 = (pw + cm.pad) % s;
      c.dh0 = (ph + cm.pad) / s; c.dw0 = (pw + cm.pad) / s;
      const int nkh = taps(cm.KH, c.kh0);
      c.nkw = taps(cm.KW, c.kw0);
      c.ntap = nkh * c.nkw;
      if (c.nkw == 0) c.nkw = 1;                        // never divided by
      c.tiles = (int)ceil_div(c.rows, tile);
      if (c.rows > 0) p[n++] = c;
    }
  int64_t total = 0;
  for (int i = 0; i < n; ++i) {                         // selection by taps, stable
    int best = -1;
    for (int j = 0; j < n; ++j)
      if (p[j].tiles >= 0 && (best < 0 || p[j].ntap > p[best].ntap)) best = j;
    ConvPhase c = p[best];
    p[best].tiles = -1;
    c.tile0 = (int)total;
    total += c.tiles;
    if (out) out[i] = c;
  }
  if (nphase) *nphase = n;
  return total;
}

int64_t conv_dx_strided_row_tiles(const ConvDxStridedMap& cm, int tile) { return conv_phases(cm, tile, nullptr, nullptr); }

int dx_args_strided(GemmStridedArgs* out, const bf16_t* dy_tok, int64_t ldc, const bf16_t* wqT, int64_t ldb, int64_t M, int64_t N,
                    const ConvDxStridedMap& cm, const GemmPlan& plan, const GemmEpilogueDx& epi) {
  if (M <= 0 || N <= 0 || (ldc % 64) || (ldb % 8) || cm.H > 65535 || cm.W > 65535 || cm.stride < 2 ||
      cm.stride > kMaxConvStride || (plan.tile != 128 && plan.tile != 64) || plan.split_k != 1 || M > INT32_MAX || N > INT32_MAX)
    return EFQAT_ERR_BAD_SHAPE;
  GemmStridedArgs a{};
  a.A = dy_tok; a.lda = ldc; a.B = wqT; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N;
  fill_epilogue(a, epi);
  a.cv_H = cm.H; a.cv_W = cm.W; a.cv_Ho = cm.Ho; a.cv_Wo = cm.Wo; a.cv_KW = cm.KW; a.cv_pad = cm.pad;
  a.cv_stride = cm.stride;
  a.cv_spt = (int)(ldc / 64);
  a.cv_m_spt = (1ull << 32) / (uint64_t)a.cv_spt + 1;
  a.tiles_n = plan.tiles_n;
  a.tiles_m = (int)conv_phases(cm, plan.tile, a.phase, &a.nphase);
  if (a.tiles_m != plan.tiles_m) return EFQAT_ERR_BAD_SHAPE;
  *out = a;
  return EFQAT_OK;
}

// Tile of the int8 forward product.  `lone` / `full`: microseconds per K stage of 128 codes and per block (launch, first
// loads, epilogue) with one block on a CU and with all `bpc` that fit (LDS); between the two by the number resident.  A
// product is its whole rounds of 256 * bpc blocks plus what is left.  Fitted to measured launches; against the tile that
// is fastest by measurement at 12 sizes of 128 .. 16384 tokens the choice loses 5 % at most.  T x C_in -> C_out, us with
// tiles of 256x256 / 192x128 / 128x128 / 64x64:
//   8192 x 4096 -> 4096    136 / 146 / 151 / 229    whole rounds of large tiles: fewest LDS bytes per operation
//   2048 x 4096 -> 11008   138 / 105 / 120 / 161    two 192x128 blocks fill the 160 KB of LDS and overlap their epilogues
//   12288 x 768 -> 3072     67 /  43 /  50 /  66
//   2048 x 4096 -> 4096    few tiles: 128x128 is one round of two blocks a CU
//   512 x 4096 -> 4096      57 /  31 /  26 /  21    less than one tile per CU: latency, the smallest tile
struct FwdTile { int bm, bn, bpc; double lone[2], full[2]; };
static const FwdTile kFwdTiles[] = {{256, 256, 1, {1.75, 13.5}, {1.75, 13.5}},
                                    {192, 128, 2, {0.77, 5.9}, {1.30, 7.0}},
                                    {128, 128, 2, {0.67, 4.3}, {1.06, 5.0}},
                                    {64, 64, 5, {0.53, 2.4}, {1.00, 3.0}}};
static FwdTile fwd_tile(int64_t M, int64_t N, int64_t K) {
  const double stages = (double)ceil_div(K, 128);
  const FwdTile* best = nullptr;
  double best_t = 0.0;
  for (const FwdTile& c : kFwdTiles) {
    const int64_t tiles = ceil_div(M, c.bm) * ceil_div(N, c.bn), round = 256 * c.bpc;
    if (tiles >= (1 << 24) && c.bm < 256) continue;     // a grid dimension holds less than 2^32 work items
    const double lone = c.lone[0] * stages + c.lone[1], full = c.full[0] * stages + c.full[1];
    double t = (double)(tiles / round) * full;
    if (const int64_t rest = tiles % round) {
      const int64_t resident = ceil_div(rest, 256);
      t += lone + (full - lone) * (double)(resident - 1) / (double)std::max(1, c.bpc - 1);
    }
    if (!best || t < best_t) { best = &c; best_t = t; }
  }
  return *best;
}

int fwd_tile_columns(int64_t M, int64_t N, int64_t K) { return fwd_tile(M, N, K).bn; }

int launch_gemm_fwd_i8(const uint8_t* x_codes, int64_t lda, const int8_t* w_codes, int64_t ldb, int64_t M, int64_t N,
                       int64_t K, const float* s_x, const float* z_x, const float* s_w, void* y, int y_dtype,
                       hipStream_t stream) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 16) || (lda % 16) || (ldb % 16)) return EFQAT_ERR_BAD_SHAPE;
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return EFQAT_ERR_BAD_SHAPE;
  GemmArgs a{};
  a.A = x_codes; a.lda = lda; a.a_rows = nullptr; a.B = w_codes; a.ldb = ldb;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.k_per_split = (int)(ceil_div(K, 2 * KALIGN) * 2 * KALIGN);
  a.s_x = s_x; a.z_x = z_x; a.s_w = s_w; a.y = y; a.y_dtype = y_dtype;
  a.epi_vec = ((N % 8) == 0 && ((uintptr_t)y % 16) == 0) ? 1 : 0;
  const FwdTile t = fwd_tile(M, N, K);
  a.tiles_m = (int)ceil_div(M, t.bm);
  a.tiles_n = (int)ceil_div(N, t.bn);
  switch (t.bm) {
    case 256: return launch_cfg<256, 256, EPI_FWD, true>(a, 1, stream);
    case 192: return launch_cfg<192, 128, EPI_FWD, true>(a, 1, stream);
    case 128: return launch_cfg<128, 128, EPI_FWD, true>(a, 1, stream);
    default: return launch_cfg<64, 64, EPI_FWD, true>(a, 1, stream);
  }
}

}  // namespace efqat
