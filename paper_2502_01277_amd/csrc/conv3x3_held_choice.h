// What a model keeps for a 3x3 layer that may run on conv3x3_held_kernel, and which launches do.  Host arithmetic only.
#pragma once
#include "octo_internal.h"
#include <algorithm>

namespace octo {

// The three tiles: channels x pixels, the wavefronts that share K, and the time of a launch in us in its place in a model, by stride: a constant, per 64 input channels, and
// what a compute unit does - half way between its mean number of tiles and the next whole one, at least one - per tile and 64 channels, per tile and per 4 KB
// of patch, and the memory traffic in MB.  Fitted, without negative terms, to 988 launches that the rule below allows (residual error 5 - 8 %; of the best
// tile's time the choice takes 1.002).
struct HeldTile { int bc, bp, ks; double cost[2][6]; };
constexpr HeldTile HELD_TILE[3] = {
    {64, 32, 4, {{3.321, 0.112, 0.677, 0.000, 0.0000, 0.198}, {3.203, 0.248, 0.517, 0.399, 0.0249, 0.057}}},
    {64, 64, 4, {{4.001, 0.017, 0.609, 0.000, 0.0548, 0.287}, {4.243, 0.258, 0.000, 1.145, 0.0519, 0.063}}},
    {64, 128, 2, {{4.590, 0.000, 1.105, 0.366, 0.0501, 0.138}, {0, 0, 0, 0, 0, 0}}}};

// Geometry of a tile: TH rows of the stack of output images (consecutive in memory, so a tile may span several) x TW columns; a patch of PH x PW input pixels, `halo` of
// its columns left of the tile (0 where the tile spans the image); rows: the patch and two rows of zeros in whole passes of the loader.  rows = 0: none.
struct HeldGeom {
  int TH, TW, PW, PH, halo, tiles_x, rows, lds;
  FastDiv div_tw, div_pw, div_tx, div_th;
};
struct HeldPlan {
  const void* w = nullptr;       // device: the weights in the kernel's order
  HeldGeom geom[3]{};
  FastDiv div_ho{}, div_tc{};
};

// Layers that get a plan: 16-bit types, 3x3, padding 1, input channels in 64s up to 512, output channels in 64s, and at stride 2 an even height: output row v of the
// stack then needs input rows 2 v - 1 .. 2 v + 1.
inline bool held_layer(int kh, int kw, int stride, int pad, int H, int cin, int cout) {
  return kh == 3 && kw == 3 && pad == 1 && (stride == 1 || (stride == 2 && H % 2 == 0)) && cin % 64 == 0 && cin <= 512 && cout % 64 == 0 && (long long)cout * cin * 18 < 0x7FFFFFFFLL;
}

// The split of the image width into equal columns and the number of rows that give the most pixels per tile of at most bp, ties to the smaller patch; none where no
// shape fills 3/4 of the tile or the patch exceeds LDS.
inline HeldGeom held_geometry(const HeldTile& c, int S, int W, int Wo, int cin) {
  HeldGeom g{};
  const int slices = cin / 64, max_rows = 160 * 8 / slices;
  double best = 0;
  int best_patch = 0;
  for (int nx = 1; nx <= Wo; ++nx) {
    const int tw = (Wo + nx - 1) / nx, pw = nx == 1 ? W : S * (tw - 1) + 3;
    if (tw > c.bp) continue;
    if (tw < 4) break;
    const int ph = (max_rows / 32 * 32 - 2) / pw, th = std::min(c.bp / tw, ph < 3 ? 0 : (ph - 3) / S + 1);
    if (th < 1) continue;
    const int tiles_x = (Wo + tw - 1) / tw, patch = (S * (th - 1) + 3) * pw;
    const double px = (double)Wo * th / tiles_x;
    if (px > best || (px == best && patch < best_patch)) {
      best = px; best_patch = patch;
      g.TW = tw; g.TH = th; g.PW = pw; g.PH = S * (th - 1) + 3; g.halo = nx == 1 ? 0 : 1; g.tiles_x = tiles_x;
    }
  }
  if (best * 4 < c.bp * 3) return HeldGeom{};
  g.rows = (best_patch + 2 + 31) / 32 * 32;
  g.lds = std::max(slices * g.rows * 128, c.bc * c.bp * 4 * c.ks);
  g.div_tw = make_fastdiv((unsigned)g.TW); g.div_pw = make_fastdiv((unsigned)g.PW);
  g.div_tx = make_fastdiv((unsigned)g.tiles_x); g.div_th = make_fastdiv((unsigned)g.TH);
  return g;
}
inline HeldPlan held_plan(int S, int W, int Ho, int Wo, int cin, int cout) {
  HeldPlan p;
  for (int i = 0; i < (S == 1 ? 3 : 2); ++i) p.geom[i] = held_geometry(HELD_TILE[i], S, W, Wo, cin);
  p.div_ho = make_fastdiv((unsigned)Ho); p.div_tc = make_fastdiv((unsigned)(cout / 64));
  return p;
}
// Can any launch of the layer, whatever its number of items and the device, go to the kernel (held_choose)?  Where none can, no second copy of its weights is kept.
inline bool held_ever(const HeldPlan& p, int stride, int cin) {
  if (stride == 2 && cin < 128) return false;
  bool any = false;
  for (int i = 0; i < (stride == 1 ? 3 : cin < 256 ? 1 : 2); ++i) any = any || p.geom[i].rows > 0;
  return any;
}

// Weights in the order that the kernel reads them: for every block of 32 output channels, group of 16 input channels and tap the 1 KB of one wavefront's operand.
// Lane l holds channel 16 ((m / 4) % 2) + 4 (m / 8) + m % 4 of the block, m = l % 32, and input channels 8 (l / 32) .. 8 (l / 32) + 7 of the group; with that order of
// rows a lane's 16 results are consecutive channels of its pixel.
inline size_t held_weight_bytes(int cout, int cin) { return (size_t)cout * cin * 18; }

// Does the launch have the form that the kernel takes?
inline bool held_fits(const ConvArgs& a) {
  if (!a.held || a.out_f32 || a.pair_view || a.pool_y || a.up_y || a.split > 0) return false;
  if (((a.x_ld | a.x_coff | a.y_ld | a.y_coff) & 7) || (((uintptr_t)a.x | (uintptr_t)a.y) & 15)) return false;
  if (a.res && (((a.res_ld | a.res_coff) & 7) || ((uintptr_t)a.res & 15))) return false;
  // 32-bit offsets inside a tile of up to 128 pixels, and pixel numbers
  return (131LL * a.W + 256) * std::max(a.x_ld, std::max(a.y_ld, a.res ? a.res_ld : 0)) * 2 < 0x7FFFFFF0LL && (long long)a.n * a.H * a.W < 0x7FFFFF00LL;
}
inline long long held_tiles(const ConvArgs& a, long long items, int which) {
  const HeldGeom& g = a.held->geom[which];
  return (items * a.Ho + g.TH - 1) / g.TH * g.tiles_x * (a.Cout / 64);
}
inline int held_resident(const ConvArgs& a, int which, int num_cu) { return num_cu * std::min(2, 160 * 1024 / a.held->geom[which].lds); }
inline double held_cost_us(const ConvArgs& a, long long items, int which, int num_cu) {
  const double (&c)[6] = HELD_TILE[which].cost[a.stride_h - 1];
  const long long tiles = held_tiles(a, items, which);
  const double k = a.Cin / 64, per_cu = std::max(1.0, 0.5 * ((double)tiles / num_cu + (double)((tiles + num_cu - 1) / num_cu)));
  const double mb = 2e-6 * items * ((double)a.H * a.W * a.Cin + (double)a.Ho * a.Wo * a.Cout * (a.res ? 2 : 1));
  return c[0] + c[1] * k + per_cu * (c[2] * k + c[3] + c[4] * k * a.held->geom[which].rows / 32) + c[5] * mb;
}
// Where the count is taken on the device the choice is made for the stated one, so that an item's results do not depend on its neighbours' number, and the running count may be many times that.
// A kernel of the common order follows it with larger tiles, this one cannot.  Where the capacity is no more than eight times the stated count a layer goes by that like any other: up to about three
// times it this kernel is ahead, at eight times even or, at worst, 16 % behind.  Us in place, the kernel before : this one, items: 16 x 8 x 256, stated 128, 58 15.9 : 11.4, 116 18.3 : 18.0, 177 26.4 : 25.0, 336
// 47.3 : 48.4, 883 110 : 110; 14 x 14 x 256, stated 64, 32 15.0 : 11.0, 64 17.6 : 17.5, 191 43.0 : 41.9, 478 101 : 100; 28 x 28 x 128, stated 32, 24 12.0 : 11.7, 70 22.3 : 21.0, 183 46 : 43.6, 242 60 : 60;
// 32 x 16 x 128, stated 64, 32 12.4 : 8.9, 64 14.7 : 13.1, 191 30.8 : 30.9, 478 61 : 72; 8 x 8, stride 2, 128 -> 256, stated 64, 64 7.1 : 6.3, 191 10.3 : 8.7, 478 11.2 : 11.4.
// With more room than that only where it is about even at fourteen times the stated count too: in place of kernels that are tied to the stated count themselves, split-K and the narrow tiles of
// conv3x3_mid_kernel.  By tiles of 64 x 64 per compute unit at the stated count:
//   * 512 channels up to 1.7, 256 .. 448 up to 2.5: 7 x 7 x 512 at 1.5, stated 64, 59 items 26.0 : 19.0, 455 122 : 97, 843 217 : 183, at 1.95, stated 80, 78 items 27.2 : 18.4, 571 110 : 116, 1074
//     215 : 228; 14 x 14 x 256 at 2.3, stated 48, 42 items 17.4 : 17.3, 344 73.9 : 74.5, 656 132 : 133, at 3.1, stated 64, 32 items 15 : 11, 59 18.5 : 17.9, 843 172 : 180.  Beyond, where it loses
//     some 5 % at many times the stated count and gains up to a third at less than it, while no more than 32 times that count has room: passes of 10 frames with 200 items each at most and 4 or
//     8 there 903 : 869 and 1047 : 1016, of 9 with 300 and 109 there 7520 : 7580;
//   * 128 and 192 up to 2.5: 28 x 28 at 2.3, 22 items 13.3 : 12.8, 177 45.8 : 44.9, 331 78.8 : 81.2, at 3.8, 33 items 13.3 : 12.4, 294 67.2 : 74.2, 542 113 : 135;
//   * not with 64: 56 x 56, stated 16, 19 items 11.1 : 10.5, 71 23.5 : 25.2, 228 66.8 : 72.9;
//   * stride 2, in place of split-K only: 256 -> 512 on 14 x 14 at 0.22, stated 8, 6 items 7.2 : 6.9, 111 38.3 : 23.3, at 0.7, stated 24, 22 items 10.4 : 9.0, 57 13.3 : 15.6, 331 50.4 : 62.4,
//     stated 40, 542 65 : 104; 512 -> 512 on 16 x 8 at 0.5, stated 32, 27 items 18.3 : 14.0, 240 72.8 : 76.1; 128 -> 256 on 8 x 8, stated 128, 118 items 8.1 : 6.5, 923 16.5 : 20.4.
inline bool held_counted(const ConvArgs& a, long long M, int num_cu) {
  const double per_cu = (double)((M + 63) / 64 * (a.Cout / 64)) / num_cu;
  const long long room = (long long)a.n * a.Ho * a.Wo;
  if (M * 8 >= room) return true;
  if (a.stride_h == 2) return a.Cin >= 256 && per_cu <= (a.Cin >= 512 ? 0.5 : 0.25);
  if (a.Cin < 256) return a.Cin >= 128 && per_cu <= 2.5;
  return per_cu <= (a.Cin >= 512 ? 1.7 : 2.5) || M * 32 >= room;
}
// The tile of a layer with M output pixels, or -1 where another kernel is the faster one.  Measured in place, the kernels before : this one, us, by tiles of 64 x 64 per
// compute unit.  A launch is taken
//   * while its tiles are resident at a time (two workgroups per compute unit, one with more than 80 KB of patch).  256 -> 256 on 20 x 20 at 0.2 7.3 : 6.6, at 0.4
//     12.9 : 7.6, at 0.8 15.6 : 9.0, at 1.6 16.0 : 11.6, at 2.3 (three rounds of 64 x 64) 17.9 : 17.1, at 3.1 19.3 : 20.4, on 14 x 14 at 3.7 19.0 : 18.6, at 6.4
//     31.1 : 33.2; 512 -> 512 on 7 x 7 at 0.1 9.6 : 9.1, at 0.36 17.5 : 9.7, at 1.0 25.6 : 15.0, at 1.8 26.7 : 18.1, at 3.2 29.8 : 31.0; 384 -> 384 on 40 x 40 at
//     0.6 19.7 : 11.5, at 1.2 20.3 : 14.7, at 2.3 22.4 : 25.8.  At stride 2 256 -> 512 on 7 x 7 at 0.36 9.2 : 7.3, at 1.0 14.9 : 10.0, at 1.8 17.9 : 16.7;
//   * with 128 and 192 channels, whose patch leaves room for two workgroups, up to five 64 x 128 tiles per compute unit, where no count is taken on the device: 128 -> 128 on 40 x 40 at 0.2
//     5.6 : 5.1, at 1.6 9.4 : 8.7, at 2.1 13.5 : 13.2, at 3.9 16.2 : 15.6, at 4.1 (conv3x3_mid_kernel leaves its wide slices) 17.4 : 17.9, at 4.9 18.3 : 18.3, at 5.9 19.7 : 18.6, at 9.4
//     30.0 : 27.8, beyond at 10.2 35.8 : 36.6; 192 -> 192 on 80 x 80 at 1.2 13.3 : 10.7, at 4.7 23.8 : 21.2, at 9.4 36.4 : 34.3, beyond at 10.5 38.8 : 42.2, at 11.7 40.8 : 42.7;
//   * with 64 only from where conv_small_kernel leaves: 64 -> 64 on 80 x 80 at 0.8 4.7 : 5.0, at 1.6 6.8 : 7.1, at 2.3 9.2 : 8.4, at 3.9 11.1 : 9.4, at 4.7 (more than are
//     resident) 12.6 : 12.9;
//   * at stride 2 with 128 only a quarter to one 64 x 32 tile per compute unit: 128 -> 256 on 4 x 4 at 0.3 8.1 : 6.3, 128 -> 128 on 40 x 40 at 0.4 5.8 : 5.4, at 0.6 6.7 :
//     6.8, 128 -> 256 on 4 x 4 at 0.07 5.5 : 5.3; not with 64 (64 -> 128 on 40 x 40 at 0.8 4.9 : 5.7).
// Over 408 layers of three detectors and three classifiers (1 .. 48 frames) 0.85 of the time of the kernels before, at most 1.07.  Tiles of 64 x 32 and 64 x 64 sum in
// one order, so that a running count may choose between them; all else is chosen for M, which stays the same from batch to batch.
inline int held_choose(const ConvArgs& a, long long M, int num_cu) {
  const int S = a.stride_h;
  if (a.n_dyn && !held_counted(a, M, num_cu)) return -1;
  if (a.Cin < 128 && (S == 2 || (double)((M + 63) / 64 * (a.Cout / 64)) <= 1.96 * num_cu)) return -1;
  const long long hw = (long long)a.Ho * a.Wo, items = M / hw;
  int best = -1;
  double us = 0;
  for (int i = 0; i < (S == 2 ? (a.Cin < 256 ? 1 : 2) : 3); ++i) {
    if (a.held->geom[i].rows == 0) continue;
    const bool wide = i == 2 && a.Cin >= 128 && a.Cin <= 192 && !a.n_dyn;
    const long long tiles = held_tiles(a, items, i);
    if (tiles > (wide ? 5 * num_cu : S == 2 && a.Cin < 256 ? num_cu : held_resident(a, i, num_cu))) continue;
    if (S == 2 && a.Cin < 256 && tiles * 4 < num_cu) continue;
    const double t = held_cost_us(a, items, i, num_cu);
    if (best < 0 || t < us) { us = t; best = i; }
  }
  const long long now = a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n;
  if ((best == 0 || best == 1) && now != items && a.held->geom[0].rows && a.held->geom[1].rows)
    best = held_cost_us(a, now, 0, num_cu) <= held_cost_us(a, now, 1, num_cu) ? 0 : 1;
  return best;
}

}  // namespace octo
