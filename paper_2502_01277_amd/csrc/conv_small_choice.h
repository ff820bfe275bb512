// Which layers take conv_small_kernel (conv_small.h), and with which tile.  Host arithmetic only.
#pragma once
#include "octo_internal.h"
#include "conv_flow_choice.h"
#include <algorithm>

namespace octo {

// What the kernel reads.  Pointers are to the first channel of the first pixel (y2: less the split's channels), pitches in bytes.
struct SmallArgs {
  const char* x; const char* w; const float* bias; char* y;
  const int* n_dyn;
  const char* res; char* y2;
  int n, HoWo, tiles_c, per_row;         // per_row: bytes of a weight row
  int grid, c_outer;
  FastDiv div_tc, div_tp, div_howo, div_wo;       // div_tp: by the pixel tiles of n items
  int x_pitch, y_pitch, y2_pitch, res_pitch;
  int Cout, split, nk, taps_nk;          // K steps, and those of a tap
  int H, W, Wo, kw, kh, stride, pad, Cin, K;
  unsigned magic_cin, magic_kw;
  int act, res_mode, w_len, w_rows;
};

// Layers that do not depend on one another and whose arguments are collected for one launch; the first one's tile is everyone's (all tiles sum in one order).
struct SmallGroup {
  static constexpr int MAX = 3;
  int count = 0;
  int tile[MAX], mode[MAX];
  int* kernel_id[MAX];                   // of the layers: what they report; may be null
  ConvTiming timing;                     // of the first one's dispatch
  SmallArgs layer[MAX];
};
hipError_t launch_small_group_f16(const SmallGroup& g, hipStream_t s);
hipError_t launch_small_group_bf16(const SmallGroup& g, hipStream_t s);

// How addresses are made: 1x1, stride 1, no padding, whole K steps of channels; any other layer with whole K steps of channels per
// tap; any layer (a lane works out the tap of its vector at every step); in fp32, 1x1 layers without padding whose channels end inside a
// step, stride 1 or more.
enum { SMALL_POINTWISE = 0, SMALL_TAPS = 1, SMALL_ANY = 2, SMALL_PART = 3, SMALL_STRIDED_PART = 4 };

// Does a layer of values of ES bytes have the form that the kernel takes?
inline bool small_fits(const ConvArgs& a, int ES) {
  const int VN = 16 / ES;
  if (a.out_f32 || a.pair_view || a.pool_y || a.up_y || a.kh > 15 || a.kw > 15 || a.stride_h != a.stride_w || a.pad_h != a.pad_w) return false;
  if (a.Cout % VN && (a.res || a.split > 0 || a.kh > 1 || a.kw > 1 || a.stride_h > 1)) return false;      // a last vector in pieces: detector heads
  if (((a.Cin | a.x_ld | a.x_coff | a.y_ld | a.y_coff) % VN) || (((uintptr_t)a.x | (uintptr_t)a.y) & 15)) return false;
  if (a.res && (((a.res_ld | a.res_coff) % VN) || ((uintptr_t)a.res & 15))) return false;
  if (a.x_ld * ES >= 1 << 24 || a.W * 16 >= 1 << 24) return false;      // factors of 24-bit products
  // 32-bit offsets: weights, and the pixels of a tile (64 of them) in every tensor
  const long long ld = std::max(std::max(a.x_ld, a.y_ld), std::max(a.res ? a.res_ld : 0, a.split > 0 ? a.y2_ld : 0));
  return (long long)a.w_rows * a.Kp * ES < 0x7FFFFFFFLL && 256 * ld * ES < 0x7FFFFFF0LL && (long long)a.n * a.Ho * a.Wo < 0x7FFFFF00LL &&
         (2LL * a.H * a.W + 1024LL * a.stride_h * a.stride_w + (long long)a.pad_h * a.W + a.pad_w) * a.x_ld * ES < 0x7FFFFFF0LL;
}

// Time of a launch in us in its place in a cascade: see tile_cost_us, which has the form and what it was fitted to (3x3 layers: 1.006 of the best tile's time).
constexpr TileCost SMALL_COST[5] = {
    {32, 32, 2.342, 0.0943, 0.257, 0.0996, 0.0000, 0.0057},
    {32, 64, 3.337, 0.1368, 0.258, 0.1133, 0.0088, 0.0000},
    {64, 32, 2.488, 0.1123, 0.269, 0.1886, 0.0119, 0.0080},
    {64, 64, 3.083, 0.1589, 0.444, 0.1503, 0.0159, 0.0010},
    {128, 64, 3.123, 0.2288, 0.790, 0.1466, 0.0536, 0.0000}};
// Otherwise, and fp32: from a graph, input channels in whole K steps, and not.  A constant, what a compute unit does - its tiles, half way between their mean and
// the next whole number, times K steps and an epilogue -, a latency per K step and the memory traffic.  Fitted to 1070 layers (16 .. 1024 input, 24 .. 1024 output
// channels, 1x1 and 3x3 of stride 1 and 2, with and without residual, 0.04 .. 3.5 tiles of 64 x 64 per compute unit, bf16; residual error 4 - 7 %).
struct SmallCost { int bc, bp; double base, step, tile, latency, per_mb; };
constexpr SmallCost SMALL_COST_REPEATED[2][5] = {
    {{32, 32, 2.317, 0.071, 0.250, 0.054, 0.004},
     {32, 64, 2.447, 0.114, 0.287, 0.037, 0.018},
     {64, 32, 2.547, 0.115, 0.261, 0.026, 0.010},
     {64, 64, 2.557, 0.167, 0.565, 0.033, 0.020},
     {128, 64, 2.251, 0.300, 1.201, -0.031, 0.025}},
    {{32, 32, 2.585, 0.072, 0.359, 0.101, -0.016},
     {32, 64, 2.705, 0.121, 0.474, 0.091, -0.002},
     {64, 32, 2.686, 0.105, 0.401, 0.100, 0.004},
     {64, 64, 2.891, 0.167, 0.696, 0.066, 0.020},
     {128, 64, 2.682, 0.273, 1.154, 0.022, 0.074}}};
// fp32 (steps of 32 values): input channels in whole K steps, windows that are not, 1x1 layers that are not.  Fitted to 520 layers
// (4 .. 768 input, 16 .. 512 output channels, 0.04 .. 60 tiles of 64 x 64 per compute unit; residual error 3 - 6 %); 128 x 64 tiles give nothing there.
constexpr SmallCost SMALL_COST_F32[3][4] = {
    {{32, 32, 2.159, 0.136, 0.337, 0.079, -0.003},
     {32, 64, 2.329, 0.262, 0.518, 0.074, 0.018},
     {64, 32, 2.323, 0.264, 0.500, 0.071, 0.005},
     {64, 64, 2.327, 0.504, 0.867, 0.067, 0.028}},
    {{32, 32, 2.419, 0.156, 0.447, 0.126, -0.014},
     {32, 64, 3.073, 0.282, 0.757, 0.114, 0.050},
     {64, 32, 2.895, 0.260, 0.760, 0.159, 0.044},
     {64, 64, 2.674, 0.524, 0.940, 0.109, 0.047}},
    {{32, 32, 2.297, 0.145, 0.284, 0.050, 0.012},
     {32, 64, 2.446, 0.277, 0.453, 0.031, 0.033},
     {64, 32, 2.519, 0.249, 0.361, 0.047, 0.060},
     {64, 64, 2.705, 0.475, 0.479, 0.052, 0.085}}};
// (its tiles: at least one, half way between their mean and the next whole number)
template <typename Cost> double small_per_cu(const Cost& c, const LayerWork& w) {
  const long long tiles = w.tiles(c);
  return std::max(1.0, 0.5 * ((double)tiles / w.num_cu + w.rounds(tiles)));
}
inline double small_cost_us(const SmallCost& c, const LayerWork& w) {
  return c.base + small_per_cu(c, w) * (w.nk * c.step + c.tile) + c.latency * w.nk + c.per_mb * w.mb;
}
template <int N> int small_cheapest(const SmallCost (&t)[N], const LayerWork& w, double* us) {
  int best = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double v = small_cost_us(t[i], w);
    if (i == 0 || v < *us) { *us = v; best = i; }
  }
  return best;
}
// The tile (launch_small's number) with the smallest estimate for M output pixels, in place or repeated.
inline int small_choose(const ConvArgs& a, long long M, int num_cu, int ES, bool place, double* us) {
  const LayerWork w(a, M, num_cu, ES);
  const bool whole = a.Cin % (128 / ES) == 0;
  if (ES == 4) return whole ? small_cheapest(SMALL_COST_F32[0], w, us) : small_cheapest(a.kh == 1 && a.kw == 1 && !a.pad_h ? SMALL_COST_F32[2] : SMALL_COST_F32[1], w, us);
  if (!place) return whole ? small_cheapest(SMALL_COST_REPEATED[0], w, us) : small_cheapest(SMALL_COST_REPEATED[1], w, us);
  int best = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const double v = tile_cost_us(SMALL_COST[i], w);
    if (i == 0 || v < *us) { *us = v; best = i; }
  }
  return best;
}
// Layers in fp32 take the kernel at every size, but windows with steps across taps, where a lane works out addresses at every step, only up to
// eight tiles of 64 x 64 per compute unit (over 157 of them, the kernel that took the layer : here, by those tiles: up to 0.6 1.06, 2 .. 5 1.15, 8 .. 15
// 1.06, more 0.95; 4 -> 200 on 5 x 160 x 161 58.1 : 64.7).  The matrix pipe bounds it from a few tiles per compute unit on; the general kernel's blocks of
// 32 x 32 x 2 wait for one another.  Us, before : here: 16 -> 32, stride 2 on 2 x 160 x 160 5.9 : 5.2; 1x1 64 -> 192 on 10 x 16 x 17 5.4 : 3.7, 128 -> 256 on
// 11 x 56 x 56 36.8 : 29.4, 768 -> 64 on 3 x 112 x 114 59.2 : 36.5, 200 -> 512 on 837 x 7 x 8 112 : 105; 3x3 160 -> 39 on 324 x 16 x 17 170 : 135; 128 -> 384,
// stride 2 on 2 x 160 x 161 151 : 99.  Over the 520 layers 0.83 of the time and 0.75 of the error against 64 bits.
// Long reductions of few tiles stay with the split-K kernel's 32 x 32 and 64 x 32 tiles, by these estimates (same layers, up to three such tiles per
// compute unit, residual error 4 - 6 %): 284 -> 32 on 2 x 40 x 40 15.4 : 25.5, 512 -> 512 on 16 x 17 26.2 : 33.1, 256 -> 39 on 56 x 58 14.4 : 18.3.
// 1x1 layers leave beyond 64 tiles: the general kernel's 128 x 128 tiles read the pixels half as often (44 -> 352, stride 2 on 1346 x 33 x 33 at 133 266 : 312,
// 24 -> 256 on 361 x 32 x 33 at 93 146 : 158, 64 -> 256 on 22 x 153 x 120 at 98 195 : 206; 72 -> 256 on 60 x 56 x 57 at 46 116 : 112, 36 -> 128 on
// 201 x 40 x 41 at 40 128 : 108).
inline bool small_takes_f32(const ConvArgs& a, long long M, int num_cu) {
  const long long tiles = (M + 63) / 64 * ((a.Cout + 63) / 64);
  if (a.kh == 1 && a.kw == 1 && !a.pad_h) return tiles <= 64LL * num_cu;
  return a.Cin % 32 == 0 || tiles <= 8LL * num_cu;
}
constexpr SmallCost SPLIT_COST_F32[3] = {{32, 32, 2.732, 0.181, 1.363, -0.034, 0.0}, {32, 32, 3.103, 0.174, 0.691, -0.002, 0.0}, {64, 32, 3.364, 0.335, 0.952, -0.049, 0.0}};
// The split-K shape (launch_ksplit's numbers) with an estimate below `us`, or -1.
inline int small_split_f32(const ConvArgs& a, long long M, int num_cu, double us) {
  const LayerWork w(a, M, num_cu, 4);
  int best = -1;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (w.tiles(SPLIT_COST_F32[i]) > 3LL * num_cu) continue;
    const double t = small_cost_us(SPLIT_COST_F32[i], w);
    if (t < us) { us = t; best = i; }
  }
  return best;
}

// Up to how many tiles of 64 x 64 per compute unit a layer is one of few tiles: split-K is asked, and where conv_flow_kernel does not fit or the channels end
// inside a K step, and for single layers, this kernel takes the layer (us here : the kernel that took it before, from a graph unless said).  M: output pixels.
//   * windows (3x3, strides): 2.75; into one channel tile, or with steps across taps, 1.96: beyond, some unit has a third tile.  128 -> 256, stride 2 on
//     5 x 80 x 80 at 1.95 9.4 : 11.8, 256 -> 256 on 20 x 40 x 40 1.95 15.1 : 18.7, 192 -> 256 on 28 x 40 x 41 2.9 18.3 : 19.8, 96 -> 192 on 9 x 57 x 83 at 2.0 12.3 :
//     12.1, 128 -> 64 on 82 x 40 x 40 at 2.0 13.8 : 15.2.  In place up to five steps across taps 16: 32 -> 64, stride 2 on 8 x 320 x 320 at 12.5 23.1 : 28.2, on 16
//     at 25 49.0 : 47.6, on 64 207 : 188; 47 layers of 8 .. 288 channels, windows of 1 .. 5, at 1.5 .. 10 0.80 .. 0.96 of the time (32 -> 48, stride 2 on 18 x 112 x
//     110 10.8 : 11.6, 96 -> 64 1x1, stride 2 on 220 x 40 x 42 10.5 : 11.4), at 11 .. 15 0.91 .. 1.05 (24 -> 128, stride 2 on 27 x 112 x 140 18.8 : 20.1, 32 -> 128 on
//     8 x 224 x 262 23.7 : 22.6), at 17 .. 29 0.92 .. 1.11 (32 -> 192 on 31 x 112 x 106 27.2 : 24.5);
//   * 1x1 layers in whole K steps: 3, one step 4.5, or 24 into more channels than conv_flow_kernel takes.  1024 -> 512 on 7 x 28 x 29 at 2.8 11.6 : 12.4, 256 ->
//     255 on 9 x 40 x 40 at 3.5 7.5 : 7.7, 384 -> 384 on 61 x 16 x 18 at 6.4 12.8 : 12.5; 64 -> 128 on 10 x 56 x 56 at 3.8 5.5 : 6.4, 64 -> 456 with residual on 2
//     x 63 x 93 at 5.7 7.0 : 11.4.  With channel tiles less than three quarters full 1.75: half of what the second tile does is then padding (256 -> 72 on 9 x 41 x
//     39 at 1.76 4.8 : 5.3);
//   * 1x1 layers that end inside a step: 2.75 up to eight steps (32 -> 256 on 80 x 81 at 1.6 4.6 : 9.3, 24 -> 256 on 142 x 8 x 10 at 2.8 5.6 : 8.1), 1.25 with
//     more, whose every step has the taps to work out; in place up to three steps 4.5, as far as the line of the streaming kernel there (this kernel : it :
//     conv_flow_kernel, 16 -> 128 on 160 x 146 at 2.9 6.1 : 7.1 : 7.4, 96 -> 96 on 16 x 52 x 32 at 3.3 6.6 : 8.5 : 8.4, 120 -> 320 on 4 x 60 x 52 at 3.8 8.2 : 10.5
//     : 9.0, 184 -> 128 on 42 x 28 x 29 at 4.2 10.0 : 12.2 : 11.2, 48 -> 184 with residual on 2 x 97 x 125 at 4.4 8.6 : 9.5 : 10.3; the other way round 16 -> 128
//     on 148 x 14 x 16 at 4.1 7.8 : 7.4 : 9.1);
//   * up to 32 output channels 3: 256 -> 32 on 38 x 28 x 28 at 1.8 3.9 : 6.8, 320 -> 32 on 4 x 112 x 113 at 3.1 6.4 : 9.5; 1x1 layers of one K step as far as the
//     line of launch_conv1x1_stream, which has the times on both sides.
inline double small_limit(const ConvArgs& a, bool place) {
  const int nk = (a.K + 63) / 64;
  if (a.Cout <= 32) return a.Cin == 64 && nk == 1 && a.stride_h == 1 && !a.pad_h ? (place ? 24.0 : 4.5) : 3.0;
  if (a.kh > 1 || a.kw > 1 || a.stride_h > 1 || a.pad_h) return place && a.Cin % 64 && nk <= 5 ? 16.0 : a.Cout <= 64 || a.Cin % 64 ? 1.96 : 2.75;
  if (a.Cin % 64) return place && nk <= 3 ? 4.5 : nk <= 8 ? 2.75 : 1.25;
  if (nk == 1) return a.Cout > 256 ? 24.0 : 4.5;
  return a.Cout * 4 < (a.Cout + 63) / 64 * 64 * 3 ? 1.75 : 3.0;
}
inline bool small_takes(const ConvArgs& a, long long M, int num_cu, bool place) {
  return (double)((M + 63) / 64 * ((a.Cout + 63) / 64)) <= small_limit(a, place) * num_cu;
}
// 3x3 layers of stride 1, against conv3x3_mid_kernel, which reads every pixel once for all nine taps: short reductions, up to 1.96 tiles of
// 64 x 64 per compute unit.  64 -> 64 on 5 x 80 x 80 at 1.95 7.0 : 8.2, 64 -> 192 on 136 x 8 x 10 at 2.0 7.3 : 9.3, 128 -> 96 on 2 x 80 x 82 at 1.6 9.4 : 11.5, 128
// -> 256 on 8 x 20 x 22 at 0.9 7.4 : 8.2, on 11 x 28 x 29 at 2.2 13.3 : 13.9; 160 -> 384 on 56 x 57 at 1.2 11.8 : 10.9, 256 -> 128 on 80 x 80 at 0.8 10.6 : 10.1.
// Reductions that end inside a step from 128 channels on: 48 -> 384 on 13 x 20 x 22 at 2.1 8.3 : 10.4, 96 -> 256 on 4 x 40 x 42 at 1.6 9.2 : 9.1.
inline bool small_takes_3x3(const ConvArgs& a, long long M, int num_cu) {
  if (a.kh != 3 || a.kw != 3 || a.stride_h != 1 || a.stride_w != 1 || a.pad_h != 1 || a.pad_w != 1 || a.Cout <= 32) return false;
  const int nk = (a.K + 63) / 64;
  return (a.Cin % 64 ? nk <= 14 && a.Cout >= 128 : nk <= 18) && (double)((M + 63) / 64 * ((a.Cout + 63) / 64)) <= 1.96 * num_cu;
}

hipError_t launch_small_f16(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_small_f32(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_small_bf16(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);

}  // namespace octo
