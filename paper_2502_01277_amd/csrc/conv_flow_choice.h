// Which layers take conv_flow_kernel (conv_flow.h), and with which tile.  Host arithmetic only.
#pragma once
#include "octo_internal.h"
#include <algorithm>

namespace octo {

// Does a layer of values of ES bytes (16-bit types, E4M3) have the form that conv_flow_kernel takes?
inline bool flow_fits(const ConvArgs& a, int ES = 2) {
  const int VN = 16 / ES;
  if (a.out_f32 || a.pair_view || a.pool_y || a.up_y || a.kh > 15 || a.kw > 15) return false;
  const int VO = ES == 1 ? 8 : VN;                         // results and residual: E4M3 in halves of a vector
  if ((a.Cout % VO && (a.res || a.split > 0 || ES == 1)) || a.Cout < 16) return false;
  if (ES == 1 && (a.split > 0 || !a.scale)) return false;
  if (((a.Cin | a.x_ld | a.x_coff) % VN) || ((uintptr_t)a.x & 15) || ((a.y_ld | a.y_coff) % VO) || ((uintptr_t)a.y & (VO * ES - 1))) return false;
  if (a.res && (((a.res_ld | a.res_coff) % VO) || ((uintptr_t)a.res & (VO * ES - 1)))) return false;
  if (a.split > 0 && a.split % 32) return false;
  if (ES == 2 && (a.Cout <= 32 || (a.K <= 64 && a.Cout > 256))) return false;      // nothing to fill a tile with; one K step: conv1x1_stream_kernel's
  // 32-bit offsets: weights, and the pixels of a tile (256 of them) in every tensor
  const long long ld = std::max(std::max(a.x_ld, a.y_ld), std::max(a.res ? a.res_ld : 0, a.split > 0 ? a.y2_ld : 0));
  return (long long)a.w_rows * a.Kp * ES < 0x7FFFFFFFLL && 256 * ld * ES < 0x7FFFFFF0LL && (long long)a.n * a.Ho * a.Wo < 0x7FFFFF00LL &&
         (2LL * a.H * a.W + 1024LL * a.stride_h * a.stride_w + (long long)a.pad_h * a.W + a.pad_w) * a.x_ld * ES < 0x7FFFFFF0LL;
}

// Is a layer's tile chosen by tile_cost_us?
inline bool by_place(const ConvArgs& a) { return a.in_place && a.Cin % 64 == 0; }
// What the estimates of all tiles of a layer have in common: output pixels, K steps (128 bytes), megabytes.  Of the 2.6 us in which a launch is enqueued the choice
// of its kernel is 0.37; with everything worked out anew for every tile and estimates asked twice it was 0.49.  The tables are walked unrolled: divisors are constants.
struct LayerWork {
  unsigned M, Cout;
  int num_cu;
  double nk, mb;
  LayerWork(const ConvArgs& a, long long M_, int num_cu_, int ES) : M((unsigned)M_), Cout((unsigned)a.Cout), num_cu(num_cu_), nk((double)((a.K * ES + 127) / 128)) {
    const double pixels_in = (double)M_ * (a.kh >= a.stride_h ? a.stride_h : 1) * (a.kw >= a.stride_w ? a.stride_w : 1);
    mb = 1e-6 * ES * (pixels_in * a.Cin + (double)M_ * a.Cout * (a.res ? 2 : 1));
  }
  template <typename Cost> long long tiles(const Cost& c) const { return (long long)((M + (unsigned)c.bp - 1) / (unsigned)c.bp) * ((Cout + (unsigned)c.bc - 1) / (unsigned)c.bc); }
  double rounds(long long t) const { return (double)((t + num_cu - 1) / num_cu); }      // tiles of the busiest compute unit
};
// Time of a launch in us in its place in a cascade, 16-bit types, input channels in whole K steps: a constant, what a compute unit does - its tiles, a
// quarter of the way from the next whole number to their mean, times K steps and an epilogue -, a latency per K step where no unit has a second
// tile, the memory traffic, and the operands that the tiles fetch.
//   There a layer's input was written by the kernel before and comes from beyond the L2s.  Estimates from the same launch repeated on the same tensors (below)
// are low there and favour large tiles: 128 -> 128 on 8 x 80 x 80, us, in place: 128 x 256 tiles of conv_flow_kernel 11.6, 128 x 128 12, 64 x 64 of
// conv_small_kernel 9.3, where three workgroups per unit hide what one of eight wavefronts waits for; 256 -> 64 on that map 14.5 : 10.8, 256 -> 1024 with
// residual on 96 x 16 x 16 29.0 (256 x 128) : 23.6 (128 x 64).
//   Fitted, without negative terms, to 1933 layers timed in every tile: behind the launch that writes their input and 48 MB of other traffic the 696 1x1 and
// strided layers of four cascades (1 .. 64 frames), 850 random ones (64 .. 4096 channels, 0.05 .. 200 tiles of 64 x 64 per compute unit) and 266 3x3 layers of few
// tiles, in the cascades themselves 121 pairs of layers in one launch; then moved to where the choice loses least.  Of the best tile's time the choice takes
// 1.012 over the cascades' layers, 1.014 over the random ones and, among this kernel's tiles, 1.010 over the pairs; over 718 layers and pairs then timed in every
// tile in the cascades 1.015.  The constants before came from cascades alone, 1.018, 1.025, 1.026 and 1.020 here; a tile had no cost per K step and others
// a negative latency, and reductions that no cascade has lost up to 1.57: 1536 -> 1536 on 56 x 54 26.6 : 21.8, 3072 -> 512 on 11 x 28 x 28 44.8 : 37.2,
// 4096 -> 2048 on 56 x 41 50.6 : 45.3.  (64 -> 128, stride 2 on 480 x 28 x 28, near the line between the two kernels, stays on this one, 25.5 : 24.0.)
struct TileCost { int bc, bp; double base, step, tile, latency, per_mb, per_operand_mb; };
inline double tile_cost_us(const TileCost& c, const LayerWork& w) {
  const long long tiles = w.tiles(c);
  const double per_cu = std::max(1.0, 0.25 * tiles / w.num_cu + 0.75 * w.rounds(tiles)), operands = 128e-6 * tiles * w.nk * (c.bc + c.bp);
  return c.base + per_cu * (w.nk * c.step + c.tile) + (tiles <= w.num_cu ? c.latency * w.nk : 0.0) + c.per_mb * w.mb + c.per_operand_mb * operands;
}
constexpr TileCost FLOW_COST[8] = {
    {64, 64, 3.626, 0.1860, 0.372, 0.1121, 0.0276, 0.0085},
    {64, 128, 5.853, 0.2244, 0.596, 0.0847, 0.0394, 0.0097},
    {128, 64, 5.244, 0.2481, 0.996, 0.0972, 0.0000, 0.0067},
    {128, 128, 6.590, 0.3440, 1.734, 0.0000, 0.0347, 0.0019},
    {96, 256, 4.925, 0.5788, 3.260, 0.0000, 0.0185, 0.0000},
    {192, 128, 5.744, 0.4526, 2.878, 0.0000, 0.0046, 0.0059},
    {128, 256, 9.813, 0.5896, 2.726, 0.0000, 0.0239, 0.0011},
    {256, 128, 7.035, 0.6007, 3.308, 0.0000, 0.0012, 0.0000}};
// Single layers, E4M3, and layers whose channels end inside a K step, of which the cascades have too few to fit: from repeated launches of 656 layers
// (1x1 and 3x3 / stride 2, 24 .. 1536 input and 64 .. 1024 output channels, 0.3 .. 24 tiles of 64 x 128 per compute unit, bf16).  A constant, what
// the busiest compute unit does - its tiles, rounded up, times K steps and an epilogue -, a latency per K step where it has one tile only, and the
// memory traffic (residual error 8 - 11 %; the choice loses 1.3 % against always taking the fastest tile).  E4M3 uses the same numbers with steps of
// 128 values: over 64 such layers (32 .. 1024 input, 80 .. 768 output channels) the choice loses 0.9 % against the fastest tile, at most 13 % (512 -> 608 on 36 x
// 40 x 41: 256 x 128 tiles 32.4 us, 128 x 256 28.5).
struct FlowCost { int bc, bp; double base, step, tile, latency, per_mb, any_step; };
constexpr FlowCost FLOW_COST_REPEATED[8] = {
    {64, 64, 3.73, 0.165, 0.22, 0.118, 0.040, 0.031},
    {64, 128, 3.60, 0.258, 0.42, 0.091, 0.052, 0.065},
    {128, 64, 3.65, 0.255, 0.52, 0.092, 0.035, 0.028},
    {128, 128, 3.08, 0.442, 1.27, 0.000, 0.042, 0.076},
    {96, 256, 2.93, 0.580, 1.59, 0.000, 0.064, 0.145},
    {192, 128, 3.22, 0.554, 1.46, 0.000, 0.045, 0.064},
    {128, 256, 3.00, 0.674, 2.06, 0.000, 0.065, 0.093},
    {256, 128, 3.76, 0.653, 1.18, 0.000, 0.061, 0.053}};
inline double flow_cost_us(const FlowCost& c, const LayerWork& w, bool any) {
  const double per_cu = w.rounds(w.tiles(c));
  return c.base + per_cu * (w.nk * (c.step + (any ? c.any_step : 0.0)) + c.tile) + (per_cu <= 1.0 ? c.latency * w.nk : 0.0) + c.per_mb * w.mb;
}
// The tile (launch_flow's number) with the smallest estimate for M output pixels, in place or repeated.
inline int flow_choose(const ConvArgs& a, long long M, int num_cu, int ES, bool place, double* us) {
  const LayerWork w(a, M, num_cu, ES);
  const bool one = ES == 2 && a.K <= 64, any = a.Cin % (128 / ES) != 0;
  int best = -1;
  if (place) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (one && a.Cout > FLOW_COST[i].bc) continue;
      const double t = tile_cost_us(FLOW_COST[i], w);
      if (best < 0 || t < *us) { *us = t; best = i; }
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (one && a.Cout > FLOW_COST_REPEATED[i].bc) continue;
      const double t = flow_cost_us(FLOW_COST_REPEATED[i], w, any);
      if (best < 0 || t < *us) { *us = t; best = i; }
    }
  }
  return best;
}
// Output channels that are no whole vectors (detector heads: 255 in rows of 256) cost a few stores more: 192 -> 255 on 32 x 160 x 160
// 246 us on the general kernel's plain 128x128 tiles, 191 here, 128 -> 255 on 64 x 80 x 80 112 : 82.  A single K step needs its channels in
// one tile (64 -> 128, stride 2 on 4170 x 56 x 56 341 : 316).
// 1x1 / stride-1 layers that the streaming kernel (conv1x1.hip) leaves to this one: whole K steps, two or more.  Streaming : here, us:
// 128 -> 128 on 64 x 80 x 80 44.6 : 39, on 8 x 80 x 80 9.9 : 8.5, 192 -> 192 on 32 x 80 x 80 37.5 : 36.3, on 32 x 160 x 160 151 : 150.  Fewer or
// broken steps are faster there (96 -> 192 on 41 x 40 x 40 11.6 : 14.5).
// With a residual (requested a K step before the results here, a block of pixels ahead there) by the MB of all tensors together, streaming :
// here.  Three steps: while they fit the memory-side cache (192 -> 192 37 16.3 : 10.1, 147 36.8 : 32.1, 295 66.7 : 67.6, 472 104 : 111; 192 -> 96
// 197 41.5 : 35.7, 315 63.6 : 66.6), and with more channel tiles there, each of which reads the pixels, also beyond it (192 -> 256 360 92 : 91,
// 192 -> 512 311 89 : 86, 996 282 : 259; 192 -> 384 492 125 : 130).  Two steps: the same up to 128 output channels (128 -> 128 197 37.9 : 35.8, 315
// 64.8 : 71.4; 128 -> 64 210 36.3 : 32.9, 419 83 : 95), up to 64 MB with more (128 -> 192 33 10.5 : 9.3, 66 16.2 : 16.6, 419 93 : 99; 128 -> 256 41
// 12.2 : 11.8, 82 19.7 : 21.0, 328 78 : 84; 128 -> 384 57 16.4 : 16.1, 115 26.9 : 28.2, 734 169 : 178), and with more than 384 beyond the cache
// (128 -> 512 74 21.0 : 20.9, 147 33.9 : 36.0, 295 83 : 78, 944 263 : 231).  The same lines hold for a channel slice as the destination.
inline bool flow_takes_1x1(const ConvArgs& a, long long M) {
  if (a.Cin < 128 || a.Cin % 64 || !flow_fits(a)) return false;
  if (!a.res) return true;
  const double mb = 2e-6 * M * (a.Cin + 2.0 * a.Cout);
  const bool two = a.Cin == 128;
  return mb < (two && a.Cout > 128 ? 64.0 : 256.0) || (mb >= 256.0 && a.Cout > (two ? 384 : 192));
}

hipError_t launch_flow_f16(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_flow_bf16(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_flow_f8(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);

}  // namespace octo
