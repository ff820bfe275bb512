// Convolution for launches of few tiles, for layers in a cascade whose operands come late, and for fp32 of nearly any size: an implicit GEMM written for few
// instructions per wavefront.  small_limit and small_takes_f32 (conv_small_choice.h) have the lines: up to 1.25 .. 24 tiles of 64 x 64 per compute unit in the
// 16-bit types by the form of the layer, whole K steps of a layer of a model by estimated time without a bound; fp32 1x1 layers up to 64, windows in whole K steps
// at every size and with steps across taps up to 8.
//
// A launch of few tiles is one round of workgroups, and its time is what one of them takes from its first instruction to its last store. A
// wavefront alone on its SIMD issues an instruction every four cycles at best, so that time is mostly a count of instructions: of the
// 3.84 us of conv_flow_kernel on 128 -> 128 over 40 x 40 pixels (64 x 64 tile, two K steps, launches back to back from a graph) 1.23 pass
// between launches, 0.46 go to addresses, 0.34 to the first operands, 0.86 to the two K steps and 0.54 to the epilogue.  Here
//   * all arguments come in one trip to memory, in a block of their own; bias and residual are asked for before the operands, so that
//     nothing is waited for after the K loop;
//   * nothing of the next tile: no second set of addresses, no loads that only keep a count.  Workgroups are two to four per compute unit; where there are more
//     tiles than that (fp32, single K steps, layers of a model, a count on the device larger than expected) those of one follow one another, and the others
//     of its compute unit hide the gap;
//   * the fragments of a step are on their way from LDS while the loads of two steps on are issued; one barrier per step;
//   * blocks of 16 x 16, so that small tiles still have four wavefronts and the epilogue few values per lane.
// Same weights, same LDS layout and, in the 16-bit types, the same sums bit for bit as conv_flow_kernel and the general kernel (a block of 16 x 16 x 32
// adds its products in the order of two of 32 x 32 x 16).  Before (the kernel that took the layer) and after, us, bf16, from a graph: 1x1
// 256 -> 256 on 20 x 20 3.8 -> 2.8, on 5 x 40 x 40 5.4 -> 4.7; 512 -> 512 on 5 x 20 x 20 5.3 -> 4.4; 3x3 64 -> 64 on 5 x 80 x 80 8.2 -> 7.0; stride 2:
// 128 -> 256 on 5 x 80 x 80 11.8 -> 9.4, 256 -> 512 on 8 x 40 x 40 17.2 -> 13.0.
// In fp32 the matrix pipe bounds all but the smallest layers (116 of the 153 TFLOP/s that a large product reaches at 128 -> 384, stride 2 on
// 2 x 160 x 161): three or four workgroups per compute unit hide each other's latency; see conv_small_choice.h for before and after.
// What bounds it in the 16-bit types: between launches 1.2 us; then latency, and from about 20 K steps on what LDS reads take (8 KB per 32 x 32 block and step).
// Measured and left out: rings of four to eight stages, two K steps between barriers (both nothing), two or four groups of wavefronts
// that share K (20 x 20 x 256 -> 256 3x3 7.2 -> 6.7, split-K 5.9; short reductions 0.2 .. 0.5 slower), 128 x 128 tiles.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include "conv_small_choice.h"
#include <hip/hip_ext.h>

namespace octo {

// One K step (128 bytes per row) of a 16 x 16 block: lane (r16, q4) supplies vectors q4 and 4 + q4 of its row.  In fp32 the values of a step
// go to C chains of sums that are added at the end: an instruction need not wait for the one before, and a chain is as short as a
// wavefront's part of the reduction in the split-K kernel.
template <typename T, int C>
__device__ __forceinline__ void small_step(const u32x4 (&a)[2], const u32x4 (&b)[2], floatx4 (&c)[C]) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if constexpr (std::is_same<T, _Float16>::value) c[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a[k]), __builtin_bit_cast(half8, b[k]), c[0], 0, 0, 0);
    else if constexpr (std::is_same<T, __bf16>::value) c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[k]), __builtin_bit_cast(bf16x8, b[k]), c[0], 0, 0, 0);
    else {
      const floatx4 fa = __builtin_bit_cast(floatx4, a[k]), fb = __builtin_bit_cast(floatx4, b[k]);
#pragma unroll
      for (int e = 0; e < 4; ++e) c[(4 * k + e) % C] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[e], c[(4 * k + e) % C], 0, 0, 0);
    }
  }
}

// BC x BP: tile; WC, WP: wavefronts along the channels and the pixels; MINB: workgroups per compute unit; MODE: how addresses are made
// (SMALL_POINTWISE and what follows it).
template <typename T, int BC, int BP, int WC, int WP, int MINB, int MODE>
__global__ __launch_bounds__(64 * WC * WP, MINB * WC * WP / 4) void conv_small_kernel(const SmallArgs a) {
  const int block = blockIdx.x;
#include "conv_small_body.h"
}
// Up to three layers that do not depend on one another in one launch: the workgroups of one follow those of the one before (SmallGroup, conv_small_choice.h).  A launch of few
// tiles leaves compute units idle and costs 3.5 us whatever it does.  Cascades with separate launches and with a shortcut and the layer beside it, and the heads, as one, us: sweep of 1
// frame 484 -> 475, of 4 605 -> 592, traffic of 8 1050 -> 1024, surveillance of 4 953 -> 944, sweep of 64 3825 -> 3809.
struct SmallGroupArgs { SmallArgs layer[SmallGroup::MAX]; int second, third; };      // their first workgroups, multiples of 8
template <typename T, int BC, int BP, int WC, int WP, int MINB, int MODE>
__global__ __launch_bounds__(64 * WC * WP, MINB * WC * WP / 4) void conv_small_group_kernel(const SmallGroupArgs g) {
  const int b = blockIdx.x, which = b < g.second ? 0 : b < g.third ? 1 : 2, block = b - (which == 0 ? 0 : which == 1 ? g.second : g.third);
  // straight from the arguments' memory: a copy that is indexed would live in scratch
  const SmallArgs a = *(const SmallArgs*)((const char*)__builtin_amdgcn_kernarg_segment_ptr() + which * sizeof(SmallArgs));
#include "conv_small_body.h"
}

template <typename T, int BC, int BP, int WC, int WP, int MINB>
static hipError_t launch_small_cfg(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  constexpr int ES = (int)sizeof(T), BK = 128 / ES, NT = 64 * WC * WP;
  const long long M = (long long)a.n * a.Ho * a.Wo, tiles_c = (a.Cout + BC - 1) / BC, tiles_p = (M + BP - 1) / BP, tiles = tiles_p * tiles_c;
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x3FFFFFF0LL) return hipErrorNotSupported;
  long long grid = (tiles + 7) / 8 * 8;
  const long long cap = ((long long)num_cu * MINB + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  SmallArgs o{};
  o.x = (const char*)a.x + (long long)ES * a.x_coff; o.w = (const char*)a.w; o.bias = a.bias; o.y = (char*)a.y + (long long)ES * a.y_coff; o.n_dyn = a.n_dyn;
  if (a.res && a.res_mode != OCTO_RES_NONE) o.res = (const char*)a.res + (long long)ES * a.res_coff;
  if (a.split > 0) o.y2 = (char*)a.y2 + (long long)ES * (a.y2_coff - a.split);
  o.n = a.n; o.HoWo = a.Ho * a.Wo; o.tiles_c = (int)tiles_c; o.per_row = a.Kp * ES; o.grid = (int)grid;
  o.div_tc = make_fastdiv((unsigned)tiles_c); o.div_tp = make_fastdiv((unsigned)tiles_p);
  o.div_howo = make_fastdiv((unsigned)(a.Ho * a.Wo)); o.div_wo = make_fastdiv((unsigned)a.Wo);
  o.x_pitch = a.x_ld * ES; o.y_pitch = a.y_ld * ES; o.y2_pitch = a.y2_ld * ES; o.res_pitch = a.res_ld * ES;
  o.Cout = a.Cout; o.split = a.split; o.nk = (a.K + BK - 1) / BK; o.taps_nk = a.Cin / BK;
  o.H = a.H; o.W = a.W; o.Wo = a.Wo; o.kw = a.kw; o.kh = a.kh; o.stride = a.stride_h; o.pad = a.pad_h; o.Cin = a.Cin; o.K = a.K;
  o.magic_cin = a.magic_cin; o.magic_kw = a.magic_kw;
  // where the weights are the larger operand, a die keeps to its channels and all dies read the pixels; see conv_ksplit.h
  o.c_outer = (double)a.Cout * a.Kp > (double)(a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * a.H * a.W * a.Cin;
  o.act = a.act; o.res_mode = a.res_mode; o.w_len = a.w_rows * a.Kp * ES; o.w_rows = a.w_rows;
  const bool window = a.kh > 1 || a.kw > 1 || a.pad_h, part = ES == 4 && a.Cin % BK && !window;
  const int mode = part ? (a.stride_h > 1 ? SMALL_STRIDED_PART : SMALL_PART) : a.Cin % BK ? SMALL_ANY : (window || a.stride_h > 1 ? SMALL_TAPS : SMALL_POINTWISE);
  if (kernel_id) *kernel_id = small_kernel_id(BC, BP, WC, mode);
  if (a.group && a.group->count < SmallGroup::MAX) {       // launched with the others of its group
    SmallGroup& g = *a.group;
    if (g.count == 0) g.timing = tm;
    g.tile[g.count] = which; g.mode[g.count] = mode; g.kernel_id[g.count] = kernel_id; g.layer[g.count++] = o;
    return hipSuccess;
  }
  auto go = [&](auto mode_c) {
    constexpr int MODE = decltype(mode_c)::value;
    if (tm.start && tm.stop) hipExtLaunchKernelGGL((conv_small_kernel<T, BC, BP, WC, WP, MINB, MODE>), dim3((unsigned)grid), dim3(NT), 0, s, tm.start, tm.stop, 0, o);
    else hipLaunchKernelGGL((conv_small_kernel<T, BC, BP, WC, WP, MINB, MODE>), dim3((unsigned)grid), dim3(NT), 0, s, o);
    return hipGetLastError();
  };
  if constexpr (ES == 4) {
    if (part) return a.stride_h > 1 ? go(std::integral_constant<int, SMALL_STRIDED_PART>{}) : go(std::integral_constant<int, SMALL_PART>{});
  }
  return mode == SMALL_ANY ? go(std::integral_constant<int, SMALL_ANY>{})
                           : mode == SMALL_TAPS ? go(std::integral_constant<int, SMALL_TAPS>{}) : go(std::integral_constant<int, SMALL_POINTWISE>{});
}

// One entry point per storage type; `which` counts the rows of SMALL_COST (SMALL_COST_F32).
template <typename T>
static hipError_t launch_small(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (a.group && a.group->count > 0) which = a.group->tile[0];
  switch (which) {
    case 0: return launch_small_cfg<T, 32, 32, 2, 2, 4>(which, a, num_cu, s, kernel_id, tm);
    case 1: return launch_small_cfg<T, 32, 64, 1, 4, 4>(which, a, num_cu, s, kernel_id, tm);
    case 2: return launch_small_cfg<T, 64, 32, 2, 2, 4>(which, a, num_cu, s, kernel_id, tm);
    case 3: return launch_small_cfg<T, 64, 64, 2, 2, 3>(which, a, num_cu, s, kernel_id, tm);
    case 4: if constexpr (sizeof(T) == 2) return launch_small_cfg<T, 128, 64, 4, 2, 2>(which, a, num_cu, s, kernel_id, tm);
  }
  return hipErrorNotSupported;
}

// Launches what a group has collected.
template <typename T, int BC, int BP, int WC, int WP, int MINB>
static hipError_t launch_small_group_cfg(const SmallGroup& g, hipStream_t s) {
  auto go = [&](auto mode_c) {
    constexpr int MODE = decltype(mode_c)::value, NT = 64 * WC * WP;
    auto start = [&](auto kernel, int grid, const auto& args) {
      if (g.timing.start && g.timing.stop) hipExtLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NT), 0, s, g.timing.start, g.timing.stop, 0, args);
      else hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NT), 0, s, args);
      return hipGetLastError();
    };
    if (g.count == 1) return start(conv_small_kernel<T, BC, BP, WC, WP, MINB, MODE>, g.layer[0].grid, g.layer[0]);
    for (int i = 0; i < g.count; ++i)
      if (g.kernel_id[i]) *g.kernel_id[i] = i ? KID_NONE : group_kernel_id(BC, BP, g.count, MODE);
    SmallGroupArgs a{};
    for (int i = 0; i < g.count; ++i) a.layer[i] = g.layer[i];
    a.second = g.layer[0].grid;
    a.third = a.second + g.layer[1].grid;
    return start(conv_small_group_kernel<T, BC, BP, WC, WP, MINB, MODE>, a.third + (g.count > 2 ? g.layer[2].grid : 0), a);
  };
  return g.mode[0] == SMALL_TAPS ? go(std::integral_constant<int, SMALL_TAPS>{}) : go(std::integral_constant<int, SMALL_POINTWISE>{});
}
template <typename T>
static hipError_t launch_small_group_t(const SmallGroup& g, hipStream_t s) {
  for (int i = 1; i < g.count; ++i) if (g.mode[i] != g.mode[0] || g.tile[i] != g.tile[0]) return hipErrorInvalidValue;
  if (g.count < 1 || (g.mode[0] != SMALL_TAPS && g.mode[0] != SMALL_POINTWISE)) return hipErrorInvalidValue;
  switch (g.tile[0]) {
    case 0: return launch_small_group_cfg<T, 32, 32, 2, 2, 4>(g, s);
    case 1: return launch_small_group_cfg<T, 32, 64, 1, 4, 4>(g, s);
    case 2: return launch_small_group_cfg<T, 64, 32, 2, 2, 4>(g, s);
    case 3: return launch_small_group_cfg<T, 64, 64, 2, 2, 3>(g, s);
    case 4: return launch_small_group_cfg<T, 128, 64, 4, 2, 2>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace octo
