// Convolution for launches that are too small to fill the chip with large tiles: an implicit GEMM in which every
// wavefront works on its own.
//
// What bounds a small layer is not arithmetic or bandwidth but the chain of dependent trips to memory: the general
// kernel (conv.hip) has one K step in flight and a workgroup barrier per step, so a step takes 0.2 - 0.6 us whatever the
// tile, and a 128 x 128 tile leaves most compute units without work.  Here
//   * a wavefront owns a block of 32 TC channels x 32 TP pixels and a private LDS buffer of one K step (128 bytes per
//     row), which it fills itself with direct-to-LDS loads; it waits only for its own loads and there is no barrier in
//     the loop.  The fragments of a step go to registers first, so that the next step's loads run beside its MFMAs;
//   * the NW wavefronts of a workgroup split K: wavefront group k (of KS) takes steps k, k + KS, ... of the reduction, so
//     that the loads of KS steps are in flight together and a long reduction is a KS-th as long; NW / KS wavefronts take
//     different pixels.  The KS partial sums meet in LDS, where the epilogue (bias, residual, activation) adds them and
//     writes 16 bytes of consecutive channels per lane.
// Rings of two to four steps per wavefront were measured too: more, smaller workgroups per compute unit hide the
// latency better.  Same arguments, weight layout, swizzle and tile order as the general kernel; only the order of the
// sums differs.  Measured back to back against the general kernel (bf16): 20 x 20 x 256 -> 256 3x3, one image, 16.4 ->
// 6.5 us; 7 x 7 x 512 -> 512 3x3, 63 items, 53 -> 25 us; 40 x 40 x 128 -> 128 3x3, 8 images, 20.5 -> 11.5 us; 1x1 layers
// of 20 x 20 maps 5.5 - 7 -> 4.3 - 4.7 us, where an empty kernel takes about 3.5.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include <hip/hip_ext.h>

namespace octo {

// LDS of one wavefront: the operands of a K step, later its partial tile
constexpr int ksplit_region(int tc, int tp) {
  const int step = 32 * (tc + tp) * 128, part = 32 * tp * (32 * tc + 4) * 4;
  return ((step > part ? step : part) + 1023) / 1024 * 1024;
}

template <typename T, int TC, int TP, int NW, int KS>
__global__ __launch_bounds__(64 * NW) void conv_ksplit_kernel(const ConvKernelArgs a, const int c_outer) {
  using E = Elem<T>;
  constexpr int VN = E::N, ES = (int)sizeof(T);
  constexpr int KV = 8, BK = KV * VN;                    // a K step: eight 16-byte vectors per row
  constexpr int BC = 32 * TC, WBP = 32 * TP;             // block of a wavefront
  constexpr int PG = NW / KS, BP = WBP * PG;             // pixel groups; pixels of a workgroup's tile
  constexpr int LA = BC / 8, LB = WBP / 8;               // loads per wavefront and step (8 rows each)
  constexpr int RPITCH = BC + 4;                         // floats per pixel of a partial tile
  constexpr int REGION = ksplit_region(TC, TP);
  static_assert(NW % KS == 0, "whole pixel groups");
  extern __shared__ __attribute__((aligned(1024))) unsigned char dyn_lds[];

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // uniform: the step counts below are scalar
  const int ks = wave % KS, pg = wave / KS;
  unsigned char* mine = dyn_lds + wave * REGION;
  const unsigned lds_mine = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)mine);

  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int HoWo = a.Ho * a.Wo;
  const int M = n_items * HoWo;                          // < 2^31 (host)
  const int tiles_c = (a.Cout + BC - 1) / BC;
  const int tiles_p = (M + BP - 1) / BP;
  const int n_tiles = tiles_p * tiles_c;
  const int nk = a.Kp / BK;                              // the host pads Kp to whole steps
  const int n_mine = (nk - ks + KS - 1) / KS;            // steps of this wavefront
  const T* __restrict__ xg = (const T*)a.x + a.x_coff;
  const long long img_elems = (long long)a.H * a.W * a.x_ld;

  const int ld_row = lane >> 3;                          // row of a pass of 8 rows this lane fills
  // row r keeps vector v in slot v ^ ((r / 2) % 8); rows r and r + 8 i differ in that term by 4 i % 8
  const int rsw = (l32 >> 1) & 7;
  const long long w_bytes = (long long)a.w_rows * a.Kp * ES;
  const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)(w_bytes < BUF_MAX ? w_bytes : BUF_MAX), BUF_FLAGS);
  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;

  const int per_die = (n_tiles + 7) >> 3;                // contiguous chunk of the tile list per die (see conv.hip)
  for (int t = blockIdx.x; t < per_die * 8; t += gridDim.x) {
    const int tile = (t & 7) * per_die + (t >> 3);
    if (tile >= n_tiles) continue;
    int tc, tp;
    if (c_outer) { tc = tile / tiles_p; tp = tile - tc * tiles_p; }
    else { tp = tile / tiles_c; tc = tile - tp * tiles_c; }
    const int c0 = tc * BC, p0 = tp * BP, pw0 = p0 + pg * WBP;

    // the lane's logical vector in even and odd passes (the swizzle alternates between the two)
    const int v0 = (lane & 7) ^ (ld_row >> 1), v1 = v0 ^ 4;
    int woff[2];
    woff[0] = ((c0 + ld_row) * a.Kp + v0 * VN) * ES;
    woff[1] = ((c0 + ld_row + 8) * a.Kp + v1 * VN) * ES;

    const int img0 = a.HoWo_is_one ? pw0 : (int)udiv((unsigned)(pw0 < M ? pw0 : 0), a.magic_howo, a.shift_howo);
    const long long rem_bytes = ((long long)(a.n - img0) * img_elems - a.x_coff) * ES;
    const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)(xg + (long long)img0 * img_elems), 0,
        (int)(rem_bytes < 0 ? 0 : (rem_bytes < BUF_MAX ? rem_bytes : BUF_MAX)), BUF_FLAGS);
    int rowoff[LB];
    unsigned hw_ok[LB];

    auto load_w = [&](int kb) {
      const int koff = kb * (BK * ES);
#pragma unroll
      for (int i = 0; i < LA; ++i)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds_mine + i * 1024), "v"(woff[i & 1]), "s"(rsrc_w), "s"(koff + (i >> 1) * 16 * a.Kp * ES) : "memory");
    };
    auto load_x = [&](int kb) {
      int delta[2]; unsigned need[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const unsigned k = (unsigned)kb * BK + (h ? v1 : v0) * VN;
        const unsigned tap = __umulhi(k, a.magic_cin);
        const int c = (int)(k - tap * a.Cin);
        const int r = a.kw == 1 ? (int)tap : (int)__umulhi(tap, a.magic_kw);
        const int s2 = (int)tap - r * a.kw;
        delta[h] = ((r * a.W + s2) * a.x_ld + c) * ES;
        need[h] = k < (unsigned)a.K ? ((1u << r) | (0x10000u << s2)) : 0xFFFFFFFFu;
      }
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int off = (hw_ok[i] & need[i & 1]) == need[i & 1] ? rowoff[i] + delta[i & 1] : OOB;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(lds_mine + BC * 128 + i * 1024), "v"(off), "s"(rsrc_x) : "memory");
      }
    };
    // the weights of the first step need no pixel arithmetic: they are on their way while it is done
    if (n_mine > 0) load_w(ks);
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int m = pw0 + ld_row + 8 * i;
      rowoff[i] = 0; hw_ok[i] = 0u;
      if (m < M) {
        const unsigned mu = (unsigned)m;
        const unsigned img = a.HoWo_is_one ? mu : udiv(mu, a.magic_howo, a.shift_howo);
        const unsigned rem = mu - img * (unsigned)HoWo;
        const unsigned ho = a.Wo == 1 ? rem : udiv(rem, a.magic_wo, a.shift_wo);
        const unsigned wo = rem - ho * (unsigned)a.Wo;
        const int h0 = (int)ho * a.stride_h - a.pad_h, w0 = (int)wo * a.stride_w - a.pad_w;
        rowoff[i] = (int)((((long long)((int)img - img0) * a.H + h0) * a.W + w0) * a.x_ld) * ES;
        const int rlo = h0 < 0 ? -h0 : 0, rhi = a.H - h0 < a.kh ? a.H - h0 : a.kh;
        const int slo = w0 < 0 ? -w0 : 0, shi = a.W - w0 < a.kw ? a.W - w0 : a.kw;
        const unsigned rm = rhi > rlo ? ((1u << rhi) - 1u) & ~((1u << rlo) - 1u) : 0u;
        const unsigned sm = shi > slo ? ((1u << shi) - 1u) & ~((1u << slo) - 1u) : 0u;
        hw_ok[i] = rm | (sm << 16);
      }
    }
    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    if (n_mine > 0) load_x(ks);
    const u32x4* pa = (const u32x4*)mine;
    const u32x4* pb = (const u32x4*)(mine + BC * 128);
    for (int s = 0; s < n_mine; ++s) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      // all fragments of the step into registers, then the stage is free for the next step's loads, which run beside the MFMAs
      u32x4 fa[4][TC], fb[4][TP];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int i = 0; i < TC; ++i) fa[kk][i] = pa[(i * 32 + l32) * 8 + ((kk * 2 + g) ^ rsw)];
#pragma unroll
        for (int j = 0; j < TP; ++j) fb[kk][j] = pb[(j * 32 + l32) * 8 + ((kk * 2 + g) ^ rsw)];
      }
      if (s + 1 < n_mine) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        load_w(ks + (s + 1) * KS);
        load_x(ks + (s + 1) * KS);
      }
      if constexpr (ES == 1) {
        // 8-bit operands: one instruction reduces over 64 values, two vectors per lane and operand
#pragma unroll
        for (int kk = 0; kk < 4; kk += 2)
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int j = 0; j < TP; ++j) acc[i][j] = E::mfma2(fa[kk][i], fa[kk + 1][i], fb[kk][j], fb[kk + 1][j], acc[i][j]);
      } else {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int j = 0; j < TP; ++j) acc[i][j] = E::mfma(fa[kk][i], fb[kk][j], acc[i][j]);
      }
    }

    // partial sums -> this wavefront's own part of LDS as [pixel][channel]
    float* red = (float*)mine;
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
      for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(floatx4*)(red + (j * 32 + l32) * RPITCH + i * 32 + q * 8 + g * 4) =
              floatx4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
    __syncthreads();
    // epilogue: VG consecutive channels of one pixel per lane and pass
    constexpr int VG = BC * BP / 8 >= 64 * NW ? 8 : 4;
    constexpr int GPP = BC / VG;                         // lanes per pixel
    constexpr int GROUPS = BC * BP / VG, PASSES = (GROUPS + 64 * NW - 1) / (64 * NW);
    const bool second_ok = a.split > 0;
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
      constexpr int RES = decltype(res_c)::value;
      constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        const int gi = ps * 64 * NW + tid;
        const int pl = gi / GPP, cl = (gi % GPP) * VG;
        const int p = p0 + pl, c = c0 + cl;
        if (gi >= GROUPS || p >= M || c >= a.Cout) continue;
        const float* src = (const float*)(dyn_lds + (pl / WBP) * KS * REGION) + (pl % WBP) * RPITCH + cl;
        floatx4 v[VG / 4];
#pragma unroll
        for (int h = 0; h < VG / 4; ++h) {
          v[h] = *(const floatx4*)(src + h * 4);
#pragma unroll
          for (int k = 1; k < KS; ++k) {
            const floatx4 o = *(const floatx4*)(src + k * (REGION / 4) + h * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[h][e] += o[e];
          }
        }
        const bool whole = c + VG <= a.Cout;
        // two layers in one launch: a group of channels never straddles the split (a multiple of 8)
        const bool second = second_ok && c >= a.split;
        const int ld = second ? a.y2_ld : a.y_ld;
        const size_t o = (size_t)p * ld + (second ? a.y2_coff + c - a.split : a.y_coff + c);
        char* yb = (char*)(second ? a.y2 : a.y);
        const bool y_vec = whole && (o & 3) == 0 && ((uintptr_t)yb & 15) == 0;
        const T* rp = RES != OCTO_RES_NONE ? (const T*)a.res + (size_t)p * a.res_ld + a.res_coff + c : nullptr;
        const bool r_vec = whole && (((size_t)p * a.res_ld + a.res_coff + c) & 3) == 0;
#pragma unroll
        for (int h = 0; h < VG / 4; ++h) {
          floatx4 rv = {0.f, 0.f, 0.f, 0.f};
          if (RES != OCTO_RES_NONE) {
            if (r_vec) rv = load4<T>(rp + h * 4);
            else {
#pragma unroll
              for (int e = 0; e < 4; ++e) if (c + h * 4 + e < a.Cout) rv[e] = to_f32<T>(rp[h * 4 + e]);
            }
            if constexpr (ES == 1) {
#pragma unroll
              for (int e = 0; e < 4; ++e) rv[e] *= a.res_scale;
            }
          }
          // bias (and scale) are padded to whole tiles of 128 channels
          const floatx4 b4 = *(const floatx4*)(a.bias + c + h * 4);
          if constexpr (ES == 1) {
            const floatx4 s4 = *(const floatx4*)(a.scale + c + h * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[h][e] *= s4[e];
          }
          v[h] = finish4<RES, SILU>(v[h], b4, rv, act_lo);
          if constexpr (ES == 1) {
            if (!a.out_f32) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[h][e] *= a.y_inv_scale;
            }
          }
        }
        if (a.out_f32) {
#pragma unroll
          for (int h = 0; h < VG / 4; ++h) {
            if (y_vec) *(floatx4*)((float*)yb + o + h * 4) = v[h];
            else {
#pragma unroll
              for (int e = 0; e < 4; ++e) if (c + h * 4 + e < a.Cout) ((float*)yb)[o + h * 4 + e] = v[h][e];
            }
          }
          continue;
        }
        if constexpr (ES == 2 && VG == 8) {
          if (y_vec && (o & 7) == 0) {
            typedef T t8 __attribute__((ext_vector_type(8)));
            const t8 w = {(T)v[0][0], (T)v[0][1], (T)v[0][2], (T)v[0][3], (T)v[1][0], (T)v[1][1], (T)v[1][2], (T)v[1][3]};
            *(u32x4*)((T*)yb + o) = __builtin_bit_cast(u32x4, w);
            if (a.up_y) store_upsampled<T>(a, (unsigned)p, c, __builtin_bit_cast(u32x4, w));
            continue;
          }
        }
        {
#pragma unroll
          for (int h = 0; h < VG / 4; ++h) {
            if (y_vec) {
              store4<T>((T*)yb + o + h * 4, v[h]);
              if constexpr (ES == 2) {
                typedef T t4 __attribute__((ext_vector_type(4)));
                if (a.up_y) store_upsampled<T>(a, (unsigned)p, c + h * 4, __builtin_bit_cast(u32x2, t4{(T)v[h][0], (T)v[h][1], (T)v[h][2], (T)v[h][3]}));
              }
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) if (c + h * 4 + e < a.Cout) ((T*)yb)[o + h * 4 + e] = from_f32<T>(v[h][e]);
            }
          }
        }
      }
    });
    __syncthreads();                     // the partial sums have been read: the buffers may be refilled
  }
}

// ---- which launches take this kernel --------------------------------------------------------------------------------
// Time of a launch in us by a model fitted to 270 layers of the networks at 1 .. 119 items (bf16, f16 and fp32; residual
// error 6 - 8 %): a constant (start, first trip to memory, drain), plus what the busiest compute unit does: per tile the
// bytes of its operands at the rate one unit fetches them from its L2 (130 GB/s = 55 bytes per clock here, half of that in
// the general kernel) and an epilogue, plus a latency per K step.  The smallest estimate wins; over those layers the
// choice is within 1 % of always taking the fastest kernel.  The general kernel's pipelined tiles and its 64 x 256 one have no entry: the
// former are taken before this comparison where they win (general_tile), the latter only for launches far too large to split.
struct ConvCost { int bc, bp, ks; double start, per_100kb, per_tile, per_step; };
inline double conv_cost_us(const ConvCost& c, long long M, int cout, int kp_bytes, int num_cu) {
  const double tiles = (double)((M + c.bp - 1) / c.bp) * ((cout + c.bc - 1) / c.bc);
  double per_cu = tiles / num_cu;
  if (c.ks > 0 && per_cu < 4.0) per_cu = (double)(long long)(per_cu + 0.999999);      // few rounds: the last one counts in full
  if (per_cu < 1.0) per_cu = 1.0;
  const int nk = kp_bytes / 128;
  return c.start + per_cu * (c.per_100kb * (double)(c.bc + c.bp) * kp_bytes * 1e-5 + c.per_tile) + c.per_step * ((nk + c.ks - 1) / (c.ks > 0 ? c.ks : 1));
}
constexpr ConvCost KSPLIT_COST[4] = {{32, 32, 8, 3.0, 0.75, 1.00, 0.07}, {32, 32, 4, 3.0, 0.75, 0.61, 0.11},
                                     {64, 32, 4, 3.4, 0.77, 0.75, 0.085}, {64, 64, 4, 3.5, 0.84, 1.70, 0.10}};
// the general kernel's shapes (ks = 0: no split; K steps are a latency each)
constexpr ConvCost GENERAL_COST[4] = {{32, 128, 0, 3.9, 0.91, 0.80, 0.36}, {64, 64, 0, 3.7, 0.28, 0.84, 0.28},
                                      {64, 128, 0, 4.0, 1.32, 1.57, 0.12}, {128, 128, 0, 4.5, 1.27, 3.28, 0.19}};

// Index of the split-K shape with the smallest estimate below `best` us, or -1.  M: output pixels expected; shapes: the first so many of
// KSPLIT_COST; most: a shape needs fewer tiles per compute unit than this.
inline int ksplit_best(const ConvArgs& a, long long M, int es, int num_cu, double best, int shapes = 4, double most = 1e30) {
  int pick = -1;
  for (int i = 0; i < shapes; ++i) {
    const ConvCost& c = KSPLIT_COST[i];
    if ((double)((M + c.bp - 1) / c.bp) * ((a.Cout + c.bc - 1) / c.bc) >= most * num_cu) continue;
    const double t = conv_cost_us(KSPLIT_COST[i], M, a.Cout, a.Kp * es, num_cu);
    if (t < best) { best = t; pick = i; }
  }
  return pick;
}
// The one that beats the general kernel's bc x bp tile, or -1.
inline int ksplit_choose(const ConvArgs& a, long long M, int es, int bc, int bp, int num_cu) {
  double best = -1.0;
  for (const ConvCost& g : GENERAL_COST) if (g.bc == bc && g.bp == bp) best = 0.97 * conv_cost_us(g, M, a.Cout, a.Kp * es, num_cu);
  return ksplit_best(a, M, es, num_cu, best);
}

template <typename T, int TC, int TP, int NW, int KS>
static hipError_t launch_ksplit_cfg(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  constexpr int BC = 32 * TC, BP = 32 * TP * (NW / KS);
  constexpr unsigned lds = (unsigned)(NW * ksplit_region(TC, TP));
  static_assert(lds <= 80 * 1024, "two workgroups per compute unit");
  static const bool ready = [] {           // more than 64 KB of dynamic LDS needs the attribute, once per instance
    (void)hipFuncSetAttribute((const void*)conv_ksplit_kernel<T, TC, TP, NW, KS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
    return true;
  }();
  (void)ready;
  if (kernel_id) *kernel_id = ksplit_kernel_id(BC, BP, KS);
  const long long M = (long long)a.n * a.Ho * a.Wo;
  const long long tiles = ((M + BP - 1) / BP) * ((a.Cout + BC - 1) / BC);
  if (tiles <= 0) return hipSuccess;
  long long grid = (tiles + 7) / 8 * 8;
  const long long cap = ((long long)num_cu * (160 * 1024 / lds) + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  // Each die takes a contiguous piece of the tile list and has an L2 of its own.  Where the weights are the larger
  // operand, a die keeps to its channels and all dies read the pixels; otherwise the other way round.
  const int c_outer = (double)a.Cout * a.Kp > (double)(a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * a.H * a.W * a.Cin;
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv_ksplit_kernel<T, TC, TP, NW, KS>), dim3((unsigned)grid), dim3(64 * NW), lds, s, tm.start, tm.stop, 0, a, c_outer);
  else
    hipLaunchKernelGGL((conv_ksplit_kernel<T, TC, TP, NW, KS>), dim3((unsigned)grid), dim3(64 * NW), lds, s, a, c_outer);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_ksplit(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  switch (which) {
    case 0: return launch_ksplit_cfg<T, 1, 1, 8, 8>(a, num_cu, s, kernel_id, tm);
    case 1: return launch_ksplit_cfg<T, 1, 1, 4, 4>(a, num_cu, s, kernel_id, tm);
    case 2: return launch_ksplit_cfg<T, 2, 1, 4, 4>(a, num_cu, s, kernel_id, tm);
    default: return launch_ksplit_cfg<T, 2, 2, 4, 4>(a, num_cu, s, kernel_id, tm);
  }
}

}  // namespace octo
