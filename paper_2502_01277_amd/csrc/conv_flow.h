// Convolution as an implicit GEMM whose stream of loads runs on across tiles: 1x1 and strided layers of the 16-bit types and E4M3.
//
// The general kernel (conv.hip) starts every tile with addresses and an empty pipeline and ends it with a pass through LDS between
// barriers.  The 1x1 layers of a detector have 3 .. 12 K steps per tile, so most of their time was that.  Here
//   * a load cursor runs NST - 1 .. NST K steps ahead of the matrix instructions, through the workgroup's whole list of tiles: the first
//     operands of a tile arrive while the one before it is multiplied and written out;
//   * where the input channels come in whole K steps a step lies inside one kernel tap, tap and channel offsets are scalars, and a lane
//     works out addresses once per tap - for 1x1 layers without padding never: the buffer then starts at the tile's first pixel and its
//     range cuts off the pixels past the last one;
//   * weight rows are taken in an order that leaves 16 consecutive channels of a pixel in one lane (as in conv3x3_mid_kernel): results
//     leave as 16-byte stores straight from registers, and drain beside the next tile's K loop;
//   * a K step is 128 bytes, a whole cache line of every row.  What paces the large shapes is line look-ups: with steps of 64 bytes, two
//     workgroups of four wavefronts per compute unit, 128 x 256 tiles took 613 us for 128 -> 256, stride 2 on 4170 x 28 x 28; with 128 bytes
//     one workgroup of eight wavefronts fits and takes 538, as 256 x 128 512.
// Before (general kernel) and after, bf16, us: 64 -> 128, stride 2 on 4170 x 56 x 56 787 -> 676; 96 -> 192, stride 2 on 32 x 320 x 320 507 -> 387;
// 48 -> 96, stride 2 on 32 x 640 x 640 696 -> 545; 384 -> 384 on 32 x 80 x 80 124 -> 102 (3.1 TB/s); 384 -> 192 on 32 x 160 x 160 281 -> 213
// (4.4 TB/s); 192 -> 256 on 32 x 160 x 160 235 -> 164; 256 -> 256 on 64 x 40 x 40 36 -> 26; 512 -> 512 on 8 x 20 x 20 7.9 -> 6.5.
// E4M3 (a step is 128 values, two matrix instructions deep; scale and bias per channel arrive together): 96 -> 96 on 32 x 160 x 160 77 -> 50,
// 192 -> 192 149 -> 98 (3.2 TB/s), 48 -> 96, stride 2 on 32 x 640 x 640 435 -> 307, 64 -> 128, stride 2 on 4170 x 56 x 56 513 -> 416.  Its 64 x 64 tiles run
// two workgroups per compute unit: with the scales three are 2 KB more than the LDS.  Its results and residuals come in vectors of 16 and, behind the
// last of those, half a one.
// LDS rows (weights: one output channel, pixels: one output pixel) are KV vectors of 16 bytes, vector v of row r in slot
// v ^ ((r / (16 / KV)) % KV).  vmcnt bookkeeping: every wavefront issues the same number of loads per K step and of stores per tile.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace octo {

struct FlowGeom { FastDiv div_tc, div_howo, div_wo; };     // divisions by channel tiles, Ho * Wo, Wo

// How addresses are made: 1x1, stride 1, no padding, whole K steps of channels; any other layer with whole K steps of channels per
// tap; any layer (a lane works out the tap of its vector at every step).
enum { FLOW_POINTWISE = 0, FLOW_TAPS = 1, FLOW_ANY = 2 };

// Workgroups per compute unit: at most MINB, and what the LDS holds (stages, biases, E4M3 scales).
constexpr int flow_resident(int es, int NT, int BC, int BP, int KV, int NST, int MINB) {
  const int rp = NT / KV, lds = ((BC + rp - 1) / rp * rp + BP) * KV * 16 * NST + 12 * NT * (es == 1 ? 2 : 1), fit = 160 * 1024 / lds;
  return fit < MINB ? fit : MINB;
}

// NT: lanes; BC x BP: tile; WC: wavefronts along the channels (NT / 64 / WC along the pixels); KV: vectors of 16 bytes per LDS row and
// K step; NST: stages of the ring; MINB: workgroups per compute unit, where the LDS holds them.
template <typename T, int NT, int BC, int BP, int WC, int KV, int NST, int MINB, int MODE>
__global__ __launch_bounds__(NT, flow_resident(sizeof(T), NT, BC, BP, KV, NST, MINB) * NT / 256) void conv_flow_kernel(const ConvKernelArgs a, const FlowGeom gm) {
  using E = Elem<T>;
  constexpr int VN = E::N, ES = (int)sizeof(T), BK = KV * VN;
  constexpr bool PW = MODE == FLOW_POINTWISE;
  constexpr int WP = NT / 64 / WC, TC = BC / WC / 32, TP = BP / WP / 32;
  constexpr int RPW = 16 / KV, RP = NT / KV, LA = (BC + RP - 1) / RP, LB = BP / RP, NL = LA + LB;
  constexpr int ROW = KV * 16, A_BYTES = LA * RP * ROW, STAGE = A_BYTES + BP * ROW;
  constexpr int KK = ES == 1 ? KV / 4 : KV / 2, P0 = (NL + KK - 1) / KK;      // groups of MFMAs per K step, loads issued with each group
  constexpr int FV = ES == 1 ? 2 : 1, NB = ES == 1 ? 2 : 1;         // vectors per operand fragment; loads of what the epilogue needs per channel
  constexpr int HV = 16 / VN;                              // vectors of a lane's 16 consecutive output channels of a 32-channel block
  constexpr int PJ = TC * TP * HV <= 8 ? TP : 0;           // pixel blocks whose residual is requested before the K loop ends
  constexpr int NSTO = TC * TP * HV, NRES = TC * PJ * HV;
  static_assert(ES <= 2 && KK >= 2 && KK % 2 == 0 && BP % RP == 0 && TC >= 1 && TP >= 1, "tile shape");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NST * STAGE];
  __shared__ __attribute__((aligned(16))) float sBias[3][NT];               // of this tile and the next; with one channel tile of all, and a dump
  __shared__ __attribute__((aligned(16))) float sScale[3][ES == 1 ? NT : 1];             // the same of E4M3 layers' scales

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WC, wp = wave / WC;
  const int l32 = lane & 31, g = lane >> 5;
  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int HoWo = a.Ho * a.Wo, M = n_items * HoWo;        // < 2^31 (host)
  const int tiles_c = (a.Cout + BC - 1) / BC;
  const int n_tiles = (M + BP - 1) / BP * tiles_c;
  const int nk = (a.K + BK - 1) / BK;                      // the weights are padded with zeros to whole steps
  const T* __restrict__ xg = (const T*)a.x + a.x_coff;
  const long long img_elems = (long long)a.H * a.W * a.x_ld;
  const int w_len = a.w_rows * a.Kp * ES;                  // fits (host)

  const int ld_row = tid / KV;
  const int lkv = (tid % KV) ^ ((ld_row / RPW) % KV);      // logical vector of this lane's slot of a row
  const int rsw = (l32 / RPW) % KV;
  const unsigned lds_ring = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)smem + (unsigned)wave * 1024u));
  const unsigned lds_bias = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)&sBias[0][0] + (unsigned)wave * 256u));
  const unsigned lds_scale = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)&sScale[0][0] + (unsigned)wave * 256u));
  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;

  const int per_die = (n_tiles + 7) >> 3;                  // one contiguous chunk of the tile list per die, as in conv_mfma_kernel
  const int t_end = per_die * 8;
  auto next_valid = [&](int t) -> int {
    while (t < t_end && (t & 7) * per_die + (t >> 3) >= n_tiles) t += gridDim.x;
    return t;
  };
  auto locate = [&](int t, int& p0, int& c0) __attribute__((always_inline)) {
    const unsigned tile = (unsigned)((t & 7) * per_die + (t >> 3)), tp = fast_div(tile, gm.div_tc);
    c0 = (int)(tile - tp * (unsigned)tiles_c) * BC;
    p0 = (int)tp * BP;
  };

  // ---- the load cursor ----
  // LDS row m of a 32-row block holds channel 16 ((m / 4) % 2) + 4 (m / 8) + m % 4 of the block, see the epilogue
  int woff[LA], voff[LB], rowoff[PW ? 1 : LB];
  unsigned hw_ok[PW ? 1 : LB];
  {
    const int m = ld_row & 31, ch = (ld_row & ~31) + 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
#pragma unroll
    for (int i = 0; i < LA; ++i) woff[i] = ld_row + RP * i < BC ? ((ch + RP * i) * a.Kp + lkv * VN) * ES : OOB;
#pragma unroll
    for (int i = 0; i < LB; ++i) voff[i] = ((ld_row + RP * i) * a.x_ld + lkv * VN) * ES;     // PW; set per tap otherwise
  }
  int lt = next_valid(blockIdx.x);
  if (lt >= t_end) return;
  int t = lt, l_kb = 0, l_cs = 0, l_r = 0, l_s = 0, l_w = 0, l_x = 0, l_st = 0;      // tile; K step, channel offset and tap in it; scalar offsets; ring stage
  void* x_base = nullptr;
  int x_len = 0, w_now = w_len;
  auto open_tap = [&]() __attribute__((always_inline)) {
    if constexpr (MODE == FLOW_ANY) {
      // element k of the reduction is channel c of tap (r, s): k = (r * kw + s) * Cin + c, exact for k < 65536
      const unsigned k = (unsigned)l_kb * BK + lkv * VN, tap = a.Cin == 1 ? k : __umulhi(k, a.magic_cin);
      const int r = a.kw == 1 ? (int)tap : (int)__umulhi(tap, a.magic_kw), s = (int)tap - r * a.kw;
      const int delta = ((r * a.W + s) * a.x_ld + (int)(k - tap * a.Cin)) * ES;
      const unsigned need = k < (unsigned)a.K ? (1u << r) | (0x10000u << s) : 0xFFFFFFFFu;
#pragma unroll
      for (int i = 0; i < LB; ++i) voff[i] = (hw_ok[i] & need) == need ? rowoff[i] + delta : OOB;
    } else if constexpr (!PW) {
      const unsigned need = (1u << l_r) | (0x10000u << l_s);
#pragma unroll
      for (int i = 0; i < LB; ++i) voff[i] = (hw_ok[i] & need) == need ? rowoff[i] : OOB;
    }
  };
  auto open_tile = [&]() __attribute__((always_inline)) {
    int p0, c0;
    locate(lt, p0, c0);
    l_kb = 0; l_cs = 0; l_r = 0; l_s = 0; l_x = 0;
    l_w = c0 * a.Kp * ES;
    if constexpr (PW) {
      const long long bytes = ((long long)(M - p0) * a.x_ld - a.x_coff) * ES;
      x_base = (void*)(xg + (long long)p0 * a.x_ld);
      x_len = (int)(bytes < BUF_MAX ? bytes : BUF_MAX);
    } else {
      // a buffer that starts at the first image of the tile, less the padding, so that every pixel's offset is positive
      const unsigned img0 = fast_div((unsigned)p0, gm.div_howo);
      const long long shift = ((long long)a.pad_h * a.W + a.pad_w) * a.x_ld;
      const long long bytes = ((long long)(a.n - (int)img0) * img_elems - a.x_coff + shift) * ES;
      x_base = (void*)(xg + (long long)img0 * img_elems - shift);
      x_len = (int)(bytes < BUF_MAX ? bytes : BUF_MAX);
      int row = ld_row;
      asm volatile("" : "+v"(row));
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int m = p0 + row + RP * i;
        const unsigned img = fast_div((unsigned)m, gm.div_howo), rem = (unsigned)m - img * (unsigned)HoWo;
        const unsigned ho = fast_div(rem, gm.div_wo), wo = rem - ho * (unsigned)a.Wo;
        const int h0 = (int)ho * a.stride_h - a.pad_h, w0 = (int)wo * a.stride_w - a.pad_w;
        // kernel rows r with 0 <= h0 + r < H form the range [max(0, -h0), min(kh, H - h0)); same for columns
        const int rlo = h0 < 0 ? -h0 : 0, rhi = a.H - h0 < a.kh ? a.H - h0 : a.kh;
        const int slo = w0 < 0 ? -w0 : 0, shi = a.W - w0 < a.kw ? a.W - w0 : a.kw;
        const unsigned rm = rhi > rlo ? ((1u << rhi) - 1u) & ~((1u << rlo) - 1u) : 0u;
        const unsigned sm = shi > slo ? ((1u << shi) - 1u) & ~((1u << slo) - 1u) : 0u;
        rowoff[i] = ((((int)(img - img0) * a.H + (int)ho * a.stride_h) * a.W + (int)wo * a.stride_w) * a.x_ld + (MODE == FLOW_TAPS ? lkv * VN : 0)) * ES;
        hw_ok[i] = m < M ? rm | (sm << 16) : 0u;
      }
    }
    open_tap();
  };
  auto advance = [&]() __attribute__((always_inline)) {    // to the next K step, maybe of the next tile
    l_st = l_st + 1 == NST ? 0 : l_st + 1;
    l_kb += 1; l_cs += BK; l_w += BK * ES;
    if constexpr (MODE != FLOW_ANY) l_x += BK * ES;
    if (l_kb == nk) {
      lt = next_valid(lt + gridDim.x);
      if (lt < t_end) { open_tile(); return; }
      x_len = 0; w_now = 0; l_kb = -0x40000000; l_w = 0; l_x = 0;       // past the end: loads of nothing, which keep the count
      l_cs = -0x40000000;
      return;
    }
    if constexpr (MODE == FLOW_ANY) {
      if (l_kb > 0) open_tap();
    } else if constexpr (!PW) {
      if (l_cs == a.Cin) {
        l_cs = 0;
        if (++l_s == a.kw) { l_s = 0; ++l_r; }
        l_x = (l_r * a.W + l_s) * a.x_ld * ES;
        open_tap();
      }
    }
  };
  // loads [from, to) of the cursor's K step
  auto issue = [&](int from, int to) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(x_base, 0, x_len, BUF_FLAGS);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, w_now, BUF_FLAGS);
    const unsigned st = lds_ring + l_st * STAGE;
    // A tap that no pixel of the tile can use (a map no taller than the padding) may start behind the end of the buffer, where every lane is
    // out of range already.  The scalar offset must not be: the range check takes it off the length, which would wrap, and let any lane in.
    const int ox = l_x < x_len ? l_x : 0, ow = w_now ? l_w : 0;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      if (q < from || q >= to) continue;
      if (q < LB)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(st + A_BYTES + q * (NT * 16)), "v"(voff[q < LB ? q : 0]), "s"(rx), "s"(ox) : "memory");
      else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(st + (q - LB) * (NT * 16)), "v"(woff[q >= LB ? q - LB : 0]), "s"(rw), "s"(ow) : "memory");
    }
  };
  auto issue_bias = [&](int c0, int buf, bool any) __attribute__((always_inline)) {       // padded to whole tiles like the weights
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, any ? a.w_rows * 4 : 0, BUF_FLAGS);
    const int off = tid < BC ? (c0 + tid) * 4 : OOB;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_bias + buf * (NT * 4)), "v"(off), "s"(rb) : "memory");
    if constexpr (ES == 1) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.scale, 0, any ? a.w_rows * 4 : 0, BUF_FLAGS);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_scale + buf * (NT * 4)), "v"(off), "s"(rs) : "memory");
    }
  };

  u32x4 fa[2][TC][FV], fb[2][TP][FV];
  const int arow = (wc * (TC * 32) + l32) * ROW, brow = A_BYTES + (wp * (TP * 32) + l32) * ROW;
  auto frags = [&](int set, int st, int kq) __attribute__((always_inline)) {
    const unsigned char* p = smem + st * STAGE;
#pragma unroll
    for (int h = 0; h < FV; ++h) {
      const int v = (((kq * FV + h) * 2 + g) ^ rsw) << 4;
#pragma unroll
      for (int i = 0; i < TC; ++i) fa[set][i][h] = *(const u32x4*)(p + arow + i * (32 * ROW) + v);
#pragma unroll
      for (int j = 0; j < TP; ++j) fb[set][j][h] = *(const u32x4*)(p + brow + j * (32 * ROW) + v);
    }
  };

  int p0, c0;
  locate(t, p0, c0);
  open_tile();
  issue_bias(c0, 0, true);
#pragma unroll
  for (int d = 0; d < NST - 1; ++d) { issue(0, NL); advance(); }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 2) * NL) : "memory");
  __builtin_amdgcn_s_barrier();
  issue(0, P0);
  frags(0, 0, 0);

  const bool has_res = a.res && a.res_mode != OCTO_RES_NONE, tail = a.Cout % VN != 0;
  int st_rd = 0, bbuf = 0;
  auto next_bias = [](int b) { return ES == 1 ? (b == 2 ? 0 : b + 1) : b ^ 1; };      // where the next tile's bias goes, see launch_flow_cfg
  bool stored = false;                                     // the first wait of a tile counts the stores of the one before
  for (;;) {
    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int cw = c0 + wc * (TC * 32) + g * 16;           // this lane's first channel
    u32x4 rv[TP][TC][HV];
    auto load_res = [&](int from, int to) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)((const T*)a.res + a.res_coff + (long long)p0 * a.res_ld), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
      for (int j = 0; j < TP; ++j) {
        if (j < from || j >= to) continue;
        const int pl = wp * (TP * 32) + j * 32 + l32;
        const int off = (pl * a.res_ld + cw) * ES;
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int h = 0; h < HV; ++h) {
            // a half vector (E4M3 only) is asked for with the eight values before it; lanes without a pixel or channel stay out of range
            const int c = cw + i * 32 + h * VN, back = ES == 1 && c + 8 == a.Cout ? 8 : 0;
            rv[j][i][h] = __builtin_amdgcn_raw_buffer_load_b128(rr, p0 + pl < M && c < a.Cout ? off + i * 32 * ES + h * 16 - back : OOB, 0, 0);
          }
      }
    };
    const int tn = next_valid(t + gridDim.x);
    const bool more = tn < t_end;
    int pn0 = 0, cn0 = 0;
    if (more) locate(tn, pn0, cn0);
    auto step = [&](auto lastc, bool first) __attribute__((always_inline)) {
      constexpr bool LAST = decltype(lastc)::value;
      const int nxt = st_rd + 1 == NST ? 0 : st_rd + 1;
      if constexpr (LAST) {
        issue_bias(cn0, tiles_c == 1 ? 2 : next_bias(bbuf), more);
        if (PJ > 0 && has_res) load_res(0, PJ);
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        if (kk < KK - 1) {
          frags((kk + 1) & 1, st_rd, kk + 1);
          issue(P0 * (kk + 1), kk == KK - 2 ? NL : P0 * (kk + 2));
          if (kk == KK - 2) advance();
        } else {
          // this wavefront holds all it needs of the stage, and the next step's operands have landed: younger than those are the
          // loads of the step after it, in the last step of a tile its bias and residual, in the first one the stores of the tile before
          constexpr int N = (NST - 2) * NL + (LAST ? NB : 0);
          if (LAST && has_res) {
            if (first) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N + NRES + NSTO) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N + NRES) : "memory");
          } else {
            if (first) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N + NSTO) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory");
          }
          __builtin_amdgcn_s_barrier();
          frags(0, nxt, 0);
          issue(0, P0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int j = 0; j < TP; ++j) {
            if constexpr (ES == 1) acc[i][j] = E::mfma2(fa[kk & 1][i][0], fa[kk & 1][i][1], fb[kk & 1][j][0], fb[kk & 1][j][1], acc[i][j]);
            else acc[i][j] = E::mfma(fa[kk & 1][i][0], fb[kk & 1][j][0], acc[i][j]);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      st_rd = nxt;
    };
    for (int kb = 0; kb + 1 < nk; ++kb) step(std::false_type{}, stored && kb == 0);
    step(std::true_type{}, stored && nk == 1);

    // epilogue, from registers: lane (l32, g) holds channels 16 g + 4 q + e of each 32-channel block of its pixel
    if constexpr (PJ < TP) { if (has_res) load_res(PJ, TP); }
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y + a.y_coff + (long long)p0 * a.y_ld), 0, (int)BUF_MAX, BUF_FLAGS);
    const __amdgpu_buffer_rsrc_t ry2 = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y2 + a.y2_coff - a.split + (long long)p0 * a.y2_ld), 0, (int)BUF_MAX, BUF_FLAGS);
    with_epilogue_mode(has_res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
    constexpr int RES = decltype(res_c)::value;
    constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      const int pl = wp * (TP * 32) + j * 32 + l32;
      const bool in = p0 + pl < M;
      const int yo = in ? (pl * a.y_ld + cw) * ES : OOB, yo2 = in ? (pl * a.y2_ld + cw) * ES : OOB;
#pragma unroll
      for (int i = 0; i < TC; ++i) {
        // two layers in one launch: the split is a multiple of 32 channels, so a block belongs to one of them
        const bool second = a.split > 0 && c0 + wc * (TC * 32) + i * 32 >= a.split;
#pragma unroll
        for (int h = 0; h < HV; ++h) {
          u32x4 out;
          if constexpr (ES == 2) {
            typedef T t4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              floatx4 v, r4 = floatx4{0.f, 0.f, 0.f, 0.f};
              if constexpr (RES != OCTO_RES_NONE) {
                const u32x2 rw = {rv[j][i][h][2 * q], rv[j][i][h][2 * q + 1]};
                const t4 rt = __builtin_bit_cast(t4, rw);
                r4 = floatx4{(float)rt[0], (float)rt[1], (float)rt[2], (float)rt[3]};
              }
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = acc[i][j][h * VN + q * 4 + e];
              v = finish4<RES, SILU>(v, *(const floatx4*)&sBias[bbuf][wc * (TC * 32) + g * 16 + i * 32 + h * VN + q * 4], r4, act_lo);
              const t4 o = {(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
              const u32x2 ob = __builtin_bit_cast(u32x2, o);
              out[2 * q] = ob[0]; out[2 * q + 1] = ob[1];
            }
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int cq = wc * (TC * 32) + g * 16 + i * 32 + q * 4;
              floatx4 v, r4 = floatx4{0.f, 0.f, 0.f, 0.f};
              if constexpr (RES != OCTO_RES_NONE) r4 = f8_unpack4(tail && q < 2 && cw + i * 32 + 8 == a.Cout ? rv[j][i][0][(q + 2) & 3] : rv[j][i][0][q]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                v[e] = acc[i][j][q * 4 + e] * sScale[bbuf][cq + e];
                r4[e] *= a.res_scale;
              }
              v = finish4<RES, SILU>(v, *(const floatx4*)&sBias[bbuf][cq], r4, act_lo);
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] *= a.y_inv_scale;
              out[q] = f8_pack4(v);
            }
          }
          const bool ok = cw + i * 32 + h * VN + VN <= a.Cout;
          const int left = a.Cout - (c0 + wc * (TC * 32) + i * 32);
          if (ES == 2 && tail && left > 0 && left < 32 && (left / VN) % 2 == h) {    // the vector that ends past the last channel: its values in pairs
            const int to = !ok && cw + i * 32 + h * VN < a.Cout ? yo + i * 32 * ES + h * 16 : OOB;
#pragma unroll
            for (int e = 0; e < VN / 2; ++e) {
              if (2 * e + 2 <= left % VN) __builtin_amdgcn_raw_buffer_store_b32(out[e], ry, to + e * 4, 0, 0);
              else if (2 * e + 1 == left % VN) __builtin_amdgcn_raw_buffer_store_b16((short)out[e], ry, to + e * 4, 0, 0);
            }
          }
          if (ES == 1 && tail && left > 0 && left < 32)    // the half vector
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{out[0], out[1]}, ry, cw + i * 32 + 8 == a.Cout ? yo + i * 32 : OOB, 0, 0);
          if (second) __builtin_amdgcn_raw_buffer_store_b128(out, ry2, ok ? yo2 + i * 32 * ES + h * 16 : OOB, 0, 0);
          else __builtin_amdgcn_raw_buffer_store_b128(out, ry, ok ? yo + i * 32 * ES + h * 16 : OOB, 0, 0);
          __builtin_amdgcn_sched_barrier(0);               // one vector at a time: keeps the register demand low
        }
      }
    }
    });
    if (!more) break;
    stored = true;
    t = tn; p0 = pn0; c0 = cn0;
    if (tiles_c > 1) bbuf = next_bias(bbuf);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // loads issued past the last step write zeros into LDS
}

template <typename T, int NT, int BC, int BP, int WC, int KV, int NST, int MINB, int MODE>
static hipError_t launch_flow_mode(const ConvArgs& a, const FlowGeom& gm, long long tiles, int num_cu, hipStream_t s, const ConvTiming& tm) {
  long long grid = (tiles + 7) / 8 * 8;
  const long long cap = ((long long)num_cu * flow_resident(sizeof(T), NT, BC, BP, KV, NST, MINB) + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv_flow_kernel<T, NT, BC, BP, WC, KV, NST, MINB, MODE>), dim3((unsigned)grid), dim3(NT), 0, s, tm.start, tm.stop, 0, a, gm);
  else
    hipLaunchKernelGGL((conv_flow_kernel<T, NT, BC, BP, WC, KV, NST, MINB, MODE>), dim3((unsigned)grid), dim3(NT), 0, s, a, gm);
  return hipGetLastError();
}

template <typename T, int NT, int BC, int BP, int WC, int KV, int NST, int MINB>
static hipError_t launch_flow_cfg(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  constexpr int BK = KV * Elem<T>::N;
  // The bias of a tile is requested at the last step of the one before: its place must be free, and it must have landed by the epilogue (older than
  // the operands of step NST - 2).  Other wavefronts may still read that of the tile before in its epilogue: two places do where a barrier
  // lies between, which takes two K steps or a single channel tile.  E4M3, whose steps are wide, goes round three.
  static_assert(KV == 8 && NST <= 4, "operands are younger than the bias");
  if (sizeof(T) == 2 && a.K <= BK && a.Cout > BC) return hipErrorNotSupported;
  const long long M = (long long)a.n * a.Ho * a.Wo, tiles_c = (a.Cout + BC - 1) / BC, tiles = (M + BP - 1) / BP * tiles_c;
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x3FFFFFF0LL) return hipErrorNotSupported;
  const bool whole = a.Cin % BK == 0, pw = whole && a.kh == 1 && a.kw == 1 && a.stride_h == 1 && a.stride_w == 1 && !a.pad_h && !a.pad_w;
  const int mode = pw ? FLOW_POINTWISE : whole ? FLOW_TAPS : FLOW_ANY;
  if (kernel_id) *kernel_id = flow_kernel_id(BC, BP, KV, mode);
  const FlowGeom gm{make_fastdiv((unsigned)tiles_c), make_fastdiv((unsigned)(a.Ho * a.Wo)), make_fastdiv((unsigned)a.Wo)};
  if (pw) return launch_flow_mode<T, NT, BC, BP, WC, KV, NST, MINB, FLOW_POINTWISE>(a, gm, tiles, num_cu, s, tm);
  if (whole) return launch_flow_mode<T, NT, BC, BP, WC, KV, NST, MINB, FLOW_TAPS>(a, gm, tiles, num_cu, s, tm);
  return launch_flow_mode<T, NT, BC, BP, WC, KV, NST, MINB, FLOW_ANY>(a, gm, tiles, num_cu, s, tm);
}

// One entry point per storage type; `which` counts the rows of FLOW_COST.
template <typename T>
static hipError_t launch_flow(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  switch (which) {
    case 0: return launch_flow_cfg<T, 256, 64, 64, 2, 8, 3, 3>(a, num_cu, s, kernel_id, tm);
    case 1: return launch_flow_cfg<T, 256, 64, 128, 1, 8, 3, 2>(a, num_cu, s, kernel_id, tm);
    case 2: return launch_flow_cfg<T, 256, 128, 64, 2, 8, 3, 2>(a, num_cu, s, kernel_id, tm);
    case 3: return launch_flow_cfg<T, 512, 128, 128, 2, 8, 3, 1>(a, num_cu, s, kernel_id, tm);
    case 4: return launch_flow_cfg<T, 512, 96, 256, 1, 8, 3, 1>(a, num_cu, s, kernel_id, tm);
    case 5: return launch_flow_cfg<T, 512, 192, 128, 2, 8, 3, 1>(a, num_cu, s, kernel_id, tm);
    case 6: return launch_flow_cfg<T, 512, 128, 256, 2, 8, 3, 1>(a, num_cu, s, kernel_id, tm);
    case 7: return launch_flow_cfg<T, 512, 256, 128, 4, 8, 3, 1>(a, num_cu, s, kernel_id, tm);
  }
  return hipErrorNotSupported;
}

}  // namespace octo
