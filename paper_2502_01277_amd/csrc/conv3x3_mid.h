// 3x3 / stride-1 / pad-1 convolution with the input patch of a tile in LDS, for tiles of 32 to 128 channels x 64 to 256 pixels.
//
// What paces the general kernel (conv.hip) on these layers is the operand fetch from the L2s: every input pixel is
// fetched once per kernel tap, and a workgroup that is alone on its compute unit gets 18 .. 25 bytes per clock.  Here
//   * a tile is TH x TW output pixels of the image stack (the images of the batch are consecutive in memory, so a tile may
//     span several of them) times BC output channels;
//   * the K loop runs over slices of KV * 16 bytes of input channels and, inside a slice, over the nine taps.  The patch
//     of a slice - TH + 2 stack rows, and one column on each side where the tile is narrower than the image - is fetched
//     once into one of two LDS buffers; only the BC weight rows of a (slice, tap) step stream, through a ring of NST stages.
//     A 64 x 128 tile then fetches 10.5 KB per 128-byte step instead of 24 KB;
//   * the pixel operand of every tap is read from the patch with an address that the lane works out once per tile; taps
//     outside the image point at rows of zeros, so that image borders need no padding rows in LDS;
//   * the barrier of a step sits before the last group of its MFMAs, with the next step's first fragments read behind it;
//   * the stream of loads runs on across tiles: the last slice of a tile requests the first patch, weights and bias of the next one, and
//     the residual two taps before the end.  Weight rows are taken in an order that leaves 16 consecutive channels of a pixel in one
//     lane, so that results leave as 16-byte stores straight from registers, LDS stays the next tile's, and the stores drain beside
//     its K loop.
// What bounds it: the matrix pipe and the clock that the power leaves it (1.65 .. 2.1 GHz on random data), and on 28 x 28 maps the memory
// traffic.  By cycle counts of 128 -> 128 on 4170 x 28 x 28 (64 x 256 tiles) with the epilogue through LDS and a prologue of its own
// per tile, the K loop took 64 % of the time, addresses and prologue 20 %, the way out 16 %, and waiting for the residual as much as
// a quarter of it all.  Before and after, us: that layer 1022 -> 863 without and 1227 -> 989 with residual, 256 -> 256 on 4170 x 14 x 14
// 969 -> 813, 512 -> 512 on 4170 x 7 x 7 865 -> 743 (0.96 -> 1.30 PFLOP/s), 96 -> 96 on 32 x 160 x 160 214 -> 177.
// LDS rows (weights: one output channel; patch: one pixel) are KV vectors of 16 bytes, vector v of row r in slot
// v ^ ((r / (16 / KV)) % KV).  For patch pixels r counts without the halo columns (patch row * TW + column), so that the lanes of
// consecutive output pixels stay on different banks where a tile row ends (with the halo counted, 64 -> 64 on 56 x 56 maps ran
// 10 % slower), and a lane outside the image reads zeros from its own bank.
// vmcnt bookkeeping: every wavefront issues the same number of loads per tap, known at compile time, in program order.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include "conv3x3_stream.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace octo {

// Tile geometry of one layer, built on the host.
struct MidGeom {
  int TW, TH;            // output tile: TH rows of the image stack x TW columns (the last tile of a row may be narrower)
  int PW, halo;          // patch width, and its columns left of the tile (0 where the tile spans the image width)
  int tiles_x;           // tiles per image row
  FastDiv div_tw, div_pw, div_h, div_tc, div_tx;   // divisions by TW, PW, H, channel tiles, tiles_x
};

// Passes of the next slice's patch that are issued at tap t of a slice (all within the first six taps), and the loads that may
// still be in flight when the operands of the step after tap t must have landed: those issued at the NST - 2 taps before t.  The
// last slice of a tile also fetches `extra` vectors (bias, scales) of the next tile at tap 0.
constexpr int mid_ppt(int maxp) { return (maxp + 5) / 6; }
constexpr int mid_passes(int t, int maxp) {
  const int left = maxp - (t + 9) % 9 * mid_ppt(maxp);
  return left < 0 ? 0 : (left < mid_ppt(maxp) ? left : mid_ppt(maxp));
}
constexpr int mid_in_flight(int t, int nst, int la, int maxp, int extra) {
  int n = 0;
  for (int i = t + 2 - nst; i < t; ++i) n += la + mid_passes(i, maxp) + (i == 0 ? extra : 0);
  return n;
}

// The first n of a vector's values to or from memory of any alignment.
template <typename T>
__device__ __forceinline__ void mid_store_pieces(T* p, u32x4 v, int n) {
  constexpr int HN = 8 / (int)sizeof(T);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (n >= (h + 1) * HN && ((uintptr_t)p & 7) == 0) { *(u32x2*)(p + h * HN) = u32x2{v[2 * h], v[2 * h + 1]}; continue; }
#pragma unroll
    for (int e = 0; e < HN; ++e) {
      const uint32_t w = v[2 * h + e * (int)sizeof(T) / 4] >> (e * (int)sizeof(T) % 4 * 8);
      if (h * HN + e >= n) continue;
      if constexpr (sizeof(T) == 1) p[h * HN + e].bits = (uint8_t)w;
      else p[h * HN + e] = __builtin_bit_cast(T, (uint16_t)w);
    }
  }
}
template <typename T>
__device__ __forceinline__ u32x4 mid_load_pieces(const T* p, int n) {
  constexpr int HN = 8 / (int)sizeof(T);
  u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (n >= (h + 1) * HN && ((uintptr_t)p & 7) == 0) {
      const u32x2 w = *(const u32x2*)(p + h * HN);
      v[2 * h] = w[0]; v[2 * h + 1] = w[1];
      continue;
    }
#pragma unroll
    for (int e = 0; e < HN; ++e) {
      uint32_t w = 0u;
      if (h * HN + e < n) {
        if constexpr (sizeof(T) == 1) w = p[h * HN + e].bits;
        else w = __builtin_bit_cast(uint16_t, p[h * HN + e]);
      }
      v[2 * h + e * (int)sizeof(T) / 4] |= w << (e * (int)sizeof(T) % 4 * 8);
    }
  }
  return v;
}

// BC x BP: tile; WC: wavefronts along the channels (4 / WC along the pixels); KV: vectors of 16 bytes per LDS row; NST: stages
// of the weight ring; MAXP: passes of the 256 loader lanes that cover a patch buffer; MINB: workgroups per compute unit.
template <typename T, int BC, int BP, int WC, int KV, int NST, int MAXP, int MINB>
__global__ __launch_bounds__(THREADS, MINB) void conv3x3_mid_kernel(const ConvKernelArgs a, const MidGeom gm) {
  using E = Elem<T>;
  constexpr int VN = E::N, ES = (int)sizeof(T), BK = KV * VN;
  constexpr int WP = 4 / WC, TC = BC / WC / 32, TP = BP / WP / 32;
  constexpr int RPW = 16 / KV, RP = THREADS / KV, LA = (BC + RP - 1) / RP;
  constexpr int ROW = KV * 16, STAGE = LA * RP * ROW, PATCH = MAXP * 4096;
  constexpr int KK = ES == 1 ? KV / 4 : KV / 2;          // groups of MFMAs per step
  constexpr int FV = ES == 1 ? 2 : 1;                    // vectors per operand fragment
  constexpr int ZROW = MAXP * RP - RPW;                  // last rows of a patch buffer, kept zero (the host leaves them free)
  constexpr int NTAP = 9;
  constexpr int HV = 16 / VN;                            // vectors of a lane's 16 consecutive output channels of a 32-channel block
  constexpr int PJ = TC * TP * HV <= 8 ? TP : 1;         // pixel blocks whose residual is requested before the K loop ends
  constexpr int NSTO = TC * TP * HV, NRES = TC * PJ * HV, NB = ES == 1 ? 2 : 1;
  constexpr bool PACKED = TC * TP >= 8;                  // two patch offsets per register where accumulators leave few
  constexpr int BW = PACKED ? (TP + 1) / 2 : TP;
  constexpr int RTAP = NTAP - NST;                       // tap of the last slice that requests the residual
  static_assert(BC % 32 == 0 && TC >= 1 && TP >= 1 && (KK == 1 || KK % 2 == 0) && NST >= 2 && NST <= 4, "tile shape");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NST * STAGE + 2 * PATCH];
  __shared__ __attribute__((aligned(16))) float sBias[2][THREADS];               // of this tile and the next
  __shared__ __attribute__((aligned(16))) float sScale[2][ES == 1 ? THREADS : 1];
  unsigned char* ring = smem;
  unsigned char* patch = smem + NST * STAGE;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wc = wave % WC, wp = wave / WC;
  const int l32 = lane & 31, g = lane >> 5;
  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int H = a.H, W = a.W;
  const int n_rows = n_items * H;
  const int tiles_c = (a.Cout + BC - 1) / BC;
  const int n_tiles = (n_rows + gm.TH - 1) / gm.TH * gm.tiles_x * tiles_c;       // < 2^31 (host)
  const int n_slices = (a.Cin + BK - 1) / BK;
  const T* __restrict__ xg = (const T*)a.x + a.x_coff;

  const int ld_row = tid / KV;
  const int lkv = (tid % KV) ^ ((ld_row / RPW) % KV);    // logical vector of this lane's slot of a weight row
  const int rsw = (l32 / RPW) % KV;
  const unsigned lds_ring = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)ring + (unsigned)wave * 1024u));
  const unsigned lds_patch = lds_ring + NST * STAGE;
  const unsigned lds_bias = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)&sBias[0][0] + (unsigned)wave * 256u));
  const unsigned lds_scale = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)&sScale[0][0] + (unsigned)wave * 256u));
  const long long w_bytes = (long long)a.w_rows * a.Kp * ES;
  const int w_len = (int)(w_bytes < BUF_MAX ? w_bytes : BUF_MAX);
  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;
  // outputs and residuals in whole aligned vectors; anything else is written and read in pieces
  const bool vec_out = ((a.Cout | a.y_ld | a.y_coff) % VN) == 0 && ((uintptr_t)a.y & 15) == 0;
  const bool vec_res = a.res && ((a.Cout | a.res_ld | a.res_coff) % VN) == 0 && ((uintptr_t)a.res & 15) == 0;

  const int per_die = (n_tiles + 7) >> 3;      // see conv_mfma_kernel: one contiguous chunk of the tile list per die
  const int t_end = per_die * 8;
  auto next_valid = [&](int t) -> int {
    while (t < t_end && (t & 7) * per_die + (t >> 3) >= n_tiles) t += gridDim.x;
    return t;
  };
  auto locate = [&](int t, int& v0, int& x0, int& c0) __attribute__((always_inline)) {
    const unsigned tile = (unsigned)((t & 7) * per_die + (t >> 3));
    const unsigned tpx = fast_div(tile, gm.div_tc), tv = fast_div(tpx, gm.div_tx);
    c0 = (int)(tile - tpx * (unsigned)tiles_c) * BC;
    x0 = (int)(tpx - tv * (unsigned)gm.tiles_x) * gm.TW;
    v0 = (int)tv * gm.TH;
  };

  // Loaders.  Patch: this lane's vector of every pass, relative to the first patch row of a tile; vectors past `channels` of a slice
  // read as zeros.  (Lane values are opaque to the compiler, which would otherwise keep the tile-independent part of every
  // address in registers of its own.)
  int poff[MAXP], woff[LA], p_len = 0;
  void* p_base = nullptr;
  auto patch_of = [&](int v0, int x0, int channels) __attribute__((always_inline)) {
    const long long pix0 = (long long)(v0 - 1) * W;                  // may be -W: lanes of that row are out of range
    const long long rem_bytes = (((long long)a.n * H * W - pix0) * a.x_ld - a.x_coff) * ES;
    p_len = (int)(rem_bytes < BUF_MAX ? rem_bytes : BUF_MAX);
    p_base = (void*)(xg + pix0 * a.x_ld);
    int lrow = ld_row;
    asm volatile("" : "+v"(lrow));
#pragma unroll
    for (int i = 0; i < MAXP; ++i) {
      const int pp = i * RP + lrow;
      const int pr = (int)fast_div((unsigned)pp, gm.div_pw), pc = pp - pr * gm.PW;
      const int v = v0 - 1 + pr, x = x0 - gm.halo + pc;
      const int vec = (tid % KV) ^ ((int)((unsigned)(pr * gm.TW + pc) / RPW) % KV);
      const bool ok = pr < gm.TH + 2 && (unsigned)v < (unsigned)n_rows && (unsigned)x < (unsigned)W && vec * VN < channels;
      poff[i] = ok ? ((pr * W + x) * a.x_ld + vec * VN) * ES : OOB;
    }
  };
  // Weights: LDS row m of a 32-row block holds channel 16 ((m / 4) % 2) + 4 (m / 8) + m % 4 of the block: register 4 q + e of half g of
  // a wavefront's result is row 8 q + 4 g + e, so a lane gets 16 consecutive channels of its pixel
  {
    const int m = ld_row & 31, ch = (ld_row & ~31) + 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
#pragma unroll
    for (int i = 0; i < LA; ++i) woff[i] = ld_row + RP * i < BC ? ((ch + RP * i) * a.Kp + lkv * VN) * ES : OOB;
  }
  // weights of the channels from c0 on, (slice, tap), into ring stage st; nothing is fetched if !any
  auto issue_w = [&](int c0, int sl, int tap, int st, bool any) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, any ? w_len : 0, BUF_FLAGS);
    const int koff = any ? (c0 * a.Kp + tap * a.Cin + sl * BK) * ES : 0;
#pragma unroll
    for (int i = 0; i < LA; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(lds_ring + st * STAGE + i * 4096), "v"(woff[i]), "s"(rs), "s"(koff) : "memory");
  };
  // passes of a slice's patch into buffer buf
  auto issue_p = [&](int buf, int sl, int from, int count, bool any) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(p_base, 0, any ? p_len : 0, BUF_FLAGS);
    const int koff = any ? sl * BK * ES : 0;
#pragma unroll
    for (int i = 0; i < MAXP; ++i)
      if (i >= from && i < from + count)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds_patch + buf * PATCH + i * 4096), "v"(poff[i]), "s"(rs), "s"(koff) : "memory");
  };
  auto issue_bias = [&](int c0, int buf, bool any) __attribute__((always_inline)) {       // (and scales); padded to whole tiles like the weights
    const int off = tid < BC ? (c0 + tid) * 4 : OOB, len = any ? a.w_rows * 4 : 0;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, len, BUF_FLAGS);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_bias + buf * (THREADS * 4)), "v"(off), "s"(rb) : "memory");
    if constexpr (ES == 1) {
      const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void*)a.scale, 0, len, BUF_FLAGS);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_scale + buf * (THREADS * 4)), "v"(off), "s"(rc) : "memory");
    }
  };

  int t = next_valid(blockIdx.x);
  if (t >= t_end) return;
  int v0, x0, c0;
  locate(t, v0, x0, c0);
  issue_bias(c0, 0, true);
  patch_of(v0, x0, a.Cin);
  issue_p(0, 0, 0, MAXP, true);
  constexpr int AHEAD = KK == 1 ? NST - 1 : NST;         // steps whose weights are requested ahead
#pragma unroll
  for (int d = 0; d < AHEAD; ++d) issue_w(c0, 0, d, d, true);
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((AHEAD - 1) * LA) : "memory");
  __builtin_amdgcn_s_barrier();

  int rd = 0, pbuf = 0, bbuf = 0;                        // ring stage of the current step, patch buffer of the current slice, bias buffer
  bool stored = false;                                   // the vmcnt of the first steps counts the stores of the tile before
  for (;;) {
    // byte offset inside a patch buffer of this lane's first vector, per tap and block
    int baddr[NTAP][BW], lpix = wp * (TP * 32) + l32;
    asm volatile("" : "+v"(lpix));
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      const int q = lpix + j * 32;
      const int ty = (int)fast_div((unsigned)q, gm.div_tw), tx = q - ty * gm.TW;
      const int v = v0 + ty, x = x0 + tx;
      const int yy = v - (int)fast_div((unsigned)v, gm.div_h) * H;
      const bool ok = ty < gm.TH && v < n_rows && x < W;
#pragma unroll
      for (int tap = 0; tap < NTAP; ++tap) {
        const int r = tap / 3, s = tap % 3 - 1;
        const bool in = ok && (unsigned)(yy + r - 1) < (unsigned)H && (unsigned)(x + s) < (unsigned)W;
        const int px = (ty + r) * gm.PW + tx + s + gm.halo, pos = px - (ty + r) * (gm.PW - gm.TW);
        const int off = (in ? px : ZROW + (px & (RPW - 1))) * ROW + ((g ^ ((pos >> (RPW == 2 ? 1 : 2)) & (KV - 1))) << 4);
        if (!PACKED) baddr[tap][j] = off;
        else baddr[tap][j / 2] = j % 2 ? baddr[tap][j / 2] | off << 16 : off;
      }
    }

    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    u32x4 fa[2][TC][FV], fb[2][TP][FV];
    const int arow = (wc * (TC * 32) + l32) * ROW;
    auto frags = [&](int set, int st, const int (&ba)[BW], int buf, int kq) __attribute__((always_inline)) {
      const unsigned char* pa = ring + st * STAGE + arow;
      const unsigned char* pb = patch + buf * PATCH;
#pragma unroll
      for (int h = 0; h < FV; ++h) {
        const int v = (kq * FV + h) * 2;
#pragma unroll
        for (int i = 0; i < TC; ++i) fa[set][i][h] = *(const u32x4*)(pa + i * (32 * ROW) + (((v + g) ^ rsw) << 4));
#pragma unroll
        for (int j = 0; j < TP; ++j) fb[set][j][h] = *(const u32x4*)(pb + ((PACKED ? (j % 2 ? (int)((unsigned)ba[j / 2] >> 16) : ba[j / 2] & 0xFFFF) : ba[j]) ^ (v << 4)));
      }
    };
    // output and residual: offset of this lane's first channel from the tile's first pixel, per pixel block
    const int cw = c0 + wc * (TC * 32) + g * 16;
    const long long pix0 = (long long)v0 * W + x0;
    auto pixel_off = [&](int j, int ld) __attribute__((always_inline)) -> int {
      const int q = lpix + j * 32;
      const int ty = (int)fast_div((unsigned)q, gm.div_tw), tx = q - ty * gm.TW;
      return ty < gm.TH && v0 + ty < n_rows && x0 + tx < W ? ((ty * W + tx) * ld + cw) * ES : OOB;
    };
    u32x4 rv[TP][TC][HV];
    auto load_res = [&](int from, int to) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)((const T*)a.res + a.res_coff + pix0 * a.res_ld), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
      for (int j = 0; j < TP; ++j) {
        if (j < from || j >= to) continue;
        const int off = pixel_off(j, a.res_ld);
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int h = 0; h < HV; ++h)
            rv[j][i][h] = __builtin_amdgcn_raw_buffer_load_b128(rr, cw + i * 32 + h * VN < a.Cout ? off + i * 32 * ES + h * 16 : OOB, 0, 0);
      }
    };

    int vn0 = 0, xn0 = 0, cn0 = 0;                       // the next tile, whose operands are requested during the last slice
    bool more = false;
    // Waits until the operands of the step after tap TAP of a slice have landed.  In program order later than those: the loads of
    // the NST - 2 taps before, the residual's after tap RTAP of the last slice, and, in the first steps, the stores of the tile before
    auto landed = [&](auto tapc, auto lastc, bool first) __attribute__((always_inline)) {
      constexpr int TAP = decltype(tapc)::value;
      constexpr bool LAST = decltype(lastc)::value;
      constexpr int N = mid_in_flight(TAP, NST, LA, MAXP, LAST ? NB : 0);
      constexpr bool AFTER_RES = LAST && TAP > RTAP, AFTER_STORES = TAP < NST - 1;
      if constexpr (AFTER_STORES) {
        if (first) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N + NSTO) : "memory"); return; }
      }
      if constexpr (AFTER_RES) {
        if (vec_res) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N + NRES) : "memory"); return; }
      }
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory");
    };
    auto step = [&](auto tapc, auto lastc, int sl) __attribute__((always_inline)) {
      constexpr int TAP = decltype(tapc)::value, NEXT = (TAP + 1) % NTAP;
      constexpr bool LAST = decltype(lastc)::value;
      const int cur = NTAP % NST == 0 ? TAP % NST : rd;
      const int nxt = NTAP % NST == 0 ? NEXT % NST : (rd + 1 == NST ? 0 : rd + 1);
      // loads that go out at this tap: the next slice's patch, weights AHEAD steps on, both of the next tile after the last slice
      auto issue = [&](int st) __attribute__((always_inline)) {
        issue_p(pbuf ^ 1, LAST ? 0 : sl + 1, TAP * mid_ppt(MAXP), mid_passes(TAP, MAXP), !LAST || more);
        constexpr bool WRAP = TAP + AHEAD >= NTAP;
        issue_w(LAST && WRAP ? cn0 : c0, WRAP ? (LAST ? 0 : sl + 1) : sl, (TAP + AHEAD) % NTAP, st, !(LAST && WRAP) || more);
        if constexpr (LAST && TAP == 0) issue_bias(cn0, bbuf ^ 1, more);
        if constexpr (LAST && TAP == RTAP) { if (vec_res) load_res(0, PJ); }
      };
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        if constexpr (KK == 1) {
          // a single group per step: its fragments are read here, and the loads go to the stage that the previous step has left
          landed(tapc, lastc, stored && sl == 0);
          __builtin_amdgcn_s_barrier();
          frags(0, cur, baddr[TAP], pbuf, 0);
          issue(NTAP % NST == 0 ? (TAP + NST - 1) % NST : (rd == 0 ? NST - 1 : rd - 1));
        } else if (kk < KK - 1) {
          frags((kk + 1) & 1, cur, baddr[TAP], pbuf, kk + 1);
        } else {
          // this wavefront holds all it needs of the stage in registers, and the next step's operands have landed
          landed(tapc, lastc, stored && sl == 0);
          __builtin_amdgcn_s_barrier();
          if constexpr (!(LAST && TAP == NTAP - 1)) frags(0, nxt, baddr[NEXT], TAP == NTAP - 1 ? pbuf ^ 1 : pbuf, 0);
          issue(cur);
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
      rd = nxt;
    };
    auto slice = [&](auto lastc, int sl) __attribute__((always_inline)) {
      if constexpr (PACKED) {        // opaque: the unpacked offsets would otherwise be kept in registers of their own
#pragma unroll
        for (int tap = 0; tap < NTAP; ++tap)
#pragma unroll
          for (int j = 0; j < BW; ++j) asm volatile("" : "+v"(baddr[tap][j]));
      }
      step(std::integral_constant<int, 0>{}, lastc, sl); step(std::integral_constant<int, 1>{}, lastc, sl); step(std::integral_constant<int, 2>{}, lastc, sl);
      step(std::integral_constant<int, 3>{}, lastc, sl); step(std::integral_constant<int, 4>{}, lastc, sl); step(std::integral_constant<int, 5>{}, lastc, sl);
      step(std::integral_constant<int, 6>{}, lastc, sl); step(std::integral_constant<int, 7>{}, lastc, sl); step(std::integral_constant<int, 8>{}, lastc, sl);
      pbuf ^= 1;
    };
    if constexpr (KK > 1) frags(0, rd, baddr[0], pbuf, 0);
    for (int sl = 0; sl + 1 < n_slices; ++sl) {
      // the last slice, fetched from here on, may be partial: its missing channels are zeros (the weights there anything finite)
      if (sl + 2 == n_slices && a.Cin % BK) patch_of(v0, x0, a.Cin % BK);
      slice(std::false_type{}, sl);
    }
    t = next_valid(t + gridDim.x);
    more = t < t_end;
    if (more) { locate(t, vn0, xn0, cn0); patch_of(vn0, xn0, a.Cin); }
    slice(std::true_type{}, n_slices - 1);

    // epilogue, from registers: lane (l32, g) holds channels 16 g + 4 q + e of each 32-channel block of its pixel
    if constexpr (PJ < TP) { if (vec_res) load_res(PJ, TP); }
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y + a.y_coff + pix0 * a.y_ld), 0, (int)BUF_MAX, BUF_FLAGS);
    const int cl = wc * (TC * 32) + g * 16;
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
    constexpr int RES = decltype(res_c)::value;
    constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      const int yo = pixel_off(j, a.y_ld);
#pragma unroll
      for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int h = 0; h < HV; ++h) {
          const int c = cw + i * 32 + h * VN;              // first channel of the vector
          u32x4 rvec = {0u, 0u, 0u, 0u}, out;
          if constexpr (RES != OCTO_RES_NONE) {
            if (vec_res) rvec = rv[j][i][h];
            else if (yo != OOB) rvec = mid_load_pieces<T>((const T*)a.res + a.res_coff + pix0 * a.res_ld + (pixel_off(j, a.res_ld) / ES - cw + c), a.Cout - c);
          }
#pragma unroll
          for (int q = 0; q < VN / 4; ++q) {
            const int cq = cl + i * 32 + h * VN + q * 4;
            const floatx4 b4 = *(const floatx4*)&sBias[bbuf][cq];
            floatx4 v, r4 = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (RES != OCTO_RES_NONE) r4 = load4<T>((const T*)&rvec + q * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float av = acc[i][j][h * VN + q * 4 + e];
              v[e] = ES == 1 ? av * sScale[bbuf][cq + e] : av;
              if (ES == 1) r4[e] *= a.res_scale;
            }
            v = finish4<RES, SILU>(v, b4, r4, act_lo);
            if constexpr (ES == 1) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] *= a.y_inv_scale;
            }
            store4<T>((T*)&out + q * 4, v);
          }
          if (vec_out) __builtin_amdgcn_raw_buffer_store_b128(out, ry, c < a.Cout ? yo + i * 32 * ES + h * 16 : OOB, 0, 0);
          else if (yo != OOB) mid_store_pieces<T>((T*)a.y + a.y_coff + pix0 * a.y_ld + (yo / ES - cw + c), out, a.Cout - c);
          __builtin_amdgcn_sched_barrier(0);               // one vector at a time: keeps the register demand low
        }
    }
    });
    if (!more) break;
    stored = vec_out;
    if (!vec_out || (a.res && !vec_res)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); stored = false; }     // a number of accesses that is not known here
    v0 = vn0; x0 = xn0; c0 = cn0;
    bbuf ^= 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // loads issued past the last step write zeros into LDS
}

// Tile of at most BP pixels whose patch leaves four of `rows` LDS rows free: the split of the image width into equal columns and
// the number of rows that give the most pixels per tile, ties to the smaller patch.  False if no shape fills 3/4 of the tile.
inline bool mid_geometry(const ConvArgs& a, int BC, int BP, int rows, MidGeom* gm) {
  double best = 0;
  int best_patch = 0;
  for (int nx = 1; nx <= a.W; ++nx) {
    const int tw = (a.W + nx - 1) / nx, pw = nx == 1 ? tw : tw + 2;
    if (tw > BP) continue;
    if (tw < 4) break;
    const int th = std::min(BP / tw, (rows - 4) / pw - 2);
    if (th < 1) continue;
    const int tiles_x = (a.W + tw - 1) / tw, patch = (th + 2) * pw;
    const double px = (double)a.W * th / tiles_x;
    if (px > best || (px == best && patch < best_patch)) {
      best = px; best_patch = patch;
      gm->TW = tw; gm->TH = th; gm->PW = pw; gm->halo = nx == 1 ? 0 : 1; gm->tiles_x = tiles_x;
    }
  }
  if (best * 4 < BP * 3) return false;
  gm->div_tw = make_fastdiv((unsigned)gm->TW); gm->div_pw = make_fastdiv((unsigned)gm->PW);
  gm->div_h = make_fastdiv((unsigned)a.H); gm->div_tx = make_fastdiv((unsigned)gm->tiles_x);
  gm->div_tc = make_fastdiv((unsigned)((a.Cout + BC - 1) / BC));
  return true;
}

template <typename T, int BC, int BP, int WC, int KV, int NST, int MAXP, int MINB>
hipError_t launch_mid_cfg(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  MidGeom gm{};
  constexpr int ROWS = MAXP * (THREADS / KV);
  if (!mid_geometry(a, BC, BP, ROWS, &gm)) return hipErrorNotSupported;
  const long long n_rows = (long long)a.n * a.H;
  const long long tiles = ((n_rows + gm.TH - 1) / gm.TH) * gm.tiles_x * ((a.Cout + BC - 1) / BC);
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x7FFFFFF0LL || n_rows * a.W >= 0x7FFFFFFFLL) return hipErrorNotSupported;
  if ((long long)(gm.TH + 2) * a.W * std::max(a.x_ld, std::max(a.y_ld, a.res ? a.res_ld : 0)) * (int)sizeof(T) > 0x7FFFFFF0LL) return hipErrorNotSupported;     // 32-bit offsets inside a tile
  if (kernel_id) *kernel_id = mid_kernel_id(BC, BP, KV, Elem<T>::N, MAXP, a.Cin, a.Cout);
  long long grid = (tiles + 7) / 8 * 8;
  const long long cap = ((long long)num_cu * MINB + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv3x3_mid_kernel<T, BC, BP, WC, KV, NST, MAXP, MINB>), dim3((unsigned)grid), dim3(THREADS), 0, s, tm.start, tm.stop, 0, a, gm);
  else
    hipLaunchKernelGGL((conv3x3_mid_kernel<T, BC, BP, WC, KV, NST, MAXP, MINB>), dim3((unsigned)grid), dim3(THREADS), 0, s, a, gm);
  return hipGetLastError();
}

// Does the layer have the form that conv3x3_mid_kernel takes?  Input alignment is the caller's to check.
inline bool mid_fits(const ConvArgs& a) {
  return a.kh == 3 && a.kw == 3 && a.stride_h == 1 && a.stride_w == 1 && a.pad_h == 1 && a.pad_w == 1 && !a.out_f32 && !a.pair_view &&
         !a.pool_y && !a.up_y && a.split == 0;
}

// Tiles of one configuration for a layer with that many items, per compute unit and rounded up; 0 where no tile shape fits.
inline long long mid_rounds(const ConvArgs& a, long long items, int BC, int BP, int rows, int num_cu) {
  MidGeom gm{};
  if (!mid_geometry(a, BC, BP, rows, &gm)) return 0;
  const long long tiles = (items * a.H + gm.TH - 1) / gm.TH * gm.tiles_x * ((a.Cout + BC - 1) / BC);
  return (tiles + num_cu - 1) / num_cu;
}

// Tile of a 16-bit layer with M output pixels, or hipErrorNotSupported where the split-K or general kernel is the better one
// (measured on MI355X, bf16, us; layers of H x W x C -> C, by the number of images).  per_cu: 64 x 128 tiles per compute unit.
//   * up to 64 channels and many pixels: conv3x3_stream_kernel;
//   * below 0.25 the split-K kernel spreads the K loop of the few tiles over more wavefronts.  Against 64 x 64 tiles: 14 x 14 x 256 at
//     0.22 9.5 : 9.8, at 0.24 9.8 : 9.9, at 0.26 11.9 : 10.0, at 0.33 12.2 : 10.2; 20 x 20 x 64 at 0.24 6.1 : 5.9, at 0.29 6.8 : 6.0; 40 x 40 x 128
//     at 0.20 7.1 : 7.4, at 0.29 9.2 : 7.6; 13 x 13 x 384 at 0.22 11.8 : 12.4, at 0.25 15.0 : 12.4.  Longer reductions turn at 0.35: 7 x 7 x 512 at
//     0.24 14.1 : 19.1, at 0.33 18.1 : 19.3;
//   * layers whose last 64-channel slice would be half padding (slices of 32, 64 x 128 or 96 x 128 tiles) turn at 0.5, where split-K's 64 x 64
//     tiles no longer are one round: 96 -> 96 on 80 x 80 at 0.39 7.9 : 8.8, on 28 x 28 at 0.48 8.0 : 9.0, at 0.53 8.9 : 9.0, at 0.96 11.3 : 9.3; 288 ->
//     96 on 40 x 40 at 0.49 13.6 : 17.1, at 0.59 18.0 : 17.2; 80 -> 128 on 40 x 40 at 0.49 7.8 : 8.5, at 0.59 8.6 : 8.5; 96 -> 192 there is even from 0.3
//     on (8.1 : 8.0 at 0.44).  96 x 128 tiles with a last slice that even then is partly padding turn at 1.0: 80 -> 80 on 80 x 80 at 0.39 7.8 :
//     9.4, at 0.78 9.0 : 9.7, at 1.17 11.3 : 10.3; 72 -> 72 on 40 x 40 at 0.98 8.7 : 9.4, at 1.07 10.2 : 9.6;
//   * 64 x 64 tiles up to 0.8.  Against 64 x 128: 14 x 14 x 256 at 0.79 13.0 : 13.4, at 1.0 19.8 : 18.1; 7 x 7 x 512 at 0.6 20.7 : 21.3, at 1.0
//     36.2 : 30.1; 28 x 28 x 128 at 0.81 9.3 : 9.9, at 1.0 13.3 : 12.2;
//   * tiles of 32 channels for layers with no more: 32 -> 32 with residual on 16 x 160 x 160 24 us (33).  From 0.8: 80 x 80 x 32 at 0.59 5.8
//     on either, at 0.78 5.7 (general kernel 7.0);
//   * tiles of 96 channels where those of 64 would pad: 96 -> 96 on 32 x 160 x 160 177 us (64 x 256 218), of 256 pixels from four per
//     compute unit on (80 x 80 x 96, 128 : 256 pixels, 15.2 : 17.9 for 10 images, 36.6 : 37.4 for 30, 46.9 : 46.3 for 40);
//   * otherwise by estimated time: tiles per compute unit, rounded up, times what a tile costs beside a 64 x 128 one.  A launch whose
//     compute units have to do one tile more takes that much longer, and large tiles are cheaper by the pixel (128 x 256: four
//     wavefronts that hold all 128 channels read the weights half as often from LDS and the patch half as often from memory).
//     14 x 14 x 256, 64 x 128 (128-byte slices) : 64 x 256 : 128 x 256, at 3.0 34.7 : 33.6 : 35.8, at 4.0 43.6 : 50.0 : 54.7, at 5.0 52.2 :
//     50.4 : 55.9, at 6.0 59.8 : 64.2 : 59.0, at 8.0 78.2 : 77.7 : 85.3, at 10 94.1 : 98.7 : 87.6, at 24 227 : 221 : 211, at 40 383 : 363 :
//     342; 7 x 7 x 512 at 10 175 : 184 : 159, at 40 696 : 669 : 623; 28 x 28 x 128 at 8 46.0 : 48.4 : 53.1, at 10 56.1 : 57.2 : 54.8, at 40 242 : 221 :
//     209.  With less than two tiles per compute unit nothing overlaps a large tile's prologue and epilogue: 64 x 128 then.
//     96 x 256 tiles where 128 would pad but 96 do not: 192 -> 192 on 32 x 80 x 80 123 us (64 x 256 134).
// Reductions over at least 192 channels are paced by the operand fetch: 64 x 128 tiles take slices of 128 bytes (whole cache lines)
// there, and of 64 bytes, half the LDS and up to four workgroups per compute unit elsewhere (28 x 28 x 128 at 2.0 16.0 : 18.8).
// In place in a cascade, where a tile's first operands come from beyond the L2s, 128 channels take the wide slices, which have half the waits, while every
// tile has one of the two places that a compute unit has for them, where the count is not taken on the device (else larger tiles could not be taken for
// more items).  Wide : narrow, over 330 layers of nine maps, 64 .. 384 output channels, with and without residual, 0.91 .. 1.00 of the time up to two tiles per
// compute unit (8 x 40 x 40 at 1.5 12.1 : 13.6, with residual at 1.6 16.7 : 17.8; 41 x 16 x 17 x 256 at 1.4 14.0 : 14.4, 162 x 14 x 12 with residual at 1.7 15.6 :
// 16.5), 1.05 .. 1.13 from there to 2.4, as at 2.1 with residual 269 x 16 x 16 x 64 22.3 : 20.5, and 1.00 .. 1.05 at 2.6 .. 3.2.  64 x 256 tiles of three or four
// whole slices cost 2.05 there (64 x 256 : 64 x 128, traced in two cascades, 192 x 32 x 16 x 128 at 6 30.3 : 27.1, 192 x 28 x 28 with residual at 9.2 42.8 : 38.9;
// where the two costs differ, over 98 layers of 96 channels 1.015, over 78 of 128 0.99), and 1.9 as elsewhere with part of a slice or more of them, which read the
// patch more often (35 x 80 x 80 x 184 -> 128 100 : 118, 13 x 80 x 70 x 184 -> 256 69 : 78; 67 layers of 112 .. 184 channels 0.92).
// The two slice widths sum in different orders; the choice between them is made for a count that stays the same from batch to
// batch (M, from a.n_split), and so the results do.
template <typename T>
hipError_t launch_mid(const ConvArgs& a, long long M, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (!mid_fits(a)) return hipErrorNotSupported;
  const hipError_t es = launch_stream3<T>(a, M, num_cu, s, kernel_id, tm);
  if (es != hipErrorNotSupported) return es;
  const int pad32 = (a.Cin + 31) / 32 * 32, pad64 = (a.Cin + 63) / 64 * 64;
  if (a.Cin * 4 < pad32 * 3) return hipErrorNotSupported;       // more than a quarter of the MFMAs would be padding
  if (a.Cout <= 32) return (double)M / 128 < 0.8 * num_cu ? hipErrorNotSupported : launch_mid_cfg<T, 32, 128, 1, 4, 3, 3, 4>(a, num_cu, s, kernel_id, tm);
  const double per_cu = (double)M / 128 * ((a.Cout + 63) / 64) / num_cu;
  const bool k8 = pad32 == pad64, by96 = (a.Cout + 95) / 96 * 96 < (a.Cout + 63) / 64 * 64;
  if (per_cu < (k8 ? (a.Cin <= 384 ? 0.25 : 0.35) : by96 && a.Cin % 32 ? 1.0 : 0.5)) return hipErrorNotSupported;
  if (k8 && per_cu < 0.8) return launch_mid_cfg<T, 64, 64, 2, 8, 3, 4, 2>(a, num_cu, s, kernel_id, tm);
  if (by96 && !(k8 && a.Cin >= 192 && per_cu < 6))
    return M / 256 * ((a.Cout + 95) / 96) >= 4 * num_cu ? launch_mid_cfg<T, 96, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm)
                                                        : launch_mid_cfg<T, 96, 128, 1, 4, 3, 3, 3>(a, num_cu, s, kernel_id, tm);
  const bool fits128 = (a.Cout + 127) / 128 * 2 == (a.Cout + 63) / 64, long_k = a.Cin >= 192;
  // the cheapest of the large tiles for that many items: 0 none, 1 64 x 256, 2 96 x 256, 3 128 x 256
  auto large = [&](long long items, double* cost) -> int {
    int best = 0;
    auto offer = [&](int which, int bc, double c) {
      const long long r = mid_rounds(a, items, bc, 256, 384, num_cu);
      if (r >= 2 && c * r < *cost) { *cost = c * r; best = which; }
    };
    if (a.Cin >= 96) offer(1, 64, long_k ? 1.83 : a.in_place && a.Cin <= 128 && a.Cin % 32 == 0 ? 2.05 : 1.9);
    if (long_k && !fits128 && a.Cout % 96 == 0) offer(2, 96, 2.56);
    if (a.Cin >= 128 && fits128) offer(3, 128, long_k ? 3.26 : 3.5);
    return best;
  };
  if (a.in_place && a.n_split == 0 && a.Cin == 128) {
    const long long tiles = mid_rounds(a, M / ((long long)a.Ho * a.Wo), 64, 128, 192, num_cu);
    if (tiles == 1 || tiles == 2) return launch_mid_cfg<T, 64, 128, 1, 8, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
  }
  const long long hw = (long long)a.Ho * a.Wo, now = a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n;
  if (k8 && long_k) {
    double cost = (double)mid_rounds(a, M / hw, 64, 128, 192, num_cu);
    if (!large(M / hw, &cost)) {
      // tiles whose patch fits five passes of the loader (whole images of up to 14 columns) save the sixth, which would fetch
      // nothing: 512 -> 512 on 200 x 7 x 7 51 us (56).  Same slices, so a running count may choose: 128 channels with plenty of
      // tiles after all (64 : 128 channels, 7 x 7 x 512 at 12 208 : 210, at 16 276 : 271, at 24 415 : 408, at 40 696 : 674)
      MidGeom g5{}, g6{};
      const bool five = mid_geometry(a, 64, 128, 160, &g5) && mid_geometry(a, 64, 128, 192, &g6) && g5.TH * g5.TW == g6.TH * g6.TW;
      if (five && fits128 && (double)now * hw / 128 * ((a.Cout + 63) / 64) / num_cu >= 24)
        return launch_mid_cfg<T, 128, 128, 2, 8, 2, 5, 2>(a, num_cu, s, kernel_id, tm);
      if (five) return launch_mid_cfg<T, 64, 128, 1, 8, 3, 5, 2>(a, num_cu, s, kernel_id, tm);
      return launch_mid_cfg<T, 64, 128, 1, 8, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
    }
  }
  double cost = (double)mid_rounds(a, now, 64, 128, 192, num_cu) * (long_k ? 1.08 : 1.0);
  if (cost == 0) cost = 1e30;
  switch (large(now, &cost)) {
    case 1: return launch_mid_cfg<T, 64, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
    case 2: return launch_mid_cfg<T, 96, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
    case 3: return launch_mid_cfg<T, 128, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
  }
  return launch_mid_cfg<T, 64, 128, 1, 4, 3, 3, 4>(a, num_cu, s, kernel_id, tm);
}

}  // namespace octo
