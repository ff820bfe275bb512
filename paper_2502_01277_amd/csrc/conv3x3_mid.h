// 3x3 / stride-1 / pad-1 convolution with the input patch of a tile in LDS, for tiles of 64 or 128 channels x 128 or 256 pixels.
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
//   * the barrier of a step sits before the last group of its MFMAs, with the next step's first fragments read behind it.
// Several workgroups share a compute unit, so that the prologue and epilogue of one overlap the K loop of another.
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
// still be in flight when the operands of the step after tap t must have landed: those issued at the NST - 2 taps before t.
constexpr int mid_ppt(int maxp) { return (maxp + 5) / 6; }
constexpr int mid_passes(int t, int maxp) {
  const int left = maxp - (t + 9) % 9 * mid_ppt(maxp);
  return left < 0 ? 0 : (left < mid_ppt(maxp) ? left : mid_ppt(maxp));
}
constexpr int mid_in_flight(int t, int nst, int la, int maxp) {
  int n = 0;
  for (int i = t + 2 - nst; i < t; ++i) n += la + mid_passes(i, maxp);
  return n;
}

// BC x BP: tile; WC: wavefronts along the channels (4 / WC along the pixels); KV: vectors of 16 bytes per LDS row; NST: stages
// of the weight ring; MAXP: passes of the 256 loader lanes that cover a patch buffer; MINB: workgroups per compute unit.
template <typename T, int BC, int BP, int WC, int KV, int NST, int MAXP, int MINB>
__global__ __launch_bounds__(THREADS, MINB) void conv3x3_mid_kernel(const ConvArgs a, const MidGeom gm) {
  using E = Elem<T>;
  constexpr int VN = E::N, ES = (int)sizeof(T), BK = KV * VN;
  constexpr int WP = 4 / WC, TC = BC / WC / 32, TP = BP / WP / 32;
  constexpr int RPW = 16 / KV, RP = THREADS / KV, LA = (BC + RP - 1) / RP;
  constexpr int ROW = KV * 16, STAGE = LA * RP * ROW, PATCH = MAXP * 4096;
  constexpr int KK = ES == 1 ? KV / 4 : KV / 2;          // groups of MFMAs per step
  constexpr int FV = ES == 1 ? 2 : 1;                    // vectors per operand fragment
  constexpr int ZROW = MAXP * RP - RPW;                  // last rows of a patch buffer, kept zero (the host leaves them free)
  constexpr int NTAP = 9;
  static_assert(BC % 32 == 0 && TC >= 1 && TP >= 1 && (KK == 1 || KK % 2 == 0) && NST >= 2 && NST <= 4, "tile shape");
  constexpr int OPITCH = BC * ES + 16;
  constexpr int OPER = NST * STAGE + 2 * PATCH, OSTAGE = BP * OPITCH;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[OPER > OSTAGE ? OPER : OSTAGE];
  __shared__ float sBias[BC];
  __shared__ float sScale[ES == 1 ? BC : 1];
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
  const long long w_bytes = (long long)a.w_rows * a.Kp * ES;
  const int w_len = (int)(w_bytes < BUF_MAX ? w_bytes : BUF_MAX);
  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;

  const int per_die = (n_tiles + 7) >> 3;      // see conv_mfma_kernel: one contiguous chunk of the tile list per die
  for (int t = blockIdx.x; t < per_die * 8; t += gridDim.x) {
    const int tile = (t & 7) * per_die + (t >> 3);
    if (tile >= n_tiles) continue;
    const unsigned tpx = fast_div((unsigned)tile, gm.div_tc);
    const int c0 = (int)((unsigned)tile - tpx * (unsigned)tiles_c) * BC;
    const unsigned tv = fast_div(tpx, gm.div_tx);
    const int x0 = (int)(tpx - tv * (unsigned)gm.tiles_x) * gm.TW;
    const int v0 = (int)tv * gm.TH;

    // loaders: this lane's vector of every pass of the patch (relative to the first patch row) and of the weight rows
    const long long pix0 = (long long)(v0 - 1) * W;                  // may be -W: lanes of that row are out of range
    const long long rem_bytes = (((long long)a.n * H * W - pix0) * a.x_ld - a.x_coff) * ES;
    const int p_len = (int)(rem_bytes < BUF_MAX ? rem_bytes : BUF_MAX);
    void* p_base = (void*)(xg + pix0 * a.x_ld);
    // (opaque to the compiler, which would otherwise keep the tile-independent part of every address in registers of its own)
    int poff[MAXP], woff[LA], lrow = ld_row, lpix = wp * (TP * 32) + l32;
    asm volatile("" : "+v"(lrow), "+v"(lpix));
    auto patch_offsets = [&](int channels) __attribute__((always_inline)) {      // vectors past that many channels of a slice read as zeros
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
    patch_offsets(a.Cin);
#pragma unroll
    for (int i = 0; i < LA; ++i) woff[i] = ld_row + RP * i < BC ? ((c0 + ld_row + RP * i) * a.Kp + lkv * VN) * ES : OOB;
    // byte offset inside a patch buffer of this lane's first vector, per tap and block
    int baddr[NTAP][TP];
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
        baddr[tap][j] = (in ? px : ZROW + (px & (RPW - 1))) * ROW + ((g ^ ((pos >> (RPW == 2 ? 1 : 2)) & (KV - 1))) << 4);
      }
    }

    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    __syncthreads();   // the previous tile's LDS reads are done
    if (tid < BC) sBias[tid] = a.bias[c0 + tid];
    if constexpr (ES == 1) { if (tid < BC) sScale[tid] = a.scale[c0 + tid]; }

    // weights of (slice SL, tap TAP) into ring stage ST; nothing is fetched past the last slice
    auto issue_w = [&](int sl, int tap, int st) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, sl < n_slices ? w_len : 0, BUF_FLAGS);
      const int koff = (tap * a.Cin + sl * BK) * ES;
#pragma unroll
      for (int i = 0; i < LA; ++i)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds_ring + st * STAGE + i * 4096), "v"(woff[i]), "s"(rs), "s"(koff) : "memory");
    };
    // passes of slice sl's patch
    auto issue_p = [&](int sl, int from, int count) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(p_base, 0, sl < n_slices ? p_len : 0, BUF_FLAGS);
      const int koff = sl * BK * ES;
#pragma unroll
      for (int i = 0; i < MAXP; ++i)
        if (i >= from && i < from + count)
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                       :: "s"(lds_patch + (sl & 1) * PATCH + i * 4096), "v"(poff[i]), "s"(rs), "s"(koff) : "memory");
    };
    u32x4 fa[2][TC][FV], fb[2][TP][FV];
    const int arow = (wc * (TC * 32) + l32) * ROW;
    auto frags = [&](int set, int st, const int (&ba)[TP], int pbuf, int kq) __attribute__((always_inline)) {
      const unsigned char* pa = ring + st * STAGE + arow;
      const unsigned char* pb = patch + pbuf * PATCH;
#pragma unroll
      for (int h = 0; h < FV; ++h) {
        const int v = (kq * FV + h) * 2;
#pragma unroll
        for (int i = 0; i < TC; ++i) fa[set][i][h] = *(const u32x4*)(pa + i * (32 * ROW) + (((v + g) ^ rsw) << 4));
#pragma unroll
        for (int j = 0; j < TP; ++j) fb[set][j][h] = *(const u32x4*)(pb + (ba[j] ^ (v << 4)));
      }
    };

    issue_p(0, 0, MAXP);
    constexpr int AHEAD = KK == 1 ? NST - 1 : NST;         // steps whose weights are requested up front
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) issue_w(0, d, d);
    if constexpr (KK > 1) {
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 1) * LA) : "memory");
      __builtin_amdgcn_s_barrier();
      frags(0, 0, baddr[0], 0, 0);
    }
    int rd = 0;                                // ring stage of the current step
    auto step = [&](auto tapc, int sl) __attribute__((always_inline)) {
      constexpr int TAP = decltype(tapc)::value, NEXT = (TAP + 1) % NTAP, LTAP = (TAP + NST) % NTAP;
      const int cur = NTAP % NST == 0 ? TAP % NST : rd;
      const int nxt = NTAP % NST == 0 ? NEXT % NST : (rd + 1 == NST ? 0 : rd + 1);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        if constexpr (KK == 1) {
          // a single group per step: its fragments are read here, and the loads go to the stage that the previous step has left
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(mid_in_flight(TAP, NST, LA, MAXP)) : "memory");
          __builtin_amdgcn_s_barrier();
          frags(0, cur, baddr[TAP], sl & 1, 0);
          issue_p(sl + 1, TAP * mid_ppt(MAXP), mid_passes(TAP, MAXP));
          issue_w(TAP + NST - 1 >= NTAP ? sl + 1 : sl, (TAP + NST - 1) % NTAP, NTAP % NST == 0 ? (TAP + NST - 1) % NST : (rd == 0 ? NST - 1 : rd - 1));
        } else if (kk < KK - 1) {
          frags((kk + 1) & 1, cur, baddr[TAP], sl & 1, kk + 1);
        } else {
          // this wavefront holds all it needs of the stage in registers, and the next step's operands have landed
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(mid_in_flight(TAP, NST, LA, MAXP)) : "memory");
          __builtin_amdgcn_s_barrier();
          frags(0, nxt, baddr[NEXT], TAP == NTAP - 1 ? (sl + 1) & 1 : sl & 1, 0);
          issue_p(sl + 1, TAP * mid_ppt(MAXP), mid_passes(TAP, MAXP));
          issue_w(TAP + NST >= NTAP ? sl + 1 : sl, LTAP, cur);
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
    for (int sl = 0; sl < n_slices; ++sl) {
      // the last slice, fetched from here on, may be partial: its missing channels are zeros (the weights there anything finite)
      if (sl + 2 == n_slices && a.Cin % BK) patch_offsets(a.Cin % BK);
      step(std::integral_constant<int, 0>{}, sl); step(std::integral_constant<int, 1>{}, sl); step(std::integral_constant<int, 2>{}, sl);
      step(std::integral_constant<int, 3>{}, sl); step(std::integral_constant<int, 4>{}, sl); step(std::integral_constant<int, 5>{}, sl);
      step(std::integral_constant<int, 6>{}, sl); step(std::integral_constant<int, 7>{}, sl); step(std::integral_constant<int, 8>{}, sl);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // loads issued past the last step wrote zeros into the ring
    __syncthreads();

    // epilogue: through LDS as [pixel][channel], so that residual and output move in 16-byte pieces of whole rows
    constexpr int VPR = BC / VN, PPP = THREADS / VPR;      // vectors per pixel, pixels per pass
    constexpr int NPASS = (BP + PPP - 1) / PPP;
    const int ov = tid % VPR, opr = tid / VPR;
    const int oc = c0 + ov * VN;
    auto out_pixel = [&](int pl) -> int {                  // pixel of the batch, or -1
      const int ty = (int)fast_div((unsigned)pl, gm.div_tw), tx = pl - ty * gm.TW;
      return ty < gm.TH && v0 + ty < n_rows && x0 + tx < W && oc < a.Cout && (THREADS % VPR == 0 || opr < PPP) ? (v0 + ty) * W + x0 + tx : -1;
    };
    const bool whole = oc + VN <= a.Cout;
    const bool vec_out = whole && ((a.y_ld | a.y_coff) % VN) == 0 && ((uintptr_t)a.y & 15) == 0;
    const bool vec_res = whole && ((a.res_ld | a.res_coff) % VN) == 0 && ((uintptr_t)a.res & 15) == 0;
    if (a.res) {
#pragma unroll
      for (int ps = 0; ps < NPASS; ++ps) {
        const int pl = ps * PPP + opr, p = out_pixel(pl);
        if (p < 0) continue;
        const T* r = (const T*)a.res + (size_t)p * a.res_ld + a.res_coff + oc;
        T* o = (T*)(smem + pl * OPITCH + ov * 16);
        if (vec_res) *(u32x4*)o = *(const u32x4*)r;
        else
#pragma unroll 1
          for (int e = 0; e < VN && oc + e < a.Cout; ++e) o[e] = r[e];
      }
      __syncthreads();
    }
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
    constexpr int RES = decltype(res_c)::value;
    constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      const int pl = wp * (BP / WP) + j * 32 + l32;
#pragma unroll
      for (int i = 0; i < TC; ++i) {
        const int cblk = wc * (BC / WC) + i * 32 + g * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          T* o = (T*)(smem + pl * OPITCH) + cblk + q * 8;
          floatx4 rv = floatx4{0.f, 0.f, 0.f, 0.f}, v;
          if (RES != OCTO_RES_NONE) rv = load4<T>(o);
          const floatx4 b4 = *(const floatx4*)&sBias[cblk + q * 8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = ES == 1 ? acc[i][j][q * 4 + e] * sScale[cblk + q * 8 + e] : acc[i][j][q * 4 + e];
            if (ES == 1) rv[e] *= a.res_scale;
          }
          v = finish4<RES, SILU>(v, b4, rv, act_lo);
          if constexpr (ES == 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= a.y_inv_scale;
          }
          store4<T>(o, v);
        }
      }
    }
    });
    __syncthreads();
#pragma unroll
    for (int ps = 0; ps < NPASS; ++ps) {
      const int pl = ps * PPP + opr, p = out_pixel(pl);
      if (p < 0) continue;
      T* y = (T*)a.y + (size_t)p * a.y_ld + a.y_coff + oc;
      const T* o = (const T*)(smem + pl * OPITCH + ov * 16);
      if (vec_out) *(u32x4*)y = *(const u32x4*)o;
      else
#pragma unroll 1
        for (int e = 0; e < VN && oc + e < a.Cout; ++e) y[e] = o[e];
    }
  }
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
  if ((long long)(gm.TH + 2) * a.W * a.x_ld * (int)sizeof(T) > 0x7FFFFFF0LL) return hipErrorNotSupported;     // 32-bit offsets inside a patch
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

// Tile of a 16-bit layer with M output pixels, or hipErrorNotSupported where the split-K or general kernel is the better one
// (measured on MI355X, bf16, us; layers of H x W x C -> C, by the number of images).  per_cu: 64 x 128 tiles per compute unit.
//   * up to 64 channels and many pixels: conv3x3_stream_kernel;
//   * below 0.35 the split-K kernel spreads the K loop of the few tiles over more wavefronts.  Against 64 x 64 tiles: 14 x 14 x 256 at
//     0.22 9.0 : 9.5, at 0.36 11.0 : 9.7; 20 x 20 x 64 at 0.24 5.7 : 6.1, at 0.34 7.2 : 6.2; 40 x 40 x 128 at 0.20 6.7 : 7.2, at 0.29
//     8.4 : 7.3; the long reduction of 7 x 7 x 512 turns later, at 0.43 16.5 : 19.2, at 0.60 24.7 : 19.9;
//   * 64 x 64 tiles up to 0.8.  Against 64 x 128: 14 x 14 x 256 at 0.72 12.0 : 12.3, at 0.96 12.8 : 12.8, at 1.2 18.9 : 17.2;
//     7 x 7 x 512 at 0.72 20.4 : 20.8, at 0.96 23.1 : 21.7;
//   * reductions over at least 192 channels with fewer than six tiles per compute unit are paced by the operand fetch: slices of
//     128 bytes (whole cache lines), and 64 x 64 tiles while those leave compute units idle.  256 -> 256 on 63 x 14 x 14: 19 us
//     on 64 x 128 (general kernel 27), 512 -> 512 on 63 x 7 x 7: 22 us on 64 x 64 (split-K 29);
//   * otherwise slices of 64 bytes, half the LDS and up to four workgroups per compute unit, which hide each other's prologue
//     and epilogue: 64 -> 64 with residual on 64 x 80 x 80 46 us (general kernel 74).  Tiles of 256 pixels fetch the weights half
//     as often and pay once there are plenty of them: 384 -> 384 on 32 x 40 x 40 116 us (64 x 128: 136, general kernel 156).
//     From 96 channels that is at 12 (64 x 128 : 64 x 256): 28 x 28 x 128 at 8 43.7 : 44.6, at 12 61.8 : 60.3, at 20 99.7 : 93.9;
//     56 x 56 x 96 -> 64 at 8.6 37.7 : 39.4, at 19 77.9 : 74.9.  From 192 channels it is a matter of rounds: 14 x 14 x 256, slices of 128
//     bytes : 64 x 256, at 2.0 27.3 : 28.9, at 3.8 37.1 : 35.2, at 5.0 52.4 : 47.5, at 6.0 59.2 : 61.5, at 7.2 70.2 : 63.1, at 14
//     128 : 127; the line at 6 is right on both sides of itself and 10 % off in the last third of a round below it;
//   * tiles of 32 channels for layers with no more: 32 -> 32 with residual on 16 x 160 x 160 24 us (33).  From 0.8: 80 x 80 x 32 at 0.59 5.8
//     on either, at 0.78 5.7 (general kernel 7.0);
//   * tiles of 96 channels where those of 64 would pad: 96 -> 96 on 32 x 160 x 160 156 us (187), of 256 pixels from four per compute
//     unit on (80 x 80 x 96, 128 : 256 pixels, 15.2 : 17.9 for 10 images, 36.6 : 37.4 for 30, 46.9 : 46.3 for 40, 89.4 : 86.2 for 80).
// The two slice widths sum in different orders; M is taken for a count that stays the same from batch to batch (a.n_split), and
// so do the results.
template <typename T>
hipError_t launch_mid(const ConvArgs& a, long long M, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (!mid_fits(a)) return hipErrorNotSupported;
  const hipError_t es = launch_stream3<T>(a, M, num_cu, s, kernel_id, tm);
  if (es != hipErrorNotSupported) return es;
  const int pad32 = (a.Cin + 31) / 32 * 32, pad64 = (a.Cin + 63) / 64 * 64;
  if (a.Cin * 4 < pad32 * 3) return hipErrorNotSupported;       // more than a quarter of the MFMAs would be padding
  if (a.Cout <= 32) return (double)M / 128 < 0.8 * num_cu ? hipErrorNotSupported : launch_mid_cfg<T, 32, 128, 1, 4, 3, 3, 4>(a, num_cu, s, kernel_id, tm);
  const double per_cu = (double)M / 128 * ((a.Cout + 63) / 64) / num_cu;
  if (per_cu < 0.35) return hipErrorNotSupported;
  if (pad32 == pad64) {
    if (per_cu < 0.8) return launch_mid_cfg<T, 64, 64, 2, 8, 3, 4, 2>(a, num_cu, s, kernel_id, tm);
    if (a.Cin >= 192 && per_cu < 6) {
      // tiles whose patch fits five passes of the loader (whole images of up to 14 columns) save the sixth, which would fetch
      // nothing: 512 -> 512 on 200 x 7 x 7 51 us (56).  Same slices, so a running count may choose: 128 channels with plenty of
      // tiles after all (64 : 128 channels, 7 x 7 x 512 at 18 300 : 313 us, at 24 397 : 389, at 30 497 : 502, at 48 814 : 780;
      // 14 x 14 x 256 at 24 212 : 206, at 36 328 : 312)
      MidGeom g5{}, g6{};
      const bool five = mid_geometry(a, 64, 128, 160, &g5) && mid_geometry(a, 64, 128, 192, &g6) && g5.TH * g5.TW == g6.TH * g6.TW;
      const double now = (double)(a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * a.Ho * a.Wo / 128 * ((a.Cout + 63) / 64) / num_cu;
      if (five && now >= 24 && a.Cout % 128 == 0) return launch_mid_cfg<T, 128, 128, 2, 8, 2, 5, 2>(a, num_cu, s, kernel_id, tm);
      if (five) return launch_mid_cfg<T, 64, 128, 1, 8, 3, 5, 2>(a, num_cu, s, kernel_id, tm);
      return launch_mid_cfg<T, 64, 128, 1, 8, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
    }
  }
  if ((a.Cout + 95) / 96 * 96 < (a.Cout + 63) / 64 * 64)
    return M / 256 * ((a.Cout + 95) / 96) >= 4 * num_cu ? launch_mid_cfg<T, 96, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm)
                                                        : launch_mid_cfg<T, 96, 128, 1, 4, 3, 3, 3>(a, num_cu, s, kernel_id, tm);
  if (a.Cin >= 192 || (a.Cin >= 96 && per_cu >= 12)) return launch_mid_cfg<T, 64, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm);
  return launch_mid_cfg<T, 64, 128, 1, 4, 3, 3, 4>(a, num_cu, s, kernel_id, tm);
}

}  // namespace octo
