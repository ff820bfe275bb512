// 3x3 / stride-1 / pad-1 convolution with at most 64 input and 64 output channels on many pixels: resident weights, streamed patches.
//
// Such layers (the 56 x 56 stage of a classifier, the wide early stages of a detector) have so short a reduction that a tile of
// conv3x3_mid_kernel spends its time on fetching weights - 73 KB for 64 -> 64 channels, more than the patch and the output
// together - and on vector arithmetic around the MFMAs, most of it addresses.  Their floor is the memory traffic of the
// activations.  Here
//   * every wavefront keeps the weights of its 32 output channels in registers (36 for every 16 input channels), so a workgroup
//     strides over tiles of up to 256 / WC pixels without touching weights again, and LDS is read for the pixel operand alone;
//   * tiles divide the image, with a one-pixel border of the patch in LDS that reads as zeros outside: every LDS and memory
//     offset of a lane is then the same for all tiles, and a pass of the loader costs three vector instructions;
//   * patch and residual of the next tile stream into LDS while a tile is multiplied; there is one barrier per tile;
//   * weight rows are taken in an order that leaves 16 consecutive channels of a pixel in one lane, so that residual and output
//     move in 16-byte pieces without a detour through LDS.
// Patch rows are swizzled as in conv3x3_mid_kernel.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace octo {

struct Stream3Geom {
  int TW, TH, tiles_x, tiles_y;            // output tile; tiles per image
  FastDiv div_tw, div_pw, div_tx, div_ty;  // divisions by TW, TW + 2, tiles_x, tiles_y
};

// WC: 32-channel blocks of the output, one per wavefront of a group; 4 / WC groups of wavefronts of 64 pixels each; KC: 16-channel groups
// of the input; KV: 16-byte vectors per patch row; MAXP: passes of the loader lanes that cover a patch; PD: depth of the ring of
// pixel fragments.
template <typename T, int WC, int KC, int KV, int MAXP, int PD, int MINB>
__global__ __launch_bounds__(THREADS, MINB) void conv3x3_stream_kernel(const ConvKernelArgs a, const Stream3Geom gm) {
  using E = Elem<T>;
  constexpr int VN = 8, ES = 2, TP = 2, NTAP = 9, NT = THREADS;
  constexpr int RPW = 16 / KV, RP = NT / KV, ROW = KV * 16, PATCH = MAXP * NT * 16;
  static_assert(sizeof(T) == 2 && KC * 2 <= KV && MAXP <= 8, "16-bit types, a patch row holds all input channels");
  __shared__ __attribute__((aligned(1024))) unsigned char patch[2 * PATCH];
  __shared__ __attribute__((aligned(1024))) unsigned char sRes[4 * 4096];     // residual: 4 KB per wavefront
  __shared__ __attribute__((aligned(16))) float sBias[WC * 32];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wc = wave % WC, wp = wave / WC;
  const int l32 = lane & 31, g = lane >> 5;
  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int W = a.W, PW = gm.TW + 2;
  const int n_tiles = n_items * gm.tiles_y * gm.tiles_x;
  const unsigned lds_patch = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)patch + (unsigned)wave * 1024u));
  const unsigned lds_res = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)sRes + (unsigned)wave * 4096u));
  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;

  const int per_die = (n_tiles + 7) >> 3;      // one contiguous chunk of the tile list per die, as in conv_mfma_kernel
  auto next_valid = [&](int t) -> int {
    while (t < per_die * 8 && (t & 7) * per_die + (t >> 3) >= n_tiles) t += gridDim.x;
    return t;
  };
  // first pixel of tile t (in pixels of the batch) and the image sides it touches: 1 top, 2 bottom, 4 left, 8 right
  auto origin = [&](int t, long long& pix0, unsigned& sides) __attribute__((always_inline)) {
    const unsigned tile = (unsigned)((t & 7) * per_die + (t >> 3)), row = fast_div(tile, gm.div_tx), img = fast_div(row, gm.div_ty);
    const int tx = (int)(tile - row * (unsigned)gm.tiles_x), ty = (int)(row - img * (unsigned)gm.tiles_y);
    pix0 = ((long long)img * a.H + ty * gm.TH) * W + tx * gm.TW;
    sides = (ty == 0 ? 1u : 0u) | (ty == gm.tiles_y - 1 ? 2u : 0u) | (tx == 0 ? 4u : 0u) | (tx == gm.tiles_x - 1 ? 8u : 0u);
  };

  // loader: byte offset of this lane's vector of every pass from the patch origin, and the patch sides its pixel lies on
  int poff[MAXP];
  unsigned pside = 0;
#pragma unroll
  for (int i = 0; i < MAXP; ++i) {
    const int pp = i * RP + tid / KV;
    const int pr = (int)fast_div((unsigned)pp, gm.div_pw), pc = pp - pr * PW;
    const int vec = (tid % KV) ^ ((int)((unsigned)(pr * gm.TW + pc) / RPW) % KV);
    poff[i] = pr < gm.TH + 2 && vec * VN < a.Cin ? ((pr * W + pc) * a.x_ld + vec * VN) * ES : OOB;
    pside |= ((pr == 0 ? 1u : 0u) | (pr == gm.TH + 1 ? 2u : 0u) | (pc == 0 ? 4u : 0u) | (pc == PW - 1 ? 8u : 0u)) << (4 * i);
  }
  // consumer: LDS offset of this lane's first vector per tap and block, output and residual offsets from the tile's first pixel
  const int cl = wc * 32 + g * 16;         // this lane's 16 channels
  int baddr[NTAP][TP], yoff[TP], roff[TP];
#pragma unroll
  for (int j = 0; j < TP; ++j) {
    const int q = wp * (TP * 32) + j * 32 + l32;
    const int ty = (int)fast_div((unsigned)q, gm.div_tw), tx = q - ty * gm.TW;
    const bool ok = ty < gm.TH;
    yoff[j] = ok && cl < a.Cout ? ((ty * W + tx) * a.y_ld + cl) * ES : OOB;
    roff[j] = ok && cl < a.Cout ? ((ty * W + tx) * a.res_ld + cl) * ES : OOB;
#pragma unroll
    for (int tap = 0; tap < NTAP; ++tap) {
      const int r = tap / 3, s = tap % 3;
      const int px = ok ? (ty + r) * PW + tx + s : 0, pos = ok ? (ty + r) * gm.TW + tx + s : 0;
      baddr[tap][j] = px * ROW + ((g ^ ((pos / RPW) & (KV - 1))) << 4);
    }
  }
  const bool half = cl + 8 >= a.Cout;      // only the first 8 of this lane's channels exist
  // patch of tile t into buffer buf; nothing is fetched past the last tile
  auto load_patch = [&](int t, int buf) __attribute__((always_inline)) {
    if (t >= per_die * 8) return;
    long long pix0;
    unsigned sides;
    origin(t, pix0, sides);
    pix0 -= W + 1;
    const long long rem_bytes = (((long long)a.n * a.H * W - pix0) * a.x_ld - a.x_coff) * ES;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)((const T*)a.x + a.x_coff + pix0 * a.x_ld), 0, (int)(rem_bytes < BUF_MAX ? rem_bytes : BUF_MAX), BUF_FLAGS);
#pragma unroll
    for (int i = 0; i < MAXP; ++i) {
      const int off = pside & (sides << (4 * i)) ? OOB : poff[i];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(lds_patch + buf * PATCH + i * (NT * 16)), "v"(off), "s"(rs) : "memory");
    }
  };
  // every lane's own four residual vectors of tile t, in the order the epilogue takes them
  auto load_res = [&](int t) __attribute__((always_inline)) {
    if (!a.res) return;
    long long pix0;
    unsigned sides;
    origin(t, pix0, sides);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)((const T*)a.res + a.res_coff + pix0 * a.res_ld), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int off = h && half ? OOB : roff[j] + h * 16;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(lds_res + (j * 2 + h) * 1024), "v"(off), "s"(rs) : "memory");
      }
  };

  int t = next_valid(blockIdx.x);
  if (t >= per_die * 8) return;
  load_patch(t, 0);
  if (tid < WC * 32) sBias[tid] = a.bias[tid];
  // weights: row m of a 32-row block is channel 16 ((m / 4) % 2) + 4 (m / 8) + m % 4, see the epilogue
  u32x4 wr[NTAP * KC];
  {
    const T* w = (const T*)a.w + (size_t)(wc * 32 + 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3)) * a.Kp + g * VN;
#pragma unroll
    for (int k = 0; k < NTAP * KC; ++k) wr[k] = *(const u32x4*)(w + (k / KC) * a.Cin + (k % KC) * 16);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  int tn = next_valid(t + gridDim.x), buf = 0;
  load_patch(tn, 1);
  load_res(t);
  for (;;) {
    // opaque: the exclusive-or of every group of channels would otherwise be kept in a register of its own
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
      for (int tap = 0; tap < NTAP; ++tap) asm volatile("" : "+v"(baddr[tap][j]));
    floatx16 acc[TP];
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
    const unsigned char* pb = patch + buf * PATCH;
    u32x4 fb[PD][TP];
    auto read = [&](int k) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < TP; ++j) fb[k % PD][j] = *(const u32x4*)(pb + (baddr[k / KC][j] ^ ((k % KC) << 5)));
    };
#pragma unroll
    for (int k = 0; k < PD - 1; ++k) read(k);
#pragma unroll
    for (int k = 0; k < NTAP * KC; ++k) {
      if (k + PD - 1 < NTAP * KC) read(k + PD - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TP; ++j) acc[j] = E::mfma(wr[k], fb[k % PD][j], acc[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next tile's patch (and this tile's residual) have landed, and everyone is done reading this tile's patch
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    const int t2 = tn < per_die * 8 ? next_valid(tn + gridDim.x) : tn;
    load_patch(t2, buf);

    // epilogue: lane (l32, g) holds channels 16 g + 4 q + e of each 32-channel block
    long long pix0;
    unsigned sides;
    origin(t, pix0, sides);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y + a.y_coff + pix0 * a.y_ld), 0, (int)BUF_MAX, BUF_FLAGS);
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
    constexpr int RES = decltype(res_c)::value;
    constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
    for (int j = 0; j < TP; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        typedef T t4 __attribute__((ext_vector_type(4)));
        u32x4 out;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          floatx4 v, r4 = floatx4{0.f, 0.f, 0.f, 0.f};
          if (RES != OCTO_RES_NONE) r4 = load4<T>((const T*)(sRes + wave * 4096 + (j * 2 + h) * 1024 + lane * 16) + q * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[j][(h * 2 + q) * 4 + e];
          v = finish4<RES, SILU>(v, *(const floatx4*)&sBias[cl + h * 8 + q * 4], r4, act_lo);
          const t4 o = {(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
          const u32x2 ob = __builtin_bit_cast(u32x2, o);
          out[2 * q] = ob[0]; out[2 * q + 1] = ob[1];
        }
        __builtin_amdgcn_raw_buffer_store_b128(out, ry, h && half ? OOB : yoff[j] + h * 16, 0, 0);
      }
    });
    if (tn >= per_die * 8) break;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // this wavefront's residual has been read: its place is free
    t = tn; tn = t2; buf ^= 1;
    load_res(t);
  }
}

// The tile of up to BP pixels that divides an H x W image, has its patch in `rows` LDS rows and fills the most of BP (ties: the smallest
// patch); false if none fills 3/4.
inline bool stream3_geometry(int H, int W, int BP, int rows, Stream3Geom* gm) {
  int best = 0, best_patch = 0;
  for (int tw = std::min(W, 64); tw >= 4; --tw) {
    if (W % tw) continue;
    for (int th = std::min(H, BP / tw); th >= 1; --th) {
      const int px = th * tw, patch = (th + 2) * (tw + 2);
      if (H % th || patch > rows || px < best || (px == best && patch >= best_patch)) continue;
      best = px; best_patch = patch;
      gm->TW = tw; gm->TH = th;
    }
  }
  if (best * 4 < BP * 3) return false;
  gm->tiles_x = W / gm->TW; gm->tiles_y = H / gm->TH;
  gm->div_tw = make_fastdiv((unsigned)gm->TW); gm->div_pw = make_fastdiv((unsigned)gm->TW + 2u);
  gm->div_tx = make_fastdiv((unsigned)gm->tiles_x); gm->div_ty = make_fastdiv((unsigned)gm->tiles_y);
  return true;
}

template <typename T, int WC, int KC, int KV, int MAXP, int PD, int MINB>
hipError_t launch_stream3_cfg(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  Stream3Geom gm{};
  if (!stream3_geometry(a.H, a.W, 256 / WC, MAXP * (THREADS / KV), &gm)) return hipErrorNotSupported;
  const long long tiles = (long long)a.n * gm.tiles_y * gm.tiles_x;
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x3FFFFFF0LL) return hipErrorNotSupported;
  // 32-bit offsets inside a tile
  if ((long long)(gm.TH + 2) * a.W * std::max(a.x_ld, std::max(a.y_ld, a.res ? a.res_ld : 0)) * 2 > 0x7FFFFFF0LL) return hipErrorNotSupported;
  if (kernel_id) *kernel_id = stream3_kernel_id(WC, KC, KV, a.Cin);
  long long grid = (tiles + 7) / 8 * 8;
  const long long cap = ((long long)num_cu * MINB + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv3x3_stream_kernel<T, WC, KC, KV, MAXP, PD, MINB>), dim3((unsigned)grid), dim3(THREADS), 0, s, tm.start, tm.stop, 0, a, gm);
  else
    hipLaunchKernelGGL((conv3x3_stream_kernel<T, WC, KC, KV, MAXP, PD, MINB>), dim3((unsigned)grid), dim3(THREADS), 0, s, a, gm);
  return hipGetLastError();
}

// Layers of up to 64 input and output channels whose tiles give every workgroup enough to do: loading 73 KB of weights into
// registers pays after three tiles of a workgroup (64 -> 64 on 32 x 80 x 80: 28 us, 29 on conv3x3_mid_kernel; at 16 images
// 21 against 18), with up to 32 channels and a quarter of the weights after one and a half.  64 -> 64 with residual on
// 600 x 56 x 56: 179 us, 4.1 TB/s (conv3x3_mid_kernel 248); 48 -> 48 with residual on 32 x 320 x 320: 237 us (395, general kernel
// 440); 32 -> 32 with residual on 64 x 160 x 160: 64 us, 4.9 TB/s (109, 117 on the patch kernel before it).
// In its place in a cascade, where the first pixels come late, 64 -> 64 turns later (here : conv3x3_mid_kernel): without residual 8 x 160 x 160 28.0 : 24.8,
// 96 x 56 x 56 28.0 : 23.7, 192 x 64 x 32 29.2 : 28.0, 16 x 160 x 160 41.2 : 40.5, 256 x 56 x 56 67 : 76; with residual 96 x 56 x 56 28.4 : 27.9, 128 x 56 x 56
// 37.7 : 41.3.  Over 120 layers of nine maps, 56 and 64 channels into 40 and 64, by tiles of 128 pixels per compute unit, of the other's time: without residual at
// 8 1.03 .. 1.2, at 11 0.97 .. 1.14, at 12.5 0.92 .. 1.09, at 16 0.88 .. 1.05; with residual at 8 0.99 .. 1.07, at 9.5 0.97 .. 1.08, at 11 0.87 .. 1.01, at 14 0.80
// .. 0.93.
template <typename T>
hipError_t launch_stream3(const ConvArgs& a, long long M, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (a.Cin < 24 || a.Cin > 64 || a.Cout > 64 || ((a.Cout | a.y_ld | a.y_coff) & 7) || ((uintptr_t)a.y & 15) ||
      (a.res && (((a.res_ld | a.res_coff) & 7) || ((uintptr_t)a.res & 15)))) return hipErrorNotSupported;
  const bool narrow = a.Cout <= 32;
  if (narrow && a.Cin > 32) return hipErrorNotSupported;
  if (M < (long long)(narrow ? 256 * 3 : 128 * (a.Cin <= 32 ? 3 : !a.in_place || a.Cin <= 48 ? 6 : a.res ? 10 : 13)) * num_cu) return hipErrorNotSupported;
  if (narrow) return launch_stream3_cfg<T, 1, 2, 4, 6, 3, 2>(a, num_cu, s, kernel_id, tm);
  if (a.Cin <= 32) return launch_stream3_cfg<T, 2, 2, 4, 3, 3, 3>(a, num_cu, s, kernel_id, tm);
  if (a.Cin <= 48) return launch_stream3_cfg<T, 2, 3, 8, 6, 4, 2>(a, num_cu, s, kernel_id, tm);
  return launch_stream3_cfg<T, 2, 4, 8, 6, 3, 2>(a, num_cu, s, kernel_id, tm);
}

}  // namespace octo
