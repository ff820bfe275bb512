// 3x3 / pad-1 convolution of stride 1 or 2 for launches of about one round of workgroups: the input patch of a tile, all of its channels, is held in LDS, and the
// wavefronts of a workgroup share the reduction.
//
// In such a launch a workgroup runs alone or with one other on its compute unit, and its time is a chain of waits: the kernels that took these layers fetch their operands
// K step by K step (64 x 64 tiles of 256 -> 256: 36 steps with a wait and a barrier each, 16 KB of operands per 8 MFLOP), the patch kernel two slices of the patch at a time.  Here
//   * the whole patch is asked for at once, a tile has one wait for it and one barrier before the K loop, and none in it;
//   * weights come straight from the L2 into registers, in an order in which an instruction reads 1 KB in a row (held_weight_bytes; a copy that a model makes when it is
//     created), nine taps ahead: by the time a group of 16 input channels is done the next one's weights have come;
//   * four wavefronts share K (two, and two halves of the pixels, in 64 x 128 tiles): every one reads its own quarter of the weights, so that no byte is
//     fetched twice by a workgroup, and takes 64 x 32 or 64 x 64 results of it, half an LDS read per matrix instruction.  Partial sums meet in LDS, in fp32.
// A tile is TH x TW output pixels of the image stack (see conv3x3_mid.h), its patch in slices of 64 channels; pixel p keeps vector v of a slice in slot
// v ^ (p / 2) % 8, p counted without the halo columns at stride 1; taps outside the image read a row of zeros.
// What bounds it: start, first trip to memory and drain (about 4 us), then the time that loads take from the L2: every pixel tile reads its weights once, with the patch some 16 bytes per clock and
// compute unit (counters; a stream of loads alone reaches 54).  Wavefronts wait in 27 - 56 % of their cycles, the matrix pipe is busy in 9 - 32 % of a launch.  Before (the
// fastest kernel that could take the layer) and after, us, in place in a model: 512 -> 512 on 11 x 7 x 7 14.3 -> 9.6, on 63 x 7 x 7 26.5 -> 20.0 (735 TFLOP/s); 256 -> 256 on
// 4 x 20 x 20 12.1 -> 7.1, on 8 x 20 x 20 15.6 -> 9.0, on 11 x 14 x 14 10.3 -> 7.8; 384 -> 384 on 40 x 40 19.7 -> 11.5; 128 -> 128 on 40 x 40 5.6 -> 5.1, on 8 x 40 x 40 9.6 ->
// 8.3; stride 2: 256 -> 512 on 15 x 14 x 14 9.2 -> 7.3, 256 -> 256 on 8 x 40 x 40 14.5 -> 9.9.
// Measured and left out: eight wavefronts sharing K (0 - 2 us slower but for 512 channels on less than a tile per unit), 64 x 128 tiles of one wavefront per SIMD with 64 x 128 results
// each (15 - 60 % slower: nothing overlaps its waits), 32 x 64 tiles, and the 1x1 layer in front of a bottleneck's 3x3 layer computed on the patch in the same launch: bit-identical and
// one launch less, but every workgroup repeats it for its halo and channel tile, and an activation per value costs 50 cycles there (64 -> 64 -> 64 on 80 x 80 7.2 : 4.0 + 4.4, 128 on 40 x
// 40 9.7 : 4.1 + 5.3, 256 on 20 x 20 16.8 : 4.1 + 6.5; the detector of one frame 8 us slower with it).
// vmcnt bookkeeping: the patch loads are older than the first nine taps' weights, 9 TC loads, so that waiting for all but those waits for the patch.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include "conv3x3_held_choice.h"
#include <hip/hip_ext.h>

namespace octo {

// What the kernel reads.  Pointers are to the first channel of the first pixel.
struct HeldArgs {
  const char* x; const char* w; const float* bias; char* y;
  const int* n_dyn; const char* res;
  int n, H, W, Ho, Wo, C;
  int x_pitch, y_pitch, res_pitch;         // bytes of a pixel
  int TH, TW, PW, PH, halo, tiles_x, rows; // see HeldGeom
  int tiles_c, grid, c_outer, act, res_mode;
  FastDiv div_tw, div_pw, div_ho, div_tx, div_tc, div_th;
};

// floor(n / d) without a branch: for d of at least 2, and for any (the multiplier of 1 is zero)
__device__ __forceinline__ int held_div(unsigned n, const FastDiv& f) { return (int)(__umulhi(n, f.mul) >> f.shift); }
__device__ __forceinline__ int held_div1(unsigned n, const FastDiv& f) { return (int)((__umulhi(n, f.mul) >> f.shift) | (n & (0u - (unsigned)f.is_one))); }

// A wavefront: TC x TP blocks of 32 channels x 32 pixels.  Of the four, KS share the reduction of a tile's part, 4 / KS the tile's pixels.  S: stride.
template <typename T, int TC, int TP, int KS, int S>
__global__ __launch_bounds__(256, 2) void conv3x3_held_kernel(const HeldArgs a) {
  using E = Elem<T>;
  constexpr int BC = 32 * TC, B = TC * TP;
  constexpr int QW = 4 * B / KS, NV = QW / 2;              // quads of 4 channels that a wavefront finishes
  static_assert(sizeof(T) == 2 && QW >= 2 && QW % 2 == 0, "tile shape");
  extern __shared__ __attribute__((aligned(1024))) unsigned char held_smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = wave % KS, wp = wave / KS, l32 = lane & 31, g = lane >> 5;
  asm volatile("" :: "s"(a.x), "s"(a.w), "s"(a.bias), "s"(a.y), "s"(a.res), "s"(a.C), "s"(a.x_pitch), "s"(a.TH), "s"(a.tiles_c));
  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int n_rows = n_items * a.Ho;                       // output rows of the image stack
  const int tiles_s = held_div1((unsigned)(n_rows + a.TH - 1), a.div_th) * a.tiles_x, n_tiles = tiles_s * a.tiles_c, per_die = (n_tiles + 7) >> 3;
  const int SL = a.rows * 128, ZROW = a.rows - 2;
  const int n16 = a.C >> 4, per_wave = n16 / KS, slices = a.C >> 6;
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)held_smem + (unsigned)wave * 1024u));

  for (int t = blockIdx.x; t < per_die * 8; t += a.grid) {
    const int tile = (t & 7) * per_die + (t >> 3);       // contiguous chunk of the tile list per die, see conv_mfma_kernel
    if (tile >= n_tiles) continue;
    int tc, ts;
    if (!a.c_outer) { ts = held_div1((unsigned)tile, a.div_tc); tc = tile - ts * a.tiles_c; }
    else { int d = tiles_s; asm volatile("" : "+s"(d)); tc = (int)((unsigned)tile / (unsigned)d); ts = tile - tc * tiles_s; }
    const int tv = held_div1((unsigned)ts, a.div_tx);
    const int c0 = tc * BC, x0 = (ts - tv * a.tiles_x) * a.TW, v0 = tv * a.TH;

    // this wavefront's part of the results: QW of the quads of 4 channels of its pixels' part of the tile, in one or more 32 x 32 blocks
    const int q0 = kq * QW;
    int yo[(QW + 3) / 4], ro[(QW + 3) / 4];              // byte offset from the tile's first pixel, per block
    const long long pix0 = (long long)v0 * a.Wo + x0;
    auto channel = [&](int k) __attribute__((always_inline)) { return c0 + ((q0 + k) >> 2) / TP * 32 + g * 16 + ((q0 + k) & 3) * 4; };     // of quad k
#pragma unroll
    for (int k = 0; k < QW; k += 4) {
      const int q = (wp * TP + ((q0 + k) >> 2) % TP) * 32 + l32, ty = held_div((unsigned)q, a.div_tw), tx = q - ty * a.TW;
      const bool in = ty < a.TH && v0 + ty < n_rows && x0 + tx < a.Wo;
      yo[k / 4] = in ? (ty * a.Wo + tx) * a.y_pitch : OOB;
      ro[k / 4] = in ? (ty * a.Wo + tx) * a.res_pitch : OOB;
    }
    u32x4 rv[NV];
    if (a.res) {                                         // asked for first, so that it has landed with the patch
      const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)(a.res + pix0 * a.res_pitch), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
      for (int k = 0; k < NV; ++k) rv[k] = __builtin_amdgcn_raw_buffer_load_b128(rr, ro[k / 2] + channel(2 * k) * 2, 0, 0);
    }

    // patch: lane t of the workgroup fills slot t % 8 of row t / 8 of a pass
    {
      const long long p0 = (long long)(S * v0 - 1) * a.W;            // may be -W: lanes of that row are out of range
      const long long rem = ((long long)a.n * a.H * a.W - p0) * a.x_pitch;
      const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)(a.x + p0 * a.x_pitch), 0, (int)(rem < BUF_MAX ? rem : BUF_MAX), BUF_FLAGS);
      for (int r0 = 0; r0 < a.rows; r0 += 32) {
        const int pp = r0 + (tid >> 3), pr = held_div((unsigned)pp, a.div_pw), pc = pp - pr * a.PW;
        const int v = S * v0 - 1 + pr, x = S * x0 - a.halo + pc;
        const int vec = (tid & 7) ^ (((S == 1 ? pr * a.TW + pc : pp) >> 1) & 7);
        const bool ok = pr < a.PH && (unsigned)v < (unsigned)(n_items * a.H) && (unsigned)x < (unsigned)a.W;
        const int po = ok ? (pr * a.W + x) * a.x_pitch + vec * 16 : OOB;
        for (int sl = 0; sl < slices; ++sl)
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                       :: "s"(lds0 + sl * SL + r0 * 128), "v"(po), "s"(rx), "s"(sl * 128) : "memory");
      }
    }
    // weights: for every block of 32 channels, group of 16 input channels and tap the 1 KB that a wavefront's instruction takes
    const int wblk = n16 * 9 * 1024;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)(a.w + ((size_t)tc * TC * n16 + kq * per_wave) * 9 * 1024), 0,
                                                                        (a.tiles_c - tc) * TC * wblk - kq * per_wave * 9 * 1024, BUF_FLAGS);
    u32x4 ring[9][TC];
    auto load_w = [&](int c, int tap) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TC; ++i) ring[tap][i] = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16, (c * 9 + tap) * 1024 + i * wblk, 0);
    };
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) load_w(0, tap);

    // byte offset inside a slice of the patch of this lane's first vector, per tap and block; taps outside the image read a row of zeros
    int baddr[9][TP];
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      const int q = (wp * TP + j) * 32 + l32;
      const int ty = held_div((unsigned)q, a.div_tw), tx = q - ty * a.TW;
      const int v = v0 + ty, x = S * (x0 + tx);
      const int yy = S * (v - held_div1((unsigned)v, a.div_ho) * a.Ho);
      const bool ok = ty < a.TH && v < n_rows && x0 + tx < a.Wo;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int r = tap / 3, s = tap % 3 - 1;
        const bool in = ok && (unsigned)(yy + r - 1) < (unsigned)a.H && (unsigned)(x + s) < (unsigned)a.W;
        const int px = (S * ty + r) * a.PW + S * tx + s + a.halo, pos = S == 1 ? px - (ty + r) * (a.PW - a.TW) : px;
        baddr[tap][j] = (in ? px : ZROW + (px & 1)) * 128 + ((g ^ ((pos >> 1) & 7)) << 4);
      }
    }
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(9 * TC) : "memory");       // all but the weights have landed
    __syncthreads();

    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    auto group = [&](auto more, int c) __attribute__((always_inline)) {
      const int c16 = kq * per_wave + c, sx = (c16 & 3) << 5;
      const unsigned char* pb = held_smem + (c16 >> 2) * SL;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        u32x4 fb[TP];
#pragma unroll
        for (int j = 0; j < TP; ++j) fb[j] = *(const u32x4*)(pb + (baddr[tap][j] ^ sx));
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int j = 0; j < TP; ++j) acc[i][j] = E::mfma(ring[tap][i], fb[j], acc[i][j]);
        if constexpr (decltype(more)::value) load_w(c + 1, tap);
      }
    };
    for (int c = 0; c + 1 < per_wave; ++c) group(std::true_type{}, c);
    group(std::false_type{}, per_wave - 1);

    floatx4 bv[QW], sum[QW];
    {
      const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, a.tiles_c * (BC * 4), BUF_FLAGS);
#pragma unroll
      for (int k = 0; k < QW; ++k) bv[k] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rb, channel(k) * 4, 0, 0));
    }
    // partial sums meet in LDS
    __syncthreads();
    unsigned char* red = held_smem + lane * 16;
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(floatx4*)(red + ((wave * B + i * TP + j) * 4 + q) * 1024) = floatx4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    __syncthreads();
#pragma unroll
    for (int k = 0; k < QW; ++k) {
      floatx4 p[KS];
#pragma unroll
      for (int w = 0; w < KS; ++w) p[w] = *(const floatx4*)(red + ((wp * KS + w) * B * 4 + q0 + k) * 1024);
#pragma unroll
      for (int w = 1; w < KS; ++w)
#pragma unroll
        for (int e = 0; e < 4; ++e) p[0][e] += p[w][e];
      sum[k] = p[0];
    }
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)(a.y + pix0 * a.y_pitch), 0, (int)BUF_MAX, BUF_FLAGS);
    const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, a.act == OCTO_ACT_SILU, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
      constexpr int RES = decltype(res_c)::value;
      constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        u32x4 out;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          floatx4 r4 = {0.f, 0.f, 0.f, 0.f};
          if constexpr (RES != OCTO_RES_NONE) r4 = load4<T>((const T*)&rv[k] + h * 4);
          store4<T>((T*)&out + h * 4, finish4<RES, SILU>(sum[2 * k + h], bv[2 * k + h], r4, act_lo));
        }
        __builtin_amdgcn_raw_buffer_store_b128(out, ry, yo[k / 2] + channel(2 * k) * 2, 0, 0);
      }
    });
    if (t + a.grid < per_die * 8) __syncthreads();       // the partial sums have been read: the patch may be refilled
  }
}

template <typename T, int TC, int TP, int KS, int S>
hipError_t launch_held_cfg(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  constexpr int BC = 32 * TC, BP = 32 * TP * (4 / KS);
  const HeldGeom& g = a.held->geom[which];
  HeldArgs h{};
  h.x = (const char*)a.x + a.x_coff * 2; h.w = (const char*)a.held->w; h.bias = a.bias; h.y = (char*)a.y + a.y_coff * 2;
  h.n_dyn = a.n_dyn; h.res = a.res ? (const char*)a.res + a.res_coff * 2 : nullptr;
  h.n = a.n; h.H = a.H; h.W = a.W; h.Ho = a.Ho; h.Wo = a.Wo; h.C = a.Cin;
  h.x_pitch = a.x_ld * 2; h.y_pitch = a.y_ld * 2; h.res_pitch = a.res_ld * 2;
  h.TH = g.TH; h.TW = g.TW; h.PW = g.PW; h.PH = g.PH; h.halo = g.halo; h.tiles_x = g.tiles_x; h.rows = g.rows;
  h.tiles_c = a.Cout / BC;
  h.act = a.act; h.res_mode = a.res_mode;
  h.div_tw = g.div_tw; h.div_pw = g.div_pw; h.div_ho = a.held->div_ho; h.div_tx = g.div_tx; h.div_tc = a.held->div_tc; h.div_th = g.div_th;
  const long long tiles = held_tiles(a, a.n, which);
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x7FFFFFF0LL) return hipErrorNotSupported;
  static const bool ready = [] {           // more than 64 KB of dynamic LDS needs the attribute, once per instance
    (void)hipFuncSetAttribute((const void*)conv3x3_held_kernel<T, TC, TP, KS, S>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipGetLastError();
    return true;
  }();
  (void)ready;
  if (kernel_id) *kernel_id = held_kernel_id(BC, BP, KS, S);
  // Each die takes a contiguous piece of the tile list and has an L2 of its own.  Where the weights are the larger operand, a die keeps to its channels and all dies read the
  // pixels; otherwise the other way round.
  const long long now = a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n;
  h.c_outer = (double)a.Cout * 9 > (double)now * a.H * a.W;
  const long long grid = std::min((tiles + 7) / 8 * 8, (long long)(held_resident(a, which, num_cu) + 7) / 8 * 8);
  h.grid = (int)grid;
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv3x3_held_kernel<T, TC, TP, KS, S>), dim3((unsigned)grid), dim3(256), (unsigned)g.lds, s, tm.start, tm.stop, 0, h);
  else
    hipLaunchKernelGGL((conv3x3_held_kernel<T, TC, TP, KS, S>), dim3((unsigned)grid), dim3(256), (unsigned)g.lds, s, h);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_held(const ConvArgs& a, long long M, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (!held_fits(a)) return hipErrorNotSupported;
  const int which = held_choose(a, M, num_cu), st = a.stride_h;
  if (which == 0 && st == 1) return launch_held_cfg<T, 2, 1, 4, 1>(0, a, num_cu, s, kernel_id, tm);
  if (which == 1 && st == 1) return launch_held_cfg<T, 2, 2, 4, 1>(1, a, num_cu, s, kernel_id, tm);
  if (which == 2 && st == 1) return launch_held_cfg<T, 2, 2, 2, 1>(2, a, num_cu, s, kernel_id, tm);
  if (which == 0) return launch_held_cfg<T, 2, 1, 4, 2>(0, a, num_cu, s, kernel_id, tm);
  if (which == 1) return launch_held_cfg<T, 2, 2, 4, 2>(1, a, num_cu, s, kernel_id, tm);
  return hipErrorNotSupported;
}

}  // namespace octo
