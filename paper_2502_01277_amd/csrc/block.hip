// A cross-stage block of 32 channels behind its two entry convolutions, in one launch: 1x1, 3x3 (with the shortcut, where there is one), and the 1x1 layer on the
// concatenation of that with the block's other half.  Types of 16 bits, SiLU.
//
// Three launches moved 15 MB a frame of 160 x 160 for 420 MFLOP, of which the block's inputs and its output are 6.6.  Here a workgroup takes 16 x 8 pixels at a time.  Layers of 1x1 need no
// LDS: a lane's 16 bytes of a pixel are its operand of a block of 16 x 16 x 32, and with the rows of the weights permuted its 8 results are consecutive channels of that pixel - the
// operand of the next 1x1 layer as they are.  Only the 3x3 layer's input, 18 x 10 pixels, goes through LDS (vector v of pixel p in slot v ^ (p / 4) % 4; two
// buffers, one barrier per tile).  All weights and biases are in registers for the workgroup's lifetime, sums start from the bias, and the next tile's
// pixels are asked for a tile ahead.
// What bounds it, by counters on 64 frames (122 us): issue and memory together.  The vector units are active in half of the cycles (two fifths of that the exponential and the reciprocal of 72
// activations a lane and tile), the matrix pipe in 17 %, LDS in 13 % - 47 % of that conflicts of banks, which the slots do not prevent -, and its tensors move at 3.5 TB/s (420 MB).
// Before, the three launches, and after, us: 1 frame 13.5 -> 8.3, 5 28.4 -> 16.7, 8 40.5 -> 23.0, 16 58.8 -> 36.5, 64 200 -> 121 (130 with stores of 32 bytes of a pixel and the other half
// asked for at the start of its own tile).
#include "octo_internal.h"
#include "mfma_common.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace octo {

constexpr int BLOCK_TW = 16, BLOCK_TH = 8;                                        // output tile
constexpr int BLOCK_PW = BLOCK_TW + 2, BLOCK_PX = BLOCK_PW * (BLOCK_TH + 2);      // its pixels with their neighbours

struct BlockKernelArgs {
  const char* x; const char* z; char* y;               // input of the block's inner layers, its other half, output: first channel of the first pixel
  const char* w0; const char* w1; const char* w2;
  const float* b0; const float* b1; const float* b2;
  int x_pitch, z_pitch, y_pitch;                       // bytes of a pixel
  int row0, row1, row2;                                // bytes of a weight row
  int H, W, n_tiles, grid, tiles_x;
  FastDiv div_tx, div_ty;
};

template <typename T, bool SHORTCUT>
__global__ __launch_bounds__(256, 2) void block_kernel(const BlockKernelArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char s_h[2][192 * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;

  // weights: row r of block b of a pair has channel 8 (r / 4) + 4 b + r % 4, so that a lane gets 8 consecutive channels of its pixel, and a store 64 bytes of it
  u32x4 w0[2], w1[2][9], w2[4][2];
  floatx4 b0[2], b1[2], b2[4];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int ch = 8 * (r16 >> 2) + 4 * b + (r16 & 3);
    w0[b] = *(const u32x4*)(a.w0 + (size_t)ch * a.row0 + q4 * 16);
#pragma unroll
    for (int s = 0; s < 9; ++s) w1[b][s] = *(const u32x4*)(a.w1 + (size_t)ch * a.row1 + s * 64 + q4 * 16);
    b0[b] = *(const floatx4*)(a.b0 + q4 * 8 + b * 4);
    b1[b] = *(const floatx4*)(a.b1 + q4 * 8 + b * 4);
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int ch = 32 * (b >> 1) + 8 * (r16 >> 2) + 4 * (b & 1) + (r16 & 3);
#pragma unroll
    for (int s = 0; s < 2; ++s) w2[b][s] = *(const u32x4*)(a.w2 + (size_t)ch * a.row2 + s * 64 + q4 * 16);
    b2[b] = *(const floatx4*)(a.b2 + 32 * (b >> 1) + q4 * 8 + 4 * (b & 1));
  }
  // pixels of the tile with their neighbours, blocks wave, wave + 4, wave + 8: row and column, LDS offset; taps of the wavefront's two rows of the tile
  int at0[3], wr0[3], rd1[2][9];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int p = (wave + 4 * i) * 16 + r16, r = p / BLOCK_PW, c = p - r * BLOCK_PW;
    at0[i] = p < BLOCK_PX ? r << 16 | c : 0x7FFF0000;
    wr0[i] = p * 64 + ((q4 ^ ((p >> 2) & 3)) << 4);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int p = (wave * 2 + j + tap / 3) * BLOCK_PW + r16 + tap % 3;
      rd1[j][tap] = p * 64 + ((q4 ^ ((p >> 2) & 3)) << 4);
    }

  const int per_die = (a.n_tiles + 7) >> 3, t_end = per_die * 8;       // one contiguous chunk of the tile list per die, see conv_mfma_kernel
  auto next_valid = [&](int t) -> int {
    while (t < t_end && (t & 7) * per_die + (t >> 3) >= a.n_tiles) t += a.grid;
    return t;
  };
  int img = 0, y0 = 0, x0 = 0;
  auto locate = [&](int t) __attribute__((always_inline)) {
    const unsigned tile = (unsigned)((t & 7) * per_die + (t >> 3)), row = fast_div(tile, a.div_tx);
    img = (int)fast_div(row, a.div_ty);
    x0 = (int)(tile - row * (unsigned)a.tiles_x) * BLOCK_TW;
    y0 = (int)(row - (unsigned)img * (unsigned)((a.H + BLOCK_TH - 1) / BLOCK_TH)) * BLOCK_TH;
  };
  // a lane's vector of a pixel; zeros outside the image
  auto load = [&](const char* p, int pitch, int Y, int X) __attribute__((always_inline)) -> u32x4 {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(p + (size_t)img * a.H * a.W * pitch), 0, a.H * a.W * pitch, BUF_FLAGS);
    return __builtin_amdgcn_raw_buffer_load_b128(r, (unsigned)Y < (unsigned)a.H && (unsigned)X < (unsigned)a.W ? (Y * a.W + X) * pitch + q4 * 16 : OOB, 0, 0);
  };
  u32x4 f0[3], other[2];
  auto load_x = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 3; ++i) f0[i] = load(a.x, a.x_pitch, y0 - 1 + (at0[i] >> 16), x0 - 1 + (at0[i] & 0xFFFF));
  };
  int t = next_valid(blockIdx.x);
  if (t >= t_end) return;
  locate(t);
  load_x();
#pragma unroll
  for (int j = 0; j < 2; ++j) other[j] = load(a.z, a.z_pitch, y0 + wave * 2 + j, x0 + r16);
  for (int buf = 0;; buf ^= 1) {
    const int cy = y0, cx = x0;
    u32x4 res[2];
    if constexpr (SHORTCUT) {
#pragma unroll
      for (int j = 0; j < 2; ++j) res[j] = load(a.x, a.x_pitch, cy + wave * 2 + j, cx + r16);
    }
    char* const yb = a.y + (size_t)img * a.H * a.W * a.y_pitch;
    // pixels outside the image are the padding of the 3x3 layer: only a tile on an edge has any
    const bool inside = cy > 0 && cx > 0 && cy + BLOCK_TH < a.H && cx + BLOCK_TW < a.W;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      u32x4 out = silu8<T>(mfma16<T>(w0[0], f0[i], b0[0]), mfma16<T>(w0[1], f0[i], b0[1]));
      if (!inside && ((unsigned)(cy - 1 + (at0[i] >> 16)) >= (unsigned)a.H || (unsigned)(cx - 1 + (at0[i] & 0xFFFF)) >= (unsigned)a.W)) out = u32x4{0u, 0u, 0u, 0u};
      *(u32x4*)(s_h[buf] + wr0[i]) = out;
    }
    t = next_valid(t + a.grid);
    const bool more = t < t_end;
    if (more) { locate(t); load_x(); }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      floatx4 acc[2];
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const u32x4 f = *(const u32x4*)(s_h[buf] + rd1[j][tap]);
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = mfma16<T>(w1[b][tap], f, tap == 0 ? b1[b] : acc[b]);
      }
      // a lane's 8 channels of its pixel are its operand of the last layer
      u32x4 h;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        floatx4 v = {silu(acc[b][0]), silu(acc[b][1]), silu(acc[b][2]), silu(acc[b][3])};
        if constexpr (SHORTCUT) {
          const floatx4 r = load4<T>((const T*)&res[j] + b * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += r[e];
        }
        store4<T>((T*)&h + b * 4, v);
      }
      floatx4 o[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) o[b] = mfma16<T>(w2[b][1], other[j], mfma16<T>(w2[b][0], h, b2[b]));
      if (more) other[j] = load(a.z, a.z_pitch, y0 + wave * 2 + j, x0 + r16);
      const int Y = cy + wave * 2 + j, X = cx + r16;
      if (Y < a.H && X < a.W) {
        u32x4* q = (u32x4*)(yb + (size_t)(Y * a.W + X) * a.y_pitch + q4 * 16);
        q[0] = silu8<T>(o[0], o[1]);
        q[4] = silu8<T>(o[2], o[3]);
      }
    }
    if (!more) break;
  }
}

hipError_t launch_block(int dtype, const BlockArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm) {
  if (dtype != OCTO_F16 && dtype != OCTO_BF16) return hipErrorNotSupported;
  if (((a.x_ld | a.x_coff | a.z_ld | a.z_coff | a.y_ld | a.y_coff) & 7) || (((uintptr_t)a.x | (uintptr_t)a.z | (uintptr_t)a.y) & 15)) return hipErrorNotSupported;
  if ((long long)a.H * a.W * std::max(a.x_ld, std::max(a.z_ld, a.y_ld)) * 2 >= 0x7FFFFFF0LL) return hipErrorNotSupported;      // 32-bit offsets inside an image
  BlockKernelArgs k{};
  k.x = (const char*)a.x + (size_t)a.x_coff * 2; k.z = (const char*)a.z + (size_t)a.z_coff * 2; k.y = (char*)a.y + (size_t)a.y_coff * 2;
  k.w0 = (const char*)a.w[0]; k.w1 = (const char*)a.w[1]; k.w2 = (const char*)a.w[2];
  k.b0 = a.bias[0]; k.b1 = a.bias[1]; k.b2 = a.bias[2];
  k.x_pitch = a.x_ld * 2; k.z_pitch = a.z_ld * 2; k.y_pitch = a.y_ld * 2;
  k.row0 = a.kp[0] * 2; k.row1 = a.kp[1] * 2; k.row2 = a.kp[2] * 2;
  k.H = a.H; k.W = a.W; k.tiles_x = (a.W + BLOCK_TW - 1) / BLOCK_TW;
  const int tiles_y = (a.H + BLOCK_TH - 1) / BLOCK_TH;
  const long long tiles = (long long)a.n * k.tiles_x * tiles_y;
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x7FFFFF00LL) return hipErrorNotSupported;
  k.n_tiles = (int)tiles;
  k.div_tx = make_fastdiv((unsigned)k.tiles_x); k.div_ty = make_fastdiv((unsigned)tiles_y);
  k.grid = (int)std::min((tiles + 7) / 8 * 8, ((long long)num_cu * 2 + 7) / 8 * 8);
  if (kernel_id) *kernel_id = block_kernel_id(a.shortcut);
  auto go = [&](auto kernel) {
    if (tm.start && tm.stop) hipExtLaunchKernelGGL(kernel, dim3((unsigned)k.grid), dim3(256), 0, s, tm.start, tm.stop, 0, k);
    else hipLaunchKernelGGL(kernel, dim3((unsigned)k.grid), dim3(256), 0, s, k);
    return hipGetLastError();
  };
  if (dtype == OCTO_F16) return a.shortcut ? go(block_kernel<_Float16, true>) : go(block_kernel<_Float16, false>);
  return a.shortcut ? go(block_kernel<__bf16, true>) : go(block_kernel<__bf16, false>);
}

}  // namespace octo
