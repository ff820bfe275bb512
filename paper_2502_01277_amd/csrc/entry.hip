// The first layers of a detector in one launch: the first convolution (3-channel input as pixel pairs, 6x6 / stride 2 / pad 2, 32 channels), the down-sampling 3x3 / stride 2 /
// pad 1 layer behind it (64 channels), and the two 1x1 layers (32 channels each) that are the only readers of that one.  Types of 16 bits, SiLU.
//
// In launches of their own these layers write and read the two largest tensors of a detector (26 MB a frame of 640 x 640 moved for them) and are bound by that: 127, 203 and 79 us on 64
// frames.  Here a workgroup takes 8 x 8 pixels of the second layer's output at a time: the 38 x 38 input pixels come into LDS (the next tile's while this one is computed), the
// first layer's 17 x 17 and the second's 8 x 8 pixels stay there.  All weights and biases are in registers for the workgroup's lifetime.  13 % of the first layer is computed twice.
// Blocks of 16 x 16 x 32, a block's rows permuted so that a lane gets 8 consecutive channels of its pixel: one LDS write or store per block.  The first layer's pixels
// lie in LDS by parity of their column, even ones first, so that the stride-2 taps of 8 neighbouring pixels read neighbours; vector v of pixel p in slot v ^ (p / 4) % 4,
// of the second layer's in v ^ (p / 2) % 8.
// What bounds it, by counters on 64 frames (223 us): issue.  The vector units are active in 56 % of the cycles (two fifths of that the exponential and the reciprocal of 72 activations a lane
// and tile), the matrix pipe in 29 %, LDS in 35 % - 45 % of that conflicts of banks, which the slots do not prevent -, and an instruction of some kind is under way in 74 %.  Sums start from the
// bias, which saves an addition each (252 -> 235 us on 64 frames with that and the next block's operands read ahead of a block's activations).  Before, the three launches, and after, us: 1 frame 21.0 ->
// 14.5, 5 42.5 -> 29.2, 8 57.5 -> 37.6, 16 109 -> 62, 64 399 -> 235.
#include "octo_internal.h"
#include "mfma_common.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace octo {

constexpr int ENTRY_PITCH = 20;                  // LDS row of the input tile in pairs, and of the first layer's tile in pixels
constexpr int ENTRY_ROWS = 38, ENTRY_PAIRS = 19; // input rows and pairs of an 8 x 8 tile
constexpr int ENTRY_T0 = 17;                     // rows and columns of the first layer's tile
constexpr int ENTRY_BYTES = 3 * 4096;         // 38 rows of 20 vectors, in whole passes of the loader

struct EntryKernelArgs {
  const char* x; const char* w0; const char* w1; const char* w2;
  const float* b0; const float* b1; const float* b2;
  char* y[2];
  int y_pitch[2];
  int row0, row1, row2;                    // bytes of a weight row
  int H, W2, H0, W0, H1, W1;
  int n_tiles, grid, tiles_x;
  FastDiv div_tx, div_ty;
};

template <typename T>
__global__ __launch_bounds__(256, 2) void entry_kernel(const EntryKernelArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char s_in[2][ENTRY_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char s_t0[ENTRY_T0 * ENTRY_PITCH * 64];
  __shared__ __attribute__((aligned(1024))) unsigned char s_t1[64 * 128];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q4 = lane >> 4, wc = wave & 1, wp = wave >> 1;

  // weights: block b of a wavefront's two has channel 8 (r / 4) + 4 b + r % 4 in row r, so that a lane gets 8 consecutive channels of its pixel
  u32x4 w0[2][5], w1[2][9], w2[2][2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int ch = 8 * (r16 >> 2) + 4 * b + (r16 & 3);
#pragma unroll
    for (int s = 0; s < 5; ++s) w0[b][s] = *(const u32x4*)(a.w0 + (size_t)ch * a.row0 + s * 64 + q4 * 16);
#pragma unroll
    for (int s = 0; s < 9; ++s) w1[b][s] = *(const u32x4*)(a.w1 + (size_t)(wc * 32 + ch) * a.row1 + s * 64 + q4 * 16);
#pragma unroll
    for (int s = 0; s < 2; ++s) w2[b][s] = *(const u32x4*)(a.w2 + (size_t)(wc * 32 + ch) * a.row2 + s * 64 + q4 * 16);
  }
  // biases of a lane's channels, where the sums start
  floatx4 b0[2], b1[2], b2[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    b0[h] = *(const floatx4*)(a.b0 + q4 * 8 + h * 4);
    b1[h] = *(const floatx4*)(a.b1 + wc * 32 + q4 * 8 + h * 4);
    b2[h] = *(const floatx4*)(a.b2 + wc * 32 + q4 * 8 + h * 4);
  }

  // first layer: LDS offsets of a pixel's window (two vectors past its 18th are zeros from behind the last row) and of its result, blocks wave, wave + 4 ...
  int voff[5], rd0[5], wr0[5], at0[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) { const int v = 4 * s + q4; voff[s] = (v / 3 * ENTRY_PITCH + v % 3) * 16; }
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int px = (wave + 4 * i) * 16 + r16, p = px / ENTRY_T0, c = px - p * ENTRY_T0, pp = p * ENTRY_PITCH + (c & 1 ? 9 + (c >> 1) : c >> 1);
    const bool in = px < ENTRY_T0 * ENTRY_T0;
    rd0[i] = in ? (2 * p * ENTRY_PITCH + c) * 16 : 0;
    wr0[i] = in ? pp * 64 + ((q4 ^ ((pp >> 2) & 3)) << 4) : (ENTRY_PITCH - 1) * 64;      // (a column that nothing reads)
    at0[i] = p << 16 | c;
  }
  // second layer: offsets of a tap's vector, of the result; third: of its vectors
  int rd1[2][9], wr1[2], rd2[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int t = (wp * 2 + j) * 16 + r16, ty = t >> 3, tx = t & 7;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int r = tap / 3, s = tap % 3, pp = (2 * ty + r) * ENTRY_PITCH + (s == 1 ? 9 + tx : tx + (s >> 1));
      rd1[j][tap] = pp * 64 + ((q4 ^ ((pp >> 2) & 3)) << 4);
    }
    wr1[j] = t * 128 + (((wc * 4 + q4) ^ ((t >> 1) & 7)) << 4);
#pragma unroll
    for (int s = 0; s < 2; ++s) rd2[j][s] = t * 128 + (((s * 4 + q4) ^ ((t >> 1) & 7)) << 4);
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
    x0 = (int)(tile - row * (unsigned)a.tiles_x) * 8;
    y0 = (int)(row - (unsigned)img * (unsigned)((a.H1 + 7) >> 3)) * 8;
  };
  const int img_bytes = a.H * a.W2 * 16;
  const unsigned lds_in = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)&s_in[0][0] + (unsigned)wave * 1024u));
  auto load_in = [&](int buf) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)(a.x + (size_t)img * img_bytes), 0, img_bytes, BUF_FLAGS);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int v = i * 256 + tid, r = v / ENTRY_PITCH, c = v - r * ENTRY_PITCH, Y = 4 * y0 - 4 + r, P = 2 * x0 - 2 + c;
      const int o = r < ENTRY_ROWS && c < ENTRY_PAIRS && (unsigned)Y < (unsigned)a.H && (unsigned)P < (unsigned)a.W2 ? (Y * a.W2 + P) * 16 : OOB;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds_in + buf * ENTRY_BYTES + i * 4096), "v"(o), "s"(rx) : "memory");
    }
  };
  int t = next_valid(blockIdx.x);
  if (t >= t_end) return;
  locate(t);
  load_in(0);
  for (int buf = 0;; buf ^= 1) {
    const int cur_img = img, cy = y0, cx = x0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (the results of the tile before have left too)
    __syncthreads();
    t = next_valid(t + a.grid);
    const bool more = t < t_end;
    if (more) { locate(t); load_in(buf ^ 1); }

    const unsigned char* in = s_in[buf];
    // pixels outside the first layer's output are the padding of the second layer's input: only a tile on an edge has any
    const bool inside = cy > 0 && cx > 0 && 2 * cy + ENTRY_T0 - 2 < a.H0 && 2 * cx + ENTRY_T0 - 2 < a.W0;
    u32x4 f[2][5];
    auto read0 = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 5; ++s) f[i & 1][s] = *(const u32x4*)(in + (s < 4 || q4 < 2 ? rd0[i] + voff[s] : ENTRY_ROWS * ENTRY_PITCH * 16));
    };
    auto block0 = [&](int i, bool next) __attribute__((always_inline)) {
      floatx4 acc[2];
#pragma unroll
      for (int s = 0; s < 5; ++s)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = mfma16<T>(w0[b][s], f[i & 1][s], s == 0 ? b0[b] : acc[b]);
      if (next) read0(i + 1);
      u32x4 out = silu8<T>(acc[0], acc[1]);
      if (!inside) {
        const int Y = 2 * cy - 1 + (at0[i] >> 16), X = 2 * cx - 1 + (at0[i] & 0xFFFF);
        if ((unsigned)Y >= (unsigned)a.H0 || (unsigned)X >= (unsigned)a.W0) out = u32x4{0u, 0u, 0u, 0u};
      }
      *(u32x4*)(s_t0 + wr0[i]) = out;
    };
    read0(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) block0(i, true);
    if (wave < 3) block0(4, false);                      // the last wavefront has four blocks
    __syncthreads();
    {
      floatx4 acc[2][2];
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const u32x4 f = *(const u32x4*)(s_t0 + rd1[j][tap]);
#pragma unroll
          for (int b = 0; b < 2; ++b) acc[j][b] = mfma16<T>(w1[b][tap], f, tap == 0 ? b1[b] : acc[j][b]);
        }
#pragma unroll
      for (int j = 0; j < 2; ++j) *(u32x4*)(s_t1 + wr1[j]) = silu8<T>(acc[j][0], acc[j][1]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      floatx4 acc[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const u32x4 f = *(const u32x4*)(s_t1 + rd2[j][s]);
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = mfma16<T>(w2[b][s], f, s == 0 ? b2[b] : acc[b]);
      }
      const u32x4 out = silu8<T>(acc[0], acc[1]);
      const int q = (wp * 2 + j) * 16 + r16, Y = cy + (q >> 3), X = cx + (q & 7);
      if (Y < a.H1 && X < a.W1) *(u32x4*)(a.y[wc] + ((size_t)(cur_img * a.H1 + Y) * a.W1 + X) * a.y_pitch[wc] + q4 * 16) = out;
    }
    if (!more) break;
  }
}

hipError_t launch_entry(int dtype, const EntryArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm) {
  EntryKernelArgs k{};
  k.x = (const char*)a.x; k.w0 = (const char*)a.w[0]; k.w1 = (const char*)a.w[1]; k.w2 = (const char*)a.w[2];
  k.b0 = a.bias[0]; k.b1 = a.bias[1]; k.b2 = a.bias[2];
  k.row0 = a.kp[0] * 2; k.row1 = a.kp[1] * 2; k.row2 = a.kp[2] * 2;
  for (int i = 0; i < 2; ++i) {
    if (((a.y_ld[i] | a.y_coff[i]) & 7) || ((uintptr_t)a.y[i] & 15)) return hipErrorNotSupported;
    k.y[i] = (char*)a.y[i] + (size_t)a.y_coff[i] * 2; k.y_pitch[i] = a.y_ld[i] * 2;
  }
  if ((dtype != OCTO_F16 && dtype != OCTO_BF16) || ((uintptr_t)a.x & 15) || a.kp[0] < 160 || (long long)a.H * a.W * 8 >= 0x7FFFFFF0LL) return hipErrorNotSupported;
  k.H = a.H; k.W2 = a.W / 2; k.H0 = (a.H - 2) / 2 + 1; k.W0 = (a.W - 2) / 2 + 1; k.H1 = (k.H0 - 1) / 2 + 1; k.W1 = (k.W0 - 1) / 2 + 1;
  k.tiles_x = (k.W1 + 7) / 8;
  const int tiles_y = (k.H1 + 7) / 8;
  const long long tiles = (long long)a.n * k.tiles_x * tiles_y;
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x7FFFFF00LL || (long long)a.n * k.H1 * k.W1 >= 0x7FFFFFFFLL) return hipErrorNotSupported;
  k.n_tiles = (int)tiles;
  k.div_tx = make_fastdiv((unsigned)k.tiles_x); k.div_ty = make_fastdiv((unsigned)tiles_y);
  k.grid = (int)std::min((tiles + 7) / 8 * 8, ((long long)num_cu * 2 + 7) / 8 * 8);
  if (kernel_id) *kernel_id = KID_ENTRY;
  auto go = [&](auto kernel) {
    if (tm.start && tm.stop) hipExtLaunchKernelGGL(kernel, dim3((unsigned)k.grid), dim3(256), 0, s, tm.start, tm.stop, 0, k);
    else hipLaunchKernelGGL(kernel, dim3((unsigned)k.grid), dim3(256), 0, s, k);
    return hipGetLastError();
  };
  return dtype == OCTO_F16 ? go(entry_kernel<_Float16>) : go(entry_kernel<__bf16>);
}

}  // namespace octo
