// The entry of a cross-stage block in one launch: its two 1x1 convolutions of the same input, and the 1x1 layer of the block's first bottleneck on the first one's output.  Types of
// 16 bits, SiLU, 64 or 128 channels each.
//
// Two launches (the entry layers as one, the third layer) wrote the first layer's output to memory, read it back, and each waited for its pixels anew.  Here a workgroup, a wavefront to 32 of the
// stacked layers' channels, brings a tile of pixels to LDS (vector v of pixel p in slot v ^ p % 16: no two lanes of a read on one bank), all its weights are in registers for its
// lifetime, and the first layer's results - 8 consecutive channels of a pixel to a lane, the weights' rows being permuted - go through LDS to the third layer.  Sums start from the bias; the
// next tile's pixels are asked for a tile ahead; where nothing else reads the first layer's output it is not written.
// What bounds it: with many frames the memory traffic of its tensors (64 x 80 x 80, 128 -> 64: 262 MB in 56 us, 4.7 TB/s); with few the time until the weights and the first pixels are there.
// Before, the two launches, and after, us, s detector: 64 channels of 80 x 80 from 128 and from 256 input channels, 1 frame 8.5 -> 4.9 and 8.6 -> 5.6, 5 16.1 -> 13.2 and 14.3 -> 12.5,
// 8 19.9 -> 13.9 and 17.5 -> 14.3, 16 23.7 -> 15.8 and 28 -> 19.7, 64 73 -> 56 and 94 -> 59; 128 channels of 40 x 40, 16 18.6 -> 15.6, 64 49 -> 33.6.  Whole passes 0.3 - 2 % less.
#include "octo_internal.h"
#include "mfma_common.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace octo {

struct LeadKernelArgs {
  const char* x; char* a; char* b; char* h;            // first channel of the first pixel; a may be null: nobody else reads it
  const char* w0; const char* w1;                      // the two entry layers' weights, stacked; the third one's
  const float* b0; const float* b1;
  int x_pitch, a_pitch, b_pitch, h_pitch;              // bytes of a pixel
  int row0, row1;                                      // bytes of a weight row
  long long pixels;
  int n_tiles, grid;
};

// C: channels of each layer; KS: input channels / 32; NP: blocks of 16 pixels of a tile
template <typename T, int C, int KS, int NP>
__global__ __launch_bounds__(C * 4, 1) void lead_kernel(const LeadKernelArgs a) {
  constexpr int WAVES = C / 16, TP = NP * 16, XV = KS * 4, HV = C / 8, K2 = C / 32;
  constexpr int LV = TP * XV / (WAVES * 64);                       // vectors of a tile a lane brings
  constexpr int PG = NP == 1 ? 1 : 2, CB = PG;                     // second step: groups of pixel blocks, channel blocks of a wavefront
  static_assert(LV * WAVES * 64 == TP * XV, "whole vectors");
  __shared__ __attribute__((aligned(1024))) unsigned char s_x[TP * XV * 16], s_h[TP * HV * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;

  // first step: 32 channels of the stacked layers; row r of block b of a pair has channel 8 (r / 4) + 4 b + r % 4, so that a lane gets 8 consecutive channels of its pixel
  u32x4 w0[2][KS], w1[CB][K2];
  floatx4 b0[2], b1[CB];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const char* row = a.w0 + (size_t)(wave * 32 + 8 * (r16 >> 2) + 4 * b + (r16 & 3)) * a.row0 + q4 * 16;
#pragma unroll
    for (int s = 0; s < KS; ++s) w0[b][s] = *(const u32x4*)(row + s * 64);
    b0[b] = *(const floatx4*)(a.b0 + wave * 32 + q4 * 8 + b * 4);
  }
  // second step: 16 channels of all pixels, or 32 of every other block of 16
  const int c2 = PG == 1 ? wave * 16 : wave % (C / 32) * 32, pg = PG == 1 ? 0 : wave / (C / 32);
#pragma unroll
  for (int b = 0; b < CB; ++b) {
    const char* row = a.w1 + (size_t)(c2 + (CB == 1 ? r16 : 8 * (r16 >> 2) + 4 * b + (r16 & 3))) * a.row1 + q4 * 16;
#pragma unroll
    for (int s = 0; s < K2; ++s) w1[b][s] = *(const u32x4*)(row + s * 64);
    b1[b] = *(const floatx4*)(a.b1 + c2 + (CB == 1 ? q4 * 4 : q4 * 8 + b * 4));
  }
  const bool first = wave < WAVES / 2;                             // this wavefront's channels are the first layer's
  char* const y0 = first ? a.a : a.b;
  const int y0_pitch = first ? a.a_pitch : a.b_pitch, c0 = (first ? wave : wave - WAVES / 2) * 32 + q4 * 8;

  const int per_die = (a.n_tiles + 7) >> 3, t_end = per_die * 8;   // one contiguous chunk of the tile list per die, see conv_mfma_kernel
  auto next_valid = [&](int t) -> int {
    while (t < t_end && (t & 7) * per_die + (t >> 3) >= a.n_tiles) t += a.grid;
    return t;
  };
  u32x4 in[LV];
  long long p0 = 0;
  int left = 0;                                                    // pixels of the tile inside the tensor
  auto load = [&](int t) __attribute__((always_inline)) {
    p0 = (long long)((t & 7) * per_die + (t >> 3)) * TP;
    left = (int)(a.pixels - p0 < TP ? a.pixels - p0 : TP);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(a.x + (size_t)p0 * a.x_pitch), 0, left * a.x_pitch, BUF_FLAGS);
#pragma unroll
    for (int i = 0; i < LV; ++i) {
      const int v = tid + i * WAVES * 64, p = v / XV;
      in[i] = __builtin_amdgcn_raw_buffer_load_b128(r, p < left ? p * a.x_pitch + (v & (XV - 1)) * 16 : OOB, 0, 0);
    }
  };
  int t = next_valid(blockIdx.x);
  if (t >= t_end) return;
  load(t);
  for (;;) {
    const long long cp = p0;
    const int cl = left;
#pragma unroll
    for (int i = 0; i < LV; ++i) {
      const int v = tid + i * WAVES * 64, p = v / XV;
      *(u32x4*)(s_x + (p * XV + ((v & (XV - 1)) ^ (p & 15))) * 16) = in[i];
    }
    t = next_valid(t + a.grid);
    const bool more = t < t_end;
    if (more) load(t);
    __syncthreads();                                               // (also: every wavefront has read s_h of the tile before)
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int p = j * 16 + r16;
      floatx4 acc[2] = {b0[0], b0[1]};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const u32x4 f = *(const u32x4*)(s_x + (p * XV + ((s * 4 + q4) ^ r16)) * 16);
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = mfma16<T>(w0[b][s], f, acc[b]);
      }
      const u32x4 o = silu8<T>(acc[0], acc[1]);
      if (first) *(u32x4*)(s_h + (p * HV + ((c0 >> 3) ^ (p & (HV - 1)))) * 16) = o;
      if (p < cl && y0) *(u32x4*)(y0 + (size_t)(cp + p) * y0_pitch + c0 * 2) = o;
    }
    __syncthreads();                                               // (also: every wavefront has read s_x)
#pragma unroll
    for (int j = 0; j < NP / PG; ++j) {
      const int p = (j * PG + pg) * 16 + r16;
      floatx4 acc[CB];
#pragma unroll
      for (int b = 0; b < CB; ++b) acc[b] = b1[b];
#pragma unroll
      for (int s = 0; s < K2; ++s) {
        const u32x4 f = *(const u32x4*)(s_h + (p * HV + ((s * 4 + q4) ^ (p & (HV - 1)))) * 16);
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[b] = mfma16<T>(w1[b][s], f, acc[b]);
      }
      if (p < cl) {
        char* q = a.h + (size_t)(cp + p) * a.h_pitch + c2 * 2;
        if constexpr (CB == 1) store4<T>((T*)q + q4 * 4, floatx4{silu(acc[0][0]), silu(acc[0][1]), silu(acc[0][2]), silu(acc[0][3])});
        else *(u32x4*)(q + q4 * 16) = silu8<T>(acc[0], acc[CB - 1]);
      }
    }
    if (!more) break;
  }
}

bool lead_fits(int c, int cin) { return (c == 64 && (cin == 128 || cin == 256)) || (c == 128 && cin == 256); }

hipError_t launch_lead(int dtype, const LeadArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm) {
  if ((dtype != OCTO_F16 && dtype != OCTO_BF16) || !lead_fits(a.C, a.Cin)) return hipErrorNotSupported;
  if (((a.x_ld | a.x_coff | a.a_ld | a.a_coff | a.b_ld | a.b_coff | a.h_ld | a.h_coff) & 7) ||
      (((uintptr_t)a.x | (uintptr_t)a.a | (uintptr_t)a.b | (uintptr_t)a.h) & 15)) return hipErrorNotSupported;
  if (a.x_ld > 1 << 20) return hipErrorNotSupported;               // 32-bit offsets inside a tile
  LeadKernelArgs k{};
  k.x = (const char*)a.x + (size_t)a.x_coff * 2; k.a = a.a ? (char*)a.a + (size_t)a.a_coff * 2 : nullptr;
  k.b = (char*)a.b + (size_t)a.b_coff * 2; k.h = (char*)a.h + (size_t)a.h_coff * 2;
  k.w0 = (const char*)a.w[0]; k.w1 = (const char*)a.w[1]; k.b0 = a.bias[0]; k.b1 = a.bias[1];
  k.x_pitch = a.x_ld * 2; k.a_pitch = a.a_ld * 2; k.b_pitch = a.b_ld * 2; k.h_pitch = a.h_ld * 2;
  k.row0 = a.kp[0] * 2; k.row1 = a.kp[1] * 2;
  k.pixels = a.pixels;
  if (a.pixels <= 0) return hipSuccess;
  // 128 channels: a workgroup's weights are 160 KB, one workgroup to a CU.  They are worth their time from two tiles of 32 pixels to a CU: 40 x 40, 1 frame 8.3 -> 7.1 us (and no less for the
  // whole pass), 5 10.3 -> 11.6, 8 12.4 -> 12.9 and 11.8 -> 10.6, 16 18.6 -> 15.6.
  if (a.C == 128 && a.pixels < 64LL * num_cu) return hipErrorNotSupported;
  // Tiles of 16 pixels while they all have a CU to themselves; of 64 from 8 to a CU, where there are registers for them (64 x 80 x 80, 32 against 64 pixels: 60 -> 57 and 63 -> 59 us; 8 frames
  // 13.8 -> 15 and 13.9 -> 15.6); else of 32 (80 x 80, 1 frame, 16 against 32: 5.4 -> 4.9 and 6.8 -> 5.4).
  const int np = a.pixels <= 16LL * num_cu ? 1 : a.C == 64 && a.pixels >= 64LL * 8 * num_cu ? 4 : 2;
  const long long tiles = (a.pixels + np * 16 - 1) / (np * 16);
  if (tiles >= 0x7FFFFF00LL) return hipErrorNotSupported;
  k.n_tiles = (int)tiles;
  // two workgroups to a CU keep more loads in flight (64 frames, one: 73 and 80 us, two: 60 and 63, three: 61 and 70); of 128 channels one has room
  const long long resident = (long long)num_cu * (a.C == 64 ? 2 : 1);
  k.grid = (int)std::min((tiles + 7) / 8 * 8, (resident + 7) / 8 * 8);
  if (kernel_id) *kernel_id = lead_kernel_id(a.C, a.Cin, np);
  auto go = [&](auto kernel) {
    if (tm.start && tm.stop) hipExtLaunchKernelGGL(kernel, dim3((unsigned)k.grid), dim3((unsigned)a.C * 4), 0, s, tm.start, tm.stop, 0, k);
    else hipLaunchKernelGGL(kernel, dim3((unsigned)k.grid), dim3((unsigned)a.C * 4), 0, s, k);
    return hipGetLastError();
  };
  auto form = [&](auto zero) {
    using T = decltype(zero);
    if (a.C == 128) return go(lead_kernel<T, 128, 8, 2>);          // (refused where tiles of 16 pixels would be chosen)
    if (a.Cin == 128) return np == 1 ? go(lead_kernel<T, 64, 4, 1>) : np == 2 ? go(lead_kernel<T, 64, 4, 2>) : go(lead_kernel<T, 64, 4, 4>);
    return np == 1 ? go(lead_kernel<T, 64, 8, 1>) : np == 2 ? go(lead_kernel<T, 64, 8, 2>) : go(lead_kernel<T, 64, 8, 4>);
  };
  return dtype == OCTO_F16 ? form(_Float16()) : form(__bf16());
}

}  // namespace octo
