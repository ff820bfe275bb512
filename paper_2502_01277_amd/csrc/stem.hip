// First-layer convolution (3 input channels, stride 2) on the matrix cores, and the 3x3 / stride-2 / pad-1 max-pool behind it where the
// layer's output feeds nothing else (only the pooled tensor is written then).
//
// The input is stored with 4 channels, so two neighbouring pixels form one 16-byte vector of 8 values, and a
// stride-2 convolution becomes a stride-1 convolution over pixel pairs with a kernel of KH x PKW pairs (see
// pipeline.hip, which also re-packs the weights as [Cout][(row, pair, 8 values)]).  The general implicit-GEMM kernel
// gathers every K vector of every output pixel from global memory: for a 7x7 kernel that is 28 loads of 16 bytes per
// output pixel, almost all of them re-reads.  Here
//   * the weights live in registers for the lifetime of a wavefront (112 registers for 64 channels x 7x7).  Out of LDS they cost as many
//     bytes per MFMA as the pixel operand, and the two together are exactly what a compute unit's LDS delivers at the full MFMA rate;
//   * a wavefront works on its own: it walks down a segment of a strip of 64 convolution columns, one row at a time, with the input rows
//     in a ring of eight row pairs in LDS, fetched four rows ahead straight from memory.  No barrier after the weights.  (A workgroup that
//     loaded a patch, computed a tile, staged it in LDS and wrote or pooled it took turns at each: matrix pipe 29 % busy with the pool.)
//   * the 16 channels that a lane gets of a pixel are consecutive (rows of the weight operand are permuted to that end), and results leave
//     from the registers, 64 bytes of a pixel at a time;
//   * for the pool, one block of 32 pixels is the even columns of a row and the other the odd ones, so that the two or three columns of a
//     window lie in one lane and its neighbour: the horizontal maximum is two instructions per accumulator, the vertical one another, on
//     registers that the wavefront carries from row to row.  Bias and activation come after the maximum (before it for SiLU, which is not
//     monotonous), on a quarter of the values.  Rounding keeps the order, so the result is that of the separate kernels bit for bit.  The
//     ring then stores the even and the odd pixel pairs of a row apart: either way an operand read is 32 consecutive vectors.
// Bound by the matrix pipe with the pool (28 vectors of 8 products, of which 147 are real), without it by memory and SiLU.
// Measured against tiles staged in LDS, us: 7x7 with the pool, bf16, 4170 crops of 224 x 224 2146 -> 1300, some 380 crops 232 -> 148, some 6
// crops 23 -> 18, on 224 x 224 with SiLU (stem_pool_any_kernel) 8 crops 19.5 -> 18.5, 380 283 -> 249, 2000 1438 -> 1105, 36 channels with ReLU
// (the same) 17.1 -> 14.4, 237 -> 163, 1190 -> 800; 6x6 on 32 frames of 1280 x 1280 to 64 channels 496 -> 434, on 64 of 640 x 640 to 32 channels 170 -> 127 (5 TB/s).
#include "mfma_common.h"
#include "stem_segment.h"
#include <hip/hip_ext.h>

namespace octo {

// A maximum of accumulators ignores NaN (as bias and activation by fmaxf do one by one), one of SiLU's results keeps it.  In assembly:
// fmaxf would quiet both operands first, three instructions for one.
template <bool KEEP_NAN>
__device__ __forceinline__ float max3_raw(float a, float b, float c) {
  float r;
  if constexpr (KEEP_NAN) asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  else asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
constexpr int SP_STRIP = 64, SP_POOLED = 31; // convolution columns per strip; pooled ones: windows 2 l .. 2 l + 2
constexpr int SP_PAIRS = 8, SP_ROW = 68, SP_PAIR = 2 * SP_ROW * 16;      // ring of row pairs; vectors of a row (a half: even, odd); bytes of a pair

// PLAIN: no SiLU and a multiple of 8 channels; with the pool the other code would cost the row loop registers that it has not got
template <typename T, int BC, int KH, int PKW, bool POOL, bool PLAIN>
__device__ __forceinline__ void stem_walk(const ConvKernelArgs& a) {
  using E = Elem<T>;
  static_assert(sizeof(T) == 2 && E::N == 8, "pixel pairs are 16-byte vectors of 8 values");
  constexpr int TC = BC / 32, NV = KH * PKW, NJ = NV / 2, PD = 3, NP = (KH + 1) / 2;
  constexpr bool BY_ROWS = PKW % 2 != 0;     // the two vectors of an MFMA step: of two rows of a pair, or neighbours in a row
  static_assert(BY_ROWS ? KH % 2 == 0 : true, "an even number of vectors");
  constexpr int AHEAD = SP_PAIRS - NP;       // rows between a pair's fetch and its first use
  constexpr int STORES = POOL ? AHEAD / 2 * 2 * TC : AHEAD * 4 * TC;      // stores of that many rows
  static_assert(AHEAD * 3 + STORES < 64, "counter");
  __shared__ __attribute__((aligned(1024))) unsigned char ring_all[4 * SP_PAIRS * SP_PAIR];
  __shared__ __attribute__((aligned(16))) float sBias[BC];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, g = lane >> 5;
  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  constexpr int WIDTH = POOL ? SP_POOLED : SP_STRIP;         // of a strip, and the size it is cut from
  const int out_w = POOL ? a.pool_wo : a.Wo, out_h = POOL ? a.pool_ho : a.Ho;
  const int strips = (out_w + WIDTH - 1) / WIDTH, seg = a.stem_seg, segs = (out_h + seg - 1) / seg, per_img = strips * segs;
  const int n_units = n_items * per_img;     // < 2^31 (host)
  const bool is_silu = !(POOL && PLAIN) && a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;
  unsigned char* ring = ring_all + wave * (SP_PAIRS * SP_PAIR);
  const unsigned lds = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)ring);

  // weights -> registers, once; row m of a 32-channel operand is channel 16 ((m / 4) % 2) + 4 (m / 8) + m % 4: register 4 q + e of half g
  // of a lane is channel 16 g + 4 q + e of the block (rows beyond Cout are zero in the packed matrix)
  u32x4 wreg[TC][NJ];
  {
    const long long w_bytes = (long long)a.w_rows * a.Kp * 2;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)(w_bytes < BUF_MAX ? w_bytes : BUF_MAX), BUF_FLAGS);
    const int row = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int v = BY_ROWS ? (2 * (j / PKW) + g) * PKW + j % PKW : 2 * j + g;
        wreg[i][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, ((i * 32 + row) * a.Kp + v * 8) * 2, 0, 0);
      }
    if (tid < BC) sBias[tid] = a.bias[tid];
  }
  __syncthreads();

  // operand reads; with the pool column 2 l + tp + s of a row is vector l + (tp + s) / 2 of its even or odd half, and s = 2 (j % 2) + g
  int bbase[2];
#pragma unroll
  for (int tp = 0; tp < 2; ++tp)
    bbase[tp] = (POOL ? ((tp + g) & 1) * (SP_ROW / 2) + l32 + ((tp + g) >> 1) : tp * 32 + l32 + g * (BY_ROWS ? SP_ROW : 1)) * 16;
  const long long img_elems = (long long)a.H * a.W * 8;
  const int img_bytes = (int)(img_elems * 2), row_bytes = a.W * 16;          // fits (host)
  const bool tail = !(POOL && PLAIN) && a.Cout % 8 != 0;
  const int cs = (lane >> 4) * 8;            // channels of the vector this lane stores, of pixel lane % 16 (see swap_rows16)

  // 32 pixels x 32 channels, two vectors of consecutive channels per lane, to row y0 of the output
  auto store_block = [&](const __amdgpu_buffer_rsrc_t& ry, u32x4 (&out)[2], int i, int col0, int cols, int ld) __attribute__((always_inline)) {
    swap_rows16(out[0], out[1]);
    const int c = i * 32 + cs;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int pc = col0 + v * 16 + (lane & 15);
      const int yo = pc < cols ? (pc * ld + c) * 2 : OOB;
      __builtin_amdgcn_raw_buffer_store_b128(out[v], ry, c + 8 <= a.Cout ? yo : OOB, 0, 0);
      if (tail && a.Cout > i * 32 && a.Cout < i * 32 + 32) {           // the vector that ends past the last channel: value by value
        const int to = c < a.Cout && c + 8 > a.Cout ? yo : OOB;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e < a.Cout % 8) __builtin_amdgcn_raw_buffer_store_b16((short)(out[v][e / 2] >> (e % 2 * 16)), ry, to + e * 2, 0, 0);
      }
    }
  };

  // runs of four units (one per wavefront) go round the dies
  for (int unit = blockIdx.x * 4 + wave; unit < n_units; unit += gridDim.x * 4) {
    const int img = unit / per_img, rem = unit - img * per_img, sx = rem / segs, sy = rem - sx * segs;
    const int px0 = sx * WIDTH, py0 = sy * seg, py1 = py0 + seg < out_h ? py0 + seg : out_h;
    // convolution columns and rows; with the pool a segment also computes the row that its first windows share with the segment above,
    // and its last row may lie outside
    const int ox0 = POOL ? 2 * px0 - 1 : px0, ys = POOL ? (py0 > 0 ? 2 * py0 - 1 : 0) : py0, ye = POOL ? 2 * py1 - 1 : py1 - 1;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)((const T*)a.x + a.x_coff + (long long)img * img_elems), 0, img_bytes, BUF_FLAGS);
    // loader: vector p = 64 k + lane of a pair; columns outside the image read as zeros, and so do rows, whose offsets lie outside the buffer
    int loff[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int p = k * 64 + lane, sub = p >= SP_ROW ? 1 : 0, pos = p - sub * SP_ROW;
      const int col = !POOL ? pos : pos < SP_ROW / 2 ? 2 * pos : 2 * (pos - SP_ROW / 2) + 1, ix = ox0 - a.pad_w + col;
      loff[k] = col < SP_STRIP + PKW - 1 && (unsigned)ix < (unsigned)a.W ? (sub * a.W + ix) * 16 : OOB;
    }
    const int last_pair = ye + NP - 1;
    auto load_pair = [&](int q) __attribute__((always_inline)) {       // input rows 2 q - pad, 2 q + 1 - pad
      const int base = (2 * q - a.pad_h) * row_bytes;
      const unsigned at = lds + (unsigned)(q & (SP_PAIRS - 1)) * SP_PAIR;
      const bool any = q <= last_pair;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int off = any && loff[k] != OOB ? loff[k] + base : OOB;
        if (k < 2 || lane < 2 * SP_ROW - 128)
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(at + k * 1024), "v"(off), "s"(rx) : "memory");
      }
    };
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll 1
    for (int q = ys; q < ys + SP_PAIRS - 1; ++q) load_pair(q);

    // pool: columns outside the image do not take part - convolution column -1, and the last one plus 1 of an odd width
    const bool edge = px0 == 0 || 2 * (px0 + SP_POOLED) > a.Wo, col_in = (unsigned)(ox0 + 2 * l32) < (unsigned)a.Wo;
    float run[POOL ? TC : 1][16];            // maximum over the window's rows so far
    if constexpr (POOL) {
#pragma unroll
      for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int k = 0; k < 16; ++k) run[i][k] = -INFINITY;
    }
    for (int y = ys; y <= ye; ++y) {
      load_pair(y + SP_PAIRS - 1);           // into the place of the pair that the row before used last
      // Younger than this row's last pair: the loads of the AHEAD pairs after it, and the stores of the AHEAD rows before this one, if there
      // were that many (with the pool those of a second row each: AHEAD rows are sure to hold that many from row AHEAD + 1 on)
      if (y - ys >= AHEAD + (POOL ? 1 : 0)) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * AHEAD + STORES) : "memory");
      else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * AHEAD) : "memory");
      floatx16 acc[TC][2];
#pragma unroll
      for (int i = 0; i < TC; ++i)
#pragma unroll
        for (int tp = 0; tp < 2; ++tp)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][tp][r] = 0.0f;
      u32x4 fb[PD][2];
      auto read = [&](int j) __attribute__((always_inline)) {
        const int row = BY_ROWS ? 2 * (j / PKW) : 2 * j / PKW, s = BY_ROWS ? j % PKW : 2 * j % PKW;      // of half 0
        const unsigned char* p = ring + ((y + row / 2) & (SP_PAIRS - 1)) * SP_PAIR;
#pragma unroll
        for (int tp = 0; tp < 2; ++tp) fb[j % PD][tp] = *(const u32x4*)(p + bbase[tp] + (row & 1) * (SP_ROW * 16) + (POOL ? s / 2 : s) * 16);
      };
#pragma unroll
      for (int j = 0; j < PD - 1; ++j) read(j);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j + PD - 1 < NJ) read(j + PD - 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int tp = 0; tp < 2; ++tp) acc[i][tp] = E::mfma(wreg[i][j], fb[j % PD][tp], acc[i][tp]);
        __builtin_amdgcn_sched_barrier(0);
      }
      typedef T t4 __attribute__((ext_vector_type(4)));
      if constexpr (!POOL) {
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y + (((size_t)img * a.Ho + y) * a.Wo + px0) * a.y_ld + a.y_coff), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
        for (int i = 0; i < TC; ++i)
#pragma unroll
          for (int tp = 0; tp < 2; ++tp) {
            u32x4 out[2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const floatx4 b4 = *(const floatx4*)&sBias[i * 32 + g * 16 + q * 4];
              t4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float v = fmaxf(acc[i][tp][q * 4 + e] + b4[e], act_lo);
                o[e] = (T)(is_silu ? silu(v) : v);
              }
              const u32x2 ob = __builtin_bit_cast(u32x2, o);
              out[q / 2][q % 2 * 2] = ob[0]; out[q / 2][q % 2 * 2 + 1] = ob[1];
            }
            store_block(ry, out, i, tp * 32, a.Wo - px0, a.y_ld);
          }
      } else {
        // the matrix results are read by inline assembly below: wait states that the compiler would insert for its own instructions
#pragma unroll
        for (int i = TC - 1; i >= 0; --i) {
          if (i == TC - 1) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(acc[i][0]), "+v"(acc[i][1]));
          else asm volatile("" : "+v"(acc[i][0]), "+v"(acc[i][1]));
        }
        if (is_silu) {
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const floatx4 b4 = *(const floatx4*)&sBias[i * 32 + g * 16 + q * 4];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][tp][q * 4 + e] = silu(fmaxf(acc[i][tp][q * 4 + e] + b4[e], -INFINITY));
              }
        }
        if (edge) {
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[i][0][k] = col_in ? acc[i][0][k] : -INFINITY;
        }
        // horizontal maximum of columns 2 l, 2 l + 1 and the next lane's 2 l (lane 31 of a half has no next one, and no pooled column)
        auto across = [&](auto keep_nan) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int k = 0; k < 16; ++k) {
              const float c0 = acc[i][0][k];
              const float next = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(c0), 0x130, 0xF, 0xF, true));
              acc[i][0][k] = max3_raw<keep_nan.value>(c0, acc[i][1][k], next);
            }
        };
        if (is_silu) across(std::true_type{});
        else across(std::false_type{});
        if (y >= a.Ho) {                     // the last row of an odd height is missing
#pragma unroll
          for (int i = 0; i < TC; ++i) acc[i][0] = -INFINITY;
        }
        // the window's rows so far
        auto down = [&](auto keep_nan) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int k = 0; k < 16; ++k) run[i][k] = max3_raw<keep_nan.value>(run[i][k], acc[i][0][k], acc[i][0][k]);
        };
        if (is_silu) down(std::true_type{});
        else down(std::false_type{});
        if (!(y & 1) || (y == ys && py0 > 0)) continue;    // the first row of a pair, or the row shared with the segment above
        // row y ends the windows of pooled row y / 2 and begins those of the next
        const int cols = px0 + SP_POOLED < a.pool_wo ? SP_POOLED : a.pool_wo - px0;
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
            (void*)((T*)a.pool_y + (((size_t)img * a.pool_ho + (y >> 1)) * a.pool_wo + px0) * a.pool_ld + a.pool_coff), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
        for (int i = 0; i < TC; ++i) {
          u32x4 out[2];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const floatx4 b4 = *(const floatx4*)&sBias[i * 32 + g * 16 + q * 4];
            t4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int k = q * 4 + e;
              o[e] = (T)(is_silu ? run[i][k] : fmaxf(run[i][k] + b4[e], act_lo));
              run[i][k] = acc[i][0][k];
            }
            const u32x2 ob = __builtin_bit_cast(u32x2, o);
            out[q / 2][q % 2 * 2] = ob[0]; out[q / 2][q % 2 * 2 + 1] = ob[1];
          }
          store_block(ry, out, i, 0, cols, a.pool_ld);
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the last loads write into LDS
}

template <typename T, int BC, int KH, int PKW, bool POOL>
__global__ __launch_bounds__(THREADS, 2) void stem_conv_kernel(const ConvKernelArgs a) { stem_walk<T, BC, KH, PKW, POOL, true>(a); }
template <typename T, int BC, int KH, int PKW>
__global__ __launch_bounds__(THREADS, 2) void stem_pool_any_kernel(const ConvKernelArgs a) { stem_walk<T, BC, KH, PKW, true, false>(a); }

template <typename T, int BC, int KH, int PKW, bool POOL>
static hipError_t launch_stem_cfg(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (kernel_id) *kernel_id = stem_kernel_id(BC, KH, PKW, POOL);
  ConvArgs b = a;
  const int out_w = POOL ? a.pool_wo : a.Wo, out_h = POOL ? a.pool_ho : a.Ho, width = POOL ? SP_POOLED : SP_STRIP;
  const long long strips = (out_w + width - 1) / width;
  const long long items = a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n;       // expected
  b.stem_seg = stem_segment(out_h, items * strips, 8LL * num_cu, POOL);
  const long long units = out_h > 0 ? (long long)a.n * strips * ((out_h + b.stem_seg - 1) / b.stem_seg) : 0;
  if (units <= 0) return hipSuccess;
  if (units >= 0x7FFF0000LL) return hipErrorNotSupported;
  long long grid = ((units + 3) / 4 + 7) / 8 * 8;
  if (grid > 2LL * num_cu) grid = 2LL * num_cu;
  void (*kernel)(ConvKernelArgs) = stem_conv_kernel<T, BC, KH, PKW, POOL>;
  if constexpr (POOL) {
    if (a.act == OCTO_ACT_SILU || a.Cout % 8 != 0) kernel = stem_pool_any_kernel<T, BC, KH, PKW>;
  }
  if (tm.start && tm.stop) hipExtLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(THREADS), 0, s, tm.start, tm.stop, 0, b);
  else hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(THREADS), 0, s, b);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_stem_typed(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (a.pool_y) {
    if (a.kh != 7 || a.kw != 4 || a.Cout > 64) return hipErrorNotSupported;
    return launch_stem_cfg<T, 64, 7, 4, true>(a, num_cu, s, kernel_id, tm);
  }
  if (a.kh == 7 && a.kw == 4 && a.Cout <= 64) return launch_stem_cfg<T, 64, 7, 4, false>(a, num_cu, s, kernel_id, tm);
  if (a.kh == 6 && a.kw == 3 && a.Cout <= 32) return launch_stem_cfg<T, 32, 6, 3, false>(a, num_cu, s, kernel_id, tm);
  if (a.kh == 6 && a.kw == 3 && a.Cout <= 64) return launch_stem_cfg<T, 64, 6, 3, false>(a, num_cu, s, kernel_id, tm);
  if (a.kh == 3 && a.kw == 2 && a.Cout <= 32) return launch_stem_cfg<T, 32, 3, 2, false>(a, num_cu, s, kernel_id, tm);
  return hipErrorNotSupported;
}

// Pixel-pair first layers in the 16-bit types, stride 2, with one of the kernel shapes above, 16-byte aligned output
// rows and no residual; anything else is left to the general kernel (hipErrorNotSupported).  With a fused max-pool:
// the 7x7 shape only, pooled size (Ho + 1) / 2 x (Wo + 1) / 2, 16-byte aligned pooled rows.
hipError_t launch_stem(int dtype, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm) {
  if (!a.pair_view || (dtype != OCTO_F16 && dtype != OCTO_BF16) || a.stride_h != 2 || a.stride_w != 1 || a.Cin != 8 || a.x_ld != 8 || a.res || a.out_f32)
    return hipErrorNotSupported;
  if (a.pool_y) {
    if (a.pool_ho != (a.Ho + 1) / 2 || a.pool_wo != (a.Wo + 1) / 2 || ((a.pool_ld | a.pool_coff) & 7) || ((uintptr_t)a.pool_y & 15)) return hipErrorNotSupported;
  } else if (((a.y_ld | a.y_coff) & 7) || ((uintptr_t)a.y & 15)) {
    return hipErrorNotSupported;
  }
  if (((uintptr_t)a.x & 15) || (a.x_coff & 7)) return hipErrorNotSupported;
  if ((long long)a.H * a.W * 16 > BUF_MAX || a.w_rows < 64) return hipErrorNotSupported;
  return dtype == OCTO_F16 ? launch_stem_typed<_Float16>(a, num_cu, s, kernel_id, tm) : launch_stem_typed<__bf16>(a, num_cu, s, kernel_id, tm);
}

}  // namespace octo
