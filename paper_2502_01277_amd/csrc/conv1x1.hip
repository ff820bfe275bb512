// 1x1 / stride-1 convolution of large maps with short reductions: a stream of pixels past resident weights.
//
// Such a layer (96 -> 96 on 32 x 160 x 160) moves as many bytes as a copy and multiplies little.  The general kernel
// (conv.hip) fetches the weights again for every tile - more bytes than the tile's pixels - and runs fetch, K steps,
// epilogue and write-out one after the other between barriers: 2.9 TB/s where a copy does 4.7.  Here
//   * a workgroup keeps the weights of its BC = 32 TC output channels in LDS for its lifetime;
//   * every wavefront works on its own on blocks of 32 pixels: it fetches a block (and the residual's) with direct-to-LDS
//     loads, 1 KB of consecutive memory per instruction, multiplies, and requests its next block as soon as the operands
//     are in registers, so the fetch runs beside the epilogue and the stores.  No barrier after the first;
//   * weight rows are permuted so that a lane of the matrix instruction's result holds 16 consecutive channels of its pixel:
//     results leave as 16-byte stores, 64 consecutive bytes per pixel and instruction (see swap_rows16), without a detour
//     through LDS.
// LDS rows (a pixel's or an output channel's K values) have an odd pitch in 16-byte vectors: reads of one vector of 32
// rows hit all banks evenly.
#include "mfma_common.h"
#include "conv_small_choice.h"
#include <hip/hip_ext.h>

namespace octo {

struct StreamGeom {
  int waves;             // wavefronts per workgroup
  int kvp, rvp;          // LDS pitch in vectors: a row of K values, a pixel's BC residual values (0: no residual)
  int x_vecs, r_vecs;    // vectors of a wavefront's pixel block and residual block, whole passes of 64
  int w_vecs;            // weights, whole passes of all lanes
  int tiles_c, lanes;    // channel tiles; workgroups per die that share a channel tile
  FastDiv div_k, div_r;  // by kvp, rvp
};

// channel (within a block of 32) that row m of the matrix instruction computes: result register 4 q + e of half g of the
// wavefront is row 8 q + 4 g + e, and shall be channel 16 g + 4 q + e
__device__ __forceinline__ int row_channel(int m) { return 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3); }

template <typename T, int TC>
__global__ __launch_bounds__(512) void conv1x1_stream_kernel(const ConvKernelArgs a, const StreamGeom gm) {
  using E = Elem<T>;
  static_assert(sizeof(T) == 2, "16-bit storage types");
  constexpr int BC = 32 * TC;
  extern __shared__ __attribute__((aligned(1024))) unsigned char dyn_lds[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  u32x4* sW = (u32x4*)dyn_lds;
  float* sBias = (float*)(sW + gm.w_vecs);
  u32x4* sX = (u32x4*)(sBias + BC) + wave * (gm.x_vecs + gm.r_vecs);
  u32x4* sR = sX + gm.x_vecs;

  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int M = n_items * a.Ho * a.Wo;                   // < 2^31 (host)
  const int n_blk = (M + 31) >> 5;
  // A workgroup takes runs of as many consecutive blocks as it has wavefronts; the runs go round the dies (workgroup b runs on die b % 8),
  // so that the chip reads and writes one window of memory at a time: 64 -> 64 on 64 x 160 x 160 85 -> 81 us against a contiguous piece
  // of the tensor for every die, 64 -> 256 with residual on 119 x 64 x 32 63 -> 57.  The workgroups of the channel tiles of one pixel
  // range are neighbours on a die and advance together, so they meet in its L2
  const int die = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int ct = j % gm.tiles_c, pl = j / gm.tiles_c;
  if (pl >= gm.lanes) return;
  const int stride = gm.lanes * 8 * gm.waves;
  int blk = (pl * 8 + die) * gm.waves + wave;
  const int c0 = ct * BC, cs = c0 + (lane >> 4) * 8;     // channels of the vector this lane stores, of pixel lane % 16
  const int kv = a.Cin >> 3;                             // vectors per pixel

  // weights, once
  {
    const long long w_bytes = (long long)a.w_rows * a.Kp * 2;
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)(w_bytes < BUF_MAX ? w_bytes : BUF_MAX), BUF_FLAGS);
    for (int i = tid; i < gm.w_vecs; i += 64 * gm.waves) {
      const int m = (int)fast_div((unsigned)i, gm.div_k), v = i - m * gm.kvp;
      const int c = c0 + (m & ~31) + row_channel(m & 31);
      sW[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, m < BC && v < kv && c < a.w_rows ? (c * a.Kp + v * 8) * 2 : OOB, 0, 0);
    }
    for (int i = tid; i < BC; i += 64 * gm.waves) sBias[i] = c0 + i < a.w_rows ? a.bias[c0 + i] : 0.0f;
  }
  // a block's rows into LDS, `vecs` / 64 passes of 1 KB; bytes past the tensor's end and pitch padding read as zeros
  auto fetch = [&](const T* base, int ld, long long rows_left, int row_vecs, int pitch, const FastDiv& div, u32x4* dst, int vecs) {
    const long long bytes = rows_left * ld * 2;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)(bytes < BUF_MAX ? bytes : BUF_MAX), BUF_FLAGS);
    const unsigned lds = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)dst);
    for (int ps = 0; ps < vecs / 64; ++ps) {
      const int i = ps * 64 + lane;
      const int r = (int)fast_div((unsigned)i, div), v = i - r * pitch;
      const int off = r < 32 && v < row_vecs ? (r * ld + v * 8) * 2 : OOB;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(lds + ps * 1024), "v"(off), "s"(rsrc) : "memory");
    }
  };
  // buffers end where the last row's own channels end (the tensor may be a channel slice of a wider one)
  const T* xg = (const T*)a.x + a.x_coff;
  const T* rg = (const T*)a.res + a.res_coff + c0;
  auto fetch_x = [&](int b) { fetch(xg + (size_t)b * 32 * a.x_ld, a.x_ld, M - b * 32 < 32 ? M - b * 32 : 32, kv, gm.kvp, gm.div_k, sX, gm.x_vecs); };
  const int res_vecs = a.Cout - c0 < BC ? (a.Cout - c0) >> 3 : BC >> 3;
  auto fetch_r = [&](int b) { fetch(rg + (size_t)b * 32 * a.res_ld, a.res_ld, M - b * 32 < 32 ? M - b * 32 : 32, res_vecs, gm.rvp, gm.div_r, sR, gm.r_vecs); };
  const bool has_res = a.res && a.res_mode != OCTO_RES_NONE;
  if (blk < n_blk) { fetch_x(blk); if (has_res) fetch_r(blk); }
  __syncthreads();                                       // the weights are in place

  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;
  const int nkk = (kv + 1) >> 1;
  const u32x4* pa = sW + l32 * gm.kvp + g;
  const u32x4* pb = sX + l32 * gm.kvp + g;
  const int wstep = 32 * gm.kvp;
  for (; blk < n_blk; blk += stride) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    floatx16 acc[TC];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
    for (int kk = 0; kk < nkk; ++kk) {
      const u32x4 fb = pb[2 * kk];
#pragma unroll
      for (int i = 0; i < TC; ++i) acc[i] = E::mfma(pa[i * wstep + 2 * kk], fb, acc[i]);
    }
    const int next = blk + stride;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the block's operands have been read: its buffer takes the next one
    if (next < n_blk) fetch_x(next);

    const int p0 = blk * 32;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y + a.y_coff + (size_t)p0 * a.y_ld), 0, (int)BUF_MAX, BUF_FLAGS);
    const __amdgpu_buffer_rsrc_t ry2 = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)a.y2 + a.y2_coff - a.split + (size_t)p0 * a.y2_ld), 0, (int)BUF_MAX, BUF_FLAGS);
    int yo[2], yo2[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int pl = h * 16 + (lane & 15);
      yo[h] = p0 + pl < M ? (pl * a.y_ld + cs) * 2 : OOB; yo2[h] = p0 + pl < M ? (pl * a.y2_ld + cs) * 2 : OOB;
    }
    with_epilogue_mode(has_res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
      constexpr int RES = decltype(res_c)::value;
      constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
      for (int i = 0; i < TC; ++i) {
        u32x4 out[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int cl = i * 32 + g * 16 + h * 8;        // eight consecutive channels
          typedef T t8 __attribute__((ext_vector_type(8)));
          t8 r8 = {};
          if (RES != OCTO_RES_NONE) r8 = __builtin_bit_cast(t8, sR[l32 * gm.rvp + (cl >> 3)]);
          t8 o8;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const floatx4 b4 = *(const floatx4*)(sBias + cl + q * 4);
            floatx4 v, rv;
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = acc[i][h * 8 + q * 4 + e]; rv[e] = (float)r8[q * 4 + e]; }
            v = finish4<RES, SILU>(v, b4, rv, act_lo);
#pragma unroll
            for (int e = 0; e < 4; ++e) o8[q * 4 + e] = (T)v[e];
          }
          out[h] = __builtin_bit_cast(u32x4, o8);
        }
        swap_rows16(out[0], out[1]);
        // two layers in one launch: a block of 32 channels belongs to one of them, or (a split that is a multiple of 8 only) each vector to its own
        const int left = a.split - c0 - i * 32;
        const bool any = cs + i * 32 < a.Cout, second = a.split > 0 && cs + i * 32 >= a.split;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (a.split == 0 || left > 0) __builtin_amdgcn_raw_buffer_store_b128(out[h], ry, any && !second ? yo[h] + i * 64 : OOB, 0, 0);
          if (a.split > 0 && left < 32) __builtin_amdgcn_raw_buffer_store_b128(out[h], ry2, any && second ? yo2[h] + i * 64 : OOB, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);               // one block of channels at a time: keeps the register demand low
      }
      if (RES != OCTO_RES_NONE) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (next < n_blk) fetch_r(next);
      }
    });
  }
}

constexpr int STREAM_LDS = 160 * 1024;

// Geometry of a launch with BC = 32 tc channels per workgroup; 0 wavefronts when it does not fit.
inline StreamGeom stream_geometry(const ConvArgs& a, int tc, int num_cu, size_t* lds) {
  StreamGeom g{};
  const int kv = a.Cin / 8, bc = 32 * tc;
  const bool res = a.res && a.res_mode != OCTO_RES_NONE;
  g.kvp = ((kv + 1) & ~1) + 1;
  g.rvp = res ? bc / 8 + 1 : 1;
  g.x_vecs = (32 * g.kvp + 63) / 64 * 64;
  g.r_vecs = res ? (32 * g.rvp + 63) / 64 * 64 : 0;
  g.w_vecs = (bc * g.kvp + 63) / 64 * 64;
  const int fixed = g.w_vecs * 16 + bc * 4, per_wave = (g.x_vecs + g.r_vecs) * 16;
  g.waves = (STREAM_LDS - fixed) / per_wave;
  if (g.waves > 8) g.waves = 8;
  *lds = (size_t)fixed + (size_t)g.waves * per_wave;
  g.tiles_c = (a.Cout + bc - 1) / bc;
  g.div_k = make_fastdiv((unsigned)g.kvp); g.div_r = make_fastdiv((unsigned)g.rvp);
  return g;
}

template <typename T, int TC>
static hipError_t launch_stream_cfg(const ConvArgs& a, long long M, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  size_t lds;
  StreamGeom g = stream_geometry(a, TC, num_cu, &lds);
  if (g.waves < 3) return hipErrorNotSupported;
  static const bool ready = [] {
    (void)hipFuncSetAttribute((const void*)conv1x1_stream_kernel<T, TC>, hipFuncAttributeMaxDynamicSharedMemorySize, STREAM_LDS);
    (void)hipGetLastError();
    return true;
  }();
  (void)ready;
  // two workgroups per compute unit while the tensors fit the 256 MB memory-side cache; beyond it one streams better
  // (48 -> 48 on 32 x 320 x 320, 630 MB: 128 against 144 us)
  const bool cached = (double)M * (a.Cin + a.Cout * (g.r_vecs ? 2 : 1)) * 2 < 256e6;
  const int per_cu = lds <= STREAM_LDS / 2 && cached ? 2 : 1;
  const int per_die = num_cu * per_cu / 8;
  if (g.tiles_c > per_die) return hipErrorNotSupported;
  g.lanes = per_die / g.tiles_c;
  if (kernel_id) *kernel_id = stream1_kernel_id(TC, a.Cin);
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv1x1_stream_kernel<T, TC>), dim3((unsigned)(8 * per_die)), dim3(64 * g.waves), (unsigned)lds, s, tm.start, tm.stop, 0, a, g);
  else
    hipLaunchKernelGGL((conv1x1_stream_kernel<T, TC>), dim3((unsigned)(8 * per_die)), dim3(64 * g.waves), (unsigned)lds, s, a, g);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_stream_typed(const ConvArgs& a, long long M, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (a.Cout <= 32) return launch_stream_cfg<T, 1>(a, M, num_cu, s, kernel_id, tm);
  if (a.Cout > 64 && a.Cout % 96 == 0) return launch_stream_cfg<T, 3>(a, M, num_cu, s, kernel_id, tm);
  if (a.Cout >= 256 && a.Cin <= 64) return launch_stream_cfg<T, 4>(a, M, num_cu, s, kernel_id, tm);
  return launch_stream_cfg<T, 2>(a, M, num_cu, s, kernel_id, tm);
}

// 1x1 / stride-1 layers in the 16-bit types with at most 192 input channels and a block of pixels for every other
// wavefront of the chip; hipErrorNotSupported otherwise.  Longer reductions have work enough per byte for the larger tiles of
// conv_flow_kernel (flow_takes_1x1 has the line; 384 -> 192 on 80 x 80 took 63 us on the general kernel and 95 here), and channel counts
// that are no multiple of 8 would have their last vectors written element by element.  The sums are those of both other kernels.
// Bound by memory.  Measured, bf16, with stores of 32 consecutive bytes per pixel and a contiguous piece of the tensor for every die, and
// now: 96 -> 96 on 32 x 160 x 160 84 -> 68 us (4.6 TB/s; a copy of that size does 5.3), on 32 x 320 x 320 300 -> 249 (5.0); 64 -> 64 on
// 64 x 160 x 160 103 -> 81; 64 -> 256 with residual on 119 x 64 x 32 74 -> 57.  A second block per wavefront in flight gave nothing.
hipError_t launch_conv1x1_stream(int dtype, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm) {
  if ((dtype != OCTO_F16 && dtype != OCTO_BF16) || a.pair_view || a.pool_y || a.up_y || a.out_f32 || a.kh != 1 || a.kw != 1 || a.stride_h != 1 || a.stride_w != 1 ||
      a.pad_h || a.pad_w || a.Cin > 192 || a.Cin < 16)
    return hipErrorNotSupported;
  if (((a.Cin | a.x_ld | a.x_coff | a.Cout | a.y_ld | a.y_coff) & 7) || (((uintptr_t)a.x | (uintptr_t)a.y) & 15)) return hipErrorNotSupported;
  if (a.res && (((a.res_ld | a.res_coff) & 7) || ((uintptr_t)a.res & 15))) return hipErrorNotSupported;
  // Below the line lies the split-K kernel too, which sums in another order: as everywhere, that choice is made for a.n_split items where the
  // count is taken on the device, and not for the running one
  const long long hw = (long long)a.Ho * a.Wo, M = (a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * hw;
  const long long M_split = a.n_split > 0 ? (a.n_split < a.n ? a.n_split : a.n) * hw : M;
  if (flow_takes_1x1(a, M_split)) return hipErrorNotSupported;
  // Several channel tiles read the pixels several times and need more of them.  Us, by blocks times channel tiles of 64 per compute unit.
  // Here : conv_flow_kernel (32 channels: general): 16 -> 32 at 3 3.9 : 4.6; 32 -> 64 at 2 4.8 : 4.5, at 3 4.9 : 5.5, at 4 5.1 : 6.1; 96 -> 64 at 3
  // 5.7 : 5.8, at 4 5.9 : 6.6; 32 -> 96 at 4 5.6 : 5.1, at 5 5.6 : 6.0; 96 -> 192 at 5 6.9 : 6.7, at 6 7.1 : 6.9, at 7 7.2 : 7.5; 120 -> 128 at 4 6.2 : 5.7,
  // at 5 6.5 : 6.8.
  // In their place in a cascade, where the input comes from beyond the L2s, here : conv_small_kernel: 96 -> 96 at 6.2 9.9 : 6.7, at 25 14.0 : 15.6.
  // 64 input channels, a whole K step, go to conv_small_kernel for longer, where it takes them (here : there): alone 64 -> 128 at 6.2 6.1 : 5.2, at 7.7
  // 6.4 : 5.5, 64 -> 16 at 7 4.3 : 3.6, 64 -> 32 at 10.5 5.8 : 4.5; in place 64 -> 64 at 12.5 11.8 : 8.3, at 25 14.5 : 11.4, at 50 21.3 : 21.3, at 100 43.7 : 42.4, in
  // two tensors at 12.5 13.1 : 9.9, at 50 21.2 : 19.7, at 100 49.2 : 53.3; 64 -> 256 at 48 18.4 : 16.5 (conv_flow_kernel), with residual 19.9 : 18.1, at
  // 192 37.0 : 40.8; 64 -> 32 at 6.4 5.7 : 5.1, at 16 7.9 : 7.1, at 33 11.8 : 11.1, with residual at 41 16.7 : 14.8, at 59 15.7 : 15.1, 64 -> 8 at 72 16.3 : 17.1.
  // Up to 32 channels before an upsampling, or of items counted on the device, have only the general kernel below the line (64 -> 32 in place at 6.4
  // 5.7 : 7.1, at 33 11.8 : 14.5; alone at 7 4.3 : 5.4).
  // A count on the device that runs beyond the line of a layer in place, while the stated one lies between that line and the one alone, goes by the running
  // count: this kernel, conv_small_kernel and conv_flow_kernel sum in one order, and above the line alone nothing is split (here : what the stated count alone would
  // give, twice as many items as stated: 64 -> 640 on 15 x 57 x 57 21.4 : 32.4, 16 -> 80 with residual on 278 x 14 x 14 8.7 : 11.3, 96 -> 288 on 580 x 7 x 7 12.0 : 14.8).
  const bool step = a.Cin == 64 && small_fits(a, 2) && (a.Cout > 32 || (a.n_split == 0 && !a.up_next));
  const long long alone = step ? 9 : a.Cout <= 64 ? 4 : 6, line = !a.in_place ? alone : step ? 48 : a.Cout <= 64 ? 4 : 9;
  auto below = [&](long long m, long long l) { return (m + 31) / 32 * ((a.Cout + 63) / 64) < l * num_cu; };
  if (below(M_split, alone) || (below(M_split, line) && below(M, line))) return hipErrorNotSupported;
  return dtype == OCTO_F16 ? launch_stream_typed<_Float16>(a, M, num_cu, s, kernel_id, tm) : launch_stream_typed<__bf16>(a, M, num_cu, s, kernel_id, tm);
}

}  // namespace octo
