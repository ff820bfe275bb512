// Convolution for launches of few tiles, for layers in a cascade whose operands come late, and for fp32 of nearly any size: an implicit GEMM written for few
// instructions per wavefront.  small_limit and small_takes_f32 (conv_small_choice.h) have the lines: up to 1.25 .. 24 tiles of 64 x 64 per compute unit in the
// 16-bit types by the form of the layer, whole K steps of a layer of a model by estimated time without a bound; fp32 1x1 layers up to 64, windows in whole K steps
// at every size and with steps across taps up to 8.
//
// A launch of few tiles is one round of workgroups, and its time is what one of them takes from its first instruction to its last store. A
// wavefront alone on its SIMD issues an instruction every four cycles at best, so that time is mostly a count of instructions: of the
// 3.84 us of conv_flow_kernel on 128 -> 128 over 40 x 40 pixels (64 x 64 tile, two K steps, launches back to back from a graph) 1.23 pass
// between launches, 0.46 go to addresses, 0.34 to the first operands, 0.86 to the two K steps and 0.54 to the epilogue.  Here
//   * all arguments come in one trip to memory, in a block of their own; bias and residual are asked for before the operands, so that
//     nothing is waited for after the K loop;
//   * nothing of the next tile: no second set of addresses, no loads that only keep a count.  Workgroups are two to four per compute unit; where there are more
//     tiles than that (fp32, single K steps, layers of a model, a count on the device larger than expected) those of one follow one another, and the others
//     of its compute unit hide the gap;
//   * the fragments of a step are on their way from LDS while the loads of two steps on are issued; one barrier per step;
//   * blocks of 16 x 16, so that small tiles still have four wavefronts and the epilogue few values per lane.
// Same weights, same LDS layout and, in the 16-bit types, the same sums bit for bit as conv_flow_kernel and the general kernel (a block of 16 x 16 x 32
// adds its products in the order of two of 32 x 32 x 16).  Before (the kernel that took the layer) and after, us, bf16, from a graph: 1x1
// 256 -> 256 on 20 x 20 3.8 -> 2.8, on 5 x 40 x 40 5.4 -> 4.7; 512 -> 512 on 5 x 20 x 20 5.3 -> 4.4; 3x3 64 -> 64 on 5 x 80 x 80 8.2 -> 7.0; stride 2:
// 128 -> 256 on 5 x 80 x 80 11.8 -> 9.4, 256 -> 512 on 8 x 40 x 40 17.2 -> 13.0.
// In fp32 the matrix pipe bounds all but the smallest layers (116 of the 153 TFLOP/s that a large product reaches at 128 -> 384, stride 2 on
// 2 x 160 x 161): three or four workgroups per compute unit hide each other's latency; see conv_small_choice.h for before and after.
// What bounds it in the 16-bit types: between launches 1.2 us; then latency, and from about 20 K steps on what LDS reads take (8 KB per 32 x 32 block and step).
// Measured and left out: rings of four to eight stages, two K steps between barriers (both nothing), two or four groups of wavefronts
// that share K (20 x 20 x 256 -> 256 3x3 7.2 -> 6.7, split-K 5.9; short reductions 0.2 .. 0.5 slower), 128 x 128 tiles.
#pragma once
#include "octo_internal.h"
#include "mfma_common.h"
#include "conv_small_choice.h"
#include <hip/hip_ext.h>

namespace octo {

// One K step (128 bytes per row) of a 16 x 16 block: lane (r16, q4) supplies vectors q4 and 4 + q4 of its row.  In fp32 the values of a step
// go to C chains of sums that are added at the end: an instruction need not wait for the one before, and a chain is as short as a
// wavefront's part of the reduction in the split-K kernel.
template <typename T, int C>
__device__ __forceinline__ void small_step(const u32x4 (&a)[2], const u32x4 (&b)[2], floatx4 (&c)[C]) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if constexpr (std::is_same<T, _Float16>::value) c[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a[k]), __builtin_bit_cast(half8, b[k]), c[0], 0, 0, 0);
    else if constexpr (std::is_same<T, __bf16>::value) c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[k]), __builtin_bit_cast(bf16x8, b[k]), c[0], 0, 0, 0);
    else {
      const floatx4 fa = __builtin_bit_cast(floatx4, a[k]), fb = __builtin_bit_cast(floatx4, b[k]);
#pragma unroll
      for (int e = 0; e < 4; ++e) c[(4 * k + e) % C] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[e], c[(4 * k + e) % C], 0, 0, 0);
    }
  }
}

// BC x BP: tile; WC, WP: wavefronts along the channels and the pixels; MINB: workgroups per compute unit; MODE: how addresses are made
// (SMALL_POINTWISE and what follows it).
template <typename T, int BC, int BP, int WC, int WP, int MODE>
__device__ __forceinline__ void conv_small_tiles(const SmallArgs& a, const int block) {
  constexpr bool PART = MODE == SMALL_PART || MODE == SMALL_STRIDED_PART, PW = MODE == SMALL_POINTWISE || MODE == SMALL_PART;
  constexpr int ES = (int)sizeof(T), VN = 16 / ES, BK = 8 * VN;
  constexpr int NT = 64 * WC * WP, RP = NT / 8, NS = 3;       // lanes, rows that they load per pass, stages of the ring
  constexpr int NB = BC / WC / 16, NP = BP / WP / 16;         // blocks of 16 channels and of 16 pixels of a wavefront
  constexpr int LA = BC / RP, LB = BP / RP, NL = LA + LB, STAGE = (BC + BP) * 128;
  constexpr int NC = ES == 4 ? (NB * NP <= 2 ? 8 : 4) : 1;    // chains of sums
  constexpr int CH = 4 * NB;                                  // consecutive channels of a lane
  constexpr int UQ = ES == 4 ? 1 : (ES == 2 ? (NB < 2 ? NB : 2) : (NB < 4 ? NB : 4)), VC = 4 * UQ, NV = NB / UQ;     // quads and channels of a store, stores
  typedef uint32_t vec __attribute__((ext_vector_type(UQ * ES)));
  static_assert(BC % RP == 0 && BP % RP == 0 && NB >= 1 && NP >= 1 && NB % UQ == 0, "tile shape");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NS * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WC, wp = wave / WC, r16 = lane & 15, q4 = lane >> 4;
  // one trip to memory for all arguments (the compiler would ask for some of them when it needs them)
  asm volatile("" :: "s"(a.x), "s"(a.w), "s"(a.bias), "s"(a.y), "s"(a.res), "s"(a.Cout), "s"(a.x_pitch), "s"(a.w_len), "s"(a.H));
  int n_items = a.n;
  if (a.n_dyn) { const int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const int M = n_items * a.HoWo, tiles_p = (int)((unsigned)(M + BP - 1) / BP), n_tiles = tiles_p * a.tiles_c, per_die = (n_tiles + 7) >> 3;

  // loads: lane t of the workgroup fills slot t % 8 of row t / 8 of a pass; row r keeps vector v in slot v ^ ((r / 2) % 8)
  const int row = tid >> 3, lkv = (tid & 7) ^ ((row >> 1) & 7);
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)smem + (unsigned)wave * 1024u));
  // LDS row m of a wavefront's 16 NB rows holds channel CH (m / 4 % 4) + 4 (m / 16) + m % 4 of them, so a lane gets CH consecutive channels
  int woff[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = row + i * RP, m = r % (16 * NB);
    woff[i] = (r - m + CH * ((m >> 2) & 3) + 4 * (m >> 4) + (m & 3)) * a.per_row + lkv * 16;
  }
  const int fswz = (r16 >> 1) & 7;
  const int fa0 = (wc * 16 * NB + r16) * 128, fb0 = BC * 128 + (wp * 16 * NP + r16) * 128;
  const int fv[2] = {(q4 ^ fswz) << 4, ((4 + q4) ^ fswz) << 4};
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, a.w_len, BUF_FLAGS);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, a.w_rows * 4, BUF_FLAGS);      // padded to whole tiles like the weights

  for (int t = block; t < per_die * 8; t += a.grid) {
    const int tile = (t & 7) * per_die + (t >> 3);       // contiguous chunk of the tile list per die, see conv_mfma_kernel
    if (tile >= n_tiles) continue;
    int tc, tp;
    if (!a.c_outer) { tp = (int)fast_div((unsigned)tile, a.div_tc); tc = tile - tp * a.tiles_c; }
    else {
      if (!a.n_dyn) tc = (int)fast_div((unsigned)tile, a.div_tp);
      else { int d = tiles_p; asm volatile("" : "+s"(d)); tc = (int)((unsigned)tile / (unsigned)d); }      // (opaque: its reciprocal would be taken by every launch)
      tp = tile - tc * tiles_p;
    }
    const int c0 = tc * BC, p0 = tp * BP;
    int wk = c0 * a.per_row;

    // pixels, as in conv_flow_kernel: a buffer that starts at the tile, or at the first image of the tile less the padding
    const char* xb;
    long long x_bytes;
    int voff[LB], rowoff[PW ? 1 : LB];
    unsigned ok[PW ? 1 : LB];
    int xk = 0, ist = 0, l_kb = 0, tr = 0, ts = 0;       // load cursor: scalar offset, stage, step in its tap (SMALL_ANY: of all), tap
    auto open_tap = [&]() __attribute__((always_inline)) {
      if constexpr (!PW) {
        int delta = 0;
        unsigned need = (1u << tr) | (0x10000u << ts);
        if constexpr (MODE == SMALL_ANY) {
          // element k of the reduction is channel c of tap (r, s): k = (r * kw + s) * Cin + c, exact for k < 65536.  24-bit products are four
          // times as fast (their factors fit, small_fits)
          const unsigned k = (unsigned)l_kb * BK + lkv * VN, tap = __umulhi(k, a.magic_cin);
          const unsigned r = a.kw == 1 ? tap : __umulhi(tap, a.magic_kw), s = tap - __umul24(r, (unsigned)a.kw);
          delta = (int)(__umul24(__umul24(r, (unsigned)a.W) + s, (unsigned)a.x_pitch) + (k - __umul24(tap, (unsigned)a.Cin)) * ES);
          need = k < (unsigned)a.K ? (1u << r) | (0x10000u << s) : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) voff[i] = (ok[i] & need) == need ? rowoff[i] + delta : OOB;
      }
    };
    if constexpr (PW) {
      xb = a.x + (long long)p0 * a.x_pitch;
      x_bytes = (long long)(M - p0) * a.x_pitch;
#pragma unroll
      for (int i = 0; i < LB; ++i) voff[i] = (row + RP * i) * a.x_pitch + lkv * 16;
    } else {
      const unsigned img0 = fast_div((unsigned)p0, a.div_howo);
      const long long shift = ((long long)a.pad * a.W + a.pad) * a.x_pitch, img = (long long)a.H * a.W * a.x_pitch;
      xb = a.x + (long long)img0 * img - shift;
      x_bytes = (long long)(a.n - (int)img0) * img + shift;
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int m = p0 + row + RP * i;
        const unsigned im = fast_div((unsigned)m, a.div_howo), rem = (unsigned)m - im * (unsigned)a.HoWo;
        const unsigned ho = fast_div(rem, a.div_wo), wo = rem - ho * (unsigned)a.Wo;
        const int h0 = (int)ho * a.stride - a.pad, w0 = (int)wo * a.stride - a.pad;
        // kernel rows r with 0 <= h0 + r < H form the range [max(0, -h0), min(kh, H - h0)); same for columns
        const int rlo = h0 < 0 ? -h0 : 0, rhi = a.H - h0 < a.kh ? a.H - h0 : a.kh;
        const int slo = w0 < 0 ? -w0 : 0, shi = a.W - w0 < a.kw ? a.W - w0 : a.kw;
        const unsigned rm = rhi > rlo ? ((1u << rhi) - 1u) & ~((1u << rlo) - 1u) : 0u;
        const unsigned sm = shi > slo ? ((1u << shi) - 1u) & ~((1u << slo) - 1u) : 0u;
        rowoff[i] = (((int)(im - img0) * a.H + (int)ho * a.stride) * a.W + (int)wo * a.stride) * a.x_pitch + (MODE == SMALL_ANY ? 0 : lkv * 16);
        ok[i] = m < M ? rm | (sm << 16) : 0u;
      }
      open_tap();
    }
    const int x_len = (int)(x_bytes < BUF_MAX ? x_bytes : BUF_MAX);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)xb, 0, x_len, BUF_FLAGS);
    auto issue = [&]() __attribute__((always_inline)) {
      const unsigned st = lds0 + ist * STAGE;
      // a tap that no pixel of the tile can use may start behind the buffer's end, where a scalar offset must not be (see conv_flow_kernel)
      const int ox = PW ? xk : MODE == SMALL_ANY ? 0 : xk < x_len ? xk : 0;
#pragma unroll
      for (int i = 0; i < LA; ++i)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(st + i * (NT * 16)), "v"(woff[i]), "s"(rw), "s"(wk) : "memory");
      const bool cut = PART && l_kb == a.nk - 1 && lkv * VN >= a.K - (a.nk - 1) * BK;      // behind the last channel
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int vo = cut ? OOB : voff[i];
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(st + BC * 128 + i * (NT * 16)), "v"(vo), "s"(rx), "s"(ox) : "memory");
      }
      ist = ist + 1 == NS ? 0 : ist + 1;
      wk += 128; xk += 128;
      if constexpr (MODE == SMALL_ANY) {
        ++l_kb;
        open_tap();
      } else if constexpr (PART) {
        ++l_kb;
      } else if constexpr (!PW) {
        if (++l_kb == a.taps_nk) {
          l_kb = 0;
          if (++ts == a.kw) { ts = 0; ++tr; }
          xk = (tr * a.W + ts) * a.x_pitch;
          open_tap();
        }
      }
    };
    // what the epilogue needs is asked for first: it has landed with the first operands
    const int cw = c0 + wc * 16 * NB + q4 * CH;          // this lane's first channel
    floatx4 bias[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) bias[b] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rb, (cw + 4 * b) * 4, 0, 0));
    vec rv[NP][NV];
    if (a.res) {
      const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)(a.res + (long long)p0 * a.res_pitch), 0, (int)BUF_MAX, BUF_FLAGS);
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int h = 0; h < NV; ++h) {
          const int pl = (wp * NP + j) * 16 + r16, off = p0 + pl < M && cw + VC * h < a.Cout ? pl * a.res_pitch + (cw + VC * h) * ES : OOB;
          if constexpr (sizeof(vec) == 16) rv[j][h] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(rr, off, 0, 0));
          else if constexpr (sizeof(vec) == 8) rv[j][h] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(rr, off, 0, 0));
          else rv[j][h] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b32(rr, off, 0, 0));
        }
    }
    const int ahead = a.nk < NS - 1 ? a.nk : NS - 1;
    for (int d = 0; d < ahead; ++d) issue();

    floatx4 acc[NB][NP][NC];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[b][j][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    int rst = 0;
    // one K step; `between` runs while its fragments are on their way from LDS
    auto compute = [&](auto between) __attribute__((always_inline)) {
      const unsigned char* p = smem + rst * STAGE;
      u32x4 fa[NB][2], fb[NP][2];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int b = 0; b < NB; ++b) fa[b][kk] = *(const u32x4*)(p + fa0 + b * 2048 + fv[kk]);
#pragma unroll
        for (int j = 0; j < NP; ++j) fb[j][kk] = *(const u32x4*)(p + fb0 + j * 2048 + fv[kk]);
      }
      between();
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < NP; ++j) small_step<T, NC>(fa[b], fb[j], acc[b][j]);
      rst = rst + 1 == NS ? 0 : rst + 1;
    };
    int s = NS - 1;                                      // steps requested
    for (; s < a.nk; ++s) {
      // the stage of the step before is free behind the barrier: every wavefront's fragments of it have returned (lgkmcnt; matrix instructions are
      // no memory accesses, and the compiler may move them, and its own wait for what they read, past this one)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((NS - 2) * NL) : "memory");
      __builtin_amdgcn_s_barrier();
      compute(issue);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    for (s -= NS - 1; s < a.nk; ++s) compute([] {});

    // epilogue: lane (r16, q4) holds CH consecutive channels of pixel r16 of each block
    const bool is_silu = a.act == OCTO_ACT_SILU;
    const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
      constexpr int RES = decltype(res_c)::value;
      constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int pl = (wp * NP + j) * 16 + r16;
#pragma unroll
        for (int h = 0; h < NV; ++h) {
          const int c = cw + VC * h;
          const bool second = a.split > 0 && c >= a.split;       // two layers in one launch: a store never straddles the split (a multiple of 8)
          vec out;
#pragma unroll
          for (int q = 0; q < UQ; ++q) {
            const int b = UQ * h + q;
            floatx4 r4 = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (RES != OCTO_RES_NONE) r4 = load4<T>((const T*)&rv[j][h] + 4 * q);
            floatx4 v = acc[b][j][0];
            if constexpr (NC == 4) v = (v + acc[b][j][1]) + (acc[b][j][2] + acc[b][j][3]);
            if constexpr (NC == 8) v = ((v + acc[b][j][1]) + (acc[b][j][2] + acc[b][j][3])) + ((acc[b][j][4] + acc[b][j][5]) + (acc[b][j][6] + acc[b][j][7]));
            v = finish4<RES, SILU>(v, bias[b], r4, act_lo);
            if constexpr (std::is_same<T, _Float16>::value) {
              // rounded to 32 bits and then to 16, as in the other kernels (the compiler would fuse SiLU's last product with the conversion)
#pragma unroll
              for (int e = 0; e < 4; ++e) asm("" : "+v"(v[e]));
            }
            store4<T>((T*)&out + 4 * q, v);
          }
          if (p0 + pl >= M) continue;
          const int pitch = second ? a.y2_pitch : a.y_pitch;
          char* p = (second ? a.y2 : a.y) + (long long)p0 * pitch + pl * pitch + c * ES;
          if (c + VC <= a.Cout) *(vec*)p = out;
          else {
#pragma unroll
            for (int e = 0; e < VC; ++e) if (c + e < a.Cout) ((T*)p)[e] = ((const T*)&out)[e];
          }
        }
      }
    });
    if (t + a.grid < per_die * 8) __syncthreads();       // the stages may be refilled
  }
}

template <typename T, int BC, int BP, int WC, int WP, int MINB, int MODE>
__global__ __launch_bounds__(64 * WC * WP, MINB * WC * WP / 4) void conv_small_kernel(const SmallArgs a) {
  conv_small_tiles<T, BC, BP, WC, WP, MODE>(a, blockIdx.x);
}
// Up to three layers that do not depend on one another in one launch: the workgroups of one follow those of the one before (SmallGroup, conv_small_choice.h).  A launch of few
// tiles leaves compute units idle and costs 3.5 us whatever it does.  Cascades with separate launches and with a shortcut and the layer beside it, and the heads, as one, us: sweep of 1
// frame 484 -> 475, of 4 605 -> 592, traffic of 8 1050 -> 1024, surveillance of 4 953 -> 944, sweep of 64 3825 -> 3809.
struct SmallGroupArgs { SmallArgs layer[SmallGroup::MAX]; int second, third; };      // their first workgroups, multiples of 8
template <typename T, int BC, int BP, int WC, int WP, int MINB, int MODE>
__global__ __launch_bounds__(64 * WC * WP, MINB * WC * WP / 4) void conv_small_group_kernel(const SmallGroupArgs g) {
  const int b = blockIdx.x, which = b < g.second ? 0 : b < g.third ? 1 : 2, first = which == 0 ? 0 : which == 1 ? g.second : g.third;
  // straight from the arguments' memory: a copy that is indexed would live in scratch
  const SmallArgs a = *(const SmallArgs*)((const char*)__builtin_amdgcn_kernarg_segment_ptr() + which * sizeof(SmallArgs));
  conv_small_tiles<T, BC, BP, WC, WP, MODE>(a, b - first);
}

template <typename T, int BC, int BP, int WC, int WP, int MINB>
static hipError_t launch_small_cfg(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  constexpr int ES = (int)sizeof(T), BK = 128 / ES, NT = 64 * WC * WP;
  const long long M = (long long)a.n * a.Ho * a.Wo, tiles_c = (a.Cout + BC - 1) / BC, tiles_p = (M + BP - 1) / BP, tiles = tiles_p * tiles_c;
  if (tiles <= 0) return hipSuccess;
  if (tiles >= 0x3FFFFFF0LL) return hipErrorNotSupported;
  long long grid = (tiles + 7) / 8 * 8;
  const long long cap = ((long long)num_cu * MINB + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  SmallArgs o{};
  o.x = (const char*)a.x + (long long)ES * a.x_coff; o.w = (const char*)a.w; o.bias = a.bias; o.y = (char*)a.y + (long long)ES * a.y_coff; o.n_dyn = a.n_dyn;
  if (a.res && a.res_mode != OCTO_RES_NONE) o.res = (const char*)a.res + (long long)ES * a.res_coff;
  if (a.split > 0) o.y2 = (char*)a.y2 + (long long)ES * (a.y2_coff - a.split);
  o.n = a.n; o.HoWo = a.Ho * a.Wo; o.tiles_c = (int)tiles_c; o.per_row = a.Kp * ES; o.grid = (int)grid;
  o.div_tc = make_fastdiv((unsigned)tiles_c); o.div_tp = make_fastdiv((unsigned)tiles_p);
  o.div_howo = make_fastdiv((unsigned)(a.Ho * a.Wo)); o.div_wo = make_fastdiv((unsigned)a.Wo);
  o.x_pitch = a.x_ld * ES; o.y_pitch = a.y_ld * ES; o.y2_pitch = a.y2_ld * ES; o.res_pitch = a.res_ld * ES;
  o.Cout = a.Cout; o.split = a.split; o.nk = (a.K + BK - 1) / BK; o.taps_nk = a.Cin / BK;
  o.H = a.H; o.W = a.W; o.Wo = a.Wo; o.kw = a.kw; o.kh = a.kh; o.stride = a.stride_h; o.pad = a.pad_h; o.Cin = a.Cin; o.K = a.K;
  o.magic_cin = a.magic_cin; o.magic_kw = a.magic_kw;
  // where the weights are the larger operand, a die keeps to its channels and all dies read the pixels; see conv_ksplit.h
  o.c_outer = (double)a.Cout * a.Kp > (double)(a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * a.H * a.W * a.Cin;
  o.act = a.act; o.res_mode = a.res_mode; o.w_len = a.w_rows * a.Kp * ES; o.w_rows = a.w_rows;
  const bool window = a.kh > 1 || a.kw > 1 || a.pad_h, part = ES == 4 && a.Cin % BK && !window;
  const int mode = part ? (a.stride_h > 1 ? SMALL_STRIDED_PART : SMALL_PART) : a.Cin % BK ? SMALL_ANY : (window || a.stride_h > 1 ? SMALL_TAPS : SMALL_POINTWISE);
  if (kernel_id) *kernel_id = small_kernel_id(BC, BP, WC, mode);
  if (a.group && a.group->count < SmallGroup::MAX) {       // launched with the others of its group
    SmallGroup& g = *a.group;
    if (g.count == 0) g.timing = tm;
    g.tile[g.count] = which; g.mode[g.count] = mode; g.kernel_id[g.count] = kernel_id; g.layer[g.count++] = o;
    return hipSuccess;
  }
  auto go = [&](auto mode_c) {
    constexpr int MODE = decltype(mode_c)::value;
    if (tm.start && tm.stop) hipExtLaunchKernelGGL((conv_small_kernel<T, BC, BP, WC, WP, MINB, MODE>), dim3((unsigned)grid), dim3(NT), 0, s, tm.start, tm.stop, 0, o);
    else hipLaunchKernelGGL((conv_small_kernel<T, BC, BP, WC, WP, MINB, MODE>), dim3((unsigned)grid), dim3(NT), 0, s, o);
    return hipGetLastError();
  };
  if constexpr (ES == 4) {
    if (part) return a.stride_h > 1 ? go(std::integral_constant<int, SMALL_STRIDED_PART>{}) : go(std::integral_constant<int, SMALL_PART>{});
  }
  return mode == SMALL_ANY ? go(std::integral_constant<int, SMALL_ANY>{})
                           : mode == SMALL_TAPS ? go(std::integral_constant<int, SMALL_TAPS>{}) : go(std::integral_constant<int, SMALL_POINTWISE>{});
}

// One entry point per storage type; `which` counts the rows of SMALL_COST (SMALL_COST_F32).
template <typename T>
static hipError_t launch_small(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (a.group && a.group->count > 0) which = a.group->tile[0];
  switch (which) {
    case 0: return launch_small_cfg<T, 32, 32, 2, 2, 4>(which, a, num_cu, s, kernel_id, tm);
    case 1: return launch_small_cfg<T, 32, 64, 1, 4, 4>(which, a, num_cu, s, kernel_id, tm);
    case 2: return launch_small_cfg<T, 64, 32, 2, 2, 4>(which, a, num_cu, s, kernel_id, tm);
    case 3: return launch_small_cfg<T, 64, 64, 2, 2, 3>(which, a, num_cu, s, kernel_id, tm);
    case 4: if constexpr (sizeof(T) == 2) return launch_small_cfg<T, 128, 64, 4, 2, 2>(which, a, num_cu, s, kernel_id, tm);
  }
  return hipErrorNotSupported;
}

// Launches what a group has collected.
template <typename T, int BC, int BP, int WC, int WP, int MINB>
static hipError_t launch_small_group_cfg(const SmallGroup& g, hipStream_t s) {
  auto go = [&](auto mode_c) {
    constexpr int MODE = decltype(mode_c)::value, NT = 64 * WC * WP;
    auto start = [&](auto kernel, int grid, const auto& args) {
      if (g.timing.start && g.timing.stop) hipExtLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NT), 0, s, g.timing.start, g.timing.stop, 0, args);
      else hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(NT), 0, s, args);
      return hipGetLastError();
    };
    if (g.count == 1) return start(conv_small_kernel<T, BC, BP, WC, WP, MINB, MODE>, g.layer[0].grid, g.layer[0]);
    for (int i = 0; i < g.count; ++i)
      if (g.kernel_id[i]) *g.kernel_id[i] = i ? KID_NONE : group_kernel_id(BC, BP, g.count, MODE);
    SmallGroupArgs a{};
    for (int i = 0; i < g.count; ++i) a.layer[i] = g.layer[i];
    a.second = g.layer[0].grid;
    a.third = a.second + g.layer[1].grid;
    return start(conv_small_group_kernel<T, BC, BP, WC, WP, MINB, MODE>, a.third + (g.count > 2 ? g.layer[2].grid : 0), a);
  };
  return g.mode[0] == SMALL_TAPS ? go(std::integral_constant<int, SMALL_TAPS>{}) : go(std::integral_constant<int, SMALL_POINTWISE>{});
}
template <typename T>
static hipError_t launch_small_group_t(const SmallGroup& g, hipStream_t s) {
  for (int i = 1; i < g.count; ++i) if (g.mode[i] != g.mode[0] || g.tile[i] != g.tile[0]) return hipErrorInvalidValue;
  if (g.count < 1 || (g.mode[0] != SMALL_TAPS && g.mode[0] != SMALL_POINTWISE)) return hipErrorInvalidValue;
  switch (g.tile[0]) {
    case 0: return launch_small_group_cfg<T, 32, 32, 2, 2, 4>(g, s);
    case 1: return launch_small_group_cfg<T, 32, 64, 1, 4, 4>(g, s);
    case 2: return launch_small_group_cfg<T, 64, 32, 2, 2, 4>(g, s);
    case 3: return launch_small_group_cfg<T, 64, 64, 2, 2, 3>(g, s);
    case 4: return launch_small_group_cfg<T, 128, 64, 4, 2, 2>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace octo
