// Convolution as an implicit GEMM on the CDNA4 matrix cores.
//
//   y[n,p,q,k] = act(bias[k] + sum_{r,s,c} x[n, p*stride + r - pad, q*stride + s - pad, c] * w[k,r,s,c]  (+ residual))
// (vertical and horizontal stride / padding are separate arguments: a 3-channel first layer is run on the
// pixel-pair view of a 4-channel-padded input, see pipeline.hip)
//
// GEMM view: rows = output channels (weights, [Cout][K] with K = kh*kw*Cin contiguous),
// columns = output pixels (gathered on the fly from the NHWC input), reduction = K.
// One workgroup = 4 wavefronts (256 lanes) computes a BC x BP tile with
// v_mfma_f32_32x32x16 (fp16 / bf16) or v_mfma_f32_32x32x2 (fp32).  Operands reach LDS in one of two ways: straight
// from global memory (buffer loads with the LDS bit, a ring of stages, one barrier per K step; the path of all layers
// with more than 32 output channels), or through registers (double buffered; 3-channel first layers, whose gather is
// element-wise, and layers with up to 32 output channels).  A tile row is 64 or 128 bytes of K; its 16-byte vectors
// are XOR-swizzled so that both the fills and the MFMA operand reads (16 bytes per lane) are bank-conflict free.
//
// The inner loop is kept nearly free of vector-ALU work, which would otherwise
// starve the matrix cores: operands are fetched with buffer loads whose 32-bit
// offsets are "row offset + tap offset", an out-of-image tap gets an offset beyond
// the buffer range so the hardware returns zeros, and the weight offsets advance
// through the scalar offset operand.
//
// The grid is persistent: workgroups stride over the tile list, whose length may
// depend on an item count that lives in device memory (a variable number of ROIs),
// so no host round trip is needed.
#include "octo_internal.h"
#include "mfma_common.h"
#include "conv_ksplit.h"
#include "conv3x3_mid.h"
#include "conv3x3_held.h"
#include "conv_flow_choice.h"
#include "conv_small_choice.h"
#include <hip/hip_ext.h>

namespace octo {

// BC: output channels per tile, BP: pixels per tile, WC x WP: wavefront grid (WC * WP == 4),
// KV: 16-byte vectors per tile row and K step (one K step = KV*16 bytes of K per row),
// D: K steps whose global loads are in flight in registers (even), MINB: workgroups per CU to fit registers for.
// DMA: operands go global -> LDS directly (buffer loads with the LDS bit), D K-steps ahead, into a ring of D + 1 LDS
// stages; no registers are spent on staging and no LDS store instructions are issued.  The loads are issued from
// inline assembly (the wave's LDS destination is base M0 + lane * 16), and their completion is awaited with explicit
// vmcnt waits whose counts rely on every wave issuing the same number of loads per K step.  M0 is reserved by the
// compiler (it writes M0 immediately before each of its own uses), so setting it inside the asm statement is safe.
template <typename T, int BC, int BP, int WC, int WP, int KV, int D, int MINB, bool VEC, bool DMA = false, bool PIPE = false>
__global__ __launch_bounds__(THREADS, MINB) void conv_mfma_kernel(const ConvKernelArgs a) {
  using E = Elem<T>;
  constexpr int VN = E::N;
  constexpr int ES = (int)sizeof(T);
  constexpr int BK = KV * VN;            // elements per K step
  constexpr int ROWV = KV;               // LDS row pitch in vectors; the vector slot of a row is XOR-swizzled (below)
  constexpr int RPW = 16 / KV;           // tile rows per 256 bytes of LDS (one pass over all banks)
  static_assert(KV == 4 || KV == 8 || KV == 16, "swizzle assumes 64-, 128- or 256-byte rows");
  constexpr int RP = THREADS / KV;       // tile rows covered by one pass of the 256 loader lanes
  constexpr int TC = BC / WC / 32;       // 32x32 blocks per wavefront along channels
  constexpr int TP = BP / WP / 32;
  constexpr int LA = (BC + RP - 1) / RP; // vectors per lane per K step (weights)
  constexpr int LB = BP / RP;            // (pixels)
  static_assert(DMA || D % 2 == 0, "pipeline depth must be even");
  static_assert(WC * WP == 4 && TC >= 1 && TP >= 1 && LB >= 1 && BP % RP == 0 && BC % 32 == 0, "tile shape");
  static_assert(!PIPE || DMA, "the pipelined loop loads straight to LDS");
  static_assert(!DMA || (VEC && BC % RP == 0), "direct-to-LDS loads need whole passes of all lanes");
  constexpr int NST = DMA ? D + 1 : 2;   // LDS stages
  constexpr int STAGE_VECS_OP = (BC + BP) * ROWV;
  constexpr int NL = LA + LB;            // load instructions per wave and K step

  // operand tiles; after the K loop the same memory stages the output tile as [pixel][channel] so that it can be
  // written with 16-byte stores that cover whole cache lines
  constexpr int OPITCH = BC * ES + 16;                                    // bytes per staged output row
  constexpr int OPER_VECS = NST * (BC + BP) * ROWV;                       // operand tiles, all stages
  constexpr int STAGE_VECS = BP * OPITCH / 16;                            // output tile
  constexpr bool STAGED = STAGE_VECS <= 4096 || STAGE_VECS <= OPER_VECS;  // stage outputs of up to 64 KB, or what the operands took
  constexpr int SMEM_VECS = STAGED && STAGE_VECS > OPER_VECS ? STAGE_VECS : OPER_VECS;
  __shared__ u32x4 smem[SMEM_VECS];
  __shared__ float sBias[BC];
  __shared__ float sScale[ES == 1 ? BC : 1];       // 8-bit storage: factor on the accumulator, per output channel
  u32x4 (*sA)[BC][ROWV] = (u32x4 (*)[BC][ROWV])smem;
  u32x4 (*sB)[BP][ROWV] = (u32x4 (*)[BP][ROWV])(smem + 2 * BC * ROWV);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wc = wave % WC, wp = wave / WC;
  const int l32 = lane & 31, g = lane >> 5;

  int n_items = a.n;
  if (a.n_dyn) { int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const long long M = (long long)n_items * a.Ho * a.Wo;
  const int tiles_c = (a.Cout + BC - 1) / BC;
  const long long tiles_p = (M + BP - 1) / BP;
  const long long n_tiles = tiles_p * tiles_c;
  // register path: a multiple of D (the host pads Kp to a multiple of 128 bytes); direct-to-LDS path: any count, and a
  // last step that runs past Kp multiplies zero-filled pixels
  const int nk = DMA ? (a.Kp + BK - 1) / BK : a.Kp / BK;
  const T* __restrict__ xg = (const T*)a.x + a.x_coff;
  const int HoWo = a.Ho * a.Wo;
  const long long img_elems = (long long)a.H * a.W * a.x_ld;

  const int ld_row = tid / KV;
  const int ld_kv = tid % KV;
  // Row r keeps its 16-byte vector v in slot v ^ ((r / RPW) % KV).  Sixteen lanes that write RPW whole rows, and sixteen
  // lanes that read the same logical vector of sixteen consecutive rows, then each touch a different 16-byte bank group.
  // 32 and THREADS / KV are multiples of RPW * KV, so the swizzle term depends only on the lane.
  const int wsw = ld_kv ^ ((ld_row / RPW) % KV);      // slot this lane writes
  // direct-to-LDS: the lane's slot is fixed by its lane id (ld_kv), so it fetches the vector that belongs there
  const int lkv = DMA ? wsw : ld_kv;                  // logical vector this lane fetches
  const int rsw = (l32 / RPW) % KV;                   // XOR term for this lane's fragment reads
  const bool vec_ok = ((a.y_ld | a.y_coff) & 3) == 0 && (!a.res || ((a.res_ld | a.res_coff) & 3) == 0);
  const bool is_silu = a.act == OCTO_ACT_SILU;
  const float act_lo = a.act == OCTO_ACT_RELU ? 0.0f : -INFINITY;

  // weights: one buffer for the whole packed matrix (padded, so never out of range)
  const long long w_bytes = (long long)a.w_rows * a.Kp * ES;
  const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)(w_bytes < BUF_MAX ? w_bytes : BUF_MAX), BUF_FLAGS);

  // Workgroups are handed to the eight dies in turn (workgroup b runs on die b % 8) and every die has its own L2.  The
  // tile list is therefore cut into eight contiguous chunks, one per die: tiles that share input rows (neighbouring
  // pixel tiles, and all channel tiles of the same pixels) then meet in one L2 instead of being fetched by every die.
  // The grid is a multiple of 8, so a workgroup stays on its chunk while it strides.
  const long long per_die = (n_tiles + 7) >> 3;
  for (long long t = blockIdx.x; t < per_die * 8; t += gridDim.x) {
    const long long tile = (t & 7) * per_die + (t >> 3);
    if (tile >= n_tiles) continue;
    const int tc = (int)(tile % tiles_c);
    const long long tp = tile / tiles_c;
    const int c0 = tc * BC;
    const long long p0 = tp * BP;

    // activations: a buffer that starts at the first image this tile touches, so that 32-bit offsets suffice
    const int img0 = (int)(p0 / HoWo);
    const long long rem_bytes = ((long long)(a.n - img0) * img_elems - a.x_coff) * ES;
    const __amdgpu_buffer_rsrc_t rsrc_x =
        __builtin_amdgcn_make_buffer_rsrc((void*)(xg + (long long)img0 * img_elems), 0, (int)(rem_bytes < BUF_MAX ? rem_bytes : BUF_MAX), BUF_FLAGS);

    // per-lane pixel rows of the gather: byte offset of the (possibly out-of-image) pixel of tap (0, 0) and the
    // sets of kernel rows / columns that fall inside the image (bit r: row r ok; bit 16+s: column s ok)
    int rowoff[LB];
    unsigned hw_ok[LB];
    int hi0[LB], wi0[LB];   // only used by the element-wise gather
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const long long m = p0 + ld_row + RP * i;
      rowoff[i] = 0; hw_ok[i] = 0u; hi0[i] = -1000000; wi0[i] = 0;
      if (m < M) {
        // m < 2^31 (checked on the host): pixel -> (image, row, column) with precomputed reciprocals
        const unsigned mu = (unsigned)m;
        const unsigned img = a.HoWo_is_one ? mu : udiv(mu, a.magic_howo, a.shift_howo);
        const unsigned rem = mu - img * (unsigned)HoWo;
        const unsigned ho = a.Wo == 1 ? rem : udiv(rem, a.magic_wo, a.shift_wo);
        const unsigned wo = rem - ho * (unsigned)a.Wo;
        const int h0 = (int)ho * a.stride_h - a.pad_h, w0 = (int)wo * a.stride_w - a.pad_w;
        hi0[i] = h0; wi0[i] = w0;
        rowoff[i] = (int)((((long long)((int)img - img0) * a.H + h0) * a.W + w0) * a.x_ld) * ES;
        // kernel rows r with 0 <= h0 + r < H form the range [max(0, -h0), min(kh, H - h0)); same for columns
        const int rlo = h0 < 0 ? -h0 : 0, rhi = a.H - h0 < a.kh ? a.H - h0 : a.kh;
        const int slo = w0 < 0 ? -w0 : 0, shi = a.W - w0 < a.kw ? a.W - w0 : a.kw;
        const unsigned rm = rhi > rlo ? ((1u << rhi) - 1u) & ~((1u << rlo) - 1u) : 0u;
        const unsigned sm = shi > slo ? ((1u << shi) - 1u) & ~((1u << slo) - 1u) : 0u;
        hw_ok[i] = rm | (sm << 16);
      }
    }
    int woff[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i) woff[i] = ((c0 + ld_row + RP * i) * a.Kp + lkv * VN) * ES;

    floatx16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; ++i)
#pragma unroll
      for (int j = 0; j < TP; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // Operands of K step KB.  Element k = KB*BK + lkv*VN of the reduction is channel c of tap (r, s):
    // k = (r*kw + s)*Cin + c; the two divisions use precomputed reciprocals (exact for k < 65536).
    __syncthreads();   // the previous tile's LDS reads are done
    if (tid < BC) sBias[tid] = a.bias[c0 + tid];     // bias is padded to a multiple of 128 channels
    if constexpr (ES == 1) { if (tid < BC) sScale[tid] = a.scale[c0 + tid]; }     // padded alike
    if constexpr (DMA) {
      // LDS byte address of this wave's 1 KB slice of pass 0 of stage 0 (lane l writes at + 16 l)
      const unsigned lds_wave = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(uintptr_t)smem + (unsigned)wave * 1024u));
      constexpr unsigned STAGE_BYTES = STAGE_VECS_OP * 16, PASS_BYTES = RP * ROWV * 16, A_BYTES = BC * ROWV * 16;
      if constexpr (PIPE) {
      // Pipelined form: a K step is KK groups of matrix instructions.  The fragments of a group are read from LDS while the
      // group before it is multiplied, the loads of step kb + NST - 1 .. kb + NST go out between the groups, and the barrier sits
      // before the last group: behind it the next step's operands are complete and the stage of this one is free.
      constexpr int KK = ES == 1 ? KV / 4 : KV / 2;
      constexpr int FV = ES == 1 ? 2 : 1;
      constexpr int P0 = (NL + KK - 1) / KK;       // loads issued with each group
      unsigned need = 0u; int delta = 0, koff = 0; unsigned sbase = 0;
#define OCTO_CONV_ADDR(KB, ST)                                                                                      \
      {                                                                                                             \
        sbase = lds_wave + (unsigned)(ST) * STAGE_BYTES;                                                            \
        koff = (KB) * (BK * ES);                                                                                    \
        const unsigned k = (unsigned)(KB) * BK + lkv * VN;                                                          \
        const unsigned tap = __umulhi(k, a.magic_cin);                                                              \
        const int c = (int)(k - tap * a.Cin);                                                                       \
        const int r = a.kw == 1 ? (int)tap : (int)__umulhi(tap, a.magic_kw);                                        \
        const int s2 = (int)tap - r * a.kw;                                                                         \
        delta = ((r * a.W + s2) * a.x_ld + c) * ES;                                                                 \
        need = k < (unsigned)a.K ? ((1u << r) | (0x10000u << s2)) : 0xFFFFFFFFu;                                    \
      }
#define OCTO_CONV_PART(FROM, TO)                                                                                    \
      _Pragma("unroll") for (int q = (FROM); q < (TO) && q < NL; ++q) {                                             \
        if (q < LB) {                                                                                               \
          const int off = (hw_ok[q < LB ? q : 0] & need) == need ? rowoff[q < LB ? q : 0] + delta : OOB;            \
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"                   \
                       :: "s"(sbase + A_BYTES + q * PASS_BYTES), "v"(off), "s"(rsrc_x) : "memory");                  \
        } else {                                                                                                    \
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"                  \
                       :: "s"(sbase + (q - LB) * PASS_BYTES), "v"(woff[q >= LB ? q - LB : 0]), "s"(rsrc_w), "s"(koff) : "memory");             \
        }                                                                                                           \
      }
      u32x4 fa[2][TC][FV], fb[2][TP][FV];
#define OCTO_CONV_FRAGS(SET, ST, KQ)                                                                                \
      {                                                                                                             \
        const u32x4* pa = smem + (ST) * STAGE_VECS_OP;                                                              \
        const u32x4* pb = pa + BC * ROWV;                                                                           \
        _Pragma("unroll") for (int h = 0; h < FV; ++h) {                                                            \
          _Pragma("unroll") for (int i = 0; i < TC; ++i)                                                            \
            fa[SET][i][h] = pa[(wc * (BC / WC) + i * 32 + l32) * ROWV + ((((KQ) * FV + h) * 2 + g) ^ rsw)];         \
          _Pragma("unroll") for (int j = 0; j < TP; ++j)                                                            \
            fb[SET][j][h] = pb[(wp * (BP / WP) + j * 32 + l32) * ROWV + ((((KQ) * FV + h) * 2 + g) ^ rsw)];         \
        }                                                                                                           \
      }
#pragma unroll
      for (int d = 0; d < NST - 1; ++d) { OCTO_CONV_ADDR(d, d) OCTO_CONV_PART(0, NL) }
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 2) * NL) : "memory");
      __builtin_amdgcn_s_barrier();
      OCTO_CONV_ADDR(NST - 1, NST - 1)
      OCTO_CONV_PART(0, P0)
      OCTO_CONV_FRAGS(0, 0, 0)
      int st_rd = 0;
      for (int kb = 0; kb < nk; ++kb) {
        const int st_nx = st_rd + 1 == NST ? 0 : st_rd + 1;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          if (kk < KK - 1) {
            OCTO_CONV_FRAGS((kk + 1) & 1, st_rd, kk + 1)
            OCTO_CONV_PART(P0 * (kk + 1), (kk == KK - 2 ? NL : P0 * (kk + 2)))
          } else {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((NST - 2) * NL) : "memory");
            __builtin_amdgcn_s_barrier();
            OCTO_CONV_FRAGS(0, st_nx, 0)
            OCTO_CONV_ADDR(kb + NST, st_rd)
            OCTO_CONV_PART(0, P0)
          }
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int j = 0; j < TP; ++j) {
              if constexpr (ES == 1) acc[i][j] = E::mfma2(fa[kk & 1][i][0], fa[kk & 1][i][1], fb[kk & 1][j][0], fb[kk & 1][j][1], acc[i][j]);
              else acc[i][j] = E::mfma(fa[kk & 1][i][0], fb[kk & 1][j][0], acc[i][j]);
            }
        }
        st_rd = st_nx;
      }
#undef OCTO_CONV_ADDR
#undef OCTO_CONV_PART
#undef OCTO_CONV_FRAGS
      } else {
#define OCTO_CONV_DMA(KB, ST)                                                                                       \
      {                                                                                                             \
        const unsigned sbase = lds_wave + (unsigned)(ST) * STAGE_BYTES;                                             \
        const int koff = (KB) * (BK * ES);                                                                          \
        _Pragma("unroll") for (int i = 0; i < LA; ++i)                                                              \
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"                  \
                       :: "s"(sbase + i * PASS_BYTES), "v"(woff[i]), "s"(rsrc_w), "s"(koff) : "memory");             \
        const unsigned k = (unsigned)(KB) * BK + lkv * VN;                                                          \
        const unsigned tap = __umulhi(k, a.magic_cin);                                                              \
        const int c = (int)(k - tap * a.Cin);                                                                       \
        const int r = a.kw == 1 ? (int)tap : (int)__umulhi(tap, a.magic_kw);                                        \
        const int s2 = (int)tap - r * a.kw;                                                                         \
        const int delta = ((r * a.W + s2) * a.x_ld + c) * ES;                                                       \
        const unsigned need = k < (unsigned)a.K ? ((1u << r) | (0x10000u << s2)) : 0xFFFFFFFFu;                     \
        _Pragma("unroll") for (int i = 0; i < LB; ++i) {                                                            \
          const int off = (hw_ok[i] & need) == need ? rowoff[i] + delta : OOB;                                      \
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"                   \
                       :: "s"(sbase + A_BYTES + i * PASS_BYTES), "v"(off), "s"(rsrc_x) : "memory");                  \
        }                                                                                                           \
      }
      int st_rd = 0, st_wr = D;          // ring positions: stage read in this step, stage filled for step kb + D
#pragma unroll
      for (int d = 0; d < D; ++d) OCTO_CONV_DMA(d, d)
      for (int kb = 0; kb < nk; ++kb) {
        // loads of the D - 1 later steps may stay in flight; those of step kb (issued before them) are complete, and so are this wavefront's reads of
        // step kb - 1 (said here: the compiler's own wait for them goes with the matrix instructions, which no barrier holds)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((D - 1) * NL) : "memory");
        __builtin_amdgcn_s_barrier();    // everyone's part of step kb is in LDS, and everyone is done reading step kb - 1
        OCTO_CONV_DMA(kb + D, st_wr)     // refills the stage that step kb - 1 read; past the last step: zeros, never read
        const u32x4* pa = smem + st_rd * STAGE_VECS_OP;
        const u32x4* pb = pa + BC * ROWV;
        if constexpr (ES == 1) {
          // 8-bit operands: one instruction reduces over 64 values, two vectors per lane and operand
#pragma unroll
          for (int kk = 0; kk < KV / 4; ++kk) {
            u32x4 fa[TC][2], fb[TP][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
              for (int i = 0; i < TC; ++i) fa[i][h] = pa[(wc * (BC / WC) + i * 32 + l32) * ROWV + ((kk * 4 + h * 2 + g) ^ rsw)];
#pragma unroll
              for (int j = 0; j < TP; ++j) fb[j][h] = pb[(wp * (BP / WP) + j * 32 + l32) * ROWV + ((kk * 4 + h * 2 + g) ^ rsw)];
            }
#pragma unroll
            for (int i = 0; i < TC; ++i)
#pragma unroll
              for (int j = 0; j < TP; ++j) acc[i][j] = E::mfma2(fa[i][0], fa[i][1], fb[j][0], fb[j][1], acc[i][j]);
          }
        } else {
#pragma unroll
        for (int kk = 0; kk < KV / 2; ++kk) {
          u32x4 fa[TC], fb[TP];
#pragma unroll
          for (int i = 0; i < TC; ++i) fa[i] = pa[(wc * (BC / WC) + i * 32 + l32) * ROWV + ((kk * 2 + g) ^ rsw)];
#pragma unroll
          for (int j = 0; j < TP; ++j) fb[j] = pb[(wp * (BP / WP) + j * 32 + l32) * ROWV + ((kk * 2 + g) ^ rsw)];
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int j = 0; j < TP; ++j) acc[i][j] = E::mfma(fa[i], fb[j], acc[i][j]);
        }
        }
        st_rd = st_rd + 1 == NST ? 0 : st_rd + 1;
        st_wr = st_wr + 1 == NST ? 0 : st_wr + 1;
      }
#undef OCTO_CONV_DMA
      }
      // the loads issued past the last step still write (zeros) into the ring: drain them before the memory is reused
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    } else {
    u32x4 ra[D][LA], rb[D][LB];
#define OCTO_CONV_LOAD(KB, SL)                                                                                      \
    {                                                                                                               \
      _Pragma("unroll") for (int i = 0; i < LA; ++i)                                                                \
        if (BC % RP == 0 || ld_row + RP * i < BC)                                                                   \
          ra[SL][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, woff[i], (KB) * (BK * ES), 0);                  \
      if (VEC) {                                                                                                    \
        const unsigned k = (unsigned)(KB) * BK + lkv * VN;                                                          \
        const unsigned tap = __umulhi(k, a.magic_cin);                                                              \
        const int c = (int)(k - tap * a.Cin);                                                                       \
        const int r = a.kw == 1 ? (int)tap : (int)__umulhi(tap, a.magic_kw);                                        \
        const int s2 = (int)tap - r * a.kw;                                                                         \
        const int delta = ((r * a.W + s2) * a.x_ld + c) * ES;                                                       \
        const unsigned need = k < (unsigned)a.K ? ((1u << r) | (0x10000u << s2)) : 0xFFFFFFFFu;                     \
        _Pragma("unroll") for (int i = 0; i < LB; ++i) {                                                            \
          const int off = (hw_ok[i] & need) == need ? rowoff[i] + delta : OOB;                                      \
          rb[SL][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, off, 0, 0);                                     \
        }                                                                                                           \
      } else {                                                                                                      \
        const int kbase = (KB) * BK + ld_kv * VN;                                                                   \
        _Pragma("unroll") for (int i = 0; i < LB; ++i) {                                                            \
          typedef T tv __attribute__((ext_vector_type(VN)));                                                        \
          tv pk;                                                                                                    \
          const T* rowp = xg + (long long)img0 * img_elems + rowoff[i] / ES;                                        \
          _Pragma("unroll") for (int e = 0; e < VN; ++e) {                                                          \
            const int k = kbase + e;                                                                                \
            T val = (T)0.0f;                                                                                        \
            if (k < a.K) {                                                                                          \
              const int tap = k / a.Cin, c = k - tap * a.Cin;                                                       \
              const int r = tap / a.kw, s2 = tap - r * a.kw;                                                        \
              if ((unsigned)(hi0[i] + r) < (unsigned)a.H && (unsigned)(wi0[i] + s2) < (unsigned)a.W)                \
                val = rowp[(r * a.W + s2) * a.x_ld + c];                                                            \
            }                                                                                                       \
            pk[e] = val;                                                                                            \
          }                                                                                                         \
          rb[SL][i] = __builtin_bit_cast(u32x4, pk);                                                                \
        }                                                                                                           \
      }                                                                                                             \
    }

    // nk is a multiple of D (the packed K extent is padded accordingly); loads past the end return zeros
#pragma unroll
    for (int d = 0; d < D; ++d) OCTO_CONV_LOAD(d, d)
    for (int kb0 = 0; kb0 < nk; kb0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int kb = kb0 + d;
        const int buf = d & 1;           // D is even, so kb & 1 == d & 1
        // operands of step kb: registers -> LDS
#pragma unroll
        for (int i = 0; i < LA; ++i)
          if (BC % RP == 0 || ld_row + RP * i < BC) sA[buf][ld_row + RP * i][wsw] = ra[d][i];
#pragma unroll
        for (int i = 0; i < LB; ++i) sB[buf][ld_row + RP * i][wsw] = rb[d][i];
        __syncthreads();
        OCTO_CONV_LOAD(kb + D, d)
#pragma unroll
        for (int kk = 0; kk < KV / 2; ++kk) {
          u32x4 fa[TC], fb[TP];
#pragma unroll
          for (int i = 0; i < TC; ++i) fa[i] = sA[buf][wc * (BC / WC) + i * 32 + l32][(kk * 2 + g) ^ rsw];
#pragma unroll
          for (int j = 0; j < TP; ++j) fb[j] = sB[buf][wp * (BP / WP) + j * 32 + l32][(kk * 2 + g) ^ rsw];
#pragma unroll
          for (int i = 0; i < TC; ++i)
#pragma unroll
            for (int j = 0; j < TP; ++j) acc[i][j] = E::mfma(fa[i], fb[j], acc[i][j]);
        }
      }
    }
#undef OCTO_CONV_LOAD
    }

    // epilogue: a lane holds pixel column l32 of each 32x32 block and 4 groups of 4 consecutive channels
    // (a launch with a second output tensor always takes the staged path: the host has checked its alignment)
    const bool staged = STAGED && !a.out_f32 && ((a.y_ld | a.y_coff) & (VN - 1)) == 0 && (((uintptr_t)a.y & 15) == 0);
    if (staged) __syncthreads();       // every wavefront is done reading the operand tiles
    // the arithmetic is compiled once per (residual mode, SiLU or not): see finish4
    with_epilogue_mode(a.res ? a.res_mode : OCTO_RES_NONE, is_silu, [&](auto res_c, auto silu_c) __attribute__((always_inline)) {
    constexpr int RES = decltype(res_c)::value;
    constexpr bool SILU = decltype(silu_c)::value;
#pragma unroll
    for (int j = 0; j < TP; ++j) {
      const int pl = wp * (BP / WP) + j * 32 + l32;          // pixel inside the tile
      const long long p = p0 + pl;
      if (p >= M) continue;
#pragma unroll
      for (int i = 0; i < TC; ++i) {
        const int cblk = wc * (BC / WC) + i * 32 + g * 4;     // channel (inside the tile) of this lane's group q = 0
        if (staged || (vec_ok && c0 + cblk + 28 <= a.Cout)) {
          // all four 4-channel groups are inside the tensor and 8/16-byte accesses are aligned (a staged tile may
          // carry channels past Cout; they are dropped when the tile is written out)
          floatx4 rv[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) rv[q] = floatx4{0.f, 0.f, 0.f, 0.f};
          if (RES != OCTO_RES_NONE) {
            const T* rp = (const T*)a.res + (size_t)p * a.res_ld + a.res_coff + c0 + cblk;
            if (vec_ok && c0 + cblk + 28 <= a.Cout) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const floatx4 r4 = load4<T>(rp + q * 8);
#pragma unroll
                for (int e = 0; e < 4; ++e) rv[q][e] = ES == 1 ? r4[e] * a.res_scale : r4[e];
              }
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (c0 + cblk + q * 8 + e < a.Cout) rv[q][e] = ES == 1 ? to_f32<T>(rp[q * 8 + e]) * a.res_scale : to_f32<T>(rp[q * 8 + e]);
            }
          }
          const size_t o = (size_t)p * a.y_ld + a.y_coff + c0 + cblk;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const floatx4 b4 = *(const floatx4*)&sBias[cblk + q * 8];
            floatx4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = ES == 1 ? acc[i][j][q * 4 + e] * sScale[cblk + q * 8 + e] : acc[i][j][q * 4 + e];
            v = finish4<RES, SILU>(v, b4, rv[q], act_lo);
            if (a.out_f32) { store4<float>((float*)a.y + o + q * 8, v); continue; }
            if constexpr (ES == 1) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] *= a.y_inv_scale;
            }
            if (staged) store4<T>((T*)((char*)smem + (size_t)pl * OPITCH) + cblk + q * 8, v);
            else store4<T>((T*)a.y + o + q * 8, v);
          }
        } else {
          // edge path: channel tail of the tensor or unaligned pitch - element by element
#pragma unroll
          for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int cl = cblk + q * 8 + e;
              const int c = c0 + cl;
              if (c < a.Cout) {
                float r = 0.f, av = acc[i][j][q * 4 + e];
                if (RES != OCTO_RES_NONE) r = to_f32<T>(((const T*)a.res)[(size_t)p * a.res_ld + a.res_coff + c]);
                if constexpr (ES == 1) { r *= a.res_scale; av *= sScale[cl]; }
                float t = finish1<RES, SILU>(av, sBias[cl], r, act_lo);
                const size_t o = (size_t)p * a.y_ld + a.y_coff + c;
                if (a.out_f32) { ((float*)a.y)[o] = t; continue; }
                if constexpr (ES == 1) t *= a.y_inv_scale;
                ((T*)a.y)[o] = from_f32<T>(t);
              }
            }
          }
        }
      }
    }
    });
    if (staged) {
      // staged tile -> global memory: consecutive lanes write consecutive 16-byte pieces of a pixel's channels
      __syncthreads();
      constexpr int VPR = BC / VN;                 // 16-byte vectors per pixel row of the tile
      constexpr int PPP = THREADS / VPR;           // pixels per pass
      const int v = tid % VPR, pr = tid / VPR;
      const int c = c0 + v * VN;
#pragma unroll
      for (int ps = 0; ps < BP / PPP; ++ps) {
        const int pl = ps * PPP + pr;
        const long long p = p0 + pl;
        if (p < M && c < a.Cout) {
          const u32x4 val = *(const u32x4*)((const char*)smem + (size_t)pl * OPITCH + (size_t)v * 16);
          // two layers in one launch: a vector never straddles the split (a multiple of 8 channels)
          const bool second = a.split > 0 && c >= a.split;
          T* yp = second ? (T*)a.y2 + (size_t)p * a.y2_ld + a.y2_coff + (c - a.split) : (T*)a.y + (size_t)p * a.y_ld + a.y_coff + c;
          if (c + VN <= a.Cout) {
            *(u32x4*)yp = val;
          } else if constexpr (ES == 1) {
            typedef uint8_t bv __attribute__((ext_vector_type(16)));
            const bv b = __builtin_bit_cast(bv, val);
#pragma unroll
            for (int e = 0; e < VN; ++e) if (c + e < a.Cout) yp[e].bits = b[e];
          } else {
            typedef T tv __attribute__((ext_vector_type(VN)));
            const tv tvv = __builtin_bit_cast(tv, val);
#pragma unroll
            for (int e = 0; e < VN; ++e) if (c + e < a.Cout) yp[e] = tvv[e];
          }
        }
      }
    }
  }
}

// This file is compiled once per storage type, so that the types build in parallel: conv_f16.hip, conv_bf16.hip,
// conv_f32.hip and conv_f8.hip define OCTO_CONV_ONLY_<type> and include it; each then holds the kernel instances of
// its type behind one entry point (launch_general_<type>).  Compiled as itself it holds no kernel, only the dispatch
// (launch_conv) and the host helpers.
#ifndef OCTO_CONV_NO_LAUNCHERS
template <typename T, int BC, int BP, int WC, int WP, int KV, int D, int MINB, bool VEC, bool DMA = false, bool PIPE = false>
static hipError_t launch_cfg(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  if (kernel_id) *kernel_id = conv_kernel_id(BC, BP, KV, MINB, VEC, DMA, PIPE);
  const long long M = (long long)a.n * a.Ho * a.Wo;
  const long long tiles = ((M + BP - 1) / BP) * ((a.Cout + BC - 1) / BC);
  if (tiles <= 0) return hipSuccess;
  long long grid = (tiles + 7) / 8 * 8;          // a multiple of the die count (see the kernel's tile order)
  const long long cap = ((long long)num_cu * MINB + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  // with timing events the dispatch itself carries them, so their difference is the kernel's own run time
  if (tm.start && tm.stop)
    hipExtLaunchKernelGGL((conv_mfma_kernel<T, BC, BP, WC, WP, KV, D, MINB, VEC, DMA, PIPE>), dim3((unsigned)grid), dim3(THREADS), 0, s, tm.start, tm.stop, 0, a);
  else
    hipLaunchKernelGGL((conv_mfma_kernel<T, BC, BP, WC, WP, KV, D, MINB, VEC, DMA, PIPE>), dim3((unsigned)grid), dim3(THREADS), 0, s, a);
  return hipGetLastError();
}

// Tile choice of the general kernel (measured on MI355X) for M output pixels.  Up to 32 output channels: register-staged
// 32x128 tiles.  Otherwise operands go straight into LDS with K steps of 128 bytes: 128x128 tiles where 128 channels per
// tile pad the channel count no further than 64 do (192 = 3 x 64, but 2 x 128), 64x128 tiles for the middle ground (64x256
// with 64-byte K steps for very large, narrow layers), 64x64 tiles for layers with few output pixels.  How many tiles a
// shape must yield depends on the length of the reduction.  A layer with a short K loop is dominated by start-up and
// epilogue and runs fastest on the shape that spreads it over all compute units.  A long K loop is paced by the operand
// fetch from the L2s, so the shape with the most arithmetic per fetched byte wins as soon as a quarter of the compute
// units get a tile: alone it takes a little longer, but it moves half the bytes, and kernels of other streams use the
// rest of the chip meanwhile (+4 % on the traffic cascade with four pipeline instances).
// Very many pixels: 256-pixel tiles of 64 channels with 64-byte K steps, three workgroups per compute unit.  For layers of
// at most 64 channels (store-bound first layers, wide early stages), and for short reductions - all epilogue and memory
// traffic - whose channel count the 128-channel tile would pad (192 = 3 x 64): 192 -> 192 on 32 x 160 x 160 runs 11 %
// faster than on 64x128 tiles; beyond K = 384 the larger K step wins.
// k_scale: values per 2 bytes of K (2 for 8-bit storage, whose reductions are half as long in bytes).
// 16-bit layers also have shapes of the pipelined form, whose deeper ring leaves room for two workgroups per compute unit (three
// with 64x64).  Aligned layers reach one of them only, 64x64 (launch_typed says when; conv_flow_kernel has the rest); the others serve
// pixel-pair first layers that the first-layer kernel declines, two layers whose split lies inside a block of 32 channels,
// outputs and residuals that are no whole 16-byte vectors, fp32 outputs and single K steps into more than 256 channels, and their
// lines were drawn by the aligned layers below, which they took before that kernel: 128x64 (64x128 where 128 channels would pad)
// where their tiles fill one round of those and not more - 128 -> 256, stride 2 on 8 x 80 x 80 15.6 us (128x128: 19.6), 1024 -> 512 on 60 x 16 x 8 14.7 (18.2); one tile more than a round and the
// others win again -, 64x64 in the same way for fewer pixels and a reduction of at least 1 KB (256 -> 512, stride 2 on
// 63 x 14 x 14 16.4 us, split-K 18.2; where 64x128 would do too, up to 1.3 of those per compute unit, beyond which the three
// per unit that 64x64 tiles fit run out: 192 -> 192, stride 2 on 56 x 56, 64x64 : 64x128 at 1.08 17.0 : 17.1, at 1.29 17.7 : 17.6, at
// 1.58 23.8 : 18.9; 128 -> 192, stride 2 on 57 x 57 at 1.15 13.1 : 13.5, at 1.31 13.3 : 13.7, at 1.54 17.3 : 14.0), and 128x256 with 64-byte K steps for long reductions over enough pixels to keep its
// rounds three quarters full (256 -> 512, stride 2 on 64 x 40 x 40 76 us, 128x128: 88).
struct GeneralTile { int bc, bp; bool pipe = false; };
static GeneralTile general_tile(const ConvArgs& a, long long M, int num_cu, int k_scale, bool pipe_ok = false) {
  auto tiles = [&](int bc, int bp) { return ((M + bp - 1) / bp) * ((a.Cout + bc - 1) / bc); };
  if (a.Cout <= 32 && k_scale == 1) return {32, 128};
  const bool fits128 = a.Cout >= 96 && (a.Cout + 127) / 128 * 128 == (a.Cout + 63) / 64 * 64;
  if (tiles(64, 256) >= 4 * num_cu && (a.Cout <= 64 || (k_scale == 1 && !fits128 && a.Kp <= 384))) return {64, 256};
  if (pipe_ok) {
    const long long big = tiles(128, 256), rounds = (big + 2 * num_cu - 1) / (2 * num_cu);
    if (fits128 && a.Kp >= 512 && big * 4 >= rounds * 2 * num_cu * 3) return {128, 256, true};
    auto one_round = [&](long long t, int per_cu) { return t > num_cu && t <= (long long)per_cu * num_cu; };
    if (fits128 && one_round(tiles(128, 64), 2)) return {128, 64, true};
    if (!fits128 && a.Cout > 64 && one_round(tiles(64, 128), 2) && tiles(64, 128) * 10 >= 13 * num_cu) return {64, 128, true};
    if (a.Kp >= 512 && one_round(tiles(64, 64), fits128 ? 2 : 3)) return {64, 64, true};
  }
  if (fits128 && tiles(128, 128) >= (a.Kp >= 1024 * k_scale ? num_cu / 4 : 5 * num_cu / 4)) return {128, 128};
  if (tiles(64, 128) >= (a.Kp >= 512 * k_scale ? num_cu / 4 : 9 * num_cu / 8)) return {64, 128};
  return {64, 64};
}

template <typename T>
static hipError_t launch_typed(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  constexpr int VN = Elem<T>::N;
  const bool vec = (a.Cin % VN == 0) && (a.x_ld % VN == 0) && (a.x_coff % VN == 0) && (((uintptr_t)a.x & 15) == 0) &&
                   a.kh <= 15 && a.kw <= 15;
  // the tile shape is chosen for the expected number of items (any shape is correct for any count: the grid strides
  // over however many tiles the device-side count gives)
  const long long M = (long long)(a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * a.Ho * a.Wo;
  if (!vec) {
    // element-wise gather (first layers with 3 input channels)
    if (a.Cout <= 32) return launch_cfg<T, 32, 128, 1, 4, 4, 2, 2, false>(a, num_cu, s, kernel_id, tm);
    return launch_cfg<T, 64, 128, 2, 2, 4, 2, 2, false>(a, num_cu, s, kernel_id, tm);
  }
  // Launches that leave compute units idle or wait on their K loop go to the split-K kernel instead, by estimated time.
  // That kernel sums in another order, so the choice is made for a.n_split items where the count is taken on the device:
  // unlike the running average behind n_hint it stays the same from batch to batch, and so do the results.
  const long long M_split = a.n_split > 0 ? (long long)(a.n_split < a.n ? a.n_split : a.n) * a.Ho * a.Wo : M;
  // fp32: conv_small_kernel or split-K, wherever the layer has the form of the former (conv_small_choice.h).  Tiles sum in chains of different lengths, so that
  // every choice is made for M_split.
  if constexpr (sizeof(T) == 4) {
    if (small_fits(a, 4) && small_takes_f32(a, M_split, num_cu)) {
      double us = 0;
      const int which = small_choose(a, M_split, num_cu, 4, false, &us);
      int ks = small_split_f32(a, M_split, num_cu, us);
      // Shorter sums round less: where the estimates that serve the other types have a split of eight ahead, one of four is no faster than it to speak of,
      // and eight it is (eight : four, us: 3x3 60 .. 130 K steps into 32 x 32 tiles 36.1 : 35.5, 42.4 : 42.0, 63.9 : 64.0, over 40 layers 1.01 of the
      // time; 90 .. 535 K steps, 64 x 32 tiles at two and a bit per compute unit 76 : 80, 134 : 143, 309 : 341, over 40 layers 0.95)
      if (ks > 0) {
        const GeneralTile st = general_tile(a, M_split, num_cu, 1);
        if (ksplit_choose(a, M_split, 4, st.bc, st.bp, num_cu) == 0) ks = 0;
      }
      return ks >= 0 ? launch_ksplit<T>(ks, a, num_cu, s, kernel_id, tm) : launch_small_f32(which, a, num_cu, s, kernel_id, tm);
    }
  }
  // Split-K or not is decided from estimates of repeated launches for M_split, in a cascade too: a layer of a model and a single call sum in one order there.  Over
  // 726 layers of few tiles in their place that choice, then the tile by place, takes 1.013 of the fastest kernel's time (by the estimates in place times
  // 0.80 .. 0.92 1.015 .. 1.044, never splitting 1.031).
  // Launches of few tiles go to conv_small_kernel, or to split-K where that is estimated to be faster; small_limit and TileCost have the lines.
  // conv_flow_kernel and the general kernel sum in the order of conv_small_kernel, so that place and running count may choose between those (the count not where
  // a last vector has less than eight channels, whose values they convert one by one); against the patch kernel it is M_split as well.
  bool to_small = false, not_split = false;
  [[maybe_unused]] const long long M_small = a.Cout % 8 || a.Cout <= 32 ? M_split : M;
  int small_tile = -1, flow_tile = -1;                     // the cheapest for M_small, where they have been asked for
  [[maybe_unused]] auto run_small = [&](long long m) -> hipError_t {
    double us = 0;
    const int which = small_tile >= 0 ? small_tile : small_choose(a, m, num_cu, 2, by_place(a), &us);
    return std::is_same<T, __bf16>::value ? launch_small_bf16(which, a, num_cu, s, kernel_id, tm) : launch_small_f16(which, a, num_cu, s, kernel_id, tm);
  };
  [[maybe_unused]] const bool pipe_ok = sizeof(T) == 2, pw = a.kh == 1 && a.kw == 1 && a.stride_h == 1 && a.stride_w == 1 && !a.pad_h && !a.pad_w;
  // Against the kernels of this order split-K is for few tiles: from four per compute unit on it loses whatever the estimates say (384 -> 768, stride 2
  // on 7 x 40 x 40 at 4.1 38.0 : 28.0, 512 -> 64 1x1 on 82 x 20 x 20 at 4.0 11.1 : 8.2).  Its 64 x 64 tiles serve long reductions (256 -> 256,
  // stride 2 on 6 x 40 x 40 11.0 : 13.8), not 1x1 layers (512 -> 512 on 5 x 20 x 20 7.3 : 5.8, 1024 -> 512 8.7 : 7.3).
  [[maybe_unused]] const int shapes = pw ? 3 : 4;
  [[maybe_unused]] const bool splittable = (M_split + (pw ? 31 : 63)) / (pw ? 32 : 64) * ((a.Cout + 63) / 64) < 4LL * num_cu;      // the last shape's tiles, the largest
  // strided layers of up to two 64x64 tiles per compute unit that the general kernel would run in one round of pipelined tiles: never split
  [[maybe_unused]] auto stays = [&](long long m) {
    const GeneralTile t = general_tile(a, m, num_cu, 1, pipe_ok);
    return !pw && t.pipe && t.bc == 64 && t.bp == 64 && (m + 63) / 64 * ((a.Cout + 63) / 64) <= 2LL * num_cu;
  };
  if constexpr (sizeof(T) == 2) {
    const hipError_t eh = launch_held<T>(a, M_split, num_cu, s, kernel_id, tm);
    if (eh != hipErrorNotSupported) return eh;
    const bool fits = small_fits(a, 2), patch = fits && small_takes_3x3(a, M_split, num_cu);
    if (!patch) {
      const hipError_t em = launch_mid<T>(a, M_split, num_cu, s, kernel_id, tm);
      if (em != hipErrorNotSupported) return em;
    }
    // (up to 32 channels only where the count is not taken on the device; not before an upsampling, which the split-K kernel writes along)
    to_small = fits && (a.Cout > 32 || (a.n_split == 0 && !a.up_next));
    if (patch || (to_small && !a.up_next && small_takes(a, M_split, num_cu, false))) {
      // Split-K has to beat every other kernel: below the patch kernel's line, never where one round of tiles fills the chip, and
      // conv_flow_kernel's estimate (96 -> 192, stride 2 on 9 x 57 x 83: split-K 14.1, estimated 12.1, conv_flow_kernel 13.3)
      if (splittable && (patch ? (double)M_split / 128 * ((a.Cout + 63) / 64) < 0.25 * num_cu : !stays(M_split))) {
        double us = 0, uf = 0;
        small_choose(a, M_split, num_cu, 2, false, &us);
        if (!patch && flow_fits(a)) { flow_choose(a, M_split, num_cu, 2, false, &uf); us = std::min(us, uf); }
        const int kf = ksplit_best(a, M_split, 2, num_cu, us, shapes, 4.0);
        if (kf >= 0) return launch_ksplit<T>(kf, a, num_cu, s, kernel_id, tm);
      }
      if (patch) return run_small(M_split);
      not_split = true;
    }
    // (two layers in one launch: by small_limit; beyond it conv_flow_kernel's best tile takes 1.03 .. 1.1 of this kernel's time)
    if (to_small && by_place(a) && a.split == 0 && flow_fits(a)) {
      double us = 0, uf = 0;
      small_tile = small_choose(a, M_small, num_cu, 2, true, &us);
      flow_tile = flow_choose(a, M_small, num_cu, 2, true, &uf);
      to_small = us <= uf;
    } else if (to_small) {
      to_small = small_takes(a, M_small, num_cu, a.in_place);
    }
  }
  // Only the split-K kernel writes an upsampled copy.  Where its estimate is below that of the general kernel's tile one launch beats
  // conv_flow_kernel and a launch for the upsampling at every size tried (us: 512 -> 256 on 20 x 20, 1 image 5.2 : 7.4, 8 8.4 : 9.4, 12
  // 9.7 : 11.2; 256 -> 128 on 40 x 40, 2 images 5.8 : 7.5; 384 -> 192 on 40 x 40 5.9 : 7.6; 768 -> 384 on 20 x 20, 8 images 11.1 : 12.5); the next
  // larger batches are left to those two.  The same layer on its own takes it too, so that fused and separate launches sum in one order.
  if (sizeof(T) == 2 && (a.up_y || a.up_next)) {
    const GeneralTile st = general_tile(a, M_split, num_cu, 1, false);
    const int ks = ksplit_choose(a, M_split, (int)sizeof(T), st.bc, st.bp, num_cu);
    if (ks >= 0) return launch_ksplit<T>(ks, a, num_cu, s, kernel_id, tm);
  }
  if (a.up_y) return hipErrorNotSupported;
  if constexpr (sizeof(T) == 2) {
    // conv_flow_kernel takes what has its form, except what conv_small_kernel takes (in a cascade by estimate).  A single strided layer of up to two pipelined
    // 64x64 tiles per compute unit stays with the general kernel: 256 -> 512,
    // stride 2 on 42 x 14 x 14 16.1 us here, 18.1 there, 128 -> 128, stride 2 on 8 x 80 x 80 10.5 : 11.1 (a step of such a tile is four matrix
    // instructions per wavefront, fewer than the cursor's scalar ones).  By tiles per compute unit: 256 -> 256 on 20 x 40 x 40 at 1.95 17.1 :
    // 18.4, 128 -> 64 on 82 x 40 x 40 at 2.0 (513 tiles) 14.6 : 13.9, 96 -> 192 on 9 x 57 x 83 at 2.02 13.4 : 12.5, 192 -> 192 on 7 x 80 x 80 at
    // 2.05 18.0 : 17.2.  Their order of summation is the same, so the running count may choose between these; split-K or not is
    // decided for M_split.
    if (flow_fits(a)) {
      double us = 0;
      int kf = -1;
      if (splittable && !not_split && !stays(M_split)) {
        flow_choose(a, M_split, num_cu, 2, false, &us);
        kf = ksplit_best(a, M_split, 2, num_cu, pw ? 0.85 * us : us, shapes, 4.0);      // (this kernel's estimate of 1x1 layers is 15 % high while it has few tiles)
      }
      if (kf >= 0) return launch_ksplit<T>(kf, a, num_cu, s, kernel_id, tm);
      if (to_small) return run_small(M_small);
      if (!by_place(a) && stays(M)) return launch_cfg<T, 64, 64, 2, 2, 8, 2, 3, true, true, true>(a, num_cu, s, kernel_id, tm);
      const int which = flow_tile >= 0 && M_small == M ? flow_tile : flow_choose(a, M, num_cu, 2, by_place(a), &us);
      return std::is_same<T, __bf16>::value ? launch_flow_bf16(which, a, num_cu, s, kernel_id, tm) : launch_flow_f16(which, a, num_cu, s, kernel_id, tm);
    }
  }
  const GeneralTile st = general_tile(a, M_split, num_cu, 1, pipe_ok);
  const int ks = not_split || st.pipe ? -1 : ksplit_choose(a, M_split, (int)sizeof(T), st.bc, st.bp, num_cu);
  if (ks >= 0) return launch_ksplit<T>(ks, a, num_cu, s, kernel_id, tm);
  const GeneralTile t = general_tile(a, M, num_cu, 1, pipe_ok);
  if constexpr (sizeof(T) == 2) {
    if (to_small) return run_small(M_small);
    if (t.pipe && t.bp == 256) return launch_cfg<T, 128, 256, 2, 2, 4, 2, 2, true, true, true>(a, num_cu, s, kernel_id, tm);
    if (t.pipe && t.bc == 128) return launch_cfg<T, 128, 64, 2, 2, 8, 2, 2, true, true, true>(a, num_cu, s, kernel_id, tm);
    if (t.pipe && t.bp == 128) return launch_cfg<T, 64, 128, 2, 2, 8, 2, 2, true, true, true>(a, num_cu, s, kernel_id, tm);
    if (t.pipe) return launch_cfg<T, 64, 64, 2, 2, 8, 2, 3, true, true, true>(a, num_cu, s, kernel_id, tm);
  }
  if (t.bc == 32) return launch_cfg<T, 32, 128, 1, 4, 4, 2, 4, true>(a, num_cu, s, kernel_id, tm);
  if (t.bp == 256) return launch_cfg<T, 64, 256, 1, 4, 4, 1, 3, true, true>(a, num_cu, s, kernel_id, tm);
  if (t.bc == 128) return launch_cfg<T, 128, 128, 2, 2, 8, 1, 2, true, true>(a, num_cu, s, kernel_id, tm);
  if (t.bp == 128) return launch_cfg<T, 64, 128, 2, 2, 8, 1, 3, true, true>(a, num_cu, s, kernel_id, tm);
  return launch_cfg<T, 64, 64, 2, 2, 8, 1, 4, true, true>(a, num_cu, s, kernel_id, tm);
}

// 8-bit floating point (E4M3) storage: the direct-to-LDS tile shapes only, so the input channels must come in whole
// 16-byte vectors.  Same choice of shape as for the 16-bit types; a K step is 128 (or 64) bytes of K as there, that is
// twice as many values.
#if defined(OCTO_CONV_ONLY_F8)
static hipError_t launch_f8(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) {
  const bool vec = (a.Cin % 16 == 0) && (a.x_ld % 16 == 0) && (a.x_coff % 16 == 0) && (((uintptr_t)a.x & 15) == 0) && a.kh <= 15 && a.kw <= 15;
  if (!vec || !a.scale || a.pair_view) return hipErrorInvalidValue;
  const long long M = (long long)(a.n_hint > 0 && a.n_hint < a.n ? a.n_hint : a.n) * a.Ho * a.Wo;
  // 3x3 layers with enough tiles for every compute unit: input patch in LDS, slices of 64 channels, four workgroups per compute unit
  // (256 -> 256 on 300 x 14 x 14: 39 us, slices of 128 channels 46).  The lines, by 64 x 128 tiles per compute unit: split-K : patch
  // 14 x 14 x 256 at 0.48 8.8 : 9.0, at 0.81 11.4 : 9.2 (7 x 7 x 512 turns below 0.6: 16.3 : 13.1).  128 x 256 tiles where they are the
  // cheaper by whole tiles per compute unit, as in launch_mid (256 -> 256 with residual, 64 x 128 : 128 x 128 : 128 x 256, on 250 x 14 x 14
  // 34.6 : 37.4 : 35.8, on 420 52.9 : 54.5 : 50.6, on 1021 119 : 115 : 113, on 4170 503 : 485 : 454); else 128 channels per tile
  // (and for a single slice, which leaves a large tile mostly epilogue) halve the fetch of the patch from 12 on (at 6 34.6 : 37.4, at 12 112 : 110 (7 x 7 x 512), at 24 119 : 115)
  if (mid_fits(a) && a.Cout > 32 && a.Cin * 4 >= (a.Cin + 63) / 64 * 64 * 3) {
    const double per_cu = (double)M / 128 * ((a.Cout + 63) / 64) / num_cu;
    const bool fits128 = (a.Cout + 127) / 128 * 2 == (a.Cout + 63) / 64;
    const long long items = M / ((long long)a.Ho * a.Wo), huge = fits128 && a.Cin >= 128 ? mid_rounds(a, items, 128, 256, 384, num_cu) : 0;
    const hipError_t em = per_cu < 0.8 ? hipErrorNotSupported
                          : huge >= 2 && 3.5 * huge < mid_rounds(a, items, 64, 128, 192, num_cu) ? launch_mid_cfg<f8, 128, 256, 1, 4, 3, 6, 2>(a, num_cu, s, kernel_id, tm)
                          : per_cu >= 12 && fits128 ? launch_mid_cfg<f8, 128, 128, 1, 4, 3, 3, 3>(a, num_cu, s, kernel_id, tm)
                                                    : launch_mid_cfg<f8, 64, 128, 1, 4, 3, 3, 4>(a, num_cu, s, kernel_id, tm);
    if (em != hipErrorNotSupported) return em;
  }
  const GeneralTile t = general_tile(a, M, num_cu, 2);
  const int ks = ksplit_choose(a, M, 1, t.bc, t.bp, num_cu);
  if (ks >= 0) return launch_ksplit<f8>(ks, a, num_cu, s, kernel_id, tm);
  // conv_flow_kernel as for the 16-bit types, by the same estimate with steps of 128 values (general : flow, us: 96 -> 96 1x1 on 32 x 160 x 160
  // 76.8 : 50.1, 192 -> 192 148.7 : 97.7, 1024 -> 256 on 60 x 14 x 14 11.2 : 8.1, 48 -> 96, stride 2 on 32 x 640 x 640 435 : 307, 256 -> 512, stride 2 on
  // 4170 x 14 x 14 298 : 257, 128 -> 256, stride 2 on 8 x 80 x 80 12.2 : 10.2).  Half a step into one 64-channel tile stays on the 64 x 256
  // tiles with 64-byte steps (48 -> 48 on 32 x 320 x 320 124 : 130, 32 -> 64 on 16 x 160 x 160 20.1 : 21.6) but for 56 channels, which those tiles
  // write byte by byte (16 -> 56 on 104 x 57 x 59 34.9 : 20.7); so do up to 40 channels of short reductions (32 -> 40 on 1651 x 21 x 13 21.9 : 30.3, 3x3
  // 16 -> 32 on 256 x 73 x 94 79 : 96, 48 -> 24 77 : 87; 96 -> 24 on 56 x 158 x 133 55 : 57, 256 -> 24 on 209 x 34 x 38 25.5 : 18.9, 3x3 304 -> 24 on
  // 1526 x 25 x 15 268 : 159).  Other half vectors and single steps into several channel tiles: 16 -> 88 on 45 x 159 x 224 339 : 149, 96 -> 184, stride 2 on
  // 142 x 75 x 96 60.5 : 32.7, 16 -> 648, stride 2 on 780 x 33 x 37 202 : 131; over 164 such layers 0.80 of the general kernel's time.
  if (flow_fits(a, 1) && (a.Cout >= 48 ? a.K > 64 || a.Cout > 64 || a.Cout % 16 : a.Cin >= 96)) {
    double us = 0;
    return launch_flow_f8(flow_choose(a, M, num_cu, 1, false, &us), a, num_cu, s, kernel_id, tm);
  }
  if (t.bc == 128) return launch_cfg<f8, 128, 128, 2, 2, 8, 1, 2, true, true>(a, num_cu, s, kernel_id, tm);
  if (t.bp == 256) return launch_cfg<f8, 64, 256, 1, 4, 4, 1, 3, true, true>(a, num_cu, s, kernel_id, tm);
  if (t.bp == 128) return launch_cfg<f8, 64, 128, 2, 2, 8, 1, 3, true, true>(a, num_cu, s, kernel_id, tm);
  return launch_cfg<f8, 64, 64, 2, 2, 8, 1, 4, true, true>(a, num_cu, s, kernel_id, tm);
}
#endif

#if defined(OCTO_CONV_ONLY_F16)
hipError_t launch_general_f16(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_typed<_Float16>(a, num_cu, s, kernel_id, tm); }
#elif defined(OCTO_CONV_ONLY_BF16)
hipError_t launch_general_bf16(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_typed<__bf16>(a, num_cu, s, kernel_id, tm); }
#elif defined(OCTO_CONV_ONLY_F32)
hipError_t launch_general_f32(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_typed<float>(a, num_cu, s, kernel_id, tm); }
#elif defined(OCTO_CONV_ONLY_F8)
hipError_t launch_general_f8(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_f8(a, num_cu, s, kernel_id, tm); }
#else
hipError_t launch_general_f16(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_general_bf16(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_general_f32(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);
hipError_t launch_general_f8(const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm);

size_t conv_packed_weight_elems(int cout, int kh, int kw, int cin, int dtype, int* kp_out, int* cout_pad_out) {
  const int vn = 16 / dtype_size(dtype);
  const int bk = 8 * vn;   // largest K step of any tile configuration
  const int K = kh * kw * cin;
  const int kp = (K + bk - 1) / bk * bk;
  const int cp = (cout + 127) / 128 * 128;
  if (kp_out) *kp_out = kp;
  if (cout_pad_out) *cout_pad_out = cp;
  return (size_t)kp * cp;
}

// Checks the limits the kernel relies on and fills the precomputed reciprocals.
bool conv_prepare(ConvArgs& a, int dtype) {
  if (a.Cin < 1 || a.kw < 1 || a.kh < 1 || a.stride_h < 1 || a.stride_w < 1 || a.Kp >= 65536 || a.w_rows < 1) return false;
  // a tile addresses its pixels with 32-bit byte offsets from the first image it touches: at most two images plus
  // 256 output pixels' worth of further images
  if ((2LL * a.H * a.W + 1024LL * a.stride_h * a.stride_w) * a.x_ld * dtype_size(dtype) > 0x7FFFFFF0LL) return false;
  if ((long long)a.n * a.Ho * a.Wo >= 0x7FFFFFFFLL) return false;
  // floor(n / d) = umulhi(n, magic) >> shift, exact for n < 2^31
  auto magic = [](unsigned d, unsigned* mg, unsigned* sh) {
    unsigned s = 0;
    while ((1ull << s) < d) ++s;
    const unsigned long long m = ((1ull << (32 + s)) + d - 1) / d;
    if (m >> 32) { *mg = (unsigned)(((1ull << (31 + s)) + d - 1) / d); *sh = s - 1; }
    else { *mg = (unsigned)m; *sh = s; }
  };
  a.HoWo_is_one = (a.Ho * a.Wo == 1) ? 1 : 0;
  if (!a.HoWo_is_one) magic((unsigned)(a.Ho * a.Wo), &a.magic_howo, &a.shift_howo);
  if (a.Wo > 1) magic((unsigned)a.Wo, &a.magic_wo, &a.shift_wo);
  a.magic_cin = a.Cin > 1 ? (unsigned)((1ull << 32) / (unsigned)a.Cin) + 1u : 0u;
  a.magic_kw = a.kw > 1 ? (unsigned)((1ull << 32) / (unsigned)a.kw) + 1u : 0u;
  return true;
}

__global__ __launch_bounds__(256) void held_pack_kernel(const u32x4* w, int kp, int cin, int n, u32x4* out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int lane = i & 63, m = lane & 31, g = i >> 6, tap = g % 9, c = g / 9 % (cin / 16), k = g / 9 / (cin / 16) * 32 + 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
  out[i] = w[((size_t)k * kp + tap * cin + c * 16 + (lane >> 5) * 8) / 8];
}
hipError_t launch_held_pack(const void* w, int kp, int cin, int cout, void* out, hipStream_t s) {
  const int n = cout * (cin / 8) * 9;
  hipLaunchKernelGGL(held_pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const u32x4*)w, kp, cin, n, (u32x4*)out);
  return hipGetLastError();
}

hipError_t launch_conv(int dtype, const ConvArgs& a0, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm) {
  ConvArgs a = a0;
  if (!conv_prepare(a, dtype)) return hipErrorInvalidValue;
  if (a.split > 0) {
    // two layers in one launch: the streaming 1x1 kernel, conv_flow_kernel (a split in whole blocks of 32 channels), the split-K kernel and
    // the general kernel's staged epilogue write two tensors
    const bool ok = (dtype == OCTO_F16 || dtype == OCTO_BF16) && a.y2 && !a.res && !a.out_f32 && !a.pair_view && !a.pool_y && a.split < a.Cout &&
                    ((a.split | a.Cout | a.y_ld | a.y_coff | a.y2_ld | a.y2_coff) & 7) == 0 && ((((uintptr_t)a.y | (uintptr_t)a.y2) & 15) == 0);
    if (!ok) return hipErrorNotSupported;
    const hipError_t e1 = launch_conv1x1_stream(dtype, a, num_cu, s, kernel_id, tm);
    if (e1 != hipErrorNotSupported) return e1;
    return dtype == OCTO_F16 ? launch_general_f16(a, num_cu, s, kernel_id, tm) : launch_general_bf16(a, num_cu, s, kernel_id, tm);
  }
  if (a.up_y) {
    // the output and its upsampled copy from one launch: the split-K kernel (launch_typed refuses the others; in the
    // general kernel's epilogue the test for it alone cost every layer 2 %)
    const bool ok = (dtype == OCTO_F16 || dtype == OCTO_BF16) && !a.out_f32 && !a.pair_view && !a.pool_y && a.kh == 1 && a.kw == 1 &&
                    ((a.Cout | a.y_ld | a.y_coff | a.up_ld | a.up_coff) & 7) == 0 && (a.Cin & 7) == 0 && ((a.x_ld | a.x_coff) & 7) == 0 &&
                    ((((uintptr_t)a.x | (uintptr_t)a.y | (uintptr_t)a.up_y) & 15) == 0);
    if (!ok) return hipErrorNotSupported;
    return dtype == OCTO_F16 ? launch_general_f16(a, num_cu, s, kernel_id, tm) : launch_general_bf16(a, num_cu, s, kernel_id, tm);
  }
  const hipError_t es = launch_stem(dtype, a, num_cu, s, kernel_id, tm);
  if (es != hipErrorNotSupported || a.pool_y) return es;      // only the first-layer kernel can pool its own output
  const hipError_t e1 = launch_conv1x1_stream(dtype, a, num_cu, s, kernel_id, tm);
  if (e1 != hipErrorNotSupported) return e1;
  switch (dtype) {
    case OCTO_F8: return launch_general_f8(a, num_cu, s, kernel_id, tm);
    case OCTO_F16: return launch_general_f16(a, num_cu, s, kernel_id, tm);
    case OCTO_BF16: return launch_general_bf16(a, num_cu, s, kernel_id, tm);
    case OCTO_F32: return launch_general_f32(a, num_cu, s, kernel_id, tm);
  }
  return hipErrorInvalidValue;
}
#endif   // the main translation unit
#endif   // launchers

}  // namespace octo
