// The body of conv_small_kernel and conv_small_group_kernel (conv_small.h, which includes it inside each): all tiles of a workgroup.  `a`: the layer's SmallArgs, `block`: the workgroup's number
// in its layer.  Not a function that both call: conv_small_kernel then gets other registers and more spills, and fp32 layers of windows take 1 - 3 % longer (28 -> 24, 3x3 on 11 x 83 x 70
// 14.8 : 15.3 us, 384 -> 656 on 27 x 14 x 12 175.6 : 178.2).
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
