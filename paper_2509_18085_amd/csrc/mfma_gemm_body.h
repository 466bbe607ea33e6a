  // (body of gemm_bf16_mfma_kernel and gemm_tile: EPI, BN, SD, BMT, SA, a, tiles_i, tiles_j, wave)
  constexpr int BM = BMT;                         // rows of the output tile: 256, or 128 / 64 / 32 when there are few rows
  constexpr int WM = waves_m(EPI, BMT, BN), WN = waves_n(EPI, BMT, BN), NW = WM * WN;
  constexpr int RW = BM / WM, CW = wave_cols(EPI, BMT, BN);  // rows and columns of the tile that one wavefront owns
  constexpr int NW_MATH = WM * (BN / CW);          // wavefronts that own a part of the tile (all but one of a 96-column tile's)
  static_assert(EPI != EPI_LMHEAD || (NW == 4 && RW == 128), "a part of the summaries is 128 vocabulary rows");
  static_assert(RW % 32 == 0 && CW % 32 == 0, "a wavefront owns whole MFMA tiles");
  // which operand is the weight matrix (deep ring): Y for the projections, X for the LM head
  constexpr bool XDEEP = (EPI == EPI_LMHEAD);
  // The deep operand (weights) rides a ring of SD stages and is loaded SD tiles ahead; the shallow one (activations)
  // a ring of SH stages, SH tiles ahead.  The load counter retires in order, so waiting for the shallow operand of
  // the next tile also waits for every older load: across a barrier stay in flight the deep loads issued with that
  // shallow tile and the SH-2 whole groups after it (SH = 2: only the newest weight tile, whatever SD; SH = SD, the
  // weight-streaming shapes with few rows: SD-2 whole tiles).
  constexpr int SH = shallow_stages(EPI, BN, BMT, SD, SA);
  static_assert(SH >= 2 && SH <= SD, "the shallow ring is at most as deep as the deep one");
  constexpr int SX = XDEEP ? SD : SH, SY = XDEEP ? SH : SD;
  constexpr int TM = RW / 32, TN = CW / 32;
  constexpr int LX = BM / (8 * NW), LY = BN / (8 * NW);   // 1-KB wave-loads (8 rows x 128 B) per wavefront per K-tile
  constexpr int NL = LX + LY;
  constexpr int XSTAGE = BM * BKK, YSTAGE = BN * BKK;
  constexpr int NMF = TM * TN, NF = TM + TN;
  constexpr int NSLOT = 4 * NMF;                  // MFMAs between two barriers
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* Xs = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* Ys = Xs + SX * XSTAGE;

  const int lane = EPI == EPI_LMHEAD ? lane_id() : threadIdx.x & 63;
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, hh = lane >> 5;
  const bool math = NW_MATH == NW || wave < NW_MATH;    // wavefront-uniform

  int i_max, j_max, kz, ti, tj;
  if (EPI == EPI_LMHEAD) {
    // The grid covers the row capacity; the number of rows in use is only known on the device.  The first
    // (vocabulary tiles x token tiles in use) workgroup ids take the real tiles, token tiles running fastest
    // so that the workgroups sharing a vocabulary tile sit next to each other on one XCD; the rest leave.
    i_max = a.N;
    j_max = a.M_dev ? min(*a.M_dev, a.M) : a.M;
    const int used_j = (j_max + BN - 1) / BN;
    const int used = tiles_i * used_j;
    if ((int)blockIdx.x >= used) return;
    const int L = xcd_contiguous(blockIdx.x, used);
    kz = 0;
    ti = L / used_j;
    tj = L % used_j;
  } else {
    // XCD-aware order: workgroup ids go round-robin over the 8 XCDs; give each XCD a contiguous range
    // of logical tiles, running fastest over the activation tiles, so the workgroups that stream the
    // same weight tile share one L2 and run at the same time.
    const int per_z = tiles_i * tiles_j;
    kz = blockIdx.x / per_z;
    const int L = xcd_contiguous(blockIdx.x % per_z, per_z);
    ti = L % tiles_i;
    tj = L / tiles_i;
    i_max = a.M_dev ? min(*a.M_dev, a.M) : a.M;
    j_max = a.N;
    if (ti * BM >= i_max) return;
  }
  const int i0 = ti * BM, j0 = tj * BN;

  const int ldw = a.ldw ? a.ldw : a.K;
  // K range of this slice
  const int KT_all = a.K / BKK;
  const int kt0 = (int)(((long long)KT_all * kz) / a.ksplit);
  const int KT = (int)(((long long)KT_all * (kz + 1)) / a.ksplit) - kt0;

  // ---- global sources.  A wave-load covers 8 rows; lane -> (row, swizzled 16-byte chunk).  Addresses are a
  // wavefront-uniform base (scalar registers) plus a 32-bit per-lane byte offset that never changes: the
  // loads take the scalar-base form and the K loop needs no vector arithmetic for them.
  const char* xbase;
  const char* ybase[LY];
  unsigned xoff[LX], yoff[LY];
  {
    const bf16_t* X = (EPI == EPI_LMHEAD) ? (const bf16_t*)a.W[0] : (const bf16_t*)a.A;
    const int ldx = (EPI == EPI_LMHEAD) ? ldw : a.lda;
    xbase = reinterpret_cast<const char*>(X + (size_t)kt0 * BKK);
#pragma unroll
    for (int q = 0; q < LX; ++q) {
      const int row = 8 * (wave * LX + q) + (lane >> 3);
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      int gi = min(i0 + row, i_max - 1);
      if (EPI == EPI_PARTIAL && a.a_rows) gi = a.a_rows[gi];
      xoff[q] = (unsigned)gi * (unsigned)(ldx * 2) + chunk * 16;
    }
#pragma unroll
    for (int q = 0; q < LY; ++q) {
      const int row0 = 8 * (wave * LY + q);            // first row of the wave-load: uniform
      const int row = row0 + (lane >> 3);
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      const bf16_t* base;
      int r;                                            // row inside the matrix `base` points to
      if (EPI == EPI_LMHEAD) {
        base = (const bf16_t*)a.A;
        r = min(j0 + row, j_max - 1);
        yoff[q] = (unsigned)r * (unsigned)(a.lda * 2) + chunk * 16;
      } else {
        if (EPI == EPI_SWIGLU) {
          // rows of every 32-row MFMA tile: 16 gate rows then the 16 up rows of the same features
          base = (row0 & 16) ? (const bf16_t*)a.W[1] : (const bf16_t*)a.W[0];
          r = tj * (BN / 2) + (row >> 5) * 16 + (row & 15);
        } else {
          base = (const bf16_t*)a.W[0];
          r = j0 + row;
          if (EPI == EPI_QKV) {
            const int n0 = j0 + row0;   // column of the fused q | k | v output; 8-row groups never straddle
            if (n0 >= a.Nseg[0] + a.Nseg[1]) { base = (const bf16_t*)a.W[2]; r -= a.Nseg[0] + a.Nseg[1]; }
            else if (n0 >= a.Nseg[0]) { base = (const bf16_t*)a.W[1]; r -= a.Nseg[0]; }
            // rows of every 32-row MFMA tile: 16 columns of a head, then the 16 columns 64 further on that rotate with them
            r = (r & ~127) + 16 * ((r >> 5) & 3) + 64 * ((r >> 4) & 1) + (r & 15);
          }
        }
        yoff[q] = (unsigned)r * (unsigned)(ldw * 2) + chunk * 16;
      }
      ybase[q] = reinterpret_cast<const char*>(base + (size_t)kt0 * BKK);
    }
  }
  // 16 bytes per lane, global (scalar base + 32-bit lane offset) -> LDS (M0 = destination of lane 0).  Written
  // out because the compiler only emits the 64-bit-lane-address form, which costs a 64-bit vector add per load.
  auto dma16 = [](const char* ubase, unsigned lane_off, const bf16_t* lds_dst) {
    const unsigned m0v = (unsigned)(size_t)(lds_ptr_t)lds_dst;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(m0v), "v"(lane_off), "s"(ubase) : "memory");
  };
  auto load_x = [&](int q, int t) {
    dma16(xbase + (size_t)t * (BKK * 2), xoff[q], Xs + (t % SX) * XSTAGE + (wave * LX + q) * 512);
  };
  auto load_y = [&](int q, int t) {
    dma16(ybase[q] + (size_t)t * (BKK * 2), yoff[q], Ys + (t % SY) * YSTAGE + (wave * LY + q) * 512);
  };
  constexpr int LS = XDEEP ? LY : LX, LD = XDEEP ? LX : LY;   // wave-loads of the shallow / deep operand
  auto load_sh = [&](int q, int t) { if (XDEEP) load_y(q, t); else load_x(q, t); };
  auto load_dp = [&](int q, int t) { if (XDEEP) load_x(q, t); else load_y(q, t); };
  // load `idx` of group g (the loads issued after barrier g): shallow operand of tile g+SH first, then
  // the deep operand of tile g+SD
  constexpr int SH_AHEAD = SH;
  auto group_load = [&](int idx, int g, bool checked = true) {
    if (idx < LS) { if (!checked || g + SH_AHEAD < KT) load_sh(idx, g + SH_AHEAD); }
    else { if (!checked || g + SD < KT) load_dp(idx - LS, g + SD); }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // short K: not enough tiles for the steady-state wait counts, wait for everything each time
  const bool short_k = KT <= SD;
  // prologue, in the order the partial waits rely on: D0 S0 | D1 [S1] .. D(SD-2) [S(SD-2)] (shallow tiles up to SH-2)
  // | first quarter of group -1 (what a "K step 3 of tile -1" would have issued); the loop issues the rest
  static_assert(SD >= 3, "the steady-state wait keeps one deep-operand tile in flight across the barrier");
#pragma unroll
  for (int q = 0; q < LD; ++q) load_dp(q, 0);
#pragma unroll
  for (int q = 0; q < LS; ++q) load_sh(q, 0);
#pragma unroll
  for (int t = 1; t < SD - 1; ++t)
    if (t < KT) {
#pragma unroll
      for (int q = 0; q < LD; ++q) load_dp(q, t);
      if (t < SH - 1) {
#pragma unroll
        for (int q = 0; q < LS; ++q) load_sh(q, t);
      }
    }
#pragma unroll
  for (int idx = 0; idx < NL / 4; ++idx) group_load(idx, -1);

  const int sw_r = (l32 >> 1) & 7;
  const int xrow = (wm * RW + l32) * BKK;
  const int yrow = (wn * CW + l32) * BKK;
  bf16x8 fx[2][TM], fy[2][TN];
  auto ldfrag = [&](int buf, const bf16_t* xs, const bf16_t* ys, int kk, int r) {
    if (!math) return;
    const int slot = ((kk * 2 + hh) ^ sw_r) * 8;
    if (r < TM) fx[buf][r] = *reinterpret_cast<const bf16x8*>(xs + xrow + r * 32 * BKK + slot);
    else fy[buf][r - TM] = *reinterpret_cast<const bf16x8*>(ys + yrow + (r - TM) * 32 * BKK + slot);
  };
  // loads younger than tile 0's: the deep halves of tiles 1 .. SD-2, the shallow halves of tiles 1 .. SH-2, and the
  // start of group -1.  Steady state: younger than the shallow operand of the next tile are the deep loads of its
  // own group and the SH-2 groups after it (every group when both rings have the same depth).
  constexpr int W_FIRST = (SD - 2) * LD + (SH - 2) * LS + NL / 4;
  constexpr int W_STEADY = SH == SD ? (SD - 2) * NL : LD + (SH - 2) * NL;
  static_assert(W_FIRST <= 63 && W_STEADY <= 63, "vmcnt is a 6-bit counter");
  if (short_k) wait_vmcnt<0>(); else wait_vmcnt<W_FIRST>();   // tile 0 is in LDS
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int r = 0; r < NF; ++r) ldfrag(0, Xs, Ys, 0, r);

  // fragment reads of the next K step issued after MFMA m of the current one: [frag_lo(m), frag_lo(m+1)).
  // One per MFMA from the second on when there are enough MFMAs, else spread over all but the last.
  auto frag_lo = [](int m) {
    if (NMF == 1) return m < 1 ? 0 : NF;
    if (NF <= NMF - 1) return m < 1 ? 0 : (m - 1 < NF ? m - 1 : NF);
    return m < NMF - 1 ? (m * NF) / (NMF - 1) : NF;
  };
  // Weights as the A operand (ROW_LANES): a lane owns one row of the result (a token) and runs of four columns, so the
  // epilogues work inside a lane - no partner values to fetch - and store 16 bytes at a time (gate/up at 1024 rows
  // 160 -> 157 us, 768 rows of 18944 features 146 -> 139).  The LM head has its vocabulary there anyway; fp32 partials keep
  // 32 columns side by side in the lanes, whole 128-byte lines a store (1 - 2 us faster at 1024 rows than 16-byte runs of
  // 32 rows).
  constexpr bool ROW_LANES = EPI != EPI_LMHEAD && EPI != EPI_PARTIAL;
  auto mfma = [&](int i, int j, int buf) {
    if (!math) return;
    acc[i][j] = !ROW_LANES ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[buf][i], fy[buf][j], acc[i][j], 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fy[buf][j], fx[buf][i], acc[i][j], 0, 0, 0);
  };
  // one K-tile; STEADY = every tile this iteration prefetches exists (no bounds checks, no branches)
  auto k_tile = [&](int kt, auto steady_tag) {
    constexpr bool STEADY = decltype(steady_tag)::value;
    const bf16_t* xs = Xs + (kt % SX) * XSTAGE;
    const bf16_t* ys = Ys + (kt % SY) * YSTAGE;
    // K steps 0..2 of the tile: MFMAs on fragment buffer kk&1, fragments of step kk+1 into the other
    // buffer, remaining loads of group kt-1
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
#pragma unroll
      for (int m = 0; m < NMF; ++m) {
        const int i = m / TN, j = m % TN;
        mfma(i, j, kk & 1);
#pragma unroll
        for (int r = frag_lo(m); r < frag_lo(m + 1); ++r) ldfrag((kk + 1) & 1, xs, ys, kk + 1, r);
        const int slot = NMF + kk * NMF + m;      // position among the NSLOT MFMAs that follow barrier kt-1
#pragma unroll
        for (int idx = (slot * NL) / NSLOT; idx < ((slot + 1) * NL) / NSLOT; ++idx) group_load(idx, kt - 1, !STEADY);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // barrier kt: tile kt+1 is in LDS for every wavefront (only the deep-operand loads of group kt-1
    // may still fly), and no wavefront reads the stages of tile kt after this point
    if (STEADY || (!short_k && kt + SD - 1 < KT)) wait_vmcnt<W_STEADY>(); else wait_vmcnt<0>();
    wait_lgkm0();
    __builtin_amdgcn_s_barrier();
    const bf16_t* xs1 = Xs + ((kt + 1) % SX) * XSTAGE;
    const bf16_t* ys1 = Ys + ((kt + 1) % SY) * YSTAGE;
    // K step 3: MFMAs on buffer 1, fragments (kt+1, step 0) into buffer 0, first loads of group kt
#pragma unroll
    for (int m = 0; m < NMF; ++m) {
      const int i = m / TN, j = m % TN;
      mfma(i, j, 1);
#pragma unroll
      for (int r = frag_lo(m); r < frag_lo(m + 1); ++r) ldfrag(0, xs1, ys1, 0, r);
#pragma unroll
      for (int idx = (m * NL) / NSLOT; idx < ((m + 1) * NL) / NSLOT; ++idx) group_load(idx, kt, !STEADY);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // steady state: kt >= 1 (group kt-1 exists as a whole) and kt + SD < KT (everything prefetched exists)
  int kt = 0;
  if (!short_k) {
    k_tile(0, std::false_type{});
    for (kt = 1; kt + SD < KT; ++kt) k_tile(kt, std::true_type{});
  }
  for (; kt < KT; ++kt) k_tile(kt, std::false_type{});
  if (!math) return;      // (no barrier follows the K loop)


  if (EPI == EPI_LMHEAD) {
    const int lane_e = lane_id(), e32 = lane_e & 31, eh = lane_e >> 5;
    // accumulator element (i,j,v) of this lane: row = i0 + wm*RW + i*32 + 8*(v/4) + 4*eh + v%4, column wn*CW + j*32 + e32
    // of the tile
    // Per token column: top value, its lowest vocabulary index, runner-up and sum of exponentials over the
    // lane's 64 vocabulary rows, on the unscaled accumulators (the scale is positive, so the order is the
    // same); the lane's rows are visited in increasing vocabulary index, so "strictly greater" keeps the
    // lowest index among equals.  One median-of-three per value maintains the runner-up.
    TopPartial* part = reinterpret_cast<TopPartial*>(a.C);
    const float c = a.scale * 1.4426950408889634f;
    auto reduce_columns = [&](auto checked_tag) {
      constexpr bool CHECKED = decltype(checked_tag)::value;   // the last vocabulary tile: rows beyond V count as -inf
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        float m = -INFINITY, m2 = -INFINITY;
        int code = 0;      // 16 * i + v of the top value
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float l = acc[i][j][v];
            if (CHECKED) {
              const int idx = i0 + wm * RW + i * 32 + 8 * (v >> 2) + 4 * eh + (v & 3);
              if (idx >= i_max) l = -INFINITY;
              acc[i][j][v] = l;
            }
            m2 = __builtin_amdgcn_fmed3f(m, m2, l);
            code = l > m ? 16 * i + v : code;
            m = __builtin_amdgcn_fmed3f(m, l, INFINITY);   // max(m, l) as one instruction
          }
        // in the last tile a lane may have no row below V: it keeps m = -inf and contributes nothing
        const float mc = (m == -INFINITY) ? 0.f : m * c;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][v], c, -mc));
        Top t;
        t.m = m * a.scale;
        t.m2 = m2 * a.scale;
        t.s = sum;
        t.idx = (m == -INFINITY) ? 0x7fffffff
                                 : i0 + wm * RW + (code >> 4) * 32 + 8 * ((code & 15) >> 2) + 4 * eh + (code & 3);
        t = top_merge(t, top_shfl_xor(t, 32));
        const int tokr = j0 + wn * CW + j * 32 + e32;
        if (eh == 0 && tokr < j_max) part[(size_t)(ti * WM + wm) * a.ldc + tokr] = TopPartial{t.m, t.m2, t.s, t.idx};
      }
    };
    if (i0 + BM <= i_max) reduce_columns(std::false_type{}); else reduce_columns(std::true_type{});
    return;
  }

  if (EPI == EPI_PARTIAL) {
    // accumulator elements as for the LM head
    float* P = reinterpret_cast<float*>(a.C) + (size_t)kz * (a.Mz ? a.Mz : a.M) * a.ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = i0 + wm * RW + i * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
        if (r >= i_max) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) P[(size_t)r * a.ldc + j0 + wn * CW + j * 32 + l32] = acc[i][j][v];
      }
    return;
  }

  // accumulator element (i,j,v) of this lane: row i0 + wm*RW + i*32 + l32, column wn*CW + j*32 + 8*(v/4) + 4*hh + v%4 of the
  // tile: four runs of four columns, the lane 32 further on holds the runs in between
  const int r_lane = i0 + wm * RW + l32;
  // Sixteen consecutive columns of the lane's row: run 0 of the lower lane, run 0 of the upper, run 1 of the lower, run 1 of
  // the upper.  The lanes trade run 1 against run 0 and hold eight columns each: columns 8*hh .. 8*hh+7, one 16-byte store.
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  auto pack2 = [](float x, float y) {
    bf16x2 t;
    t[0] = static_cast<bf16_t>(x);
    t[1] = static_cast<bf16_t>(y);
    return __builtin_bit_cast(unsigned int, t);
  };
  auto pack16 = [&](const float (&x)[8]) {     // x: run 0, run 1
    const u32x2 s0 = __builtin_amdgcn_permlane32_swap(pack2(x[0], x[1]), pack2(x[4], x[5]), false, false);
    const u32x2 s1 = __builtin_amdgcn_permlane32_swap(pack2(x[2], x[3]), pack2(x[6], x[7]), false, false);
    return u32x4{s0[0], s1[0], s0[1], s1[1]};
  };

  // A 256 x 256 tile's accumulators fill the accumulation registers.  Its epilogues take each out where it is used: copied
  // ahead of time, as the compiler likes to, they pushed 2 (gate/up) and 144 (QKV) registers into scratch memory (QKV, 12288
  // columns: 1056 rows of 4096 110.1 -> 103.3 us, 4096 rows 358.9 -> 327.6, 4096 rows of 1024 139 -> 110).
  auto keep_in_place = [](f32x16& x) {
    if constexpr (TM * TN >= 16) asm volatile("" : "+a"(x));
  };

  bf16_t* C = reinterpret_cast<bf16_t*>(a.C);
  if (EPI == EPI_SWIGLU) {
    // columns 0 .. 15 of a 32-column block are gate values, 16 .. 31 the up values of the same features
    bf16_t* Cl = C + tj * (BN / 2) + wn * TN * 16 + 8 * hh;
    auto silu_mul = [](float g, float u) { return g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * u; };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = r_lane + i * 32;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        keep_in_place(acc[i][j]);
        float h[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) h[v] = silu_mul(acc[i][j][v], acc[i][j][v + 8]);
        const u32x4 o = pack16(h);
        if (r < i_max) *reinterpret_cast<u32x4*>(Cl + (size_t)r * a.ldc + j * 16) = o;
      }
    }
    return;
  }

  if (EPI == EPI_QKV) {
    // columns 0 .. 15 of a 32-column block are columns c of a head, 16 .. 31 the columns c + 64 that rotate with them.
    // The launch takes 0.3 - 2.6 us more than with the plain store (1024 rows of 4096 88.0 -> 90.6, 768 rows of 3584 38.7 -> 40.9, 256
    // rows 43.7 -> 44.0).  It pays through the attention kernel, which rotated queries and own keys in front of its first product,
    // one wavefront at a time (3 us), and the launch of its own that extended the cache (5 us).
    const QkvArgs& q = a.qkv;
    auto seg_of = [&](int n0) { return n0 < a.Nseg[0] ? 0 : (n0 < a.Nseg[0] + a.Nseg[1] ? 1 : 2); };
    auto col_of = [&](int n0) { const int s = seg_of(n0); return n0 - (s == 0 ? 0 : (s == 1 ? a.Nseg[0] : a.Nseg[0] + a.Nseg[1])); };
    // The angles of the next 32 rows are loaded in front of the stores of these: vector stores and loads retire in order, and
    // a load behind a store waits for it.
    f32x4 ang[2][TN][4];                           // (cos, sin) of frequencies 0, 1 | 2, 3 of run 0, then of run 1
    auto load_angles = [&](int i) {
      const int g = min(r_lane + i * 32, i_max - 1) + q.row0;
      const int trow = g >= q.rows ? g - q.rows + q.B : q.B > 1 ? g - (int)__umulhi((unsigned)g, q.magic) * q.B : 0;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int fr = 16 * ((col_of(j0 + wn * CW + j * 32) >> 5) & 3);
        const f32x4* t = reinterpret_cast<const f32x4*>(q.rope) + (size_t)(fr / 2 + 2 * hh) * q.rope_rows + trow;
#pragma unroll
        for (int u = 0; u < 4; ++u) ang[i & 1][j][u] = t[(size_t)(4 * (u >> 1) + (u & 1)) * q.rope_rows];
      }
    };
    load_angles(0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i + 1 < TM) load_angles(i + 1);
      const int r = r_lane + i * 32, g = r + q.row0;
      // row of the cache this row extends it by, or -1
      const int dst = r >= i_max ? -1 : g < q.n_head ? q.dst_head + g : g >= q.rows && q.dst_tail >= 0 ? q.dst_tail + g - q.rows : -1;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n0 = j0 + wn * CW + j * 32;      // uniform; a 32-column block is part of one head of q, k or v
        const int seg = seg_of(n0), c0 = col_of(n0);
        const int hcol = c0 & ~127, fr = 16 * ((c0 >> 5) & 3);       // head's first column, first frequency
        keep_in_place(acc[i][j]);
        float x1[8], x2[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) { x1[v] = acc[i][j][v]; x2[v] = acc[i][j][v + 8]; }
        const void* bias = seg == 0 ? a.bias[0] : (seg == 1 ? a.bias[1] : a.bias[2]);
        if (bias) {
          const bf16_t* bp = (const bf16_t*)bias + hcol + fr + 4 * hh;
#pragma unroll
          for (int v = 0; v < 8; v += 4) {
            const bf16x4 b1 = *reinterpret_cast<const bf16x4*>(bp + 2 * v), b2 = *reinterpret_cast<const bf16x4*>(bp + 64 + 2 * v);
#pragma unroll
            for (int e = 0; e < 4; ++e) { x1[v + e] += static_cast<float>(b1[e]); x2[v + e] += static_cast<float>(b2[e]); }
          }
        }
        if (seg < 2) {
          const float scale = seg == 0 ? q.q_scale : 1.f;
#pragma unroll
          for (int v = 0; v < 8; v += 4) {
            const f32x4 ta = ang[i & 1][j][v >> 1], tb = ang[i & 1][j][(v >> 1) + 1];
            const float c[4] = {ta[0], ta[2], tb[0], tb[2]}, s[4] = {ta[1], ta[3], tb[1], tb[3]};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              // rotated as the rounded values that a reader of the unrotated columns would rotate
              const float u1 = static_cast<float>(static_cast<bf16_t>(x1[v + e])), u2 = static_cast<float>(static_cast<bf16_t>(x2[v + e]));
              x1[v + e] = (u1 * c[e] - u2 * s[e]) * scale;
              x2[v + e] = (u2 * c[e] + u1 * s[e]) * scale;
            }
          }
        }
        const u32x4 o1 = pack16(x1), o2 = pack16(x2);
        if (r < i_max) {
          bf16_t* p = C + (size_t)r * a.ldc + (n0 - c0) + hcol + fr + 8 * hh;
          *reinterpret_cast<u32x4*>(p) = o1;
          *reinterpret_cast<u32x4*>(p + 64) = o2;
        }
        if (seg > 0 && dst >= 0) {
          bf16_t* p = reinterpret_cast<bf16_t*>(seg == 1 ? q.ck : q.cv) + ((size_t)(hcol >> 7) * q.ldp + dst) * 128 + fr + 8 * hh;
          *reinterpret_cast<u32x4*>(p) = o1;
          *reinterpret_cast<u32x4*>(p + 64) = o2;
        }
      }
    }
    return;
  }

  const bf16_t* R = reinterpret_cast<const bf16_t*>(a.R);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = r_lane + i * 32;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v0 = 0; v0 < 16; v0 += 8) {       // sixteen columns
        const int n = j0 + wn * CW + j * 32 + 2 * v0;
        float x[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) x[v] = acc[i][j][v0 + v];
        if (EPI == EPI_RESID && r < i_max) {
          const bf16_t* rp = R + (size_t)r * a.ldc + n + 4 * hh;
#pragma unroll
          for (int v = 0; v < 8; v += 4) {
            const bf16x4 rr = *reinterpret_cast<const bf16x4*>(rp + 2 * v);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[v + e] += static_cast<float>(rr[e]);
          }
        }
        const u32x4 o = pack16(x);
        if (r < i_max) *reinterpret_cast<u32x4*>(C + (size_t)r * a.ldc + n + 8 * hh) = o;
      }
  }
