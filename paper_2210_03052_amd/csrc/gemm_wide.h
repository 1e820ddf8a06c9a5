// The wide-tile product kernel (included by gemm.hip).
//
//   C = epilogue(A W^T),  block tile BM x BN x 64, four wavefronts in a 2 x 2 grid (one per SIMD), wave tile
//   (BM/2) x (BN/2) of 16x16x32 MFMA blocks, three operand stages in LDS (NS; four for some, see wide_stages), tiles taken
//   one after another.
//
// What it is built around:
//  - LDS traffic.  With eight wavefronts of 64 x 64 the fragment reads of a 256 x 128 x 64 slab are 128 KB and, with the
//    48 KB that the DMA writes, keep LDS busy for about as long as the slab's MFMAs take (1 294 cycles a slab measured,
//    1 024 of them MFMA); four wavefronts of 128 x 64 read 96 KB.
//  - Issue order.  One wavefront per SIMD has nobody to fill its gaps, so every instruction is placed by hand: a 16-cycle
//    MFMA leaves room for about two others, and each is followed by at most one fragment read or one DMA request.
//  - No seams between tiles.  The slabs of all tiles of a workgroup form one stream through the ring of stages:
//    the last slabs of a tile already fetch the first ones of the next, which land during the epilogue.  The
//    epilogue stages 16 rows at a time in LDS of its own, so the ring keeps its contents.
//
// Slab g of the stream lives in stage g mod NS.  Its two k-steps (32 deep), with three stages (with four everything is
// requested one slab earlier, and one more may be in flight):
//    k-step 0   MFMAs on fragments in registers; reads the fragments of k-step 1; requests the second half of slab g+2
//    hand-over  every fragment of slab g is in registers, slab g+1 has landed (vmcnt), barrier: its stage is free
//    k-step 1   MFMAs; reads the first fragments of slab g+1; requests the first half of slab g+3 into that stage
// A wait "at most TOT memory instructions in flight" at the hand-over is exact: what may still be in flight
// is slab g+2.  Additional older requests (the bias of a tile) only make it stricter.  Loads return in order
// among themselves, but stores may overtake them, so the epilogue waits for every request in flight before its
// first store; the first hand-over of the next tile then needs no wait, and at the second the stores have drained.

// DMA with the address split into a wave-uniform base and a 32-bit byte offset per lane; the LDS target is lds + OFF.  Two
// parts, so that the hand-scheduled loop can put an MFMA into the wait state that the hardware wants between them.  No operand
// ties the parts together (m0 cannot be one); a test reads off the library's listing that every pair is whole.  As one
// statement with a wait state of its own (dma16_sv) the loop is slower: 9 894 x 768 x 3072 40.5 -> 41.0 us, 9 894 x 2304 x 768
// 38.2 -> 38.9, 4 648 x 4096 x 1024 46.5 -> 46.8.
template <int OFF>
__device__ __forceinline__ void dma_target(uint32_t lds) {
  asm volatile("s_add_u32 m0, %0, %1" ::"s"(lds), "n"(OFF) : "m0", "scc");
}
__device__ __forceinline__ void dma_load(const void* sbase, uint32_t voff) {
  asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase) : "memory");
}
__device__ __forceinline__ void dma4_sv(const void* sbase, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(voff), "s"(sbase) : "memory", "m0");
}

// Stages.  Three hold all that LDS has room for from 192 rows on.  Deep reductions (SHAPE 2) on smaller tiles take four: a
// slab of theirs is multiplied in a third to two thirds of the time its operands travel, and what the fourth stage costs, a
// slab's requests ahead of the first product, they do not notice.  us, three stages / four: 1 400 x 1024 x 4096 with 96 x 128
// tiles 22.8 / 20.7, 128 x 128 24.5 / 23.3; 2 192 x 768 x 3072 18.7 / 18.0, 20.3 / 20.2; with 96 x 96 17.1 / 15.8.  Five and six
// are level with four, 160 rows level (33.8 / 33.8), and K = 768 has nothing of it (1 200 x 2304, 128 x 128: 7.70 / 7.96; 160 x 128
// 8.73 / 8.93).
constexpr int wide_stages(int bm, int epi, int shape) { return shape == 2 && epi == EPI_PLAIN && bm <= 128 ? 4 : 3; }

template <int BM, int BN, int STAGES>
struct WideTile {
  static constexpr int WM = BM / 2, WN = BN / 2, MI = WM / 16, NI = WN / 16;
  static constexpr int LA = BM / 32, LB = BN / 32, TOT = LA + LB;  // DMA instructions (8 rows each) per wave and slab
  static constexpr int NS = STAGES, STAGE = (BM + BN) * 128;  // operand stages, bytes per stage
  static constexpr int EPI_LD = WN + 8;                           // row pitch of the epilogue's staging rows, halves
  static constexpr int EPI_BYTES = 16 * EPI_LD * 2, BIAS_BYTES = 1024;
  static constexpr int LDS = NS * STAGE + 4 * EPI_BYTES + 2 * BIAS_BYTES;
  static_assert(LDS <= 160 * 1024, "LDS");
  static_assert((NS - 2) * TOT + TOT / 2 < 64, "vmcnt range");
};

// smem: WideTile<BM, BN, NS>::LDS bytes, 1024-byte aligned.
template <int BM, int BN, int ACT, int EPI, int NS>
__device__ __forceinline__ void gemm_wide_tiles(char* smem, const half_t* __restrict__ A, const half_t* __restrict__ W,
                                                const int32_t* __restrict__ a_rows, const half_t* __restrict__ bias, int M, int N,
                                                int K, int tiles_n, int tiles_m, int group_m, half_t* __restrict__ C,
                                                const GemmEpi& ep) {
  using T = WideTile<BM, BN, NS>;
  constexpr int MI = T::MI, NI = T::NI, LA = T::LA, LB = T::LB, TOT = T::TOT, STAGE = T::STAGE;
  static_assert(EPI == EPI_PLAIN || EPI == EPI_FOLD, "epilogue form");
  // Several tiles per workgroup; FOLD: one.  It runs in one round of tiles nearly everywhere; where it does not (192- and
  // 128-row tiles at 2 561 to 2 688 tokens of width 768) the second round starts anew.
  constexpr bool STREAM = EPI == EPI_PLAIN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, quad = lane >> 4;
  const int n_tiles = tiles_m * tiles_n, per_group = group_m * tiles_n;

  // Tile order as in gemm_pipe_kernel: a contiguous run per XCD, strips of group_m tile rows column by column.
  auto tile_at = [&](int id, int& m0, int& n0) {
    const int lin = xcd_remap(id, n_tiles);
    const int g = lin / per_group, first_m = g * group_m, in_group = lin - g * per_group;
    const int rows_here = min(tiles_m - first_m, group_m);
    const int tn = in_group / rows_here;
    m0 = (first_m + in_group - tn * rows_here) * BM;
    n0 = tn * BN;
  };
  // DMA source offsets of this lane (bytes).  Instruction q of this wave fills rows [8 (wave*L + q), +8) of the operand;
  // lane i lands in row i/8, physical 16-byte chunk i%8, and fetches the logical chunk (i%8) ^ ((row>>1)&7).
  const int r8 = lane >> 3;
  const uint32_t c_even = ((lane & 7) ^ (r8 >> 1)) * 16;  // row>>1 & 7 = (r8 >> 1) + 4 (q odd)
  auto offsets_of = [&](int m0, int n0, uint32_t (&va)[LA], uint32_t (&vb)[LB]) {
#pragma unroll
    for (int q = 0; q < LA; ++q) {
      const int blk = wave * LA + q, r = min(m0 + blk * 8 + r8, M - 1);  // rows past M: clamped reads, never stored
      va[q] = (uint32_t)(a_rows ? a_rows[r] : r) * (uint32_t)(K * 2) + (c_even ^ ((blk & 1) * 64));
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) {
      const int blk = wave * LB + q, r = min(n0 + blk * 8 + r8, N - 1);
      vb[q] = (uint32_t)r * (uint32_t)(K * 2) + (c_even ^ ((blk & 1) * 64));
    }
  };
  const uint32_t lds0 = lds_addr(smem);
  const uint32_t dma_a = lds0 + wave * LA * 1024, dma_b = lds0 + BM * 128 + wave * LB * 1024;
  const int nk = K / 64;  // > NS (checked by the launcher)

  // ---- fetch cursor: the slab whose requests are being issued
  uint32_t va[LA], vb[LB], nva[LA], nvb[LB];
  int id = blockIdx.x, m0, n0;  // tile being computed
  tile_at(id, m0, n0);
  offsets_of(m0, n0, va, vb);
  const half_t *fa_base = A, *fb_base = W;
  uint32_t fstage = 0;  // byte offset of the stage the cursor writes to
  auto request = [&](auto q_c) {
    constexpr int Q = decltype(q_c)::value;
    if constexpr (Q < LA) dma16_sv<Q * 1024>(fa_base, va[Q], dma_a + fstage);
    else dma16_sv<(Q - LA) * 1024>(fb_base, vb[Q - LA], dma_b + fstage);
  };
  // The tile's per-column operands for the epilogue (columns past N: clamped, never stored), one DMA instruction.
  // PLAIN: BN bias values, a pair per lane (a bias is 8-byte aligned, not 16).  FOLD: BN values of fold_c, then BN of
  // fold_d = fold_c + N.
  auto request_bias = [&](int n_first, int parity) {
    const uint32_t to = lds0 + NS * STAGE + 4 * T::EPI_BYTES + parity * T::BIAS_BYTES;
    if constexpr (EPI == EPI_PLAIN) {
      static_assert(BN <= 128, "one DMA instruction: 64 pairs");
      if (bias && wave == 0) dma4_sv(bias, (uint32_t)min(n_first + lane * 2, N - 2) * 2u, to);
    } else {
      static_assert(BN == 128, "one DMA instruction: 32 lanes for each vector");
      if (wave == 0) dma16_sv<0>(ep.fold_c, (uint32_t)((lane >> 5) * N + min(n_first + (lane & 31) * 4, N - 4)) * 4u, to);
    }
  };
  auto advance = [&]() {
    fa_base += 64;
    fb_base += 64;
    fstage = fstage == (NS - 1u) * STAGE ? 0u : fstage + STAGE;
  };

  request_bias(n0, 0);
  static_for<TOT>(request);
  advance();
  // the requests of slab 0 of every wavefront go ahead of those of slab 1: the pipeline starts half a slab earlier
  __builtin_amdgcn_s_barrier();
  static_for<NS - 2>([&](auto) {
    static_for<TOT>(request);
    advance();
  });
  constexpr int HALF = TOT / 2;
  static_for<HALF>(request);
  int nm0 = 0, nn0 = 0;  // the tile after this one
  if (STREAM && id + (int)gridDim.x < n_tiles) {
    tile_at(id + gridDim.x, nm0, nn0);
    offsets_of(nm0, nn0, nva, nvb);
  }

  // ---- fragments
  const int swz = (l16 >> 1) & 7;
  const uint32_t row_a = lds0 + (wm * T::WM + l16) * 128, row_b = lds0 + BM * 128 + (wn * T::WN + l16) * 128;
  const uint32_t co0 = (uint32_t)((quad ^ swz) * 16), co1 = co0 ^ 64u;  // chunk 4ks + quad, swizzled
  half8_t fa[2][MI], fb[2][NI];
  float4_t acc[MI][NI];
  uint32_t rstage = 0;  // byte offset of the stage being read
  auto read_one = [&](auto idx_c, auto slot_c, uint32_t a_at, uint32_t b_at) {  // W fragments first: all of a row's MFMAs need them
    constexpr int I = decltype(idx_c)::value, SLOT = decltype(slot_c)::value;
    if constexpr (I < NI) fb[SLOT][I] = *reinterpret_cast<BT_AS3 const half8_t*>(b_at + I * 2048);
    else fa[SLOT][I - NI] = *reinterpret_cast<BT_AS3 const half8_t*>(a_at + (I - NI) * 2048);
  };
  using std::integral_constant;
  // MFMAs of one k-step on fragment slot SLOT; meanwhile the other slot is filled from (a_at, b_at) (READ) and the requests
  // [Q0, Q1) of the cursor's slab are issued.
  auto kstep = [&](auto slot_c, auto zero_c, auto read_c, auto q0_c, auto q1_c, uint32_t a_at, uint32_t b_at) {
    constexpr int SLOT = decltype(slot_c)::value, Q0 = decltype(q0_c)::value, Q1 = decltype(q1_c)::value;
    constexpr bool ZERO = decltype(zero_c)::value, READ = decltype(read_c)::value;
    constexpr int NM = MI * NI, NR = MI + NI;
    constexpr int RSPAN = NM * 3 / 4;  // the reads go into the first three quarters: they are back when the step ends
    static_for<NM>([&](auto m_c) {
      // Back and forth over the columns: at a turn the column fragment stays and the row changes, elsewhere the row stays, and
      // operands that do not change cost no switching.  On ordinary data the chip runs at its power limit, so that is time, if
      // little: 8 232 x 3072 x 768 42.9 -> 42.2 us on one card, level on zeros; whole stacks 0 to 1 % by card and run.
      constexpr int m = decltype(m_c)::value, i = m / NI, j = (i & 1) ? NI - 1 - m % NI : m % NI;
      constexpr int dlo = Q0 + m * (Q1 - Q0) / NM, dhi = Q0 + (m + 1) * (Q1 - Q0) / NM;
      static_assert(dhi - dlo <= 1, "at most one request per MFMA");
      if constexpr (dhi > dlo) {
        if constexpr (dlo < LA) dma_target<dlo * 1024>(dma_a + fstage);
        else dma_target<(dlo - LA) * 1024>(dma_b + fstage);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (ZERO)  // transposed product: D[n][m] += W[n][k] * A[m][k]
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[SLOT][j], fa[SLOT][i], float4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      else
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[SLOT][j], fa[SLOT][i], acc[i][j], 0, 0, 0);
      if constexpr (READ) {
        constexpr int lo = m < RSPAN ? m * NR / RSPAN : NR, hi = m + 1 < RSPAN ? (m + 1) * NR / RSPAN : NR;
        static_for<hi - lo>([&](auto k_c) {
          read_one(integral_constant<int, lo + decltype(k_c)::value>{}, integral_constant<int, 1 - SLOT>{}, a_at, b_at);
        });
      }
      if constexpr (dhi > dlo) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (dlo < LA) dma_load(fa_base, va[dlo < LA ? dlo : 0]);
        else dma_load(fb_base, vb[dlo < LA ? 0 : dlo - LA]);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using yes = std::true_type;
  using no = std::false_type;
  // fetch1_c: 0 = nothing more to request, 1 = the next slab of the cursor's tile, 2 = the first slab of the next tile
  auto slab = [&](auto zero_c, auto fetch0_c, auto fetch1_c, auto last_c, auto younger_c, bool wait, int next_parity) {
    constexpr int F1 = decltype(fetch1_c)::value;
    constexpr bool F0 = decltype(fetch0_c)::value, LAST = decltype(last_c)::value;
    kstep(integral_constant<int, 0>{}, zero_c, yes{}, integral_constant<int, HALF>{},
          integral_constant<int, F0 ? TOT : HALF>{}, row_a + rstage + co1, row_b + rstage + co1);
    rstage = rstage == (NS - 1u) * STAGE ? 0u : rstage + STAGE;
    if constexpr (!LAST) {
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      if (wait) wait_vmcnt<(F0 ? (NS - 2) * TOT : 0) + decltype(younger_c)::value>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (F1 == 1) {
      fa_base += 64;
      fb_base += 64;
    } else if constexpr (F1 == 2) {
      fa_base = A;
      fb_base = W;
#pragma unroll
      for (int q = 0; q < LA; ++q) va[q] = nva[q];
#pragma unroll
      for (int q = 0; q < LB; ++q) vb[q] = nvb[q];
      request_bias(nn0, next_parity);
    }
    if constexpr (F1 > 0) fstage = fstage == (NS - 1u) * STAGE ? 0u : fstage + STAGE;
    __builtin_amdgcn_sched_barrier(0);
    kstep(integral_constant<int, 1>{}, no{}, integral_constant<bool, !LAST>{}, integral_constant<int, 0>{},
          integral_constant<int, (F1 > 0 ? HALF : 0)>{}, row_a + rstage + co0, row_b + rstage + co0);
    if constexpr (!LAST) __builtin_amdgcn_s_waitcnt(0xc07f);  // one wait instead of one per use: the reads are long back
  };

  // first fragments of slab 0 (slab 1 and half of slab 2 may be in flight)
  wait_vmcnt<(NS - 2) * TOT + HALF>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  static_for<MI + NI>([&](auto i_c) { read_one(i_c, integral_constant<int, 0>{}, row_a + co0, row_b + co0); });

  half_t* const stage = reinterpret_cast<half_t*>(smem + NS * STAGE + wave * T::EPI_BYTES);
  bool first = true;
  for (int parity = 0;; parity ^= 1) {
    const bool last = !STREAM || id + (int)gridDim.x >= n_tiles;
    using next = integral_constant<int, 1>;
    using switch_tile = integral_constant<int, 2>;
    using none = integral_constant<int, 0>;
    float2 psum[EPI == EPI_FOLD ? MI : 1][row_sum_requests(BM, BN)];
    slab(yes{}, yes{}, next{}, no{}, none{}, first, 0);
    for (int k = nk - NS - 1; k > 0; --k) slab(no{}, yes{}, next{}, no{}, none{}, true, 0);
    if (last) {
      slab(no{}, yes{}, none{}, no{}, none{}, true, 0);
      // FOLD: the row sums arrive under the last two slabs.  They are younger than the last operand requests, and the only
      // wait left before the epilogue's own lets them stay in flight.  Straight-line code from here to that wait, with the
      // destinations live all the way, so that nothing touches them before the data is there (tests read it off the listing).
      // Requested behind the last slab, their round trip stood alone in every tile: six folded layers of width 768 at 2 308
      // tokens 408.3 -> 405.4 us, at 1 500 tokens 340.2 -> 335.0 us; width 1024 at 1 600 tokens 452.6 -> 443.7 us.
      if constexpr (EPI == EPI_FOLD) request_row_sums(ep.ln_part, ep.ln_np, M, m0 + wm * T::WM, l16, quad, psum);
      static_for<NS - 2>([&](auto t_c) {  // the slabs behind the next one may be in flight
        slab(no{}, no{}, none{}, no{},
             integral_constant<int, (EPI == EPI_FOLD ? MI * row_sum_requests(BM, BN) : 0) + (NS - 3 - decltype(t_c)::value) * TOT>{},
             true, 0);
      });
      slab(no{}, no{}, none{}, yes{}, none{}, true, 0);
    } else {
      slab(no{}, yes{}, switch_tile{}, no{}, none{}, true, parity ^ 1);
      for (int k = NS - 1; k > 0; --k) slab(no{}, yes{}, next{}, no{}, none{}, true, 0);
    }
    first = false;

    // ---- epilogue: acc[i][j][t] = C[m][n], m = m_base + i*16 + l16, n = n_base + j*16 + 4 quad + t
    const int m_base = m0 + wm * T::WM, n_base = n0 + wn * T::WN;
    float mu[MI], rstd[MI];
    const char* const col_lds = smem + NS * STAGE + 4 * T::EPI_BYTES + parity * T::BIAS_BYTES;
    float4_t c4[NI], d4[NI];  // PLAIN: d4 = bias;  FOLD: c4, d4
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int nl = wn * T::WN + j * 16 + 4 * quad;
      if constexpr (EPI == EPI_FOLD) {
        c4[j] = *reinterpret_cast<const float4_t*>(col_lds + nl * 4);
        d4[j] = *reinterpret_cast<const float4_t*>(col_lds + (BN + nl) * 4);
      } else {
        d4[j] = float4_t{0.f, 0.f, 0.f, 0.f};
        if (bias) d4[j] = __builtin_convertvector(*reinterpret_cast<const half4_t*>(col_lds + nl * 2), float4_t);
      }
    }
    if constexpr (EPI == EPI_FOLD) {
      wait_vmcnt<0>();
      finish_row_sums(ep.ln_part, ep.ln_np, M, m_base, l16, quad, ep.inv_h, ep.eps, psum, mu, rstd);
    }
    half4_t out[MI][NI];
    auto arithmetic = [&](int i) {
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          v[t] = acc[i][j][t];
          if constexpr (EPI == EPI_FOLD) v[t] = __builtin_fmaf(rstd[i], v[t] - mu[i] * c4[j][t], d4[j][t]);
          else v[t] += d4[j][t];
          if (ACT == BT_ACT_GELU_ERF) v[t] = gelu_erf(v[t]);
          else if (ACT == BT_ACT_GELU_TANH) v[t] = gelu_tanh(v[t]);
          out[i][j][t] = (half_t)v[t];
        }
      }
    };
    constexpr int LPR = T::WN / 8, RPP = 64 / LPR;  // lanes per row of the row-contiguous pass, rows per pass
    const int rr = lane / LPR, cc = (lane % LPR) * 8;
    // The arithmetic runs MI/2 blocks ahead of the stores: the requests in flight for the next tile land under it.
    // (FOLD has waited for them already, with its row sums.)
    constexpr int AHEAD = EPI == EPI_FOLD ? 0 : MI / 2;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) arithmetic(i);
    wait_vmcnt<0>();
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if (i + AHEAD < MI) arithmetic(i + AHEAD);
      if constexpr (EPI == EPI_FOLD) __builtin_amdgcn_sched_barrier(0);  // one block's registers at a time
#pragma unroll
      for (int j = 0; j < NI; ++j) *reinterpret_cast<half4_t*>(stage + l16 * T::EPI_LD + j * 16 + 4 * quad) = out[i][j];
      // same wavefront reads what it wrote: LDS operations of a wave complete in order
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += RPP) {  // 96 columns: six lanes a row, ten rows a pass, the last four lanes idle
        if (RPP * LPR != 64 && (rr >= RPP || r0 + rr >= 16)) continue;
        const int mr = m_base + i * 16 + r0 + rr, n = n_base + cc;
        const uint4_t o4 = *reinterpret_cast<const uint4_t*>(stage + (r0 + rr) * T::EPI_LD + cc);
        if (mr < M && n < N) store_through(C + ((size_t)mr * N + n), o4);  // written through: see store_tile
      }
    }
    if (last) break;
    id += gridDim.x;
    m0 = nm0;
    n0 = nn0;
    if (id + (int)gridDim.x < n_tiles) {
      tile_at(id + gridDim.x, nm0, nn0);
      offsets_of(nm0, nn0, nva, nvb);
    }
  }
}

template <int BM, int BN, int ACT, int EPI, int SHAPE>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(
    // in the order of first use: the first 14 dwords are preloaded into SGPRs at wave launch
    const half_t* __restrict__ A, const half_t* __restrict__ W, const int32_t* __restrict__ a_rows /* = ep.a_rows */,
    const half_t* __restrict__ bias /* = ep.bias */, int M, int N, int K, int tiles_n, int tiles_m, int group_m,
    half_t* __restrict__ C, const GemmEpi ep) {
  constexpr int NS = wide_stages(BM, EPI, SHAPE);
  __shared__ __attribute__((aligned(1024))) char smem[WideTile<BM, BN, NS>::LDS];
  gemm_wide_tiles<BM, BN, ACT, EPI, NS>(smem, A, W, a_rows, bias, M, N, K, tiles_n, tiles_m, group_m, C, ep);
}
