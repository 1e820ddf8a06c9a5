// The layer's products for few tokens, with the LayerNorm between two of them inside the second one.
//
// With a hundred tokens a layer is seven dependent launches of 3 to 5 us, of which the launch itself and one round trip to
// data that another XCD has written (0.7 us) are the larger part, and the host needs nearly as long to enqueue them.  Here
// add-bias + residual + LayerNorm (Sec. III-C1) is no launch of its own:
//   few_resid_gemm_kernel   z = A W^T + residual + bias, fp32, the whole reduction in one workgroup (its wavefronts share it
//                           out and add their parts through LDS in wavefront order)
//   few_ln_gemm_kernel      C = act(LN(z) W^T + bias): every workgroup normalises the rows it multiplies, 16 or 32 of them,
//                           while the first slabs of its weights are on their way
// Included at the end of gemm.hip.
// z stays fp32 between the two and is summed in the order of the product over K slices and the LayerNorm kernel behind it, the
// statistics in the order of that kernel: a layer's output is the same bits in 5, 6 and 7 launches.

namespace bt {

// At most `younger` (wave-uniform, taken as MAX where larger) slabs of TOT requests each stay in flight.
template <int MAX, int TOT>
__device__ __forceinline__ void wait_younger(int younger) {
  if constexpr (MAX == 0) wait_vmcnt<0>();
  else if (younger >= MAX) wait_vmcnt<MAX * TOT>();
  else wait_younger<MAX - 1, TOT>(younger);
}
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xc07f); }  // lgkmcnt(0), other counters untouched

// The LayerNorm kernel's arithmetic (layernorm.hip) with the roundings the compiler gives it there written out: a row normalised
// here and one normalised by that kernel are the same bits.  Deviations are fused from the row sum; the output of rows of more
// than one piece a lane starts from the rounded mean instead; the output's last multiply-add and its conversion to fp16 round
// once, but twice from the third element on where a lane has one piece.
__device__ __forceinline__ float ln_square(float v, float sum, float inv_h, float sq) {
  const float d = __builtin_fmaf(-inv_h, sum, v);
  return __builtin_fmaf(d, d, sq);
}
template <bool ONE_PIECE>
__device__ __forceinline__ half8_t ln_out(const float4_t (&v)[2], float sum, float inv_h, float rstd, uint4_t gamma, uint4_t beta) {
#pragma clang fp contract(off)
  const half8_t g8 = __builtin_bit_cast(half8_t, gamma), b8 = __builtin_bit_cast(half8_t, beta);
  const float mean = sum * inv_h;
  half8_t o;
  static_for<8>([&](auto e_c) {
#pragma clang fp contract(off)
    constexpr int e = decltype(e_c)::value;
    const float x = v[e / 4][e % 4], d = ONE_PIECE ? __builtin_fmaf(-inv_h, sum, x) : x - mean;
    float y = __builtin_fmaf(d * rstd, (float)g8[e], (float)b8[e]);
    if constexpr (ONE_PIECE && e >= 2) asm volatile("" : "+v"(y));
    o[e] = (half_t)y;
  });
  return o;
}
// Lower halves of two registers side by side, and the upper ones; a second swap puts them back.
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  const auto t = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  a = __builtin_bit_cast(float, (unsigned)t[0]);
  b = __builtin_bit_cast(float, (unsigned)t[1]);
}

// C [T,N] = act(LN(z) W^T + bias), y [T,K] = LN(z); z fp32 [T,K], K = 256 NL, N % 16 == 0.
// NW wavefronts, block tile 16 MI x 16 NW; a wavefront owns 16 columns: its slabs of W (16 rows, 64 deep) go through a ring of
// its own, NC chunks of two slabs, so that nothing but the normalised rows is shared and one barrier is all there is.
// Bound: a chain of launch, round trip to z, row statistics and a K loop of its own per wavefront; no single unit is full.  186 tokens,
// FFN-up of width 768: 7.4 us, in which LDS is active for 1.8 us of a compute unit's time, 0.6 of them bank conflicts of the reads of
// the normalised rows (4 cycles a read, and all NW wavefronts read every row).
// Per launch, weights of twelve layers in turn, graph replays, width 768, z to 2304 / 3072 + GELU columns: 48 tokens 5.2 / 5.2 us,
// 90 tokens 5.2 / 5.8 us, 256 tokens 7.2 / 7.5 us, where the LayerNorm kernel over K slices (3.2 to 3.8 us) and the product (5.0 /
// 5.4 us) take 8 to 9 us together.  One slab per hand-over without fragments read ahead took 6.3 us, a ring of 64-deep slabs
// twice as long 5.4 us.
template <int MI, int NW, int NC, int NL, int ACT>
__global__ __launch_bounds__(NW * 64) void few_ln_gemm_kernel(
    // in the order of first use: the first 14 dwords are preloaded into SGPRs at wave launch
    const float* __restrict__ z, const half_t* __restrict__ W, int T, int N, int tiles_m, int tiles_n,
    const half_t* __restrict__ gamma, const half_t* __restrict__ beta, const half_t* __restrict__ bias, float eps,
    half_t* __restrict__ C, half_t* __restrict__ y) {
  constexpr int K = 256 * NL, BM = MI * 16, RW = BM / NW;  // rows a wavefront normalises
  constexpr int SLAB = 2048, NCH = NL * 2;                 // bytes of a slab, chunks of a reduction
  constexpr int PITCH = K * 2 + 16;                        // of a normalised row in LDS
  // A lane holds pieces of eight columns, piece lane + 64 i of a row, as in the LayerNorm kernel: its sums are then the same
  // sums.  The second pieces of 768 columns fill half a wavefront, so two rows share one (one row each: 1 us a layer more).
  constexpr int SHARE = NL == 3 ? 2 : 1, TAILS = NL == 2 ? 0 : RW / SHARE;  // rows to a second piece, second pieces
  static_assert(RW == 2 || RW == 4, "rows per wavefront");
  static_assert(NC <= NCH, "ring");
  __shared__ __attribute__((aligned(1024))) char s_ring[NW * NC * 2 * SLAB];
  __shared__ __attribute__((aligned(16))) char s_a[BM * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, quad = lane >> 4;
  // all row tiles of a column tile stand together, so that an XCD reads its share of W once
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int tn = id / tiles_m, m0 = (id - tn * tiles_m) * BM, n0 = (tn * NW + wave) * 16;

  // DMA source of this lane: row i/8 of 8, the logical chunk (i%8) ^ ((row>>1)&7) lands in physical chunk i%8
  const int r8 = lane >> 3;
  const uint32_t chunk = (uint32_t)((lane & 7) ^ (r8 >> 1)) * 16;
  uint32_t w0 = (uint32_t)min(n0 + r8, N - 1) * (uint32_t)(K * 2) + chunk;  // columns past N: clamped, never stored
  uint32_t w1 = (uint32_t)min(n0 + 8 + r8, N - 1) * (uint32_t)(K * 2) + (chunk ^ 64u);
  const uint32_t ring = lds_addr(s_ring) + wave * (NC * 2 * SLAB);

  // Rows, gamma, beta and bias, behind them the whole ring, and the wait for all but the ring, as ONE statement: the compiler does
  // not count the DMA requests and would wait for them too before it touches a row.
  const int tail_lane = lane & (kWave / SHARE - 1), tail_row = lane / (kWave / SHARE);
  const uint32_t vh = lane * 16, vz = vh * 2, th = (kWave + tail_lane) * 16;
  const uint32_t vb = (uint32_t)min(n0 + 4 * quad, N - 4) * 2;
  const int row0 = m0 + wave * RW;
  auto clamped = [&](int r) { return min(row0 + r, T - 1); };  // rows past T: never stored
  const float *zr[RW], *zt[4];
  uint32_t tz[4];
#pragma unroll
  for (int r = 0; r < RW; ++r) zr[r] = z + (size_t)clamped(r) * K;
#pragma unroll
  for (int p = 0; p < TAILS; ++p) {
    zt[p] = zr[p * SHARE];
    tz[p] = th * 2 + (tail_row ? (uint32_t)(clamped(p * SHARE + 1) - clamped(p * SHARE)) * (K * 4) : 0u);
  }
  float4_t v[RW][2], t[4][2];
  uint4_t gm[2], be[2];
  uint2_t bs;
#define BT_ROW(r) "global_load_dwordx4 %[z" #r "0], %[vz], %[b" #r "]\n\tglobal_load_dwordx4 %[z" #r "1], %[vz], %[b" #r "] offset:16\n\t"
#define BT_TAIL(p) "global_load_dwordx4 %[t" #p "0], %[u" #p "], %[c" #p "]\n\tglobal_load_dwordx4 %[t" #p "1], %[u" #p "], %[c" #p "] offset:16\n\t"
#define BT_VEC "global_load_dwordx4 %[g0], %[vh], %[g]\n\tglobal_load_dwordx4 %[e0], %[vh], %[e]\n\t"
#define BT_TAIL_VEC "global_load_dwordx4 %[g1], %[th], %[g]\n\tglobal_load_dwordx4 %[e1], %[th], %[e]\n\t"
#define BT_ROWS_2 BT_ROW(0) BT_ROW(1) BT_VEC
#define BT_ROWS_4 BT_ROW(0) BT_ROW(1) BT_ROW(2) BT_ROW(3) BT_VEC
#define BT_TAILS_0
#define BT_TAILS_1 BT_TAIL(0) BT_TAIL_VEC
#define BT_TAILS_2 BT_TAIL(0) BT_TAIL(1) BT_TAIL_VEC
#define BT_TAILS_4 BT_TAIL(0) BT_TAIL(1) BT_TAIL(2) BT_TAIL(3) BT_TAIL_VEC
#define BT_RING                                    \
  "global_load_dwordx2 %[bs], %[vb], %[bias]\n\t"  \
  ".set bt_ring_at, 0\n\t"                         \
  ".rept %c[slabs]\n\t"                            \
  "s_add_u32 m0, %[lds], bt_ring_at\n\t"           \
  "s_nop 0\n\t"                                    \
  "global_load_lds_dwordx4 %[w0], %[w]\n\t"        \
  "s_add_u32 m0, %[lds], bt_ring_at + 0x400\n\t"   \
  "v_add_u32 %[w0], 0x80, %[w0]\n\t"               \
  "global_load_lds_dwordx4 %[w1], %[w]\n\t"        \
  "v_add_u32 %[w1], 0x80, %[w1]\n\t"               \
  ".set bt_ring_at, bt_ring_at + 0x800\n\t"        \
  ".endr\n\t"                                      \
  "s_waitcnt vmcnt(%c[dma])"
#define BT_ROW_OUT(r) [z##r##0] "=&v"(v[r][0]), [z##r##1] "=&v"(v[r][1])
#define BT_TAIL_OUT(p) , [t##p##0] "=&v"(t[p][0]), [t##p##1] "=&v"(t[p][1])
#define BT_TAIL_VEC_OUT , [g1] "=&v"(gm[1]), [e1] "=&v"(be[1])
#define BT_ROWS_OUT_2 BT_ROW_OUT(0), BT_ROW_OUT(1)
#define BT_ROWS_OUT_4 BT_ROW_OUT(0), BT_ROW_OUT(1), BT_ROW_OUT(2), BT_ROW_OUT(3)
#define BT_TAILS_OUT_0
#define BT_TAILS_OUT_1 BT_TAIL_OUT(0) BT_TAIL_VEC_OUT
#define BT_TAILS_OUT_2 BT_TAIL_OUT(0) BT_TAIL_OUT(1) BT_TAIL_VEC_OUT
#define BT_TAILS_OUT_4 BT_TAIL_OUT(0) BT_TAIL_OUT(1) BT_TAIL_OUT(2) BT_TAIL_OUT(3) BT_TAIL_VEC_OUT
#define BT_ROWS_IN_2 [b0] "s"(zr[0]), [b1] "s"(zr[1])
#define BT_ROWS_IN_4 BT_ROWS_IN_2, [b2] "s"(zr[2]), [b3] "s"(zr[3])
#define BT_TAIL_IN(p) , [u##p] "v"(tz[p]), [c##p] "s"(zt[p])
#define BT_TAILS_IN_0
#define BT_TAILS_IN_1 , [th] "v"(th) BT_TAIL_IN(0)
#define BT_TAILS_IN_2 BT_TAILS_IN_1 BT_TAIL_IN(1)
#define BT_TAILS_IN_4 BT_TAILS_IN_2 BT_TAIL_IN(2) BT_TAIL_IN(3)
#define BT_LOAD(R, P)                                                                                                          \
  asm volatile(BT_ROWS_##R BT_TAILS_##P BT_RING                                                                                \
               : BT_ROWS_OUT_##R BT_TAILS_OUT_##P, [g0] "=&v"(gm[0]), [e0] "=&v"(be[0]), [bs] "=&v"(bs), [w0] "+&v"(w0), [w1] "+&v"(w1) \
               : BT_ROWS_IN_##R BT_TAILS_IN_##P, [vz] "v"(vz), [vh] "v"(vh), [vb] "v"(vb), [g] "s"(gamma), [e] "s"(beta),      \
                 [bias] "s"(bias), [w] "s"(W), [lds] "s"(ring), [slabs] "n"(2 * NC), [dma] "n"(4 * NC)                         \
               : "memory", "m0", "scc")
  if constexpr (RW == 2 && TAILS == 0) BT_LOAD(2, 0);
  if constexpr (RW == 2 && TAILS == 1) BT_LOAD(2, 1);
  if constexpr (RW == 2 && TAILS == 2) BT_LOAD(2, 2);
  if constexpr (RW == 4 && TAILS == 0) BT_LOAD(4, 0);
  if constexpr (RW == 4 && TAILS == 2) BT_LOAD(4, 2);
  if constexpr (RW == 4 && TAILS == 4) BT_LOAD(4, 4);
#undef BT_LOAD

  // Two-pass statistics in fp32, normalised rows to LDS in fp16.  tails(s, add): add(p, s) goes on with the sums s of the rows of
  // second piece p, in the lanes that hold them.
  constexpr float inv_k = 1.0f / (float)K;
  auto tails = [&](float (&s)[RW], auto&& add) {
    static_for<TAILS>([&](auto p_c) {
      constexpr int a = decltype(p_c)::value * SHARE, b = a + SHARE - 1;
      if constexpr (SHARE == 2) swap_halves(s[a], s[b]);  // the lanes 0 to 31 of both rows
      add(p_c, s[a]);
      if constexpr (SHARE == 2) swap_halves(s[a], s[b]);
    });
  };
  auto of_tail = [&](const float (&s)[RW], auto p_c) {
    constexpr int a = decltype(p_c)::value * SHARE, b = a + SHARE - 1;
    return tail_row ? s[b] : s[a];
  };
  float sum[RW], sq[RW], rstd[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    sum[r] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[r] += v[r][e / 4][e % 4];
  }
  tails(sum, [&](auto p_c, float& s) {
    constexpr int p = decltype(p_c)::value;
#pragma unroll
    for (int e = 0; e < 8; ++e) s += t[p][e / 4][e % 4];
  });
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    sum[r] = wave_sum(sum[r]);
    sq[r] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = k < 2 ? 1 - k : k;  // the first two the other way round, as there
      sq[r] = ln_square(v[r][e / 4][e % 4], sum[r], inv_k, sq[r]);
    }
  }
  tails(sq, [&](auto p_c, float& q) {
    constexpr int p = decltype(p_c)::value;
    const float s = of_tail(sum, p_c);
#pragma unroll
    for (int e = 0; e < 8; ++e) q = ln_square(t[p][e / 4][e % 4], s, inv_k, q);
  });
#pragma unroll
  for (int r = 0; r < RW; ++r) rstd[r] = rsqrtf(__builtin_fmaf(inv_k, wave_sum(sq[r]), eps));
  char* const rows_at = s_a + wave * RW * PITCH;
#pragma unroll
  for (int r = 0; r < RW; ++r)
    *reinterpret_cast<half8_t*>(rows_at + r * PITCH + vh) = ln_out<TAILS == 0>(v[r], sum[r], inv_k, rstd[r], gm[0], be[0]);
  static_for<TAILS>([&](auto p_c) {
    constexpr int p = decltype(p_c)::value;
    *reinterpret_cast<half8_t*>(rows_at + (p * SHARE + tail_row) * PITCH + th) =
        ln_out<false>(t[p], of_tail(sum, p_c), inv_k, of_tail(rstd, p_c), gm[1], be[1]);
  });
  wait_lds();
  __builtin_amdgcn_s_barrier();

  // Chunk c (128 deep) lives in ring slot c % NC.  Its fragments are read while the MFMAs of chunk c-1 run, and its slot is
  // refilled as soon as they are in registers.  Every offset and wait is a constant.
  float4_t acc[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
  const uint32_t wf0 = ring + l16 * 128 + (quad ^ ((l16 >> 1) & 7)) * 16, wf1 = wf0 ^ 64u;
  const uint32_t a_at = lds_addr(s_a) + l16 * PITCH + quad * 16;
  half8_t fa[2][4][MI], fb[2][4];
  auto read = [&](auto c_c) {
    constexpr int c = decltype(c_c)::value, SLOT = c & 1, ST = (c % NC) * 2 * SLAB;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      fb[SLOT][k] = *reinterpret_cast<BT_AS3 const half8_t*>(((k & 1) ? wf1 : wf0) + ST + (k >> 1) * SLAB);
#pragma unroll
      for (int i = 0; i < MI; ++i)
        fa[SLOT][k][i] = *reinterpret_cast<BT_AS3 const half8_t*>(a_at + i * 16 * PITCH + c * 256 + k * 64);
    }
  };
  wait_vmcnt<(NC - 1) * 4>();
  read(std::integral_constant<int, 0>{});
  static_for<NCH>([&](auto c_c) {
    constexpr int c = decltype(c_c)::value, SLOT = c & 1;
    wait_lds();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (c + NC < NCH) {
      static_for<2>([&](auto k_c) {
        constexpr int at = ((c % NC) * 2 + decltype(k_c)::value) * SLAB;
        dma16_sv<at>(W, w0, ring);
        dma16_sv<at + 1024>(W, w1, ring);
        w0 += 128;
        w1 += 128;
      });
    }
    if constexpr (c + 1 < NCH) {
      wait_vmcnt<((c + NC < NCH ? c + NC : NCH - 1) - (c + 1)) * 4>();
      read(std::integral_constant<int, c + 1>{});
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < MI; ++i)  // transposed product: D[n][m] += W[n][k] * A[m][k]
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[SLOT][k], fa[SLOT][k][i], acc[i], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  });

  // The normalised rows are the residual of the product after next; the column tiles take one row of the tile each.
  for (int r = tn; r < BM; r += tiles_n)
    if (m0 + r < T)
      for (int c = tid; c < K / 8; c += NW * 64)
        store_through(y + (size_t)(m0 + r) * K + c * 8, *reinterpret_cast<const uint4_t*>(s_a + r * PITCH + c * 16));

  // acc[i][t] = C[m0 + i*16 + l16][n0 + 4 quad + t]
  const half4_t b4 = __builtin_bit_cast(half4_t, bs);
  const int n = n0 + 4 * quad;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int m = m0 + i * 16 + l16;
    half4_t o;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float x = acc[i][t] + (float)b4[t];
      if (ACT == BT_ACT_GELU_ERF) x = gelu_erf(x);
      else if (ACT == BT_ACT_GELU_TANH) x = gelu_tanh(x);
      o[t] = (half_t)x;
    }
    if (m < T && n < N) store_through(C + (size_t)m * N + n, __builtin_bit_cast(uint2_t, o));
  }
}

// z [T,N] = A W^T + residual + bias, fp32; A fp16 [T,K], K % 64 == 0, N % 8 == 0; row m of the residual is row
// resid_rows[m] of `resid` where given (pack fused into the read).
// WK wavefronts, block tile 16 MI x 16 NI: a wavefront multiplies the whole tile over one slice of the reduction, `per` of the K/64
// slabs, from a ring of NS slabs of its own (no barrier until the parts are added).  The slices are those of the product over K
// slices and are added in their order, then residual, then bias: z is what the LayerNorm kernel over K slices normalises, bit for
// bit, and a layer's output does not depend on which form made it.  Wavefronts past the last slice add zeros.
// Bound: operand bytes per compute unit.  768 columns, K = 768 / 3072, graph replays: 30 tokens 2.9 / 4.8 us, 90 tokens 3.3 / 5.7 us,
// 256 tokens 3.4 / 6.6 us; the products over K slices 3.3 / 4.4, 3.4 / 4.4 and 3.6 / 5.3 us, but they leave 4 to 8 slices to be added.
template <int MI, int NI, int WK, int NS>
__global__ __launch_bounds__(WK * 64) void few_resid_gemm_kernel(
    const half_t* __restrict__ A, const half_t* __restrict__ W, int T, int N, int K, int per,
    const half_t* __restrict__ resid, const int32_t* __restrict__ resid_rows, const half_t* __restrict__ bias,
    float* __restrict__ z) {
  constexpr int BM = MI * 16, BN = NI * 16, LA = BM / 8, LB = BN / 8, TOT = LA + LB;
  constexpr int SLAB = (BM + BN) * 128, ACC_LD = BN + 4;  // bytes of a slab, pitch of a partial tile (floats)
  constexpr int C4 = BN / 4, Q = BM * C4;                 // 16-byte pieces per row and per tile
  static_assert(NS * TOT < 64, "vmcnt range");
  static_assert(BM * ACC_LD * 4 <= NS * SLAB, "a partial tile fits the ring");
  static_assert(Q <= WK * 64, "at most one piece per thread");
  __shared__ __attribute__((aligned(1024))) char smem[WK * NS * SLAB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, quad = lane >> 4;
  const int id = xcd_remap(blockIdx.x, gridDim.x), tiles_m = (T + BM - 1) / BM;
  const int tn = id / tiles_m, m0 = (id - tn * tiles_m) * BM, n0 = tn * BN;
  const int s0 = wave * per, my = s0 < K / 64 ? per : 0;

  const int r8 = lane >> 3;
  const uint32_t chunk = (uint32_t)((lane & 7) ^ (r8 >> 1)) * 16;
  uint32_t va[LA], vb[LB];
#pragma unroll
  for (int q = 0; q < LA; ++q) va[q] = (uint32_t)min(m0 + q * 8 + r8, T - 1) * (uint32_t)(K * 2) + (chunk ^ ((q & 1) * 64));
#pragma unroll
  for (int q = 0; q < LB; ++q) vb[q] = (uint32_t)min(n0 + q * 8 + r8, N - 1) * (uint32_t)(K * 2) + (chunk ^ ((q & 1) * 64));
  const uint32_t ring = lds_addr(smem) + wave * (NS * SLAB);
  const half_t *fa = A + (size_t)s0 * 64, *fb = W + (size_t)s0 * 64;
  auto fetch = [&](int stage) {
    static_for<LA>([&](auto q) { dma16_sv<decltype(q)::value * 1024>(fa, va[decltype(q)::value], ring + stage * SLAB); });
    static_for<LB>([&](auto q) { dma16_sv<BM * 128 + decltype(q)::value * 1024>(fb, vb[decltype(q)::value], ring + stage * SLAB); });
    fa += 64;
    fb += 64;
  };
  // the residual piece this thread adds at the end, requested ahead of the slabs (clamped where it has none)
  const int r = tid / C4, c = (tid - r * C4) * 4, m = m0 + r, n = n0 + c;
  const bool mine = tid < Q && m < T && n < N;
  const int rm = min(m, T - 1), rn = min(n, N - 4);
  const half4_t r4 = *reinterpret_cast<const half4_t*>(resid + (size_t)(resid_rows ? resid_rows[rm] : rm) * N + rn);
  const half4_t b4 = *reinterpret_cast<const half4_t*>(bias + rn);
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < my) fetch(s);

  float4_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  const uint32_t f0 = ring + l16 * 128 + (quad ^ ((l16 >> 1) & 7)) * 16, f1 = f0 ^ 64u;
  half8_t a[2][2][MI], b[2][2][NI];
  auto read = [&](auto slot_c, int stage) {
    constexpr int S = decltype(slot_c)::value;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const uint32_t at = (ks ? f1 : f0) + stage * SLAB;
#pragma unroll
      for (int j = 0; j < NI; ++j) b[S][ks][j] = *reinterpret_cast<BT_AS3 const half8_t*>(at + BM * 128 + j * 2048);
#pragma unroll
      for (int i = 0; i < MI; ++i) a[S][ks][i] = *reinterpret_cast<BT_AS3 const half8_t*>(at + i * 2048);
    }
  };
  // Slab `it` is in registers; its stage is refilled, and slab it+1 read, under its MFMAs.
  int st = 0;
  auto step = [&](auto slot_c, int it) {
    constexpr int S = decltype(slot_c)::value;
    wait_lds();
    __builtin_amdgcn_sched_barrier(0);
    if (it + NS < my) fetch(st);
    st = st + 1 == NS ? 0 : st + 1;
    if (it + 1 < my) {
      wait_younger<NS - 1, TOT>(my - 2 - it);
      read(std::integral_constant<int, 1 - S>{}, st);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[S][ks][j], a[S][ks][i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  using c0 = std::integral_constant<int, 0>;
  using c1 = std::integral_constant<int, 1>;
  if (my > 0) {
    wait_younger<NS - 1, TOT>(my - 1);
    read(c0{}, 0);
    int it = 0;
    for (; it + 1 < my; it += 2) {
      step(c0{}, it);
      step(c1{}, it + 1);
    }
    if (it < my) step(c0{}, it);
  }

  // the parts of the reduction meet in LDS, each in the ring of the wavefront that has finished with it
  float* const part = reinterpret_cast<float*>(smem + wave * (NS * SLAB));
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) *reinterpret_cast<float4_t*>(part + (i * 16 + l16) * ACC_LD + j * 16 + 4 * quad) = acc[i][j];
  __syncthreads();
  if (mine) {
    float4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WK; ++w) s += *reinterpret_cast<const float4_t*>(smem + w * (NS * SLAB) + (r * ACC_LD + c) * 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) s[t] = (s[t] + (float)r4[t]) + (float)b4[t];
    store_through(z + (size_t)m * N + n, s);
  }
}

// Shapes by the number of tiles: the smallest ones while a round of the compute units holds them, since a compute unit
// then fetches the fewest operand bytes (90 x 2304 x 768: 16 x 64 tiles 5.1 us, 16 x 128 5.5, 32 x 128 7.3; 90 x 3072, where the
// first need 288 of them, 6.5, 5.6, 7.4).
constexpr int kFewRound = 256;

static long long few_tiles(int T, int N, int bm, int bn) { return (long long)((T + bm - 1) / bm) * ((N + bn - 1) / bn); }

bt_status few_ln_gemm_dispatch(const float* z, const bt_half* w, int T, int N, int K, const bt_half* gamma, const bt_half* beta,
                               const bt_half* bias, float eps, bt_act act, bt_half* c, bt_half* y, hipStream_t st) {
  auto h = [](const bt_half* p) { return reinterpret_cast<const half_t*>(p); };
#define BT_LAUNCH(MI, NW, NC, NL, ACT)                                                                              \
  do {                                                                                                              \
    const int tm = (T + MI * 16 - 1) / (MI * 16), tn = (N + NW * 16 - 1) / (NW * 16);                               \
    few_ln_gemm_kernel<MI, NW, NC, NL, ACT><<<tm * tn, NW * 64, 0, st>>>(                                           \
        z, h(w), T, N, tm, tn, h(gamma), h(beta), h(bias), eps, reinterpret_cast<half_t*>(c), reinterpret_cast<half_t*>(y)); \
  } while (0)
#define BT_ACT(MI, NW, NC, NL)                                                          \
  do {                                                                                  \
    if (act == BT_ACT_NONE) BT_LAUNCH(MI, NW, NC, NL, BT_ACT_NONE);                     \
    else if (act == BT_ACT_GELU_ERF) BT_LAUNCH(MI, NW, NC, NL, BT_ACT_GELU_ERF);        \
    else BT_LAUNCH(MI, NW, NC, NL, BT_ACT_GELU_TANH);                                   \
  } while (0)
#define BT_WIDTH(MI, NW, NC)                            \
  do {                                                  \
    if (K == 512) BT_ACT(MI, NW, NC, 2);                \
    else if (K == 768) BT_ACT(MI, NW, NC, 3);           \
    else if (K == 1024) BT_ACT(MI, NW, NC, 4);          \
    else return BT_ERR_UNSUPPORTED;                     \
  } while (0)
  if (few_tiles(T, N, 16, 64) <= kFewRound) BT_WIDTH(1, 4, 3);
  else if (few_tiles(T, N, 16, 128) <= kFewRound) BT_WIDTH(1, 8, 3);
  else BT_WIDTH(2, 8, 2);
#undef BT_WIDTH
#undef BT_ACT
#undef BT_LAUNCH
  return launch_status();
}

// slices: as gemm_splitk_choice gives them, 2 to 8 and a divisor of K/64
bt_status few_resid_gemm_dispatch(const bt_half* a, const bt_half* w, int T, int N, int K, int slices, const bt_half* resid,
                                  const int32_t* resid_rows, const bt_half* bias, float* z, hipStream_t st) {
  auto h = [](const bt_half* p) { return reinterpret_cast<const half_t*>(p); };
  if (slices < 1 || slices > 8 || K % (64 * slices) != 0) return BT_ERR_UNSUPPORTED;
#define BT_LAUNCH(MI, NI, WK, NS)                                                                                   \
  do {                                                                                                              \
    const int tm = (T + MI * 16 - 1) / (MI * 16), tn = (N + NI * 16 - 1) / (NI * 16);                               \
    few_resid_gemm_kernel<MI, NI, WK, NS><<<tm * tn, WK * 64, 0, st>>>(h(a), h(w), T, N, K, K / 64 / slices, h(resid), resid_rows, h(bias), z); \
  } while (0)
#define BT_SLICES(MI, NI, NS)                      \
  do {                                             \
    if (slices <= 4) BT_LAUNCH(MI, NI, 4, NS);     \
    else BT_LAUNCH(MI, NI, 8, NS);                 \
  } while (0)
  if (few_tiles(T, N, 16, 16) <= kFewRound) BT_SLICES(1, 1, 3);
  else if (few_tiles(T, N, 16, 32) <= kFewRound && K >= 2 * N) BT_SLICES(1, 2, 3);
  else BT_SLICES(2, 2, 2);
#undef BT_SLICES
#undef BT_LAUNCH
  return launch_status();
}

}  // namespace bt
