// bf16 GEMM on the gfx950 matrix cores:  C[M][N] = A[M][K] * W[N][K]^T  (+ epilogue).
//
// Used for every dense contraction of the denoising step except attention: QKV, attention
// output projection, both MLP matmuls, the embeddings and the final projection.
//
// Tiling.  A workgroup owns a BM x BN tile of C and walks K in slabs of BK (32 or 64).  Slabs
// of A and W go from global memory straight into LDS (global_load_lds_dwordx4: each lane
// deposits 16 bytes at wave-base + 16*lane, no staging registers) into a ring of NS stages.
// Which 16-byte chunk a lane fetches is XOR-swizzled on the global side, so that the 128-bit
// LDS reads that feed the MFMA operands are bank-conflict free (LDS on gfx950 serves 16 lanes
// x 16 bytes per clock from 64 banks: 16 consecutive slab rows must fall into 16 distinct
// 16-byte slots of a 256-byte window; the key is (row >> 1) & 7 for 128-byte rows and
// (row >> 2) & 3 for 64-byte rows).  A wave owns a (BM/WM) x (BN/WN) sub-tile made of 32x32
// MFMA tiles (v_mfma_f32_32x32x16_bf16: 64 lanes, A operand = 32 rows x 16 k, B operand =
// 16 k x 32 columns, each lane supplies 8 consecutive k), or of 16x16 ones
// (v_mfma_f32_16x16x32_bf16) in the two-group forms.  MFMA rows are rows of A (tokens), MFMA
// columns are rows of W (output features); the two-group forms have it the other way round.
//
// Pipeline.  NS-1 slabs are in flight from global memory while one is computed: measured on
// MI355X a 64 KB slab takes about 1.4 us from issue to landing, as long as its MFMA work, so
// a single slab in flight leaves the matrix cores waiting.  In the 2- and 4-wave tiles operand
// fragments are double buffered in registers: while the MFMAs of k-step kk run, the fragments of
// kk+1 are read from LDS.  The one barrier per slab sits before the slab's last k-step: by then every
// wave holds the slab's last fragments in registers, so the slab's stage is free for the loads of
// slab+NS, and the next slab becomes visible, so the last k-step already prefetches the next
// slab's first fragments.  The 8-wave tiles with a 64-wide slab alternate instead: four waves multiply
// while the other four read and load (gemm8_kernel below).
//
// Several problems (for example the text and the image stream of one joint block, which
// have different weights) are launched as one grid.  Workgroup ids are first de-interleaved
// over the 8 XCDs (ids are dealt round-robin to XCDs by the hardware) so that workgroups
// sharing an L2 work on neighbouring tiles, then mapped to tiles in groups of 8 tile rows.
#include "dit_internal.h"
#include "gemm_rows.h"
#include <type_traits>

namespace dit {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));


__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// two floats -> packed bf16 pair, round-to-nearest-even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2bf(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return *(uint32_t*)&r;
}

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// two floats -> packed fp16 pair, round-to-nearest-even
__device__ __forceinline__ uint32_t pack2h(float a, float b) {
  f32x2 v = {a, b};
  f16x2 r = __builtin_convertvector(v, f16x2);
  return *(uint32_t*)&r;
}

__device__ __forceinline__ float gelu_tanh(float x) {
  // 0.5 x (1 + tanh(u)) == x * sigmoid(2u) == x / (1 + 2^(-2 log2(e) u)),
  // u = sqrt(2/pi) (x + 0.044715 x^3); hardware exp2 and reciprocal (1 ulp each)
  const float t = x * (0.7978845608028654f + 0.035677408136300125f * x * x);
  const float e = __builtin_amdgcn_exp2f(-2.8853900817779268f * t);
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

template <int BKT>
__device__ __forceinline__ int swz_key(int r) { return BKT == 64 ? ((r >> 1) & 7) : ((r >> 2) & 3); }

typedef __attribute__((address_space(3))) void* lptr_t;

#define SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)
// scheduling hint for one k-step: NR LDS reads spread over NM MFMAs
template <int NR, int NM>
__device__ __forceinline__ void interleave_hint() {
  if constexpr (NM >= 16) {
    // one wave per SIMD: nothing else covers LDS latency, so all reads go out in the first half
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      SGB(0x100, 1);
      SGB(0x008, 1);
    }
    SGB(0x008, NM - NR);
    return;
  }
  constexpr int per = NM / NR, extra = NM - per * NR;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    SGB(0x100, 1);      // one DS read
    if constexpr (per > 0) SGB(0x008, per);    // `per` MFMAs
  }
  if (extra > 0) SGB(0x008, extra);
}
// s_waitcnt immediate for "at most N vector-memory loads outstanding" (and LDS reads done if LGKM0)
template <int N, bool LGKM0>
__device__ __forceinline__ void wait_vm() {
  constexpr int imm = (N & 15) | ((N >> 4) << 14) | (7 << 4) | ((LGKM0 ? 0 : 15) << 8);
  __builtin_amdgcn_s_waitcnt(imm);
  asm volatile("" ::: "memory");
}

// Workgroup barrier without the memory fence of __syncthreads(): the callers wait for exactly the
// loads and LDS reads they need (wait_vm) just before it; a fence would make the compiler wait for
// EVERY slab still in flight.
__device__ __forceinline__ void wg_barrier() {
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// 16 bytes per lane from global memory straight into LDS through a buffer descriptor: address =
// base + voff (per lane) + soff (wave-uniform), all in bytes; the descriptor (raw buffer, no bounds
// in practice) is rebuilt from the base pointer at each call site and hoisted by the compiler.
__device__ __forceinline__ void buffer_load_lds16(const void* base, lptr_t dst, uint32_t voff, int soff) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)0xFFFFFFFFu, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, soff, 0, 0);
}

// tile t of a problem -> (tile row, tile column): groups of 8 tile rows, column-major inside
template <class PROBLEM>
__device__ __forceinline__ void tile_coords(const PROBLEM& P, int t, int& tm, int& tn) {
  constexpr int GM = 8;
  int per = GM * P.tiles_n;
  int g = t / per, r = t - g * per;
  int first = g * GM;
  int gsz = P.tiles_m - first < GM ? P.tiles_m - first : GM;
  tm = first + r % gsz;
  tn = r / gsz;
}

// MODE: 0 = production; 4 = split-K: workgroup b = tile*splits + s walks the s-th share of the
// k-slabs and leaves its fp32 accumulators, in register order, in chunk b of batch.partial for
// splitk_reduce_kernel (small-M problems have too few tiles to fill the chip and a lone
// tile's k-loop runs at global-memory latency per slab).
// CONV: every problem of the batch is a 3x3 convolution (GemmProblem::conv_w > 0); a separate
// instantiation so that the plain product's address arithmetic stays as it is.
// Slabs are fetched with buffer_load ... lds: descriptor in SGPRs, one 32-bit byte offset per lane, taken
// from the tile's first row (for a convolution: from that row's window) and never changing, the k advance
// in an SGPR: no vector address arithmetic in the loop and a cheaper issue than global_load_lds with
// 64-bit lane addresses (measured +2..7 %, convolutions +2.5 %).
template <int BM, int BN, int WM, int WN, int BKT, int NS, int MODE, bool CONV = false>
__global__ __launch_bounds__(WM * WN * 64) void gemm_kernel(const GemmBatch batch) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int ROWB = BKT * 2;                        // bytes of one slab row in LDS
  constexpr int CPR = BKT / 8;                         // 16-byte chunks per slab row
  constexpr int KK = BKT / 16;                         // k-steps per slab (2 or 4)
  constexpr int LA = BM * CPR / NT, LB = BN * CPR / NT;   // chunks per thread per slab
  constexpr int LPS = LA + LB;
  static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads");
  static_assert((NS - 1) * LPS < 64, "vmcnt range");
  extern __shared__ __attribute__((aligned(128))) unsigned char smem[];
  constexpr int STAGE = (BM + BN) * ROWB;   // one slab of A then one slab of W
  constexpr int OFFB = BM * ROWB;

  // ---- workgroup -> (problem, tile) ----------------------------------------------------
  int bid = blockIdx.x, nb = gridDim.x;
  {
    int x = bid & 7, idx = bid >> 3, q = nb >> 3, rem = nb & 7;
    bid = x * q + (x < rem ? x : rem) + idx;
  }
  const int chunk = bid;          // split-K: this workgroup's slot in batch.partial
  int split = 0;
  if (MODE == 4) { split = bid % batch.splits; bid /= batch.splits; }
  GemmProblem P = batch.p[0];   // static indices only: keeps the argument block in SGPRs
  if (batch.n > 1 && bid >= batch.p[1].tile_start) P = batch.p[1];
  if (batch.n > 2 && bid >= batch.p[2].tile_start) P = batch.p[2];
  int tm, tn;
  tile_coords(P, bid - P.tile_start, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  constexpr int RPL = 64 / CPR;                        // slab rows that one load of a wave fills

  // ---- per-thread global source offsets ------------------------------------------------
  // (element offsets from the matrix base; every operand is far below 2^31 elements)
  uint32_t ga[LA], gb[LB];
  size_t conv_pix0 = 0;        // convolution: window of row m0 in the stack of bordered images
  if constexpr (CONV) {
    const int mm = m0 < P.M ? m0 : P.M - 1;
    const int b = mm / P.conv_img, r = mm - b * P.conv_img;
    const int y = r / P.conv_w, x = r - y * P.conv_w;
    conv_pix0 = (size_t)(b * (P.conv_img / P.conv_w + 2) + y) * (P.conv_w + 2) + x;
  }
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (i * (WM * WN) + wave) * RPL + lane / CPR, pc = lane % CPR, c = pc ^ swz_key<BKT>(r);
    int m = m0 + r; if (m >= P.M) m = P.M - 1;            // clamp: rows past M are never stored
    if constexpr (CONV) {    // top-left pixel of the 3x3 window in the stack of bordered images
      const int b = m / P.conv_img, r = m - b * P.conv_img;
      const int y = r / P.conv_w, x = r - y * P.conv_w;
      const size_t pix = (size_t)(b * (P.conv_img / P.conv_w + 2) + y) * (P.conv_w + 2) + x;
      // from the window of the tile's first row (pixels of later rows lie behind it)
      ga[i] = (uint32_t)((pix - conv_pix0) * (size_t)P.conv_cin) + c * 8;
    } else {
      ga[i] = (uint32_t)(m - m0) * (uint32_t)P.lda + c * 8;    // from the tile's first row (the buffer's base)
    }
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int r = (i * (WM * WN) + wave) * RPL + lane / CPR, pc = lane % CPR, c = pc ^ swz_key<BKT>(r);
    const int rw = !CONV && MODE == 0 && P.out_kind == OUT_GEGLU ? (r >> 6) * 32 + (r & 31) : r;
    gb[i] = (uint32_t)rw * (uint32_t)P.ldw + c * 8; // weights are padded to N_pad rows
  }


  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  // place of element e in its 32x32 tile
  auto acc_row = [&](int e) { return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); };
  const int acc_col = lane & 31;

  int nk = P.K / BKT;           // slabs of the product
  int kb = 0;                   // first slab of my share
  if (MODE == 4) {              // my share of the slabs (shares differ by at most one slab)
    const int ke = (split + 1) * nk / batch.splits;
    kb = split * nk / batch.splits;
    nk = ke - kb;
  }
  // With a second term of A the same slabs of both, the second term's first: its sum is small when the first term's begins and costs
  // no precision (behind it, a second chain of additions at full size made the error 1.6 to 1.8 times that of two products).
  const int n_lo = !CONV && P.A2 ? nk : 0;
  nk += n_lo;
  // lanes address their tile by 32-bit byte offsets from its first row, so no operand size limit
  const bf16_t* const tileA = CONV ? P.A + conv_pix0 * (size_t)P.conv_cin : P.A + (size_t)m0 * P.lda;
  const bf16_t* const tileA2 = !CONV && P.A2 ? P.A2 + (size_t)m0 * P.lda : tileA;
  // a gated pair: every 64 columns of the tile are 32 of the gate and the same 32 of the values
  const bool pair = !CONV && MODE == 0 && P.out_kind == OUT_GEGLU;
  const bf16_t* const tileW = P.W + (size_t)(pair ? n0 >> 1 : n0) * P.ldw;
  const bf16_t* const tileW2 = pair ? P.W2 + (size_t)(n0 >> 1) * P.ldw : tileW;
  const int half = lane >> 5;
  // LDS byte offsets of this lane's fragment rows (the chunk index is XORed in per k-step;
  // the key is the same for rows 32 apart)
  const int arow = wm * (BM / WM) + (lane & 31);
  const int brow = wn * (BN / WN) + (lane & 31);
  const int akey = swz_key<BKT>(arow), bkey = swz_key<BKT>(brow);
  const int abase = arow * ROWB, bbase = OFFB + brow * ROWB;

  // A load's lanes land at LDS byte row*ROWB + lane*16 of their slab (row: its first).  Slab indices
  // past the end are clamped (the copy is redundant but keeps the load count per slab fixed,
  // which the vmcnt arithmetic below relies on).
  auto issue = [&](int kt) {
    unsigned char* dA = smem + (kt % NS) * STAGE;
    unsigned char* dB = dA + OFFB;
    const int slab = kt < nk ? kt : nk - 1;
    const bool lo = slab < n_lo;
    const int ks = (kb + (lo ? slab : slab - n_lo)) * BKT;
    int ka = ks;             // A-side offset of the slab
    if constexpr (CONV) {    // slab = 64 channels of one tap (ky, kx): shift by ky rows and kx pixels
      int tap = ks / P.conv_cin;
      const int c0 = ks - tap * P.conv_cin;
      int kf = 0;            // 27 taps: the first index is the frame, 0 = two frames back (the stack starts two frames early)
      if (P.conv_kt == 3) { kf = tap / 9; tap -= 9 * kf; }
      const int ky = tap / 3, kx = tap - 3 * ky;
      ka = ((kf * (P.conv_img / P.conv_w + 2) + ky) * (P.conv_w + 2) + kx) * P.conv_cin + c0;
    }
#pragma unroll
    for (int i = 0; i < LA; ++i) buffer_load_lds16(lo ? tileA2 : tileA, (lptr_t)(dA + (i * NT + wave * 64) * 16), ga[i] * 2u, ka * 2);
#pragma unroll
    for (int i = 0; i < LB; ++i)      // (a load's rows lie in one half of their 64)
      buffer_load_lds16(((i * (WM * WN) + wave) * RPL >> 5) & 1 ? tileW2 : tileW, (lptr_t)(dB + (i * NT + wave * 64) * 16), gb[i] * 2u, ks * 2);
  };
  auto load_frags = [&](const unsigned char* st, int kk, bf16x8 (&a)[TM], bf16x8 (&b)[TN]) {
    const int c = kk * 2 + half;
    const unsigned char* pa = st + abase + ((c ^ akey) << 4);
    const unsigned char* pb = st + bbase + ((c ^ bkey) << 4);
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = *(const bf16x8*)(pa + i * 32 * ROWB);
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = *(const bf16x8*)(pb + j * 32 * ROWB);
  };
  auto mfma_all = [&](const bf16x8 (&a)[TM], const bf16x8 (&b)[TN]) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };

  bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
#pragma unroll
  for (int sidx = 0; sidx < NS; ++sidx) issue(sidx);
  wait_vm<(NS - 1) * LPS, false>();          // slab 0 has landed (mine)
  wg_barrier();   // ... and everyone's
  load_frags(smem, 0, a0, b0);
  int st_cur = 0;                            // stage of slab kt
  for (int kt = 0; kt < nk; ++kt) {
    const unsigned char* cur = smem + st_cur * STAGE;
    const int st_nxt = st_cur + 1 == NS ? 0 : st_cur + 1;
    const unsigned char* nxt = smem + st_nxt * STAGE;
    load_frags(cur, 1, a1, b1);
    mfma_all(a0, b0);
    interleave_hint<TM + TN, TM * TN>();
    if (KK == 4) {
      load_frags(cur, 2, a0, b0);
      mfma_all(a1, b1);
      interleave_hint<TM + TN, TM * TN>();
      load_frags(cur, 3, a1, b1);
      mfma_all(a0, b0);
      interleave_hint<TM + TN, TM * TN>();
    }
    // The last fragments of this slab are on their way to registers; slabs kt+1..kt+NS-1 are in
    // flight.  Wait for slab kt+1 (mine) and my fragments; after the barrier nobody reads `cur`
    // any more and `nxt` is visible to all.
    wait_vm<(NS - 2) * LPS, true>();
    wg_barrier();
    issue(kt + NS);                          // into the stage of slab kt
    load_frags(nxt, 0, a0, b0);              // (after the last slab this reads a stale stage; unused)
    mfma_all(a1, b1);
    interleave_hint<TM + TN, TM * TN>();
    st_cur = st_nxt;
  }
  wait_vm<0, true>();                        // drain the redundant tail loads before LDS is released
  if (MODE == 4) {
    // float4 number q = (((wave*TM + i)*TN + j)*4 + g)*64 + lane of the chunk holds
    // C[32i + 8g + 4*half + 0..3][32j + lane%32] of wave's sub-tile: 1 KB per store instruction
    float* pc = batch.partial + (size_t)chunk * (BM * BN);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 v4 = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
          *(f32x4*)(pc + ((((wave * TM + i) * TN + j) * 4 + g) * 64 + lane) * 4) = v4;
        }
    return;
  }

  // ---- epilogue ---------------------------------------------------------------------------
  // acc[i][j][e] is C[32i + acc_row(e)][32j + acc_col] of the wave's sub-tile: a lane
  // holds one or two columns, so direct stores would be 2- or 4-byte pieces.  Each wave therefore turns
  // its sub-tile 32 rows at a time through a private LDS patch (row stride TN*128 + 32 bytes:
  // the two half-waves, 4 rows apart, then fall into disjoint bank halves) and reads it back
  // row-major, 4 (fp32 out) or 8 (bf16 out) consecutive columns per lane: global accesses are
  // 16 bytes per lane and whole rows of the sub-tile per instruction.
  __syncthreads();     // every wave's ring loads have landed and all fragment reads are done
  constexpr int RS = TN * 128 + 32;
  unsigned char* stg = smem + wave * (32 * RS);
  static_assert(WM * WN * 32 * RS <= NS * STAGE, "staging patch fits the ring");
  auto epilogue = [&](auto kind_tag) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool F32OUT = KIND == OUT_F32 || KIND == OUT_RESID_F32;
    constexpr int VEC = F32OUT ? 4 : 8;          // columns per lane
    constexpr int LPR = TN * 32 / VEC;           // lanes per row
    constexpr int RPI = 64 / LPR;                // rows per instruction
    const int lr = lane / LPR, lc = (lane % LPR) * VEC;
    const int n = n0 + wn * (BN / WN) + lc;      // first of this lane's columns
    const bool full = n + VEC <= P.N;
    float bv[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) bv[c] = (P.bias && n + c < P.N) ? P.bias[n + c] : 0.f;
    // convolutions with fp32 output: per-column sums and sums of squares of the values stored,
    // over this wave's rows (the statistics pass of the group norm that follows).  Rows 8 apart are added one after the other,
    // then the eight sums in pairs: the order of gemm8_kernel, so that an image's statistics do not move with the tile.
    constexpr bool STATS = CONV && F32OUT;
    constexpr int CLS = STATS ? 8 / RPI : 1;     // rows of this lane modulo 8
    static_assert(!STATS || RPI == 4, "two classes of rows a lane");
    float cs[CLS][STATS ? VEC : 1], cq[CLS][STATS ? VEC : 1];
    if constexpr (STATS) {
#pragma unroll
      for (int k = 0; k < CLS; ++k)
#pragma unroll
        for (int c = 0; c < VEC; ++c) { cs[k][c] = 0.f; cq[k][c] = 0.f; }
    }
    // Gated residual: the loads of an output row (request index -> gate vector, and the residual itself)
    // depend on each other and may not be moved across the stores by the compiler, so they are issued
    // by hand for all rows of a 32-row patch at once: two memory latencies per patch instead of two per row.
    constexpr int NIT = 32 / RPI;
    constexpr bool RESID = KIND == OUT_RESID_F32;
    int rq[RESID ? NIT : 1];
    auto load_rq = [&](int i) {
      if constexpr (RESID) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int m = m0 + wm * (BM / WM) + i * 32 + it * RPI + lr;
          rq[it] = (P.row_req && m < P.M) ? P.row_req[m] : 0;
        }
      }
    };
    load_rq(0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          *(float*)(stg + acc_row(e) * RS + (j * 32 + acc_col) * 4) = acc[i][j][e];
      f32x4 xr[RESID ? NIT : 1], gr[RESID ? NIT : 1];
      // (tiles with 128 or more accumulator registers per lane fetch half a patch at a time)
      constexpr int GRP = (RESID && TM * TN >= 8) ? NIT / 2 : NIT;
      auto load_resid = [&](int first) {
        if constexpr (RESID) {
#pragma unroll
          for (int it = first; it < first + GRP; ++it) {
            const int m = m0 + wm * (BM / WM) + i * 32 + it * RPI + lr;
            xr[it] = f32x4{0.f, 0.f, 0.f, 0.f};
            gr[it] = f32x4{1.f, 1.f, 1.f, 1.f};
            if (full && m < P.M) {
              xr[it] = *(const f32x4*)((const float*)P.out + (size_t)m * P.ldc + n);
              if (P.gate) gr[it] = *(const f32x4*)(P.gate + (size_t)rq[it] * P.gate_stride + n);
            }
          }
        }
      };
      load_resid(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        if (GRP < NIT && it == GRP) load_resid(GRP);
        if (RESID && it == NIT - 1 && i + 1 < TM) load_rq(i + 1);
        const int row = it * RPI + lr;
        const int m = m0 + wm * (BM / WM) + i * 32 + row;
        float v[VEC];
#pragma unroll
        for (int c4 = 0; c4 < VEC / 4; ++c4) {
          const f32x4 t4 = *(const f32x4*)(stg + row * RS + (lc + 4 * c4) * 4);
#pragma unroll
          for (int c = 0; c < 4; ++c) v[4 * c4 + c] = t4[c] + bv[4 * c4 + c];
        }
        if (m >= P.M || n >= P.N) continue;
        const size_t o = (size_t)m * P.ldc + n;
        if constexpr (KIND == OUT_RESID_F32) {
          float* xp = (float*)P.out + o;
          if (full) {
            f32x4 x4 = xr[it];
#pragma unroll
            for (int c = 0; c < 4; ++c) x4[c] += gr[it][c] * v[c];
            *(f32x4*)xp = x4;
            if constexpr (STATS) {
#pragma unroll
              for (int c = 0; c < 4; ++c) { cs[it % CLS][c] += x4[c]; cq[it % CLS][c] += x4[c] * x4[c]; }
            }
          } else {
            // (ragged last columns: the request index is read here, rq[] may already hold the next patch's)
            const float* gp = P.gate ? P.gate + (size_t)(P.row_req ? P.row_req[m] : 0) * P.gate_stride + n : nullptr;
            for (int c = 0; c < VEC && n + c < P.N; ++c) {
              const float r = xp[c] + (gp ? gp[c] : 1.f) * v[c];
              xp[c] = r;
              if constexpr (STATS) { cs[it % CLS][c] += r; cq[it % CLS][c] += r * r; }
            }
          }
        } else if constexpr (KIND == OUT_F32) {
          float* xp = (float*)P.out + o;
          if (full) {
            f32x4 x4 = {v[0], v[1], v[2], v[3]};
            *(f32x4*)xp = x4;
          } else {
            for (int c = 0; c < VEC && n + c < P.N; ++c) xp[c] = v[c];
          }
          if constexpr (STATS) {
#pragma unroll
            for (int c = 0; c < VEC; ++c) { cs[it % CLS][c] += v[c]; cq[it % CLS][c] += v[c] * v[c]; }   // (columns past N are not written out)
          }
        } else {
          if constexpr (KIND == OUT_GELU_BF16) {
#pragma unroll
            for (int c = 0; c < VEC; ++c) v[c] = gelu_tanh(v[c]);
          }
          bf16_t* xp = (bf16_t*)P.out + o;
          if (full) {
            u32x4 w;
#pragma unroll
            for (int c = 0; c < 4; ++c) w[c] = pack2bf(v[2 * c], v[2 * c + 1]);
            *(u32x4*)xp = w;
          } else {
            for (int c = 0; c < VEC && n + c < P.N; ++c) xp[c] = f2bf(v[c]);
          }
        }
      }
      asm volatile("" ::: "memory");
    }
    if constexpr (STATS) {
      if (P.stats) {      // partial[(tile row * WM + wm)][column][2]: rows of one wave of one tile
#pragma unroll
        for (int c = 0; c < VEC; ++c)
#pragma unroll
          for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
            for (int k = 0; k < CLS; ++k) { cs[k][c] += __shfl_xor(cs[k][c], o); cq[k][c] += __shfl_xor(cq[k][c], o); }
        if (lr == 0) {
          float* sp = P.stats + ((size_t)(tm * WM + wm) * P.N + n) * 2;
          for (int c = 0; c < VEC && n + c < P.N; ++c) { sp[2 * c] = cs[0][c] + cs[CLS - 1][c]; sp[2 * c + 1] = cq[0][c] + cq[CLS - 1][c]; }
        }
      }
    }
  };
  // q/k columns of a QKV product: RMS norm per head, gain, rotary code, scale, scatter by row.
  // A wave's 64 columns are one head (head_dim 64) or half of one (128: the two waves of a
  // pair exchange their partial sums of squares through LDS).
  auto epilogue_qk = [&]() {
    if constexpr (BN / WN == 64) {
      constexpr int VEC = 8, LPR = 8, RPI = 8;
      const QkNorm& Q = P.qk;
      const int lr = lane / LPR, lc = (lane % LPR) * VEC;
      const int n = n0 + wn * 64 + lc;               // first of this lane's 8 output columns
      const bool is_k = n >= Q.nq;
      const int col_in = is_k ? n - Q.nq : n;        // column inside the q (k) range
      const int hc = col_in & (Q.head_dim - 1);      // ... inside the head
      const bool wide = Q.head_dim == 128;
      const float inv_dh = 1.0f / (float)Q.head_dim;
      const float osc = is_k ? 1.0f : Q.qscale;
      float bv[VEC], gv[VEC];
      {
        const float* gp = (is_k ? Q.kgain : Q.qgain) + hc;
        const f32x4 g0 = *(const f32x4*)gp, g1 = *(const f32x4*)(gp + 4);
#pragma unroll
        for (int c = 0; c < 4; ++c) { gv[c] = g0[c]; gv[4 + c] = g1[c]; }
#pragma unroll
        for (int c = 0; c < VEC; ++c) bv[c] = P.bias ? P.bias[n + c] : 0.f;
      }
      float* xch = (float*)(smem + WM * WN * 32 * RS);   // [2][waves][32] partial sums of squares
      static_assert(WM * WN * 32 * RS + 2 * WM * WN * 32 * 4 <= NS * STAGE, "exchange area fits the ring");
      bf16_t* dst = is_k ? Q.ko : Q.qo;
      // Destination rows one patch ahead, and per patch the rotary pairs of its rows while the patch
      // turns through LDS: the compiler may not move these loads across the stores, and issued row by row
      // each would cost a full memory latency.
      int dnext[4];
      auto load_drows = [&](int i) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int m = m0 + wm * (BM / WM) + i * 32 + it * RPI + lr;
          dnext[it] = (Q.dst_row && m < P.M) ? Q.dst_row[m] : m;
        }
      };
      load_drows(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            *(float*)(stg + acc_row(e) * RS + (j * 32 + acc_col) * 4) = acc[i][j][e];
        int drows[4];
        f32x4 rc0[4], rc1[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) drows[it] = dnext[it];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int m = m0 + wm * (BM / WM) + i * 32 + it * RPI + lr;
          rc0[it] = f32x4{1.f, 0.f, 1.f, 0.f}; rc1[it] = f32x4{1.f, 0.f, 1.f, 0.f};      // (cos, sin) pairs
          if (Q.rope && m < P.M) {
            const f32x4* rp = (const f32x4*)(Q.rope + (size_t)drows[it] * (Q.head_dim / 2) + (hc >> 1));
            rc0[it] = rp[0]; rc1[it] = rp[1];
          }
        }
        if (i + 1 < TM) load_drows(i + 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        float v[4][VEC], ss[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = it * RPI + lr;
          const f32x4 t0 = *(const f32x4*)(stg + row * RS + lc * 4), t1 = *(const f32x4*)(stg + row * RS + (lc + 4) * 4);
          float s2 = 0.f;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            v[it][c] = t0[c] + bv[c]; v[it][4 + c] = t1[c] + bv[4 + c];
            s2 += v[it][c] * v[it][c] + v[it][4 + c] * v[it][4 + c];
          }
          s2 += __shfl_xor(s2, 1); s2 += __shfl_xor(s2, 2); s2 += __shfl_xor(s2, 4);
          ss[it] = s2;
        }
        if (wide) {
          float* mine = xch + ((i & 1) * (WM * WN) + wave) * 32;
          const float* other = xch + ((i & 1) * (WM * WN) + (wave ^ 1)) * 32;
          if ((lane % LPR) == 0) {
#pragma unroll
            for (int it = 0; it < 4; ++it) mine[it * RPI + lr] = ss[it];
          }
          __syncthreads();
#pragma unroll
          for (int it = 0; it < 4; ++it) ss[it] += other[it * RPI + lr];
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int m = m0 + wm * (BM / WM) + i * 32 + it * RPI + lr;
          if (m >= P.M) continue;
          const float r = rsqrtf(ss[it] * inv_dh + 1e-6f) * osc;
          const int drow = drows[it];
          const f32x4 c0 = rc0[it], c1 = rc1[it];
          const float cs[8] = {c0[0], c0[1], c0[2], c0[3], c1[0], c1[1], c1[2], c1[3]};
          u32x4 w;
#pragma unroll
          for (int pz = 0; pz < 4; ++pz) {
            const float a = v[it][2 * pz] * r * gv[2 * pz], b = v[it][2 * pz + 1] * r * gv[2 * pz + 1];
            const float ra = a * cs[2 * pz] - b * cs[2 * pz + 1], rb = a * cs[2 * pz + 1] + b * cs[2 * pz];
            w[pz] = Q.f16 ? pack2h(ra, rb) : pack2bf(ra, rb);
          }
          *(u32x4*)(dst + (size_t)drow * Q.ldo + col_in) = w;
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);    // patches one after the other: work hoisted across them costs registers
      }
    }
  };
  // value columns of a QKV product written transposed (the layout the attention kernel reads): the
  // wave's 32-row patch goes through LDS column-major, and a lane writes two consecutive rows of one
  // output column as one 4-byte piece when they are neighbours in the transposed matrix (always, except
  // across a request boundary or at an odd start), else as single elements.
  auto epilogue_vt = [&]() {
   if constexpr (BN / WN == 64) {                      // (the tile variants that take q/k-norm problems)
    const QkNorm& Q = P.qk;
    constexpr int CS = 36 * 4;                         // bytes per patch column: 32 rows + padding, 16-byte aligned
    static_assert(TN * 32 * CS <= 32 * RS, "transposed patch fits the wave's staging area");
    const int nv0 = n0 + wn * (BN / WN) - (Q.nq + Q.nk);   // first value column of the wave
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          *(float*)(stg + (j * 32 + acc_col) * CS + acc_row(e) * 4) = acc[i][j][e];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const int mb = m0 + wm * (BM / WM) + i * 32;     // first row of the patch
      // whole patch in range, its 32 rows neighbours in the transposed matrix, starting at a multiple of 8:
      // a lane writes 8 rows of one column as one 16-byte piece
      bool consec = mb + 32 <= P.M;
      int cb = 0;
      if (consec) {
        cb = Q.vt_col[mb];
        consec = Q.vt_col[mb + 31] == cb + 31;
      }
      if (consec && (cb & 7) != 0) {
        // Neighbours, but starting off a multiple of 8 (a request's image rows follow 154 text rows): three
        // 16-byte pieces from the first aligned column on, written by lanes 0-2 of each group of four; the
        // fourth lane writes the 8 rows before and after them as pairs (even start) or single elements.
        const int r0 = 8 - (cb & 7);                   // patch row of the first aligned column
        const int rg = lane & 3, cl = lane >> 2;
#pragma unroll
        for (int it = 0; it < TN * 32 / 16; ++it) {
          const int col = it * 16 + cl, nv = nv0 + col;
          if (nv + Q.nq + Q.nk >= P.N) continue;
          const float* pc = (const float*)(stg + col * CS);
          const float bv = P.bias ? P.bias[nv + Q.nq + Q.nk] : 0.f;
          bf16_t* dst = Q.vt + (size_t)nv * Q.ldvt + cb;
          if (rg < 3) {
            const float* t = pc + r0 + 8 * rg;
            u32x4 w = {pack2bf(t[0] + bv, t[1] + bv), pack2bf(t[2] + bv, t[3] + bv), pack2bf(t[4] + bv, t[5] + bv), pack2bf(t[6] + bv, t[7] + bv)};
            *(u32x4*)(dst + r0 + 8 * rg) = w;
          } else if ((cb & 1) == 0) {
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
              const int r = k < r0 ? k : k + 24;
              *(uint32_t*)(dst + r) = pack2bf(pc[r] + bv, pc[r + 1] + bv);
            }
          } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int r = k < r0 ? k : k + 24;
              dst[r] = f2bf(pc[r] + bv);
            }
          }
        }
      } else if (consec) {
        const int rg = lane & 3, cl = lane >> 2;
#pragma unroll
        for (int it = 0; it < TN * 32 / 16; ++it) {
          const int col = it * 16 + cl, nv = nv0 + col;
          const f32x4 t0 = *(const f32x4*)(stg + col * CS + rg * 32), t1 = *(const f32x4*)(stg + col * CS + rg * 32 + 16);
          if (nv + Q.nq + Q.nk >= P.N) continue;
          const float bv = P.bias ? P.bias[nv + Q.nq + Q.nk] : 0.f;
          u32x4 w = {pack2bf(t0[0] + bv, t0[1] + bv), pack2bf(t0[2] + bv, t0[3] + bv), pack2bf(t1[0] + bv, t1[1] + bv), pack2bf(t1[2] + bv, t1[3] + bv)};
          *(u32x4*)(Q.vt + (size_t)nv * Q.ldvt + cb + rg * 8) = w;
        }
      } else {
        const int rp = lane & 15, cl = lane >> 4;      // this lane's row pair and column phase
        const int m = mb + 2 * rp;
        const bool ok0 = m < P.M, ok1 = m + 1 < P.M;
        const int c0 = ok0 ? Q.vt_col[m] : 0, c1 = ok1 ? Q.vt_col[m + 1] : -1;
        const bool pair = ok1 && c1 == c0 + 1 && (c0 & 1) == 0;
#pragma unroll
        for (int it = 0; it < TN * 32 / 4; ++it) {
          const int col = it * 4 + cl;                 // column inside the wave's patch
          const int nv = nv0 + col;                    // value column = row of the transposed matrix
          const f32x2 t2 = *(const f32x2*)(stg + col * CS + rp * 8);
          if (nv + Q.nq + Q.nk >= P.N) continue;
          const float bv = P.bias ? P.bias[nv + Q.nq + Q.nk] : 0.f;
          bf16_t* dst = Q.vt + (size_t)nv * Q.ldvt;
          if (pair) *(uint32_t*)(dst + c0) = pack2bf(t2[0] + bv, t2[1] + bv);
          else {
            if (ok0) dst[c0] = f2bf(t2[0] + bv);
            if (ok1) dst[c1] = f2bf(t2[1] + bv);
          }
        }
      }
      asm volatile("" ::: "memory");
    }
   }
  };
  // gated pair: the wave's 64 columns are 32 of the gate, then the same 32 of the values
  auto epilogue_pair = [&]() {
    if constexpr (BN / WN == 64) {
      const int lr = lane >> 2, lc = (lane & 3) * 8;
      const int n = (n0 >> 1) + wn * 32 + lc, n_end = P.N >> 1;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            *(float*)(stg + acc_row(e) * RS + (j * 32 + acc_col) * 4) = acc[i][j][e];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int row = it * 16 + lr, m = m0 + wm * (BM / WM) + i * 32 + row;
          float v[8];
#pragma unroll
          for (int c4 = 0; c4 < 2; ++c4) {
            const f32x4 g = *(const f32x4*)(stg + row * RS + (lc + 4 * c4) * 4), u = *(const f32x4*)(stg + row * RS + (32 + lc + 4 * c4) * 4);
#pragma unroll
            for (int c = 0; c < 4; ++c) v[4 * c4 + c] = gelu_tanh(g[c]) * u[c];
          }
          if (m >= P.M || n >= n_end) continue;
          bf16_t* xp = (bf16_t*)P.out + (size_t)m * P.ldc + n;
          if (n + 8 <= n_end) {
            u32x4 w;
#pragma unroll
            for (int c = 0; c < 4; ++c) w[c] = pack2bf(v[2 * c], v[2 * c + 1]);
            *(u32x4*)xp = w;
          } else {
            for (int c = 0; c < n_end - n; ++c) xp[c] = f2bf(v[c]);
          }
        }
        asm volatile("" ::: "memory");
      }
    }
  };
  if (P.out_kind == OUT_GEGLU) { if constexpr (!CONV) epilogue_pair(); }
  else if (P.out_kind == OUT_VT) { if constexpr (!CONV) epilogue_vt(); }
  else if (P.out_kind == OUT_QKNORM) {
    if (n0 < P.qk.nq + P.qk.nk) epilogue_qk();
    else if (P.qk.vt) epilogue_vt();
    else epilogue(std::integral_constant<int, OUT_BF16>{});
  }
  else if (P.out_kind == OUT_BF16) epilogue(std::integral_constant<int, OUT_BF16>{});
  else if (P.out_kind == OUT_F32) epilogue(std::integral_constant<int, OUT_F32>{});
  else if (P.out_kind == OUT_GELU_BF16) epilogue(std::integral_constant<int, OUT_GELU_BF16>{});
  else epilogue(std::integral_constant<int, OUT_RESID_F32>{});
}

// ---- 8-wave tiles: two groups of waves, tiles in one stream ------------------------------------------------
//
// 256x256 and 320x256 tiles (NS = 2 stages, two phases per slab) and the 256x128 tile (3 stages, one phase).
//
// Loop.  Two groups of four waves (wave / 4; each has one wave on every SIMD), half a phase apart: while one group's
// waves do nothing but multiply, the other's read the fragments of their next product and issue loads, so the matrix
// cores change hands at a barrier instead of idling while a wave waits for LDS (8192^3: 839 us with each wave
// interleaving reads and products, matrix cores 78 % busy; 768 us this way with the same MFMA form, 91 %).  They
// multiply with v_mfma_f32_16x16x32_bf16: the same cycles per flop as 32x32x16, but at that load the board lowers its
// clock to what it can feed, and per flop the 16x16 form draws less (714 us).
//   A group's reads are in registers before the barrier that ends its reading half, so what it read may be
// overwritten by loads of either group from its next phase on.  The wait at the end of a reading half covers
// the group's own loads of what the NEXT phase reads; the barriers in between make them visible to the other.
//
// Stream.  A workgroup stays on its CU and walks over its tiles (as many apart as its XCD has workgroups); the slabs of
// its tiles are ONE stream: behind the last slab of a tile the loads go on with the first of the next, which
// therefore arrive under the last products and the epilogue.
//
// Epilogue.  The operands are swapped, W in the place of MFMA rows: a lane then holds consecutive columns of ONE row, and
// with the rows of W fed in the order {0-3, 8-11, 16-19, 24-27}, {4-7, 12-15, ...} the two products of a pair of 16
// columns give it 8 neighbours: bias, GELU, norm and rotary code act on whole 16-byte pieces in registers, which are
// turned into runs of 128 bytes by 16-byte LDS accesses in a 2 KB patch per wave beside the ring.  Tiles of transposed
// values do the same with the operands in their first order and the rows of A permuted: 8 neighbouring tokens of a column.
//   The XOR key of a slab row takes its bits 1, 3 and 2^4, so that 16 rows fall into 16 distinct 16-byte slots in both
// orders.
//
// What bounds it: the matrix cores in the loop (1.32 us a slab of 256x256x64, 1.6 PFLOP/s); a tile's fixed part, 10 us
// with a workgroup per tile and the results turned as fp32 in 4-byte LDS stores, is a quarter of the time at K = 1536.
// Now 8 to 8.5 us, of which tanh-GELU is 3.6 and the stores 3 (each measured by leaving it out).  Before and after:
// 18384 x 6144 x 1536 with GELU 303 -> 292 us, 18384 x 4608 x 1536 226 -> 216, 18384 x 1536 x 6144 into the residual
// 307 -> 297, 32760 x 5120 x 5120 into the residual 1400 -> 1363 (as bf16 1177), 8192^3 722 -> 709; 3x3 convolutions of a million
// pixels with 128 channels 449 -> 426.  Counters at 8192^3: matrix cores busy in 90 % of the cycles at 1.57 GHz, no bank conflicts but
// the epilogue's.  The 320-row tile has no registers to hold the next tile's offsets and starts each tile anew.
// Tried: two workgroups of 4 waves a CU with 256x128 tiles, to let one's epilogue run under the other's loop (8192^3 at
// 1088 TFLOP/s); starts staggered over the CUs so that their stores do not collide (as much lost as gained);
// non-temporal stores (0.4 % at 32760 tokens, nothing elsewhere).
__device__ __forceinline__ int swz_key8(int r) { return ((r >> 1) & 1) | ((r >> 2) & 2) | (((r ^ (r >> 2)) & 4)); }

typedef const __attribute__((address_space(4))) GemmBatch Batch;
typedef const __attribute__((address_space(4))) GemmProblem Problem;
typedef const __attribute__((address_space(4))) QkNorm Norm;

template <int BM, int BN, int WM, int WN, int NS, bool CONV>
__global__ __launch_bounds__(512) void gemm8_kernel(const GemmBatch) {
  Batch& batch = *(Batch*)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int ROWB = 128, BKT = 64;                  // bytes of a slab row, columns of a slab
  constexpr int RT = BM / WM / 16, CT = 4;             // 16-row and 16-column tiles of a wave
  constexpr int PH = NS == 2 ? 2 : 1, RP = RT / PH;    // phases per slab, row tiles per phase
  constexpr int LA = BM / 64, LB = BN / 64, LPS = LA + LB;   // loads per wave and slab
  constexpr int LAU = NS == 2 ? WM : LA;               // ... of the first part of A: 64 rows of every wave row
  constexpr int STAGE = (BM + BN) * ROWB, OFFB = BM * ROWB;
  static_assert(WM * WN == 8 && BN / WN == 64 && BM % 64 == 0 && RT % PH == 0, "two groups of four waves, 64 columns a wave");
  static_assert(NS == 3 || (NS == 2 && RP * 16 >= 64), "two stages: the first part of A is read in phase 0 alone");
  constexpr bool STREAM = RT <= 8;                     // (320 rows: no registers to hold the next tile's offsets under the epilogue)
  constexpr bool LATE = RP * 16 == 64;                 // phase 0 reads none of the rest of A, which has a phase more to arrive
  extern __shared__ __attribute__((aligned(128))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  unsigned char* const patch = smem + NS * STAGE + wave * 2048;

  // ---- my tiles: XCD x (workgroup ids are dealt round-robin) owns a contiguous range of them -----------------
  int t_first, t_count, t_step;
  {
    const int x = blockIdx.x & 7, T = batch.total_tiles, G = gridDim.x;
    t_first = x * (T >> 3) + (x < (T & 7) ? x : (T & 7));
    t_count = (T >> 3) + (x < (T & 7) ? 1 : 0);
    t_step = (G >> 3) + (x < (G & 7) ? 1 : 0);
  }
  // The argument block is read where it lies, in the kernel's argument segment (its only argument): a copy of the
  // problem at hand would take half of the scalar registers.
  auto problem = [&](int bid) -> Problem& {
    const int i = batch.n > 2 && bid >= batch.p[2].tile_start ? 2 : batch.n > 1 && bid >= batch.p[1].tile_start ? 1 : 0;
    return batch.p[i];
  };

  // ---- the stream of slabs -----------------------------------------------------------------------------------
  // One load of a wave fills 8 slab rows.  With two stages A is fetched in two parts, the first 64 rows of every
  // wave row and the rest; row_a: first of the rows that the wave's i-th load of A fills.
  auto row_a = [&](int i) {
    if constexpr (NS == 2) {
      const bool up = i < LAU;
      const int per = up ? 64 : RT * 16 - 64;
      const int rr = ((up ? i : i - LAU) * 8 + wave) * 8;
      return rr / per * (RT * 16) + rr % per + (up ? 0 : 64);
    } else {
      return (i * 8 + wave) * 8;
    }
  };
  uint32_t oa[LA], ob[LB];        // byte offsets of my lane's 16-byte chunk of each load, from the tile's first row
  const bf16_t *sA, *sW;          // first rows of the tile whose slabs are fetched
  int ld_t = blockIdx.x >> 3;     // that tile (index in my XCD's range)
  int ks = 0, ks_n = 0, ka = 0;   // slab of it, their number, byte offset of the slab in A (in W: 128 ks)
  int run_left = 0, rows_left = 0, run_len = 0, run_skip = 0, frame_skip = 0;   // convolutions: see advance()
  auto aim = [&](int t) {
    const int bid = t_first + t;
    Problem& P = problem(bid);
    int tm, tn;
    tile_coords(P, bid - P.tile_start, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const bool pair = !CONV && P.out_kind == OUT_GEGLU;                      // every 64 columns: 32 of the gate, the same 32 of the values
    int ln = lane;
    asm volatile("" : "+v"(ln));                                           // (made anew for each tile: kept, these would cost registers)
    auto window = [&](int m) {    // convolution: top-left pixel of row m's 3x3 window in the stack of bordered images
      const int b = m / P.conv_img, r = m - b * P.conv_img;
      const int y = r / P.conv_w, x = r - y * P.conv_w;
      return (size_t)(b * (P.conv_img / P.conv_w + 2) + y) * (P.conv_w + 2) + x;
    };
    size_t pix0 = 0;
    if constexpr (CONV) pix0 = window(m0 < P.M ? m0 : P.M - 1);
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = row_a(i) + (ln >> 3), c = (ln & 7) ^ swz_key8(r);
      const int m = m0 + r < P.M ? m0 + r : P.M - 1;                       // clamp: rows past M are never stored
      if constexpr (CONV) oa[i] = (uint32_t)((window(m) - pix0) * (size_t)P.conv_cin + c * 8) * 2u;
      else oa[i] = ((uint32_t)(m - m0) * (uint32_t)P.lda + c * 8) * 2u;    // (32-bit offsets inside a tile: no operand limit)
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int r = (i * 8 + wave) * 8 + (ln >> 3), c = (ln & 7) ^ swz_key8(r);
      const int rw = pair ? (r >> 6) * 32 + (r & 31) : r;
      ob[i] = ((uint32_t)rw * (uint32_t)P.ldw + c * 8) * 2u;               // weights are padded to N_pad rows
    }
    sA = P.A + (CONV ? pix0 * (size_t)P.conv_cin : (size_t)m0 * P.lda);
    sW = (pair && (wave & 4) ? P.W2 : P.W) + (size_t)(pair ? n0 >> 1 : n0) * P.ldw;   // (waves 4-7 load the upper half of each 64 rows)
    ks = 0; ks_n = P.K / BKT; ka = 0;
    if constexpr (CONV) {
      run_len = run_left = 3 * P.conv_cin / BKT; rows_left = 3;
      run_skip = (P.conv_w - 1) * P.conv_cin * 2;
      frame_skip = (P.conv_img / P.conv_w - 1) * (P.conv_w + 2) * P.conv_cin * 2;
    }
  };
  // Next slab of the stream: of the same tile (a convolution's taps of one image row are neighbours in memory, 3 conv_cin
  // columns; then the next row of the window, then the next frame) ...
  auto next_slab = [&]() {
    ++ks; ka += BKT * 2;
    if constexpr (CONV)
      if (--run_left == 0) {
        run_left = run_len; ka += run_skip;
        if (--rows_left == 0) { rows_left = 3; ka += frame_skip; }
      }
  };
  // ... or the first of the next tile.  (Behind the very last one the same again: redundant, but it keeps the number of
  // loads per slab fixed, which the vmcnt arithmetic relies on.)
  auto advance = [&]() {
    if (ks + 1 < ks_n) next_slab();
    else if (STREAM && ld_t + t_step < t_count) {
      ld_t += t_step;
      aim(ld_t);
    }
  };
  auto issue_a = [&](int st, auto first, auto last) {
#pragma unroll
    for (int i = decltype(first)::value; i < decltype(last)::value; ++i)
      buffer_load_lds16(sA, (lptr_t)(smem + st * STAGE + row_a(i) * ROWB), oa[i], ka);
  };
  auto issue_b = [&](int st) {
#pragma unroll
    for (int i = 0; i < LB; ++i) buffer_load_lds16(sW, (lptr_t)(smem + st * STAGE + OFFB + (i * 8 + wave) * 1024), ob[i], ks * (BKT * 2));
  };
  constexpr std::integral_constant<int, 0> A_FIRST{};
  constexpr std::integral_constant<int, LAU> A_REST{};
  constexpr std::integral_constant<int, LA> A_END{};

  // ---- the loop over one tile's slabs ------------------------------------------------------------------------
  f32x4 acc[RT][CT];
  const bool second = wave >= 4;
  int stage = 0;                  // stage of the slab that is read next
  // Byte offsets of this lane's fragments.  Consecutive rows: 16-row tile i starts 16 i rows on, permuted rows
  // (8 rows for every 4 lanes): pairs of tiles 32 rows on, the odd one 4 rows on.  Odd tiles flip bit 2 of the key.
  // VT: the first operand is A with permuted rows (tiles of transposed values), else W with permuted rows.
  auto run = [&](auto vt_tag, int nk) {
    constexpr bool VT = decltype(vt_tag)::value;
    int ln = lane;
    asm volatile("" : "+v"(ln));                         // (made anew for each tile, as in aim())
    const int l16 = ln & 15, kq = ln >> 4;
    const int row_c = l16, row_p = (l16 >> 2) * 8 + (l16 & 3);
    const int off_c = row_c * ROWB + ((kq ^ swz_key8(row_c)) << 4), off_p = row_p * ROWB + ((kq ^ swz_key8(row_p)) << 4);
    bf16x8 fa[2][RP], fb[2][CT];
    auto tile_off = [](bool perm, int i) { return perm ? (i >> 1) * 32 + (i & 1) * 4 : i * 16; };
    const int a0 = wm * (RT * 16) * ROWB + (VT ? off_p : off_c), b0 = OFFB + wn * 64 * ROWB + (VT ? off_c : off_p);
    auto read_a = [&](const unsigned char* st, auto phase) {
      const unsigned char* p[2] = {st + a0, st + (a0 ^ 64)};
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          const int i = decltype(phase)::value * RP + r;
          fa[k][r] = *(const bf16x8*)(p[k ^ (i & 1)] + tile_off(VT, i) * ROWB);
        }
    };
    auto read_b = [&](const unsigned char* st) {
      const unsigned char* p[2] = {st + b0, st + (b0 ^ 64)};
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < CT; ++c) fb[k][c] = *(const bf16x8*)(p[k ^ (c & 1)] + tile_off(!VT, c) * ROWB);
    };
    auto multiply = [&](auto phase) {
      wg_barrier();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < RP; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            f32x4& d = acc[decltype(phase)::value * RP + r][c];
            if constexpr (VT) d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[k][r], fb[k][c], d, 0, 0, 0);
            else d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[k][c], fa[k][r], d, 0, 0, 0);
          }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      wg_barrier();
    };
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, PH - 1> P1{};
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (Waits that allow for the last epilogue's stores, two slabs long, cost more by their branches than they gain.)
    // One slab.  same: the stream's next slab is known to be of this tile, which keeps the aiming out of the loop.
    auto slab = [&](auto same) {
      const unsigned char* cur = smem + stage * STAGE;
      const int nxt = stage + 1 == NS ? 0 : stage + 1;
      if constexpr (decltype(same)::value) next_slab(); else advance();      // (here: no fragments are held)
      read_b(cur);
      read_a(cur, P0);
      if constexpr (NS == 2) {
        // Phase 0 of slab s reads the upper half of A and W; phase 1 reads the lower half of A and issues W and the first
        // part of A of slab s+2; when it is over the rest of A follows (over that of slab s, which everybody has read).
        wait_vm<LATE ? LPS : 63, true>();              // rest of A of slab s (mine; without LATE slab s is complete)
        multiply(P0);
        read_a(cur, P1);
        issue_b(stage); issue_a(stage, A_FIRST, A_REST);
        // W and the first part of A of slab s+1 (mine; without LATE all of it)
        wait_vm<LATE ? LPS : LB + LAU, true>();
        multiply(P1);
        issue_a(stage, A_REST, A_END);
      } else {
        // phase s reads slab s and issues slab s+2 into the stage that slab s-1 left
        const int free_st = nxt + 1 == NS ? 0 : nxt + 1;
        issue_a(free_st, A_FIRST, A_END); issue_b(free_st);
        wait_vm<LPS, true>();                          // slab s+1 (mine)
        multiply(P0);
      }
      stage = nxt;
    };
    if (second) wg_barrier();
    int kt = 0;
    for (; kt < nk - 2; ++kt) slab(std::true_type{});
    for (; kt < nk; ++kt) slab(std::false_type{});
    if (!second) wg_barrier();
  };

  // ---- epilogues: non-VT tiles hold C[16 r + l16][32 j + 8 kq + 0..7] of the wave's sub-tile in acc[r][2 j], acc[r][2 j + 1] ----
  // (Row addresses: a scalar base per 8 rows and one lane offset.  The scheduling barriers keep a unit's work from
  // being hoisted over the ones before it, which costs registers.)
  auto epilogue = [&](Problem& P, int tm, int m0, int n0, bool vt) {
    int ln = lane;
    asm volatile("" : "+v"(ln));                         // (lane numbers are made anew: kept through the loop they would cost registers)
    const int l16 = ln & 15, kq = ln >> 4;
    const int prow = ln >> 3, pchunk = ln & 7;           // my row (and the one 8 on) and 16-byte chunk when a patch is read back
    const int mw = m0 + wm * (RT * 16), nw = n0 + wn * 64;
    const int M = P.M, N = P.N, kind = P.out_kind;
    const float* const bias = P.bias;
    constexpr bool PIPE = RT <= 8;                       // a unit is turned while the one before it is stored (where registers allow)
    auto patch_at = [&](int row, int chunk) { return patch + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); };
    auto turn = [&](const u32x4& lo, const u32x4& hi, int c_lo, int c_hi, u32x4 (&out)[2]) {    // 16 rows x 128 bytes
      *(u32x4*)patch_at(l16, c_lo) = lo;
      *(u32x4*)patch_at(l16, c_hi) = hi;
      asm volatile("" ::: "memory");                     // (a wave's LDS accesses are executed in order)
      out[0] = *(const u32x4*)patch_at(prow, pchunk);
      out[1] = *(const u32x4*)patch_at(prow + 8, pchunk);
      asm volatile("" ::: "memory");
    };
    auto load_cols = [&](const float* p, float (&v)[2][8]) {   // per-column values of my 16 columns
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int n = nw + j * 32 + kq * 8 + c;
          v[j][c] = p && n < N ? p[n] : 0.f;
        }
    };
    auto raw = [&](int r, int j, float (&v)[8]) {
#pragma unroll
      for (int c = 0; c < 4; ++c) { v[c] = acc[r][2 * j][c]; v[4 + c] = acc[r][2 * j + 1][c]; }
    };
    // bf16 results: value(r, j, v) makes the 8 values of row tile r, columns 32 j + 8 kq ...; row_ptr(r, h): where my 8
    // columns of row 16 r + 8 h + prow go
    auto store_bf16 = [&](auto value, auto pack2, auto row_ptr) {
      const bool full = nw + pchunk * 8 + 8 <= N;
      auto make = [&](int r, u32x4 (&w)[2]) {
        u32x4 p[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          float v[8];
          value(r, j, v);
#pragma unroll
          for (int c = 0; c < 4; ++c) p[j][c] = pack2(v[2 * c], v[2 * c + 1]);
        }
        turn(p[0], p[1], kq, 4 + kq, w);
      };
      u32x4 w[2], nx[2];
      if (PIPE) make(0, w);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        if (!PIPE) make(r, w);
        else if (r + 1 < RT) make(r + 1, nx);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          char* const xp = row_ptr(r, h);
          if (prow < M - mw - (r * 16 + h * 8)) {
            if (full) *(u32x4*)xp = w[h];
            else
              for (int c = 0; c < N - nw - pchunk * 8; ++c) ((bf16_t*)xp)[c] = (bf16_t)(w[h][c >> 1] >> (16 * (c & 1)));
          }
        }
#pragma unroll
        for (int h = 0; h < 2 && PIPE; ++h) w[h] = nx[h];
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto plain_bf16 = [&](auto gelu_tag) {
      constexpr bool GELU = decltype(gelu_tag)::value;
      float bv[2][8];
      load_cols(bias, bv);
      bf16_t* const out = (bf16_t*)P.out;
      const int ldc = P.ldc;
      const uint32_t voff = (uint32_t)(prow * ldc + pchunk * 8) * 2u;
      store_bf16([&](int r, int j, float (&v)[8]) {
        raw(r, j, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          v[c] += bv[j][c];
          if constexpr (GELU) v[c] = gelu_tanh(v[c]);
        }
      }, [](float a, float b) { return pack2bf(a, b); },
      [&](int r, int h) { return (char*)(out + (size_t)(mw + r * 16 + h * 8) * ldc + nw) + voff; });
    };
    // fp32 results in units of 16 rows x 32 columns: plain, or added to what is there times the row's gate
    auto plain_f32 = [&](auto resid_tag) {
      constexpr bool RESID = decltype(resid_tag)::value;
      constexpr bool STATS = CONV;
      float bv[2][8];
      load_cols(bias, bv);
      const int nb = nw + pchunk * 4, ldc = P.ldc;       // my columns on the way out: nb + 32 j ... + 3
      float* const out = (float*)P.out;
      const uint32_t voff = (uint32_t)(prow * ldc + pchunk * 4) * 4u;
      auto row_at = [&](int u, int h) { return (char*)(out + (size_t)(mw + (u >> 1) * 16 + h * 8) * ldc + nw + 32 * (u & 1)) + voff; };
      auto row_in = [&](int u, int h) { return prow < M - mw - (u >> 1) * 16 - h * 8; };
      float cs[2][4], cq[2][4];                          // convolutions: their sums and sums of squares (see GemmProblem::stats)
      if constexpr (STATS) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int c = 0; c < 4; ++c) { cs[j][c] = 0.f; cq[j][c] = 0.f; }
      }
      // One gate vector for all rows of the wave (nearly always: a request has hundreds) is kept in registers.
      const float* const gate = RESID && !CONV ? P.gate : nullptr;
      const int* const rreq = P.row_req;
      const int gstride = P.gate_stride;
      bool one_gate = true;
      constexpr int RQ = (RT * 16 + 63) / 64;
      int rq[RQ];                                        // request of row 64 k + lane
      f32x4 gv[2] = {{1.f, 1.f, 1.f, 1.f}, {1.f, 1.f, 1.f, 1.f}};
      auto load_gate = [&](int req, int j) {
        f32x4 g;
        const float* gp = gate + (size_t)req * gstride + nb + 32 * j;
        if (nb + 32 * j + 4 <= N) {
#pragma unroll
          for (int c = 0; c < 4; ++c) g[c] = gp[c];
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) g[c] = nb + 32 * j + c < N ? gp[c] : 0.f;
        }
        return g;
      };
      if (RESID && gate) {
#pragma unroll
        for (int k = 0; k < RQ; ++k) {
          const int m = mw + k * 64 + ln;
          rq[k] = rreq ? rreq[m < M ? m : M - 1] : 0;
        }
        const int req0 = __builtin_amdgcn_readfirstlane(rq[0]);
        bool same = true;
#pragma unroll
        for (int k = 0; k < RQ; ++k) same = same && (rq[k] == req0 || k * 64 + ln >= RT * 16);
        one_gate = __builtin_amdgcn_ballot_w64(!same) == 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) gv[j] = load_gate(req0, j);
      }
      // What is there is loaded AHEAD units before it is used (the compiler may not move loads across the stores).
      constexpr int U = RT * 2;
      f32x4 xr[RESID ? 4 : 1][2], gr[2];
      // (rows of several requests: their gates, a unit ahead)
      auto load_gr = [&](int u) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int i = (u >> 1) * 16 + h * 8;
          gr[h] = load_gate(__shfl(rq[i >> 6], (i & 63) + prow), u & 1);
        }
      };
      auto load_x = [&](int u, f32x4 (&x)[2]) {
        if constexpr (RESID) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            x[h] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (row_in(u, h) && nb + 32 * (u & 1) + 4 <= N) x[h] = *(const f32x4*)row_at(u, h);
          }
        }
      };
      auto make = [&](int u, u32x4 (&w)[2]) {
        union { float f[8]; u32x4 q[2]; } v;
        raw(u >> 1, u & 1, v.f);
#pragma unroll
        for (int c = 0; c < 8; ++c) v.f[c] += bv[u & 1][c];
        turn(v.q[0], v.q[1], 2 * kq, 2 * kq + 1, w);
      };
      auto units = [&](auto one_tag) {
      constexpr bool ONE = decltype(one_tag)::value;
      constexpr int AHEAD = !RESID ? 1 : ONE && PIPE ? 4 : 2;
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) load_x(u, xr[u]);
      if (!ONE) load_gr(0);
      u32x4 w[2], nx[2];
      if (PIPE) make(0, w);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = u & 1, n = nb + 32 * j;
        if (!PIPE) make(u, w);
        else if (u + 1 < U) make(u + 1, nx);
        // (used here on every path: a load that some path leaves pending would be waited for in the next tile's loop)
        if constexpr (RESID) asm volatile("" :: "v"(xr[u % AHEAD][0]), "v"(xr[u % AHEAD][1]), "v"(gv[j]));
        if constexpr (RESID && !ONE) asm volatile("" :: "v"(gr[0]), "v"(gr[1]));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (row_in(u, h) && n < N) {
            f32x4 x4;
#pragma unroll
            for (int c = 0; c < 4; ++c) x4[c] = __uint_as_float(w[h][c]);
            float* xp = (float*)row_at(u, h);
            if constexpr (RESID) {
              const f32x4 g = ONE ? gv[j] : gr[h];
              if (n + 4 <= N) {
#pragma unroll
                for (int c = 0; c < 4; ++c) x4[c] = xr[u % AHEAD][h][c] + g[c] * x4[c];
              } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) x4[c] = n + c < N ? xp[c] + g[c] * x4[c] : 0.f;
              }
            }
            if (n + 4 <= N) *(f32x4*)xp = x4;
            else {
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (n + c < N) xp[c] = x4[c];
            }
            if constexpr (STATS) {
#pragma unroll
              for (int c = 0; c < 4; ++c) { cs[j][c] += x4[c]; cq[j][c] += x4[c] * x4[c]; }     // (columns past N are not written out)
            }
          }
        }
        if (u + AHEAD < U) load_x(u + AHEAD, xr[u % AHEAD]);
        if (!ONE && u + 1 < U) load_gr(u + 1);
#pragma unroll
        for (int h = 0; h < 2 && PIPE; ++h) w[h] = nx[h];
        __builtin_amdgcn_sched_barrier(0);
      }
      };
      // (two copies: loads of a path that the compiler thinks may be left pending are waited for in the next tile's loop)
      if (!RESID || CONV || one_gate) units(std::true_type{});
      else units(std::false_type{});
      if constexpr (STATS) {
        float* const stats = P.stats;
        if (stats) {      // partial[(tile row * WM + wm)][column][2]: rows of one wave of one tile
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
              for (int o = 8; o < 64; o <<= 1) { cs[j][c] += __shfl_xor(cs[j][c], o); cq[j][c] += __shfl_xor(cq[j][c], o); }
              const int n = nb + 32 * j + c;
              if (prow == 0 && n < N) *(f32x2*)(stats + ((size_t)(tm * WM + wm) * N + n) * 2) = f32x2{cs[j][c], cq[j][c]};
            }
        }
      }
    };
    // q/k columns of a QKV product: RMS norm per head, gain, rotary code, scale, scatter by row.  The wave's 64 columns are
    // one head (head_dim 64) or half of one (128: the two waves of a pair exchange their sums of squares).
    auto norm_rope = [&]() {
      Norm& Q = P.qk;
      const int head_dim = Q.head_dim, nq = Q.nq;
      const bool is_k = n0 >= nq;                        // (nq is a multiple of the tile's width)
      const int col0 = nw - (is_k ? nq : 0);             // first of the wave's columns in the q (k) range
      // destination rows of my rows 16 r + l16 (what is loaded here arrives under the sums)
      const int* const map = Q.dst_row;
      int dr[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) dr[r] = dest_row(map, mw + r * 16 + l16, M);
      float ss[RT];
      {
        float bv[2][8];
        load_cols(bias, bv);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          float s2 = 0.f;
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              const float v = acc[r][2 * j + (c >> 2)][c & 3] + bv[j][c];
              acc[r][2 * j + (c >> 2)][c & 3] = v;
              s2 += v * v;
            }
          s2 += __shfl_xor(s2, 16); s2 += __shfl_xor(s2, 32);
          ss[r] = s2;
        }
      }
      if (head_dim == 128) {
        float* mine = (float*)patch;
        const float* other = (const float*)(smem + NS * STAGE + (wave ^ 1) * 2048);
        if (kq == 0) {
#pragma unroll
          for (int r = 0; r < RT; ++r) mine[r * 16 + l16] = ss[r];
        }
        wait_vm<63, true>();
        wg_barrier();
#pragma unroll
        for (int r = 0; r < RT; ++r) ss[r] += other[r * 16 + l16];
        wait_vm<63, true>();
        wg_barrier();                                    // (the patches are written again from here on)
      }
      const float inv_dh = 1.0f / (float)head_dim, osc = is_k ? 1.0f : Q.qscale;
#pragma unroll
      for (int r = 0; r < RT; ++r) ss[r] = rsqrtf(ss[r] * inv_dh + 1e-6f) * osc;
      const int hc = (col0 & (head_dim - 1)) + kq * 8;   // my first column inside the head
      float gv[2][8];
      {
        const float* gain = is_k ? Q.kgain : Q.qgain;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int c = 0; c < 8; ++c) gv[j][c] = gain[hc + j * 32 + c];
      }
      const float2* const rope = Q.rope;
      const int half = head_dim >> 1;
      // rotary pairs of row tile r, a tile ahead
      f32x4 rc[2][2];
      auto load_rope = [&](int r) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 (&c)[2] = rc[j];
          c[0] = c[1] = f32x4{1.f, 0.f, 1.f, 0.f};       // (cos, sin)
          if (rope) {
            const f32x4* rp = (const f32x4*)(rope + (size_t)dr[r] * half + (hc >> 1) + 16 * j);
            c[0] = rp[0]; c[1] = rp[1];
          }
        }
      };
      load_rope(0);
      auto value = [&](int r, int j, float (&v)[8]) {
        const f32x4 c0 = rc[j][0], c1 = rc[j][1];
        const float cs[8] = {c0[0], c0[1], c0[2], c0[3], c1[0], c1[1], c1[2], c1[3]};
        raw(r, j, v);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float a = v[2 * p] * ss[r] * gv[j][2 * p], b = v[2 * p + 1] * ss[r] * gv[j][2 * p + 1];
          v[2 * p] = a * cs[2 * p] - b * cs[2 * p + 1];
          v[2 * p + 1] = a * cs[2 * p + 1] + b * cs[2 * p];
        }
        if (j == 1 && r + 1 < RT) load_rope(r + 1);
      };
      const bool f16 = Q.f16 != 0;
      bf16_t* const out = is_k ? Q.ko : Q.qo;
      const int ldo = Q.ldo;
      store_bf16(value, [&](float a, float b) { return f16 ? pack2h(a, b) : pack2bf(a, b); },
                 [&](int r, int h) { return (char*)(out + (size_t)__shfl(dr[r], h * 8 + prow) * ldo + col0 + pchunk * 8); });
    };
    // Value columns written transposed: acc[2 i][c], acc[2 i + 1][c] hold rows 32 i + 8 kq + 0..7 of column 16 c + l16.  Units of
    // 32 rows x 32 columns; a lane writes 8 rows of a column as one 16-byte piece (at any 2-byte offset: a request's
    // image rows follow its text rows) when the 32 rows are neighbours in the transposed matrix, else element by element.
    auto transposed = [&]() {
      Norm& Q = P.qk;
      typedef u32x4 u32x4_any __attribute__((aligned(2)));
      const int nv0 = nw - (Q.nq + Q.nk), ldvt = Q.ldvt;
      const int* const map = Q.vt_col;
      bf16_t* const vt_out = Q.vt;
      float bv[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) bv[c] = bias && nw + c * 16 + l16 < N ? bias[nw + c * 16 + l16] : 0.f;
      const int fr = ln >> 2, fc = ln & 3;               // my column (and the one 16 on) and piece when a unit is read back
      auto at = [&](int f, int chunk) { return patch + f * 64 + ((chunk ^ ((f >> 2) & 3)) << 4); };
      const uint32_t voff = (uint32_t)(fr * ldvt + fc * 8) * 2u;
#pragma unroll
      for (int i = 0; i < RT / 2; ++i) {
        const int mb = mw + i * 32;                      // first row of the unit
        bool consec = mb + 32 <= M;
        int cb = 0;
        if (consec) {
          cb = map[mb];
          consec = map[mb + 31] == cb + 31;
        }
        int col[8];                                      // else the columns of my piece's rows, fetched together and
        if (!consec) {                                   // waited for here (one by one they cost a memory latency each)
#pragma unroll
          for (int e = 0; e < 8; ++e) col[e] = mb + fc * 8 + e < M ? map[mb + fc * 8 + e] : -1;
          asm volatile("" :: "v"(col[0]), "v"(col[1]), "v"(col[2]), "v"(col[3]), "v"(col[4]), "v"(col[5]), "v"(col[6]), "v"(col[7]));
        }
#pragma unroll
        for (int cp = 0; cp < 2; ++cp) {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int c = cp * 2 + q;
            const f32x4 t0 = acc[2 * i][c], t1 = acc[2 * i + 1][c];
            const u32x4 w = {pack2bf(t0[0] + bv[c], t0[1] + bv[c]), pack2bf(t0[2] + bv[c], t0[3] + bv[c]),
                             pack2bf(t1[0] + bv[c], t1[1] + bv[c]), pack2bf(t1[2] + bv[c], t1[3] + bv[c])};
            *(u32x4*)at(q * 16 + l16, kq) = w;
          }
          asm volatile("" ::: "memory");
          u32x4 w[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) w[h] = *(const u32x4*)at(h * 16 + fr, fc);
          asm volatile("" ::: "memory");
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int f = cp * 32 + h * 16;
            if (fr >= N - nw - f) continue;
            if (consec) *(u32x4_any*)((char*)(vt_out + (size_t)(nv0 + f) * ldvt + cb) + voff) = w[h];
            else {
              bf16_t* dst = vt_out + (size_t)(nv0 + f + fr) * ldvt;
#pragma unroll
              for (int e = 0; e < 8; e += 2) {           // (pairs where two rows are neighbours at an even column)
                if (col[e + 1] == col[e] + 1 && (col[e] & 1) == 0) *(uint32_t*)(dst + col[e]) = w[h][e >> 1];
                else {
                  if (col[e] >= 0) dst[col[e]] = (bf16_t)w[h][e >> 1];
                  if (col[e + 1] >= 0) dst[col[e + 1]] = (bf16_t)(w[h][e >> 1] >> 16);
                }
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    // gated pair: the wave's 64 columns are 32 of the gate (acc[.][0, 1]) and the same 32 of the values (acc[.][2, 3])
    auto gated = [&]() {
      const int n_end = N >> 1, nw2 = nw >> 1;
      bf16_t* const out = (bf16_t*)P.out;
      const int ldc = P.ldc, fr = ln >> 2, fc = ln & 3;  // my row (and the one 16 on) and piece when 32 rows are read back
      auto at = [&](int f, int chunk) { return patch + f * 64 + ((chunk ^ ((f >> 2) & 3)) << 4); };
      const bool full = nw2 + fc * 8 + 8 <= n_end;
      const uint32_t voff = (uint32_t)(fr * ldc + fc * 8) * 2u;
#pragma unroll
      for (int i = 0; i < RT / 2; ++i) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = 2 * i + q;
          float v[8], u[8];
          raw(r, 0, v); raw(r, 1, u);
          u32x4 w;
#pragma unroll
          for (int c = 0; c < 4; ++c) w[c] = pack2bf(gelu_tanh(v[2 * c]) * u[2 * c], gelu_tanh(v[2 * c + 1]) * u[2 * c + 1]);
          *(u32x4*)at(q * 16 + l16, kq) = w;
        }
        asm volatile("" ::: "memory");
        u32x4 w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) w[h] = *(const u32x4*)at(h * 16 + fr, fc);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = i * 32 + h * 16;
          char* const xp = (char*)(out + (size_t)(mw + k) * ldc + nw2) + voff;
          if (fr < M - mw - k) {
            if (full) *(u32x4*)xp = w[h];
            else
              for (int c = 0; c < n_end - nw2 - fc * 8; ++c) ((bf16_t*)xp)[c] = (bf16_t)(w[h][c >> 1] >> (16 * (c & 1)));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if constexpr (!CONV) {
      if (kind == OUT_GEGLU) { gated(); return; }
      if (kind == OUT_QKNORM && n0 < P.qk.nq + P.qk.nk) { norm_rope(); return; }
      if (vt) { transposed(); return; }
      if (kind == OUT_GELU_BF16) { plain_bf16(std::true_type{}); return; }
      if (kind == OUT_BF16 || kind == OUT_QKNORM) { plain_bf16(std::false_type{}); return; }
    }
    if (kind == OUT_F32) plain_f32(std::false_type{});
    else plain_f32(std::true_type{});
  };

  // ---- all my tiles ------------------------------------------------------------------------------------------
  auto start = [&]() {
    aim(ld_t);
    issue_b(0); issue_a(0, A_FIRST, A_END);
    advance();
    issue_b(1); issue_a(1, A_FIRST, A_END);
    wait_vm<LPS, false>();
    wg_barrier();
  };
  if (STREAM) start();
  for (int t = blockIdx.x >> 3; t < t_count; t += t_step) {
    if (!STREAM) {
      ld_t = t; stage = 0;
      start();
    }
    const int bid = t_first + t;
    Problem& P = problem(bid);
    int tm, tn;
    tile_coords(P, bid - P.tile_start, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const bool vt = !CONV && (P.out_kind == OUT_VT || (P.out_kind == OUT_QKNORM && P.qk.vt && n0 >= P.qk.nq + P.qk.nk));
    if (!CONV && vt) run(std::true_type{}, P.K / BKT);
    else run(std::false_type{}, P.K / BKT);
    if (!STREAM) {                           // the redundant tail loads, before the stages are filled again
      wait_vm<0, true>();
      wg_barrier();
    }
    epilogue(P, tm, m0, n0, vt);
  }
  wait_vm<0, true>();                        // drain the redundant tail loads before LDS is released
}

// N shares, STRIDE floats apart, fetched together and added in their order.
template <int N, int STRIDE>
__device__ __forceinline__ void add_shares(f32x4& acc, const float* pc) {
  f32x4 t[N];
#pragma unroll
  for (int u = 0; u < N; ++u) t[u] = *(const f32x4*)(pc + (size_t)u * STRIDE);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] += t[u][c];
}
// The shares of one float4 of a split product, STRIDE floats apart, added in their order.  Eight loads are in flight and none
// waits alone behind them: with four, and the rest one by one, 16 shares cost six memory latencies, with eight two (32 tokens
// through the encoder 2985 -> 2962 us).  The last ones have a branch for their number: a condition for each load costs
// more than it saves at few shares (see splitk_reduce_kernel).
template <int STRIDE>
__device__ __forceinline__ f32x4 sum_shares(const float* pc, int splits) {
  f32x4 acc = *(const f32x4*)pc;
  int left = splits - 1;
  for (pc += STRIDE; left >= 8; left -= 8, pc += 8 * STRIDE) add_shares<8, STRIDE>(acc, pc);
  switch (left) {
    case 7: add_shares<7, STRIDE>(acc, pc); break;
    case 6: add_shares<6, STRIDE>(acc, pc); break;
    case 5: add_shares<5, STRIDE>(acc, pc); break;
    case 4: add_shares<4, STRIDE>(acc, pc); break;
    case 3: add_shares<3, STRIDE>(acc, pc); break;
    case 2: add_shares<2, STRIDE>(acc, pc); break;
    case 1: add_shares<1, STRIDE>(acc, pc); break;
  }
  return acc;
}

// Second half of a split-K product: sums the `splits` partial tiles in fixed order (so the
// result does not depend on which workgroup finished first) and applies the epilogue.  One
// thread per float4 of the chunk layout written above: 4 consecutive rows of one column, the
// 32 lanes of a half-wave on 32 consecutive columns.
//   GEGLU: a gated pair's reduction covers the tiles of the gate and adds up both; VT: some problem is OUT_VT, where 4 rows
// of a column are 4 neighbours of a row of the transposed matrix.  Both have instantiations of their own: in one kernel for all, with a
// condition for each share, 6 and 7 shares of 235 rows took 7.75 us, 2 shares of 515 rows 9.6; now 7.35 and 9.4 (before
// these forms were here 7.25 and 9.15).
template <int BM, int BN, int WM, int WN, bool GEGLU, bool VT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmBatch batch) {
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int QPT = BM * BN / 4;                 // float4s per tile
  constexpr int BPT = QPT / 256;                   // workgroups per tile
  const int tile = blockIdx.x / BPT;
  const int q = (blockIdx.x % BPT) * 256 + threadIdx.x;
  GemmProblem P = batch.p[0];
  if (batch.n > 1 && tile >= batch.p[1].tile_start) P = batch.p[1];
  if (batch.n > 2 && tile >= batch.p[2].tile_start) P = batch.p[2];
  int tm, tn;
  tile_coords(P, tile - P.tile_start, tm, tn);
  const int lane = q & 63, g = (q >> 6) & 3, j = (q >> 8) % TN, i = (q >> 8) / TN % TM, wave = (q >> 8) / (TN * TM);
  const int wm = wave / WN, wn = wave % WN;
  const int n = tn * BN + wn * (BN / WN) + j * 32 + (lane & 31);
  const int mrow = tm * BM + wm * (BM / WM) + i * 32 + 8 * g + 4 * (lane >> 5);
  auto sum = [&](int t) {
    const float* pc = batch.partial + (size_t)t * batch.splits * (BM * BN) + (size_t)q * 4;
    return sum_shares<BM * BN>(pc, batch.splits);
  };
  f32x4 acc = sum(tile);
  if constexpr (GEGLU) {
    const f32x4 up = sum(tile + batch.p[1].tile_start);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = gelu_tanh(acc[c]) * up[c];
  }
  if (VT && P.out_kind == OUT_VT) {
    if (n >= P.N) return;
    const float bias = P.bias ? P.bias[n] : 0.f;
    bf16_t* dst = P.qk.vt + (size_t)n * P.qk.ldvt;
    int col[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) col[c] = mrow + c < P.M ? P.qk.vt_col[mrow + c] : -1;
    if (col[3] == col[0] + 3 && col[1] == col[0] + 1 && col[2] == col[0] + 2 && col[0] >= 0 && (col[0] & 3) == 0) {
      *(uint2*)(dst + col[0]) = make_uint2(pack2bf(acc[0] + bias, acc[1] + bias), pack2bf(acc[2] + bias, acc[3] + bias));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (col[c] >= 0) dst[col[c]] = f2bf(acc[c] + bias);
    }
    return;
  }
  float cs = 0.f, cq = 0.f;               // sum and sum of squares of the values stored, this thread's rows of the column
  if (n < P.N) {
    const float bias = P.bias ? P.bias[n] : 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int m = mrow + c;
      if (m >= P.M) continue;
      float v = acc[c] + bias;
      const size_t o = (size_t)m * P.ldc + n;
      if (P.out_kind == OUT_RESID_F32) {
        const float gt = P.gate ? P.gate[(size_t)(P.row_req ? P.row_req[m] : 0) * P.gate_stride + n] : 1.f;
        v = ((float*)P.out)[o] + gt * v;
        ((float*)P.out)[o] = v;
      } else if (P.out_kind == OUT_F32) {
        ((float*)P.out)[o] = v;
      } else {
        ((bf16_t*)P.out)[o] = f2bf(P.out_kind == OUT_GELU_BF16 ? gelu_tanh(v) : v);
      }
      cs += v; cq += v * v;
    }
  }
  if (P.stats) {                          // a workgroup holds one 32x32 tile: a chunk of 32 rows
    __shared__ float red[4][32][2];
    cs += __shfl_xor(cs, 32); cq += __shfl_xor(cq, 32);
    if (lane < 32) { red[g][lane][0] = cs; red[g][lane][1] = cq; }
    __syncthreads();
    if (threadIdx.x < 32 && n < P.N) {
      float* sp = P.stats + ((size_t)((tm * BM + wm * (BM / WM)) / 32 + i) * P.N + n) * 2;
#pragma unroll
      for (int c = 0; c < 2; ++c) sp[c] = (red[0][lane][c] + red[1][lane][c]) + (red[2][lane][c] + red[3][lane][c]);
    }
  }
}

// The reduction of a residual product with the layer norm that follows it: a workgroup takes four whole rows (of each
// partial tile's float4s, four rows of a column), 512 columns at a time, writes the residual rows and, from registers,
// their modulated norm.  What counts here is the number of launches: apart, the reduction of 410 rows of 1536 columns in 5
// shares takes 7.5 us and the norm 5, both at the latency of a launch; together 2.6 us less.
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(512) void splitk_reduce_ln_kernel(const GemmBatch batch) {
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int MAXP = 3;                          // up to 1536 columns
  __shared__ float red[2][8][4];
  int row4 = blockIdx.x;                           // my four rows: 4 row4 ... of the problem
  GemmProblem P = batch.p[0];
  if (batch.n > 1 && row4 >= (P.M + 3) / 4) { row4 -= (P.M + 3) / 4; P = batch.p[1]; }
  const int tid = threadIdx.x, wv = tid >> 6;
  const int m0 = row4 * 4, d = P.N;
  const int tm = m0 / BM, r = m0 % BM;
  const int i = r % (BM / WM) / 32, g = (r & 31) >> 3, half = (r >> 2) & 1, wm = r / (BM / WM);
  const int first = tm & ~7, gsz = P.tiles_m - first < 8 ? P.tiles_m - first : 8;
  const int tile0 = P.tile_start + first * P.tiles_n + (tm - first);      // (tile_coords() backwards; + tn * gsz)
  int mr[4];
  const float* gp[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    mr[c] = m0 + c < P.M ? m0 + c : P.M - 1;       // rows past the end repeat the last one and are not stored
    const size_t req = (size_t)(P.row_req ? P.row_req[mr[c]] : 0) * P.gate_stride;
    gp[c] = P.gate ? P.gate + req : nullptr;
  }
  float x[MAXP][4], s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    const int n = p * 512 + tid;
    if (n >= d) { x[p][0] = x[p][1] = x[p][2] = x[p][3] = 0.f; continue; }
    const int tn = n / BN, cc = n % BN, wn = cc / (BN / WN), j = cc % (BN / WN) / 32;
    const int q = ((((wm * WN + wn) * TM + i) * TN + j) * 4 + g) * 64 + half * 32 + (cc & 31);
    const float* pc = batch.partial + (size_t)(tile0 + tn * gsz) * batch.splits * (BM * BN) + (size_t)q * 4;
    const float bias = P.bias ? P.bias[n] : 0.f;
    float x0[4], gt[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x0[c] = ((const float*)P.out)[(size_t)mr[c] * P.ldc + n];
      gt[c] = gp[c] ? gp[c][n] : 1.f;
    }
    // (the order of sum_shares(); several columns a thread have enough loads in flight, whose conditions cost 0.6 % of a step)
    f32x4 acc = *(const f32x4*)pc;
    int k = 1;
    for (; k + 3 < batch.splits; k += 4) {
      f32x4 t4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t4[u] = *(const f32x4*)(pc + (size_t)(k + u) * (BM * BN));
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] += t4[u][c];
    }
    for (; k < batch.splits; ++k) {
      const f32x4 t4 = *(const f32x4*)(pc + (size_t)k * (BM * BN));
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] += t4[c];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[p][c] = x0[c] + gt[c] * (acc[c] + bias);
      s[c] += x[p][c];
    }
  }
  auto block_sum = [&](float (&v)[4], float (&buf)[8][4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v[c] += __shfl_xor(v[c], o);
    if ((tid & 63) == 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c) buf[wv][c] = v[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      v[c] = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) v[c] += buf[w][c];
    }
  };
  block_sum(s, red[0]);
  float qs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 4; ++c) s[c] /= (float)d;
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    const int n = p * 512 + tid;
    if (n >= d) continue;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (m0 + c < P.M) ((float*)P.out)[(size_t)mr[c] * P.ldc + n] = x[p][c];
      x[p][c] -= s[c];
      qs[c] += x[p][c] * x[p][c];
    }
  }
  block_sum(qs, red[1]);
#pragma unroll
  for (int c = 0; c < 4; ++c) qs[c] = rsqrtf(qs[c] / (float)d + 1e-6f);
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    const int n = p * 512 + tid;
    if (n >= d) continue;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (m0 + c >= P.M) continue;
      const size_t mo = (size_t)(P.row_req ? P.row_req[mr[c]] : 0) * P.gate_stride + n;
      P.ln_y[(size_t)mr[c] * d + n] = f2bf(x[p][c] * qs[c] * (1.f + P.ln_scale[mo]) + P.ln_shift[mo]);
    }
  }
}

// tiles of the whole batch, numbered through
static int count_tiles(GemmBatch& b, int bm, int bn) {
  int total = 0;
  for (int i = 0; i < b.n; ++i) {
    GemmProblem& p = b.p[i];
    p.tiles_m = (p.M + bm - 1) / bm;
    p.tiles_n = (p.N + bn - 1) / bn;
    p.tile_start = total;
    total += p.tiles_m * p.tiles_n;
  }
  return b.total_tiles = total;
}

template <int BM, int BN, int WM, int WN, int NS, bool CONV = false>
static void launch8_t(hipStream_t s, GemmBatch& b) {
  const int total = count_tiles(b, BM, BN);
  if (total == 0) return;
  constexpr int lds = NS * (BM + BN) * 128 + 8 * 2048;      // the ring and a patch per wave
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  auto kern = gemm8_kernel<BM, BN, WM, WN, NS, CONV>;
  static std::atomic<unsigned> seen{0};
  if (first_use_on_device(seen))
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  // One workgroup per CU.  Its tiles are fixed: beside other streams a workgroup whose CU is held starts late, and its tiles with it (a
  // stage in a stream beside small calls of another: 0.82 to 0.98 of the time of one after the other, with a workgroup per tile
  // 0.83 to 0.96; no pair of stages takes longer than it did).
  hipLaunchKernelGGL(kern, dim3(total < 256 ? total : 256), dim3(512), lds, s, b);
}

template <int BM, int BN, int WM, int WN, int BKT, int NS, int MODE = 0, bool CONV = false>
static void launch_t(hipStream_t s, GemmBatch& b) {
  const int total = count_tiles(b, BM, BN);
  if (total == 0) return;
  size_t lds = (size_t)NS * (BM + BN) * BKT * 2;
  auto kern = gemm_kernel<BM, BN, WM, WN, BKT, NS, MODE, CONV>;
  static std::atomic<unsigned> seen{0};
  if (first_use_on_device(seen))
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (MODE == 4) {
    hipLaunchKernelGGL(kern, dim3(total * b.splits), dim3(WM * WN * 64), lds, s, b);
    // The norm that follows as well, from 96 workgroups of four rows on and up to 1536 columns: there it takes 2 % off a step (eight
    // blocks of 1536 columns: 410 rows 1122 -> 1101 us, 700 rows 1209 -> 1184, 1178 rows 1542 -> 1513).  Below that too few
    // workgroups read the partial sums (80 rows 817 -> 826 us, 272 rows 974 -> 976), and with 3072 columns a workgroup
    // reads twice as many (256 rows 1278 -> 1295 us, 640 rows 1633 -> 1632).  (The smaller tiles serve problems of at most 128
    // rows, two of which are 64 workgroups.)
    bool ln = BM == 128 && !b.geglu && b.n <= 2;
    int rows = 0;
    for (int i = 0; i < b.n; ++i) {
      ln = ln && b.p[i].ln_y && b.p[i].out_kind == OUT_RESID_F32 && b.p[i].N <= 1536;
      rows += (b.p[i].M + 3) / 4;
    }
    ln = ln && rows >= 96;
    b.ln_done = ln;
    if constexpr (BM == 128)
      if (ln) hipLaunchKernelGGL((splitk_reduce_ln_kernel<BM, BN, WM, WN>), dim3(rows), dim3(512), 0, s, b);
    bool vt = false;
    for (int i = 0; i < b.n; ++i) vt = vt || b.p[i].out_kind == OUT_VT;
    const dim3 grid((b.geglu ? total / 2 : total) * (BM * BN / 1024));
    if (b.geglu) hipLaunchKernelGGL((splitk_reduce_kernel<BM, BN, WM, WN, true, false>), grid, dim3(256), 0, s, b);
    else if (vt) hipLaunchKernelGGL((splitk_reduce_kernel<BM, BN, WM, WN, false, true>), grid, dim3(256), 0, s, b);
    else if (!ln) hipLaunchKernelGGL((splitk_reduce_kernel<BM, BN, WM, WN, false, false>), grid, dim3(256), 0, s, b);
  } else {
    hipLaunchKernelGGL(kern, dim3(total), dim3(WM * WN * 64), lds, s, b);
  }
}

// variant codes: BM*1000 + BN, plus
//   +1000000  8 waves (2x4) instead of 4 (2x2); 1320256: 320x256 with 8 waves
//   +10000000 k-slab 32 with a 4-stage ring, +20000000 k-slab 32 with a 5-stage ring
//             (default: k-slab 64, 2 stages)
//   31256128 / 32256128 / 31128256  256x128 (4 waves / 8 waves) and 128x256 with a 3-stage ring
//   30128128  128x128, k-slab 64, 4-stage ring (one workgroup per CU: for grids below 256 tiles)
//   30128064 / 33128064  128x64 (4 waves of 32x64), 6- / 3-stage ring;  30064128 / 32064128  64x128 (4 waves of 64x32 / 32x64), 6-stage ring
//   40128128  the same as split-K over b.splits shares of K plus the reduction kernel
//   30032128 / 30064064  32x128 (4 waves of 32x32) and 64x64 (2 waves of 32x64), two workgroups per CU, 4- / 5-stage ring;
//   40032128 / 40064064  the same as split-K
// Few rows: what counts is how many bytes are in flight and how long the chain of slabs of one workgroup is.
// Tiles of 32x128 (up to 64 rows) and 64x64 (up to 128) take 80 KB of LDS, so two workgroups share a CU and K is
// split over up to 512 of them.  Where one row of tiles covers a problem they take 0.63 to 0.99 of the 128-row tiles'
// time (32 rows: 12288 x 4096 25.9 against 31.4 us, 5120 x 13824 34.5 against 36.1).  Under two rows of tiles every
// slab of W is fetched into LDS twice, and large weights lose more by that than the shorter chain gives.  At 64 rows:
// 4096 x 4096 16.6 against 18.8 us, 6144 x 3072 17.5 against 17.9, 5120 x 5120 21.7 against 20.8, 3072 x 12288 27.5
// against 25.0, 5120 x 13824 41.3 against 35.3; with fewer than four shares of K also 12288 x 1536, 19.0 against 18.1.
// At 96 rows: 1536 x 6144 15.8 against 16.0, 3072 x 3072 16.5 against 17.2, 6144 x 3072 20.7 against 18.1,
// 5120 x 13824 49.5 against 36.9.  Hence the limits on the weights under two rows of tiles: 21 million at 32x128 with at
// least four shares (up to 128 tiles), 17 million with fewer and in the q/k-norm form, which is never split (two streams of
// 4608 x 1536 at 64 and 100 rows 15.0 against 16.8 us), 10.5 million at 64x64.  Beyond 256 tiles nothing is split and
// a second round begins (3072-wide streams of 64 and 16 rows, N = 12288: 46 against 37 us).  0: not such a launch.
static int small_m_tile(GemmBatch& b) {
  int max_m = 0, min_nk = 1 << 30;
  long long t128 = 0;
  bool qk = false;
  for (int i = 0; i < b.n; ++i) {
    const GemmProblem& p = b.p[i];
    if (p.M <= 0 || p.N <= 0) continue;
    if (p.conv_w > 0 || (p.out_kind == OUT_QKNORM && p.qk.head_dim > 64)) return 0;
    qk = qk || p.out_kind == OUT_QKNORM;
    max_m = p.M > max_m ? p.M : max_m;
    min_nk = p.K / 64 < min_nk ? p.K / 64 : min_nk;
    t128 += (long long)((p.M + 127) / 128) * ((p.N + 127) / 128);
  }
  if (max_m == 0 || max_m > 128 || t128 > 256) return 0;
  const bool rows32 = max_m <= 64 && !qk;       // (the q/k-norm epilogue needs waves of 64 columns, the reduction has none)
  const int bm = rows32 ? 32 : 64, bn = rows32 ? 128 : 64;
  long long t = 0, twice = 0;                   // tiles; weights under two rows of them
  for (int i = 0; i < b.n; ++i) {
    const GemmProblem& p = b.p[i];
    if (p.M <= 0 || p.N <= 0) continue;
    t += (long long)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn);
    if (p.M > bm) twice += (long long)p.N * p.K;
  }
  if (t > 256 || twice > (rows32 ? (t <= 128 ? 5 << 22 : 1 << 24) : qk ? 1 << 24 : 5 << 21)) return 0;
  long long sp = qk || !b.partial ? 1 : 512 / t;
  if (sp > min_nk / 4) sp = min_nk / 4;
  const long long cap = (long long)(b.partial_bytes / (bm * bn * 4)) / t;
  if (sp > cap) sp = cap;
  if (sp < 2) return rows32 ? 30032128 : 30064064;
  b.splits = (int)sp;
  return rows32 ? 40032128 : 40064064;
}

int choose_tile(GemmBatch& b, int force_tile) {
  // Tile choice.  The 256x256 tile (8 waves) halves the L2->LDS traffic per flop of the 128x128
  // tile and takes 0.71 to 0.74 of its time where rounds are full (bf16 results, 8192^3 709 against 964 us,
  // 32760 x 5120 x 5120 1177 against 1605), but one workgroup fills a CU, so its grid runs
  // in rounds of 256 tiles: use it from one full round on, unless the last round would hold only
  // a few tiles (a partly filled last round runs faster than a full one, lone tiles see less
  // contention; 4250 x 4608 x 1536, 306 tiles: 71.1 us against 71.6 as 1224 of 128x128); otherwise the
  // 128x128 tile (three workgroups per CU, finer granularity).  The thresholds were set when every wave
  // interleaved its reads and products; the two-group loop has made the 8-wave tiles 6 to 17 % faster since, and
  // a call that they keep on the 128x128 tile is as fast as it was.
  int tile = force_tile;
  if (tile > 40000000 && (!b.partial || b.splits < 1)) tile -= 10000000;   // no scratch: no split
  if (tile < 40000000) b.splits = 1;
  if (!tile) tile = small_m_tile(b);
  if (!tile) {
    // Few tiles (small M): a lone tile's k-loop runs at memory latency per slab, so keep three
    // slabs in flight (4-stage ring, one workgroup per CU) and, when K is long enough, split it
    // over up to 256 workgroups.
    long long t128 = 0;
    int min_nk = 1 << 30;
    for (int i = 0; i < b.n; ++i) {
      if (b.p[i].M <= 0 || b.p[i].N <= 0) continue;
      t128 += (long long)((b.p[i].M + 127) / 128) * ((b.p[i].N + 127) / 128);
      min_nk = b.p[i].K / 64 < min_nk ? b.p[i].K / 64 : min_nk;
    }
    if (t128 > 0 && t128 <= 256) {
      long long sp = 256 / t128;
      if (sp > min_nk / 4) sp = min_nk / 4;
      const long long cap = (long long)(b.partial_bytes / (128 * 128 * 4)) / t128;
      if (sp > cap) sp = cap;
      bool qk = false;                       // the reduction kernel has no q/k-norm epilogue
      // (A video's convolutions are left unsplit as well: their shares of K would follow the frame count, on top of what
      // does already, the 1x1 products' shares and the tile height, which is that of the group norm's partial sums.  The
      // first frames of a narrow video, tested to keep their bits when one is added, would move with it.)
      for (int i = 0; i < b.n; ++i) qk = qk || b.p[i].out_kind == OUT_QKNORM || (b.p[i].conv_w > 0 && b.p[i].conv_kt == 3);
      if (b.partial && sp >= 2 && !qk) { b.splits = (int)sp; tile = 40128128; }
      else {
        // no split (q/k-norm epilogue, or K too short): 128x64 tiles with a 6-stage ring when twice the
        // workgroups still fit one round: these launches run at memory latency, and twice as many CUs with
        // more bytes in flight each fetch the weights faster (108 -> 216 workgroups: 17.4 -> 13.2 us)
        long long t64 = 0;
        for (int i = 0; i < b.n; ++i)
          if (b.p[i].M > 0 && b.p[i].N > 0) t64 += (long long)((b.p[i].M + 127) / 128) * ((b.p[i].N + 63) / 64);
        bool narrow_ok = true;        // not for convolutions; a 128-wide head must lie inside one workgroup's columns
        for (int i = 0; i < b.n; ++i)
          narrow_ok = narrow_ok && b.p[i].conv_w <= 0 && !(b.p[i].out_kind == OUT_QKNORM && b.p[i].qk.head_dim > 64);
        tile = (t64 <= 256 && narrow_ok) ? 30128064 : 30128128;
        if (tile == 30128128) {
          // ... or 64-row tiles when that gives more workgroups in one round, with the q/k norm in waves of 32 x 64: two
          // streams of 256 and 154 rows, N = 4608: 252 workgroups instead of 144, a step of eight blocks 1101 -> 1058 us
          long long t6 = 0;
          bool plain = true;
          for (int i = 0; i < b.n; ++i) {
            if (b.p[i].M > 0 && b.p[i].N > 0) t6 += (long long)((b.p[i].M + 63) / 64) * ((b.p[i].N + 127) / 128);
            plain = plain && b.p[i].conv_w <= 0;
          }
          if (plain && t6 <= 256 && t6 > t128) tile = qk ? 32064128 : 30064128;
        }
      }
    }
  }
  if (!tile) {
    // One round of 256x128 tiles (8 waves, 3-stage ring) when that fits the chip and K is not short:
    // a workgroup per CU with two slabs in flight, against 1.6 128x128 workgroups per CU (4250 rows, N = 1536:
    // 74 against 85 us at K = 6144, 24.1 against 27.1 at K = 1536; a 3x3 convolution of 16384 pixels, 512 channels:
    // 67 against 75).
    long long t21 = 0;
    int min_k = 1 << 30;
    bool plain = true;
    for (int i = 0; i < b.n; ++i) {
      if (b.p[i].M <= 0 || b.p[i].N <= 0) continue;
      t21 += (long long)((b.p[i].M + 255) / 256) * ((b.p[i].N + 127) / 128);
      min_k = b.p[i].K < min_k ? b.p[i].K : min_k;
      plain = plain && b.p[i].out_kind != OUT_QKNORM;
    }
    if (plain && t21 > 128 && t21 <= 256 && min_k >= 1536) tile = 32256128;
  }
  if (!tile) {
    int max_n = 0;
    for (int i = 0; i < b.n; ++i)
      if (b.p[i].M > 0 && b.p[i].N > max_n) max_n = b.p[i].N;
    // half or more of a 256-wide tile would be padding; convolutions take the 8-wave 256x128 tile from one round on
    if (max_n <= 128) {
      long long t21 = 0;
      bool all_conv = b.n > 0;
      for (int i = 0; i < b.n; ++i) {
        all_conv = all_conv && b.p[i].conv_w > 0;
        if (b.p[i].M > 0) t21 += (b.p[i].M + 255) / 256;
      }
      tile = all_conv && t21 >= 256 ? 32256128 : 128128;
    }
  }
  if (!tile) {
    long long t256 = 0;
    for (int i = 0; i < b.n; ++i)
      t256 += (long long)((b.p[i].M + 255) / 256) * ((b.p[i].N + 255) / 256);
    const long long rem = t256 % 256;
    tile = (t256 >= 1024 || (t256 >= 256 && (rem == 0 || rem >= 64))) ? 1256256 : 128128;
    // Below one round of 256x256 tiles: a round of them does the work of two rounds of 128x128 pairs in about
    // 1.42 times the time of one, so the big tile wins whenever the small one needs two rounds or more of its
    // 512 slots (216 tiles of 256x256 against 864 of 128x128 at 4608 x 3072 x 15360: 292 against 411 us).
    if (tile == 128128 && t256 < 256) {
      long long t128 = 0;
      for (int i = 0; i < b.n; ++i)
        t128 += (long long)((b.p[i].M + 127) / 128) * ((b.p[i].N + 127) / 128);
      if (100 * ((t128 + 511) / 512) > 142) tile = 1256256;      // (t256 < 256: one round of the big tile)
    }
    // A 320-row tile when it saves rounds: the 4250-row QKV product of the 1024^2 request is 306 tiles of
    // 256x256 (a second round for 50 tiles) but 252 of 320x256, one round of tiles 1.25 times as long (52 us
    // against 71 us with 128x128 and with 256x256 tiles); 864 tiles (4 rounds) against 720 (3 rounds x 1.25):
    // 252 against 267 us at 4608 x 12288 x 3072.  Per unit of work it is 3 to 12 % slower (18384 x 6144 x 1536 279
    // against 271 us, 8192^3 797 against 709), of which the rule, rounds alone, has 5 % as its margin.
    bool any_conv = false;                  // (convolutions have no 320-row instantiation)
    for (int i = 0; i < b.n; ++i) any_conv = any_conv || b.p[i].conv_w > 0;
    if (t256 > 256 && !any_conv) {
      long long t320 = 0;
      for (int i = 0; i < b.n; ++i)
        t320 += (long long)((b.p[i].M + 319) / 320) * ((b.p[i].N + 255) / 256);
      const long long r256 = (t256 + 255) / 256, r320 = (t320 + 255) / 256;
      if (125 * r320 <= 95 * r256) tile = 1320256;
    }
  }
  return tile;
}

int launch_gemm(hipStream_t s, GemmBatch& b, int force_tile) {
  b.ln_done = 0;
  int tile = choose_tile(b, force_tile);
  // The streams of the 8-wave tiles do not know second terms of A: there it is added by a launch of its own.
  if (tile == 1256256 || tile == 1320256 || tile == 32256128) {
    GemmBatch first = b, second = b;
    second.n = 0;
    for (int i = 0; i < b.n; ++i) {
      if (!b.p[i].A2) continue;
      if (b.p[i].out_kind != OUT_F32 && b.p[i].out_kind != OUT_RESID_F32) return -1;
      first.p[i].A2 = nullptr;
      GemmProblem& q = second.p[second.n++] = b.p[i];
      q.A = q.A2; q.A2 = nullptr; q.bias = nullptr; q.out_kind = OUT_RESID_F32;
    }
    if (second.n) {
      tile = launch_gemm(s, first, force_tile);
      return tile < 0 ? tile : launch_gemm(s, second, force_tile);
    }
  }
  // a gated pair: two problems of one A and one shape, nothing but the product
  if (b.geglu && (b.n != 2 || b.p[0].A != b.p[1].A || b.p[0].lda != b.p[1].lda || b.p[0].M != b.p[1].M || b.p[0].N != b.p[1].N ||
                  b.p[0].K != b.p[1].K || b.p[0].ldw != b.p[1].ldw || b.p[0].bias || b.p[1].bias)) return -1;
  bool narrow = b.geglu && tile < 40000000;      // epilogues that need waves of 64 columns (the split reduction has its own ...
  bool conv = false, plain = false, qknorm = false;
  for (int i = 0; i < b.n; ++i) {
    conv = conv || b.p[i].conv_w > 0; plain = plain || b.p[i].conv_w <= 0;
    qknorm = qknorm || b.p[i].out_kind == OUT_QKNORM;
    narrow = narrow || (b.p[i].out_kind == OUT_VT && tile < 40000000);
  }
  if (narrow && tile == 30064128) tile = 32064128;
  if (narrow && tile == 30032128) tile = 30128128;
  // ... but none for the q/k norm)
  if ((qknorm || narrow) && !(tile == 1256256 || tile == 1320256 || tile == 11256256 || tile == 21256256 || tile == 128128 || tile == 10128128 ||
                              tile == 30128128 || tile == 30128064 || tile == 32064128 || tile == 30064064 || tile == 33128064 || tile == 256128 ||
                              tile == 31256128 || tile == 32256128))
    return -1;
  if (b.geglu && tile < 40000000) {     // unsplit: one problem whose tiles hold both products of their columns
    b.p[0].W2 = b.p[1].W;
    b.p[0].N *= 2;
    b.p[0].out_kind = OUT_GEGLU;
    b.n = 1;
  }
  if (qknorm && (tile == 30128064 || tile == 33128064 || tile == 30064064))      // 64 columns per workgroup: heads of 64 only
    for (int i = 0; i < b.n; ++i)
      if (b.p[i].out_kind == OUT_QKNORM && b.p[i].qk.head_dim > 64) return -1;
  if (conv) {     // convolutions: never mixed with plain products, three tile shapes
    if (plain) return -1;
    for (int i = 0; i < b.n; ++i)        // whole images of whole rows
      if (b.p[i].conv_img <= 0 || b.p[i].conv_img % b.p[i].conv_w || b.p[i].M % b.p[i].conv_img ||
          (b.p[i].conv_kt != 1 && b.p[i].conv_kt != 3) || b.p[i].K != 9 * b.p[i].conv_kt * b.p[i].conv_cin) return -1;
    if (tile == 1256256) launch8_t<256, 256, 2, 4, 2, true>(s, b);
    else if (tile == 32256128) launch8_t<256, 128, 4, 2, 3, true>(s, b);
    else if (tile == 40128128) launch_t<128, 128, 2, 2, 64, 4, 4, true>(s, b);
    else if (tile == 30128128) launch_t<128, 128, 2, 2, 64, 4, 0, true>(s, b);
    else { tile = 128128; launch_t<128, 128, 2, 2, 64, 2, 0, true>(s, b); }
    return tile;
  }
  switch (tile) {
    case 256256: launch_t<256, 256, 2, 2, 64, 2>(s, b); break;
    case 1256256: launch8_t<256, 256, 2, 4, 2>(s, b); break;
    case 1320256: launch8_t<320, 256, 2, 4, 2>(s, b); break;
    case 10256256: launch_t<256, 256, 2, 2, 32, 4>(s, b); break;
    case 11256256: launch_t<256, 256, 2, 4, 32, 4>(s, b); break;
    case 20256256: launch_t<256, 256, 2, 2, 32, 5>(s, b); break;
    case 21256256: launch_t<256, 256, 2, 4, 32, 5>(s, b); break;
    case 256128: launch_t<256, 128, 2, 2, 64, 2>(s, b); break;
    case 128256: launch_t<128, 256, 2, 2, 64, 2>(s, b); break;
    case 10128128: launch_t<128, 128, 2, 2, 32, 4>(s, b); break;
    case 30128128: launch_t<128, 128, 2, 2, 64, 4>(s, b); break;
    case 30128064: launch_t<128, 64, 4, 1, 64, 6>(s, b); break;
    case 30064128: launch_t<64, 128, 1, 4, 64, 6>(s, b); break;
    case 32064128: launch_t<64, 128, 2, 2, 64, 6>(s, b); break;
    case 30032128: launch_t<32, 128, 1, 4, 64, 4>(s, b); break;
    case 40032128: launch_t<32, 128, 1, 4, 64, 4, 4>(s, b); break;
    case 30064064: launch_t<64, 64, 2, 1, 64, 5>(s, b); break;
    case 40064064: launch_t<64, 64, 2, 1, 64, 5, 4>(s, b); break;
    case 33128064: launch_t<128, 64, 4, 1, 64, 3>(s, b); break;
    case 31256128: launch_t<256, 128, 2, 2, 64, 3>(s, b); break;
    case 32256128: launch8_t<256, 128, 4, 2, 3>(s, b); break;
    case 31128256: launch_t<128, 256, 2, 2, 64, 3>(s, b); break;
    case 40128128: launch_t<128, 128, 2, 2, 64, 4, 4>(s, b); break;
    default: tile = 128128; launch_t<128, 128, 2, 2, 64, 2>(s, b); break;
  }
  return tile;
}

}  // namespace dit
