// MFMA GEMM for gfx950 with fused epilogues.
//
//   C[M][N] = A[M][K] * W[N][K]^T   (A row-major, W = weights [out][in])
//
// Two kernels on direct global->LDS loads: k_gemm_w4 (bf16) and k_gemm_ring
// (bf16 and fp32); ragged M and N tails are handled by the loads' buffer ranges
// (zeros) and by masking stores.
//
// The accumulation order over K depends on the element type only, never on the
// kernel, the tile shape or M: a row's result is bitwise the same whatever
// other rows share the launch (batch invariance).
//
// Every projection of the model has a bias; the accumulators start from it
// (each column's bias, then the products in a fixed K order), so the epilogue
// reads no bias.
#pragma once
#include "kernels.hpp"

#include <type_traits>

namespace cs {

// LDS layout: a tile row holds 128 bytes of one K slice (64 bf16 or 32 fp32, 8
// chunks of 16 bytes); logical chunk c of row r is stored at c ^ gemm_swz(r),
// gemm_swz(r) = r mod 8.  A fragment read (16 rows, each lane one 16-byte
// chunk) measured free of LDS bank conflicts with this swizzle (a variant
// that also flips chunk bit 0 for rows 8..15 of each 16 stalled the LDS on
// conflicts 14% of the kernel's cycles).  Rows r and r + 16 share the
// swizzle, so the fragment reads of the 16-row blocks of a wave tile differ
// by an immediate offset.
CS_DEV int gemm_swz(int r) { return r & 7; }

// 16x16 accumulators: the products are formed as C^T tiles (W fragment as the
// MFMA A operand), so accumulator (i, j) of a lane holds row i*16 + lane%16
// of the wave's sub-tile and, in registers 0..3, columns j*16 + 4(lane/16) ..
// +3, one vector access in the epilogue.
template <int TM, int TN>
CS_DEV void init_acc16_bias(f32x4 (&acc)[TM][TN], const float* __restrict__ bias, int col_base,
                            int lane, int N) {
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col0 = col_base + j * 16 + 4 * (lane >> 4);
    float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col0 < N) b = *reinterpret_cast<const float4*>(bias + col0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      acc[i][j][0] = b.x;
      acc[i][j][1] = b.y;
      acc[i][j][2] = b.z;
      acc[i][j][3] = b.w;
    }
  }
}

// Epilogue over 16x16 accumulators with the epilogue operands of PD - 1
// chunks in flight (a ring of PD slots): with one wave per SIMD nothing else
// hides the latency of the residual reads, so they are requested well ahead.
template <bool CHECK, int PD, int TM, int TN, class Epi>
CS_DEV void gemm_epilogue16_deep_impl(const f32x4 (&acc)[TM][TN], int row_base, int col_base,
                                      int lane, int M, int N, const Epi& epi) {
  constexpr int NQ = TM * TN;
  typename Epi::Pre pre[PD];
  auto fetch = [&](int q) {
    const int i = q / TN, j = q % TN;
    const int row = row_base + i * 16 + (lane & 15);
    const int col0 = col_base + j * 16 + 4 * (lane >> 4);
    if (!CHECK || (row < M && col0 < N)) pre[q % PD] = epi.pre(row, col0);
  };
#pragma unroll
  for (int q = 0; q < PD - 1 && q < NQ; ++q) fetch(q);
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (q + PD - 1 < NQ) fetch(q + PD - 1);
    const int i = q / TN, j = q % TN;
    const int row = row_base + i * 16 + (lane & 15);
    const int col0 = col_base + j * 16 + 4 * (lane >> 4);
    if (!CHECK || (row < M && col0 < N)) {
      const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      epi(row, col0, v, pre[q % PD]);
    }
  }
}

template <int PD, int TM, int TN, class Epi>
CS_DEV void gemm_epilogue16_deep(const f32x4 (&acc)[TM][TN], int row_base, int col_base, int lane,
                                 int M, int N, const Epi& epi) {
  if (row_base + TM * 16 <= M && col_base + TN * 16 <= N)
    gemm_epilogue16_deep_impl<false, PD>(acc, row_base, col_base, lane, M, N, epi);
  else
    gemm_epilogue16_deep_impl<true, PD>(acc, row_base, col_base, lane, M, N, epi);
}

// ---------------------------------------------------------------------------
// Direct global->LDS loads (gfx950 buffer_load_dwordx4 ... lds) and 16x16
// MFMAs (x32 in bf16, x4 in fp32).
//
// Each load instruction of a wave moves 64 x 16 bytes into 1 KB of LDS at
// base + 16*lane, with an arbitrary source offset per lane, so no registers
// stage the tiles and no LDS store instructions are issued.  LDS rows are
// unpadded and swizzled (gemm_swz), which keeps the fragment reads (16 rows x
// 4 chunks per instruction) free of bank conflicts.  W is stored in blocks of
// 256 rows x 128 bytes (gemm_tile_weight); a tile of BN < 256 columns takes
// BN consecutive rows of a block, which are contiguous there.
//
// Two kernels, one per limit.  k_gemm_w4 (below) is for bf16 tiles whose
// products fill the matrix pipe; k_gemm_ring (further down) for grids that
// leave most CUs with a single small tile, where the latency from one K slice
// to the next is what counts, and for fp32, whose products take 16 times as
// long per byte loaded.  In either type every tile shape sums in the same order
// (bias, then K in steps of 32 in bf16, of 16 in fp32), so results are bitwise
// equal whichever is chosen: the choice (k_gemm.hip) may follow M without
// making a row's result depend on how many other rows share the launch.
// ---------------------------------------------------------------------------
constexpr int W_BLOCK_ROWS = 256;   // rows of a block of the tiled weights

// Batched launches (blockIdx.y = item): the same A against n weight matrices
// w_stride elements apart, with an epilogue that moves to item z (Epi::item).
template <class Epi> struct EpiBatched : std::false_type {};

// Tile order: the launch is split into 8 contiguous ranges, one per XCD
// (workgroups are dealt round-robin to the 8 dies).  Inside a range, tiles are
// visited in groups of GM tile-rows, column-major within the group, so the
// workgroups resident on one die at a time share both rows of A and columns of
// W in its L2.
template <int GM>
CS_DEV void gemm_tile_of(int tiles_m, int tiles_n, int& tm_i, int& tn_i) {
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int group = bid / (GM * tiles_n), first_m = group * GM;
  const int gm = min(tiles_m - first_m, GM);
  const int in = bid - group * GM * tiles_n;
  tm_i = first_m + in % gm;
  tn_i = in / gm;
}

// ---------------------------------------------------------------------------
// bf16 GEMM, 4 waves of (BM/2) x (BN/2): one wave per SIMD at BN = 256 (BM =
// 256, 224, 192, 160), two workgroups per CU (OCC = 2) at 128 x 128 and three
// at 64 x 64; the accumulators are held in AGPRs.
//
// Fragment reads from LDS per product: (BM/32 + 8) reads per BM/4 products,
// against 12 per 32 with 8 waves of 128x64, so the LDS, which also absorbs
// the direct loads, is less of a co-limit.  With a single wave per SIMD no
// other wave hides a stall, so every LDS read is issued half a K slice (one
// k-step of products) ahead of its use, and the direct loads are spread
// evenly over the slice (clumped, they back up the address unit and stall
// the issuing wave):
//
//   slice k, half 1: products of k-step 0 | reads of k-step 1 of slice k |
//                    loads of the A rows of slice k+2
//   wait: own loads of slice k+1 landed, own reads done; barrier
//   slice k, half 2: products of k-step 1 | reads of k-step 0 of slice k+1 |
//                    loads of the W rows of slice k+2
//
// A tiles rotate through three LDS buffers and W tiles through two (160 KB
// at 256 x 256, 80 KB at 128 x 128): the A buffer of slice k+2 held slice k-1, which every wave
// finished reading before the previous barrier, and the W buffer of slice
// k+2 held slice k, whose last reads precede this slice's barrier.
//
// The products are issued as volatile inline assembly with the accumulators
// bound to AGPRs: that fixes the issue order exactly (LDS reads and loads
// are ordered against them) and keeps the register allocator from moving
// accumulators between the register files.  The compiler does not see them
// as matrix instructions, so the hazards it would otherwise cover are
// covered here: the accumulators are written (bias) long before the first
// product, none is read until 24 wait states after the last product, an
// accumulator's next product comes NM >= 4 products later, and a fragment
// register is rewritten by an LDS read issued no sooner than two products
// after the last product that used it (products issue in order and read
// their operands in their first cycles; the read's data returns later still).
// ---------------------------------------------------------------------------
// Epilogues that route a workgroup's tile through LDS on its way out
// (staged_tile / store_staged_tile), once the main loop has released the
// ring: each wave gets a region of max(WN (WM + 8), WM (WN + 8)) elements.
template <class Epi> struct EpiStagesTiles : std::false_type {};

CS_DEV void mfma_16x16x32_agpr(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

template <int BM, int BN, int OCC, int GM, int PD, class Epi>
__global__ __launch_bounds__(256, OCC) void k_gemm_w4(const bf16* __restrict__ A, long lda,
                                                    const bf16* __restrict__ W, int M, int N,
                                                    int K, long w_stride, Epi epi) {
  if constexpr (EpiBatched<Epi>::value) {
    W += blockIdx.y * w_stride;
    epi.item(blockIdx.y);
  }
  constexpr int BK = 64, NWAVE = 4, WM = BM / 2, WN = BN / 2;
  constexpr int CH = 8;                       // bf16 per 16-byte chunk
  constexpr int CPR = BK / CH;                // chunks per LDS row
  constexpr int RPI = 64 / CPR;               // rows filled by one wave instruction
  constexpr int A_INST = BM / RPI / NWAVE;    // load instructions per wave per slice
  constexpr int B_INST = BN / RPI / NWAVE;
  constexpr int A_BUF = BM * BK, B_BUF = BN * BK;  // elements per buffer
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int NF = TM + TN, NM = TM * TN;   // reads and products per k-step
  // products per read: as far apart as fits a half, at most 3
  constexpr int RPM = (NM - 1) / (NF - 1) < 3 ? (NM - 1) / (NF - 1) : 3;
  static_assert(A_INST * RPI * NWAVE == BM && B_INST * RPI * NWAVE == BN, "load split");
  static_assert(W_BLOCK_ROWS % BN == 0 && RPI * BK * 2 == 1024, "part of a tiled W block");
  static_assert(RPM * (NF - 1) < NM && NM % A_INST == 0 && NM % B_INST == 0, "interleave");
  __shared__ __attribute__((aligned(1024))) bf16 smem[3 * A_BUF + 2 * B_BUF];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  const int tiles_n = (N + BN - 1) / BN;
  const int tiles_m = (M + BM - 1) / BM;
  int tm_i, tn_i;
  gemm_tile_of<GM>(tiles_m, tiles_n, tm_i, tn_i);
  const int m0 = tm_i * BM, n0 = tn_i * BN;

  const bf16* a_base = A + (long)m0 * lda;
  const int n_in = n0 % W_BLOCK_ROWS;         // first row of the tile in its W block
  const bf16* b_base = W + (long)(n0 - n_in) * K + n_in * BK;
  const int a_bytes = min(BM, M - m0) * (int)lda * 2, b_bytes = (W_BLOCK_ROWS * K - n_in * BK) * 2;
  int a_off[A_INST], b_off[B_INST];
  {
    const int rin = lane / CPR, phys = lane % CPR;
#pragma unroll
    for (int i = 0; i < A_INST; ++i) {
      const int row = (wave * A_INST + i) * RPI + rin;
      a_off[i] = (row * (int)lda + (phys ^ gemm_swz(row)) * CH) * 2;
    }
#pragma unroll
    for (int i = 0; i < B_INST; ++i) b_off[i] = (wave * B_INST + i) * 1024 + lane * 16;
  }
  bf16* const sb0 = smem + 3 * A_BUF;
  // load instruction r of the A (W) rows of slice `slice` into A buffer ab (W buffer bb)
  auto load_a = [&](int r, int slice, int ab) {
    buffer_load_lds16(a_base, a_bytes, smem + ab * A_BUF + (wave * A_INST + r) * RPI * BK, a_off[r],
                      slice * BK * 2);
  };
  auto load_b = [&](int r, int slice, int bb) {
    buffer_load_lds16(b_base, b_bytes, sb0 + bb * B_BUF + (wave * B_INST + r) * RPI * BK, b_off[r],
                      slice * W_BLOCK_ROWS * BK * 2);
  };

  f32x4 acc[TM][TN];
  init_acc16_bias(acc, epi.bias, n0 + wn * WN, lane, N);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));  // in AGPRs from here on

  // fragment addressing (16x16x32 operands): lane reads row (lane & 15) of
  // each 16-row block at logical chunk 4*ks + (lane >> 4); the swizzle of
  // row r + 16i equals that of row r, so block i is at an immediate offset
  const int a_row0 = wm * WM + (lane & 15);
  const int b_row0 = wn * WN + (lane & 15);
  const int quad = lane >> 4;
  const int a_lds[2] = {a_row0 * BK + (quad ^ gemm_swz(a_row0)) * CH,
                        a_row0 * BK + ((4 + quad) ^ gemm_swz(a_row0)) * CH};
  const int b_lds[2] = {b_row0 * BK + (quad ^ gemm_swz(b_row0)) * CH,
                        b_row0 * BK + ((4 + quad) ^ gemm_swz(b_row0)) * CH};
  // read r (< NF) of k-step ks from A buffer ab / W buffer bb: W fragments
  // first (the first products of the next half use all of them)
  auto read = [&](int r, int ab, int bb, int ks, bf16x8(&fa)[TM], bf16x8(&fb)[TN]) {
    if (r < TN)
      fb[r] = *reinterpret_cast<const bf16x8*>(sb0 + bb * B_BUF + b_lds[ks] + r * 16 * BK);
    else
      fa[r - TN] = *reinterpret_cast<const bf16x8*>(smem + ab * A_BUF + a_lds[ks] + (r - TN) * 16 * BK);
  };

  bf16x8 f0a[TM], f0b[TN], f1a[TM], f1b[TN];
  // One half: the NM products of (pa, pb); after product RPM*r, read r into
  // (na, nb) (RD); NL loads spread evenly, through `ld` (LD).
  auto half = [&](auto rd, auto ldf, auto nl, const bf16x8(&pa)[TM], const bf16x8(&pb)[TN],
                  bf16x8(&na)[TM], bf16x8(&nb)[TN], int ab, int bb, int ks) {
    constexpr int NL = decltype(nl)::value;
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      mfma_16x16x32_agpr(acc[q / TN][q % TN], pb[q % TN], pa[q / TN]);
      if constexpr (NL > 0) {
        if (q % (NM / NL) == NM / NL / 2) ldf(q / (NM / NL));
      }
      if constexpr (decltype(rd)::value) {
        if (q % RPM == 0 && q / RPM < NF) read(q / RPM, ab, bb, ks, na, nb);
      }
    }
  };
  typedef std::integral_constant<bool, true> Y;
  typedef std::integral_constant<bool, false> F;
  typedef std::integral_constant<int, 0> L0;
  typedef std::integral_constant<int, A_INST> LA;
  typedef std::integral_constant<int, B_INST> LB;
  auto no_load = [](int) {};

  const int nk = K / BK;
#pragma unroll
  for (int r = 0; r < A_INST; ++r) load_a(r, 0, 0);
#pragma unroll
  for (int r = 0; r < B_INST; ++r) load_b(r, 0, 0);
  if (nk > 1) {
#pragma unroll
    for (int r = 0; r < A_INST; ++r) load_a(r, 1, 1);
#pragma unroll
    for (int r = 0; r < B_INST; ++r) load_b(r, 1, 1);
    wait_vm_barrier<A_INST + B_INST>();   // slice 0 landed (slice 1 may be in flight)
  } else {
    wait_vm_barrier<0>();
  }
#pragma unroll
  for (int r = 0; r < NF; ++r) read(r, 0, 0, 0, f0a, f0b);

  // HN: slice k+1 exists (barrier, its k-step 0 reads); IS: slice k+2
  // exists (its loads).  Slice k uses A buffer k % 3 and W buffer k % 2.
  auto slice = [&](int kt, int a3, auto hn, auto is) {
    const int b2 = kt & 1;
    const int a_next = a3 == 2 ? 0 : a3 + 1, a_far = a3 == 0 ? 2 : a3 - 1;
    if constexpr (decltype(is)::value) {
      half(Y{}, [&](int r) { load_a(r, kt + 2, a_far); }, LA{}, f0a, f0b, f1a, f1b, a3, b2, 1);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(A_INST) : "memory");
      half(Y{}, [&](int r) { load_b(r, kt + 2, b2); }, LB{}, f1a, f1b, f0a, f0b, a_next, b2 ^ 1, 0);
    } else if constexpr (decltype(hn)::value) {
      half(Y{}, no_load, L0{}, f0a, f0b, f1a, f1b, a3, b2, 1);
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      half(Y{}, no_load, L0{}, f1a, f1b, f0a, f0b, a_next, b2 ^ 1, 0);
    } else {
      half(Y{}, no_load, L0{}, f0a, f0b, f1a, f1b, a3, b2, 1);
      half(F{}, no_load, L0{}, f1a, f1b, f0a, f0b, 0, 0, 0);
    }
  };
  int kt = 0, a3 = 0;
  for (; kt + 2 < nk; ++kt, a3 = a3 == 2 ? 0 : a3 + 1) slice(kt, a3, Y{}, Y{});
  if (kt + 1 < nk) {
    slice(kt, a3, Y{}, F{});
    ++kt;
    a3 = a3 == 2 ? 0 : a3 + 1;
  }
  slice(kt, a3, F{}, F{});

  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));  // read only after the nops
  if constexpr (EpiStagesTiles<Epi>::value && WM >= 32 && WN >= 32) {
    constexpr int STG = WN * (WM + 8) > WM * (WN + 8) ? WN * (WM + 8) : WM * (WN + 8);
    static_assert(NWAVE * STG <= 3 * A_BUF + 2 * B_BUF, "staging fits the ring");
    if (epi.staged_tile(n0)) {   // uniform over the workgroup
      __syncthreads();           // every wave's last fragment reads are done
      epi.store_staged_tile(acc, smem + wave * STG, m0 + wm * WM, n0 + wn * WN, lane, M, N);
      return;
    }
  }
  gemm_epilogue16_deep<PD>(acc, m0 + wm * WM, n0 + wn * WN, lane, M, N, epi);
}

// ---------------------------------------------------------------------------
// GEMM on a ring of LDS stages.  In bf16 for small grids (few rows, narrow
// outputs): BM x BN tiles of 128 x 128, 64 x 128 and 64 x 64 (8 waves), 32 x 64
// and 32 x 32 (4 waves).  In fp32 for all of them.
//
// With a tile or less per CU nothing runs beside it, so a slice costs its
// latency chain: barrier, fragment reads, products.  The chain is shortened in
// three ways: one step covers two K slices (SL; one at 128 x 128, whose
// products cover the latency), so the barrier and the read latency are paid
// half as often; the reads of step k+1 are issued before the
// products of step k, into a second register set; and STAGES steps of loads
// are in flight (the buffer of step k is free as soon as its reads are done,
// before its products).  Measured at 384 x 1536 x 8960, one stream of 384
// tokens on the 1.3B FFN-down projection, 144 tiles of 64 x 64: 30 us, against
// 156 us with 256 x 256 tiles (12 of them) and 41 us with one slice per
// barrier; 891 x 256 x 512 with 32 x 32 tiles: 3.4 us against 24.8 us.  With
// weights from HBM the loads in flight count too: 1536 x 1536 x 8960 takes 70 us
// with 128 x 128 ring tiles (three slices ahead) against 94 us with k_gemm_w4's
// (one and a half), 384 x 4608 x 1536 13.7 us with 64 x 128 against 17.9 us.
//
// In bf16 the counters of such launches (384 and 1,536 rows) show neither pipe
// busy on the CUs that have a tile: products 16 to 40% of the cycles, LDS reads 24
// to 30%, no bank conflicts, waves waiting for the LDS 5 to 8% of their time.
//
// In fp32 a 32 x 32 x 32 slice of products takes 256 cycles per CU, four times
// what the counters show for its fragment reads (matrix pipe busy 61% of all
// cycles against 15% at 768 x 1536 x 8960), and the matrix pipe is the limit once
// the chip is full: 88 to 90% busy with 64 x 64 tiles at 12,480 rows.  Below that
// the last round counts: the smallest tile wins by filling the chip evenly, with
// four workgroups per CU covering each other's barriers.  768 x 1536 x 8960: 183 us
// (115 TFLOP/s), against 391 us (up to 660) with 128 x 128 register-staged tiles;
// 1024 x 128 x 512: 5.1 against 43 us.  A lane's 16-byte chunk holds four consecutive k;
// product e of a chunk takes element e of the four lanes of a row, so four
// products consume a chunk of each operand without any shuffle.  The distance
// of whole evaluations and rollouts to 64-bit results (8 shapes, 8 seeds each)
// is that of sums in natural k order: 4.4e-7 at d = 128, 1.45e-6 at d = 1536.
// ---------------------------------------------------------------------------
template <typename T> struct Mfma16;
template <> struct Mfma16<bf16> {
  typedef bf16x8 chunk;
  static CS_DEV f32x4 mma(const chunk& a, const chunk& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma16<float> {
  typedef f32x4 chunk;
  static CS_DEV f32x4 mma(const chunk& a, const chunk& b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
  }
};

template <typename T, int BM, int BN, int WGM, int WGN, int SL, int STAGES, int OCC, int GM, class Epi>
__global__ __launch_bounds__(64 * WGM * WGN, OCC) void k_gemm_ring(const T* __restrict__ A, long lda,
                                                                  const T* __restrict__ W, int M,
                                                                  int N, int K, long w_stride, Epi epi) {
  if constexpr (EpiBatched<Epi>::value) {
    W += blockIdx.y * w_stride;
    epi.item(blockIdx.y);
  }
  typedef typename Mfma16<T>::chunk chunk;
  constexpr int ES = (int)sizeof(T), CH = 16 / ES, BK = 8 * CH, RPI = 8, NWAVE = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16, NF = TM + TN;
  constexpr int A_INST = BM / RPI / NWAVE, B_INST = BN / RPI / NWAVE;
  constexpr int PER = (A_INST + B_INST) * SL;               // load instructions per wave per step
  constexpr int SLICE = (BM + BN) * BK, STAGE = SLICE * SL;  // elements
  static_assert(A_INST * RPI * NWAVE == BM && B_INST * RPI * NWAVE == BN, "load split");
  static_assert(W_BLOCK_ROWS % BN == 0, "part of a tiled W block");
  static_assert(STAGES >= 2 && STAGES <= 4, "wait counts below");
  // the ring, then 1 KB of bias per wave.  One array: the compiler waits for all
  // direct loads before a read of a second one.
  __shared__ __attribute__((aligned(1024))) T smem[STAGES * STAGE + NWAVE * 1024 / ES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
  const int wm = wave / WGN, wn = wave % WGN;
  const int tiles_n = (N + BN - 1) / BN, tiles_m = (M + BM - 1) / BM;
  int tm_i, tn_i;
  gemm_tile_of<GM>(tiles_m, tiles_n, tm_i, tn_i);
  const int m0 = tm_i * BM, n0 = tn_i * BN;

  // per-lane offsets as in k_gemm_w4; the bases move from slice to slice, so
  // that the 32-bit ranges cover one slice: the tile's rows of A up to its end,
  // and the tile's part of a W block
  const T* a_base = A + (long)m0 * lda;
  const int n_in = n0 % W_BLOCK_ROWS;
  const T* b_base = W + (long)(n0 - n_in) * K + n_in * BK;
  const int a_bytes = ((min(BM, M - m0) - 1) * (int)lda + BK) * ES, b_bytes = BN * BK * ES;
  int a_off[A_INST], b_off[B_INST];
#pragma unroll
  for (int i = 0; i < A_INST; ++i) {
    const int row = (wave * A_INST + i) * RPI + lane / 8;
    a_off[i] = (row * (int)lda + ((lane % 8) ^ gemm_swz(row)) * CH) * ES;
  }
#pragma unroll
  for (int i = 0; i < B_INST; ++i) b_off[i] = (wave * B_INST + i) * 1024 + lane * 16;
  // An odd slice count leaves half a step at the end: the last slice is loaded
  // twice (the wait counts stay uniform) and multiplied once.
  const int nslice = K / BK, nstep = (nslice + SL - 1) / SL;
  auto issue = [&](int step, int st) {
#pragma unroll
    for (int l = 0; l < SL; ++l) {
      T* sa = smem + st * STAGE + l * SLICE;
      T* sb = sa + BM * BK;
      const int slice = min(step * SL + l, nslice - 1);
#pragma unroll
      for (int i = 0; i < A_INST; ++i)
        buffer_load_lds16(a_base + (long)slice * BK, a_bytes, sa + (wave * A_INST + i) * RPI * BK, a_off[i], 0);
#pragma unroll
      for (int i = 0; i < B_INST; ++i)
        buffer_load_lds16(b_base + (long)slice * W_BLOCK_ROWS * BK, b_bytes,
                          sb + (wave * B_INST + i) * RPI * BK, b_off[i], 0);
    }
  };

  // The bias from the wave's first column on (zeros past N) comes in by the first
  // of the direct loads: the wait for step 0 covers it.  A load into registers
  // would be waited for by the compiler, which cannot count the conditional loads
  // behind it and waits for all of them, the whole ring, before the first product.
  T* const s_bias = smem + STAGES * STAGE + wave * (1024 / ES);
  buffer_load_lds16(epi.bias, N * 4, s_bias, (n0 + wn * WN) * 4 + lane * 16, 0);

#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < nstep) issue(s, s);

  // fragment addressing (16x16x32 operands) as in k_gemm_w4
  const int a_row0 = wm * WM + (lane & 15), b_row0 = wn * WN + (lane & 15), quad = lane >> 4;
  const int a_lds[2] = {a_row0 * BK + (quad ^ gemm_swz(a_row0)) * CH,
                        a_row0 * BK + ((4 + quad) ^ gemm_swz(a_row0)) * CH};
  const int b_lds[2] = {(BM + b_row0) * BK + (quad ^ gemm_swz(b_row0)) * CH,
                        (BM + b_row0) * BK + ((4 + quad) ^ gemm_swz(b_row0)) * CH};
  chunk f[2][2 * SL][NF];   // two register sets of one step's fragments
  auto read = [&](int st, chunk(&o)[2 * SL][NF]) {
#pragma unroll
    for (int ks = 0; ks < 2 * SL; ++ks) {
      const T* s = smem + st * STAGE + (ks >> 1) * SLICE;
#pragma unroll
      for (int j = 0; j < TN; ++j) o[ks][TM + j] = *reinterpret_cast<const chunk*>(s + b_lds[ks & 1] + j * 16 * BK);
#pragma unroll
      for (int i = 0; i < TM; ++i) o[ks][i] = *reinterpret_cast<const chunk*>(s + a_lds[ks & 1] + i * 16 * BK);
    }
  };
  if (nstep >= STAGES) wait_all_barrier<(STAGES - 1) * PER>();   // bias and step 0 landed
  else wait_all_barrier<0>();
  f32x4 acc[TM][TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
      acc[i][j] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(s_bias) + 16 * j + 4 * (lane >> 4));
  read(0, f[0]);
  auto mul = [&](int step, const chunk(&o)[2 * SL][NF]) {
#pragma unroll
    for (int ks = 0; ks < 2 * SL; ++ks) {
      if (SL == 2 && ks == 2 && step * SL + 1 >= nslice) break;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = Mfma16<T>::mma(o[ks][TM + j], o[ks][i], acc[i][j]);
    }
  };
  // step k: products of k from registers `cur`, reads of k+1 into `nxt`
  auto step = [&](int k, const chunk(&cur)[2 * SL][NF], chunk(&nxt)[2 * SL][NF]) {
    if (k + 1 < nstep) {
      // step k+1 landed (later ones may be in flight) and, past the barrier,
      // every wave's reads of step k are done: its buffer is free
      const int later = nstep - 2 - k;
      if (later >= STAGES - 2) wait_all_barrier<(STAGES - 2) * PER>();
      else if (STAGES == 4 && later == 1) wait_all_barrier<PER>();
      else wait_all_barrier<0>();
      if (k + STAGES < nstep) issue(k + STAGES, k % STAGES);
      read((k + 1) % STAGES, nxt);
    }
    mul(k, cur);
  };
  int k = 0;
  for (; k + 1 < nstep; k += 2) {
    step(k, f[0], f[1]);
    step(k + 1, f[1], f[0]);
  }
  if (k < nstep) step(k, f[0], f[1]);

  gemm_epilogue16_deep<2>(acc, m0 + wm * WM, n0 + wn * WN, lane, M, N, epi);
}

// ------------------------------------------------------------- epilogues
// Each epilogue is called per (row, 4 consecutive columns col0..col0+3) with
// the accumulated values v (bias included); N is a multiple of 4.  `Pre` is
// what it reads from memory besides v, fetched ahead by `pre`.
template <typename T> CS_DEV void store4(T* p, const float* y) {
  if constexpr (sizeof(T) == 2) {
    bf16x4 q;
#pragma unroll
    for (int r = 0; r < 4; ++r) q[r] = to_t<T>(y[r]);
    *reinterpret_cast<bf16x4*>(p) = q;
  } else {
    *reinterpret_cast<float4*>(p) = make_float4(y[0], y[1], y[2], y[3]);
  }
}
struct NoPre {};

// Row-major bf16 store of one wave's TM*16 x TN*16 block of 16x16
// accumulators (lane holds row row_base + 16i + (lane & 15), columns
// col_base + 16j + 4(lane >> 4) + r) through `stage` (TM*16 rows of TN*16 + 8
// elements): written as 8-byte pieces, read back and stored as 16-byte runs,
// 256 contiguous bytes per row, where the direct path stores 32-byte pieces
// of 16 rows per instruction.  f maps each value before its rounding.
// Contains one workgroup barrier: every wave of the workgroup calls a staged
// store exactly once.
template <int TM, int TN, class F>
CS_DEV void store_rows_staged(const f32x4 (&acc)[TM][TN], bf16* stage, int row_base, int col_base,
                              int lane, int M, int N, bf16* out, long ldo, F f) {
  constexpr int R = TM * 16, C = TN * 16, SP = C + 8;
  constexpr int LPR = C / 8, RPI = 64 / LPR;   // lanes per row, rows per instruction
  static_assert(64 % LPR == 0 && R % RPI == 0, "readback split");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      bf16x4 q;
#pragma unroll
      for (int r = 0; r < 4; ++r) q[r] = (bf16)f(acc[i][j][r]);
      *reinterpret_cast<bf16x4*>(stage + (16 * i + (lane & 15)) * SP + 16 * j + 4 * (lane >> 4)) = q;
    }
  __syncthreads();
  const int c = 8 * (lane % LPR), col = col_base + c;
  const bool whole = col + 8 <= N && ((ldo | col) & 7) == 0;
#pragma unroll 4
  for (int q = 0; q < R / RPI; ++q) {
    const int r = RPI * q + lane / LPR, row = row_base + r;
    if (row >= M) continue;
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(stage + r * SP + c);
    bf16* dst = out + (long)row * ldo + col;
    if (whole && ((uintptr_t)dst & 15) == 0) {
      *reinterpret_cast<bf16x8*>(dst) = v;
    } else {
      for (int e = 0; e < 8 && col + e < N; ++e) dst[e] = v[e];
    }
  }
}

struct IdentityF { CS_DEV float operator()(float x) const { return x; } };
struct GeluF { CS_DEV float operator()(float x) const { return gelu_tanh(x); } };

// On the bf16 kernel every tile goes out through LDS (store_rows_staged).
// Measured against the element-wise path at 8 x 32,760 rows, d = 1536, same
// process: cross q (N = 1536) 1.036 -> 0.938 ms, q|k (N = 3072) 2.032 ->
// 1.895 ms, FFN up + GELU (N = 8960) unchanged (5.877 vs 5.886 ms); same
// values.
template <typename T, int ACT> struct EpiStore {  // ACT: 0 none, 1 tanh-GELU
  T* out; long ldo; const float* bias; long out_stride = 0, bias_stride = 0;
  CS_DEV void item(int z) { out += z * out_stride; bias += z * bias_stride; }
  typedef NoPre Pre;
  CS_DEV Pre pre(int, int) const { return {}; }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre&) const {
    float y[4] = {v[0], v[1], v[2], v[3]};
    if constexpr (ACT == 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = gelu_tanh(y[r]);
    }
    store4<T>(out + (long)row * ldo + col0, y);
  }

  CS_DEV bool staged_tile(int) const { return true; }
  template <int TM, int TN>
  CS_DEV void store_staged_tile(const f32x4 (&acc)[TM][TN], bf16* stage, int row_base, int col_base,
                                int lane, int M, int N) const {
    static_assert(sizeof(T) == 2, "bf16 tiles only");
    if constexpr (ACT == 1)
      store_rows_staged(acc, stage, row_base, col_base, lane, M, N, out, ldo, GeluF{});
    else
      store_rows_staged(acc, stage, row_base, col_base, lane, M, N, out, ldo, IdentityF{});
  }
};
template <int ACT> struct EpiStagesTiles<EpiStore<bf16, ACT>> : std::true_type {};
template <typename T> struct EpiBatched<EpiStore<T, 0>> : std::true_type {};

// Self-attention projection: columns [0, 2d) are q and k, stored row-major
// [row][2d]; columns [2d, 3d) are v, stored transposed per stream as
// vT[stream][channel][token] with a padded token stride.
//
// On the bf16 kernel every tile goes out through LDS.  A wave whose 128
// columns lie in v (2d is a multiple of 128) writes its 128 x 128 block there
// as [channel][token] (token stride 136, 16-byte aligned rows) and stores it
// back as 16-byte runs of 8 tokens, 256 contiguous bytes per channel, where
// the element-wise path below issues a 2-byte store per value (measured: the
// v part alone: 3.386 -> 3.167 ms for the QKV projection at 8 x 32,760 rows,
// d = 1536, within 0.5% of storing v row-major); a wave in q|k stores its
// rows through store_rows_staged (both parts staged: 3.203 -> 2.886 ms;
// bitwise equal).
template <typename T> struct EpiQKV {
  T* qk; T* vt; const float* bias; int d; int L; long vt_ld; long vt_ss;
  typedef NoPre Pre;
  CS_DEV Pre pre(int, int) const { return {}; }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre&) const {
    if (col0 < 2 * d) {
      store4<T>(qk + (long)row * (2 * d) + col0, v);
    } else {
      const int s = row / L, tok = row - s * L;
      T* dst = vt + (long)s * vt_ss + (long)(col0 - 2 * d) * vt_ld + tok;
#pragma unroll
      for (int r = 0; r < 4; ++r) dst[(long)r * vt_ld] = to_t<T>(v[r]);
    }
  }

  CS_DEV bool staged_tile(int) const { return true; }

  template <int TM, int TN>
  CS_DEV void store_staged_tile(const f32x4 (&acc)[TM][TN], bf16* stage, int row_base, int col_base,
                                int lane, int M, int N) const {
    static_assert(sizeof(T) == 2, "bf16 tiles only");
    if (col_base >= 2 * d)
      store_v_transposed(acc, stage, row_base, col_base, lane, M, N);
    else
      store_rows_staged(acc, stage, row_base, col_base, lane, M, 2 * d, qk, 2L * d, IdentityF{});
  }

  // One wave's TM*16 x TN*16 block of 16x16 accumulators (lane holds row
  // row_base + 16i + (lane & 15), columns col_base + 16j + 4(lane >> 4) + r)
  // through `stage` (TN*16 rows of TM*16 + 8 tokens) to vT; one workgroup
  // barrier, like store_rows_staged.
  template <int TM, int TN>
  CS_DEV void store_v_transposed(const f32x4 (&acc)[TM][TN], bf16* stage, int row_base,
                                 int col_base, int lane, int M, int N) const {
    constexpr int R = TM * 16, C = TN * 16, SP = R + 8, CHUNKS = R / 8;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          stage[(16 * j + 4 * (lane >> 4) + r) * SP + 16 * i + (lane & 15)] = to_t<T>(acc[i][j][r]);
    __syncthreads();
    // lane: tokens row0..row0+7 of channels c = CPI*q + lane / CHUNKS (with 96
    // rows, 12 chunks, the last 4 lanes have none; likewise 80 and 112 rows)
    constexpr int CPI = 64 / CHUNKS;
    if (lane >= CPI * CHUNKS) return;
    const int k = lane % CHUNKS;
    const int row0 = row_base + 8 * k;
    const int s = row0 / L, tok = row0 - s * L;
    const bool whole = row0 + 8 <= M && tok + 8 <= L;   // one stream, all rows valid
    T* const base = vt + (long)s * vt_ss + tok;
#pragma unroll 4
    for (int q = 0; q < (C + CPI - 1) / CPI; ++q) {
      const int c = CPI * q + lane / CHUNKS;
      const int col = col_base + c;
      if (c >= C || col >= N) continue;
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(stage + c * SP + 8 * k);
      T* dst = base + (long)(col - 2 * d) * vt_ld;
      if (whole && ((uintptr_t)dst & 15) == 0) {
        *reinterpret_cast<bf16x8*>(dst) = v;
      } else {
        for (int e = 0; e < 8; ++e) {
          const int row = row0 + e;
          if (row >= M) break;
          const int se = row / L;
          vt[(long)se * vt_ss + (long)(col - 2 * d) * vt_ld + (row - se * L)] = v[e];
        }
      }
    }
  }
};
template <> struct EpiStagesTiles<EpiQKV<bf16>> : std::true_type {};

// Transposed store of a single-stream projection: out[col][row].
template <typename T> struct EpiStoreT {
  T* out; long ldo; const float* bias; long out_stride = 0, bias_stride = 0;
  CS_DEV void item(int z) { out += z * out_stride; bias += z * bias_stride; }
  typedef NoPre Pre;
  CS_DEV Pre pre(int, int) const { return {}; }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre&) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(long)(col0 + r) * ldo + row] = to_t<T>(v[r]);
  }
};

template <typename T> struct EpiBatched<EpiStoreT<T>> : std::true_type {};

// Residual update z += gate * (acc + bias) (GATED = 0: gate 1).  The
// updated residual is stored non-temporally: it is read again only by the
// next row pass, so it need not displace the operand tiles the GEMM keeps in
// L2 (measured +2.6% on the K = 8960 projection, neutral at K = 1536).
typedef float f32x4v __attribute__((ext_vector_type(4)));
template <int GATED> struct EpiResidual {
  float* z; long ldz; const float* bias; const float* gate;
  struct Pre { float4 z, g; };
  CS_DEV Pre pre(int row, int col0) const {
    Pre p;
    p.z = *reinterpret_cast<const float4*>(z + (long)row * ldz + col0);
    p.g = make_float4(1.f, 1.f, 1.f, 1.f);
    if constexpr (GATED) p.g = *reinterpret_cast<const float4*>(gate + col0);
    return p;
  }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre& p) const {
    float4 o = p.z;
    o.x += p.g.x * v[0];
    o.y += p.g.y * v[1];
    o.z += p.g.z * v[2];
    o.w += p.g.w * v[3];
    const f32x4v ov = {o.x, o.y, o.z, o.w};
    __builtin_nontemporal_store(ov, reinterpret_cast<f32x4v*>(z + (long)row * ldz + col0));
  }
};

// Residual update that also keeps the branch output y = acc + bias in y
// (row stride N, compute type) for later reuse: z += gate * y.
template <int GATED, typename T> struct EpiResidualStore {
  float* z; long ldz; const float* bias; const float* gate; T* y;
  typedef typename EpiResidual<GATED>::Pre Pre;
  CS_DEV Pre pre(int row, int col0) const {
    return EpiResidual<GATED>{z, ldz, bias, gate}.pre(row, col0);
  }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre& p) const {
    store4<T>(y + (long)row * ldz + col0, v);
    EpiResidual<GATED>{z, ldz, bias, gate}(row, col0, v, p);
  }
};

// Patch embedding: z = acc + bias (fp32 residual stream).
struct EpiPatch {
  float* z; long ldz; const float* bias;
  typedef NoPre Pre;
  CS_DEV Pre pre(int, int) const { return {}; }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre&) const {
    *reinterpret_cast<float4*>(z + (long)row * ldz + col0) = make_float4(v[0], v[1], v[2], v[3]);
  }
};

// Head: acc + bias, scattered back to latent layout (unpatchify).  Row
// = slot * L + token (token = (f, h, w) row-major on the patch grid);
// columns c*4 .. c*4+3 are the 2x2 patch (dy, dx) of channel c.  The slot's
// output latent is out + slot_id[slot] * D.
struct EpiHead {
  float* out; const int* slot_id; const float* bias; int L, gh, gw, F, H, Wd; long D;
  struct Pre { int slot; };
  CS_DEV Pre pre(int row, int) const { return {slot_id[row / L]}; }
  CS_DEV void operator()(int row, int col0, const float* v, const Pre& p) const {
    const int c = col0 >> 2;
    const int tok = row % L;
    const int f = tok / (gh * gw), rem = tok - f * gh * gw;
    const int hh = rem / gw, ww = rem - hh * gw;
    float* dst = out + (long)p.slot * D + (((long)c * F + f) * H + 2 * hh) * Wd + 2 * ww;
    *reinterpret_cast<float2*>(dst) = make_float2(v[0], v[1]);
    *reinterpret_cast<float2*>(dst + Wd) = make_float2(v[2], v[3]);
  }
};

}  // namespace cs
