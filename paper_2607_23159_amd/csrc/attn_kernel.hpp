// Flash attention for gfx950: softmax(q k^T / sqrt(dh)) v per (stream, head),
// non-causal, online softmax in fp32, MFMA for both products.
//
// Work split.  bf16: a workgroup of NW waves shares each K/V tile, staged
// through LDS; each wave owns 32 queries, and the hardware overlaps one wave's
// softmax (VALU) with another's matrix products.  fp32: the waves of a
// workgroup share 32 queries and split the keys.
//
// Orientation.  Each wave computes the
// transposed scores S^T = K Q^T (A = K tile from LDS, B = Q^T held in
// registers for the whole key loop), so that after the softmax the
// probabilities P^T already sit in the B-operand layout of the second
// product O^T = V^T P^T (A = V^T).  The MFMA's contraction index may visit
// keys in any order as long as both operands agree: accumulator register j of
// lane l holds row 8(j/4) + 4(l/32) + j%4 of a 32-key block.  No shuffle of P
// through LDS is needed.
//
// The softmax row of query q lives in lanes l and l^32 (16 keys each per
// 32-key block), so row maxima and sums need one cross-lane exchange.
//
// Keys past lk are masked to -inf in the last tile; K rows past lk are read as
// zeros or clamped, and V^T columns past lk must be finite (the runtime
// zero-fills the padding of every V^T buffer).
#pragma once
#include "kernels.hpp"

namespace cs {

constexpr float RESCALE_LOG2 = 8.0f;

// OCC is the number of waves per SIMD the register budget is sized for.
// CROSS distinguishes the cross-attention instantiation (text keys) from the
// self-attention one, so that profiles report them separately.
//
// ---------------------------------------------------------------------------
// fp32.  A 32 x 32 score block takes 32 DH cycles of products against 256 DH
// bytes of K and V, so the matrix pipe is the limit even with every fragment
// read straight from L2: no LDS staging, no barriers, each wave on its own.
// At the sizes fp32 is used at the chip is nearly empty, so the NW waves of a
// workgroup share 32 queries and split the keys (wave w takes 32-key blocks w,
// w + NW, ...), and their partial softmax states are merged through LDS at the
// end in the fixed order of the waves.  The split depends on lk alone, never on
// the batch.  Each wave loads the next block's K under the value product and V
// under the score product, 16 bytes per lane (four consecutive channels of K
// and Q, four consecutive keys of V^T: the contraction visits both operands in
// the same permuted order).
//
// Two streams of 384 tokens, 12 x 128 heads: 46 us (self) and 54 us (512 text
// keys), against 69 and 87 us with 128-query workgroups staged through LDS; four
// of 256 tokens, 4 x 32 heads: 7.1 us against 15.6.
//
// A fragment load of 32 rows touches 32 lines for 32 bytes each, and at head dims
// 32 and 64 these loads, not the products, set the pace once the chip is full.
// There a wave then takes QB = 2 blocks of 32 queries per K and V fragment (each
// block's arithmetic is the same, so results are bitwise those of QB = 1): 4 x
// 24,000 tokens, 4 x 64 heads 20.4 -> 18.6 ms, 8 x 16,384 tokens, 4 x 32 heads
// 10.0 -> 9.0 ms (18.5 and 8.8 with the LDS-staged workgroups).  At head dim 128
// two blocks do not fit the registers; from some 10,000 queries on the staged
// workgroups were faster there (32,760 queries: 512 keys 1.00 against 1.20 ms,
// self 53.9 against 55.3 ms, 2% of it).
// ---------------------------------------------------------------------------
template <int DH, int QB, int NW, int OCC, bool CROSS>
__global__ __launch_bounds__(64 * NW, OCC) void k_flash_f32(AttnArgs<float> a) {
  typedef Mfma32<float> MF;
  constexpr int NG = DH / 8;      // 8-channel groups of the score product
  constexpr int NDT = DH / 32;    // 32-channel blocks of the output
  constexpr int OLD = DH + 4;     // padded row of a partial output
  __shared__ __attribute__((aligned(16))) float s_o[NW][32 * OLD];
  __shared__ float s_m[QB][NW][32], s_l[QB][NW][32];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int n_qt = (a.lq + 32 * QB - 1) / (32 * QB);
  const int vid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int qt = vid % n_qt, hs = vid / n_qt;
  const int head = hs % a.heads, s = hs / a.heads;
  const int kvs = a.kv_sel ? a.kv_sel[s] : s;
  const int q0 = qt * 32 * QB;

  const float* kb_ = a.k + (long)kvs * a.k_ss + head * DH + 4 * half;
  const float* vb_ = a.vt + (long)kvs * a.vt_ss + ((long)head * DH + l32) * a.vt_ld + 4 * half;

  // lane: query 32 qb + l32, channels 8g + 4 half + e in qf[qb][g][e]
  f32x4 qf[QB][NG];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float* src =
        a.q + (long)s * a.q_ss + (long)min(q0 + 32 * qb + l32, a.lq - 1) * a.q_ld + head * DH + 4 * half;
#pragma unroll
    for (int g = 0; g < NG; ++g) qf[qb][g] = *reinterpret_cast<const f32x4*>(src + 8 * g);
  }
  const int nblk = (a.lk + 31) / 32;
  f32x4 kf[NG];
  auto load_k = [&](int blk) {   // lane: key l32 of the block (past lk: the last one, masked)
    const float* src = kb_ + (long)min(blk * 32 + l32, a.lk - 1) * a.k_ld;
#pragma unroll
    for (int g = 0; g < NG; ++g) kf[g] = *reinterpret_cast<const f32x4*>(src + 8 * g);
  };

  f32x16 o[QB][NDT];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_run[qb] = -INFINITY;
    l_run[qb] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[qb][dt][r] = 0.0f;
  }

  if (wave < nblk) load_k(wave);
  for (int blk = wave; blk < nblk; blk += NW) {
    const int kv0 = blk * 32;
    // lane: channel 32 dt + l32, keys kv0 + 8g + 4 half + e in vf[dt][g][e]
    // (columns past lk are finite padding, met by zero probabilities)
    f32x4 vf[NDT][4];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        vf[dt][g] = *reinterpret_cast<const f32x4*>(vb_ + (long)dt * 32 * a.vt_ld + kv0 + 8 * g);

    float p[QB][16];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      // S^T = K Q^T; two chains, so that no product waits for the one before
      f32x16 sc[2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[c][r] = 0.0f;
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[e & 1] = MF::mma(kf[g][e], qf[qb][g][e], sc[e & 1]);
      if (qb == QB - 1 && blk + NW < nblk) load_k(blk + NW);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sc[0][r] += sc[1][r];
        if (kv0 + 32 > a.lk && kv0 + acc_row(r, lane) >= a.lk) sc[0][r] = -INFINITY;
      }

      // online softmax.  The running maximum is only raised (and O, l rescaled)
      // when some lane's block maximum exceeds it by more than RESCALE_LOG2;
      // otherwise the stale maximum is kept and probabilities may reach
      // 2^RESCALE_LOG2, which fp32 accumulation carries without loss of relative
      // precision.  The branch is uniform across the wave.
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[0][r]);
      mx = max_lane_pair32(mx) * a.scale_log2;
      if (__any(mx > m_run[qb] + RESCALE_LOG2)) {
        const float m_new = fmaxf(m_run[qb], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        m_run[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[qb][dt][r] *= alpha;
      }
      float lsum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[qb][r] = __builtin_amdgcn_exp2f(fmaf(sc[0][r], a.scale_log2, -m_run[qb]));
        lsum += p[qb][r];
      }
      l_run[qb] += lsum;
    }

    // O^T += V^T P^T: register 4g + e of P^T holds key 8g + 4 half + e
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) o[qb][dt] = MF::mma(vf[dt][g][e], p[qb][4 * g + e], o[qb][dt]);
  }

  // merge: every wave's maximum and sum, then its output scaled to the common
  // maximum (a wave without a block has maximum -inf, sum and output 0)
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 32, WAVE);
    if (half == 0) {
      s_m[qb][wave][l32] = m_run[qb];
      s_l[qb][wave][l32] = l_tot;
    }
  }
  __syncthreads();
  float* dst = a.o + (long)s * a.o_ss + head * DH;
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    float m_all = s_m[qb][0][l32];
#pragma unroll
    for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, s_m[qb][w][l32]);
    float l_all = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l_all += s_l[qb][w][l32] * __builtin_amdgcn_exp2f(s_m[qb][w][l32] - m_all);
    const float f = __builtin_amdgcn_exp2f(m_run[qb] - m_all) / l_all;
    if (qb > 0) __syncthreads();   // the previous block's outputs are read
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {o[qb][dt][4 * g] * f, o[qb][dt][4 * g + 1] * f, o[qb][dt][4 * g + 2] * f,
                         o[qb][dt][4 * g + 3] * f};
        *reinterpret_cast<f32x4*>(&s_o[wave][l32 * OLD + dt * 32 + 8 * g + 4 * half]) = v;
      }
    __syncthreads();
#pragma unroll
    for (int i = tid; i < 32 * DH / 4; i += 64 * NW) {
      const int q = i / (DH / 4), c = 4 * (i % (DH / 4));
      f32x4 v = *reinterpret_cast<const f32x4*>(&s_o[0][q * OLD + c]);
#pragma unroll
      for (int w = 1; w < NW; ++w) v += *reinterpret_cast<const f32x4*>(&s_o[w][q * OLD + c]);
      const int row = q0 + 32 * qb + q;
      if (row < a.lq) *reinterpret_cast<f32x4*>(dst + (long)row * a.o_ld + c) = v;
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 variant with direct global->LDS tile loads.
//
// K and V^T tiles of KVT keys travel from global memory straight into a ring
// of STAGES LDS buffers by buffer loads (no staging registers, no LDS store
// instructions; keys past lk arrive as zeros);
// tile t+STAGES-1 is requested while tile t is processed, and one barrier per
// tile separates the reads of a buffer from its refill.  Rows are unpadded;
// 16-byte chunks are XOR-swizzled so that the fragment reads are free of bank
// conflicts.
//
// V^T is stored in natural key order.  The key order of P^T in the
// accumulators is made to match it instead: the score product reads, for its
// output row u, K row pi(u), where pi swaps bits 2 and 3 of u.  Accumulator
// register j of lane l holds output row u = 8(j/4) + 4(l/32) + j%4, so it
// holds key pi(u) = 16(j/8) + 8(l/32) + j%8, which is exactly element j%8 of
// k-step j/8 of the value product's B operand for lane l.  The K swizzle is
// taken in pi-space, f(r) = swz(pi(r)), so the permuted reads stay
// conflict-free.
// ---------------------------------------------------------------------------
CS_DEV int swap_bits23(int u) { return (u & ~12) | ((u & 4) << 1) | ((u & 8) >> 1); }

template <int DH, int QB, int KVT, int NW, int OCC, int STAGES, bool CROSS>
__global__ __launch_bounds__(64 * NW, OCC) void k_flash_dl(AttnArgs<bf16> a) {
  typedef Mfma32<bf16> MF;
  constexpr int KSTEP = MF::KSTEP;             // 16 keys / channels per MFMA step
  constexpr int CPR_K = DH / 8, RPI_K = 64 / CPR_K;    // K: chunks per row, rows per load
  constexpr int CPR_V = KVT / 8, RPI_V = 64 / CPR_V;   // V^T
  constexpr int K_INST = KVT / RPI_K / NW, V_INST = DH / RPI_V / NW;
  constexpr int PER_TILE = K_INST + V_INST;    // load instructions per wave per tile
  constexpr int K_ELEMS = KVT * DH, STAGE = 2 * KVT * DH;
  constexpr int NKT = KVT / 32, NDT = DH / 32, NKS = DH / KSTEP, NPS = 32 / KSTEP;
  static_assert(K_INST * RPI_K * NW == KVT && V_INST * RPI_V * NW == DH, "tile split");
  static_assert(STAGES >= 3 && STAGES <= 4, "ring depth");
  __shared__ __attribute__((aligned(1024))) bf16 smem[STAGES * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  constexpr int QPW = QB * 32;                 // queries per wave
  const int n_qt = (a.lq + NW * QPW - 1) / (NW * QPW);
  const int vid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int qt = vid % n_qt, hs = vid / n_qt;
  const int head = hs % a.heads, s = hs / a.heads;
  const int kvs = a.kv_sel ? a.kv_sel[s] : s;
  const int q0 = qt * (NW * QPW) + wave * QPW;

  const bf16* qb_ = a.q + (long)s * a.q_ss + head * DH;
  const bf16* kb_ = a.k + (long)kvs * a.k_ss + head * DH;
  const bf16* vb_ = a.vt + (long)kvs * a.vt_ss + (long)head * DH * a.vt_ld;

  // Q^T fragments (B operand), kept for the whole key loop
  typename MF::frag qf[QB][NKS];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int row = min(q0 + qb * 32 + l32, a.lq - 1);
    const bf16* src = qb_ + (long)row * a.q_ld + MF::KPL * half;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[qb][ks] = MF::load(src + ks * KSTEP);
  }
  // all requested before the first is waited for, and waited for before the
  // direct loads, which are counted
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[qb][ks]));

  // per-lane load sources: lane covers row (lane / CPR) of its instruction's
  // rows and physical chunk lane % CPR, i.e. logical chunk phys ^ f(row)
  // Buffer ranges: the lk key rows of this (stream, head), and its DH rows
  // of V^T (padded key length); keys past lk load as zeros and are masked.
  const int k_bytes = (int)(((long)(a.lk - 1) * a.k_ld + DH) * 2);
  const int v_bytes = (int)((long)DH * a.vt_ld * 2);
  int k_off[K_INST], v_off[V_INST];
#pragma unroll
  for (int i = 0; i < K_INST; ++i) {
    const int row = (wave * K_INST + i) * RPI_K + lane / CPR_K;
    k_off[i] = (row * (int)a.k_ld + ((lane % CPR_K) ^ chunk_swz<CPR_K>(swap_bits23(row))) * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < V_INST; ++i) {
    const int row = (wave * V_INST + i) * RPI_V + lane / CPR_V;
    v_off[i] = (row * (int)a.vt_ld + ((lane % CPR_V) ^ chunk_swz<CPR_V>(row)) * 8) * 2;
  }
  auto issue = [&](int tile, int st) {
    const int kv0 = tile * KVT;
    bf16* sk = smem + st * STAGE;
    bf16* sv = sk + K_ELEMS;
#pragma unroll
    for (int i = 0; i < K_INST; ++i)
      buffer_load_lds16(kb_, k_bytes, sk + (wave * K_INST + i) * RPI_K * DH, k_off[i],
                        kv0 * (int)a.k_ld * 2);
#pragma unroll
    for (int i = 0; i < V_INST; ++i)
      buffer_load_lds16(vb_, v_bytes, sv + (wave * V_INST + i) * RPI_V * KVT, v_off[i], kv0 * 2);
  };

  f32x16 o[QB][NDT];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[qb][dt][r] = 0.0f;
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) { m_run[qb] = -INFINITY; l_run[qb] = 0.0f; }

  const int ntiles = (a.lk + KVT - 1) / KVT;
#pragma unroll
  for (int t = 0; t < STAGES - 1; ++t)
    if (t < ntiles) issue(t, t);

  // fragment rows: the score product reads K row pi(l32) of each 32-key
  // block; the value product reads V^T row (channel) l32 of each 32-block
  const int k_frag_row = swap_bits23(l32);

  for (int t = 0; t < ntiles; ++t) {
    // tile t has landed once at most min(rem, STAGES-2) later tiles are in flight
    const int rem = ntiles - 1 - t;
    if (rem >= STAGES - 2) wait_vm_barrier<(STAGES - 2) * PER_TILE>();
    else if (STAGES == 4 && rem == 1) wait_vm_barrier<PER_TILE>();
    else wait_vm_barrier<0>();
    if (t + STAGES - 1 < ntiles) issue(t + STAGES - 1, (t + STAGES - 1) % STAGES);
    const bf16* sk = smem + (t % STAGES) * STAGE;
    const bf16* sv = sk + K_ELEMS;
    const int kv0 = t * KVT;

    // S^T = K Q^T (rows in pi order)
    f32x16 sc[NKT][QB];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[kt][qb][r] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        const int row = kt * 32 + k_frag_row;
        const int c = 2 * ks + half;
        typename MF::frag kf = MF::load(sk + row * DH + (c ^ chunk_swz<CPR_K>(kt * 32 + l32)) * 8);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) sc[kt][qb] = MF::mma(kf, qf[qb][ks], sc[kt][qb]);
      }
    }
    // every V^T fragment of the tile is requested before the softmax, whose
    // arithmetic then hides the read latency of the value product
    typename MF::frag vf[NKT][NPS][NDT];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int row = dt * 32 + l32;
          const int c = 4 * kt + 2 * ps + half;
          vf[kt][ps][dt] = MF::load(sv + row * KVT + (c ^ chunk_swz<CPR_V>(row)) * 8);
        }
    if (kv0 + KVT > a.lk) {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kv0 + kt * 32 + swap_bits23(acc_row(r, lane));
          if (key >= a.lk)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) sc[kt][qb][r] = -INFINITY;
        }
    }

    // online softmax with lazy rescaling (see k_flash_f32); P^T packed into
    // B-operand fragments, row sums over the rounded operands
    typename MF::frag pf[QB][NKT][NPS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[kt][qb][r]);
      mx = max_lane_pair32(mx) * a.scale_log2;
      if (__any(mx > m_run[qb] + RESCALE_LOG2)) {
        const float m_new = fmaxf(m_run[qb], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        m_run[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[qb][dt][r] *= alpha;
      }
      float lsum = 0.0f;
      const bf16x2 one = {(bf16)1.0f, (bf16)1.0f};
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
          p[r] = __builtin_amdgcn_exp2f(fmaf(sc[kt][qb][r], a.scale_log2, -m_run[qb]));
#pragma unroll
        for (int ps = 0; ps < NPS; ++ps) {
          typename MF::frag f;
#pragma unroll
          for (int i = 0; i < 8; ++i) f[i] = (bf16)p[ps * 8 + i];
          pf[qb][kt][ps] = f;
#pragma unroll
          for (int i = 0; i < 8; i += 2) {
            const bf16x2 pr = {f[i], f[i + 1]};
            lsum = __builtin_amdgcn_fdot2_f32_bf16(pr, one, lsum, false);
          }
        }
      }
      l_run[qb] += lsum;
    }

    // O^T += V^T P^T
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) o[qb][dt] = MF::mma(vf[kt][ps][dt], pf[qb][kt][ps], o[qb][dt]);
  }

  // normalise and store O[q][head*DH + channel]
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 32, WAVE);
    const float inv = 1.0f / l_tot;
    const int row = q0 + qb * 32 + l32;
    if (row < a.lq) {
      bf16* dst = a.o + (long)s * a.o_ss + (long)row * a.o_ld + head * DH;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int ch = dt * 32 + 8 * g + 4 * half;
          bf16x4 q;
#pragma unroll
          for (int r = 0; r < 4; ++r) q[r] = (bf16)(o[qb][dt][4 * g + r] * inv);
          *reinterpret_cast<bf16x4*>(dst + ch) = q;
        }
    }
  }
}


// O^T accumulators of a wave's 32 queries, normalised and stored as row
// query l32 of dst (row stride o_ld).  A lane holds 4 consecutive channels per
// group of 8 and the lane 32 away the other 4: exchanging them between two
// groups (v_permlane32_swap) gives each lane 8 consecutive channels of one
// group, one 16-byte store instead of two of 8 bytes.  Measured with the Q
// loads behind the first tile's: 32,760 queries x 512 keys x 12 heads, 8
// streams 1045 -> 988 us, one stream 159 -> 144 us; 384 x 512, one stream 19.9
// -> 17.6 us; neutral over 32,760 keys (bitwise equal).
template <int NDT>
CS_DEV void store_o_rows(const f32x16 (&o)[NDT], float inv, bf16* dst, int half, bool valid) {
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
      union { bf16x4 v; uint32_t u[2]; } x, y;   // groups g and g + 1
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x.v[r] = (bf16)(o[dt][4 * g + r] * inv);
        y.v[r] = (bf16)(o[dt][4 * g + 4 + r] * inv);
      }
      const auto w0 = __builtin_amdgcn_permlane32_swap(x.u[0], y.u[0], false, false);
      const auto w1 = __builtin_amdgcn_permlane32_swap(x.u[1], y.u[1], false, false);
      if (valid) *reinterpret_cast<uint4*>(dst + dt * 32 + 8 * (g + half)) = make_uint4(w0[0], w1[0], w0[1], w1[1]);
    }
}

// ---------------------------------------------------------------------------
// bf16 variant with padded LDS rows (head dims 64 and 128).
//
// The direct loads place any 16-byte chunk of global memory anywhere in the
// 1 KB an instruction fills, so the tiles are stored with padded rows instead
// of a swizzle: a K row of DH/8 chunks takes DH/8 + 1 chunk slots and a V^T
// row of 8 chunks takes 9.  The extra slot of a row receives a copy of the
// row's last chunk (same cache line, no extra traffic) and is never read.
// Row strides of 272 and 144 bytes spread 16 consecutive rows over all 64
// banks, and since no chunk index is permuted every fragment read of a tile is
// one base register plus a compile-time offset: the per-read address
// arithmetic of the swizzled layout disappears from the key loop.  Stage t of
// the ring holds K (64 x 17 chunks = 17 KB) then V^T (DH x 9 chunks), all
// whole 1 KB load instructions, spread over the waves (the first few waves
// issue one more than the others).  Results are bitwise those of k_flash_dl.
//
// Occupancy.  With 12 waves of 32 queries the V^T fragments are read inside
// the value product, each just before its MFMA, instead of all ahead of the
// softmax: that saves 64 registers and brings a wave to 160, so three waves
// fit per SIMD, and the third wave hides LDS latency better than early reads
// (measured 4% faster at 32,760 tokens).  With 8 waves (two per SIMD, 256
// registers) and head dim 128 a tile's K fragments are requested together and its
// V^T fragments ahead of the softmax (EARLY: 5711 -> 5583 us, one 32,760-token
// stream of 12 heads); at head dim 64, with half the products per tile to cover
// them, that costs (two 16,384-token streams of 4 heads 555 us without, 580 with,
// one of 32,760 1101 and 1151).  4
// waves, one per SIMD, are for grids that leave CUs idle otherwise: 384 tokens
// x 12 heads 12.4 us against 14.8 with 8 waves and 19.0 with 12.
//
// The first tile is requested before Q, and all of Q before any of it is waited
// for, so that their latencies overlap.  (One wait after each of the eight loads:
// 40 us for 4 x 32,760 queries, 4 x 64 heads and 19 keys, 34.5 without; longer key
// loops do not show it.)
// ---------------------------------------------------------------------------
template <int DH, int NW, int OCC, int STAGES, bool EARLY, bool CROSS>
__global__ __launch_bounds__(64 * NW, OCC) void k_flash_pad(AttnArgs<bf16> a) {
  typedef Mfma32<bf16> MF;
  typedef typename MF::frag frag;
  constexpr int KVT = 64, KSTEP = MF::KSTEP;
  constexpr int CK = DH / 8 + 1, CV = KVT / 8 + 1;   // chunk slots per padded row
  constexpr int KRS = CK * 16, VRS = CV * 16;        // padded row strides (bytes)
  constexpr int K_INSTR = KVT * CK / 64, V_INSTR = DH * CV / 64;
  static_assert(K_INSTR * 64 == KVT * CK && V_INSTR * 64 == DH * CV, "whole 1 KB loads");
  constexpr int KB = K_INSTR * 1024, STAGE = KB + V_INSTR * 1024;
  constexpr int TOT = K_INSTR + V_INSTR;             // load instructions per tile
  constexpr int NPW = (TOT + NW - 1) / NW;           // per wave, for the first NBUSY waves
  constexpr int NBUSY = TOT - (NPW - 1) * NW;        // the others issue NPW - 1
  constexpr int NKT = KVT / 32, NDT = DH / 32, NKS = DH / KSTEP, NPS = 32 / KSTEP;
  static_assert(STAGES >= 3 && STAGES <= 4, "ring depth");
  __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: loads use SGPR ranges
  const int half = lane >> 5, l32 = lane & 31;
  const int n_qt = (a.lq + NW * 32 - 1) / (NW * 32);
  const int vid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int qt = vid % n_qt, hs = vid / n_qt;
  const int head = hs % a.heads, s = hs / a.heads;
  const int kvs = a.kv_sel ? a.kv_sel[s] : s;
  const int q0 = qt * (NW * 32) + wave * 32;
  // With 12 waves, a wave past the last query only loads: a head's last tile has
  // up to 11 of them (8 x 1,560 tokens: 153 -> 145 us, 4 x 3,120: 255 -> 248 us,
  // 27,280 tokens: 1%).  With 8 and 4 waves the branch in the key loop costs the
  // full tiles more (1.4% and 4%) than the few idle waves take.
  const bool active = NW < 12 || q0 < a.lq;

  const bf16* qb_ = a.q + (long)s * a.q_ss + head * DH;
  const bf16* kb_ = a.k + (long)kvs * a.k_ss + head * DH;
  const bf16* vb_ = a.vt + (long)kvs * a.vt_ss + (long)head * DH * a.vt_ld;

  // load instruction i of this wave fills slots [64g, 64g + 64) of the stage,
  // g = wave + NW*i; slot p of the K part is row p / CK, chunk p % CK (the
  // padding slot takes the row's last chunk), likewise for V^T.  Keys past
  // lk load as zeros (K range) or are finite padding (V^T) and are masked.
  const int k_bytes = (int)(((long)(a.lk - 1) * a.k_ld + DH) * 2);
  const int v_bytes = (int)((long)DH * a.vt_ld * 2);
  int voff[NPW];
#pragma unroll
  for (int i = 0; i < NPW; ++i) {
    const int g = wave + NW * i;
    if (g < K_INSTR) {
      const int p = g * 64 + lane, row = p / CK, ch = min(p % CK, CK - 2);
      voff[i] = (row * (int)a.k_ld + ch * 8) * 2;
    } else {
      const int p = (g - K_INSTR) * 64 + lane, row = p / CV, ch = min(p % CV, CV - 2);
      voff[i] = (row * (int)a.vt_ld + ch * 8) * 2;
    }
  }
  const bool busy = wave < NBUSY;
  auto issue = [&](int tile, int st) {
    const int kv0 = tile * KVT;
    char* base = smem + st * STAGE;
#pragma unroll
    for (int i = 0; i < NPW; ++i) {
      const int g = wave + NW * i;
      if (i < NPW - 1 || busy) {
        if (g < K_INSTR)
          buffer_load_lds16(kb_, k_bytes, base + g * 1024, voff[i], kv0 * (int)a.k_ld * 2);
        else
          buffer_load_lds16(vb_, v_bytes, base + g * 1024, voff[i], kv0 * 2);
      }
    }
  };

  f32x16 o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
  float m_run = -INFINITY, l_run = 0.0f;

  const int ntiles = (a.lk + KVT - 1) / KVT;
  issue(0, 0);
  // Q^T fragments (B operand), kept for the whole key loop
  frag qf[NKS];
  {
    const int row = min(q0 + l32, a.lq - 1);
    const bf16* src = qb_ + (long)row * a.q_ld + MF::KPL * half;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = MF::load(src + ks * KSTEP);
    // all requested before the first is waited for, and waited for before the
    // direct loads of the later tiles, which are counted
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[ks]));
  }
#pragma unroll
  for (int t = 1; t < STAGES - 1; ++t)
    if (t < ntiles) issue(t, t);

  // fragment bases: the score product reads K row pi(l32) of each 32-key
  // block (pi swaps bits 2 and 3, see k_flash_dl), the value product V^T row
  // (channel) l32 of each 32-channel block
  const int lane_k = swap_bits23(l32) * KRS + half * 16;
  const int lane_v = KB + l32 * VRS + half * 16;
  const bf16x2 one = {(bf16)1.0f, (bf16)1.0f};

  for (int t = 0; t < ntiles; ++t) {
    // tile t has landed once at most min(rem, STAGES-2) later tiles are in flight
    const int inflight = min(ntiles - 1 - t, STAGES - 2);
    if (busy) {
      if (inflight >= 2) wait_vm_barrier<2 * NPW>();
      else if (inflight == 1) wait_vm_barrier<NPW>();
      else wait_vm_barrier<0>();
    } else {
      if (inflight >= 2) wait_vm_barrier<2 * (NPW - 1)>();
      else if (inflight == 1) wait_vm_barrier<NPW - 1>();
      else wait_vm_barrier<0>();
    }
    if (t + STAGES - 1 < ntiles) issue(t + STAGES - 1, (t + STAGES - 1) % STAGES);
    if (NW >= 12 && !active) continue;
    const char* pk = smem + (t % STAGES) * STAGE + lane_k;
    const char* pv = smem + (t % STAGES) * STAGE + lane_v;
    const int kv0 = t * KVT;

    // S^T = K Q^T (rows in pi order)
    frag kf[EARLY ? NKS : 1][NKT];
    if constexpr (EARLY) {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
          kf[ks][kt] = MF::load(reinterpret_cast<const bf16*>(pk + kt * 32 * KRS + ks * 32));
    }
    f32x16 sc[NKT];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[kt][r] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        if constexpr (EARLY)
          sc[kt] = MF::mma(kf[ks][kt], qf[ks], sc[kt]);
        else
          sc[kt] = MF::mma(MF::load(reinterpret_cast<const bf16*>(pk + kt * 32 * KRS + ks * 32)), qf[ks], sc[kt]);
      }
    auto load_v = [&](int kt, int ps, int dt) {
      return MF::load(reinterpret_cast<const bf16*>(pv + dt * 32 * VRS + kt * 64 + ps * 32));
    };
    frag vf[EARLY ? NKT : 1][NPS][NDT];
    if constexpr (EARLY) {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt) vf[kt][ps][dt] = load_v(kt, ps, dt);
    }
    if (kv0 + KVT > a.lk) {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kv0 + kt * 32 + swap_bits23(acc_row(r, lane));
          if (key >= a.lk) sc[kt][r] = -INFINITY;
        }
    }

    // online softmax with lazy rescaling (see k_flash_f32)
    frag pf[NKT][NPS];
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[kt][r]);
    mx = max_lane_pair32(mx) * a.scale_log2;
    if (__any(mx > m_run + RESCALE_LOG2)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
    float lsum = 0.0f;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      float p[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(sc[kt][r], a.scale_log2, -m_run));
#pragma unroll
      for (int ps = 0; ps < NPS; ++ps) {
        frag f;
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = (bf16)p[ps * 8 + i];
        pf[kt][ps] = f;
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          const bf16x2 pr = {f[i], f[i + 1]};
          lsum = __builtin_amdgcn_fdot2_f32_bf16(pr, one, lsum, false);
        }
      }
    }
    l_run += lsum;

    // O^T += V^T P^T
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int ps = 0; ps < NPS; ++ps)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          if constexpr (EARLY)
            o[dt] = MF::mma(vf[kt][ps][dt], pf[kt][ps], o[dt]);
          else
            o[dt] = MF::mma(load_v(kt, ps, dt), pf[kt][ps], o[dt]);
        }
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, WAVE);
  const int row = q0 + l32;
  store_o_rows(o, 1.0f / l_tot, a.o + (long)s * a.o_ss + (long)row * a.o_ld + head * DH, half, row < a.lq);
}

}  // namespace cs
