// Attention launchers: tile shapes per element type and head size.
#include "attn_kernel.hpp"

namespace cs {

int attn_kv_tile(int dtype_bytes, int head_dim) {
  if (dtype_bytes == 2) return 64;
  return head_dim > 64 ? 32 : 64;
}

static int cu_count() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cus[dev]) {
    int v = 0;
    cus[dev] = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0
                   ? v : 256;
  }
  return cus[dev];
}

// fp32: 32 QB queries per workgroup, keys split over four waves.
template <int DH, int QB, int OCC>
static hipError_t launch_flash_f32_qb(const AttnArgs<float>& a, hipStream_t st) {
  constexpr int NW = 4;
  const long nwg = (long)cdiv(a.lq, 32 * QB) * a.heads * a.n_streams;
  if (nwg * 64 * NW > 0xFFFFFFFFL) return hipErrorInvalidConfiguration;
  // 16-byte rows of q, k and o; every 32-key block of V^T inside its padded row
  if (a.q_ld % 4 || a.k_ld % 4 || a.o_ld % 4 || a.vt_ld % 4 || a.vt_ld < round_up(a.lk, 32))
    return hipErrorInvalidValue;
  if (a.kv_sel)
    hipLaunchKernelGGL((k_flash_f32<DH, QB, NW, OCC, true>), dim3((unsigned)nwg), dim3(64 * NW), 0, st, a);
  else
    hipLaunchKernelGGL((k_flash_f32<DH, QB, NW, OCC, false>), dim3((unsigned)nwg), dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

// Head dims 32 and 64: 64 queries per workgroup where that takes less than 1 / 1.85
// of the rounds of the CUs that 32 take (time of a round 41 and 75 us at head dim 64
// and 2,048 keys; 4 heads of 1, 2, 3, 4 and 8 streams: 45, 89, 127, 166 and 326 us with
// 32 queries, 80, 82, 148, 149 and 293 with 64), and the keys are more than one
// 32-key block per wave.  Results are bitwise the same.
template <int DH, int OCC1, int OCC2>
static hipError_t launch_flash_f32(const AttnArgs<float>& a, hipStream_t st) {
  const long cus = cu_count(), sh = (long)a.heads * a.n_streams;
  const int r1 = cdiv(cdiv(a.lq, 32) * sh, cus), r2 = cdiv(cdiv(a.lq, 64) * sh, cus);
  if (a.lk > 128 && 1.85 * r2 < r1) return launch_flash_f32_qb<DH, 2, OCC2>(a, st);
  return launch_flash_f32_qb<DH, 1, OCC1>(a, st);
}

// bf16, head dim 32: XOR-swizzled direct-to-LDS tiles of 64 keys in a
// 4-deep ring, one 32-query block per wave.
template <int DH, int QB, int NW, int OCC>
static hipError_t launch_flash_dl(const AttnArgs<bf16>& a, hipStream_t st) {
  constexpr int KVT = 64, STAGES = 4;
  const long nwg = (long)cdiv(a.lq, NW * QB * 32) * a.heads * a.n_streams;
  if (nwg * 64 * NW > 0xFFFFFFFFL) return hipErrorInvalidConfiguration;
  // buffer ranges and offsets are 32-bit byte counts
  if ((long)a.lk * a.k_ld * 2 > 0x7FFFFFFFL || (long)DH * a.vt_ld * 2 > 0x7FFFFFFFL)
    return hipErrorInvalidValue;
  if (a.vt_ld < round_up(a.lk, KVT)) return hipErrorInvalidValue;
  if (a.kv_sel)
    hipLaunchKernelGGL((k_flash_dl<DH, QB, KVT, NW, OCC, STAGES, true>), dim3((unsigned)nwg),
                       dim3(64 * NW), 0, st, a);
  else
    hipLaunchKernelGGL((k_flash_dl<DH, QB, KVT, NW, OCC, STAGES, false>), dim3((unsigned)nwg),
                       dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

// bf16, head dims 64 and 128: padded-row tiles of 64 keys in a 3-deep ring (4
// waves: 4-deep), 105 to 140 KB of LDS at 128: one workgroup per CU.  12 waves
// of 32 queries (three per SIMD) are the fastest shape per query; 8 (two per
// SIMD) and 4 (one) take 256 and 128 instead of 384 queries per workgroup,
// which matters when the grid is a few rounds of the CUs long or shorter than
// one: at one 32,760-token stream of 12 heads, 1032 twelve-wave workgroups fill
// 256 CUs 4.03 times while 1536 eight-wave ones fill them exactly six times.
// Each wave's arithmetic is the same in all shapes (same key order, same
// per-wave rescale decisions), so the outputs are bitwise equal and the choice
// never changes a result.
template <int DH, int NW, int OCC, int STAGES, bool EARLY>
static hipError_t launch_flash_pad_nw(const AttnArgs<bf16>& a, hipStream_t st) {
  const long nwg = (long)cdiv(a.lq, NW * 32) * a.heads * a.n_streams;
  if (nwg * 64 * NW > 0xFFFFFFFFL) return hipErrorInvalidConfiguration;
  if (a.kv_sel)
    hipLaunchKernelGGL((k_flash_pad<DH, NW, OCC, STAGES, EARLY, true>), dim3((unsigned)nwg), dim3(64 * NW), 0, st, a);
  else
    hipLaunchKernelGGL((k_flash_pad<DH, NW, OCC, STAGES, EARLY, false>), dim3((unsigned)nwg), dim3(64 * NW), 0, st,
                       a);
  return hipGetLastError();
}

template <int DH>
static hipError_t launch_flash_pad(const AttnArgs<bf16>& a, hipStream_t st) {
  if ((long)a.lk * a.k_ld * 2 > 0x7FFFFFFFL || (long)DH * a.vt_ld * 2 > 0x7FFFFFFFL)
    return hipErrorInvalidValue;
  // every 64-key tile of V^T must lie inside its padded row; outputs are
  // stored 16 bytes at a time
  if (a.vt_ld < round_up(a.lk, 64) || a.o_ld % 8 || a.o_ss % 8) return hipErrorInvalidValue;
  // Estimated time: rounds of the CUs x queries per workgroup x time per query
  // against 12 waves; a partly filled last round costs at least 0.7 of a full one.
  // In whole rounds (49,152 tokens, 12 heads of 128) 12, 8 and 4 waves take 11.1,
  // 12.1 and 17.4 ms: 9% and 57% more.  8 waves are weighted with 6% instead, for
  // their last rounds: at 2 x 32,760 tokens, 12 whole rounds of 8 waves and 8.06 of
  // 12, they take 10.8 against 10.9 ms, at 4 x 32,760 tokens of 4 x 64 heads 4.2
  // against 4.7.  Over 40 shapes (96 to 49,152 tokens, 1 to 8 streams, 4, 12 and 40
  // heads of 64 and 128) the choice costs 0.2% on average against the best of the
  // three, with 9% in its place 0.5%.
  const long cus = cu_count(), sh = (long)a.heads * a.n_streams;
  auto cost = [&](int queries, double per_query) {
    const long nwg = (long)cdiv(a.lq, queries) * sh;
    const double r = (double)(nwg % cus) / (double)cus;
    return ((double)(nwg / cus) + (r > 0 ? 0.7 + 0.3 * r : 0.0)) * queries * per_query;
  };
  const double t12 = cost(384, 1.0), t8 = cost(256, 1.06), t4 = cost(128, 1.55);
  if (t4 < t8 && t4 < t12) return launch_flash_pad_nw<DH, 4, 1, 4, false>(a, st);
  if (t8 < t12) return launch_flash_pad_nw<DH, 8, 2, 3, (DH > 64)>(a, st);
  return launch_flash_pad_nw<DH, 12, 3, 3, false>(a, st);
}

template <>
hipError_t flash_attention<bf16>(const AttnArgs<bf16>& a, int head_dim, hipStream_t st) {
  if (a.lq <= 0 || a.n_streams <= 0) return hipSuccess;
  switch (head_dim) {
    case 128: return launch_flash_pad<128>(a, st);
    case 64: return launch_flash_pad<64>(a, st);
    case 32: return launch_flash_dl<32, 1, 4, 1>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <>
hipError_t flash_attention<float>(const AttnArgs<float>& a, int head_dim, hipStream_t st) {
  if (a.lq <= 0 || a.n_streams <= 0) return hipSuccess;
  switch (head_dim) {
    case 128: return launch_flash_f32_qb<128, 1, 1>(a, st);
    case 64: return launch_flash_f32<64, 2, 2>(a, st);
    case 32: return launch_flash_f32<32, 4, 3>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace cs
