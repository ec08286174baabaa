// GEMM launchers: tile shapes per element type and the fused epilogues.
#include "gemm_kernel.hpp"
#include "gemm_tile.hpp"

namespace cs {

// ------------------------------------------------------------- launchers
// Direct-to-LDS kernels on 16x16 MFMAs, tile shape chosen per launch
// (choose_tile in bf16, F32_64_TILES in fp32), K slices of 128 bytes, tile
// groups of 4 tile-rows; all shapes of a type sum in the same order (bitwise
// equal results).  K must be a multiple of a slice.
template <typename T> constexpr int SLICE_K = 128 / (int)sizeof(T);
constexpr int GROUP_M = 4;

// ------------------------------------------------------- weight tiling
// Weights for the direct-load kernels: [N][K] fp32 row-major -> blocks of
// W_BLOCK_ROWS rows x SLICE_K columns in the compute type, block (tn, kt) at
// ((tn * K/SLICE_K + kt) * W_BLOCK_ROWS * SLICE_K) elements; inside a block row
// r holds its 8 chunks of 16 bytes with logical chunk c at physical position
// c ^ gemm_swz(r), the LDS layout of the kernels.  Rows past N are zero.
template <typename T>
__global__ __launch_bounds__(256) void k_tile_weight(const float* __restrict__ src, int N, int K,
                                                     T* __restrict__ dst, long n_chunks) {
  constexpr int BN = W_BLOCK_ROWS, BK = SLICE_K<T>, CPR = 8, CH = BK / CPR;
  const long q = (long)blockIdx.x * 256 + threadIdx.x;
  if (q >= n_chunks) return;
  const long blk = q / (BN * CPR);
  const int within = (int)(q - blk * BN * CPR);
  const int r = within / CPR, p = within % CPR;
  const int nk = K / BK;
  const int tn = (int)(blk / nk), kt = (int)(blk % nk);
  const int n = tn * BN + r;
  const int k0 = kt * BK + (p ^ gemm_swz(r)) * CH;
  typename Mfma16<T>::chunk v;
#pragma unroll
  for (int e = 0; e < CH; ++e) v[e] = n < N ? to_t<T>(src[(long)n * K + k0 + e]) : to_t<T>(0.0f);
  *reinterpret_cast<typename Mfma16<T>::chunk*>(dst + q * CH) = v;
}

long gemm_tiled_weight_elems(int N, int K) { return round_up(N, W_BLOCK_ROWS) * (long)K; }

template <typename T>
hipError_t gemm_tile_weight(const float* src, int N, int K, T* dst, hipStream_t st) {
  if (N <= 0 || K % SLICE_K<T> != 0) return hipErrorInvalidValue;
  const long n_chunks = gemm_tiled_weight_elems(N, K) / (16 / (long)sizeof(T));
  hipLaunchKernelGGL(k_tile_weight<T>, dim3((unsigned)cdiv(n_chunks, 256)), dim3(256), 0, st, src, N, K, dst,
                     n_chunks);
  return hipGetLastError();
}

// Residual updates read and write the fp32 residual stream in their epilogue,
// which then weighs several times a bf16 store.
template <class Epi> struct EpiIsResidual : std::false_type {};
template <int G> struct EpiIsResidual<EpiResidual<G>> : std::true_type {};
template <int G, typename T> struct EpiIsResidual<EpiResidualStore<G, T>> : std::true_type {};

struct GemmBatch { int n; long w_stride; };

template <int BM, int BN, int OCC, int PD, class Epi>
static void launch_w4(const bf16* A, long lda, const bf16* W, int M, int N, int K, GemmBatch b, const Epi& epi,
                      hipStream_t st) {
  const unsigned tiles = (unsigned)((long)cdiv(M, BM) * cdiv(N, BN));
  hipLaunchKernelGGL((k_gemm_w4<BM, BN, OCC, GROUP_M, PD, Epi>), dim3(tiles, (unsigned)b.n), dim3(256), 0, st, A, lda,
                     W, M, N, K, b.w_stride, epi);
}

template <typename T, int BM, int BN, int WGM, int WGN, int SL, int STAGES, int OCC, class Epi>
static void launch_ring(const T* A, long lda, const T* W, int M, int N, int K, GemmBatch b, const Epi& epi,
                        hipStream_t st) {
  const unsigned tiles = (unsigned)((long)cdiv(M, BM) * cdiv(N, BN));
  hipLaunchKernelGGL((k_gemm_ring<T, BM, BN, WGM, WGN, SL, STAGES, OCC, GROUP_M, Epi>), dim3(tiles, (unsigned)b.n),
                     dim3(64 * WGM * WGN), 0, st, A, lda, W, M, N, K, b.w_stride, epi);
}

// fp32: 64 x 64 tiles from six per CU on (768 x 8960 x 1536: 180 us against
// 183 with 32 x 32, 3000 x 8960 x 1536: 629 against 661, half the loads), below
// that 32 x 32 (768 x 1536 x 8960, 288 tiles of 64 x 64: 183 against 267 us).
constexpr long F32_64_TILES = 6 * 256;

// W is in the tiled layout (row stride K).
template <typename T, class Epi>
static hipError_t launch(const T* A, long lda, const T* W, int M, int N, int K, Epi epi, hipStream_t st,
                         GemmBatch b = {1, 0}) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (b.n < 1 || b.n > MAX_BATCH || (b.n > 1 && !EpiBatched<Epi>::value)) return hipErrorInvalidValue;
  if (K <= 0 || K % SLICE_K<T> != 0 || N % 4 != 0) return hipErrorInvalidValue;
  // buffer ranges are 32-bit byte counts: k_gemm_w4's of a whole W block row,
  // k_gemm_ring's of a tile's rows of A
  const long row_bytes = std::max(lda, (long)K) * (long)sizeof(T);
  if ((sizeof(T) == 2 ? W_BLOCK_ROWS : 32) * row_bytes > 0x7FFFFFFFL) return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 2) {
    constexpr bool RES = EpiIsResidual<Epi>::value;
    // residual operands in flight per wave: with one wave per SIMD nothing
    // else hides their latency, with two workgroups per CU half as many do
    constexpr int PD = RES ? 8 : 2, PD2 = RES ? 4 : 2;
    switch (choose_tile(M, N, K, b.n, RES)) {
      case W4_256x256: launch_w4<256, 256, 1, PD>(A, lda, W, M, N, K, b, epi, st); break;
      case W4_224x256: launch_w4<224, 256, 1, PD>(A, lda, W, M, N, K, b, epi, st); break;
      case W4_160x256: launch_w4<160, 256, 1, PD>(A, lda, W, M, N, K, b, epi, st); break;
      case W4_192x256: launch_w4<192, 256, 1, PD>(A, lda, W, M, N, K, b, epi, st); break;
      case W4_128x128: launch_w4<128, 128, 2, PD2>(A, lda, W, M, N, K, b, epi, st); break;
      case W4_64x64: launch_w4<64, 64, 3, 2>(A, lda, W, M, N, K, b, epi, st); break;
      case RING_128x128: launch_ring<T, 128, 128, 2, 4, 1, 4, 2>(A, lda, W, M, N, K, b, epi, st); break;
      case RING_64x128: launch_ring<T, 64, 128, 2, 4, 2, 3, 2>(A, lda, W, M, N, K, b, epi, st); break;
      case RING_64x64: launch_ring<T, 64, 64, 2, 4, 2, 4, 2>(A, lda, W, M, N, K, b, epi, st); break;
      case RING_32x64: launch_ring<T, 32, 64, 1, 4, 2, 3, 2>(A, lda, W, M, N, K, b, epi, st); break;
      default: launch_ring<T, 32, 32, 2, 2, 2, 4, 2>(A, lda, W, M, N, K, b, epi, st);
    }
  } else {
    if ((long)cdiv(M, 64) * cdiv(N, 64) * b.n >= F32_64_TILES && 64 * row_bytes <= 0x7FFFFFFFL)
      launch_ring<T, 64, 64, 2, 4, 2, 2, 4>(A, lda, W, M, N, K, b, epi, st);
    else
      launch_ring<T, 32, 32, 2, 2, 2, 2, 4>(A, lda, W, M, N, K, b, epi, st);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t gemm_store(const T* A, long lda, const T* W, int M, int N, int K, const float* bias,
                      int act, T* out, long ldo, hipStream_t st) {
  if (!bias) return hipErrorInvalidValue;
  if (act == 1) return launch<T>(A, lda, W, M, N, K, EpiStore<T, 1>{out, ldo, bias}, st);
  return launch<T>(A, lda, W, M, N, K, EpiStore<T, 0>{out, ldo, bias}, st);
}

template <typename T>
hipError_t gemm_store_batch(const T* A, long lda, const T* W, long w_stride, int n, int M, int N, int K,
                            const float* bias, long bias_stride, T* out, long ldo, long out_stride,
                            hipStream_t st) {
  if (!bias) return hipErrorInvalidValue;
  return launch<T>(A, lda, W, M, N, K, EpiStore<T, 0>{out, ldo, bias, out_stride, bias_stride}, st, {n, w_stride});
}

template <typename T>
hipError_t gemm_store_t_batch(const T* A, long lda, const T* W, long w_stride, int n, int M, int N, int K,
                              const float* bias, long bias_stride, T* out, long ldo, long out_stride,
                              hipStream_t st) {
  if (!bias) return hipErrorInvalidValue;
  return launch<T>(A, lda, W, M, N, K, EpiStoreT<T>{out, ldo, bias, out_stride, bias_stride}, st, {n, w_stride});
}

template <typename T>
hipError_t gemm_qkv(const T* A, const T* W, int M, int d, const float* bias, int L, T* qk, T* vt,
                    long vt_ld, hipStream_t st) {
  EpiQKV<T> e{qk, vt, bias, d, L, vt_ld, (long)d * vt_ld};
  return launch<T>(A, d, W, M, 3 * d, d, e, st);
}

template <typename T>
hipError_t gemm_residual(const T* A, long lda, const T* W, int M, int N, int K, const float* bias,
                         const float* gate, float* z, T* y, hipStream_t st) {
  if (!bias) return hipErrorInvalidValue;
  if (y) {
    if (gate) return launch<T>(A, lda, W, M, N, K, EpiResidualStore<1, T>{z, N, bias, gate, y}, st);
    return launch<T>(A, lda, W, M, N, K, EpiResidualStore<0, T>{z, N, bias, nullptr, y}, st);
  }
  if (gate) return launch<T>(A, lda, W, M, N, K, EpiResidual<1>{z, N, bias, gate}, st);
  return launch<T>(A, lda, W, M, N, K, EpiResidual<0>{z, N, bias, nullptr}, st);
}

template <typename T>
hipError_t gemm_patch(const T* A, const T* W, int M, int d, int P, const float* bias, float* z,
                      hipStream_t st) {
  EpiPatch e{z, d, bias};
  return launch<T>(A, P, W, M, d, P, e, st);
}

template <typename T>
hipError_t gemm_head(const T* A, const T* W, int M, int d, int P, const float* bias, float* out,
                     const int* slot_id, int L, int gh, int gw, int F, int H, int Wd, long D,
                     hipStream_t st) {
  EpiHead e{out, slot_id, bias, L, gh, gw, F, H, Wd, D};
  return launch<T>(A, d, W, M, P, d, e, st);
}

#define CS_INST(T)                                                                              \
  template hipError_t gemm_tile_weight<T>(const float*, int, int, T*, hipStream_t);             \
  template hipError_t gemm_store<T>(const T*, long, const T*, int, int, int, const float*, int, \
                                    T*, long, hipStream_t);                                     \
  template hipError_t gemm_store_batch<T>(const T*, long, const T*, long, int, int, int, int,   \
                                          const float*, long, T*, long, long, hipStream_t);     \
  template hipError_t gemm_store_t_batch<T>(const T*, long, const T*, long, int, int, int, int, \
                                            const float*, long, T*, long, long, hipStream_t);   \
  template hipError_t gemm_qkv<T>(const T*, const T*, int, int, const float*, int, T*, T*,     \
                                  long, hipStream_t);                                           \
  template hipError_t gemm_residual<T>(const T*, long, const T*, int, int, int, const float*,  \
                                       const float*, float*, T*, hipStream_t);                  \
  template hipError_t gemm_patch<T>(const T*, const T*, int, int, int, const float*, float*,   \
                                    hipStream_t);                                               \
  template hipError_t gemm_head<T>(const T*, const T*, int, int, int, const float*, float*,    \
                                   const int*, int, int, int, int, int, int, long, hipStream_t);
CS_INST(bf16)
CS_INST(float)
#undef CS_INST

}  // namespace cs
