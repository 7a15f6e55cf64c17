// Passes over a BF16 A on the matrix cores (mixed-precision range finder):
// C[M x L] (FP32) = op(A) Xb with A and Xb in BF16 and FP32 accumulation,
// v_mfma_f32_16x16x32_bf16.  The skinny operand arrives in FP32 or FP64 and is
// rounded to BF16 (to nearest even) and transposed (Xt = X^T, rup(L, 16) x K, k
// contiguous) by convert_bf16_kernel before the pass; everything after the
// pass (CholeskyQR, Jacobi, pivoted QR) stays in FP64.  The product itself is
// the narrow-type pass kernel of gemm_lowp.h.
#include "gemm_lowp.h"

namespace rsvd {
namespace {

// RNE rounding of an FP32 value to BF16 bits (NaN kept quiet)
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Xt[c * ldo + k] = bf16(x) (MODE 0) or bf16(x - bf16(x)) (MODE 1: the low
// part of a two-term BF16 split; the subtraction is exact in FP32), x =
// X[k][c] rounded to FP32, for c < cols, k < rows; the padding k in [rows,
// ldo) is zero.  One 64 x 64 tile per workgroup passes through LDS, so that
// the reads (c contiguous) and the writes (k contiguous) are both coalesced.
constexpr int TT = 64;

template <typename T, int MODE>
__global__ __launch_bounds__(256) void convert_bf16_kernel(const T* __restrict__ in, int64_t ldi,
                                                           int64_t rows, int cols,
                                                           uint16_t* __restrict__ out,
                                                           int64_t ldo) {
  __shared__ uint16_t tile[TT][TT + 2];
  const int64_t k0 = (int64_t)blockIdx.x * TT;
  const int c0 = blockIdx.y * TT;
  const int lo = threadIdx.x & 63, hi = threadIdx.x >> 6;
  for (int i = hi; i < TT; i += 4) {
    const int64_t k = k0 + i;
    const int c = c0 + lo;
    uint16_t v = 0;
    if (k < rows && c < cols) {
      const float x = (float)in[k * ldi + c];
      if (MODE == 0) {
        v = to_bf16(x);
      } else {
        const float h = __uint_as_float((uint32_t)to_bf16(x) << 16);
        v = to_bf16(x - h);
      }
    }
    tile[i][lo] = v;
  }
  __syncthreads();
  for (int i = hi; i < TT; i += 4) {
    const int c = c0 + i;
    const int64_t k = k0 + lo;
    if (c < cols && k < ldo) out[(int64_t)c * ldo + k] = tile[lo][i];
  }
}

}  // namespace

size_t gemm_bf16_part_bytes(int64_t M, int64_t K, int64_t L, int ncu) {
  return lowp::part_bytes(lowp::plan(2, M, K, L, ncu));
}

hipError_t launch_gemm_bf16(bool trans, const uint16_t* A, int64_t lda, const uint16_t* Xt,
                            int64_t ldx, float* C, int64_t ldc, int64_t M, int64_t K, int64_t L,
                            int ncu, void* part, size_t part_cap, bool accumulate,
                            hipStream_t s) {
  if (M <= 0 || L <= 0) return hipSuccess;
  // whole 16-byte chunks of A and Xt
  if (K <= 0 || lda % 8 || ldx % 8 || (reinterpret_cast<uintptr_t>(A) & 15) ||
      (reinterpret_cast<uintptr_t>(Xt) & 15))
    return hipErrorInvalidValue;
  lowp::Args g;
  g.A = reinterpret_cast<const uint8_t*>(A); g.lda = lda * 2;
  g.X = reinterpret_cast<const uint8_t*>(Xt); g.ldx = ldx * 2;
  g.C = C; g.ldc = ldc;
  g.M = M; g.K = K; g.L = L;
  g.part = static_cast<float*>(part);
  g.xs = nullptr;
  g.rs = nullptr;
  g.accumulate = accumulate ? 1 : 0;
  return trans ? lowp::launch<2, true>(g, ncu, part_cap, s)
               : lowp::launch<2, false>(g, ncu, part_cap, s);
}

hipError_t launch_bf16_residual(const float* X, int64_t ldx, int64_t rows, int cols,
                                uint16_t* out, int64_t ldo, hipStream_t s) {
  if (cols <= 0 || ldo <= 0) return hipSuccess;
  const dim3 grid((unsigned)cdiv(ldo, TT), (unsigned)cdiv(cols, TT));
  hipLaunchKernelGGL((convert_bf16_kernel<float, 1>), grid, dim3(256), 0, s, X, ldx, rows, cols,
                     out, ldo);
  return hipGetLastError();
}

hipError_t launch_convert_bf16(bool in_f32, const void* in, int64_t ldi, int64_t rows, int cols,
                               uint16_t* out, int64_t ldo, hipStream_t s) {
  if (cols <= 0 || ldo <= 0) return hipSuccess;
  const dim3 grid((unsigned)cdiv(ldo, TT), (unsigned)cdiv(cols, TT));
  if (in_f32)
    hipLaunchKernelGGL((convert_bf16_kernel<float, 0>), grid, dim3(256), 0, s, (const float*)in,
                       ldi, rows, cols, out, ldo);
  else
    hipLaunchKernelGGL((convert_bf16_kernel<double, 0>), grid, dim3(256), 0, s,
                       (const double*)in, ldi, rows, cols, out, ldo);
  return hipGetLastError();
}

}  // namespace rsvd
