// Passes over an FP8 A on the matrix cores (mixed-precision range finder with
// A stored as FP8 E4M3 codes and one FP32 scale per column, A ~ A8 diag(s)).
//
//   Y = A X    = A8 (diag(s) X)          : the column scales sit on the
//                                          reduction index, so they are folded
//                                          into the skinny operand before it is
//                                          quantized;
//   Z = A^T X  = diag(s) (A8^T X)        : they are an epilogue row scale.
// The skinny operand X' (diag(s) X, or X) is quantized per output column:
// t_j = max_k |X'_kj| / 448, X8 = e4m3(X' / t) (nearest, ties to even), and
// the product is (op(A8) X8) diag(t) (diag(s) in the transposed case), with
// v_mfma_scale_f32_16x16x128_f8f6f4 on E4M3 x E4M3 (unit block scales) and
// FP32 accumulation.  A two-term split X' ~ t X8 + t2 X8lo (X8lo the codes of
// the residual with their own column scales t2) keeps about twice the
// significand bits in the last projection, as the BF16 passes do.
//
// The product itself is the narrow-type pass kernel of gemm_lowp.h, which
// applies the scales to its results.
#include "gemm_lowp.h"

namespace rsvd {
namespace {

// ---- the skinny operand in FP8 ---------------------------------------------
//
// E4M3 code of an FP32 value (nearest, ties to even, saturated to +-448; NaN
// to 0x7F): with e the binary exponent of |y| (at least -6, the smallest
// normal), the spacing is 2^(e-3); the rounded magnitude is re-read as
// (exponent, significand) fields.
__device__ __forceinline__ uint8_t e4m3_from_float(float y) {
  if (y != y) return 0x7F;
  const uint32_t sign = y < 0.f ? 0x80u : 0u;
  const float a = fabsf(y);
  uint32_t code;
  if (a >= 448.f) {
    code = 0x7E;
  } else {
    int e;
    (void)frexpf(a, &e);                       // a = f 2^e, f in [0.5, 1)
    const int E = max(e - 1, -6);
    const float step = ldexpf(1.f, E - 3);
    const float q = fminf(rintf(a / step) * step, 448.f);
    if (q >= 0x1.0p-6f) {
      int e2;
      (void)frexpf(q, &e2);
      const int E2 = e2 - 1;
      const uint32_t mant = (uint32_t)rintf((ldexpf(q, -E2) - 1.f) * 8.f);
      code = ((uint32_t)(E2 + 7) << 3) | mant;
    } else {
      code = (uint32_t)rintf(q * 512.f);
    }
  }
  return (uint8_t)(code | sign);
}

__device__ __forceinline__ float e4m3_to_float(uint8_t c) {
  const int e = (c >> 3) & 0xF, m = c & 7;
  const float v = e == 0 ? (float)m * 0x1.0p-9f : ldexpf(1.f + (float)m * 0.125f, e - 7);
  return (c & 0x80) ? -v : v;
}

// Element (k, c) of the operand being quantized: X'(k, c) = s_k X(k, c) (s may
// be null), or in residual mode the part that the first term leaves,
// X'(k, c) - t0_c dec(X8_0[c][k]).
template <typename TX>
__device__ __forceinline__ float xval(const TX* X, int64_t ldx, const float* s, int64_t k, int c,
                                      const uint8_t* prev, int64_t ldp, const float* t0) {
  float v = (float)X[k * ldx + c];
  if (s) v *= s[k];
  if (prev) v -= t0[c] * e4m3_to_float(prev[(int64_t)c * ldp + k]);
  return v;
}

// tmax[c] = max_k |X'(k, c)| as FP32 bits (non-negative floats order as
// integers); tmax zeroed beforehand.  Block: 64 columns x 4 row groups.
template <typename TX>
__global__ __launch_bounds__(256) void colmax_kernel(const TX* __restrict__ X, int64_t ldx,
                                                     int64_t rows, int cols, const float* s,
                                                     const uint8_t* prev, int64_t ldp,
                                                     const float* t0, uint32_t* tmax) {
  __shared__ float part[4][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rg = threadIdx.x >> 6;
  // four independent maxima (a maximum does not depend on the order), so
  // that four loads per thread are in flight
  float m0 = 0.f, m1 = 0.f, m2 = 0.f, m3 = 0.f;
  if (c < cols) {
    const int64_t st = (int64_t)gridDim.y * 4;
    int64_t k = blockIdx.y * 4 + rg;
    for (; k + 3 * st < rows; k += 4 * st) {
      m0 = fmaxf(m0, fabsf(xval(X, ldx, s, k, c, prev, ldp, t0)));
      m1 = fmaxf(m1, fabsf(xval(X, ldx, s, k + st, c, prev, ldp, t0)));
      m2 = fmaxf(m2, fabsf(xval(X, ldx, s, k + 2 * st, c, prev, ldp, t0)));
      m3 = fmaxf(m3, fabsf(xval(X, ldx, s, k + 3 * st, c, prev, ldp, t0)));
    }
    for (; k < rows; k += st) m0 = fmaxf(m0, fabsf(xval(X, ldx, s, k, c, prev, ldp, t0)));
  }
  part[rg][threadIdx.x & 63] = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
  __syncthreads();
  // one atomic per column and workgroup
  if (rg == 0 && c < cols) {
    const int i = threadIdx.x;
    const float m = fmaxf(fmaxf(part[0][i], part[1][i]), fmaxf(part[2][i], part[3][i]));
    atomicMax(tmax + c, __float_as_uint(m));
  }
}

// t[c] = tmax[c] / 448 (1 for a zero column)
__global__ __launch_bounds__(256) void colscale_kernel(const uint32_t* tmax, int cols, float* t) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= cols) return;
  const float m = __uint_as_float(tmax[c]);
  t[c] = m > 0.f ? m / 448.f : 1.f;
}

// Xt[c][k] = e4m3(X'(k, c) / t[c]); padding k in [rows, ldo) zero.  One 64 x
// 64 tile per workgroup: s_k X(k, c) goes through LDS (read with c
// contiguous), the residual term and the code are formed with k contiguous
// (the reads of prev and the writes of Xt), so all three are coalesced.  The
// arithmetic is xval's, in its order.
constexpr int TT = 64;

template <typename TX>
__global__ __launch_bounds__(256) void encode_kernel(const TX* __restrict__ X, int64_t ldx,
                                                     int64_t rows, int cols, const float* s,
                                                     const uint8_t* prev, int64_t ldp,
                                                     const float* t0, const float* t,
                                                     uint8_t* __restrict__ Xt, int64_t ldo) {
  __shared__ float tile[TT][TT + 1];
  const int64_t k0 = (int64_t)blockIdx.x * TT;
  const int c0 = blockIdx.y * TT;
  const int lo = threadIdx.x & 63, hi = threadIdx.x >> 6;
  for (int i = hi; i < TT; i += 4) {
    const int64_t k = k0 + i;
    const int c = c0 + lo;
    float v = 0.f;
    if (k < rows && c < cols) {
      v = (float)X[k * ldx + c];
      if (s) v *= s[k];
    }
    tile[i][lo] = v;
  }
  __syncthreads();
  for (int i = hi; i < TT; i += 4) {
    const int c = c0 + i;
    const int64_t k = k0 + lo;
    if (c >= cols || k >= ldo) continue;
    uint8_t code = 0;
    if (k < rows) {
      float v = tile[lo][i];
      if (prev) v -= t0[c] * e4m3_to_float(prev[(int64_t)c * ldp + k]);
      code = e4m3_from_float(v / t[c]);
    }
    Xt[(int64_t)c * ldo + k] = code;
  }
}

__global__ void zero_u32_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

template <typename TX>
hipError_t quant_x(const TX* X, int64_t ldx, int64_t rows, int cols, const float* s,
                   const uint8_t* prev, int64_t ldp, const float* t0, uint8_t* Xt, int64_t ldo,
                   float* t, uint32_t* tmax, hipStream_t st) {
  const unsigned cb = (unsigned)cdiv(cols, 256);
  hipLaunchKernelGGL(zero_u32_kernel, dim3(cb), dim3(256), 0, st, tmax, cols);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned gx = (unsigned)cdiv(cols, 64);
  int64_t gy = cdiv(rows, 256);
  if (gy > 256) gy = 256;
  if (gy < 1) gy = 1;
  hipLaunchKernelGGL(colmax_kernel<TX>, dim3(gx, (unsigned)gy), dim3(256), 0, st, X, ldx, rows,
                     cols, s, prev, ldp, t0, tmax);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(colscale_kernel, dim3(cb), dim3(256), 0, st, tmax, cols, t);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const dim3 grid((unsigned)cdiv(ldo, TT), (unsigned)cdiv(cols, TT));
  hipLaunchKernelGGL(encode_kernel<TX>, grid, dim3(256), 0, st, X, ldx, rows, cols, s, prev, ldp,
                     t0, t, Xt, ldo);
  return hipGetLastError();
}

}  // namespace

size_t gemm_f8_part_bytes(int64_t M, int64_t K, int64_t L, int ncu) {
  return lowp::part_bytes(lowp::plan(1, M, K, L, ncu));
}

hipError_t launch_gemm_f8(bool trans, const uint8_t* A, int64_t lda, const uint8_t* Xt,
                          int64_t ldx, const float* xscale, const float* rscale, float* C,
                          int64_t ldc, int64_t M, int64_t K, int64_t L, int ncu, void* part,
                          size_t part_cap, bool accumulate, hipStream_t s) {
  if (M <= 0 || L <= 0) return hipSuccess;
  // whole 16-byte chunks of A and Xt
  if (K <= 0 || lda % 16 || ldx % 16 || (reinterpret_cast<uintptr_t>(A) & 15) ||
      (reinterpret_cast<uintptr_t>(Xt) & 15))
    return hipErrorInvalidValue;
  lowp::Args g;
  g.A = A; g.lda = lda; g.X = Xt; g.ldx = ldx; g.C = C; g.ldc = ldc;
  g.M = M; g.K = K; g.L = L;
  g.part = static_cast<float*>(part);
  g.xs = xscale;
  g.rs = rscale;
  g.accumulate = accumulate ? 1 : 0;
  return trans ? lowp::launch<1, true>(g, ncu, part_cap, s)
               : lowp::launch<1, false>(g, ncu, part_cap, s);
}

hipError_t launch_quant_x_f8(bool x_f32, const void* X, int64_t ldx, int64_t rows, int cols,
                             const float* rowscale, const uint8_t* prev, int64_t ldp,
                             const float* t0, uint8_t* Xt, int64_t ldo, float* t, uint32_t* tmax,
                             hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (x_f32)
    return quant_x(static_cast<const float*>(X), ldx, rows, cols, rowscale, prev, ldp, t0, Xt, ldo,
                   t, tmax, s);
  return quant_x(static_cast<const double*>(X), ldx, rows, cols, rowscale, prev, ldp, t0, Xt, ldo,
                 t, tmax, s);
}

}  // namespace rsvd
