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
// v_mfma_f32_16x16x128_f8f6f4 on E4M3 x E4M3 (no block scales) and FP32
// accumulation.  A two-term split X' ~ t X8 + t2 X8lo (X8lo the codes of
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
// E4M3 codes of four FP32 values (nearest, ties to even, saturated to +-448;
// NaN to 0x7F), packed with the first in the low byte.  The conversion
// instruction rounds to nearest even down to the subnormals; its input is
// clamped, since it does not saturate (checked against the definition over
// every FP32 value: only -0 differs, in its sign).
__device__ __forceinline__ float e4m3_clamp(float y) {
  return fminf(fmaxf(y, -448.f), 448.f);           // (NaN is put back below)
}
__device__ __forceinline__ uint32_t e4m3_pack(const float (&y)[4]) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_clamp(y[0]), e4m3_clamp(y[1]), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_clamp(y[2]), e4m3_clamp(y[3]), w, true);
  uint32_t u = (uint32_t)w;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (y[j] != y[j]) u = (u & ~(0xFFu << (8 * j))) | (0x7Fu << (8 * j));
  return u;
}

// value of code J of a word of four
template <int J> __device__ __forceinline__ float e4m3_value(uint32_t w) {
  return __builtin_amdgcn_cvt_f32_fp8((int)w, J);
}

// The operand being quantized: X'(k, c) = s_k X(k, c) (s may be null), or for
// the second term the part that the first leaves, X'(k, c) - t0_c dec(X8_0[c][k]).
template <int J> __device__ __forceinline__ float residual(float x, float t0, uint32_t codes) {
  return x - t0 * e4m3_value<J>(codes);
}

// t = tmax / 448 (1 for a zero column)
__device__ __forceinline__ float col_scale(uint32_t tmax) {
  const float m = __uint_as_float(tmax);
  return m > 0.f ? m / 448.f : 1.f;
}

// tmax[c] = max_k |X'(k, c)| as FP32 bits (non-negative floats order as
// integers; a maximum does not depend on the order); tmax zeroed beforehand.
// Block: 64 columns x 4 row groups, eight loads in flight per thread, one
// atomic per column and workgroup.
template <typename TX>
__global__ __launch_bounds__(256) void colmax_kernel(const TX* __restrict__ X, int64_t ldx,
                                                     int64_t rows, int cols,
                                                     const float* __restrict__ s,
                                                     uint32_t* tmax) {
  constexpr int U = 8;
  __shared__ float part[4][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cc = c < cols ? c : cols - 1;
  float m[U];
#pragma unroll
  for (int u = 0; u < U; ++u) m[u] = 0.f;
  const int64_t st = (int64_t)gridDim.y * 4;
  for (int64_t k = blockIdx.y * 4 + rg; k < rows; k += U * st) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t ku = k + u * st < rows ? k + u * st : k;   // (a repeated row)
      float v = (float)X[ku * ldx + cc];
      if (s) v *= s[ku];
      m[u] = fmaxf(m[u], fabsf(v));
    }
  }
#pragma unroll
  for (int u = 1; u < U; ++u) m[0] = fmaxf(m[0], m[u]);
  part[rg][threadIdx.x & 63] = m[0];
  __syncthreads();
  if (rg == 0 && c < cols) {
    const int i = threadIdx.x;
    const float v = fmaxf(fmaxf(part[0][i], part[1][i]), fmaxf(part[2][i], part[3][i]));
    atomicMax(tmax + c, __float_as_uint(v));
  }
}

// Xt[c][k] = e4m3(X'(k, c) / t[c]), t from tmax (and written by the first k
// block); padding k in [rows, ldo) zero (ldo a multiple of 16).  One tile of
// 128 k x 64 columns per workgroup: s_k X(k, c) goes through LDS (read with c
// contiguous), then a thread forms four codes of consecutive k (one word of
// prev and of Xt), so every access is coalesced.  With rmax (RMAX), the column
// maxima of what these codes leave go there: the second term needs no pass
// of its own for them (and the workgroup takes ENC_TILES tiles, for fewer
// atomics on the few column words: 286 -> 117 us at 65536 x 576).
constexpr int TK = 128, TC = 64;
constexpr int ENC_TILES = 4;

template <typename TX, bool PREV, bool RMAX>
__global__ __launch_bounds__(256) void encode_kernel(const TX* __restrict__ X, int64_t ldx,
                                                     int64_t rows, int cols,
                                                     const float* __restrict__ s,
                                                     const uint8_t* __restrict__ prev,
                                                     int64_t ldp, const float* __restrict__ t0,
                                                     const uint32_t* __restrict__ tmax, float* t,
                                                     uint8_t* __restrict__ Xt, int64_t ldo,
                                                     uint32_t* rmax) {
  __shared__ float tile[TK][TC + 1];
  constexpr int CI = TC / 8;                      // columns per thread
  const int c0 = blockIdx.y * TC;
  const int lo = threadIdx.x & 63, hi = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cl = min(c0 + lo, cols - 1);
  const int kq = threadIdx.x & 31, cg = threadIdx.x >> 5;   // four k values, column group
  if (blockIdx.x == 0 && hi == 0 && c0 + lo < cols) t[c0 + lo] = col_scale(tmax[c0 + lo]);
  float m[CI];
#pragma unroll
  for (int x = 0; x < CI; ++x) m[x] = 0.f;
  constexpr int NTILE = RMAX ? ENC_TILES : 1;
  for (int ti = 0; ti < NTILE; ++ti) {
    const int64_t k0 = ((int64_t)blockIdx.x * NTILE + ti) * TK;
    if (k0 >= ldo) break;                         // (the whole workgroup)
    if (ti > 0) __syncthreads();
#pragma unroll 16
    for (int i = hi; i < TK; i += 4) {
      const int64_t k = min(k0 + i, rows - 1);    // (rows past the end are not used)
      float v = (float)X[k * ldx + cl];
      if (s) v *= s[k];
      tile[i][lo] = v;
    }
    __syncthreads();
    const int64_t k = k0 + 4 * kq;
#pragma unroll
    for (int x = 0; x < CI; ++x) {
      const int i = cg + 8 * x, c = c0 + i;
      if (c >= cols) break;
      const float tc = col_scale(tmax[c]);
      const float p0 = PREV ? t0[c] : 0.f;
      uint32_t pw = 0u;
      if (PREV && k < ldp) pw = *reinterpret_cast<const uint32_t*>(prev + (int64_t)c * ldp + k);
      float v[4], y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = tile[4 * kq + j][i];
      if (PREV) {
        v[0] = residual<0>(v[0], p0, pw);
        v[1] = residual<1>(v[1], p0, pw);
        v[2] = residual<2>(v[2], p0, pw);
        v[3] = residual<3>(v[3], p0, pw);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[j] = k + j < rows ? v[j] : 0.f;
        y[j] = v[j] / tc;
      }
      const uint32_t code = e4m3_pack(y);
      if (k < ldo) *reinterpret_cast<uint32_t*>(Xt + (int64_t)c * ldo + k) = code;
      if (RMAX) {
        m[x] = fmaxf(m[x], fmaxf(fabsf(residual<0>(v[0], tc, code)),
                                 fabsf(residual<1>(v[1], tc, code))));
        m[x] = fmaxf(m[x], fmaxf(fabsf(residual<2>(v[2], tc, code)),
                                 fabsf(residual<3>(v[3], tc, code))));
      }
    }
  }
  if (RMAX) {
#pragma unroll
    for (int x = 0; x < CI; ++x) {
      const int c = c0 + cg + 8 * x;
#pragma unroll
      for (int d = 1; d < 32; d <<= 1) m[x] = fmaxf(m[x], __shfl_xor(m[x], d, 32));
      if (kq == 0 && c < cols) atomicMax(rmax + c, __float_as_uint(m[x]));
    }
  }
}

__global__ void zero_u32_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

template <typename TX>
hipError_t quant_x(const TX* X, int64_t ldx, int64_t rows, int cols, const float* s,
                   const uint8_t* prev, int64_t ldp, const float* t0, uint8_t* Xt, int64_t ldo,
                   float* t, uint32_t* tmax, uint32_t* rmax, hipStream_t st) {
  hipError_t e;
  if (!prev) {
    const unsigned cb = (unsigned)cdiv(cols, 256);
    hipLaunchKernelGGL(zero_u32_kernel, dim3(cb), dim3(256), 0, st, tmax, cols);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (rmax) {
      hipLaunchKernelGGL(zero_u32_kernel, dim3(cb), dim3(256), 0, st, rmax, cols);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const unsigned gx = (unsigned)cdiv(cols, 64);
    int64_t gy = cdiv(rows, 128);
    if (gy > 256) gy = 256;
    hipLaunchKernelGGL(colmax_kernel<TX>, dim3(gx, (unsigned)gy), dim3(256), 0, st, X, ldx, rows,
                       cols, s, tmax);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const dim3 grid((unsigned)cdiv(ldo, rmax ? TK * ENC_TILES : TK), (unsigned)cdiv(cols, TC));
  if (prev)
    hipLaunchKernelGGL((encode_kernel<TX, true, false>), grid, dim3(256), 0, st, X, ldx, rows, cols,
                       s, prev, ldp, t0, tmax, t, Xt, ldo, nullptr);
  else if (rmax)
    hipLaunchKernelGGL((encode_kernel<TX, false, true>), grid, dim3(256), 0, st, X, ldx, rows, cols,
                       s, nullptr, 0, nullptr, tmax, t, Xt, ldo, rmax);
  else
    hipLaunchKernelGGL((encode_kernel<TX, false, false>), grid, dim3(256), 0, st, X, ldx, rows,
                       cols, s, nullptr, 0, nullptr, tmax, t, Xt, ldo, nullptr);
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
                             uint32_t* rmax, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ldo % 16 || (prev && ldp % 16)) return hipErrorInvalidValue;   // whole words of codes
  if (x_f32)
    return quant_x(static_cast<const float*>(X), ldx, rows, cols, rowscale, prev, ldp, t0, Xt, ldo,
                   t, tmax, rmax, s);
  return quant_x(static_cast<const double*>(X), ldx, rows, cols, rowscale, prev, ldp, t0, Xt, ldo,
                 t, tmax, rmax, s);
}

}  // namespace rsvd
