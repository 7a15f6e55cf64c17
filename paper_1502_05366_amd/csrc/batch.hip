// Batched randomized SVD of many small FP32 matrices in persistent launches:
// Alg. 5 (RSVD version II) with re-orthonormalization after every product (Sec.
// 3.2, s = 1), applied to each matrix of the batch on its own.
// The matrices are independent, as the blocks of Alg. 8 are, so each one is
// the work of a single workgroup:
//
//   Omega_i (n x l, Philox stream 0, batch = the matrix's index);
//   Y = A Omega; q times { Q = orth(Y); Z = A^T Q; Z = orth(Z); Y = A Z };
//   Q = orth(Y); B^T = A^T Q; Qh = orth(B^T); Rh = Qh^T B^T;
//   Rh = Uh diag(sigma) Vh^T (one-sided Jacobi); U = Q Vh_k, V = Qh Uh_k.
//
// A workgroup of 8 waves pops matrices off a work queue (an atomic counter;
// the host orders the queue by decreasing work) until it is empty, so the
// grid is one workgroup per CU (two where l <= 64) whatever the batch size, and
// no workgroup ever waits for another.  Per matrix:
//  * passes over A (FP32 MFMA 16x16x4, FP32 accumulation): 128- or 256-row
//    (column for A^T) tiles of A loaded straight into registers, 64- or 32-deep
//    chunks of the skinny operand double-buffered in LDS;
//  * orth = CholeskyQR2 in FP64: Gram X^T X on FP64 MFMA (upper blocks,
//    rows split over the waves), Cholesky (one barrier per step) and the
//    inverse of R (four lanes per column) in LDS, Q = Y R^{-1} on FP64 MFMA;
//    a pivot below 1e-13 G_jj marks a dependent column (unit row of R, info
//    bit 1), which after the first pass is replaced by a fresh Gaussian
//    column (Philox stream 7) for the second pass to orthonormalize, as the
//    single-matrix orth does; a non-finite pivot sets info bit 8; the second
//    pass is skipped when the first already left ||Q^T Q - I||_F <= 2^-30,
//    far below the FP32 rounding of the bases;
//  * the Jacobi SVD of the l x l factor in LDS (the rotations of the
//    single-matrix small SVD, one column pair per 16 lanes);
//  * U and V on FP64 MFMA, written in FP32.
// Skinny matrices live in a per-workgroup slot of the workspace (L2-resident
// for the sizes of a batch), small factors in LDS (l <= 80).  A slot holds three,
// each used in place for what follows it: Y and its basis Q; Omega, Z and its basis;
// the FP64 first pass of an orth and, of the last one, its FP64 basis Qh.
#include "common.h"
#include "internal.h"
#include "jacobi_dev.h"
#include "philox_dev.h"

namespace rsvd {
namespace {

constexpr int BNT = 512;             // 8 waves
// Pass shapes (the batch autotuner picks one per matrix): a pass over A
// takes tiles of TM = 128 RPW rows of A (A^T: columns), RPW 16-row blocks
// per wave, and KC-deep chunks, A in registers and the skinny operand double
// buffered in LDS.
//   variant 0: TM = 128, KC = 64;  variant 1: TM = 256, KC = 32;
//   variant 2: TM = 128, KC = 32.
// LDS row stride of the skinny chunk (floats): lane (li, lk) reads row lk at
// column li, and 80 = 16 mod 64 puts the four rows on distinct banks.
constexpr int XLD = 80;              // skinny chunk row stride, KC x lp
constexpr int STAGE_FLOATS = 2 * 64 * XLD;
constexpr double ETA_DEP = 1e-13;
constexpr int JAC_MAX_SWEEPS = 40;

// LDS of a workgroup: the passes stage the skinny operand over the whole union;
// the small factorizations use a, b (lp x lp FP64, stride SL).  Declared at
// namespace scope so that every helper addresses it as LDS even when it is not
// inlined.  Two layouts, ML = 64 and 80 (the largest lp that fits): 68 KB lets two
// workgroups share a compute unit, 105 KB does not.
template <int ML> struct alignas(16) BatchLds {
  static constexpr int SL = ML + 1;              // row stride of the small FP64 matrices
  union {
    struct {
      double a[ML * SL];
      double b[ML * SL];
    } sm;
    float stage[STAGE_FLOATS];
  } u;
  double sig[ML];
  double dgn[ML];
  int depc[ML];        // columns found dependent by the last Cholesky
  int ndep;            // how many
  int nonfinite;       // a non-finite pivot was met (this matrix)
  int flag;
  int item;
};
__shared__ BatchLds<BATCH_SMALL_LP> g_lds_small;
__shared__ BatchLds<BATCH_MAX_LP> g_lds_large;
template <int ML> __device__ __forceinline__ BatchLds<ML>& batch_lds() {
  if constexpr (ML == BATCH_SMALL_LP) return g_lds_small;
  else return g_lds_large;
}
// the LDS layout of a matrix with lp = 16 NB
template <int NB> constexpr int ml_of() {
  return 16 * NB <= BATCH_SMALL_LP ? BATCH_SMALL_LP : BATCH_MAX_LP;
}

__device__ __forceinline__ double to_d(float x) { return (double)x; }
__device__ __forceinline__ double to_d(double x) { return x; }
template <typename T> __device__ __forceinline__ T from_d(double x);
template <> __device__ __forceinline__ float from_d<float>(double x) { return (float)x; }
template <> __device__ __forceinline__ double from_d<double>(double x) { return x; }

// The arguments of a function that is not inlined arrive in vector registers;
// these are the same in every lane.
__device__ __forceinline__ int64_t uniform(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename T> __device__ __forceinline__ T* uniform(T* p) {
  return reinterpret_cast<T*>(uniform((int64_t)reinterpret_cast<intptr_t>(p)));
}

__device__ __forceinline__ float4 ld4(const float* p) {
  return *reinterpret_cast<const float4*>(p);
}

// Omega (n x lp, FP32): column j < l holds normals j*n .. j*n + n-1 of stream
// 0, batch `batch`; columns l .. lp-1 are zero.
template <int ML>   // (a copy per kernel: they differ in registers)
__device__ __noinline__ void b_sketch(float* Om, int64_t n, int l, int lp, uint32_t k0,
                                      uint32_t k1, uint32_t batch) {
  const int tid = threadIdx.x;
  const int64_t total = n * l;
  const int64_t npairs = (total + 1) / 2;
  for (int64_t p = tid; p < npairs; p += BNT) {
    const Words w = philox10((uint32_t)p, (uint32_t)((uint64_t)p >> 32), 0u, batch, k0, k1);
    double z[2];
    box_muller(w, z[0], z[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t t = 2 * p + h;
      if (t < total) {
        const int64_t j = t / n, i = t - (t / n) * n;
        Om[i * lp + j] = (float)z[h];
      }
    }
  }
  if (lp > l) {
    const int pad = lp - l;
    for (int64_t e = tid; e < n * pad; e += BNT) {
      const int64_t i = e / pad;
      Om[i * lp + l + (e - i * pad)] = 0.0f;
    }
  }
  __syncthreads();
}

// 16-byte store (p is 16-byte aligned: every tile stride is a multiple of 4)
__device__ __forceinline__ void st4(float* p, const float4& v) {
  *reinterpret_cast<float4*>(p) = v;
}

// Both passes keep A in registers and the skinny operand X in LDS.  Every
// element of A is used by one wave only, so staging A in LDS (as before) bought
// nothing but its barriers: a chunk of A had to arrive, be stored and be read
// back while nothing else of the pass could run, and one chunk in flight per
// compute unit (32 KB) covers a third of the memory's latency.  Here a wave
// loads the A of its own rows (columns for A^T) straight into the layout of the
// products, two chunks ahead, each register replaced as soon as it is consumed;
// X chunks are double buffered in LDS with one barrier per chunk that waits for
// LDS only, so loads of A stay in flight across it.
//
// Order of the FP32 sums: k ascending in steps of 4.  4096 matrices of up to 2048
// x 1024, k <= 64, one power step, the whole batch: 44.2 -> 36.8 ms.
// Chunks of A in flight per wave: with two workgroups on a compute unit one
// chunk each (and half the registers), otherwise two.
template <int NCB> constexpr int pass_ahead() { return 16 * NCB <= BATCH_SMALL_LP ? 1 : 2; }

// X chunk kc (KC rows x lp; rows >= n are zero) through registers to LDS
template <int NCB, int KC> struct XChunk {
  static constexpr int lp = 16 * NCB, XQ = lp / 4, XN = KC * XQ;
  static constexpr int F4 = (XN + BNT - 1) / BNT;
  float4 v[F4];
  bool in[F4];
  __device__ __forceinline__ void load(const float* X, int64_t n, int64_t kc) {
    const bool past = kc * KC >= n;
    const int64_t r0 = past ? 0 : kc * KC;
#pragma unroll
    for (int u = 0; u < F4; ++u) {
      const int idx = min((int)threadIdx.x + BNT * u, XN - 1);
      // clamped and selected: no branch waits for the load
      const int left = (int)min(n - r0, (int64_t)KC);
      const int r = idx / XQ;
      v[u] = ld4(X + r0 * lp + min(r, left - 1) * lp + (idx % XQ) * 4);
      in[u] = r < left && !past;
    }
  }
  __device__ __forceinline__ void store(float* xs) const {
#pragma unroll
    for (int u = 0; u < F4; ++u) {
      const int idx = threadIdx.x + BNT * u;
      const float4 z = in[u] ? v[u] : make_float4(0.f, 0.f, 0.f, 0.f);
      if (idx < XN) st4(xs + (idx / XQ) * XLD + (idx % XQ) * 4, z);
    }
  }
};

// LDS stores of this wave done, then the workgroup's barrier (outstanding loads
// from memory are not waited for)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// x[c] of lane group g = value (g, c)  ->  x[t] of lane group g = value (t, g)
// (lane groups of 16; a 4 x 4 transposition over the groups)
__device__ __forceinline__ void transpose_groups(float (&x)[4]) {
  auto sw32 = [](float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  auto sw16 = [](float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  sw32(x[0], x[2]);
  sw32(x[1], x[3]);
  sw16(x[0], x[1]);
  sw16(x[2], x[3]);
}

// Y (m x lp) = A X, A m x n (FP32, lda % 4 == 0), X n x lp (FP32), lp = 16 NCB.
// Row tiles of TM (16 RPW rows per wave), KC-deep chunks.  A lane loads 4
// consecutive k of its row (16 bytes); transpose_groups brings them into the
// order of the products.
template <int NCB, int RPW, int KC>
__device__ __noinline__ void b_pass_n(const float* __restrict__ A, int64_t lda, int64_t m,
                                      int64_t n, const float* __restrict__ X,
                                      float* __restrict__ Y) {
  auto& g_lds = batch_lds<ml_of<NCB>()>();
  constexpr int SL = BatchLds<ml_of<NCB>()>::SL;
  (void)SL;
  constexpr int lp = 16 * NCB, TM = 128 * RPW, NG = KC / 16;
  A = uniform(A); X = uniform(X); Y = uniform(Y);
  lda = uniform(lda); m = uniform(m); n = uniform(n);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  float* const xs0 = g_lds.u.stage;
  const int64_t nkc = cdiv(n, KC);
  for (int64_t row0 = 0; row0 < m; row0 += TM) {
    f4 acc[RPW][NCB];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = f4{0.f, 0.f, 0.f, 0.f};
    const float* ar[RPW];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
      ar[rb] = A + min(row0 + (wave * RPW + rb) * 16 + li, m - 1) * lda;
    constexpr int D = pass_ahead<NCB>();
    float4 a[D][NG][RPW];
    // group j of chunk kc: columns kc KC + 16 j + 4 lk .. + 3 of the lane's rows
    auto aload = [&](float4 (&d)[RPW], int64_t kc, int j) {
      const int64_t c = min(kc * KC + 16 * j, lda - 4);
      const int e = min(4 * lk, (int)min(lda - 4 - c, (int64_t)12));
#pragma unroll
      for (int rb = 0; rb < RPW; ++rb) d[rb] = ld4(ar[rb] + c + e);
    };
    XChunk<NCB, KC> x;
    x.load(X, n, 0);
#pragma unroll
    for (int h = 0; h < D; ++h)
#pragma unroll
      for (int j = 0; j < NG; ++j) aload(a[h][j], h, j);
    x.store(xs0);
    x.load(X, n, 1);
    lds_barrier();
    auto chunk = [&](int h, int64_t kc) {      // h = kc mod D
      const int xb = (int)(kc & 1);
      const float* xs = xs0 + xb * (KC * XLD);
      x.store(xs0 + (xb ^ 1) * (KC * XLD));     // chunk kc + 1 (read from the barrier on)
      x.load(X, n, kc + 2);
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        float y[RPW][4];
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb) {
          const float4 v = a[h][j][rb];
          y[rb][0] = v.x; y[rb][1] = v.y; y[rb][2] = v.z; y[rb][3] = v.w;
          if (kc * KC + 16 * j + 16 > n) {     // entries at columns >= n count as zero
#pragma unroll
            for (int c = 0; c < 4; ++c)
              y[rb][c] = kc * KC + 16 * j + 4 * lk + c < n ? y[rb][c] : 0.f;
          }
          transpose_groups(y[rb]);
        }
        aload(a[h][j], kc + D, j);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          float xv[NCB];
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) xv[cb] = xs[(16 * j + 4 * t + lk) * XLD + cb * 16 + li];
#pragma unroll
          for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
              acc[rb][cb] = Mfma<float>::mma(y[rb][t], xv[cb], acc[rb][cb]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      lds_barrier();
    };
    int64_t kc = 0;
    if constexpr (D == 2) {
      for (; kc + 1 < nkc; kc += 2) {
        chunk(0, kc);
        chunk(1, kc + 1);
      }
      if (kc < nkc) chunk(0, kc);
    } else {
      for (; kc < nkc; ++kc) chunk(0, kc);
    }
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t r = row0 + (wave * RPW + rb) * 16 + Mfma<float>::row(lk, v);
          if (r < m) Y[r * lp + cb * 16 + li] = acc[rb][cb][v];
        }
      }
  }
  __syncthreads();
}

// Z (n x lp) = A^T X, A m x n (FP32, lda % 4 == 0), X m x lp (FP32), lp = 16 NCB.
// Tiles of TM columns of A, 16 RPW per wave (block rb of a wave holds every
// RPW-th of them, so a lane loads RPW neighbours), KC-row chunks.
template <int NCB, int RPW, int KC>
__device__ __noinline__ void b_pass_t(const float* __restrict__ A, int64_t lda, int64_t m,
                                      int64_t n, const float* __restrict__ X,
                                      float* __restrict__ Z) {
  auto& g_lds = batch_lds<ml_of<NCB>()>();
  constexpr int SL = BatchLds<ml_of<NCB>()>::SL;
  (void)SL;
  constexpr int lp = 16 * NCB, TM = 128 * RPW, NS = KC / 4;
  A = uniform(A); X = uniform(X); Z = uniform(Z);
  lda = uniform(lda); m = uniform(m); n = uniform(n);
  static_assert(RPW <= 2, "");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  float* const xs0 = g_lds.u.stage;
  const int64_t nkc = cdiv(m, KC);
  const int64_t last = (m - 1) & ~(int64_t)3;            // first row of the last 4-row step
  const int tail = (int)(m - 1 - last);
  for (int64_t col0 = 0; col0 < n; col0 += TM) {
    f4 acc[RPW][NCB];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = f4{0.f, 0.f, 0.f, 0.f};
    // the lane's columns (past the last ones: loaded, not stored)
    const int64_t c0 = min(col0 + (wave * 16 + li) * RPW, lda - RPW);
    const float* const al = A + lk * lda + c0;                     // row lk of a step
    const float* const at = A + min(lk, tail) * lda + c0;          // ... of the last step
    constexpr int D = pass_ahead<NCB>();
    float a[D][NS][RPW];
    auto aload = [&](float (&d)[RPW], int64_t kc, int j) {
      const int64_t r = min(kc * KC + 4 * j, last);
      const float* p = (r == last ? at : al) + r * lda;
      if constexpr (RPW == 2) {
        const float2 v = *reinterpret_cast<const float2*>(p);
        d[0] = v.x;
        d[1] = v.y;
      } else {
        d[0] = *p;
      }
    };
    XChunk<NCB, KC> x;
    x.load(X, m, 0);
#pragma unroll
    for (int h = 0; h < D; ++h)
#pragma unroll
      for (int j = 0; j < NS; ++j) aload(a[h][j], h, j);
    x.store(xs0);
    x.load(X, m, 1);
    lds_barrier();
    auto chunk = [&](int h, int64_t kc) {      // h = kc mod D
      const int xb = (int)(kc & 1);
      const float* xs = xs0 + xb * (KC * XLD);
      x.store(xs0 + (xb ^ 1) * (KC * XLD));
      x.load(X, m, kc + 2);
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        float y[RPW];
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb) y[rb] = a[h][j][rb];
        if (kc * KC + 4 * j + 4 > m) {         // rows >= m count as zero
#pragma unroll
          for (int rb = 0; rb < RPW; ++rb) y[rb] = kc * KC + 4 * j + lk < m ? y[rb] : 0.f;
        }
        float xv[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) xv[cb] = xs[(4 * j + lk) * XLD + cb * 16 + li];
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            acc[rb][cb] = Mfma<float>::mma(y[rb], xv[cb], acc[rb][cb]);
        aload(a[h][j], kc + D, j);
        if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      lds_barrier();
    };
    int64_t kc = 0;
    if constexpr (D == 2) {
      for (; kc + 1 < nkc; kc += 2) {
        chunk(0, kc);
        chunk(1, kc + 1);
      }
      if (kc < nkc) chunk(0, kc);
    } else {
      for (; kc < nkc; ++kc) chunk(0, kc);
    }
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t c = col0 + (wave * 16 + Mfma<float>::row(lk, v)) * RPW + rb;
          if (c < n) Z[c * lp + cb * 16 + li] = acc[rb][cb][v];
        }
      }
  }
  __syncthreads();
}

// a (lp x lp, stride SL) = X^T Y for X, Y rows x lp (FP32 or FP64), on FP64
// MFMA.  Tasks (16x16 block, row slice) are spread over the 8 waves; with
// fewer than 8 blocks the rows are cut into slices whose partial blocks are
// added in slice order.  Eight 4-row steps are loaded before their products.
template <int ML, typename TX, typename TY>
__device__ __noinline__ void b_xty(const TX* __restrict__ X, const TY* __restrict__ Y,
                                   int64_t rows, int lp) {
  auto& g_lds = batch_lds<ML>();
  constexpr int SL = BatchLds<ML>::SL;
  (void)SL;
  X = uniform(X); Y = uniform(Y); rows = uniform(rows);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int nb = lp / 16, nblk = nb * nb;
  const int S = nblk >= 8 ? 1 : 8 / nblk;
  const int ntask = nblk * S;
  const int64_t nsteps = cdiv(rows, 4);
  double* out = g_lds.u.sm.a;
  double* part = out + 32 * SL;     // (sliced only with at most two column blocks)
  for (int task = wave; task < ntask; task += 8) {
    const int b = task / S, sl = task - (task / S) * S;
    const int bi = b / nb, bj = b - (b / nb) * nb;
    const int64_t st0 = sl * nsteps / S, st1 = (sl + 1) * nsteps / S;
    d4 acc = d4{0.0, 0.0, 0.0, 0.0};
    for (int64_t st = st0; st < st1; st += 8) {
      double av[8], bv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        // (clamped, not branched around)
        const int64_t r = min((st + u) * 4 + lk, rows - 1) * lp;
        av[u] = to_d(X[r + bi * 16 + li]);
        bv[u] = to_d(Y[r + bj * 16 + li]);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool ok = st + u < st1 && (st + u) * 4 + lk < rows;
        acc = Mfma<double>::mma(ok ? av[u] : 0.0, ok ? bv[u] : 0.0, acc);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (S == 1)
        out[(bi * 16 + drow(lk, v)) * SL + bj * 16 + li] = acc[v];
      else
        part[task * 256 + drow(lk, v) * 16 + li] = acc[v];
    }
  }
  __syncthreads();
  if (S > 1) {
    for (int e = tid; e < nblk * 256; e += BNT) {
      const int b = e >> 8, rr = (e >> 4) & 15, cc = e & 15;
      const int bi = b / nb, bj = b - (b / nb) * nb;
      double t = 0.0;
      for (int sl = 0; sl < S; ++sl) t += part[(b * S + sl) * 256 + rr * 16 + cc];
      out[(bi * 16 + rr) * SL + bj * 16 + cc] = t;
    }
    __syncthreads();
  }
}

// a (upper 16x16 blocks, stride SL) = X^T X for X rows x lp (FP32 or FP64)
// on FP64 MFMA.  Wave w forms every upper block over its eighth of the rows; the eight partial Grams are added into a in wave order.
template <int NB, typename TX>
__device__ __noinline__ void b_gram(const TX* __restrict__ X, int64_t rows) {
  auto& g_lds = batch_lds<ml_of<NB>()>();
  constexpr int SL = BatchLds<ml_of<NB>()>::SL;
  (void)SL;
  constexpr int lp = 16 * NB, nb = NB;
  X = uniform(X); rows = uniform(rows);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  double* out = g_lds.u.sm.a;
  const int64_t nsteps = cdiv(rows, 4);
  const int64_t st0 = wave * nsteps / 8, st1 = (wave + 1) * nsteps / 8;
  d4 acc[NB][NB];
#pragma unroll
  for (int bi = 0; bi < NB; ++bi)
#pragma unroll
    for (int bj = bi; bj < NB; ++bj) acc[bi][bj] = d4{0.0, 0.0, 0.0, 0.0};
  // U steps at a time, the next U in flight meanwhile (the registers: 128 up to
  // NB = 4); addresses are clamped and steps outside the wave's eighth or past
  // the last row count as zero, so no branch waits for a load
  constexpr int U = NB <= 2 ? 4 : (NB == 4 && sizeof(TX) == 8 ? 1 : 2);
  const int64_t last = (rows - 1) / 4;
  const int off = lk * lp + li, off_last = min(lk, (int)(rows - 1 - 4 * last)) * lp + li;
  TX x0[U][NB], x1[U][NB];
  auto load = [&](TX (&x)[U][NB], int64_t st) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t t = min(st + u, last);
      const TX* p = X + t * (4 * lp);
      const int o = t == last ? off_last : off;
#pragma unroll
      for (int bi = 0; bi < NB; ++bi) x[u][bi] = p[o + bi * 16];
    }
  };
  auto products = [&](const TX (&x)[U][NB], int64_t st) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = st + u < st1 && (st + u) * 4 + lk < rows;
      double xv[NB];
#pragma unroll
      for (int bi = 0; bi < NB; ++bi) xv[bi] = ok ? to_d(x[u][bi]) : 0.0;
#pragma unroll
      for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = bi; bj < NB; ++bj)
          acc[bi][bj] = Mfma<double>::mma(xv[bi], xv[bj], acc[bi][bj]);
    }
  };
  load(x0, st0);
#pragma unroll 1
  for (int64_t st = st0; st < st1; st += 2 * U) {
    load(x1, st + U);
    products(x0, st);
    load(x0, st + 2 * U);
    products(x1, st + U);
  }
  for (int w = 0; w < 8; ++w) {
    if (wave == w) {
#pragma unroll
      for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = bi; bj < NB; ++bj)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double* o = out + (bi * 16 + drow(lk, v)) * SL + bj * 16 + li;
            *o = (w == 0 ? 0.0 : *o) + acc[bi][bj][v];
          }
    }
    __syncthreads();
  }
}

// Cholesky G = R^T R of the leading l x l block (G = a, R = b; only the upper
// triangle of G is read, and G is overwritten).  R is upper triangular with
// zeros below the diagonal and the identity in rows / columns l .. lp-1.  A
// pivot <= ETA_DEP * G_jj (or not positive) gives a unit row and sets the
// flag.  Step j reads only row j of G and updates rows > j, so one barrier
// per step suffices.
template <int ML>
__device__ __noinline__ void b_chol(int l, int lp) {
  auto& g_lds = batch_lds<ML>();
  constexpr int SL = BatchLds<ML>::SL;
  (void)SL;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double* G = g_lds.u.sm.a;
  double* R = g_lds.u.sm.b;
  for (int e = tid; e < lp * lp; e += BNT) {
    const int r = e / lp, c = e - (e / lp) * lp;
    R[r * SL + c] = (r == c && r >= l) ? 1.0 : 0.0;
  }
  for (int i = tid; i < l; i += BNT) g_lds.dgn[i] = G[i * SL + i];
  if (tid == 0) g_lds.ndep = 0;
  __syncthreads();
  for (int j = 0; j < l; ++j) {
    const double d = G[j * SL + j];
    const bool dep = !(d > ETA_DEP * g_lds.dgn[j]);
    if (tid == 0) g_lds.depc[j] = dep ? 1 : 0;
    if (dep) {
      for (int c = j + tid; c < l; c += BNT) R[j * SL + c] = (c == j) ? 1.0 : 0.0;
      if (tid == 0) {
        g_lds.flag = 1;
        ++g_lds.ndep;
        if (!(fabs(d) <= 1.7976931348623157e308)) g_lds.nonfinite = 1;
      }
    } else {
      const double sq = sqrt(d);
      const double inv = 1.0 / d;
      for (int c = j + tid; c < l; c += BNT) R[j * SL + c] = G[j * SL + c] / sq;
      // G[r][c] -= G[j][r] G[j][c] / G[j][j] for j < r <= c < l
      for (int r = j + 1 + wave; r < l; r += BNT / 64) {
        const double gr = G[j * SL + r] * inv;
        for (int c = r + lane; c < l; c += 64) G[r * SL + c] -= gr * G[j * SL + c];
      }
    }
    __syncthreads();
  }
}

// a = R^{-1} with R = b (upper triangular, lp x lp): four lanes per column c
// solve R x = e_c by back substitution, each summing a quarter of every dot
// product; rows / columns l .. lp-1 are the identity.
template <int ML>
__device__ __noinline__ void b_rinv(int l, int lp) {
  auto& g_lds = batch_lds<ML>();
  constexpr int SL = BatchLds<ML>::SL;
  (void)SL;
  const int tid = threadIdx.x;
  const double* R = g_lds.u.sm.b;
  double* X = g_lds.u.sm.a;
  for (int e = tid; e < lp * lp; e += BNT) {
    const int r = e / lp, c = e - (e / lp) * lp;
    X[r * SL + c] = (r == c && r >= l) ? 1.0 : 0.0;
  }
  __syncthreads();
  const int grp = tid >> 2, sub = tid & 3;
  for (int c = grp; c < l; c += BNT / 4) {
    for (int i = c; i >= 0; --i) {
      double t0 = 0.0, t1 = 0.0, t2 = 0.0, t3 = 0.0;
      int u = i + 1 + sub;
      for (; u + 12 <= c; u += 16) {
        t0 += R[i * SL + u] * X[u * SL + c];
        t1 += R[i * SL + u + 4] * X[(u + 4) * SL + c];
        t2 += R[i * SL + u + 8] * X[(u + 8) * SL + c];
        t3 += R[i * SL + u + 12] * X[(u + 12) * SL + c];
      }
      for (; u <= c; u += 4) t0 += R[i * SL + u] * X[u * SL + c];
      double t = (t0 + t1) + (t2 + t3);
      t += __shfl_xor(t, 1, 64);
      t += __shfl_xor(t, 2, 64);
      if (sub == 0) X[i * SL + c] = ((i == c ? 1.0 : 0.0) - t) / R[i * SL + i];
    }
  }
  __syncthreads();
}

// Out (rows x ncols, ldo) = In (rows x lp, lp = 16 NB) a (lp x lp in LDS,
// stride SL; columns >= ncols are formed but not written), on FP64 MFMA; a
// 16-row block's operands are loaded before its products.
// Out may be In (ldo = lp): a wave's block is read before it is written, by no other
// wave.
template <int NB, typename TI, typename TO>
__device__ __noinline__ void b_apply(const TI* In, int64_t rows, int ncols, TO* Out,
                                     int64_t ldo) {
  auto& g_lds = batch_lds<ml_of<NB>()>();
  constexpr int SL = BatchLds<ml_of<NB>()>::SL;
  (void)SL;
  constexpr int lp = 16 * NB;
  In = uniform(In); Out = uniform(Out); rows = uniform(rows); ldo = uniform(ldo);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const double* B = g_lds.u.sm.a;
  const int64_t nrb = cdiv(rows, 16);
  for (int64_t rb = wave; rb < nrb; rb += 8) {
    const int64_t r = min(rb * 16 + li, rows - 1);   // (rows past the last: not stored)
    double av[4 * NB];
#pragma unroll
    for (int t = 0; t < 4 * NB; ++t) av[t] = to_d(In[r * lp + 4 * t + lk]);
    d4 acc[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) acc[cb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 4 * NB; ++t) {
      const int k = 4 * t + lk;
#pragma unroll
      for (int cb = 0; cb < NB; ++cb)
        acc[cb] = Mfma<double>::mma(av[t], B[k * SL + cb * 16 + li], acc[cb]);
      // keep each step's LDS reads next to its products (bounded registers)
      if (t % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      const int c = cb * 16 + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t rr = rb * 16 + drow(lk, v);
        if (rr < rows && c < ncols) Out[rr * ldo + c] = from_d<TO>(acc[cb][v]);
      }
    }
  }
  __syncthreads();
}

// ||G - I||_F^2 of the leading l x l block of the Gram in a (upper blocks:
// diagonal terms once, off-diagonal ones twice), the same value on every
// thread
template <int ML>
__device__ double b_gram_offset2(int l) {
  auto& g_lds = batch_lds<ML>();
  constexpr int SL = BatchLds<ML>::SL;
  (void)SL;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* G = g_lds.u.sm.a;
  double t = 0.0;
  for (int e = tid; e < l * l; e += BNT) {
    const int i = e / l, j = e - (e / l) * l;
    if (i == j) {
      const double d = G[i * SL + i] - 1.0;
      t = fma(d, d, t);
    } else if (i < j) {
      const double x = G[i * SL + j];
      t = fma(2.0 * x, x, t);
    }
  }
  t = wave_allsum(t);
  if (lane == 0) g_lds.sig[wave] = t;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < BNT / 64; ++w) r += g_lds.sig[w];
  __syncthreads();
  return r;
}

// Q = T rounded to TO (rows x lp; lp is a multiple of 16, both 256-byte aligned)
template <typename TO>
__device__ void b_copy(const double* T, int64_t rows, int lp, TO* Q) {
  struct alignas(4 * sizeof(TO)) Vec { TO v[4]; };
  struct alignas(32) DVec { double v[4]; };
#pragma unroll 4
  for (int64_t e = threadIdx.x; e < rows * lp / 4; e += BNT) {
    const DVec x = reinterpret_cast<const DVec*>(T)[e];
    Vec y;
#pragma unroll
    for (int i = 0; i < 4; ++i) y.v[i] = from_d<TO>(x.v[i]);
    reinterpret_cast<Vec*>(Q)[e] = y;
  }
  __syncthreads();
}

// Largest ||Q1^T Q1 - I||_F after the first pass for which the second pass
// is skipped: 2^-30, far below the unit roundoff of the FP32 bases (2^-24),
// so the orthogonality of the stored basis is set by its own rounding.
constexpr double ORTH_SKIP2 = 0x1.0p-60;   // (2^-30)^2

// The columns of T (rows x lp) found dependent by the first Cholesky get
// N(0, 1/rows) entries: normal number j*rows + i of Philox stream 7 with
// batch word (orth call << 20 | matrix index), under the call's seed.
template <int ML>
__device__ __noinline__ void b_replace(double* T, int64_t rows, int l, int lp, uint32_t k0,
                                       uint32_t k1, uint32_t word) {
  auto& g_lds = batch_lds<ML>();
  constexpr int SL = BatchLds<ML>::SL;
  (void)SL;
  const double scale = 1.0 / sqrt((double)rows);
  for (int j = 0; j < l; ++j) {
    if (!g_lds.depc[j]) continue;
    for (int64_t i2 = threadIdx.x; 2 * i2 < rows; i2 += BNT) {
      const uint64_t t = (uint64_t)j * (uint64_t)rows + 2 * (uint64_t)i2;   // even number
      // normals t and t + 1 come from one counter when t is even; rows may be
      // odd, so each value is computed from its own pair
      double z[2];
      for (int h = 0; h < 2; ++h) {
        const uint64_t th = t + h;
        const uint64_t pr = th >> 1;
        const Words w = philox10((uint32_t)pr, (uint32_t)(pr >> 32), 7u, word, k0, k1);
        double z0, z1;
        box_muller(w, z0, z1);
        z[h] = (th & 1) ? z1 : z0;
      }
      const int64_t i = 2 * i2;
      T[i * lp + j] = z[0] * scale;
      if (i + 1 < rows) T[(i + 1) * lp + j] = z[1] * scale;
    }
  }
  __syncthreads();
}

// Q (rows x lp) = orth(In) by CholeskyQR2 in FP64; T (rows x lp FP64) holds
// the first pass.  Q may be In, or T where it is FP64.
template <int NB, typename TI, typename TO>
__device__ void b_orth(const TI* In, int64_t rows, int l, double* T, TO* Q, uint32_t k0,
                       uint32_t k1, uint32_t word) {
  auto& g_lds = batch_lds<ml_of<NB>()>();
  constexpr int SL = BatchLds<ml_of<NB>()>::SL;
  (void)SL;
  constexpr int lp = 16 * NB, ML = ml_of<NB>();
  b_gram<NB>(In, rows);
  b_chol<ML>(l, lp);
  b_rinv<ML>(l, lp);
  b_apply<NB>(In, rows, lp, T, (int64_t)lp);
  if (g_lds.ndep > 0) b_replace<ML>(T, rows, l, lp, k0, k1, word);
  b_gram<NB>(T, rows);
  if (b_gram_offset2<ML>(l) <= ORTH_SKIP2) {
    if ((const void*)T != (const void*)Q) b_copy(T, rows, lp, Q);
    return;
  }
  b_chol<ML>(l, lp);
  b_rinv<ML>(l, lp);
  b_apply<NB>(T, rows, lp, Q, (int64_t)lp);
}

// One-sided Jacobi on the l x l Rh held in a (stride SL): W (column j
// contiguous, ld l) goes to b and V = I to a.  Round-robin rounds of
// disjoint pairs, one pair per group of 16 lanes (32 groups), NB = lp / 16
// rows per lane.  Writes the k
// largest sigma to S and Uh, Vh (l x k, ld lp) to global scratch.
template <int NB>
__device__ __noinline__ void b_jacobi(int l, int k, double* S, double* Uh, double* Vh, int lp,
                                      int32_t* info) {
  auto& g_lds = batch_lds<ml_of<NB>()>();
  constexpr int SL = BatchLds<ml_of<NB>()>::SL;
  (void)SL;
  const int tid = threadIdx.x;
  const int grp = tid >> 4, li = tid & 15;
  double* W = g_lds.u.sm.b;
  double* V = g_lds.u.sm.a;
  for (int e = tid; e < l * l; e += BNT) {
    const int j = e / l, i = e - (e / l) * l;
    W[j * l + i] = V[i * SL + j];
  }
  __syncthreads();
  for (int e = tid; e < l * l; e += BNT) {
    const int j = e / l, i = e - (e / l) * l;
    V[j * l + i] = (i == j) ? 1.0 : 0.0;
  }
  __syncthreads();
  const double tol = (double)l * 2.220446049250313e-16;
  const int N = l + (l & 1);
  int sweep = 0;
  bool converged = (l < 2);
  while (!converged && sweep < JAC_MAX_SWEEPS) {
    ++sweep;
    if (tid == 0) g_lds.flag = 0;
    __syncthreads();
    for (int r = 0; r < N - 1; ++r) {
      for (int pi = grp; pi < N / 2; pi += BNT / 16) {
        int a = rr_player(pi, r, N), b = rr_player(N - 1 - pi, r, N);
        if (a >= l || b >= l) continue;
        if (a > b) { const int t = a; a = b; b = t; }
        if (rotate_pair16<NB>(W + a * l, W + b * l, V + a * l, V + b * l, l, li, tol) && li == 0)
          g_lds.flag = 1;
      }
      __syncthreads();
    }
    converged = (g_lds.flag == 0);
    __syncthreads();
  }
  if (!converged && tid == 0) info_or(info, INFO_JACOBI_CAP);
  jacobi_finish<BNT>(W, V, l, l, k, g_lds.sig, S, Uh, lp, Vh, lp);
  __syncthreads();
}

// a (stride SL, lp x lp) = the l x k matrix M (ld lp, global), zero elsewhere
template <int ML>
__device__ void b_load_small(const double* M, int l, int k, int lp) {
  auto& g_lds = batch_lds<ML>();
  constexpr int SL = BatchLds<ML>::SL;
  (void)SL;
  double* B = g_lds.u.sm.a;
  const int nc = lp;
  for (int e = threadIdx.x; e < lp * nc; e += BNT) {
    const int r = e / nc, c = e - (e / nc) * nc;
    B[r * SL + c] = (r < l && c < k) ? M[r * lp + c] : 0.0;
  }
  __syncthreads();
}

// The decomposition of one matrix after its sketch (in Z), for lp = 16 NB.
template <int NB, int RPW, int KC>
__device__ __noinline__ void b_one(const BatchArgs& g, const BatchDesc& d, const float* A,
                                   float* Y, float* Z, double* T, double* Uh, double* Vh) {
  auto& g_lds = batch_lds<ml_of<NB>()>();
  constexpr int SL = BatchLds<ml_of<NB>()>::SL;
  (void)SL;
  constexpr int lp = 16 * NB, ML = ml_of<NB>();
  const int64_t m = d.m, n = d.n;
  const int l = d.l, k = d.k;
  // batch word of the replacement columns: orth call (high bits), matrix
  const uint32_t mw = (uint32_t)d.index & 0xFFFFFu;
  uint32_t call = 0;
  b_pass_n<NB, RPW, KC>(A, d.lda, m, n, Z, Y);
  for (int j = 0; j < g.q; ++j) {
    b_orth<NB>(Y, m, l, T, Y, g.k0, g.k1, (call++ << 20) | mw);
    b_pass_t<NB, RPW, KC>(A, d.lda, m, n, Y, Z);
    b_orth<NB>(Z, n, l, T, Z, g.k0, g.k1, (call++ << 20) | mw);
    b_pass_n<NB, RPW, KC>(A, d.lda, m, n, Z, Y);
  }
  float* Q = Y;
  b_orth<NB>(Y, m, l, T, Q, g.k0, g.k1, (call++ << 20) | mw);
  b_pass_t<NB, RPW, KC>(A, d.lda, m, n, Q, Z);   // B^T
  double* Qh = T;
  b_orth<NB>(Z, n, l, T, Qh, g.k0, g.k1, (call++ << 20) | mw);
  b_xty<ML>(Qh, Z, n, lp);                         // Rh = Qh^T B^T
  if (threadIdx.x == 0 && g_lds.flag) info_or(g.info, INFO_ORTH_FALLBACK);
  if (threadIdx.x == 0 && g_lds.nonfinite) info_or(g.info, INFO_NONFINITE);
  b_jacobi<NB>(l, k, g.S + d.s_off, Uh, Vh, lp, g.info);
  b_load_small<ML>(Vh, l, k, lp);
  b_apply<NB>(Q, m, k, g.U + d.u_off, (int64_t)k);
  b_load_small<ML>(Uh, l, k, lp);
  b_apply<NB>(Qh, n, k, g.V + d.v_off, (int64_t)k);
}

template <int ML> __device__ __forceinline__ void batch_rsvd(const BatchArgs& g) {
  auto& g_lds = batch_lds<ML>();
  const int tid = threadIdx.x;
  char* slot = g.scratch + (int64_t)blockIdx.x * g.slot_bytes;
  float* Y = reinterpret_cast<float*>(slot + g.off_y);
  float* Z = reinterpret_cast<float*>(slot + g.off_z);
  double* T = reinterpret_cast<double*>(slot + g.off_t);
  double* Uh = reinterpret_cast<double*>(slot + g.off_uh);
  double* Vh = reinterpret_cast<double*>(slot + g.off_vh);
  for (;;) {
    if (tid == 0) g_lds.item = atomicAdd(g.counter, 1);
    __syncthreads();
    const int64_t it = g_lds.item;
    __syncthreads();
    if (it >= g.count) break;
    const BatchDesc d = g.desc[it];
    const int lp = d.lp;
    const float* A = g.A + d.a_off;
    if (tid == 0) {
      g_lds.flag = 0;
      g_lds.nonfinite = 0;
    }
    __syncthreads();
    b_sketch<ML>(Z, d.n, d.l, lp, g.k0, g.k1, (uint32_t)d.index);
    // (lp / 16, pass shape) -> one instantiation
#define RSVD_B1(NBV)                                                                     \
  switch (d.variant) {                                                                   \
    case 1: b_one<NBV, 2, 32>(g, d, A, Y, Z, T, Uh, Vh); break;                          \
    case 2: b_one<NBV, 1, 32>(g, d, A, Y, Z, T, Uh, Vh); break;                          \
    default: b_one<NBV, 1, 64>(g, d, A, Y, Z, T, Uh, Vh); break;                         \
  }
    if constexpr (ML == BATCH_SMALL_LP) {
      switch (lp / 16) {
        case 1: RSVD_B1(1); break;
        case 2: RSVD_B1(2); break;
        case 3: RSVD_B1(3); break;
        default: RSVD_B1(4); break;
      }
    } else {
      RSVD_B1(5);
    }
#undef RSVD_B1
  }
}

// Half of a matrix's time goes to phases of one workgroup's latency (Cholesky,
// inverse, Jacobi) in which a compute unit's matrix cores and memory wait: with
// two workgroups on it the phases of two matrices overlap (the batch above: 36.8
// -> 32.0 ms, and 29.3 ms with the loads of the FP64 steps in flight across their
// products).
__global__ __launch_bounds__(BNT) __attribute__((amdgpu_waves_per_eu(4, 4))) void
batch_small_kernel(BatchArgs g) {
  batch_rsvd<BATCH_SMALL_LP>(g);
}
__global__ __launch_bounds__(BNT) void batch_large_kernel(BatchArgs g) {
  batch_rsvd<BATCH_MAX_LP>(g);
}

}  // namespace

hipError_t launch_batch_rsvd(const BatchArgs& g, int grid, bool small, hipStream_t st) {
  if (g.count < 1) return hipSuccess;
  if (grid < 1) return hipErrorInvalidValue;
  hipError_t e = launch_set_word(g.counter, 0, st);
  if (e != hipSuccess) return e;
  if (small) hipLaunchKernelGGL(batch_small_kernel, dim3((unsigned)grid), dim3(BNT), 0, st, g);
  else hipLaunchKernelGGL(batch_large_kernel, dim3((unsigned)grid), dim3(BNT), 0, st, g);
  return hipGetLastError();
}

}  // namespace rsvd
