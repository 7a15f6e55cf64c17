// orth(Y) by CholeskyQR (the unpivoted QR `[Q, ~] = qr(Y, 0)` of Sec. 2.1,
// used between the products of the power scheme of Sec. 3.2 and in Alg. 5):
//   G = Y^T Y (FP64),  G = R^T R (Cholesky),  Q = Y R^{-1}  (triangular solve),
// applied twice (CholeskyQR2) so that Q is orthonormal to working precision.
//
// Kernels here:
//  * chol_factor: one workgroup factors an lp x lp Gram matrix (lp <= 256)
//    held in 16x16 matrix-core accumulator tiles (right-looking, block size
//    16, one-step lookahead).  It writes R (upper triangular, zero below), the inverses
//    of its 16x16 diagonal blocks, and a flag per column.  A column whose
//    Schur pivot is not above eta * G_jj (numerically dependent on the
//    columns before it) gets a unit row in R, so it is removed from the
//    factorization of the later columns and can be replaced afterwards.
//  * the factor of the second pass's Gram matrix, which is I + E with E of the
//    order of the unit roundoff times cond(Y)^2.  With R = I + F (F upper
//    triangular), R^T R = I + E reads F = Phi(E - F^T F), Phi taking the strict
//    upper triangle and half the diagonal, so F = Phi(E) + O(||E||^2) and
//    R^{-1} = I - F + O(||F||^2).  When ||E||_F^2 <= NI_TAU2 (a quarter of the
//    unit roundoff) both truncations sit below rounding: the tiles of R = I +
//    Phi(E) are written where the tiles of G are summed, with the parts of
//    ||E||_F^2, and the factorization runs only when the test fails.
//  * gram_kernel sums Y^T Y over row ranges into partial tiles;
//    gram_chol_kernel, one workgroup per tile, adds them in a fixed order, and
//    its last workgroup to finish tests and factors G: separate kernels for the
//    sums, the test and the factorization cost a launch of 4 - 5 us each where
//    the work is shorter.  (The last workgroup of gram_kernel doing all of it is
//    slower even at l = 30: 28 us against 8 + 9.)
//  * trsm_kernel: Q = Y R^{-1} for a tall Y, one wave per 16 rows, column
//    block by column block (Q_c = (Y_c - sum_{b<c} Q_b R_bc) R_cc^{-1}); a
//    flagged column of Q gets fresh Gaussian numbers (Philox stream 7) scaled to
//    unit expected norm instead.
//  * trmm_kernel: R = R2 R1 for the two passes.
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace rsvd {
namespace {

constexpr double NI_TAU2 = 2.5e-17;   // bound on ||G - I||_F^2 (about a quarter of 2^-52)
// ||G - I||_F^2 of the second Gram below which an FP32 basis is the first
// pass rounded to FP32: (2^-30)^2, far below the FP32 unit roundoff 2^-24
constexpr double TRSM_SKIP2 = 0x1.0p-60;
constexpr int MAXNB = 16;          // lp <= 256
// LDS row stride of the Cholesky's panel row (doubles): rows k and k+1 fall
// on different halves of the banks
constexpr int CH_LDP = 272;

// f(integral_constant<int, i>) for i = 0 .. N-1 (compile-time indices)
template <int I, int N, typename F> __device__ __forceinline__ void static_for_(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    static_for_<I + 1, N>(f);
  }
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_<0, N>(f);
}

// Tile t of the row-major enumeration of the upper triangle of an nb x nb
// tile grid: row a starts at t = a*nb - a*(a-1)/2.  Arguments are uniform.
__device__ __forceinline__ int tile_row(int t, int nb) {
  int a = 0;
  while (a + 1 < nb && (a + 1) * nb - (a + 1) * a / 2 <= t) ++a;
  return a;
}
__device__ __forceinline__ int tile_col(int t, int nb) {
  const int a = tile_row(t, nb);
  return a + (t - (a * nb - a * (a - 1) / 2));
}

// Load tile (a, b) of the symmetric G (upper triangle read; padding rows and
// columns >= l are those of the identity) in accumulator layout.
__device__ __forceinline__ d4 load_gtile(const double* G, int64_t ldg, int l, int a, int b,
                                         int lane) {
  d4 t;
  const int col = b * 16 + (lane & 15);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = a * 16 + drow(lane >> 4, v);
    // one load per element (clamped address), no branches
    const bool in = row < l && col < l;
    const int64_t off = in ? (int64_t)min(row, col) * ldg + max(row, col) : 0;
    const double g = ld_agent(G + off);   // (written by other workgroups of this launch)
    t[v] = in ? g : ((row == col) ? 1.0 : 0.0);
  }
  return t;
}

// Row broadcasts (DPP row_newbcast, the form that FP64 operations take): lane L of
// every row of 16 lanes.  A register that a VALU operation wrote is not read through
// DPP within two wait states: dpp_source stands between (bcast has its own).
__device__ __forceinline__ void dpp_source(double& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 1" : "+v"(x));
#endif
}
template <int L> __device__ __forceinline__ double bcast(double x) {
  double d = x;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
      : "=v"(d) : "v"(x), "n"(L));
#endif
  return d;
}
// acc = fma(-(r of lane L), y, acc)
template <int L> __device__ __forceinline__ void fnma_bcast(double& acc, double r, double y) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
      : "+v"(acc) : "v"(r), "v"(y), "n"(L));
#endif
}

// Right-looking block Cholesky with a one-step lookahead, one workgroup of
// NW waves.  Waves 1 .. NW-1 hold the upper 16x16 tiles of G in matrix-core
// accumulator layout (tile t of the row-major enumeration of the upper
// triangle lives in slot t / (NW-1) of wave 1 + t % (NW-1)); wave 0 owns no
// tile and factors the diagonal blocks.  Block step s has two phases:
//   1. wave 0 takes the diagonal tile (s, s), which its owner handed over in
//      the previous step with the panels 0 .. s-2 applied, applies panel
//      s-1 and factors it (R_ss and X = R_ss^{-1}); meanwhile the other waves
//      apply panel s-1 to every tile of rows >= s, and the owner of
//      (s+1, s+1) hands that tile over for the next step;
//   2. the owners of the tiles (s, b), b > s, form the panel row
//      R_sb = X^T G_sb (rows of dependent columns zeroed) in LDS and in R.
// The panel lives in LDS (16 x lp, one buffer: phase 2 of a step writes it
// after phase 1 has read the previous one).
template <int NW, int TPW>
__device__ __forceinline__ void chol_factor(const double* G, int64_t ldg, int l, int lp,
                                            double eta, double* R, int64_t ldr, double* Rdinv,
                                            int32_t* dep, int32_t* info) {
  constexpr int NT = 64 * NW, NU = NW - 1;
  const int nb = lp / 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;

  __shared__ double P[16 * CH_LDP];     // panel row of R (rows 16s .. 16s+15)
  __shared__ double Dn[2][16 * 17];     // diagonal tile handed to wave 0
  __shared__ double Dw[16 * 17];        // wave 0: the updated diagonal tile
  __shared__ double Rs[16 * 16];        // R_ss, row-major
  __shared__ double Xs[16 * 16];        // R_ss^{-1}, row-major
  __shared__ double diag0[256];
  __shared__ int depblk[16];

  for (int j = tid; j < lp; j += NT)
    diag0[j] = (j < l) ? ld_agent(G + (int64_t)j * ldg + j) : 1.0;
  // zero the strictly lower part of R
  for (int r = 1 + wave; r < lp; r += NW)
    for (int c = lane; c < r; c += 64) R[(int64_t)r * ldr + c] = 0.0;

  // slot table of an update wave: lane q holds (a | b << 8) of slot q's tile
  // (a = 255: no tile)
  const int ntiles = nb * (nb + 1) / 2;
  int coord = 255;
  if (wave > 0 && lane < TPW) {
    const int t = (wave - 1) + NU * lane;
    if (t < ntiles) {
      int a = 0;
      while (a + 1 < nb && (a + 1) * nb - (a + 1) * a / 2 <= t) ++a;
      const int b = a + (t - (a * nb - a * (a - 1) / 2));
      coord = a | (b << 8);
    }
  }
  d4 acc[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int ab = __builtin_amdgcn_readlane(coord, q);
    const int a = ab & 255, b = ab >> 8;
    // (a slot without a tile reads identity values: no branch around the loads)
    acc[q] = load_gtile(G, ldg, l, a, b, lane);
    if (a == 0 && b == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) Dn[0][drow(lk, v) * 17 + li] = acc[q][v];
    }
  }
  __syncthreads();

  // Wave 0 and the update waves run separate loops over s that meet at the
  // same two barriers per step, so the tiles' registers are live only in the
  // update waves' loop.
  if (wave == 0) {
    for (int s = 0; s < nb; ++s) {
      // (1, wave 0) the diagonal tile with panel s-1 applied, in accumulator
      // layout, then as columns: lane c (all four row groups alike) holds
      // x[a] = G'[a][c]
      d4 t;
#pragma unroll
      for (int v = 0; v < 4; ++v) t[v] = Dn[s & 1][drow(lk, v) * 17 + li];
      if (s > 0) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const double pv = P[(4 * kk + lk) * CH_LDP + s * 16 + li];
          t = Mfma<double>::mma(-pv, pv, t);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) Dw[drow(lk, v) * 17 + li] = t[v];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // c = li through an opaque move, so that the per-lane constants derived
      // from it are formed here and not kept live across the whole s loop
      int c;
      asm volatile("v_mov_b32 %0, %1" : "=v"(c) : "v"(li));
      double x[16];
#pragma unroll
      for (int a = 0; a < 16; ++a) x[a] = Dw[a * 17 + c];
      // right-looking elimination inside the block: step j takes the pivot
      // d = G'[j][j] from lane j and turns x[j] into row j of R (lane c >= j
      // gets x[j] / sqrt(d), which is sqrt(d) itself in lane j), then
      // subtracts R[j][a] R[j][c] from the rows a > j.  Lanes c < j compute
      // values that are never read (rows below the diagonal are dropped at
      // the end).  A column whose pivot is not above eta * G_jj gets a unit
      // row.  Entries of other lanes come by row broadcasts inside the FMAs
      // (fnma_bcast): with two readlanes per entry and a store per step a step took
      // 430 cycles, and it takes 250.
      const double thr = eta * diag0[s * 16 + c];
      double inv[16];
      bool okc = true, nfc = false;      // of the lane's own column
      static_for<16>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const double d = bcast<j>(x[j]);
        const bool finite = __builtin_isfinite(d);
        const bool ok = finite && d > bcast<j>(thr);
        okc = c == j ? ok : okc;
        nfc = c == j ? !finite : nfc;
        // branch-free: the estimate is formed for any d and then selected
        const double inv0 = rsq_nr(d);
        inv[j] = ok ? inv0 : 1.0;
        double r = ok ? x[j] * inv0 : ((c == j) ? 1.0 : 0.0);
        dpp_source(r);
        x[j] = r;
        static_for<15 - j>([&](auto ii) {
          constexpr int a = j + 1 + decltype(ii)::value;
          fnma_bcast<a>(x[a], r, r);
        });
      });
      // R_ss to LDS (the four row groups of the wave hold the same columns
      // and store the same values); the update waves copy it to R in phase 2
#pragma unroll
      for (int a = 0; a < 16; ++a) Rs[a * 16 + c] = (a <= c) ? x[a] : 0.0;
      if (lane < 16) {
        const int dj = okc ? 0 : 1;
        depblk[c] = dj;
        if (s * 16 + c < l) dep[s * 16 + c] = dj;
      }
      // columns of the block below l that failed the test
      const uint64_t bad = __ballot(lane < 16 && s * 16 + c < l && !okc);
      const uint64_t nf = __ballot(nfc);
      if (lane == 0) {
        if ((bad & nf) != 0u) info_or(info, INFO_NONFINITE);
        if ((bad & ~nf) != 0u) info_or(info, INFO_ORTH_FALLBACK);
      }
      // X = R_ss^{-1}, column c in lane c by back substitution (the entries
      // below the diagonal come out zero), R[a][b] broadcast from lane b; the terms
      // of rows b > a+1 are summed in two chains before X[a+1] is known, so each
      // row adds one product to the dependent chain (250 -> 190 cycles a row against
      // reads of R from LDS).
      double X[16];
      static_for<16>([&](auto ii) { dpp_source(x[decltype(ii)::value]); });
      static_for<16>([&](auto ii) {
        constexpr int a = 15 - decltype(ii)::value;
        double u0 = (a == c) ? 1.0 : 0.0, u1 = 0.0;
        static_for<(a < 14 ? 14 - a : 0)>([&](auto kk) {
          constexpr int b = 15 - decltype(kk)::value;      // 15 .. a + 2
          if constexpr ((b & 1) == 0) fnma_bcast<b>(u0, x[a], X[b]);
          else fnma_bcast<b>(u1, x[a], X[b]);
        });
        double u = u0 + u1;
        if constexpr (a < 15) fnma_bcast<a + 1>(u, x[a], X[a + 1]);
        X[a] = u * inv[a];
      });
#pragma unroll
      for (int a = 0; a < 16; ++a) Xs[a * 16 + c] = X[a];
      __syncthreads();
      __syncthreads();   // (2) the update waves form the panel row
    }
  } else {
    for (int s = 0; s < nb; ++s) {
      // (1, update waves) panel s-1 on every tile of rows >= s but (s, s);
      // the k-steps run outermost so that consecutive products go to
      // different tiles
      if (s > 0) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int k = 4 * kk + lk;
#pragma unroll
          for (int q = 0; q < TPW; ++q) {
            const int ab = __builtin_amdgcn_readlane(coord, q);
            const int a = ab & 255, b = ab >> 8;
            if (a >= s && a < nb && b > s) {
              const double av = -P[k * CH_LDP + a * 16 + li];
              const double bv = P[k * CH_LDP + b * 16 + li];
              acc[q] = Mfma<double>::mma(av, bv, acc[q]);
            }
          }
          // (operands of one k-step at a time in registers)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int q = 0; q < TPW; ++q) {
        const int ab = __builtin_amdgcn_readlane(coord, q);
        if (ab == ((s + 1) | ((s + 1) << 8))) {
#pragma unroll
          for (int v = 0; v < 4; ++v) Dn[(s + 1) & 1][drow(lk, v) * 17 + li] = acc[q][v];
        }
      }
      __syncthreads();
      // (2) panel row s: R_sb = X^T G_sb.  The accumulator layout of G_sb is
      // the B-operand layout of the k-steps (element kk of lane (i, g) is
      // row 4 kk + g, column i).  The update waves also copy R_ss and its
      // inverse from LDS to R and Rdinv.
      for (int e = tid - 64; e < 512; e += NT - 64) {
        if (e < 256) R[(int64_t)(s * 16 + (e >> 4)) * ldr + s * 16 + (e & 15)] = Rs[e];
        else Rdinv[(int64_t)s * 256 + (e - 256)] = Xs[e - 256];
      }
#pragma unroll
      for (int q = 0; q < TPW; ++q) {
        const int ab = __builtin_amdgcn_readlane(coord, q);
        const int a = ab & 255, b = ab >> 8;
        if (a == s && b > s) {
          d4 r = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
            r = Mfma<double>::mma(Xs[(4 * kk + lk) * 16 + li], acc[q][kk], r);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = drow(lk, v);
            const double x = depblk[row] ? 0.0 : r[v];
            P[row * CH_LDP + b * 16 + li] = x;
            R[(int64_t)(s * 16 + row) * ldr + b * 16 + li] = x;
          }
        }
      }
      __syncthreads();
    }
  }
}

// Normal number t of a Philox stream.  A flagged column j of Q (M rows) is
// replaced by N(0, 1/M) entries from stream 7, number j*M + i for row i, batch =
// the orth call.
__device__ __forceinline__ double normal_at(uint32_t k0, uint32_t k1, uint32_t sid, uint32_t batch,
                                            uint64_t t) {
  uint32_t c0 = (uint32_t)(t >> 1), c1 = (uint32_t)(t >> 33), c2 = sid, c3 = batch;
  const uint32_t PM0 = 0xD2511F53u, PM1 = 0xCD9E8D57u, PW0 = 0x9E3779B9u, PW1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += PW0; k1 += PW1; }
    const uint32_t hi0 = __umulhi(PM0, c0), lo0 = PM0 * c0;
    const uint32_t hi1 = __umulhi(PM1, c2), lo1 = PM1 * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  const double a = (double)(c0 >> 5) * 67108864.0 + (double)(c1 >> 6);
  const double b = (double)(c2 >> 5) * 67108864.0 + (double)(c3 >> 6);
  const double u1 = (a + 1.0) * 0x1.0p-53, u2 = b * 0x1.0p-53;
  const double r = sqrt(-2.0 * log(u1)), th = 6.283185307179586 * u2;
  return (t & 1) ? r * sin(th) : r * cos(th);
}

// Q = Y R^{-1}: a workgroup of 4 waves takes 64 rows of Y (a wave 16),
// column block by column block, in transposed form
// Q_c^T = R_cc^{-T} (Y_c^T - sum_{b<c} R_bc^T Q_b^T).  The accumulator layout
// of a 16x16 product (lane (j, g) holds rows 4v + g of column j) is also the
// B-operand layout of the next products, so every Q_b^T stays in registers
// (4 doubles per lane) from the step that makes it to the last column block.
// The A operands of column block c (-R_bc for b < c, then R_cc^{-1}) are
// staged in LDS in operand order, shared by the four waves and double
// buffered: thread (kk, lane) fetches the k-step kk operands of the next
// column (and each wave its next Y values) into registers while the current
// column is multiplied, and one barrier per column block separates the two.
template <typename TY, typename TQ, int NB>
__global__ __launch_bounds__(256) void trsm_kernel(const TY* __restrict__ Y, int64_t ldy,
                                                   int64_t M, int l, int lp,
                                                   const double* __restrict__ R, int64_t ldr,
                                                   const double* __restrict__ Rdinv,
                                                   TQ* __restrict__ Q, int64_t ldq,
                                                   const double* __restrict__ skip_e2,
                                                   const int32_t* __restrict__ dep, uint64_t seed,
                                                   uint32_t call) {
  __shared__ double Rb[2][NB * 256];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int nb = lp / 16;
  // (a wave past the last row still stages its share of the operands)
  const int64_t r = ((int64_t)blockIdx.x * 4 + wave) * 16 + li;
  const bool rok = r < M;
  const TY* yr = Y + (rok ? r : 0) * ldy;
  TQ* qr = Q + (rok ? r : 0) * ldq;
  if (skip_e2) {
    // when Y is orthonormal to within TRSM_SKIP2, Q = Y rounded to TQ
    if (*skip_e2 <= TRSM_SKIP2) {
      for (int c = 0; c < nb; ++c) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int col = c * 16 + 4 * v + lk;
          if (rok && col < l) qr[col] = (TQ)yr[col];
        }
      }
      return;
    }
  }
  double pre[NB], ypre[4];
  // operands of column block c (compile-time slot count) read at column cf
  // (equal to c but past the last block, where the values go unused); no
  // branches around the loads, so they stay in flight across the products
  auto fetch = [&](auto cc, int cf) {
    constexpr int c = decltype(cc)::value;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i < c) pre[i] = -R[(int64_t)(i * 16 + 4 * wave + lk) * ldr + cf * 16 + li];
      else if (i == c) pre[i] = Rdinv[(int64_t)cf * 256 + (4 * wave + lk) * 16 + li];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int col = cf * 16 + 4 * v + lk;
      const bool ok = rok && col < l;
      const double y = (double)yr[ok ? col : 0];
      ypre[v] = ok ? y : 0.0;
    }
  };
  auto stash = [&](int c) {
    double* rb = Rb[c & 1];
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i <= c) rb[i * 256 + wave * 64 + lane] = pre[i];
  };
  fetch(std::integral_constant<int, 0>(), 0);
  stash(0);
  __syncthreads();
  d4 qt[NB];
  static_for<NB>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    if (c < nb) {
      d4 acc;
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = ypre[v];
      if constexpr (c + 1 < NB) fetch(std::integral_constant<int, c + 1>(), min(c + 1, nb - 1));
      // (the loads issue before the products)
      __builtin_amdgcn_sched_barrier(0);
      const double* rb = Rb[c & 1];
#pragma unroll
      for (int b = 0; b < c; ++b) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          acc = Mfma<double>::mma(rb[b * 256 + kk * 64 + lane], qt[b][kk], acc);  // -R_bc[k][i]
      }
      d4 out = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        out = Mfma<double>::mma(rb[c * 256 + kk * 64 + lane], acc[kk], out);  // Rinv_cc[k][i]
      qt[c] = out;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int col = c * 16 + 4 * v + lk;
        if (rok && col < l) qr[col] = (TQ)out[v];
      }
      if (c + 1 < nb) stash(c + 1);
      __syncthreads();
    }
  });
  if (dep != nullptr) {
    // the flagged columns (usually none)
    const double scale = 1.0 / sqrt((double)M);
    for (int j0 = 0; j0 < l; j0 += 64) {
      uint64_t flag = __ballot(j0 + lane < l && dep[min(j0 + lane, l - 1)] != 0);
      for (; flag != 0; flag &= flag - 1) {
        const int col = j0 + __builtin_ctzll(flag);
        if (rok && lk == (col & 3)) {              // (the lane that stored this column above)
          const double z = normal_at((uint32_t)seed, (uint32_t)(seed >> 32), 7u, call,
                                     (uint64_t)col * (uint64_t)M + (uint64_t)r);
          qr[col] = (TQ)(z * scale);
        }
      }
    }
  }
}

// C = A B for upper-triangular lp x lp A, B (C upper triangular, zero below);
// rows k of B with bdep[k] != 0 count as zero (the unit rows that the
// Cholesky gives dependent columns stand for a zero residual, so the product
// is the R of Y = Q R).  One wave per 16 x 16 tile of C, on the matrix cores.
__global__ __launch_bounds__(256) void trmm_kernel(const double* __restrict__ Am, int64_t lda,
                                                   const double* __restrict__ Bm, int64_t ldb,
                                                   const int32_t* __restrict__ bdep,
                                                   double* __restrict__ C, int64_t ldc, int lp) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int nb = lp / 16;
  const int t = blockIdx.x * 4 + wave;
  if (t >= nb * nb) return;
  const int a = t / nb, b = t - (t / nb) * nb;
  d4 acc = d4{0.0, 0.0, 0.0, 0.0};
  for (int q = a; q <= b; ++q) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int kx = q * 16 + 4 * kk + lk;
      const double av = Am[(int64_t)(a * 16 + li) * lda + kx];
      const double bv = (bdep != nullptr && bdep[kx] != 0) ? 0.0 : Bm[(int64_t)kx * ldb + b * 16 + li];
      acc = Mfma<double>::mma(av, bv, acc);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = a * 16 + drow(lk, v), col = b * 16 + li;
    C[(int64_t)row * ldc + col] = (row <= col) ? acc[v] : 0.0;
  }
}

__global__ void set_word_kernel(int32_t* w, int32_t v) { *w = v; }
// the status words of a call and the sync words of its orths
__global__ void reset_kernel(int32_t* info, OrthSync* s0, OrthSync* s1) {
  if (threadIdx.x < 2) info[threadIdx.x] = 0;
  if (threadIdx.x == 2 && s0) s0->ticket = 0u;
  if (threadIdx.x == 3 && s1) s1->ticket = 0u;
}

// T = Y - T: the residual of a projection of Y (block orthonormalization)
template <typename TY>
__global__ __launch_bounds__(256) void rsub_kernel(const TY* __restrict__ Y, int64_t ldy,
                                                   double* __restrict__ T, int64_t ldt,
                                                   int64_t rows, int cols) {
  const int64_t total = rows * cols;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / cols, c = e - r * cols;
    T[r * ldt + c] = (double)Y[r * ldy + c] - T[r * ldt + c];
  }
}

// rows of R that belong to dependent columns, zeroed (their unit rows are
// placeholders, not part of Y = Q R)
__global__ __launch_bounds__(64) void zero_dep_rows_kernel(double* __restrict__ R, int64_t ldr,
                                                           int lp, const int32_t* __restrict__ dep) {
  const int j = blockIdx.x;
  if (!dep[j]) return;
  for (int c = threadIdx.x; c < lp; c += blockDim.x) R[(int64_t)j * ldr + c] = 0.0;
}

// Gram matrix G = Y^T Y (FP64) of a tall Y (rows x l), upper 16x16 tiles only.
// The column blocks are cut into segments of 4; a tile group is a pair of
// segments (sa <= sb) and holds the at most 16 upper tiles between them, so a
// workgroup of the group needs only the <= 128 columns of its two segments.
// Each group owns a number of workgroups proportional to its tiles per wave
// (1 or 2), and workgroup j of the group reduces the j-th of that many equal
// row ranges.  16-row chunks of the group's columns are staged in LDS (row
// stride 144 doubles, so the four row groups of a wave fall on different bank
// halves), the next chunk is fetched into registers while the current one is
// multiplied, and each tile accumulates on one wave's matrix cores.  Partial
// tiles go to part[workgroup][slot]; gram_chol_kernel adds a tile's partials in
// workgroup order (deterministic).
constexpr int GR_NT = 512;
constexpr int GR_NW = GR_NT / 64;
constexpr int GR_SEG = 4;                   // column blocks per segment
constexpr int GR_MAXSEG = MAXNB / GR_SEG;   // 4
constexpr int GR_MAXG = GR_MAXSEG * (GR_MAXSEG + 1) / 2;
constexpr int GR_LDS = 144;                 // LDS row stride (doubles)

struct GramPlan {
  int nb, nseg, ngroups, total;
  int sa[GR_MAXG], sb[GR_MAXG];
  int off[GR_MAXG + 1];                     // first workgroup of each group
};

// What follows the sums of the partial tiles: the factorization.
struct CholArgs {
  double* G; int64_t ldg;
  int l, lp;
  double eta;
  double* R; int64_t ldr;
  double* Rdinv;
  int32_t* dep;
  int32_t* info;
  double* parts;                  // NI: the tiles' parts of ||G - I||_F^2
  OrthSync* sync;
};

// Tile t of G (512 threads): the sum over the workgroups of its group of their
// partial tiles, in workgroup order (four interleaved chains added in a fixed
// order; two halves of the workgroup take two chains each, sixteen loads in
// flight).  NI: also the tile of R = I + Phi(G - I) (and the zeros below the
// diagonal), the inverse I - F + F^2 of a diagonal block, clear flags and the
// tile's part of ||G - I||_F^2 (off-diagonal entries twice).  What another
// workgroup reads or rewrites in the same launch is stored past the L2.
template <bool NI>
__device__ __forceinline__ void reduce_tile(const double* part, const GramPlan& gp, int t,
                                            const CholArgs& c) {
  __shared__ double half1[256];
  __shared__ double Fd[16 * 17];
  __shared__ double red[4];
  const int tid = threadIdx.x, e = tid & 255, h = tid >> 8;
  const int a = tile_row(t, gp.nb), b = tile_col(t, gp.nb);
  const int sa = a / GR_SEG, sb = b / GR_SEG;
  const int g = sa * gp.nseg - sa * (sa - 1) / 2 + (sb - sa);
  const int u = 4 * (a - GR_SEG * sa) + (b - GR_SEG * sb);
  const int w0 = gp.off[g], ng = gp.off[g + 1] - w0;
  const double* p = part + ((int64_t)w0 * 16 + u) * 256 + e;
  auto ld = [&](int w) { return p[(int64_t)w * 4096]; };
  constexpr int U = 8;
  double s0 = 0.0, s1 = 0.0;
  const int n4 = ng & ~3;                          // the interleaved part
  for (int w = 0; w < n4; w += 4 * U) {
    double x[U], y[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {                  // (past the end: the last one, not added)
      const int v = min(w + 4 * i, n4 - 4) + 2 * h;
      x[i] = ld(v);
      y[i] = ld(v + 1);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const bool in = w + 4 * i < n4;
      s0 = in ? s0 + x[i] : s0;
      s1 = in ? s1 + y[i] : s1;
    }
  }
  if (h == 0 && n4 < ng) {
    double x[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) x[i] = ld(min(n4 + i, ng - 1));
#pragma unroll
    for (int i = 0; i < 3; ++i) s0 = n4 + i < ng ? s0 + x[i] : s0;
  }
  if (h == 1) half1[e] = s0 + s1;
  __syncthreads();
  const int i = e >> 4, j = e & 15;
  const int gi = a * 16 + i, gj = b * 16 + j;
  if (h == 0) {
    const double x = (s0 + s1) + half1[e];
    st_agent(c.G + (int64_t)gi * c.ldg + gj, x);
    if constexpr (NI) {
      const bool in = gi < c.l && gj < c.l && gi <= gj;
      const double d = x - (gi == gj ? 1.0 : 0.0);
      double s = in ? ((gi == gj ? 1.0 : 2.0) * d) * d : 0.0;
      const double f = in ? (gi == gj ? 0.5 * d : d) : 0.0;
      st_agent(c.R + (int64_t)gi * c.ldr + gj, (gi == gj ? 1.0 : 0.0) + f);
      if (a == b) {
        Fd[i * 17 + j] = f;
        if (i == 0 && gj < c.l)
          __hip_atomic_store(c.dep + gj, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      s = wave_allsum(s);
      if ((tid & 63) == 0) red[tid >> 6] = s;
    }
  } else if constexpr (NI) {
    if (a != b) st_agent(c.R + (int64_t)(b * 16 + i) * c.ldr + a * 16 + j, 0.0);
  }
  if constexpr (NI) {
    __syncthreads();
    if (tid == 0) st_agent(c.parts + t, ((red[0] + red[1]) + red[2]) + red[3]);
    if (a == b && h == 0) {
      double f2 = 0.0;
      for (int q = i; q <= j; ++q) f2 = fma(Fd[i * 17 + q], Fd[q * 17 + j], f2);
      st_agent(c.Rdinv + (int64_t)a * 256 + e, ((i == j) ? 1.0 : 0.0) - Fd[i * 17 + j] + f2);
    }
  }
}

// Whether this workgroup is the last of the launch to get here; what the others
// stored past the L2 before is then visible to agent-scope loads.  (No
// workgroup waits for another one.)
__device__ __forceinline__ bool last_workgroup(OrthSync* sync) {
  __shared__ int last;
  stores_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t n =
        __hip_atomic_fetch_add(&sync->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = n + 1u == gridDim.x;
    if (last) st_agent_u32(&sync->ticket, 0u);       // for the next launch
  }
  __syncthreads();
  return last != 0;
}

// the near-identity test (NI), or the factorization
template <int TPW, bool NI>
__device__ __forceinline__ void test_and_factor(const CholArgs& c) {
  if constexpr (NI) {
    const int nb = c.lp / 16, ntiles = nb * (nb + 1) / 2, ln = threadIdx.x & 63;
    double e2 = 0.0;                               // (the same on every wave)
    for (int t = ln; t < ntiles; t += 64) e2 += ld_agent(c.parts + t);
    e2 = wave_allsum(e2);
    if (threadIdx.x == 0) c.sync->e2 = e2;
    if (e2 <= NI_TAU2) return;                     // false for NaN
  }
  chol_factor<8, TPW>(c.G, c.ldg, c.l, c.lp, c.eta, c.R, c.ldr, c.Rdinv, c.dep, c.info);
}

template <typename TY>
__global__ __launch_bounds__(GR_NT) void gram_kernel(const TY* __restrict__ Y, int64_t ldy,
                                                     int64_t rows, int l, GramPlan gp,
                                                     double* __restrict__ part) {
  __shared__ double Ys[2][16 * GR_LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int x = blockIdx.x;
  int g = 0;
  while (g + 1 < gp.ngroups && gp.off[g + 1] <= x) ++g;
  const int sa = gp.sa[g], sb = gp.sb[g];
  const int ng = gp.off[g + 1] - gp.off[g], j = x - gp.off[g];
  const int64_t r0 = ((int64_t)j * rows) / ng, r1 = ((int64_t)(j + 1) * rows) / ng;
  const bool diag = sa == sb;
  const int ncol = diag ? 64 : 128;
  const int sh = diag ? 6 : 7;
  // the (up to) two tiles of this wave: slot u = 4 * (ta - 4 sa) + (tb - 4 sb)
  bool tv[2];
  int ca[2], cb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int u = wave + GR_NW * q;
    const int ta = GR_SEG * sa + (u >> 2), tb = GR_SEG * sb + (u & 3);
    tv[q] = ta < gp.nb && tb < gp.nb && ta <= tb;
    ca[q] = (u >> 2) * 16;
    cb[q] = (diag ? 0 : 64) + (u & 3) * 16;
  }
  d4 acc[2];
  acc[0] = d4{0.0, 0.0, 0.0, 0.0};
  acc[1] = d4{0.0, 0.0, 0.0, 0.0};
  const int nch = (int)cdiv(r1 - r0, 16);
  double pre[4];
  auto fetch = [&](int ch) {
    const int64_t base = r0 + (int64_t)ch * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + GR_NT * i;
      const int rr = e >> sh, cc = e & (ncol - 1);
      const int gcol = (cc < 64) ? sa * 64 + cc : sb * 64 + (cc - 64);
      const int64_t r = base + rr;
      pre[i] = (e < 16 * ncol && r < r1 && gcol < l) ? (double)Y[r * ldy + gcol] : 0.0;
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + GR_NT * i;
      if (e < 16 * ncol) Ys[buf][(e >> sh) * GR_LDS + (e & (ncol - 1))] = pre[i];
    }
  };
  if (nch > 0) {
    fetch(0);
    stash(0);
  }
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    const int buf = ch & 1;
    if (ch + 1 < nch) fetch(ch + 1);
    const double* ys = Ys[buf];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (tv[q]) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int k = 4 * kk + lk;
          acc[q] = Mfma<double>::mma(ys[k * GR_LDS + ca[q] + li], ys[k * GR_LDS + cb[q] + li],
                                     acc[q]);
        }
      }
    }
    if (ch + 1 < nch) stash(buf ^ 1);
    __syncthreads();
  }
  double* P = part + (int64_t)x * 16 * 256;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (tv[q]) {
      const int u = wave + GR_NW * q;
#pragma unroll
      for (int v = 0; v < 4; ++v) P[u * 256 + drow(lk, v) * 16 + li] = acc[q][v];
    }
  }
}

// one workgroup per tile: the sums, and in the last one the factorization
template <int TPW, bool NI>
__global__ __launch_bounds__(GR_NT) void gram_chol_kernel(const double* __restrict__ part,
                                                          GramPlan gp, CholArgs ca) {
  reduce_tile<NI>(part, gp, blockIdx.x, ca);
  if (!last_workgroup(ca.sync)) return;
  test_and_factor<TPW, NI>(ca);
}

GramPlan plan_gram(int64_t rows, int lp, int ncu) {
  GramPlan gp;
  gp.nb = lp / 16;
  gp.nseg = (int)cdiv(gp.nb, GR_SEG);
  gp.ngroups = 0;
  int wsum = 0;
  int wt[GR_MAXG];
  for (int sa = 0; sa < gp.nseg; ++sa)
    for (int sb = sa; sb < gp.nseg; ++sb) {
      const int na = std::min(GR_SEG, gp.nb - GR_SEG * sa);
      const int nbb = std::min(GR_SEG, gp.nb - GR_SEG * sb);
      const int tiles = (sa == sb) ? na * (na + 1) / 2 : na * nbb;
      gp.sa[gp.ngroups] = sa;
      gp.sb[gp.ngroups] = sb;
      wt[gp.ngroups] = (int)cdiv(tiles, GR_NW);   // tiles per wave: 1 or 2
      wsum += wt[gp.ngroups];
      ++gp.ngroups;
    }
  // about two workgroups per CU in all, at least 64 rows per workgroup
  const int64_t budget = 2 * (int64_t)ncu;
  int64_t unit = budget / wsum;
  const int64_t maxunit = std::max<int64_t>(1, rows / (64 * 2));
  unit = std::max<int64_t>(1, std::min(unit, maxunit));
  gp.off[0] = 0;
  for (int g = 0; g < gp.ngroups; ++g) gp.off[g + 1] = gp.off[g] + (int)(unit * wt[g]);
  gp.total = gp.off[gp.ngroups];
  return gp;
}

}  // namespace

size_t gram_part_bytes(int lp, int ncu) {
  (void)lp;
  return (size_t)2 * ncu * 16 * 256 * sizeof(double);
}

hipError_t launch_gram_chol(bool y_f32, const void* Y, int64_t ldy, int64_t rows, int l, int lp,
                            double* Gm, int64_t ldg, double* part, int ncu, double eta, double* R,
                            int64_t ldr, double* Rdinv, int32_t* dep, int32_t* info,
                            OrthSync* sync, double* ni_parts, hipStream_t s) {
  if (lp > 256 || lp % 16) return hipErrorInvalidValue;
  const GramPlan gp = plan_gram(rows, lp, ncu);
  const bool ni = ni_parts != nullptr;
  CholArgs c;
  c.G = Gm; c.ldg = ldg; c.l = l; c.lp = lp; c.eta = eta; c.R = R; c.ldr = ldr;
  c.Rdinv = Rdinv; c.dep = dep; c.info = info; c.parts = ni_parts; c.sync = sync;
  const int ntiles = gp.nb * (gp.nb + 1) / 2;
  if (y_f32)
    hipLaunchKernelGGL(gram_kernel<float>, dim3(gp.total), dim3(GR_NT), 0, s, (const float*)Y, ldy,
                       rows, l, gp, part);
  else
    hipLaunchKernelGGL(gram_kernel<double>, dim3(gp.total), dim3(GR_NT), 0, s, (const double*)Y,
                       ldy, rows, l, gp, part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // 8 waves: wave 0 factors the diagonal blocks, 7 hold the tiles (2 waves
  // per SIMD leave each up to 256 registers)
#define RSVD_CHOL(T)                                                                        \
  do {                                                                                      \
    if (ni) hipLaunchKernelGGL((gram_chol_kernel<T, true>), dim3(ntiles), dim3(GR_NT), 0, s, part, \
                               gp, c);                                                      \
    else hipLaunchKernelGGL((gram_chol_kernel<T, false>), dim3(ntiles), dim3(GR_NT), 0, s, part, \
                            gp, c);                                                         \
  } while (0)
  const int tpw = (int)cdiv(ntiles, 7);
  if (tpw <= 1) RSVD_CHOL(1);
  else if (tpw <= 2) RSVD_CHOL(2);
  else if (tpw <= 4) RSVD_CHOL(4);
  else if (tpw <= 8) RSVD_CHOL(8);
  else if (tpw <= 15) RSVD_CHOL(15);
  else RSVD_CHOL(20);
#undef RSVD_CHOL
  return hipGetLastError();
}

template <int NB>
hipError_t launch_trsm_nb(bool y_f32, bool q_f32, const void* Y, int64_t ldy, int64_t M, int l,
                          int lp, const double* R, int64_t ldr, const double* Rdinv, void* Q,
                          int64_t ldq, const double* skip_e2, const int32_t* dep, uint64_t seed,
                          uint32_t call, hipStream_t s) {
  const dim3 grid((unsigned)cdiv(M, 64));
  if (!y_f32 && !q_f32)
    hipLaunchKernelGGL((trsm_kernel<double, double, NB>), grid, dim3(256), 0, s,
                       (const double*)Y, ldy, M, l, lp, R, ldr, Rdinv, (double*)Q, ldq, skip_e2, dep,
                       seed, call);
  else if (y_f32 && q_f32)
    hipLaunchKernelGGL((trsm_kernel<float, float, NB>), grid, dim3(256), 0, s,
                       (const float*)Y, ldy, M, l, lp, R, ldr, Rdinv, (float*)Q, ldq, skip_e2, dep, seed,
                       call);
  else if (y_f32 && !q_f32)
    hipLaunchKernelGGL((trsm_kernel<float, double, NB>), grid, dim3(256), 0, s,
                       (const float*)Y, ldy, M, l, lp, R, ldr, Rdinv, (double*)Q, ldq, skip_e2, dep,
                       seed, call);
  else
    hipLaunchKernelGGL((trsm_kernel<double, float, NB>), grid, dim3(256), 0, s,
                       (const double*)Y, ldy, M, l, lp, R, ldr, Rdinv, (float*)Q, ldq, skip_e2, dep, seed,
                       call);
  return hipGetLastError();
}

hipError_t launch_trsm(bool y_f32, bool q_f32, const void* Y, int64_t ldy, int64_t M, int l,
                       int lp, const double* R, int64_t ldr, const double* Rdinv, void* Q,
                       int64_t ldq, hipStream_t s, const double* skip_e2, const int32_t* dep,
                       uint64_t seed, uint32_t call) {
  if (M <= 0) return hipSuccess;
  if (lp > 256 || lp % 16) return hipErrorInvalidValue;
  const int nb = lp / 16;
  if (nb <= 2)
    return launch_trsm_nb<2>(y_f32, q_f32, Y, ldy, M, l, lp, R, ldr, Rdinv, Q, ldq,
                             skip_e2, dep, seed, call, s);
  if (nb <= 4)
    return launch_trsm_nb<4>(y_f32, q_f32, Y, ldy, M, l, lp, R, ldr, Rdinv, Q, ldq,
                             skip_e2, dep, seed, call, s);
  if (nb <= 8)
    return launch_trsm_nb<8>(y_f32, q_f32, Y, ldy, M, l, lp, R, ldr, Rdinv, Q, ldq,
                             skip_e2, dep, seed, call, s);
  if (nb <= 12)
    return launch_trsm_nb<12>(y_f32, q_f32, Y, ldy, M, l, lp, R, ldr, Rdinv, Q, ldq,
                             skip_e2, dep, seed, call, s);
  return launch_trsm_nb<16>(y_f32, q_f32, Y, ldy, M, l, lp, R, ldr, Rdinv, Q, ldq, skip_e2, dep,
                            seed, call, s);
}

hipError_t launch_trmm_upper(const double* A, int64_t lda, const double* B, int64_t ldb,
                             const int32_t* bdep, double* C, int64_t ldc, int lp, hipStream_t s) {
  if (lp > 256 || lp % 16) return hipErrorInvalidValue;
  const int nb = lp / 16;
  hipLaunchKernelGGL(trmm_kernel, dim3((unsigned)cdiv(nb * nb, 4)), dim3(256), 0, s, A, lda, B,
                     ldb, bdep, C, ldc, lp);
  return hipGetLastError();
}

hipError_t launch_set_word(int32_t* w, int32_t v, hipStream_t s) {
  hipLaunchKernelGGL(set_word_kernel, dim3(1), dim3(1), 0, s, w, v);
  return hipGetLastError();
}

hipError_t launch_reset(int32_t* info, OrthSync* s0, OrthSync* s1, hipStream_t s) {
  hipLaunchKernelGGL(reset_kernel, dim3(1), dim3(64), 0, s, info, s0, s1);
  return hipGetLastError();
}

hipError_t launch_rsub(bool y_f32, const void* Y, int64_t ldy, double* T, int64_t ldt,
                       int64_t rows, int cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  int64_t grid = cdiv(rows * cols, 256);
  if (grid > 16384) grid = 16384;
  if (y_f32)
    hipLaunchKernelGGL(rsub_kernel<float>, dim3((unsigned)grid), dim3(256), 0, s,
                       (const float*)Y, ldy, T, ldt, rows, cols);
  else
    hipLaunchKernelGGL(rsub_kernel<double>, dim3((unsigned)grid), dim3(256), 0, s,
                       (const double*)Y, ldy, T, ldt, rows, cols);
  return hipGetLastError();
}

hipError_t launch_zero_dep_rows(double* R, int64_t ldr, int l, int lp, const int32_t* dep,
                                hipStream_t s) {
  if (l <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_dep_rows_kernel, dim3(l), dim3(64), 0, s, R, ldr, lp, dep);
  return hipGetLastError();
}

}  // namespace rsvd
