// The passes over A (and the other products of one type) in FP64 and FP32 with
// A in registers: C[M x L] = op(A) X on the stream-K units of gemm.hip.
//
// The tile kernel of gemm.hip stages both operands in LDS behind one barrier
// per 16-deep k-step, where its eight waves drain the matrix cores together
// (72% of the FP64 matrix peak at l = 220, FP32 54%).  Here:
//  * 4 waves per workgroup, a wave owns 32 rows of all BN = 16 NB columns; no
//    other wave needs its rows of A, so they go from memory straight into its
//    registers, one k-step ahead (a k-step is 2 NB products x 4: 3 us of matrix
//    time at NB = 14).  FP64: one wave per SIMD (2 x NB accumulator blocks of 8
//    registers); FP32: two workgroups per compute unit.
//  * X, which all four waves read, passes through three LDS stages of 16
//    k-rows: loaded into registers and stored two steps ahead, so that the
//    first operand reads of a step go out in the step before, behind its
//    products.  One barrier per step, which no wave reaches before its
//    products are issued.
//  * Loads, LDS stores and operand reads are spread over the products.
//  * The accumulators stay in the accumulation registers through the k loop
//    (assembly products: through the builtins the register allocator moves them
//    inside it).  The waits around these products are in the source (settle,
//    settle_operands), tied to the registers that they stand for.
//
// Products (16 x 16 x 4; lane l, g = l / 16, c = l % 16): A operand A[row c][k g],
// B operand X[k g][col c].  A product sums over k in any order, so k is dealt to
// (product, g) as the loads of A give it: not transposed, a lane's load holds KN
// consecutive k of row 16 rb + c (FP32: 4.  FP64: 1, or 2 dealt by lane swaps, so
// that product i sums k = 4 i .. 4 i + 3, as in the tile kernel and as transposed:
// both kernels then give the same bits for the same work ranges); transposed (a row of A's storage is
// one k), it holds the two rows m = 2 c, 2 c + 1 of k = 4 i + g, which go to
// accumulator blocks rb = 0, 1.  Columns 2 c and 2 c + 1 of 32 go to two
// accumulator blocks, so a lane reads both with one LDS access and writes two
// consecutive results (an odd last block holds column c).
//
// Loads need the element's own alignment only.  Every k-step but a tile's last
// reads rows k <= K - 2 only: a pair that crosses the edge of op(A)'s rows or
// of X's columns then reads the start of the next row (its results are
// discarded), never past the end.  The last step reads element by element
// with zeros outside.
// Measured (the tile kernel -> this one, A X / A^T X, with the fix-up; FP64 bits
// equal), 20000 x 10000: FP64 l = 220 1539 / 1502 -> 1334 / 1338 us (65.8 TFLOP/s;
// a large library product reaches 73), l = 64 576 / 590 -> 480 / 444, l = 40 592 /
// 590 -> 433 / 379 (the tile kernel's columns are a multiple of 32), l = 32 359 /
// 346 -> 328 / 314; FP32 l = 220 1072 / 999 -> 714 / 708, l = 30 (against a
// streaming kernel without LDS) 259 / 239 -> 199 / 187 us.  FP64 16384 x 8192, l =
// 576: 2549 / 2578 -> 2244 / 2272 us; 8192 x 4096, l = 80: 163 / 148 -> 132 / 113.
#pragma once

#include <type_traits>

#include "common.h"
#include "internal.h"

namespace rsvd {
namespace gemmreg {

constexpr int BM = 128;
constexpr int BK = 16;
constexpr int NT = 256;
constexpr int NS = 3;

struct Args {
  const void* A; int64_t lda;
  const void* X; int64_t ldx;
  void* C; int64_t ldc;
  int64_t M, K, L;
  int64_t nct, KI, U, G;
  void* part;
};

template <typename T> struct Vec;
template <> struct Vec<double> {
  typedef double v2 __attribute__((ext_vector_type(2)));            // aligned (LDS, partial tiles)
  typedef double u2 __attribute__((ext_vector_type(2), aligned(8)));   // as stored by the caller
  typedef d4 acc;
};
template <> struct Vec<float> {
  typedef float v2 __attribute__((ext_vector_type(2)));
  typedef float u2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef f4 acc;
};

// k values of a lane's load of A, not transposed (FP32: 16 bytes; FP64: 16
// bytes where the pass is bound by reading A, else 8, which need no lane swaps)
template <typename T, int NB> constexpr int kload() {
  return sizeof(T) == 4 ? 4 : NB <= 5 ? 2 : 1;
}
template <typename T, int N> struct KVec;
template <> struct KVec<double, 1> { typedef double type; };
template <> struct KVec<double, 2> { typedef Vec<double>::u2 type; };
template <> struct KVec<float, 4> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};

#if defined(__HIP_DEVICE_COMPILE__)
// AC: the accumulator in the accumulation registers, else in ordinary ones
template <bool AC> __device__ __forceinline__ void mma(d4& acc, double a, double b) {
  if constexpr (AC) asm volatile("v_mfma_f64_16x16x4_f64 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f64_16x16x4_f64 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
template <bool AC> __device__ __forceinline__ void mma(f4& acc, float a, float b) {
  if constexpr (AC) asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// Wait states that the compiler does not insert, since it does not see the matrix
// instructions: two between a vector instruction and the products that read what it
// wrote, their own length (19 states in FP64, 10 in FP32) between the last products
// and a read of the accumulators.  Each is tied to the registers it stands for: a
// bare wait leaves the compiler free to move their other accesses across it.
template <bool AC, typename V> __device__ __forceinline__ void tie(V& x) {
  if constexpr (AC) asm volatile("" : "+a"(x));
  else asm volatile("" : "+v"(x));
}
// the accumulators: what was written before is read by the products after this, and
// the results of the products before are there after it
template <bool AC, typename V, int S, int N>
__device__ __forceinline__ void settle(V (&acc)[S][2][N]) {
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) tie<AC>(acc[s][i / N][i % N]);
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) tie<AC>(acc[s][i / N][i % N]);
}
__device__ __forceinline__ int opaque_zero() {
  int z;
  asm volatile("v_mov_b32 %0, 0" : "=v"(z));
  return z;
}
// a step's A
template <typename R> __device__ __forceinline__ void settle_operands(R& r) {
#pragma unroll
  for (int i = (int)(sizeof(r.v) / sizeof(r.v[0])) - 1; i > 0; --i) asm volatile("" : "+v"(r.v[i]));
  asm volatile("s_nop 1" : "+v"(r.v[0]));
}
// a column group's X
template <typename V> __device__ __forceinline__ void settle_operands(V (&x)[4]) {
#pragma unroll
  for (int i = 3; i > 0; --i) tie<false>(x[i]);
  asm volatile("s_nop 1" : "+v"(x[0]));
}
#else   // (the host pass does not know the register constraints)
template <typename R> __device__ void settle_operands(R& r);
template <typename V> __device__ void settle_operands(V (&x)[4]);
__device__ int opaque_zero();
template <bool AC> __device__ void mma(d4& acc, double a, double b);
template <bool AC> __device__ void mma(f4& acc, float a, float b);
template <bool AC, typename V, int S, int N> __device__ void settle(V (&acc)[S][2][N]);
#endif

__device__ __forceinline__ int64_t range_begin(int64_t w, int64_t U, int64_t G) {
  return (w * U) / G;
}

// every load has arrived (s_waitcnt vmcnt(0), the other counters left alone)
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// workgroups per compute unit that the registers allow (FP64: 16 NB for the
// accumulators)
template <typename T, int NB> constexpr int wgs() { return sizeof(T) == 4 || NB <= 4 ? 2 : 1; }

template <typename T, bool TRANS, int NB>
__global__ __launch_bounds__(NT)
    __attribute__((amdgpu_waves_per_eu(wgs<T, NB>(), wgs<T, NB>()))) void kernel(Args g) {
  typedef Vec<T> V;
  typedef typename V::v2 v2;
  typedef typename V::u2 u2;
  constexpr int BN = 16 * NB;
  constexpr bool DEEP = NB <= 2;                  // short steps: loads several steps ahead
  // FP32 sums of a short step in four chains, one per product of the step (registers
  // are free there): relative error of a pair of passes at 20000 x 10000, l = 30
  // against 64 bits 9.6e-7 -> 4.8e-7 at the same time
  constexpr int SETS = sizeof(T) == 4 && DEEP ? 4 : 1;
  constexpr int NG = (NB + 1) / 2;                // column groups (two blocks; the last may be one)
  constexpr int XPT = (NB + 1) / 2;               // pairs of X per thread and step
  constexpr int XP = BK * BN / 2;                 // pairs of X per step
  // A loads per step: not transposed, N k's per load; transposed, two rows
  constexpr int KN = kload<T, NB>();
  constexpr int NA = TRANS ? 4 : 2 * (BK / 4 / KN);
  __shared__ __attribute__((aligned(16))) T sm[NS][BK * BN];

  const T* __restrict__ A = static_cast<const T*>(g.A);
  const T* __restrict__ X = static_cast<const T*>(g.X);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15;
  const int q = lane >> 4;

  const int64_t w = blockIdx.x;
  int64_t u = range_begin(w, g.U, g.G);
  const int64_t uend = range_begin(w + 1, g.U, g.G);

  // one step's A in registers: operand(p, rb) of product p, row block rb
  struct RawN { typename KVec<T, KN>::type v[TRANS ? 1 : NA]; };
  struct RawT { u2 v[4]; };
  typedef typename std::conditional<TRANS, RawT, RawN>::type raw_t;
  auto operand = [](const raw_t& r, int p, int rb) -> T {
    if constexpr (TRANS) return r.v[p][rb];
    else if constexpr (KN == 1) return r.v[rb * (NA / 2) + p];
    else return r.v[rb * (NA / 2) + p / KN][p % KN];
  };
  // k-row (of the 16 of a step) of product p in lane group g
  auto krow = [](int p, int g_) {
    return TRANS || KN <= 2 ? 4 * p + g_ : 4 * KN * (p / KN) + KN * g_ + p % KN;
  };
  // FP64, not transposed: the pairs k = 8 h + 2 g, + 1 as loaded become the
  // operands k = 8 h + g and 8 h + 4 + g of products 2 h, 2 h + 1
  auto deal = [](raw_t& r) {
    if constexpr (!TRANS && KN == 2) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const long long x = __double_as_longlong(r.v[i][0]), y = __double_as_longlong(r.v[i][1]);
        uint32_t o[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const auto s = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> (32 * h)),
                                                          (uint32_t)(y >> (32 * h)), false, false);
          const auto t = __builtin_amdgcn_permlane32_swap(s[0], s[1], false, false);
          o[0][h] = t[0];
          o[1][h] = t[1];
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
          r.v[i][j] = __longlong_as_double(((long long)o[j][1] << 32) | o[j][0]);
      }
    }
  };

  while (u < uend) {
    const int64_t tile = u / g.KI;
    const int64_t kb = u - tile * g.KI;
    const int64_t ke = min(g.KI, kb + (uend - u));
    u += ke - kb;
    const int64_t row0 = (tile / g.nct) * BM;
    const int64_t col0 = (tile % g.nct) * BN;
    const int64_t m0 = row0 + wave * 32;          // the wave's first row
    const int64_t lastf = g.KI - 2;               // the last step that reads freely (KI >= 2)

    typename V::acc acc[SETS][2][NB];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[s][i][j] = Mfma<T>::zero();

    // addresses of this lane's loads at k = 0 (rows past M and columns past L
    // read others, which are discarded)
    const T* ap[TRANS ? 1 : 2];
    if constexpr (TRANS) {
      const int64_t m = m0 + 2 * c;
      ap[0] = A + q * g.lda + (m < g.M ? m : 0);
    } else {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) ap[rb] = A + min(m0 + 16 * rb + c, g.M - 1) * g.lda + KN * q;
    }
    // (one address where a thread's pairs lie in one column, XR rows apart: with one
    // per pair the 16 blocks of FP32 do not fit, and an accumulator block left the
    // accumulation registers in every step)
    constexpr int XR = NT % (BN / 2) == 0 ? NT / (BN / 2) : 0;
    const T* xp[XR ? 1 : XPT];
#pragma unroll
    for (int i = 0; i < (XR ? 1 : XPT); ++i) {
      const int ch = tid + i * NT;
      const int64_t col = col0 + 2 * (ch % (BN / 2));
      xp[i] = X + (ch < XP ? ch / (BN / 2) : 0) * g.ldx + (col < g.L ? col : 0);
    }
    auto aload1 = [&](raw_t& r, int i, int64_t kt) {
      if constexpr (TRANS) r.v[i] = *reinterpret_cast<const u2*>(ap[0] + (kt * BK + 4 * i) * g.lda);
      else
        r.v[i] = *reinterpret_cast<const typename KVec<T, KN>::type*>(
            ap[i / (NA / 2)] + kt * BK + 4 * KN * (i % (NA / 2)));
    };
    auto xload1 = [&](u2 (&rx)[XPT], int i, int64_t kt) {
      rx[i] = *reinterpret_cast<const u2*>(xp[XR ? 0 : i] + (kt * BK + XR * i) * g.ldx);
    };
    auto xstore1 = [&](const u2 (&rx)[XPT], int i, int b) {
      const int ch = tid + i * NT;
      if (XP % NT == 0 || i + 1 < XPT || ch < XP) *reinterpret_cast<v2*>(&sm[b][2 * ch]) = v2(rx[i]);
    };

    v2 bq[2][4];                                  // operands of a column group: current, next
    auto bread = [&](int slot, int b, int grp) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const T* s = &sm[b][krow(p, q) * BN + 32 * grp];
        if (NB % 2 && grp == NG - 1) bq[slot][p][0] = s[c];
        else bq[slot][p] = *reinterpret_cast<const v2*>(s + 2 * c);
      }
    };
    // The products of one step on LDS stage b, group i's operands in slot (s0 + i)
    // & 1; group 0 of stage nx is read behind the last ones.  extra(e), e < NE,
    // are the step's other memory operations, spread evenly over its products.
    constexpr int NE = DEEP ? 2 * XPT + NA : 2 * (XPT + NA);
    auto step = [&](const raw_t& r, int b, int nx, int s0, auto&& extra) {
      constexpr int NM = 8 * NB;
      int m = 0;
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        const int cur = (s0 + i) & 1;
        const int nb = (NB % 2 && i == NG - 1) ? 1 : 2;
        if (i + 1 < NG) bread(cur ^ 1, b, i + 1);
        else bread(cur ^ 1, nx, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int j = 0; j < nb; ++j)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
              mma<!DEEP>(acc[p % SETS][rb][2 * i + j], operand(r, p, rb), bq[cur][p][j]);
#pragma unroll
              for (int e = m * NE / NM; e < (m + 1) * NE / NM; ++e) {
                __builtin_amdgcn_sched_barrier(0);
                extra(e);
                __builtin_amdgcn_sched_barrier(0);
              }
              ++m;
            }
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    // the tile's last step: zeros outside the operands (their addresses are
    // formed there: left to itself the compiler keeps them in registers
    // through the whole loop; and their loads are waited for there: where the
    // paths join, it would wait for the loads in flight of the other one)
    auto aload_last = [&](raw_t& r) {
      const int z = opaque_zero(), c = (lane & 15) + z, q = (lane >> 4) + z;
      const int64_t k0 = (g.KI - 1) * BK;
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          const int64_t k = k0 + krow(p, q);
          const int64_t m = m0 + (TRANS ? 2 * c + rb : 16 * rb + c);
          const T v = (k < g.K && m < g.M) ? A[TRANS ? k * g.lda + m : m * g.lda + k] : T(0);
          if constexpr (TRANS) r.v[p][rb] = v;
          else if constexpr (KN == 1) r.v[rb * (NA / 2) + p] = v;
          else r.v[rb * (NA / 2) + p / KN][p % KN] = v;
        }
      wait_loads();
    };
    auto xstore_last = [&](int b) {
      const int tid = threadIdx.x + opaque_zero();
      const int64_t k0 = (g.KI - 1) * BK;
#pragma unroll
      for (int i = 0; i < XPT; ++i) {
        const int ch = tid + i * NT;
        if (ch < XP) {
          const int64_t k = k0 + ch / (BN / 2), col = col0 + 2 * (ch % (BN / 2));
          v2 v;
#pragma unroll
          for (int j = 0; j < 2; ++j)
            v[j] = (k < g.K && col + j < g.L) ? X[k * g.ldx + col + j] : T(0);
          *reinterpret_cast<v2*>(&sm[b][2 * ch]) = v;
        }
      }
      wait_loads();
    };

    // Prologue: stages kb and kb + 1, the first A.  (Loads past the last free
    // step re-read it; what they bring is replaced or not used.)
    raw_t ra[DEEP ? 4 : 2];
    u2 rx[DEEP ? 2 : 1][XPT];
#pragma unroll
    for (int i = 0; i < XPT; ++i) xload1(rx[0], i, min(kb, lastf));
#pragma unroll
    for (int s = 0; s < (DEEP ? 3 : 1); ++s)
#pragma unroll
      for (int i = 0; i < NA; ++i) aload1(ra[s], i, min(kb + s, lastf));
#pragma unroll
    for (int i = 0; i < XPT; ++i) xstore1(rx[0], i, 0);
#pragma unroll
    for (int i = 0; i < XPT; ++i) xload1(rx[0], i, min(kb + 1, lastf));
#pragma unroll
    for (int i = 0; i < XPT; ++i) xstore1(rx[0], i, 1);
    if constexpr (DEEP) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < XPT; ++i) xload1(rx[s], i, min(kb + 2 + s, lastf));
    }
    if (kb >= lastf) {
      xstore_last(kb == lastf ? 1 : 0);
      if (kb > lastf) aload_last(ra[0]);
    }
    if constexpr (!DEEP) {
      if (kb <= lastf) deal(ra[0]);
      settle_operands(ra[0]);
    }
    __syncthreads();
    bread(0, 0, 0);
    settle<!DEEP>(acc);
    int b = 0;
    if constexpr (!DEEP) {
      // Step t: the loads of A for t + 1 and of X for t + 2 go out in its first
      // half, X is stored in its second half; the barrier at its end makes
      // stage t + 2 visible (one step early) and frees stage t.  The loaded A
      // then moves to its place (a few moves per step; two buffers in turn
      // would need two copies of the step, between which the allocator moves
      // accumulators).
      for (int64_t t = kb; t < ke; ++t) {
        const int b1 = b == NS - 1 ? 0 : b + 1, b2 = b1 == NS - 1 ? 0 : b1 + 1;
        const int64_t ta = min(t + 1, lastf), tx = min(t + 2, lastf);
        step(ra[0], b, b1, 0, [&](int e) {
          if (e < XPT) xload1(rx[0], e, tx);
          else if (e < XPT + NA) aload1(ra[1], e - XPT, ta);
          else if (e >= 2 * NA + XPT) xstore1(rx[0], e - (2 * NA + XPT), b2);
        });
        ra[0] = ra[1];
        if (t < lastf) deal(ra[0]);
        if (t + 1 >= lastf) {
          if (t + 1 == lastf) xstore_last(b2);
          else if (t == lastf) aload_last(ra[0]);
        }
        settle_operands(ra[0]);
        b = b1;
        if (NG & 1) {
#pragma unroll
          for (int p = 0; p < 4; ++p) bq[0][p] = bq[1][p];
        }                                         // (the barrier's wait follows)
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
      }
    } else {
      // The same with short steps (up to 32 columns: bound by reading A), whose
      // loads take several of them: A is loaded three steps ahead (four buffers
      // in turn), X two steps before it is stored.  The loop has no branch: where
      // the paths of one join, the compiler waits for loads in flight.  The last
      // steps of the range run one by one.
      int64_t t = kb;
      auto dstep = [&](auto sc, int64_t t) {
        constexpr int S = decltype(sc)::value;    // t - kb modulo 4
        const int b1 = b == NS - 1 ? 0 : b + 1, b2 = b1 == NS - 1 ? 0 : b1 + 1;
        const int64_t ta = min(t + 3, lastf), tx = min(t + 4, lastf);
        deal(ra[S]);
        settle_operands(ra[S]);
        step(ra[S], b, b1, (S * NG) & 1, [&](int e) {
          if (e < NA) aload1(ra[(S + 3) % 4], e, ta);
          else if (e < NA + XPT) xstore1(rx[S % 2], e - NA, b2);
          else xload1(rx[S % 2], e - NA - XPT, tx);
        });
        b = b1;
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
      };
      for (const int64_t te = min(ke, lastf - 1); t + 3 < te; t += 4) {
        dstep(std::integral_constant<int, 0>(), t);
        dstep(std::integral_constant<int, 1>(), t + 1);
        dstep(std::integral_constant<int, 2>(), t + 2);
        dstep(std::integral_constant<int, 3>(), t + 3);
      }
      for (; t < ke; ++t) {
        const int b1 = b == NS - 1 ? 0 : b + 1, b2 = b1 == NS - 1 ? 0 : b1 + 1;
        const int64_t ta = min(t + 3, lastf), tx = min(t + 4, lastf);
        if (t <= lastf) deal(ra[0]);
        settle_operands(ra[0]);
        step(ra[0], b, b1, 0, [&](int e) {
          if (e < NA) aload1(ra[3], e, ta);
          else if (e < NA + XPT) xstore1(rx[0], e - NA, b2);
        });
#pragma unroll
        for (int s = 0; s < 3; ++s) ra[s] = ra[s + 1];
#pragma unroll
        for (int i = 0; i < XPT; ++i) rx[0][i] = rx[1][i];
#pragma unroll
        for (int i = 0; i < XPT; ++i) xload1(rx[1], i, tx);
        if (t + 1 == lastf) xstore_last(b2);
        if (t == lastf) aload_last(ra[0]);
        b = b1;
        if (NG & 1) {
#pragma unroll
          for (int p = 0; p < 4; ++p) bq[0][p] = bq[1][p];
          settle_operands(bq[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
      }
    }
    settle<!DEEP>(acc);
    if constexpr (SETS == 4) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[0][i][j] = (acc[0][i][j] + acc[1][i][j]) + (acc[2][i][j] + acc[3][i][j]);
    }

    // results: element v of block rb is row Mfma::row(q, v) of the block's 16
    const bool full = (kb == 0) && (ke == g.KI);
    T* C = static_cast<T*>(g.C);
    T* P = static_cast<T*>(g.part) + (2 * w + (kb == 0 ? 1 : 0)) * (int64_t)(BM * BN);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int rr = Mfma<T>::row(q, v);
        const int rl = wave * 32 + (TRANS ? 2 * rr + rb : 16 * rb + rr);
        const int64_t r = row0 + rl;
        if (full) {
          if (r < g.M) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              const int64_t col = col0 + ((NB % 2 && j == NB - 1) ? 16 * j + c
                                                                  : 32 * (j / 2) + 2 * c + j % 2);
              if (col < g.L) C[r * g.ldc + col] = acc[0][rb][j][v];
            }
          }
        } else {
#pragma unroll
          for (int i = 0; i < NG; ++i) {
            if (NB % 2 && i == NG - 1) P[rl * BN + 32 * i + c] = acc[0][rb][2 * i][v];
            else
              *reinterpret_cast<v2*>(&P[rl * BN + 32 * i + 2 * c]) =
                  v2{acc[0][rb][2 * i][v], acc[0][rb][(2 * i + 1) % NB][v]};
          }
        }
      }
    __syncthreads();                              // (the next tile's stages)
  }
}

}  // namespace gemmreg
}  // namespace rsvd
