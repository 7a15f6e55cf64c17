// The passes over a narrow A (BF16, or FP8 E4M3 codes) on the matrix cores:
//
//   C[M x L] (FP32) = op(A) X,  op(A) = A (M x K) or A^T (A stored K x M),
//
// with the skinny operand given transposed and narrow (Xt, L x K, k
// contiguous).  One kernel template for both element sizes: a k-step is 128
// bytes of a row of Xt (64 BF16 or 128 FP8 values).
//
// Tiles: 4 waves per workgroup, one per SIMD, BM = 256 rows x BN = 16 NB
// columns (NB <= 18, so l = 576 takes two column tiles); a wave owns 64 rows
// of all BN columns (4 x NB accumulator blocks, 288 registers at NB = 18).
//  * A goes from memory straight into the registers of the wave that uses
//    it: no other wave needs those rows, so LDS would only add a round trip.
//    Its loads go out two k-steps ahead (a k-step is ~1 us of products at
//    NB = 18, the loaded-memory latency 1 - 2 us).
//  * Xt, which all four waves read, is moved by the direct-to-LDS loads into
//    four LDS stages.  Per k-step the LDS then serves 4 x 2 NB KB of operand
//    reads and 2 NB KB of writes, 62% of the products' time at any NB.  (With
//    both operands in LDS and 8 waves of 32 x 288 rows the operand reads
//    alone took 110% of the products' time, and the pass ran at their rate.)
//  * A^T: a row of A's storage holds one k for consecutive rows m of the
//    result.  A lane loads the m = 4 c .. 4 c + 3 of its k values and takes row
//    4 c + rb into accumulator block rb, so the transposition is a byte
//    permutation among its own registers.
// One barrier per k-step.  It makes the next stage visible one step before it
// is multiplied, so the first operand reads of a step are issued in the step
// before, behind its products.
//
// MFMA operand layouts (lane l, g = l / 16, c = l % 16): 16x16x32 BF16: lane l
// holds 8 consecutive k (16 bytes) of row c; 16x16x128 FP8: 32 bytes of row
// c.  A product sums over k in any order, so the 16-byte chunks g and 4 + g of
// the 128-byte row stand for the two products of a BF16 k-step and for the two
// halves of an FP8 operand alike.  D: lane l element v holds D[4 g + v][c].
#pragma once

#include <type_traits>

#include "common.h"
#include "internal.h"

namespace rsvd {
namespace lowp {

typedef unsigned int u4v __attribute__((ext_vector_type(4)));   // 16 bytes
typedef int i8v __attribute__((ext_vector_type(8)));            // 32 bytes
typedef __attribute__((address_space(3))) void* lds_vp;
typedef __attribute__((address_space(1))) void* gbl_vp;

constexpr int BM = 256;            // rows per tile (4 waves x 64)
constexpr int NT = 256;
constexpr int NW = 4;
constexpr int SB = 128;            // bytes of k per step
constexpr int NS = 4;              // LDS stages of Xt
constexpr int MAX_NB = 18;

struct Args {
  const uint8_t* A; int64_t lda;   // bytes
  const uint8_t* X; int64_t ldx;   // bytes; Xt: rup(L, 16) rows, zero from K to ldx
  float* C; int64_t ldc;
  int64_t M, K, L;                 // elements
  int64_t nrt, nct;
  int64_t P, W;                    // tile numbers; the first W are whole tiles, the
  int S;                           // others (W = 0: all tiles) in S k splits (in part)
  float* part;
  const float* xs;                 // FP8: L column scales (null: none)
  const float* rs;                 // FP8: M row scales (null: none)
  int accumulate;                  // C += instead of C =
};

// s_waitcnt that waits until at most N vector-memory operations are in
// flight (lgkm and exp counters left alone)
template <int N> __device__ __forceinline__ void wait_vm() {
  constexpr int n = N > 63 ? 63 : N;
  __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));
}

// One operand of 16 rows for a k-step: two 16-byte chunks per lane.
template <int ELT> struct Opnd;
template <> struct Opnd<2> {
  u4v h[2];
  __device__ __forceinline__ void set(int kk, const u4v& v) { h[kk] = v; }
};
template <> struct Opnd<1> {
  i8v h;
  __device__ __forceinline__ void set(int kk, const u4v& v) {
#pragma unroll
    for (int d = 0; d < 4; ++d) h[4 * kk + d] = (int)v[d];
  }
};

// One product (product KK of a BF16 k-step) on one accumulator block.  Written as assembly
// so that the accumulator stays in place: AC = true in the accumulation
// registers (256 of them: 16 column blocks x 4), AC = false in ordinary ones.
// (Through the builtins the register allocator moved accumulators between
// the two files inside the k loop, 150 - 250 moves per step, and spilled.)
// The compiler does not see a matrix instruction here: a value written by an
// ordinary vector instruction is used two wait states later at the earliest
// (opnd_settle), and the accumulators are read or moved only after acc_settle (the
// register allocator spills some between the k loop and its rest).  Both are tied
// to the registers they stand for: a bare wait leaves the compiler free to move
// other accesses of them across it.
#if defined(__HIP_DEVICE_COMPILE__)
template <int ELT, bool AC, int KK>
__device__ __forceinline__ void mma(f4& acc, const Opnd<ELT>& a, const Opnd<ELT>& b) {
  if constexpr (ELT == 2) {
    if constexpr (AC)
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                   : "+a"(acc) : "v"(a.h[KK]), "v"(b.h[KK]));
    else
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                   : "+v"(acc) : "v"(a.h[KK]), "v"(b.h[KK]));
  } else {
    if constexpr (AC)
      asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+a"(acc) : "v"(a.h), "v"(b.h));
    else
      asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+v"(acc) : "v"(a.h), "v"(b.h));
  }
}
// vector writes of the operands have reached the matrix core (two wait states)
template <int ELT> __device__ __forceinline__ void opnd_settle(Opnd<ELT> (&av)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (ELT == 2) asm volatile("" : "+v"(av[i].h[0]), "+v"(av[i].h[1]));
    else asm volatile("" : "+v"(av[i].h));
  }
  asm volatile("s_nop 1" ::: "memory");
}
// the accumulators (block j < 16 in the accumulation registers)
template <int NB> __device__ __forceinline__ void acc_tie(f4 (&acc)[4][NB]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j < 16) asm volatile("" : "+a"(acc[i][j]));
      else asm volatile("" : "+v"(acc[i][j]));
    }
}
// the last products (at most 8 passes, 32 cycles) have written their results
template <int NB> __device__ __forceinline__ void acc_settle(f4 (&acc)[4][NB]) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  acc_tie(acc);
}
// a copy the optimizer keeps: the loaded register is free for the next load
__device__ __forceinline__ uint32_t move_u32(uint32_t x) {
  uint32_t y;
  asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
  return y;
}

#else   // (the host pass does not know the register constraints)
template <int ELT, bool AC, int KK>
__device__ void mma(f4& acc, const Opnd<ELT>& a, const Opnd<ELT>& b);
template <int ELT> __device__ void opnd_settle(Opnd<ELT> (&av)[4]);
template <int NB> __device__ void acc_tie(f4 (&acc)[4][NB]);
template <int NB> __device__ void acc_settle(f4 (&acc)[4][NB]);
__device__ uint32_t move_u32(uint32_t x);
#endif

// mask of the first n bytes of a word (n clamped to 0..4)
__device__ __forceinline__ uint32_t byte_mask(int64_t n) {
  return n >= 4 ? 0xFFFFFFFFu : n <= 0 ? 0u : (0xFFFFFFFFu >> (32 - 8 * (int)n));
}

// The A registers of one k-step, as loaded (32 words per lane; element types as
// loaded, so that a load's registers stay one tuple):
//  not transposed: chunk kk of row block rb in v[2 rb + kk];
//  transposed, BF16: k value i of chunk kk, rows 4 c .. 4 c + 3 in v[8 kk + i];
//  transposed, FP8: the same in v[16 kk + i].
typedef unsigned int u2v __attribute__((ext_vector_type(2)));
template <int ELT, bool TRANS> struct RawT { typedef u4v type; };
template <> struct RawT<2, true> { typedef u2v type; };
template <> struct RawT<1, true> { typedef unsigned int type; };
template <int ELT, bool TRANS> struct Raw {
  typedef typename RawT<ELT, TRANS>::type vec;
  static constexpr int N = 128 / (int)sizeof(vec);
  vec v[N];
};

// chunk kk of row block rb from the loaded words
template <int ELT, bool TRANS>
__device__ __forceinline__ u4v operand(const Raw<ELT, TRANS>& r, int rb, int kk) {
  u4v o;
  if constexpr (!TRANS) {
#pragma unroll
    for (int d = 0; d < 4; ++d) o[d] = move_u32(r.v[2 * rb + kk][d]);
  } else if constexpr (ELT == 2) {
    // halves (rb & 1) of two k values
#pragma unroll
    for (int d = 0; d < 4; ++d)
      o[d] = __builtin_amdgcn_perm(r.v[8 * kk + 2 * d + 1][rb >> 1], r.v[8 * kk + 2 * d][rb >> 1],
                                   (rb & 1) ? 0x07060302u : 0x05040100u);
  } else {
    // byte rb of four k values: pairs first, then the pairs together
    const uint32_t sel = 0x0c0c0000u | ((uint32_t)(4 + rb) << 8) | (uint32_t)rb;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const unsigned int* p = &r.v[16 * kk + 4 * d];
      const uint32_t lo = __builtin_amdgcn_perm(p[1], p[0], sel);
      const uint32_t hi = __builtin_amdgcn_perm(p[3], p[2], sel);
      o[d] = lo | (hi << 16);
    }
  }
  return o;
}

template <int ELT, bool TRANS, int NB>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1))) void pass_kernel(Args g) {
  constexpr int BN = 16 * NB;
  constexpr int KS = SB / ELT;                    // elements of k per step
  constexpr int STAGE = BN * SB;                  // bytes
  constexpr int NDMA = BN * SB / 1024 / NW;       // 1 KB wave loads per step and wave
  constexpr int NA = Raw<ELT, TRANS>::N;          // A loads per step and wave
  constexpr int GB = (NB % 3 == 0) ? 3 : 2;       // column blocks per operand group
  constexpr int NG = NB / GB;
  static_assert(NB % 2 == 0 && NB <= MAX_NB, "column blocks");
  extern __shared__ __attribute__((aligned(16))) uint8_t sm[];    // NS x STAGE

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15;
  const int q = lane >> 4;

  // Workgroup -> (tile, split).  Tiles are numbered so that number p runs on
  // XCD p % 8 (workgroups are dealt to the XCDs in turn) and the workgroups of
  // one XCD that run at the same time take the column tiles of one row tile
  // (the second read of A hits that XCD's L2) and the same k range of different
  // row tiles (the same lines of Xt).  The first g.W tiles are whole, the others
  // in S splits.  Numbers past the last row tile (of 8) have no tile.
  // With W = 0 the pairs (row tile, split) take the place of the row tiles, so that a
  // few row tiles in many splits reach all XCDs.
  const int64_t w = blockIdx.x;
  const int64_t rest = g.P - g.W;
  const bool whole = w < g.W, pairs = g.W == 0;
  const int64_t p = whole || pairs ? w : g.W + (w - g.W) % rest;
  const int S = whole ? 1 : g.S;
  const int64_t ct = (p / 8) % g.nct;
  const int64_t gt = p % 8 + 8 * (p / 8 / g.nct);
  const int64_t rt = pairs ? gt % g.nrt : gt;
  const int sp = whole ? 0 : (int)(pairs ? gt / g.nrt : (w - g.W) / rest);
  if (sp >= S) return;
  if (rt >= g.nrt) return;                        // (the whole workgroup)
  const int64_t row0 = rt * BM;
  const int64_t col0 = ct * BN;
  // pairs of whole k-steps are dealt to the splits; what is left (less than
  // two steps) goes to the last split's masked steps
  const int64_t npair = g.K / (2 * KS);
  const int64_t kb = 2 * ((sp * npair) / S);
  const int64_t ke = 2 * (((sp + 1) * npair) / S);

  // --- addresses -----------------------------------------------------------
  const int64_t m0 = row0 + wave * 64;            // the wave's first row
  const uint8_t* ap[TRANS ? 1 : 4];
  if constexpr (!TRANS) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)                // (rows past M are discarded)
      ap[rb] = g.A + min(m0 + 16 * rb + c, g.M - 1) * g.lda + 16 * q;
  } else {
    // four rows m of one k: inside the row's storage when the first is below M
    const int64_t m = m0 + 4 * c;
    ap[0] = g.A + (int64_t)q * (16 / ELT) * g.lda + (m < g.M ? m : 0) * ELT;
  }
  // A DMA load moves 8 rows of Xt, lane l to slot l % 8 of row l / 8 (chunk s of
  // row r in slot s ^ (r & 7): the lanes that read one chunk of 8 rows hit 8
  // slots).  Xt has rup(L, 16) rows, so 8 rows lie inside it or past it.
  const uint8_t* xp = g.X + (lane >> 3) * g.ldx + 16 * ((lane & 7) ^ (lane >> 3));
  const int64_t xlast = rup(g.L, 16) - 8;

  auto dma1 = [&](int i, int64_t kt, int b) {     // load i of k-step kt into stage b
    const int64_t gj = min(col0 + (wave + NW * i) * 8, xlast);
    __builtin_amdgcn_global_load_lds((gbl_vp)(xp + (gj * g.ldx + kt * SB)),
                                     (lds_vp)(sm + b * STAGE + (wave + NW * i) * 1024), 16, 0, 0);
  };
  auto dma = [&](int64_t kt, int b) {
#pragma unroll
    for (int i = 0; i < NDMA; ++i) dma1(i, kt, b);
  };
  typedef Raw<ELT, TRANS> raw_t;
  typedef typename raw_t::vec avec;
  // address of A load i of the k-step that starts at element k0
  auto aaddr = [&](int i, int64_t k0) {
    if constexpr (!TRANS) return ap[i >> 1] + (k0 * ELT + 64 * (i & 1));
    else return ap[0] + (k0 + (i / (16 / ELT)) * (64 / ELT) + i % (16 / ELT)) * g.lda;
  };
  auto aload1 = [&](raw_t& r, int i, int64_t kt) {
    r.v[i] = *reinterpret_cast<const avec*>(aaddr(i, kt * KS));
  };
  auto aload = [&](raw_t& r, int64_t kt) {
#pragma unroll
    for (int i = 0; i < raw_t::N; ++i) aload1(r, i, kt);
  };

  f4 acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  acc_tie(acc);

  Opnd<ELT> bq[2][GB];                            // operand groups of Xt: current, next
  auto bread = [&](int slot, const uint8_t* st, int grp) {
#pragma unroll
    for (int i = 0; i < GB; ++i)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int r = (grp * GB + i) * 16 + c;
        bq[slot][i].set(
            kk, *reinterpret_cast<const u4v*>(st + r * SB + 16 * ((4 * kk + q) ^ (r & 7))));
      }
  };
  // The products of one k-step: group i's operands are in slot (s0 + i) & 1, read
  // behind the products of the group before (group 0's behind the last
  // products of the step before; nx is the next step's stage).  The reads
  // come after the group's first product: with direct-to-LDS loads in flight
  // the compiler waits for every LDS read there, so these must not be among them.
  // The two products of a BF16 step on one block are 4 GB products apart.
  // load(i), i < NV, issues the step's memory loads, spread evenly over its
  // products: issued together they queue at the address unit (16 cycles per
  // load, four waves), and the wave issues no product meanwhile (2.4 -> 1.9 ms
  // per pass at 65536 x 32768, l = 576, BF16).
  constexpr int KPM = ELT == 2 ? 2 : 1;           // products per block and step
  constexpr int NM = 4 * NB * KPM;
  constexpr int NV = NA + NDMA;
  auto step = [&](const Opnd<ELT> (&av)[4], const uint8_t* st, const uint8_t* nx, int s0,
                  auto&& load) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int cur = (s0 + i) & 1;
#pragma unroll
      for (int x = 0; x < 4 * GB * KPM; ++x) {
        const int j = (x / 4) % GB, rb = x % 4;
        f4& a = acc[rb][i * GB + j];
        if (x < 4 * GB) {
          if (i * GB + j < 16) mma<ELT, true, 0>(a, av[rb], bq[cur][j]);
          else mma<ELT, false, 0>(a, av[rb], bq[cur][j]);
        } else {
          if (i * GB + j < 16) mma<ELT, true, KPM - 1>(a, av[rb], bq[cur][j]);
          else mma<ELT, false, KPM - 1>(a, av[rb], bq[cur][j]);
        }
        if (x == 0) {
          __builtin_amdgcn_sched_barrier(0);
          if (i + 1 < NG) bread(cur ^ 1, st, i + 1);
          else bread(cur ^ 1, nx, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        const int m = i * 4 * GB * KPM + x;       // this product's number
#pragma unroll
        for (int v = m * NV / NM; v < (m + 1) * NV / NM; ++v) {
          __builtin_amdgcn_sched_barrier(0);
          load(v);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  if (ke > kb) {
    const int64_t last = ke - 1;
    raw_t r0, r1;
    // (loads past the range re-read its last step; no one uses them)
    dma(kb, 0);
    aload(r0, kb);
    dma(min(kb + 1, last), 1);
    aload(r1, min(kb + 1, last));
    dma(min(kb + 2, last), 2);
    wait_vm<NDMA + NA + NDMA>();                  // stage 0
    asm volatile("s_barrier" ::: "memory");
    bread(0, sm, 0);
    // One k-step: stage t + 1 and the A of step t have landed when at most
    // step t - 1's loads (A of t + 1, stage t + 2) are in flight; the barrier
    // makes every wave's part of the stage visible and frees stage t - 1.
    auto kstep = [&](raw_t& r, int64_t t, int s0) {
      __builtin_amdgcn_sched_barrier(0);
      wait_vm<NA + NDMA>();
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      Opnd<ELT> av[4];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) av[rb].set(kk, operand<ELT, TRANS>(r, rb, kk));
      opnd_settle<ELT>(av);
      __builtin_amdgcn_sched_barrier(0);
      const int64_t ta = min(t + 2, last), tx = min(t + 3, last);
      const int bx = (int)((t - kb + 3) % NS);
      step(av, sm + (int)((t - kb) % NS) * STAGE, sm + (int)((t - kb + 1) % NS) * STAGE, s0,
           [&](int v) {
             if (v < NA) aload1(r, v, ta);
             else dma1(v - NA, tx, bx);
           });
    };
    for (int64_t t = kb; t < ke; t += 2) {        // (each buffer keeps its registers)
      kstep(r0, t, 0);
      kstep(r1, t + 1, NG & 1);
    }
    acc_settle(acc);
  }
  if (sp == S - 1) {
    // the rest: both operands masked to zero past K
    for (int64_t k0 = 2 * npair * KS; k0 < g.K; k0 += KS) {
      wait_vm<0>();
      __syncthreads();
      for (int ch = tid; ch < BN * 8; ch += NT) {
        const int r = ch >> 3, s = ch & 7;
        const int64_t gj = col0 + r, gk = k0 + s * (16 / ELT);
        u4v v = u4v{0u, 0u, 0u, 0u};
        // (Xt rows are zero from K to whole chunks)
        if (gj < g.L && gk < g.K) v = *reinterpret_cast<const u4v*>(g.X + gj * g.ldx + gk * ELT);
        *reinterpret_cast<u4v*>(sm + r * SB + 16 * (s ^ (r & 7))) = v;
      }
      raw_t r;
#pragma unroll
      for (int i = 0; i < raw_t::N; ++i) {
        // a chunk that starts below K lies inside its row's storage
        if constexpr (!TRANS) {
          const int64_t nb = g.K * ELT - (k0 * ELT + 64 * (i & 1) + 16 * q);   // bytes left
          u4v v = u4v{0u, 0u, 0u, 0u};
          if (nb > 0) v = *reinterpret_cast<const u4v*>(aaddr(i, k0));
#pragma unroll
          for (int d = 0; d < 4; ++d) v[d] &= byte_mask(nb - 4 * d);
          r.v[i] = v;
        } else {
          const int64_t k = k0 + (i / (16 / ELT)) * (64 / ELT) + i % (16 / ELT) + q * (16 / ELT);
          avec v = avec(0u);
          if (k < g.K) v = *reinterpret_cast<const avec*>(aaddr(i, k0));
          r.v[i] = v;
        }
      }
      Opnd<ELT> av[4];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) av[rb].set(kk, operand<ELT, TRANS>(r, rb, kk));
      __syncthreads();
      opnd_settle<ELT>(av);
      bread(0, sm, 0);
      step(av, sm, sm, 0, [](int) {});
      acc_settle(acc);
    }
  }

  // --- results -------------------------------------------------------------
  // row of element v of block rb: 16 rb + 4 q + v, or 4 (4 q + v) + rb transposed.  The
  // scales, and for C += the old values of a row, are loaded before the first
  // store: a load between stores is waited for before the next one (FP8 pass
  // kernel, 1000 x 1000, l = 250: 59 -> 36 us; three passes at 65536 x 32768, l = 576,
  // one of them C +=: 4.29 -> 4.15 ms).
  float* P = nullptr;
  if (S > 1) P = g.part + ((pairs ? rt * g.nct + ct : p - g.W) * S + sp) * (int64_t)(BM * BN);
  auto rowloc = [&](int rb, int v) {
    return wave * 64 + (TRANS ? 4 * (4 * q + v) + rb : 16 * rb + 4 * q + v);
  };
  if (P) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) P[rowloc(rb, v) * BN + cb * 16 + c] = acc[rb][cb][v];
    return;
  }
  float xs[ELT == 1 ? NB : 1], rs[ELT == 1 ? 16 : 1];
  if constexpr (ELT == 1) {
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) xs[cb] = g.xs[min(col0 + cb * 16 + c, g.L - 1)];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      rs[i] = g.rs ? g.rs[min(row0 + rowloc(i / 4, i % 4), g.M - 1)] : 1.f;
  }
  auto value = [&](int rb, int cb, int v) {
#pragma clang fp contract(off)                    // (the scaled value is rounded before C +=)
    if constexpr (ELT == 1) return acc[rb][cb][v] * (xs[cb] * rs[4 * rb + v]);
    else return acc[rb][cb][v];
  };
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t r = row0 + rowloc(rb, v);
      if (r >= g.M) continue;
      float* cp = g.C + r * g.ldc + col0 + c;
      if (g.accumulate) {
        float y[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) y[cb] = col0 + cb * 16 + c < g.L ? cp[cb * 16] : 0.f;
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
          if (col0 + cb * 16 + c < g.L) cp[cb * 16] = y[cb] + value(rb, cb, v);
      } else {
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
          if (col0 + cb * 16 + c < g.L) cp[cb * 16] = value(rb, cb, v);
      }
    }
}

// Split mode: C = the sum of the S partial tiles of each tile, in split order
// (deterministic), scaled.  One column quad per thread: bound by reading the
// partial tiles, so the reads are 16 bytes wide.
template <int ELT, int NB>
__global__ __launch_bounds__(256) void split_sum_kernel(Args g) {
  constexpr int BN = 16 * NB;
  const int64_t tile = blockIdx.x, p0 = g.W + tile;
  const bool pairs = g.W == 0;
  const int64_t row0 = (pairs ? tile / g.nct : p0 % 8 + 8 * (p0 / 8 / g.nct)) * BM;
  const int64_t col0 = (pairs ? tile % g.nct : p0 / 8 % g.nct) * BN;
  const int e = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (e >= BM * BN) return;
  const int64_t r = row0 + e / BN;
  const int64_t c0 = col0 + e % BN;
  if (r >= g.M || c0 >= g.L) return;
  const float* p = g.part + tile * g.S * (int64_t)(BM * BN) + e;
  f4 s = *reinterpret_cast<const f4*>(p);
  for (int sp = 1; sp < g.S; ++sp) s += *reinterpret_cast<const f4*>(p + sp * (int64_t)(BM * BN));
  const float rsc = g.rs ? g.rs[r] : 1.f;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const int64_t col = c0 + d;
    if (col >= g.L) break;
    float x = s[d];
    if constexpr (ELT == 1) x *= g.rs ? g.xs[col] * rsc : g.xs[col];
    float* cp = g.C + r * g.ldc + col;
    *cp = g.accumulate ? *cp + x : x;
  }
}

// column blocks per tile: the fewest column tiles of at most 18 blocks, as
// even as pairs of blocks allow
inline void col_tiles(int64_t L, int64_t& nct, int& nb) {
  const int64_t ncb = cdiv(L, 16);
  nct = cdiv(ncb, MAX_NB);
  nb = (int)rup(cdiv(ncb, nct), 2);
}

template <int ELT, bool TRANS, int NB>
hipError_t run(const Args& g, hipStream_t s) {
  constexpr size_t shm = (size_t)NS * 16 * NB * SB;
  hipError_t e = hipFuncSetAttribute((const void*)pass_kernel<ELT, TRANS, NB>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  if (e != hipSuccess) return e;
  const int64_t rest = g.P - g.W;
  const int64_t grid = g.W ? g.W + rest * g.S : 8 * g.nct * cdiv(g.nrt * g.S, 8);
  hipLaunchKernelGGL((pass_kernel<ELT, TRANS, NB>), dim3((unsigned)grid), dim3(NT), shm, s, g);
  e = hipGetLastError();
  if (e != hipSuccess || g.S == 1) return e;
  hipLaunchKernelGGL((split_sum_kernel<ELT, NB>),
                     dim3((unsigned)(g.W ? rest : g.nrt * g.nct),
                          (unsigned)cdiv(BM * 16 * NB, 1024)), dim3(256), 0, s, g);
  return hipGetLastError();
}

// The tiling of a pass: column blocks per tile, tiles, and how the last round
// over the compute units (one workgroup each) is filled: the first W tile
// numbers are whole tiles in full rounds, the `rest` others run in S splits of
// the reduction, S minimizing the rounds they take times the k-steps of a
// split, with 8 steps added for a workgroup's start, its partial tile and the
// sum (258 tiles on 256 compute units: 2 rounds whole, 1 + 1/16 split).  At
// least 8 steps per split, and at most 2 ncu partial tiles of up to 256 columns.
struct Plan {
  int nb, S;
  int64_t nrt, nct, P, W;
};
inline Plan plan(int elt, int64_t M, int64_t K, int64_t L, int ncu) {
  Plan p;
  col_tiles(L, p.nct, p.nb);
  p.nrt = cdiv(M, BM);
  p.P = 8 * p.nct * cdiv(p.nrt, 8);
  p.W = ncu % 8 ? p.P : p.P / ncu * ncu;          // (multiples of 8)
  const int64_t rest = p.P - p.W, steps = K / (SB / elt);   // (whole k-steps)
  // tile numbers of the rest that have a tile (the padding ends at once)
  const int64_t pad = p.P - p.nct * p.nrt, live = rest > pad ? rest - pad : rest;
  p.S = 1;
  double best = (double)cdiv(live, ncu) * (double)steps;
  for (int64_t S = 2; S <= steps / 8; ++S) {
    if (rest * S * 16 * p.nb > (int64_t)2 * ncu * (16 * p.nb < 256 ? 16 * p.nb : 256)) break;
    const double t = (double)cdiv(live * S, ncu) * ((double)cdiv(steps, S) + 8.0);
    if (t < best) {
      best = t;
      p.S = (int)S;
    }
  }
  if (p.S == 1) p.W = p.P;
  // Where that leaves more than half of the compute units idle (few row tiles and a
  // short reduction: 1000 x 1000, l = 250, ran on 4 workgroups), also narrower column
  // tiles and splits of as few as two steps: more workgroups, each with fewer steps
  // and less code, which a small product waits for.  Chosen by a sum of microseconds
  // as measured: a k-step 1.1 (the latency of its loads) or its products, a
  // workgroup's start and end 4 + 1.1 per column block (code that runs once), the sum
  // of the splits 5 and its partial tiles at 2 TB/s.  Pass and sum at l = 250, BF16 /
  // FP8: 1000 x 1000 43 -> 16 / 59 -> 14 us, 4096 x 512 27 -> 16 / 51 -> 14; A^T X of
  // 512 columns and 4096 rows the same way round, 25 + 5 -> 10 + 8 / 19 + 4 -> 8 + 6;
  // 300 x 20000, l = 220: 44 + 13 -> 17 + 11 / 26 + 7 -> 20 + 8.
  if (p.nrt * p.nct * p.S * 2 <= ncu) {
    const int64_t ncb = cdiv(L, 16);
    const int nb_max = p.nb;
    double least = 1e30;
    for (int nb = nb_max; nb >= 2; nb -= 2) {
      const int64_t nct = cdiv(ncb, nb), tiles = p.nrt * nct, P = 8 * nct * cdiv(p.nrt, 8);
      if (tiles > ncu) break;
      for (int64_t S = 1; S == 1 || (S <= steps / 2 && tiles * S <= ncu); ++S) {
        if (S > 1 && tiles * S * nb > (int64_t)2 * ncu * 16) break;
        const double step = 0.055 * nb > 1.1 ? 0.055 * nb : 1.1;
        const double t = (double)(cdiv(steps, S) + 1) * step + 4.0 + 1.1 * nb +
                         (S > 1 ? 5.0 + (double)(S * p.nrt * nct * BM * 16 * nb) * 4.0 / 2e6 : 0.0);
        if (t < least) {
          least = t;
          p.nb = nb;
          p.nct = nct;
          p.P = P;
          p.S = (int)S;
          p.W = S > 1 ? 0 : P;
        }
      }
    }
  }
  return p;
}
inline size_t part_bytes(const Plan& p) {
  const int64_t tiles = p.W ? p.P - p.W : p.nrt * p.nct;
  return p.S > 1 ? (size_t)(tiles * p.S) * (size_t)(BM * 16 * p.nb) * sizeof(float) : 0;
}

// Fills in the tiling and launches (whole tiles when `part_cap` bytes do not
// hold the partial ones).
template <int ELT, bool TRANS>
hipError_t launch(Args g, int ncu, size_t part_cap, hipStream_t s) {
  const Plan p = plan(ELT, g.M, g.K, g.L, ncu);
  g.nct = p.nct;
  g.nrt = p.nrt;
  g.P = p.P;
  const bool fits = part_bytes(p) <= part_cap;
  g.S = fits ? p.S : 1;
  g.W = fits ? p.W : p.P;
  switch (p.nb) {
    case 2: return run<ELT, TRANS, 2>(g, s);
    case 4: return run<ELT, TRANS, 4>(g, s);
    case 6: return run<ELT, TRANS, 6>(g, s);
    case 8: return run<ELT, TRANS, 8>(g, s);
    case 10: return run<ELT, TRANS, 10>(g, s);
    case 12: return run<ELT, TRANS, 12>(g, s);
    case 14: return run<ELT, TRANS, 14>(g, s);
    case 16: return run<ELT, TRANS, 16>(g, s);
    case 18: return run<ELT, TRANS, 18>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lowp
}  // namespace rsvd
