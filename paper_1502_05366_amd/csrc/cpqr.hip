// k steps of the column-pivoted QR (Sec. 2.3) of the short, wide B = Q^T A
// (l x n), which selects the skeleton columns of the ID computed from B
// (Sec. 3.5, last part) and, applied to C^T, the rows of the CUR (Sec. 2.5,
// Sec. 3.6).  Then T = S11^{-1} S12 (Sec. 2.4) by back substitution.
//
// One launch of G <= (compute units) workgroups that wait for each other with
// bounded spins (below); workgroup g keeps columns
// [g*cs, (g+1)*cs) of B for the whole factorization, in registers
// (cpqr_reg_kernel) or, where they do not fit, in LDS (cpqr_kernel).  Step s:
//   1. each workgroup finds its unchosen column with the largest residual
//      norm ||B(s:, j)|| (FP64, lowest column index on ties) and publishes
//      the norm, the index and rows s.. of that column;
//   2. grid barrier;
//   3. every workgroup reads the G candidates, picks the global pivot the
//      same way, builds the Householder reflector H = I - beta v v^T of the
//      pivot column (v = x + sign(x_0)||x|| e_1, beta = 2 / v^T v) from the
//      published values, and applies it to rows s.. of its unchosen columns;
//   4. residual norms are recomputed exactly over rows s+1.. .
// Chosen columns keep their place; the remaining columns are listed in
// ascending index order.  The rank tolerance is max(r, c) * eps * ||B||_F.
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace rsvd {
namespace {

constexpr int CQ_NT = 512;
constexpr double DEPS = 2.220446049250313e-16;

struct CpqrArgs {
  const void* Bt; int64_t ldb;     // column j of B at Bt + j * ldb
  int r; int64_t c; int k;
  int G; int64_t cs; int rp;
  double* slots;                   // [2][G][slot_len]: norm^2, index, ||.||_F^2 part, column
  int64_t slot_len;
  uint32_t* tags;                  // [2][G] (FLAG_STRIDE apart) step + 1 of the last post
  uint32_t* abort_flag;            // set when a wait exceeds its spin cap
  uint32_t wait_bias;              // 0; 1 only in the forced give-up test mode
  uint32_t spin_cap;
  int64_t* J;                      // [c]
  double* S11t;                    // column t = top k rows of pivot column t (ld = lds)
  double* S12t;                    // column rho = top k rows of residual column rho
  int64_t lds;
  double* pivn;                    // [k] pivot norms
  int32_t* info;                   // [2]
};

// Exchange between the workgroups of one step (columns in LDS): every workgroup posts its
// candidate into its own slot and then raises the slot's tag to step + 1
// (release); readers wait for each tag (acquire) and read the slot with
// agent-scope loads.  No counter is shared, so no atomic is contended.  A wait
// longer than its spin cap raises the abort flag and INFO_BARRIER; all later
// waits then return at once, so the kernel always runs to its end (its
// results are then flagged invalid).  In the forced give-up test mode the
// host sets wait_bias = 1, so every wait is for a value that no workgroup
// posts, and a small spin cap.
constexpr uint32_t SPIN_CAP = 1u << 22;
constexpr uint32_t SPIN_CAP_TEST = 1u << 10;

// Called by every thread of the workgroup after the slot data has been stored
// with agent-scope stores: each wave waits for its stores, then thread 0
// raises the tag.
__device__ __forceinline__ void post_tag(uint32_t* tag, uint32_t value) {
  stores_done();
  __syncthreads();
  if (threadIdx.x == 0) st_agent_u32(tag, value);
}

// Relaxed polling; the slot data is then read with agent-scope loads.
__device__ __forceinline__ void wait_tag(const uint32_t* tag, uint32_t value, uint32_t* abort_flag,
                                         uint32_t spin_cap, int32_t* info) {
  uint32_t spins = 0;
  while (ld_agent_u32(tag) != value) {
    if ((++spins & 63) == 0) {
      if (ld_agent_u32(abort_flag) != 0) break;
      if (spins > spin_cap) {
        st_agent_u32(abort_flag, 1u);
        info_or(info, INFO_BARRIER);
        break;
      }
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// argmax of (val, idx): larger val wins, lower idx on equal val
__device__ __forceinline__ bool better(double v1, int64_t i1, double v2, int64_t i2) {
  return v1 > v2 || (v1 == v2 && i1 < i2);
}

// Selection key of a squared residual norm: NaN (from non-finite entries of
// B) maps to -0.5, below every finite norm and above the empty-candidate
// value -1, so such columns are still chosen, last and lowest index first:
// the k pivots are always k distinct columns and the index bookkeeping
// below stays a permutation.  The step then reports INFO_NONFINITE.
__device__ __forceinline__ double sel_key(double s2) { return s2 == s2 ? s2 : -0.5; }

constexpr int CQ_NW = CQ_NT / 64;
// A column is handled by one row of 16 lanes, RPL rows per lane (rows
// rl + 16 e, e < RPL); the plan takes the smallest instantiated RPL with
// 16 RPL >= r and a column stride rp >= 16 RPL, so every row a lane touches is
// in its column (rows r .. 16 RPL - 1 hold zeros) and no access needs a
// per-lane test.
constexpr int CQ_RPLS[] = {2, 4, 8, 12, 13, 14, 16};

// sum over the 16 lanes of a row, returned in each of them
__device__ __forceinline__ double row16_sum(double x) {
  x += dpp_d<0xB1>(x);
  x += dpp_d<0x4E>(x);
  x += dpp_d<0x141>(x);
  x += dpp_d<0x140>(x);
  return x;
}

template <typename TB, int RPL>
__global__ __launch_bounds__(CQ_NT) void cpqr_kernel(CpqrArgs a) {
  extern __shared__ double smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cg = lane >> 4, rl = lane & 15;
  const int g = blockIdx.x;
  const int64_t j0 = (int64_t)g * a.cs;
  int64_t ncols = a.c - j0;
  if (ncols > a.cs) ncols = a.cs;
  if (ncols < 0) ncols = 0;
  const int r = a.r, rp = a.rp;

  double* slab = smem;                         // [cs][rp]
  double* nrm = slab + a.cs * rp;              // [cs]
  double* v = nrm + a.cs;                      // [rp]
  int* chosen_at = (int*)(v + rp);             // [cs] step at which chosen, -1 if not
  int64_t* piv = (int64_t*)(chosen_at + a.cs + (a.cs & 1));  // [k]
  __shared__ double redv[2][CQ_NW];
  __shared__ int64_t redi[2][CQ_NW];
  __shared__ int redg[2][CQ_NW];
  __shared__ double redf[CQ_NW];
  __shared__ double sh_beta, sh_alpha, sh_gv;
  __shared__ int64_t sh_gi;
  __shared__ int sh_gg;

  const TB* Bt = static_cast<const TB*>(a.Bt);
  for (int64_t e = tid; e < ncols * rp; e += CQ_NT) {
    const int64_t jj = e / rp;
    const int i = (int)(e - jj * rp);
    slab[e] = (i < r) ? (double)Bt[(j0 + jj) * a.ldb + i] : 0.0;
  }
  // the reflector's rows >= r stay zero (the steps write rows s .. r-1)
  for (int i = tid; i < rp; i += CQ_NT) v[i] = 0.0;
  __syncthreads();
  // initial norms, the workgroup's share of ||B||_F^2 and each lane's best
  // column (largest norm, lowest index on ties).  A column is handled by one
  // row of 16 lanes (rows rl + 16 e of the column), four columns per wave.
  double fpart = 0.0;
  double bv = -1.0;
  int64_t bi = INT64_MAX;
  for (int64_t jb = 0; jb < ncols; jb += CQ_NW * 4) {
    const int64_t jj = jb + wave * 4 + cg;
    const bool act = jj < ncols;
    const double* col = slab + (act ? jj : 0) * rp;
    double s2 = 0.0;
#pragma unroll
    for (int e = 0; e < RPL; ++e) {
      const double x = col[rl + 16 * e];
      s2 = fma(x, x, s2);
    }
    s2 = row16_sum(s2);
    if (act) {
      if (rl == 0) {
        nrm[jj] = s2; chosen_at[jj] = -1; fpart += s2;
        if (!(s2 <= 1.7976931348623157e308)) info_or(a.info, INFO_NONFINITE);   // NaN or Inf in B
      }
      if (better(sel_key(s2), j0 + jj, bv, bi)) { bv = sel_key(s2); bi = j0 + jj; }
    }
  }
  fpart = wave_allsum(fpart);
  if (lane == 0) redf[wave] = fpart;
  double tol = 0.0;
  int frank = a.k;

  for (int s = 0; s < a.k; ++s) {
    const int par = s & 1;
    // 1. the workgroup's candidate (lanes' bests, fixed order), posted
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      const double ov = __shfl_xor(bv, off, 64);
      const int64_t oi = __shfl_xor(bi, off, 64);
      if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if (lane == 0) { redv[par][wave] = bv; redi[par][wave] = bi; }
    __syncthreads();
    double* myslot = a.slots + ((int64_t)par * a.G + g) * a.slot_len;
    double cv = redv[par][0];
    int64_t ci = redi[par][0];
    for (int w = 1; w < CQ_NW; ++w)
      if (better(redv[par][w], redi[par][w], cv, ci)) { cv = redv[par][w]; ci = redi[par][w]; }
    if (tid == 0) {
      double f = 0.0;
      if (s == 0)
        for (int w = 0; w < CQ_NW; ++w) f += redf[w];
      st_agent(myslot + 0, cv);
      st_agent(myslot + 1, (double)(ci == INT64_MAX ? -1 : ci));
      st_agent(myslot + 2, f);
    }
    if (ci != INT64_MAX) {
      const int64_t jj = ci - j0;
      for (int i = s + tid; i < r; i += CQ_NT) st_agent(myslot + 3 + i, slab[jj * rp + i]);
    }
    post_tag(a.tags + (par * a.G + g) * FLAG_STRIDE, (uint32_t)s + 1u);
    // 2./3. thread w waits for workgroup w's tag and reads its candidate; the
    // global pivot is the best candidate (lowest index on ties)
    double gv = -1.0;
    int64_t gi = INT64_MAX;
    int gg = 0;
    double fro_part = 0.0;
    for (int w = tid; w < a.G; w += CQ_NT) {
      wait_tag(a.tags + (par * a.G + w) * FLAG_STRIDE, (uint32_t)s + 1u + a.wait_bias,
               a.abort_flag, a.spin_cap, a.info);
      const double* sl = a.slots + ((int64_t)par * a.G + w) * a.slot_len;
      const double vv = ld_agent(sl + 0);
      const double iv = ld_agent(sl + 1);
      if (s == 0) fro_part += ld_agent(sl + 2);
      if (iv >= 0.0) {
        const int64_t ii = (int64_t)iv;
        if (better(vv, ii, gv, gi)) { gv = vv; gi = ii; gg = w; }
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double ov = __shfl_xor(gv, off, 64);
      const int64_t oi = __shfl_xor(gi, off, 64);
      const int og = __shfl_xor(gg, off, 64);
      if (better(ov, oi, gv, gi)) { gv = ov; gi = oi; gg = og; }
    }
    if (s == 0) fro_part = wave_allsum(fro_part);
    const int rb = par ^ 1;                // the other half of the reduction buffers
    if (lane == 0) { redv[rb][wave] = gv; redi[rb][wave] = gi; redg[rb][wave] = gg; }
    if (s == 0 && lane == 0) redf[wave] = fro_part;
    __syncthreads();
    gv = redv[rb][0]; gi = redi[rb][0]; gg = redg[rb][0];
    for (int w = 1; w < CQ_NW; ++w)
      if (better(redv[rb][w], redi[rb][w], gv, gi)) { gv = redv[rb][w]; gi = redi[rb][w]; gg = redg[rb][w]; }
    if (s == 0) {
      double fro2 = 0.0;
      for (int w = 0; w < CQ_NW; ++w) fro2 += redf[w];
      tol = (double)(r > a.c ? r : a.c) * DEPS * sqrt(fro2);
    }
    // without a valid candidate (possible only after an aborted wait, whose
    // results are flagged invalid) column 0 stands in, so that every index
    // stays in range
    if (gi < 0 || gi >= a.c) { gi = 0; gg = 0; }
    // the pivot's posted norm^2 is ||x||^2 of its rows s..r-1; a non-finite
    // pivot (NaN key -0.5, or Inf) is taken with a zero reflector
    const bool pfin = gv >= 0.0 && gv <= 1.7976931348623157e308;
    if (!pfin && g == 0 && tid == 0) info_or(a.info, INFO_NONFINITE);
    const double pnorm = pfin ? sqrt(gv) : 0.0;
    if (frank == a.k && pnorm <= tol) frank = s;
    const double* psl = a.slots + ((int64_t)par * a.G + gg) * a.slot_len;
    for (int i = s + tid; i < r; i += CQ_NT) v[i] = ld_agent(psl + 3 + i);
    __syncthreads();
    if (tid == 0) {
      const double normx = pnorm;
      const double x0 = v[s];
      if (normx == 0.0) {
        sh_beta = 0.0;
        sh_alpha = 0.0;
      } else {
        const double sg = x0 >= 0.0 ? 1.0 : -1.0;
        v[s] = x0 + sg * normx;
        sh_alpha = -sg * normx;
        // v^T v = 2 ||x|| (||x|| + |x_0|)
        sh_beta = 1.0 / (normx * (normx + fabs(x0)));
      }
      if (g == 0) {
        a.J[s] = gi;
        a.pivn[s] = pnorm;
      }
      piv[s] = gi;
    }
    __syncthreads();
    const double beta = sh_beta, alpha = sh_alpha;
    // apply H to the unchosen owned columns, recompute their norms over rows
    // s+1.. and track each lane's best column.  Rows above s enter as exact
    // zeros through v (selected per lane), rows r .. 16 RPL - 1 are zero in
    // the slab and in v; a column's stores run under one test.
    bv = -1.0;
    bi = INT64_MAX;
    double vr[RPL];
#pragma unroll
    for (int e = 0; e < RPL; ++e) {
      const int i = rl + 16 * e;
      const double vv = v[i];
      vr[e] = i >= s ? vv : 0.0;
    }
    for (int64_t jb = 0; jb < ncols; jb += CQ_NW * 4) {
      const int64_t jj = jb + wave * 4 + cg;
      const bool inr = jj < ncols;
      const int64_t jc = inr ? jj : 0;       // a column of the slab for the loads
      const bool act = inr && chosen_at[jc] < 0;
      const bool is_piv = act && (j0 + jj == gi);
      double* col = slab + jc * rp;
      double x[RPL];
      double dp[4] = {0.0, 0.0, 0.0, 0.0};   // four partial sums: short FMA chains
#pragma unroll
      for (int e = 0; e < RPL; ++e) {
        x[e] = col[rl + 16 * e];
        dp[e & 3] = fma(vr[e], x[e], dp[e & 3]);
      }
      const double wdot = beta * row16_sum((dp[0] + dp[1]) + (dp[2] + dp[3]));
      const bool upd = act && !is_piv && beta != 0.0;
#pragma unroll
      for (int e = 0; e < RPL; ++e) {
        const int i = rl + 16 * e;
        const double y = fma(-wdot, vr[e], x[e]);
        x[e] = (upd && i >= s) ? y : x[e];
      }
      if (upd) {
#pragma unroll
        for (int e = 0; e < RPL; ++e) col[rl + 16 * e] = x[e];
      }
      if (is_piv) {
#pragma unroll
        for (int e = 0; e < RPL; ++e) {
          const int i = rl + 16 * e;
          col[i] = (i == s) ? alpha : (i > s ? 0.0 : x[e]);
        }
        if (rl == 0) { chosen_at[jj] = s; nrm[jj] = 0.0; }
      }
      double sp[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < RPL; ++e) {
        const int i = rl + 16 * e;
        const double f = fma(x[e], x[e], sp[e & 3]);
        sp[e & 3] = i > s ? f : sp[e & 3];
      }
      const double s2 = row16_sum((sp[0] + sp[1]) + (sp[2] + sp[3]));
      if (act && !is_piv) {
        if (rl == 0) nrm[jj] = s2;
        if (better(sel_key(s2), j0 + jj, bv, bi)) { bv = sel_key(s2); bi = j0 + jj; }
      }
    }
  }
  __syncthreads();
  if (g == 0 && tid == 0 && frank < a.k) {
    info_or(a.info, INFO_RANK);
    a.info[1] = frank;
  }
  // After an aborted wait the workgroups may disagree on the pivots, so the
  // positions below would not be a permutation: then J lists the columns in
  // order and the factors are not written (the call reports INFO_BARRIER).
  if (ld_agent_u32(a.abort_flag) != 0) {
    for (int64_t jj = tid; jj < ncols; jj += CQ_NT) a.J[j0 + jj] = j0 + jj;
    return;
  }
  // outputs: top k rows of every owned column
  for (int64_t jj = wave; jj < ncols; jj += CQ_NW) {
    const int64_t j = j0 + jj;
    const int t = chosen_at[jj];
    double* dst;
    if (t >= 0) {
      dst = a.S11t + (int64_t)t * a.lds;
    } else {
      int64_t before = 0;
      for (int q = lane; q < a.k; q += 64) before += (piv[q] < j) ? 1 : 0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
      const int64_t rho = j - before;
      dst = a.S12t + rho * a.lds;
      if (lane == 0) a.J[a.k + rho] = j;
    }
    for (int i = lane; i < a.k; i += 64) dst[i] = (i < r) ? slab[jj * rp + i] : 0.0;
  }
}

// ---- columns in registers ---------------------------------------------------
//
// Up to 96 columns per workgroup (c <= 24576 on 256 compute units) the columns
// stay in registers: lane rl of a row of 16 lanes holds rows rl + 16 e of its
// NSET columns (column 32 q + 4 wave + group of the workgroup), so a step reads
// no column from LDS and writes none.  What bounds a step is the exchange, not
// the arithmetic (~0.5 us): three trips to memory that all compute units see.
// The slot protocol of the kernel above takes five (data, tag, poll, candidate,
// column), so here every 64-bit word carries 32 bits of data and the step
// number and is its own flag: a candidate is two words, the column 32 RPL, a
// writer waits for nothing, and one wave reads all candidates (contiguous, two
// words per lane), picks the pivot, reads its column and forms the reflector,
// while the others wait at a barrier (two barriers per step instead of five).
// The arithmetic and its order are those of the kernel above.  Per step, LDS
// kernel -> this one: 6.7 -> 4.5 us (210 x 1024), 7.1 -> 4.8 (210 x 4096), 8.7 ->
// 6.0 (210 x 10000, two columns per lane group), 9.6 -> 6.6 (200 x 20000, three).
// Candidates lie 128 bytes apart: eight to a line cost 0.4 - 0.9 us more, the
// writers of one line waiting for each other.
//
// A word of step s is overwritten at step s + 2 (two halves), which its owner
// reaches only after the candidates of step s + 1 of all workgroups, and those
// follow their reads of step s.  The words are cleared before the launch.
constexpr int CQ_MAXSET = 3;                 // 32 columns each
constexpr int CQ_NOCAND = 0xFFFF;
constexpr int CQ_LINE = 16;                  // words between candidates: 128 bytes

__device__ __forceinline__ uint64_t ld_agent_u64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent_u64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a double as two words with a tag in their low halves
__device__ __forceinline__ void st_tagged(uint64_t* p, double x, uint32_t tag_hi,
                                          uint32_t tag_lo) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  st_agent_u64(p, (b & 0xFFFFFFFF00000000ull) | tag_hi);
  st_agent_u64(p + 1, (b << 32) | tag_lo);
}
__device__ __forceinline__ double tagged_value(uint64_t hi, uint64_t lo) {
  return __longlong_as_double((long long)((hi & 0xFFFFFFFF00000000ull) | (lo >> 32)));
}

// (val, key) of the better candidate among the lanes that a DPP or swap
// exchange brings together; keys rise with the column index
__device__ __forceinline__ void keep_better(double& v, uint32_t& k, double ov, uint32_t ok) {
  const bool b = ov > v || (ov == v && ok < k);
  v = b ? ov : v;
  k = b ? ok : k;
}
template <int CTRL> __device__ __forceinline__ void best_dpp(double& v, uint32_t& k) {
  const double ov = dpp_d<CTRL>(v);
  const uint32_t ok = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, CTRL, 0xF, 0xF, false);
  keep_better(v, k, ov, ok);
}
// the best over the lanes i, i ^ 16 (H = 16) or i, i ^ 32 (H = 32)
template <int H> __device__ __forceinline__ void best_swap(double& v, uint32_t& k) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  auto sw = [](uint32_t x) {
    if constexpr (H == 16) return __builtin_amdgcn_permlane16_swap(x, x, false, false);
    else return __builtin_amdgcn_permlane32_swap(x, x, false, false);
  };
  const auto lo = sw((uint32_t)b), hi = sw((uint32_t)(b >> 32)), kk = sw(k);
  const double v0 = __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0]));
  const double v1 = __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
  v = v0;
  k = kk[0];
  keep_better(v, k, v1, kk[1]);
}

template <int RPL, int NSET>
__global__ __launch_bounds__(CQ_NT) void cpqr_reg_kernel(CpqrArgs a, int b_f32) {
  __shared__ double v[16 * RPL];
  __shared__ double redf[CQ_NW];
  __shared__ double redv[CQ_NW];
  __shared__ uint32_t redk[CQ_NW];
  __shared__ int32_t piv[256];
  __shared__ double sh_beta, sh_alpha;
  __shared__ int32_t sh_gi;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cg = lane >> 4, rl = lane & 15;
  const int g = blockIdx.x, G = a.G;
  const int cs = (int)a.cs, r = a.r;
  const int64_t j0 = (int64_t)g * cs;
  const int ncols = (int)max((int64_t)0, min(a.c - j0, (int64_t)cs));
  uint64_t* const cand = reinterpret_cast<uint64_t*>(a.slots);       // [2][G] CQ_LINE apart
  uint64_t* const fro = cand + (int64_t)CQ_LINE * 2 * G;                       // [G][2]
  uint64_t* const colw = fro + (int64_t)2 * G;                       // [2][G][16 RPL][2]

  double x[NSET][RPL];
  int chosen_at[NSET];                     // step at which chosen, -1 if not, -2 no column
  double bv = -1.0;
  uint32_t bk = CQ_NOCAND;
  double fpart = 0.0;
#pragma unroll
  for (int q = 0; q < NSET; ++q) {
    const int jj = 32 * q + 4 * wave + cg;
    const bool in = jj < ncols;
    const int64_t base = (j0 + (in ? jj : 0)) * a.ldb;
    chosen_at[q] = in ? -1 : -2;
#pragma unroll
    for (int e = 0; e < RPL; ++e) {
      const int i = rl + 16 * e;
      const int64_t off = (in && i < r) ? base + i : 0;
      const double y = b_f32 ? (double)static_cast<const float*>(a.Bt)[off]
                             : static_cast<const double*>(a.Bt)[off];
      x[q][e] = (in && i < r) ? y : 0.0;
    }
  }
#pragma unroll
  for (int q = 0; q < NSET; ++q) {
    double s2 = 0.0;
#pragma unroll
    for (int e = 0; e < RPL; ++e) s2 = fma(x[q][e], x[q][e], s2);
    s2 = row16_sum(s2);
    if (chosen_at[q] == -1) {
      if (rl == 0) {
        fpart += s2;
        if (!(s2 <= 1.7976931348623157e308)) info_or(a.info, INFO_NONFINITE);   // NaN or Inf in B
      }
      keep_better(bv, bk, sel_key(s2), (uint32_t)(32 * q + 4 * wave + cg));
    }
  }
  fpart = wave_allsum(fpart);
  if (lane == 0) redf[wave] = fpart;
  double tol = 0.0;                        // (tol, frank and dead: wave 0)
  int frank = a.k;
  bool dead = false;

  for (int s = 0; s < a.k; ++s) {
    const int par = s & 1;
    const uint32_t tag = (uint32_t)s + 1u;
    // 1. the workgroup's candidate: the owning wave posts it and its column
    best_swap<16>(bv, bk);
    best_swap<32>(bv, bk);
    if (lane == 0) { redv[wave] = bv; redk[wave] = bk; }
    __syncthreads();
    {
      double cv = redv[lane & 7];
      uint32_t ck = redk[lane & 7];
      best_dpp<0xB1>(cv, ck);
      best_dpp<0x4E>(cv, ck);
      best_dpp<0x141>(cv, ck);
      const uint32_t loc = (uint32_t)__builtin_amdgcn_readfirstlane((int)ck);
      const int owner = loc == CQ_NOCAND ? 0 : (int)(loc >> 2) & 7;
      if (wave == owner) {
        if (lane == 0) st_tagged(cand + (int64_t)CQ_LINE * (par * G + g), cv, (loc << 16) | tag, tag);
        if (loc != CQ_NOCAND) {
          uint64_t* cw = colw + ((int64_t)par * G + g) * (32 * RPL);
          if (cg == (int)(loc & 3)) {
#pragma unroll
            for (int q = 0; q < NSET; ++q)
              if (q == (int)(loc >> 5)) {
#pragma unroll
                for (int e = 0; e < RPL; ++e)
                  if (16 * e + 15 >= s) st_tagged(cw + 2 * (rl + 16 * e), x[q][e], tag, tag);
              }
          }
        }
      }
      if (s == 0 && tid == 0) {
        double f = 0.0;
        for (int w = 0; w < CQ_NW; ++w) f += redf[w];
        st_tagged(fro + 2 * g, f, tag, tag);
      }
    }
    // 2. wave 0: all candidates, the pivot (largest norm, lowest index on
    // ties), its column and the reflector
    if (wave == 0) {
      const uint32_t want = tag + a.wait_bias;
      auto waits = [&](auto&& poll) {
        for (uint32_t spins = 1; !poll() && !dead; ++spins) {
          if ((spins & 63) == 0) {
            if (ld_agent_u32(a.abort_flag) != 0) dead = true;
            else if (spins > a.spin_cap) {
              if (lane == 0) {
                st_agent_u32(a.abort_flag, 1u);
                info_or(a.info, INFO_BARRIER);
              }
              dead = true;
            }
          }
          __builtin_amdgcn_s_sleep(1);
        }
      };
      constexpr int NQ = 4;                // G <= 256
      // (a lane past the last workgroup holds an empty candidate)
      uint64_t c0[NQ], c1[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const bool in = 64 * q + lane < G;
        c0[q] = in ? 0u : ((uint32_t)CQ_NOCAND << 16) | want;
        c1[q] = in ? 0u : want;
      }
      const uint64_t* cp = cand + (int64_t)CQ_LINE * par * G;
      waits([&]() {
        bool ok = true;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (((uint32_t)c0[q] & 0xFFFFu) != want || (uint32_t)c1[q] != want) {
            const int w = 64 * q + lane;
            c0[q] = ld_agent_u64(cp + CQ_LINE * w);
            c1[q] = ld_agent_u64(cp + CQ_LINE * w + 1);
          }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          ok = ok && ((uint32_t)c0[q] & 0xFFFFu) == want && (uint32_t)c1[q] == want;
        return __all(ok) != 0;
      });
      double gv = -1.0;
      uint32_t gk = 0xFFFFFFFFu;           // workgroup << 16 | its column
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const uint32_t loc = (uint32_t)c0[q] >> 16;
        const bool ok = ((uint32_t)c0[q] & 0xFFFFu) == want && (uint32_t)c1[q] == want &&
                        loc < (uint32_t)cs;
        if (ok)
          keep_better(gv, gk, tagged_value(c0[q], c1[q]), ((uint32_t)(64 * q + lane) << 16) | loc);
      }
      best_dpp<0xB1>(gv, gk);
      best_dpp<0x4E>(gv, gk);
      best_dpp<0x141>(gv, gk);
      best_dpp<0x140>(gv, gk);
      best_swap<16>(gv, gk);
      best_swap<32>(gv, gk);
      gk = (uint32_t)__builtin_amdgcn_readfirstlane((int)gk);
      gv = readlane_d(gv, 0);
      // without a valid candidate (possible only after an aborted wait, whose
      // results are flagged invalid) column 0 stands in, so that every index
      // stays in range
      int gg = (int)(gk >> 16);
      int64_t gi = (int64_t)gg * cs + (gk & 0xFFFFu);
      if (gk == 0xFFFFFFFFu || gi >= a.c) { gi = 0; gg = 0; }
      constexpr int NR = (16 * RPL + 63) / 64;
      uint64_t h[NR], o[NR];
      const uint64_t* cw = colw + ((int64_t)par * G + gg) * (32 * RPL);
      // (rows not posted: zero)
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = 64 * q + lane;
        h[q] = o[q] = ((i | 15) >= s && i < 16 * RPL) ? 0u : want;
      }
      waits([&]() {
        bool ok = true;
#pragma unroll
        for (int q = 0; q < NR; ++q)
          if ((uint32_t)h[q] != want || (uint32_t)o[q] != want) {
            h[q] = ld_agent_u64(cw + 2 * (64 * q + lane));
            o[q] = ld_agent_u64(cw + 2 * (64 * q + lane) + 1);
          }
#pragma unroll
        for (int q = 0; q < NR; ++q) ok = ok && (uint32_t)h[q] == want && (uint32_t)o[q] == want;
        return __all(ok) != 0;
      });
      if (s == 0) {
        // the workgroups' shares of ||B||_F^2
        double fro2 = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (64 * q < G) {
            const bool in = 64 * q + lane < G;
            const int w = min(64 * q + lane, G - 1);
            uint64_t f0 = 0, f1 = 0;
            waits([&]() {
              f0 = ld_agent_u64(fro + 2 * w);
              f1 = ld_agent_u64(fro + 2 * w + 1);
              return __all((uint32_t)f0 == want && (uint32_t)f1 == want) != 0;
            });
            fro2 += wave_allsum(in ? tagged_value(f0, f1) : 0.0);
          }
        tol = (double)(r > a.c ? r : a.c) * DEPS * sqrt(fro2);
      }
      // the pivot's posted norm^2 is ||x||^2 of its rows s..r-1; a non-finite
      // pivot (NaN key -0.5, or Inf) is taken with a zero reflector
      const bool pfin = gv >= 0.0 && gv <= 1.7976931348623157e308;
      if (!pfin && g == 0 && lane == 0) info_or(a.info, INFO_NONFINITE);
      const double normx = pfin ? sqrt(gv) : 0.0;
      if (frank == a.k && normx <= tol) frank = s;
      double x0 = 0.0;
#pragma unroll
      for (int q = 0; q < NR; ++q)
        if (q == s >> 6) x0 = readlane_d(tagged_value(h[q], o[q]), s & 63);
      double beta = 0.0, alpha = 0.0, v0 = x0;
      if (normx != 0.0) {
        const double sg = x0 >= 0.0 ? 1.0 : -1.0;
        v0 = x0 + sg * normx;
        alpha = -sg * normx;
        // v^T v = 2 ||x|| (||x|| + |x_0|)
        beta = 1.0 / (normx * (normx + fabs(x0)));
      }
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = 64 * q + lane;
        const double y = tagged_value(h[q], o[q]);
        if (i < 16 * RPL) v[i] = (i < s || i >= r) ? 0.0 : (i == s ? v0 : y);
      }
      if (lane == 0) {
        sh_beta = beta;
        sh_alpha = alpha;
        sh_gi = (int32_t)gi;
        piv[s] = (int32_t)gi;
        if (g == 0) {
          a.J[s] = gi;
          a.pivn[s] = normx;
        }
      }
    }
    __syncthreads();
    // 3. the reflector on the unchosen columns, their norms over rows s+1..
    // and each lane's best column (rows outside s .. r-1 of v are zero)
    const double beta = sh_beta, alpha = sh_alpha;
    const int gl = (int)min(max((int64_t)sh_gi - j0, (int64_t)-1), (int64_t)CQ_NOCAND);
    double vr[RPL];
#pragma unroll
    for (int e = 0; e < RPL; ++e) vr[e] = v[rl + 16 * e];
    bv = -1.0;
    bk = CQ_NOCAND;
#pragma unroll
    for (int q = 0; q < NSET; ++q) {
      const int jj = 32 * q + 4 * wave + cg;
      const bool act = chosen_at[q] == -1;
      const bool is_piv = act && jj == gl;
      double dp[4] = {0.0, 0.0, 0.0, 0.0};   // four partial sums: short FMA chains
#pragma unroll
      for (int e = 0; e < RPL; ++e) dp[e & 3] = fma(vr[e], x[q][e], dp[e & 3]);
      const double wdot = beta * row16_sum((dp[0] + dp[1]) + (dp[2] + dp[3]));
      const bool upd = act && !is_piv && beta != 0.0;
#pragma unroll
      for (int e = 0; e < RPL; ++e) {
        const int i = rl + 16 * e;
        const double y = fma(-wdot, vr[e], x[q][e]);
        x[q][e] = (upd && i >= s) ? y : x[q][e];
      }
      if (is_piv) {
#pragma unroll
        for (int e = 0; e < RPL; ++e) {
          const int i = rl + 16 * e;
          x[q][e] = (i == s) ? alpha : (i > s ? 0.0 : x[q][e]);
        }
        chosen_at[q] = s;
      }
      double sp[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < RPL; ++e) {
        const int i = rl + 16 * e;
        const double f = fma(x[q][e], x[q][e], sp[e & 3]);
        sp[e & 3] = i > s ? f : sp[e & 3];
      }
      const double s2 = row16_sum((sp[0] + sp[1]) + (sp[2] + sp[3]));
      if (act && !is_piv) keep_better(bv, bk, sel_key(s2), (uint32_t)jj);
    }
  }
  if (g == 0 && tid == 0 && frank < a.k) {
    info_or(a.info, INFO_RANK);
    a.info[1] = frank;
  }
  // (after an aborted wait: as in the kernel above)
  const bool dead_all = ld_agent_u32(a.abort_flag) != 0;
  // outputs: top k rows of every owned column
#pragma unroll
  for (int q = 0; q < NSET; ++q) {
    const int64_t j = j0 + 32 * q + 4 * wave + cg;
    const int t = chosen_at[q];
    if (t == -2) continue;
    if (dead_all) {
      if (rl == 0) a.J[j] = j;
      continue;
    }
    int before = 0;
    for (int i = rl; i < a.k; i += 16) before += (piv[i] < j) ? 1 : 0;
    before += __builtin_amdgcn_update_dpp(0, before, 0xB1, 0xF, 0xF, false);
    before += __builtin_amdgcn_update_dpp(0, before, 0x4E, 0xF, 0xF, false);
    before += __builtin_amdgcn_update_dpp(0, before, 0x141, 0xF, 0xF, false);
    before += __builtin_amdgcn_update_dpp(0, before, 0x140, 0xF, 0xF, false);
    double* dst = t >= 0 ? a.S11t + (int64_t)t * a.lds : a.S12t + (j - before) * a.lds;
    if (t < 0 && rl == 0) a.J[a.k + (j - before)] = j;
#pragma unroll
    for (int e = 0; e < RPL; ++e)
      if (rl + 16 * e < a.k) dst[rl + 16 * e] = x[q][e];
  }
}

// Upper-triangular solve X = S^{-1} B with many right-hand sides (k <= 256),
// by block back substitution over 16 x 16 blocks:
//   X_c = M_c (B_c - sum_{b>c} S_cb X_b),  c = nb-1 .. 0,
// where M_c is the solve with the diagonal block S_cc under the rule that a
// zero pivot gives a zero unknown (x_i = 0 when S_ii = 0); that rule is
// linear in the right-hand side, so M_c is the matrix of 16 such solves with
// the unit vectors, formed in LDS by every workgroup.  One wave takes 16
// right-hand sides; as in the orth triangular solve, the 16 x 16 product
// in accumulator layout (lane (j, g) holds rows 4v + g of column j) is the
// B operand of the later products, so each X_b stays in registers.  Strided
// access: S(i, j) = S[i*s_r + j*s_c], right-hand side `col` element i =
// Bm[col*b_c + i*b_r], X(i, col) = X[i*x_r + col*x_c].
constexpr int BSB_MAXNB = 16;

template <int NB>
__global__ __launch_bounds__(256) void backsub_kernel(const double* __restrict__ S, int64_t s_r,
                                                      int64_t s_c, const double* __restrict__ Bm,
                                                      int64_t b_r, int64_t b_c, int k,
                                                      int64_t nrhs, double* __restrict__ X,
                                                      int64_t x_r, int64_t x_c) {
  __shared__ double Sd[BSB_MAXNB][16 * 17];   // diagonal blocks of S
  __shared__ double Md[BSB_MAXNB][16 * 17];   // their solve matrices M_c
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int nb = (int)cdiv(k, 16);
  for (int e = tid; e < nb * 256; e += 256) {
    const int c = e >> 8, i = (e >> 4) & 15, j = e & 15;
    const int gi = c * 16 + i, gj = c * 16 + j;
    Sd[c][i * 17 + j] = (gi < k && gj < k && i <= j) ? S[gi * s_r + gj * s_c] : 0.0;
  }
  __syncthreads();
  if (tid < nb * 16) {
    // column j of M_c: back substitution with the unit vector e_j
    const int c = tid >> 4, j = tid & 15;
    const double* sd = Sd[c];
    double x[16];
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      double t = (i == j) ? 1.0 : 0.0;
#pragma unroll
      for (int q = i + 1; q < 16; ++q) t -= sd[i * 17 + q] * x[q];
      const double sii = sd[i * 17 + i];
      x[i] = (sii != 0.0) ? t / sii : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) Md[c][i * 17 + j] = x[i];
  }
  __syncthreads();
  const int64_t col0 = ((int64_t)blockIdx.x * 4 + wave) * 16;
  if (col0 >= nrhs) return;
  const int64_t col = col0 + li;
  const bool cok = col < nrhs;
  const double* bc = Bm + (cok ? col : 0) * b_c;
  double* xc = X + (cok ? col : 0) * x_c;
  // The loads of a block step are unconditional, from clamped indices, with
  // a select after them (under a branch each load was waited for at once);
  // blocks past nb contribute zeros (their X blocks start at zero).
  d4 xt[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) xt[c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int c = NB - 1; c >= 0; --c) {
    if (c < nb) {
      d4 acc;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = c * 16 + 4 * v + lk;
        const double bv = bc[min(i, k - 1) * b_r];
        acc[v] = (cok && i < k) ? bv : 0.0;
      }
#pragma unroll
      for (int b = c + 1; b < NB; ++b) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int i = c * 16 + li, j = b * 16 + 4 * kk + lk;
          const double sv = S[min(i, k - 1) * s_r + min(j, k - 1) * s_c];
          const double av = (i < k && j < k) ? -sv : 0.0;   // S_cb[li][k]
          acc = Mfma<double>::mma(av, xt[b][kk], acc);
        }
      }
      d4 out = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        out = Mfma<double>::mma(Md[c][li * 17 + 4 * kk + lk], acc[kk], out);
      xt[c] = out;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = c * 16 + 4 * v + lk;
        if (cok && i < k) xc[i * x_r] = out[v];
      }
    }
  }
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

}  // namespace

size_t cpqr_lds_bytes(int64_t cs, int rp, int k) {
  return (size_t)(cs * rp + cs + rp) * sizeof(double) + (size_t)(cs + (cs & 1)) * sizeof(int) +
         (size_t)k * sizeof(int64_t);
}

CpqrPlan plan_cpqr(int r, int64_t c, int k, int ncu) {
  CpqrPlan p;
  // rows per lane: the smallest instantiated RPL with 16 RPL >= r
  p.rpl = 0;
  for (int v : CQ_RPLS)
    if (p.rpl == 0 && 16 * v >= r) p.rpl = v;
  // column stride of the LDS slab: rp = 16 (mod 32) doubles puts consecutive
  // columns on opposite halves of the LDS banks; rp >= 16 RPL
  p.rp = (int)(rup(std::max(r, 16 * p.rpl) + 16, 32) - 16);
  int64_t G = cdiv(c, 32);
  if (G > ncu) G = ncu;
  if (G < 1) G = 1;
  p.G = (int)G;
  p.cs = cdiv(c, G);
  p.lds = cpqr_lds_bytes(p.cs, p.rp, k);
  p.slot_len = 3 + p.rp;
  p.ok = p.lds <= 150 * 1024 && r <= 256 && k <= 256 && k <= r && k <= c && p.rpl > 0;
  return p;
}

// The words of the kernel with columns in registers, in 64-bit words: the abort
// flag (the first), candidates, shares of ||B||_F^2, columns.
static int64_t cpqr_reg_words(const CpqrPlan& p) {
  return FLAG_STRIDE / 2 + (int64_t)p.G * (2 * CQ_LINE + 2 + 2 * 32 * p.rpl);
}

size_t cpqr_work_bytes(const CpqrPlan& p) {
  return std::max((size_t)(2 * p.G * p.slot_len) * sizeof(double) +
                      (size_t)(2 * p.G + 1) * FLAG_STRIDE * sizeof(uint32_t),
                  (size_t)cpqr_reg_words(p) * sizeof(uint64_t)) + 64;
}

hipError_t launch_cpqr(bool b_f32, const void* Bt, int64_t ldb, int r, int64_t c, int k,
                       const CpqrPlan& p, void* work, int64_t* J, double* S11t, double* S12t,
                       int64_t lds, double* pivn, int32_t* info, bool giveup_test,
                       hipStream_t s) {
  if (!p.ok) return hipErrorInvalidValue;
  CpqrArgs a;
  a.Bt = Bt; a.ldb = ldb; a.r = r; a.c = c; a.k = k;
  a.G = p.G; a.cs = p.cs; a.rp = p.rp;
  double* w = static_cast<double*>(work);
  a.slots = w;
  a.slot_len = p.slot_len;
  a.tags = reinterpret_cast<uint32_t*>(w + 2 * p.G * p.slot_len);
  a.abort_flag = a.tags + 2 * p.G * FLAG_STRIDE;
  a.J = J; a.S11t = S11t; a.S12t = S12t; a.lds = lds; a.pivn = pivn; a.info = info;
  a.wait_bias = giveup_test ? 1u : 0u;
  a.spin_cap = giveup_test ? SPIN_CAP_TEST : SPIN_CAP;
  const void* fn = nullptr;
  const int nset = (int)cdiv(p.cs, 32);
  // Three column sets of 16 rows per lane fill the 256 registers of a wave;
  // wider B stays in LDS.
  if (nset <= CQ_MAXSET && p.G <= 256) {
    a.abort_flag = static_cast<uint32_t*>(work);
    a.slots = w + FLAG_STRIDE / 2;
    hipError_t e = launch_fill_u32(a.abort_flag, 0u, 2 * cpqr_reg_words(p), s);
    if (e != hipSuccess) return e;
    int f = b_f32 ? 1 : 0;
    void* args[] = {&a, &f};
#define RSVD_CQ1(V, N) \
  if (p.rpl == V && nset == N) fn = (const void*)cpqr_reg_kernel<V, N>;
#define RSVD_CQ(V) RSVD_CQ1(V, 1) RSVD_CQ1(V, 2) RSVD_CQ1(V, 3)
    RSVD_CQ(2) RSVD_CQ(4) RSVD_CQ(8) RSVD_CQ(12) RSVD_CQ(13) RSVD_CQ(14) RSVD_CQ(16)
#undef RSVD_CQ
#undef RSVD_CQ1
    if (!fn) return hipErrorInvalidValue;
    e = hipLaunchKernel(fn, dim3(p.G), dim3(CQ_NT), args, 0, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  hipError_t e = launch_fill_u32(a.tags, 0u, (2 * p.G + 1) * FLAG_STRIDE, s);
  if (e != hipSuccess) return e;
  void* args[] = {&a};
#define RSVD_CQ(V)                                                                       \
  if (p.rpl == V)                                                                        \
    fn = b_f32 ? (const void*)cpqr_kernel<float, V> : (const void*)cpqr_kernel<double, V>;
  RSVD_CQ(2) RSVD_CQ(4) RSVD_CQ(8) RSVD_CQ(12) RSVD_CQ(13) RSVD_CQ(14) RSVD_CQ(16)
#undef RSVD_CQ
  if (!fn) return hipErrorInvalidValue;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
  if (e != hipSuccess) return e;
  e = hipLaunchKernel(fn, dim3(p.G), dim3(CQ_NT), args, p.lds, s);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t launch_backsub(const double* S, int64_t s_r, int64_t s_c, const double* Bm,
                          int64_t b_r, int64_t b_c, int k, int64_t nrhs, double* X, int64_t x_r,
                          int64_t x_c, hipStream_t s) {
  if (nrhs <= 0 || k <= 0) return hipSuccess;
  if (k > 256) return hipErrorInvalidValue;
  const dim3 grid((unsigned)cdiv(nrhs, 64));
  const int nb = (int)cdiv(k, 16);
#define RSVD_BSB(NBV)                                                                           \
  hipLaunchKernelGGL(backsub_kernel<NBV>, grid, dim3(256), 0, s, S, s_r, s_c, Bm, b_r, b_c, k, \
                     nrhs, X, x_r, x_c)
  if (nb <= 2) RSVD_BSB(2);
  else if (nb <= 4) RSVD_BSB(4);
  else if (nb <= 8) RSVD_BSB(8);
  else if (nb <= 13) RSVD_BSB(13);
  else RSVD_BSB(16);
#undef RSVD_BSB
  return hipGetLastError();
}

}  // namespace rsvd
