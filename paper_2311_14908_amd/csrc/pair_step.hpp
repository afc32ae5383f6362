// pair_step.hpp -- device pieces shared by the solver kernels: DPP wave reductions with
// index tie-breaking, relaxed agent-scope word access for the exchanges, and the
// two-multiplier step (paper, Section III.B) with its gradient update.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "solver_params.hpp"

namespace svmx {

constexpr int IBIG = 0x7fffffff;

__device__ __forceinline__ bool lt_min(double v2, int i2, double v, int i) { return v2 < v || (v2 == v && i2 < i); }
__device__ __forceinline__ bool gt_max(double v2, int i2, double v, int i) { return v2 > v || (v2 == v && i2 < i); }

__device__ __forceinline__ double readlane_d(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, ROW_MASK, 0xf, false);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_mov_d(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned hi = (unsigned)dpp_mov<CTRL, ROW_MASK>((int)(b >> 32));
  const unsigned lo = (unsigned)dpp_mov<CTRL, ROW_MASK>((int)b);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int CTRL>
__device__ __forceinline__ double dpp_full_d(double v) {  // every lane reads its source lane
  const long long b = __double_as_longlong(v);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Wave-wide min (MAX = false) or max (MAX = true) of v, returned to every lane.  DPP row
// operations (xor 1 and 2 inside quads, rotations by 4 and 8 inside rows of 16, then the
// row-15 and row-31 broadcasts) leave the result in lane 63.  Lanes outside a broadcast's row
// mask keep their own value, which min/max leaves unchanged.  Compare and select: the values
// are finite or +-inf, so fmin/fmax's quieting of NaN inputs is not needed (either zero may
// come out of -0 against +0; callers compare with ==, for which they are equal).
template <bool MAX>
__device__ __forceinline__ double wave_extreme(double v) {
#define SVMX_EXT_FULL(CTRL)                           \
  {                                                   \
    const double o = dpp_full_d<CTRL>(v);             \
    v = MAX ? (o > v ? o : v) : (o < v ? o : v);      \
  }
#define SVMX_EXT_MASK(CTRL, RM)                       \
  {                                                   \
    const double o = dpp_mov_d<CTRL, RM>(v);          \
    v = MAX ? (o > v ? o : v) : (o < v ? o : v);      \
  }
  SVMX_EXT_FULL(0xB1)         // quad_perm [1,0,3,2]
  SVMX_EXT_FULL(0x4E)         // quad_perm [2,3,0,1]
  SVMX_EXT_FULL(0x124)        // row_ror:4
  SVMX_EXT_FULL(0x128)        // row_ror:8
  SVMX_EXT_MASK(0x142, 0xA)   // row_bcast:15 -> rows 1, 3
  SVMX_EXT_MASK(0x143, 0xC)   // row_bcast:31 -> rows 2, 3
#undef SVMX_EXT_FULL
#undef SVMX_EXT_MASK
  return readlane_d(v, 63);
}

// Wave-wide min of an int, returned to every lane (same DPP pattern).
__device__ __forceinline__ int wave_min_int(int v) {
  v = min(v, dpp_mov<0xB1, 0xF>(v));
  v = min(v, dpp_mov<0x4E, 0xF>(v));
  v = min(v, dpp_mov<0x124, 0xF>(v));
  v = min(v, dpp_mov<0x128, 0xF>(v));
  v = min(v, dpp_mov<0x142, 0xA>(v));
  v = min(v, dpp_mov<0x143, 0xC>(v));
  return __builtin_amdgcn_readlane(v, 63);
}

// Lane of the winner among the lanes with `hit` (those holding the extreme value): the one with
// the smallest index i; an index reduction runs only when several lanes tie.
__device__ __forceinline__ int tie_lane(bool hit, int i) {
  const unsigned long long tie = (unsigned long long)__ballot(hit);
  if (__popcll(tie) == 1) return __ffsll(tie) - 1;
  const int best = wave_min_int(hit ? i : IBIG);
  return __ffsll((unsigned long long)__ballot(hit && i == best)) - 1;
}

// Lane holding the winner of one side: the extreme value, then the smallest index among the
// lanes holding it.  This is the (value, index) lexicographic order: -0 and +0 compare equal.
template <bool MAX>
__device__ __forceinline__ int winner_lane(double v, int i) {
  const double rv = wave_extreme<MAX>(v);
  return tie_lane(v == rv, i);
}

// Total order of (value, index) on 32-bit words, for reductions whose every round is one
// v_min_u32 with a DPP operand: the words of an ascending key of a double (negate for a maximum;
// -0 must not occur, it would order below +0).
__device__ __forceinline__ void order_words(double v, unsigned &hi, unsigned &lo) {
  const long long b = __double_as_longlong(v);
  const int s = (int)(b >> 63);
  hi = (unsigned)(b >> 32) ^ ((unsigned)s | 0x80000000u);
  lo = (unsigned)b ^ (unsigned)s;
}

template <int CTRL>
__device__ __forceinline__ unsigned dpp_min_u32(unsigned v) {  // every lane reads its source lane
  const unsigned o = (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
  return o < v ? o : v;
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_min_u32_rows(unsigned v) {
  const unsigned o = (unsigned)dpp_mov<CTRL, ROW_MASK>((int)v);
  return o < v ? o : v;
}

// Minimum over groups of N lanes (N = 4, 8, 16: DPP inside rows, to every lane of the group; 64:
// to every lane of the wave, in a scalar register).
template <int N>
__device__ __forceinline__ void lanes_min2(unsigned &a, unsigned &b) {
  a = dpp_min_u32<0xB1>(a);  // quad_perm [1,0,3,2]
  b = dpp_min_u32<0xB1>(b);
  a = dpp_min_u32<0x4E>(a);  // quad_perm [2,3,0,1]
  b = dpp_min_u32<0x4E>(b);
  if (N >= 8) {
    a = dpp_min_u32<0x124>(a);  // row_ror:4
    b = dpp_min_u32<0x124>(b);
  }
  if (N >= 16) {
    a = dpp_min_u32<0x128>(a);  // row_ror:8
    b = dpp_min_u32<0x128>(b);
  }
  if (N == 64) {
    a = dpp_min_u32_rows<0x142, 0xA>(a);  // row_bcast:15 -> rows 1, 3
    b = dpp_min_u32_rows<0x142, 0xA>(b);
    a = dpp_min_u32_rows<0x143, 0xC>(a);  // row_bcast:31 -> rows 2, 3
    b = dpp_min_u32_rows<0x143, 0xC>(b);
    a = (unsigned)__builtin_amdgcn_readlane((int)a, 63);
    b = (unsigned)__builtin_amdgcn_readlane((int)b, 63);
  }
}

// The first of the N lowest lanes that holds the smallest (hi, lo, i), given those with the
// smallest hi: lo and i are only looked at when several lanes share the smallest hi (the 20
// leading mantissa bits).
template <int N>
__device__ __forceinline__ int first_of(unsigned long long m, unsigned lo, unsigned i) {
  if (N < 64) m &= (1ull << (N & 63)) - 1ull;
  if (__builtin_expect((m & (m - 1)) == 0, 1)) return __builtin_ctzll(m);
  const int lane = threadIdx.x & 63;
  unsigned a = (m >> lane) & 1 ? lo : 0xffffffffu, b = a;
  lanes_min2<64>(a, b);
  m &= (unsigned long long)__ballot(lo == a);
  if ((m & (m - 1)) == 0) return __builtin_ctzll(m);
  a = b = (m >> lane) & 1 ? i : 0xffffffffu;
  lanes_min2<64>(a, b);
  return __builtin_ctzll(m & (unsigned long long)__ballot(i == a));
}

// Lanes of the two winners among the N lowest lanes (N < 64: lanes q, q + N, ... hold the same):
// smallest (vu, iu) and largest (vl, smallest il).  Called by all 64 lanes; uniform results.
template <int N>
__device__ __forceinline__ void winner_lanes(double vu, unsigned iu, double vl, unsigned il, int &lu, int &ll) {
  unsigned hu, ou, hl, ol;
  order_words(vu, hu, ou);
  order_words(-vl, hl, ol);
  unsigned mu = hu, ml = hl;
  lanes_min2<N>(mu, ml);
  lu = first_of<N>((unsigned long long)__ballot(hu == mu), ou, iu);
  ll = first_of<N>((unsigned long long)__ballot(hl == ml), ol, il);
}

__device__ __forceinline__ double uniform_d(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32));
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)b);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ void st_word(u64 *p, u64 v) {
  __hip_atomic_store(gp(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 ld_word(const u64 *p) {
  return __hip_atomic_load(gp(const_cast<u64 *>(p)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// 2x2 sub-problem on (u, l): eta = K_uu + K_ll - 2 K_ul with K_uu = K_ll = 1 for the RBF
// kernel, the box [L, H] on a_l, the partner clamped to [0, C], values within 1e-12 C of a
// bound snapped onto it.  Written without contraction so the fp64 rounding is that of the
// plain expression.
struct PairStep {
  double au, al;  // new multipliers of u and l
};

__device__ __forceinline__ PairStep solve_pair(double C, double bu, double bl, double au, double al, double yu,
                                               double yl, double kul) {
#pragma clang fp contract(off)
  double eta = (1.0 + 1.0) - 2.0 * kul;
  if (eta <= 0.0) eta = 1e-12;
  const double s = yu * yl;
  double L, H;
  if (s < 0) {
    L = fmax(0.0, al - au);
    H = fmin(C, C + al - au);
  } else {
    L = fmax(0.0, au + al - C);
    H = fmin(C, au + al);
  }
  // Clamps as max and min, and the two snaps side by side (a value cannot be within 1e-12 C of both
  // bounds): the same values with a shorter chain, and the chain is what a step waits for.  (A
  // zero's sign may differ before its snap; the snap makes it +0.)
  const double aln = fmin(fmax(al + yl * (bu - bl) / eta, L), H);
  const double aun = fmin(fmax(au + s * (al - aln), 0.0), C);
  const double snap = 1e-12 * C;
  const bool l0 = fabs(aln) <= snap, lC = fabs(aln - C) <= snap, u0 = fabs(aun) <= snap, uC = fabs(aun - C) <= snap;
  return PairStep{u0 ? 0.0 : (uC ? C : aun), l0 ? 0.0 : (lC ? C : aln)};
}

// f_j + (c_u K_uj + c_l K_lj), rounded as written (no contraction), so that every solver
// variant -- whatever its unrolling -- produces the same bits.
__device__ __forceinline__ double f_update(double f, double cu, float ku, double cl, float kl) {
#pragma clang fp contract(off)
  return f + (cu * (double)ku + cl * (double)kl);
}

}  // namespace svmx
