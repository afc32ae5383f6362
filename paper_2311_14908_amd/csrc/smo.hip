// smo.hip -- persistent SMO solver for gfx950 (paper, Section III.B: SMO with two Lagrange
// multipliers per step; the data-parallel work runs one thread per training sample).
//
// One cooperative launch advances every running problem by up to `steps` SMO steps.  A
// problem is served by nwg workgroups; workgroup r owns local samples [r*per_wg,
// (r+1)*per_wg) and keeps their f, alpha and label in registers for the whole launch.
// Each step:
//   1. every workgroup selects its own candidates  u_r = argmin_{I_up} f,  l_r = argmax_{I_low} f
//      (ties to the smaller index) with DPP wave reductions and one LDS hand-off;
//   2. the nwg partial results are exchanged through global memory as records of six
//      self-stamped 64-bit words (step stamp | payload, xchg_record.hpp), so no fence or cache
//      flush is needed: a reader simply waits until every word it needs carries the current
//      stamp.  With one level every
//      workgroup polls all records, one record per lane over as many waves as needed; with
//      two levels (the default above 128 workgroups) group leaders reduce about sqrt(nwg)
//      records each and publish a group record, and every workgroup then reads the group
//      records;
//   3. every workgroup reduces the same nwg records to the same pair (u, l), tests the stop
//      rule, and solves the 2x2 sub-problem redundantly (identical fp64 arithmetic);
//   4. every workgroup fetches K(u, j) and K(l, j) for its own samples -- from the Gram, or
//      computed from X as a GEMV against x_u and x_l with the squared row norms, the first
//      rows of its slice of X held in LDS for the whole launch -- and applies
//      f_j += da_u y_u K_uj + da_l y_l K_lj.
// Every wait is bounded by a wall-clock limit; on expiry the kernel records an error and
// all waits end, so a launch always drains.
#include "common.hpp"
#include "rbf_rows.hpp"
#include "pair_step.hpp"
#include "xchg_record.hpp"

#include <math.h>

namespace svmx {

// Gram path: 256-thread workgroups, up to 16 samples per thread.  Row path: 512-thread
// workgroups, one per CU (8 waves, each with a batch of samples x the lane's loads in flight,
// keep the streaming of X busy without spilling), up to 8 samples per thread.
constexpr int BS_GRAM = 256, MAXP_GRAM = 16;
constexpr int BS_ROWS = 512, MAXP_ROWS = 8;
constexpr int ROW_BATCH = 2;   // samples per lane group and batch of rows read from LDS
constexpr int ROW_SBATCH = 2;  // samples per lane group and batch of rows streamed from HBM
constexpr int ROW_MAXM = ROW_POSITIONS;  // feature positions per lane whose loads are issued together

int solver_block_size(bool gram) { return gram ? BS_GRAM : BS_ROWS; }
int max_per_thread(bool gram) { return gram ? MAXP_GRAM : MAXP_ROWS; }


// Candidates of one selection: min f over I_up (vu at index iu) and max f over I_low (vl at
// il), each with the multiplier and label of its sample.
struct Sel {
  double vu, au, vl, al;
  int iu, yu, il, yl;
};

__device__ __forceinline__ void sel_init(Sel &s) {
  s.vu = INFINITY; s.au = 0.0; s.iu = IBIG; s.yu = 0;
  s.vl = -INFINITY; s.al = 0.0; s.il = IBIG; s.yl = 0;
}

__device__ __forceinline__ void sel_merge(Sel &s, const Sel &o) {
  if (lt_min(o.vu, o.iu, s.vu, s.iu)) { s.vu = o.vu; s.iu = o.iu; s.au = o.au; s.yu = o.yu; }
  if (gt_max(o.vl, o.il, s.vl, s.il)) { s.vl = o.vl; s.il = o.il; s.al = o.al; s.yl = o.yl; }
}

// Candidate of the second-order choice of l (used with p.second_order): the largest gain
// g = (f_t - b_up)^2 / a_ut over the members t of I_low above b_up (ties to the smaller index),
// with f, multiplier, label and K(u, t) of that sample.
struct Sel2 {
  double g, fl, al, kul;
  int il, yl;
};

__device__ __forceinline__ void rec_init(Sel2 &s) {
  s.g = -INFINITY; s.fl = 0.0; s.al = 0.0; s.kul = 0.0; s.il = IBIG; s.yl = 0;
}
__device__ __forceinline__ void rec_merge(Sel2 &s, const Sel2 &o) {
  if (gt_max(o.g, o.il, s.g, s.il)) s = o;
}
__device__ __forceinline__ Sel2 rec_wave(const Sel2 &mine) {
  const int lane = winner_lane<true>(mine.g, mine.il);
  Sel2 r;
  r.g = readlane_d(mine.g, lane);
  r.fl = readlane_d(mine.fl, lane);
  r.al = readlane_d(mine.al, lane);
  r.kul = readlane_d(mine.kul, lane);
  r.il = __builtin_amdgcn_readlane(mine.il, lane);
  r.yl = __builtin_amdgcn_readlane(mine.yl, lane);
  return r;
}

__device__ __forceinline__ unsigned pack_index(int i, int y) { return (unsigned)i | (y < 0 ? 0x80000000u : 0u); }
__device__ __forceinline__ void unpack_index(unsigned w, int &i, int &y) {
  i = (int)(w & 0x7fffffffu);
  y = (w >> 31) ? -1 : 1;
}

// LDS hand-off between the waves of a workgroup.  Two buffers used alternately, so one
// barrier per hand-off suffices: a buffer is rewritten only after another hand-off's barrier.
template <class R, int NW>
struct RecLds {
  R slot[2][NW];
};

// Combine the wave results of all waves; every thread returns the same workgroup result.
template <class R, int NW>
__device__ __forceinline__ R rec_block(const R &wave_res, RecLds<R, NW> &L, int &buf) {
  if ((threadIdx.x & 63) == 0) L.slot[buf][threadIdx.x >> 6] = wave_res;
  __syncthreads();
  R r = L.slot[buf][0];
#pragma unroll
  for (int q = 1; q < NW; ++q) rec_merge(r, L.slot[buf][q]);
  buf ^= 1;
  return r;
}

// The same hand-off for the two candidates of the first-order rule.  A wave's two winning lanes
// write their own fields; after the barrier lane q of every wave reads wave q's candidates, the
// winners are found among those lanes, and their fields come out in scalar registers, so that
// the addresses, tests and the pair's multipliers that follow are scalar.
// The step of a problem is a chain of such short stages and bound by their latency, instruction
// after instruction of one wave a SIMD: reducing 32-bit leading words (a move and a v_min_u32 a
// round) instead of (value, index) pairs of doubles, letting lanes combine the waves instead of
// every thread in turn, branch-free offers, scalar addresses and tests, and issuing the rows'
// loads before the tests took a step from 4.08 to 3.29 us at 20,000 x 784 (40 workgroups; 2.0 us
// of it the exchange) and from 2.1 to 1.5 us at 1,000 x 16 (one workgroup), from 4.61 to 3.72 us at
// 50,000 x 128 and from 5.23 to 4.01 at 100,000 x 32, bit for bit the same.
struct SelRec {
  double vu, au, vl, al;
  unsigned wu, wl;  // index | label
};

template <int NW>
struct SelLds {
  SelRec slot[2][NW];
};

// The lane of each winner writes it.
__device__ __forceinline__ void sel_put(SelRec &r, const Sel &s, int lu, int ll) {
  const int lane = threadIdx.x & 63;
  if (lane == lu) { r.vu = s.vu; r.au = s.au; r.wu = pack_index(s.iu, s.yu); }
  if (lane == ll) { r.vl = s.vl; r.al = s.al; r.wl = pack_index(s.il, s.yl); }
}

// The winners of lanes 0 .. N-1, each a candidate of its own, in scalar registers.
__device__ __forceinline__ Sel sel_from_lanes(const SelRec &r, int lu, int ll) {
  Sel s;
  s.vu = readlane_d(r.vu, lu);
  s.au = readlane_d(r.au, lu);
  unpack_index((unsigned)__builtin_amdgcn_readlane((int)r.wu, lu), s.iu, s.yu);
  s.vl = readlane_d(r.vl, ll);
  s.al = readlane_d(r.al, ll);
  unpack_index((unsigned)__builtin_amdgcn_readlane((int)r.wl, ll), s.il, s.yl);
  return s;
}

__device__ __forceinline__ void rec_limbs_of(const Sel &s, u64 (&L)[5]) {
  L[0] = (u64)__double_as_longlong(s.vu);
  L[1] = (u64)__double_as_longlong(s.au);
  L[2] = (u64)pack_index(s.iu, s.yu) | ((u64)pack_index(s.il, s.yl) << 32);
  L[3] = (u64)__double_as_longlong(s.vl);
  L[4] = (u64)__double_as_longlong(s.al);
}
// A record of scalar fields: the six words are packed by the scalar unit and dealt to lanes 0-5.
__device__ __forceinline__ void put_record_uniform(u64 *rec, unsigned stamp, const Sel &s) {
  u64 L[5];
  rec_limbs_of(s, L);
  const int t = threadIdx.x & 63;
  u64 mine = rec_word(L, 0, stamp);
#pragma unroll
  for (int w = 1; w < REC_WORDS; ++w) {
    const u64 v = rec_word(L, w, stamp);
    mine = t == w ? v : mine;
  }
  if (t < REC_WORDS) st_word(rec + t, mine);
}

// slots: one record per wave, written before the call; ends with the workgroup's winners.
template <int NW>
__device__ __forceinline__ Sel sel_combine(const SelRec (&slot)[NW]) {
  __syncthreads();
  const SelRec r = slot[threadIdx.x & (NW - 1)];
  int lu, ll;
  winner_lanes<NW>(r.vu, r.wu & 0x7fffffffu, r.vl, r.wl & 0x7fffffffu, lu, ll);
  return sel_from_lanes(r, lu, ll);
}

// Limbs of a record (xchg_record.hpp): v_up, a_up, index words, v_low, a_low; the label travels
// in bit 31 of the index word.
__device__ __forceinline__ void rec_from_limbs(const u64 (&L)[5], Sel &o) {
  o.vu = __longlong_as_double((long long)L[0]);
  o.au = __longlong_as_double((long long)L[1]);
  unpack_index((unsigned)L[2], o.iu, o.yu);
  unpack_index((unsigned)(L[2] >> 32), o.il, o.yl);
  o.vl = __longlong_as_double((long long)L[3]);
  o.al = __longlong_as_double((long long)L[4]);
}
// Second-order record: gain, f_l, index word, a_l, K(u, l).
__device__ __forceinline__ void rec_limbs_of(const Sel2 &s, u64 (&L)[5]) {
  L[0] = (u64)__double_as_longlong(s.g);
  L[1] = (u64)__double_as_longlong(s.fl);
  L[2] = (u64)pack_index(s.il, s.yl);
  L[3] = (u64)__double_as_longlong(s.al);
  L[4] = (u64)__double_as_longlong(s.kul);
}
__device__ __forceinline__ void rec_from_limbs(const u64 (&L)[5], Sel2 &o) {
  o.g = __longlong_as_double((long long)L[0]);
  o.fl = __longlong_as_double((long long)L[1]);
  unpack_index((unsigned)L[2], o.il, o.yl);
  o.al = __longlong_as_double((long long)L[3]);
  o.kul = __longlong_as_double((long long)L[4]);
}

// Lanes 0..REC_WORDS-1 of the calling wave each write one word of the record.
template <class R>
__device__ __forceinline__ void put_record(u64 *rec, unsigned stamp, const R &s) {
  const int t = threadIdx.x & 63;
  if (t < REC_WORDS) {
    u64 L[5];
    rec_limbs_of(s, L);
    st_word(rec + t, rec_word(L, t, stamp));
  }
}

// Wave-level: wait for records q0 + lane, q0 + lane + stride, ... below q1 of `words` to carry
// `stamp`, reduce them, and return the result to every lane of the wave (all 64 lanes must
// call).
template <class R>
__device__ R poll_reduce(const u64 *words, int q0, int q1, int stride, unsigned stamp, uint64_t spin_limit,
                         int32_t *err, int *abort_flag) {
  R s;
  rec_init(s);
  for (int q = q0 + (int)(threadIdx.x & 63); q < q1; q += stride) {
    const u64 *rec = words + (size_t)q * SLOT_WORDS;
    u64 w[REC_WORDS];
    const uint64_t t0 = wall_clock64();
    for (;;) {
      bool ok = true;
#pragma unroll
      for (int k = 0; k < REC_WORDS; ++k) {
        w[k] = ld_word(rec + k);
        ok = ok && rec_stamped(w[k], stamp);
      }
      if (ok) break;
      if (wall_clock64() - t0 > spin_limit) {
        __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *abort_flag = 1;
        break;
      }
    }
    u64 L[5];
    rec_limbs(w, L);
    R o;
    rec_from_limbs(L, o);
    rec_merge(s, o);
  }
  return rec_wave(s);
}

// Exchange of the workgroup results of one problem (see file comment, item 2).  Wave 0
// publishes the record.  With one level, the records are polled by as many waves as needed
// for one record per lane (wave w takes records w*64 + lane, then every 64*pollers-th), each
// wave reduces its share, and the shares meet in LDS.  With two levels, wave 0 does the
// global-memory work of both levels.  The stamp's parity selects the buffer.
template <class R, int NW>
__device__ R exchange(const Prob &P, int rank, unsigned stamp, const R &mine, RecLds<R, NW> &L, int &buf,
                      uint64_t spin_limit, int32_t *err, int *abort_flag) {
  const size_t par = stamp & 1u;
  u64 *lv1 = P.slots + par * (size_t)P.nwg * SLOT_WORDS;
  const int wave = threadIdx.x >> 6;
  int pollers = 1;
  if (wave == 0) put_record(lv1 + (size_t)rank * SLOT_WORDS, stamp, mine);
  if (P.g1 > 0) {
    if (wave == 0) {
      u64 *lv2 = P.slots2 + par * (size_t)P.ng * SLOT_WORDS;
      const int g = rank / P.g1;
      if (rank == group_leader(P, g)) {
        const int q0 = g * P.g1, q1 = min(P.nwg, q0 + P.g1);
        const R gs = poll_reduce<R>(lv1, q0, q1, 64, stamp, spin_limit, err, abort_flag);
        put_record(lv2 + (size_t)g * SLOT_WORDS, stamp, gs);
      }
      const R s = poll_reduce<R>(lv2, 0, P.ng, 64, stamp, spin_limit, err, abort_flag);
      if (threadIdx.x == 0) L.slot[buf][0] = s;
    }
  } else {
    pollers = min(NW, (P.nwg + 63) >> 6);
    if (wave < pollers) {
      const R s = poll_reduce<R>(lv1, wave * 64, P.nwg, 64 * pollers, stamp, spin_limit, err, abort_flag);
      if ((threadIdx.x & 63) == 0) L.slot[buf][wave] = s;
    }
  }
  __syncthreads();
  R r = L.slot[buf][0];
  for (int q = 1; q < pollers; ++q) rec_merge(r, L.slot[buf][q]);
  buf ^= 1;
  return r;
}

// exchange for the first-order candidates: the same protocol; the lanes that hold the winning
// records write them to LDS, and every wave reads the one result into scalar registers.
__device__ __forceinline__ void poll_lanes(const u64 *words, int q0, int q1, int stride, unsigned stamp,
                                           uint64_t spin_limit, int32_t *err, int *abort_flag, Sel &s, int &lu, int &ll) {
  sel_init(s);
  for (int q = q0 + (int)(threadIdx.x & 63); q < q1; q += stride) {
    const u64 *rec = words + (size_t)q * SLOT_WORDS;
    u64 w[REC_WORDS];
    const uint64_t t0 = wall_clock64();
    for (;;) {
      bool ok = true;
#pragma unroll
      for (int k = 0; k < REC_WORDS; ++k) {
        w[k] = ld_word(rec + k);
        ok = ok && rec_stamped(w[k], stamp);
      }
      if (ok) break;
      if (wall_clock64() - t0 > spin_limit) {
        __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *abort_flag = 1;
        break;
      }
    }
    u64 L[5];
    rec_limbs(w, L);
    Sel o;
    rec_from_limbs(L, o);
    if (q < q0 + 64)
      s = o;
    else
      sel_merge(s, o);
  }
  winner_lanes<64>(s.vu, (unsigned)s.iu, s.vl, (unsigned)s.il, lu, ll);
}

// What the exchange needs of a problem and of the workgroup's place in it.
struct Xchg {
  u64 *slots, *slots2;
  int nwg, g1, ng, rank, group, q0, q1;  // q0 .. q1: the group whose leader this workgroup is (else empty)
};

__device__ __forceinline__ Xchg xchg_of(const Prob &P, int rank) {
  Xchg x;
  x.slots = P.slots;
  x.slots2 = P.slots2;
  x.nwg = P.nwg;
  x.g1 = P.g1;
  x.ng = P.ng;
  x.rank = rank;
  x.group = P.g1 > 0 ? __builtin_amdgcn_readfirstlane(rank / P.g1) : 0;
  const bool leads = P.g1 > 0 && rank == group_leader(P, x.group);
  x.q0 = x.group * P.g1;
  x.q1 = leads ? min(P.nwg, x.q0 + P.g1) : x.q0;
  return x;
}

template <int NW>
__device__ __forceinline__ Sel sel_exchange(const Xchg &x, unsigned stamp, const Sel &mine, SelLds<NW> &L, int &buf,
                                            uint64_t spin_limit, int32_t *err, int *abort_flag, bool &aborted) {
  const unsigned par = stamp & 1u;
  u64 *lv1 = x.slots + par * (unsigned)x.nwg * SLOT_WORDS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave == 0) put_record_uniform(lv1 + x.rank * SLOT_WORDS, stamp, mine);
  int pollers = 1, lu, ll;
  Sel s;
  if (x.g1 > 0) {
    if (wave == 0) {
      u64 *lv2 = x.slots2 + par * (unsigned)x.ng * SLOT_WORDS;
      if (x.q1 > x.q0) {
        poll_lanes(lv1, x.q0, x.q1, 64, stamp, spin_limit, err, abort_flag, s, lu, ll);
        SelRec r{s.vu, s.au, s.vl, s.al, pack_index(s.iu, s.yu), pack_index(s.il, s.yl)};
        put_record_uniform(lv2 + x.group * SLOT_WORDS, stamp, sel_from_lanes(r, lu, ll));
      }
      poll_lanes(lv2, 0, x.ng, 64, stamp, spin_limit, err, abort_flag, s, lu, ll);
      sel_put(L.slot[buf][0], s, lu, ll);
    }
  } else {
    pollers = min(NW, (x.nwg + 63) >> 6);
    if (wave < pollers) {
      poll_lanes(lv1, wave * 64, x.nwg, 64 * pollers, stamp, spin_limit, err, abort_flag, s, lu, ll);
      sel_put(L.slot[buf][wave], s, lu, ll);
    } else if (pollers > 1) {  // an empty candidate, for the combination
      sel_init(s);
      sel_put(L.slot[buf][wave], s, 0, 0);
    }
  }
  Sel r;
  if (__builtin_expect(pollers > 1, 0)) {
    r = sel_combine<NW>(L.slot[buf]);
    aborted = *abort_flag != 0;
  } else {
    __syncthreads();
    const SelRec rec = L.slot[buf][0];
    const int ab = *abort_flag;
    r = sel_from_lanes(rec, 0, 0);
    aborted = __builtin_amdgcn_readfirstlane(ab) != 0;
  }
  buf ^= 1;
  return r;
}

__device__ __forceinline__ int64_t gmap(const Prob &P, int64_t j) { return j < P.len0 ? P.off0 + j : P.off1 + (j - P.len0); }
__device__ __forceinline__ int label_of(const Prob &P, int64_t j) {
  return P.y ? gp(P.y)[gmap(P, j)] : (j < P.len0 ? 1 : -1);
}

// Gain of the second-order rule for a member t of I_low above b_up: (f_t - b_up)^2 / a_ut with
// a_ut = K_uu + K_tt - 2 K_ut, K_uu = K_tt = 1 for the RBF kernel, 1e-12 when not positive.
// Rounded as written (no contraction).
__device__ __forceinline__ double so_gain(double ft, double bup, float kut) {
#pragma clang fp contract(off)
  const double bt = ft - bup;
  double at = (1.0 + 1.0) - 2.0 * (double)kut;
  if (at <= 0.0) at = 1e-12;
  return bt * bt / at;
}

// This thread's samples and their candidates.  Membership of I_up and I_low is kept per sample and
// only changes for u and l.  Gram path: as what is added to its f before it is compared, 0 for a
// member (which also turns -0 into +0), +-infinity otherwise, so offering a sample costs an
// addition, a compare and three selects a side and no branch.  FLAGS: as bits, where the registers are
// needed: on the row path by the rows, and with 8 samples a thread or more.  With 16 the 64 registers of
// addends spilled (second-order rule, 500 steps at 2,500 x 64 4.46 -> 3.32 ms, at 4,096 x 10 5.36 ->
// 3.62; first-order 1.70 -> 1.62); with 8 a CU held two workgroups instead of three, which splits
// one-vs-one trainings into more batches (36 classes of 1,000, 630 pairs, 2.75 -> 2.16 ms; 10 of 9,000
// with 16 workgroups a pair 9.26 -> 7.10).
template <int BS, int PER, bool FLAGS>
struct Own {
  static constexpr int NP = FLAGS ? 1 : PER;
  double f[PER], a[PER], pu[NP], pl[NP];
  unsigned mu, ml;  // FLAGS: bit k: sample k is in I_up, in I_low
  unsigned ypos;    // bit k: the label of sample k is +1
  double bu, bl;    // best value of each side, and which of the PER samples has it
  int ku, kl;

  __device__ __forceinline__ void member(int k, bool up, bool low) {
    if (FLAGS) {
      mu = (mu & ~(1u << k)) | (up ? 1u << k : 0u);
      ml = (ml & ~(1u << k)) | (low ? 1u << k : 0u);
    } else {
      pu[FLAGS ? 0 : k] = up ? 0.0 : INFINITY;
      pl[FLAGS ? 0 : k] = low ? 0.0 : -INFINITY;
    }
  }
  __device__ __forceinline__ bool in_low(int k) const { return FLAGS ? ((ml >> k) & 1u) != 0 : pl[FLAGS ? 0 : k] == 0.0; }
  __device__ __forceinline__ void start() { bu = INFINITY; bl = -INFINITY; ku = kl = 0; }
  __device__ __forceinline__ void offer(int k) {
    double u, l;
    if (FLAGS) {
      const double v = f[k] + 0.0;
      u = (mu >> k) & 1u ? v : INFINITY;
      l = (ml >> k) & 1u ? v : -INFINITY;
    } else {
      u = f[k] + pu[FLAGS ? 0 : k];
      l = f[k] + pl[FLAGS ? 0 : k];
    }
    ku = u < bu ? k : ku;
    bu = u < bu ? u : bu;
    kl = l > bl ? k : kl;
    bl = l > bl ? l : bl;
  }
  // The wave's two winners to r (local index base + thread + k BS).  Every lane picks the
  // multiplier and label of its own candidates, in the shadow of the reduction's rounds.
  __device__ __forceinline__ void put_wave(SelRec &r, int base) const {
    const int j = base + (int)threadIdx.x;
    unsigned wu = (unsigned)(j + ku * BS), wl = (unsigned)(j + kl * BS);
    wu = bu < INFINITY ? wu : (unsigned)IBIG;
    wl = bl > -INFINITY ? wl : (unsigned)IBIG;
    int lu, ll;
    winner_lanes<64>(bu, wu, bl, wl, lu, ll);
    double au = a[0], al = a[0];
#pragma unroll
    for (int k = 1; k < PER; ++k) {
      au = ku == k ? a[k] : au;
      al = kl == k ? a[k] : al;
    }
    wu |= (~ypos >> ku) << 31;  // (an empty side carries some label, which nobody reads)
    wl |= (~ypos >> kl) << 31;
    const int lane = threadIdx.x & 63;
    if (lane == lu) { r.vu = bu; r.au = au; r.wu = wu; }
    if (lane == ll) { r.vl = bl; r.al = al; r.wl = wl; }
  }
  // Sample j (uniform, of label y) of this workgroup's slice [base, base + cnt) has a new multiplier.
  __device__ __forceinline__ void assign(int j, int base, int cnt, int y, double v, double C) {
    const unsigned q = (unsigned)(j - base);
    if (q >= (unsigned)cnt) return;
    const bool mine = threadIdx.x == q % BS;
    const bool up = y > 0 ? v < C : v > 0.0, low = y > 0 ? v > 0.0 : v < C;
#pragma unroll
    for (int k = 0; k < PER; ++k) {  // selects: branches on k would keep the arrays in scratch memory
      const bool hit = mine && k == (int)(q / BS);
      a[k] = hit ? v : a[k];
      if (!FLAGS) {
        pu[FLAGS ? 0 : k] = hit ? (up ? 0.0 : INFINITY) : pu[FLAGS ? 0 : k];
        pl[FLAGS ? 0 : k] = hit ? (low ? 0.0 : -INFINITY) : pl[FLAGS ? 0 : k];
      }
    }
    if (FLAGS) {
      const unsigned bit = mine ? 1u << (q / BS) : 0u;
      mu = up ? mu | bit : mu & ~bit;
      ml = low ? ml | bit : ml & ~bit;
    }
  }
};

// ---------------------------------------------------------------------------------------
// SO (Gram path): the second index of the pair by the second-order rule (p.second_order).
template <int BS, int PER, bool GRAM, int V, bool ONE = false, bool SO = false>
__global__ void __launch_bounds__(BS) smo_solve(SolveParams p) {
  constexpr int NW = BS / 64;
  // Samples per lane group and batch (a sample's arithmetic does not depend on them): scalar
  // lanes hold a quarter of the registers per sample, so they take twice as many; ONE: one at
  // a time (row_batch_one).
  constexpr int SB = ONE ? 1 : V != ROW_SCALAR ? ROW_BATCH : 2 * ROW_BATCH;
  // Row path, dynamic LDS: dot products against x_u and x_l [2][per_wg] (fp64), cache tags
  // [cap], then the rows of X this workgroup keeps resident [res][d] (16-byte aligned).
  extern __shared__ float4 dyn4[];
  __shared__ SelLds<NW> sh;
  __shared__ RecLds<Sel2, NW> sh2;
  __shared__ int s_abort;
  __shared__ double s_kul;
  int buf = 0, buf2 = 0;

  const int32_t pid = __builtin_amdgcn_readfirstlane(p.wg_prob[blockIdx.x]);
  const Prob P = p.probs[pid];
  const int rank = (int)blockIdx.x - P.wg0;
  Ctl *ctl = P.ctl;
  if (ctl->status != ST_RUNNING || input_invalid(p.check)) return;
  const int64_t t0 = ctl->t;
  int64_t t = ((int64_t)__builtin_amdgcn_readfirstlane((int)(t0 >> 32)) << 32) |
              (unsigned)__builtin_amdgcn_readfirstlane((int)t0);
  if (threadIdx.x == 0) s_abort = 0;

  const int64_t base = (int64_t)rank * P.per_wg;
  const int64_t lim = min(base + (int64_t)P.per_wg, P.n);
  const double C = p.C;
  const bool from_zero = t == 0 && p.warm == 0;
  Own<BS, PER, !GRAM || PER >= 8> own;
  own.ypos = own.mu = own.ml = 0;
  unsigned col[PER];  // Gram path: byte offset of sample k's column in a row of the Gram
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t j = base + threadIdx.x + (int64_t)k * BS;
    const int64_t jc = min(j, lim - 1);  // past the end: some column, read and not used
    if (GRAM) col[k] = (unsigned)(4 * gmap(P, jc));
    if (j < lim) {
      own.f[k] = gp(P.f)[j];
      own.a[k] = from_zero ? 0.0 : gp(P.alpha)[j];
      const bool pos = label_of(P, j) > 0;
      own.ypos |= pos ? 1u << k : 0u;
      own.member(k, pos ? own.a[k] < C : own.a[k] > 0.0, pos ? own.a[k] > 0.0 : own.a[k] < C);
    } else {
      own.f[k] = 0.0;
      own.a[k] = 0.0;
      own.member(k, false, false);
    }
  }

  double *dotu = reinterpret_cast<double *>(dyn4), *dotl = dotu + P.per_wg;
  int *tags = reinterpret_cast<int *>(dotl + P.per_wg);
  float *xres = reinterpret_cast<float *>(dyn4 + ((16 * (int64_t)P.per_wg + 4 * (int64_t)p.cache_cap + 15) >> 4));
  const bool use_cache = !GRAM && p.cache != nullptr && p.cache_cap > 0;
  // Resident rows: the first `res` samples of the slice, copied once per launch; every step
  // reads them from LDS instead of HBM.
  const int64_t res = GRAM ? 0 : min<int64_t>(p.res_rows, max<int64_t>(0, lim - base));
  double sq[PER];  // squared norms of the own samples (row path)
  if (!GRAM) {
    if (use_cache) {
      for (int s = threadIdx.x; s < p.cache_cap; s += BS) tags[s] = gp(p.cache_tags)[(size_t)blockIdx.x * p.cache_cap + s];
    }
    typedef typename Lane<V>::T T;
    const int64_t units = row_units(p.d, V);
    T *xr = reinterpret_cast<T *>(xres);
    for (int64_t e = threadIdx.x; e < res * units; e += BS) {
      const int64_t r = e / units, k = e - r * units;
      xr[e] = Lane<V>::load(p.X + gmap(P, base + r) * p.d, k, p.d);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int64_t j = base + threadIdx.x + (int64_t)k * BS;
      sq[k] = j < lim ? gp(p.sqn)[gmap(P, j)] : 0.0;
    }
  }
  __syncthreads();

  const int64_t t_end = min(t + p.steps, p.max_iter);
  // Candidates of this thread's samples; after the first scan they are gathered in the same
  // pass as the f update of the previous step.
  own.start();
#pragma unroll
  for (int k = 0; k < PER; ++k) own.offer(k);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // What the loop needs of the problem, in scalar registers (local samples and rows are below 2^31).
  const int n = (int)P.n, nwg = P.nwg, len0 = (int)P.len0, cnt = (int)(lim - base);
  const int64_t off0 = P.off0, off1 = P.off1 - P.len0, trace_len = P.trace_len;
  const Xchg xc = xchg_of(P, rank);
  for (;;) {
    // 1. workgroup candidates
    own.put_wave(sh.slot[buf][wave], (int)base);
    Sel s = sel_combine<NW>(sh.slot[buf]);
    buf ^= 1;
    // 2. exchange across the problem's workgroups (with the second-order rule every step has two
    // exchanges, stamped 2t + 1 and 2t + 2)
    const unsigned stamp1 = SO ? (unsigned)(2 * t + 1) : (unsigned)(t + 1);
    bool aborted = false;
    if (nwg > 1) s = sel_exchange<NW>(xc, stamp1, s, sh, buf, p.spin_limit, p.error, &s_abort, aborted);
    // The rows of the pair are on their way before anything else happens (an empty selection, which
    // ends the launch below, reads row n - 1).
    const int64_t u = min(s.iu, n - 1);
    int64_t l = min(s.il, n - 1);
    const int64_t gu = u + (u < len0 ? off0 : off1);
    float ku[PER], kl[PER];
    double kul = 0.0;
    if (GRAM && !SO) {
      const int64_t gl = l + (l < len0 ? off0 : off1);
      const SVMX_GLOBAL char *Ru = gp(reinterpret_cast<const char *>(p.gram + gu * p.ld));
      const SVMX_GLOBAL char *Rl = gp(reinterpret_cast<const char *>(p.gram + gl * p.ld));
      kul = (double)*reinterpret_cast<const SVMX_GLOBAL float *>(Ru + 4 * gl);
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        unsigned c = col[k];
        asm volatile("" : "+v"(c));  // stays a 32-bit offset to a scalar base
        ku[k] = *reinterpret_cast<const SVMX_GLOBAL float *>(Ru + c);
        kl[k] = *reinterpret_cast<const SVMX_GLOBAL float *>(Rl + c);
      }
    }
    // 3. stop rule
    if (t < trace_len && rank == 0 && threadIdx.x == 0) {
      if (P.trace_ul) { gp(P.trace_ul)[2 * t] = s.iu; gp(P.trace_ul)[2 * t + 1] = s.il; }
      if (P.trace_b) { gp(P.trace_b)[2 * t] = s.vu; gp(P.trace_b)[2 * t + 1] = s.vl; }
    }
    const bool done = s.iu == IBIG || s.il == IBIG || s.vl - s.vu <= p.tol;
    if (__builtin_expect(aborted || done || t >= t_end, 0)) {
      if (rank == 0 && threadIdx.x == 0) {
        ctl->t = t;
        ctl->status = aborted ? ST_TIMEOUT : done ? ST_CONVERGED : t >= p.max_iter ? ST_MAXITER : ST_RUNNING;
        ctl->b_up = s.vu;
        ctl->b_low = s.vl;
        ctl->u = s.iu;
        ctl->l = s.il;
      }
      break;
    }
    double yl = (double)s.yl, fl = s.vl, al = s.al;
    const double yu = (double)s.yu;

    // 4. kernel rows of u and l for the own samples, K_ul, 2x2 solve, f update
    if (!GRAM || SO) {
#pragma unroll
      for (int k = 0; k < PER; ++k) ku[k] = kl[k] = 0.f;
    }
    if (GRAM && SO) {
      // Second-order rule: row u first, the gains of the own members of I_low above b_up, a
      // second exchange for l (its record carries f_l, a_l, y_l and K(u, l)), then row l.
      const SVMX_GLOBAL float *Ru = gp(p.gram) + gu * p.ld;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int64_t j = base + threadIdx.x + (int64_t)k * BS;
        if (j < lim) ku[k] = Ru[gmap(P, j)];
      }
      Sel2 c;
      rec_init(c);
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int64_t j = base + threadIdx.x + (int64_t)k * BS;
        if (own.in_low(k) && own.f[k] > s.vu) {
          const double g = so_gain(own.f[k], s.vu, ku[k]);
          if (gt_max(g, (int)j, c.g, c.il)) {
            c.g = g; c.fl = own.f[k]; c.al = own.a[k]; c.kul = (double)ku[k]; c.il = (int)j;
            c.yl = (own.ypos >> k) & 1u ? 1 : -1;
          }
        }
      }
      c = rec_block<Sel2, NW>(rec_wave(c), sh2, buf2);
      if (P.nwg > 1)
        c = exchange<Sel2, NW>(P, rank, (unsigned)(2 * t + 2), c, sh2, buf2, p.spin_limit, p.error, &s_abort);
      if (s_abort != 0) {
        if (rank == 0 && threadIdx.x == 0) {
          ctl->t = t;
          ctl->status = ST_TIMEOUT;
        }
        break;
      }
      // A member of I_low above b_up exists whenever the stop rule fails (b_low > b_up + tol);
      // the maximal violating pair's l stands in should none have been found.
      if (c.il != IBIG) {
        l = c.il;
        yl = (double)c.yl;
        fl = c.fl;
        al = c.al;
      }
      if (rank == 0 && threadIdx.x == 0 && t < P.trace_len && P.trace_ul) P.trace_ul[2 * t + 1] = (int)l;
      const int64_t gl = gmap(P, l);
      const SVMX_GLOBAL float *Rl = gp(p.gram) + gl * p.ld;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int64_t j = base + threadIdx.x + (int64_t)k * BS;
        if (j < lim) kl[k] = Rl[gmap(P, j)];
      }
      kul = c.il != IBIG ? c.kul : (double)Ru[gl];
    } else if (!GRAM) {
      const int64_t gl = gmap(P, l);
      const int64_t d = p.d;
      const int gs = group_size_for(d, V);
      const int lig = threadIdx.x & (gs - 1);
      const int ngroups = BS / gs;
      const int grp = threadIdx.x / gs;
      // Block 0 of x_u and x_l is held in registers for the whole step; the samples stream
      // past it in batches of SB.
      const float *xu = p.X + gu * d, *xl = p.X + gl * d;
      const double nu = gp(p.sqn)[gu], nl = gp(p.sqn)[gl];
      RowPair<V, ROW_MAXM> rp;
      load_pair(rp, xu, xl, d, lig, gs);
      int su = -1, sl = -1;
      bool hit_u = false, hit_l = false;
      if (use_cache) {
        su = (int)(gu % p.cache_cap);
        sl = (int)(gl % p.cache_cap);
        hit_u = tags[su] == (int)gu;
        hit_l = tags[sl] == (int)gl;
      }
      // K_ul: x_l as the sample against x_u, exactly as the row of u evaluates sample l
      if (grp == 0) {
        const float *xs1[1] = {xl};
        double pu1[1], pl1[1];
        dot_batch<V, 1, ROW_MAXM>(xs1, 1, xu, xl, d, lig, gs, rp, pu1, pl1);
        if (lig == 0) s_kul = (double)rbf_from_dot(nu, nl, pu1[0], p.gamma);
      }
      if (!(hit_u && hit_l)) {
        typedef typename Lane<V>::T T;
        // Streamed samples [res, cnt) go in batches of SBS per group; the first batch of each
        // group is loaded before the resident samples are computed, so its HBM latency
        // overlaps that work.
        constexpr int SBS = ONE ? 1 : V != ROW_SCALAR ? ROW_SBATCH : 2 * ROW_SBATCH;
        const int64_t sstride = (int64_t)ngroups * SBS;
        int64_t qs = res + (int64_t)grp * SBS;
        int nbs = 0;
        const float *xs[SBS];
        T vs[SBS][ROW_MAXM];
        if (qs < cnt) {
          nbs = (int)min<int64_t>(SBS, cnt - qs);
#pragma unroll
          for (int b = 0; b < SBS; ++b) xs[b] = p.X + gmap(P, base + qs + min(b, nbs - 1)) * d;
          load_block0<V, SBS, ROW_MAXM>(vs, xs, nbs, d, lig, gs);
        }
        for (int64_t q0 = (int64_t)grp * SB; q0 < res; q0 += (int64_t)ngroups * SB) {
          const int nb = (int)min<int64_t>(SB, res - q0);
          const float *xr[SB];
#pragma unroll
          for (int b = 0; b < SB; ++b) xr[b] = xres + (q0 + min(b, nb - 1)) * row_lds_pitch(d, V);
          T vr[SB][ROW_MAXM];
          load_block0<V, SB, ROW_MAXM, true>(vr, xr, nb, d, lig, gs);
          typename Lane<V>::Acc fu[SB], fl[SB];
          dot_partials<V, SB, ROW_MAXM, true>(vr, xr, nb, xu, xl, d, lig, gs, rp, fu, fl);
          group_sums_store<V, SB>(fu, fl, nb, gs, lig, dotu + q0, dotl + q0);
        }
        while (qs < cnt) {
          typename Lane<V>::Acc fu[SBS], fl[SBS];
          dot_partials<V, SBS, ROW_MAXM>(vs, xs, nbs, xu, xl, d, lig, gs, rp, fu, fl);
          group_sums_store<V, SBS>(fu, fl, nbs, gs, lig, dotu + qs, dotl + qs);
          qs += sstride;
          if (qs < cnt) {
            nbs = (int)min<int64_t>(SBS, cnt - qs);
#pragma unroll
            for (int b = 0; b < SBS; ++b) xs[b] = p.X + gmap(P, base + qs + min(b, nbs - 1)) * d;
            load_block0<V, SBS, ROW_MAXM>(vs, xs, nbs, d, lig, gs);
          }
        }
      }
      __syncthreads();
      kul = s_kul;
      const bool store_u = use_cache && !hit_u;
      const bool store_l = use_cache && !hit_l && !(sl == su && store_u);
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int64_t j = base + threadIdx.x + (int64_t)k * BS;
        if (j < lim) {
          const int64_t q = j - base;
          ku[k] = hit_u ? gp(p.cache)[(size_t)su * p.ld + j] : rbf_from_dot(nu, sq[k], dotu[q], p.gamma);
          kl[k] = hit_l ? gp(p.cache)[(size_t)sl * p.ld + j] : rbf_from_dot(nl, sq[k], dotl[q], p.gamma);
          if (store_u) gp(p.cache)[(size_t)su * p.ld + j] = ku[k];
          if (store_l) gp(p.cache)[(size_t)sl * p.ld + j] = kl[k];
        }
      }
      if (use_cache) {
        __syncthreads();
        if (threadIdx.x == 0) {
          if (store_u) tags[su] = (int)gu;
          if (store_l) tags[sl] = (int)gl;
        }
      }
    }
    const PairStep ps = solve_pair(C, s.vu, fl, s.au, al, yu, yl, kul);
    const double au_new = ps.au, al_new = ps.al;
    const double cu = (au_new - s.au) * yu, cl = (al_new - al) * yl;
    own.assign((int)u, (int)base, cnt, s.yu, au_new, C);
    own.assign((int)l, (int)base, cnt, l == s.il ? s.yl : (int)yl, al_new, C);
    own.start();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      own.f[k] = f_update(own.f[k], cu, ku[k], cl, kl[k]);
      own.offer(k);
    }
    ++t;
  }

#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t j = base + threadIdx.x + (int64_t)k * BS;
    if (j < lim) {
      gp(P.f)[j] = own.f[k];
      gp(P.alpha)[j] = own.a[k];
    }
  }
  if (use_cache) {
    __syncthreads();
    for (int s2 = threadIdx.x; s2 < p.cache_cap; s2 += BS) gp(p.cache_tags)[(size_t)blockIdx.x * p.cache_cap + s2] = tags[s2];
  }
}

// One problem at a = 0 (which the solvers start from): f = -y; exchange words and control block cleared.
__device__ __forceinline__ void init_problem(const Prob &P, int64_t i0, int64_t stride) {
  for (int64_t j = i0; j < P.n; j += stride) P.f[j] = -(double)label_of(P, j);
  for (int64_t q = i0; q < 2 * (int64_t)P.nwg * SLOT_WORDS; q += stride) P.slots[q] = 0ull;
  if (P.slots2)
    for (int64_t q = i0; q < 2 * (int64_t)P.ng * SLOT_WORDS; q += stride) P.slots2[q] = 0ull;
  if (i0 == 0) {
    P.ctl->t = 0;
    P.ctl->status = ST_RUNNING;
    P.ctl->b_up = 0.0;
    P.ctl->b_low = 0.0;
    P.ctl->u = -1;
    P.ctl->l = -1;
  }
}

__global__ void smo_init(const Prob *probs) {
  const Prob P = probs[blockIdx.y];
  init_problem(P, blockIdx.x * (int64_t)blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// Is any of the count values at X not finite?  (16 bytes a load, at any alignment.)
__device__ __forceinline__ bool any_nonfinite(const float *__restrict__ X, int64_t count, int64_t i0, int64_t stride) {
  typedef unsigned u4 __attribute__((ext_vector_type(4), aligned(4)));
  bool bad = false;
  const auto test = [&](unsigned u) { bad |= (u & 0x7f800000u) == 0x7f800000u; };
#pragma unroll 4
  for (int64_t i = i0; i < count / 4; i += stride) {
    const u4 v = *reinterpret_cast<const u4 *>(X + 4 * i);
    test(v[0]);
    test(v[1]);
    test(v[2]);
    test(v[3]);
  }
  for (int64_t i = count / 4 * 4 + i0; i < count; i += stride) test(__builtin_bit_cast(unsigned, X[i]));
  return bad;
}

// Everything a binary training needs before its kernels: the descriptor and the workgroup table
// written, the state initialised, the labels counted and checked, and (count > 0) X checked.
__global__ void __launch_bounds__(256) train_prep_k(Prob P, Prob *dprob, int32_t *wgp, int32_t nwgp,
                                                    const float *__restrict__ X, int64_t count, InputCheck *chk) {
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  if (i0 == 0) {
    *dprob = P;
    chk->both = 1;
  }
  for (int64_t q = i0; q < nwgp; q += stride) wgp[q] = 0;
  int64_t pos = 0, neg = 0;
  int bad = 0;
  for (int64_t j = i0; j < P.n; j += stride) {
    const int32_t y = P.y[j];
    pos += y == 1;
    neg += y == -1;
    if (y != 1 && y != -1) bad = max(bad, (int)(0x7fffffff - j));
  }
  for (int o = 32; o > 0; o >>= 1) {
    pos += __shfl_xor(pos, o);
    neg += __shfl_xor(neg, o);
    bad = max(bad, __shfl_xor(bad, o));
  }
  __shared__ int64_t rp[4], rn[4];
  __shared__ int rb[4];
  if ((threadIdx.x & 63) == 0) {
    rp[threadIdx.x >> 6] = pos;
    rn[threadIdx.x >> 6] = neg;
    rb[threadIdx.x >> 6] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // one atomic of each kind a workgroup: they all meet in one line
    pos = (rp[0] + rp[1]) + (rp[2] + rp[3]);
    neg = (rn[0] + rn[1]) + (rn[2] + rn[3]);
    bad = max(max(rb[0], rb[1]), max(rb[2], rb[3]));
    if (pos) atomicAdd(reinterpret_cast<u64 *>(&chk->pos), (u64)pos);
    if (neg) atomicAdd(reinterpret_cast<u64 *>(&chk->neg), (u64)neg);
    if (bad) atomicMax(&chk->bad_label, bad);
  }
  init_problem(P, i0, stride);
  if (any_nonfinite(X, count, i0, stride)) chk->nonfinite = 1;
}

__global__ void __launch_bounds__(256) nonfinite_k(const float *__restrict__ X, int64_t count, InputCheck *chk) {
  if (any_nonfinite(X, count, blockIdx.x * (int64_t)blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x))
    chk->nonfinite = 1;
}

constexpr int FBS = 256;

// Workgroups that finalize a problem of n samples.
__host__ __device__ inline int finalize_blocks(int64_t n) {
  const int64_t b = (n + 4 * FBS - 1) / (4 * FBS);
  return b > FINALIZE_BLOCKS_MAX ? FINALIZE_BLOCKS_MAX : b < 1 ? 1 : (int)b;
}

// Per problem that is not running any more: out[4p+0] = sum a, out[4p+1] = sum a y f, out[4p+2] =
// #(a>0), out[4p+3] = #(a>=C).  Each workgroup sums its share into part; the one that finds the
// others done (ticket, left at 0 again) adds the shares up in order.  100,000 samples: 15 us,
// against 184 us in one workgroup.
__global__ void __launch_bounds__(FBS) smo_finalize(const Prob *probs, double C, double *part, int32_t *ticket, double *out) {
  const int pid = blockIdx.y;
  const Prob P = probs[pid];
  const int blocks = finalize_blocks(P.n);
  if ((int)blockIdx.x >= blocks || P.ctl->status == ST_RUNNING) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t j = (int64_t)blockIdx.x * FBS + threadIdx.x; j < P.n; j += (int64_t)blocks * FBS) {
    const double aj = P.alpha[j];
    s[0] += aj;
    s[1] += aj * (double)label_of(P, j) * P.f[j];
    s[2] += aj > 0.0 ? 1.0 : 0.0;
    s[3] += aj >= C ? 1.0 : 0.0;
  }
  __shared__ double red[4][FBS / 64];
  __shared__ int last;
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] += __shfl_xor(s[c], o);
  if ((threadIdx.x & 63) == 0)
    for (int c = 0; c < 4; ++c) red[c][threadIdx.x >> 6] = s[c];
  __syncthreads();
  part += (int64_t)pid * FINALIZE_BLOCKS_MAX * 4;
  double v = 0.0;
  if (threadIdx.x < 4) {
    for (int q = 0; q < FBS / 64; ++q) v += red[threadIdx.x][q];
    if (blocks > 1) st_word(reinterpret_cast<u64 *>(part) + blockIdx.x * 4 + threadIdx.x, (u64)__double_as_longlong(v));
  }
  if (blocks > 1) {
    // The words are written and read at agent scope, so the ticket only has to follow the words of
    // its wave (waiting for them does it; a fence would write back a whole L2, 48 us for the 45
    // pairs of 12,000 samples).
    if (threadIdx.x < 64) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(gp(&ticket[pid]), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == blocks - 1;
    }
    __syncthreads();
    if (!last) return;
    v = 0.0;
    if (threadIdx.x < 4)
      for (int q = 0; q < blocks; ++q)
        v += __longlong_as_double((long long)ld_word(reinterpret_cast<const u64 *>(part) + q * 4 + threadIdx.x));
    if (threadIdx.x == 0) __hip_atomic_store(gp(&ticket[pid]), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x < 4) out[4 * (int64_t)pid + threadIdx.x] = v;
}

hipError_t launch_train_prep(const Prob &P, Prob *dprob, int32_t *wgp, int32_t nwgp, const float *X, int64_t count,
                             InputCheck *chk, hipStream_t s) {
  int64_t bx = (P.n + 1023) / 1024;
  if (bx < (count + 4095) / 4096) bx = (count + 4095) / 4096;
  if (bx > 4096) bx = 4096;
  hipLaunchKernelGGL(train_prep_k, dim3((unsigned)bx), dim3(256), 0, s, P, dprob, wgp, nwgp, X, count, chk);
  return hipGetLastError();
}

hipError_t launch_check_finite(const float *X, int64_t count, InputCheck *chk, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  int64_t bx = (count + 4095) / 4096;
  if (bx > 4096) bx = 4096;
  hipLaunchKernelGGL(nonfinite_k, dim3((unsigned)bx), dim3(256), 0, s, X, count, chk);
  return hipGetLastError();
}

hipError_t launch_solver_init(const Prob *probs, int32_t nprob, int64_t max_n, hipStream_t s) {
  int64_t bx = (max_n + 255) / 256;
  if (bx < 1) bx = 1;
  if (bx > 4096) bx = 4096;
  hipLaunchKernelGGL(smo_init, dim3((unsigned)bx, (unsigned)nprob), dim3(256), 0, s, probs);
  return hipGetLastError();
}

int64_t finalize_scratch_bytes(int64_t max_n, int32_t nprob) {
  return finalize_blocks(max_n) > 1 ? 32LL * FINALIZE_BLOCKS_MAX * nprob : 0;
}

hipError_t launch_finalize(const Prob *probs, int32_t nprob, int64_t max_n, double C, double *part, int32_t *ticket,
                           double *out, hipStream_t s) {
  hipLaunchKernelGGL(smo_finalize, dim3((unsigned)finalize_blocks(max_n), (unsigned)nprob), dim3(FBS), 0, s, probs, C,
                     part, ticket, out);
  return hipGetLastError();
}

static int row_kind(const SolveParams &p) { return row_kind_of(p.X, p.d); }

// Dynamic LDS of the row path: the fp64 dot products [2][per_wg], the cache tags, then `res`
// resident rows of d floats from a 16-byte boundary.
static size_t row_path_lds(const SolveParams &p, int64_t res) {
  const int64_t head = (16 * (int64_t)p.max_per_wg + 4 * (int64_t)p.cache_cap + 15) & ~(int64_t)15;
  return (size_t)(head + 4 * res * row_lds_pitch(p.d, row_kind(p)));
}

// Row path, float4 lanes with 8 samples a thread: there batches of two samples spill registers.
// For lane groups of up to 8 lanes (rows of up to 128 features) batches of one are faster
// (1,000,000 x 16: 25.8 -> 17.5 us a step; 1,000,000 x 64: 55.0 -> 46.0; 600,000 x 128: 55.2 ->
// 49.1); for wider groups the loads one batch keeps in flight matter more than the spill
// (batches of one: 600,000 x 256 115 -> 120 us, x 512 214 -> 238, x 784 326 -> 362).  Units at any
// address take the same line, which has not been measured for them; they spill more (with 8 samples a
// thread and batches of two 164 bytes a lane against 128, with 4 samples 48 against 12).
static bool row_batch_one(const SolveParams &p, int32_t per_thread) {
  return per_thread == 8 && row_kind(p) != ROW_SCALAR && group_size_for(p.d, row_kind(p)) <= 8;
}

template <int BS, int PER, bool GRAM, int V, bool ONE = false, bool SO = false>
static const void *kernel_of() {
  return reinterpret_cast<const void *>(&smo_solve<BS, PER, GRAM, V, ONE, SO>);
}

// The solver variant for a path, samples per thread, (row path) the kind of units and batches of
// one, (Gram path) the second-order rule; NULL if none.
static const void *solver_kernel(bool gram, int32_t per_thread, int kind, bool one = false, bool so = false) {
  if (gram && so) {
    switch (per_thread) {
      case 1: return kernel_of<BS_GRAM, 1, true, 0, false, true>();
      case 2: return kernel_of<BS_GRAM, 2, true, 0, false, true>();
      case 4: return kernel_of<BS_GRAM, 4, true, 0, false, true>();
      case 8: return kernel_of<BS_GRAM, 8, true, 0, false, true>();
      case 16: return kernel_of<BS_GRAM, 16, true, 0, false, true>();
      default: return nullptr;
    }
  }
  if (gram) {
    switch (per_thread) {
      case 1: return kernel_of<BS_GRAM, 1, true, 0>();
      case 2: return kernel_of<BS_GRAM, 2, true, 0>();
      case 4: return kernel_of<BS_GRAM, 4, true, 0>();
      case 8: return kernel_of<BS_GRAM, 8, true, 0>();
      case 16: return kernel_of<BS_GRAM, 16, true, 0>();
      default: return nullptr;
    }
  }
  switch (per_thread * 4 + kind) {
    case 1 * 4 + ROW_SCALAR: return kernel_of<BS_ROWS, 1, false, ROW_SCALAR>();
    case 1 * 4 + ROW_F4: return kernel_of<BS_ROWS, 1, false, ROW_F4>();
    case 1 * 4 + ROW_F4U: return kernel_of<BS_ROWS, 1, false, ROW_F4U>();
    case 2 * 4 + ROW_SCALAR: return kernel_of<BS_ROWS, 2, false, ROW_SCALAR>();
    case 2 * 4 + ROW_F4: return kernel_of<BS_ROWS, 2, false, ROW_F4>();
    case 2 * 4 + ROW_F4U: return kernel_of<BS_ROWS, 2, false, ROW_F4U>();
    case 4 * 4 + ROW_SCALAR: return kernel_of<BS_ROWS, 4, false, ROW_SCALAR>();
    case 4 * 4 + ROW_F4: return kernel_of<BS_ROWS, 4, false, ROW_F4>();
    case 4 * 4 + ROW_F4U: return kernel_of<BS_ROWS, 4, false, ROW_F4U>();
    case 8 * 4 + ROW_SCALAR: return kernel_of<BS_ROWS, 8, false, ROW_SCALAR>();
    case 8 * 4 + ROW_F4: return one ? kernel_of<BS_ROWS, 8, false, ROW_F4, true>()
                              : kernel_of<BS_ROWS, 8, false, ROW_F4>();
    case 8 * 4 + ROW_F4U: return one ? kernel_of<BS_ROWS, 8, false, ROW_F4U, true>()
                              : kernel_of<BS_ROWS, 8, false, ROW_F4U>();
    default: return nullptr;
  }
}

// Workgroups of a kernel the current device holds at once; asked once per thread, kernel, LDS size
// and device (the answer does not change, and asking costs more than the launch).
hipError_t coresident_workgroups(const void *fn, int bs, size_t shmem, int *capacity) {
  struct Key {
    const void *fn;
    int dev, bs, capacity;
    size_t shmem;
  };
  static thread_local Key known[8] = {};
  static thread_local unsigned next = 0;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  for (const Key &k : known)
    if (k.fn == fn && k.dev == dev && k.bs == bs && k.shmem == shmem) {
      *capacity = k.capacity;
      return hipSuccess;
    }
  int cus = 0, per_cu = 0;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, bs, shmem);
  if (e != hipSuccess) return e;
  *capacity = per_cu * cus;
  known[next++ % 8] = Key{fn, dev, bs, *capacity, shmem};
  return hipSuccess;
}

hipError_t launch_solver(const SolveParams &p, int32_t total_wg, int32_t per_thread, bool gram, hipStream_t s,
                         int32_t *max_coresident) {
  if (p.second_order && !gram) return hipErrorInvalidValue;
  const void *fn = solver_kernel(gram, per_thread, gram ? 0 : row_kind(p), !gram && row_batch_one(p, per_thread),
                                 p.second_order != 0);
  if (!fn) return hipErrorInvalidValue;
  const int bs = gram ? BS_GRAM : BS_ROWS;
  const size_t shmem = gram ? 0 : row_path_lds(p, p.res_rows);
  if (shmem > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return e;
  }
  int capacity = 0;
  const hipError_t e = coresident_workgroups(fn, bs, shmem, &capacity);
  if (e != hipSuccess) return e;
  if (max_coresident) *max_coresident = capacity;
  if (total_wg <= 0) return hipSuccess;  // capacity query only
  if (total_wg > capacity) return hipErrorCooperativeLaunchTooLarge;
  SolveParams pp = p;
  void *args[] = {&pp};
  // problems of one workgroup each exchange nothing, so they need not run at once
  if (p.alone) return hipLaunchKernel(fn, dim3((unsigned)total_wg), dim3(bs), args, shmem, s);
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)total_wg), dim3(bs), args, (unsigned)shmem, s);
}

int64_t solver_res_rows_max(const SolveParams &p, int32_t per_thread) {
  int dev = 0, max_lds = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -1;
  if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return -1;
  const void *fn = solver_kernel(false, per_thread, row_kind(p), row_batch_one(p, per_thread));
  if (!fn) return -1;
  hipFuncAttributes attr;
  if (hipFuncGetAttributes(&attr, fn) != hipSuccess) return -1;
  const int64_t avail = (int64_t)max_lds - (int64_t)attr.sharedSizeBytes - (int64_t)row_path_lds(p, 0);
  return avail > 0 ? avail / (4 * row_lds_pitch(p.d, row_kind(p))) : 0;
}

}  // namespace svmx
