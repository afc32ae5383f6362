// split_rows.hpp -- splitting rows of X into scaled fp16 halves (the layout of SplitX), shared by
// the Gram build and predict.
#pragma once

#include "common.hpp"

#include <math.h>

namespace svmx {

// Rows to split: `count` positions of X into s, gs lanes a row (a power of two covering the row's
// chunks of 8 features, at most 64).
struct SplitRows {
  const float *X;
  int64_t count;
  SplitX s;
  int32_t gs;
  const int32_t *perm;  // position pos of s is row perm[pos] of X (NULL: the row itself)
  InputCheck *chk;      // its nonfinite is set where a row read holds a value that is not finite
};

inline SplitRows split_rows_of(const float *X, int64_t count, const SplitX &s) {
  SplitRows r;
  r.X = X;
  r.count = count;
  r.s = s;
  r.perm = nullptr;
  r.chk = nullptr;
  r.gs = 1;
  while (r.gs < 64 && (int64_t)r.gs * 8 < s.dp) r.gs <<= 1;
  return r;
}

// Workgroups of 256 threads that split_rows_block wants for them.
inline int64_t split_rows_blocks(const SplitRows &r) {
  const int64_t per = 256 / r.gs, b = (r.count + per - 1) / per;
  return b > 8192 ? 8192 : b;
}

typedef _Float16 split_h8 __attribute__((ext_vector_type(8)));
typedef float split_f4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int SPLIT_KEEP = 4;

__device__ __forceinline__ void split_chunk_load(const float *__restrict__ x, int64_t d, int64_t k, float (&v)[8]) {
  if (k + 8 <= d) {
    const split_f4u a = *reinterpret_cast<const split_f4u *>(x + k), b = *reinterpret_cast<const split_f4u *>(x + k + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = a[e];
      v[4 + e] = b[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = k + e < d ? x[k + e] : 0.f;
  }
}

__device__ __forceinline__ void split_chunk_store(_Float16 *__restrict__ row, int64_t k, float inv, const float (&v)[8]) {
  split_h8 h, l;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float w = v[e] * inv;  // exact (power of two)
    h[e] = (_Float16)w;
    l[e] = (_Float16)(w - (float)h[e]);  // w - h is exact in fp32
  }
  _Float16 *p = row + (k >> 5) * 64 + (k & 31);
  *reinterpret_cast<split_h8 *>(p) = h;
  *reinterpret_cast<split_h8 *>(p + 32) = l;
}

// s = 2^e with max|x| < 2^e, h = fp16(x / s), l = fp16(x / s - h), and the norm |x|^2 as an fp64
// sum rounded to fp32, for every position of p: row_of(pos) is its row of X and of p.s, or
// negative to leave it out (called by all lanes of the wave, pos the same in the gs lanes of a
// row and -1 past the end).  Each lane reads 8 consecutive features at once (two 16-byte loads,
// whatever the alignment of the row) and writes 16 bytes of each half; up to SPLIT_KEEP chunks a
// lane stay in registers between the two passes.  Bound by reading X and writing as many bytes
// (20,000 x 784: 20 us, against 34 us with one feature a lane and 2-byte stores).
// Block `block` of `blocks` workgroups of 256 threads.
template <class RowOf>
__device__ __forceinline__ void split_rows_block(const SplitRows &p, int64_t d, int64_t block, int64_t blocks,
                                                 RowOf row_of) {
  const int gs = p.gs, per = 256 / gs;
  const int g = threadIdx.x & (gs - 1), mine = threadIdx.x / gs;
  const int chunks = (int)(p.s.dp >> 3);
  // every lane of a wave runs the same number of rounds (the reductions cross lanes)
  for (int64_t r0 = block * per; r0 < p.count; r0 += blocks * per) {
    const int64_t r = row_of(r0 + mine < p.count ? r0 + mine : -1);
    const bool in = r >= 0;
    const float *x = p.X + (in ? (p.perm ? (int64_t)p.perm[r] : r) : 0) * d;
    float v[SPLIT_KEEP][8];
    float m = 0.f;
    double q = 0.0;
    auto take = [&](const float (&c)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        m = fmaxf(m, fabsf(c[e]));
        q = __builtin_fma((double)c[e], (double)c[e], q);
      }
    };
    if (in) {
#pragma unroll
      for (int i = 0; i < SPLIT_KEEP; ++i)
        if (g + i * gs < chunks) split_chunk_load(x, d, 8 * (int64_t)(g + i * gs), v[i]);
#pragma unroll
      for (int i = 0; i < SPLIT_KEEP; ++i)
        if (g + i * gs < chunks) take(v[i]);
      for (int c = g + SPLIT_KEEP * gs; c < chunks; c += gs) {
        float w[8];
        split_chunk_load(x, d, 8 * (int64_t)c, w);
        take(w);
      }
    }
    for (int o = gs >> 1; o > 0; o >>= 1) {
      m = fmaxf(m, __shfl_xor(m, o));
      q += __shfl_xor(q, o);
    }
    if (!in) continue;
    int e = 0;
    if (m > 0.f) (void)frexpf(m, &e);  // m = f 2^e, f in [0.5, 1)
    const float inv = ldexpf(1.0f, -e);
    _Float16 *row = p.s.rows + r * 2 * p.s.dp;
#pragma unroll
    for (int i = 0; i < SPLIT_KEEP; ++i)
      if (g + i * gs < chunks) split_chunk_store(row, 8 * (int64_t)(g + i * gs), inv, v[i]);
    for (int c = g + SPLIT_KEEP * gs; c < chunks; c += gs) {
      float w[8];
      split_chunk_load(x, d, 8 * (int64_t)c, w);
      split_chunk_store(row, 8 * (int64_t)c, inv, w);
    }
    if (g == 0) {
      p.s.scale[r] = ldexpf(1.0f, e);
      p.s.nrm[r] = (float)q;
      // squares of finite floats do not overflow an fp64 sum
      if (p.chk && !__builtin_isfinite(q)) p.chk->nonfinite = 1;
    }
  }
}

}  // namespace svmx
