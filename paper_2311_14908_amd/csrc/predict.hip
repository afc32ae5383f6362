// predict.hip -- decision values d(x) = sum_{a_i>0} a_i y_i K(x_i, x) - b and one-vs-one votes.
//
// 1. predict_prep: in one launch, the support vectors (a_i > 0) of every problem in increasing
//    local index, as rows of X with coefficient a_i y_i (chunks of samples, each counting the
//    support vectors before it; deterministic order), and the split-fp16 rows of the test samples
//    and of the training rows that are a support vector of some problem.
// 2. predict_f16x3: 128 support vectors x 128 test samples per tile; the contraction runs on
//    v_mfma_f32_16x16x32_f16 over the split rows, as in the Gram build (split_tile.hpp), K =
//    exp2(c * max(0, |t|^2 + |x|^2 - 2 t.x)) with c = -gamma log2(e), and each lane adds coef * K
//    of its support vectors in fp64 to the sums of its four test samples.  Support-vector tiles
//    are split over `nsplit` workgroups per test tile; each split writes its own partial sums.
//    `gram_mfma = SVM_MFMA_F32` takes predict_mfma instead: v_mfma_f32_16x16x4f32, fp32 in, norms
//    from the same LDS slabs.
// 3. predict_final: dec = sum over splits (fixed order) - b, and the one-vs-one votes.
// Few test samples (few_rule.hpp) take one pass over the training rows (predict_few) in place of all
// of these.
// Results are deterministic: no atomics touch values.
#include "split_rows.hpp"
#include "split_tile.hpp"

#include <math.h>

namespace svmx {

constexpr int PT = 128;        // tile edge
constexpr int PKC = 16;        // k per LDS stage
constexpr int PPAD = PT + 16;  // LDS pitch (conflict-free operand reads)
constexpr int PBS = 256;

__device__ __forceinline__ int64_t pm_pos(const PredPair &m, int64_t j) {
  return j < m.len0 ? m.off0 + j : m.off1 + (j - m.len0);
}

// Samples a compaction workgroup handles: every workgroup counts the support vectors before its
// chunk itself (no second launch, no flags), so at most 64 of them per problem keep that linear in
// ntr: 50,000 samples 9 us under the rows' splitting, where one workgroup walking them all took
// 70 us on its own.
constexpr int COMPACT_MIN = 1024;

__host__ __device__ inline int64_t compact_chunk(int64_t ntr) {
  const int64_t c = (ntr + 63) / 64;
  return c < COMPACT_MIN ? COMPACT_MIN : (c + PBS - 1) / PBS * PBS;
}

struct PrepParams {
  const double *alpha;
  const PredPair *pairs;  // [npairs], or NULL: the one problem is `one`
  PredPair one;
  int32_t npairs;
  int32_t compact_blocks;  // per problem (blocks past a problem's samples leave)
  int32_t *sv_row;
  double *sv_coef;
  int64_t *count;
  int64_t d;
  SplitRows test, train;  // rows to split: all test rows; training positions 0 .. n-1
  const int32_t *perm;    // training position -> row (NULL: the same)
  int32_t all_train;      // split every training row, not only support vectors
  int32_t test_blocks;
};

__device__ __forceinline__ PredPair pair_of(const PredPair *pairs, const PredPair &one, int p) {
  return pairs ? pairs[p] : one;
}

// Sum of v over the workgroup, to every thread.
__device__ __forceinline__ int64_t block_sum(int v, int *red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if (lane == 0) red[w] = v;
  __syncthreads();
  int64_t s = 0;
  for (int q = 0; q < PBS / 64; ++q) s += red[q];
  __syncthreads();
  return s;
}

// Chunk `blk` of one problem's samples: its support vectors to their places.
__device__ __forceinline__ void compact_block(const PrepParams &p, int pid, int64_t blk, int *red) {
  const PredPair map = pair_of(p.pairs, p.one, pid);
  const double *alpha = p.alpha + map.alpha_off;
  const int64_t n = map.ntr, chunk = compact_chunk(n);
  const int64_t c0 = blk * chunk, c1 = min(n, c0 + chunk);
  if (c0 >= n) return;
  int32_t *sv_row = p.sv_row + map.sv_off;
  double *sv_coef = p.sv_coef + map.sv_off;
  int before = 0;
#pragma unroll 16
  for (int64_t j = threadIdx.x; j < c0; j += PBS) before += alpha[j] > 0.0 ? 1 : 0;
  int64_t base = block_sum(before, red);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int64_t j0 = c0; j0 < c1; j0 += PBS) {
    const int64_t j = j0 + threadIdx.x;
    const double a = j < c1 ? alpha[j] : 0.0;
    const bool sv = a > 0.0;
    const unsigned long long mask = __ballot(sv);
    if (lane == 0) red[w] = __popcll(mask);
    __syncthreads();
    int off = __popcll(mask & ((1ull << lane) - 1ull)), tot = 0;
#pragma unroll
    for (int q = 0; q < PBS / 64; ++q) {
      off += q < w ? red[q] : 0;
      tot += red[q];
    }
    if (sv) {
      const int64_t pos = pm_pos(map, j);
      const int64_t row = map.perm ? (int64_t)map.perm[pos] : pos;
      const double y = map.y ? (double)map.y[row] : (j < map.len0 ? 1.0 : -1.0);
      sv_row[base + off] = (int32_t)row;
      sv_coef[base + off] = a * y;
    }
    base += tot;
    __syncthreads();
  }
  if (c1 == n && threadIdx.x == 0) p.count[pid] = base;
}

// Is training position pos a support vector of some problem?  Wave-uniform pos; lane p looks at
// problem p (at most 64).
__device__ __forceinline__ bool any_sv(const PrepParams &p, int64_t pos) {
  const int lane = threadIdx.x & 63;
  bool sv = false;
  if (lane < p.npairs) {
    const PredPair m = pair_of(p.pairs, p.one, lane);
    int64_t j = -1;
    if (pos >= m.off0 && pos < m.off0 + m.len0) j = pos - m.off0;
    else if (pos >= m.off1 && pos < m.off1 + (m.ntr - m.len0)) j = m.len0 + (pos - m.off1);
    sv = j >= 0 && p.alpha[m.alpha_off + j] > 0.0;
  }
  return __ballot(sv) != 0;
}

// Blocks: the compaction (npairs x compact_blocks), the test rows, the training rows.
__global__ void __launch_bounds__(PBS) predict_prep_k(PrepParams p) {
  __shared__ int red[PBS / 64];
  int64_t b = blockIdx.x;
  const int64_t nc = (int64_t)p.npairs * p.compact_blocks;
  if (b < nc) {
    compact_block(p, (int)(b / p.compact_blocks), b % p.compact_blocks, red);
    return;
  }
  b -= nc;
  if (b < p.test_blocks) {
    split_rows_block(p.test, p.d, b, p.test_blocks, [](int64_t pos) { return pos; });
    return;
  }
  b -= p.test_blocks;
  const int lane = threadIdx.x & 63;
  split_rows_block(p.train, p.d, b, (int64_t)gridDim.x - nc - p.test_blocks, [&](int64_t pos) -> int64_t {
    const int64_t row = p.perm && pos >= 0 ? (int64_t)p.perm[pos] : pos;
    if (p.all_train) return row;
    if (p.npairs == 1) {
      const PredPair m = pair_of(p.pairs, p.one, 0);
      return pos >= 0 && p.alpha[m.alpha_off + pos] > 0.0 ? row : -1;
    }
    // the wave's rows one after the other: lane -> problem
    bool need = false;
    for (int l = 0; l < 64; l += p.train.gs) {
      const int64_t q = ((int64_t)__builtin_amdgcn_readlane((int)(pos >> 32), l) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)pos, l);
      const bool sv = q >= 0 && any_sv(p, q);
      if (lane >= l && lane < l + p.train.gs) need = sv;
    }
    return need ? row : -1;
  });
}

// Load 128 rows x 16 columns into LDS transposed to [k][row] and add the squares into the
// thread's norm partials (thread t: rows t/4 and 64 + t/4, columns 4*(t%4) .. +3).  Rows come
// from `idx` (row numbers of X) when given, else r0.. directly; rows at or past `nrows` are 0.
template <bool VEC4>
__device__ __forceinline__ void load_rows(const float *__restrict__ X, const int32_t *__restrict__ idx, int64_t nrows,
                                          int64_t d, int64_t r0, int64_t k0, float (*S)[PPAD], float nacc[2]) {
  const int t = threadIdx.x;
  const int kq = (t & 3) * 4;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = h * 64 + (t >> 2);
    const int64_t r = r0 + row;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (r < nrows) {
      const int64_t xr = idx ? (int64_t)idx[r] : r;
      const float *src = X + xr * d + k0 + kq;
      if (VEC4 && k0 + kq + 3 < d) {
        const float4 q = *reinterpret_cast<const float4 *>(src);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (k0 + kq + e < d) v[e] = src[e];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      S[kq + e][row] = v[e];
      nacc[h] += v[e] * v[e];
    }
  }
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
  const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sum over the 16 lanes of a DPP row; every lane of the row gets the same bits.
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_d<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_d<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_d<0x141>(v);  // row_half_mirror
  v += dpp_d<0x140>(v);  // row_mirror
  return v;
}

// Workgroup (x, y, z): test rows 128 x .. +128, split y of problem z's support-vector tiles.
template <bool VEC4>
__global__ void __launch_bounds__(PBS) predict_mfma_k(const float *__restrict__ T, int64_t m, const float *__restrict__ X,
                                                      const PredPair *__restrict__ pairs, PredPair one,
                                                      const int32_t *__restrict__ sv_row_all,
                                                      const double *__restrict__ sv_coef_all,
                                                      const int64_t *__restrict__ sv_count, int64_t d, float c,
                                                      double *__restrict__ part_all) {
  const PredPair pp = pair_of(pairs, one, blockIdx.z);
  const int nsplit = pp.nsplit;
  if ((int)blockIdx.y >= nsplit) return;
  const int32_t *sv_row = sv_row_all + pp.sv_off;
  const double *sv_coef = sv_coef_all + pp.sv_off;
  double *part = part_all + pp.part_off;
  __shared__ float As[PKC][PPAD];
  __shared__ float Bs[PKC][PPAD];
  __shared__ float nA[PT], nB[PT];
  __shared__ double cB[PT];
  __shared__ double rs[2][PT];
  const int64_t nsv = sv_count[blockIdx.z];
  const int64_t q0 = (int64_t)blockIdx.x * PT;
  const int split = blockIdx.y;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wm = w >> 1, wn = w & 1;
  double row_acc = 0.0;  // thread t < 128 owns test row q0 + t
  const int64_t ntile = (nsv + PT - 1) / PT;
  for (int64_t st = split; st < ntile; st += nsplit) {
    const int64_t s0 = st * PT;
    v4f acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = (v4f){0.f, 0.f, 0.f, 0.f};
    float na[2] = {0.f, 0.f}, nb[2] = {0.f, 0.f};
    for (int64_t k0 = 0; k0 < d; k0 += PKC) {
      load_rows<VEC4>(T, nullptr, m, d, q0, k0, As, na);
      load_rows<VEC4>(X, sv_row + s0, nsv - s0, d, 0, k0, Bs, nb);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < PKC; kk += 4) {
        float av[4], bv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) av[q] = As[kk + (lane >> 4)][wm * 64 + q * 16 + (lane & 15)];
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[q] = Bs[kk + (lane >> 4)][wn * 64 + q * 16 + (lane & 15)];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
      }
      __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      na[h] += __shfl_xor(na[h], 1);
      na[h] += __shfl_xor(na[h], 2);
      nb[h] += __shfl_xor(nb[h], 1);
      nb[h] += __shfl_xor(nb[h], 2);
    }
    if ((threadIdx.x & 3) == 0) {
      nA[threadIdx.x >> 2] = na[0];
      nA[64 + (threadIdx.x >> 2)] = na[1];
      nB[threadIdx.x >> 2] = nb[0];
      nB[64 + (threadIdx.x >> 2)] = nb[1];
    }
    if (threadIdx.x < PT) cB[threadIdx.x] = s0 + threadIdx.x < nsv ? sv_coef[s0 + threadIdx.x] : 0.0;
    __syncthreads();
    // per test row: sum over this wave's 64 columns (4 blocks x 16 lanes), then the two halves
#pragma unroll
    for (int a = 0; a < 4; ++a) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int lr = wm * 64 + a * 16 + 4 * (lane >> 4) + e;
        double sacc = 0.0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int lc = wn * 64 + b * 16 + (lane & 15);
          float t = nA[lr] + nB[lc] - 2.0f * acc[a][b][e];
          t = t > 0.f ? t : 0.f;
          sacc = __builtin_fma(cB[lc], (double)__builtin_amdgcn_exp2f(c * t), sacc);
        }
        sacc = row16_sum(sacc);
        if ((lane & 15) == 0) rs[wn][lr] = sacc;
      }
    }
    __syncthreads();
    if (threadIdx.x < PT) row_acc += rs[0][threadIdx.x] + rs[1][threadIdx.x];
    __syncthreads();
  }
  if (threadIdx.x < PT && q0 + threadIdx.x < m) part[(int64_t)split * m + q0 + threadIdx.x] = row_acc;
}

struct PredCols {
  alignas(16) float s[PT], n[PT];  // scales and norms of a tile's support vectors
  alignas(16) double c[PT];        // coefficients (0 past the end)
};

// predict on the split rows: the support vectors (gathered through sv_row; past the end the last
// one again, with coefficient 0) are the row operand, the test samples the columns, so a lane
// holds 16 support vectors of each of 4 test samples and adds them up by itself, over all tiles
// of its split; lanes meet once, at the end.  (With the roles exchanged every tile needed 16
// sums over 16 lanes.)  Short rows are bound by this epilogue's vector instructions (an exp2, a
// conversion, an fp64 multiply-add and five fp32 ones an entry: about as long as the products of
// 128 features), long ones by the matrix cores.  Three workgroups a CU: 168 registers, and 10 more
// spilled (44 bytes a lane, not in the stage loop).  10,000 x 15,000 x 784: 0.56 ms, 1,280 TFLOP/s of
// fp16 work (1.24 ms before); 4,097 x 30,000 x 127: 131 us (202 us; without the next tile's first stage
// and rows read ahead 140 us).
__global__ void __launch_bounds__(PBS, 3) predict_f16x3_k(SplitX st, int64_t m, SplitX sx,
                                                       const PredPair *__restrict__ pairs, PredPair one, int32_t npairs,
                                                       const int32_t *__restrict__ sv_row_all,
                                                       const double *__restrict__ sv_coef_all,
                                                       const int64_t *__restrict__ sv_count, float c, int32_t nrt,
                                                       double *__restrict__ part_all) {
  __shared__ SplitStage S;
  __shared__ PredCols cols[2];  // this tile's support vectors and the next one's
  __shared__ int rows[2][PT];   // their rows of X, one tile further ahead
  __shared__ float sB[PT], nB[PT];
  __shared__ double sums[4][PBS];  // each lane's four sums (kept here, not in registers, over the products)
  __shared__ int64_t ends[64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int kq = lane >> 4, r16 = lane & 15;
  // Items: for every problem, test tiles x the splits that have a tile, in the order (8 test
  // tiles) x splits x (groups of 8 test tiles).  Workgroup b runs on XCD b % 8 and takes items of
  // that XCD's contiguous share of them, so the workgroups an XCD holds at once share 8 slabs of
  // test rows and a dozen of support vectors in its L2.  ends[p]: the end
  // of problem p's items.
  if (w == 0) {
    int64_t end = 0;
    if (lane < npairs)
      end = (int64_t)nrt * min<int64_t>(pair_of(pairs, one, lane).nsplit, (sv_count[lane] + PT - 1) / PT);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t v = __shfl_up(end, o);
      if (lane >= o) end += v;
    }
    ends[lane] = end;
  }
  __syncthreads();
  const int64_t items = ends[63], share = (items + 7) / 8;
  for (int64_t i = blockIdx.x / 8; i < share; i += gridDim.x / 8) {
    const int64_t item = (blockIdx.x % 8) * share + i;
    if (item >= items) break;
    const int pid = __builtin_amdgcn_readfirstlane(__popcll(__ballot(ends[lane] <= item)));
    const PredPair pp = pair_of(pairs, one, pid);
    const int nsv = (int)sv_count[pid];  // at most n < 2^31 - 1
    const int ntile = (int)(((int64_t)nsv + PT - 1) / PT);
    const uint32_t used = min(pp.nsplit, ntile);
    const uint32_t lin = (uint32_t)(item - (pid > 0 ? ends[pid - 1] : 0));
    const uint32_t sup = lin / (8 * used), rem = lin - sup * 8 * used;
    const uint32_t wide = min(8u, (uint32_t)nrt - 8 * sup);
    const int split = __builtin_amdgcn_readfirstlane((int)(rem / wide));
    const int64_t q0 = (int64_t)__builtin_amdgcn_readfirstlane((int)(8 * sup + rem % wide)) * PT;
    const int32_t *sv_row = sv_row_all + pp.sv_off;
    const double *sv_coef = sv_coef_all + pp.sv_off;
    // While a tile's sums are added up, the first stage of the next tile is on its way; its
    // support vectors' rows were read a tile earlier, so nothing waits for a chain of loads.
    const auto row_at = [&](int tile) {  // row of support vector `threadIdx.x` of the tile, past the end the last one's
      const int q = min((int)threadIdx.x, nsv - 1 - tile * PT);
      return sv_row[tile * PT + q];
    };
    const char *src[SCH];  // waves 0 and 1 load the support vectors, 2 and 3 the test rows
    const auto aim = [&](const int (&r)[PT]) {
#pragma unroll
      for (int q = 0; q < SCH; ++q) {
        const int i = ((w & 1) * SCH + q) * 8 + (lane >> 3);
        src[q] = w < 2 ? split_src(sx, r[i]) : split_src(st, min<int64_t>(q0 + i, m - 1));
      }
    };
    int tile = split, buf = 0;
    if (threadIdx.x < PT) {
      const int r0 = row_at(tile), r1 = tile + pp.nsplit < ntile ? row_at(tile + pp.nsplit) : 0;
      const int64_t q = min<int64_t>(q0 + threadIdx.x, m - 1);
      sB[threadIdx.x] = -2.0f * st.scale[q];  // the test samples: -2 x the scale, and the norm
      nB[threadIdx.x] = st.nrm[q];
      rows[0][threadIdx.x] = r0;
      rows[1][threadIdx.x] = r1;
      cols[0].s[threadIdx.x] = sx.scale[r0];
      cols[0].n[threadIdx.x] = sx.nrm[r0];
      cols[0].c[threadIdx.x] = tile * PT + (int)threadIdx.x < nsv ? sv_coef[tile * PT + threadIdx.x] : 0.0;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) sums[b][threadIdx.x] = 0.0;
    __syncthreads();
    aim(rows[0]);
    split_stage_load(S, src);
    for (;;) {
      v4f acc[4][4];
      split_tile_loaded(S, src, st.dp / SKS, wm, wn, acc);
      const int next = tile + pp.nsplit;
      const bool more = next < ntile;
      float ns = 0.f, nn = 0.f;
      double nc = 0.0;
      int nr = 0;
      if (more) {
        aim(rows[buf ^ 1]);
        split_stage_load(S, src);
        if (threadIdx.x < PT) {
          const int r = rows[buf ^ 1][threadIdx.x];
          ns = sx.scale[r];
          nn = sx.nrm[r];
          nc = next * PT + (int)threadIdx.x < nsv ? sv_coef[next * PT + threadIdx.x] : 0.0;
          nr = next + pp.nsplit < ntile ? row_at(next + pp.nsplit) : 0;
        }
      }
      const PredCols &A = cols[buf];
      float sb[4], nb[4];
      double sum[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        sum[b] = sums[b][threadIdx.x];
        sb[b] = sB[wn * 64 + b * 16 + r16];
        nb[b] = nB[wn * 64 + b * 16 + r16];
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int lr = wm * 64 + a * 16 + 4 * kq;
        const v4f sa = *reinterpret_cast<const v4f *>(&A.s[lr]), na = *reinterpret_cast<const v4f *>(&A.n[lr]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double ca = A.c[lr + e];
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            // the scales are powers of two, so this is n_i + n_j - 2 s_i s_j acc with one rounding
            float t = __builtin_fmaf(acc[a][b][e] * sa[e], sb[b], na[e] + nb[b]);
            t = t > 0.f ? t : 0.f;
            sum[b] = __builtin_fma(ca, (double)__builtin_amdgcn_exp2f(c * t), sum[b]);
          }
        }
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) sums[b][threadIdx.x] = sum[b];
      if (!more) break;
      if (threadIdx.x < PT) {
        cols[buf ^ 1].s[threadIdx.x] = ns;
        cols[buf ^ 1].n[threadIdx.x] = nn;
        cols[buf ^ 1].c[threadIdx.x] = nc;
        rows[buf][threadIdx.x] = nr;
      }
      tile = next;
      buf ^= 1;
    }
    __syncthreads();
    // test sample t: column block b = t / 16 % 4 of the waves of its half, lanes t % 16 + 16 kq
    if (threadIdx.x < PT && q0 + threadIdx.x < m) {
      const int b = (threadIdx.x >> 4) & 3, col = threadIdx.x & 15, half = threadIdx.x >> 6;
      double r[2];
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const double *l = &sums[b][(2 * v + half) * 64 + col];
        r[v] = (l[0] + l[16]) + (l[32] + l[48]);
      }
      part_all[pp.part_off + (int64_t)split * m + q0 + threadIdx.x] = r[0] + r[1];
    }
    __syncthreads();  // sums, sB and nB are rewritten by the next item
  }
}

// A few test samples (at most FEW_MAX): a pass over the training rows instead of tiles of 128, most
// of whose columns would be empty, and neither the compaction nor the split rows first.  Workgroup
// (x, y, z): chunk x of problem y's samples, test samples MQ z .. MQ z + MQ - 1.  The chunk's
// support vectors are listed in LDS in index order; gs lanes take a row each (float4 positions g,
// g + gs, ..; the first FEW_POS positions of the test samples stay in registers), K = exp2(c |x -
// t|^2) from the fp32 differences, squared and summed in fp64 (in fp32 the roundings of features
// that are zero in most rows are the same for all of them and do not average out), and each row
// group adds coef * K in fp64.  Bound by launches and by reading the support vectors once, for more
// samples, and for many problems that share rows, by the fp64 sums.  few_rule.hpp says when it is
// taken.  Us a call of a binary prediction: one sample against 1,000 x 16 28 (35 by tiles), 8 against
// 5,000 x 100 37 (39), 1 against 20,000 x 784 49 (106), 16 against 20,000 x 784 76 (107), against 50,000 x
// 300 79 (116), against 50,000 x 8 44 (52); 32 against 20,000 x 784 take 124 (107).
constexpr int FEW_BS = 512, FEW_POS = 4;

// Chunks of a problem: about 8 rows for each row group to take one after the other; at most 64 and
// one per 128 samples, so never more than predict_splits().
__host__ __device__ inline int few_chunks(int64_t ntr, int gs) {
  const int64_t rows = 8 * (FEW_BS / gs) > 128 ? 8 * (FEW_BS / gs) : 128;
  const int64_t c = (ntr + rows - 1) / rows;
  return c > 64 ? 64 : c < 1 ? 1 : (int)c;
}

typedef float few_f4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ few_f4u few_load(const float *__restrict__ x, int64_t d, int64_t k) {
  if (k + 4 <= d) return *reinterpret_cast<const few_f4u *>(x + k);
  few_f4u v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (k + e < d) v[e] = x[k + e];
  return v;
}

// exp2(c d2), c d2 <= 0: exp2 of the fp32 part of the exponent, then the rest to first order.
__device__ __forceinline__ double rbf_of_d2(double c, double d2) {
  const double x2 = c * (d2 > 0.0 ? d2 : 0.0);
  const float hi = (float)x2, e2 = __builtin_amdgcn_exp2f(hi);
  return hi > -150.f ? (double)__builtin_fmaf(e2, 0.6931472f * (float)(x2 - (double)hi), e2) : 0.0;
}

template <int MQ>
__global__ void __launch_bounds__(FEW_BS) predict_few_k(const float *__restrict__ T, int64_t m, const float *__restrict__ X,
                                                        int64_t d, const double *__restrict__ alpha_all,
                                                        const PredPair *__restrict__ pairs, PredPair one, double c, int gs,
                                                        double *__restrict__ part_all, double *__restrict__ dec,
                                                        int64_t stride) {
  const PredPair map = pair_of(pairs, one, blockIdx.y);
  const double *alpha = alpha_all + map.alpha_off;
  const int chunks = few_chunks(map.ntr, gs);
  if ((int)blockIdx.x >= chunks) return;
  const int64_t per = (map.ntr + chunks - 1) / chunks;
  const int64_t c0 = blockIdx.x * per, c1 = min(map.ntr, c0 + per);
  __shared__ int32_t rows[FEW_BS];
  __shared__ double coefs[FEW_BS];
  __shared__ int cnt[FEW_BS / 64];
  __shared__ double sums[MQ][FEW_BS];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = threadIdx.x & (gs - 1), grp = threadIdx.x / gs, groups = FEW_BS / gs;
  const int64_t units = (d + 3) / 4, q0 = (int64_t)blockIdx.z * MQ;
  few_f4u t[MQ][FEW_POS];
#pragma unroll
  for (int q = 0; q < MQ; ++q) {
    const float *tr = T + min(q0 + q, m - 1) * d;
#pragma unroll
    for (int i = 0; i < FEW_POS; ++i)
      if (g + i * gs < units) t[q][i] = few_load(tr, d, 4 * (int64_t)(g + i * gs));
  }
  double sum[MQ];
#pragma unroll
  for (int q = 0; q < MQ; ++q) sum[q] = 0.0;
  for (int64_t j0 = c0; j0 < c1; j0 += FEW_BS) {
    const int64_t j = j0 + threadIdx.x;
    const double a = j < c1 ? alpha[j] : 0.0;
    const bool sv = a > 0.0;
    const unsigned long long mask = __ballot(sv);
    if (lane == 0) cnt[w] = __popcll(mask);
    __syncthreads();
    int off = __popcll(mask & ((1ull << lane) - 1ull)), nsv = 0;
    for (int q = 0; q < FEW_BS / 64; ++q) {
      off += q < w ? cnt[q] : 0;
      nsv += cnt[q];
    }
    if (sv) {
      const int64_t pos = pm_pos(map, j);
      const int64_t row = map.perm ? (int64_t)map.perm[pos] : pos;
      rows[off] = (int32_t)row;
      coefs[off] = a * (map.y ? (double)map.y[row] : (j < map.len0 ? 1.0 : -1.0));
    }
    __syncthreads();
    few_f4u v[FEW_POS], nv[FEW_POS];  // this row, and the next one on its way
    const auto fetch = [&](int r, few_f4u (&o)[FEW_POS]) {
      const float *x = X + (int64_t)rows[r] * d;
#pragma unroll
      for (int i = 0; i < FEW_POS; ++i)
        if (g + i * gs < units) o[i] = few_load(x, d, 4 * (int64_t)(g + i * gs));
    };
    if (grp < nsv) fetch(grp, nv);
    for (int r = grp; r < nsv; r += groups) {  // a row group is inside one wave
      const float *x = X + (int64_t)rows[r] * d;
#pragma unroll
      for (int i = 0; i < FEW_POS; ++i) v[i] = nv[i];
      if (r + groups < nsv) fetch(r + groups, nv);
      double s[MQ];
#pragma unroll
      for (int q = 0; q < MQ; ++q) s[q] = 0.0;
#pragma unroll
      for (int i = 0; i < FEW_POS; ++i)
        if (g + i * gs < units) {
#pragma unroll
          for (int q = 0; q < MQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double f = (double)(v[i][e] - t[q][i][e]);
              s[q] = __builtin_fma(f, f, s[q]);
            }
        }
      for (int64_t u = g + (int64_t)FEW_POS * gs; u < units; u += gs) {  // rows past 1,024 features
        const few_f4u xv = few_load(x, d, 4 * u);
#pragma unroll
        for (int q = 0; q < MQ; ++q) {
          const few_f4u tq = few_load(T + min(q0 + q, m - 1) * d, d, 4 * u);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const double f = (double)(xv[e] - tq[e]);
            s[q] = __builtin_fma(f, f, s[q]);
          }
        }
      }
      for (int o = gs >> 1; o > 0; o >>= 1)
#pragma unroll
        for (int q = 0; q < MQ; ++q) s[q] += __shfl_xor(s[q], o);
      const double coef = coefs[r];
#pragma unroll
      for (int q = 0; q < MQ; ++q) sum[q] = __builtin_fma(coef, rbf_of_d2(c, s[q]), sum[q]);
    }
    __syncthreads();  // rows, coefs and cnt are rewritten
  }
  // every lane of a row group holds the same sums: group grp's to place grp, added up in order
#pragma unroll
  for (int q = 0; q < MQ; ++q)
    if (g == 0) sums[q][grp] = sum[q];
  __syncthreads();
  for (int h = groups >> 1; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h)
#pragma unroll
      for (int q = 0; q < MQ; ++q) sums[q][threadIdx.x] += sums[q][threadIdx.x + h];
    __syncthreads();
  }
  const int q = threadIdx.x;
  if (q < MQ && q0 + q < m) {
    if (chunks == 1)
      dec[(q0 + q) * stride + blockIdx.y] = sums[q][0] - map.b;
    else
      part_all[map.part_off + (int64_t)blockIdx.x * m + q0 + q] = sums[q][0];
  }
}

// Sum of the chunks' partials in order, - the bias (problems of one chunk are done already).
__global__ void __launch_bounds__(64) predict_few_final_k(const double *__restrict__ part_all, int64_t m,
                                                          const PredPair *__restrict__ pairs, PredPair one, int gs,
                                                          double *dec, int64_t stride) {
  const PredPair pp = pair_of(pairs, one, blockIdx.x);
  const int chunks = few_chunks(pp.ntr, gs);
  if (chunks == 1 || (int)threadIdx.x >= m) return;
  const double *part = part_all + pp.part_off + threadIdx.x;
  double s = 0.0;
#pragma unroll 16
  for (int k = 0; k < chunks; ++k) s += part[k * m];
  dec[threadIdx.x * stride + blockIdx.x] = s - pp.b;
}

static hipError_t launch_predict_few(const PredictLaunch &L, hipStream_t s) {
  const PredPair *pairs = L.npairs > 1 ? L.ws.pairs : nullptr;
  int gs = 1;
  while (gs < 64 && 4LL * FEW_POS * gs < L.d) gs <<= 1;
  int chunks = 1;
  for (int32_t q = 0; q < L.npairs; ++q) {
    const int c = few_chunks(L.host_pairs[q].ntr, gs);
    chunks = c > chunks ? c : chunks;
  }
  const double c = -L.gamma * 1.4426950408889634;
  const auto go = [&](auto kernel, int mq) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)chunks, (unsigned)L.npairs, (unsigned)((L.m + mq - 1) / mq)), dim3(FEW_BS), 0,
                       s, L.T, L.m, L.Xtr, L.d, L.alpha, pairs, L.host_pairs[0], c, gs, L.ws.part, L.dec, L.dec_stride);
  };
  if (L.m == 1)
    go(predict_few_k<1>, 1);
  else
    go(predict_few_k<4>, 4);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || chunks == 1) return e;
  hipLaunchKernelGGL(predict_few_final_k, dim3((unsigned)L.npairs), dim3(64), 0, s, L.ws.part, L.m, pairs,
                     L.host_pairs[0], gs, L.dec, L.dec_stride);
  return hipGetLastError();
}

// dec[q * stride + p] = the sum of problem p's (blockIdx.y) split partials - its bias.  A split
// without a tile wrote nothing.  nrm (split-fp16 rows): the norms of the test samples; where one is
// infinite (squares above the largest float), the tiles' |t|^2 + |x|^2 - 2 t.x is infinite even for t = x,
// and the wave takes the sample again by differences in fp64, as predict_few does.
__global__ void __launch_bounds__(64) predict_final_k(const double *__restrict__ part_all, int64_t m,
                                                      const PredPair *__restrict__ pairs, PredPair one,
                                                      const int64_t *__restrict__ sv_count, double *dec, int64_t stride,
                                                      const float *__restrict__ nrm, const float *__restrict__ T,
                                                      const float *__restrict__ X, int64_t d,
                                                      const int32_t *__restrict__ sv_row_all,
                                                      const double *__restrict__ sv_coef_all, double c) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const PredPair pp = pair_of(pairs, one, blockIdx.y);
  const double *part = part_all + pp.part_off;
  const int64_t nsv = sv_count[blockIdx.y];
  const int used = (int)min<int64_t>(pp.nsplit, (nsv + PT - 1) / PT);
  double s = 0.0;
  if (q < m) {
#pragma unroll 8
    for (int k = 0; k < used; ++k) s += part[(int64_t)k * m + q];
  }
  unsigned long long again = nrm ? __ballot(q < m && nrm[q < m ? q : m - 1] == INFINITY) : 0;
  while (again) {
    const int lane = __builtin_ctzll(again);
    again &= again - 1;
    const float *t = T + (q - threadIdx.x + lane) * d;
    double sum = 0.0;
    for (int64_t v = threadIdx.x; v < nsv; v += 64) {
      const float *x = X + (int64_t)sv_row_all[pp.sv_off + v] * d;
      double d2 = 0.0;
      for (int64_t k = 0; k < d; ++k) {
        const double f = (double)(x[k] - t[k]);
        d2 = __builtin_fma(f, f, d2);
      }
      sum = __builtin_fma(sv_coef_all[pp.sv_off + v], rbf_of_d2(c, d2), sum);
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    s = (int)threadIdx.x == lane ? sum : s;
  }
  if (q < m) dec[q * stride + blockIdx.y] = s - pp.b;
}

// Workgroups of a launch at most: of the worst case (every training sample a support vector) most
// splits may turn out empty, and a workgroup that finds nothing to do still takes a turn (45 pairs
// of 12,000 samples with 480 support vectors each, 138,000 workgroups: 270 us of them).
constexpr int64_t PREDICT_GRID_MAX = 8192;

// Splits of a problem's support-vector tiles: about four workgroups for each of the 768 the
// device holds at once (they take what comes, so an uneven last round costs a quarter of one),
// at most one per tile and 64.
int predict_splits(int64_t m, int64_t nsv_max) {
  if (m <= 0) return 1;
  const int64_t row_tiles = (m + PT - 1) / PT;
  const int64_t sv_tiles = nsv_max > 0 ? (nsv_max + PT - 1) / PT : 1;
  int64_t s = (3072 + row_tiles - 1) / row_tiles;
  if (s > sv_tiles) s = sv_tiles;
  if (s > 64) s = 64;
  if (s < 1) s = 1;
  return (int)s;
}

hipError_t launch_predict_pairs(const PredictLaunch &L, hipStream_t s) {
  if (L.m <= 0 || L.npairs <= 0) return hipSuccess;
  if (L.few) return launch_predict_few(L, s);
  const PredictScratch &ws = L.ws;
  // Items of one problem fit 32 bits (test tiles x splits, at most 3,072 more than the test tiles).
  const int64_t nrt = (L.m + PT - 1) / PT;
  if (nrt > 0x7fffffff - 4096) return hipErrorInvalidValue;
  PrepParams p{};
  p.alpha = L.alpha;
  p.pairs = L.npairs > 1 ? ws.pairs : nullptr;
  p.one = L.host_pairs[0];
  p.npairs = L.npairs;
  p.sv_row = ws.sv_row;
  p.sv_coef = ws.sv_coef;
  p.count = ws.count;
  p.d = L.d;
  int64_t cb = 1;
  int32_t nsplit = 1;
  for (int32_t q = 0; q < L.npairs; ++q) {
    const int64_t n = L.host_pairs[q].ntr;
    cb = n > 0 && (n + compact_chunk(n) - 1) / compact_chunk(n) > cb ? (n + compact_chunk(n) - 1) / compact_chunk(n) : cb;
    nsplit = L.host_pairs[q].nsplit > nsplit ? L.host_pairs[q].nsplit : nsplit;
  }
  p.compact_blocks = (int32_t)cb;
  int64_t blocks = cb * L.npairs;
  if (L.split) {
    p.test = split_rows_of(L.T, L.split_test_rows ? L.m : 0, ws.split_test);
    p.train = split_rows_of(L.Xtr, L.split_train_rows ? L.n : 0, ws.split_train);
    p.perm = L.perm;
    p.all_train = L.all_train;
    p.test_blocks = (int32_t)split_rows_blocks(p.test);
    blocks += p.test_blocks + split_rows_blocks(p.train);
  }
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(predict_prep_k, dim3((unsigned)blocks), dim3(PBS), 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const float c = (float)(-L.gamma * 1.4426950408889634);
  int64_t items = 0;  // at most: the device counts the splits that have a tile
  for (int32_t q = 0; q < L.npairs; ++q) items += nrt * L.host_pairs[q].nsplit;
  if (L.split) {
    int64_t grid = (items + 7) / 8 * 8;
    if (grid > PREDICT_GRID_MAX) grid = PREDICT_GRID_MAX;
    hipLaunchKernelGGL(predict_f16x3_k, dim3((unsigned)grid), dim3(PBS), 0, s, ws.split_test, L.m, ws.split_train,
                       p.pairs, p.one, L.npairs, ws.sv_row, ws.sv_coef, ws.count, c, (int32_t)nrt, ws.part);
  } else {
    const dim3 grid((unsigned)nrt, (unsigned)nsplit, (unsigned)L.npairs);
    const bool vec4 = (L.d % 4 == 0) && ((reinterpret_cast<uintptr_t>(L.T) & 15) == 0) &&
                      ((reinterpret_cast<uintptr_t>(L.Xtr) & 15) == 0);
    if (vec4)
      hipLaunchKernelGGL(predict_mfma_k<true>, grid, dim3(PBS), 0, s, L.T, L.m, L.Xtr, p.pairs, p.one, ws.sv_row,
                         ws.sv_coef, ws.count, L.d, c, ws.part);
    else
      hipLaunchKernelGGL(predict_mfma_k<false>, grid, dim3(PBS), 0, s, L.T, L.m, L.Xtr, p.pairs, p.one, ws.sv_row,
                         ws.sv_coef, ws.count, L.d, c, ws.part);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(predict_final_k, dim3((unsigned)((L.m + 63) / 64), (unsigned)L.npairs), dim3(64), 0, s, ws.part,
                     L.m, p.pairs, p.one, ws.count, L.dec, L.dec_stride, L.split ? ws.split_test.nrm : nullptr, L.T, L.Xtr, L.d,
                     ws.sv_row, ws.sv_coef, -L.gamma * 1.4426950408889634);
  return hipGetLastError();
}

// pred[q] = class with most votes over the k(k-1)/2 pairs (a<b, lexicographic), pair (a,b)
// voting a iff its decision value is > 0; ties to the smaller class.  One wave a test sample:
// lanes take the pairs (whole lines of dec), votes are counted in LDS.  10,000 x 45 pairs: 25 us
// with one thread a sample.
__global__ void __launch_bounds__(PBS) ovo_vote_k(const double *__restrict__ dec, int64_t m, int32_t k,
                                                  int32_t *__restrict__ pred) {
  __shared__ uint8_t first[64 * 63 / 2], second[64 * 63 / 2];
  __shared__ int votes[PBS / 64][64];
  const int P = k * (k - 1) / 2;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x < k - 1) {  // thread a writes its pairs (a, a + 1) ..
    const int a = threadIdx.x;
    int p = a * (2 * k - a - 1) / 2;
    for (int b = a + 1; b < k; ++b, ++p) {
      first[p] = (uint8_t)a;
      second[p] = (uint8_t)b;
    }
  }
  votes[w][lane] = 0;
  __syncthreads();
  for (int64_t q = (int64_t)blockIdx.x * (PBS / 64) + w; q < m; q += (int64_t)gridDim.x * (PBS / 64)) {
    for (int p = lane; p < P; p += 64) atomicAdd(&votes[w][dec[q * P + p] > 0.0 ? first[p] : second[p]], 1);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // most votes, then the smaller class
    int best = lane < k ? (votes[w][lane] << 6) | (63 - lane) : -1;
    votes[w][lane] = 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o));
    if (lane == 0) pred[q] = 63 - (best & 63);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
}

hipError_t launch_ovo_vote(const double *dec, int64_t m, int32_t k, int32_t *pred, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  int64_t blocks = (m + 3) / 4;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(ovo_vote_k, dim3((unsigned)blocks), dim3(PBS), 0, s, dec, m, k, pred);
  return hipGetLastError();
}

}  // namespace svmx
