// gram_split.hip -- RBF Gram on the fp16 MFMA path with fp32 accuracy (gfx950).
//
// G_ij = exp(-gamma * max(0, |x_i|^2 + |x_j|^2 - 2 x_i.x_j)) as in gram.hip (the Gaussian RBF
// the paper names, Section III.C), but the contraction X X^T runs on v_mfma_f32_16x16x32_f16:
// every row is scaled by a power of two s_i (so that |x| < 1), split as x = h + l with h, l fp16
// (h the nearest fp16, l the nearest fp16 to the remainder; together 22 significant bits), and
// x_i.x_j = s_i s_j (h_i.h_j + h_i.l_j + l_i.h_j) up to the l_i.l_j term (2^-22 relative) and
// the rounding of l; all three products go into one fp32 accumulator per output, as in an fp32
// contraction.  Three fp16 MFMA products per fp32 product on a 2.5 PFLOP/s path instead of one
// fp32 product on the 157 TFLOP/s path; measured against the fp64 difference form, the values
// are as accurate as those of the fp32 MFMA kernel.  The row norms are fp64 sums of the fp32
// inputs.
#include "split_rows.hpp"
#include "split_tile.hpp"
#include "tile_order.hpp"
#include "tile_store.hpp"

#include <math.h>

namespace svmx {

int64_t split_pitch(int64_t d) { return (d + SKS - 1) / SKS * SKS; }

// Scratch of the split rows: [n][dp / 32][hi 32 | lo 32] halves (dp = d rounded up to 32, zero
// padded), the power-of-two row scales and the row norms.  The rows start on a 128-byte boundary
// whatever the address of the caller's workspace (the 256 bytes more leave room for it): their
// 16-byte pieces are loaded to LDS, and a row's 128 bytes of a stage are one line.
int64_t gram_split_scratch_bytes(int64_t n, int64_t d) {
  const int64_t dp = split_pitch(d);
  return 2 * (2 * n * dp) + 8 * n + 256;
}

SplitX split_views(void *scratch, int64_t n, int64_t d) {
  SplitX s;
  s.dp = split_pitch(d);
  s.rows = reinterpret_cast<_Float16 *>((reinterpret_cast<uintptr_t>(scratch) + 127) & ~(uintptr_t)127);
  s.scale = reinterpret_cast<float *>(s.rows + 2 * n * s.dp);
  s.nrm = s.scale + n;
  return s;
}

__global__ void __launch_bounds__(256) gram_split_k(SplitRows p, int64_t d) {
  split_rows_block(p, d, blockIdx.x, gridDim.x, [](int64_t pos) { return pos; });
}

// One 128x128 tile of the upper triangle per workgroup; workgroup b runs on XCD b % 8 and takes
// tile b / 8 of that XCD's contiguous share of the super-tile order (tile_order.hpp), so the
// tiles an XCD holds at once share their row and column slabs in its L2.  An off-diagonal
// tile is stored twice, as itself and mirrored.  Lane l of an MFMA holds D[4*(l/16) + e][l%16]
// of each 16x16 block.
// Long rows are bound by the matrix cores (20,000 x 784: the products alone 0.66 ms at the
// 1,450 TFLOP/s the stage loop reaches, 0.91 ms in all against 1.16 ms with stages staged through
// registers; 60,000 x 784 7.7 against 9.8 ms), short ones by the stores (100,000 x 32: 40 GB in
// 7.0 ms).  Four workgroups a CU: one's products run under the others' loads and stores (three:
// 50,000 x 128 2.07 instead of 2.01 ms, 60,000 x 784 7.88 instead of 7.70); they leave 128 registers,
// and 5 are spilled (20 bytes a lane, not in the stage loop).
// In a diagonal tile the cross products h.l and l.h are accumulated in the order of the operand
// roles, so K(x_r, x_c) and K(x_c, x_r) can differ in the last bit; the upper one (row index <=
// column index, the role every off-diagonal tile uses) is written to both places, so that
// K(x_i, x_j) of i < j is always computed with x_i as the row operand.
template <bool NT>
__global__ void __launch_bounds__(SBS, 4) gram_rbf_f16x3(SplitX s, int64_t n, float c, float *__restrict__ G, int64_t ld,
                                                      int64_t nt, int64_t ntiles, int64_t sup, const InputCheck *chk) {
  __shared__ SplitStage S;
  __shared__ float sA[ST], sB[ST], nA[ST], nB[ST];
  const int64_t per_xcd = (ntiles + 7) / 8;
  const int64_t b = (int64_t)blockIdx.x;
  const int64_t lin = (b % 8) * per_xcd + b / 8;
  if (lin >= ntiles || input_invalid(chk)) return;
  int64_t ti, tj;
  upper_tile_super(lin, nt, ti, tj, sup);
  // (uniform by construction; said so, the store addresses stay in scalar registers)
  const int64_t i0 = (int64_t)__builtin_amdgcn_readfirstlane((int)ti) * ST;
  const int64_t j0 = (int64_t)__builtin_amdgcn_readfirstlane((int)tj) * ST;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int kq = lane >> 4, r16 = lane & 15;
  if (threadIdx.x < ST) {
    const int64_t gi = i0 + threadIdx.x, gj = j0 + threadIdx.x;
    sA[threadIdx.x] = gi < n ? s.scale[gi] : 0.f;
    nA[threadIdx.x] = gi < n ? s.nrm[gi] : 0.f;
    sB[threadIdx.x] = gj < n ? s.scale[gj] : 0.f;
    nB[threadIdx.x] = gj < n ? s.nrm[gj] : 0.f;
  }
  const char *src[SCH];  // waves 0 and 1 load the rows of A, 2 and 3 those of B (past the end: the last row again)
#pragma unroll
  for (int q = 0; q < SCH; ++q)
    src[q] = split_src(s, min<int64_t>((w < 2 ? i0 : j0) + ((w & 1) * SCH + q) * 8 + (lane >> 3), n - 1));
  v4f acc[4][4];
  split_stage_load(S, src);
  split_tile_loaded(S, src, s.dp / SKS, wm, wn, acc);
  const bool diag = i0 == j0;
  float kv[4][4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int lr0 = wm * 64 + a * 16 + 4 * kq;
    const int64_t gr0 = i0 + lr0;
#pragma unroll
    for (int bb = 0; bb < 4; ++bb) {
      const int lc = wn * 64 + bb * 16 + r16;
      const int64_t gc = j0 + lc;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        kv[a][bb][e] = (gr0 + e == gc) ? 1.0f : split_rbf(acc[a][bb][e], sA[lr0 + e], sB[lc], nA[lr0 + e], nB[lc], c);
      if (diag && gc < n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (gr0 + e < n && lr0 + e <= lc) {
            __builtin_nontemporal_store(kv[a][bb][e], &G[(gr0 + e) * ld + gc]);
            if (lr0 + e < lc) __builtin_nontemporal_store(kv[a][bb][e], &G[gc * ld + gr0 + e]);
          }
        }
      }
    }
  }
  if (!diag) store_tile_128<NT>(G, ld, n, i0 + wm * 64, j0 + wn * 64, kq, r16, kv);
}

hipError_t launch_split_rows(const float *X, int64_t n, int64_t d, const SplitX &s, hipStream_t st, const int32_t *perm,
                             InputCheck *chk) {
  if (n <= 0) return hipSuccess;
  SplitRows p = split_rows_of(X, n, s);
  p.perm = perm;
  p.chk = chk;
  hipLaunchKernelGGL(gram_split_k, dim3((unsigned)split_rows_blocks(p)), dim3(256), 0, st, p, d);
  return hipGetLastError();
}

hipError_t launch_gram_split(const float *X, int64_t n, int64_t d, float gamma, float *G, int64_t ld, void *scratch,
                             hipStream_t st, const int32_t *perm, InputCheck *chk) {
  const SplitX s = split_views(scratch, n, d);
  hipError_t e = launch_split_rows(X, n, d, s, st, perm, chk);
  if (e != hipSuccess) return e;
  const int64_t nt = (n + ST - 1) / ST;
  const int64_t ntiles = nt * (nt + 1) / 2;
  const int64_t grid = ((ntiles + 7) / 8) * 8;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  const float c = -gamma * 1.4426950408889634f;
  // Non-temporal stores where the Gram is larger than the 256 MB Infinity Cache (it is not read
  // again here, so its lines should not displace the operand slabs from L2: 60,000 x 784 7.7
  // against 8.3 ms, 50,000 x 128 2.0 against 2.3); a smaller one stays in the caches, for the
  // solver to read (8,000 x 64 81 against 93 us, 10,000 x 64, 400 MB, the same), and rows that
  // are not 16-byte aligned need L2 to put their lines together (tile_store.hpp).
  const bool aligned = (ld % 4 == 0) && ((reinterpret_cast<uintptr_t>(G) & 15) == 0);
  const bool nt_store = aligned && 4.0 * (double)n * (double)ld > 256e6;
  // super-tiles of 32 x 32 tiles for rows of up to 128 features, whose build is bound by its
  // stores (measured: 8.7 -> 7.7 ms at 100,000 x 32, 16.6 -> 13.2 ms at 130,000 x 32, 2.44 ->
  // 2.37 ms at 50,000 x 128), 8 x 8 for longer rows (1.09 against 1.25 ms at 20,000 x 784)
  const int64_t sup = s.dp <= 4 * SKS ? 32 : 8;
  if (nt_store)
    hipLaunchKernelGGL(gram_rbf_f16x3<true>, dim3((unsigned)grid), dim3(SBS), 0, st, s, n, c, G, ld, nt, ntiles, sup,
                       chk);
  else
    hipLaunchKernelGGL(gram_rbf_f16x3<false>, dim3((unsigned)grid), dim3(SBS), 0, st, s, n, c, G, ld, nt, ntiles, sup,
                       chk);
  return hipGetLastError();
}

}  // namespace svmx
