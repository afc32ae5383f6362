// split_tile.hpp -- 128 x 128 tiles of row products on the split-fp16 rows (gram_split.hip):
// the stage loads, the LDS layout and the MFMA sweep shared by the Gram build and predict.
//
// A stage is 32 features of 128 rows of A and 128 rows of B.  The 128 bytes a row contributes
// (hi 32 | lo 32 halves, one line) go from memory to LDS without passing through registers
// (load-to-LDS, 16 bytes a lane: one instruction moves 8 whole rows), so a stage costs a wave
// eight instructions, no LDS store instructions and no registers beyond the addresses.  LDS row
// r holds its eight 16-byte pieces permuted by piece ^ (r % 8): the 16 lanes that read one MFMA
// operand (16 rows, the same piece) would otherwise all hit the same four banks.  The rows of B
// may be any rows (predict gathers its support vectors here).
// Staging through registers into [k chunk][row] slabs instead (two 2-way conflicting 16-byte
// LDS stores a thread and slab) kept the LDS pipe as busy as the matrix cores.  Contraction
// alone, 10,000 x 15,016 x 800: 1,370-1,400 TFLOP/s of fp16 MFMA work this way, 1,700 with no
// loads at all.
#pragma once

#include "common.hpp"

namespace svmx {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int ST = 128;   // tile edge (rows and columns)
constexpr int SKS = 32;   // k per stage: one MFMA K
constexpr int SBS = 256;  // 4 waves, 2x2 over the tile, 64x64 each
constexpr int SCH = 2 * ST / 8 / (SBS / 64);  // 8-row chunks of a stage that each wave loads

struct SplitStage {
  h8 v[2 * ST * 8];  // rows of A, then rows of B; 8 pieces a row
};

// Where this lane reads its piece of one 8-row chunk from: row `row` (already in range) of s,
// piece (lane % 8) ^ (lane / 8) of the stage at feature 0.
__device__ __forceinline__ const char *split_src(const SplitX &s, int64_t row) {
  const int lane = threadIdx.x & 63;
  return reinterpret_cast<const char *>(s.rows) + row * 4 * s.dp + (((lane & 7) ^ (lane >> 3)) << 4);
}

// Load one stage: chunk q of this wave from src[q] + 128 bytes a stage passed.
__device__ __forceinline__ void split_stage_load(SplitStage &S, const char *(&src)[SCH]) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int q = 0; q < SCH; ++q) {
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) const void *)src[q],
                                     (__attribute__((address_space(3))) void *)&S.v[(w * SCH + q) * 64], 16, 0, 0);
    src[q] += 4 * SKS;
  }
}

// One stage of the tile's products: wave (wm, wn) accumulates its 64 x 64 block.  The three
// products of a block go into one accumulator in the order h.h, h.l, l.h.
__device__ __forceinline__ void split_stage_mma(const SplitStage &S, int wm, int wn, v4f (&acc)[4][4]) {
  const int lane = threadIdx.x & 63;
  const int kq = lane >> 4, r16 = lane & 15;
  const int ph = r16 * 8 + (kq ^ (r16 & 7)), pl = r16 * 8 + ((kq | 4) ^ (r16 & 7));
  h8 ah[4], al[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    ah[a] = S.v[(wm * 4 + a) * 128 + ph];
    al[a] = S.v[(wm * 4 + a) * 128 + pl];
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const h8 bh = S.v[(8 + wn * 4 + b) * 128 + ph], bl = S.v[(8 + wn * 4 + b) * 128 + pl];
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[a], bh, acc[a][b], 0, 0, 0);
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[a], bl, acc[a][b], 0, 0, 0);
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[a], bh, acc[a][b], 0, 0, 0);
  }
}

// The contraction of a tile whose first stage is already on its way: one LDS stage (32 KB),
// loaded, then multiplied; the other workgroups of the CU multiply meanwhile.  Ends with a barrier
// after the last operand has been read.
__device__ __forceinline__ void split_tile_loaded(SplitStage &S, const char *(&src)[SCH], int64_t stages, int wm, int wn,
                                                  v4f (&acc)[4][4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int64_t st = 1;; ++st) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's loads to LDS (a barrier alone asks for no wait)
    __syncthreads();
    split_stage_mma(S, wm, wn, acc);
    __syncthreads();  // this stage's operands have been read
    if (st >= stages) break;
    split_stage_load(S, src);
  }
}

}  // namespace svmx
