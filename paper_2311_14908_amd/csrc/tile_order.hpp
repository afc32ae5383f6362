// tile_order.hpp -- order of the upper-triangle tiles (ti <= tj) of a symmetric tile grid.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace svmx {

// Linear index -> tile (ti, tj), ti <= tj < nt, in super-tile order: super-rows I of SUPER tile
// rows; in each, the diagonal super-tile (its upper triangle, row-major), then the super-tiles
// to its right (each row-major; the last one may be narrower).  A run of consecutive indices
// (what the workgroups of one XCD hold at once) therefore reads SUPER row slabs and SUPER column
// slabs, which stay in that XCD's L2, instead of one row slab and a different column slab per
// tile.  Bijective onto the upper triangle for every nt >= 1 and SUPER >= 1.  SUPER = 8 suits
// long rows, whose slabs are the traffic; short rows are bound by the tile stores, which a
// wider super-tile (32) keeps on fewer rows of the Gram at a time.
constexpr int64_t SUPER = 8;

__host__ __device__ inline void upper_tile_super(int64_t lin64, int64_t nt64, int64_t &ti, int64_t &tj,
                                                 const int64_t super = svmx::SUPER) {
  // A launch has fewer than 2^31 tiles, so 32-bit arithmetic (a 64-bit division costs a hundred
  // instructions, before the first load of a tile).
  const uint32_t lin = (uint32_t)lin64, nt = (uint32_t)nt64, S = (uint32_t)super;
  uint32_t r0 = 0, base = 0, r = 0, right = 0;
  for (;;) {
    r = nt - r0 < S ? nt - r0 : S;
    right = nt - r0 - r;
    const uint32_t cnt = r * (r + 1) / 2 + r * right;
    if (lin < base + cnt) break;
    base += cnt;
    r0 += S;
  }
  uint32_t off = lin - base;
  const uint32_t dcnt = r * (r + 1) / 2;
  if (off < dcnt) {  // diagonal super-tile: row a holds r - a tiles
    uint32_t a = 0;
    while (off >= r - a) {
      off -= r - a;
      ++a;
    }
    ti = r0 + a;
    tj = r0 + a + off;
    return;
  }
  off -= dcnt;  // only a super-row of full height has tiles to its right
  const uint32_t J = off / (r * S), nfull = right / S;
  const uint32_t o2 = off - J * r * S;
  const uint32_t c = J < nfull ? S : right - nfull * S;  // width of this super-tile (the last may be narrower)
  ti = r0 + o2 / c;
  tj = r0 + S + J * S + o2 % c;
}

}  // namespace svmx
