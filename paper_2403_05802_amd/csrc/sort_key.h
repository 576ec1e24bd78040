// The packed target tuple of an entry (the index map of the target format evaluated at its coordinates), as the kernels
// that sort by it build it.
#pragma once
#include "common.h"

namespace us {

typedef uint64_t Key;  // keys live in registers and LDS as 64-bit words whatever their storage

__device__ __forceinline__ Key build_key(const KeySpec &ks, uint32_t r, uint32_t c) {
  uint32_t a = ks.swap ? c : r, b = ks.swap ? r : c;
  if (ks.mode == 0) return ((Key)a << ks.b_bits) | (Key)b;
  // (a coordinate out of range is reported, not sorted; its second field is still cut to b_bits so that it cannot
  // leak into the leading field, whose digits the first histogram may take from a / bh alone)
  const Key field = ((Key)1 << ks.b_bits) - 1;
  if (ks.mode == 2) {   // Skew(0,1,-1) then TileSplit(0,bh): (a/bh, b-a, a%bh), the diagonal biased to be >= 0
    uint32_t ab = a / ks.bh, ai = a - ab * ks.bh, dg = b - a + (ks.a_extent - 1);
    return ((((Key)ab << ks.b_bits) | ((Key)dg & field)) << ks.ih_bits) | (Key)ai;
  }
  uint32_t ab = a / ks.bh, ai = a - ab * ks.bh, bb = b / ks.bw, bi = b - bb * ks.bw;
  return (((((Key)ab << ks.b_bits) | ((Key)bb & field)) << ks.ih_bits | (Key)ai) << ks.iw_bits) | (Key)bi;
}

__device__ __forceinline__ bool coo_out_of_range(const KeySpec &ks, uint32_t r, uint32_t c) {
  return ((ks.swap ? c : r) >= ks.a_extent) | ((ks.swap ? r : c) >= ks.b_extent);
}

// Workgroups are dealt round-robin to the 8 XCDs.  Mapping launch index i to tile
// (i % 8) * tiles_per_xcd + i / 8 lets each XCD work through one contiguous range of tiles, so
// the partial cache lines at the ends of neighbouring tiles' runs meet in the same L2.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t i, uint32_t per_xcd) { return (i & 7u) * per_xcd + (i >> 3); }

}  // namespace us
