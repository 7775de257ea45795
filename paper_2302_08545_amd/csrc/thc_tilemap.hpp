// The tiling table shared by the host planner and the kernels (plain data, no GPU types).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define THC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define THC_HOST_DEVICE inline
#endif

namespace thc {

constexpr int LOG_TILE = 13;

// ---------------------------------------------------------------------------------------------
// Bit-permuted tiling.  Every transform pass cuts a block of 2^L coordinates into tiles of 8192: a tile is
// 2^nrows rows of 2^logw consecutive coordinates (nrows + logw = 13).  The offset bits of a coordinate
// inside its block are dealt out as
//   bits [0, logw)                          the column inside the row,
//   [sh0, sh0 + n0) and [sh1, ...)          the row index: its low n0 bits, then the rest,
//   runs (flen, fpos)                       the bit positions the tile index inside the block is scattered to.
// The host orders the runs so that the low three bits of the tile index (workgroup ids are dealt round-robin to
// the 8 XCDs) land on the offset bits that measured fastest for that pass.
// ---------------------------------------------------------------------------------------------
struct TileMap {
  // 32-bit fields throughout: the geometry is uniform per workgroup and stays in scalar registers
  uint32_t L;        // log2 of the span the tile index runs over (the block, or 13 for blocks below 8192)
  uint32_t logw;
  uint32_t nrows;
  uint32_t nfixed;   // = L - 13
  uint32_t n0, sh0, sh1;
  // the tile index inside the span, cut into up to four runs of consecutive bits: run i starts at bit fcum[i]
  // of the tile index, has mask fmask[i] = 2^length - 1 (0 for an unused run) and lands at offset bit fpos[i]
  uint32_t fcum[4];
  uint32_t fmask[4];
  uint32_t fpos[4];
};

// Kernels that walk a vector in consecutive 8192-coordinate tiles, one per workgroup: workgroup ids are dealt
// round-robin to the 8 XCDs, and streaming is faster (measured 5.7 against 5.3 TB/s) when an XCD keeps to its own
// value of byte-address bits 18..20 rather than 15..17.  Inside every whole group of 8 << S = 64 tiles the low three bits
// of the workgroup id therefore select tile bits S..S+2 = 3..5.
template <int S = 3>
THC_HOST_DEVICE uint32_t xcd_tile(uint32_t wg, uint32_t ntiles) {
  constexpr uint32_t G = (8u << S) - 1u;
  return (wg | G) < ntiles ? (wg & ~G) | ((wg & 7u) << S) | ((wg >> 3) & ((1u << S) - 1u)) : wg;
}

}  // namespace thc
