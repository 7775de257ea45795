// Host-side planner: how the butterfly stages of a block are split over the passes and how every pass tiles a
// block.  Plain C++ (no GPU types), so that it can be built and run under the host sanitizers.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "thc.h"
#include "thc_tilemap.hpp"

namespace thc {

inline int ilog2(uint64_t v) {
  int l = 0;
  while ((1ull << l) < v) ++l;
  return l;
}

// Split of the log2(B) butterfly stages over the passes, and each pass's tiling (see TileMap).
//
// Stage order.  THC_ORDER_ASCENDING: bits 0, 1, ..., L-1.  THC_ORDER_SPLIT (blocks of at least 2^16):
// bits 0..9, 13, 14, 15, then 10, 11, 12, 16, ..., L-1.  In the split order the first pass works on eight rows
// of 1024 consecutive coordinates (4 KB) that are 32 KB apart instead of 8192 consecutive ones, which lets a
// workgroup -- hence its XCD -- stay on one value of byte-address bits 12..14 for both its reads and writes.
struct Plan {
  int L, L1;        // lo pass does L1 = min(L, 13) bits
  bool split;       // stage order THC_ORDER_SPLIT in effect
  int nmid;
  int mid[3];       // bit counts of the in-place middle passes
  int R;            // the last pass does R bits
  int bits[4][16];  // the butterfly bits of every pass after the first, in processing order (mids, then the last)
  TileMap lo, midmap[3], hi;
  bool ok() const {
    if (!lo.L || !hi.L) return false;
    for (int m = 0; m < nmid; ++m) if (!midmap[m].L) return false;
    return true;
  }
};

inline TileMap make_tilemap(int L, int logw, const std::vector<int>& rows, const int (&pref)[3]) {
  TileMap m{};
  m.L = (uint32_t)L;
  m.logw = (uint32_t)logw;
  m.nrows = (uint32_t)rows.size();
  m.nfixed = (uint32_t)(L - LOG_TILE);
  // rows: at most two runs of consecutive bit positions
  size_t run = 0;
  while (run + 1 < rows.size() && rows[run + 1] == rows[run] + 1) ++run;
  m.n0 = (uint32_t)(rows.empty() ? 0 : run + 1);
  m.sh0 = (uint32_t)(rows.empty() ? 0 : rows[0]);
  m.sh1 = (uint32_t)(m.n0 < rows.size() ? rows[m.n0] : 0);
  bool taken[32] = {};
  for (int r : rows) taken[r] = true;
  std::vector<int> fixed;
  for (int b : pref)
    if (b >= logw && b < L && !taken[b]) { fixed.push_back(b); taken[b] = true; }
  for (int b = logw; b < L; ++b)
    if (!taken[b]) fixed.push_back(b);
  // cut into runs of consecutive positions (at most four with the orders and splits used here)
  int nrun = 0;
  uint32_t cum = 0;
  for (size_t i = 0; i < fixed.size();) {
    size_t j = i;
    while (j + 1 < fixed.size() && fixed[j + 1] == fixed[j] + 1) ++j;
    if (nrun == 4) { m.L = 0; return m; }   // cannot happen; L = 0 makes validation fail loudly
    const uint32_t len = (uint32_t)(j - i + 1);
    m.fcum[nrun] = cum;
    m.fmask[nrun] = (1u << len) - 1u;
    m.fpos[nrun] = (uint32_t)fixed[i];
    cum += len;
    ++nrun;
    i = j + 1;
  }
  return m;
}

inline std::vector<int> bit_range(int lo, int hi) {
  std::vector<int> v;
  for (int b = lo; b < hi; ++b) v.push_back(b);
  return v;
}

inline Plan make_plan(uint64_t block, uint32_t stage_order) {
  Plan pl{};
  pl.L = ilog2(block);
  pl.L1 = pl.L < LOG_TILE ? pl.L : LOG_TILE;
  pl.split = stage_order == THC_ORDER_SPLIT && pl.L >= 16;
  // Up to 9 bits left after the lo pass: one strided pass takes them all (8 and 9 bits mean rows of only 128 and
  // 64 bytes, still far cheaper than another trip through HBM).  More than that: ceil(rem / 7) strided passes of
  // nearly equal size (wider rows make longer contiguous segments); the last one, fused with the quantizer or
  // the final scaling, gets the smallest.  In the split order the first of them starts with bits 10, 11, 12: its
  // rows are 1024 coordinates wide at most, so it must own all three, which any share of at least 3 bits guarantees.
  const int rem = pl.L - pl.L1;
  const int npass = rem <= 9 ? 1 : (rem + 6) / 7;
  pl.nmid = npass - 1;
  pl.R = rem / npass;
  for (int m = 0, left = rem - pl.R; m < pl.nmid; ++m) {
    pl.mid[m] = (left + (pl.nmid - m) - 1) / (pl.nmid - m);
    left -= pl.mid[m];
  }
  const int Lg = pl.L < LOG_TILE ? LOG_TILE : pl.L;   // blocks below 8192: tiles are just 8192 consecutive coordinates
  // bits still to do after the lo pass, in processing order
  std::vector<int> todo;
  if (pl.split) {
    todo = {10, 11, 12};
    for (int b = 16; b < pl.L; ++b) todo.push_back(b);
  } else {
    todo = bit_range(pl.L1, pl.L);
  }
  const int none[3] = {-1, -1, -1}, low[3] = {10, 11, 12}, grp[3] = {13, 14, 15};
  pl.lo = pl.split ? make_tilemap(Lg, 10, {13, 14, 15}, low) : make_tilemap(Lg, LOG_TILE, {}, none);
  size_t at = 0;
  for (int m = 0; m < pl.nmid; ++m) {
    std::vector<int> rows(todo.begin() + at, todo.begin() + at + pl.mid[m]);
    std::copy(rows.begin(), rows.end(), pl.bits[m]);
    pl.midmap[m] = make_tilemap(Lg, LOG_TILE - pl.mid[m], rows, pl.split ? grp : low);
    at += pl.mid[m];
  }
  std::vector<int> rows(todo.begin() + at, todo.end());
  std::copy(rows.begin(), rows.end(), pl.bits[pl.nmid]);
  pl.hi = make_tilemap(Lg, LOG_TILE - pl.R, rows, pl.split ? grp : low);
  return pl;
}

// Tiling of the first pass over `len` coordinates.  Consecutive 8192-coordinate tiles (ascending order, or blocks
// below 2^16) stream faster (measured: 5.7 against 5.3 TB/s) when the tile order is permuted inside spans of at least
// 2^19 coordinates so that the low three bits of the tile index, i.e. the XCD, select offset bits 16..18 rather
// than 13..15.  Vectors that are not whole spans keep the natural order.
inline TileMap lo_tilemap(const Plan& pl, uint64_t len) {
  if (pl.split) return pl.lo;
  const int span = pl.L < 19 ? 19 : pl.L;
  if (len & ((1ull << span) - 1)) return pl.lo;
  const int far[3] = {16, 17, 18};
  const TileMap m = make_tilemap(span, LOG_TILE, {}, far);
  return m.L ? m : pl.lo;
}

// Whether the quantizer finds the range itself.  Small calls are bound by their launches, about 2.4 us each on the host and
// 3 on the device.  Against that, every workgroup reads its block's partial sums over again, while its tile's loads travel.
// Measured, first pass and quantizer with the range found there against a launch of its own (time of the first over the
// second), by the workgroups of the launch:
//   blocks of 2^17 to 2^20, up to 128 partial sums a worker: 1 to 4 workers 0.93 to 0.97 at 512 and 1024, 0.96 to 1.00 at 1280,
//     0.98 to 1.02 at 1536; 8 workers 0.95 to 0.98 at 512 and 1024, 1.01 from 1280 on; 32 workers 0.96 at 512, 1.03 at 1024.
//   blocks of up to 2^16, at most 8 partial sums a worker: 1 to 4 workers 0.88 to 0.95 at up to 1024, 0.96 to 0.98 at 2048,
//     0.97 to 0.99 at 3072 and 3584, 0.98 to 1.01 at 4096; 8 workers 0.89 to 0.98 at up to 3072, 0.98 to 1.01 at 4096; 32
//     workers 0.81 to 0.95 at up to 2048, 0.94 to 0.99 at 4096, 0.96 to 1.01 at 5120 and 6144.  With up to four workers
//     another 1 to 3 % would be had up to 3584.
// Blocks of 2^22 lose 2 % at 1024.
inline bool find_range(const Plan& pl, uint64_t tiles, uint32_t W) {   // 8192-coordinate tiles of each of W vectors
  if (pl.L > 20) return false;
  if (pl.L > 16) return tiles * W <= (W > 16 ? 512u : W > 4 ? 1024u : 1280u);
  return tiles * W <= (W > 4 ? 4096u : W > 2 ? 3072u : 2048u);
}

// Blocks of up to 2^14: whether the worker side of W vectors goes block by block (thc_whole.hpp) instead of pass by pass,
// and where the range comes from.
//   GIVEN  range known (thc_compress): one launch instead of two, with error feedback three.  Faster at every size measured
//          (2^15 to 2^28 worker-coordinates): 7.5 to 10.9 us -> 5.4 to 7.8 for small calls, 620 -> 290 for large ones.
//   FIND   every workgroup adds up its block's squares of all workers: one launch, W times the reads.  Time over that of the
//          passes: one worker (no reads more) up to 2^13 0.80 to 0.85 at 4 to 3104 workgroups (of 8192 coordinates), 2^14 0.47
//          to 0.79 at 512 to 1024, 1.00 at 1280.  2 and 4 workers up to 2^13 0.51 to 0.95 at up to 512; at 1024 0.70 to 0.91,
//          with 4 workers behind NORMS; 8 workers no gain (10.4 to 12.5 -> 10.2 to 12.1 us at up to 256).  2^14 with 2 workers
//          0.95 to 1.07 at up to 128, 0.50 to 0.76 at 256 to 512; with 3 and 4 1.08 to 1.22 at up to 192 (9.2 -> 11.2 us), and
//          a launch less, which is what bounds such a round on the host: two blocks x 4 workers, rounds one after the other,
//          21.7 -> 19.7 us.
//   NORMS  a pass that keeps the sums only, the range, the blocks: three launches instead of two or three, 8.5 bytes a
//          coordinate instead of 12.5.  Time over that of the passes, 2 to 32 workers: up to 2^13 1.10 to 1.17 at 256 (8 and
//          more), 1.01 to 1.10 at 384 and 448, 0.70 to 0.75 at 512 with up to 8 workers and 0.99 to 1.03 with more, 0.88 to
//          0.95 at 576, 0.74 to 0.96 at 640 and 768, 0.79 to 0.88 at 1024, 622 -> 463 us at 32768.  2^14, whose 1024 threads
//          leave room for two workgroups a compute unit: where they fill the chip evenly 0.71 to 0.95 (up to 8 workers, 449 to
//          512) and 0.79 to 1.02 (up to 16, 897 to 1024; with more 0.98 to 1.04); 0.80 to 1.11 at 576 to 896, 0.94 to 1.13 at
//          1152 to 1536, 0.96 to 1.03 at 2048, 0.91 to 0.97 at 3072 and 3584, 0.91 to 0.94 at 4096, 607 -> 477 us at 32768.
//          There is more to gain from 3072 on and, with up to 8 workers, at 320 to 448 (0.80 to 0.99).
//          With error feedback (29 bytes -> 20.5) up to 2^13 always: 13.5 to 18.7 -> 12.6 to 16.9 us at up to 256, 26 to 28 ->
//          21 at 512, 45 -> 41 at 1024, 1459 -> 1019 at 32768; 2^14, one workgroup a compute unit: 0.65 to 0.84 at up to 512,
//          0.90 to 1.06 at 576, 1.02 to 1.07 at 768 to 2048, 1.00 at 3072, 0.92 to 0.94 at 4096, 1448 -> 1263 us at 32768.
enum class Whole { NO, GIVEN, FIND, NORMS };
constexpr uint32_t WHOLE_FIND_WORKERS = 4;

inline Whole whole_route(const Plan& pl, uint64_t tiles, uint32_t W, bool ef, bool range_given) {
  if (pl.L > 14) return Whole::NO;
  if (range_given) return Whole::GIVEN;
  const uint64_t wg = tiles * W;
  if (ef) return pl.L <= 13 || wg <= 512 || wg >= 4096 ? Whole::NORMS : Whole::NO;
  if (W == 1 && (pl.L <= 13 || wg <= 1024)) return Whole::FIND;
  if (W <= WHOLE_FIND_WORKERS && wg <= 512) return Whole::FIND;
  if (pl.L <= 13) return wg >= (W > 8 ? 640u : 512u) ? Whole::NORMS : Whole::NO;
  const bool even = (wg > 448 && wg <= 512 && W <= 8) || (wg > 896 && wg <= 1024 && W <= 16);
  return even || wg >= 4096 ? Whole::NORMS : Whole::NO;
}

// FIND at 2^14: whether two workgroups share a block's quantization.  A call of a few blocks leaves most of the chip idle, and a
// workgroup's chain is long: halving its longest part pays for a second transform.  Time of a round over that of one workgroup
// a block, by workgroups before the split: 1 0.94, 4 0.97, 8 0.96 (19.6 -> 18.8 us), 32 0.96, 64 0.98, 128 1.02 to 1.03.  Four to a
// block 0.96 at 8 and 32, 1.05 at 64; blocks of up to 2^13, 512 threads to a workgroup, 0.99 to 1.00 at any size.
inline bool whole_split(const Plan& pl, uint64_t tiles, uint32_t W) { return pl.L == 14 && (tiles / 2) * W <= 64; }

// Blocks of 2^14, inverse transform in one launch: a block to a workgroup of 1024 threads (k_inv_whole) or two blocks to
// one of 512 (k_big_inv_whole).  With few blocks the first has half the work on each of twice the compute units; 512 of its
// workgroups are on the chip at once, and 1024 of the other's, which is why neither is better throughout.  From 1025 blocks on it
// is the faster one as long as the estimate is stored plainly (keep_estimate, 2560 blocks).  Time of the first over that of the
// second, by the number of blocks, sums that no cache holds:
//                  128 to 512     640            704 to 1024    1040 to 1280   1281 to 1792   1920 to 2560   2816 to 3600   from 4200 on
//   8-bit sums     0.69 to 0.95   0.98           1.02 to 1.15   0.90 to 0.94   0.94 to 0.95   0.95 to 0.99   1.03 to 1.05   1.07 to 1.13
//   4 bits         0.65 to 0.88   0.99           1.01 to 1.07   0.82 to 0.86   0.87 to 0.93   0.87 to 0.93   0.98 to 1.00   1.04 to 1.13
//   5, 9 and 12    0.64 to 0.96   1.03 to 1.04   1.05 to 1.15   0.84 to 0.90   0.88 to 0.99   0.91 to 1.00   0.98 to 1.06   0.99 to 1.17
//   16 bits        the first always; the second has no form of its own for them
// With error feedback the second: the rotated uniform variant, and thc_compress_all where whole_route leaves it to the passes.
inline bool inv_whole_14(uint64_t len, bool ef, uint32_t bits) {
  const uint64_t K = len >> 14;
  if (ef) return false;
  if (bits == 16) return true;
  if (K <= 1024) return K <= (bits == 4 || bits == 8 ? 640 : 512);
  return K <= 2560;
}

// Which passes of a call over W vectors of d coordinates, walked in launches of `len` coordinates of each, take tiles of
// 2^15 coordinates (thc_big.hpp).  Blocks of 2^23 to 2^25: all (two passes instead of three: 1.16x at one block of one
// vector, 1.5x at 16 of them).  2^22: both tile sizes take two passes, and the larger one pays once its few large tiles
// fill the chip many times over (rounds of 256 to 3072 tiles: 0.91x to 1.05x; of 16384: 1.12x).  The forward passes go by
// the tiles of a launch (64 blocks of one vector, 512 tiles a launch: 707 us with the smaller tiles, 752 with the larger
// ones), the inverse ones by those of the call (787 and 740 us) as long as a launch has a tile for each of the 512
// workgroups the chip holds (thc_decompress_noalloc, 256 tiles a launch: 1030 and 1140 us, 995 and 1260 ascending).
constexpr int LOG_BIG = 15;
constexpr uint64_t BIG_MIN_TILES_22 = 8192, BIG_RESIDENT = 512;

inline bool big_forward(const Plan& pl, uint64_t len, uint32_t W) {
  if (pl.L == 22) return W * (len >> LOG_BIG) >= BIG_MIN_TILES_22;
  return pl.L > 22 && pl.L <= LOG_BIG + 10;
}

inline bool big_inverse(const Plan& pl, uint64_t d, uint64_t len, uint32_t W) {
  return big_forward(pl, d, W) && (pl.L > 22 || W * (len >> LOG_BIG) >= BIG_RESIDENT);
}

// Whether the quantizer and, with error feedback, the inverse's last pass walk a launch's tiles last one first: where the
// half-transformed vectors of the launch, with error feedback these and the vectors themselves, exceed the 256 MB
// memory-side cache.  In order -> last first: rounds of 2^20-point blocks with error feedback, 25 x 4 vectors 733 -> 707 us,
// 25 x 8 1430 -> 1407, 9 x 16 1042 -> 1017, 64 x 8 3633 -> 3612; 2^25 x 8 2154 -> 2094; the range pass of the rotated
// uniform variant behind its first pass, 25 x 4 vectors, 221 -> 214.  Below that size it gives nothing (25 x 1 167 either
// way, one block without error feedback 31.3 -> 31.6), and the decompression's two passes lose 3 %.  Tiles of 2^15, the worker
// side with error feedback, time of last first over in order: 2^25 0.96 to 0.97, 2^24 0.98 to 0.99, 2^23 0.99 to 1.00, 2^22
// 0.985 to 1.00 (32 workers in bf16, ascending, 1.004); without it 1.00 to 1.01 at all four.  The rule takes 2^25 only.
inline bool last_first(const Plan& pl, uint64_t len, uint32_t W, bool ef, bool big) {
  return W * len > (1ull << (ef ? 25 : 26)) && (!big || pl.L == 25);
}

// Cache hints (see Mem) that depend on the size of a launch: `len` coordinates of each of W vectors.  The memory-side cache
// holds 256 MB, and what is read again before that much else has come by should be left in it.
//
// stream_inputs: the first pass reads its vectors non-temporally.  Without error feedback nothing of the call reads them again,
// so that only small ones, which the caller has just written, are better left alone; with it the update does, at the end.  Time
// of streamed over kept: one block of 2^20 x 4 vectors 1.01, x 10 1.04, 4 x 8 (128 MB) 0.99, 10 x 8 0.97, 41 x 16 0.96, 256 x 8
// 0.96.  With error feedback, inputs that no cache held before: 128 MB 0.99 to 1.04 and at 2^14 1.11, 160 MB 0.98 to 1.09, 192 MB
// 1.00 to 1.09, 224 MB 0.98 to 1.09, 256 MB 0.96 to 1.02, 320 to 768 MB 0.92 to 0.98.
// stream_big_inputs: the bf16 gradients of that pass on tiles of 2^15, with error feedback.  Two instructions of 16 bytes a lane share
// their lines, and still it gains from a size on.  Streamed over kept, thc_compress_all, gradients and buffers together: 2^23 (48
// MB) 1.01 to 1.02, 2 x 2^23 and 2^24 (96 MB) 1.01 to 1.02, 4 x 2^23 (192 MB) 0.98 to 0.99, 2^25 (192 MB) 0.99 to 1.00, 2 x 2^24 x 4
// vectors 0.99 to 1.00, 4 x 2^23 x 8, 2^25 x 8 and 16 x 2^22 x 16 0.99.
// stream_norms: the pass that keeps the norms only.  Time of streamed over kept, with the compression behind it, inputs that no
// cache held before.  Blocks of 2^10 to 2^14, whose compression is one launch: 32 MB 1.08 to 1.18 in binary32, 64 MB 0.94 to 1.00,
// 96 to 192 MB 0.92 to 1.00, 256 MB to 1 GB 0.88 to 1.00; in bf16 without error feedback 0.98 to 1.01 throughout.  Blocks of
// 2^20: 64 MB 1.00 to 1.11, 96 and 128 MB 0.97 to 1.02, 160 and 192 MB 0.94 to 1.00, 256 MB and more 0.92 to 1.00.
// stream_minmax: the uniform variant's range pass without rotation; its quantizer reads the vectors again and finds what the
// cache holds.  Streamed over kept, prepare and compress: 64 MB 0.97 to 1.07, 96 to 160 MB 0.99 to 1.08, 192 and 224 MB 0.98 to
// 1.09, 255 and 256 MB 0.93 to 1.02, 320 MB and more 0.92 to 1.01.
// stream_rotated: the half-rotated vectors in the uniform variant's range pass, which the quantizer reads once more.  Streamed over
// kept, prepare and compress, rotated, blocks of 2^16 and 2^20: 16 MB 1.01 to 1.02, 64 MB 1.03 to 1.05, 128 MB 1.02 to 1.03, 192 MB
// 1.03 to 1.04, 256 MB 1.01 to 1.02, 384 MB 0.95 to 0.97, 512 MB 0.90 to 0.93, 1.6 GB 0.94 to 0.96.
// plain_first_pass: the forward first pass stores plainly, or else through the L2.  Where a few workgroups write, there is no
// eviction to spare, and a launch ends later.  Through over plain, thc_compress_all, by workgroups of 8192 coordinates: 4 1.00 to
// 1.01, 16 to 24 1.01 to 1.03, 64 0.99, 84 1.00 to 1.02, 128 0.93 to 1.00, 512 0.92 to 0.94.
// through_inverse: the inverse's first pass writes through the L2, or else non-temporally.  Through over non-temporal, decompressions
// that no cache holds parts of, blocks of 2^16 to 2^21: 4 MB 0.92 to 0.93, 16 and 64 MB 0.76 to 0.82, 100 and 128 MB 0.86 to 0.89,
// 160 to 256 MB 0.84 to 0.89, and 512 MB to 1 GB, walked in shares of 256 MB, 0.87; 2^23 and 2^24 up to 256 MB 0.83 to 0.95, 384 and
// 512 MB in one share 1.01 to 1.09; 2^25 0.91 to 1.00, 1.01 to 1.04.  Again and again on the same buffers the two are closer
// (4 MB 0.98, 128 MB 1.01).  With error feedback, 2^20: 128 MB 0.95 to 0.97, 160 MB 1.00 to 1.02, 192 MB 1.01 to 1.02, 256 MB 1.00 to 1.05.
// stream_blocks: the gradients of blocks of up to 2^14 that go block by block, behind the norms.  Time of streamed over kept, 64 MB
// to 1 GB: 2^10 0.95 to 1.00, 2^13 and 2^14 0.97 to 1.01, with error feedback 0.98 to 1.01; in bf16 0.98 to 1.02, no gain.
// stream_sums: the aggregation.  Time of streamed over kept, by the streams' bytes together, on three sets of them in turn: 34 MB
// 1.05, 66 MB 1.02 to 1.19 (0.80 to 0.95 with 3-bit indices, 16-bit sums or 3 workers), 82 MB 0.80 to 0.93, 100 to 190 MB 0.76 to
// 0.94, 840 MB 0.85 to 0.95; behind the quantizer of the same round 67 MB 0.99, 105 MB 1.00.  A single stream of 3-bit indices, whose
// three loads a thread share their lines, 1.12 to 1.15 from 100 MB on, of 2-bit ones 0.98 to 1.02: kept.
// sums_four_loads: streamed sums of 4-bit indices at other widths than 8 with four workers' loads in flight, where a call has few
// wavefronts to hide them.  Time over that of one, 16-bit sums: 32 workers of 5 * 2^20 coordinates 0.70, 6.25 * 2^20 0.77, 8 * 2^20
// 0.86, 12 * 2^20 1.04, 16 * 2^20 1.13; 16 workers of 10 * 2^20 0.95, 12.5 * 2^20 1.00, 16 * 2^20 1.05, 24 * 2^20 1.03; 8 workers
// of 20 * 2^20 0.95, 25 * 2^20 0.99, 32 * 2^20 1.02.
// keep_estimate: the estimate, which the caller reads next, is stored plainly, or else non-temporally.  Kept over streamed, the
// decompression and a step that reads the estimate (w -= lr * out) together, by the size of the estimate:
//                  4 to 12 MB     16 MB          24 and 32 MB   48 to 96 MB    128 MB   160 MB         176 and 192 MB  208 to 256 MB
//   2^10 to 2^14   1.00 to 1.03   1.01 to 1.03   0.98 to 1.02   0.93 to 1.00   0.92     1.00           1.03 to 1.07    1.06 to 1.08
//   2^15           1.00 to 1.02   1.04           0.96 to 0.98   0.94 to 0.97   0.93     0.98           1.00 to 1.03    1.01 to 1.02
//   2^16 to 2^21   1.00 to 1.03   1.03 to 1.04   0.95 to 1.01   0.94 to 0.99   0.92     0.93 to 0.95   0.96 to 1.01    1.00 to 1.08
//   2^22                          1.00           0.90 to 1.00   0.90 (48), 0.98 (64), 1.05 (96)  1.14  1.20   1.11 to 1.15   1.00 to 1.10
//   2^23, 2^24                                   1.00           0.92 to 0.96   0.91 to 0.93  0.90 to 0.97  0.90 to 1.00  0.97 to 1.06
//   no rotation    0.94 to 1.01   0.94           0.92 to 0.94   0.92 to 0.96   0.92     0.99           1.02 to 1.04    1.04
// Blocks of 2^15, whose one workgroup a block writes all of an estimate of 0.1 to 1 MB, 0.98 to 0.99; 2^10 to 2^14 0.99 to 1.01.
// The decompression by itself gains by the hint at every size above 4 MB (2^10 x 2^15, 128 MB, 30 us against 37): what it gains
// below 160 MB, the reader loses and more.
constexpr uint64_t MB = 1ull << 20;

inline uint64_t input_bytes(uint64_t len, uint32_t W, bool bf16, bool ef) { return W * len * ((bf16 ? 2 : 4) + (ef ? 4 : 0)); }
inline bool stream_inputs(uint64_t len, uint32_t W, bool bf16, bool ef) {
  return input_bytes(len, W, bf16, ef) >= (ef ? 240 : 64) * MB;
}
inline bool stream_big_inputs(uint64_t len, uint32_t W) { return input_bytes(len, W, true, true) >= 160 * MB; }
inline bool stream_norms(const Plan& pl, uint64_t len, uint32_t W, bool bf16, bool ef) {
  return input_bytes(len, W, bf16, ef) >= (pl.L > 14 ? 128 : 64) * MB;
}
inline bool stream_blocks(uint64_t len, uint32_t W, bool bf16) { return !bf16 && input_bytes(len, W, bf16, false) >= 64 * MB; }
inline bool plain_first_pass(uint64_t tiles, uint32_t W) { return tiles * W < 64; }
inline bool stream_rotated(uint64_t len, uint32_t W) { return W * len * 4 > 256 * MB; }
inline bool through_inverse(uint64_t len, uint32_t W) { return W * len * 4 <= 256 * MB; }
inline bool stream_sums(uint64_t d, uint32_t n, uint32_t b) { return n * (d / 8) * b >= 80 * MB && (n > 1 || b == 1 || b > 3); }
inline bool sums_four_loads(uint64_t d) { return d <= 10 * MB; }   // coordinates

inline bool stream_minmax(uint64_t len, uint32_t W, bool bf16, bool ef) { return input_bytes(len, W, bf16, ef) >= 240 * MB; }

inline bool keep_estimate(uint64_t d, int L) {
  return (L == 15 && 4 * d <= MB) || (4 * d > 16 * MB && 4 * d <= (L == 22 ? 80 : 160) * MB);
}
inline bool keep_plain_estimate(uint64_t d) { return 4 * d > 4 * MB && 4 * d <= 160 * MB; }   // uniform variant without rotation

// Uniform quantizer on a vector of d coordinates: one group of eight coordinates to a thread, 4096 to a workgroup, or two.
// One group / two, us:
//   error feedback, binary32: 2^18 4.0 / 4.3, 2^20 4.7 / 4.8, 2^21 6.2 / 5.8, 6 * 2^20 14.6 / 13.7, 2^24 33.1 / 32.0, 25 * 2^20
//     48.5 / 48.5, 2^28 605 / 584 (2^25 to 40 * 2^20, called again and again on the same vector, 64 / 65 and 79 / 84);
//   bf16: 2^20 4.7 / 4.9, 2^21 6.0 / 5.8, 6 * 2^20 13.0 / 10.8, 25 * 2^20 43.4 / 41.6, 2^28 512 / 496 (48 and 56 * 2^20, again and
//     again, 81 / 85 and 99 / 106);
//   without it, binary32: 2^20 3.3 / 3.9, 2^22 4.8 / 4.9, 6 * 2^20 6.2 / 5.8, 12 * 2^20 12.3 / 11.3, 2^24 14.9 / 14.6, 25 * 2^20
//     20.5 / 20.7, 2^26 55.8 / 57.4, 2^28 214 / 221;
//   bf16: 2^20 3.4 / 3.8, 12 * 2^20 10.4 / 9.9, 2^24 12.3 / 12.3, 2^28 181 / 189.
inline bool uniform_one_group(uint64_t d, bool bf16, bool ef) {
  if (ef) return d <= 1ull << 20;
  return bf16 || d <= 1ull << 22 || d > 1ull << 24;
}

// Kernels that take a whole vector, one launch after another of at most LAUNCH_COORDS coordinates (whole blocks): a launch
// holds fewer than 2^32 threads, which at eight coordinates a thread is 2^35, a bf16 vector of 64 GB.
constexpr uint64_t LAUNCH_COORDS = 1ull << 34;

template <class Piece>
inline void for_pieces(uint64_t d, Piece&& piece) {
  for (uint64_t x0 = 0; x0 < d; x0 += LAUNCH_COORDS) piece(x0, d - x0 < LAUNCH_COORDS ? d - x0 : LAUNCH_COORDS);
}

// Whether a walk goes in shares smaller than the ring (even_share): where one pass leaves in memory what the next one reads.  A
// decompression that takes the inverse in one launch leaves nothing, and each share costs a launch and its drain; walked in
// shares of 2^26 coordinates / in one launch, us: 2^27 coordinates from 8-bit sums in blocks of 2^10 110 / 108, 2^14 129 / 112,
// 2^15 116 / 109; 2^29 501 / 478, 542 / 467 and 506 / 472; 2^28 from 16-bit sums 283 / 268, 298 / 283, 305 / 285.
inline bool walks_in_shares(uint64_t block, bool inverse) {
  return block < (1ull << 22) && (!inverse || block > (1ull << LOG_BIG));
}

// What a walk in even shares counts in: whole blocks, and whole 2^20 coordinates (the first pass's tiling wants 2^19, see
// lo_tilemap).
inline uint64_t share_unit(uint64_t block) { return block > (1ull << 20) ? block : 1ull << 20; }

// Coordinates of each of W vectors in the largest step of a walk over d of them in even shares.  A step takes about `target`
// coordinates of all vectors together, rounded to whole units, or with `most` at most that.
inline uint64_t even_share(uint64_t d, uint64_t block, uint32_t W, uint64_t target, bool most) {
  const uint64_t unit = share_unit(block);
  const uint64_t whole = (W * d + (most ? target - 1 : 0)) / target, steps = whole ? whole : 1;
  const uint64_t share = ((d + steps - 1) / steps + unit - 1) / unit * unit;
  return share < d ? share : d;
}

// The groups of whole blocks, at most `gc` coordinates of each of W vectors, in which a call walks its d coordinates:
// group(first coordinate, coordinates, whether the forward and the inverse launches take the larger tiles).  Groups of gc and
// a rest, or with `unit` (of which gc is a multiple, or all of d) as many groups that differ by at most one unit.
template <class Group>
inline void for_groups(const Plan& pl, uint64_t d, uint64_t gc, uint32_t W, Group&& group, uint64_t unit = 0) {
  const uint64_t steps = (d + gc - 1) / gc, units = unit ? (d + unit - 1) / unit : 0;
  for (uint64_t x0 = 0, i = 0; x0 < d; ++i) {
    const uint64_t want = unit ? (units / steps + (i < units % steps ? 1 : 0)) * unit : gc, len = d - x0 < want ? d - x0 : want;
    group(x0, len, big_forward(pl, len, W), big_inverse(pl, d, len, W));
    x0 += len;
  }
}

}  // namespace thc
