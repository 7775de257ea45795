// C-ABI of libthc (see include/thc.h): host-side validation and kernel dispatch.
#include "thc.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "thc_kernels.hpp"
#include "thc_plan.hpp"

namespace {

using namespace thc;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int validate(const thc_params* p) {
  if (!p) return THC_EINVAL;
  if (p->block < (1ull << 10) || p->block > (1ull << 27) || (p->block & (p->block - 1))) return THC_EINVAL;
  if (p->d == 0 || p->d % p->block || p->d >> 40) return THC_EINVAL;   // grids are 32-bit tile counts
  if (p->n < 1) return THC_EINVAL;
  if (p->n > THC_MAX_WORKERS) return THC_EUNSUPPORTED;
  if (p->b < 1 || p->b > 8) return THC_EINVAL;
  if (p->g < (1u << p->b) - 1 || p->g > 255) return THC_EINVAL;
  if (p->agg_bits < 1 || p->agg_bits > 16) return THC_EINVAL;
  if (p->in_dtype != THC_DTYPE_F32 && p->in_dtype != THC_DTYPE_BF16) return THC_EINVAL;
  if (!(p->t_p > 0.f) || !std::isfinite(p->t_p)) return THC_EINVAL;
  if (p->stage_order != THC_ORDER_ASCENDING && p->stage_order != THC_ORDER_SPLIT) return THC_EINVAL;
  if (p->group_log2 != 0 && (p->group_log2 < 10 || p->group_log2 > 40)) return THC_EINVAL;
  if (p->single_launch > 1) return THC_EINVAL;
  const uint32_t top = (1u << p->b) - 1;
  if (p->table[0] != 0 || p->table[top] != p->g) return THC_ETABLE;
  for (uint32_t z = 0; z < top; ++z)
    if (p->table[z] >= p->table[z + 1]) return THC_ETABLE;
  if ((uint64_t)p->g * p->n >= (1ull << p->agg_bits)) return THC_EOVERFLOW;
  return THC_OK;
}


// ---- workspace layout --------------------------------------------------------------------------------------
// [0, header)  status word of the last single-launch sweep (0 = fine), the rest reserved.  The header is 2 MiB
//              (4 KiB for small rings) so that the ring is aligned like the workspace itself: the passes' tilings
//              count on address bits up to 2^20.
// ring         the half-rotated vectors in flight: one group of blocks (launch-by-launch path) or a few block-sized
//              slots per vector (single-launch path); ring_floats(p, ef) binary32 values
// partials     n * (d >> min(L, 13)) binary64 partial sums of squares (one per 8192 coordinates, or per block)
// sync         counters of the single-launch path, K * SYNC_PER_UNIT words
// lut          device copy of the quantizer's grid-cell table, 256 words
//
// Launch-by-launch path: a group is a run of whole blocks of every vector in the call, sized so that the group's
// intermediate (all vectors of the call together) is about 2^group_log2 coordinates, or by default what measured best
// (walk_coords); the workspace does not grow with d.  Random streams are indexed by global coordinate, so the grouping never changes a result.
constexpr size_t WS_HEADER_BIG = 1u << 21, WS_HEADER_SMALL = 4096;
constexpr uint32_t DEFAULT_GROUP_LOG2 = 29;
constexpr uint32_t DEFAULT_GROUP_LOG2_SMALL = 25;   // with thc_params.single_launch: the caller is after a small workspace
// From a unit's last first-pass workgroup being dispatched to its range being visible, the chip gets through about
// this many workgroups (measured on the VGG16-shaped workload: trailing by fewer steps leaves consumers waiting,
// by more pushes the ring out of the memory-side cache).  A unit's next phase trails by at least that.
constexpr uint32_t LATENCY_WORKGROUPS = 1024;

uint64_t group_coords(const thc_params* p, uint32_t W) {
  const uint64_t target =
      1ull << (p->group_log2 ? p->group_log2 : p->single_launch ? DEFAULT_GROUP_LOG2_SMALL : DEFAULT_GROUP_LOG2);
  uint64_t gc = target / W / p->block * p->block;
  if (gc < p->block) gc = p->block;
  if (gc > p->d) gc = p->d;
  return gc;
}

struct GroupWalk {
  uint64_t most, unit;   // for_groups' `gc` and `unit`
};

// Coordinates of each of W vectors that one group takes, by default; at most what the ring holds.  The smaller a group, the more
// of what its first pass writes is still in the memory-side cache when the last one reads it; against that stand two or three
// launches a group.  Blocks of up to 2^21, groups of 2^29 / 2^28 / 2^27 / 2^26 coordinates, us: 256 x 8 vectors of 2^20 (half of it
// padding) 5070 / 4950 / 4813 / 4788, 321 x 16 12250 / 12090 / 12000 / 12160, 512 x 8 of 2^17 1259 / 1245 / 1231 / 1258, with error
// feedback 64 x 4 1802 / 1799 / 1784 / 1847.  A walk in steps of exactly 2^27 took 3 % more where it left a short rest (20 x 8):
// hence even shares.  The decompression, two launches a group: rounds of one worker, 200 blocks of 2^20, 997 us at 2^29, 990 at
// 2^27, 968 at 2^26 (256 MB), 978 at 2^25, and 1005 where shares exceed 2^26 a little.  Blocks of 2^22 and more lose up to 7 % (8 x 8 of 2^23) and keep their groups.
GroupWalk walk_coords(const thc_params* p, uint32_t W, bool inverse) {
  const uint64_t most = group_coords(p, W);
  if (p->group_log2 || p->single_launch || !walks_in_shares(p->block, inverse)) return {most, 0};
  const uint64_t share = even_share(p->d, p->block, W, 1ull << (inverse ? 26 : 27), inverse);
  if (share > most) return {most, 0};
  return {share, share_unit(p->block)};
}

// Shape of the single-launch sweep over W vectors (thc_pipeline.hpp), or ok = false where it does not apply:
// it is asked for by thc_params.single_launch and takes the split stage order, blocks of 2^17 .. 2^22 coordinates,
// at least four blocks, and the default grouping.
struct PipeShape {
  bool ok;
  uint32_t nphase, lag, slots;
};

PipeShape pipe_shape(const thc_params* p, const Plan& pl, uint32_t W, bool ef) {
  PipeShape sh{};
  const uint64_t K = p->d / p->block;
  sh.ok = p->single_launch == 1 && pl.split && pl.nmid == 0 && pl.L >= 17 && K >= 4 && K <= 65536 && p->group_log2 == 0;
  sh.nphase = ef ? 4 : 2;
  // A consumer should find its producers finished and published: they are `lag` steps ahead, a step being
  // nphase * Tu workgroups.
  const uint64_t per_step = (uint64_t)sh.nphase * ((uint64_t)W << pl.R);
  sh.lag = 1 + (uint32_t)((LATENCY_WORKGROUPS + per_step - 1) / per_step);
  sh.slots = (sh.nphase - 1) * sh.lag + 2;
  return sh;
}

uint64_t ring_floats(const thc_params* p, const Plan& pl, bool ef) {
  uint64_t need = group_coords(p, 1);
  const uint64_t all = (uint64_t)p->n * group_coords(p, p->n);
  if (all > need) need = all;
  for (uint32_t W : {1u, p->n}) {
    const PipeShape sh = pipe_shape(p, pl, W, ef);
    if (sh.ok && (uint64_t)sh.slots * W * p->block > need) need = (uint64_t)sh.slots * W * p->block;
  }
  return need;
}

size_t partial_count(const thc_params* p, const Plan& pl) { return (size_t)p->n * (size_t)(p->d >> pl.L1); }

size_t sync_words(const thc_params* p) {
  const uint64_t K = p->d / p->block;
  return (p->single_launch == 1 && K <= 65536) ? (size_t)K * SYNC_PER_UNIT : 0;
}

struct WsLayout {
  uint32_t* status;
  float* ring;
  double* partials;
  uint32_t* sync;
  uint32_t* lut;
  size_t bytes;
};

// The ring is sized for error feedback whenever the caller asked for it in thc_workspace_bytes; the calls take
// the layout that goes with what they are given (ef or not), which is the same or smaller.
WsLayout ws_layout(void* ws, const thc_params* p, const Plan& pl, bool ef) {
  char* base = static_cast<char*>(ws);
  WsLayout w{};
  const size_t ring_bytes = ring_floats(p, pl, ef) * sizeof(float);
  size_t at = ring_bytes >= WS_HEADER_BIG ? WS_HEADER_BIG : WS_HEADER_SMALL;
  w.status = reinterpret_cast<uint32_t*>(base);
  w.ring = reinterpret_cast<float*>(base + at);
  at += ring_bytes;
  w.partials = reinterpret_cast<double*>(base + at);
  at += partial_count(p, pl) * sizeof(double);
  w.sync = reinterpret_cast<uint32_t*>(base + at);
  at += sync_words(p) * sizeof(uint32_t);
  w.lut = reinterpret_cast<uint32_t*>(base + at);
  at += 256 * sizeof(uint32_t);
  w.bytes = at + 256;
  return w;
}

uint64_t tiles_of(uint64_t d) { return (d + TILE - 1) / TILE; }

Walk walk_over(bool last_first, uint64_t tiles, uint32_t W) {
  return last_first ? Walk{(uint32_t)tiles - 1u, W - 1u, ~0u} : Walk{};
}

// global coordinate of the buffers' first element
uint64_t base_coord(const thc_params* p) { return (uint64_t)p->first_block * p->block; }

void fill_lut(const thc_params* p, uint32_t (&lut)[256]) {
  const uint32_t top = (1u << p->b) - 1;
  uint32_t k = 0;
  for (uint32_t z = 0; z < top; ++z) {
    const uint32_t lo = p->table[z], next = p->table[z + 1], ent = lo | (next - lo) << 8 | z << 16;
    for (; k < next; ++k) lut[k] = ent;
  }
  for (; k < 256; ++k) lut[k] = p->g | 255u << 8 | top << 16;   // 255: the top value never rounds up
}

int check_launch() {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return THC_OK;
  std::fprintf(stderr, "libthc: kernel launch failed: %s\n", hipGetErrorString(e));
  return THC_ELAUNCH;
}

template <template <int> class Launcher, class... A>
void dispatch_0_7(int r, A&&... args) {
  switch (r) {
    case 0: Launcher<0>::run(args...); break;
    case 1: Launcher<1>::run(args...); break;
    case 2: Launcher<2>::run(args...); break;
    case 3: Launcher<3>::run(args...); break;
    case 4: Launcher<4>::run(args...); break;
    case 5: Launcher<5>::run(args...); break;
    case 6: Launcher<6>::run(args...); break;
    default: Launcher<7>::run(args...); break;
  }
}

// the last pass of a transform may take 8 or 9 bits
template <template <int> class Launcher, class... A>
void dispatch_0_9(int r, A&&... args) {
  switch (r) {
    case 8: Launcher<8>::run(args...); break;
    case 9: Launcher<9>::run(args...); break;
    default: dispatch_0_7<Launcher>(r, args...); break;
  }
}

// every launcher takes the number of vectors W of the launch: grid = (tiles, W)
template <int R> struct LaunchMid {
  static void run(const MidArgs& a, uint64_t tiles, uint32_t W, hipStream_t s) {
    k_mid<R><<<dim3((unsigned)tiles, W), dim3(NT), 0, s>>>(a);
  }
};
template <int R> struct LaunchQuant {
  static void run(const QuantArgs& a, bool cfold, uint64_t tiles, uint32_t W, hipStream_t s) {
    if (cfold && R >= 2) go<R >= 2>(a, tiles, W, s);
    else go<false>(a, tiles, W, s);
  }
  template <bool CFOLD>
  static void go(const QuantArgs& a, uint64_t tiles, uint32_t W, hipStream_t s) {
    if constexpr (R <= 7) {                        // find_range: blocks of up to 2^20
      if (a.partials) {
        k_fwd_hi_quant<R, CFOLD, true><<<dim3((unsigned)tiles, W), dim3(NT), 0, s>>>(a);
        return;
      }
    }
    k_fwd_hi_quant<R, CFOLD, false><<<dim3((unsigned)tiles, W), dim3(NT), 0, s>>>(a);
  }
};
template <int R> struct LaunchHiMinMax {
  static void run(const HiMinMaxArgs& a, uint64_t tiles, uint32_t W, hipStream_t s) {
    const dim3 grid((unsigned)tiles, W), blk(NT);
    if constexpr (R >= 2 && hi_mem<R>() == STREAM) {
      if (stream_rotated(a.d, W)) {
        k_fwd_hi_minmax<R, STREAM><<<grid, blk, 0, s>>>(a);
        return;
      }
    }
    k_fwd_hi_minmax<R, KEEP><<<grid, blk, 0, s>>>(a);
  }
};
template <int R> struct LaunchInvHi {
  static void run(const InvHiArgs& a, bool keep, uint64_t tiles, uint32_t W, hipStream_t s) {
    const dim3 grid((unsigned)tiles, W), blk(NT);
    if (keep) k_inv_hi<R, KEEP><<<grid, blk, 0, s>>>(a);
    else k_inv_hi<R, STREAM><<<grid, blk, 0, s>>>(a);
  }
};

template <int L1, bool BF16, bool EF, bool XO, Mem LOAD>
void launch_fwd_lo_x(const FwdLoArgs& a, bool norm_only, uint64_t tiles, uint32_t n, hipStream_t s) {
  const dim3 grid((unsigned)tiles, n), blk(NT);
  if (norm_only) {
    k_fwd_lo<L1, BF16, EF, XO, true, LOAD, KEEP><<<grid, blk, 0, s>>>(a);
    return;
  }
  if constexpr (LOAD == KEEP) {
    if (plain_first_pass(tiles, n)) {
      k_fwd_lo<L1, BF16, EF, XO, false, LOAD, KEEP><<<grid, blk, 0, s>>>(a);
      return;
    }
  }
  k_fwd_lo<L1, BF16, EF, XO, false, LOAD, THROUGH><<<grid, blk, 0, s>>>(a);
}

template <int L1, bool BF16, bool EF, Mem LOAD>
void launch_fwd_lo_k(const FwdLoArgs& a, bool split, bool norm_only, uint64_t tiles, uint32_t n, hipStream_t s) {
  if constexpr (L1 == LOG_TILE) {
    if (split) {
      launch_fwd_lo_x<L1, BF16, EF, true, LOAD>(a, norm_only, tiles, n, s);
      return;
    }
  }
  launch_fwd_lo_x<L1, BF16, EF, false, LOAD>(a, norm_only, tiles, n, s);
}

template <int L1, Mem LOAD>
void launch_fwd_lo_t(const FwdLoArgs& a, bool bf16, bool ef, bool split, bool norm_only, uint64_t tiles, uint32_t n,
                     hipStream_t s) {
  if (bf16) {
    if (ef) launch_fwd_lo_k<L1, true, true, LOAD>(a, split, norm_only, tiles, n, s);
    else launch_fwd_lo_k<L1, true, false, LOAD>(a, split, norm_only, tiles, n, s);
  } else {
    if (ef) launch_fwd_lo_k<L1, false, true, LOAD>(a, split, norm_only, tiles, n, s);
    else launch_fwd_lo_k<L1, false, false, LOAD>(a, split, norm_only, tiles, n, s);
  }
}

template <Mem LOAD>
void launch_fwd_lo_m(const Plan& pl, const FwdLoArgs& a, bool bf16, bool ef, bool norm_only, uint64_t tiles, uint32_t n,
                     hipStream_t s) {
  switch (pl.L1) {
    case 10: launch_fwd_lo_t<10, LOAD>(a, bf16, ef, false, norm_only, tiles, n, s); break;
    case 11: launch_fwd_lo_t<11, LOAD>(a, bf16, ef, false, norm_only, tiles, n, s); break;
    case 12: launch_fwd_lo_t<12, LOAD>(a, bf16, ef, false, norm_only, tiles, n, s); break;
    default: launch_fwd_lo_t<13, LOAD>(a, bf16, ef, pl.split, norm_only, tiles, n, s); break;
  }
}

void launch_fwd_lo(const Plan& pl, const FwdLoArgs& a, bool bf16, bool ef, bool norm_only, bool stream, uint64_t tiles,
                   uint32_t n, hipStream_t s) {
  if (stream) launch_fwd_lo_m<STREAM>(pl, a, bf16, ef, norm_only, tiles, n, s);
  else launch_fwd_lo_m<KEEP>(pl, a, bf16, ef, norm_only, tiles, n, s);
}

void launch_range(const RangeArgs& r, hipStream_t s) {
  const uint64_t K = r.d >> r.L;
  if (r.L - r.L1 <= 3) k_range_small<<<dim3((unsigned)((K + RANGE_SMALL_BLOCKS - 1) / RANGE_SMALL_BLOCKS)), dim3(256), 0, s>>>(r);
  else k_range<<<dim3((unsigned)K), dim3(RANGE_NT), 0, s>>>(r);
}

template <int SB, bool TABLE>
void launch_inv_lo_k(const InvLoArgs& a, bool split, bool through, dim3 grid, hipStream_t s) {
  const dim3 blk(NT);
  if (split) {
    if (through) k_inv_lo<true, SB, TABLE, THROUGH><<<grid, blk, 0, s>>>(a);
    else k_inv_lo<true, SB, TABLE, STREAM><<<grid, blk, 0, s>>>(a);
  } else {
    if (through) k_inv_lo<false, SB, TABLE, THROUGH><<<grid, blk, 0, s>>>(a);
    else k_inv_lo<false, SB, TABLE, STREAM><<<grid, blk, 0, s>>>(a);
  }
}

void launch_inv_lo(const Plan& pl, const InvLoArgs& a, uint64_t tiles, uint32_t W, hipStream_t s) {
  const dim3 grid((unsigned)tiles, W);
  const bool through = through_inverse(a.d, W);
  if (a.use_table) {
    if (a.src_bits == 4) launch_inv_lo_k<4, true>(a, pl.split, through, grid, s);
    else launch_inv_lo_k<0, true>(a, pl.split, through, grid, s);
  } else {
    if (a.src_bits == 8) launch_inv_lo_k<8, false>(a, pl.split, through, grid, s);
    else if (a.src_bits == 16) launch_inv_lo_k<16, false>(a, pl.split, through, grid, s);
    else launch_inv_lo_k<0, false>(a, pl.split, through, grid, s);
  }
}

// ---- passes on tiles of 2^15 coordinates (thc_big.hpp) ------------------------------------------------------------
template <template <int> class Launcher, class... A>
void dispatch_big(int r, A&&... args) {
  switch (r) {
    case 7: Launcher<7>::run(args...); break;
    case 8: Launcher<8>::run(args...); break;
    case 9: Launcher<9>::run(args...); break;
    default: Launcher<10>::run(args...); break;
  }
}

template <bool BF16, bool EF, Mem LOAD = KEEP>
void launch_big_lo_k(const BigLoArgs& a, bool split, dim3 grid, hipStream_t s) {
  if (split) k_big_lo<BF16, EF, true, LOAD><<<grid, dim3(NT), 0, s>>>(a);
  else k_big_lo<BF16, EF, false, LOAD><<<grid, dim3(NT), 0, s>>>(a);
}

void launch_big_lo(const Plan& pl, const BigLoArgs& a, bool bf16, bool ef, uint32_t W, hipStream_t s) {
  const dim3 grid((unsigned)(a.d >> LOG_BIG), W);
  if (bf16) {
    if (ef && stream_big_inputs(a.d, W)) launch_big_lo_k<true, true, STREAM>(a, pl.split, grid, s);
    else if (ef) launch_big_lo_k<true, true>(a, pl.split, grid, s);
    else launch_big_lo_k<true, false>(a, pl.split, grid, s);
  } else {
    if (ef) launch_big_lo_k<false, true>(a, pl.split, grid, s);
    else launch_big_lo_k<false, false>(a, pl.split, grid, s);
  }
}

template <int R> struct LaunchBigQuant {
  static void run(const BigQuantArgs& a, bool split, uint32_t W, hipStream_t s) {
    const dim3 grid((unsigned)(a.d >> LOG_BIG), W);
    if (split) k_big_quant<R, true><<<grid, dim3(NT), 0, s>>>(a);
    else k_big_quant<R, false><<<grid, dim3(NT), 0, s>>>(a);
  }
};

template <int R> struct LaunchBigInvHi {
  template <bool XO>
  static void go(const BigInvHiArgs& a, int mode, bool keep, dim3 grid, hipStream_t s) {
    if constexpr (R == 8 || R == 9) {   // R = 7: calls beyond keep_estimate's limit; R = 10 stores plainly
      if (mode == 0 && keep) {
        k_big_inv_hi<R, XO, 0, KEEP><<<grid, dim3(NT), 0, s>>>(a);
        return;
      }
    }
    if (mode == 0) k_big_inv_hi<R, XO, 0><<<grid, dim3(NT), 0, s>>>(a);
    else if (mode == 1) k_big_inv_hi<R, XO, 1><<<grid, dim3(NT), 0, s>>>(a);
    else k_big_inv_hi<R, XO, 2><<<grid, dim3(NT), 0, s>>>(a);
  }
  static void run(const BigInvHiArgs& a, bool split, int mode, bool keep, uint32_t W, hipStream_t s) {
    const dim3 grid((unsigned)(a.d >> LOG_BIG), W);
    if (split) go<true>(a, mode, keep, grid, s);
    else go<false>(a, mode, keep, grid, s);
  }
};

template <int SB, bool TABLE>
void launch_big_inv_lo_k(const BigInvLoArgs& a, bool split, dim3 grid, hipStream_t s) {
  const dim3 blk(NT);
  if constexpr (!TABLE) {
    if (through_inverse(a.d, grid.y)) {
      if (split) k_big_inv_lo<SB, TABLE, true, THROUGH><<<grid, blk, 0, s>>>(a);
      else k_big_inv_lo<SB, TABLE, false, THROUGH><<<grid, blk, 0, s>>>(a);
      return;
    }
  }
  if (split) k_big_inv_lo<SB, TABLE, true, STREAM><<<grid, blk, 0, s>>>(a);
  else k_big_inv_lo<SB, TABLE, false, STREAM><<<grid, blk, 0, s>>>(a);
}

void launch_big_inv_lo(const Plan& pl, const BigInvLoArgs& a, uint32_t W, hipStream_t s) {
  const dim3 grid((unsigned)(a.d >> LOG_BIG), W);
  if (a.use_table) {
    if (a.src_bits == 4) launch_big_inv_lo_k<4, true>(a, pl.split, grid, s);
    else launch_big_inv_lo_k<0, true>(a, pl.split, grid, s);
  } else {
    if (a.src_bits == 8) launch_big_inv_lo_k<8, false>(a, pl.split, grid, s);
    else if (a.src_bits == 16) launch_big_inv_lo_k<16, false>(a, pl.split, grid, s);
    else launch_big_inv_lo_k<0, false>(a, pl.split, grid, s);
  }
}

// middle passes of W vectors of `d` coordinates each, in place
void run_mids(const Plan& pl, float* x, uint64_t d, uint32_t W, hipStream_t s) {
  for (int m = 0; m < pl.nmid; ++m) {
    MidArgs a{x, d, pl.midmap[m]};
    switch (pl.mid[m]) {   // blocks of 2^23 and more
      case 5: LaunchMid<5>::run(a, tiles_of(d), W, s); break;
      case 6: LaunchMid<6>::run(a, tiles_of(d), W, s); break;
      default: LaunchMid<7>::run(a, tiles_of(d), W, s); break;
    }
  }
}

template <int L1>
void launch_inv_whole_ef(const InvWholeArgs& a, int efm, dim3 grid, hipStream_t s) {
  const dim3 blk(NT);
  const bool b4 = a.lo.src_bits == 4;
  if (efm == 1) {
    if (b4) k_inv_whole<L1, 4, 1><<<grid, blk, 0, s>>>(a);
    else k_inv_whole<L1, 0, 1><<<grid, blk, 0, s>>>(a);
  } else {
    if (b4) k_inv_whole<L1, 4, 2><<<grid, blk, 0, s>>>(a);
    else k_inv_whole<L1, 0, 2><<<grid, blk, 0, s>>>(a);
  }
}

// Blocks of up to 2^15 coordinates: the inverse transform in one launch.
template <int L1>
void launch_inv_whole(const InvWholeArgs& a, int efm, bool keep, uint32_t W, hipStream_t s) {
  constexpr int N = inv_whole_threads(L1);
  const dim3 grid((unsigned)((a.lo.d + 16 * N - 1) / (16 * N)), W), blk(N);
  const uint32_t bits = a.lo.src_bits;
  if (efm == 0) {
    if (bits == 8) {
      if (keep) k_inv_whole<L1, 8, 0, KEEP><<<grid, blk, 0, s>>>(a);
      else k_inv_whole<L1, 8, 0><<<grid, blk, 0, s>>>(a);
    } else {
      if (keep) k_inv_whole<L1, 0, 0, KEEP><<<grid, blk, 0, s>>>(a);
      else k_inv_whole<L1, 0, 0><<<grid, blk, 0, s>>>(a);
    }
    return;
  }
  if constexpr (L1 <= LOG_TILE) launch_inv_whole_ef<L1>(a, efm, grid, s);
}

template <int L, Mem OUT>
void launch_big_inv_whole_sums(const InvWholeArgs& a, dim3 grid, hipStream_t s) {
  const dim3 blk(NT);
  if (a.lo.src_bits == 8) {
    k_big_inv_whole<L, 8, 0, OUT><<<grid, blk, 0, s>>>(a);
    return;
  }
  if constexpr (L == 15) {               // 16-bit sums of 2^14-point blocks: k_inv_whole
    if (a.lo.src_bits == 16) {
      k_big_inv_whole<L, 16, 0, OUT><<<grid, blk, 0, s>>>(a);
      return;
    }
  }
  k_big_inv_whole<L, 0, 0, OUT><<<grid, blk, 0, s>>>(a);
}

template <int L>
void launch_big_inv_whole(const InvWholeArgs& a, int efm, bool keep, uint32_t W, hipStream_t s) {
  const dim3 grid((unsigned)((a.lo.d + BIG - 1) >> LOG_BIG), W), blk(NT);
  const uint32_t bits = a.lo.src_bits;
  if (efm == 0) {
    if (keep) launch_big_inv_whole_sums<L, KEEP>(a, grid, s);
    else launch_big_inv_whole_sums<L, STREAM>(a, grid, s);
  } else if (efm == 1) {
    if (bits == 4) k_big_inv_whole<L, 4, 1><<<grid, blk, 0, s>>>(a);
    else k_big_inv_whole<L, 0, 1><<<grid, blk, 0, s>>>(a);
  } else {
    if (bits == 4) k_big_inv_whole<L, 4, 2><<<grid, blk, 0, s>>>(a);
    else k_big_inv_whole<L, 0, 2><<<grid, blk, 0, s>>>(a);
  }
}

// inverse transform of W vectors of `len` coordinates that the first pass is about to produce in `wsx`
void run_inverse(const thc_params* p, const Plan& pl, InvLoArgs lo, float* wsx, InvHiArgs hi, uint64_t len, bool big,
                 uint32_t W, hipStream_t s) {
  const bool keep = hi.mode == 0 && keep_estimate(p->d, pl.L);
  if (big) {
    BigInvLoArgs a{lo.src, lo.range_M, lo.range_m, wsx, len, lo.L, lo.src_bits, lo.use_table, lo.divisor, {}};
    std::memcpy(a.table, lo.table, 256);
    launch_big_inv_lo(pl, a, W, s);
    const BigInvHiArgs h{wsx, hi.out, hi.grad, len, hi.j0,
                         walk_over(hi.mode == 1 && last_first(pl, len, W, true, true), len >> LOG_BIG, W), hi.round, hi.k0, hi.k1,
                         (float)(1.0 / std::sqrt((double)p->block))};
    dispatch_big<LaunchBigInvHi>(pl.L - LOG_BIG, h, pl.split, hi.mode == 0 ? 0 : hi.bf16 ? 2 : 1, keep, W, s);
    return;
  }
  lo.tm = lo_tilemap(pl, len);
  lo.ws_x = wsx;
  lo.d = len;
  if (pl.L <= LOG_BIG) {
    const InvWholeArgs a{lo, hi.out, hi.grad, hi.j0, hi.round, hi.k0, hi.k1, (float)(1.0 / std::sqrt((double)p->block))};
    const int efm = hi.mode == 0 ? 0 : hi.bf16 ? 2 : 1;
    switch (pl.L) {
      case 10: launch_inv_whole<10>(a, efm, keep, W, s); break;
      case 11: launch_inv_whole<11>(a, efm, keep, W, s); break;
      case 12: launch_inv_whole<12>(a, efm, keep, W, s); break;
      case 13: launch_inv_whole<13>(a, efm, keep, W, s); break;
      case 14:
        if (inv_whole_14(len, efm != 0, lo.src_bits)) launch_inv_whole<14>(a, efm, keep, W, s);
        else launch_big_inv_whole<14>(a, efm, keep, W, s);
        break;
      default: launch_big_inv_whole<15>(a, efm, keep, W, s); break;
    }
    return;
  }
  launch_inv_lo(pl, lo, tiles_of(len), W, s);
  run_mids(pl, wsx, len, W, s);
  hi.x = wsx;
  hi.d = len;
  hi.walk = walk_over(hi.mode == 1 && last_first(pl, len, W, true, false), tiles_of(len), W);
  hi.tm = pl.hi;
  hi.c = (float)(1.0 / std::sqrt((double)p->block));
  switch (pl.R) {   // blocks of 2^16 and more: 3 bits at least
    case 3: LaunchInvHi<3>::run(hi, keep, tiles_of(len), W, s); break;
    case 4: LaunchInvHi<4>::run(hi, keep, tiles_of(len), W, s); break;
    case 5: LaunchInvHi<5>::run(hi, keep, tiles_of(len), W, s); break;
    case 6: LaunchInvHi<6>::run(hi, keep, tiles_of(len), W, s); break;
    case 7: LaunchInvHi<7>::run(hi, keep, tiles_of(len), W, s); break;
    case 8: LaunchInvHi<8>::run(hi, keep, tiles_of(len), W, s); break;
    default: LaunchInvHi<9>::run(hi, keep, tiles_of(len), W, s); break;
  }
}

// Worker side of one round (Alg. 3) for W co-resident vectors.  Blocks of up to 2^14 go block by block where whole_route says
// so; else the passes, group by group:
//   first pass (x = grad + e, diagonal, 13 stages; with `range_out` also the norms) -> [range] -> middle passes ->
//   last pass + quantizer -> [error feedback: indices -> inverse first pass -> middle passes -> inverse last pass].
// Every kernel of a group covers all W vectors (grid.y), so a group costs the same number of launches for any W.
struct Forward {
  const thc_params* p;
  uint64_t round;
  uint32_t W;                  // vectors in the call
  uint32_t worker0;            // worker id of vector 0 (vector i is worker worker0 + i)
  const void* const* grads;    // W device pointers
  float* const* efs;           // W device pointers, or null: no error feedback
  float* range_out;            // not null: M_k from the W vectors' norms, written here and used
  const float* range_in;       // used when range_out is null
  uint8_t* const* packed;      // W device pointers
  void* ws;
  hipStream_t s;
};

template <int R>
void launch_pipe_forward(const PipeArgs& a, bool bf16, bool ef, unsigned grid, hipStream_t s) {
  if (bf16) {
    if (ef) k_pipe_forward<R, true, true><<<dim3(grid), dim3(NT), 0, s>>>(a);
    else k_pipe_forward<R, true, false><<<dim3(grid), dim3(NT), 0, s>>>(a);
  } else {
    if (ef) k_pipe_forward<R, false, true><<<dim3(grid), dim3(NT), 0, s>>>(a);
    else k_pipe_forward<R, false, false><<<dim3(grid), dim3(NT), 0, s>>>(a);
  }
}

// The whole sweep as one launch (plus a small one that clears the counters).
void run_forward_pipe(const Forward& f, const Plan& pl, const PipeShape& sh) {
  const thc_params* p = f.p;
  const bool bf16 = p->in_dtype == THC_DTYPE_BF16, ef = f.efs != nullptr;
  const WsLayout wl = ws_layout(f.ws, p, pl, ef);
  const uint32_t K = (uint32_t)(p->d / p->block);

  PipeSetupArgs su{};
  su.sync = wl.sync;
  su.nsync = (uint64_t)K * SYNC_PER_UNIT;
  su.status = wl.status;
  su.lut_out = wl.lut;
  fill_lut(p, su.lut);
  const unsigned setup_grid = (unsigned)((su.nsync + 4095) / 4096);
  k_pipe_setup<<<dim3(setup_grid ? setup_grid : 1), dim3(256), 0, f.s>>>(su);

  PipeArgs a{};
  for (uint32_t i = 0; i < f.W; ++i) {
    a.grads.p[i] = f.grads[i];
    if (ef) a.efs.p[i] = f.efs[i];
    a.packed.p[i] = f.packed[i];
  }
  a.ring = wl.ring;
  a.partials = wl.partials;
  a.pstride = p->d >> pl.L1;
  a.range_M = f.range_out ? f.range_out : const_cast<float*>(f.range_in);
  a.lut = wl.lut;
  a.sync = wl.sync;
  a.status = wl.status;
  a.d = p->d;
  a.j0 = base_coord(p);
  a.lo_tm = pl.lo;
  a.hi_tm = pl.hi;
  a.L = (uint32_t)pl.L;
  a.W = f.W;
  a.K = K;
  a.slots = sh.slots;
  a.lag = sh.lag;
  a.nphase = sh.nphase;
  a.compute_range = f.range_out ? 1u : 0u;
  a.b = p->b;
  a.g = p->g;
  a.round = (uint32_t)f.round;
  a.worker0 = f.worker0;
  a.k0 = (uint32_t)p->seed;
  a.k1 = (uint32_t)(p->seed >> 32);
  a.bf16 = bf16;
  a.c = (float)(1.0 / std::sqrt((double)p->block));
  a.t_p = p->t_p;
  std::memcpy(a.table, p->table, 256);
  const uint64_t Tu = (uint64_t)f.W << pl.R;
  const uint64_t steps = (uint64_t)K + (uint64_t)(sh.nphase - 1) * sh.lag;
  const uint64_t grid = steps * ((Tu >> 3) * sh.nphase + 1) * 8;
  switch (pl.R) {
    case 4: launch_pipe_forward<4>(a, bf16, ef, (unsigned)grid, f.s); break;
    case 5: launch_pipe_forward<5>(a, bf16, ef, (unsigned)grid, f.s); break;
    case 6: launch_pipe_forward<6>(a, bf16, ef, (unsigned)grid, f.s); break;
    case 7: launch_pipe_forward<7>(a, bf16, ef, (unsigned)grid, f.s); break;
    case 8: launch_pipe_forward<8>(a, bf16, ef, (unsigned)grid, f.s); break;
    default: launch_pipe_forward<9>(a, bf16, ef, (unsigned)grid, f.s); break;
  }
}

template <int L, bool BF16>
void launch_whole_k(const WholeArgs& a, bool ef, bool find, bool stream, dim3 grid, hipStream_t s) {
  const dim3 blk(WholeTile<L>::N);
  if constexpr (!BF16) {
    if (stream && !find) {
      if (ef) k_whole<L, BF16, true, false, false, STREAM><<<grid, blk, 0, s>>>(a);
      else k_whole<L, BF16, false, false, false, STREAM><<<grid, blk, 0, s>>>(a);
      return;
    }
  }
  if (ef) k_whole<L, BF16, true, false><<<grid, blk, 0, s>>>(a);
  else if (find) k_whole<L, BF16, false, true><<<grid, blk, 0, s>>>(a);
  else k_whole<L, BF16, false, false><<<grid, blk, 0, s>>>(a);
}

template <int L>
void launch_whole(const WholeArgs& a, bool bf16, bool ef, bool find, bool split, bool stream, uint32_t W, hipStream_t s) {
  const dim3 grid((unsigned)((a.d + (1ull << WholeTile<L>::LOG) - 1) >> WholeTile<L>::LOG), W);
  if constexpr (L == 14) {
    if (find && split) {
      const dim3 twice(2 * grid.x, W), blk(WholeTile<L>::N);
      if (bf16) k_whole<L, true, false, true, true><<<twice, blk, 0, s>>>(a);
      else k_whole<L, false, false, true, true><<<twice, blk, 0, s>>>(a);
      return;
    }
  }
  if (bf16) launch_whole_k<L, true>(a, ef, find, stream, grid, s);
  else launch_whole_k<L, false>(a, ef, find, stream, grid, s);
}

// the norms of `len` coordinates, from x0 on, of W vectors and their range (Alg. 3's preliminary stage)
void run_norms(const thc_params* p, const Plan& pl, const void* const* grads, const float* const* ef, uint32_t W, uint64_t x0,
               uint64_t len, float* range_M, double* partials, hipStream_t s) {
  const bool bf16 = p->in_dtype == THC_DTYPE_BF16;
  FwdLoArgs a{};
  for (uint32_t i = 0; i < W; ++i) {
    a.grads.p[i] = static_cast<const char*>(grads[i]) + x0 * (bf16 ? 2 : 4);
    if (ef) a.efs.p[i] = ef[i] + x0;
  }
  a.partials = partials;
  a.pstride = len >> pl.L1;
  a.d = len;
  a.tm = lo_tilemap(pl, len);
  launch_fwd_lo(pl, a, bf16, ef != nullptr, true, stream_norms(pl, len, W, bf16, ef != nullptr), tiles_of(len), W, s);
  launch_range(RangeArgs{partials, range_M + x0 / p->block, a.pstride, len, W, (uint32_t)pl.L, (uint32_t)pl.L1, p->t_p}, s);
}

// Blocks of up to 2^14, block by block: nothing of the vectors goes through the workspace.
void run_forward_whole(const Forward& f, const Plan& pl, Whole route) {
  const thc_params* p = f.p;
  const bool bf16 = p->in_dtype == THC_DTYPE_BF16, ef = f.efs != nullptr, find = route == Whole::FIND;
  float* const range_M = f.range_out ? f.range_out : const_cast<float*>(f.range_in);
  WholeArgs a{};
  a.L = (uint32_t)pl.L;
  a.b = p->b;
  a.g = p->g;
  a.round = (uint32_t)f.round;
  a.worker = f.worker0;
  a.k0 = (uint32_t)p->seed;
  a.k1 = (uint32_t)(p->seed >> 32);
  a.n = f.W;
  a.c = (float)(1.0 / std::sqrt((double)p->block));
  a.t_p = p->t_p;
  fill_lut(p, a.lut);
  std::memcpy(a.table, p->table, 256);
  for_pieces(p->d, [&](uint64_t x0, uint64_t len) {
    if (route == Whole::NORMS)
      run_norms(p, pl, f.grads, f.efs, f.W, x0, len, range_M, ws_layout(f.ws, p, pl, ef).partials, f.s);
    for (uint32_t i = 0; i < f.W; ++i) {
      a.grads.p[i] = static_cast<const char*>(f.grads[i]) + x0 * (bf16 ? 2 : 4);
      if (ef) a.efs.p[i] = f.efs[i] + x0;
      a.packed.p[i] = f.packed[i] + x0 / 8 * p->b;
    }
    a.range_M = range_M + x0 / p->block;
    a.d = len;
    const bool stream = stream_blocks(len, f.W, bf16), split = whole_split(pl, tiles_of(len), f.W);
    a.j0 = base_coord(p) + x0;
    switch (pl.L) {
      case 10: launch_whole<10>(a, bf16, ef, find, split, stream, f.W, f.s); break;
      case 11: launch_whole<11>(a, bf16, ef, find, split, stream, f.W, f.s); break;
      case 12: launch_whole<12>(a, bf16, ef, find, split, stream, f.W, f.s); break;
      case 13: launch_whole<13>(a, bf16, ef, find, split, stream, f.W, f.s); break;
      default: launch_whole<14>(a, bf16, ef, find, split, stream, f.W, f.s); break;
    }
  });
}

void run_forward(const Forward& f) {
  const thc_params* p = f.p;
  const Plan pl = make_plan(p->block, p->stage_order);
  const Whole route = whole_route(pl, tiles_of(p->d), f.W, f.efs != nullptr, f.range_out == nullptr);
  if (route != Whole::NO) {
    run_forward_whole(f, pl, route);
    return;
  }
  {
    const PipeShape sh = pipe_shape(p, pl, f.W, f.efs != nullptr);
    const uint64_t Tu = (uint64_t)f.W << pl.R;
    const uint64_t grid = ((uint64_t)(p->d / p->block) + (uint64_t)(sh.nphase - 1) * sh.lag) * ((Tu >> 3) * sh.nphase + 1) * 8;
    if (sh.ok && grid < (1ull << 31)) {
      run_forward_pipe(f, pl, sh);
      return;
    }
  }
  const bool bf16 = p->in_dtype == THC_DTYPE_BF16;
  const size_t in_size = bf16 ? 2 : 4;
  const GroupWalk walk = walk_coords(p, f.W, false);
  const WsLayout wl = ws_layout(f.ws, p, pl, f.efs != nullptr);
  float* const slot = wl.ring;
  double* const partials = wl.partials;
  const float* const range = f.range_out ? f.range_out : f.range_in;

  QuantArgs q{};
  q.tm = pl.hi;
  q.L = (uint32_t)pl.L;
  q.b = p->b;
  q.g = p->g;
  q.round = (uint32_t)f.round;
  q.worker = f.worker0;
  q.k0 = (uint32_t)p->seed;
  q.k1 = (uint32_t)(p->seed >> 32);
  q.c = (float)(1.0 / std::sqrt((double)p->block));
  fill_lut(p, q.lut);   // per grid cell k: the largest index z0 with T[z0] <= k, its value and the gap to the next
  InvLoArgs ilo{};
  InvHiArgs ihi{};
  if (f.efs) {
    ilo.L = (uint32_t)pl.L;
    ilo.src_bits = p->b;
    ilo.use_table = 1;
    ilo.divisor = p->g;
    std::memcpy(ilo.table, p->table, 256);
    ihi.round = (uint32_t)f.round;
    ihi.k0 = q.k0;
    ihi.k1 = q.k1;
    ihi.mode = 1;
    ihi.bf16 = bf16;
  }
  for_groups(pl, p->d, walk.most, f.W, [&](uint64_t x0, uint64_t len, bool big, bool inv_big) {
    const uint64_t tiles = tiles_of(len);
    FwdLoArgs a{};
    for (uint32_t i = 0; i < f.W; ++i) {
      a.grads.p[i] = static_cast<const char*>(f.grads[i]) + x0 * in_size;
      if (f.efs) a.efs.p[i] = f.efs[i] + x0;
      q.packed.p[i] = f.packed[i] + x0 / 8 * p->b;
      if (f.efs) {
        ilo.src.p[i] = q.packed.p[i];
        ihi.out.p[i] = f.efs[i] + x0;
        ihi.grad.p[i] = a.grads.p[i];
      }
    }
    a.ws_x = slot;
    a.partials = f.range_out ? partials + (x0 >> pl.L1) : nullptr;
    a.pstride = p->d >> pl.L1;
    a.d = len;
    a.j0 = base_coord(p) + x0;
    a.round = (uint32_t)f.round;
    a.k0 = q.k0;
    a.k1 = q.k1;
    q.range_M = range + x0 / p->block;
    q.j0 = a.j0;
    if (big) {
      const BigLoArgs bl{a.grads, a.efs, slot, a.partials, a.pstride, len, a.j0, a.round, a.k0, a.k1};
      launch_big_lo(pl, bl, bf16, f.efs != nullptr, f.W, f.s);
    } else {
      a.tm = lo_tilemap(pl, len);
      launch_fwd_lo(pl, a, bf16, f.efs != nullptr, false, stream_inputs(len, f.W, bf16, f.efs != nullptr), tiles, f.W, f.s);
    }
    const bool find = f.range_out && !big && find_range(pl, tiles, f.W);
    if (f.range_out && !find) {
      RangeArgs r{a.partials, f.range_out + x0 / p->block, a.pstride, len, f.W, (uint32_t)pl.L, (uint32_t)pl.L1, p->t_p};
      launch_range(r, f.s);
    }
    if (big) {
      BigQuantArgs bq{slot, q.range_M, q.packed, len, q.j0,
                      walk_over(last_first(pl, len, f.W, f.efs != nullptr, true), len >> LOG_BIG, f.W), q.b, q.g, q.round,
                      q.worker, q.k0, q.k1, q.c, {}};
      std::memcpy(bq.lut, q.lut, sizeof q.lut);
      dispatch_big<LaunchBigQuant>(pl.L - LOG_BIG, bq, pl.split, f.W, f.s);
    } else {
      run_mids(pl, slot, len, f.W, f.s);
      q.x = slot;
      q.d = len;
      q.walk = walk_over(last_first(pl, len, f.W, f.efs != nullptr, false), tiles, f.W);
      q.partials = find ? a.partials : nullptr;
      q.pstride = a.pstride;
      q.range_out = find ? f.range_out + x0 / p->block : nullptr;
      q.n = f.W;
      q.t_p = p->t_p;
      dispatch_0_9<LaunchQuant>(pl.R, q, (pl.L & 1) == 0, tiles, f.W, f.s);
    }
    if (f.efs) {
      // e <- (grad + e) - RHT^-1(X_i): the group's slot is free again and takes the inverse's intermediate
      ilo.range_M = q.range_M;
      ihi.j0 = a.j0;
      run_inverse(p, pl, ilo, slot, ihi, len, inv_big, f.W, f.s);
    }
  }, walk.unit);
}

template <Mem LOAD>
void launch_minmax(const MinMaxArgs& a, bool bf16, bool ef, uint32_t W, hipStream_t s) {
  const dim3 grid((unsigned)tiles_of(a.d), W), blk(NT);
  if (bf16) {
    if (ef) k_minmax<true, true, LOAD><<<grid, blk, 0, s>>>(a);
    else k_minmax<true, false, LOAD><<<grid, blk, 0, s>>>(a);
  } else {
    if (ef) k_minmax<false, true, LOAD><<<grid, blk, 0, s>>>(a);
    else k_minmax<false, false, LOAD><<<grid, blk, 0, s>>>(a);
  }
}

template <bool BF16, int G>
void launch_uniform_quant_g(const UQuantArgs& q, bool ef, hipStream_t s) {
  const dim3 grid((unsigned)((q.d + (G << LOG_UTILE) - 1) / (G << LOG_UTILE))), blk(NT);
  if (ef) k_uniform_quant<BF16, true, G><<<grid, blk, 0, s>>>(q);
  else k_uniform_quant<BF16, false, G><<<grid, blk, 0, s>>>(q);
}

template <bool BF16>
void launch_uniform_quant(const UQuantArgs& q, bool ef, bool one_group, hipStream_t s) {
  if (one_group) launch_uniform_quant_g<BF16, 1>(q, ef, s);
  else launch_uniform_quant_g<BF16, 2>(q, ef, s);
}

// ---- scratch of the entry point that allocates nothing -------------------------------------------------------
// One array per GPU the library's code object is loaded on, held until the process ends.  Its name is a host-side
// stand-in: the device address comes from hipGetSymbolAddress, once per device, with that device current.
constexpr uint64_t STATIC_SCRATCH_FLOATS = 1ull << 23;   // 32 MB
static __device__ __align__(256) float g_static_scratch[STATIC_SCRATCH_FLOATS];

constexpr int MAX_DEVICES = 64;
float* g_scratch_ptr[MAX_DEVICES] = {};

int static_scratch(float** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return THC_ELAUNCH;
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_static_scratch));
    if (e != hipSuccess || !ptr) {
      std::fprintf(stderr, "libthc: hipGetSymbolAddress failed: %s\n", hipGetErrorString(e));
      return THC_ELAUNCH;
    }
    g_scratch_ptr[dev] = static_cast<float*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return THC_OK;
}

// ---- aggregation ----------------------------------------------------------------------------------------------
template <Mem M>
int run_aggregate(const thc_params* p, const uint8_t* const* packed, uint8_t* out, hipStream_t s) {
  const dim3 blk(256);
  auto fill = [&](auto& a, uint32_t per_thread) {
    for (uint32_t i = 0; i < p->n; ++i) a.packed.p[i] = packed[i];
    a.out = out;
    a.nvec = p->d / per_thread;
    a.n = p->n;
    return dim3((unsigned)((a.nvec + 255) / 256));
  };
  if (p->b == 4 && p->agg_bits == 8) {
    AggB4Args a{};
    const dim3 grid = fill(a, 32);
    std::memcpy(a.tb, p->table, 16);
    k_aggregate_b4w8<M><<<grid, blk, 0, s>>>(a);
  } else if (p->b == 2 && p->agg_bits == 8) {
    AggB2Args a{};
    const dim3 grid = fill(a, 64);
    std::memcpy(&a.tb, p->table, 4);
    k_aggregate_b2w8<M><<<grid, blk, 0, s>>>(a);
  } else if (p->b == 4) {
    AggB4WxArgs a{};
    const dim3 grid = fill(a, 32);
    a.chunk = 255u / p->g;              // g <= 255, so at least one worker per run
    std::memcpy(a.tb, p->table, 16);
    switch (p->agg_bits) {
#define THC_AGG_WX(W)                                                                         \
  case W:                                                                                     \
    if (M == KEEP || sums_four_loads(p->d)) k_aggregate_b4wx<W, M, true><<<grid, blk, 0, s>>>(a); \
    else k_aggregate_b4wx<W, M, M == KEEP><<<grid, blk, 0, s>>>(a);                           \
    break;
      THC_AGG_WX(4) THC_AGG_WX(5) THC_AGG_WX(6) THC_AGG_WX(7) THC_AGG_WX(9) THC_AGG_WX(10) THC_AGG_WX(11)
      THC_AGG_WX(12) THC_AGG_WX(13) THC_AGG_WX(14) THC_AGG_WX(15) THC_AGG_WX(16)
#undef THC_AGG_WX
      default: return THC_EINVAL;       // 4-bit tables reach at least g = 15: the sums need 4 bits or more
    }
  } else {
    AggArgs a{};
    const dim3 grid = fill(a, 32);
    a.agg_bits = p->agg_bits;
    a.chunk = 255u / p->g;              // g <= 255, so at least one worker per run
    std::memcpy(a.tb, p->table, 8);
    std::memcpy(a.table, p->table, 256);
    switch (p->b) {
#define THC_AGG_ANY(B) case B: k_aggregate_any<B, M><<<grid, blk, 0, s>>>(a); break;
      THC_AGG_ANY(1) THC_AGG_ANY(2) THC_AGG_ANY(3) THC_AGG_ANY(5) THC_AGG_ANY(6) THC_AGG_ANY(7) THC_AGG_ANY(8)
#undef THC_AGG_ANY
      default: return THC_EINVAL;       // 4-bit indices have kernels of their own
    }
  }
  return check_launch();
}

const char* const kNames[] = {"THC_OK", "THC_EINVAL", "THC_ETABLE", "THC_EOVERFLOW", "THC_EUNSUPPORTED", "THC_ELAUNCH"};

}  // namespace

extern "C" {

int thc_version(void) { return 200; }

const char* thc_strerror(int status) {
  const int i = -status;
  return (i >= 0 && i <= 5) ? kNames[i] : "THC_E?";
}

int thc_workspace_bytes(const thc_params* p, int ef_enabled, size_t* bytes_out) {
  const int rc = validate(p);
  if (rc) return rc;
  if (!bytes_out) return THC_EINVAL;
  const Plan pl = make_plan(p->block, p->stage_order);
  *bytes_out = ws_layout(nullptr, p, pl, ef_enabled != 0).bytes;
  return THC_OK;
}

int thc_describe_plan(const thc_params* p, uint32_t* out, size_t cap_records) {
  const int rc = validate(p);
  if (rc) return rc;
  const Plan pl = make_plan(p->block, p->stage_order);
  if (!pl.ok()) return THC_EUNSUPPORTED;
  const int npass = 2 + pl.nmid;
  if (!out) return npass;
  if (cap_records < (size_t)npass) return THC_EINVAL;
  auto put = [&](int rec, uint32_t kind, const int* bits, int nbits, const TileMap& m) {
    uint32_t* r = out + (size_t)rec * THC_PLAN_RECORD_WORDS;
    std::fill(r, r + THC_PLAN_RECORD_WORDS, 0xFFFFFFFFu);
    r[0] = kind;
    r[1] = (uint32_t)nbits;
    for (int i = 0; i < nbits; ++i) r[2 + i] = (uint32_t)bits[i];
    const uint32_t tm[19] = {m.L, m.logw, m.nrows, m.nfixed, m.n0, m.sh0, m.sh1, m.fcum[0], m.fcum[1], m.fcum[2],
                             m.fcum[3], m.fmask[0], m.fmask[1], m.fmask[2], m.fmask[3], m.fpos[0], m.fpos[1],
                             m.fpos[2], m.fpos[3]};
    std::copy(tm, tm + 19, r + 18);
  };
  int first[16];
  for (int i = 0; i < pl.L1; ++i) first[i] = (pl.split && i >= 10) ? i + 3 : i;
  put(0, pl.split ? 3u : 0u, first, pl.L1, lo_tilemap(pl, walk_coords(p, p->n, false).most));
  for (int m = 0; m < pl.nmid; ++m) put(1 + m, 1u, pl.bits[m], pl.mid[m], pl.midmap[m]);
  put(npass - 1, 2u, pl.bits[pl.nmid], pl.R, pl.hi);
  return npass;
}

namespace {

int check_vectors(const thc_params* p, const void* const* grads, const float* const* ef) {
  if (!grads) return THC_EINVAL;
  for (uint32_t i = 0; i < p->n; ++i) {
    if (!grads[i] || !aligned16(grads[i])) return THC_EINVAL;
    if (ef && (!ef[i] || !aligned16(ef[i]))) return THC_EINVAL;
  }
  return THC_OK;
}

}  // namespace

int thc_prepare_range(const thc_params* p, const void* const* grads, const float* const* ef, float* range_M, void* ws,
                      void* stream) {
  const int rc = validate(p);
  if (rc) return rc;
  if (!ws || !aligned16(ws) || !range_M || (reinterpret_cast<uintptr_t>(range_M) & 3u)) return THC_EINVAL;
  const int rv = check_vectors(p, grads, ef);
  if (rv) return rv;
  const Plan pl = make_plan(p->block, p->stage_order);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // The same partial sums, in the same order, as the first pass of thc_compress_all takes them group by group, on tiles
  // of either size and in the single launch: all give the same M bit for bit.
  run_norms(p, pl, grads, ef, p->n, 0, p->d, range_M, ws_layout(ws, p, pl, false).partials, s);
  return check_launch();
}

int thc_compress(const thc_params* p, uint32_t worker_id, uint64_t round, const void* grad, float* ef_inout,
                 const float* range_M, uint8_t* packed_out, void* ws, void* stream) {
  const int rc = validate(p);
  if (rc) return rc;
  if (worker_id >= p->n || round >> 32 || !range_M || !packed_out || !ws || !grad) return THC_EINVAL;
  if (!aligned16(packed_out) || !aligned16(ws) || !aligned16(grad)) return THC_EINVAL;
  if (ef_inout && !aligned16(ef_inout)) return THC_EINVAL;
  Forward f{p, round, 1, worker_id, &grad, ef_inout ? &ef_inout : nullptr, nullptr, range_M, &packed_out, ws,
            static_cast<hipStream_t>(stream)};
  run_forward(f);
  return check_launch();
}

int thc_compress_all(const thc_params* p, uint64_t round, const void* const* grads, float* const* ef_inout,
                     float* range_M, uint8_t* const* packed_out, void* ws, void* stream) {
  const int rc = validate(p);
  if (rc) return rc;
  if (round >> 32 || !ws || !aligned16(ws) || !range_M || (reinterpret_cast<uintptr_t>(range_M) & 3u) || !packed_out)
    return THC_EINVAL;
  const int rv = check_vectors(p, grads, ef_inout);
  if (rv) return rv;
  for (uint32_t i = 0; i < p->n; ++i)
    if (!packed_out[i] || !aligned16(packed_out[i])) return THC_EINVAL;
  Forward f{p, round, p->n, 0, grads, ef_inout, range_M, nullptr, packed_out, ws, static_cast<hipStream_t>(stream)};
  run_forward(f);
  return check_launch();
}

int thc_aggregate(const thc_params* p, const uint8_t* const* packed, void* agg_out, void* stream) {
  const int rc = validate(p);
  if (rc) return rc;
  if (!packed || !agg_out || !aligned16(agg_out)) return THC_EINVAL;
  for (uint32_t i = 0; i < p->n; ++i)
    if (!packed[i] || !aligned16(packed[i])) return THC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (stream_sums(p->d, p->n, p->b)) return run_aggregate<STREAM>(p, packed, static_cast<uint8_t*>(agg_out), s);
  return run_aggregate<KEEP>(p, packed, static_cast<uint8_t*>(agg_out), s);
}

namespace {

// m + (Y/n)(M-m)/g and the inverse RHT, group by group through `slot` (room for `walk.most` coordinates, whole blocks)
void run_decompress(const thc_params* p, const Plan& pl, uint64_t round, const void* agg, const float* range_M,
                    float* out, float* slot, GroupWalk walk, hipStream_t s) {
  InvLoArgs lo{};
  lo.L = (uint32_t)pl.L;
  lo.src_bits = p->agg_bits;
  lo.use_table = 0;
  lo.divisor = p->g * p->n;
  InvHiArgs hi{};
  hi.round = (uint32_t)round;
  hi.k0 = (uint32_t)p->seed;
  hi.k1 = (uint32_t)(p->seed >> 32);
  hi.mode = 0;
  for_groups(pl, p->d, walk.most, 1, [&](uint64_t x0, uint64_t len, bool, bool big) {
    lo.src.p[0] = static_cast<const uint8_t*>(agg) + x0 / 8 * p->agg_bits;
    lo.range_M = range_M + x0 / p->block;
    hi.out.p[0] = out + x0;
    hi.j0 = base_coord(p) + x0;
    run_inverse(p, pl, lo, slot, hi, len, big, 1, s);
  }, walk.unit);
}

}  // namespace

int thc_decompress(const thc_params* p, uint64_t round, const void* agg, const float* range_M, float* out,
                   void* ws, void* stream) {
  const int rc = validate(p);
  if (rc) return rc;
  if (round >> 32 || !agg || !range_M || !out || !ws) return THC_EINVAL;
  if (!aligned16(agg) || !aligned16(out) || !aligned16(ws)) return THC_EINVAL;
  const Plan pl = make_plan(p->block, p->stage_order);
  run_decompress(p, pl, round, agg, range_M, out, ws_layout(ws, p, pl, false).ring, walk_coords(p, 1, true),
                 static_cast<hipStream_t>(stream));
  return check_launch();
}

int thc_decompress_noalloc(const thc_params* p, uint64_t round, const void* agg, const float* range_M, float* out,
                           void* stream) {
  const int rc = validate(p);
  if (rc) return rc;
  if (round >> 32 || !agg || !range_M || !out) return THC_EINVAL;
  if (!aligned16(agg) || !aligned16(out)) return THC_EINVAL;
  if (p->block > STATIC_SCRATCH_FLOATS) {
    std::fprintf(stderr, "libthc: thc_decompress_noalloc takes blocks of at most %llu coordinates (got %llu)\n",
                 (unsigned long long)STATIC_SCRATCH_FLOATS, (unsigned long long)p->block);
    return THC_EUNSUPPORTED;
  }
  float* scratch = nullptr;
  const int rs = static_scratch(&scratch);
  if (rs) return rs;
  const Plan pl = make_plan(p->block, p->stage_order);
  uint64_t gc = STATIC_SCRATCH_FLOATS / p->block * p->block;   // whole blocks that fit the scratch array
  if (gc > p->d) gc = p->d;
  run_decompress(p, pl, round, agg, range_M, out, scratch, {gc, 0}, static_cast<hipStream_t>(stream));
  return check_launch();
}

// ---- uniform THC (Alg. 1) -----------------------------------------------------------------------

namespace {

int validate_uniform(const thc_params* p) {
  const int rc = validate(p);
  if (rc) return rc;
  if (p->g != (1u << p->b) - 1) return THC_ETABLE;     // identity table: T[z] = z (checked by validate: strictly increasing 0..g)
  return THC_OK;
}

// Workspace of the uniform entry points: with rotation the half-rotated vectors of all n workers (n*d binary32
// values, kept from thc_uniform_prepare_range to thc_uniform_compress), then per-tile minima and maxima.
size_t uni_x_bytes(const thc_params* p, int rotate) { return rotate ? (size_t)p->n * (size_t)p->d * sizeof(float) : 0; }

float* pmin_of(const thc_params* p, int rotate, void* ws) {
  return reinterpret_cast<float*>(static_cast<char*>(ws) + uni_x_bytes(p, rotate));
}

}  // namespace

int thc_uniform_workspace_bytes(const thc_params* p, int rotate, size_t* bytes_out) {
  const int rc = validate_uniform(p);
  if (rc) return rc;
  if (!bytes_out) return THC_EINVAL;
  const Plan pl = make_plan(p->block, p->stage_order);
  *bytes_out = uni_x_bytes(p, rotate) + partial_count(p, pl) * 2 * sizeof(float) + 256;
  return THC_OK;
}

int thc_uniform_prepare_range(const thc_params* p, uint64_t round, const void* const* grads, const float* const* ef,
                              int rotate, float* range_m, float* range_M, void* ws, void* stream) {
  const int rc = validate_uniform(p);
  if (rc) return rc;
  if (!grads || !ws || !aligned16(ws) || round >> 32 || !range_m || !range_M) return THC_EINVAL;
  for (uint32_t i = 0; i < p->n; ++i) {
    if (!grads[i] || !aligned16(grads[i])) return THC_EINVAL;
    if (ef && (!ef[i] || !aligned16(ef[i]))) return THC_EINVAL;
  }
  const Plan pl = make_plan(p->block, p->stage_order);
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* pmin = pmin_of(p, rotate, ws);
  float* pmax = pmin + partial_count(p, pl);
  const bool bf16 = p->in_dtype == THC_DTYPE_BF16;
  if (rotate) {
    // every worker's forward RHT up to its last pass, kept in the workspace, and the range of what that pass gives
    FwdLoArgs a{};
    for (uint32_t i = 0; i < p->n; ++i) {
      a.grads.p[i] = grads[i];
      if (ef) a.efs.p[i] = ef[i];
    }
    a.ws_x = static_cast<float*>(ws);
    a.d = p->d;
    a.j0 = base_coord(p);
    a.round = (uint32_t)round;
    a.k0 = (uint32_t)p->seed;
    a.k1 = (uint32_t)(p->seed >> 32);
    a.tm = lo_tilemap(pl, p->d);
    launch_fwd_lo(pl, a, bf16, ef != nullptr, false, stream_inputs(p->d, p->n, bf16, ef != nullptr), tiles_of(p->d), p->n, s);
    run_mids(pl, static_cast<float*>(ws), p->d, p->n, s);
    const HiMinMaxArgs h{static_cast<float*>(ws), pmin, pmax, p->d,
                        walk_over(last_first(pl, p->d, p->n, false, false), tiles_of(p->d), p->n), pl.hi, (uint32_t)pl.L,
                        (float)(1.0 / std::sqrt((double)p->block))};
    dispatch_0_9<LaunchHiMinMax>(pl.R, h, tiles_of(p->d), p->n, s);
  } else {
    MinMaxArgs a{};
    for (uint32_t i = 0; i < p->n; ++i) {
      a.grads.p[i] = grads[i];
      if (ef) a.efs.p[i] = ef[i];
    }
    a.pmin = pmin;
    a.pmax = pmax;
    a.d = p->d;
    a.L1 = (uint32_t)pl.L1;
    if (stream_minmax(p->d, p->n, bf16, ef != nullptr)) launch_minmax<STREAM>(a, bf16, ef != nullptr, p->n, s);
    else launch_minmax<KEEP>(a, bf16, ef != nullptr, p->n, s);
  }
  MinMaxFinalArgs f{pmin, pmax, range_m, range_M, p->d, p->n, (uint32_t)pl.L, (uint32_t)pl.L1};
  k_minmax_final<<<dim3((unsigned)(p->d / p->block)), dim3(64), 0, s>>>(f);
  return check_launch();
}

int thc_uniform_compress(const thc_params* p, uint32_t worker_id, uint64_t round, const void* grad, float* ef_inout,
                         int rotate, const float* range_m, const float* range_M, uint8_t* packed_out, void* ws,
                         void* stream) {
  const int rc = validate_uniform(p);
  if (rc) return rc;
  if (worker_id >= p->n || round >> 32 || !range_m || !range_M || !packed_out || !aligned16(packed_out)) return THC_EINVAL;
  if (rotate && (!ws || !aligned16(ws))) return THC_EINVAL;
  if (!rotate && (!grad || !aligned16(grad))) return THC_EINVAL;
  if (ef_inout && (!grad || !aligned16(grad) || !aligned16(ef_inout))) return THC_EINVAL;
  const Plan pl = make_plan(p->block, p->stage_order);
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* wsx = rotate ? static_cast<float*>(ws) + (size_t)worker_id * p->d : nullptr;
  const uint32_t k0 = (uint32_t)p->seed, k1 = (uint32_t)(p->seed >> 32);
  if (rotate) {
    QuantArgs q{};
    q.x = wsx;
    q.range_M = range_M;
    q.range_m = range_m;
    q.packed.p[0] = packed_out;
    q.d = p->d;
    q.j0 = base_coord(p);
    q.tm = pl.hi;
    q.L = (uint32_t)pl.L;
    q.b = p->b;
    q.g = p->g;
    q.round = (uint32_t)round;
    q.worker = worker_id;
    q.k0 = k0;
    q.k1 = k1;
    q.c = (float)(1.0 / std::sqrt((double)p->block));
    fill_lut(p, q.lut);
    dispatch_0_9<LaunchQuant>(pl.R, q, (pl.L & 1) == 0, tiles_of(p->d), 1, s);
  } else {
    UQuantArgs q{};
    q.L = (uint32_t)pl.L;
    q.b = p->b;
    q.g = p->g;
    q.round = (uint32_t)round;
    q.worker = worker_id;
    q.k0 = k0;
    q.k1 = k1;
    fill_lut(p, q.lut);
    const bool bf16 = p->in_dtype == THC_DTYPE_BF16, one = uniform_one_group(p->d, bf16, ef_inout != nullptr);
    for_pieces(p->d, [&](uint64_t x0, uint64_t len) {
      q.grad = static_cast<const char*>(grad) + x0 * (bf16 ? 2 : 4);
      q.ef = ef_inout ? ef_inout + x0 : nullptr;
      q.range_M = range_M + x0 / p->block;
      q.range_m = range_m + x0 / p->block;
      q.packed = packed_out + x0 / 8 * p->b;
      q.d = len;
      q.j0 = base_coord(p) + x0;
      if (bf16) launch_uniform_quant<true>(q, ef_inout != nullptr, one, s);
      else launch_uniform_quant<false>(q, ef_inout != nullptr, one, s);
    });
  }
  if (rotate && ef_inout) {
    // e <- (grad + e) - RHT^-1(X_i): rebuild X_i from the indices, inverse transform, subtract
    InvLoArgs lo{};
    lo.src.p[0] = packed_out;
    lo.range_M = range_M;
    lo.range_m = range_m;
    lo.ws_x = wsx;
    lo.d = p->d;
    lo.L = (uint32_t)pl.L;
    lo.src_bits = p->b;
    lo.use_table = 1;
    lo.divisor = p->g;
    std::memcpy(lo.table, p->table, 256);
    InvHiArgs hi{};
    hi.out.p[0] = ef_inout;
    hi.grad.p[0] = grad;
    hi.round = (uint32_t)round;
    hi.k0 = k0;
    hi.k1 = k1;
    hi.mode = 1;
    hi.bf16 = p->in_dtype == THC_DTYPE_BF16;
    hi.j0 = base_coord(p);
    run_inverse(p, pl, lo, wsx, hi, p->d, big_inverse(pl, p->d, p->d, 1), 1, s);
  }
  return check_launch();
}

int thc_uniform_decompress(const thc_params* p, uint64_t round, const void* agg, int rotate, const float* range_m,
                           const float* range_M, float* out, void* ws, void* stream) {
  const int rc = validate_uniform(p);
  if (rc) return rc;
  if (round >> 32 || !agg || !range_m || !range_M || !out || !aligned16(agg) || !aligned16(out)) return THC_EINVAL;
  if (rotate && (!ws || !aligned16(ws))) return THC_EINVAL;
  const Plan pl = make_plan(p->block, p->stage_order);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!rotate) {
    UDequantArgs a{agg, range_M, range_m, out, p->d, (uint32_t)pl.L, p->agg_bits, p->g * p->n};
    const uint64_t threads = p->d / 16;
    const dim3 grid((unsigned)((threads + 255) / 256)), blk(256);
    if (keep_plain_estimate(p->d)) k_uniform_dequant<KEEP><<<grid, blk, 0, s>>>(a);
    else k_uniform_dequant<STREAM><<<grid, blk, 0, s>>>(a);
    return check_launch();
  }
  float* wsx = static_cast<float*>(ws);
  InvLoArgs lo{};
  lo.src.p[0] = agg;
  lo.range_M = range_M;
  lo.range_m = range_m;
  lo.ws_x = wsx;
  lo.d = p->d;
  lo.L = (uint32_t)pl.L;
  lo.src_bits = p->agg_bits;
  lo.use_table = 0;
  lo.divisor = p->g * p->n;
  InvHiArgs hi{};
  hi.out.p[0] = out;
  hi.round = (uint32_t)round;
  hi.k0 = (uint32_t)p->seed;
  hi.k1 = (uint32_t)(p->seed >> 32);
  hi.mode = 0;
  hi.j0 = base_coord(p);
  run_inverse(p, pl, lo, wsx, hi, p->d, big_inverse(pl, p->d, p->d, 1), 1, s);
  return check_launch();
}

}  // extern "C"
