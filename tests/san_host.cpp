// Host code of the library under AddressSanitizer and UndefinedBehaviorSanitizer (no GPU involved): the table
// solver, its exhaustive cross-check, the threshold, and the pass planner with an emulation of the addressing the
// kernels derive from its tables.  Built and run by tests/test_host_sanitizers.py.
#include <cstdio>
#include <cstdlib>
#include <cmath>
#include <vector>

#include "thc.h"
#include "thc_bigmap.hpp"
#include "thc_plan.hpp"
#include "thc_quant.hpp"

using namespace thc;

static uint64_t tile_base(const TileMap& m, uint32_t tile) {
  const uint32_t tib = tile & ((1u << m.nfixed) - 1u);
  uint32_t off = 0;
  for (int i = 0; i < 4; ++i) off |= ((tib >> m.fcum[i]) & m.fmask[i]) << m.fpos[i];
  return ((uint64_t)(tile >> m.nfixed) << m.L) | off;
}

static uint32_t tile_row(const TileMap& m, uint32_t r) {
  return ((r & ((1u << m.n0) - 1u)) << m.sh0) | ((r >> m.n0) << m.sh1);
}

// every coordinate of a span of 2^L is touched exactly once by the 2^(L-13) tiles of a strided pass
static int check_cover(const TileMap& m, bool first_pass_rows) {
  if (!m.L) return 1;
  const uint64_t span = 1ull << m.L;
  if (span > (1ull << 24)) return 0;                        // keep the run short; the Python test covers the rest
  std::vector<unsigned char> seen(span, 0);
  const uint32_t tiles = 1u << m.nfixed, W = 1u << m.logw;
  for (uint32_t t = 0; t < tiles; ++t) {
    const uint64_t base = tile_base(m, t);
    for (uint32_t idx = 0; idx < 8192; ++idx) {
      uint64_t o;
      if (first_pass_rows) o = (idx & 1023u) | ((uint64_t)(idx >> 10) << 13);
      else o = tile_row(m, idx >> m.logw) + (idx & (W - 1));
      const uint64_t j = base + o;
      if (j >= span || seen[j]) return 1;
      seen[j] = 1;
    }
  }
  return 0;
}

// Tiles of 2^15 coordinates: the tiles of either pass cover a block once, the first does the first 15 bits of the
// stage order and the last pass the rest, each with the row bit it is meant for in the slot index when its turn comes.
template <int R, bool XO, bool SPREAD = false>
static int check_big() {
  using H = BigHi<R, SPREAD>;
  constexpr int L = LOG_BIG + R;
  std::vector<uint32_t> order;                     // offset each stage pairs
  if (XO) {
    for (int b : {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 14, 15, 10, 11, 12}) order.push_back(1u << b);
    for (int b = 16; b < L; ++b) order.push_back(1u << b);
  } else {
    for (int b = 0; b < L; ++b) order.push_back(1u << b);
  }
  int bad = 0;
  for (int i = 0; i < LOG_BIG; ++i) bad += big_p<XO>(1u << i) != order[i];
  for (int i = 0; i < R; ++i) bad += big_q<XO>(1u << i) != order[LOG_BIG + i];
  const BigLayout a = H::first(), b = H::second(), c = H::third(), e = H::last();
  for (int i = 0; i < 3; ++i) bad += a.slot[i] != i || (i < H::E && c.slot[i] != 5 + i);
  bad += b.slot[0] != 3 || b.slot[1] != 4;
  bad += (H::E >= 4 && e.slot[0] != 8) || (H::E >= 5 && e.slot[1] != 9);
  // every map takes bits to bits, so single bits show that the tiles' coordinates are disjoint and complete
  uint64_t lo = 0, hi = 0, out = 0;
  auto add = [&bad](uint64_t& seen, uint64_t bit) { bad += !bit || (bit & (bit - 1)) || (seen & bit); seen |= bit; };
  for (int i = 0; i < LOG_BIG; ++i) add(lo, big_p<XO>(1u << i));
  for (int i = 0; i < R; ++i) {
    add(lo, big_lo_base<XO>(1u << i));
    add(hi, big_hi_base<R, XO>(1u << i));
    add(out, big_hi_base<R, XO>(1u << i));
  }
  for (int i = 0; i < 9; ++i) {
    add(hi, H::template thread_off<XO, 0>(a, 1 << i));
    add(out, H::template thread_off<XO, 0>(e, 1 << i));
  }
  for (int i = 0; i < 3; ++i) {
    add(hi, H::template slot_off<XO>(a, 1 << i));
    add(out, H::template slot_off<XO>(e, 1 << i));
  }
  add(hi, H::template half_off<XO>());
  add(out, H::template half_off<XO>());
  const uint64_t most = (1ull << L) - 4;          // the low two bits are four of a thread's eight columns
  bad += lo != most + 3 || hi != most || out != most;
  return bad + (big_hi_base<R, XO>(3u << R | 1) != (3ull << L) + big_hi_base<R, XO>(1));
}

// a walk covers the vector in whole groups; forward passes pick the tile size by what one launch holds, inverse passes
// by the call, but not where a launch is too short to fill the chip
static int check_groups(uint64_t block, uint64_t d, uint64_t gc, uint32_t W, bool fwd_full, bool inv_full, bool fwd_last,
                        bool inv_last) {
  const Plan pl = make_plan(block, THC_ORDER_SPLIT);
  uint64_t at = 0;
  int bad = 0;
  for_groups(pl, d, gc, W, [&](uint64_t x0, uint64_t len, bool fwd, bool inv) {
    bad += x0 != at || len != (d - x0 < gc ? d - x0 : gc) || fwd != (len == gc ? fwd_full : fwd_last) ||
           inv != (len == gc ? inv_full : inv_last);
    at += len;
  });
  return bad + (at != d);
}

// whole vectors in launches of whole blocks and fewer than 2^32 threads, at eight coordinates a thread or more
static int check_pieces(uint64_t d, int want) {
  uint64_t at = 0;
  int bad = 0, n = 0;
  for_pieces(d, [&](uint64_t x0, uint64_t len) {
    bad += x0 != at || !len || x0 % (1ull << 27) || len / 8 >= (1ull << 32);
    at += len;
    ++n;
  });
  return bad + (at != d) + (n != want);
}

// the order in which workgroups take consecutive tiles leaves none out and takes none twice
template <int S>
static int check_xcd_tile() {
  int bad = 0;
  for (uint32_t n : {1u, 7u, (8u << S) - 1, 8u << S, (8u << S) + 1, 3 * (8u << S) + 5, 4096u}) {
    std::vector<unsigned char> seen(n, 0);
    for (uint32_t wg = 0; wg < n; ++wg) {
      const uint32_t t = xcd_tile<S>(wg, n);
      if (t >= n || seen[t]) { ++bad; break; }
      seen[t] = 1;
    }
    if (n >= 8u << S)
      for (uint32_t x = 0; x < 8; ++x) bad += (xcd_tile<S>(x, n) >> S & 7u) != x;
  }
  return bad;
}

// Both sides of every limit of whole_route: vectors of `tiles` 8192-coordinate tiles, W of them.
static int check_whole_route() {
  const struct { int L; uint32_t W; bool ef; uint64_t tiles; Whole want; } at[] = {
      // no error feedback, up to 2^13
      {10, 1, false, 1, Whole::FIND}, {13, 1, false, 1ull << 20, Whole::FIND}, {13, 2, false, 256, Whole::FIND},
      {13, 2, false, 257, Whole::NORMS}, {10, 4, false, 128, Whole::FIND}, {10, 4, false, 129, Whole::NORMS},
      {12, 5, false, 1, Whole::NO}, {12, 5, false, 102, Whole::NO}, {12, 5, false, 103, Whole::NORMS},
      {13, 8, false, 63, Whole::NO}, {13, 8, false, 64, Whole::NORMS}, {11, 16, false, 39, Whole::NO},
      {11, 16, false, 40, Whole::NORMS}, {13, 10, false, 63, Whole::NO}, {13, 10, false, 64, Whole::NORMS},
      // 2^14: where its two workgroups a compute unit fill the chip evenly, and in large calls
      {14, 1, false, 1024, Whole::FIND}, {14, 1, false, 1026, Whole::NO}, {14, 4, false, 128, Whole::FIND},
      {14, 4, false, 130, Whole::NO}, {14, 4, false, 224, Whole::NO}, {14, 4, false, 226, Whole::NORMS},
      {14, 4, false, 256, Whole::NORMS}, {14, 4, false, 258, Whole::NO}, {14, 4, false, 1022, Whole::NO},
      {14, 4, false, 1024, Whole::NORMS}, {14, 8, false, 56, Whole::NO}, {14, 5, false, 90, Whole::NORMS},
      {14, 8, false, 64, Whole::NORMS}, {14, 8, false, 66, Whole::NO}, {14, 9, false, 56, Whole::NO},
      {14, 16, false, 32, Whole::NO}, {14, 16, false, 56, Whole::NO}, {14, 16, false, 58, Whole::NORMS},
      {14, 16, false, 64, Whole::NORMS}, {14, 16, false, 66, Whole::NO}, {14, 17, false, 60, Whole::NO},
      {14, 32, false, 126, Whole::NO}, {14, 32, false, 128, Whole::NORMS},
      // error feedback
      {10, 1, true, 1, Whole::NORMS}, {13, 64, true, 1000, Whole::NORMS}, {14, 1, true, 512, Whole::NORMS},
      {14, 1, true, 514, Whole::NO}, {14, 8, true, 64, Whole::NORMS}, {14, 8, true, 66, Whole::NO},
      {14, 8, true, 510, Whole::NO}, {14, 8, true, 512, Whole::NORMS},
      {15, 1, false, 4, Whole::NO}, {15, 1, true, 4, Whole::NO}, {20, 8, false, 1024, Whole::NO}};
  int bad = 0;
  for (const auto& c : at) {
    const Plan pl = make_plan(1ull << c.L, THC_ORDER_SPLIT);
    bad += whole_route(pl, c.tiles, c.W, c.ef, false) != c.want;
    bad += whole_route(pl, c.tiles, 1, c.ef, true) != (c.L <= 14 ? Whole::GIVEN : Whole::NO);
  }
  return bad;
}

// ... of the kernel that takes the inverse transform of blocks of 2^14 ...
static int check_inv_whole_14() {
  auto one = [](uint64_t K, bool ef, uint32_t bits) { return inv_whole_14(K << 14, ef, bits); };
  int bad = 0;
  for (uint32_t bits : {1u, 4u, 5u, 8u, 9u, 15u}) {
    const uint64_t a = bits == 4 || bits == 8 ? 640 : 512;
    bad += !one(1, false, bits) || !one(a, false, bits) || one(a + 1, false, bits) || one(1024, false, bits);
    bad += !one(1025, false, bits) || !one(2560, false, bits) || one(2561, false, bits) || one(1ull << 20, false, bits);
  }
  for (uint64_t K : {1ull, 704ull, 705ull, 1024ull, 1025ull, 2048ull, 16384ull})
    bad += !one(K, false, 16) || one(K, true, 4) || one(K, true, 8);
  return bad;
}

// ... and of the walk from the last tile.
static int check_last_first() {
  int bad = 0;
  for (int L : {14, 16, 20, 21, 25}) {
    const Plan pl = make_plan(1ull << L, THC_ORDER_SPLIT);
    const uint64_t B = 1ull << L, a = 1ull << 26, b = 1ull << 25;
    bad += last_first(pl, a, 1, false, false) || !last_first(pl, a + B, 1, false, false);
    bad += last_first(pl, b, 1, true, false) || !last_first(pl, b + B, 1, true, false);
    bad += last_first(pl, b / 8 > B ? b / 8 : B, b / 8 > B ? 8 : b / B, true, false);
    bad += !last_first(pl, b, 2, true, false) || last_first(pl, b, 2, false, false) || !last_first(pl, b, 3, false, false);
    bad += last_first(pl, 4 * a, 8, true, true) != (L == 25);
  }
  return bad;
}

// even shares cover the vector in whole blocks, at least (or at most) the target where that can be
static int check_even_share() {
  int bad = 0;
  for (uint64_t block : {1ull << 15, 1ull << 20, 1ull << 21})
    for (uint32_t W : {1u, 3u, 8u, 64u})
      for (uint64_t K : {1ull, 2ull, 7ull, 41ull, 63ull, 64ull, 65ull, 321ull, 4097ull})
        for (bool most : {false, true}) {
          const uint64_t d = K * block, T = 1ull << 26, s = even_share(d, block, W, T, most);
          const uint64_t unit = block > (1ull << 20) ? block : 1ull << 20;
          bad += !s || s > d || s % block || (s < d && s % (1ull << 19));
          bad += most ? s > unit && W * (s - unit) >= T : s < d && W * s < T;
          bad += W * d < T && s != d;
          bad += W * d >= 2 * T && d >= 4 * unit && s == d;
        }
  return bad + (even_share(20ull << 20, 1ull << 20, 8, 1ull << 27, false) != 20ull << 20) +
         (even_share(41ull << 20, 1ull << 20, 16, 1ull << 27, false) != 9ull << 20) +
         (even_share(100ull << 20, 1ull << 20, 1, 1ull << 26, true) != 50ull << 20);
}

// ... and the walk in them: whole vector, no step above the largest share, all of them within a unit of each other but for the
// last one's rest of a unit
static int check_even_walk() {
  int bad = 0;
  for (uint64_t block : {1ull << 16, 1ull << 20, 1ull << 21}) {
    const Plan pl = make_plan(block, THC_ORDER_SPLIT);
    for (uint32_t W : {1u, 3u, 8u, 16u, 24u, 64u})
      for (uint64_t K : {1ull, 2ull, 7ull, 41ull, 43ull, 73ull, 273ull, 321ull, 4097ull})
        for (bool most : {false, true}) {
          const uint64_t d = K * block, unit = share_unit(block), s = even_share(d, block, W, 1ull << 27, most);
          uint64_t at = 0, least = ~0ull, steps = 0;
          for_groups(pl, d, s, W, [&](uint64_t x0, uint64_t len, bool, bool) {
            bad += x0 != at || !len || len > s || len % block;
            at += len;
            const uint64_t units = (len + unit - 1) / unit;
            least = units < least ? units : least;
            ++steps;
          }, unit);
          bad += at != d || steps != (d + s - 1) / s || (s < d && least + 1 < s / unit);
        }
  }
  return bad;
}

// a decompression whose blocks take the inverse in one launch has no intermediate to keep in the cache, and is not cut
static int check_walks_in_shares() {
  int bad = 0;
  for (int L = 10; L <= 27; ++L)
    bad += walks_in_shares(1ull << L, true) != (L >= 16 && L <= 21) || walks_in_shares(1ull << L, false) != (L <= 21);
  return bad;
}

// ... of the two workgroups to a block of 2^14
static int check_whole_split() {
  const Plan p14 = make_plan(1 << 14, THC_ORDER_ASCENDING), p13 = make_plan(1 << 13, THC_ORDER_ASCENDING);
  return !whole_split(p14, 2, 1) + !whole_split(p14, 32, 4) + whole_split(p14, 34, 4) + !whole_split(p14, 128, 1) +
         whole_split(p14, 130, 1) + whole_split(p13, 2, 1);
}

// ... of the estimate's stores
static int check_keep_estimate() {
  int bad = 0;
  for (int L = 10; L <= 25; ++L) {
    const uint64_t most = (L == 22 ? 80 : 160) * MB / 4;
    bad += keep_estimate(MB / 4, L) != (L == 15) || keep_estimate(MB / 4 + 1024, L);
    bad += keep_estimate(4 * MB, L) || !keep_estimate(4 * MB + 1024, L) || !keep_estimate(most, L) || keep_estimate(most + 1024, L);
  }
  return bad + keep_plain_estimate(MB) + !keep_plain_estimate(MB + 1024) + !keep_plain_estimate(40 * MB) +
         keep_plain_estimate(40 * MB + 1024);
}

// ... and of the cache hints: a call just below each limit and one at it.
static int check_hints() {
  int bad = 0;
  for (uint32_t W : {1u, 4u, 32u}) {
    for (bool bf16 : {false, true}) {
      const uint64_t plain = 64 * MB / (bf16 ? 2 : 4) / W, with_ef = 240 * MB / (bf16 ? 6 : 8) / W;
      const uint64_t norms_ef = 64 * MB / (bf16 ? 6 : 8) / W;
      bad += stream_inputs(plain - 1024, W, bf16, false) || !stream_inputs(plain, W, bf16, false);
      bad += stream_inputs(with_ef - 1024, W, bf16, true) || !stream_inputs(with_ef + 1024, W, bf16, true);
      for (int L : {10, 14, 15, 20}) {
        const Plan pl = make_plan(1ull << L, THC_ORDER_SPLIT);
        const uint64_t x = L > 14 ? 2 : 1;
        bad += stream_norms(pl, x * plain - 1024, W, bf16, false) || !stream_norms(pl, x * plain, W, bf16, false);
        bad += stream_norms(pl, x * norms_ef - 1024, W, bf16, true) || !stream_norms(pl, x * norms_ef + 1024, W, bf16, true);
      }
    }
    for (bool bf16 : {false, true})
      for (bool ef : {false, true}) {
        const uint64_t d = 240 * MB / ((bf16 ? 2 : 4) + (ef ? 4 : 0)) / W;
        bad += stream_minmax(d - 1024, W, bf16, ef) || !stream_minmax(d + 1024, W, bf16, ef);
      }
    bad += stream_big_inputs(160 * MB / 6 / W - 1024, W) || !stream_big_inputs(160 * MB / 6 / W + 1024, W);
    bad += stream_rotated(64 * MB / W, W) || !stream_rotated(64 * MB / W + 1024, W);
    bad += !through_inverse(64 * MB / W, W) || through_inverse(64 * MB / W + 1024, W);
    for (uint32_t b : {1u, 3u, 4u, 8u}) {
      const uint64_t d = 80 * MB / W / b * 8;
      bad += stream_sums(d - 1024, W, b) || stream_sums(d + 1024, W, b) == (W == 1 && b == 3);
    }
  }
  bad += !plain_first_pass(63, 1) + plain_first_pass(64, 1) + !plain_first_pass(7, 9) + plain_first_pass(8, 8);
  return bad + stream_sums(80 * MB * 4 + 1024, 1, 2) + !stream_sums(40 * MB * 4 + 1024, 2, 2) + !sums_four_loads(10 * MB) +
         sums_four_loads(10 * MB + 1024);
}

// The index of a coordinate above the range, for the largest rounding draw: what the quantizer's fast form, which does
// not clamp, makes of M itself.
static bool fast_form_ends_at_the_top(const QuantScalars& q, uint32_t g, uint32_t wd) {
  const float y = (q.M - q.lo) * q.sc;
  if (y >= (float)g * GRID_SCALE) return true;
  const float t = y - (float)(g - wd) * GRID_SCALE;               // in the last cell: up if the draw's product is below
  return (65535.0f + 0.5f) * (float)wd * 256.0f < t;
}

static int check_quant_form() {
  int bad = 0;
  uint64_t seed = 12345;
  auto uniform = [&] { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return (float)(seed >> 40) * 0x1p-24f; };
  auto form = [](float M, float m, uint32_t g, uint32_t wd, QuantScalars& q) {
    bool careful = false;
    q = quant_scalars(M, m, g, (g - wd) | wd << 8, 0x1p-10f, true, careful);
    return careful;
  };
  QuantScalars q;
  // empty blocks: every index is 0 in either form, so they take the short one
  for (uint32_t g : {1u, 30u, 255u})
    for (float M : {0.f, 1.f, -3.f, 1e-45f}) bad += form(M, M == 1e-45f ? -M : M, g, 1, q) || q.sc != 0.f;
  bad += !form(1e-30f, -1e-30f, 30, 3, q);                          // scale beyond what the scaled form can hold
  for (uint32_t wd : {1u, 2u, 5u})
    for (uint32_t g = wd; g <= 255; ++g) {
      int careful = 0;
      for (int i = 0; i < 400; ++i) {
        const float M = std::ldexp(0.5f + uniform(), (int)(uniform() * 40.f) - 30), m = i & 1 ? -M : -M * uniform();
        if (form(M, m, g, wd, q)) ++careful;
        else bad += !fast_form_ends_at_the_top(q, g, wd);
      }
      bad += g <= 42 * wd && careful;
    }
  return bad;
}

int main() {
  int bad = 0;
  bad += check_quant_form();
  bad += check_big<7, false>() + check_big<7, true>() + check_big<8, false>() + check_big<8, true>();
  bad += check_big<7, false, true>() + check_big<7, true, true>() + check_big<8, true, true>() + check_big<9, false, true>();
  bad += check_big<9, true, true>() + check_big<8, false, true>();
  bad += check_big<9, false>() + check_big<9, true>() + check_big<10, false>() + check_big<10, true>();
  const uint64_t M22 = 1ull << 22;
  bad += check_groups(M22, 64 * M22, 2 * M22, 1, false, false, false, false);   // thc_decompress_noalloc: 32 MB at a time
  bad += check_groups(M22, 64 * M22, 4 * M22, 1, false, true, false, true);
  bad += check_groups(M22, 66 * M22, 4 * M22, 1, false, true, false, false);     // the last group is too short
  bad += check_groups(M22, 63 * M22, 63 * M22, 1, false, false, false, false);
  bad += check_groups(M22, 64 * M22, 64 * M22, 1, true, true, true, true);
  bad += check_groups(M22, 96 * M22, 64 * M22, 1, true, true, false, true);
  bad += check_groups(M22, 16 * M22, 4 * M22, 32, true, true, true, true);
  bad += check_groups(2 * M22, 3 * M22 * 2, 2 * M22, 1, true, true, true, true);
  bad += check_groups(M22 / 2, 256 * M22, 128 * M22, 8, false, false, false, false);
  bad += check_groups(16 * M22, 32 * M22, 16 * M22, 8, false, false, false, false);
  bad += check_pieces(1ull << 10, 1) + check_pieces(1ull << 34, 1) + check_pieces((1ull << 34) + 1024, 2);
  bad += check_pieces((1ull << 36) - 1024, 4) + check_pieces(5ull << 34, 5);
  bad += check_xcd_tile<2>() + check_xcd_tile<3>() + check_xcd_tile<4>() + check_xcd_tile<6>();
  bad += check_whole_route() + check_inv_whole_14() + check_last_first() + check_hints() + check_keep_estimate() + check_even_share() + check_even_walk() + check_walks_in_shares() + check_whole_split();
  // the uniform quantizer's groups of coordinates: the limits, and that bf16 without error feedback has none
  for (bool bf16 : {false, true}) bad += !uniform_one_group(1 << 20, bf16, true) || uniform_one_group((1 << 20) + 1024, bf16, true);
  bad += !uniform_one_group(1 << 22, false, false) || uniform_one_group((1 << 22) + 1024, false, false);
  bad += uniform_one_group(1 << 24, false, false) || !uniform_one_group((1 << 24) + 1024, false, false);
  for (uint64_t d : {1ull << 10, 1ull << 23, 1ull << 34}) bad += !uniform_one_group(d, true, false);
  // largest number of workgroups at which the quantizer finds the range itself (where whole_route leaves it to the passes:
  // from 2^15 on, in 2^14, and up to 2^13 with more than four workers)
  const struct { int L; uint32_t W; uint64_t most; } find[] = {
      {10, 1, 2048},  {13, 2, 1024},  {14, 3, 1024}, {16, 4, 768},  {16, 8, 512},  {10, 32, 128}, {17, 1, 1280}, {20, 4, 320},
      {15, 1, 2048},  {16, 2, 1024},  {15, 3, 1024}, {15, 4, 768},  {15, 5, 819},  {14, 2, 1024}, {14, 4, 768},  {14, 8, 512},
      {16, 64, 64},   {18, 5, 204},   {20, 16, 64},  {17, 17, 30},  {20, 32, 16}};
  for (const auto& f : find) {
    const Plan pl = make_plan(1ull << f.L, THC_ORDER_ASCENDING);
    bad += !find_range(pl, f.most, f.W) || find_range(pl, f.most + 1, f.W);
  }
  bad += find_range(make_plan(1ull << 21, THC_ORDER_SPLIT), 256, 1);
  for (int L = 10; L <= 27; ++L)
    for (uint32_t order = 0; order <= 1; ++order) {
      const Plan pl = make_plan(1ull << L, order);
      if (!pl.ok()) { std::printf("plan L=%d order=%u not ok\n", L, order); ++bad; continue; }
      int bits = pl.L1 + pl.R;
      for (int m = 0; m < pl.nmid; ++m) bits += pl.mid[m];
      if (bits != L) { std::printf("plan L=%d order=%u covers %d bits\n", L, order, bits); ++bad; }
      if (L >= 13) {
        if (pl.split) bad += check_cover(pl.lo, true);
        for (int m = 0; m < pl.nmid; ++m) bad += check_cover(pl.midmap[m], false);
        bad += check_cover(pl.hi, false);
        const TileMap lt = lo_tilemap(pl, 1ull << (L < 19 ? 19 : L));
        if (!pl.split) {
          // consecutive tiles in a permuted order: the bases are a permutation of the multiples of 8192
          const uint32_t tiles = 1u << lt.nfixed;
          std::vector<unsigned char> seen(tiles, 0);
          for (uint32_t t = 0; t < tiles; ++t) {
            const uint64_t b = tile_base(lt, t);
            if ((b & 8191u) || (b >> 13) >= tiles || seen[b >> 13]) { ++bad; break; }
            seen[b >> 13] = 1;
          }
        }
      }
    }
  uint8_t table[256];
  double cost = 0.0, cost2 = 0.0;
  uint64_t count = 0;
  for (uint32_t b = 1; b <= 4; ++b)
    for (uint32_t g = (1u << b) - 1; g <= (b == 4 ? 22u : 40u); g += 3) {
      if (thc_solve_table(b, g, 1.0 / 32, table, &cost) != THC_OK) ++bad;
      uint8_t t2[256];
      const int rc = thc_solve_table_bruteforce(b, g, 1.0 / 32, t2, &cost2, &count);
      if (rc == THC_OK) {
        for (uint32_t z = 0; z < (1u << b); ++z) bad += table[z] != t2[z];
      } else if (rc != THC_EUNSUPPORTED) {
        ++bad;
      }
    }
  if (thc_solve_table(8, 255, 1.0 / 1024, table, nullptr) != THC_OK) ++bad;
  if (thc_solve_table(4, 14, 0.1, table, nullptr) != THC_EINVAL) ++bad;       // g < 2^b - 1
  if (!(thc_threshold(1.0 / 32) > 2.15 && thc_threshold(1.0 / 32) < 2.16)) ++bad;
  std::printf("sanitizer run: %d problem(s)\n", bad);
  return bad ? 1 : 0;
}
