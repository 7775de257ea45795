// Which coordinates the tiles of 2^15 coordinates hold, and where (plain data and arithmetic, no GPU types).
#pragma once

#include "thc_plan.hpp"

namespace thc {

// ---------------------------------------------------------------------------------------------
// Coordinates of a block, as the big tiles see them.  The first pass does the first 15 bits of the stage order
// (processing bits p0..p14), the last pass the remaining R = L - 15 (row bits q0..).
//   ascending: p = coordinate bits 0..14,                    q = 15, 16, ...
//   split:     p = coordinate bits 0..9, 13, 14, 15, 10, 11, q = 12, 16, 17, ...
// ---------------------------------------------------------------------------------------------
template <bool XO>
THC_HOST_DEVICE constexpr uint32_t big_p(uint32_t p) {   // processing index inside a first-pass tile -> offset
  return XO ? (p & 1023u) | (((p >> 10) & 7u) << 13) | (((p >> 13) & 3u) << 10) : p;
}
template <bool XO>
THC_HOST_DEVICE constexpr uint32_t big_u(uint32_t u) {   // the same 15 bits in address order -> offset
  return XO ? (u & 4095u) | ((u >> 12) << 13) : u;
}
template <bool XO>
THC_HOST_DEVICE constexpr uint32_t big_q(uint32_t q) {   // row index of the last pass -> offset
  return XO ? ((q & 1u) << 12) | ((q >> 1) << 16) : q << 15;
}
template <bool XO>
THC_HOST_DEVICE uint64_t big_lo_base(uint32_t tile) {
  return XO ? ((uint64_t)(tile & 1u) << 12) | ((uint64_t)(tile >> 1) << 16) : (uint64_t)tile << 15;
}

// ---------------------------------------------------------------------------------------------
// What the 3 slot bits and the 9 thread bits stand for: >= 0: row bit q; < 0: column bit -1 - c.
struct BigLayout {
  int slot[3];
  int thr[9];
};

// A thread's eight values of a slot are columns 0..7 (what one Philox call and one packed word cover), or, SPREAD, columns 0..3
// of each half of the row: a wave's 16-byte accesses then take whole lines, where neighbouring eights take every other 16 bytes.
template <int R, bool SPREAD = false>
struct BigHi {
  static_assert(R >= 7 && R <= 10, "the last pass takes 7 to 10 row bits");
  static constexpr int C = LOG_BIG - R;
  static constexpr int E = R - 5;                // row bits that need LDS

  // columns first, then the row bits that are still missing
  static constexpr BigLayout first() {
    BigLayout m{{0, 1, 2}, {}};
    int c = SPREAD ? 2 : 3, q = 5;
    for (int i = 0; i < 9; ++i)
      m.thr[i] = i == 4 ? 3 : i == 5 ? 4 : c < C - SPREAD ? -1 - c++ : q++;
    return m;
  }
  static constexpr void swap(BigLayout& m, int slot, int thr) {
    const int x = m.slot[slot];
    m.slot[slot] = m.thr[thr];
    m.thr[thr] = x;
  }
  static constexpr int pos(const BigLayout& m, int what) {   // thread bit that stands for `what`
    for (int i = 0; i < 9; ++i)
      if (m.thr[i] == what) return i;
    return -1;
  }
  // after the lane swaps of q3 and q4
  static constexpr BigLayout second() {
    BigLayout m = first();
    swap(m, 0, 4);
    swap(m, 1, 5);
    return m;
  }
  // after the LDS exchange: q5..q7 in the slots, q8 and q9 on lane bits 4 and 5
  static constexpr BigLayout third() {
    BigLayout m = second();
    for (int i = 0; i < 3; ++i)
      if (i < E) swap(m, i, pos(m, 5 + i));
    for (int i = 3; i < E; ++i) {
      const int a = 1 + i, b = pos(m, 5 + i);    // thread bits 4, 5
      const int x = m.thr[a];
      m.thr[a] = m.thr[b];
      m.thr[b] = x;
    }
    return m;
  }
  static constexpr BigLayout last() {
    BigLayout m = third();
    if (E >= 4) swap(m, 0, 4);
    if (E >= 5) swap(m, 1, 5);
    return m;
  }

  // offset of a slot's fifth value from its first
  template <bool XO>
  static constexpr uint32_t half_off() { return SPREAD ? big_u<XO>(1u << (C - 1)) : 4u; }

  template <bool XO>
  static constexpr uint32_t what_off(int what) {
    return what >= 0 ? big_q<XO>(1u << what) : big_u<XO>(1u << (-1 - what));
  }
  static constexpr int log2c(uint32_t v) { return v <= 1 ? 0 : 1 + log2c(v >> 1); }
  template <bool XO, int B>
  static THC_HOST_DEVICE uint32_t thread_off(const BigLayout& m, int t) {
    if constexpr (B == 9) return 0u;
    else return (((uint32_t)t >> B) & 1u) << log2c(what_off<XO>(m.thr[B])) | thread_off<XO, B + 1>(m, t);
  }
  template <bool XO>
  static constexpr uint32_t slot_off(const BigLayout& m, int k) {
    return (k & 1 ? what_off<XO>(m.slot[0]) : 0u) | (k & 2 ? what_off<XO>(m.slot[1]) : 0u) |
           (k & 4 ? what_off<XO>(m.slot[2]) : 0u);
  }
};

// offset of a tile's first coordinate inside its vector
template <int R, bool XO>
THC_HOST_DEVICE uint64_t big_hi_base(uint32_t tile) {
  return ((uint64_t)(tile >> R) << (LOG_BIG + R)) | big_u<XO>((tile & ((1u << R) - 1u)) << (LOG_BIG - R));
}

}  // namespace thc
