// Per-block constants of the quantizer.  Plain C++ arithmetic (no GPU types), so that the choice of its form can be
// checked on the host; to be compiled with -ffp-contract=off.
#pragma once

#include "thc_tilemap.hpp"

namespace thc {

struct QuantScalars {
  float M, lo, sc, c;    // range [lo, M]; fast form: scale * 2^24, and lo, M and the scale folded with c where it is a power of two
};

constexpr float GRID_SCALE = 0x1p24f;

// scale = g / (M - m): the width in binary64, the quotient rounded once to binary32.  Where that is not a finite
// number (M = m, or a width so small that the quotient overflows binary32) the range is empty: scale 0, every index 0.
THC_HOST_DEVICE float scale_of(float M, float m, uint32_t g) {
  const float sc = (float)((double)g / ((double)M - (double)m));
  return sc <= 3.4028234663852886e38f ? sc : 0.f;     // also false for NaN
}

// scale * 2^24 (and the fold with 1/sqrt(B)) stay finite below this
constexpr float WIDE_SCALE = 0x1p102f;

// Per-block constants of the quantizer and which form it takes.  `last`: the table's last cell, lut[g - 1].
THC_HOST_DEVICE QuantScalars quant_scalars(float M, float m, uint32_t g, uint32_t last, float c, bool cfold,
                                           bool& careful) {
  const float sc = scale_of(M, m, g);
  QuantScalars q{M, m, sc * GRID_SCALE, c};
  if (cfold) q = QuantScalars{M * (1.0f / c), m * (1.0f / c), sc * GRID_SCALE * c, c};
  // what a clamped coordinate comes to, and whether the largest draw still lets it reach the top index
  const float top = (q.M - q.lo) * q.sc, wd = (float)((last >> 8) & 255u) * 256.0f;
  const bool ends = top >= (float)g * GRID_SCALE ||
                    __builtin_fmaf(65535.0f, wd, 0.5f * wd) < top - (float)(last & 255u) * GRID_SCALE;
  careful = sc >= WIDE_SCALE || (sc != 0.f && !ends);   // an empty block: index 0 in either form
  return careful ? QuantScalars{M, m, sc, c} : q;
}

}  // namespace thc
