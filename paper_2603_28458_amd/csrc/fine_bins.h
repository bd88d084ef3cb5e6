// Bin addresses of the one-pass top-k (select_topk_fine): plain arithmetic, so that a host compiler can
// take the same lines.  constexpr functions are callable from host and device code alike.
#pragma once
#include <stdint.h>

namespace hisa {

// bin(x) = 1 + floor((x - lo) * scale) in 1 .. NBIN-1 for lo <= x <= hi, 0 for NaN.  What is computed per
// score is the bin's LDS byte address, base + 4 * bin: one multiply-add, one conversion that rounds down
// (negative and NaN give 0), one mask and one clamp to the bins.
// Monotone in x, so every score in a higher bin is larger than every score in a lower one.  scale stops a
// hair short of (NBIN - 2) / (hi - lo), and in exact arithmetic the top bin needs no clamp; but bias4 is
// rounded at the magnitude of lo * scale4, and past 2^24 (a row whose spread is below 5e-4 of its scores) its
// error exceeds the four bytes of slack: 64 scores from 777.7 upwards, one unit in the last place apart,
// reach address base + 8208 of 8192.  The clamp keeps every such score in the top bin (or in bin 0, which
// makes the search decline), takes the place of the clamp from below and costs nothing more.
struct FineBins {
  float scale4, bias4;
  uint32_t base, top;   // addresses of the first and the last bin
};

template <int NBIN>
constexpr inline __attribute__((always_inline)) FineBins fine_bins(float lo, float hi, uint32_t base) {
  const float scale4 = 4.0f * (float)(NBIN - 2) * (1.0f - 0x1p-18f) / (hi - lo);
  return {scale4, __builtin_fmaf(-lo, scale4, 4.0f + (float)base), base, base + 4u * (NBIN - 1)};
}

// cvt(x): x rounded down to uint32_t, saturating, NaN to 0; med3: the median of three.
template <class Cvt, class Med3>
constexpr inline __attribute__((always_inline)) uint32_t fine_bin_address(float x, const FineBins& b, Cvt cvt,
                                                                          Med3 med3) {
  return med3(cvt(__builtin_fmaf(x, b.scale4, b.bias4)) & ~3u, b.base, b.top);
}

}  // namespace hisa
