// scan_units.hpp -- the units of the sweep's integer scan (host code without HIP,
// so that its bound can be checked on any machine).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace pr {

// Positions in units of L / 2^m, as floor(position * scale) modulo 2^16, and the
// squared distance in these units below which a pair is a candidate.
struct ScanUnits {
  float scale;
  uint32_t thr;
};

// L / 2^m with m from 16 (the integers wrap at 2^16 and the box at a multiple of
// it) to 22 (positions times 2^m / L keep their FP32 rounding below two units),
// the cutoff 4096 to 8191 units where that allows.  The threshold lets every pair
// through that the FP32 test can accept: the truncations move a component
// difference by less than one unit, the rounding of the two products by less than
// 2^(m - 22), that of the FP32 distance itself by less than 2^-20 of the cutoff
// and 2^(m - 23) units.
inline ScanUnits scan_units(float L, float rc) {
  int m = 16;
  while (m < 22 && (double)rc / (double)L * (double)(1u << m) < 4096.0) ++m;
  ScanUnits u;
  u.scale = (float)((double)(1u << m) / (double)L);
  const double e = 1.0 + std::ldexp(1.0, m - 21);
  const double r = (double)rc / (double)L * (double)(1u << m) * (1.0 + 1.0 / (1 << 16)) + 2.0 * e;
  u.thr = (uint32_t)std::min(std::ceil(r * r), 4294967295.0);
  // near the smallest FP32 numbers the FP32 test itself is that coarse: every
  // pair of a block is a candidate
  if (rc * rc < 1e-30f) u.thr = 4294967295u;
  return u;
}

}  // namespace pr
