// Checks scan_units against the two tests it stands between, on the host: every
// pair that the FP32 distance test accepts must be a candidate of the integer
// one.  Prints, per L and rc: pairs tried, accepted, candidates, accepted but no
// candidate (which must be none).  Built with FP contraction off.
#include "../paper_1409_7498_amd/csrc/scan_units.hpp"

#include <cstdio>
#include <cstdlib>
#include <random>

static float min_image(float d, float L, float half) {
  return d > half ? d - L : (d < -half ? d + L : d);
}

int main(int argc, char** argv) {
  const float L = std::strtof(argv[1], nullptr), rc = std::strtof(argv[2], nullptr);
  const long tries = std::atol(argv[3]);
  const pr::ScanUnits u = pr::scan_units(L, rc);
  const float half = 0.5f * L, rc2 = rc * rc;
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> uni(0.0, 1.0);
  std::normal_distribution<double> nrm;
  auto at = [&](double v) {  // a position of the box, FP32
    v = std::fmod(v, (double)L);
    if (v < 0.0) v += L;
    const float f = (float)v;
    return f < 0.0f || f >= L ? 0.0f : f;
  };
  auto q = [&](float x) { return (int16_t)(uint16_t)(uint32_t)(int)(x * u.scale); };
  long in = 0, cand = 0, lost = 0;
  for (long t = 0; t < tries; ++t) {
    float a[3], b[3];
    double dir[3], len = 0.0;
    const int kind = (int)(t % 4);  // a direction: any, along an axis, a face's diagonal, the box's
    for (int d = 0; d < 3; ++d)
      dir[d] = kind == 0 ? nrm(rng) : kind == 1 ? (d == (int)(t / 4 % 3)) : kind == 2 ? (d < 2) : 1.0;
    for (int d = 0; d < 3; ++d) {
      if (kind && (rng() & 1)) dir[d] = -dir[d];
      len += dir[d] * dir[d];
    }
    // the distance: within a few FP32 roundings of the cutoff, or of a unit of the scan
    const double near = t % 3 ? 1e-7 : 3.0 / (u.scale * (double)rc);
    const double r = rc * (1.0 + near * (2.0 * uni(rng) - 1.0));
    for (int d = 0; d < 3; ++d) {
      // anywhere, or at the edges of the box
      const double p = t % 5 ? uni(rng) * L : (t % 2 ? 0.0 : (double)std::nextafter(L, 0.0f));
      a[d] = at(p);
      b[d] = at((double)a[d] + r * dir[d] / std::sqrt(len));
    }
    float f[3];
    uint32_t s = 0;
    for (int d = 0; d < 3; ++d) {
      f[d] = min_image(a[d] - b[d], L, half);
      const int32_t i = (int16_t)(uint16_t)((uint32_t)(uint16_t)q(a[d]) - (uint16_t)q(b[d]));
      s += (uint32_t)(i * i);
    }
    const bool ok = (f[0] * f[0] + f[1] * f[1]) + f[2] * f[2] < rc2, c = s < u.thr;
    in += ok;
    cand += c;
    lost += ok && !c;
  }
  std::printf("%ld %ld %ld %ld\n", tries, in, cand, lost);
  return 0;
}
