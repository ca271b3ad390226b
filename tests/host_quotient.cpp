// quotient() against the division, over integers below 2^26 of every size, scaled alike by powers of
// two, with the reciprocal off by up to `off` units in the last place; returns the differing ones
#include <cmath>
#include <cstdint>
#include <cstring>
#include <random>

#include "geom.hpp"

extern "C" long hq_differ(long n, int off, int scale, unsigned seed) {
  std::mt19937_64 g(seed);
  const double f = std::ldexp(1.0, scale);
  long bad = 0;
  for (long i = 0; i < n; ++i) {
    const int ba = 1 + int(g() % 26), bd = 1 + int(g() % 26);
    int64_t a = int64_t(g() % (uint64_t(1) << ba)), d = 1 + int64_t(g() % ((uint64_t(1) << bd) - 1));
    if (g() & 1) a = -a;
    if (g() & 1) d = -d;
    const double x = double(a) * f, y = double(d) * f;
    double r = 1.0 / y;
    int64_t bits;
    std::memcpy(&bits, &r, 8);
    bits += int64_t(g() % uint64_t(2 * off + 1)) - off;
    std::memcpy(&r, &bits, 8);
    bad += vx::quotient(x, y, r) != x / y;
  }
  return bad;
}
