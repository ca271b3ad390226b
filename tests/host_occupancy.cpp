// Host build of the capsules' sub-cell masks, exported for tests/test_host_occupancy.py.
#include "occ_capsule.hpp"

extern "C" {
// bits by which the pair's mask differs from the exact test of every sub-cell; touched: the exact hits
int ho_wrong(const int32_t* r6, const int64_t* v3, int Sb, int64_t rho, int* touched) {
  uint64_t word[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  vx::cap_occ_pair(r6, v3, Sb, rho, [&](int oct, uint64_t w) { word[oct] |= w; });
  int wrong = 0;
  *touched = 0;
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 8; ++j)
      for (int k = 0; k < 8; ++k) {
        const int64_t u[3] = {8 * v3[0] + i, 8 * v3[1] + j, 8 * v3[2] + k};
        const bool in = vx::cap_touch(r6, u, int64_t(1) << (Sb - 3), Sb - 3, rho);
        int m = 0;
        for (int b = 0; b < 3; ++b) m |= ((i >> b) & 1) << (3 * b) | ((j >> b) & 1) << (3 * b + 1) | ((k >> b) & 1) << (3 * b + 2);
        wrong += in != bool((word[m >> 6] >> (m & 63)) & 1);
        *touched += in;
      }
  return wrong;
}
int ho_touch(const int32_t* r6, const int64_t* v3, int Sb, int64_t rho) {
  return vx::cap_touch(r6, v3, int64_t(1) << Sb, Sb, rho) ? 1 : 0;
}
}
