// Host build of the unit kernel's area by integration, exported for tests/test_host_area.py.
#include "geom.hpp"

extern "C" {
// the triangle's piece in voxel v (voxel^2); dir4: unit normal and twice the area
float ha_area(const int32_t* q9, const int32_t* v3, int Sb, const float* dir4) {
  uint32_t how;
  double scale;
  vx::tri_area_setup(q9, make_float4(dir4[0], dir4[1], dir4[2], dir4[3]), Sb, how, scale);
  return vx::tri_area_under(q9, v3, Sb, how, scale);
}
// the same by the routine that small pieces take
float ha_small(const int32_t* q9, const int32_t* v3, int Sb, const float* dir4) {
  const int64_t v[3] = {v3[0], v3[1], v3[2]};
  return vx::tri_area(q9, v, Sb, dir4[3]);
}
}
