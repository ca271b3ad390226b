// occ_capsule.hpp -- the sub-cells of a voxel that a capsule touches (device and host: the host side
// serves a check against the exact test).
#pragma once

#include "geom.hpp"

namespace vx {

// exchanges index bits lo < hi of a 64-bit mask (bit number <-> bit number with the two swapped)
template <int LO, int HI>
VX_HD inline uint64_t swap_index(uint64_t x) {
  constexpr int d = (1 << HI) - (1 << LO);
  uint64_t m = 0;                                        // bit LO set, bit HI clear
#pragma unroll
  for (int i = 0; i < 64; ++i)
    if (((i >> LO) & 1) && !((i >> HI) & 1)) m |= 1ull << i;
  const uint64_t t = ((x >> d) ^ x) & m;
  return x ^ t ^ (t << d);
}

// the words of a pair in rotated coordinates, turned back and handed to put(word index, word)
template <class Put>
VX_HD inline void put_turned(uint64_t (&word)[8], int turn, const Put& put) {
  // (a, b, c) are axes turn, turn + 1, turn + 2
  if (turn != 0) {
#pragma unroll
    for (int o = 0; o < 8; ++o) word[o] = swap_index<3, 4>(swap_index<0, 1>(word[o]));
  }
  if (turn == 1) {
#pragma unroll
    for (int o = 0; o < 8; ++o) word[o] = swap_index<3, 5>(swap_index<0, 2>(word[o]));
  } else if (turn == 2) {
#pragma unroll
    for (int o = 0; o < 8; ++o) word[o] = swap_index<4, 5>(swap_index<1, 2>(word[o]));
  }
#pragma unroll
  for (int o = 0; o < 8; ++o) put(((o << turn) | (o >> (3 - turn))) & 7, word[o]);
}

// ---------------------------------------------------------------------------------------------
// capsules: the distance from a sub-cell's centre to the segment decides most (the box holds the ball
// of radius h around its centre and lies in the one of radius h sqrt(3)): along a column of sub-cells,
// the centres within a radius of the segment are one interval, solved for; those between the two
// radii take cheap bounds and the exact voxel-level test on the sub-box.
// Bound by VALU issue: 12.8 M pairs of a weave (radius of four sub-cells) 17.0 -> 10.1 ms, of it 4.8 the
// columns, 2.5 the cheap bounds and 3 the exact tests; with the exact test inside the loop of the bounds
// (a few lanes at a time) 14.0; before, every sub-cell was tried by its own distance.
// ---------------------------------------------------------------------------------------------
struct CapOcc {
  double c[3], d[3];         // segment start from the voxel's corner, direction (lattice units)
  double inv_dd;             // 1 / |d|^2 (0 for a point)
  double err;                // rounding bound of a squared distance, as in cap_ball: M^2 2^-44
  int lo[3], hi[3];
};

VX_HD inline void cap_occ_setup(const int32_t* r, const int64_t v[3], int Sb, int64_t rho, CapOcc& C) {
  const double s = double(int64_t(1) << Sb), sl = 0.125 * s, isl = 1.0 / sl;
  double M = s;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int32_t ci = r[a] - (int32_t(v[a]) << Sb);
    const int32_t di = r[3 + a] - r[a];
    C.c[a] = double(ci);
    C.d[a] = double(di);
    M = fmax(M, fabs(C.c[a]) + fabs(C.d[a]) + s);
    const double mn = fmin(C.c[a], C.c[a] + C.d[a]) - double(rho), mx = fmax(C.c[a], C.c[a] + C.d[a]) + double(rho);
    C.lo[a] = int(fmax(ceil(mn * isl) - 1.0, 0.0));
    C.hi[a] = int(fmin(floor(mx * isl), 7.0));
  }
  C.inv_dd = cap_inv_len2(r);
  C.err = M * M * 0x1p-44;
}

VX_HD inline __attribute__((noinline)) bool cap_occ_exact(const int32_t* r, int64_t u0, int64_t u1, int64_t u2,
                                                          int64_t sl, int Sbl, int64_t rho) {
  const int64_t u[3] = {u0, u1, u2};
  return cap_touch(r, u, sl, Sbl, rho);
}

// A sub-cell whose centre lies between the two balls.  P, the segment's point nearest the centre
// X, and u = (X - P) / |X - P|: the segment projects onto u at or below u . P (P is its nearest
// point to X) and the box at or above u . X - h (|u_x| + |u_y| + |u_z|), so the box lies farther
// than |X - P| - h sum |u_a| from the segment; and the box lies within the distance from P to the
// box.  Either settles most; the margins (2 err on squared lengths) cover every rounding.  The
// rest take the exact test.
VX_HD inline int cap_occ_band(const CapOcc& C, int a, int b, int c, double sl, int64_t rho) {
  const double h = 0.5 * sl, rh = double(rho);
  const double o[3] = {a * sl, b * sl, c * sl};
  double w[3];
#pragma unroll
  for (int x = 0; x < 3; ++x) w[x] = (o[x] + h) - C.c[x];
  double tc = (w[0] * C.d[0] + w[1] * C.d[1] + w[2] * C.d[2]) * C.inv_dd;
  tc = fmin(fmax(tc, 0.0), 1.0);
  double dc2 = 0.0, s1 = 0.0, f = 0.0;
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    const double wx = fma(-tc, C.d[x], w[x]);
    dc2 = fma(wx, wx, dc2);
    s1 += fabs(wx);
    const double p = fma(tc, C.d[x], C.c[x]) - o[x];          // P from the box's corner
    const double e = p < 0 ? p : (p > sl ? p - sl : 0.0);
    f = fma(e, e, f);
  }
  if (f + C.err <= rh * rh) return 1;
  const double lhs = dc2 - h * s1 - 2.0 * C.err;
  return lhs > 0.0 && lhs > rh * sqrt(dc2 + C.err) * (1.0 + 0x1p-40) ? 0 : -1;
}

// 1 / sqrt(x), x > 0, within 2^-45.4 of itself: one Newton step on an estimate good to 2^-23 (the
// host's check takes an estimate no better than that)
VX_HD inline double rsqrt_fast(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double r = __builtin_amdgcn_rsq(x);
#else
  const double r = (1.0 + 0x1p-23) / sqrt(x);
#endif
  const double h = 0.5 * x * r;
  return fma(r, fma(-h, r, 0.5), r);
}

// A row of sub-cells (bit 8 b + c) as the quarters of the words they lie in: quarter b2 + 2 c2, bit
// 2 b0 + 4 c0 + 16 b1 + 32 c1
VX_HD inline uint32_t occ_spread(uint32_t t) {          // bits 0, 8, 16, 24 -> 0, 2, 16, 18
  return (t & 0x00010001u) | ((t >> 6) & 0x00040004u);
}
VX_HD inline uint64_t occ_quarter(uint64_t row, int b2, int c2) {
  const uint32_t y = uint32_t(row >> (32 * b2)) >> (4 * c2);
  const uint32_t lo = occ_spread(y & 0x01010101u) | (occ_spread((y >> 1) & 0x01010101u) << 4);
  const uint32_t hi = occ_spread((y >> 2) & 0x01010101u) | (occ_spread((y >> 3) & 0x01010101u) << 4);
  return uint64_t(lo) | uint64_t(hi) << 32;
}

// the sub-cells il .. ih of a column
VX_HD inline uint32_t occ_bits(double l, double h) {
  const int il = int(fmax(l, 0.0)), n = int(fmax(fmin(h, 7.0), -1.0)) - il + 1;      // (l, h whole numbers)
  return n > 0 && il < 8 ? ((1u << n) - 1u) << il : 0u;
}

// The pair's mask, handed to put(word index, word).  Coordinates come rotated by `turn` axes so that
// columns run along the axis that the segment moves least along: the quadratic of the cylinder then
// has a leading coefficient of at least 2/3.  In units of a sub-cell and from the segment's start: a
// column at (x, y) is within r of the segment for heights s in the union of three intervals with
// a common point each, the two end balls' and the cylinder's between its two end planes.
//
// The radii are taken inwards and outwards by a bound on every rounding, as an amount of squared
// distance: the heights found belong exactly to a squared distance that is off by less than it.  With M
// the largest of |c| + |d| + 8 over the axes and the radius (sub-cells), every product below is at most
// 3 M^2: c0, which is a difference of such products where the segment starts far away, is off by less
// than 27 M^2 2^-53, the quadratic's other coefficients, the middle and the rounded heights change it
// by less than 190 M^2 2^-53 in all, and the roots, good to 2^-45.4, by 10 M^2 2^-45.4 (a root is at
// most 2.2 M): together less than M^2 2^-41.  Taken: M^2 2^-40.  (An end plane's place matters to the
// square of its error only, since the end's ball takes over there.)  On a grid of 1024^3 that is below
// 2^-13 of a sub-cell squared for any segment inside it; a fixed 2^-30 of a sub-cell set sub-cells that
// were not touched on segments of 2^18 sub-cells and more.
template <class Put>
VX_HD inline void cap_occ_mask(const CapOcc& C, const int32_t* r, const int64_t v[3], int turn, double sl, int Sb,
                               int64_t rho, const Put& put) {
  const double isl = 1.0 / sl, rh = double(rho) * isl;
  const double px = C.c[0] * isl, py = C.c[1] * isl, pz = C.c[2] * isl - 0.5;      // (of the centres)
  const double dx = C.d[0] * isl, dy = C.d[1] * isl, dz = C.d[2] * isl;
  const double idd = C.inv_dd * sl * sl, dd = dx * dx + dy * dy + dz * dz;
  const double A = 1.0 - dz * dz * idd, iA = rcp_fast(A), idz = dz != 0.0 ? rcp_fast(dz) : 0.0;
  const double margin = 16.0 * fmax(C.err * isl * isl, (rh + 1.0) * (rh + 1.0) * 0x1p-44);
  const double rin = rh + 0.5, rout = rh + 0.8660254037844387;
  const double r2[2] = {rin * rin - margin, rout * rout + margin};
  uint64_t word[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
  for (int a = C.lo[0]; a <= C.hi[0]; ++a) {
    const double x = (a + 0.5) - px;
    uint64_t row = 0, band = 0;
#pragma unroll 1
    for (int b = C.lo[1]; b <= C.hi[1]; ++b) {
      const double y = (b + 0.5) - py;
      const double e = fma(x, dx, y * dy), q0 = fma(x, x, y * y);
      const double x1 = x - dx, y1 = y - dy, q1 = fma(x1, x1, y1 * y1);
      const double B = e * dz * idd, mid = B * iA, c0 = q0 - e * e * idd;
      double t0 = -e * idz, t1 = (dd - e) * idz;                 // heights of the end planes
      const bool within = e >= 0.0 && e <= dd;
      if (dz == 0.0) {
        t0 = within ? -1e9 : 1e9;
        t1 = -t0;
      } else if (dz < 0.0) {
        const double t = t0;
        t0 = t1;
        t1 = t;
      }
      uint32_t bits[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        double l = 1e9, h = -1e9;
        const double disc = fma(B, B, A * (r2[k] - c0)), s0 = r2[k] - q0, s1 = r2[k] - q1;
        if (disc > 0.0) {
          const double w = disc * rsqrt_fast(disc) * iA;
          const double cl = fmax(mid - w, t0), ch = fmin(mid + w, t1);
          l = cl <= ch ? cl : l;
          h = cl <= ch ? ch : h;
        }
        if (s0 > 0.0) {
          const double w = s0 * rsqrt_fast(s0);
          l = fmin(l, -w);
          h = fmax(h, w);
        }
        if (s1 > 0.0) {
          const double w = s1 * rsqrt_fast(s1);
          l = fmin(l, dz - w);
          h = fmax(h, dz + w);
        }
        bits[k] = occ_bits(ceil(fmin(l + pz, 64.0)), floor(fmax(h + pz, -64.0)));
      }
      const uint32_t box = (2u << C.hi[2]) - (1u << C.lo[2]);
      row |= uint64_t(bits[0] & box) << (8 * b);
      band |= uint64_t(bits[1] & ~bits[0] & box) << (8 * b);
    }
    // the cheap bounds first, so that the lanes that need the exact test take it together
    uint64_t hard = 0;
    for (; band; band &= band - 1) {
      const int t = __builtin_ctzll(band), in = cap_occ_band(C, a, t >> 3, t & 7, sl, rho);
      row |= in > 0 ? 1ull << t : 0ull;
      hard |= in < 0 ? 1ull << t : 0ull;
    }
    for (; hard; hard &= hard - 1) {
      const int t = __builtin_ctzll(hard), b = t >> 3, c = t & 7;
      // (a, b, c) are axes turn, turn + 1, turn + 2; the record and the voxel are not rotated
      const int i = turn == 0 ? a : (turn == 1 ? c : b), j = turn == 0 ? b : (turn == 1 ? a : c),
                k = turn == 0 ? c : (turn == 1 ? b : a);
      if (cap_occ_exact(r, 8 * v[0] + i, 8 * v[1] + j, 8 * v[2] + k, int64_t(sl), Sb - 3, rho)) row |= 1ull << t;
    }
    const int at = (a & 1) | ((a & 2) << 2);
#pragma unroll
    for (int o = 0; o < 4; ++o) {                        // b2 + 2 c2
      const uint64_t p = occ_quarter(row, o & 1, o >> 1) << at;
      word[2 * o] |= a < 4 ? p : 0ull;
      word[2 * o + 1] |= a < 4 ? 0ull : p;
    }
  }
  put_turned(word, turn, put);
}

// The mask of the pair (segment record r, voxel v) on a grid of 2^Sb lattice units a voxel: rotated so
// that the axis the segment moves least along comes last
template <class Put>
VX_HD inline void cap_occ_pair(const int32_t* r, const int64_t v[3], int Sb, int64_t rho, const Put& put) {
  const int32_t e0 = abs(r[3] - r[0]), e1 = abs(r[4] - r[1]), e2 = abs(r[5] - r[2]);
  const int turn = e2 <= e0 && e2 <= e1 ? 0 : (e0 <= e1 ? 1 : 2);
  int32_t q[6];
  int64_t vt[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int b = (a + 1) % 3, c = (a + 2) % 3;
    vt[a] = turn == 0 ? v[a] : (turn == 1 ? v[b] : v[c]);
#pragma unroll
    for (int k = 0; k < 6; k += 3) q[k + a] = turn == 0 ? r[k + a] : (turn == 1 ? r[k + b] : r[k + c]);
  }
  CapOcc C;
  cap_occ_setup(q, vt, Sb, rho, C);
  cap_occ_mask(C, r, v, turn, double(int64_t(1) << (Sb - 3)), Sb, rho, put);
}

}  // namespace vx
