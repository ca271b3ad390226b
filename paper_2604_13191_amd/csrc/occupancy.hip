// occupancy.hip -- sub-voxel occupancy and projected densities (Sec. 3.5 occupancy equation and
// XY / XZ / YZ projections; Sec. 4.2 the same projections for the coarser levels).
//
// Every voxel of every level holds 8^3 sub-cells.  At the leaf a sub-cell is hit when a primitive
// touches its closed box (the voxel level's exact predicate on the same lattice, with boxes of
// s / 8 lattice units).  The pairs (primitive, voxel) come from the candidate pipeline; for each
// pair the sub-cells inside the primitive's bounding box are decided (triangles through their three
// axis projections and the plane, capsules by the distance of sub-cell centres), and the pair's 512-bit
// mask is OR-ed into its voxel's mask.  OR is order-free, so the result does not
// depend on the order of the atomics.
// A coarser voxel's sub-cell is the union of 2 x 2 x 2 sub-cells of one child, so its mask is its
// children's masks with every byte OR-reduced to one bit.
//
// Mask layout: sub-cell (i, j, k) in [0, 8)^3 has the Morton index m (x bits at 0, 3, 6); word
// m >> 6, bit m & 63.  Word c therefore covers the octant c of the voxel, byte b of it the octant
// b of that octant, and bit b' of the byte the sub-cell b' of that.
#include "geom.hpp"
#include "occ_capsule.hpp"
#include "vx_internal.hpp"

namespace vx {
namespace {

__device__ __forceinline__ void occ_flag(int64_t* stats, int64_t bit) {
  atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)bit);
}

// ---------------------------------------------------------------------------------------------
// triangles
// ---------------------------------------------------------------------------------------------
// The closed-box test is the separating-axis test on the box axes, the plane normal and the nine
// edge x box-axis directions.  The three edge directions perpendicular to axis k and the two box
// axes other than k are the separating-axis test of the triangle and the box projected along k, so
// a sub-cell (i, j, k) is touched exactly when
//     P_z(i, j)  and  P_y(i, k)  and  P_x(j, k)  and  the plane meets the box,
// with P_z, P_y, P_x the 8 x 8 masks of the squares the projected triangle meets.  Coordinates are
// lattice units from the voxel's corner.  The projections and every box bound of the edge tests are
// integers below 2^53 (see tri_touch), so FP64 holds them exactly.
// The tests are linear in each sub-cell coordinate, so they are solved instead of tried: in a row of
// squares each edge leaves a range, and in a column of sub-cells the plane does.  A row's ends are
// rounded quotients settled by an exact remainder; a column's come from FP64 with a bound on its
// error, and a column whose end lies within the bound of a whole number (or a plane too nearly
// parallel to z) takes the plane test with its exact fallback cell by cell.
// Bound by VALU issue: about 4,500 instructions a pair, 8,300 when every square and sub-cell was tried in
// divergent loops: a 1025^2 piece of the brushed surface (9.4 M pairs) 2.42 -> 1.65 ms.
struct TriOcc {
  double c0[3];
  double e[3][3];
  double pmin[9], pmax[9];   // the triangle on the nine edge x axis directions (edge j, axis k: 3j + k)
  double n[3], nlo, nhi;     // plane normal, sums of its negative and positive parts
  double base;               // -n . c0
  double err;                // bound on the rounding of every plane evaluation in this voxel
  int lo[3], hi[3];          // sub-cells the bounding box meets, per axis
};

__device__ __forceinline__ void tri_occ_setup(const int32_t* q, const int64_t v[3], int Sb, TriOcc& T) {
  double c[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int a = 0; a < 3; ++a) c[i][a] = double(q[3 * i + a] - (int32_t(v[a]) << Sb));
  const double sl = double(int64_t(1) << (Sb - 3)), isl = 1.0 / sl;    // exact: powers of two
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    T.c0[a] = c[0][a];
    T.e[0][a] = c[1][a] - c[0][a];
    T.e[1][a] = c[2][a] - c[1][a];
    T.e[2][a] = c[0][a] - c[2][a];
    const double mn = fmin(fmin(c[0][a], c[1][a]), c[2][a]), mx = fmax(fmax(c[0][a], c[1][a]), c[2][a]);
    // box [i sl, (i+1) sl] meets [mn, mx] for ceil(mn / sl) - 1 <= i <= floor(mx / sl)
    T.lo[a] = int(fmax(ceil(mn * isl) - 1.0, 0.0));
    T.hi[a] = int(fmin(floor(mx * isl), 7.0));
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int u = (k + 1) % 3, w = (k + 2) % 3;
      const double au = -T.e[j][w], aw = T.e[j][u];
      const double p0 = fma(au, c[j][u], aw * c[j][w]);
      const double p2 = fma(au, c[(j + 2) % 3][u], aw * c[(j + 2) % 3][w]);
      T.pmin[3 * j + k] = fmin(p0, p2);
      T.pmax[3 * j + k] = fmax(p0, p2);
    }
  }
  T.n[0] = fma(T.e[0][2], T.e[2][1], -(T.e[0][1] * T.e[2][2]));
  T.n[1] = fma(T.e[0][0], T.e[2][2], -(T.e[0][2] * T.e[2][0]));
  T.n[2] = fma(T.e[0][1], T.e[2][0], -(T.e[0][0] * T.e[2][1]));
  T.nlo = (fmin(T.n[0], 0.0) + fmin(T.n[1], 0.0) + fmin(T.n[2], 0.0)) * sl;
  T.nhi = (fmax(T.n[0], 0.0) + fmax(T.n[1], 0.0) + fmax(T.n[2], 0.0)) * sl;
  T.base = -(T.n[0] * c[0][0] + T.n[1] * c[0][1] + T.n[2] * c[0][2]);
  const double mag0 = fabs(T.n[0] * c[0][0]) + fabs(T.n[1] * c[0][1]) + fabs(T.n[2] * c[0][2]);
  // every sub-box corner offset is at most 8 sl per axis, and its bounds add sl more
  T.err = (mag0 + 9.0 * sl * (fabs(T.n[0]) + fabs(T.n[1]) + fabs(T.n[2]))) * 0x1p-48;
}

// The squares of the plane perpendicular to axis K that the projected triangle meets, row by row:
// rows along axis R, bits along axis B (R, B and K are the three axes).  Edge j holds in square
// (row a, bit b) when  lo_j <= A a + W b <= hi_j; with the signs turned so that W > 0, b runs from
// ceil((lo_j - A a) / W) to floor((hi_j - A a) / W).
struct OccRows {
  double A[3], W[3], iW[3], lo[3], hi[3], mul[3];
  int r0, r1, b0, b1;        // rows and bits of the triangle's bounding box
};

template <int K, int R, int B>
__device__ __forceinline__ OccRows tri_occ_rows(const TriOcc& T, double sl) {
  constexpr int u = (K + 1) % 3, w = (K + 2) % 3;
  static_assert((R == u && B == w) || (R == w && B == u), "rows and bits span the projection");
  OccRows P;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double au = -T.e[j][w], aw = T.e[j][u];
    const double up = T.pmax[3 * j + K] - (fmin(au, 0.0) + fmin(aw, 0.0)) * sl;
    const double dn = T.pmin[3 * j + K] - (fmax(au, 0.0) + fmax(aw, 0.0)) * sl;
    const double cr = (R == u ? au : aw) * sl, cb = (R == u ? aw : au) * sl;
    const bool neg = cb < 0.0, flat = cb == 0.0;
    P.A[j] = neg ? -cr : cr;
    P.W[j] = flat ? 1.0 : fabs(cb);
    P.iW[j] = flat ? 0.0 : rcp_fast(P.W[j]);
    P.hi[j] = neg ? -dn : up;
    P.lo[j] = neg ? -up : dn;
    // an edge along the bits decides the row alone: its quotients come out 0 or past it (-1 and 1),
    // stretched to the whole row or none of it
    P.mul[j] = flat ? 8.0 : 1.0;
  }
  P.r0 = T.lo[R];
  P.r1 = T.hi[R];
  P.b0 = T.lo[B];
  P.b1 = T.hi[B];
  return P;
}

// Row a's eight bits.  A quotient rounded to the nearest whole number is settled by the sign of its
// exact remainder.
__device__ __forceinline__ uint32_t occ_row(const OccRows& P, int a) {
  double h = 7.0, l = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double dh = fma(-P.A[j], double(a), P.hi[j]), dl = fma(-P.A[j], double(a), P.lo[j]);
    const double kh = rint(dh * P.iW[j]), kl = rint(dl * P.iW[j]);
    const double past = kh + (fma(-kh, P.W[j], dh) < 0.0 ? 0.0 : 1.0);      // floor + 1
    const double from = kl + (fma(-kl, P.W[j], dl) > 0.0 ? 1.0 : 0.0);      // ceil
    h = fmin(h, fma(past, P.mul[j], -1.0));
    l = fmax(l, from * P.mul[j]);
  }
  const int ih = min(int(fmax(h, -1.0)), P.b1), il = max(int(fmin(l, 8.0)), P.b0);
  const int n = a >= P.r0 && a <= P.r1 ? max(ih - il + 1, 0) : 0;
  return ((1u << n) - 1u) << il;
}

// does the plane meet the closed box at sub-cell (i, j, k)?  Operands by value, out of line: taken
// where a column's range is too close to call
__device__ __attribute__((noinline)) bool tri_occ_plane(double n0, double n1, double n2, double nlo, double nhi,
                                                        double base, double err, double c0, double c1, double c2,
                                                        int i, int j, int k, double sl) {
  const double o0 = i * sl, o1 = j * sl, o2 = k * sl;
  const double b = base + (n0 * o0 + n1 * o1 + n2 * o2);
  const double lo = b + nlo, hi = b + nhi;
  if (lo > err || hi < -err) return false;
  if (lo < -err && hi > err) return true;
  return plane_exact(int64_t(n0), int64_t(n1), int64_t(n2), int64_t(o0 - c0), int64_t(o1 - c1), int64_t(o2 - c2),
                     int64_t(sl));
}

// The pair's mask, handed to put(word index, word) in Morton order.  Coordinates come rotated by
// `turn` axes (axis 0 here is axis `turn`, the one the triangle is thinnest along: rows run along it
// and there are few) and the words are rotated back.  One row of columns at a time in a rolled loop:
// unrolled, the spills of its registers alone write 12 GB per 9 M pairs.  Rolled, 27 registers are
// spilled at the kernel's three waves per SIMD (capsules: 21), 128 (160) bytes a lane.
template <class Put>
__device__ __forceinline__ void tri_occ_mask(const TriOcc& T, double sl, int turn, const Put& put) {
  uint64_t px = 0;                                       // row y, bits z
  {
    const OccRows P = tri_occ_rows<0, 1, 2>(T, sl);
#pragma unroll 1
    for (int b = 0; b < 8; ++b) px |= uint64_t(occ_row(P, b)) << (8 * b);
  }
  const OccRows PZ = tri_occ_rows<2, 0, 1>(T, sl);       // row x, bits y
  const OccRows PY = tri_occ_rows<1, 0, 2>(T, sl);       // row x, bits z
  // the plane meets column (a, b) in the sub-cells ceil(q - span) .. floor(q), q = q0 + qa a + qb b;
  // T.err covers the rounding of the plane's value, and that of the quotients is smaller.  An end
  // within eps of a whole number leaves that one sub-cell open.
  const bool neg = T.n[2] < 0.0;
  const double W = fabs(T.n[2]) * sl, iW = W > 0.0 ? rcp_fast(W) : 0.0;
  const double qa = (neg ? T.n[0] : -T.n[0]) * sl * iW, qb = (neg ? T.n[1] : -T.n[1]) * sl * iW;
  const double q0 = (neg ? T.base + T.nhi : -(T.base + T.nlo)) * iW;
  const double span = (T.nhi - T.nlo) * iW;
  const double eps = 4.0 * T.err * iW + 0x1p-40;
  const bool steep = !(W > 0.0) || !(eps < 0.25);
  uint64_t word[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  uint64_t hard = 0, py = 0;                             // columns with an open sub-cell (bit 8 a + b); PY
#pragma unroll 1
  for (int a = T.lo[0]; a <= T.hi[0]; ++a) {
    const uint32_t rz = occ_row(PZ, a), ry = occ_row(PY, a);
    py |= uint64_t(ry) << (8 * a);
    uint32_t part[8] = {0, 0, 0, 0, 0, 0, 0, 0};         // index c1 + 2 b2 + 4 c2: half of a word
    uint32_t open = 0;
    const double h0 = fma(qa, double(a), q0);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int j = b & 3, o = 2 * (b >> 2), at = ((j & 1) << 1) | ((j & 2) << 3);
      const double h = fma(qb, double(b), h0), l = h - span;
      const double fh = floor(h - eps), cl = ceil(l + eps);
      const bool near = floor(h + eps) != fh || ceil(l - eps) != cl || steep;
      const int ih = min(int(fh), 7), il = max(int(cl), 0);
      const uint32_t z = (rz >> b) & 1u ? ry & uint32_t(px >> (8 * b)) & 255u : 0u;
      open |= near && z != 0u ? 1u << b : 0u;
      const uint32_t in = ih >= il && !steep ? z & (((2u << (ih - il)) - 1u) << il) : 0u;
      // sub-cell (a, b, c) is bit a0 b0 c0 a1 b1 c1 of word a2 b2 c2
      part[o] |= ((in & 1u) | ((in << 3) & 0x10u)) << at;
      part[o + 1] |= (((in >> 2) & 1u) | ((in << 1) & 0x10u)) << at;
      part[o + 4] |= (((in >> 4) & 1u) | ((in >> 1) & 0x10u)) << at;
      part[o + 5] |= (((in >> 6) & 1u) | ((in >> 3) & 0x10u)) << at;
    }
    hard |= uint64_t(open) << (8 * a);
    const int at = (a & 1) | ((a & 2) << 2);
#pragma unroll
    for (int o = 0; o < 4; ++o) {                        // b2 + 2 c2
      const uint64_t p = (uint64_t(part[2 * o]) | (uint64_t(part[2 * o + 1]) << 32)) << at;
      word[2 * o] |= a < 4 ? p : 0ull;
      word[2 * o + 1] |= a < 4 ? 0ull : p;
    }
  }
  for (; hard; hard &= hard - 1) {
    const int t = __builtin_ctzll(hard), a = t >> 3, b = t & 7;
    const uint32_t z = uint32_t(py >> (8 * a)) & uint32_t(px >> (8 * b)) & 255u;
    const double h = fma(qb, double(b), fma(qa, double(a), q0)), l = h - span;
    const double kh = floor(h + eps), kl = ceil(l - eps);
    uint32_t m = steep ? z : 0u;
    if (kh >= 0.0 && kh <= 7.0 && kh != floor(h - eps)) m |= z & (1u << int(kh));
    if (kl >= 0.0 && kl <= 7.0 && kl != ceil(l + eps)) m |= z & (1u << int(kl));
    for (; m; m &= m - 1) {
      const int c = __builtin_ctz(m);
      if (!tri_occ_plane(T.n[0], T.n[1], T.n[2], T.nlo, T.nhi, T.base, T.err, T.c0[0], T.c0[1], T.c0[2], a, b, c, sl))
        continue;
      const int o = (a >> 2) | ((b >> 1) & 2) | (c & 4);
      const uint64_t bit = 1ull << ((a & 1) | ((b & 1) << 1) | ((c & 1) << 2) | ((a & 2) << 2) | ((b & 2) << 3) | ((c & 2) << 4));
#pragma unroll
      for (int w = 0; w < 8; ++w) word[w] |= w == o ? bit : 0ull;
    }
  }
  put_turned(word, turn, put);
}

// ---------------------------------------------------------------------------------------------
// per pair: find the voxel in the leaf, build each octant's word, OR it in
// ---------------------------------------------------------------------------------------------
template <class Key>
__device__ __forceinline__ int64_t find_key(const Key* __restrict__ keys, int64_t n, Key k) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (keys[mid] < k) lo = mid + 1; else hi = mid;
  }
  return lo < n && keys[lo] == k ? lo : -1;
}

// Leaf index of every pair's voxel (kNoVoxel: the leaf lacks it), a pass of its own: a chain of some 20
// dependent loads with few registers, where many waves hide each other's; in the mask kernel, at
// three waves per SIMD, the same search took 0.4 ms per 9 M pairs.
constexpr uint32_t kNoVoxel = 0xffffffffu;
template <class Key>
__global__ void __launch_bounds__(kBlock) k_occ_find(const Key* __restrict__ pkeys, const int64_t* __restrict__ ctl,
                                                     const Key* __restrict__ leaf_keys,
                                                     const int64_t* __restrict__ n_leaf, int64_t leaf_cap, int64_t cap,
                                                     uint32_t* __restrict__ at, int64_t* stats) {
  const int64_t n = ctl[CTL_N_PAIRS];
  // a leaf over either capacity is flagged by k_occ_check; searching a clamped prefix keeps every
  // access in bounds
  const int64_t nl = imin(imin(*n_leaf, leaf_cap), cap);
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const int64_t idx = find_key<Key>(leaf_keys, nl, pkeys[i]);
    if (idx < 0) occ_flag(stats, VX_FLAG_OCC_LEAF);      // the leaf given is not this voxelization's
    at[i] = idx < 0 ? kNoVoxel : uint32_t(idx);
  }
}

template <int KIND, class Key>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3))) k_occ_pairs(
    const int32_t* __restrict__ rec, const Key* __restrict__ pkeys, const uint32_t* __restrict__ prim,
    const uint32_t* __restrict__ at, const int64_t* __restrict__ ctl, Lat L, unsigned long long* __restrict__ mask,
    int64_t cap) {
  const int64_t n = ctl[CTL_N_PAIRS];
  const int Sb = L.Sb;
  const double sl = double(int64_t(1) << (Sb - 3));
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const Key key = pkeys[i];
    const uint32_t idx = at[i];
    if (idx == kNoVoxel) continue;
    const int64_t v[3] = {int64_t(compact3(uint64_t(key))), int64_t(compact3(uint64_t(key) >> 1)),
                          int64_t(compact3(uint64_t(key) >> 2))};
    const int32_t* r = rec + int64_t(prim[i]) * kRec;
    if (KIND == 0) {
      // rotated so that the triangle's thinnest axis comes first
      int32_t q[9];
      int32_t ext[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int32_t mn = min(min(r[a], r[3 + a]), r[6 + a]), mx = max(max(r[a], r[3 + a]), r[6 + a]);
        ext[a] = mx - mn;
      }
      const int turn = ext[0] <= ext[1] && ext[0] <= ext[2] ? 0 : (ext[1] <= ext[2] ? 1 : 2);
      int64_t vt[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int b = (a + 1) % 3, c = (a + 2) % 3;
        vt[a] = turn == 0 ? v[a] : (turn == 1 ? v[b] : v[c]);
#pragma unroll
        for (int k = 0; k < 9; k += 3) q[k + a] = turn == 0 ? r[k + a] : (turn == 1 ? r[k + b] : r[k + c]);
      }
      TriOcc T;
      tri_occ_setup(q, vt, Sb, T);
      tri_occ_mask(T, sl, turn, [&](int oct, uint64_t word) {
        if (word) atomicOr(mask + int64_t(oct) * cap + idx, (unsigned long long)word);
      });
    } else {
      cap_occ_pair(r, v, Sb, L.rho, [&](int oct, uint64_t word) {
        if (word) atomicOr(mask + int64_t(oct) * cap + idx, (unsigned long long)word);
      });
    }
  }
}

// ---------------------------------------------------------------------------------------------
// counts and the coarser levels
// ---------------------------------------------------------------------------------------------
// hits and the cells of the XY, XZ and YZ planes whose column holds a hit
__device__ __forceinline__ void occ_counts(const uint64_t m[8], uint16_t out[4]) {
  int h = 0, xy = 0, xz = 0, yz = 0;
#pragma unroll
  for (int w = 0; w < 8; ++w) h += __popcll(m[w]);
  // along z: the word's z bit is 4, in-word z bits are 2 and 5
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint64_t x = m[w] | m[w + 4];
    x |= x >> 32;
    x |= x >> 4;
    xy += __popcll(x & 0x0f0f0f0full);
  }
  // along y: word bit 2, in-word bits 1 and 4
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int w = (t & 1) | ((t & 2) << 1);
    uint64_t x = m[w] | m[w + 2];
    x |= x >> 16;
    x |= x >> 2;
    xz += __popcll(x & 0x0000333300003333ull);
  }
  // along x: word bit 1, in-word bits 0 and 3
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int w = 2 * t;
    uint64_t x = m[w] | m[w + 1];
    x |= x >> 8;
    x |= x >> 1;
    yz += __popcll(x & 0x0055005500550055ull);
  }
  out[0] = uint16_t(h);
  out[1] = uint16_t(xy);
  out[2] = uint16_t(xz);
  out[3] = uint16_t(yz);
}

__global__ void __launch_bounds__(kBlock) k_occ_zero(unsigned long long* __restrict__ mask, int64_t cap,
                                                     const int64_t* __restrict__ n_ptr) {
  const int64_t n = *n_ptr < cap ? *n_ptr : cap;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
#pragma unroll
    for (int w = 0; w < 8; ++w) mask[w * cap + i] = 0ull;
}

__global__ void __launch_bounds__(kBlock) k_occ_leaf_counts(const unsigned long long* __restrict__ mask, int64_t cap,
                                                            const int64_t* __restrict__ n_ptr,
                                                            uint16_t* __restrict__ hits) {
  const int64_t n = *n_ptr < cap ? *n_ptr : cap;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    uint64_t m[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) m[w] = mask[w * cap + i];
    uint16_t c[4];
    occ_counts(m, c);
#pragma unroll
    for (int t = 0; t < 4; ++t) hits[t * cap + i] = c[t];
  }
}

// the byte-wise OR of one 64-bit word, byte b -> bit b
__device__ __forceinline__ uint32_t byte_any(uint64_t x) {
  x |= x >> 4;
  x |= x >> 2;
  x |= x >> 1;
  x &= 0x0101010101010101ull;
  return uint32_t((x * 0x0102040810204080ull) >> 56);
}

// Parent p's children are the voxels of the level below with key >> 3 == key_p, contiguous in
// key order: found by a search for key_p << 3.
// cstride / pstride: the occupancy capacities (mask and count strides); cmax / pmax: the most
// voxels both the level and its occupancy hold
template <class Key>
__global__ void __launch_bounds__(kBlock) k_occ_up(const Key* __restrict__ ckeys, const int64_t* __restrict__ n_child,
                                                   const unsigned long long* __restrict__ cmask, int64_t cstride,
                                                   int64_t cmax, const Key* __restrict__ pkeys,
                                                   const int64_t* __restrict__ n_par,
                                                   unsigned long long* __restrict__ pmask, uint16_t* __restrict__ hits,
                                                   int64_t pstride, int64_t pmax, int64_t* stats) {
  const int64_t np = *n_par, nc = *n_child;
  if (np > pmax || nc > cmax) {
    if (blockIdx.x == 0 && threadIdx.x == 0) occ_flag(stats, VX_FLAG_VOXEL_CAPACITY);
    return;
  }
  for (int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x; p < np; p += int64_t(gridDim.x) * kBlock) {
    const Key pk = pkeys[p];
    const Key first = Key(pk << 3);
    int64_t lo = 0, hi = nc;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (ckeys[mid] < first) lo = mid + 1; else hi = mid;
    }
    uint64_t m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t c = lo; c < nc && Key(ckeys[c] >> 3) == pk; ++c) {
      const int oct = int(ckeys[c] & 7);
      uint64_t word = 0;
#pragma unroll
      for (int w = 0; w < 8; ++w) word |= uint64_t(byte_any(cmask[w * cstride + c])) << (8 * w);
#pragma unroll
      for (int w = 0; w < 8; ++w)
        if (w == oct) m[w] = word;
    }
#pragma unroll
    for (int w = 0; w < 8; ++w) pmask[w * pstride + p] = m[w];
    uint16_t cnt[4];
    occ_counts(m, cnt);
#pragma unroll
    for (int t = 0; t < 4; ++t) hits[t * pstride + p] = cnt[t];
  }
}

// the leaf's count against its occupancy capacity
__global__ void k_occ_check(const int64_t* __restrict__ n_leaf, int64_t vcap, int64_t ocap, int64_t* stats) {
  if (threadIdx.x == 0 && (*n_leaf > vcap || *n_leaf > ocap)) occ_flag(stats, VX_FLAG_VOXEL_CAPACITY);
}

int occ_blocks(int64_t n) {
  const int64_t b = (n + kBlock - 1) / kBlock;
  return int(b < 1 ? 1 : (b > 4 * kGrid ? 4 * kGrid : b));
}

}  // namespace

size_t occupancy_ws_bytes(int64_t n_prims, int64_t max_cand, int64_t max_pairs, bool key64) {
  Carver cv(nullptr);
  front_ws_carve(cv, n_prims, max_cand, max_pairs, key64, nullptr);
  return cv.off + 256;
}

vx_status occupancy_run(int kind, const vx_grid* g, const float* data, int64_t n_prims, const int64_t* offsets,
                        int64_t n_fib, float radius, const vx_voxels* leaf, const vx_voxels* out,
                        const int64_t* n_levels, int levels, int64_t max_cand, int64_t max_pairs,
                        const vx_occupancy* occ, void* ws, int64_t* stats, hipStream_t s) {
  const bool key64 = g->log2_res > 10;
  Carver cv(ws);
  FrontWs w;
  front_ws_carve(cv, n_prims, max_cand, max_pairs, key64, &w);
  voxelize_front(kind, g, data, n_prims, offsets, n_fib, radius, max_cand, max_pairs, w, stats, s, nullptr, false);
  const Lat L = make_lat(g, kind, radius);
  hipLaunchKernelGGL(k_occ_check, dim3(1), dim3(64), 0, s, n_levels, leaf->cap, occ[0].cap, stats);
  hipLaunchKernelGGL(k_occ_zero, dim3(occ_blocks(occ[0].cap)), dim3(kBlock), 0, s,
                     reinterpret_cast<unsigned long long*>(occ[0].mask), occ[0].cap, n_levels);
  {
    VX_TIMED(kind == 0 ? "occ_pairs_tri" : "occ_pairs_fib", s);
    uint32_t* at = reinterpret_cast<uint32_t*>(w.pa.w);    // the pairs' weights are not computed here
#define VX_OCC(KD, K)                                                                                           \
  do {                                                                                                          \
    hipLaunchKernelGGL(k_occ_find<K>, dim3(kGrid * 4), dim3(kBlock), 0, s, (const K*)w.pa.keys, w.ctl,          \
                       (const K*)leaf->keys, n_levels, leaf->cap, occ[0].cap, at, stats);                       \
    hipLaunchKernelGGL((k_occ_pairs<KD, K>), dim3(kGrid * 4), dim3(kBlock), 0, s, w.rec, (const K*)w.pa.keys, \
                       w.pa.prim, at, w.ctl, L, reinterpret_cast<unsigned long long*>(occ[0].mask),             \
                       occ[0].cap);                                                                             \
  } while (0)
    if (kind == 0) {
      if (key64) VX_OCC(0, uint64_t); else VX_OCC(0, uint32_t);
    } else {
      if (key64) VX_OCC(1, uint64_t); else VX_OCC(1, uint32_t);
    }
#undef VX_OCC
  }
  VX_TIMED("occ_levels", s);
  hipLaunchKernelGGL(k_occ_leaf_counts, dim3(occ_blocks(occ[0].cap)), dim3(kBlock), 0, s,
                     reinterpret_cast<const unsigned long long*>(occ[0].mask), occ[0].cap, n_levels, occ[0].hits);
  for (int l = 1; l < levels; ++l) {
    const vx_voxels& C = l == 1 ? *leaf : out[l - 2];
    const vx_voxels& P = out[l - 1];
    const int64_t pmax = imin(P.cap, occ[l].cap), cmax = imin(C.cap, occ[l - 1].cap);
#define VX_UP(K)                                                                                                  \
  hipLaunchKernelGGL(k_occ_up<K>, dim3(occ_blocks(pmax)), dim3(kBlock), 0, s, (const K*)C.keys, n_levels + l - 1, \
                     reinterpret_cast<const unsigned long long*>(occ[l - 1].mask), occ[l - 1].cap, cmax,        \
                     (const K*)P.keys, n_levels + l, reinterpret_cast<unsigned long long*>(occ[l].mask),        \
                     occ[l].hits, occ[l].cap, pmax, stats)
    if (key64) VX_UP(uint64_t); else VX_UP(uint32_t);
#undef VX_UP
  }
  return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
}

}  // namespace vx
