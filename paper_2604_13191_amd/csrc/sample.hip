// sample.hip -- the paper's sampling voxelizer (Sec. 3.2), a baseline for the exact path.
//
// Points are generated on the primitives from kernel indices (no random numbers) and each is
// stored in the voxel that contains it:
//   * fibers: the uniform Catmull-Rom span of every segment (control points i-1 .. i+2, the
//     fiber's end points repeated) cut at t = j / m into m chords, n samples per chord at
//     fractions (k + 1/2) / n, each weighing chord length / n along the chord's tangent;
//   * triangles: max(1, floor(N A / A_max)) samples per triangle (in proportion to its area
//     relative to the largest), sample k at ((k + 1/2) / n_T, radical inverse of k) mapped to
//     barycentric coordinates by Heitz's low-distortion triangle map, each weighing A / n_T.
// Per voxel: the number of samples, their weight and their moments (n n^T or I - t t^T), summed
// in sample order.  Positions are FP64 in grid units with the operation order fixed (no
// contraction, explicit fused multiply-adds), so every sample's voxel is reproducible; samples
// outside the grid get a key above every voxel's and are dropped after the sort.
#pragma clang fp contract(off)

#include "geom.hpp"
#include "vx_internal.hpp"

namespace vx {
namespace {

enum { SC_TOTAL = 0, SC_SEGS = 1, SC_VOX = 2, SC_QMAX = 3, SC_SORT = 4, SC_OUTSIDE = 5, SC_WORDS = 6 };

// A record: the voxel's key, the id of a chord or triangle and how many of its samples lie there, in
// one word or with the key apart.
struct RecordBits {
  int id, cnt;        // of the id, and above it of the count less one
  bool packed;        // key << (cnt + id) | (count - 1) << id | id; else the key and the rest apart
};

struct SampWs {
  int64_t* ctl;       // [8] (SC_*)
  int64_t* cnt;       // [n_prims + 1] samples per primitive, then their offsets
  double* q;          // triangles: [n] squared twice-area
  float4* dirs;       // fibers: [n_pts * m] chord tangents; triangles: [n] normals; with the weight of
                      // each of the chord's or triangle's samples
  PairBufs a, b;      // sample records (key, chord or triangle id), ping-pong for the sort; packed: no prim
  RecordBits bits;
  int32_t* filled;    // triangles: [kEmitGrid * kWaves] records that each wave of the emission wrote
  int32_t* hist;
  int64_t* partial;
  uint64_t* mask;     // [max_samples / 64] one bit per sorted sample: the first of its key
  int64_t* start;     // [max_vox + 2] first sample of every key
};

// One word where 64-bit keys, the bit for samples outside (fibers) and the id fit it: a sort pass then moves 16 bytes a
// record, not 24 (41.7 M: 0.19 ms, 0.25 ms apart).  32-bit keys stay apart: packing them would save
// nothing and double what the digit counts read.  Counts take what bits are left, up to the 6 that a
// wave's 64 samples need.
RecordBits record_bits(int kind, int64_t n_prims, int log2R, int sub) {
  const int64_t ids = n_prims * (kind == 0 ? 1 : int64_t(sub));
  RecordBits r{1, 0, false};
  while (r.id < 32 && (int64_t(1) << r.id) < ids) ++r.id;
  const int left = 64 - (3 * log2R + (kind == 0 ? 0 : 1) + r.id);
  r.packed = log2R > 10 && left >= 0;
  const int room = r.packed ? left : 32 - r.id;
  r.cnt = kind != 0 ? 0 : (room < 6 ? room : 6);
  return r;
}

// Blocks of the emission of triangles' samples, whose waves take equal stretches of them, a few rows of 64
// at least: 512 samples a wave up to 1,024 blocks, 1,024 above (the sort's first pass serves the
// stretches one by one, so more of them cost it what the emission gains: emission and sort of 1.0 M samples
// 160 us, at 1,024 a wave 165, at 256 190; of 5 M 187, at 512 a wave 224).  One fill of the chip at most: six
// blocks a CU by their LDS (41.7 M samples: 0.30 ms; 0.33 with four, 0.31 with eight).
constexpr int kEmitGrid = 1536;
int emit_blocks(int64_t max_samples) {
  const int64_t few = (max_samples + 512 * kWaves - 1) / (512 * kWaves);
  const int64_t many = (max_samples + 1024 * kWaves - 1) / (1024 * kWaves);
  const int64_t b = few < kGrid ? few : (many < kGrid ? kGrid : many);
  return int(b < 1 ? 1 : (b > kEmitGrid ? kEmitGrid : b));
}

size_t samp_ws_layout(int kind, int64_t n_prims, int64_t max_samples, int64_t max_vox, int log2R, int sub,
                      void* base, SampWs* w) {
  Carver cv(base);
  SampWs x;
  x.ctl = cv.take<int64_t>(8);
  x.cnt = cv.take<int64_t>(n_prims + 1);
  x.q = cv.take<double>(kind == 0 ? n_prims : 1);
  x.dirs = cv.take<float4>(kind == 0 ? n_prims : n_prims * int64_t(sub));
  const int kb = log2R > 10 ? 8 : 4;
  x.bits = record_bits(kind, n_prims, log2R, sub);
  for (PairBufs* p : {&x.a, &x.b}) {
    p->keys = cv.take<uint8_t>(max_samples * kb);
    p->w = nullptr;
    p->prim = x.bits.packed ? nullptr : cv.take<uint32_t>(max_samples);
  }
  x.filled = cv.take<int32_t>(kind == 0 ? kEmitGrid * kWaves : 0);
  x.hist = cv.take<int32_t>(int64_t(kRadixBuckets) * kGrid);
  x.partial = cv.take<int64_t>(kGrid + 1);
  x.mask = cv.take<uint64_t>((max_samples + 63) / 64);
  x.start = cv.take<int64_t>(max_vox + 2);
  if (w) *w = x;
  return cv.off + 256;
}

struct Grid64 {
  double bmin[3];
  double vs;       // grid units per world unit, R / extent
  int64_t R;
};

__device__ __forceinline__ void to_grid(const float* p, const Grid64& G, double g[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) g[a] = (double(p[a]) - G.bmin[a]) * G.vs;
}

// the key of grid point X, or `outside` when X lies outside [0, R)^3
template <class Key>
__device__ __forceinline__ Key sample_key(const double X[3], const Grid64& G, Key outside) {
  uint32_t v[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double f = floor(X[a]);
    if (!(f >= 0.0 && f < double(G.R))) return outside;
    v[a] = uint32_t(f);
  }
  return Key(morton3(v[0], v[1], v[2]));
}

__device__ __forceinline__ bool finite3(const float* p) {
  return isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]);
}
__device__ __forceinline__ void flag_input(int64_t* stats) {
  atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_INPUT);
}
// samples that fell outside the grid, one atomic per wave
__device__ __forceinline__ void add_outside(int64_t n, int64_t* ctl) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
  if (lane_id() == 0 && n) atomicAdd(reinterpret_cast<unsigned long long*>(ctl + SC_OUTSIDE), (unsigned long long)n);
}

// offsets: 0 first, non-decreasing, n_pts last
__global__ void k_samp_offsets(const int64_t* __restrict__ off, int64_t F, int64_t n_pts, int64_t* stats) {
  for (int64_t f = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; f <= F; f += int64_t(gridDim.x) * blockDim.x) {
    bool bad = f == 0 ? off[0] != 0 : off[f] < off[f - 1];
    if (f == F) bad = bad || off[F] != n_pts;
    if (bad)
      atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_OFFSETS);
  }
}

// the Catmull-Rom span of segment (i, i+1) of a fiber [a, b): polynomial coefficients
__device__ __forceinline__ void span_coeffs(const float* __restrict__ pts, int64_t i, int64_t a, int64_t b,
                                            const Grid64& G, double c[4][3]) {
  double P[4][3];
  to_grid(pts + 3 * (i > a ? i - 1 : i), G, P[0]);
  to_grid(pts + 3 * i, G, P[1]);
  to_grid(pts + 3 * (i + 1), G, P[2]);
  to_grid(pts + 3 * (i + 2 < b ? i + 2 : i + 1), G, P[3]);
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    c[0][x] = P[1][x];
    c[1][x] = 0.5 * (P[2][x] - P[0][x]);
    c[2][x] = ((P[0][x] - 2.5 * P[1][x]) + 2.0 * P[2][x]) - 0.5 * P[3][x];
    c[3][x] = 0.5 * (P[3][x] - P[0][x]) + 1.5 * (P[1][x] - P[2][x]);
  }
}

__device__ __forceinline__ void span_point(const double c[4][3], double t, double out[3]) {
#pragma unroll
  for (int x = 0; x < 3; ++x) out[x] = fma(fma(fma(c[3][x], t, c[2][x]), t, c[1][x]), t, c[0][x]);
}

// fiber [a, b) holding point i (offsets non-decreasing): the last f with offsets[f] <= i
__device__ __forceinline__ int64_t fiber_of(const int64_t* __restrict__ off, int64_t F, int64_t i) {
  int64_t lo = 0, hi = F;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// per point: the samples of its segment (m * n, or 0 when the point ends its fiber) and the
// chords' tangents and sample weights
__global__ void __launch_bounds__(kBlock) k_samp_fib_count(const float* __restrict__ pts, int64_t n_pts,
                                                           const int64_t* __restrict__ off, int64_t F, int sub,
                                                           int per, Grid64 G, int64_t* __restrict__ cnt,
                                                           float4* __restrict__ dirs, int64_t* stats) {
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n_pts; i += int64_t(gridDim.x) * kBlock) {
    const int64_t f = fiber_of(off, F, i);
    const int64_t a = off[f], b = off[f + 1];
    const bool seg = a >= 0 && i >= a && i + 1 < b && b <= n_pts;   // in bounds whatever the offsets hold
    cnt[i] = seg ? int64_t(sub) * per : 0;
    if (!seg) continue;
    if (!finite3(pts + 3 * i) || !finite3(pts + 3 * (i + 1))) flag_input(stats);
    double c[4][3];
    span_coeffs(pts, i, a, b, G, c);
    for (int j = 0; j < sub; ++j) {
      double A[3], B[3];
      span_point(c, double(j) / double(sub), A);
      span_point(c, double(j + 1) / double(sub), B);
      const double d0 = B[0] - A[0], d1 = B[1] - A[1], d2 = B[2] - A[2];
      const double len = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
      const double il = len > 0.0 ? 1.0 / len : 0.0;
      dirs[i * sub + j] = make_float4(float(d0 * il), float(d1 * il), float(d2 * il), float(len / double(per)));
    }
  }
}

// the emitted records: the sort's buffers
template <class Key>
struct SampOut {
  Key* keys;
  uint32_t* ids;
  RecordBits bits;
  __device__ __forceinline__ void put(int64_t o, Key key, uint32_t id, int count) const {
    const uint64_t low = uint64_t(count - 1) << bits.id | id;
    if (bits.packed) {
      keys[o] = Key(uint64_t(key) << (bits.id + bits.cnt) | low);
    } else {
      keys[o] = key;
      ids[o] = uint32_t(low);
    }
  }
};

template <class Key>
__global__ void __launch_bounds__(kBlock) k_samp_fib_emit(const float* __restrict__ pts, int64_t n_pts,
                                                          const int64_t* __restrict__ off, int64_t F, int sub,
                                                          int per, Grid64 G, const int64_t* __restrict__ soff,
                                                          int64_t* __restrict__ ctl, int64_t cap, Key outside,
                                                          SampOut<Key> out) {
  if (ctl[SC_TOTAL] > cap) return;                  // over capacity: nothing is written
  int64_t outs = 0;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n_pts; i += int64_t(gridDim.x) * kBlock) {
    if (soff[i + 1] == soff[i]) continue;
    const int64_t f = fiber_of(off, F, i);
    const int64_t a = off[f], b = off[f + 1];
    double c[4][3];
    span_coeffs(pts, i, a, b, G, c);
    int64_t o = soff[i];
    for (int j = 0; j < sub; ++j) {
      double A[3], B[3], d[3];
      span_point(c, double(j) / double(sub), A);
      span_point(c, double(j + 1) / double(sub), B);
#pragma unroll
      for (int x = 0; x < 3; ++x) d[x] = B[x] - A[x];
      const uint32_t id = uint32_t(i * sub + j);
      for (int k = 0; k < per; ++k) {
        const double fr = (double(k) + 0.5) / double(per);
        double X[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) X[x] = fma(fr, d[x], A[x]);
        const Key key = sample_key<Key>(X, G, outside);
        outs += key == outside;
        out.put(o, key, id, 1);
        ++o;
      }
    }
  }
  add_outside(outs, ctl);
}

__device__ __forceinline__ void tri_grid(const float* __restrict__ tris, int64_t t, const Grid64& G, double g[3][3],
                                         double c[3]) {
#pragma unroll
  for (int v = 0; v < 3; ++v) to_grid(tris + 9 * t + 3 * v, G, g[v]);
  double e0[3], e1[3];
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    e0[x] = g[1][x] - g[0][x];
    e1[x] = g[2][x] - g[0][x];
  }
  c[0] = e0[1] * e1[2] - e0[2] * e1[1];
  c[1] = e0[2] * e1[0] - e0[0] * e1[2];
  c[2] = e0[0] * e1[1] - e0[1] * e1[0];
}

// squared twice-areas and their maximum (non-negative doubles order like their bits)
__global__ void __launch_bounds__(kBlock) k_samp_tri_q(const float* __restrict__ tris, int64_t n, Grid64 G,
                                                       double* __restrict__ q, int64_t* __restrict__ ctl,
                                                       int64_t* stats) {
  __shared__ uint64_t red[kWaves];
  uint64_t best = 0;
  for (int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x; t < n; t += int64_t(gridDim.x) * kBlock) {
    double g[3][3], c[3];
    tri_grid(tris, t, G, g, c);
    double qq = c[0] * c[0] + c[1] * c[1] + c[2] * c[2];
    if (!finite3(tris + 9 * t) || !finite3(tris + 9 * t + 3) || !finite3(tris + 9 * t + 6) || !isfinite(qq)) {
      flag_input(stats);
      qq = 0.0;
    }
    q[t] = qq;
    const uint64_t b = qq > 0.0 ? uint64_t(__double_as_longlong(qq)) : 0ull;
    best = b > best ? b : best;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t u = uint64_t(__shfl_xor((unsigned long long)best, o, 64));
    best = u > best ? u : best;
  }
  if (lane_id() == 0) red[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t m = 0;
    for (int i = 0; i < kWaves; ++i) m = red[i] > m ? red[i] : m;
    atomicMax(reinterpret_cast<unsigned long long*>(ctl + SC_QMAX), (unsigned long long)m);
  }
}

// max(1, floor(N sqrt(q / qmax))): the guess from the square root, settled on products
__device__ __forceinline__ int64_t tri_samples(double q, double qmax, int N) {
  if (!(qmax > 0.0)) return 1;
  const double nn = double(N) * double(N) * q;
  int64_t k = int64_t(floor(double(N) * sqrt(q / qmax)));
  if (k < 0) k = 0;
  while (double(k + 1) * double(k + 1) * qmax <= nn) ++k;
  while (k > 0 && double(k) * double(k) * qmax > nn) --k;
  return k > 1 ? k : 1;
}

__global__ void __launch_bounds__(kBlock) k_samp_tri_count(const float* __restrict__ tris, int64_t n, Grid64 G, int N,
                                                           const double* __restrict__ q,
                                                           const int64_t* __restrict__ ctl,
                                                           int64_t* __restrict__ cnt, float4* __restrict__ dirs) {
  const double qmax = __longlong_as_double((long long)ctl[SC_QMAX]);
  for (int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x; t < n; t += int64_t(gridDim.x) * kBlock) {
    const int64_t nt = tri_samples(q[t], qmax, N);
    cnt[t] = nt;
    double g[3][3], c[3];
    tri_grid(tris, t, G, g, c);
    const double a2 = sqrt(q[t]);
    const double ia = a2 > 0.0 ? 1.0 / a2 : 0.0;
    dirs[t] = make_float4(float(c[0] * ia), float(c[1] * ia), float(c[2] * ia), float(0.5 * a2 / double(nt)));
  }
}

__device__ __forceinline__ double radical_inverse2(uint32_t k) { return double(__brev(k)) * 0x1p-32; }

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Each wave takes an equal stretch of the samples, whatever triangles they fall in, and walks through
// its triangles 64 at a time: their frames and first samples go to LDS, then one lane a sample finds
// its triangle by bisection there.  A triangle's samples that fall in one voxel leave as one record
// with their count, where the first of them stood: the sort keeps records in this order, so the
// voxel adds the same numbers in the same order.  They find each other, within a row of 64, through
// a table in LDS: the lowest lane of a slot is taken for the first if key and triangle agree (two
// voxels in one slot: the other's samples stay single).  A wave's records lie at the start of its
// stretch; samples outside the grid leave none.  Bound by FP64 arithmetic (41.7 M samples of 4.7 M triangles: 0.30 ms, leaving 16.7 M
// records; 0.24 ms as records of one sample each, but every sort pass 0.25 ms instead of 0.11).
constexpr int kSampSlots = 256;
template <class Key>
__global__ void __launch_bounds__(kBlock) k_samp_tri_emit(const float* __restrict__ tris, int64_t n, Grid64 G,
                                                          const int64_t* __restrict__ soff,
                                                          int64_t* __restrict__ ctl, int64_t cap, Key outside,
                                                          SampOut<Key> out, int32_t* __restrict__ filled) {
  __shared__ double frames[kWaves][10][64];         // third vertex; edges from it to the others; 1 / samples
  __shared__ int32_t firsts[kWaves][65];            // less the tile's first sample
  __shared__ uint32_t slots[kWaves][kSampSlots], more[kWaves][64];
  const int lane = lane_id(), wv = threadIdx.x >> 6, wave = int(blockIdx.x) * kWaves + wv;
  double(*fr)[64] = frames[wv];
  int32_t* first = firsts[wv];
  uint32_t* slot = slots[wv];
  const int64_t total = ctl[SC_TOTAL];
  const int64_t waves = int64_t(gridDim.x) * kWaves, range = (total + waves - 1) / waves;
  const int64_t o0 = wave * range, o1 = o0 + range < total ? o0 + range : total;
  if (total > cap || o0 >= o1) {                    // over capacity: nothing is written
    if (lane == 0) filled[wave] = 0;
    return;
  }
  // the triangle of sample o0: the last t with soff[t] <= o0, 64 probes a round
  int64_t tlo = 0, thi = n;
  while (thi - tlo > 1) {
    const int64_t step = (thi - tlo + 63) / 64, p = tlo + lane * step;
    const int64_t c = __popcll(__ballot(p < thi && soff[p] <= o0));
    tlo += (c - 1) * step;
    thi = tlo + step < thi ? tlo + step : thi;
  }
#pragma unroll
  for (int i = 0; i < kSampSlots; i += 64) slot[i + lane] = 0xffffffffu;
  uint32_t row = 0xffffffffu >> 6;                  // counts down: a row's entries are below all earlier ones
  const int most = 1 << out.bits.cnt;               // samples of a record
  int64_t outs = 0, o = o0;
  for (int64_t t0 = tlo; t0 < n; t0 += 64) {
    const int nt = int(n - t0 < 64 ? n - t0 : 64);
    const int64_t base = soff[t0];
    if (base >= o1) break;
    if (lane < nt) {
      double g[3][3], c[3];
      tri_grid(tris, t0 + lane, G, g, c);
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        fr[x][lane] = g[2][x];
        fr[3 + x][lane] = g[0][x] - g[2][x];
        fr[6 + x][lane] = g[1][x] - g[2][x];
      }
      const int64_t s0 = soff[t0 + lane];
      first[lane] = int32_t(s0 - base);
      fr[9][lane] = recip(double(soff[t0 + lane + 1] - s0));
    }
    if (lane == 0) first[nt] = int32_t(soff[t0 + nt] - base);
    wave_lds_fence();
    const int32_t q0 = int32_t(o0 > base ? o0 - base : 0);
    const int32_t q1 = int32_t(o1 - base < first[nt] ? o1 - base : first[nt]);
    for (int32_t qr = q0; qr < q1; qr += 64, --row) {
      const int32_t q = qr + lane < q1 ? qr + lane : q1 - 1;     // past the end: the last sample again, dropped
      const bool on = qr + lane < q1;
      int lo = 0, hi = nt;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first[mid] <= q) lo = mid; else hi = mid;
      }
      const int32_t k = q - first[lo];
      // (half-odd numbers below 2^21 over integers below it: the correctly rounded quotient)
      const double u1 = quotient(double(k) + 0.5, double(first[lo + 1] - first[lo]), fr[9][lo]);
      const double u2 = radical_inverse2(uint32_t(k));
      // Heitz's map, both halves by selects
      const bool up = u2 > u1;
      const double h1 = 0.5 * u1, h2 = 0.5 * u2;
      const double b0 = up ? h1 : u1 - h2;
      const double b1 = up ? u2 - h1 : h2;
      double X[3];
#pragma unroll
      for (int x = 0; x < 3; ++x) X[x] = fma(b0, fr[3 + x][lo], fma(b1, fr[6 + x][lo], fr[x][lo]));
      const Key key = sample_key<Key>(X, G, outside);
      outs += on && key == outside;
      bool put = on;
      int count = 1;
      if (most > 1) {
        const uint32_t h = (uint32_t(key) * 0x9e3779b1u + uint32_t(uint64_t(key) >> 32) + uint32_t(lo) * 0x85ebca6bu) >> 24;
        more[wv][lane] = 0;
        if (on) atomicMin(&slot[h], row << 6 | uint32_t(lane));
        wave_lds_fence();
        const int lead = on ? int(slot[h] & 63u) : lane;
        bool same = __shfl(lo, lead, 64) == lo && __shfl(uint32_t(key), lead, 64) == uint32_t(key);
        if (sizeof(Key) == 8)
          same = same && __shfl(uint32_t(uint64_t(key) >> 32), lead, 64) == uint32_t(uint64_t(key) >> 32);
        if (on && same && lead != lane)              // joins the first's record while that has room
          put = int(atomicAdd(&more[wv][lead], 1u)) >= most - 1;
        wave_lds_fence();
        const int joined = int(more[wv][lane]);
        if (put && (lead == lane || !same)) count = 1 + (joined < most - 1 ? joined : most - 1);
        wave_lds_fence();
      }
      put = put && key != outside;
      const uint64_t m = __ballot(put);
      if (put)
        out.put(o + __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0)), key,
                uint32_t(t0 + lo), count);
      o += __popcll(m);
    }
    wave_lds_fence();
  }
  if (lane == 0) filled[wave] = int32_t(o - o0);
  add_outside(outs, ctl);
}

struct SampTotal {
  int64_t* ctl;
  int64_t* stats;
  int64_t cap;
  __device__ void operator()(int64_t total, int64_t n) const {
    ctl[SC_TOTAL] = total;
    stats[VX_STAT_CAND] = total;
    if (total > cap) {
      atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_PAIR_CAPACITY);
    }
    (void)n;
  }
};
struct CntOut {
  int64_t* o;
  __device__ void operator()(int64_t i, int64_t ex, int64_t) const { o[i] = ex; }
};
struct CntIn {
  const int64_t* a;
  __device__ int64_t operator()(int64_t i) const { return a[i]; }
};
// The sort's element count: the samples, or the records (filled: what each of the emission's waves
// wrote, added here -- counted by the waves, on one address 16 ns apart, they took a third of the emission),
// or none when they did not fit; and its 64s.
__global__ void __launch_bounds__(kBlock) k_samp_n(int64_t* ctl, int64_t cap, const int32_t* __restrict__ filled,
                                                   int waves) {
  __shared__ int64_t tmp[kWaves + 1];
  const int64_t total = ctl[SC_TOTAL];
  int64_t mine = 0, n = total;
  if (filled) {
    for (int i = threadIdx.x; i < waves; i += kBlock) mine += filled[i];
    (void)block_exclusive_scan(mine, tmp, n);
  }
  if (threadIdx.x != 0) return;
  n = total <= cap ? n : 0;
  ctl[SC_SORT] = n;
  ctl[SC_WORDS] = (n + 63) / 64;
}
// voxels = key segments, less the trailing one of samples outside the grid (fibers)
__global__ void k_samp_finish(int kind, int64_t* ctl, int64_t* stats, int64_t cap, int64_t vcap) {
  if (threadIdx.x != 0) return;
  const int64_t out = ctl[SC_OUTSIDE];
  const int64_t nv = ctl[SC_SEGS] - (kind == 1 && out > 0);
  stats[VX_STAT_PAIRS] = ctl[SC_TOTAL] <= cap ? ctl[SC_TOTAL] - out : 0;
  stats[VX_STAT_VOXELS] = nv;
  if (nv > vcap)
    atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_VOXEL_CAPACITY);
  ctl[SC_VOX] = nv <= vcap ? nv : 0;
}

// the sorted records' keys, ids and counts
template <class Key>
struct Sorted {
  const Key* keys;
  const uint32_t* ids;
  RecordBits bits;
  __device__ __forceinline__ Key key(int64_t i) const {
    return bits.packed ? Key(uint64_t(keys[i]) >> (bits.id + bits.cnt)) : keys[i];
  }
  template <bool PACKED>
  __device__ __forceinline__ uint32_t id(int64_t i, int& count) const {
    const uint64_t r = PACKED ? uint64_t(keys[i]) : uint64_t(ids[i]);
    count = 1 + int((r >> bits.id) & ((uint64_t(1) << bits.cnt) - 1));
    return uint32_t(r & ((uint64_t(1) << bits.id) - 1));
  }
};

// One bit a record: does its voxel start here?  One read of the records instead of the two that a scan over
// them takes (16.7 M records, 3.1 M voxels: 0.061 ms with the starts).  A block serves a stretch of words
// and leaves its number of starts: of 32 words at least, and eight waves, whose loads in flight a large
// set needs (with four 0.077 ms).
constexpr int kHeadRows = 8;
constexpr int kHeadBlock = 512, kHeadWaves = kHeadBlock / 64;
__device__ __forceinline__ int64_t head_chunk(int64_t words) {
  const int64_t c = (words + gridDim.x - 1) / gridDim.x;
  return (c + kHeadRows - 1) / kHeadRows * kHeadRows;
}
int head_blocks(int64_t max_samples) {
  const int64_t b = ((max_samples + 63) / 64 + 31) / 32;
  return int(b < 1 ? 1 : (b > kGrid ? kGrid : b));
}
template <class Key>
__global__ void __launch_bounds__(kHeadBlock) k_samp_heads(Sorted<Key> s, const int64_t* __restrict__ ctl,
                                                       uint64_t* __restrict__ mask, int64_t* __restrict__ partial) {
  __shared__ int64_t tmp[kHeadWaves + 1];
  const int64_t n = ctl[SC_SORT], words = ctl[SC_WORDS], chunk = head_chunk(words);
  const int64_t b0 = int64_t(blockIdx.x) * chunk, b1 = b0 + chunk < words ? b0 + chunk : words;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  int64_t count = 0;
  for (int64_t w0 = b0 + wave * kHeadRows; w0 < b1; w0 += kHeadWaves * kHeadRows) {
    Key k[kHeadRows], p[kHeadRows];
#pragma unroll
    for (int r = 0; r < kHeadRows; ++r) {
      const int64_t i = (w0 + r) * 64 + lane;
      k[r] = i < n ? s.key(i) : Key(0);
      p[r] = i < n && i > 0 ? s.key(i - 1) : Key(0);
    }
#pragma unroll
    for (int r = 0; r < kHeadRows; ++r) {
      const int64_t i = (w0 + r) * 64 + lane;
      const uint64_t m = __ballot(i < n && (i == 0 || k[r] != p[r]));
      if (lane == 0 && w0 + r < b1) mask[w0 + r] = m;
      count += w0 + r < b1 ? __popcll(m) : 0;
    }
  }
  int64_t all;
  (void)block_exclusive_scan_n<kHeadWaves>(lane == 0 ? count : int64_t(0), tmp, all);
  if (threadIdx.x == 0) partial[blockIdx.x] = all;
}

// Voxel starts from the masks: a word's offset is the voxels that start before it.  A block scans its
// words' counts, one a thread, and its waves write the starts, a lane per bit and four words at a time
// (a thread writing all the starts of a word took 20 us of 20,000 samples in as many voxels).  start has cap
// entries, the voxels' capacity + 2.
__global__ void __launch_bounds__(kBlock) k_samp_starts(const uint64_t* __restrict__ mask, int64_t* __restrict__ ctl,
                                                        const int64_t* __restrict__ partial,
                                                        int64_t* __restrict__ start, int64_t cap) {
  __shared__ int64_t tmp[kWaves + 1];
  __shared__ uint64_t word[kBlock];
  __shared__ int32_t at[kBlock];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const int64_t words = ctl[SC_WORDS], chunk = head_chunk(words);
  const int64_t b0 = int64_t(blockIdx.x) * chunk, b1 = b0 + chunk < words ? b0 + chunk : words;
  int64_t all, base = block_scan_base(partial, tmp, all);
  if (blockIdx.x == 0 && tid == 0) {
    if (all < cap) start[all] = ctl[SC_SORT];
    ctl[SC_SEGS] = all;
  }
  for (int64_t t0 = b0; t0 < b1; t0 += kBlock) {
    const uint64_t m = t0 + tid < b1 ? mask[t0 + tid] : 0;
    int64_t tot;
    at[tid] = int32_t(block_exclusive_scan(int64_t(__popcll(m)), tmp, tot));
    word[tid] = m;
    __syncthreads();
    for (int q0 = wave * 4; q0 < kBlock && t0 + q0 < b1; q0 += kWaves * 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {                  // (words past b1 are empty)
        const uint64_t x = word[q0 + r];
        const int64_t v = base + at[q0 + r] + __popcll(x & lt);
        if (((x >> lane) & 1) && v < cap) start[v] = 64 * (t0 + q0 + r) + lane;
      }
    }
    base += tot;
    __syncthreads();
  }
}

// after a conditional pass: its result back to where the passes before it ended
template <class Key>
__global__ void __launch_bounds__(kBlock) k_samp_back(const Key* __restrict__ kin, const uint32_t* __restrict__ iin,
                                                      Key* __restrict__ kout, uint32_t* __restrict__ iout,
                                                      const int64_t* __restrict__ ctl) {
  if (ctl[SC_OUTSIDE] == 0) return;
  const int64_t n = ctl[SC_SORT];
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    kout[i] = kin[i];
    if (iin) iout[i] = iin[i];
  }
}

// A wave sums 64 voxels, one a lane, each voxel's samples in order, a record's direction as often as it
// counts.  Bound by the gathers.  Triangles, where the 64 voxels' records fit one tile: they are one stretch
// of the sorted list, so their ids are read and their directions gathered together into LDS, and each lane
// takes its own from there (41.7 M samples in 16.7 M records, 3.1 M voxels: 0.096 ms, 0.117 by the other way).
// Else each lane gathers its own records, eight at a time: through tiles the lanes of a crowded stretch
// wait for one another (0.8 M samples in 4,096 voxels: 45 us, 310 by tiles; fibers, 159,920 in 588: 0.38 ms,
// 2.9), and fibers' records, one a sample, are no faster by tiles (4.1 M in 1.8 M voxels: 36 us, 47).
constexpr int kReduceTile = 512;
constexpr int kReduceAtOnce = 8;
template <int KIND, class Key, bool PACKED>
__global__ void __launch_bounds__(kBlock) k_samp_reduce(Sorted<Key> sorted, const int64_t* __restrict__ start,
                                                        const float4* __restrict__ dirs,
                                                        const int64_t* __restrict__ ctl, vx_voxels out) {
  __shared__ float4 stage[KIND == 0 ? kWaves : 1][KIND == 0 ? kReduceTile : 1];
  __shared__ uint8_t counts[KIND == 0 ? kWaves : 1][KIND == 0 ? kReduceTile : 1];   // 1 to 64
  float4* st = stage[KIND == 0 ? threadIdx.x >> 6 : 0];
  uint8_t* sc = counts[KIND == 0 ? threadIdx.x >> 6 : 0];
  const int64_t nv = ctl[SC_VOX];
  const int64_t waves = int64_t(gridDim.x) * kWaves, wave = int64_t(blockIdx.x) * kWaves + (threadIdx.x >> 6);
  for (int64_t v0 = wave * 64; v0 < nv; v0 += waves * 64) {
    const int64_t v = v0 + lane_id(), vend = v0 + 64 < nv ? v0 + 64 : nv;
    const int64_t a = start[v < vend ? v : vend], b = start[v < vend ? v + 1 : vend];
    const int64_t first = start[v0], last = start[vend];
    Moment m{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    uint32_t samples = 0;
    if (KIND == 0 && last - first <= kReduceTile) {
      float4 d[kReduceTile / 64];
#pragma unroll
      for (int r = 0; r < kReduceTile / 64; ++r) {
        const int64_t j = first + r * 64 + lane_id();
        int c;
        d[r] = dirs[sorted.template id<PACKED>(j < last ? j : last - 1, c)];
        sc[r * 64 + lane_id()] = uint8_t(c);
      }
#pragma unroll
      for (int r = 0; r < kReduceTile / 64; ++r) st[r * 64 + lane_id()] = d[r];
      wave_lds_fence();
      for (int q = int(a - first); q < int(b - first); ++q) {
        const float4 t = st[q];
        const int c = sc[q];
        samples += uint32_t(c);
        for (int i = 0; i < c; ++i) accum_pair<KIND>(m, t.w, t);
      }
      wave_lds_fence();
    } else {
      for (int64_t j0 = a; j0 < b; j0 += kReduceAtOnce) {
        float4 d[kReduceAtOnce];
        int c[kReduceAtOnce];
#pragma unroll
        for (int r = 0; r < kReduceAtOnce; ++r)
          d[r] = dirs[sorted.template id<PACKED>(j0 + r < b ? j0 + r : b - 1, c[r])];
#pragma unroll
        for (int r = 0; r < kReduceAtOnce; ++r) {
          const int n = j0 + r < b ? (KIND == 0 ? c[r] : 1) : 0;
          samples += uint32_t(n);
          for (int i = 0; i < n; ++i) accum_pair<KIND>(m, d[r].w, d[r]);
        }
      }
    }
    if (v >= vend) continue;
    static_cast<Key*>(out.keys)[v] = sorted.key(a);
    out.count[v] = samples;
    out.w[v] = m.W;
    out.S[v] = m.xx;
    out.S[out.cap + v] = m.yy;
    out.S[2 * out.cap + v] = m.zz;
    out.S[3 * out.cap + v] = m.xy;
    out.S[4 * out.cap + v] = m.xz;
    out.S[5 * out.cap + v] = m.yz;
  }
}

int blocks_for(int64_t n) {
  const int64_t b = (n + kBlock - 1) / kBlock;
  return int(b < 1 ? 1 : (b > 4 * kGrid ? 4 * kGrid : b));
}

template <class Key>
void samp_back(int kind, const vx_grid* g, int64_t max_samples, const SampWs& w, const vx_voxels* out,
               int64_t* stats, hipStream_t s) {
  // Fibers: one bit above the voxels' keys holds the samples outside the grid.  Where the voxels' bits
  // fill the digits, that bit would cost a pass of its own (0.26 ms of 41.7 M samples): it runs only
  // when there are such samples, and its empty launches take 15 us.
  const int voxel_bits = 3 * g->log2_res;
  const bool own_pass = kind == 1 && voxel_bits % kRadixBits == 0;
  hipLaunchKernelGGL(k_samp_n, dim3(1), dim3(kBlock), 0, s, w.ctl, max_samples,
                     kind == 0 ? (const int32_t*)w.filled : nullptr, emit_blocks(max_samples) * kWaves);
  const int low = w.bits.packed ? w.bits.id + w.bits.cnt : 0;
  const PairBufs P = radix_sort_pairs(sizeof(Key) == 8, kind == 0 || own_pass ? voxel_bits : voxel_bits + 1, w.a, w.b, w.a,
                                      w.ctl + SC_SORT, max_samples, w.hist, w.partial, s, low,
                                      SortRegions{w.ctl + SC_TOTAL, kind == 0 ? w.filled : nullptr,
                                                  emit_blocks(max_samples) * kWaves});
  if (own_pass) {
    const PairBufs Q = P.keys == w.a.keys ? w.b : w.a;
    radix_sort_pass(sizeof(Key) == 8, P, Q, w.ctl + SC_SORT, max_samples, voxel_bits + low, w.hist,
                    w.partial, w.ctl + SC_OUTSIDE, s);
    hipLaunchKernelGGL(k_samp_back<Key>, dim3(blocks_for(max_samples)), dim3(kBlock), 0, s, (const Key*)Q.keys,
                       Q.prim, (Key*)P.keys, P.prim, w.ctl);
  }
  const Sorted<Key> sorted{(const Key*)P.keys, P.prim, w.bits};
  {
    VX_TIMED("sample_heads", s);
    const int blocks = head_blocks(max_samples);
    hipLaunchKernelGGL(k_samp_heads<Key>, dim3(blocks), dim3(kHeadBlock), 0, s, sorted, w.ctl, w.mask, w.partial);
    hipLaunchKernelGGL(k_samp_starts, dim3(blocks), dim3(kBlock), 0, s, w.mask, w.ctl, w.partial, w.start,
                       out->cap + 2);
    hipLaunchKernelGGL(k_samp_finish, dim3(1), dim3(64), 0, s, kind, w.ctl, stats, max_samples, out->cap);
  }
  VX_TIMED("sample_reduce", s);
  const auto reduce = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks_for(out->cap)), dim3(kBlock), 0, s, sorted, w.start, w.dirs, w.ctl, *out);
  };
  if constexpr (sizeof(Key) == 8) {
    if (w.bits.packed) return kind == 0 ? reduce(k_samp_reduce<0, Key, true>) : reduce(k_samp_reduce<1, Key, true>);
  }
  kind == 0 ? reduce(k_samp_reduce<0, Key, false>) : reduce(k_samp_reduce<1, Key, false>);
}

}  // namespace

size_t sample_ws_bytes(int kind, int64_t n_prims, int64_t max_samples, int64_t max_vox, int log2R, int sub) {
  return samp_ws_layout(kind, n_prims, max_samples, max_vox, log2R, sub, nullptr, nullptr);
}

vx_status sample_voxelize(int kind, const vx_grid* g, const float* data, int64_t n_prims, const int64_t* offsets,
                          int64_t n_fib, const vx_sampling* sp, int64_t max_samples, void* ws, const vx_voxels* out,
                          int64_t* stats, hipStream_t s) {
  const bool key64 = g->log2_res > 10;
  SampWs w;
  samp_ws_layout(kind, n_prims, max_samples, out->cap, g->log2_res, sp->chords_per_segment, ws, &w);
  Grid64 G;
  for (int a = 0; a < 3; ++a) G.bmin[a] = g->bmin[a];
  G.vs = ldexp(1.0, g->log2_res) / g->extent;
  G.R = int64_t(1) << g->log2_res;
  launch_fill_i64(w.ctl, 8, 0, s);
  launch_fill_i64(stats, VX_NSTAT, 0, s);
  launch_fill_i64(w.cnt + n_prims, 1, 0, s);      // the scan's last element: the total
  {
    VX_TIMED(kind == 0 ? "sample_tri_count" : "sample_fib_count", s);
    if (kind == 0) {
      hipLaunchKernelGGL(k_samp_tri_q, dim3(blocks_for(n_prims)), dim3(kBlock), 0, s, data, n_prims, G, w.q, w.ctl,
                         stats);
      hipLaunchKernelGGL(k_samp_tri_count, dim3(blocks_for(n_prims)), dim3(kBlock), 0, s, data, n_prims, G,
                         sp->max_triangle_samples, w.q, w.ctl, w.cnt, w.dirs);
    } else {
      hipLaunchKernelGGL(k_samp_offsets, dim3(blocks_for(n_fib + 1)), dim3(kBlock), 0, s, offsets, n_fib, n_prims,
                         stats);
      hipLaunchKernelGGL(k_samp_fib_count, dim3(blocks_for(n_prims)), dim3(kBlock), 0, s, data, n_prims, offsets,
                         n_fib, sp->chords_per_segment, sp->samples_per_chord, G, w.cnt, w.dirs, stats);
    }
    device_scan(CntIn{w.cnt}, CntOut{w.cnt}, SampTotal{w.ctl, stats, max_samples}, nullptr, n_prims + 1, w.partial,
                s);
  }
  {
    VX_TIMED(kind == 0 ? "sample_tri_emit" : "sample_fib_emit", s);
    const uint64_t out64 = uint64_t(1) << (3 * g->log2_res);
#define VX_SAMP_EMIT(K)                                                                                              \
  if (kind == 0)                                                                                                     \
    hipLaunchKernelGGL(k_samp_tri_emit<K>, dim3(emit_blocks(max_samples)), dim3(kBlock), 0, s, data, n_prims, G,     \
                       w.cnt, w.ctl, max_samples, K(out64), (SampOut<K>{(K*)w.a.keys, w.a.prim, w.bits}), w.filled);      \
  else                                                                                                               \
    hipLaunchKernelGGL(k_samp_fib_emit<K>, dim3(blocks_for(n_prims)), dim3(kBlock), 0, s, data, n_prims, offsets,   \
                       n_fib, sp->chords_per_segment, sp->samples_per_chord, G, w.cnt, w.ctl, max_samples, K(out64), \
                       (SampOut<K>{(K*)w.a.keys, w.a.prim, w.bits}))
    if (key64) { VX_SAMP_EMIT(uint64_t); } else { VX_SAMP_EMIT(uint32_t); }
#undef VX_SAMP_EMIT
  }
  if (key64)
    samp_back<uint64_t>(kind, g, max_samples, w, out, stats, s);
  else
    samp_back<uint32_t>(kind, g, max_samples, w, out, stats, s);
  return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
}

}  // namespace vx
