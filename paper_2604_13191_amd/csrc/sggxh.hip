// sggxh.hip -- the paper's SGGX-H lobe reduction (Sec. 4.4) on the GPU.
//
// A coarse voxel gathers the lobes of its children (the leaf's voxel is one lobe), drops those of
// zero weight and, when more than K remain, compares them through histograms of samples drawn
// from their normal distributions and merges the closest pair (pooling the samples) until K are
// left:
//   * lobe (w, S): the SGGX of S / w, its diagonal raised by 1e-3 of its trace; with S = L L^T
//     (Cholesky), a sample is n = L u / |L u| for u uniform on the sphere, accepted with
//     probability |L u| / sqrt(tr S) (the normals of the ellipsoid x^T S x = 1 weighted by area);
//     u from the cube [-1, 1]^3 by rejection, so only correctly rounded IEEE double operations
//     decide a sample's bin;
//   * random numbers: draw d of sample k of a lobe is SplitMix64 output number k 2^32 + d of the
//     lobe's seed, keyed by the level, the voxel's Morton key and the lobe's slot;
//   * histogram: 5 bins per axis, floor((n_a + 1) 2.5); only the three axis marginals are kept
//     (the distance uses nothing else);
//   * distance: Wasserstein-1 between the axis marginals, summed over the axes; for lobes pooling
//     m_i, m_j sample sets it is proportional to sum |C_i(b) m_j - C_j(b) m_i| / (m_i m_j) over
//     the cumulative counts C, compared exactly in 64-bit integers; ties to the first pair in
//     slot order;
//   * merge: w and S added (FP32), counts pooled; the survivors sorted by descending weight.
// One block of W waves per coarse voxel.  A wave samples one lobe at a time, dealing it to its
// lanes: a lane whose sample was accepted takes the next one, so that no lane waits for another's
// attempts.  The lobes of a voxel go to its waves in turn; then one wave merges, lane i holding
// row i of the pair distances.
//
// Sampling is bound by VALU issue: about four 64-bit hashes per attempt (six quarter-rate 32-bit
// multiplies each) and three attempts per sample.  An attempt is therefore decided in FP32 from the
// upper 32 bits of its draws, with margins several times the largest error (below); about one in
// 10^4 falls inside a margin and repeats the FP64 arithmetic, so every count is that of the FP64
// definition.  A lane keeps its counts in bytes of three registers.  Pyramid of a 257^2 piece of the
// brushed surface, K = 4, 5,000 samples per lobe: 47.1 -> 12.8 ms (FP64 attempts with a square root and three
// divisions, one wave per voxel: levels of 18 to 569 voxels took 3.6 to 3.9 ms each).
#pragma clang fp contract(off)

#include "vx_internal.hpp"

namespace vx {
namespace {

constexpr int kMaxLobes = 64;        // 8 children x K <= 8
constexpr int kMaxAttempts = 10000;
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t draw(uint64_t key, uint64_t k, uint64_t d) {
  return mix64(key + kGamma * (((k << 32) | d) + 1));
}
__device__ __forceinline__ double unit(uint64_t x) { return double(x >> 11) * 0x1p-53; }
__device__ __forceinline__ uint64_t lobe_key(int level, uint64_t voxel_key, int slot) {
  return mix64(mix64(voxel_key + kGamma * uint64_t(level + 1)) + kGamma * uint64_t(slot + 1));
}

struct Chol {
  double l00, l10, l11, l20, l21, l22, tr;
};

// lobe (w, S) with S = (xx, yy, zz, xy, xz, yz)
__device__ __forceinline__ Chol lobe_chol(float wf, float xx, float yy, float zz, float xy, float xz, float yz) {
  const double w = double(wf);
  double a00 = double(xx) / w, a11 = double(yy) / w, a22 = double(zz) / w;
  const double a10 = double(xy) / w, a20 = double(xz) / w, a21 = double(yz) / w;
  const double e = 1e-3 * ((a00 + a11) + a22);
  a00 = a00 + e;
  a11 = a11 + e;
  a22 = a22 + e;
  Chol c;
  c.tr = (a00 + a11) + a22;
  c.l00 = sqrt(a00);
  c.l10 = a10 / c.l00;
  c.l20 = a20 / c.l00;
  double d1 = a11 - c.l10 * c.l10;
  if (!(d1 > 0.0)) d1 = e;
  c.l11 = sqrt(d1);
  c.l21 = (a21 - c.l20 * c.l10) / c.l11;
  double d2 = (a22 - c.l20 * c.l20) - c.l21 * c.l21;
  if (!(d2 > 0.0)) d2 = e;
  c.l22 = sqrt(d2);
  return c;
}

__device__ __forceinline__ int bin_of(double n) {
  const double f = floor((n + 1.0) * 2.5);
  return !(f >= 0.0) ? 0 : (f > 4.0 ? 4 : int(f));
}

// attempt `at` of sample k of the lobe: true (and the three bins) when it is accepted
__device__ __forceinline__ bool lobe_attempt(const Chol& c, uint64_t key, uint64_t k, int at, int b[3]) {
  const uint64_t d = 4 * uint64_t(at);
  const double x = 2.0 * unit(draw(key, k, d)) - 1.0;
  const double y = 2.0 * unit(draw(key, k, d + 1)) - 1.0;
  const double z = 2.0 * unit(draw(key, k, d + 2)) - 1.0;
  const double r2 = (x * x + y * y) + z * z;
  if (r2 > 1.0 || r2 == 0.0) return false;
  const double p0 = c.l00 * x;
  const double p1 = c.l10 * x + c.l11 * y;
  const double p2 = (c.l20 * x + c.l21 * y) + c.l22 * z;
  const double q = (p0 * p0 + p1 * p1) + p2 * p2;
  const double U = unit(draw(key, k, d + 3));
  if (((U * U) * c.tr) * r2 > q) return false;
  const double len = sqrt(q);
  b[0] = bin_of(p0 / len);
  b[1] = bin_of(p1 / len);
  b[2] = bin_of(p2 / len);
  return true;
}

// Upper 32 bits of mix64(z).
__device__ __forceinline__ uint32_t mix64_hi(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  const uint32_t h = uint32_t(z >> 32);
  return h ^ (h >> 31);
}

// The attempt in FP32.  L is divided by sqrt(tr), so its rows are at most 1 long (else the lobe takes
// the FP64 path throughout).  Coordinates from the upper 32 bits are off by at most 2^-24.9, r2 by
// 2^-21.7, a component of p = L u by 2^-21.9 (the vector by 2^-21.1), q = |p|^2 by 2^-19.9 and
// U^2 r2 by 2^-21.2; n_a = p_a / |p| by 2^-20.4 / |p| + 2^-21.5, and (n_a + 1) 2.5 by
// 2^-19.1 / |p| + 2^-20.2.  The margins leave a factor of at least four.
constexpr float kMarginR2 = 0x1p-19f, kMarginQ = 0x1p-17f, kMarginBin = 0x1p-17f;

struct CholF {
  float l00, l10, l11, l20, l21, l22;
};

// 1: accepted (with its bins), 0: rejected, -1: inside a margin
__device__ __forceinline__ int fast_attempt(const CholF& c, uint64_t z, int b[3]) {
  const float x = float(int32_t(mix64_hi(z) ^ 0x80000000u)) * 0x1p-31f;
  const float y = float(int32_t(mix64_hi(z + kGamma) ^ 0x80000000u)) * 0x1p-31f;
  const float w = float(int32_t(mix64_hi(z + 2 * kGamma) ^ 0x80000000u)) * 0x1p-31f;
  const float U = float(mix64_hi(z + 3 * kGamma)) * 0x1p-32f;
  const float r2 = fmaf(w, w, fmaf(y, y, x * x));
  const float p0 = c.l00 * x;
  const float p1 = fmaf(c.l11, y, c.l10 * x);
  const float p2 = fmaf(c.l22, w, fmaf(c.l21, y, c.l20 * x));
  const float q = fmaf(p2, p2, fmaf(p1, p1, p0 * p0));
  const float over = fmaf(U * U, r2, -q);
  const float rs = __builtin_amdgcn_rsqf(q);
  float f[3], edge = 0.f;
  const float p[3] = {p0, p1, p2};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    // the outer halves of the end bins hold no boundary
    f[a] = __builtin_amdgcn_fmed3f(fmaf(p[a] * rs, 2.5f, 2.5f), 0.5f, 4.5f);
    edge = fmaxf(edge, fabsf(__builtin_amdgcn_fractf(f[a]) - 0.5f));
    b[a] = int(f[a]);
  }
  // every decision is a comparison that holds: a NaN decides nothing
  const bool out = r2 > 1.0f + kMarginR2 || over > kMarginQ;
  const bool in = r2 < 1.0f - kMarginR2 && over < -kMarginQ && edge < fmaf(rs, -kMarginBin, 0.5f - kMarginBin);
  return in ? 1 : (out ? 0 : -1);
}

// the FP64 attempt, out of line: taken by about one attempt in 10^4
__device__ __attribute__((noinline)) int exact_attempt(const Chol* c, uint64_t key, uint64_t k, int at) {
  int b[3];
  if (!lobe_attempt(*c, key, k, at, b)) return -1;
  return b[0] | (b[1] << 4) | (b[2] << 8);
}

// counts of the lobe's N samples in bins 0 to 3 of each axis (bin 4 follows), added to cnt[12]
__device__ __forceinline__ void sample_lobe(const Chol& c, const Chol* c_lds, uint64_t key, int N, int32_t* cnt) {
  const int lane = lane_id();
  CholF f;
  {
    const double is = 1.0 / sqrt(c.tr);
    f.l00 = float(c.l00 * is);
    f.l10 = float(c.l10 * is);
    f.l11 = float(c.l11 * is);
    f.l20 = float(c.l20 * is);
    f.l21 = float(c.l21 * is);
    f.l22 = float(c.l22 * is);
    const float n1 = fmaf(f.l10, f.l10, f.l11 * f.l11);
    const float n2 = fmaf(f.l20, f.l20, fmaf(f.l21, f.l21, f.l22 * f.l22));
    if (!(f.l00 * f.l00 <= 1.0f && n1 <= 1.0f && n2 <= 1.0f)) f.l00 = __builtin_nanf("");
  }
  auto first = [&](int k) {                        // draw 0 of sample k is mix64 of this
    return key + kGamma + (uint64_t(uint32_t(kGamma) * uint32_t(k)) << 32);
  };
  uint32_t acc[3] = {0, 0, 0};
  int k = lane, at = 0, next = 64, rounds = 0;
  uint64_t z = first(k);
  auto flush = [&]() {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int v = int((acc[a] >> (8 * b)) & 255u);
        if (v) atomicAdd(&cnt[4 * a + b], v);
      }
      acc[a] = 0;
    }
    rounds = 0;
  };
  while (__ballot(k < N)) {
    int b[3];
    int res = fast_attempt(f, z, b);
    if (k >= N) res = 0;
    if (__ballot(res < 0)) {
      if (res < 0) {
        const int e = exact_attempt(c_lds, key, uint64_t(k), at);
        res = e >= 0 ? 1 : 0;
        b[0] = e & 15;
        b[1] = (e >> 4) & 15;
        b[2] = (e >> 8) & 15;
      }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) acc[a] += res == 1 && b[a] < 4 ? 1u << (8 * b[a]) : 0u;
    const bool take = k < N && (res == 1 || at + 1 >= kMaxAttempts);
    const uint64_t m = __ballot(take);
    const int before = int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0)));
    k = take ? next + before : k;
    at = take ? 0 : at + 1;
    z = take ? first(k) : z + 4 * kGamma;
    next += __popcll(m);
    if (++rounds == 255) flush();                  // a byte holds 255
  }
  flush();
}

// Child lobes come from a vx_lobes level (lob != nullptr) or from the leaf (one lobe per voxel).
// W waves per voxel, at most ML lobes.
template <class Key, int W, int ML>
__global__ void __launch_bounds__(64 * W) k_sggxh_level(const Key* __restrict__ ckeys,
                                                        const int64_t* __restrict__ n_child, int64_t cmax,
                                                        const float* __restrict__ leaf_w,
                                                        const float* __restrict__ leaf_S, int64_t leaf_cap,
                                                        vx_lobes clob, int Kc, const Key* __restrict__ pkeys,
                                                        const int64_t* __restrict__ n_par, int64_t pmax, vx_lobes plob,
                                                        int K, int level, int N, int64_t* stats) {
  static_assert(ML <= kMaxLobes, "lobes fit one wave");
  __shared__ float sw[ML];
  __shared__ float sS[6][ML];
  __shared__ __attribute__((aligned(16))) int32_t cum[ML][12];   // bins 0..3 per axis: counts, then cumulative
  __shared__ int32_t mass[ML];               // sample sets pooled
  __shared__ double dist[ML][ML + 1];
  __shared__ Chol chol[W];
  __shared__ int32_t s_n, s_next;
  const int64_t nparents = *n_par, nc = *n_child;
  if (nparents > pmax || nc > cmax) {
    if (blockIdx.x == 0 && threadIdx.x == 0)
      atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_VOXEL_CAPACITY);
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  for (int64_t p = blockIdx.x; p < nparents; p += gridDim.x) {
    const Key pk = pkeys[p];
    if (wave == 0) {
      // children: key >> 3 == pk, contiguous from the first key >= pk << 3
      int64_t lo = 0, hi = nc;
      const Key first = Key(pk << 3);
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ckeys[mid] < first) lo = mid + 1; else hi = mid;
      }
      // gather the positive lobes, child-major then lobe order: lane = child * Kc + lobe
      bool have = false;
      float lw = 0.0f;
      float lS[6] = {0, 0, 0, 0, 0, 0};
      const int ci = lane / Kc, k = lane % Kc;
      const int64_t c = lo + ci;
      if (ci < 8 && c < nc && Key(ckeys[c] >> 3) == pk) {
        if (clob.nl == nullptr) {
          if (k == 0) {
            lw = leaf_w[c];
#pragma unroll
            for (int t = 0; t < 6; ++t) lS[t] = leaf_S[t * leaf_cap + c];
            have = lw > 0.0f;
          }
        } else if (k < int(clob.nl[c])) {
          lw = clob.w[int64_t(k) * clob.cap + c];
#pragma unroll
          for (int t = 0; t < 6; ++t) lS[t] = clob.S[(int64_t(t) * Kc + k) * clob.cap + c];
          have = lw > 0.0f;
        }
      }
      const uint64_t hv = __ballot(have);
      const int slot = __popcll(hv & lt);
      if (have) {
        sw[slot] = lw;
#pragma unroll
        for (int t = 0; t < 6; ++t) sS[t][slot] = lS[t];
      }
      if (lane == 0) {
        s_n = __popcll(hv);
        s_next = 0;
      }
      for (int i = lane; i < ML * 12; i += 64) (&cum[0][0])[i] = 0;
    }
    __syncthreads();
    const int n = s_n;
    if (n > K) {
      while (true) {
        int j = 0;
        if (lane == 0) j = atomicAdd(&s_next, 1);
        j = __builtin_amdgcn_readfirstlane(j);
        if (j >= n) break;
        const Chol c = lobe_chol(sw[j], sS[0][j], sS[1][j], sS[2][j], sS[3][j], sS[4][j], sS[5][j]);
        if (lane == 0) chol[wave] = c;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        sample_lobe(c, &chol[wave], lobe_key(level, uint64_t(pk), j), N, cum[j]);
      }
      __syncthreads();
    }
    if (wave == 0) {
      bool on = lane < n;
      if (n > K) {
        if (on) {
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            int32_t run = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              run += cum[lane][4 * a + b];
              cum[lane][4 * a + b] = run;
            }
          }
          mass[lane] = 1;
        }
        auto fence = [] {
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        };
        fence();
        // sum |C_i m_j - C_j m_i| / (m_i m_j): C below 2^22, m at most 64, the sum below 2^30.
        // Two different quotients differ by 2^-20 at least on values below 2^20, far more than an
        // FP64 rounding, and equal ones round alike: the quotients order like the fractions.
        auto pair = [&](int i, int j) {
          const int mi = mass[i], mj = mass[j];
          int num = 0;
#pragma unroll
          for (int t = 0; t < 12; ++t) {
            const int d = __mul24(cum[i][t], mj) - __mul24(cum[j][t], mi);
            num += d < 0 ? -d : d;
          }
          return double(num) / double(mi * mj);
        };
        if (on) {
          for (int j = 0; j < n; ++j) dist[lane][j] = INFINITY;
        }
        fence();
        if (on) {
          for (int d = 1; 2 * d <= n; ++d) {
            const int j = lane + d < n ? lane + d : lane + d - n;
            const double v = pair(lane, j);
            dist[lane][j] = v;
            dist[j][lane] = v;
          }
        }
        fence();
        // the closest pair, ties to the first in (i, j) order: i is the first lane whose row holds
        // the least distance, j the first column of that row (the matrix is symmetric)
        for (int active = n; active > K; --active) {
          double best = INFINITY;
          if (on)
            for (int j = 0; j < n; ++j) best = fmin(best, dist[lane][j]);
          double least = best;
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) least = fmin(least, __shfl_xor(least, o, 64));
          const int i = __ffsll((unsigned long long)__ballot(on && best == least)) - 1;
          const int j = __ffsll((unsigned long long)__ballot(lane < n && dist[i][lane < n ? lane : 0] == least)) - 1;
          if (lane < 12) cum[i][lane] += cum[j][lane];
          else if (lane < 18) sS[lane - 12][i] = sS[lane - 12][i] + sS[lane - 12][j];
          else if (lane == 18) sw[i] = sw[i] + sw[j];
          else if (lane == 19) mass[i] += mass[j];
          fence();
          if (lane == j) on = false;
          if (lane == i) {
            dist[i][j] = INFINITY;
          } else if (on) {
            const double v = pair(lane, i);
            dist[lane][i] = v;
            dist[i][lane] = v;
            dist[lane][j] = INFINITY;
          }
          fence();
        }
      }
      // survivors by descending weight (ties in slot order)
      const int m = n > K ? K : n;
      const uint64_t left = __ballot(on);
      if (on) {
        const float w = sw[lane];
        int rank = 0;
        for (int t = 0; t < n; ++t)
          if (((left >> t) & 1) && (sw[t] > w || (sw[t] == w && t < lane))) ++rank;
        plob.w[int64_t(rank) * plob.cap + p] = w;
#pragma unroll
        for (int t = 0; t < 6; ++t) plob.S[(int64_t(t) * K + rank) * plob.cap + p] = sS[t][lane];
      }
      if (lane >= m && lane < K) {
        plob.w[int64_t(lane) * plob.cap + p] = 0.0f;
#pragma unroll
        for (int t = 0; t < 6; ++t) plob.S[(int64_t(t) * K + lane) * plob.cap + p] = 0.0f;
      }
      if (lane == 0) plob.nl[p] = uint8_t(m);
    }
    __syncthreads();
  }
}

}  // namespace

vx_status sggxh_run(const vx_grid* g, const vx_voxels* leaf, const vx_voxels* out, const int64_t* n_levels,
                    int levels, int K, int N, const vx_lobes* lobes, int64_t* stats, hipStream_t s) {
  const bool key64 = g->log2_res > 10;
  launch_fill_i64(stats, VX_NSTAT, 0, s);
  for (int l = 1; l < levels; ++l) {
    const vx_voxels& C = l == 1 ? *leaf : out[l - 2];
    const vx_voxels& P = out[l - 1];
    const vx_lobes clob = l == 1 ? vx_lobes{nullptr, nullptr, nullptr, 0} : lobes[l - 2];
    const int Kc = l == 1 ? 1 : K;
    const int64_t cmax = l == 1 ? C.cap : (C.cap < clob.cap ? C.cap : clob.cap);
    const int64_t pmax = P.cap < lobes[l - 1].cap ? P.cap : lobes[l - 1].cap;
    const int grid = int(pmax < 16384 ? (pmax < 1 ? 1 : pmax) : 16384);
    VX_TIMED("sggxh_level", s);
    // Waves per voxel: a lobe takes one wave about 0.1 ms at 5,000 samples, so four a voxel fill the
    // chip (1,024 SIMDs) from about a thousand voxels on; on smaller levels the voxels' own lobes are
    // all there is to spread, and sixteen waves take up to 32 of them in two turns.
    const bool wide = pmax < 1024;
#define VX_SH(Ky, W, ML)                                                                                          \
  hipLaunchKernelGGL((k_sggxh_level<Ky, W, ML>), dim3(grid), dim3(64 * W), 0, s, (const Ky*)C.keys, n_levels + l - 1, \
                     cmax, leaf->w, leaf->S, leaf->cap, clob, Kc, (const Ky*)P.keys, n_levels + l, pmax,          \
                     lobes[l - 1], K, l, N, stats)
#define VX_SH_W(Ky, ML)                                            \
  do {                                                            \
    if (wide) VX_SH(Ky, 16, ML); else VX_SH(Ky, 4, ML);           \
  } while (0)
    if (Kc <= 4) {
      if (key64) VX_SH_W(uint64_t, 32); else VX_SH_W(uint32_t, 32);
    } else {
      if (key64) VX_SH_W(uint64_t, 64); else VX_SH_W(uint32_t, 64);
    }
#undef VX_SH_W
#undef VX_SH
  }
  return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
}

}  // namespace vx
