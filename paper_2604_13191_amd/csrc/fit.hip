// fit.hip -- differentiable two-lobe fit over the pyramid, forward and hand-written backward.
//
// For every voxel u of levels lo..hi with w_u > 0, two lobes given by lower-triangular L_1, L_2
// (6 parameters each: L00 L10 L11 L20 L21 L22) have projected area
// f_u(omega) = |L_1^T omega| + |L_2^T omega|; the target is the density-weighted projected area
// of u's children, tau_u(omega) = sum_c sqrt(w_c omega^T S_c omega) / sum_c w_c (Sec. 4.1 gives
// sigma(omega) = sqrt(omega^T S omega) for an SGGX S = S_c / w_c).  The loss is the sum over
// voxels of the mean over the direction set of (f_u - tau_u)^2.
//
// Backward: d loss / d L per voxel; d loss / d (S_c, w_c) per child, accumulated top-down so
// that every leaf voxel holds the gradient of all its ancestors' sums; then, per fiber segment,
// through the clipped lengths (weights) and the tangent (moment I - t t^T) to the control
// points.  Intermediates are recomputed instead of stored: the per-direction profiles are
// re-evaluated in the backward kernel, and the (segment, voxel) pairs are re-emitted in
// primitive order by the voxelize front half.
#include <type_traits>

#include "geom.hpp"
#include "vx_internal.hpp"

namespace vx {

template <class Key>
__device__ __forceinline__ int64_t key_lower_bound(const Key* __restrict__ keys, int64_t n, uint64_t k) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (uint64_t(keys[mid]) < k) lo = mid + 1; else hi = mid;
  }
  return lo;
}

constexpr int kMaxChild = 8;

// ---------------------------------------------------------------------------------------------
// Layout of both passes: one wave per voxel, the voxels of all fitted levels in one launch (sixteen
// lanes per voxel ran as long as the largest of a wave's four, and the upper levels' launches stood
// nearly empty).  Each lane keeps ndir / 64 directions as their products
// x^2 .. 2yz, so that w^T S w is six fused multiply-adds; a child's sums are the same for all lanes
// and come from LDS.
// ---------------------------------------------------------------------------------------------
constexpr int kMaxFit = 20;
constexpr int kFitGrid = 2 * kGrid;
struct FitLevel {
  const int64_t* n;        // voxels
  int64_t rows;            // parameter rows: voxels past them are not fitted
  const float* w;
  const int64_t* cstart;   // children of voxel u in the level below: [cstart[u], cstart[u + 1]), at most 8
  const float* Lp;
  const float* chw;        // forward: the children's sums, and the loss per voxel
  const float* chS;
  int64_t chcap;
  float* loss;
  const double* c64;       // backward: the children's FP64 sums [7][gcap] (S, then w), their gradients
  double* gch;             // [7][gcap] likewise, and the parameters'
  int64_t gcap;
  float* dLp;
};
struct FitLevels {
  FitLevel l[kMaxFit];
  int count;
};

// the i-th voxel of all levels: its level, and i reduced to its index there; false past the last
__device__ __forceinline__ bool fit_level(const FitLevels& lv, int64_t& i, int& L) {
  for (L = 0; L < lv.count; ++L) {
    const int64_t n = *lv.l[L].n;
    if (i < n) return true;
    i -= n;
  }
  return false;
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// the products of direction k (zeros past the set: its terms vanish)
template <class T>
__device__ __forceinline__ void dir_products(const float* __restrict__ dirs, int ndir, int k, T x[3], T m[6]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] = k < ndir ? T(dirs[3 * k + a]) : T(0);
  m[0] = x[0] * x[0];
  m[1] = x[1] * x[1];
  m[2] = x[2] * x[2];
  m[3] = T(2) * x[0] * x[1];
  m[4] = T(2) * x[0] * x[2];
  m[5] = T(2) * x[1] * x[2];
}
template <class T>
__device__ __forceinline__ T quad(const T* S, const T m[6]) {
  T q = S[0] * m[0];
#pragma unroll
  for (int t = 1; t < 6; ++t) q = fma(S[t], m[t], q);
  return q;
}

// ---------------------------------------------------------------------------------------------
// forward.  Bound by FP32 arithmetic (0.69 M voxels, 2.7 M children, 128 directions: 0.25 ms;
// with sixteen lanes per voxel, the sums read from LDS for every direction, 0.58 ms).
// ---------------------------------------------------------------------------------------------
// sqrt(x): the reciprocal root's estimate, refined on the residual x - s^2; zeros, numbers so small
// that the residual underflows, infinities and NaN take the library's function (whatever lies outside
// [2^-96, inf), by one comparison of the bits)
__device__ __forceinline__ float sqrt_nrf(float x) {
  constexpr uint32_t least = 0x0f800000u, inf = 0x7f800000u;
  if (__builtin_amdgcn_ballot_w64(__float_as_uint(x) - least >= inf - least)) return sqrtf(x);
  const float r = __builtin_amdgcn_rsqf(x), s = x * r;
  return fmaf(fmaf(-s, s, x), 0.5f * r, s);
}

template <int DPL>
__global__ void __launch_bounds__(kBlock) k_fit_fwd(FitLevels lv, const float* __restrict__ dirs, int ndir) {
  __shared__ float stage[kWaves][kMaxChild][8];      // per child: S, then w
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float x[DPL][3], m[DPL][6];
#pragma unroll
  for (int i = 0; i < DPL; ++i) {
    // past the set the last direction again, its residual dropped: zeros there would send every root of
    // the wave to the library's function (0.69 M voxels, 100 directions: 0.267 -> 0.255 ms)
    const int k = lane + 64 * i;
    dir_products(dirs, ndir, k < ndir ? k : ndir - 1, x[i], m[i]);
  }
  const float rdir = float(ndir);
  for (int64_t i0 = int64_t(blockIdx.x) * kWaves + wv;; i0 += int64_t(gridDim.x) * kWaves) {
    int64_t u = i0;
    int L;
    if (!fit_level(lv, u, L)) return;
    const FitLevel& F = lv.l[L];
    if (u >= F.rows) continue;                       // never past the parameter rows
    const float W = F.w[u];
    if (!(W > 0.f)) {
      if (lane == 0) F.loss[u] = 0.f;
      continue;
    }
    const int64_t first = F.cstart[u], nch = F.cstart[u + 1] - first;
    const int nc = int(nch < kMaxChild ? nch : kMaxChild);
    const int lt = lane >> 3, lc = lane & 7;
    if (lc < nc && lt < 7) stage[wv][lc][lt] = lt < 6 ? F.chS[int64_t(lt) * F.chcap + first + lc] : F.chw[first + lc];
    wave_sync_lds();
    float tau[DPL];
#pragma unroll
    for (int i = 0; i < DPL; ++i) tau[i] = 0.f;
    for (int c = 0; c < nc; ++c) {
      float S[6];
#pragma unroll
      for (int t = 0; t < 6; ++t) S[t] = stage[wv][c][t];
      const float wc = stage[wv][c][6];
      if (!(wc > 0.f)) continue;
#pragma unroll
      for (int i = 0; i < DPL; ++i) tau[i] += sqrt_nrf(fmaxf(wc * quad(S, m[i]), 0.f));
    }
    float l[12], acc = 0.f;
#pragma unroll
    for (int t = 0; t < 12; ++t) l[t] = F.Lp[u * 12 + t];
    const float invW = 1.0f / W;
#pragma unroll
    for (int i = 0; i < DPL; ++i) {
      float f = 0.f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float* lj = l + 6 * j;
        const float y0 = lj[0] * x[i][0] + lj[1] * x[i][1] + lj[3] * x[i][2];
        const float y1 = lj[2] * x[i][1] + lj[4] * x[i][2], y2 = lj[5] * x[i][2];
        f += sqrt_nrf(y0 * y0 + y1 * y1 + y2 * y2);
      }
      const float r = lane + 64 * i < ndir ? f - tau[i] * invW : 0.f;
      acc = fmaf(r, r, acc);
    }
    acc = wave_sum(acc);
    if (lane == 0) F.loss[u] = acc / rdir;
    wave_sync_lds();                                  // the wave's LDS slots are reused next
  }
}

// deterministic sum, in FP64, of the per-voxel losses of all levels into loss[0]: fixed per-block
// chunks of every level, then one block adds the block sums in order
struct LossLevels {
  const float* p[24];
  const int64_t* n[24];
  int64_t rows[24];       // the forward wrote at most this many per-voxel losses
  int count;
};

__global__ void __launch_bounds__(kBlock) k_fit_partial(LossLevels lv, double* __restrict__ part) {
  __shared__ double red[kWaves];
  double acc = 0.0;
  for (int i = 0; i < lv.count; ++i) {
    const int64_t n = *lv.n[i] < lv.rows[i] ? *lv.n[i] : lv.rows[i];
    const int64_t chunk = (n + kGrid - 1) / kGrid;
    const int64_t b0 = int64_t(blockIdx.x) * chunk, b1 = b0 + chunk < n ? b0 + chunk : n;
    for (int64_t j = b0 + threadIdx.x; j < b1; j += kBlock) acc += double(lv.p[i][j]);
  }
  acc = wave_sum(acc);
  if (lane_id() == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += red[w];
    part[blockIdx.x] = t;
  }
}

__global__ void __launch_bounds__(1024) k_fit_total(const double* __restrict__ part, float* loss) {
  __shared__ double red[16];
  double acc = threadIdx.x < kGrid ? part[threadIdx.x] : 0.0;
  acc = wave_sum(acc);
  if (lane_id() == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < 16; ++w) t += red[w];
    loss[0] = float(t);
  }
}

// ---------------------------------------------------------------------------------------------
// backward per voxel: lobe gradients and the gradient of the target w.r.t. the children's sums.
// FP64: the derivative of the target along a child's own (w, S) direction nearly cancels (the
// target is invariant when all children scale alike), so the parts must be accurate.  Bound by
// FP64 arithmetic (the workload of the forward: 0.97 ms; with sixteen lanes per voxel, whose children
// were evaluated again for their gradients and summed over the lanes by LDS permutes, 2.46 ms).
// ---------------------------------------------------------------------------------------------
// 1 / sqrt(x), x > 0: the hardware estimate (good to 2^-24 as measured) refined by one Newton step,
// r' = r (3/2 - x r^2 / 2), which squares its relative error: good to 2^-47
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x * r;
  return fma(r, fma(-h, r, 0.5), r);
}

// cross-lane moves of a double: a DPP pattern; v_permlane{16,32}_swap of a and b, added
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppRor8 = 0x128;
__device__ __forceinline__ double swap_add32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double swap_add16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// sum over eight lanes / a row of sixteen, in every lane of them
__device__ __forceinline__ double sum8(double v) {
  v += dpp64<kDppXor1>(v);
  v += dpp64<kDppXor2>(v);
  return v + dpp64<kDppHalfMirror>(v);
}
__device__ __forceinline__ double sum16(double v) { return sum8(v + dpp64<kDppRor8>(v)); }
// sums of eight values over the wave: lane l gets that of value 4 * bit 5 + 2 * bit 4 + bit 3 of l.
// Each step halves the values a lane still carries, where a butterfly per value would add all.
__device__ __forceinline__ double wave_sum8(const double v[8], int lane) {
  double a[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = swap_add32(v[i], v[i + 4]);
  const double b0 = swap_add16(a[0], a[2]), b1 = swap_add16(a[1], a[3]);
  const bool up = lane & 8;
  const double mine = up ? b1 : b0, other = up ? b0 : b1;
  return sum8(mine + dpp64<kDppRor8>(other));
}
// sums of four values: lane l gets that of value 2 * bit 5 + bit 4 of l
__device__ __forceinline__ double wave_sum4(const double v[4]) {
  return sum16(swap_add16(swap_add32(v[0], v[2]), swap_add32(v[1], v[3])));
}

template <int DPL>
__global__ void __launch_bounds__(kBlock, DPL <= 2 ? 3 : 1) k_fit_bwd(FitLevels lv, const float* __restrict__ dirs, int ndir,
                                                    const float* __restrict__ dloss) {
  // per child: S and w; later sqrt(w) and 1 / (2 sqrt(w)) in the last two, the gradients in the first seven
  __shared__ double stage[kWaves][kMaxChild][8];
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double(*st)[8] = stage[wv];
  double x[DPL][3], m[DPL][6];
#pragma unroll
  for (int i = 0; i < DPL; ++i) dir_products(dirs, ndir, lane + 64 * i, x[i], m[i]);
  const double g2 = 2.0 / double(ndir) * double(dloss[0]);
  const int lt = lane >> 3, lc = lane & 7;
  for (int64_t i0 = int64_t(blockIdx.x) * kWaves + wv;; i0 += int64_t(gridDim.x) * kWaves) {
    int64_t u = i0;
    int L;
    if (!fit_level(lv, u, L)) return;
    const FitLevel& F = lv.l[L];
    const bool fitted = u < F.rows;
    const bool active = fitted && F.w[u] > 0.f && F.c64 != nullptr;   // no FP64 sums: no points, nothing to fit
    const int64_t first = F.cstart[u], nch = F.cstart[u + 1] - first;
    const int nc = int(nch < kMaxChild ? nch : kMaxChild);
    if (!active) {
      if (fitted && lane < 12) F.dLp[u * 12 + lane] = 0.f;
      if (lc < nc && lt < 7) F.gch[int64_t(lt) * F.gcap + first + lc] = 0.0;
      continue;
    }
    // lane 8 t + c: component t of child c (w in the last two rows, as its root and half its reciprocal)
    double wc = 0.0;
    if (lc < nc) {
      const double v = F.c64[int64_t(lt < 6 ? lt : 6) * F.gcap + first + lc];
      wc = v;
      const double r = v > 0.0 ? rsqrt_nr(v) : 0.0;
      st[lc][lt] = lt < 6 ? v : lt == 6 ? v * r : 0.5 * r;
    }
    // the parent's weight as the FP64 sum of its children's
    const double Ws = sum8(wc);
    const double Wd = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(Ws), 48),
                                       __builtin_amdgcn_readlane(__double2loint(Ws), 48));
    const double invW = Wd > 0.0 ? 1.0 / Wd : 0.0;
    wave_sync_lds();
    // pass 1: the target, with every child's root s and 1 / s kept
    double s[kMaxChild][DPL], r[kMaxChild][DPL], tau[DPL], g[DPL];
#pragma unroll
    for (int i = 0; i < DPL; ++i) tau[i] = 0.0;
#pragma unroll
    for (int c = 0; c < kMaxChild; ++c) {
      if (c >= nc) continue;
      double S[6];
#pragma unroll
      for (int t = 0; t < 6; ++t) S[t] = st[c][t];
      const double sw = st[c][6];
#pragma unroll
      for (int i = 0; i < DPL; ++i) {
        const double q = quad(S, m[i]);
        r[c][i] = q > 0.0 ? rsqrt_nr(q) : 0.0;
        s[c][i] = q * r[c][i];
        tau[i] = fma(sw, s[c][i], tau[i]);
      }
    }
    // fit, residual and lobe gradients
    double gl[12];
#pragma unroll
    for (int t = 0; t < 12; ++t) gl[t] = 0.0;
#pragma unroll
    for (int i = 0; i < DPL; ++i) {
      tau[i] *= invW;
      double f = 0.0, y[2][3], ry[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float* lj = F.Lp + u * 12 + 6 * j;
        y[j][0] = double(lj[0]) * x[i][0] + double(lj[1]) * x[i][1] + double(lj[3]) * x[i][2];
        y[j][1] = double(lj[2]) * x[i][1] + double(lj[4]) * x[i][2];
        y[j][2] = double(lj[5]) * x[i][2];
        const double n2 = y[j][0] * y[j][0] + y[j][1] * y[j][1] + y[j][2] * y[j][2];
        ry[j] = n2 > 0.0 ? rsqrt_nr(n2) : 0.0;                 // 1 / |L_j^T w|
        f += n2 * ry[j];
      }
      g[i] = (f - tau[i]) * g2;                                 // d loss / d f;  d loss / d tau = -g
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const double sj = g[i] * ry[j];
        const double a0 = sj * y[j][0], a1 = sj * y[j][1], a2 = sj * y[j][2];
        double* gj = gl + 6 * j;
        gj[0] = fma(a0, x[i][0], gj[0]);
        gj[1] = fma(a0, x[i][1], gj[1]);
        gj[2] = fma(a1, x[i][1], gj[2]);
        gj[3] = fma(a0, x[i][2], gj[3]);
        gj[4] = fma(a1, x[i][2], gj[4]);
        gj[5] = fma(a2, x[i][2], gj[5]);
      }
    }
    {
      const double v8 = wave_sum8(gl, lane), v4 = wave_sum4(gl + 8);
      if (lc == 0) F.dLp[u * 12 + lt] = float(v8);
      if ((lane & 15) == 0) F.dLp[u * 12 + 8 + (lane >> 4)] = float(v4);
    }
    // pass 2: d loss / d (S_c, w_c).  d tau / d (w^T S_c w) = sqrt(w_c) / (2 s) / W and
    // d tau / d w_c = (s / (2 sqrt(w_c)) - tau) / W
#pragma unroll
    for (int c = 0; c < kMaxChild; ++c) {
      if (c >= nc) continue;
      const double sw = st[c][6], hs = st[c][7];
      double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < DPL; ++i) {
        const double gr = g[i] * r[c][i];
#pragma unroll
        for (int t = 0; t < 6; ++t) acc[t] = fma(gr, m[i][t], acc[t]);
        acc[6] = fma(g[i], fma(hs, s[c][i], -tau[i]), acc[6]);
      }
      const double v = wave_sum8(acc, lane) * -invW * (lt < 6 ? 0.5 * sw : sw > 0.0 ? 1.0 : 0.0);
      wave_sync_lds();
      if (lc == 0) st[c][lt] = v;                               // (the eighth is not read)
    }
    wave_sync_lds();
    if (lc < nc && lt < 7) F.gch[int64_t(lt) * F.gcap + first + lc] = st[lc][lt];
    wave_sync_lds();                                  // the wave's LDS slots are reused next
  }
}

// the leaf's gradients: its own and those of all its ancestors, added from the top down (levels
// below the first fitted one hold none).  One pass over the leaf instead of one per level.
struct FitDown {
  const int32_t* pidx[kMaxFit];    // index of every voxel's parent
  double* g[kMaxFit];              // [7][gcap]
  int64_t gcap[kMaxFit];
  uint32_t last[kMaxFit];          // gcap - 1 (indexes are 32-bit)
  int lo, hi;                      // levels lo .. hi - 1 hold gradients
};
__global__ void __launch_bounds__(kBlock) k_fit_down(FitDown d, const int64_t* n_p) {
  const int64_t n = *n_p;
  for (int64_t c = int64_t(blockIdx.x) * kBlock + threadIdx.x; c < n; c += int64_t(gridDim.x) * kBlock) {
    // A level over its capacity (flagged: the gradients are invalid) leaves children without a parent and
    // their index unset: held inside the buffers, whatever it is
    int32_t at[kMaxFit];
    at[0] = int32_t(c);
#pragma unroll
    for (int L = 1; L < kMaxFit; ++L)
      if (L < d.hi) at[L] = int32_t(min(uint32_t(d.pidx[L - 1][at[L - 1]]), d.last[L]));
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int L = kMaxFit - 1; L >= 0; --L)
      if (L < d.hi && L >= d.lo)
#pragma unroll
        for (int t = 0; t < 7; ++t) acc[t] = d.g[L][int64_t(t) * d.gcap[L] + at[L]] + acc[t];
#pragma unroll
    for (int t = 0; t < 7; ++t) d.g[0][int64_t(t) * d.gcap[0] + c] = acc[t];
  }
}

// leaf lookup table: first and end leaf index of every 16^3 tile (empty tiles: 0, 0).  A leaf over its
// capacity (flagged) was not written, so its keys may be anything: those past the grid are left out.
template <class Key>
__global__ void __launch_bounds__(kBlock) k_tile_index(const Key* __restrict__ keys, const int64_t* n_p,
                                                       int64_t tiles, int64_t* __restrict__ tfirst,
                                                       int64_t* __restrict__ tend) {
  const int64_t n = *n_p;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const uint64_t t = uint64_t(keys[i]) >> (3 * kTileBits);
    if (t >= uint64_t(tiles)) continue;
    if (i == 0 || (uint64_t(keys[i - 1]) >> (3 * kTileBits)) != t) tfirst[t] = i;
    if (i == n - 1 || (uint64_t(keys[i + 1]) >> (3 * kTileBits)) != t) tend[t] = i + 1;
  }
}

// per segment: chain rule over its (segment, voxel) pairs, which the front half emitted
// contiguously in primitive order; seg_grad[p] = (d/dA, d/dB) in world units.  Sixteen lanes take a
// segment's pairs: each pair is a chain of dependent lookups, and one thread a segment left too few of
// them in flight (128,000 segments, 3.2 M pairs: 0.109 ms; one thread a segment 0.212 ms).
template <class Key>
__global__ void __launch_bounds__(kBlock) k_fit_pairs(const int32_t* __restrict__ rec,
                                                      const int64_t* __restrict__ cand_off, int64_t n_prims,
                                                      const uint64_t* __restrict__ masks,
                                                      const int64_t* __restrict__ wave_off,
                                                      const int64_t* __restrict__ ctl, const Key* __restrict__ pkeys,
                                                      vx_voxels leaf, const int64_t* n_leaf_p,
                                                      const double* __restrict__ gleaf, int64_t gcap, int Sb,
                                                      double vs, const int64_t* __restrict__ tfirst,
                                                      const int64_t* __restrict__ tend, double* __restrict__ seg_grad) {
  const int64_t n_leaf = *n_leaf_p;
  const int64_t n_cand = ctl[CTL_N_CAND];
  const int64_t n_pairs = ctl[CTL_N_PAIRS];
  const Key* lk = reinterpret_cast<const Key*>(leaf.keys);
  const double inv_s = 1.0 / double(int64_t(1) << Sb);
  const int gl = threadIdx.x & 15;
  constexpr int kSegs = kBlock / 16;
  // all lanes of a group take the same branches down to the loop over its pairs
  for (int64_t p = int64_t(blockIdx.x) * kSegs + (threadIdx.x >> 4); p < n_prims; p += int64_t(gridDim.x) * kSegs) {
    double gA[3] = {0, 0, 0}, gB[3] = {0, 0, 0};
    const int64_t c0 = cand_off[p], c1 = cand_off[p + 1];
    if (c1 > c0 && c1 <= n_cand) {
      auto pair_index = [&](int64_t c) -> int64_t {
        const int64_t ch = c >> 6;
        const int r = int(c & 63);
        return wave_off[ch] + (r ? __popcll(masks[ch] & ((uint64_t(1) << r) - 1)) : 0);
      };
      int64_t j0 = pair_index(c0), j1 = pair_index(c1);
      if (j0 < 0 || j1 > n_pairs || j0 > j1) j1 = j0;          // front half over capacity: no pairs
      const int32_t* r = rec + p * kRec;
      double A[3], B[3], d[3];
      for (int a = 0; a < 3; ++a) {
        A[a] = double(r[a]) * inv_s;
        B[a] = double(r[3 + a]) * inv_s;
        d[a] = B[a] - A[a];
      }
      const double len = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
      double t[3] = {0, 0, 0};
      if (len > 0)
        for (int a = 0; a < 3; ++a) t[a] = d[a] / len;
      const double M[6] = {1 - t[0] * t[0], 1 - t[1] * t[1], 1 - t[2] * t[2], -t[0] * t[1], -t[0] * t[2], -t[1] * t[2]};
      double gM[6] = {0, 0, 0, 0, 0, 0};
      for (int64_t j = j0 + gl; j < j1; j += 16) {
        const uint64_t key = uint64_t(pkeys[j]);
        const double lo[3] = {double(compact3(key)), double(compact3(key >> 1)), double(compact3(key >> 2))};
        double dA[3], dB[3];
        const double w = seg_length_grad(A, B, lo, dA, dB);
        if (!(w > 0.0)) continue;
        int64_t v;
        if (tfirst) {
          const uint64_t t = key >> (3 * kTileBits);
          const int64_t a = tfirst[t], b = tend[t];
          v = a + key_lower_bound(lk + a, b - a, key);
          if (v >= b) continue;
        } else {
          v = key_lower_bound(lk, n_leaf, key);
        }
        if (v >= n_leaf || uint64_t(lk[v]) != key) continue;
        double gS[6];
        for (int q = 0; q < 6; ++q) gS[q] = gleaf[int64_t(q) * gcap + v];
        double gw = gleaf[6 * gcap + v];
        for (int q = 0; q < 6; ++q) {
          gw += gS[q] * M[q];
          gM[q] += w * gS[q];
        }
        for (int a = 0; a < 3; ++a) {
          gA[a] += gw * dA[a];
          gB[a] += gw * dB[a];
        }
      }
#pragma unroll
      for (int q = 0; q < 6; ++q) gM[q] = sum16(gM[q]);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        gA[a] = sum16(gA[a]);
        gB[a] = sum16(gB[a]);
      }
      if (len > 0) {
        double gt[3];
        gt[0] = -2 * t[0] * gM[0] - t[1] * gM[3] - t[2] * gM[4];
        gt[1] = -2 * t[1] * gM[1] - t[0] * gM[3] - t[2] * gM[5];
        gt[2] = -2 * t[2] * gM[2] - t[0] * gM[4] - t[1] * gM[5];
        const double dot = gt[0] * t[0] + gt[1] * t[1] + gt[2] * t[2];
        for (int a = 0; a < 3; ++a) {
          const double gd = (gt[a] - dot * t[a]) / len;
          gA[a] -= gd;
          gB[a] += gd;
        }
      }
    }
    if (gl < 6) {
      double v = gA[0];
#pragma unroll
      for (int a = 1; a < 6; ++a) v = gl == a ? (a < 3 ? gA[a] : gB[a - 3]) : v;
      seg_grad[p * 6 + gl] = v * vs;
    }
  }
}

// a point's gradient: its segment's start end plus the previous segment's far end, added in FP64
// (the two nearly cancel along a straight fiber) and rounded once
__global__ void __launch_bounds__(kBlock) k_fit_points(const double* __restrict__ seg_grad, int64_t n,
                                                       float* __restrict__ dpts) {
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock)
    for (int a = 0; a < 3; ++a)
      dpts[i * 3 + a] = float(seg_grad[i * 6 + a] + (i > 0 ? seg_grad[(i - 1) * 6 + 3 + a] : 0.0));
}

// ---------------------------------------------------------------------------------------------
// binding of the lobe parameters: row r of a level's parameters belongs to the voxel that was at
// index r when the parameters were made.  A level whose voxel count or keys differ from that
// binding (control points moved across voxels) is flagged, and every kernel stays within the
// parameter rows.
// ---------------------------------------------------------------------------------------------
template <class Key>
__global__ void __launch_bounds__(kBlock) k_fit_bind(const Key* __restrict__ keys, const int64_t* n_p, int64_t rows,
                                                     const Key* __restrict__ bound, int64_t* stats) {
  const int64_t n = *n_p;
  if (blockIdx.x == 0 && threadIdx.x == 0 && n != rows)
    atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_FIT_ROWS);
  if (!bound) return;
  const int64_t m = n < rows ? n : rows;
  bool diff = false;
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < m; i += int64_t(gridDim.x) * kBlock)
    diff = diff || keys[i] != bound[i];
  if (__any(diff) && lane_id() == 0)
    atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_FIT_KEYS);
}

// ---------------------------------------------------------------------------------------------
// FP64 sums of the levels below the fitted ones, for the backward pass.  The target's square
// roots are ill-conditioned where a child holds nearly one fiber direction and a direction of
// the set is nearly parallel to it, so the backward differentiates at sums formed in FP64 from
// the re-emitted pairs: sorted by key (stable, so each voxel's pairs stay in primitive order),
// each leaf voxel adds its clipped lengths and moments in FP64, and every level above adds its
// children.  Layout of a level: [7][cap] (S components xx yy zz xy xz yz, then w).
// ---------------------------------------------------------------------------------------------
// start has cap + 2 entries: the first pair of every key (heads past cap are dropped), the end
// at index min(total, cap), and the number of distinct keys at index cap + 1
struct LeafSegOut {
  int64_t* start;
  int64_t cap;
  __device__ void operator()(int64_t i, int64_t ex, int64_t v) const {
    if (v && ex <= cap) start[ex] = i;
  }
};
struct LeafSegTotal {
  int64_t* start;
  int64_t cap;
  const int64_t* n_leaf;
  int64_t* stats;
  __device__ void operator()(int64_t total, int64_t n) const {
    if (total <= cap) start[total] = n;
    start[cap + 1] = total;
    if (total != *n_leaf)
      atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_FIT_KEYS);
  }
};

template <class Key>
__global__ void __launch_bounds__(kBlock) k_fit_leaf64(const Key* __restrict__ pkeys, const uint32_t* __restrict__ pprim,
                                                       const int64_t* __restrict__ sstart, const int32_t* __restrict__ rec,
                                                       const Key* __restrict__ lkeys, const int64_t* n_leaf_p,
                                                       int64_t cap, int Sb, double* __restrict__ out,
                                                       int64_t* stats) {
  // within the leaf, its capacity and the keys the pairs hold (sstart[i + 1] is written for i < n)
  int64_t n = *n_leaf_p < cap ? *n_leaf_p : cap;
  n = sstart[cap + 1] < n ? sstart[cap + 1] : n;
  const double inv_s = 1.0 / double(int64_t(1) << Sb);
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(gridDim.x) * kBlock) {
    const int64_t a = sstart[i], b = sstart[i + 1];
    double W = 0.0, S[6] = {0, 0, 0, 0, 0, 0};
    if (b > a && pkeys[a] != lkeys[i])
      atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)VX_FLAG_FIT_KEYS);
    const uint64_t key = uint64_t(lkeys[i]);
    const double lo[3] = {double(compact3(key)), double(compact3(key >> 1)), double(compact3(key >> 2))};
    for (int64_t j = a; j < b; ++j) {
      const int32_t* r = rec + int64_t(pprim[j]) * kRec;
      double A[3], B[3], d[3], gA[3], gB[3];
      for (int ax = 0; ax < 3; ++ax) {
        A[ax] = double(r[ax]) * inv_s;
        B[ax] = double(r[3 + ax]) * inv_s;
        d[ax] = B[ax] - A[ax];
      }
      const double w = seg_length_grad(A, B, lo, gA, gB);
      if (!(w > 0.0)) continue;
      const double l2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
      const double il2 = 1.0 / l2;
      W += w;
      S[0] += w * (1.0 - d[0] * d[0] * il2);
      S[1] += w * (1.0 - d[1] * d[1] * il2);
      S[2] += w * (1.0 - d[2] * d[2] * il2);
      S[3] -= w * d[0] * d[1] * il2;
      S[4] -= w * d[0] * d[2] * il2;
      S[5] -= w * d[1] * d[2] * il2;
    }
#pragma unroll
    for (int t = 0; t < 6; ++t) out[int64_t(t) * cap + i] = S[t];
    out[6 * cap + i] = W;
  }
}

// level L from level L - 1: every voxel adds its children [cstart[u], cstart[u + 1]) in order
__global__ void __launch_bounds__(kBlock) k_fit_up64(const int64_t* __restrict__ cstart, const int64_t* n_p,
                                                     int64_t cap, const double* __restrict__ in, int64_t icap,
                                                     double* __restrict__ out) {
  const int64_t n = *n_p < cap ? *n_p : cap;
  for (int64_t u = int64_t(blockIdx.x) * kBlock + threadIdx.x; u < n; u += int64_t(gridDim.x) * kBlock) {
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t c = cstart[u]; c < cstart[u + 1]; ++c)
#pragma unroll
      for (int t = 0; t < 7; ++t) acc[t] += in[int64_t(t) * icap + c];
#pragma unroll
    for (int t = 0; t < 7; ++t) out[int64_t(t) * cap + u] = acc[t];
  }
}

// ---------------------------------------------------------------------------------------------
// orchestration
// ---------------------------------------------------------------------------------------------
struct FitWs {
  float* loss_vox[21];
  double* g[21];           // [7][cap_L] per level 0..hi-1
  int64_t* cstart[21];     // [cap_L + 1] per level 1..hi: first child (in level L-1) of every voxel
  int32_t* pidx[21];       // [cap_L] per level 0..hi-1: index of every voxel's parent in level L+1
  int64_t* tfirst;         // [tiles] leaf lookup: first and end leaf index of every 16^3 tile
  int64_t* tend;
  double* part;            // [kGrid] block sums of the loss
  int64_t* partial;        // [kGrid + 1] scan partials
  double* seg_grad;        // [n_pts][6] d loss / d (segment start, segment end), world units
  FrontWs f;
  double* s64[21];         // [7][cap_L] per level 0..hi-1: FP64 sums (S, then w)
  int64_t* sstart;         // [cap_0 + 2] first sorted pair of every leaf voxel, end, key count
  PairBufs pb, pc;         // sort buffers of the re-emitted pairs, ping-pong
  int32_t* hist;           // radix digit histograms
};

// dense table of 16^3 tiles for the leaf lookup of the backward pass (grids up to 2048^3)
static int64_t leaf_tiles(int log2R) {
  return log2R > kTileBits && log2R <= 11 ? int64_t(1) << (3 * (log2R - kTileBits)) : 0;
}

static size_t fit_ws_layout(int64_t n_pts, int64_t max_cand, int64_t max_pairs, const int64_t* caps, int hi,
                            int log2R, void* base, FitWs* w) {
  const bool key64 = log2R > 10;
  Carver cv(base);
  FitWs x;
  for (int L = 0; L <= hi; ++L) x.loss_vox[L] = cv.take<float>(caps[L]);
  for (int L = 0; L < hi; ++L) x.g[L] = cv.take<double>(7 * caps[L]);
  for (int L = 1; L <= hi; ++L) x.cstart[L] = cv.take<int64_t>(caps[L] + 1);
  for (int L = 0; L < hi; ++L) x.pidx[L] = cv.take<int32_t>(caps[L]);
  const int64_t tiles = leaf_tiles(log2R);
  x.tfirst = cv.take<int64_t>(tiles);
  x.tend = cv.take<int64_t>(tiles);
  x.part = cv.take<double>(kGrid);
  x.partial = cv.take<int64_t>(kGrid + 1);
  x.seg_grad = cv.take<double>(6 * n_pts);
  front_ws_carve(cv, n_pts, max_cand, max_pairs, key64, &x.f);
  for (int L = 0; L < hi; ++L) x.s64[L] = cv.take<double>(n_pts > 0 ? 7 * caps[L] : 0);
  x.sstart = cv.take<int64_t>(n_pts > 0 ? caps[0] + 2 : 0);
  const int kb = key64 ? 8 : 4;
  for (PairBufs* pbuf : {&x.pb, &x.pc}) {
    pbuf->keys = cv.take<uint8_t>(max_pairs * kb);
    pbuf->w = nullptr;
    pbuf->prim = cv.take<uint32_t>(max_pairs);
  }
  x.hist = cv.take<int32_t>(max_pairs > 0 ? int64_t(kRadixBuckets) * kGrid : 0);
  if (w) *w = x;
  return cv.off + 256;
}

size_t fit_ws_bytes(int64_t n_pts, int64_t max_cand, int64_t max_pairs, const int64_t* caps, int hi, int log2R) {
  return fit_ws_layout(n_pts, max_cand, max_pairs, caps, hi, log2R, nullptr, nullptr);
}

static int blocks_for(int64_t n, int64_t most = kGrid) {
  const int64_t b = (n + kBlock - 1) / kBlock;
  return int(b < 1 ? 1 : (b > most ? most : b));
}

// first child of every voxel of levels 1..hi, and every child's parent, all levels in one launch: a
// voxel searches the level below for its first child (at its own index at the earliest, as each
// voxel before it has one, and at eight times that at the latest) and takes the run from there.
// (0.69 M voxels in six levels: 33 us; as two scans a level 56 us)
struct ChildLevels {
  const void* keys[kMaxFit + 1];      // per level 0..hi
  const int64_t* n[kMaxFit + 1];
  int64_t* cstart[kMaxFit + 1];       // per level 1..hi
  int32_t* pidx[kMaxFit + 1];         // per level 0..hi-1
  int hi;
};
template <class Key>
__global__ void __launch_bounds__(kBlock) k_fit_children(ChildLevels lv) {
  for (int64_t i0 = int64_t(blockIdx.x) * kBlock + threadIdx.x;; i0 += int64_t(gridDim.x) * kBlock) {
    int64_t u = i0, n = 0;
    int L = 1;
    for (; L <= lv.hi; ++L) {
      n = *lv.n[L];
      if (u <= n) break;              // one more for the end
      u -= n + 1;
    }
    if (L > lv.hi) return;
    const Key* ck = static_cast<const Key*>(lv.keys[L - 1]);
    const int64_t nc = *lv.n[L - 1];
    if (u == n) {
      lv.cstart[L][n] = nc;
      continue;
    }
    const uint64_t key = uint64_t(static_cast<const Key*>(lv.keys[L])[u]);
    const int64_t lo = u < nc ? u : nc, hi = 8 * u < nc ? 8 * u : nc;
    int64_t c = lo + key_lower_bound(ck + lo, hi - lo, key << 3);
    lv.cstart[L][u] = c;
    for (; c < nc && uint64_t(ck[c]) >> 3 == key; ++c) lv.pidx[L - 1][c] = int32_t(u);
  }
}

static void child_starts(bool key64, const vx_voxels* levels, const int64_t* n_levels, int hi, const FitWs& w,
                         const int64_t* caps, hipStream_t s) {
  VX_TIMED("fit_children", s);
  ChildLevels lv;
  lv.hi = hi;
  int64_t most = 0;
  for (int L = 0; L <= hi; ++L) {
    lv.keys[L] = levels[L].keys;
    lv.n[L] = n_levels + L;
    lv.cstart[L] = L >= 1 ? w.cstart[L] : nullptr;
    lv.pidx[L] = L < hi ? w.pidx[L] : nullptr;
    if (L >= 1) most += caps[L] + 1;
  }
  if (key64) hipLaunchKernelGGL(k_fit_children<uint64_t>, dim3(blocks_for(most, 4 * kGrid)), dim3(kBlock), 0, s, lv);
  else hipLaunchKernelGGL(k_fit_children<uint32_t>, dim3(blocks_for(most, 4 * kGrid)), dim3(kBlock), 0, s, lv);
}

template <class Key>
static void bind_check(const vx_voxels* levels, const int64_t* n_levels, int lo, int hi, const int64_t* rows,
                       const void* const* bound, int64_t* stats, hipStream_t s) {
  for (int L = lo; L <= hi; ++L)
    hipLaunchKernelGGL(k_fit_bind<Key>, dim3(blocks_for(rows[L - lo])), dim3(kBlock), 0, s,
                       (const Key*)levels[L].keys, n_levels + L, rows[L - lo],
                       bound ? (const Key*)bound[L - lo] : (const Key*)nullptr, stats);
}

// the fitted levels as the kernels take them
static FitLevels fit_levels(const vx_voxels* levels, const int64_t* n_levels, int lo, int hi,
                            const float* const* params, float* const* dparams, const int64_t* rows, const FitWs& w,
                            const int64_t* caps, bool sums64) {
  FitLevels lv{};
  for (int L = lo; L <= hi; ++L) {
    FitLevel& F = lv.l[lv.count++];
    F.n = n_levels + L;
    F.rows = rows[L - lo];
    F.w = levels[L].w;
    F.cstart = w.cstart[L];
    F.Lp = params[L - lo];
    F.chw = levels[L - 1].w;
    F.chS = levels[L - 1].S;
    F.chcap = levels[L - 1].cap;
    F.loss = w.loss_vox[L];
    F.c64 = sums64 ? w.s64[L - 1] : nullptr;
    F.gch = w.g[L - 1];
    F.gcap = caps[L - 1];
    F.dLp = dparams ? dparams[L - lo] : nullptr;
  }
  return lv;
}

// directions per lane: the set in one, two or four rows of 64
template <class F>
static void with_dirs(int ndir, F&& launch) {
  if (ndir <= 64) launch(std::integral_constant<int, 1>());
  else if (ndir <= 128) launch(std::integral_constant<int, 2>());
  else launch(std::integral_constant<int, 4>());
}

// one wave per voxel, up to as many as the chip holds at a time
static int fit_blocks(const int64_t* rows, int levels) {
  int64_t n = 0;
  for (int i = 0; i < levels; ++i) n += rows[i];
  const int64_t b = (n + kWaves - 1) / kWaves;
  return int(b < 1 ? 1 : (b > kFitGrid ? kFitGrid : b));
}

vx_status fit_forward_run(const vx_grid* g, const vx_voxels* levels, const int64_t* n_levels, int lo, int hi,
                          const float* const* params, const int64_t* rows, const void* const* bound, const float* dirs,
                          int ndir, float* loss, int64_t* stats, void* ws, const int64_t* caps, hipStream_t s) {
  const bool key64 = g->log2_res > 10;
  FitWs w;
  fit_ws_layout(0, 0, 0, caps, hi, g->log2_res, ws, &w);
  launch_fill_i64(stats, VX_NSTAT, 0, s);
  if (key64) bind_check<uint64_t>(levels, n_levels, lo, hi, rows, bound, stats, s);
  else bind_check<uint32_t>(levels, n_levels, lo, hi, rows, bound, stats, s);
  child_starts(key64, levels, n_levels, hi, w, caps, s);
  LossLevels ll;
  ll.count = 0;
  const FitLevels lv = fit_levels(levels, n_levels, lo, hi, params, nullptr, rows, w, caps, false);
  for (int i = 0; i < lv.count; ++i) {
    ll.p[i] = lv.l[i].loss;
    ll.n[i] = lv.l[i].n;
    ll.rows[i] = lv.l[i].rows;
    ++ll.count;
  }
  {
    VX_TIMED("fit_fwd", s);
    with_dirs(ndir, [&](auto dpl) {
      hipLaunchKernelGGL(k_fit_fwd<dpl.value>, dim3(fit_blocks(rows, hi - lo + 1)), dim3(kBlock), 0, s, lv, dirs, ndir);
    });
  }
  VX_TIMED("fit_total", s);
  hipLaunchKernelGGL(k_fit_partial, dim3(kGrid), dim3(kBlock), 0, s, ll, w.part);
  hipLaunchKernelGGL(k_fit_total, dim3(1), dim3(1024), 0, s, w.part, loss);
  return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
}

// FP64 sums of levels 0..hi-1 from the re-emitted pairs (f.pa, emission order, left intact)
template <class Key>
static void level_sums64(const vx_grid* g, const vx_voxels* levels, const int64_t* n_levels, int hi,
                         const FitWs& w, const int64_t* caps, int64_t max_pairs, int64_t* stats, hipStream_t s) {
  VX_TIMED("fit_sums64", s);
  // (the emission order stays in w.f.pa)
  const PairBufs P = radix_sort_pairs(sizeof(Key) == 8, 3 * g->log2_res, w.f.pa, w.pb, w.pc, w.f.ctl + CTL_N_PAIRS,
                                      max_pairs, w.hist, w.partial, s);
  device_scan(HeadIn<Key, 0>{(const Key*)P.keys}, LeafSegOut{w.sstart, caps[0]},
              LeafSegTotal{w.sstart, caps[0], n_levels, stats}, w.f.ctl + CTL_N_PAIRS, max_pairs, w.partial, s);
  const Lat lat = make_lat(g, 1, 0.0f);
  hipLaunchKernelGGL(k_fit_leaf64<Key>, dim3(blocks_for(caps[0], 4 * kGrid)), dim3(kBlock), 0, s, (const Key*)P.keys, P.prim, w.sstart,
                     w.f.rec, (const Key*)levels[0].keys, n_levels, caps[0], lat.Sb, w.s64[0], stats);
  for (int L = 1; L < hi; ++L)
    hipLaunchKernelGGL(k_fit_up64, dim3(kGrid), dim3(kBlock), 0, s, w.cstart[L], n_levels + L, caps[L],
                       w.s64[L - 1], caps[L - 1], w.s64[L]);
}

vx_status fit_backward_run(const vx_grid* g, const float* pts, int64_t n_pts, const int64_t* offsets, int64_t n_fib,
                           float radius, int64_t max_cand, int64_t max_pairs, const vx_voxels* levels,
                           const int64_t* n_levels, int lo, int hi, const float* const* params, const int64_t* rows,
                           const void* const* bound, const float* dirs, int ndir, const float* dloss,
                           float* const* dparams, float* dpts, int64_t* stats, void* ws, const int64_t* caps,
                           hipStream_t s) {
  const bool key64 = g->log2_res > 10;
  FitWs w;
  fit_ws_layout(n_pts, max_cand, max_pairs, caps, hi, g->log2_res, ws, &w);
  // re-emit the pairs in primitive order (this clears stats), then check the parameters' binding
  voxelize_front(1, g, pts, n_pts, offsets, n_fib, radius, max_cand, max_pairs, w.f, stats, s, nullptr);
  if (key64) bind_check<uint64_t>(levels, n_levels, lo, hi, rows, bound, stats, s);
  else bind_check<uint32_t>(levels, n_levels, lo, hi, rows, bound, stats, s);
  child_starts(key64, levels, n_levels, hi, w, caps, s);
  // (no points: every level is empty and the FP64 sums, sized by the points, are not read)
  if (n_pts > 0) {
    if (key64) level_sums64<uint64_t>(g, levels, n_levels, hi, w, caps, max_pairs, stats, s);
    else level_sums64<uint32_t>(g, levels, n_levels, hi, w, caps, max_pairs, stats, s);
  }
  // lobe gradients and the children's (S, w) gradients
  const FitLevels lv = fit_levels(levels, n_levels, lo, hi, params, dparams, rows, w, caps, n_pts > 0);
  {
    VX_TIMED("fit_bwd", s);
    with_dirs(ndir, [&](auto dpl) {
      hipLaunchKernelGGL(k_fit_bwd<dpl.value>, dim3(fit_blocks(rows, hi - lo + 1)), dim3(kBlock), 0, s, lv, dirs, ndir,
                         dloss);
    });
  }
  // top-down accumulation to the leaf
  if (hi > 1) {
    VX_TIMED("fit_down", s);
    FitDown d{};
    d.lo = lo - 1;
    d.hi = hi;
    for (int L = 0; L < hi; ++L) {
      d.pidx[L] = w.pidx[L];
      d.g[L] = w.g[L];
      d.gcap[L] = caps[L];
      d.last[L] = uint32_t(caps[L] - 1);
    }
    hipLaunchKernelGGL(k_fit_down, dim3(blocks_for(caps[0], 4 * kGrid)), dim3(kBlock), 0, s, d, n_levels);
  }
  // the chain rule per segment over its pairs (emission order) and per point
  const Lat lat = make_lat(g, 1, radius);
  const double vs = double(int64_t(1) << g->log2_res) / g->extent;
  const int64_t tiles = leaf_tiles(g->log2_res);
  if (tiles) {
    VX_TIMED("fit_tiles", s);
    launch_fill_i64(w.tfirst, tiles, 0, s);
    launch_fill_i64(w.tend, tiles, 0, s);
    if (key64)
      hipLaunchKernelGGL(k_tile_index<uint64_t>, dim3(kGrid), dim3(kBlock), 0, s, (const uint64_t*)levels[0].keys,
                         n_levels, tiles, w.tfirst, w.tend);
    else
      hipLaunchKernelGGL(k_tile_index<uint32_t>, dim3(kGrid), dim3(kBlock), 0, s, (const uint32_t*)levels[0].keys,
                         n_levels, tiles, w.tfirst, w.tend);
  }
  {
    VX_TIMED("fit_pairs", s);
    if (key64)
      hipLaunchKernelGGL(k_fit_pairs<uint64_t>, dim3(blocks_for(16 * n_pts, 8 * kGrid)), dim3(kBlock), 0, s, w.f.rec, w.f.cand_off,
                         n_pts, w.f.masks, w.f.wave_off, w.f.ctl, (const uint64_t*)w.f.pa.keys, levels[0], n_levels,
                         w.g[0], caps[0], lat.Sb, vs, tiles ? w.tfirst : nullptr, w.tend, w.seg_grad);
    else
      hipLaunchKernelGGL(k_fit_pairs<uint32_t>, dim3(blocks_for(16 * n_pts, 8 * kGrid)), dim3(kBlock), 0, s, w.f.rec, w.f.cand_off,
                         n_pts, w.f.masks, w.f.wave_off, w.f.ctl, (const uint32_t*)w.f.pa.keys, levels[0], n_levels,
                         w.g[0], caps[0], lat.Sb, vs, tiles ? w.tfirst : nullptr, w.tend, w.seg_grad);
  }
  {
    VX_TIMED("fit_points", s);
    hipLaunchKernelGGL(k_fit_points, dim3(blocks_for(n_pts)), dim3(kBlock), 0, s, w.seg_grad, n_pts, dpts);
  }
  return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
}

}  // namespace vx
