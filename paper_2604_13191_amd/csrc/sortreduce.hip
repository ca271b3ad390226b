// sortreduce.hip -- ordering keyed records and the parent levels of the pyramid.
//   radix sort  : Sec. 3.3 orders the samples by voxel id so that each voxel's samples are
//                 contiguous; here a stable LSD radix sort (9-bit digits) with wave-level
//                 ranking in LDS, fixed grid, no atomics on global memory -- applied to the
//                 primitive-tile records, which group the work by tile.
//   LoD level   : Sec. 4.3 aggregates 2x2x2 children into a coarser voxel; children of a parent
//                 are contiguous in Morton order, so this is a segmented sum over key >> 3.
#include "vx_internal.hpp"

namespace vx {

__device__ __forceinline__ void flag_or_s(int64_t* p, int64_t bit) {
  atomicOr(reinterpret_cast<unsigned long long*>(p), (unsigned long long)bit);
}

// ---------------------------------------------------------------------------------------------
// radix sort
// ---------------------------------------------------------------------------------------------
constexpr int kDigitBits = kRadixBits;        // 18-bit tile keys (1024^3 grids) sort in two passes
constexpr int kBuckets = 1 << kDigitBits;
static_assert(kBuckets == kRadixBuckets, "histogram workspace");
constexpr int kSortBlock = 512;               // one thread per digit, 8 waves
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kSortE = 8;                     // elements per thread of a scatter tile
constexpr int kSortTile = kSortBlock * kSortE;
static_assert(kBuckets == kSortBlock, "thread d serves digit d");
// Blocks of the sort kernels.  Large inputs: two per CU, all resident with the scatter's LDS, at least
// two tiles each.  Small ones (up to 32 blocks): the scatter adds up the digit counts of the blocks
// before it by itself (32 x 512 counts from L2) instead of leaving that to a scan's two launches
// (28,000 records, one pass: 16 us; with the scan, whose part was 11 us, 31 us).
constexpr int kSortFused = 32;
constexpr int kSortGrid = kGrid;
static_assert(kSortGrid <= kGrid, "histogram workspace");
inline int sort_blocks(int64_t cap) {
  const int64_t half = (cap + kSortTile / 2 - 1) / (kSortTile / 2), two = (cap + 2 * kSortTile - 1) / (2 * kSortTile);
  if (two <= kSortFused) return int(half < 1 ? 1 : (half < kSortFused ? half : kSortFused));
  return int(two < kSortGrid ? two : kSortGrid);
}

__device__ __forceinline__ int64_t sort_chunk(int64_t n) {
  const int64_t c = (n + gridDim.x - 1) / gridDim.x;
  return (c + kSortBlock - 1) / kSortBlock * kSortBlock;
}

// the stretches that a block serves: its chunk of dense input, or its share of the regions
struct SortSpan {
  int r, r1;
  int64_t b0, b1;
};
__device__ __forceinline__ SortSpan first_span(const SortRegions& g) {
  if (!g.filled) return SortSpan{0, 1, 0, 0};
  return SortSpan{int(int64_t(blockIdx.x) * g.regions / gridDim.x), int(int64_t(blockIdx.x + 1) * g.regions / gridDim.x),
                  0, 0};
}
__device__ __forceinline__ bool next_span(SortSpan& s, const SortRegions& g, const int64_t* n_ptr) {
  if (s.r >= s.r1) return false;
  if (g.filled) {
    s.b0 = s.r * ((*g.slots + g.regions - 1) / g.regions);
    s.b1 = s.b0 + g.filled[s.r];
  } else {
    const int64_t n = *n_ptr, chunk = sort_chunk(n);
    s.b0 = int64_t(blockIdx.x) * chunk;
    s.b1 = s.b0 + chunk < n ? s.b0 + chunk : n;
  }
  ++s.r;
  return true;
}

// Digit counts of every block's chunk: hist[d][block], or hist[block][d] for the fused scatter.
// Eight rows of 512 keys are loaded together; runs of one digit in a row (common: records of one tile)
// are added once each, by their first lanes.  Bound by the read with keys spread widely (41.7 M 64-bit
// samples: 0.089 ms = 3.7 TB/s, with four rows of 256 per block 0.16 ms), by LDS adds to the same few
// counters otherwise (47.6 M records: 0.16 ms; every lane adding by itself 0.22 ms).
template <class Key, bool FUSED>
__global__ void __launch_bounds__(kSortBlock) k_radix_hist(const Key* __restrict__ keys, const int64_t* n_ptr, int shift,
                                                           int32_t* __restrict__ hist, const int64_t* only_if,
                                                           SortRegions regions) {
  __shared__ int32_t h[kSortWaves][kBuckets];
  if (only_if && *only_if == 0) return;
  const int t = threadIdx.x, w = t >> 6, lane = lane_id();
#pragma unroll
  for (int q = 0; q < kSortWaves; ++q) h[q][t] = 0;
  __syncthreads();
  SortSpan span = first_span(regions);
  while (next_span(span, regions, n_ptr)) for (int64_t t0 = span.b0; t0 < span.b1; t0 += kSortTile) {
    int dg[kSortE];
#pragma unroll
    for (int j = 0; j < kSortE; ++j) {
      const int64_t i = t0 + j * kSortBlock + t;
      dg[j] = i < span.b1 ? int((keys[i] >> shift) & (kBuckets - 1)) : -1;
    }
#pragma unroll
    for (int j = 0; j < kSortE; ++j) {
      const int prev = __builtin_amdgcn_update_dpp(-1, dg[j], 0x138, 0xf, 0xf, false);   // of the lane before
      const bool head = lane == 0 || dg[j] != prev;
      const uint64_t heads = __builtin_amdgcn_ballot_w64(head);
      const uint64_t after = heads >> lane >> 1;
      const int len = after ? __ffsll((unsigned long long)after) : 64 - lane;
      if (head && dg[j] >= 0) atomicAdd(&h[w][dg[j]], len);
    }
  }
  __syncthreads();
  int32_t sum = 0;
#pragma unroll
  for (int q = 0; q < kSortWaves; ++q) sum += h[q][t];
  hist[FUSED ? int64_t(blockIdx.x) * kBuckets + t : int64_t(t) * gridDim.x + blockIdx.x] = sum;
}

struct I32In {
  const int32_t* a;
  __device__ int64_t operator()(int64_t i) const { return a[i]; }
};
struct I32Out {
  int32_t* o;
  __device__ void operator()(int64_t i, int64_t ex, int64_t) const { o[i] = int32_t(ex); }
};
struct NoTotal {
  __device__ void operator()(int64_t, int64_t) const {}
};

// One pass of the stable scatter.  A block takes its chunk in tiles of kSortTile elements, each wave a
// contiguous eighth of the tile, row by row: lanes holding the same digit find each other by
// ballots over its bits, and the wave's running count of the digit gives their ranks.  One scan over
// the digits places the tile digit by digit in LDS, and it is written out in that order: each
// digit's run (8 elements on average) lands contiguously at the digit's next position.  Order within
// a digit is wave, row, lane = input order: the sort is stable.
// Bound by HBM and, close behind, by the ballots: 41.7 M samples in 64-bit words, per pass 0.166 ms
// (4.0 TB/s); in tiles of 1,024, with counts per row and wave and the weights carried along, 0.39 ms.
template <class Key, bool PRIM, bool FUSED>
__global__ void __launch_bounds__(kSortBlock) k_radix_scatter(const Key* __restrict__ kin,
                                                              const uint32_t* __restrict__ pin, Key* __restrict__ kout,
                                                              uint32_t* __restrict__ pout, const int64_t* n_ptr,
                                                              int shift, const int32_t* __restrict__ hist,
                                                              const int64_t* only_if, SortRegions regions) {
  __shared__ uint16_t cnt[kSortWaves][kBuckets];       // per wave: counts, then first slots in the tile
  __shared__ int32_t place[kBuckets];                  // output position less tile slot, per digit
  __shared__ Key sk[kSortTile];
  __shared__ uint32_t sp[PRIM ? kSortTile : 1];
  __shared__ int32_t stmp[kSortWaves + 1];
  if (only_if && *only_if == 0) return;
  const int t = threadIdx.x, w = t >> 6, lane = lane_id();
  int32_t run;                                         // next output position of digit t
  if (FUSED) {
    int32_t before = 0, all = 0, total;
    constexpr int kAtOnce = 8;
    for (int g0 = 0; g0 < int(gridDim.x); g0 += kAtOnce) {
      int32_t c[kAtOnce];
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        const int g = g0 + j < int(gridDim.x) ? g0 + j : 0;
        c[j] = hist[int64_t(g) * kBuckets + t];
      }
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        const int g = g0 + j;
        before += g < int(blockIdx.x) ? c[j] : 0;
        all += g < int(gridDim.x) ? c[j] : 0;
      }
    }
    run = block_exclusive_scan_n<kSortWaves>(all, stmp, total) + before;
  } else {
    run = hist[int64_t(t) * gridDim.x + blockIdx.x];
  }
  SortSpan span = first_span(regions);
  while (next_span(span, regions, n_ptr)) for (int64_t t0 = span.b0; t0 < span.b1; t0 += kSortTile) {
    const int ntile = int(span.b1 - t0 < kSortTile ? span.b1 - t0 : kSortTile);
    Key k[kSortE];
    uint32_t pv[kSortE];
    int rk[kSortE];
#pragma unroll
    for (int j = 0; j < kSortE; ++j) {
      const int e = w * (64 * kSortE) + j * 64 + lane;
      k[j] = e < ntile ? kin[t0 + e] : Key(0);
      if (PRIM) pv[j] = e < ntile ? pin[t0 + e] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) cnt[q][t] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortE; ++j) {
      const bool valid = w * (64 * kSortE) + j * 64 + lane < ntile;
      const int dg = int((k[j] >> shift) & (kBuckets - 1));
      const uint64_t valids = __builtin_amdgcn_ballot_w64(valid);
      uint32_t plo = uint32_t(valids), phi = uint32_t(valids >> 32);
#pragma unroll
      for (int b = 0; b < kDigitBits; ++b) {            // keep the lanes whose bit is this lane's
        const int mine = __builtin_amdgcn_sbfe(dg, b, 1);
        const uint64_t m = __builtin_amdgcn_ballot_w64(mine != 0);
        plo &= ~(uint32_t(m) ^ uint32_t(mine));
        phi &= ~(uint32_t(m >> 32) ^ uint32_t(mine));
      }
      const int r = int(__builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0)));
      const int have = valid ? int(cnt[w][dg]) : 0;
      rk[j] = have + r;
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (valid && r == 0) cnt[w][dg] = uint16_t(have + __popc(plo) + __popc(phi));
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    // digit t: its counts over the waves in input order, and its first slot in the sorted tile
    int32_t c[kSortWaves], sum = 0, total;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
      c[q] = cnt[q][t];
      sum += c[q];
    }
    int32_t slot0 = block_exclusive_scan_n<kSortWaves>(sum, stmp, total);
    place[t] = run - slot0;
    run += sum;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
      cnt[q][t] = uint16_t(slot0);
      slot0 += c[q];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortE; ++j) {
      if (w * (64 * kSortE) + j * 64 + lane < ntile) {
        const int slot = int(cnt[w][int((k[j] >> shift) & (kBuckets - 1))]) + rk[j];
        sk[slot] = k[j];
        if (PRIM) sp[slot] = pv[j];
      }
    }
    __syncthreads();
    for (int q = t; q < ntile; q += kSortBlock) {
      const Key kk = sk[q];
      const int32_t pos = place[int((kk >> shift) & (kBuckets - 1))] + q;
      kout[pos] = kk;
      if (PRIM) pout[pos] = sp[q];
    }
    __syncthreads();
  }
}

template <class Key>
static void radix_pass(const PairBufs& src, const PairBufs& dst, const int64_t* n_dev, int64_t cap, int shift,
                       int32_t* hist, int64_t* partial, const int64_t* only_if, const SortRegions& regions,
                       hipStream_t s) {
  // (with gaps, a few regions a block: each costs a tile, full or not)
  const int blocks = regions.filled ? bounded_grid(kSortGrid, regions.regions / 4) : sort_blocks(cap);
  const bool fused = blocks <= kSortFused;
  {
    VX_TIMED("radix_hist", s);
    if (fused)
      hipLaunchKernelGGL((k_radix_hist<Key, true>), dim3(blocks), dim3(kSortBlock), 0, s, (const Key*)src.keys, n_dev,
                         shift, hist, only_if, regions);
    else
      hipLaunchKernelGGL((k_radix_hist<Key, false>), dim3(blocks), dim3(kSortBlock), 0, s, (const Key*)src.keys, n_dev,
                         shift, hist, only_if, regions);
  }
  if (!fused) {
    VX_TIMED("radix_scan", s);
    device_scan(I32In{hist}, I32Out{hist}, NoTotal{}, nullptr, int64_t(kBuckets) * blocks, partial, s);
  }
  VX_TIMED("radix_scatter", s);
  const auto scatter = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kSortBlock), 0, s, (const Key*)src.keys, src.prim, (Key*)dst.keys,
                       dst.prim, n_dev, shift, hist, only_if, regions);
  };
  if constexpr (sizeof(Key) == 8) {
    if (!src.prim)
      return fused ? scatter(k_radix_scatter<Key, false, true>) : scatter(k_radix_scatter<Key, false, false>);
  }
  fused ? scatter(k_radix_scatter<Key, true, true>) : scatter(k_radix_scatter<Key, true, false>);
}

void radix_sort_pass(bool key64, const PairBufs& src, const PairBufs& dst, const int64_t* n_dev, int64_t cap,
                     int shift, int32_t* hist, int64_t* partial, const int64_t* only_if, hipStream_t s) {
  if (key64) radix_pass<uint64_t>(src, dst, n_dev, cap, shift, hist, partial, only_if, {}, s);
  else radix_pass<uint32_t>(src, dst, n_dev, cap, shift, hist, partial, only_if, {}, s);
}

PairBufs radix_sort_pairs(bool key64, int key_bits, const PairBufs& in, const PairBufs& t0, const PairBufs& t1,
                          const int64_t* n_dev, int64_t cap, int32_t* hist, int64_t* partial, hipStream_t s,
                          int first_bit, const SortRegions& regions) {
  PairBufs src = in, dst = t0, spare = t1;
  for (int shift = first_bit; shift < first_bit + key_bits; shift += kDigitBits) {
    const SortRegions g = shift == first_bit ? regions : SortRegions{};
    if (key64) radix_pass<uint64_t>(src, dst, n_dev, cap, shift, hist, partial, nullptr, g, s);
    else radix_pass<uint32_t>(src, dst, n_dev, cap, shift, hist, partial, nullptr, g, s);
    src = dst;
    const PairBufs x = dst;
    dst = spare;
    spare = x;
  }
  return src;
}

// ---------------------------------------------------------------------------------------------
// LoD: parent = sum of its (<= 8, contiguous) children
// ---------------------------------------------------------------------------------------------
// sum of the children [a, b) of one parent (in Morton order, so the sums are sequential and fixed)
template <class Key, bool BATCH>
__device__ __forceinline__ void lod_parent(const vx_voxels& in, const Key* ikeys, int64_t a, int64_t b,
                                           const vx_voxels& out, int64_t p) {
  const int64_t ci = in.cap, co = out.cap;
  uint32_t c = 0, mask = 0;
  float W = 0.f, S[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // kAtOnce children at a time: their loads do not wait for one another, the sums stay in order (14
  // patches' pyramid 0.52 -> 0.46 ms; two at a time 0.48, all eight 0.50)
  constexpr int kAtOnce = 4;
  for (int64_t j0 = a; j0 < b; j0 += kAtOnce) {
    uint32_t cc[kAtOnce], low[kAtOnce];
    float ww[kAtOnce], ss[kAtOnce][6];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const int64_t j = j0 + q < b ? j0 + q : b - 1;
      cc[q] = in.count[j];
      low[q] = uint32_t(ikeys[j] & 7);
      ww[q] = in.w[j];
#pragma unroll
      for (int k = 0; k < 6; ++k) ss[q][k] = in.S[k * ci + j];
    }
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const bool on = j0 + q < b;
      c += on ? cc[q] : 0u;
      mask |= on ? 1u << low[q] : 0u;
      W = on ? W + ww[q] : W;
#pragma unroll
      for (int k = 0; k < 6; ++k) S[k] = on ? S[k] + ss[q][k] : S[k];
    }
  }
  reinterpret_cast<Key*>(out.keys)[p] = parent_key<Key, BATCH>(ikeys[a]);
  out.count[p] = c;
  out.mask[p] = uint8_t(mask);
  out.w[p] = W;
#pragma unroll
  for (int k = 0; k < 6; ++k) out.S[k * co + p] = S[k];
}

// One level: ranks of the heads as in k_scan_apply, and the parents summed right there -- a round's
// heads are listed in LDS, then each thread takes a parent and its children.  pstart (for the lobes
// of the level; may be nullptr) gets the parents' first children and, at the end, n.
template <class Key, bool BATCH>
__global__ void __launch_bounds__(kBlock) k_lod_apply(vx_voxels in, const int64_t* __restrict__ n_ptr, vx_voxels out,
                                                      int64_t* __restrict__ n_out, int64_t* flags,
                                                      int64_t* __restrict__ pstart,
                                                      const int64_t* __restrict__ partial) {
  __shared__ int64_t tmp[kWaves + 1];
  __shared__ int32_t head[kBlock * kScanRun];
  const Key* ikeys = reinterpret_cast<const Key*>(in.keys);
  const int64_t n = *n_ptr;
  const int64_t chunk = scan_chunk(n);
  const int64_t b0 = int64_t(blockIdx.x) * chunk;
  const int64_t b1 = b0 + chunk < n ? b0 + chunk : n;
  const auto total = [&](int64_t all) {
    const bool over = all > out.cap;
    if (over) flag_or_s(flags, VX_FLAG_VOXEL_CAPACITY);
    if (pstart && !over) pstart[all] = n;       // (over: the heads fill the start at out.cap themselves)
    *n_out = over ? out.cap : all;
  };
  const bool alone = gridDim.x == 1;
  int64_t base = 0;
  if (!alone) {
    int64_t all;
    base = block_scan_base(partial, tmp, all);
    if (blockIdx.x == 0 && threadIdx.x == 0) total(all);
  }
  const HeadIn<Key, 3, BATCH> is_head{ikeys};
  for (int64_t t0 = b0; t0 < b1; t0 += int64_t(kBlock) * kScanRun) {
    const int64_t i0 = t0 + int64_t(threadIdx.x) * kScanRun;
    int v[kScanRun], run = 0;
#pragma unroll
    for (int j = 0; j < kScanRun; ++j) {
      v[j] = i0 + j < b1 ? int(is_head(i0 + j)) : 0;
      run += v[j];
    }
    int64_t tot;
    int ex = int(block_exclusive_scan(int64_t(run), tmp, tot));
#pragma unroll
    for (int j = 0; j < kScanRun; ++j) {
      if (v[j]) {
        head[ex] = int(i0 - t0) + j;
        if (pstart && base + ex <= out.cap) pstart[base + ex] = i0 + j;
      }
      ex += v[j];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < int(tot); q += kBlock) {
      const int64_t a = t0 + head[q];
      int64_t b;
      if (q + 1 < int(tot)) {
        b = t0 + head[q + 1];
      } else {                          // the last parent's children may reach past the round
        const Key pk = parent_key<Key, BATCH>(ikeys[a]);
        for (b = a + 1; b < n && parent_key<Key, BATCH>(ikeys[b]) == pk;) ++b;
      }
      if (base + q < out.cap) lod_parent<Key, BATCH>(in, ikeys, a, b, out, base + q);
    }
    base += tot;
    __syncthreads();
  }
  if (alone && threadIdx.x == 0) total(base);
}

constexpr int kLodBlock = 1024;
constexpr int kLodWaves = kLodBlock / 64;

// The small top levels in one launch (one block): level after level, heads of the parent key
// in chunks, ranks by block scan, children summed as above.  The levels built here stay in LDS
// between levels (in place: every parent's sums are taken into registers before any parent is
// written back), so a level never reads global memory written by the one before.  in_cap of the
// first level <= kTailMax.
constexpr int kTailLevels = 21;
constexpr int kTailChunks = int(kTailMax / kLodBlock);
static_assert(kTailMax % kLodBlock == 0, "whole chunks");
struct TailLevels {
  vx_voxels lv[kTailLevels];    // lv[0] = the input of the first level built here
  int64_t* n[kTailLevels];      // device counts, n[0] the input's
  int count;                    // levels to build: lv[1 .. count]
};

template <class Key>
constexpr size_t tail_lds_bytes() {
  return size_t(kTailMax) * (sizeof(Key) + 4 + 4 + 24);
}

template <class Key, bool BATCH>
__global__ void __launch_bounds__(kLodBlock) k_lod_tail(TailLevels T, int64_t* __restrict__ flags) {
  extern __shared__ double tail_dyn[];
  __shared__ int64_t tmp[kLodWaves + 1];
  Key* lk = reinterpret_cast<Key*>(tail_dyn);
  uint32_t* lc = reinterpret_cast<uint32_t*>(lk + kTailMax);
  float* lw = reinterpret_cast<float*>(lc + kTailMax);
  float* lS = lw + kTailMax;                                 // [6][kTailMax]
  const int tid = threadIdx.x;
  int64_t n = *T.n[0];
  n = n < kTailMax ? n : kTailMax;
  {
    const vx_voxels& in = T.lv[0];
    const Key* k = reinterpret_cast<const Key*>(in.keys);
    for (int64_t i = tid; i < n; i += kLodBlock) {
      lk[i] = k[i];
      lc[i] = in.count[i];
      lw[i] = in.w[i];
#pragma unroll
      for (int c = 0; c < 6; ++c) lS[c * kTailMax + i] = in.S[c * in.cap + i];
    }
  }
  __syncthreads();
  for (int L = 1; L <= T.count; ++L) {
    const vx_voxels& out = T.lv[L];
    // read phase: every parent's sums into registers (chunk q of the children, one per thread)
    int64_t pp[kTailChunks];
    Key pk[kTailChunks];
    uint32_t pc[kTailChunks], pm[kTailChunks];
    float pw[kTailChunks], pS[kTailChunks][6];
    int64_t base = 0;
#pragma unroll
    for (int q = 0; q < kTailChunks; ++q) {
      pp[q] = -1;
      if (int64_t(q) * kLodBlock >= n) continue;     // uniform: no children in this chunk
      const int64_t i = int64_t(q) * kLodBlock + tid;
      const bool head = i < n && (i == 0 || parent_key<Key, BATCH>(lk[i]) != parent_key<Key, BATCH>(lk[i - 1]));
      int64_t tot;
      const int64_t ex = block_exclusive_scan_n<kLodWaves>(int64_t(head), tmp, tot);
      pp[q] = head ? base + ex : -1;
      pk[q] = 0;
      pc[q] = 0;
      pm[q] = 0;
      pw[q] = 0.f;
#pragma unroll
      for (int c = 0; c < 6; ++c) pS[q][c] = 0.f;
      if (head) {
        const Key key = parent_key<Key, BATCH>(lk[i]);
        pk[q] = key;
        for (int64_t j = i; j < n && j < i + 8 && parent_key<Key, BATCH>(lk[j]) == key; ++j) {
          pc[q] += lc[j];
          pm[q] |= 1u << uint32_t(lk[j] & 7);
          pw[q] += lw[j];
#pragma unroll
          for (int c = 0; c < 6; ++c) pS[q][c] += lS[c * kTailMax + j];
        }
      }
      base += tot;
    }
    __syncthreads();                                 // all children read before any is overwritten
    const int64_t cap = out.cap;
    Key* ok = reinterpret_cast<Key*>(out.keys);
#pragma unroll
    for (int q = 0; q < kTailChunks; ++q) {
      const int64_t p = pp[q];
      if (p >= 0 && p < cap) {
        lk[p] = pk[q];
        lc[p] = pc[q];
        lw[p] = pw[q];
#pragma unroll
        for (int c = 0; c < 6; ++c) lS[c * kTailMax + p] = pS[q][c];
        ok[p] = pk[q];
        out.count[p] = pc[q];
        out.mask[p] = uint8_t(pm[q]);
        out.w[p] = pw[q];
#pragma unroll
        for (int c = 0; c < 6; ++c) out.S[c * cap + p] = pS[q][c];
      }
    }
    const bool over = base > cap;
    if (tid == 0) {
      if (over) flag_or_s(flags, VX_FLAG_VOXEL_CAPACITY);
      *T.n[L] = over ? cap : base;
    }
    n = over ? cap : base;
    __syncthreads();
  }
}

// level counts of a pyramid build: entry 0 is the leaf count clamped to [0, cap], the other
// count - 1 entries (levels and the flag word) start at zero
__global__ void k_lod_init(const int64_t* src, int64_t cap, int64_t* n_levels, int64_t count) {
  for (int64_t i = threadIdx.x; i < count; i += blockDim.x) {
    if (i == 0) {
      const int64_t v = *src;
      n_levels[0] = v < 0 ? 0 : (v > cap ? cap : v);
    } else {
      n_levels[i] = 0;
    }
  }
}

void lod_init(const int64_t* src, int64_t cap, int64_t* n_levels, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_lod_init, dim3(1), dim3(64), 0, s, src, cap, n_levels, count);
}

template <class Key, bool BATCH>
static void lod_level_as(const vx_voxels& in, const int64_t* n_in, const vx_voxels& out, int64_t* n_out, int64_t* flags,
                         int64_t* pstart, int64_t* partial, int blocks, hipStream_t s) {
  if (blocks > 1) {
    VX_TIMED("lod_heads", s);
    using Heads = HeadIn<Key, 3, BATCH>;
    hipLaunchKernelGGL(k_scan_partial<Heads>, dim3(blocks), dim3(kBlock), 0, s, Heads{(const Key*)in.keys}, n_in,
                       int64_t(0), partial);
  }
  VX_TIMED("lod_reduce", s);
  hipLaunchKernelGGL((k_lod_apply<Key, BATCH>), dim3(blocks), dim3(kBlock), 0, s, in, n_in, out, n_out, flags, pstart,
                     partial);
}

void lod_level(bool key64, const vx_voxels& in, const int64_t* n_in, const vx_voxels& out, int64_t* n_out,
               int64_t* flags, int64_t* pstart, int64_t* partial, int grid_blocks, hipStream_t s, bool batch) {
  const int blocks = scan_blocks(in.cap, grid_blocks < kGrid ? grid_blocks : kGrid);
  if (batch) lod_level_as<uint64_t, true>(in, n_in, out, n_out, flags, pstart, partial, blocks, s);
  else if (key64) lod_level_as<uint64_t, false>(in, n_in, out, n_out, flags, pstart, partial, blocks, s);
  else lod_level_as<uint32_t, false>(in, n_in, out, n_out, flags, pstart, partial, blocks, s);
}

void lod_tail(bool key64, bool batch, const vx_voxels* lv, int64_t* const* n, int count, int64_t* flags,
              hipStream_t s) {
  if (count < 1) return;
  VX_TIMED("lod_tail", s);
  TailLevels T;
  for (int i = 0; i <= count && i < kTailLevels; ++i) {
    T.lv[i] = lv[i];
    T.n[i] = n[i];
  }
  T.count = count < kTailLevels ? count : kTailLevels - 1;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)k_lod_tail<uint64_t, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              int(tail_lds_bytes<uint64_t>()));
    (void)hipFuncSetAttribute((const void*)k_lod_tail<uint64_t, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              int(tail_lds_bytes<uint64_t>()));
    (void)hipFuncSetAttribute((const void*)k_lod_tail<uint32_t, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              int(tail_lds_bytes<uint32_t>()));
    attr = true;
  }
  if (batch)
    hipLaunchKernelGGL((k_lod_tail<uint64_t, true>), dim3(1), dim3(kLodBlock), tail_lds_bytes<uint64_t>(), s, T, flags);
  else if (key64)
    hipLaunchKernelGGL((k_lod_tail<uint64_t, false>), dim3(1), dim3(kLodBlock), tail_lds_bytes<uint64_t>(), s, T,
                       flags);
  else
    hipLaunchKernelGGL((k_lod_tail<uint32_t, false>), dim3(1), dim3(kLodBlock), tail_lds_bytes<uint32_t>(), s, T,
                       flags);
}

}  // namespace vx
