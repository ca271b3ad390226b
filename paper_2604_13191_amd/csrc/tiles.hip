// tiles.hip -- the leaf pass by spatial tiles (Sec. 3.2-3.4 on a tiled grid).
//
// Space is cut into aligned tiles of 2^tb voxels per axis (tb = 4: 16^3 voxels, one Morton
// range each).  Every primitive is listed once per tile its candidate box overlaps; the list is
// sorted by tile (a small radix sort over primitive-tile records, not over pairs).  Tiles whose
// candidate count exceeds what a work unit holds are split into octants, recursively, down to
// single voxels.  One block then takes a unit: it tests the unit's candidates, keeps the
// surviving (voxel, weight, primitive) triples in LDS, groups them by voxel and sums every
// voxel's pairs in primitive order -- the order of the pair list of the global path, so the
// sums are bit-identical -- and writes the unit's voxels.  No pair list goes through HBM.
#include "geom.hpp"
#include "vx_internal.hpp"

namespace vx {

namespace {

__device__ __forceinline__ void flag_set(int64_t* stats, int64_t bit) {
  atomicOr(reinterpret_cast<unsigned long long*>(stats + VX_STAT_FLAGS), (unsigned long long)bit);
}


// a block-wide sum (all threads get it); tmp: kWaves + 1 entries
template <class T>
__device__ __forceinline__ T block_sum(T v, T* tmp) {
  T tot;
  (void)block_exclusive_scan(v, tmp, tot);
  return tot;
}

// candidates of primitive record r inside the box [o, o + sz): per-axis first voxel and extent
__device__ __forceinline__ int64_t clip_box(const int32_t* r, const int32_t o[3], const int32_t sz[3], int32_t lo[3],
                                            int32_t n[3]) {
  int64_t c = 1;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int32_t l = r[9 + a] > o[a] ? r[9 + a] : o[a];
    const int32_t h0 = r[9 + a] + r[12 + a] - 1, h1 = o[a] + sz[a] - 1;
    const int32_t h = h0 < h1 ? h0 : h1;
    lo[a] = l;
    n[a] = h >= l ? h - l + 1 : 0;
    c *= n[a];
  }
  return c;
}

// the same from a packed box
__device__ __forceinline__ int64_t clip_packed(const ulonglong2& b, const int32_t o[3], const int32_t sz[3]) {
  int32_t bl[3], bh[3];
  unpack_box(b, bl, bh);
  int64_t c = 1;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int32_t l = bl[a] > o[a] ? bl[a] : o[a];
    const int32_t h1 = o[a] + sz[a] - 1;
    const int32_t h = bh[a] < h1 ? bh[a] : h1;
    c *= h >= l ? h - l + 1 : 0;
  }
  return c;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// primitive-tile records
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_rec_count(const ulonglong2* __restrict__ box,
                                                      const int64_t* __restrict__ cand_cnt, int64_t n_prims, int tb,
                                                      int64_t* __restrict__ rcnt) {
  for (int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x; p < n_prims; p += int64_t(gridDim.x) * kBlock) {
    int64_t c = 0;
    if (cand_cnt[p] > 0) {
      int32_t lo[3], hi[3];
      unpack_box(box[p], lo, hi);
      c = 1;
#pragma unroll
      for (int a = 0; a < 3; ++a) c *= int64_t((hi[a] >> tb) - (lo[a] >> tb) + 1);
    }
    rcnt[p] = c;
  }
}

struct RecTotal {
  int64_t* off;
  int64_t* ctl;
  int64_t* stats;
  int64_t cap;
  __device__ void operator()(int64_t total, int64_t n) const {
    off[n] = total;
    stats[VX_STAT_RECORDS] = total;
    const bool over = total > cap;
    if (over) flag_set(stats, VX_FLAG_RECORD_CAPACITY);
    ctl[CTL_N_REC] = over ? 0 : total;
  }
};

// record (tile key, primitive) for every tile a primitive's candidate box overlaps; the tile key
// is the Morton code of the tile coordinates (batched: with the patch id above it).  roff: the
// scanned record counts (n_prims + 1 entries); a primitive without candidates has none.
template <class Key>
__global__ void __launch_bounds__(kBlock) k_rec_emit(const int32_t* __restrict__ rec,
                                                     const ulonglong2* __restrict__ box,
                                                     const int64_t* __restrict__ roff, int64_t n_prims,
                                                     const int64_t* __restrict__ ctl, int tb, int batch,
                                                     Key* __restrict__ rkeys, uint32_t* __restrict__ rprim) {
  if (ctl[CTL_N_REC] == 0) return;
  for (int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x; p < n_prims; p += int64_t(gridDim.x) * kBlock) {
    if (roff[p + 1] == roff[p]) continue;
    int32_t t0[3], t1[3];
    unpack_box(box[p], t0, t1);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      t0[a] >>= tb;
      t1[a] >>= tb;
    }
    const Key hi = batch ? Key(uint64_t(uint32_t(rec[p * kRec + 15])) << (kPatchShift - 3 * tb)) : Key(0);
    int64_t o = roff[p];
    for (int32_t z = t0[2]; z <= t1[2]; ++z)
      for (int32_t y = t0[1]; y <= t1[1]; ++y)
        for (int32_t x = t0[0]; x <= t1[0]; ++x) {
          rkeys[o] = hi | Key(morton3(uint32_t(x), uint32_t(y), uint32_t(z)));
          rprim[o] = uint32_t(p);
          ++o;
        }
  }
}

struct TileTotal {
  int64_t* start;
  int64_t* ctl;
  __device__ void operator()(int64_t total, int64_t n) const {
    start[total] = n;
    ctl[CTL_N_TILES] = total;
  }
};

// ---------------------------------------------------------------------------------------------
// work units: a tile, or an octant of one, whose candidates fit a block's LDS
// ---------------------------------------------------------------------------------------------
struct Unit {
  int64_t tile;       // index into the tile list
  int64_t cand;       // candidates inside the unit
  int32_t o[3];       // first voxel
  int16_t lev;        // cells of 2^lev voxels per axis
  int16_t ncell;      // 1, 2 or 4 sibling cells, consecutive in Morton order (one box)
};

// box of a unit: ncell aligned siblings of 2^lev cells; 2 spans x, 4 spans x and y
__device__ __forceinline__ void unit_box(int lev, int ncell, int32_t sz[3]) {
  sz[0] = (ncell >= 2 ? 2 : 1) << lev;
  sz[1] = (ncell >= 4 ? 2 : 1) << lev;
  sz[2] = 1 << lev;
}

// Per tile (one block each): walk the octant tree depth first in Morton order and count (PASS 0)
// or write (PASS 1) the units.  A cell whose candidates exceed the unit budget is split; among its
// eight children, aligned groups of four or two siblings whose candidates fit together become
// one unit, the others single-cell units or further splits.  A single voxel is always a unit
// (summed in streaming order when it holds more than the budget).
namespace {
enum { kEntUnit = 0, kEntSplit = 1 };
struct PlanEntry {
  int32_t o[3];
  int16_t lev, ncell, kind, pad;
  int64_t cand;
};
}  // namespace

template <int PASS, class Key>
__global__ void __launch_bounds__(kBlock) k_unit_plan(const ulonglong2* __restrict__ box,
                                                      const Key* __restrict__ rkeys,
                                                      const uint32_t* __restrict__ rprim,
                                                      const int64_t* __restrict__ tstart,
                                                      const int64_t* __restrict__ ctl, int tb, int batch,
                                                      int64_t budget, int64_t* __restrict__ ucnt,
                                                      const int64_t* __restrict__ uoff, Unit* __restrict__ units) {
  __shared__ PlanEntry stk[48];
  __shared__ PlanEntry g[8];                         // one split's groups, before they are pushed
  __shared__ int64_t csum[8];
  __shared__ int64_t tmp[kWaves + 1];
  __shared__ int32_t s_top;
  const int64_t n_tiles = ctl[CTL_N_TILES];
  if (PASS == 1 && ctl[CTL_N_UNITS] == 0) return;
  // tile coordinates: the Morton bits below the patch id (batched) or the whole key
  const uint64_t lowmask = batch ? (uint64_t(1) << (kPatchShift - 3 * tb)) - 1 : ~uint64_t(0);
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int64_t s = tstart[t], e = tstart[t + 1];
    const uint64_t tk = uint64_t(rkeys[s]) & lowmask;
    const int32_t to[3] = {int32_t(compact3(tk)) << tb, int32_t(compact3(tk >> 1)) << tb,
                           int32_t(compact3(tk >> 2)) << tb};
    if (PASS == 1) {
      // a tile that is one unit as a whole: its candidate count came with the count pass
      const int64_t wc = ucnt[t] >> 32;
      if (wc > 0) {
        if (threadIdx.x == 0 && wc > 1) {
          Unit u;
          u.tile = t;
          u.cand = wc - 1;
          u.o[0] = to[0];
          u.o[1] = to[1];
          u.o[2] = to[2];
          u.lev = int16_t(tb);
          u.ncell = 1;
          units[uoff[t]] = u;
        }
        continue;
      }
    }
    // the whole tile
    int64_t c = 0;
    for (int64_t j = s + threadIdx.x; j < e; j += kBlock) {
      const int32_t sz[3] = {1 << tb, 1 << tb, 1 << tb};
      c += clip_packed(box[rprim[j]], to, sz);
    }
    c = block_sum(c, tmp);
    if (threadIdx.x == 0) {
      PlanEntry r;
      r.o[0] = to[0];
      r.o[1] = to[1];
      r.o[2] = to[2];
      r.lev = int16_t(tb);
      r.ncell = 1;
      r.kind = (c <= budget || tb == 0) ? kEntUnit : kEntSplit;
      r.cand = c;
      stk[0] = r;
      s_top = 1;
    }
    __syncthreads();
    int64_t nu = 0;
    int64_t out = PASS == 1 ? uoff[t] : 0;
    while (s_top > 0) {
      const PlanEntry E = stk[s_top - 1];
      __syncthreads();                               // everyone has read the top before it changes
      if (E.kind == kEntUnit) {
        if (threadIdx.x == 0) {
          s_top = s_top - 1;
          if (PASS == 1 && E.cand > 0) {
            Unit u;
            u.tile = t;
            u.cand = E.cand;
            u.o[0] = E.o[0];
            u.o[1] = E.o[1];
            u.o[2] = E.o[2];
            u.lev = E.lev;
            u.ncell = E.ncell;
            units[out] = u;
          }
        }
        if (E.cand > 0) {
          ++nu;
          ++out;
        }
        __syncthreads();
        continue;
      }
      // split: candidates of the eight children in one pass (halves per axis)
      const int32_t h = 1 << (E.lev - 1);
      if (threadIdx.x < 8) csum[threadIdx.x] = 0;
      __syncthreads();
      int64_t cc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      for (int64_t j = s + threadIdx.x; j < e; j += kBlock) {
        int32_t bl[3], bh[3];
        unpack_box(box[rprim[j]], bl, bh);
        int64_t nh[3][2];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const int32_t l = bl[a], hh = bh[a];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int32_t c0 = E.o[a] + q * h, c1 = c0 + h - 1;
            const int32_t lo = l > c0 ? l : c0, hi = hh < c1 ? hh : c1;
            nh[a][q] = hi >= lo ? hi - lo + 1 : 0;
          }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) cc[k] += nh[0][k & 1] * nh[1][(k >> 1) & 1] * nh[2][k >> 2];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int64_t v = wave_sum(cc[k]);
        if (lane_id() == 0) atomicAdd(reinterpret_cast<unsigned long long*>(&csum[k]), (unsigned long long)v);
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        int top = s_top - 1;                          // pop the split entry
        // groups in Morton order, pushed in reverse so that they pop in order
        int ng = 0;
        auto child = [&](int k, int ncell, int64_t cnt, int kind) {
          PlanEntry r;
          r.o[0] = E.o[0] + ((k & 1) ? h : 0);
          r.o[1] = E.o[1] + ((k & 2) ? h : 0);
          r.o[2] = E.o[2] + ((k & 4) ? h : 0);
          r.lev = int16_t(E.lev - 1);
          r.ncell = int16_t(ncell);
          r.kind = int16_t(kind);
          r.cand = cnt;
          g[ng++] = r;
        };
        for (int q = 0; q < 8; q += 4) {
          const int64_t s4 = csum[q] + csum[q + 1] + csum[q + 2] + csum[q + 3];
          if (s4 <= budget) {
            child(q, 4, s4, kEntUnit);
            continue;
          }
          for (int pp = q; pp < q + 4; pp += 2) {
            const int64_t s2 = csum[pp] + csum[pp + 1];
            if (s2 <= budget) {
              child(pp, 2, s2, kEntUnit);
              continue;
            }
            for (int k = pp; k < pp + 2; ++k)
              child(k, 1, csum[k], (csum[k] <= budget || E.lev - 1 == 0) ? kEntUnit : kEntSplit);
          }
        }
        for (int i = ng - 1; i >= 0; --i) stk[top++] = g[i];
        s_top = top;
      }
      __syncthreads();
    }
    // units per tile (low half); a tile that is one unit as a whole also keeps its candidate
    // count plus one (high half), so that the writing pass skips it
    if (PASS == 0 && threadIdx.x == 0)
      ucnt[t] = nu | ((c <= budget || tb == 0) && c < (int64_t(1) << 30) ? (c + 1) << 32 : 0);
    __syncthreads();
  }
}

struct UnitTotal {
  int64_t* off;
  int64_t* ctl;
  int64_t* stats;
  int64_t cap;
  __device__ void operator()(int64_t total, int64_t n) const {
    off[n] = total;
    stats[VX_STAT_UNITS] = total;
    const bool over = total > cap;
    if (over) flag_set(stats, VX_FLAG_UNIT_CAPACITY);
    ctl[CTL_N_UNITS] = over ? 0 : total;
  }
};

// ---------------------------------------------------------------------------------------------
// the unit kernel: test, weigh, group by voxel and sum in LDS
// ---------------------------------------------------------------------------------------------
struct UnitLds {
  uint16_t* key;      // [budget]   unit-local Morton code of each pair
  float* w;           // [budget]
  uint32_t* prim;     // [budget]
  uint16_t* ckey;     // [budget]   per candidate of the batch: kTouch | its unit-local key,
                      // kUndecided, or 0 for a miss
  uint16_t* queue;    // [budget]   triangles: the batch's undecided candidates, in the space of idx
                      // (fibers: in that of w, past the weights of the pairs so far)
  uint16_t* idx;      // [budget]   triangles: the slots of a batch's new pairs; after the batches:
                      // grouped order -> pair (fibers: in the space of ckey)
  uint64_t* kbits;    // [64] one-wave blocks: bit k set where a pair of key k was found
  uint64_t* sbm;      // [64] batch: bit c set where a slot's first candidate is c
  uint32_t* spre;     // [64] slot starts below each word
  int32_t* brec;      // [threads][9] the slot's primitive vertices (record words 0..8; fibers: words
                      // 0..5 and the segment's length; after the batches: the counters, then starts)
  // the current record batch; after the batches its space holds the voxels' keys
  double* binv;       // [threads] fibers: the slot's 1 / |B - A|^2 (lattice units); triangles:
                      // tri_area_under's factor from projected to true area
  int32_t* bprim;     // [threads]
  uint32_t* bbox;     // [threads] the slot's candidate box in the unit (pack_slot_box)
  int32_t* boff;      // [threads] candidate offsets within the batch
  int32_t* bpatch;    // [threads] the slot's patch (batched fibers); triangles: tri_area_under's `how`
  uint16_t* vkey;     // [budget]
  int32_t* tmp32;     // [kWaves + 1]
  int32_t* misc;      // [8]
};

// above this many pairs per voxel (unit mean) the grouping places stably instead of sorting
// (triangles: a surface voxel holds a handful of pairs, sorted per voxel in parallel faster than
// one wave places them in order; fibers: dense patches hold hundreds per voxel)
template <int KIND>
constexpr int32_t stable_mean() { return KIND == 0 ? 24 : 4; }
// keys of a unit's range: at most one 16^3 tile
constexpr int32_t kUnitKeys = 4096;

// a candidate's outcome and key in one 16-bit word (keys below 4096)
constexpr uint16_t kTouch = 0x8000, kUndecided = 0x4000;
static_assert(kUnitKeys <= kUndecided, "keys fit below the flags");

// LDS of a unit with a budget of CAND candidates, and the unit kernel's waves per SIMD that the LDS
// then allows (160 KB per CU: 4 blocks at 1024 and 1536; above, 3, but 2 for triangles at 3072).
// Much of a unit's time is latency (dependent loads, barriers, LDS), so another block per CU is worth
// more than the registers it takes.  With packed boxes, shared space and the arrival slots in registers
// the brushed surface's units (1536) went from 49 to 38 KB and 6.43 to 5.75 ms, a fabric's (3072) from
// 77 to 53 KB and 0.68 to 0.50 ms.
template <int KIND, int CAND, int NT = kBlock>
constexpr size_t unit_lds_bytes() {
  constexpr size_t batch = NT * (8 + 4 * 4) > CAND * 2 ? NT * (8 + 4 * 4) : CAND * 2;
  return size_t(CAND) * (2 + 4 + 4 + 2 + (KIND == 0 ? 2 : 0)) + 64 * 8 + (NT == 64 ? 64 * 8 : 0) + 64 * 4 + NT * 9 * 4 +
         batch + (NT / 64 + 2) * 4 + 8 * 4;
}
template <int KIND>
constexpr int unit_waves(int cand) {
  return cand <= 1536 ? 4 : (KIND == 1 || cand <= 2048 ? 3 : 2);
}
static_assert(2 * unit_lds_bytes<0, 3072>() <= 160 * 1024, "two units per CU");
static_assert(3 * unit_lds_bytes<0, 2048>() <= 160 * 1024, "three units per CU");
static_assert(4 * unit_lds_bytes<0, 1536>() <= 160 * 1024, "four units per CU");
static_assert(3 * unit_lds_bytes<1, 3072>() <= 160 * 1024, "three units per CU");
static_assert(4 * unit_lds_bytes<1, 1536>() <= 160 * 1024, "four units per CU");

// Small units (fibers), a wave each: four waves take a unit of a hundred candidates no faster than one
// does, since all that they do is wait.  The four waves of a block claim their staging ranges
// together: single claims, all on one counter, come 16 ns apart at best.  A strand's 6,300 units: 65
// us; by blocks of four waves 102 us, by single waves with claims of their own 99 us.
constexpr int kSmallCand = 384;
constexpr size_t small_lds_bytes() { return (unit_lds_bytes<1, kSmallCand, 64>() + 15) / 16 * 16; }
static_assert(4 * (kWaves * small_lds_bytes() + 64) <= 160 * 1024, "sixteen small units per CU");

// barriers and scans of the threads that share a unit: a block, or one wave of it (NT = 64)
template <int NT>
__device__ __forceinline__ void unit_sync() {
  if (NT == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}
template <int NT>
__device__ __forceinline__ int32_t unit_scan(int32_t v, int32_t* tmp, int32_t& total) {
  if constexpr (NT == 64) {
    const int32_t inc = wave_inclusive_scan(v);
    total = __builtin_amdgcn_readlane(inc, 63);
    return inc - v;
  } else {
    return block_exclusive_scan(v, tmp, total);
  }
}

template <int KIND, int CAND, int NT>
__device__ __forceinline__ UnitLds carve_unit_lds(char* base) {
  UnitLds L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base + off;
    off += (bytes + 7) & ~size_t(7);
    return p;
  };
  L.kbits = reinterpret_cast<uint64_t*>(take(NT == 64 ? 64 * 8 : 0));
  L.sbm = reinterpret_cast<uint64_t*>(take(64 * 8));
  char* batch = take(NT * (8 + 4 * 4) > CAND * 2 ? NT * (8 + 4 * 4) : CAND * 2);
  L.binv = reinterpret_cast<double*>(batch);
  L.bprim = reinterpret_cast<int32_t*>(batch + NT * 8);
  L.bbox = reinterpret_cast<uint32_t*>(batch + NT * 12);
  L.boff = reinterpret_cast<int32_t*>(batch + NT * 16);
  L.bpatch = reinterpret_cast<int32_t*>(batch + NT * 20);
  L.vkey = reinterpret_cast<uint16_t*>(batch);
  L.w = reinterpret_cast<float*>(take(CAND * 4));
  L.prim = reinterpret_cast<uint32_t*>(take(CAND * 4));
  L.key = reinterpret_cast<uint16_t*>(take(CAND * 2));
  L.ckey = reinterpret_cast<uint16_t*>(take(CAND * 2));
  L.idx = KIND == 0 ? reinterpret_cast<uint16_t*>(take(CAND * 2)) : L.ckey;
  L.queue = L.idx;
  L.spre = reinterpret_cast<uint32_t*>(take(64 * 4));
  L.brec = reinterpret_cast<int32_t*>(take(NT * 9 * 4));
  L.tmp32 = reinterpret_cast<int32_t*>(take((NT / 64 + 1) * 4));
  L.misc = reinterpret_cast<int32_t*>(take(8 * 4));
  return L;
}

// A slot's candidate box in the unit: first voxel from the unit's (4 bits per axis), extents less
// one along x and y (units span at most 16 voxels per axis)
__device__ __forceinline__ uint32_t pack_slot_box(const int32_t o[3], const int32_t lo[3], const int32_t n[3]) {
  return uint32_t(lo[0] - o[0]) | (uint32_t(lo[1] - o[1]) << 4) | (uint32_t(lo[2] - o[2]) << 8) |
         (uint32_t(n[0] - 1) << 12) | (uint32_t(n[1] - 1) << 16);
}

// Load records [j0, j0 + NT) (NT: threads of the block) of the tile clipped to the unit box, keeping those with
// candidates in it (compacted, in record order, with a copy of their vertices); returns the
// batch's candidate total and the number of slots kept.  Contains __syncthreads().
template <int KIND, int NT>
__device__ __forceinline__ int32_t load_batch(const UnitLds& S, const int32_t* __restrict__ rec,
                                              const uint32_t* __restrict__ rprim, const float4* __restrict__ dirs,
                                              int64_t j0, int64_t e, int Sb,
                                              const int32_t o[3], const int32_t sz[3], int& nslot) {
  const int tid = threadIdx.x % NT;
  const int64_t j = j0 + tid;
  int32_t c = 0, lo[3], n[3];
  uint32_t p = 0;
  // the whole record (and the triangle's normal and doubled area) in registers at once: one round
  // of loads after the primitive id, none after the scan below
  int32_t r[kRec];
  float4 dir = make_float4(0.f, 0.f, 0.f, 0.f);
  if (tid < 64) S.sbm[tid] = 0;
  if (j < e) {
    p = rprim[j];
    const int4* r4 = reinterpret_cast<const int4*>(rec + int64_t(p) * kRec);
#pragma unroll
    for (int k = 0; k < kRec / 4; ++k) {
      const int4 v = r4[k];
      r[4 * k] = v.x;
      r[4 * k + 1] = v.y;
      r[4 * k + 2] = v.z;
      r[4 * k + 3] = v.w;
    }
    if (KIND == 0) dir = dirs[p];
    else dir.w = dirs[p].w;
    c = int32_t(clip_box(r, o, sz, lo, n));
  }
  // candidates (below 2^21 per batch) and kept slots (bits 21 and up) in one scan
  int32_t tot;
  const int32_t ex = unit_scan<NT>(c | (c > 0 ? (1 << 21) : 0), S.tmp32, tot);
  if (c > 0) {
    const int q = ex >> 21;
    const int32_t off = ex & ((1 << 21) - 1);
    S.bprim[q] = int32_t(p);
    S.boff[q] = off;
    S.bbox[q] = pack_slot_box(o, lo, n);
#pragma unroll
    for (int k = 0; k < (KIND == 0 ? 9 : 6); ++k) S.brec[q * 9 + k] = r[k];
    if (KIND == 1) {
      S.bpatch[q] = r[15];
      S.brec[q * 9 + 6] = __float_as_int(dir.w);
      S.binv[q] = cap_inv_len2(r);
    } else {
      uint32_t how;
      double scale;
      tri_area_setup(r, dir, Sb, how, scale);
      S.bpatch[q] = int32_t(how);
      S.binv[q] = scale;
    }
    atomicOr(reinterpret_cast<unsigned long long*>(&S.sbm[off >> 6]), 1ull << (off & 63));
  }
  nslot = tot >> 21;
  unit_sync<NT>();
  if (tid < 64) {
    const uint32_t cnt = uint32_t(__popcll(S.sbm[tid]));
    const uint32_t inc = wave_inclusive_scan(cnt);
    S.spre[tid] = inc - cnt;
  }
  unit_sync<NT>();
  return tot & ((1 << 21) - 1);
}

// voxel of candidate li (x fastest) of the record in batch slot `slot`.  li < 16^3 and extents
// <= 16: the quotients by float reciprocal are exact (the rounding error, below 1e-3, stays
// under the 1/32 margin of (li + 1/2) / n to the next integer)
__device__ __forceinline__ void slot_voxel(const UnitLds& S, const int32_t o[3], int slot, int32_t li, int32_t v[3]) {
  const uint32_t box = S.bbox[slot];
  const int32_t nx = int32_t((box >> 12) & 15u) + 1, ny = int32_t((box >> 16) & 15u) + 1;
  const int32_t t = int32_t((float(li) + 0.5f) * __builtin_amdgcn_rcpf(float(nx)));
  const int32_t iz = int32_t((float(t) + 0.5f) * __builtin_amdgcn_rcpf(float(ny)));
  v[0] = o[0] + int32_t(box & 15u) + (li - t * nx);
  v[1] = o[1] + int32_t((box >> 4) & 15u) + (t - iz * ny);
  v[2] = o[2] + int32_t((box >> 8) & 15u) + iz;
}

// candidate c (< 4096) of the batch -> its record slot: the slot starts at or below c, less one
__device__ __forceinline__ int find_slot(const UnitLds& S, int32_t c) {
  const int wd = c >> 6;
  return int(S.spre[wd] + uint32_t(__popcll(S.sbm[wd] & ((2ull << (c & 63)) - 1)))) - 1;
}

// A voxel's Morton code within its aligned 16^3 cell (12 bits) and back: units and tiles lie in one
// such cell, so differences of these codes are differences of the whole keys.
__device__ __forceinline__ uint32_t spread4(uint32_t x) {
  x = (x | (x << 4)) & 0x0c3u;
  return (x | (x << 2)) & 0x249u;
}
__device__ __forceinline__ uint32_t cell_code(const int32_t v[3]) {
  return spread4(uint32_t(v[0]) & 15u) | (spread4(uint32_t(v[1]) & 15u) << 1) | (spread4(uint32_t(v[2]) & 15u) << 2);
}
__device__ __forceinline__ int32_t compact4(uint32_t x) {
  x &= 0x249u;
  x = (x | (x >> 2)) & 0x0c3u;
  return int32_t((x | (x >> 4)) & 15u);
}
__device__ __forceinline__ void cell_voxel(const int32_t o[3], uint32_t code, int32_t v[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) v[a] = (o[a] & ~15) | compact4(code >> a);
}

__device__ __forceinline__ float fib_weight(const int32_t* r, const int32_t v[3], int Sb, float len) {
  const int64_t w[3] = {v[0], v[1], v[2]};
  return seg_length(r, w, Sb, len);
}
// out of line: the rare streaming path keeps no second copy of the weight code
__device__ __attribute__((noinline)) float fib_weight_call(const int32_t* r, int32_t v0, int32_t v1, int32_t v2,
                                                           int Sb, float len) {
  const int32_t v[3] = {v0, v1, v2};
  return fib_weight(r, v, Sb, len);
}
__device__ __attribute__((noinline)) float tri_weight_call(const int32_t* r, int32_t v0, int32_t v1, int32_t v2,
                                                           int Sb, uint32_t how, double scale) {
  const int32_t v[3] = {v0, v1, v2};
  return tri_area_under(r, v, Sb, how, scale);
}

// does a vertex of the triangle lie in the closed box?  Decides about half the candidates of
// voxel-sized triangles (a box that holds a vertex is touched) with integer compares
__device__ __forceinline__ bool tri_vertex_in(const int32_t* r, const int32_t v[3], int Sb) {
  const uint32_t s = 1u << Sb;
  bool any = false;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) in = in & (uint32_t(r[3 * i + a] - (v[a] << Sb)) <= s);
    any = any | in;
  }
  return any;
}

// Staging of a unit's voxels (SoA, capacity cap); units claim contiguous ranges in any order.
struct Stage {
  void* key;          // u64, or u32 where the leaf's keys are 32-bit
  int key64;
  uint32_t* count;
  float* w;
  float* S;           // [6][cap]
  int64_t cap;
};

template <int KIND>
__device__ __forceinline__ void write_voxel(const Stage& st, int64_t i, uint64_t key, uint32_t cnt, const Moment& m) {
  if (st.key64) static_cast<uint64_t*>(st.key)[i] = key;
  else static_cast<uint32_t*>(st.key)[i] = uint32_t(key);
  st.count[i] = cnt;
  st.w[i] = m.W;
  st.S[i] = m.xx;
  st.S[st.cap + i] = m.yy;
  st.S[2 * st.cap + i] = m.zz;
  st.S[3 * st.cap + i] = m.xy;
  st.S[4 * st.cap + i] = m.xz;
  st.S[5 * st.cap + i] = m.yz;
}

// Bound by VALU issue (three quarters of the cycles) and the latencies above.  The whole brushed
// surface (149 M pairs): 7.95 -> 5.97 ms with the area by integration (2.4 ms of it; 3.7 before), unit
// codes spread over 4 bits instead of 21, and half the candidates decided by a vertex in the box.
// Fibers are weighed from the records in LDS, one reciprocal an axis: 14 patches (64,000 units) 2.46 ->
// 2.21 ms, a weave (10,000 units) 0.515 -> 0.460 ms against records gathered again from memory after
// the batches and two divisions an axis.
template <int KIND, int CAND, int NT>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(unit_waves<KIND>(CAND)))) k_unit(const int32_t* __restrict__ rec, const float4* __restrict__ dirs,
                                                 const uint32_t* __restrict__ rprim,
                                                 const int64_t* __restrict__ tstart, const Unit* __restrict__ units,
                                                 const int64_t* __restrict__ ctl, Lat L, const Lat* __restrict__ lats,
                                                 int64_t* __restrict__ unv, int64_t* __restrict__ unp,
                                                 int64_t* __restrict__ usoff, Stage st, int64_t* stage_ctr,
                                                 int64_t* stats, int small) {
  extern __shared__ double lds_dyn[];
  constexpr int kW = NT / 64;
  constexpr bool kOne = NT == 64;                     // a unit of up to CAND candidates per wave
  constexpr int kAtOnce = kBlock / NT;                // units in flight in the block
  static_assert(CAND <= 0xffff, "pair positions are 16-bit");
  static_assert(CAND % (kW * 64) == 0, "each wave's queue holds all of its candidates");
  char* const lds = reinterpret_cast<char*>(lds_dyn);
  const UnitLds S = carve_unit_lds<KIND, CAND, NT>(kOne ? lds + (threadIdx.x / NT) * small_lds_bytes() : lds);
  int64_t* const claims = reinterpret_cast<int64_t*>(lds + kWaves * small_lds_bytes());   // [kWaves + 1] (kOne)
  const int64_t n_units = ctl[CTL_N_UNITS];
  const int tid = threadIdx.x % NT;
  // the four waves' claims together; all waves of the block call it once a round, from one place
  const auto claim_together = [&](int32_t nv) -> int64_t {
    const int wv = threadIdx.x / 64;
    if (tid == 0) claims[wv] = nv;
    __syncthreads();
    if (threadIdx.x == 0) {
      int64_t all = 0;
      for (int i = 0; i < kWaves; ++i) {
        const int64_t n = claims[i];
        claims[i] = all;
        all += n;
      }
      claims[kWaves] = all ? int64_t(atomicAdd(reinterpret_cast<unsigned long long*>(stage_ctr), (unsigned long long)all))
                           : 0;
    }
    __syncthreads();
    return claims[kWaves] + claims[wv];               // (the next round's first barrier comes after this read)
  };
  for (int64_t u0 = int64_t(blockIdx.x) * kAtOnce; u0 < n_units; u0 += int64_t(gridDim.x) * kAtOnce) {
    // (a wave's index by readfirstlane: uniform, and so is all that hangs on it.)  A wave that has no
    // small unit this round walks through with an empty one, so that the block's barriers stand where
    // all four waves pass
    const int64_t u = kOne ? u0 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : u0;
    const Unit U = units[u < n_units ? u : u0];
    if (!kOne && U.cand <= small) continue;           // (small: what single waves take, 0: none)
    const bool live = !kOne || (u < n_units && U.cand <= CAND);
    const int64_t s = live ? tstart[U.tile] : 0, e = live ? tstart[U.tile + 1] : 0;
    int32_t usz[3];
    unit_box(U.lev, U.ncell, usz);
    const uint64_t m0 = morton3(uint32_t(U.o[0]), uint32_t(U.o[1]), uint32_t(U.o[2]));   // the unit's first key
    const uint32_t c0 = uint32_t(m0) & 4095u;                                              // its code in the cell
    const bool stream = !kOne && U.cand > CAND;          // a single voxel holding too many candidates
    int32_t np = 0;                                   // pairs so far (uniform)
    if (kOne) S.kbits[tid] = 0;                       // (the batch's barriers come before the first pair)
    Moment acc{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // streaming sums (thread 0)
    uint32_t acc_n = 0;
    for (int64_t j0 = s; j0 < e; j0 += NT) {
      int nb;
      const int32_t cb = load_batch<KIND, NT>(S, rec, rprim, dirs, j0, e, L.Sb, U.o, usz, nb);
      (void)nb;
      if (stream) {
        for (int32_t b0 = 0; b0 < cb; b0 += NT) {
          const int32_t c = b0 + tid;
          bool hit = false;
          float wgt = 0.f;
          uint32_t p = 0;
          if (c < cb) {
            const int slot = find_slot(S, c);
            int32_t v[3];
            slot_voxel(S, U.o, slot, c - S.boff[slot], v);
            const int64_t vl[3] = {v[0], v[1], v[2]};
            p = uint32_t(S.bprim[slot]);
            const int32_t* r = S.brec + slot * 9;
            if (KIND == 0) {
              hit = tri_touch(r, vl, L.s, L.Sb);
              if (hit) wgt = tri_weight_call(r, v[0], v[1], v[2], L.Sb, uint32_t(S.bpatch[slot]), S.binv[slot]);
            } else {
              const LatQ Lp = lat_q(lats, S.bpatch[slot], L);
              hit = cap_touch(r, vl, Lp.s, Lp.Sb, Lp.rho);
              if (hit) wgt = fib_weight_call(r, v[0], v[1], v[2], Lp.Sb, dirs[p].w);
            }
          }
          int32_t tot;
          const int32_t pos = unit_scan<NT>(int32_t(hit), S.tmp32, tot);
          // one voxel: sum this chunk's hits in order (thread 0), chunk by chunk
          if (hit) {
            S.w[pos] = wgt;
            S.prim[pos] = p;
          }
          unit_sync<NT>();
          if (tid == 0) {
            for (int32_t i = 0; i < tot; ++i) accum_pair<KIND>(acc, S.w[i], dirs[S.prim[i]]);
            acc_n += uint32_t(tot);
          }
          np += tot;
          unit_sync<NT>();
        }
        continue;
      }
      // Test in two rounds so that lanes stay busy: a cheap filter decides most candidates and
      // queues the rest (fibers: the centre-ball filter; triangles: a vertex in the box), then the
      // queue gets the full test.
      // Each wave works on its own candidates and drains its own queue (fibers: 16-bit entries from the
      // first free weight on; the pairs so far and the batch's candidates are within the budget, and
      // the four waves' rounded-up shares within twice the batch's, or its last); every candidate records
      // its outcome in place, and the touching ones are then compacted in candidate order,
      // which is primitive order.
      const int wv = tid >> 6, lane = tid & 63;
      const uint64_t lt = (uint64_t(1) << lane) - 1;
      uint16_t* wq = KIND == 0 ? S.queue + wv * (CAND / kW)
                               : reinterpret_cast<uint16_t*>(S.w + (np < CAND - cb ? np : CAND - cb)) +
                                     wv * 64 * ((cb + NT - 1) / NT);
      int32_t nq = 0;                                  // this wave's queue (uniform)
      for (int32_t b0 = wv * 64; b0 < cb; b0 += NT) {
        const int32_t c = b0 + lane;
        int res = 0;                                   // 0 miss, 1 touch, 2 undecided
        if (c < cb) {
          const int slot = find_slot(S, c);
          int32_t v[3];
          slot_voxel(S, U.o, slot, c - S.boff[slot], v);
          const int32_t* r = S.brec + slot * 9;
          if (KIND == 0) {
            res = tri_vertex_in(r, v, L.Sb) ? 1 : 2;
          } else {
            const LatQ Lp = lat_q(lats, S.bpatch[slot], L);
            const int64_t vl[3] = {v[0], v[1], v[2]};
            const int b = cap_ball(r, vl, Lp.s, Lp.Sb, Lp.rho, S.binv[slot]);
            res = b < 0 ? 2 : b;
          }
          S.ckey[c] = res == 1 ? uint16_t(kTouch | (cell_code(v) - c0)) : (res == 2 ? kUndecided : uint16_t(0));
        }
        const uint64_t mb = __ballot(res == 2);
        if (res == 2) wq[nq + int32_t(__popcll(mb & lt))] = uint16_t(c);
        nq += int32_t(__popcll(mb));
      }
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      for (int32_t q = lane; q < nq; q += 64) {
        const int32_t c = int32_t(wq[q]);
        const int slot = find_slot(S, c);
        int32_t v[3];
        slot_voxel(S, U.o, slot, c - S.boff[slot], v);
        const int64_t vl[3] = {v[0], v[1], v[2]};
        const int32_t* r = S.brec + slot * 9;
        bool hit;
        if (KIND == 0) {
          hit = tri_touch(r, vl, L.s, L.Sb);
        } else {
          const LatQ Lp = lat_q(lats, S.bpatch[slot], L);
          hit = cap_bracket(r, vl, Lp.s, Lp.Sb, Lp.rho);
        }
        S.ckey[c] = hit ? uint16_t(kTouch | (cell_code(v) - c0)) : uint16_t(0);
      }
      unit_sync<NT>();
      // ordered compaction: wave w takes candidates [w span, (w + 1) span)
      {
        const int32_t span = ((cb + kW * 64 - 1) / (kW * 64)) * 64;
        const int32_t w0 = wv * span, w1 = w0 + span < cb ? w0 + span : cb;
        int32_t cnt = 0;
        for (int32_t b0 = w0; b0 < w1; b0 += 64) {
          const int32_t c = b0 + lane;
          cnt += int32_t(__popcll(__ballot(c < w1 && (S.ckey[c] & kTouch) != 0)));
        }
        if (lane == 0) S.tmp32[wv] = cnt;
        unit_sync<NT>();
        int32_t base = np, tot = 0;
        for (int i = 0; i < kW; ++i) {
          if (i < wv) base += S.tmp32[i];
          tot += S.tmp32[i];
        }
        for (int32_t b0 = w0; b0 < w1; b0 += 64) {
          const int32_t c = b0 + lane;
          const bool hit = c < w1 && (S.ckey[c] & kTouch) != 0;
          const uint64_t mh = __ballot(hit);
          if (hit) {
            const int32_t q = base + int32_t(__popcll(mh & lt));
            if (q < CAND) {
              const int sl = find_slot(S, c);
              const uint32_t key = S.ckey[c] & (kTouch - 1u);
              S.key[q] = uint16_t(key);
              if (kOne) atomicOr(reinterpret_cast<uint32_t*>(S.kbits) + (key >> 5), 1u << (key & 31u));
              if (KIND == 0) {
                S.prim[q] = uint32_t(S.bprim[sl]);
                S.idx[q] = uint16_t(sl);
              } else {
                S.prim[q] = uint32_t(sl);             // until the pair is weighed
              }
            } else {
              flag_set(stats, VX_FLAG_UNIT_CAPACITY);   // planning and test disagree: never expected
            }
          }
          base += int32_t(__popcll(mh));
        }
        // the batch's pairs are weighed now, from the records still in LDS
        unit_sync<NT>();
        const int32_t q1 = np + tot < CAND ? np + tot : CAND;
        for (int32_t q = np + tid; q < q1; q += NT) {
          const int sl = KIND == 0 ? int(S.idx[q]) : int(S.prim[q]);
          const int32_t* r = S.brec + sl * 9;
          int32_t v[3];
          cell_voxel(U.o, c0 + S.key[q], v);
          if (KIND == 0) {
            S.w[q] = tri_area_under(r, v, L.Sb, uint32_t(S.bpatch[sl]), S.binv[sl]);
          } else {
            S.w[q] = fib_weight(r, v, lat_q(lats, S.bpatch[sl], L).Sb, __int_as_float(r[6]));
            S.prim[q] = uint32_t(S.bprim[sl]);
          }
        }
        np += tot;
        unit_sync<NT>();
      }
    }
    if (stream) {
      if (tid == 0) {
        const int64_t nv = acc_n > 0 ? 1 : 0;
        int64_t b = 0;
        if (nv) {
          b = int64_t(atomicAdd(reinterpret_cast<unsigned long long*>(stage_ctr), 1ull));
          const uint64_t key = morton3(uint32_t(U.o[0]), uint32_t(U.o[1]), uint32_t(U.o[2])) |
                               (lats ? uint64_t(uint32_t(rec[int64_t(rprim[s]) * kRec + 15])) << kPatchShift : 0ull);
          if (b < st.cap) write_voxel<KIND>(st, b, key, acc_n, acc);
          else flag_set(stats, VX_FLAG_VOXEL_CAPACITY);
        }
        unv[u] = nv;
        unp[u] = np;
        usoff[u] = b;
      }
      unit_sync<NT>();
      continue;
    }
    const int32_t npairs = np < CAND ? np : CAND;
    // Group the pairs by voxel with one counter per key of the unit's range (at most 4096 keys;
    // 16-bit counts packed two to a word, in the record batch's space, dead now).  Each pair's
    // arrival slot among its voxel's pairs stays in its thread's registers until it is placed.
    // One-wave blocks have room for a counter per voxel only: a key's rank among the unit's keys, by
    // the bits set as the pairs were found, numbers its voxel and takes the key's place with the pair.
    // (In the large units those bits and ranks cost more than 4096 counters: a weave 0.91 ms, 0.89.)
    uint32_t* kcw = reinterpret_cast<uint32_t*>(S.brec);                 // packed counts
    uint16_t* kst = reinterpret_cast<uint16_t*>(S.brec);                 // then starts, by key or voxel
    uint16_t* vkey = S.vkey;                                             // [nv] key of voxel v
    uint32_t slot[CAND / NT];
    int32_t nv;
    if constexpr (kOne) {
      static_assert(NT * 9 * 4 >= CAND * 2, "the voxels' counters live in the record batch's space");
      const int32_t bits = int32_t(__popcll(S.kbits[tid]));
      const int32_t upto = wave_inclusive_scan(bits);
      nv = __builtin_amdgcn_readlane(upto, 63);
      for (int32_t j = tid; j < (nv + 1) / 2; j += NT) kcw[j] = 0u;
      unit_sync<NT>();
#pragma unroll
      for (int q = 0; q < CAND / NT; ++q) {
        const int32_t i = tid + q * NT;
        slot[q] = 0;
        if (q * NT >= npairs) continue;               // (uniform)
        const uint32_t k = i < npairs ? S.key[i] : 0u;
        const uint32_t pre = uint32_t(__shfl(upto - bits, int(k >> 6), 64));
        if (i < npairs) {
          const uint32_t v = pre + uint32_t(__popcll(S.kbits[k >> 6] & ((1ull << (k & 63)) - 1)));
          const uint32_t sh = 16u * (v & 1u);
          slot[q] = (atomicAdd(&kcw[v >> 1], 1u << sh) >> sh) & 0xffffu;
          S.key[i] = uint16_t(v);
          if (slot[q] == 0) vkey[v] = uint16_t(k);
        }
      }
      unit_sync<NT>();
      // starts: lane t owns `own` voxels (whole words) from own * t on
      const int32_t own = 2 * ((nv + 2 * NT - 1) / (2 * NT)), w0 = tid * own / 2;
      uint32_t sum = 0;
      for (int32_t j = 0; j < own / 2; ++j) {
        const uint32_t n2 = 2 * (w0 + j) < nv ? kcw[w0 + j] : 0u;
        sum += (n2 & 0xffffu) + (n2 >> 16);
      }
      uint32_t at = wave_inclusive_scan(sum) - sum;
      for (int32_t j = 0; j < own / 2 && 2 * (w0 + j) < nv; ++j) {
        const uint32_t n2 = kcw[w0 + j];
        kcw[w0 + j] = at | (at + (n2 & 0xffffu)) << 16;
        at += (n2 & 0xffffu) + (n2 >> 16);
      }
    } else {
      static_assert(kOne || (NT * 9 * 4 >= kUnitKeys * 2 && NT * 16 == kUnitKeys), "sixteen keys a thread");
      for (int32_t j = tid; j < kUnitKeys / 2; j += NT) kcw[j] = 0u;
      unit_sync<NT>();
#pragma unroll
      for (int q = 0; q < CAND / NT; ++q) {
        const int32_t i = tid + q * NT;
        slot[q] = 0;
        if (i < npairs) {
          const uint32_t k = S.key[i], sh = 16u * (k & 1u);
          slot[q] = (atomicAdd(&kcw[k >> 1], 1u << sh) >> sh) & 0xffffu;
        }
      }
      unit_sync<NT>();
      // starts and the voxel list: thread t owns keys [16 t, 16 t + 16); one block scan of the
      // (pairs, voxels) counts packed in one word (at most 3072 pairs and 4096 voxels)
      {
        uint32_t c[16];
        uint32_t sp = 0, sv = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t w2 = kcw[tid * 8 + j];
          c[2 * j] = w2 & 0xffffu;
          c[2 * j + 1] = w2 >> 16;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          sp += c[k];
          sv += c[k] != 0u ? 1u : 0u;
        }
        int32_t tot;
        const uint32_t pre = uint32_t(unit_scan<NT>(int32_t(sp | (sv << 16)), S.tmp32, tot));
        nv = tot >> 16;
        uint32_t rp = pre & 0xffffu, rv = pre >> 16;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const uint32_t key = uint32_t(tid) * 16u + uint32_t(k);
          kst[key] = uint16_t(rp);
          if (c[k] != 0u) vkey[rv++] = uint16_t(key);
          rp += c[k];
        }
      }
    }
    // claim the staging range now; the claim's round trip overlaps the placement below
    int64_t b = 0;
    if constexpr (kOne) {
      b = claim_together(nv);
    } else if (tid == 0) {
      b = nv ? int64_t(atomicAdd(reinterpret_cast<unsigned long long*>(stage_ctr), (unsigned long long)nv)) : 0;
      S.misc[1] = int32_t(b & 0xffffffff);
      S.misc[2] = int32_t(b >> 32);
    }
    if (tid == 0 && live) {
      if (b + nv > st.cap) flag_set(stats, VX_FLAG_VOXEL_CAPACITY);
      unv[u] = nv;
      unp[u] = np;
      usoff[u] = b;
    }
    unit_sync<NT>();
    // Place the pairs by voxel.  Sparse units (few pairs per voxel) place by arrival slot and
    // restore primitive order per voxel by insertion sort below; dense ones place stably: one
    // wave walks the list (primitive order) and lanes holding the same key find each other by
    // ballots over the 12 key bits.
    const bool stable = npairs > stable_mean<KIND>() * nv;
    if (!stable) {
#pragma unroll
      for (int q = 0; q < CAND / NT; ++q) {
        const int32_t i = tid + q * NT;
        if (i < npairs) S.idx[kst[S.key[i]] + slot[q]] = uint16_t(i);
      }
    } else if (tid < 64) {
      const uint64_t lt = (uint64_t(1) << tid) - 1;
      for (int32_t i0 = 0; i0 < npairs; i0 += 64) {
        const int32_t i = i0 + tid;
        const bool ok = i < npairs;
        const uint32_t k = ok ? uint32_t(S.key[i]) : 0u;
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < 12; ++bit) {
          const uint64_t m = __ballot((k >> bit) & 1);
          peers &= ((k >> bit) & 1) ? m : ~m;
        }
        uint32_t q = 0;
        if (ok) q = uint32_t(kst[k]) + uint32_t(__popcll(peers & lt));
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (ok) {
          S.idx[q] = uint16_t(i);
          if ((peers & lt) == 0) kst[k] = uint16_t(kst[k] + uint32_t(__popcll(peers)));   // the group's first lane
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    unit_sync<NT>();
    if constexpr (!kOne) b = int64_t(uint32_t(S.misc[1])) | (int64_t(S.misc[2]) << 32);
    const uint64_t hi =
        lats && live ? uint64_t(uint32_t(rec[int64_t(rprim[s]) * kRec + 15])) << kPatchShift : 0ull;
    if (b + nv <= st.cap) {
      for (int32_t v = tid; v < nv; v += NT) {
        // its pairs: [start, next start), or (stably placed: the starts have run to the ends) [last
        // end, end)
        uint32_t a, z;
        if (!stable) {
          a = kst[kOne ? v : int32_t(vkey[v])];
          z = v + 1 < nv ? uint32_t(kst[kOne ? v + 1 : int32_t(vkey[v + 1])]) : uint32_t(npairs);
        } else {
          a = v ? uint32_t(kst[kOne ? v - 1 : int32_t(vkey[v - 1])]) : 0u;
          z = kst[kOne ? v : int32_t(vkey[v])];
        }
        // the voxel's pairs in list order, which is primitive order (insertion sort)
        for (uint32_t i = a + 1; !stable && i < z; ++i) {
          const uint16_t x = S.idx[i];
          uint32_t j = i;
          while (j > a && S.idx[j - 1] > x) {
            S.idx[j] = S.idx[j - 1];
            --j;
          }
          S.idx[j] = x;
        }
        Moment m{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (uint32_t i0 = a; i0 < z; i0 += 8) {
          // the loads of a group do not wait for each other, the sums stay in order.  Cleared first:
          // values that no load sets would be kept over the whole unit, and from one to the next
          // (28 registers spilled, 11 that remain at four waves per SIMD, none at three and two; the
          // brushed surface 6.07 -> 5.83 ms, 64 strands 67 -> 55 us)
          float4 t[8];
          float wv[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            t[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            wv[k] = 0.f;
            if (i0 + k < z) {
              const uint16_t x = S.idx[i0 + k];
              t[k] = dirs[S.prim[x]];
              wv[k] = S.w[x];
            }
          }
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (i0 + k < z) accum_pair<KIND>(m, wv[k], t[k]);
        }
        write_voxel<KIND>(st, b + v, hi | (m0 + vkey[v]), z - a, m);
      }
    }
    unit_sync<NT>();
  }
}

// ---------------------------------------------------------------------------------------------
// totals and the final, dense leaf
// ---------------------------------------------------------------------------------------------
struct VoxTotal {
  int64_t* pos;
  int64_t* ctl;
  int64_t* stats;
  int64_t cap;
  __device__ void operator()(int64_t total, int64_t n) const {
    pos[n] = total;
    stats[VX_STAT_VOXELS] = total;
    const bool over = total > cap;
    if (over) flag_set(stats, VX_FLAG_VOXEL_CAPACITY);
    ctl[CTL_N_VOX] = over ? 0 : total;
  }
};
struct SumTotal {
  int64_t* dst;
  __device__ void operator()(int64_t total, int64_t) const { *dst = total; }
};
struct NoOut {
  __device__ void operator()(int64_t, int64_t, int64_t) const {}
};
struct UnitCand {
  const Unit* u;
  __device__ int64_t operator()(int64_t i) const { return u[i].cand; }
};

// The three unit-level sums after the unit kernel in one two-kernel scan: totals of the pairs and
// of the candidates (statistics) and the exclusive scan of the voxels per unit (leaf positions).
// Same chunking as device_scan; partial holds 3 values per block.
__global__ void __launch_bounds__(kBlock) k_unit_sums_partial(const int64_t* __restrict__ unp,
                                                              const Unit* __restrict__ units,
                                                              const int64_t* __restrict__ unv,
                                                              const int64_t* __restrict__ ctl,
                                                              int64_t* __restrict__ partial) {
  __shared__ int64_t red[3][kWaves];
  const int64_t n = ctl[CTL_N_UNITS];
  const int64_t chunk = scan_chunk(n);
  const int64_t b0 = int64_t(blockIdx.x) * chunk;
  const int64_t b1 = b0 + chunk < n ? b0 + chunk : n;
  int64_t ap = 0, ac = 0, av = 0;
  for (int64_t i = b0 + threadIdx.x; i < b1; i += kBlock) {
    ap += unp[i];
    ac += units[i].cand;
    av += unv[i];
  }
  ap = wave_sum(ap);
  ac = wave_sum(ac);
  av = wave_sum(av);
  if (lane_id() == 0) {
    red[0][threadIdx.x >> 6] = ap;
    red[1][threadIdx.x >> 6] = ac;
    red[2][threadIdx.x >> 6] = av;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    int64_t t = 0;
    for (int i = 0; i < kWaves; ++i) t += red[threadIdx.x][i];
    partial[3 * blockIdx.x + threadIdx.x] = t;
  }
}

__global__ void __launch_bounds__(kBlock) k_unit_sums_apply(const int64_t* __restrict__ unv,
                                                            int64_t* __restrict__ ctl,
                                                            const int64_t* __restrict__ partial,
                                                            int64_t* __restrict__ upos, int64_t* __restrict__ stats,
                                                            int64_t cap) {
  __shared__ int64_t tmp[kWaves + 1];
  const int64_t n = ctl[CTL_N_UNITS];
  const int64_t chunk = scan_chunk(n);
  const int64_t b0 = int64_t(blockIdx.x) * chunk;
  const int64_t b1 = b0 + chunk < n ? b0 + chunk : n;
  int64_t pre = 0, tp = 0, tc = 0, tv = 0;
  for (int i = threadIdx.x; i < int(gridDim.x); i += kBlock) {
    const int64_t v = partial[3 * i + 2];
    if (i < int(blockIdx.x)) pre += v;
    if (blockIdx.x == 0) {
      tp += partial[3 * i];
      tc += partial[3 * i + 1];
      tv += v;
    }
  }
  int64_t base;
  (void)block_exclusive_scan(pre, tmp, base);
  if (blockIdx.x == 0) {
    int64_t t;
    (void)block_exclusive_scan(tp, tmp, t);
    if (threadIdx.x == 0) stats[VX_STAT_PAIRS] = t;
    (void)block_exclusive_scan(tc, tmp, t);
    if (threadIdx.x == 0) stats[VX_STAT_CAND] = t;
    (void)block_exclusive_scan(tv, tmp, t);
    if (threadIdx.x == 0) VoxTotal{upos, ctl, stats, cap}(t, n);
  }
  if (b0 >= b1) return;
  for (int64_t t0 = b0; t0 < b1; t0 += kBlock) {
    const int64_t i = t0 + threadIdx.x;
    const int64_t v = i < b1 ? unv[i] : 0;
    int64_t tot;
    const int64_t ex = block_exclusive_scan(v, tmp, tot);
    if (i < b1) upos[i] = base + ex;
    base += tot;
  }
}

// one block per unit: copy its staged voxels to their place in the leaf
template <class Key>
__global__ void __launch_bounds__(kBlock) k_unit_compact(const int64_t* __restrict__ unv,
                                                         const int64_t* __restrict__ usoff,
                                                         const int64_t* __restrict__ upos,
                                                         const int64_t* __restrict__ ctl, Stage st, vx_voxels out) {
  const int64_t n_units = ctl[CTL_N_UNITS];
  if (ctl[CTL_N_VOX] == 0) return;
  Key* okeys = reinterpret_cast<Key*>(out.keys);
  for (int64_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    const int64_t n = unv[u], src = usoff[u], dst = upos[u];
    for (int64_t i = threadIdx.x; i < n; i += kBlock) {
      okeys[dst + i] = static_cast<const Key*>(st.key)[src + i];
      out.count[dst + i] = st.count[src + i];
      out.w[dst + i] = st.w[src + i];
#pragma unroll
      for (int c = 0; c < 6; ++c) out.S[c * out.cap + dst + i] = st.S[c * st.cap + src + i];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// orchestration
// ---------------------------------------------------------------------------------------------
struct TileWs {
  int64_t* ctl;
  int32_t* rec;
  float4* dirs;
  int64_t* cand_cnt;
  int64_t* roff;          // [n_prims + 1]
  ulonglong2* box;        // [n_prims] packed candidate boxes
  PairBufs ra, rb;        // records (tile key, primitive; no weight), ping-pong
  int32_t* hist;
  int64_t* partial;
  int64_t* tstart;        // [max_records + 1]
  int64_t* ucnt;          // [max_records + 1] units per tile, then their offsets
  int64_t* uoff;
  Unit* units;            // [max_units]
  int64_t* unv;           // [max_units + 1]
  int64_t* unp;
  int64_t* usoff;
  int64_t* upos;          // [max_units + 1]
  int64_t* stage_ctr;
  Stage st;
};

static size_t tile_ws_layout(int64_t n_prims, int64_t max_rec, int64_t max_units, int64_t max_vox, bool key64,
                             void* base, TileWs* w) {
  Carver cv(base);
  TileWs x;
  const int kb = key64 ? 8 : 4;
  x.ctl = cv.take<int64_t>(CTL_SIZE);
  x.rec = cv.take<int32_t>(n_prims * kRec);
  x.dirs = cv.take<float4>(n_prims);
  x.cand_cnt = cv.take<int64_t>(n_prims);
  x.roff = cv.take<int64_t>(n_prims + 1);
  x.box = cv.take<ulonglong2>(n_prims);
  x.ra.keys = cv.take<uint8_t>(max_rec * kb);
  x.ra.w = nullptr;
  x.ra.prim = cv.take<uint32_t>(max_rec);
  x.rb.keys = cv.take<uint8_t>(max_rec * kb);
  x.rb.w = nullptr;
  x.rb.prim = cv.take<uint32_t>(max_rec);
  x.hist = cv.take<int32_t>(int64_t(kRadixBuckets) * kGrid);
  x.partial = cv.take<int64_t>(3 * kGrid + 1);     // 3 values per block for the unit sums
  x.tstart = cv.take<int64_t>(max_rec + 1);
  x.ucnt = cv.take<int64_t>(max_rec + 1);
  x.uoff = cv.take<int64_t>(max_rec + 1);
  x.units = cv.take<Unit>(max_units);
  x.unv = cv.take<int64_t>(max_units + 1);
  x.unp = cv.take<int64_t>(max_units + 1);
  x.usoff = cv.take<int64_t>(max_units + 1);
  x.upos = cv.take<int64_t>(max_units + 1);
  x.stage_ctr = cv.take<int64_t>(1);
  x.st.key = cv.take<uint8_t>(max_vox * kb);
  x.st.key64 = key64 ? 1 : 0;
  x.st.count = cv.take<uint32_t>(max_vox);
  x.st.w = cv.take<float>(max_vox);
  x.st.S = cv.take<float>(6 * max_vox);
  x.st.cap = max_vox;
  if (w) *w = x;
  return cv.off + 256;
}

size_t tile_ws_bytes(int64_t n_prims, int64_t max_rec, int64_t max_units, int64_t max_vox, bool key64) {
  return tile_ws_layout(n_prims, max_rec, max_units, max_vox, key64, nullptr, nullptr);
}

struct ArrIn64 {
  const int64_t* a;
  __device__ int64_t operator()(int64_t i) const { return a[i]; }
};
struct UnitCountIn {                 // units per tile: the low half of the planner's count word
  const int64_t* a;
  __device__ int64_t operator()(int64_t i) const { return a[i] & 0xffffffff; }
};
struct ArrOut64 {
  int64_t* o;
  __device__ void operator()(int64_t i, int64_t ex, int64_t) const { o[i] = ex; }
};

vx_status tile_voxelize(int kind, const vx_grid* g, const float* data, int64_t n_prims, const int64_t* offsets,
                        int64_t n_fib, float radius, int64_t max_rec, int64_t max_units, void* ws_ptr,
                        const vx_voxels* out, int64_t* stats, hipStream_t s, const BatchLattice* batch, int tb,
                        const Tuning& tu) {
  const bool key64 = batch || g->log2_res > 10;
  TileWs w;
  tile_ws_layout(n_prims, max_rec, max_units, out->cap, key64, ws_ptr, &w);
  // prep (snap, candidate boxes) is shared with the pair path
  FrontWs f{};
  f.ctl = w.ctl;
  f.rec = w.rec;
  f.dirs = w.dirs;
  f.cand_cnt = w.cand_cnt;
  f.partial = w.partial;
  f.fstart = reinterpret_cast<uint8_t*>(w.roff);       // free until the record counts
  if (kind == 0) {                                      // triangles: the prep counts the records
    f.rcnt = w.roff;
    f.tb = tb;
  }
  f.box = w.box;
  prep_prims(kind, g, data, n_prims, offsets, n_fib, radius, f, stats, s, batch, w.stage_ctr, 1);
  const int pgrid = int(n_prims / kBlock + 1 < kPrimGrid ? n_prims / kBlock + 1 : kPrimGrid);
  {
    VX_TIMED("tile_records", s);
    // fibers: their fiber-start bytes share the counts' space, so the count is a pass of its own
    if (kind != 0)
      hipLaunchKernelGGL(k_rec_count, dim3(pgrid), dim3(kBlock), 0, s, w.box, w.cand_cnt, n_prims, tb, w.roff);
    device_scan(ArrIn64{w.roff}, ArrOut64{w.roff}, RecTotal{w.roff, w.ctl, stats, max_rec}, nullptr, n_prims,
                w.partial, s);
    // a counting call without room for records (or units, below) ends at its count
    if (max_rec == 0) return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
    if (key64)
      hipLaunchKernelGGL(k_rec_emit<uint64_t>, dim3(pgrid), dim3(kBlock), 0, s, w.rec, w.box, w.roff, n_prims, w.ctl, tb,
                         batch ? 1 : 0, (uint64_t*)w.ra.keys, w.ra.prim);
    else
      hipLaunchKernelGGL(k_rec_emit<uint32_t>, dim3(pgrid), dim3(kBlock), 0, s, w.rec, w.box, w.roff, n_prims, w.ctl, tb, 0,
                         (uint32_t*)w.ra.keys, w.ra.prim);
  }
  int key_bits = 3 * (g->log2_res - tb);
  if (batch) {
    int pb = 1;
    while ((1 << pb) < batch->n_patches) ++pb;
    key_bits = kPatchShift - 3 * tb + pb;
  }
  const PairBufs R = radix_sort_pairs(key64, key_bits, w.ra, w.rb, w.ra, w.ctl + CTL_N_REC, max_rec, w.hist, w.partial, s);
  {
    VX_TIMED("tile_heads", s);
    if (key64)
      device_scan(HeadIn<uint64_t, 0>{(const uint64_t*)R.keys}, HeadOut{w.tstart}, TileTotal{w.tstart, w.ctl},
                  w.ctl + CTL_N_REC, max_rec, w.partial, s);
    else
      device_scan(HeadIn<uint32_t, 0>{(const uint32_t*)R.keys}, HeadOut{w.tstart}, TileTotal{w.tstart, w.ctl},
                  w.ctl + CTL_N_REC, max_rec, w.partial, s);
  }
  {
    VX_TIMED("unit_plan", s);
    // (a grid beyond the chip's fill only where there may be as many tiles: records are many to a tile)
    const int grid = bounded_grid(tu.grids[kTunePlan], max_rec / 8 > kGrid ? max_rec / 8 : kGrid);
    const int64_t budget = tu.unit_budget;
#define VX_PLAN(P, K)                                                                                        \
  hipLaunchKernelGGL((k_unit_plan<P, K>), dim3(grid), dim3(kBlock), 0, s, w.box, (const K*)R.keys, R.prim, w.tstart, \
                     w.ctl, tb, batch ? 1 : 0, budget, w.ucnt, w.uoff, w.units)
    if (key64) VX_PLAN(0, uint64_t); else VX_PLAN(0, uint32_t);
    device_scan(UnitCountIn{w.ucnt}, ArrOut64{w.uoff}, UnitTotal{w.uoff, w.ctl, stats, max_units}, w.ctl + CTL_N_TILES,
                max_rec, w.partial, s);
    if (max_units == 0) return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
    if (key64) VX_PLAN(1, uint64_t); else VX_PLAN(1, uint32_t);
#undef VX_PLAN
  }
  {
    VX_TIMED(kind == 0 ? "unit_tri" : "unit_fib", s);
    const Lat L = make_lat(g, kind, radius);
    const Lat* lats = batch ? batch->lats : nullptr;
    const int ugrid = bounded_grid(tu.grids[kTuneUnit], max_units);
    // Small units go to single waves where the capacities, taken from counts, say that units hold few
    // records (fewer records than units: long segments, whose units are full, or capacities that are no
    // counts, which give units the more room).  Unit
    // kernels of strands and weaves at 4.5 records a unit 104 us, 65 with single waves; at 7.4 133 and
    // 91; at 11 149 and 120; at 12.4 47 and 49; at 16.5 156 and 178, since the two kernels' rests add up.
    const int small = kind == 1 && max_units <= max_rec && max_rec <= 12 * max_units ? kSmallCand : 0;
    const int sgrid = bounded_grid(tu.grids[kTuneUnit], (max_units + kWaves - 1) / kWaves);
#define VX_UNIT(KD, C, T, GRID, BYTES)                                                                           \
  do {                                                                                                          \
    constexpr size_t bytes_ = BYTES;                                                                            \
    static bool attr_ = false;                                                                                  \
    if (!attr_) {                                                                                               \
      (void)hipFuncSetAttribute((const void*)k_unit<KD, C, T>, hipFuncAttributeMaxDynamicSharedMemorySize,     \
                                int(bytes_));                                                                   \
      attr_ = true;                                                                                             \
    }                                                                                                           \
    hipLaunchKernelGGL((k_unit<KD, C, T>), dim3(GRID), dim3(kBlock), bytes_, s, w.rec, w.dirs, R.prim, w.tstart,     \
                       w.units, w.ctl, L, lats, w.unv, w.unp, w.usoff, w.st, w.stage_ctr, stats, small);       \
  } while (0)
#define VX_UNIT_KIND(KD)                                                              \
  switch (tu.unit_budget) {                                                           \
    case 1024: VX_UNIT(KD, 1024, kBlock, ugrid, (unit_lds_bytes<KD, 1024>())); break; \
    case 1536: VX_UNIT(KD, 1536, kBlock, ugrid, (unit_lds_bytes<KD, 1536>())); break; \
    case 2048: VX_UNIT(KD, 2048, kBlock, ugrid, (unit_lds_bytes<KD, 2048>())); break; \
    default: VX_UNIT(KD, 3072, kBlock, ugrid, (unit_lds_bytes<KD, 3072>())); break;  \
  }
    if (kind == 0) {
      VX_UNIT_KIND(0);
    } else {
      VX_UNIT_KIND(1);
      if (small) VX_UNIT(1, kSmallCand, 64, sgrid, kWaves * small_lds_bytes() + 64);
    }
#undef VX_UNIT_KIND
#undef VX_UNIT
  }
  {
    VX_TIMED("unit_compact", s);
    const int blocks = scan_blocks(max_units, kGrid), cgrid = bounded_grid(tu.grids[kTuneCompact], max_units);
    hipLaunchKernelGGL(k_unit_sums_partial, dim3(blocks), dim3(kBlock), 0, s, w.unp, w.units, w.unv, w.ctl,
                       w.partial);
    hipLaunchKernelGGL(k_unit_sums_apply, dim3(blocks), dim3(kBlock), 0, s, w.unv, w.ctl, w.partial, w.upos, stats,
                       out->cap);
    if (key64)
      hipLaunchKernelGGL(k_unit_compact<uint64_t>, dim3(cgrid), dim3(kBlock), 0, s, w.unv,
                         w.usoff, w.upos, w.ctl, w.st, *out);
    else
      hipLaunchKernelGGL(k_unit_compact<uint32_t>, dim3(cgrid), dim3(kBlock), 0, s, w.unv,
                         w.usoff, w.upos, w.ctl, w.st, *out);
  }
  return hipGetLastError() == hipSuccess ? VX_OK : VX_ERR_HIP;
}

}  // namespace vx
