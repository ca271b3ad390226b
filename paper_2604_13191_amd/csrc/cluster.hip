// cluster.hip -- Sec. 4.4: per coarse voxel, merge the lobes of its children down to at most K.
//
// The paper builds a dendrogram by repeatedly merging the two most similar SGGX lobes of a
// voxel's set (its similarity compares the distributions, not the parameters).  Here the
// similarity is the L2 distance between the lobes' projected-area-squared functions,
// D(A, B) = 2 tr((A - B)^2) + (tr(A - B))^2 for normalised lobes A = S_a / w_a, and merging
// follows Ward's rule (least w_a w_b / (w_a + w_b) * D, ties to the first pair), then a few
// weighted Lloyd passes refine the K clusters.  Merging is additive: (w_a + w_b, S_a + S_b).
//
// Mapping: a block takes a run of coarse voxels.  First one lane per voxel counts its input
// lobes; voxels with at most K are finished there (their lobes, sorted).  The others are listed
// in LDS by the number of lanes they need (8, 16, 32 or 64), and the waves serve each list with
// full rounds of 64 / G voxels: lane m of a group holds input lobe m, the clusters and the
// symmetric matrix of pairwise costs live in LDS.  Every reduction has a fixed order, so the
// result is deterministic and depends neither on the group width nor on the grid.
//
// The clustering is bound by VALU issue and, on levels of a few thousand voxels, by the latency of
// one round's chain of merges.  A merge step therefore keeps no cached minima: each lane rereads
// its row (G / 4 16-byte loads) and takes its least cost with integer minima (costs are
// non-negative: their bits order like the values), about 105 instructions against 250 with cached
// minima, 64-bit keys and rescans.  Levels above the first, K = 4: the whole brushed surface (2.1 M
// voxels at level 2) 3.31 -> 2.11 ms, 14 fabric patches 5.25 -> 1.47 ms, a sphere of 1.0 M leaf
// voxels, where most voxels gather 17 to 32 lobes, 3.94 -> 0.47 ms (its levels had too few rounds
// in flight).  First level (few voxels hold more than K lobes): 0.78 -> 0.50 ms.
#include "vx_internal.hpp"

namespace vx {

constexpr uint32_t kNoCost = 0x7f800000u;        // +inf: no pair (a NaN cost orders above it)

// D between two normalised lobes a = S_a / w_a, b = S_b / w_b.  The operations and their fusions
// are spelled out: near-equal costs must compare alike wherever they are computed.
__device__ __forceinline__ float lobe_dist_n(const float* a, const float* b) {
#pragma clang fp contract(off)
  float d[6];
#pragma unroll
  for (int j = 0; j < 6; ++j) d[j] = a[j] - b[j];
  const float tr = (d[0] + d[1]) + d[2];
  const float diag = __builtin_fmaf(d[2], d[2], __builtin_fmaf(d[0], d[0], d[1] * d[1]));
  const float off = __builtin_fmaf(d[5], d[5], __builtin_fmaf(d[3], d[3], d[4] * d[4]));
  const float t2 = __builtin_fmaf(2.0f, off, diag);
  return __builtin_fmaf(tr, tr, t2 + t2);
}

// Ward's merge cost w_a w_b / (w_a + w_b) D (reciprocals to 1 ulp); symmetric bit for bit
__device__ __forceinline__ float ward_cost(float wa, float wb, const float* na, const float* nb) {
#pragma clang fp contract(off)
  return (wa * wb * __builtin_amdgcn_rcpf(wa + wb)) * lobe_dist_n(na, nb);
}

template <int G>
__device__ __forceinline__ uint64_t group_bits(uint64_t ballot, int gi) {
  if (G == 64) return ballot;
  return (ballot >> (gi * G)) & ((uint64_t(1) << G) - 1);
}

// minimum over the G lanes of a group: DPP within rows of 16 (xor 1 and 2 by quad permutes, then
// the half-row and row mirrors, each pairing every lane with a partner of the other half), then
// row and half exchanges for G = 32 and 64
template <int G>
__device__ __forceinline__ uint32_t group_min_u32(uint32_t v) {
  auto least = [](uint32_t a, int b) { return uint32_t(b) < a ? uint32_t(b) : a; };
  v = least(v, __builtin_amdgcn_update_dpp(0, int(v), 0xB1, 0xF, 0xF, true));
  v = least(v, __builtin_amdgcn_update_dpp(0, int(v), 0x4E, 0xF, 0xF, true));
  if (G > 4) v = least(v, __builtin_amdgcn_update_dpp(0, int(v), 0x141, 0xF, 0xF, true));
  if (G > 8) v = least(v, __builtin_amdgcn_update_dpp(0, int(v), 0x140, 0xF, 0xF, true));
  if (G > 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = least(r[0], int(r[1]));
  }
  if (G > 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = least(r[0], int(r[1]));
  }
  return v;
}

// a lobe in LDS: (w, xx, yy, zz), (xy, xz, yz, -)
struct LobeQ {
  float4 a, b;
};
__device__ __forceinline__ void lobe_unpack(const LobeQ& q, float& w, float* S) {
  w = q.a.x;
  S[0] = q.a.y;
  S[1] = q.a.z;
  S[2] = q.a.w;
  S[3] = q.b.x;
  S[4] = q.b.y;
  S[5] = q.b.z;
}
__device__ __forceinline__ LobeQ lobe_pack(float w, const float* S) {
  return LobeQ{make_float4(w, S[0], S[1], S[2]), make_float4(S[3], S[4], S[5], 0.f)};
}
// the lobe's weight and normalised moments
__device__ __forceinline__ void lobe_norm(const LobeQ& q, float& w, float* n) {
  float S[6];
  lobe_unpack(q, w, S);
  const float iw = __builtin_amdgcn_rcpf(w);
#pragma unroll
  for (int t = 0; t < 6; ++t) n[t] = S[t] * iw;
}

// Rows of the cost matrix are padded by four words: the 16-byte row reads of 16 lanes then cover
// all 64 banks once.  The input lobes wait in registers while the matrix is needed and take its
// place for the Lloyd passes, so that three blocks of up to 32-lane groups fit a CU's 160 KB.
template <int G>
struct ClusterLds {
  LobeQ clu[64 / G][G];          // the clusters' sums
  union {
    uint32_t mat[64 / G][G][G + 4];
    LobeQ lob[64 / G][G];        // the input lobes
  };
  uint32_t asg[64 / G][G / 4];   // Lloyd: each lobe's cluster, a byte each (255: no lobe)
};

// the lobes of a level: one per voxel (nl == nullptr, present when its weight is positive) or up
// to Kc per voxel, w[k * cap + c] and S[(j * Kc + k) * cap + c]
struct ChildLobes {
  const float* w;
  const float* S;
  const uint8_t* nl;
  int Kc;
  int64_t cap;
};

// lobe number m (child-major, then lobe order) of a voxel: nibble i of word counts child i's lobes
__device__ __forceinline__ void nth_lobe(uint32_t word, int m, int& ch, int& k) {
  ch = 0;
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const int c = int((word >> (4 * i)) & 15u);
    const bool past = ch == i && m >= c;
    m = past ? m - c : m;
    ch = past ? i + 1 : ch;
  }
  k = m;
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// One round of one wave: group gi (gi < 64 / G) reduces the n input lobes (K < n <= G; 0 when not
// live) of coarse voxel p, whose children start at cs.
template <int G>
__device__ __forceinline__ void cluster_round(int64_t p, bool live, int64_t cs, uint32_t word, int n,
                                              const ChildLobes& C, int K, int iters, const vx_lobes& out,
                                              ClusterLds<G>& L) {
  const int lane = lane_id();
  const int g = lane % G, gi = lane / G;
  const bool mine = g < n;
  float w = 0.f, nrm[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // this lane's cluster
  LobeQ own{};                                               // and its input lobe
  if (mine) {
    int ch, k;
    nth_lobe(word, g, ch, k);
    const int64_t c = cs + ch;
    float S[6];
    w = C.w[int64_t(k) * C.cap + c];
#pragma unroll
    for (int j = 0; j < 6; ++j) S[j] = C.S[(int64_t(j) * C.Kc + k) * C.cap + c];
    own = lobe_pack(w, S);
    L.clu[gi][g] = own;
    lobe_norm(own, w, nrm);
    uint4* row = reinterpret_cast<uint4*>(L.mat[gi][g]);
#pragma unroll
    for (int j = 0; j < G / 4; ++j) row[j] = make_uint4(kNoCost, kNoCost, kNoCost, kNoCost);
  }
  wave_lds_fence();
  // the costs of all pairs, each computed once: lane g against the n / 2 lobes after it (cyclic)
  if (mine) {
    for (int d = 1; 2 * d <= n; ++d) {
      const int j = g + d < n ? g + d : g + d - n;
      float wj, nj[6];
      lobe_norm(L.clu[gi][j], wj, nj);
      const uint32_t c = __float_as_uint(ward_cost(w, wj, nrm, nj));
      L.mat[gi][g][j] = c;
      L.mat[gi][j][g] = c;
    }
  }
  wave_lds_fence();
  bool alive = mine;
  int cl = g;                                      // the cluster that input lobe g belongs to
  for (int step = n; step > K; --step) {
    // the least cost of the group, then the first pair (i, j), i < j, that has it: i is the first
    // lane whose row holds it, j the first column of that row (the matrix is symmetric)
    uint32_t best = kNoCost;
    const uint4* row = reinterpret_cast<const uint4*>(L.mat[gi][g]);
#pragma unroll
    for (int q = 0; q < G / 4; ++q) {
      const uint4 r = row[q];
      best = min(best, min(min(r.x, r.y), min(r.z, r.w)));
    }
    best = alive ? best : kNoCost;
    const uint32_t least = group_min_u32<G>(best);
    if (least >= kNoCost) break;                   // no pair of finite cost
    const int i = __ffsll((unsigned long long)group_bits<G>(__ballot(best == least), gi)) - 1;
    const uint32_t col = L.mat[gi][i][g];
    const int j = __ffsll((unsigned long long)group_bits<G>(__ballot(col == least), gi)) - 1;
    // cluster i absorbs cluster j
    float wi, wj, Si[6], Sj[6], mn[6];
    lobe_unpack(L.clu[gi][i], wi, Si);
    lobe_unpack(L.clu[gi][j], wj, Sj);
    const float mw = wi + wj;
    const float inw = __builtin_amdgcn_rcpf(mw);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
#pragma clang fp contract(off)
      Si[t] = Si[t] + Sj[t];
      mn[t] = Si[t] * inw;
    }
    wave_lds_fence();
    if (cl == j) cl = i;
    if (g == j) alive = false;
    if (g == i) {
      w = mw;
#pragma unroll
      for (int t = 0; t < 6; ++t) nrm[t] = mn[t];
      L.clu[gi][i] = lobe_pack(mw, Si);
      L.mat[gi][i][j] = kNoCost;
    } else if (alive) {
      const uint32_t c = __float_as_uint(ward_cost(mw, w, mn, nrm));
      L.mat[gi][i][g] = c;
      L.mat[gi][g][i] = c;
      L.mat[gi][g][j] = kNoCost;
    }
    wave_lds_fence();
  }
  uint64_t act = group_bits<G>(__ballot(alive), gi);
  // ---- weighted Lloyd passes over the input lobes.  A pass that moves no lobe to another cluster
  // leaves every cluster as it is, and so does every later one: the group stops there.
  if (live) {
    float lw, ln[6];
    lobe_norm(own, lw, ln);
    if (mine) L.lob[gi][g] = own;
    for (int it = 0; it < iters; ++it) {
      int assign = -1;
      // nearest active centroid (ties to the lowest index), walking the active set
      float bestd = INFINITY;
      for (uint64_t m = act; m; m &= m - 1) {
        const int k = __ffsll((unsigned long long)m) - 1;
        float wk, nk[6];
        lobe_norm(L.clu[gi][k], wk, nk);
        const float d = lobe_dist_n(ln, nk);
        if (d < bestd) { bestd = d; assign = k; }
      }
      if (group_bits<G>(__ballot(mine && assign != cl), gi) == 0) break;
      cl = assign;
      reinterpret_cast<uint8_t*>(L.asg[gi])[g] = uint8_t(mine ? assign : 255);
      wave_lds_fence();
      // new cluster sums: one lane per (active cluster, component), adding the members in lobe
      // order (sequential, so the sums are fixed)
      const int na = __popcll(act);
      for (int q = g; q < 7 * na; q += G) {
        const int r = q / 7, t = q - 7 * r;        // component 0 is the weight
        uint64_t m = act;
        for (int x = 0; x < r; ++x) m &= m - 1;
        const int k = __ffsll((unsigned long long)m) - 1;
        const float* v = reinterpret_cast<const float*>(&L.lob[gi][0]) + t;
        float sum = 0.f;
        for (int x = 0; x < n; x += 4) {
          // (x + 3 < G: in bounds; a byte past the lobes matches no cluster)
          const uint32_t of = L.asg[gi][x >> 2];
          float u[4];
#pragma unroll
          for (int y = 0; y < 4; ++y) u[y] = v[8 * (x + y)];
#pragma unroll
          for (int y = 0; y < 4; ++y) sum += int((of >> (8 * y)) & 255u) == k ? u[y] : 0.f;
        }
        reinterpret_cast<float*>(&L.clu[gi][k])[t] = sum;
      }
      wave_lds_fence();
      uint64_t left = 0;
      for (uint64_t m = act; m; m &= m - 1) {
        const int k = __ffsll((unsigned long long)m) - 1;
        if (L.clu[gi][k].a.x > 0.f) left |= uint64_t(1) << k;
      }
      act = left;
    }
    // ---- output: active clusters sorted by descending weight (ties keep cluster order)
    const int nl = __popcll(act);
    if ((act >> g) & 1) {
      const LobeQ q = L.clu[gi][g];
      int rank = 0;
      for (uint64_t m = act; m; m &= m - 1) {
        const int k = __ffsll((unsigned long long)m) - 1;
        const float wk = L.clu[gi][k].a.x;
        rank += (wk > q.a.x || (wk == q.a.x && k < g)) ? 1 : 0;
      }
      if (rank < K) {                             // at most K clusters remain; never write past them
        float ow, S[6];
        lobe_unpack(q, ow, S);
        out.w[int64_t(rank) * out.cap + p] = ow;
#pragma unroll
        for (int t = 0; t < 6; ++t) out.S[(int64_t(t) * K + rank) * out.cap + p] = S[t];
      }
    }
    if (g >= nl && g < K) {
      out.w[int64_t(g) * out.cap + p] = 0.f;
#pragma unroll
      for (int t = 0; t < 6; ++t) out.S[(int64_t(t) * K + g) * out.cap + p] = 0.f;
    }
    if (g == 0) out.nl[p] = uint8_t(nl);
  }
  wave_lds_fence();
}

// A coarse voxel with at most K lobes keeps them, sorted by descending weight (ties in lobe
// order): one lane each, so that the K sorted lobes of 64 neighbours leave in whole lines.
template <int MAXK>
__device__ __forceinline__ void keep_lobes(int64_t p, int64_t cs, uint32_t word, int n, const ChildLobes& C, int K,
                                           const vx_lobes& out) {
  float w[MAXK];
  int at[MAXK];                                   // child * 16 + lobe
#pragma unroll
  for (int m = 0; m < MAXK; ++m) {
    w[m] = -1.f;
    at[m] = 0;
    if (m < n) {
      int ch, k;
      nth_lobe(word, m, ch, k);
      at[m] = ch * 16 + k;
      w[m] = C.w[int64_t(k) * C.cap + cs + ch];
    }
  }
  // odd-even transposition, neighbours exchanged only when strictly out of order: stable
#pragma unroll
  for (int r = 0; r < MAXK; ++r)
#pragma unroll
    for (int m = r & 1; m + 1 < MAXK; m += 2) {
      const bool sw = w[m + 1] > w[m];
      const float a = w[m], b = w[m + 1];
      const int x = at[m], y = at[m + 1];
      w[m] = sw ? b : a;
      w[m + 1] = sw ? a : b;
      at[m] = sw ? y : x;
      at[m + 1] = sw ? x : y;
    }
#pragma unroll
  for (int s = 0; s < MAXK; ++s) {
    if (s >= K) break;
    const bool has = s < n;
    const int64_t c = cs + (at[s] >> 4);
    const int k = at[s] & 15;
    out.w[int64_t(s) * out.cap + p] = has ? w[s] : 0.f;
#pragma unroll
    for (int t = 0; t < 6; ++t)
      out.S[(int64_t(t) * K + s) * out.cap + p] = has ? C.S[(int64_t(t) * C.Kc + k) * C.cap + c] : 0.f;
  }
  out.nl[p] = uint8_t(n);
}

// One level.  SLOTS: the most input lobes of a voxel (8: one per child; 32: up to four per child;
// 64).  A block takes runs of `run` voxels: 256, or on small levels as few as spread the level
// over three times the blocks that are resident, at least 8 (two rounds of 32 lanes per wave).
template <int SLOTS>
__global__ void __launch_bounds__(kBlock) k_cluster(const int64_t* __restrict__ pstart, const int64_t* n_par_ptr,
                                                    ChildLobes C, int K, int iters, vx_lobes out) {
  constexpr int kLists = SLOTS <= 8 ? 1 : (SLOTS <= 32 ? 3 : 4);
  union WaveLds {
    ClusterLds<8> g8;
    ClusterLds<SLOTS <= 8 ? 8 : 16> g16;
    ClusterLds<SLOTS <= 8 ? 8 : 32> g32;
    ClusterLds<SLOTS <= 32 ? 8 : 64> g64;
  };
  __shared__ WaveLds lds[kWaves];
  __shared__ int64_t first[kBlock];               // first child
  __shared__ uint32_t words[kBlock];              // lobes per child, a nibble each
  __shared__ uint8_t list[kLists][kBlock], count[kBlock];
  __shared__ int32_t len[kLists];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int64_t n_par = *n_par_ptr;
  int64_t run = ((n_par + 3 * 768 - 1) / (3 * 768) + 7) & ~int64_t(7);
  run = run < 8 ? 8 : (run > kBlock ? kBlock : run);
  for (int64_t base = int64_t(blockIdx.x) * run; base < n_par; base += int64_t(gridDim.x) * run) {
    if (tid < kLists) len[tid] = 0;
    __syncthreads();
    const int64_t p = base + tid;
    if (tid < run && p < n_par) {
      const int64_t cs = pstart[p], ce = pstart[p + 1];
      uint32_t word = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (cs + i < ce) {
          int c;
          if (SLOTS <= 8) c = C.w[cs + i] > 0.f ? 1 : 0;
          else c = int(C.nl[cs + i]) < C.Kc ? int(C.nl[cs + i]) : C.Kc;
          word |= uint32_t(c) << (4 * i);
        }
      }
      const uint32_t pairs = (word & 0x0f0f0f0fu) + ((word >> 4) & 0x0f0f0f0fu);
      const int n = int((pairs * 0x01010101u) >> 24);
      if (n <= K) {
        if (K <= 4) keep_lobes<4>(p, cs, word, n, C, K, out);
        else keep_lobes<8>(p, cs, word, n, C, K, out);
      } else {
        first[tid] = cs;
        words[tid] = word;
        count[tid] = uint8_t(n);
        const int l = SLOTS <= 8 ? 0 : (n <= 8 ? 0 : (n <= 16 ? 1 : (n <= 32 ? 2 : kLists - 1)));
        list[l][atomicAdd(&len[l], 1)] = uint8_t(tid);
      }
    }
    __syncthreads();
#define VX_ROUNDS(G, LIST, FIELD)                                                                        \
  for (int r = wave * (64 / G); r < len[LIST]; r += kWaves * (64 / G)) {                                \
    const int e = r + (tid & 63) / G;                                                                   \
    const bool live = e < len[LIST];                                                                    \
    const int q = live ? list[LIST][e] : 0;                                                             \
    cluster_round<G>(base + q, live, live ? first[q] : 0, live ? words[q] : 0, live ? count[q] : 0, C, K, iters, out, \
                     lds[wave].FIELD);                                                                  \
  }
    if constexpr (kLists > 3) { VX_ROUNDS(64, 3, g64) }
    if constexpr (kLists > 1) {
      VX_ROUNDS(32, 2, g32)
      VX_ROUNDS(16, 1, g16)
    }
    VX_ROUNDS(8, 0, g8)
#undef VX_ROUNDS
    __syncthreads();
  }
}

void cluster_level(const int64_t* pstart, const int64_t* n_par, const float* cw, const float* cS, const uint8_t* cnl,
                   int Kc, int64_t cap_c, int K, int iters, const vx_lobes& out, int grid, hipStream_t s) {
  const int need = 8 * Kc;
  // no more blocks than the level's capacity of voxels can use (the upper levels are small)
  const int64_t most = (out.cap + 7) / 8;
  const int blocks = int(most < grid ? (most < 1 ? 1 : most) : grid);
  const ChildLobes C{cw, cS, cnl, Kc, cap_c};
  // timing names: the first level (one lobe per child) and the levels above
  VX_TIMED(need <= 8 ? "lod_cluster" : "lod_cluster_up", s);
  if (cnl == nullptr) hipLaunchKernelGGL(k_cluster<8>, dim3(blocks), dim3(kBlock), 0, s, pstart, n_par, C, K, iters, out);
  else if (need <= 32) hipLaunchKernelGGL(k_cluster<32>, dim3(blocks), dim3(kBlock), 0, s, pstart, n_par, C, K, iters, out);
  else hipLaunchKernelGGL(k_cluster<64>, dim3(blocks), dim3(kBlock), 0, s, pstart, n_par, C, K, iters, out);
}

}  // namespace vx
