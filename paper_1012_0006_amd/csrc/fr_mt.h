// Multi-try FM (Sanders & Schulz, Section 4.2) on the GPU: after the
// pairwise improvements of a round, one round of localized k-way searches per
// pair, in pair order.
//
// The k-way local search of Section 2.2 moves a vertex to the adjacent block
// with the largest gain, so a search of one pair can reach any block: the
// searches of a round's pairs are not independent, and they run one after
// the other, in one workgroup.  Around them the work is spread over the chip:
//   k_mt_weights  block weights of all k blocks (grid-wide)
//   k_mt_todo     each pair's todo list: the vertices of its two blocks with
//                 a neighbour in another block, as sort keys (upper 32 bits
//                 of a SplitMix64 output, then the id), grid-wide
//   k_mt_sort     each todo list in key order (one workgroup per pair:
//                 bitonic in LDS, a tiled rank sort beyond)
//   k_mt          the searches (one workgroup): a flat queue of (gain, key,
//                 vertex) in LDS that spills to device memory, popped by a
//                 wave-wide maximum and updated by all lanes at once; each
//                 neighbour's k-way gain computed by a group of lanes;
//                 KaSPar's stopping rule in exact integer arithmetic;
//                 rollback to the best state.
// The counters of the keys (SplitMix64 outputs from mt_seed): todo order of v
// 2^40 + v + 1, queue order of v 2^41 + v + 1, tie key of target block P of v
// 2^42 + v k + P + 1.
#pragma once
#include "fr_kernels.h"

#define MT_SORT_TPB 1024
#define MT_LSORT 8192   // todo keys sorted in LDS
#define MT_LQ 2048      // queue entries in LDS (the rest in device memory)
#define MT_SCAN 1024    // a queue of up to this many entries is scanned whole
#define MT_NB 1024      // groups of 64 queue entries with a bound in LDS
#define MT_LBLK 2048    // block weights held in LDS
#define MT_TPB 320      // threads of the search kernel: one wave searches, four compute gains
#define MT_G 16         // lanes that compute one vertex's gain
#define MT_ITEMS 64     // vertices whose gains are computed per request

__device__ __forceinline__ uint64_t mt_splitmix(uint64_t seed, uint64_t n) {
  uint64_t z = seed + n * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t mt_key(uint64_t seed, int which, uint64_t x) {
  return mt_splitmix(seed, (1ull << (40 + which)) + x + 1ull);
}

// Block weights of every block (cleared by k_mt_clear).
__global__ void __launch_bounds__(256) k_mt_weights(KArgs A) {
  for (int64_t b0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) & ~(int64_t)63; b0 < A.n;
       b0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t u = b0 + lane64();
    const int key = u < A.n ? A.part[u] : -1;
    const int64_t w = u < A.n ? A.vwgt[u] : 0;
    wave_add_by_key(reinterpret_cast<unsigned long long *>(A.mtw), 1, 0, key, w);
  }
}

// Clears the weights and the todo counters of the round (one block).
__global__ void __launch_bounds__(1024) k_mt_clear(KArgs A) {
  for (int i = threadIdx.x; i < A.k; i += blockDim.x) A.mtw[i] = 0;
  for (int i = threadIdx.x; i < A.P; i += blockDim.x) A.ucnt[i] = 0;
}

// Todo keys: every vertex of a round pair's blocks with a neighbour in
// another block, appended to the pair's slice (its first entry's arena).
__global__ void __launch_bounds__(256) k_mt_todo(KArgs A) {
  const uint64_t seed = (uint64_t)(uint32_t)A.mt_seed;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < A.n;
       u += (int64_t)gridDim.x * blockDim.x) {
    const int32_t x = A.part[u];
    const int32_t p = A.blk2pair[x];
    if (p < 0) continue;
    const int32_t e1 = A.xadj[u + 1];
    bool bnd = false;
    for (int32_t e = A.xadj[u]; e < e1 && !bnd; e++) bnd = A.part[A.adjncy[e]] != x;
    if (!bnd) continue;
    const uint64_t k = ((mt_key(seed, 0, (uint64_t)u) >> 32) << 32) | (uint64_t)(uint32_t)u;
    const int32_t pos = atomicAdd(&A.ucnt[p], 1);
    if (A.voff[p] + pos < A.voff[p + 1]) A.mtk[A.voff[p] + pos] = k;
  }
}

// Each pair's todo keys in ascending order (one workgroup per pair).
__global__ void __launch_bounds__(MT_SORT_TPB) k_mt_sort(KArgs A) {
  __shared__ unsigned long long s[MT_LSORT];
  const int32_t p = blockIdx.x * A.W;  // the pair's first entry
  const int32_t T = min((int64_t)A.ucnt[p], A.voff[p + 1] - A.voff[p]);
  unsigned long long *key = A.mtk + A.voff[p];
  if (T <= 1) return;
  if (T <= MT_LSORT) {
    int32_t N = 1;
    while (N < T) N <<= 1;
    for (int32_t i = threadIdx.x; i < N; i += blockDim.x) s[i] = i < T ? key[i] : ~0ull;
    __syncthreads();
    for (int32_t len = 2; len <= N; len <<= 1)
      for (int32_t st = len >> 1; st > 0; st >>= 1) {
        for (int32_t i = threadIdx.x; i < N; i += blockDim.x) {
          const int32_t j = i ^ st;
          if (j > i) {
            const bool up = (i & len) == 0;
            const unsigned long long a = s[i], b = s[j];
            if ((a > b) == up) {
              s[i] = b;
              s[j] = a;
            }
          }
        }
        __syncthreads();
      }
    for (int32_t i = threadIdx.x; i < T; i += blockDim.x) key[i] = s[i];
    return;
  }
  // a long list: the rank of every key (the keys are distinct) by comparing
  // with all keys, tile by tile through LDS, written to the second buffer and
  // copied back
  unsigned long long *out = A.mtk2 + A.voff[p];
  for (int32_t b0 = 0; b0 < T; b0 += blockDim.x) {
    const int32_t i = b0 + threadIdx.x;
    const unsigned long long mine = i < T ? key[i] : 0ull;
    int32_t rank = 0;
    for (int32_t t0 = 0; t0 < T; t0 += MT_LSORT) {
      const int32_t tn = min(MT_LSORT, T - t0);
      __syncthreads();
      for (int32_t j = threadIdx.x; j < tn; j += blockDim.x) s[j] = key[t0 + j];
      __syncthreads();
      if (i < T)
        for (int32_t j = 0; j < tn; j++) rank += s[j] < mine ? 1 : 0;
    }
    if (i < T) out[rank] = mine;
  }
  __syncthreads();
  for (int32_t i = threadIdx.x; i < T; i += blockDim.x) key[i] = out[i];
}

// What a move of vertex v needs to know: its target and own block, weight,
// first arc and number of arcs.
struct MTVertex {
  int32_t v, to, from, c, e0, deg;
};

// The search state of the one wave.  The queue is a flat array in arrival
// order; an entry is a rank (gain, then the key's upper half) and its vertex,
// rank 0 once it has left; the entries are packed again when most have left.
// Every vertex enters the queue at most once per round of a pair.
struct MTShared {
  uint64_t qr[MT_LQ];    // queue entries in LDS
  MTVertex qv[MT_LQ];
  uint64_t bound[MT_NB];  // no rank of entries [64 b, 64 b + 64) is above
  int64_t bw[MT_LBLK];   // block weights (k <= MT_LBLK)
  // a request for gains: the vertex v0 (unless -1) and then the heads of the
  // arcs from a0 + 1, or the heads of the arcs from a0; cnt vertices, -1 ends
  // the kernel; the pair's stamp
  int32_t v0, a0, cnt, stamp;
  // its answer per vertex: the vertex (v -1 none, target -1 none), queue slot
  // (-1 none), rank in the queue, weighted degree of 2^31 or more
  MTVertex iv[MT_ITEMS];
  int32_t islot[MT_ITEMS];
  uint64_t ir[MT_ITEMS];
  bool iovf[MT_ITEMS];
};

// Orders this lane's memory operations with the other lanes' for the
// compiler (the hardware keeps a wave's in order).
__device__ __forceinline__ void mt_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ uint64_t read_lane64(uint64_t x, int l) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(x >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int32_t)x, l);
}

// The largest value in the wave.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  const int32_t m = group_reduce<16>((int32_t)x, [](int32_t a, int32_t b) {
    return (int32_t)max((uint32_t)a, (uint32_t)b);
  });
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane(m, 0),
                 b = (uint32_t)__builtin_amdgcn_readlane(m, 16),
                 c = (uint32_t)__builtin_amdgcn_readlane(m, 32),
                 d = (uint32_t)__builtin_amdgcn_readlane(m, 48);
  return max(max(a, b), max(c, d));
}
__device__ __forceinline__ uint64_t wave_max64(uint64_t x) {
  const uint32_t h = (uint32_t)(x >> 32), hm = wave_max(h);
  return ((uint64_t)hm << 32) | wave_max(h == hm ? (uint32_t)x : 0u);
}

// Ranks order queue entries by gain, then by the upper half of the key.
__device__ __forceinline__ uint64_t mt_rank(int32_t g, uint64_t key) {
  return ((uint64_t)((uint32_t)g ^ 0x80000000u) << 32) | (key >> 32);
}

// The queue.  Its operations are called by all lanes together.  A flat array
// because a move updates about a dozen gains: those are independent stores
// here, while a binary heap walks each of them up or down, step after
// dependent step.  The price is a scan at the pop: of all entries up to
// MT_SCAN (a search holds about a hundred), else of one bound per 64 entries
// and the groups that may hold the largest.
struct MTQueue {
  const KArgs &A;
  MTShared &sh;
  unsigned long long *gr;  // entries beyond MT_LQ
  int32_t *gv;
  int32_t len = 0, live = 0;
  uint64_t seed;
  __device__ __forceinline__ uint64_t key(int32_t v) const {
    return mt_key(seed, 1, (uint64_t)(uint32_t)v);
  }
  __device__ __forceinline__ uint64_t rank_at(int32_t i) const {
    uint64_t r = sh.qr[min(i, MT_LQ - 1)];  // two loads, not one from either space
    asm("" : "+v"(r));
    if (i >= MT_LQ) r = gr[i];
    return r;
  }
  __device__ __forceinline__ int32_t vertex_at(int32_t i) const {
    int32_t v = sh.qv[min(i, MT_LQ - 1)].v;
    asm("" : "+v"(v));
    if (i >= MT_LQ) v = gv[i];
    return v;
  }
  __device__ __forceinline__ void set_rank(int32_t i, uint64_t r) {
    if (i < MT_LQ) sh.qr[i] = r;
    else gr[i] = r;
    if (i < 64 * MT_NB) atomicMax(reinterpret_cast<unsigned long long *>(&sh.bound[i >> 6]),
                                  (unsigned long long)r);
  }
  __device__ __forceinline__ void set_target(int32_t i, int32_t v, int32_t to) {
    if (i < MT_LQ) sh.qv[i].to = to;
    else A.mtb[v] = to;
  }
  __device__ __forceinline__ void set(int32_t i, const MTVertex &x, uint64_t r) {
    if (i < MT_LQ) {
      sh.qv[i] = x;
    } else {
      gv[i] = x.v;
      A.mtb[x.v] = x.to;
    }
    set_rank(i, r);
    A.mtq[x.v] = i;
  }
  // the vertex of entry i (global loads are waited for where they are issued:
  // a wait after the branch would also be one for the stores in flight)
  __device__ __forceinline__ MTVertex info(int32_t i) const {
    MTVertex x = sh.qv[min(i, MT_LQ - 1)];
    if (i >= MT_LQ) {
      x.v = gv[i];
      x.to = A.mtb[x.v];
      x.from = A.part[x.v];
      x.c = A.vwgt[x.v];
      x.e0 = A.xadj[x.v];
      x.deg = A.xadj[x.v + 1] - x.e0;
      asm volatile("" : "+v"(x.v), "+v"(x.to), "+v"(x.from), "+v"(x.c), "+v"(x.e0), "+v"(x.deg));
    }
    return x;
  }
  __device__ __forceinline__ void drop(int32_t i, int32_t v) {  // entry i (vertex v) leaves
    if (i < MT_LQ) sh.qr[i] = 0;
    else gr[i] = 0;
    A.mtq[v] = -1;
  }
  // The lanes with want join with their vertex and rank.
  __device__ __forceinline__ void push(bool want, const MTVertex &x, uint64_t r) {
    const u64 m = ballot64(want);
    if (want) {
      const int32_t i = len + lanes_below(m);
      if ((i & 63) == 0 && i < 64 * MT_NB) sh.bound[i >> 6] = 0;
      mt_order();
      set(i, x, r);
    }
    len += (int32_t)__popcll(m);
    live += (int32_t)__popcll(m);
  }
  // Entries packed to the front, in order.
  __device__ void pack() {
    int32_t to = 0;
    for (int32_t b0 = 0; b0 < len; b0 += WAVE) {
      const int32_t i = b0 + lane64();
      uint64_t r = 0;
      MTVertex x = {};
      if (i < len) r = rank_at(i);
      if (r != 0) x = info(i);
      mt_order();
      if (lane64() == 0 && b0 < 64 * MT_NB) sh.bound[b0 >> 6] = 0;  // group b0 / 64 is read
      const u64 m = ballot64(r != 0);
      mt_order();
      if (r != 0) set(to + lanes_below(m), x, r);  // at most i: read already
      mt_order();
      to += (int32_t)__popcll(m);
    }
    len = to;
  }
  // The slot of the entry with the largest gain, then the largest key (keys
  // are distinct: the generator's finaliser is a bijection), found by its
  // rank alone: -1 when two entries hold the largest rank.
  __device__ __forceinline__ int32_t find(int32_t &gain) const {
    uint64_t top = 0;  // this lane's best entry
    int32_t at = -1;
    bool twice = false;
    for (int32_t i0 = lane64(); i0 < len; i0 += 4 * WAVE) {
      uint64_t r[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        r[j] = sh.qr[i0 + j * WAVE];  // MT_SCAN entries are there
        if (i0 + j * WAVE >= len) r[j] = 0;
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        twice = r[j] == top ? true : r[j] > top ? false : twice;
        at = r[j] > top ? i0 + j * WAVE : at;
        top = max(top, r[j]);
      }
    }
    const uint32_t h = (uint32_t)(top >> 32), hm = wave_max(h);
    const uint32_t lo = h == hm ? (uint32_t)top : 0u, lm = wave_max(lo);
    const u64 m = ballot64(h == hm && lo == lm && at >= 0);
    if (m == 0ull || (m & (m - 1)) || (m & ballot64(twice))) return -1;
    gain = (int32_t)(hm ^ 0x80000000u);
    return __builtin_amdgcn_readlane(at, __ffsll(m) - 1);
  }
  // The same for any queue: the groups of 64 entries whose bound is the
  // largest, then equal ranks by the whole key.
  __device__ __forceinline__ int32_t find_any(int32_t &gain) {
    mt_order();
    for (;;) {
      uint64_t top = 0;
      int32_t at = -1, v = -1;
      auto look = [&](int32_t i) {
        const uint64_t r = rank_at(i);
        if (r != 0 && r >= top) {
          const int32_t u = vertex_at(i);
          if (r > top || key(u) > key(v)) {
            top = r;
            at = i;
            v = u;
          }
        }
      };
      const int32_t ng = min((len + 63) >> 6, MT_NB);
      uint64_t lead = 0;  // the largest bound
      for (int32_t b = lane64(); b < ng; b += WAVE) lead = max(lead, sh.bound[b]);
      lead = wave_max64(lead);
      for (int32_t b0 = 0; b0 < ng; b0 += WAVE) {  // the groups that may hold it
        const int32_t b = b0 + lane64();
        for (u64 m = ballot64(b < ng && sh.bound[b < ng ? b : 0] == lead); m; m &= m - 1) {
          const int32_t g = b0 + __ffsll(m) - 1, i = 64 * g + lane64();
          const uint64_t hi = wave_max64(i < len ? rank_at(i) : 0ull);
          if (i < len) look(i);
          mt_order();
          if (lane64() == 0) sh.bound[g] = hi;  // exact again
          mt_order();
        }
      }
      for (int32_t i = 64 * ng + lane64(); i < len; i += WAVE) look(i);
      const uint64_t hi = wave_max64(top);
      if (hi < lead) continue;  // the bounds were above every rank: they are lower now
      u64 m = ballot64(at >= 0 && top == hi);
      if (m == 0ull) return -1;  // only after an overflow, which is reported
      int win = __ffsll(m) - 1;
      const uint64_t k = m & (m - 1) ? key(v) : 0ull;
      for (m &= m - 1; m; m &= m - 1) {
        const int l = __ffsll(m) - 1;
        if (read_lane64(k, l) > read_lane64(k, win)) win = l;
      }
      gain = (int32_t)((uint32_t)(hi >> 32) ^ 0x80000000u);
      return __builtin_amdgcn_readlane(at, win);
    }
  }
  // Takes the entry with the largest gain, then the largest key: its vertex
  // and gain in every lane; v -1 when the queue is empty.
  __device__ __forceinline__ MTVertex pop(int32_t &gain) {
    MTVertex x;
    x.v = -1;
    if (live == 0) return x;
    if (len > 2 * live + MT_SCAN / 4) pack();
    mt_order();
    int32_t i = -1;
    if (len <= MT_SCAN) i = find(gain);
    if (i < 0) i = find_any(gain);
    if (i < 0) return x;
    x = info(i);
    x = {uni(x.v), uni(x.to), uni(x.from), uni(x.c), uni(x.e0), uni(x.deg)};
    if (lane64() == 0) drop(i, x.v);
    live--;
    return x;
  }
  __device__ __forceinline__ void clear() {
    for (int32_t i = lane64(); i < len; i += WAVE)
      if (rank_at(i) != 0) A.mtq[vertex_at(i)] = -1;
    len = live = 0;
  }
};

// The k-way gains of the request's vertices (all waves but the first, MT_G
// lanes a vertex): over the blocks other than a vertex y's own that hold
// a neighbour of y, the largest weight to that block minus the weight to y's
// own block; the block reaching it is the target (equal gains: the smaller
// tie key).  y has no target when it has no neighbour outside its block.  A
// vertex touched and not queued is left out.  Up to 2 MT_G arcs lie in the
// lanes' registers, and the foreign blocks are taken in ascending order, one
// sum over the group each (a vertex has neighbours in few blocks); a vertex
// with more arcs is taken by the whole wave, which reads its arcs once and
// once more per foreign block.
__device__ __forceinline__ void mt_gains(const KArgs &A, MTShared &sh, uint64_t seed) {
  constexpr int32_t NONE = 0x7fffffff;
  constexpr int32_t GROUPS = (MT_TPB - WAVE) / MT_G;
  const int32_t v0 = uni(sh.v0), a0 = uni(sh.a0), cnt = uni(sh.cnt),
                stamp = uni(sh.stamp);
  const int gl = (int)threadIdx.x & (MT_G - 1);
  for (int32_t i0 = 0; i0 < cnt; i0 += GROUPS) {
    const int32_t i = i0 + ((int32_t)threadIdx.x - WAVE) / MT_G;
    int32_t y = -1, slot = -1, e0 = 0, e1 = 0, own = -1, cy = 0;
    uint64_t kq = 0;
    if (i < cnt) {
      y = i == 0 && v0 >= 0 ? v0 : A.adjncy[a0 + i];
      const int32_t mark = A.mtt[y];
      slot = A.mtq[y];
      e0 = A.xadj[y];
      e1 = A.xadj[y + 1];
      own = A.part[y];
      cy = A.vwgt[y];
      kq = mt_key(seed, 1, (uint64_t)(uint32_t)y);
      asm volatile("" : "+v"(kq));  // while the loads are on their way
      if (slot < 0 && mark == stamp) {
        y = -1;
        e1 = e0;
      }
    }
    int32_t best = -1;
    int32_t bg = 0;
    auto consider = [&](int32_t P, int32_t gP) {
      auto tie = [&](int32_t Q) {
        return mt_key(seed, 2, (uint64_t)(uint32_t)y * (uint64_t)A.k + (uint64_t)Q);
      };
      if (best < 0 || gP > bg || (gP == bg && tie(P) < tie(best))) {
        best = P;
        bg = gP;
      }
    };
    const bool large = e1 - e0 > 2 * MT_G;
    const bool in0 = !large && e0 + gl < e1, in1 = !large && e0 + MT_G + gl < e1;
    int32_t w0 = 0, w1 = 0, b0 = -1, b1 = -1;  // the heads' blocks (-1 no arc), weights
    if (in0) {
      w0 = A.adjwgt[e0 + gl];
      b0 = A.adjncy[e0 + gl];
    }
    if (in1) {
      w1 = A.adjwgt[e0 + MT_G + gl];
      b1 = A.adjncy[e0 + MT_G + gl];
    }
    if (in0) b0 = A.part[b0];
    if (in1) b1 = A.part[b1];
    // 32 arcs of less than 2^30: summed in halves; the sums of single blocks
    // are exact unless this one reports an overflow
    int64_t wtot = ((int64_t)group_sum<MT_G>((w0 >> 16) + (w1 >> 16)) << 16) +
                   group_sum<MT_G>((w0 & 0xffff) + (w1 & 0xffff));
    const int32_t wown = group_sum<MT_G>((b0 == own ? w0 : 0) + (b1 == own ? w1 : 0));
    auto above = [&](int32_t Q) {  // the next foreign block above Q
      return group_min<MT_G>(min(b0 > Q && b0 != own ? b0 : NONE, b1 > Q && b1 != own ? b1 : NONE));
    };
    int32_t P = above(-1);
    while (ballot64(P != NONE) != 0ull) {
      const int32_t s = group_sum<MT_G>((b0 == P ? w0 : 0) + (b1 == P ? w1 : 0));
      const int32_t next = above(P);
      if (P != NONE) consider(P, s - wown);
      P = next;
    }
    for (u64 m = ballot64(large && gl == 0); m; m &= m - 1) {
      const int l = __ffsll(m) - 1;
      const int32_t f0 = __builtin_amdgcn_readlane(e0, l), f1 = __builtin_amdgcn_readlane(e1, l);
      const int32_t mine = __builtin_amdgcn_readlane(own, l);
      const bool group = lane64() / MT_G == l / MT_G;
      int64_t wo = 0, wt = 0;
      for (int32_t Q = -1;;) {  // the own block's sum first, then one block after the other
        const int32_t want = Q < 0 ? mine : Q;
        int64_t s = 0, all = 0;
        int32_t next = NONE;
        for (int32_t e = f0 + lane64(); e < f1; e += WAVE) {
          const int32_t c = A.part[A.adjncy[e]], w = A.adjwgt[e];
          all += w;
          if (c == want) s += w;
          if (c > Q && c != mine && c < next) next = c;
        }
        for (int o = 32; o > 0; o >>= 1) {
          s += __shfl_xor((long long)s, o);
          all += __shfl_xor((long long)all, o);
          next = min(next, __shfl_xor(next, o));
        }
        if (Q < 0) {
          wo = s;
          wt = all;
        } else if (group) {
          consider(Q, (int32_t)(s - wo));
        }
        if (next == NONE) break;
        Q = next;
      }
      if (group) wtot = wt;
    }
    if (gl == 0 && i < cnt) {
      sh.iv[i] = {y, best, own, cy, e0, e1 - e0};
      sh.islot[i] = slot;
      sh.ir[i] = mt_rank(bg, kq);
      sh.iovf[i] = wtot >= 0x7fffffffLL;
    }
  }
}

// The multi-try rounds of all pairs of the round, in pair order (one
// workgroup: the first wave searches, the others compute gains at its
// request).
// A move depends on the last one, so what counts is the length of a move's
// chain: about 1,500 cycles to pop (an LDS scan and two maxima over the wave),
// 1,400 to decide, 3,000 for a request (four dependent loads that hit the L2,
// two barriers) and 900 to apply it.  Measured on a 3D round of 4 pairs
// (131,072 vertices, mean degree 12, 1,356 searches, 14,018 moves): 44 ms,
// 3.1 us per move.  With one wave, a lane per neighbour and its arcs one
// after the other: 106 ms; with a binary heap kept by lane 0 on top: 272 ms.
// Reading ahead for the neighbours of what joins the queue gave 1 ms of 46
// and isn't done.
__global__ void __launch_bounds__(MT_TPB) k_mt(KArgs A) {
  __shared__ MTShared sh;
  const int lane = lane64();
  const uint64_t seed = (uint64_t)(uint32_t)A.mt_seed;
  if (A.ctl->err != 0) return;
  if (uni((int32_t)threadIdx.x) >= WAVE) {
    for (;;) {
      __syncthreads();
      if (uni(sh.cnt) < 0) return;
      mt_gains(A, sh, seed);
      __syncthreads();
    }
  }
  MTQueue H{A, sh, A.mtr, A.mth};
  H.seed = seed;
  const bool lds_w = A.k <= MT_LBLK;
  // block weights and the blocks above L_max
  int64_t over = 0;
  for (int32_t b = lane; b < A.k; b += WAVE) {
    const int64_t w = A.mtw[b];
    if (lds_w) sh.bw[b] = w;
    over += w > A.lmax ? 1 : 0;
  }
  for (int o = 32; o > 0; o >>= 1) over += __shfl_xor(over, o);
  over = uni64(over);  // (what steers the search stays in scalar registers)
  bool ovf = false;
  // One request and its answer in the lanes (see MTShared).  The barriers also
  // order this wave's stores before them with the other waves' loads.
  struct Answer {
    MTVertex y;
    int32_t slot;
    uint64_t r;
  };
  auto request = [&](int32_t v0, int32_t a0, int32_t cnt, int32_t stamp) -> Answer {
    if (lane == 0) {
      sh.v0 = v0;
      sh.a0 = a0;
      sh.cnt = cnt;
      sh.stamp = stamp;
    }
    __syncthreads();
    __syncthreads();
    const bool on = lane < cnt;
    const int i = on ? lane : 0;
    const MTVertex &iv = sh.iv[i];
    const int32_t v = on ? iv.v : -1;
    if (v >= 0 && sh.iovf[i]) ovf = true;
    return {{v, v >= 0 ? iv.to : -1, iv.from, iv.c, iv.e0, iv.deg}, sh.islot[i], sh.ir[i]};
  };
  const int32_t npair = A.P / A.W;
  for (int32_t q = 0; q < npair; q++) {
    const int32_t p0 = q * A.W;
    const int32_t stamp = A.mt_stamp0 + q + 1;
    const int32_t T = (int32_t)min((int64_t)A.ucnt[p0], A.voff[p0 + 1] - A.voff[p0]);
    const unsigned long long *todo = A.mtk + A.voff[p0];
    int64_t searches = 0, moves = 0, kept = 0;
    // the todo list, 64 entries at a time: the first one not yet touched
    // starts a search, and the marks of the later ones are read again after it
    int32_t mine = -1, at = 0;
    for (int32_t t0 = 0, fresh = 1; t0 < T;) {
      if (fresh) {
        mine = t0 + lane < T ? (int32_t)(uint32_t)todo[t0 + lane] : -1;
        at = 0;
        fresh = 0;
      }
      const u64 open = ballot64(lane >= at && mine >= 0 && A.mtt[mine >= 0 ? mine : 0] != stamp);
      if (open == 0ull) {
        t0 += WAVE;
        fresh = 1;
        continue;
      }
      const int pick = __ffsll(open) - 1;
      const int32_t v = __builtin_amdgcn_readlane(mine, pick);
      at = pick + 1;
      // the start set: v and its untouched boundary neighbours; none when v
      // is no boundary vertex any more
      int64_t delta = 0, best = 0, best_over = over;
      int64_t nmv = 0, best_n = 0, pcount = 0;
      __int128 S1 = 0, S2 = 0;
      const int32_t s0 = uni(A.xadj[v]) - 1, s1 = uni(A.xadj[v + 1]);
      bool start = true;
      for (int32_t c0 = s0; c0 < s1 && start; c0 += MT_ITEMS) {
        const bool was = ovf;
        const Answer a = request(c0 == s0 ? v : -1, c0, min(MT_ITEMS, s1 - c0), stamp);
        if (c0 == s0) start = __builtin_amdgcn_readlane(a.y.to, 0) >= 0;
        if (!start) {
          if (lane > 0) ovf = was;  // only v was looked at
          break;
        }
        if (a.y.to >= 0) A.mtt[a.y.v] = stamp;
        H.push(a.y.to >= 0, a.y, a.r);
      }
      if (!start) continue;
      searches++;
      // the moves
      for (;;) {
        int32_t gx = 0;
        const MTVertex v = H.pop(gx);
        if (v.v < 0) break;
        const int32_t x = v.v, to = v.to, from = v.from;
        const int64_t cx = v.c;
        const int32_t e0 = v.e0, e1 = v.e0 + v.deg;
        int64_t wto = sh.bw[lds_w ? to : 0], wfrom = sh.bw[lds_w ? from : 0];
        asm("" : "+v"(wto), "+v"(wfrom));
        if (!lds_w) {
          wto = A.mtw[to];
          wfrom = A.mtw[from];
          asm volatile("" : "+v"(wto), "+v"(wfrom));
        }
        wto = uni64(wto);
        wfrom = uni64(wfrom);
        if (wto + cx > A.lmax) continue;  // the move would overload its target
        if (wfrom > A.lmax && wfrom - cx <= A.lmax) over--;
        if (lane == 0) {
          if (lds_w) {
            sh.bw[from] = wfrom - cx;
            sh.bw[to] = wto + cx;
          } else {
            A.mtw[from] = wfrom - cx;
            A.mtw[to] = wto + cx;
          }
          A.part[x] = to;
          A.mtv[nmv] = x;
          A.mtf[nmv] = from;
        }
        mt_order();
        nmv++;
        delta -= gx;
        if (over < best_over || (over == best_over && delta < best)) {
          best = delta;
          best_over = over;
          best_n = nmv;
          pcount = 0;
          S1 = S2 = 0;
        } else {
          pcount++;
          S1 += gx;
          S2 += (__int128)gx * gx;
          if (mt_stop(pcount, S1, S2, A.mt_alpha, A.mt_beta)) break;
        }
        // x's neighbours: queued ones get their gain again (or leave without
        // a target), untouched boundary ones join
        for (int32_t c0 = e0; c0 < e1; c0 += MT_ITEMS) {
          const Answer a = request(-1, c0, min(MT_ITEMS, e1 - c0), stamp);
          const bool queued = a.y.v >= 0 && a.slot >= 0, gone = queued && a.y.to < 0,
                     join = a.y.to >= 0 && a.slot < 0;
          if (gone) {
            H.drop(a.slot, a.y.v);
          } else if (queued) {
            H.set_rank(a.slot, a.r);
            H.set_target(a.slot, a.y.v, a.y.to);
          }
          H.live -= (int32_t)__popcll(ballot64(gone));
          if (join) A.mtt[a.y.v] = stamp;
          H.push(join, a.y, a.r);
        }
      }
      // the queue ends empty; roll back the moves after the best state (each
      // vertex moved at most once, so the moves go back in any order)
      H.clear();
      mt_order();
      for (int64_t j = lane; j < nmv; j += WAVE) {
        const int32_t y = A.mtv[j], fr = A.mtf[j], tb = A.part[y];
        if (j >= best_n) {
          const unsigned long long cy = (unsigned long long)(int64_t)A.vwgt[y];
          if (lds_w) {
            atomicAdd(reinterpret_cast<unsigned long long *>(sh.bw) + tb, 0ull - cy);
            atomicAdd(reinterpret_cast<unsigned long long *>(sh.bw) + fr, cy);
          } else {
            atomicAdd(reinterpret_cast<unsigned long long *>(A.mtw) + tb, 0ull - cy);
            atomicAdd(reinterpret_cast<unsigned long long *>(A.mtw) + fr, cy);
          }
          A.part[y] = fr;
        } else {
          A.mtchg[fr] = 1;
          A.mtchg[tb] = 1;
        }
      }
      // weights changed by atomics in device memory are read by plain loads
      if (!lds_w) __threadfence();
      mt_order();
      over = best_over;
      moves += nmv;
      kept += best_n;
    }
    if (lane == 0) {
      PairState &ps = A.ps[p0];
      ps.mt_searches += searches;
      ps.mt_moves += moves;
      ps.mt_kept += kept;
    }
  }
  if (lane == 0) sh.cnt = -1;  // the other waves leave
  __syncthreads();
  for (int o = 32; o > 0; o >>= 1) ovf |= __shfl_xor((int)ovf, o) != 0;
  if (lane == 0 && ovf) {
    A.ctl->err = FR_E_OVERFLOW;
    A.ctl->diag = DIAG_MT;
  }
}
