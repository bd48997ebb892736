// Multi-try FM (Sanders & Schulz, Section 4.2) on the GPU: after the
// pairwise improvements of a round, one round of localized k-way searches per
// pair, in pair order.
//
// The k-way local search of Section 2.2 moves a vertex to the adjacent block
// with the largest gain, so a search of one pair can reach any block: the
// searches of a round's pairs are not independent, and they run one after
// the other, in one wave.  Around them the work is spread over the chip:
//   k_mt_weights  block weights of all k blocks (grid-wide)
//   k_mt_todo     each pair's todo list: the vertices of its two blocks with
//                 a neighbour in another block, as sort keys (upper 32 bits
//                 of a SplitMix64 output, then the id), grid-wide
//   k_mt_sort     each todo list in key order (one workgroup per pair:
//                 bitonic in LDS, a tiled rank sort beyond)
//   k_mt          the searches (one wave): a flat queue of (gain, key, vertex)
//                 in LDS that spills to device memory, popped by a wave-wide
//                 maximum and updated by all lanes at once; each neighbour's
//                 k-way gain computed by a lane of its own; KaSPar's stopping
//                 rule in exact integer arithmetic; rollback to the best
//                 state.
// The counters of the keys (SplitMix64 outputs from mt_seed): todo order of v
// 2^40 + v + 1, queue order of v 2^41 + v + 1, tie key of target block P of v
// 2^42 + v k + P + 1.
#pragma once
#include "fr_kernels.h"

#define MT_SORT_TPB 1024
#define MT_LSORT 8192   // todo keys sorted in LDS
#define MT_LQ 3072      // queue entries in LDS (the rest in device memory)
#define MT_SCAN 256     // a queue of up to this many entries is scanned whole
#define MT_NB 1024      // groups of 64 queue entries with a bound in LDS
#define MT_LBLK 2048    // block weights held in LDS
#define MT_CH 16        // arcs of a vertex examined together by its lane

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

// The search state of the one wave.  The queue is a flat array in arrival
// order; an entry is a rank (gain, then the key's upper half) and its vertex,
// rank 0 once it has left; the entries are packed again when most have left.
// Every vertex enters the queue at most once per round of a pair.
struct MTShared {
  uint64_t qr[MT_LQ];    // queue entries in LDS
  int32_t qv[MT_LQ];
  uint64_t bound[MT_NB];  // no rank of entries [64 b, 64 b + 64) is above
  int64_t bw[MT_LBLK];   // block weights (k <= MT_LBLK)
};

// Orders this lane's memory operations with the other lanes' for the
// compiler (the hardware keeps a wave's in order).
__device__ __forceinline__ void mt_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ uint64_t read_lane64(uint64_t x, int l) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(x >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int32_t)x, l);
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
  // Ranks order entries by gain, then by the upper half of the key.
  __device__ __forceinline__ uint64_t rank(int32_t v, int32_t g) const {
    return ((uint64_t)((uint32_t)g ^ 0x80000000u) << 32) | (key(v) >> 32);
  }
  __device__ __forceinline__ uint64_t rank_at(int32_t i) const {
    uint64_t r = sh.qr[min(i, MT_LQ - 1)];  // two loads, not one from either space
    asm("" : "+v"(r));
    if (i >= MT_LQ) r = gr[i];
    return r;
  }
  __device__ __forceinline__ int32_t vertex_at(int32_t i) const {
    int32_t v = sh.qv[min(i, MT_LQ - 1)];
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
  __device__ __forceinline__ void set(int32_t i, int32_t v, uint64_t r) {
    if (i < MT_LQ) sh.qv[i] = v;
    else gv[i] = v;
    set_rank(i, r);
    A.mtq[v] = i;
  }
  __device__ __forceinline__ void drop(int32_t i, int32_t v) {  // entry i (vertex v) leaves
    if (i < MT_LQ) sh.qr[i] = 0;
    else gr[i] = 0;
    A.mtq[v] = -1;
  }
  // The lanes with want join with their vertex and gain.
  __device__ __forceinline__ void push(bool want, int32_t v, int32_t g) {
    const u64 m = ballot64(want);
    if (want) {
      const int32_t i = len + lanes_below(m);
      if ((i & 63) == 0 && i < 64 * MT_NB) sh.bound[i >> 6] = 0;
      mt_order();
      set(i, v, rank(v, g));
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
      int32_t v = -1;
      if (i < len) {
        r = rank_at(i);
        v = vertex_at(i);
      }
      mt_order();
      if (lane64() == 0 && b0 < 64 * MT_NB) sh.bound[b0 >> 6] = 0;  // group b0 / 64 is read
      const u64 m = ballot64(r != 0);
      mt_order();
      if (r != 0) set(to + lanes_below(m), v, r);  // at most i: read already
      mt_order();
      to += (int32_t)__popcll(m);
    }
    len = to;
  }
  // Takes the entry with the largest gain, then the largest key (keys are
  // distinct: the generator's finaliser is a bijection): its vertex and gain
  // in every lane; -1 when the queue is empty.
  __device__ __forceinline__ int32_t pop(int32_t &gain) {
    if (live == 0) return -1;
    if (len > 2 * live + MT_SCAN) pack();
    mt_order();
    for (;;) {
      uint64_t top = 0;  // this lane's best entry
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
      const bool groups = len > MT_SCAN;
      const int32_t ng = groups ? min((len + 63) >> 6, MT_NB) : 0;
      uint64_t lead = 0;  // the largest bound
      for (int32_t b = lane64(); b < ng; b += WAVE) lead = max(lead, sh.bound[b]);
      for (int o = 32; o > 0; o >>= 1) {
        const uint64_t x = __shfl_xor((unsigned long long)lead, o);
        lead = max(lead, x);
      }
      for (int32_t b0 = 0; b0 < ng; b0 += WAVE) {  // the groups that may hold it
        const int32_t b = b0 + lane64();
        for (u64 m = ballot64(b < ng && sh.bound[b < ng ? b : 0] == lead); m; m &= m - 1) {
          const int32_t g = b0 + __ffsll(m) - 1, i = 64 * g + lane64();
          const uint64_t r = i < len ? rank_at(i) : 0ull;
          if (i < len) look(i);
          uint64_t hi = r;
          for (int o = 32; o > 0; o >>= 1) {
            const uint64_t x = __shfl_xor((unsigned long long)hi, o);
            hi = max(hi, x);
          }
          mt_order();
          if (lane64() == 0) sh.bound[g] = hi;  // exact again
          mt_order();
        }
      }
      for (int32_t i = 64 * ng + lane64(); i < len; i += WAVE) look(i);
      // the best of all lanes: by rank, equal ranks by the whole key
      uint64_t hi = top;
      for (int o = 32; o > 0; o >>= 1) {
        const uint64_t x = __shfl_xor((unsigned long long)hi, o);
        hi = max(hi, x);
      }
      if (hi < lead) continue;  // the bounds were above every rank: they are lower now
      u64 m = ballot64(at >= 0 && top == hi);
      if (m == 0ull) return -1;  // only after an overflow, which is reported
      int win = __ffsll(m) - 1;
      if (m & (m - 1)) {
        const uint64_t k = key(v);
        for (m &= m - 1; m; m &= m - 1) {
          const int l = __ffsll(m) - 1;
          if (read_lane64(k, l) > read_lane64(k, win)) win = l;
        }
      }
      const int32_t x = __builtin_amdgcn_readlane(v, win);
      const int32_t i = __builtin_amdgcn_readlane(at, win);
      gain = (int32_t)((uint32_t)(hi >> 32) ^ 0x80000000u);
      if (lane64() == 0) drop(i, x);
      live--;
      return x;
    }
  }
  __device__ __forceinline__ void clear() {
    for (int32_t i = lane64(); i < len; i += WAVE)
      if (rank_at(i) != 0) A.mtq[vertex_at(i)] = -1;
    len = live = 0;
  }
};

// The k-way gain of vertex y (each lane for its own y, y < 0: none; all lanes
// of the wave call it): over the blocks other than y's own that hold a
// neighbour of y, the largest weight to that block minus the weight to y's
// own block; the block reaching it is the target (equal gains: the smaller
// tie key).  Returns the target or -1 when y has no neighbour outside its
// block; *ovf is set when a weighted degree reaches 2^31.  Up to 2 MT_CH arcs
// are read together and stay in registers; the foreign blocks are then taken
// in ascending order, one sum over the arcs each (a vertex has neighbours in
// few blocks).  A vertex with more arcs is taken by all lanes together, which
// read its arcs once and once more per foreign block.
__device__ __forceinline__ int32_t mt_gain(const KArgs &A, int32_t y, uint64_t seed,
                                           int32_t *gain, bool *ovf) {
  constexpr int32_t NONE = 0x7fffffff;
  const int32_t e0 = y >= 0 ? A.xadj[y] : 0, e1 = y >= 0 ? A.xadj[y + 1] : 0;
  const int32_t own = y >= 0 ? A.part[y] : -1;
  int32_t best = -1;
  int64_t bg = 0;
  uint64_t bk = 0;
  auto consider = [&](int32_t P, int64_t gP) {
    const uint64_t kP = mt_key(seed, 2, (uint64_t)(uint32_t)y * (uint64_t)A.k + (uint64_t)P);
    if (best < 0 || gP > bg || (gP == bg && kP < bk)) {
      best = P;
      bg = gP;
      bk = kP;
    }
  };
  const bool large = e1 - e0 > 2 * MT_CH;
  const bool two = __any(!large && e1 - e0 > MT_CH);
  int64_t wown = 0, wtot = 0;
  int32_t P = NONE;  // the next foreign block
  int32_t b[2 * MT_CH], w[2 * MT_CH];  // the heads' blocks (-1 past the end), weights
  auto half = [&](int h) {
#pragma unroll
    for (int j = h; j < h + MT_CH; j++) {
      const bool in = !large && e0 + j < e1;
      w[j] = in ? A.adjwgt[e0 + j] : 0;
      b[j] = in ? A.adjncy[e0 + j] : -1;
    }
  };
  auto begin = [&](int h) {
#pragma unroll
    for (int j = h; j < h + MT_CH; j++) b[j] = b[j] >= 0 ? A.part[b[j]] : -1;
#pragma unroll
    for (int j = h; j < h + MT_CH; j++) {
      wtot += w[j];
      if (b[j] == own) wown += w[j];
      if (b[j] >= 0 && b[j] != own && b[j] < P) P = b[j];
    }
  };
  half(0);
  if (two) half(MT_CH);
  begin(0);
  if (two) begin(MT_CH);
  while (__any(P != NONE)) {
    int64_t s = 0;
    int32_t next = NONE;
    auto add = [&](int h) {
#pragma unroll
      for (int j = h; j < h + MT_CH; j++) {
        if (b[j] == P) s += w[j];
        if (b[j] > P && b[j] != own && b[j] < next) next = b[j];
      }
    };
    add(0);
    if (two) add(MT_CH);
    if (P != NONE) {
      consider(P, s - wown);
      P = next;
    }
  }
  for (u64 m = ballot64(large); m; m &= m - 1) {
    const int l = __ffsll(m) - 1;
    const int32_t f0 = __builtin_amdgcn_readlane(e0, l), f1 = __builtin_amdgcn_readlane(e1, l);
    const int32_t mine = __builtin_amdgcn_readlane(own, l);
    int64_t wo = 0, wt = 0;
    int32_t Q = -1;
    for (;;) {  // the own block's sum first, then one block after the other
      const bool own_pass = Q < 0;
      const int32_t want = own_pass ? mine : Q;
      int64_t s = 0, all = 0;
      int32_t next = NONE;
      for (int32_t e = f0 + lane64(); e < f1; e += WAVE) {
        const int32_t c = A.part[A.adjncy[e]], x = A.adjwgt[e];
        all += x;
        if (c == want) s += x;
        if (c > Q && c != mine && c < next) next = c;
      }
      for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor((long long)s, o);
        all += __shfl_xor((long long)all, o);
        next = min(next, __shfl_xor(next, o));
      }
      if (own_pass) {
        wo = s;
        wt = all;
      } else if (lane64() == l) {
        consider(Q, s - wo);
      }
      if (next == NONE) break;
      Q = next;
    }
    if (lane64() == l) wtot = wt;
  }
  if (wtot >= 0x7fffffffLL) *ovf = true;
  *gain = (int32_t)bg;
  return best;
}

// KaSPar's stopping rule: p moves since the last best state with gain sum S1
// and square sum S2 stop the search when p mu^2 > alpha sigma^2 + ln n, i.e.
// 2^16 (p S1^2 - alpha (p S2 - S1^2)) > beta_fx p^2 with beta_fx = floor(ln n
// 2^16).
__device__ __forceinline__ bool mt_stop(int64_t p, __int128 S1, __int128 S2, int32_t alpha,
                                        int64_t beta_fx) {
  if (p < 4096 && S1 > -4096 && S1 < 4096 && S2 < (1 << 24) && alpha < 1024) {  // fits 64 bits
    const int64_t a = (int64_t)S1, b = (int64_t)S2;
    return (p * a * a - alpha * (p * b - a * a)) * 65536 > beta_fx * p * p;
  }
  const __int128 lhs =
      ((__int128)p * S1 * S1 - (__int128)alpha * ((__int128)p * S2 - S1 * S1)) * 65536;
  return lhs > (__int128)beta_fx * p * p;
}

// The multi-try rounds of all pairs of the round, in pair order (one wave).
// A move depends on the last one, so what counts is the length of a move's
// chain.  Measured on a 3D round of 4 pairs (131,072 vertices, mean degree 12,
// 1,356 searches, 14,018 moves): 106 ms, 7.6 us per move; with the queue as a
// binary heap kept by lane 0 and vertices of more than 16 arcs summed by
// nested loops over their arcs 272 ms, 19.4 us per move.
__global__ void __launch_bounds__(WAVE) k_mt(KArgs A) {
  __shared__ MTShared sh;
  const int lane = lane64();
  const uint64_t seed = (uint64_t)(uint32_t)A.mt_seed;
  if (A.ctl->err != 0) return;
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
  bool ovf = false;
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
      // the start set: v and its untouched boundary neighbours, a lane each;
      // none when v is no boundary vertex any more
      int64_t delta = 0, best = 0, best_over = over;
      int64_t nmv = 0, best_n = 0, pcount = 0;
      __int128 S1 = 0, S2 = 0;
      bool start = true;
      {
        const int32_t e0 = uni(A.xadj[v]), e1 = uni(A.xadj[v + 1]);
        for (int32_t c0 = e0 - 1; c0 < e1 && start; c0 += WAVE) {
          const int32_t e = c0 + lane;
          int32_t y = -1;
          if (e == e0 - 1) y = v;
          else if (e < e1) y = A.adjncy[e];
          if (y >= 0 && y != v && A.mtt[y] == stamp) y = -1;
          int32_t g = 0;
          bool o2 = false;
          const int32_t t = mt_gain(A, y, seed, &g, &o2);
          if (c0 == e0 - 1) {
            start = __builtin_amdgcn_readlane(t, 0) >= 0;
            if (!start) {
              ovf |= o2 && lane == 0;
              break;
            }
          }
          ovf |= o2;
          if (t >= 0) {
            A.mtt[y] = stamp;
            A.mtb[y] = t;
          }
          H.push(t >= 0, y, g);
        }
      }
      if (!start) continue;
      searches++;
      // the moves
      for (;;) {
        int32_t gx = 0;
        const int32_t x = H.pop(gx);
        if (x < 0) break;
        const int32_t to = uni(A.mtb[x]), from = uni(A.part[x]);
        const int64_t cx = uni(A.vwgt[x]);
        const int32_t e0 = uni(A.xadj[x]), e1 = uni(A.xadj[x + 1]);
        int64_t wto = sh.bw[lds_w ? to : 0], wfrom = sh.bw[lds_w ? from : 0];
        asm("" : "+v"(wto), "+v"(wfrom));
        if (!lds_w) {
          wto = A.mtw[to];
          wfrom = A.mtw[from];
        }
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
        // a target), untouched boundary ones join; a lane each
        for (int32_t c0 = e0; c0 < e1; c0 += WAVE) {
          const int32_t e = c0 + lane;
          int32_t y = e < e1 ? A.adjncy[e] : -1;
          int32_t slot = -1;
          if (y >= 0) {
            slot = A.mtq[y];
            if (slot < 0 && A.mtt[y] == stamp) y = -1;  // touched, not queued
          }
          int32_t g = 0;
          bool o2 = false;
          const int32_t t = mt_gain(A, y, seed, &g, &o2);
          ovf |= o2;
          if (t >= 0) A.mtb[y] = t;
          const bool gone = y >= 0 && slot >= 0 && t < 0, join = y >= 0 && slot < 0 && t >= 0;
          if (gone) H.drop(slot, y);
          else if (y >= 0 && slot >= 0) H.set_rank(slot, H.rank(y, g));
          H.live -= (int32_t)__popcll(ballot64(gone));
          if (join) A.mtt[y] = stamp;
          H.push(join, y, g);
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
  for (int o = 32; o > 0; o >>= 1) ovf |= __shfl_xor((int)ovf, o) != 0;
  if (lane == 0 && ovf) {
    A.ctl->err = FR_E_OVERFLOW;
    A.ctl->diag = DIAG_MT;
  }
}
