// Row network: the corridor network laid out for short dependent-load chains.
//
// What bounds the flow kernel is the latency of its chains, not bandwidth: a
// relabel level or a push/relabel pass handles a few hundred vertices, and
// every step of it waits for the slowest load.  In the CSR form a step reads
// the vertex's offsets, then its 16-byte arc records, then (in a pass) the
// heads' labels: three loads one after the other.  Here a vertex's arcs sit
// at a fixed place, one 128-byte row per vertex (a cache line, read by 8
// lanes with one 16-byte load each), and an arc is one 8-byte word that holds
// its head and both residuals; with the labels in LDS a step waits for one
// load.
//
// Row of vertex i: 16 words at 16 * i.  Word 0 is the header (arc count in
// the high half, first overflow row in the low half), words 1..15 are arcs,
// unused words are 0 (no residual either way, so every lane may read all).
// Arcs past the 15th follow in the vertex's overflow rows, 16 to a row, at
// 16 * (nr + first overflow row).
//
// Arc word: bits 0-15 own residual, 16-31 residual of the reverse arc,
// 32-57 head, 58-63 the reverse arc's slot in the head's row.  A push of x
// along an arc adds (x << 16) - x to its word and x - (x << 16) to the reverse
// arc's: no borrow or carry crosses the halves, as residuals stay in
// [0, 2 * weight].
//
// The form takes networks with edge weights up to 32,767, at most 63 arcs per
// vertex, and rows that fit the entry's arc slice; the others keep the CSR
// form (Arc records of any weight and degree).  Both give the same results.
// Measured on a round of 8 pairs (2D, 2^20 vertices, mean degree 8): 43 ms
// with rows in all entries but one hub's, 113 ms with every entry in the CSR
// form, where what k_net_count writes of the rows before it finds the misfit
// is lost, and 125 ms in that form before there were rows.
#pragma once  // included by fr_kernels.h, after its wave and list helpers

typedef unsigned long long u64;
typedef __attribute__((ext_vector_type(2))) unsigned long long u64x2;

#define ROW_WORDS 16
#define ROW_SLOTS 15       // arcs in a vertex's own row
#define ROW_MAX_DEG 63     // slots fit 6 bits
#define ROW_MAX_W 32767    // own + reverse residual fit 16 bits each
#define ROW_RAW 63         // slot of a word whose reverse arc has not been found yet

__device__ __forceinline__ int32_t row_own(u64 x) { return (int32_t)((uint32_t)x & 0xffffu); }
__device__ __forceinline__ int32_t row_rev(u64 x) { return (int32_t)((uint32_t)x >> 16); }
__device__ __forceinline__ int32_t row_head(u64 x) {
  return (int32_t)((uint32_t)(x >> 32) & 0x3ffffffu);
}
__device__ __forceinline__ int32_t row_rslot(u64 x) { return (int32_t)(uint32_t)(x >> 58); }
__device__ __forceinline__ u64 row_word(int32_t own, int32_t rev, int32_t head, int32_t rslot) {
  return ((u64)(uint32_t)rslot << 58) | ((u64)(uint32_t)head << 32) |
         ((u64)(uint32_t)rev << 16) | (u64)(uint32_t)own;
}
__device__ __forceinline__ int32_t row_overflow(int32_t deg) {  // overflow rows of deg arcs
  return deg > ROW_SLOTS ? (deg - ROW_SLOTS + ROW_WORDS - 1) / ROW_WORDS : 0;
}

// Index of the word at `slot` of vertex i.
__device__ __forceinline__ int64_t row_index(const u64 *L, int32_t nr, int32_t i, int32_t slot) {
  if (slot < ROW_SLOTS) return (int64_t)ROW_WORDS * i + 1 + slot;
  const int32_t ovf = (int32_t)(uint32_t)L[(int64_t)ROW_WORDS * i];
  return (int64_t)ROW_WORDS * ((int64_t)nr + ovf) + (slot - ROW_SLOTS);
}

// ---- lane groups (G = 2, 4 or 8 consecutive lanes, 16 for reductions) on the DPP crossbar: a
//      step costs a few cycles where a bpermute through LDS costs tens.  All
//      64 lanes of the wave take part.
template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false);
}
#define DPP_XOR1 0xB1        // quad_perm [1,0,3,2]
#define DPP_XOR2 0x4E        // quad_perm [2,3,0,1]
#define DPP_HALF_MIRROR 0x141  // lane i of 8 reads lane 7 - i
#define DPP_MIRROR 0x140     // lane i of 16 reads lane 15 - i
#define DPP_SHR(n) (0x110 | (n))

// value of the group's first lane
template <int G>
__device__ __forceinline__ int32_t group_first(int32_t x) {
  if (G == 2) return dpp<0xA0>(x);  // quad_perm [0,0,2,2]
  x = dpp<0x00>(x);                 // quad_perm [0,0,0,0]
  if (G == 4) return x;
  const int32_t t = dpp<DPP_SHR(4)>(x);
  return (lane64() & 4) ? t : x;
}

template <int G, typename Op>
__device__ __forceinline__ int32_t group_reduce(int32_t x, Op &&op) {
  x = op(x, dpp<DPP_XOR1>(x));
  if (G >= 4) x = op(x, dpp<DPP_XOR2>(x));
  if (G >= 8) x = op(x, dpp<DPP_HALF_MIRROR>(x));
  if (G >= 16) x = op(x, dpp<DPP_MIRROR>(x));
  return x;
}

template <int G>
__device__ __forceinline__ int32_t group_sum(int32_t x) {
  return group_reduce<G>(x, [](int32_t a, int32_t b) { return a + b; });
}

template <int G>
__device__ __forceinline__ int32_t group_min(int32_t x) {
  return group_reduce<G>(x, [](int32_t a, int32_t b) { return a < b ? a : b; });
}

// sum over the wave, the same in every lane
__device__ __forceinline__ int32_t wave_sum(int32_t x) {
  const int32_t m = group_sum<16>(x);
  return __builtin_amdgcn_readlane(m, 0) + __builtin_amdgcn_readlane(m, 16) +
         __builtin_amdgcn_readlane(m, 32) + __builtin_amdgcn_readlane(m, 48);
}

// inclusive prefix sum over the group's lanes
template <int G>
__device__ __forceinline__ int32_t group_scan(int32_t x) {
  const int gl = lane64() & (G - 1);
  int32_t t = dpp<DPP_SHR(1)>(x);
  x += gl >= 1 ? t : 0;
  if (G >= 4) {
    t = dpp<DPP_SHR(2)>(x);
    x += gl >= 2 ? t : 0;
  }
  if (G >= 8) {
    t = dpp<DPP_SHR(4)>(x);
    x += gl >= 4 ? t : 0;
  }
  return x;
}

// The lane's index, opaque to the optimiser: what is computed from it stays
// in the step that uses it.  (Hoisted out of the solver's main loop, the lane
// offsets of every group width together spill registers.)
__device__ __forceinline__ int32_t step_lane() {
  int32_t t = (int32_t)threadIdx.x & 63;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ u64 ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int32_t lanes_below(u64 m) {
  return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Appends the K values v[k] of each lane with want[k] set to a list whose
// first FR_LDS_LIST entries lie in LDS (s) and the rest in global memory (g,
// cap entries): one LDS atomic per wave for all of them.  Converged wave
// only.
template <int K>
__device__ __forceinline__ void wave_append_many(int32_t *s, int32_t *g, int64_t cap,
                                                 int32_t *counter, const bool (&want)[K],
                                                 const int32_t (&v)[K], Ctl *ctl) {
  u64 m[K];
  int32_t total = 0;
#pragma unroll
  for (int k = 0; k < K; k++) {
    m[k] = ballot64(want[k]);
    total += (int32_t)__popcll(m[k]);
  }
  if (total == 0) return;
  int32_t base = 0;
  if (lanes_below(~0ull) == 0) base = atomicAdd(counter, total);
  base = uni(base);
  if (base + total <= FR_LDS_LIST) {
#pragma unroll
    for (int k = 0; k < K; k++) {
      if (want[k]) s[base + lanes_below(m[k])] = v[k];
      base += (int32_t)__popcll(m[k]);
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int32_t pos = base + lanes_below(m[k]);
    base += (int32_t)__popcll(m[k]);
    if (!want[k]) continue;
    if (pos < FR_LDS_LIST) s[pos] = v[k];
    else put_bounded(g, pos, cap, v[k], ctl);
  }
}

// Lanes per row for `cnt` rows in a workgroup of TPB threads: 8 (a row in
// one load per lane) while that takes one pass, else 4, else 2 -- a pass more
// pays the step's load latency again, a narrower group only more loads in
// flight per lane.  (Fewer lanes also mean fewer wave instructions per row,
// which count once all waves of a SIMD are busy.)
template <int G>
struct RowLanes {
  static constexpr int g = G, k = ROW_WORDS / G;
};

template <int TPB, typename F>
__device__ __forceinline__ void by_row_width(int32_t cnt, F &&f) {
  if (cnt * 8 <= TPB) f(RowLanes<8>{});
  else if (cnt * 4 <= TPB) f(RowLanes<4>{});
  else f(RowLanes<2>{});
}

// The lane's K words of the row at `row` (zeros when off).
template <int K>
__device__ __forceinline__ void row_load(const u64 *L, int64_t row, int gl, bool on, u64 (&x)[K]) {
  // (rows lie within 4 GB: a scalar base and a 32-bit offset)
  const u64x2 *R = reinterpret_cast<const u64x2 *>(reinterpret_cast<const char *>(L) +
                                                   ((uint32_t)row * 128u + (uint32_t)(8 * K * gl)));
#pragma unroll
  for (int k = 0; k < K; k += 2) {
    u64x2 v = {0ull, 0ull};
    if (on) v = R[k / 2];
    x[k] = v.x;
    x[k + 1] = v.y;
  }
}

// Distance labels of the flow phases: 16-bit in LDS, or the entry's global
// label array.
template <bool LL>
struct Labels {
  uint16_t *s;
  int32_t *g;
  __device__ __forceinline__ int32_t get(int32_t v) const { return LL ? (int32_t)s[v] : g[v]; }
  __device__ __forceinline__ void set(int32_t v, int32_t d) const {
    if (LL) s[v] = (uint16_t)d;
    else g[v] = d;
  }
};

// LDS of the row solver for nr vertices: two bitmaps, two list heads and,
// when they fit, 16-bit labels.
__host__ __device__ __forceinline__ int64_t row_bm_words(int64_t nr) {
  return ((nr + 63) >> 6) * 2;
}
__host__ __device__ __forceinline__ int64_t row_lds_bytes(int64_t nr) {
  return 8 * (int64_t)FR_LDS_LIST + 8 * row_bm_words(nr);
}
__host__ __device__ __forceinline__ int64_t row_label_bytes(int64_t nr) {
  return 2 * ((nr + 7) & ~7ll);
}
#define ROW_LABEL_MAX 65533  // labels reach nr + 2

// Whether the entry's network takes the row form: every vertex fit (net_count
// counts the others), its rows fit the arc slice and its bitmaps the flow
// kernel's LDS.
__device__ __forceinline__ bool rows_possible(const KArgs &A, int32_t p) {
  const int64_t nr = A.ps[p].nr;
  return nr <= A.row_nr && (A.aoff[p] & 7) == 0 && 8 * nr <= A.aoff[p + 1] - A.aoff[p];
}
__device__ __forceinline__ bool rows_chosen(const KArgs &A, int32_t p) {
  return rows_possible(A, p) && A.pacc[(int64_t)p * PA_N + PA_MISFIT] == 0;
}
__device__ __forceinline__ u64 *rows_of(const KArgs &A, int32_t p) {
  return reinterpret_cast<u64 *>(A.arc + A.aoff[p]);
}

// `want` consecutive overflow rows of entry p (its counter in ctr[p]): one
// atomic per wave while its lanes share the entry, as nearly all do.
// Converged wave only; lanes with want = 0 get 0.
__device__ __forceinline__ int32_t rows_take(int32_t *ctr, int32_t p, int32_t want) {
  const u64 m = __ballot(want > 0);
  if (m == 0ull) return 0;
  const int leader = __ffsll(m) - 1;
  const int32_t p0 = __shfl(p, leader);
  if (__any(want > 0 && p != p0)) return want > 0 ? atomicAdd(ctr + p, want) : 0;
  int32_t inc = want;
  for (int o = 1; o < WAVE; o <<= 1) {
    const int32_t t = __shfl_up(inc, o);
    if (lane64() >= o) inc += t;
  }
  const int32_t total = __shfl(inc, WAVE - 1);
  int32_t base = 0;
  if (lane64() == leader) base = atomicAdd(ctr + p0, total);
  base = __shfl(base, leader);
  return want > 0 ? base + inc - want : 0;
}
