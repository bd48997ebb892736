// Maximum preflow, smallest source set and the candidate's record (Sec. 4.1,
// 4.1.1): one workgroup per entry.  Included by fr_kernels.h.
//
// Two forms of the corridor network share the control loop: rows
// (fr_rows.h), and CSR with 16-byte arc records for the networks that the
// rows do not take.
#pragma once

// Counts and device-clock times of an entry's flow in one launch.
struct FlowStats {
  int64_t gr_levels = 0, sweeps = 0, relabels = 0, cl_levels = 0;
  int64_t t_rel = 0, t_push = 0;
  bool sliced = false;
};

// ---- CSR form ------------------------------------------------------------
template <int TPB>
struct CsrSolver {
  const KArgs &A;
  const PairView &V;
  SolveShared<TPB> &sh;
  Rot &R;
  int32_t nr, NL;
  bool lds;
  ListRef cur, nxt;

  __device__ __forceinline__ int32_t relabel(int64_t &levels) {
    const int32_t cnt = global_relabel<TPB>(A, V, nr, NL, sh, R, levels, lds);
    cur = flist(V, sh, 0, lds);
    nxt = flist(V, sh, 1, lds);
    return cnt;
  }

  __device__ __forceinline__ int32_t pass(int32_t cnt, int32_t since) {
    // queued marks of this pass in bm[(since + 1) & 1]; the other bitmap
    // (the previous pass's marks, or the relabel's visited marks) is
    // cleared now and serves the next pass
    uint32_t *qbm = nullptr;
    if (lds) {
      qbm = sh.u.f.bm[(since + 1) & 1];
      uint32_t *old = sh.u.f.bm[since & 1];
      for (int w = threadIdx.x; w < (nr + 31) >> 5; w += TPB) old[w] = 0u;
    }
    pr_sweep_any<TPB>(A, V, cur, cnt, nxt, &sh.cnt[(R.c + 1) % 3], NL, sh.work, qbm);
    return advance();
  }

  __device__ __forceinline__ int32_t advance() {
    if (threadIdx.x == 0) sh.cnt[(R.c + 2) % 3] = 0;
    __syncthreads();
    R.c = (R.c + 1) % 3;
    const ListRef t = cur;
    cur = nxt;
    nxt = t;
    return uni(min(sh.cnt[R.c], (int32_t)V.nv));
  }

  // smallest source set: closure of the source border and of every vertex
  // left with excess, over arcs with residual capacity
  __device__ __forceinline__ void closure(int64_t &levels) {
    uint32_t *vis = sh.u.f.bm[0];
    nxt = flist(V, sh, 0, lds);
    cur = flist(V, sh, 1, lds);
    int32_t *ncnt = &sh.cnt[(R.c + 1) % 3];
    BLOCK_WAVE_LOOP(i, nr) {
      bool seed = false;
      if (i < nr) {
        const uint32_t f = V.fl[i];
        seed = LF_SRC(f) || (!LF_SNK(f) && V.ex[i] > 0);
        V.ins[i] = seed ? 1 : 0;
      }
      if (lds) {
        const unsigned long long m = __ballot(seed);
        if (lane64() == 0) vis[i >> 5] = (uint32_t)m;
        if (lane64() == 32) vis[i >> 5] = (uint32_t)(m >> 32);
      }
      const int pos = wave_append(ncnt, seed);
      if (seed) lput(nxt, pos, V.nv, (int32_t)i, A.ctl);
    }
    int32_t cnt = advance();
    while (cnt > 0) {
      int32_t *ncnt2 = &sh.cnt[(R.c + 1) % 3];
      for_groups<GTF>(cnt, [&](int item, bool valid, int gl) {
        const int32_t u = valid ? lget(cur, item) : 0;
        const int32_t e0 = valid ? V.lo[u] : 0, e1 = valid ? V.lo[u + 1] : 0;
        count_work(sh, W_CL_ITEMS, (valid && gl == 0) ? 1 : 0);
        count_work(sh, W_CL_ARCS, (valid && gl == 0) ? e1 - e0 : 0);
        for (int32_t c0 = e0; c0 < e1; c0 += GTF * KF) {
          int32_t v[KF], r[KF];
#pragma unroll
          for (int k = 0; k < KF; k++) {
            const int32_t ar = c0 + k * GTF + gl;
            Arc x = {0, 0, 0ull};
            if (ar < e1) x = V.arc[ar];
            r[k] = res_own(x.rc);
            v[k] = x.lh;
          }
#pragma unroll
          for (int k = 0; k < KF; k++) {
            bool claim = false;
            if (r[k] > 0) {
              if (lds) {
                const bool seen = (vis[v[k] >> 5] >> (v[k] & 31)) & 1u;
                if (!seen) {
                  claim = bm_claim(vis, v[k]);
                  if (claim) V.ins[v[k]] = 1;
                }
              } else if (V.ins[v[k]] == 0) {
                claim = atomicCAS(&V.ins[v[k]], 0, 1) == 0;
              }
            }
            const int pos = wave_append(ncnt2, claim);
            if (claim) lput(nxt, pos, V.nv, v[k], A.ctl);
          }
        }
      });
      cnt = advance();
      levels++;
    }
  }

  // (its steps count as they go)
  __device__ __forceinline__ void count_step() {}
  __device__ __forceinline__ void count_end() {}
};

// ---- row form ------------------------------------------------------------
// Same algorithm, one load per step: list entry (LDS) -> row (one cache
// line) -> labels and marks (LDS).  LL: the labels lie in LDS (corridors up
// to about 60,000 vertices with one workgroup per CU), else in the entry's
// global label array.  The bound is the latency of a step's chain.  Measured
// against the CSR form: a matching round of 32 pairs (2D, 65,536-vertex
// blocks, mean degree 6) takes 1.15 us per relabel level instead of 3.2 and
// 2.0 us per pass instead of 5.1, its flow kernels 30 ms instead of 84; one
// pair of 131,072-vertex blocks (global labels) 49 ms instead of 110.
template <int TPB, bool LL>
struct RowSolver {
  const KArgs &A;
  const PairView &V;
  SolveShared<TPB> &sh;
  u64 *L;
  int32_t nr, NL;
  Labels<LL> lab;
  uint32_t *bm0, *bm1;
  int32_t *ls;  // LDS heads of the two lists
  const int32_t wave;
  int32_t from = 1, c_next = 1;  // list read, counter of the list written
  RowWork work;
  uint32_t ahead = 0;

  __device__ __forceinline__ RowSolver(const KArgs &A_, const PairView &V_, SolveShared<TPB> &sh_,
                                       u64 *L_, int32_t nr_)
      : A(A_), V(V_), sh(sh_), L(L_), nr(nr_), NL(nr_ + 2),
        wave(uni((int32_t)threadIdx.x >> 6)) {
    unsigned char *mem = reinterpret_cast<unsigned char *>(&sh.u);
    ls = reinterpret_cast<int32_t *>(mem);
    bm0 = reinterpret_cast<uint32_t *>(mem + 8 * FR_LDS_LIST);
    bm1 = bm0 + row_bm_words(nr);
    lab.s = reinterpret_cast<uint16_t *>(bm1 + row_bm_words(nr));
    lab.g = V.lab;
    // the border marks, kept as bitmap words in the source-set array (which
    // is written at the end): every relabel starts from them
    uint32_t *border = reinterpret_cast<uint32_t *>(V.ins);
    BLOCK_WAVE_LOOP(i, nr) {
      const u64 m = __ballot(i < nr && (V.fl[i < nr ? i : 0] & LF_BORDER));
      if (lane64() == 0) border[i >> 5] = (uint32_t)m;
      if (lane64() == 32 && i < nr) border[i >> 5] = (uint32_t)(m >> 32);
    }
    __syncthreads();
  }

  // The frontier lists: slots 0 and 1 (their first FR_LDS_LIST entries in
  // LDS); `from` is read, the other one written.  from = 2: the sink list
  // (global memory), slot 0 written.
  __device__ __forceinline__ int32_t get(int32_t item, bool valid, bool in_lds) const {
    const int32_t *s = ls + (from & 1) * FR_LDS_LIST;
    if (in_lds) return s[item];
    // two loads and a select: a load through a selected pointer would be a
    // flat one, which waits for both memories
    const int32_t ns = from == 2 ? 0 : FR_LDS_LIST;
    const int32_t *g = from == 2 ? V.SNK : (from ? V.LB : V.LA);
    const int32_t a = s[min(item, FR_LDS_LIST - 1)];
    const int32_t b = valid && item >= ns ? g[item] : 0;
    return item < ns ? a : b;
  }
  // the whole list (cnt entries, read up to a wave's groups past its end) in LDS
  __device__ __forceinline__ bool list_in_lds(int32_t cnt) const {
    return from != 2 && cnt <= FR_LDS_LIST - WAVE;
  }
  template <int K>
  __device__ __forceinline__ void append(const bool (&want)[K], const int32_t (&v)[K]) {
    const int to = from == 0 ? 1 : 0;
    wave_append_many(ls + to * FR_LDS_LIST, to ? V.LB : V.LA, V.nv, &sh.cnt[c_next], want, v,
                     A.ctl);
  }

  // End of a step: the written list becomes the one to read; its length.
  __device__ __forceinline__ int32_t advance() {
    const int32_t c_clear = uni(c_next == 2 ? 0 : c_next + 1);
    if (wave == 0) sh.cnt[c_clear] = 0;
    __syncthreads();
    const int32_t n = uni(min(sh.cnt[c_next], nr));
    c_next = c_clear;
    from = uni(from == 0 ? 1 : 0);
    return n;
  }

  // One level of a search over the list: REV = backwards (over arcs whose reverse
  // has residual capacity: v can push to w), else forwards.  Heads not yet in
  // bm0 are claimed, labelled (on request) and appended.
  // ahead: the claimed heads' rows, touched here so that the next level finds
  // them in L1 or on their way (kept until the next level's own loads have
  // arrived: nothing waits for it).
  template <int G, bool REV, bool SET>
  __device__ __forceinline__ void level(int32_t cnt, int32_t d, int32_t &arcs) {
    constexpr int K = ROW_WORDS / G;
    const int wf = wave * (WAVE / G);
    if (wf >= cnt) return;  // straight to the step's barrier
    const int32_t ln = step_lane();
    const int gl = ln & (G - 1), grp = ln / G;
    auto claim_words = [&](const u64 (&x)[K]) {
      // the marks of all K heads in flight together (no look before the
      // atomic: it would cost a second LDS round trip per step)
      int32_t h[K];
      uint32_t bit[K], old[K];
#pragma unroll
      for (int k = 0; k < K; k++) {
        h[k] = row_head(x[k]);
        bit[k] = 1u << (h[k] & 31);
        old[k] = ~0u;
        if ((REV ? row_rev(x[k]) : row_own(x[k])) > 0) old[k] = atomicOr(&bm0[h[k] >> 5], bit[k]);
      }
      u64 m[K];
      int32_t total = 0;
#pragma unroll
      for (int k = 0; k < K; k++) {
        m[k] = ballot64(!(old[k] & bit[k]));
        total += (int32_t)__popcll(m[k]);
      }
      if (total == 0) return;
      int32_t at = 0;
      if (ln == 0) at = atomicAdd(&sh.cnt[c_next], total);
      at = uni(at);
      const int to = from == 0 ? 1 : 0;
      int32_t *s = ls + to * FR_LDS_LIST;
      const bool fits = at + total <= FR_LDS_LIST;
#pragma unroll
      for (int k = 0; k < K; k++) {
        const int32_t pos = at + lanes_below(m[k]);
        if (!(old[k] & bit[k])) {
          if (SET) lab.set(h[k], d);
          if (fits || pos < FR_LDS_LIST) s[pos] = h[k];
          ahead = *reinterpret_cast<const uint32_t *>(L + (int64_t)ROW_WORDS * h[k]);
        }
        at += (int32_t)__popcll(m[k]);
      }
      if (!fits) {  // the part of the list beyond LDS
        int32_t *g = to ? V.LB : V.LA;
#pragma unroll
        for (int k = K - 1; k >= 0; k--) {
          at -= (int32_t)__popcll(m[k]);
          const int32_t pos = at + lanes_below(m[k]);
          if (!(old[k] & bit[k]) && pos >= FR_LDS_LIST) put_bounded(g, pos, V.nv, h[k], A.ctl);
        }
      }
    };
    const bool in_lds = list_in_lds(cnt);
    for (int base = wf; base < cnt; base += TPB / G) {
      const int item = base + grp;
      const bool valid = item < cnt;
      const int32_t w = get(item, valid, in_lds);
      u64 x[K];
      row_load<K>(L, w, gl, valid, x);
      int32_t deg = 0, ovf = 0;
      if (gl == 0) {
        deg = (int32_t)(x[0] >> 32);
        ovf = (int32_t)(uint32_t)x[0];
        x[0] = 0ull;
      }
      arcs += deg;
      asm volatile("" ::"v"(ahead));
      claim_words(x);
      if (__any(deg > ROW_SLOTS)) {
        const int32_t more = group_first<G>(row_overflow(deg));
        const int64_t row0 = (int64_t)nr + group_first<G>(ovf);
        for (int32_t j = 0; __any(j < more); j++) {
          row_load<K>(L, row0 + j, gl, j < more, x);
          claim_words(x);
        }
      }
    }
  }

  // Exact distance labels (as global_relabel): returns the active vertices,
  // in the list.
  __device__ __forceinline__ int32_t relabel(int64_t &levels) {
    const bool term = A.terminals != 0;
    const int32_t bw = (int32_t)row_bm_words(nr);
    const int32_t nbw = (nr + 31) >> 5;
    const uint32_t *border = reinterpret_cast<const uint32_t *>(V.ins);
    for (int32_t w = threadIdx.x; w < bw; w += TPB) {
      bm0[w] = w < nbw ? border[w] : 0u;  // no border marks with contracted terminals
      bm1[w] = 0u;
    }
    if (LL) {  // every label NL, four to a store
      const uint32_t two = ((uint32_t)NL << 16) | (uint32_t)NL;
      uint2 *l4 = reinterpret_cast<uint2 *>(lab.s);
      for (int32_t i = threadIdx.x; i < (nr + 3) >> 2; i += TPB) l4[i] = make_uint2(two, two);
    } else {
      for (int32_t i = threadIdx.x; i < nr; i += TPB) lab.g[i] = NL;
    }
    from = 1;
    __syncthreads();
    int32_t cnt, lev;
    if (term) {
      // first level: the vertices with a residual arc to t, at label 1
      BLOCK_WAVE_LOOP(i, nr) {
        const bool first = i < nr && V.SNK[i] > 0;
        if (first) {
          lab.set((int32_t)i, 1);
          atomicOr(&bm0[i >> 5], 1u << (i & 31));
        }
        append<1>({first}, {(int32_t)i});
      }
      cnt = advance();
      lev = 1;
    } else {
      cnt = uni(min(sh.nsnk, nr));
      for (int32_t i = threadIdx.x; i < cnt; i += TPB) lab.set(V.SNK[i], 0);
      __syncthreads();
      from = 2;
      lev = 0;
    }
    while (cnt > 0) {
      work.gr_items += cnt;
      by_row_width<TPB>(cnt, [&](auto W) {
        level<decltype(W)::g, true, true>(cnt, lev + 1, work.arcs[1]);
      });
      cnt = advance();
      lev++;
    }
    levels += lev;
    // active vertices: excess and a label between the sink's and NL (the
    // borders have neither); the loads of four vertices per lane together
    from = 1;
    constexpr int KA = 4;
    for (int64_t b0 = (int64_t)(threadIdx.x & ~63u) * KA; b0 < nr; b0 += KA * (int64_t)TPB) {
      int32_t e[KA];
      bool act[KA];
#pragma unroll
      for (int j = 0; j < KA; j++) {
        const int64_t i = b0 + 64 * j + lane64();
        e[j] = 0;
        act[j] = false;
        if (i < nr) {
          e[j] = V.ex[i];
          const int32_t l = lab.get((int32_t)i);
          act[j] = l > 0 && l < NL;
        }
      }
#pragma unroll
      for (int j = 0; j < KA; j++) act[j] = act[j] && e[j] > 0;
      int32_t v[KA];
#pragma unroll
      for (int j = 0; j < KA; j++) v[j] = (int32_t)(b0 + 64 * j + lane64());
      append(act, v);
    }
    return advance();
  }

  // One push/relabel pass over the list with G lanes per vertex (as pr_sweep:
  // residuals and excess change by atomics, labels only grow).  A vertex that
  // received flow or stays active joins the next list once: the first lane to
  // mark it in qbm queues it.  old_bm: the previous pass's marks, cleared item
  // by item.
  //
  // A vertex pushes along the arcs below its label d; with excess left it is
  // relabelled to one above its lowest residual neighbour and pushes along the
  // arcs to that level too.  Both amounts are known before anything is
  // written, so an arc gets its atomics once.  Wide lists are bound by the
  // instructions issued (16 waves share 4 SIMDs), narrow ones by their
  // latency: either way a pass takes as long as its instructions.
  template <int G>
  __device__ __forceinline__ void pass_rows(int32_t cnt, uint32_t *qbm, uint32_t *old_bm) {
    constexpr int K = ROW_WORDS / G;
    const int wf = wave * (WAVE / G);
    if (wf >= cnt) return;  // straight to the step's barrier
    const int32_t ln = step_lane();
    const int gl = ln & (G - 1), grp = ln / G;
    const bool term = A.terminals != 0;
    const bool in_lds = list_in_lds(cnt);
    for (int base = wf; base < cnt; base += TPB / G) {
      const int item = base + grp;
      const bool valid = item < cnt;
      const int32_t w = get(item, valid, in_lds);
      const int32_t u = valid ? w : 0;
      u64 x[K];
      row_load<K>(L, u, gl, valid, x);
      int32_t e = valid ? *at32(V.ex, u) : 0;
      int32_t rt = term && valid ? *at32(V.SNK, u) : 0;
      const int32_t d = lab.get(u);
      if (old_bm && valid && gl == 0) atomicAnd(&old_bm[u >> 5], ~(1u << (u & 31)));
      int32_t deg = 0, ovf = 0;
      if (gl == 0) {
        deg = (int32_t)(x[0] >> 32);
        ovf = (int32_t)(uint32_t)x[0];
        x[0] = 0ull;
      }
      // the first lane's copy of the excess counts: it may grow
      // concurrently, and every lane must push against the same value
      e = group_first<G>(e);
      const bool work = valid && d < NL && e > 0;
      if (!work) deg = 0;
      this->work.items += deg > 0 ? 1 : 0;
      this->work.arcs[0] += deg;
      int32_t erem = work ? e : 0;
      // the arc to t first: always admissible (t is at label 0); once it is
      // saturated it takes no part in the relabel
      if (term) {
        rt = group_first<G>(rt);
        const int32_t amt = min(erem, max(rt, 0));
        if (gl == 0 && amt > 0) *at32(V.SNK, u) = rt - amt;
        erem -= amt;
      }
      int32_t r[K], dh[K], amt[K];
      residuals<K>(x, r, dh, work);
      erem -= share<G, K>(r, dh, erem, amt, [&](int32_t l) { return l < d; });
      int32_t nd = d;
      if (__any(erem > 0)) {
        int32_t minres = 0x7fffffff;
#pragma unroll
        for (int k = 0; k < K; k++)
          if (dh[k] >= d && dh[k] < minres) minres = dh[k];
        int32_t more = 0;
        if (__any(deg > ROW_SLOTS && erem > 0)) {  // the overflow rows, at label d
          more = erem > 0 ? group_first<G>(row_overflow(deg)) : 0;
          const int64_t row0 = (int64_t)nr + group_first<G>(ovf);
          for (int32_t j = 0; __any(j < more); j++) {
            u64 y[K];
            int32_t r2[K], dh2[K], amt2[K];
            row_load<K>(L, row0 + j, gl, j < more, y);
            residuals<K>(y, r2, dh2, j < more);
            erem -= share<G, K>(r2, dh2, erem, amt2, [&](int32_t l) { return l < d; });
#pragma unroll
            for (int k = 0; k < K; k++)
              if (dh2[k] >= d && dh2[k] < minres) minres = dh2[k];
            send<G, K>(row0 + j, gl, y, dh2, amt2, qbm, -1);
          }
        }
        minres = group_min<G>(minres);
        if (erem > 0) {
          const int32_t cand = minres >= NL ? NL : minres + 1;
          if (cand > d) nd = cand;
        }
        if (gl == 0 && nd > d) lab.set(u, nd);
        // (a vertex whose arcs fit its own row still holds them)
        const bool second = nd > d && nd < NL && more == 0;
        if (__any(second)) {
          int32_t amt2[K];
          erem -= share<G, K>(r, dh, second ? erem : 0, amt2,
                              [&](int32_t l) { return l >= d && l < nd; });
#pragma unroll
          for (int k = 0; k < K; k++) amt[k] += amt2[k];
        }
      }
      int32_t again = -1;
      if (work && gl == 0) {
        if (e > erem) atomicSub(at32(V.ex, u), e - erem);
        // flow pushed into u during this pass queued u already
        if (erem > 0 && nd < NL && bm_claim(qbm, u)) again = u;
      }
      send<G, K>(u, gl, x, dh, amt, qbm, again);
    }
  }

  // p[i] of an array below 4 GB: a scalar base and a 32-bit offset
  static __device__ __forceinline__ int32_t *at32(int32_t *p, int32_t i) {
    return reinterpret_cast<int32_t *>(reinterpret_cast<char *>(p) + (uint32_t)i * 4u);
  }
  __device__ __forceinline__ u64 *word_at(uint32_t i) const {
    return reinterpret_cast<u64 *>(reinterpret_cast<char *>(L) + i * 8u);
  }

  // own residuals of a row's words and their heads' labels (a large label
  // where nothing is left)
  template <int K>
  __device__ __forceinline__ void residuals(const u64 (&x)[K], int32_t (&r)[K], int32_t (&dh)[K],
                                            bool on) const {
#pragma unroll
    for (int k = 0; k < K; k++) {
      r[k] = on ? row_own(x[k]) : 0;
      dh[k] = lab.get(row_head(x[k]));
    }
#pragma unroll
    for (int k = 0; k < K; k++) dh[k] = r[k] > 0 ? dh[k] : 0x7fffffff;
  }

  // Splits the group's excess e over the words with take(label), in arc
  // order: amt[] per word; returns the sum.  (Sums of a row's residuals stay
  // far below 2^31.)
  template <int G, int K, typename Take>
  static __device__ __forceinline__ int32_t share(const int32_t (&r)[K], const int32_t (&dh)[K],
                                                  int32_t e, int32_t (&amt)[K], Take &&take) {
    int32_t adm[K], s = 0;
#pragma unroll
    for (int k = 0; k < K; k++) {
      adm[k] = take(dh[k]) ? r[k] : 0;
      s += adm[k];
    }
    int32_t left = e - (group_scan<G>(s) - s);  // for this lane's first word
#pragma unroll
    for (int k = 0; k < K; k++) {
      amt[k] = max(0, min(adm[k], left));
      left -= adm[k];
    }
    return min(e, group_sum<G>(s));
  }

  // The pushes amt[] along a row's words: both residuals, the heads' excess,
  // and the heads not queued yet (sink border apart) to the next list, with
  // vertex `again` if it is one.  The marks of all heads are in flight
  // together.
  template <int G, int K>
  __device__ __forceinline__ void send(int64_t row, int gl, const u64 (&x)[K],
                                       const int32_t (&dh)[K], const int32_t (&amt)[K],
                                       uint32_t *qbm, int32_t again) {
    uint32_t old[K];
    int32_t v[K + 1];
#pragma unroll
    for (int k = 0; k < K; k++) {
      old[k] = ~0u;
      v[k] = row_head(x[k]);
      if (amt[k] > 0) {
        const u64 a = (u64)(uint32_t)amt[k];
        const uint32_t h = (uint32_t)v[k];
        if (dh[k] > 0) old[k] = atomicOr(&qbm[h >> 5], 1u << (h & 31));
        atomicAdd(word_at(ROW_WORDS * (uint32_t)row + K * gl + k), (a << 16) - a);
        uint32_t slot = (uint32_t)row_rslot(x[k]);
        uint32_t at = ROW_WORDS * h + 1u + slot;
        if (slot >= ROW_SLOTS)
          at = ROW_WORDS * ((uint32_t)nr + (uint32_t)*word_at(ROW_WORDS * h)) + slot - ROW_SLOTS;
        atomicAdd(word_at(at), a - (a << 16));
        atomicAdd(at32(V.ex, v[k]), amt[k]);
      }
    }
    bool want[K + 1];
#pragma unroll
    for (int k = 0; k < K; k++) want[k] = !(old[k] & (1u << (v[k] & 31)));
    want[K] = again >= 0;
    v[K] = again;
    append(want, v);
  }

  __device__ __forceinline__ int32_t pass(int32_t cnt, int32_t since) {
    // queued marks of this pass in one bitmap; the other holds the previous
    // pass's marks (cleared item by item), or the relabel's visited marks
    uint32_t *qbm = (since & 1) ? bm0 : bm1, *old = (since & 1) ? bm1 : bm0;
    if (since == 0) {
      for (int32_t w = threadIdx.x; w < (int32_t)row_bm_words(nr); w += TPB) old[w] = 0u;
      old = nullptr;
    }
    if (cnt * 8 <= TPB) pass_rows<8>(cnt, qbm, old);
    else pass_rows<4>(cnt, qbm, old);
    return advance();
  }

  // smallest source set, written to V.ins (0 / 1); the labels to V.lab where
  // the candidate pass reads them
  __device__ __forceinline__ void closure(int64_t &levels) {
    from = 1;
    BLOCK_WAVE_LOOP(i, nr) {
      bool seed = false;
      if (i < nr) {
        const uint32_t f = V.fl[i];
        seed = LF_SRC(f) || (!LF_SNK(f) && V.ex[i] > 0);
      }
      const u64 m = __ballot(seed);
      if (lane64() == 0) bm0[i >> 5] = (uint32_t)m;
      if (lane64() == 32) bm0[i >> 5] = (uint32_t)(m >> 32);
      append<1>({seed}, {(int32_t)i});
    }
    int32_t cnt = advance();
    while (cnt > 0) {
      work.cl_items += cnt;
      by_row_width<TPB>(cnt, [&](auto W) { level<decltype(W)::g, false, false>(cnt, 0, work.arcs[2]); });
      cnt = advance();
      levels++;
    }
    const bool labels = LL && (A.mb_reps > 0 || A.cut_side != 0);
    for (int32_t i = threadIdx.x; i < nr; i += TPB) {
      V.ins[i] = (int32_t)((bm0[i >> 5] >> (i & 31)) & 1u);
      if (labels) V.lab[i] = lab.get(i);
    }
    __syncthreads();
  }

  // the lanes' counts since the last time into the workgroup's sums
  __device__ __forceinline__ void count_flush() {
    const int32_t n[4] = {wave_sum(work.items), wave_sum(work.arcs[0]), wave_sum(work.arcs[1]),
                          wave_sum(work.arcs[2])};
    if (lane64() == 0) {
      atomicAdd(&sh.work[W_SWEEP_ITEMS], (unsigned long long)n[0]);
      atomicAdd(&sh.work[W_SWEEP_ARCS], (unsigned long long)n[1]);
      atomicAdd(&sh.work[W_GR_ARCS], (unsigned long long)n[2]);
      atomicAdd(&sh.work[W_CL_ARCS], (unsigned long long)n[3]);
    }
    work.items = work.arcs[0] = work.arcs[1] = work.arcs[2] = 0;
  }
  __device__ __forceinline__ void count_step() {
    if (work.due()) count_flush();
  }
  __device__ __forceinline__ void count_end() {
    count_flush();
    if (threadIdx.x == 0) {
      sh.work[W_GR_ITEMS] += (unsigned long long)work.gr_items;
      sh.work[W_CL_ITEMS] += (unsigned long long)work.cl_items;
    }
    __syncthreads();
  }
};

// Global relabels and push/relabel passes until an exact relabel finds no
// active vertex, then the residual closure; or, in a sliced round, until the
// launch's time is used up.
template <int TPB, typename Solver>
__device__ __forceinline__ void run_flow(const KArgs &A, Solver &S, SolveShared<TPB> &sh,
                                         PairState &st, const int32_t *lc, FlowStats &F) {
  int64_t t0 = wall_clock64(), t1;
  const int64_t t_start = t0;
  // one relabel call site (the relabel is inlined; one copy keeps the
  // kernel within its registers): at the start, when the active list
  // runs dry and after rp_eff passes
  int32_t cnt = 0;
  int since = 0;
  // sweeps until the next global relabel: half the last relabel's BFS
  // depth (a deep corridor's relabel costs more), within [period / 4,
  // 2 period] of the tuning's period
  int32_t rp_eff = uni(st.rp_eff);
  const int32_t rp_lo = max(1, A.relabel_period / 4), rp_hi = 2 * A.relabel_period;
  const int64_t sweeps0 = uni(st.solve_sweeps);  // of this solve, in earlier launches
  bool relabel = true;
  for (;;) {
    if (relabel && A.slice_ticks > 0 && F.relabels > 0) {
      // sliced rounds: once this launch's time is used up, stop where a
      // global relabel is due anyway; the next launch starts with it
      // (only while at most a quarter of the launch's entries still run:
      // the others are waiting for it)
      if (threadIdx.x == 0) {
        int32_t stop = 0;
        if (lc && wall_clock64() - t_start >= A.slice_ticks) {
          const int32_t run = __hip_atomic_load(lc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const int32_t sta =
              __hip_atomic_load(lc + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          stop = 4 * run <= sta ? 1 : 0;
        }
        sh.slice_end = stop;
      }
      __syncthreads();
      F.sliced = uni(sh.slice_end) != 0;
      __syncthreads();
      if (F.sliced) break;
    }
    if (relabel) {
      t1 = wall_clock64();
      F.t_push += t1 - t0;
      t0 = t1;
      const int64_t lev0 = F.gr_levels;
      cnt = S.relabel(F.gr_levels);
      rp_eff = (int32_t)min((int64_t)rp_hi, max((int64_t)rp_lo, (F.gr_levels - lev0) / 2));
      t1 = wall_clock64();
      F.t_rel += t1 - t0;
      t0 = t1;
      F.relabels++;
      since = 0;
      relabel = false;
    }
    if (cnt == 0) {
      if (since == 0) break;  // an exact relabel found no active vertex
      relabel = true;
      continue;
    }
    if (sweeps0 + F.sweeps >= A.max_sweeps) {
      if (threadIdx.x == 0) {
        A.ctl->err = FR_E_SOLVER_LIMIT;
        A.ctl->diag = DIAG_SWEEPS;
      }
      break;
    }
    cnt = S.pass(cnt, since);
    S.count_step();
    F.sweeps++;
    if (++since >= rp_eff) relabel = true;
  }
  F.t_push += wall_clock64() - t0;
  if (threadIdx.x == 0) {
    st.solve_sweeps = sweeps0 + F.sweeps;
    st.rp_eff = rp_eff;
  }
  if (!F.sliced) S.closure(F.cl_levels);
  S.count_end();
}

// ---- maximum preflow, smallest source set, balance check, write-back and
//      the adaptive factor (Sec. 4.1), one workgroup per pair.
//      lc (sliced rounds): this launch's running and started flow entries.
//      ROWS: the form of the entry's network.
template <int TPB, bool ROWS>
__device__ __forceinline__ void flow_pair(const KArgs &A, int32_t p, SolveShared<TPB> &sh,
                                          PairState &st, const int32_t *lc = nullptr) {
  const PairView V = make_view(A, p);
  int64_t *pa = A.pacc + (int64_t)p * PA_N;
  if (threadIdx.x == 0) {
    st = A.ps[p];
    sh.cnt[0] = sh.cnt[1] = sh.cnt[2] = 0;
    sh.nsnk = min(A.pcnt[A.P + p], (int32_t)V.nv);
    if (st.phase == 0) {  // a new solve (else it continues from a sliced launch)
      st.solve_sweeps = 0;
      st.rp_eff = A.relabel_period;
      st.rows = ROWS ? 1 : 0;
      st.last_nr = st.nr;
    }
  }
  if (threadIdx.x < W_COUNT) sh.work[threadIdx.x] = 0ull;
  __syncthreads();
  const int32_t nr = uni(st.nr);
  int64_t t0 = wall_clock64();
  const int32_t NL = nr + 2;
  // networks that can't be solved: too large capacities (net_rev reports
  // them), and rows with an arc whose reverse is missing
  const bool torn = ROWS && pa[PA_REV] != 0;
  const bool unsolvable = pa[PA_RCAP] >= 0x7fffffffLL || torn;
  if (torn && threadIdx.x == 0) {
    A.ctl->err = FR_E_INVALID_GRAPH;
    A.ctl->diag = DIAG_REV;
  }
  Rot R;
  FlowStats F;
  if (!unsolvable) {
    if constexpr (ROWS) {
      // labels in LDS when they fit beside the bitmaps and lists
      if (nr <= ROW_LABEL_MAX && row_lds_bytes(nr) + row_label_bytes(nr) <= A.flow_lds) {
        RowSolver<TPB, true> S(A, V, sh, reinterpret_cast<u64 *>(V.arc), nr);
        run_flow<TPB>(A, S, sh, st, lc, F);
      } else {
        RowSolver<TPB, false> S(A, V, sh, reinterpret_cast<u64 *>(V.arc), nr);
        run_flow<TPB>(A, S, sh, st, lc, F);
      }
    } else {
      CsrSolver<TPB> S{A, V, sh, R, nr, NL, nr <= 32 * FR_BM_WORDS, {}, {}};
      run_flow<TPB>(A, S, sh, st, lc, F);
    }
    if (F.sliced) {
      // the solve continues in the next launch: its counters so far, its
      // relabel interval; the network, labels and excesses stay in place
      if (threadIdx.x == 0) {
        st.sweeps += F.sweeps;
        st.relabels += F.relabels;
        st.gr_levels += F.gr_levels;
        for (int j = 0; j < W_COUNT; j++) st.work[j] += (int64_t)sh.work[j];
        st.t_relabel += F.t_rel;
        st.t_push += F.t_push;
        st.phase = 1;
        st.slices++;
        A.ps[p] = st;
      }
      __syncthreads();
      return;
    }
  }
  const int64_t t1 = wall_clock64();
  const int64_t t_cl = t1 - t0 - F.t_rel - F.t_push;
  t0 = t1;
  // ---- candidate partition and its balance check (Sec. 2.1); for the most
  //      balanced cut, also the free vertices (neither in the smallest
  //      source set nor able to reach the sink: exact label NL), listed in
  //      LB with LA[i] = i for them and -1 for every other corridor vertex
  // flow, moved a->b, moved b->a, source side; the same three for the
  // largest minimum source side (label >= NL: cannot reach the sink)
  int64_t acc[7] = {0, 0, 0, 0, 0, 0, 0};
  const bool term = A.terminals != 0;
  const bool mb = A.mb_reps > 0 && !unsolvable;
  const int side_mode = (A.mb_reps > 0 || unsolvable) ? 0 : A.cut_side;
  if (mb) {
    if (threadIdx.x == 0) sh.nfree = 0;
    __syncthreads();
  }
  if (!unsolvable) {
    BLOCK_WAVE_LOOP(i, nr) {
      bool fv = false;
      if (i < nr) {
        const uint32_t f = V.fl[i];
        const int32_t w = A.vwgt[V.lg[i]];
        const bool in = V.ins[i] != 0;
        // the closure reached the sink: the preflow was not maximal
        if (in && (term ? V.SNK[i] > 0 : LF_SNK(f))) {
          A.ctl->err = FR_E_DEVICE;
          A.ctl->diag = DIAG_CLOSURE;
        }
        // flow: what reached the sink border; contracted terminals: what
        // left s and stayed nowhere in the corridor
        if (term) acc[0] -= V.ex[i];
        else if (LF_SNK(f)) acc[0] += V.ex[i];
        if (!(f & LF_SIDE_B) && !in) acc[1] += w;
        if ((f & LF_SIDE_B) && in) acc[2] += w;
        acc[3] += in ? 1 : 0;
        if (side_mode) {
          const bool inx = V.lab[i] >= NL;
          if (!(f & LF_SIDE_B) && !inx) acc[4] += w;
          if ((f & LF_SIDE_B) && inx) acc[5] += w;
          acc[6] += inx ? 1 : 0;
        }
        if (mb) {
          fv = !in && !(f & LF_BORDER) && V.lab[i] == NL;
          V.LA[i] = fv ? (int32_t)i : -1;
        }
      }
      if (mb) {
        const int pos = wave_append(&sh.nfree, fv);
        if (fv) V.LB[pos] = (int32_t)i;
      }
    }
  }
  block_sums<7>(acc, sh.red);
  // the record of this solve; the adaptive rule and the write-back run in
  // k_select, over all slots of the pair
  if (threadIdx.x == 0) {
    st.sweeps += F.sweeps;
    st.relabels += F.relabels;
    st.gr_levels += F.gr_levels;
    st.cl_levels += F.cl_levels;
    for (int j = 0; j < W_COUNT; j++) st.work[j] += (int64_t)sh.work[j];
    st.t_relabel += F.t_rel;
    st.t_push += F.t_push;
    st.t_closure += t_cl;
    fr_solve rec;
    const int64_t cut = st.cut;
    rec.alpha = st.alpha;
    if (term) acc[0] += pa[PA_CS];
    rec.flow = acc[0];
    rec.region_vertices = nr;
    rec.region_edges = pa[PA_RARCS] / 2;
    rec.source_side = acc[3];
    rec.cut_before = cut;
    int64_t cand = cut - pa[PA_RCIN] + acc[0];
    int64_t wa = st.cA - acc[1] + acc[2];
    int64_t wb = st.cB + acc[1] - acc[2];
    sh.use_max = 0;
    if (side_mode && cut != 0) {  // the largest minimum source side instead
      const int64_t wa2 = st.cA - acc[4] + acc[5], wb2 = st.cB + acc[4] - acc[5];
      const bool f1 = wa <= A.lmax && wb <= A.lmax, f2 = wa2 <= A.lmax && wb2 <= A.lmax;
      if (side_mode == 1 || (!f1 && f2)) {
        sh.use_max = 1;
        wa = wa2;
        wb = wb2;
        rec.source_side = acc[6];
      }
    }
    int dec;
    if (cut == 0) {
      dec = FR_DEC_NOT_ADJACENT;
      cand = 0;
      wa = st.cA;
      wb = st.cB;
      rec.flow = 0;
    } else {
      const bool feas = wa <= A.lmax && wb <= A.lmax;
      dec = !feas ? FR_DEC_INFEASIBLE : (cand < cut ? FR_DEC_APPLY : FR_DEC_EQUAL);
    }
    rec.cut_candidate = cand;
    rec.wa = wa;
    rec.wb = wb;
    rec.decision = dec;
    A.srec[p] = rec;
    st.t_finish += wall_clock64() - t0;
    for (int j = 0; j < PA_N; j++) pa[j] = 0;
    A.pcnt[p] = mb ? sh.nfree : 0;  // the most balanced cut kernel reads and clears it
    A.pcnt[A.P + p] = 0;
    A.pcnt[2 * A.P + p] = 0;
    st.phase = 2;
    A.ps[p] = st;
  }
  __syncthreads();
  if (sh.use_max) {  // the source side becomes every vertex that cannot reach the sink
    BLOCK_WAVE_LOOP(i, nr) {
      if (i < nr) V.ins[i] = V.lab[i] >= NL ? 1 : 0;
    }
    __syncthreads();
  }
}

// Entries whose network is in the row form, or (k_flow_csr) in the CSR form.
// Counters of launch `it`: queue, running, started.
template <int TPB, bool ROWS>
__device__ __forceinline__ void flow_entries(const KArgs &A, int32_t *ctr, SolveShared<TPB> &sh,
                                             PairState &st) {
  for (;;) {
    const int32_t p = next_pair<TPB>(A, ctr, sh, 1);
    if (p < 0) break;
    if ((A.ps[p].phase == 0 ? rows_chosen(A, p) : A.ps[p].rows != 0) != ROWS) continue;
    if (threadIdx.x == 0 && A.slice_ticks > 0) {
      atomicAdd(ctr + 1, 1);
      atomicAdd(ctr + 2, 1);
    }
    flow_pair<TPB, ROWS>(A, p, sh, st, ctr + 1);
    if (threadIdx.x == 0 && A.slice_ticks > 0) atomicSub(ctr + 1, 1);
  }
}

// Launched with at least sizeof(SolveShared<TPB>) of dynamic LDS; the union
// at its end takes the rest (A.flow_lds bytes in all).
template <int TPB>
__global__ void __launch_bounds__(TPB) k_flow(KArgs A, int32_t it) {
  extern __shared__ __align__(16) unsigned char flow_smem[];
  __shared__ PairState st;
  flow_entries<TPB, true>(A, A.queue + FR_QUEUE * (it % A.max_iters) + 1,
                          *reinterpret_cast<SolveShared<TPB> *>(flow_smem), st);
}

template <int TPB>
__global__ void __launch_bounds__(TPB) k_flow_csr(KArgs A, int32_t it) {
  __shared__ SolveShared<TPB> sh;
  __shared__ PairState st;
  flow_entries<TPB, false>(A, A.queue + FR_QUEUE * (it % A.max_iters) + 4, sh, st);
}
