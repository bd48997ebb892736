// Learned area factor: a small MLP that proposes the start factor alpha of
// each pair's adaptive flow iterations.  It has no counterpart in the paper;
// the plain adaptive search (Sec. 4.1) keeps running from the proposed
// factor, so the flow results stay exact; the search from alpha' is the
// reference for cut quality.
//
// Network: 8 features -> 64 -> 64 -> 5 classes (alpha = 1, 2, 4, 8, 16),
// ReLU hidden layers, softmax cross-entropy.  FP32 throughout, plain FMA
// (5 k parameters, no dense contraction worth a matrix core).  Parameters are
// one float array: W1[8][64], b1[64], W2[64][64], b2[64], W3[64][5], b3[5]
// (row-major [in][out]).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fr_internal.h"

#define MLP_IN 8
#define MLP_H 64
#define MLP_OUT 5
#define MLP_W1 0
#define MLP_B1 (MLP_W1 + MLP_IN * MLP_H)
#define MLP_W2 (MLP_B1 + MLP_H)
#define MLP_B2 (MLP_W2 + MLP_H * MLP_H)
#define MLP_W3 (MLP_B2 + MLP_H)
#define MLP_B3 (MLP_W3 + MLP_H * MLP_OUT)
#define MLP_NPARAMS (MLP_B3 + MLP_OUT)
#define MLP_SAMPLES_PER_BLOCK 16  // 16 samples x 64 units = 1024 threads

// Per-pair boundary statistics for the features: [P][4] = boundary vertices
// of a, of b, boundary weight of a, pair cut.  Grid over all vertices.
__global__ void __launch_bounds__(256) k_feature_stats(KArgs A, int64_t *acc) {
  __shared__ uint32_t s_bnd[256];
  __shared__ unsigned long long s_cw[256];
  const int lane = lane64();
  const int wl = (int)(threadIdx.x & ~63u);
  unsigned long long *ac = (unsigned long long *)acc;
  // boundary count a / b, boundary weight a, cut weight; keyed by pair
  KeyedSums<4> sums;
  auto out = [&](int j, int key, int64_t v) { wave_add_by_key(ac, 4, j, key, v); };
  wave_chunk_runs(A, [&](int64_t u0, int32_t blk, int32_t x0) {
    const int64_t u = u0 + lane;
    const int64_t last = min((int64_t)A.n, u0 + 64);
    int32_t p = -1, y2 = -1;
    int64_t w = 0;
    if (u < last) {
      const int32_t x = blk;
      p = A.blk2pair[x];
      if (p >= 0) {
        const int32_t a = A.pairs[2 * p], b = A.pairs[2 * p + 1];
        const int side = x == b;
        y2 = ((side ? a : b) << 1) | side;
        w = A.vwgt[u];
      }
    }
    bool bnd;
    int64_t cw;
    chunk_boundary(A, x0, y2, __shfl(x0, 0), A.xadj[last], s_bnd + wl, s_cw + wl, bnd, cw);
    const int side = y2 & 1;
    const int64_t x[4] = {bnd && !side ? 1 : 0, bnd && side ? 1 : 0, bnd && !side ? w : 0, cw};
    sums.add(p, x, out);
  });
  sums.flush(out);
}

// The 8 features of every pair (FP32): log2(1+|dA|), log2(1+|dB|), c(A)/W,
// c(B)/W, log2(1+cut), (Lmax-c(A))/W, (Lmax-c(B))/W, log2(1 + U_A(1)/c(dA))
// with W = c(V)/k and U_A(1) the alpha = 1 area bound of side a.
__global__ void __launch_bounds__(256) k_features(KArgs A, const int64_t *acc, float *feats) {
  const int64_t cV = A.ctl->cV;
  const double W = (double)cV / (double)A.k > 0 ? (double)cV / (double)A.k : 1.0;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < A.P; p += gridDim.x * blockDim.x) {
    const int32_t a = A.pairs[2 * p], b = A.pairs[2 * p + 1];
    const int64_t cA = A.bstat[a], cB = A.bstat[b];
    const int64_t *s = acc + 4 * p;
    int64_t u1 = A.base[1] - cB;
    u1 = u1 > 0 ? u1 : 0;
    const double wda = s[2] > 1 ? (double)s[2] : 1.0;
    float *f = feats + (int64_t)MLP_IN * p;
    f[0] = (float)log2(1.0 + (double)s[0]);
    f[1] = (float)log2(1.0 + (double)s[1]);
    f[2] = (float)((double)cA / W);
    f[3] = (float)((double)cB / W);
    f[4] = (float)log2(1.0 + (double)s[3]);
    f[5] = (float)((double)(A.lmax - cA) / W);
    f[6] = (float)((double)(A.lmax - cB) / W);
    f[7] = (float)log2(1.0 + (double)u1 / wda);
  }
}

// Forward pass: MLP_SAMPLES_PER_BLOCK samples per block, one thread per
// (sample, hidden unit).  Writes the class probabilities.
__global__ void __launch_bounds__(1024) k_mlp_forward(const float *prm, const float *x, int32_t n,
                                                      float *probs) {
  __shared__ float s_x[MLP_SAMPLES_PER_BLOCK][MLP_IN];
  __shared__ float s_h1[MLP_SAMPLES_PER_BLOCK][MLP_H];
  __shared__ float s_h2[MLP_SAMPLES_PER_BLOCK][MLP_H];
  __shared__ float s_z[MLP_SAMPLES_PER_BLOCK][MLP_OUT];
  const int ls = threadIdx.x / MLP_H, j = threadIdx.x % MLP_H;
  const int s = blockIdx.x * MLP_SAMPLES_PER_BLOCK + ls;
  const bool ok = s < n;
  if (j < MLP_IN) s_x[ls][j] = ok ? x[(int64_t)s * MLP_IN + j] : 0.f;
  __syncthreads();
  float a1 = prm[MLP_B1 + j];
  for (int i = 0; i < MLP_IN; i++) a1 = fmaf(s_x[ls][i], prm[MLP_W1 + i * MLP_H + j], a1);
  const float h1 = a1 > 0.f ? a1 : 0.f;
  s_h1[ls][j] = h1;
  __syncthreads();
  float a2 = prm[MLP_B2 + j];
  for (int i = 0; i < MLP_H; i++) a2 = fmaf(s_h1[ls][i], prm[MLP_W2 + i * MLP_H + j], a2);
  const float h2 = a2 > 0.f ? a2 : 0.f;
  s_h2[ls][j] = h2;
  __syncthreads();
  if (j < MLP_OUT) {
    float z = prm[MLP_B3 + j];
    for (int i = 0; i < MLP_H; i++) z = fmaf(s_h2[ls][i], prm[MLP_W3 + i * MLP_OUT + j], z);
    s_z[ls][j] = z;
  }
  __syncthreads();
  if (ok && j == 0) {
    float zm = s_z[ls][0];
    for (int c = 1; c < MLP_OUT; c++) zm = fmaxf(zm, s_z[ls][c]);
    float e[MLP_OUT], sum = 0.f;
    for (int c = 0; c < MLP_OUT; c++) {
      e[c] = expf(s_z[ls][c] - zm);
      sum += e[c];
    }
    for (int c = 0; c < MLP_OUT; c++) probs[(int64_t)s * MLP_OUT + c] = e[c] / sum;
  }
}

// Loss and parameter gradients of MLP_TILE samples per workgroup, from the
// features to partial sums (partial[tile][MLP_NPARAMS], lossp[tile]) without
// storing an activation: forward, then for the mean softmax cross-entropy
// (labels) dz = (p - onehot) / n, or, with per-class costs [n][5], for the
// mean expected cost sum_c p_c cost_c: dz_j = p_j (cost_j - sum_c p_c cost_c)
// / n; then da2 = (dz W3^T) * [h2 > 0], da1 = (da2 W2^T) * [h1 > 0] and
// dW1 = x^T da1, db1 = sum da1, dW2 = h1^T da2, db2 = sum da2, dW3 = h2^T dz,
// db3 = sum dz over the tile's samples.
//
// Each wave takes 16 of the 64 samples, a lane one hidden unit of all 16, so
// a weight is read once for 16 FMAs and the activations are LDS broadcasts;
// dW2 is a 4 x 4 tile per thread.  The sums of one thread per parameter over
// all samples, which this replaces, were a serial chain of n loads: 3.97 ms
// of a 4.4 ms call at n = 16,384; the tiles and their sum take 0.05 ms.  The
// two-level sum is also the more exact one (64 + tiles / 4 + 4 terms in a row
// instead of n).  Bound: launch latency and the LDS reads of one tile.
#define MLP_TILE 64
__global__ void __launch_bounds__(256) k_mlp_grad_tiles(const float *prm, const float *x,
                                                        const int32_t *labels, const float *costs,
                                                        int32_t n, float *partial, double *lossp) {
  constexpr int Q = MLP_TILE / 4;        // samples per wave
  constexpr int P2 = MLP_H + 1;          // pitch of W2: rows and columns free of bank conflicts
  __shared__ float s_w1[MLP_IN * MLP_H], s_w2[MLP_H * P2], s_w3[MLP_H * MLP_OUT];
  __shared__ float s_x[MLP_TILE * MLP_IN];
  __shared__ __align__(16) float s_a[MLP_TILE * MLP_H];  // h1, later da1
  __shared__ __align__(16) float s_b[MLP_TILE * MLP_H];  // h2, later da2
  __shared__ float s_p[MLP_TILE * MLP_OUT], s_dz[MLP_TILE * MLP_OUT];
  const int t = threadIdx.x, j = t & 63, s0 = (t >> 6) * Q;
  const int64_t base = (int64_t)blockIdx.x * MLP_TILE;
  const int m = (int)min((int64_t)MLP_TILE, n - base);  // samples of this tile
  float *out = partial + (int64_t)blockIdx.x * MLP_NPARAMS;
  for (int i = t; i < MLP_IN * MLP_H; i += 256) s_w1[i] = prm[MLP_W1 + i];
  for (int i = t; i < MLP_H * MLP_H; i += 256) s_w2[(i / MLP_H) * P2 + i % MLP_H] = prm[MLP_W2 + i];
  for (int i = t; i < MLP_H * MLP_OUT; i += 256) s_w3[i] = prm[MLP_W3 + i];
  for (int i = t; i < MLP_TILE * MLP_IN; i += 256)
    s_x[i] = i < m * MLP_IN ? x[base * MLP_IN + i] : 0.f;
  const float b1 = prm[MLP_B1 + j], b2 = prm[MLP_B2 + j];
  __syncthreads();
  float v[Q];
  // layer 1
#pragma unroll
  for (int q = 0; q < Q; q++) v[q] = b1;
  for (int i = 0; i < MLP_IN; i++) {
    const float w = s_w1[i * MLP_H + j];
#pragma unroll
    for (int q = 0; q < Q; q++) v[q] = fmaf(s_x[(s0 + q) * MLP_IN + i], w, v[q]);
  }
#pragma unroll
  for (int q = 0; q < Q; q++) s_a[(s0 + q) * MLP_H + j] = v[q] > 0.f ? v[q] : 0.f;
  __syncthreads();
  // layer 2
#pragma unroll
  for (int q = 0; q < Q; q++) v[q] = b2;
  for (int i = 0; i < MLP_H; i += 4) {
    const float w0 = s_w2[i * P2 + j], w1 = s_w2[(i + 1) * P2 + j], w2 = s_w2[(i + 2) * P2 + j],
                w3 = s_w2[(i + 3) * P2 + j];
#pragma unroll
    for (int q = 0; q < Q; q++) {
      const float4 h = *reinterpret_cast<const float4 *>(&s_a[(s0 + q) * MLP_H + i]);
      v[q] = fmaf(h.w, w3, fmaf(h.z, w2, fmaf(h.y, w1, fmaf(h.x, w0, v[q]))));
    }
  }
#pragma unroll
  for (int q = 0; q < Q; q++) s_b[(s0 + q) * MLP_H + j] = v[q] > 0.f ? v[q] : 0.f;
  __syncthreads();
  // logits
  for (int i = t; i < MLP_TILE * MLP_OUT; i += 256) {
    const int s = i / MLP_OUT, c = i % MLP_OUT;
    float z = prm[MLP_B3 + c];
    for (int k = 0; k < MLP_H; k++) z = fmaf(s_b[s * MLP_H + k], s_w3[k * MLP_OUT + c], z);
    s_p[i] = z;
  }
  __syncthreads();
  // softmax, loss and dz, one lane of the first wave per sample
  if (t < MLP_TILE) {
    const int64_t g = base + t;
    float *p = s_p + t * MLP_OUT, *dz = s_dz + t * MLP_OUT;
    float zm = p[0], e[MLP_OUT], sum = 0.f;
    for (int c = 1; c < MLP_OUT; c++) zm = fmaxf(zm, p[c]);
    for (int c = 0; c < MLP_OUT; c++) {
      e[c] = expf(p[c] - zm);
      sum += e[c];
    }
    for (int c = 0; c < MLP_OUT; c++) e[c] = e[c] / sum;
    double l = 0.0;
    if (t >= m) {
      for (int c = 0; c < MLP_OUT; c++) dz[c] = 0.f;
    } else if (costs) {
      const float *cs = costs + g * MLP_OUT;
      float pc = 0.f;
      for (int c = 0; c < MLP_OUT; c++) {
        pc = fmaf(e[c], cs[c], pc);
        l += (double)e[c] * (double)cs[c];
      }
      for (int c = 0; c < MLP_OUT; c++) dz[c] = e[c] * (cs[c] - pc) / (float)n;
    } else {
      const int y = labels[g];
      l = -log((double)fmaxf(e[y], 1e-30f));
      for (int c = 0; c < MLP_OUT; c++) dz[c] = (e[c] - (y == c ? 1.f : 0.f)) / (float)n;
    }
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
    if (t == 0) lossp[blockIdx.x] = l;
  }
  __syncthreads();
  // da2 (in v until dW3 has read h2), dW3, db3
  float w3r[MLP_OUT];
  for (int c = 0; c < MLP_OUT; c++) w3r[c] = s_w3[j * MLP_OUT + c];
#pragma unroll
  for (int q = 0; q < Q; q++) {
    float d = 0.f;
    for (int c = 0; c < MLP_OUT; c++) d = fmaf(s_dz[(s0 + q) * MLP_OUT + c], w3r[c], d);
    v[q] = s_b[(s0 + q) * MLP_H + j] > 0.f ? d : 0.f;
  }
  for (int i = t; i < MLP_H * MLP_OUT + MLP_OUT; i += 256) {
    const int k = i / MLP_OUT, c = i % MLP_OUT;  // row MLP_H: the bias
    float g = 0.f;
    for (int s = 0; s < m; s++) {
      const float d = s_dz[s * MLP_OUT + c];
      g = k < MLP_H ? fmaf(s_b[s * MLP_H + k], d, g) : g + d;
    }
    out[MLP_W3 + i] = g;  // b3 follows W3
  }
  static_assert(MLP_B3 == MLP_W3 + MLP_H * MLP_OUT, "b3 follows W3");
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Q; q++) s_b[(s0 + q) * MLP_H + j] = v[q];
  __syncthreads();
  // dW2 (4 x 4 per thread), db2
  {
    const int i0 = (t >> 4) * 4, j0 = (t & 15) * 4;
    float g[4][4] = {};
    for (int s = 0; s < m; s++) {
      const float4 a = *reinterpret_cast<const float4 *>(&s_a[s * MLP_H + i0]);
      const float4 b = *reinterpret_cast<const float4 *>(&s_b[s * MLP_H + j0]);
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int c = 0; c < 4; c++) g[r][c] = fmaf(av[r], bv[c], g[r][c]);
    }
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
      for (int c = 0; c < 4; c++) out[MLP_W2 + (i0 + r) * MLP_H + j0 + c] = g[r][c];
  }
  if (t < MLP_H) {
    float g = 0.f;
    for (int s = 0; s < m; s++) g += s_b[s * MLP_H + t];
    out[MLP_B2 + t] = g;
  }
  // da1 (in v until dW2 has read h1)
#pragma unroll
  for (int q = 0; q < Q; q++) v[q] = 0.f;
  for (int k = 0; k < MLP_H; k += 4) {
    const float w0 = s_w2[j * P2 + k], w1 = s_w2[j * P2 + k + 1], w2 = s_w2[j * P2 + k + 2],
                w3 = s_w2[j * P2 + k + 3];
#pragma unroll
    for (int q = 0; q < Q; q++) {
      const float4 d = *reinterpret_cast<const float4 *>(&s_b[(s0 + q) * MLP_H + k]);
      v[q] = fmaf(d.w, w3, fmaf(d.z, w2, fmaf(d.y, w1, fmaf(d.x, w0, v[q]))));
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Q; q++) {
    float &h = s_a[(s0 + q) * MLP_H + j];
    h = h > 0.f ? v[q] : 0.f;
  }
  __syncthreads();
  // dW1, db1
  for (int i = t; i < MLP_IN * MLP_H + MLP_H; i += 256) {
    const int k = i / MLP_H, c = i % MLP_H;  // row MLP_IN: the bias
    float g = 0.f;
    for (int s = 0; s < m; s++) {
      const float d = s_a[s * MLP_H + c];
      g = k < MLP_IN ? fmaf(s_x[s * MLP_IN + k], d, g) : g + d;
    }
    out[MLP_W1 + i] = g;  // b1 follows W1
  }
  static_assert(MLP_B1 == MLP_W1 + MLP_IN * MLP_H, "b1 follows W1");
}

// grad = sum of the tiles' partial gradients, loss = their mean loss, in a
// fixed order: 64 parameters per workgroup, a quarter of the tiles per wave.
__global__ void __launch_bounds__(256) k_mlp_grad_sum(const float *partial, const double *lossp,
                                                      int32_t tiles, int32_t n, float *grad,
                                                      float *loss) {
  __shared__ float s_g[4][64];
  const int seg = threadIdx.x >> 6, j = threadIdx.x & 63;
  const int p = blockIdx.x * 64 + j;
  const int lo = (int)((int64_t)tiles * seg / 4), hi = (int)((int64_t)tiles * (seg + 1) / 4);
  float g = 0.f;
  if (p < MLP_NPARAMS) {
#pragma unroll 8
    for (int i = lo; i < hi; i++) g += partial[(int64_t)i * MLP_NPARAMS + p];
  }
  s_g[seg][j] = g;
  __syncthreads();
  if (seg == 0 && p < MLP_NPARAMS) grad[p] = ((s_g[0][j] + s_g[1][j]) + s_g[2][j]) + s_g[3][j];
  if (loss && blockIdx.x == 0 && seg == 1) {
    double l = 0.0;
    for (int i = j; i < tiles; i += 64) l += lossp[i];
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
    if (j == 0) *loss = (float)(l / (n > 0 ? n : 1));
  }
}

// mean cross-entropy of n samples (labels), or their mean expected cost
// (costs [n][5]); one block
__global__ void __launch_bounds__(256) k_mlp_loss(const float *probs, const int32_t *labels,
                                                  const float *costs, int32_t n, float *loss) {
  __shared__ double s_red[256];
  double acc = 0.0;
  for (int s = threadIdx.x; s < n; s += blockDim.x) {
    if (costs) {
      for (int c = 0; c < MLP_OUT; c++)
        acc += (double)probs[(int64_t)s * MLP_OUT + c] * (double)costs[(int64_t)s * MLP_OUT + c];
    } else {
      const float p = probs[(int64_t)s * MLP_OUT + labels[s]];
      acc -= log((double)fmaxf(p, 1e-30f));
    }
  }
  s_red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(s_red[0] / (n > 0 ? n : 1));
}

// Adam (Kingma & Ba 2015) with bias correction; t >= 1.
__global__ void __launch_bounds__(256) k_adam(float *prm, const float *grad, float *m, float *v,
                                              float lr, float b1, float b2, float eps, int32_t t) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= MLP_NPARAMS) return;
  const float g = grad[i];
  const float mi = b1 * m[i] + (1.f - b1) * g;
  const float vi = b2 * v[i] + (1.f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / (1.f - powf(b1, (float)t));
  const float vh = vi / (1.f - powf(b2, (float)t));
  prm[i] -= lr * mh / (sqrtf(vh) + eps);
}

// rows idx[0..m) of (x, labels or costs) into (xb, lb or cb)
static_assert(MLP_IN >= MLP_OUT, "a row's costs are gathered by its feature lanes");
__global__ void __launch_bounds__(256) k_gather_rows(const float *x, const int32_t *labels,
                                                     const float *costs, const int32_t *idx,
                                                     int32_t m, float *xb, int32_t *lb,
                                                     float *cb) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= m * MLP_IN) return;
  const int r = t / MLP_IN, c = t % MLP_IN;
  xb[t] = x[(int64_t)idx[r] * MLP_IN + c];
  if (costs) {
    if (c < MLP_OUT) cb[r * MLP_OUT + c] = costs[(int64_t)idx[r] * MLP_OUT + c];
  } else if (c == 0) {
    lb[r] = labels[idx[r]];
  }
}

// start factor of each pair from the predicted class (first maximum, i.e.
// the smaller factor on ties)
__global__ void __launch_bounds__(256) k_alpha_from_probs(const float *probs, int32_t P,
                                                          int32_t *alpha0) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  int best = 0;
  for (int c = 1; c < MLP_OUT; c++)
    if (probs[(int64_t)p * MLP_OUT + c] > probs[(int64_t)p * MLP_OUT + best]) best = c;
  alpha0[p] = 1 << best;
}
