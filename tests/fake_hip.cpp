// Host stand-in for the HIP runtime functions that libflowrefine calls, for
// CPU tests of its host code: device memory is zero-filled host memory within
// a settable budget, copies are memcpy, kernels are not run (k_quotient: every
// two blocks are adjacent).  Every launch of k_arena, whose argument is a
// round's complete KArgs, is checked against the live allocations.  Loaded with RTLD_GLOBAL ahead of the library.
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <string.h>
#include <sys/mman.h>

#include <algorithm>
#include <map>
#include <string>

#include "fr_internal.h"

static std::map<char *, size_t> live;  // device allocations
static size_t used = 0, budget = (size_t)1 << 40;
static std::map<const void *, std::string> kernels;
static hipError_t last_error = hipSuccess;
static int64_t arenas = 0, bad = 0, mallocs = 0;
static KArgs last;

// bytes from p to the end of its allocation (0: not in a live one)
static size_t room(const void *p) {
  auto it = live.upper_bound((char *)p);
  if (it == live.begin()) return 0;
  --it;
  const size_t off = (size_t)((char *)p - it->first);
  return off < it->second ? it->second - off : 0;
}

static void need(const char *what, const void *p, int64_t bytes) {
  if (bytes <= 0) bytes = 1;
  if (p && (int64_t)room(p) >= bytes) return;
  bad++;
  fprintf(stderr, "fake_hip: %s: %p holds %zu of %lld bytes\n", what, p, p ? room(p) : (size_t)0,
          (long long)bytes);
}

// what a round of these arguments may touch, from the kernels' own indexing
static void check_round(const KArgs &A) {
  const int64_t n = A.n, W = A.W, P = A.P, w4 = 4;
  const int64_t sn = W * n;
  need("part", A.part, w4 * n);
  need("mark", A.mark, w4 * (A.mstride ? sn : n));
  need("vmap", A.vmap, w4 * (A.mstride ? sn : n));
  need("uvert", A.uvert, w4 * sn);
  need("lg", A.lg, w4 * sn);
  need("lo", A.lo, w4 * (sn + P));
  need("ex", A.ex, w4 * sn);
  need("lab", A.lab, w4 * sn);
  need("ins", A.ins, w4 * sn);
  need("LA", A.LA, w4 * sn);
  need("LB", A.LB, w4 * sn);
  need("SNK", A.SNK, w4 * sn);
  need("lflag", A.lflag, sn);
  need("arc", A.arc, std::max<int64_t>(A.arc_cap, W * A.narcs) * (int64_t)sizeof(Arc));
  need("pairs", A.pairs, 2 * w4 * P);
  need("alpha0", A.alpha0, w4 * P);
  need("order", A.order, w4 * P);
  need("ps", A.ps, P * (int64_t)sizeof(PairState));
  need("blk2pair", A.blk2pair, 3 * w4 * A.k);
  need("bstat", A.bstat, 24 * (int64_t)A.k);
  if (A.fm_limit > 0) {
    need("fmg", A.fmg, w4 * n);
    need("fmq", A.fmq, w4 * n);
  }
  if (A.mb_reps > 0) {
    need("mbq", A.mbq, w4 * W * A.narcs);
    need("mbc", A.mbc, 4 * w4 * sn);
  }
  if (A.mt_alpha > 0) {
    need("mtk", A.mtk, 8 * sn);
    need("mtk2", A.mtk2, 8 * sn);
    need("mtr", A.mtr, 8 * n);
    for (int32_t *p : {A.mtt, A.mtb, A.mtq, A.mth, A.mtv, A.mtf}) need("mt", p, w4 * n);
    need("mtw", A.mtw, 8 * (int64_t)A.k);
    need("mtchg", A.mtchg, A.k);
  }
}

static hipError_t fail(hipError_t e) { return last_error = e; }

#define API extern "C" __attribute__((visibility("default")))

API void fake_budget(int64_t bytes) { budget = (size_t)bytes; }
API int64_t fake_used() { return (int64_t)used; }
API int64_t fake_arenas() { return arenas; }
API int64_t fake_bad() { return bad; }
API int64_t fake_mallocs() { return mallocs; }
API int64_t fake_arc_cap() { return last.arc_cap; }
API int32_t fake_all_rows() { return last.all_rows; }
API int32_t fake_slots() { return last.W; }

API hipError_t hipMalloc(void **p, size_t n) {
  mallocs++;
  n = (std::max<size_t>(n, 1) + 4095) & ~(size_t)4095;
  if (used + n > budget) {
    *p = nullptr;
    return fail(hipErrorOutOfMemory);
  }
  void *m = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                 -1, 0);
  if (m == MAP_FAILED) return fail(hipErrorOutOfMemory);
  live[(char *)m] = n;
  used += n;
  *p = m;
  return hipSuccess;
}

API hipError_t hipFree(void *p) {
  if (!p) return hipSuccess;
  auto it = live.find((char *)p);
  if (it == live.end()) {
    bad++;
    fprintf(stderr, "fake_hip: hipFree of %p, which is not allocated\n", p);
    return fail(hipErrorInvalidValue);
  }
  munmap(p, it->second);
  used -= it->second;
  live.erase(it);
  return hipSuccess;
}

API hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total) {
  *free_bytes = budget > used ? budget - used : 0;
  *total = budget;
  return hipSuccess;
}

API hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  *p = calloc(1, n);
  return hipSuccess;
}
API hipError_t hipHostFree(void *p) {
  free(p);
  return hipSuccess;
}

static hipError_t copy(void *d, const void *s, size_t n) {
  if (n && (!d || !s)) return fail(hipErrorInvalidValue);
  memcpy(d, s, n);
  return hipSuccess;
}
API hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return copy(d, s, n); }
API hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  return copy(d, s, n);
}
static hipError_t set(void *d, int v, size_t n) {
  if (n && !d) return fail(hipErrorInvalidValue);
  if (v != 0) memset(d, v, n);
  else if (n) memset(d, 0, std::min<size_t>(n, 4096));  // fresh memory is zero
  return hipSuccess;
}
API hipError_t hipMemset(void *d, int v, size_t n) { return set(d, v, n); }
API hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return set(d, v, n); }

API hipError_t hipGetDeviceCount(int *n) {
  *n = 1;
  return hipSuccess;
}
API hipError_t hipSetDevice(int) { return hipSuccess; }
API hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = 160 << 10;
  return hipSuccess;
}
API hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 100000;
  return hipSuccess;
}
API hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
API hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 2;
  return hipSuccess;
}
API hipError_t hipGetSymbolAddress(void **p, const void *) {
  static void *scratch = nullptr;
  if (!scratch) scratch = calloc(1, (size_t)64 << 20);
  *p = scratch;
  return hipSuccess;
}
API hipError_t hipGetLastError() {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}

API hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)(uintptr_t)16;
  return hipSuccess;
}
API hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
API hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
API hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
API hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)(uintptr_t)16;
  return hipSuccess;
}
API hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
API hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
API hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
API hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
API hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = (hipGraph_t)(uintptr_t)16;
  return hipSuccess;
}
API hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t)(uintptr_t)16;
  return hipSuccess;
}
API hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
API hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
API hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

// launches
static struct {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
} config;
API hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  config = {g, b, s, st};
  return hipSuccess;
}
API hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
  *g = config.grid;
  *b = config.block;
  *s = config.shmem;
  *st = config.stream;
  return hipSuccess;
}
API hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **args, size_t, hipStream_t) {
  auto it = kernels.find(fn);
  if (it == kernels.end()) return hipSuccess;
  if (it->second.find("k_arena") != std::string::npos) {
    last = *(const KArgs *)args[0];
    arenas++;
    check_round(last);
  } else if (it->second.find("k_quotient") != std::string::npos) {
    const int64_t k = ((const KArgs *)args[0])->k;
    uint8_t *q = *(uint8_t **)args[1];
    need("qadj", q, k * k);
    if (room(q) >= (size_t)(k * k)) memset(q, 1, (size_t)(k * k));
  }
  return hipSuccess;
}
API void **__hipRegisterFatBinary(const void *) {
  static void *handle = nullptr;
  return &handle;
}
API void __hipUnregisterFatBinary(void **) {}
API void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned,
                               void *, void *, void *, void *, int *) {
  kernels[host] = name;
}
API void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
