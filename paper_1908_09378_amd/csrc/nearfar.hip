// Near-Far, a GPU form of Delta-stepping (Meyer and Sanders; Davidson et al.,
// IPDPS 2014): the comparison family of the paper (Sections 1.1 and 4.2).
//
// Two buckets: the "near" frontier holds vertices whose tentative distance is
// below a threshold T, the "far" pile the rest.  A relax phase scans every
// out-edge of the near frontier (atomicMin on dist); an improved vertex goes
// to the next near frontier if its new distance is below T, else to the far
// pile.  When the near frontier runs empty, T grows by Delta (or jumps to the
// first Delta step past the smallest far key) and the far vertices now below
// T become the near frontier; vertices whose distance improved since they
// were filed are re-scanned, so the result is exact for any Delta.
//
// One persistent cooperative launch over the whole GPU (one workgroup per
// CU): phases are separated by a software grid barrier whose last arriving
// workgroup also does the bookkeeping (queue sizes, next phase, T) while the
// others wait.  Every word workgroups hand to each other is written and read
// with agent-scope atomics (the XCDs' L2 caches are not coherent for plain
// stores); every wait is bounded by the real-time clock and gives up with an
// error flag, and a phase limit ends a run that would not terminate.
//
// Frontier vertices of low degree are scanned by groups of G lanes (G close
// to the mean degree), vertices of high degree by every workgroup at once.
// Pushes are deduplicated per phase by stamping vertices with the phase
// number (near) or the far pile's epoch (far), so each queue holds at most n.
//
// A phase is a chain of dependent round trips to the memory side (frontier
// entry, its distance / last scan / row, the edges, atomicMin, the stamp) and
// the queue counters, so both are kept short: what depends on the vertex alone
// is read together, and pushes are gathered in each workgroup's LDS and leave
// it with one counter update per workgroup (one per wavefront, on one address,
// is about 10 ns each: 20 us of a phase of 2,000 wavefronts).
// A phase whose frontier one workgroup covers in a few steps is not worth a
// barrier over the grid: the workgroup that arrived last runs it, and those
// that follow, by itself while the others go on waiting.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "../../include/pbh.h"
#include "nearfar_core.h"
#include "pbh_team.h"

namespace bkt {
namespace nf {

constexpr int NT = 512;          // threads per workgroup
constexpr u32 HEAVY = 1024;      // out-degree above which a vertex is scanned by the whole grid

// The GPU's grid: agent-scope accesses, since the XCDs' L2 caches are not
// coherent for plain ones.
struct DevGrid {
  static constexpr int NT = nf::NT, W = 64;
  static constexpr u32 HEAVY = nf::HEAVY;
  static constexpr u32 PUSHES = 4096;  // near / far pushes gathered per workgroup before they are written out
  using Word = u32;
  __device__ __forceinline__ u32 tid() const { return threadIdx.x; }
  __device__ __forceinline__ u32 wg() const { return blockIdx.x; }
  __device__ __forceinline__ u32 nwg() const { return gridDim.x; }
  __device__ __forceinline__ void sync() const { __syncthreads(); }
  __device__ __forceinline__ void wait_mem() const { __builtin_amdgcn_s_waitcnt(0); }
  __device__ __forceinline__ void nap() const { __builtin_amdgcn_s_sleep(2); }
  __device__ __forceinline__ u64 clock() const { return __builtin_amdgcn_s_memrealtime(); }
  __device__ __forceinline__ u32 ld32(const u32* p) const {
    return __hip_atomic_load((const u32 PBH_GLB*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ u64 ld64(const u64* p) const {
    return __hip_atomic_load((const u64 PBH_GLB*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void st32(u32* p, u32 v) const {
    __hip_atomic_store((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void st64(u64* p, u64 v) const {
    __hip_atomic_store((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ u32 xchg32(u32* p, u32 v) const {
    return __hip_atomic_exchange((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ u32 add32(u32* p, u32 v) const {
    return __hip_atomic_fetch_add((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ u32 or32(u32* p, u32 v) const {
    return __hip_atomic_fetch_or((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ u64 min64(u64* p, u64 v) const {
    return __hip_atomic_fetch_min((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // *p++ and *p = min(*p, v) in LDS
  __device__ __forceinline__ u32 lds_next(u32* p) const {
    return __hip_atomic_fetch_add((u32 PBH_LDS*)p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ void lds_min(u64* p, u64 v) const {
    __hip_atomic_fetch_min((u64 PBH_LDS*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // x of thread `from` of this wavefront
  __device__ __forceinline__ u64 from_lane(u64 x, u32 from) const { return __shfl(x, (int)(from & 63u), 64); }
  __device__ __forceinline__ u32 wave_max(u32 x) const {
    for (int o = 32; o > 0; o >>= 1) {
      const u32 y = (u32)__shfl_xor((int)x, o, 64);
      x = y > x ? y : x;
    }
    return x;
  }
};

__global__ __launch_bounds__(NT) void k_nearfar(Args a) {
  __shared__ Phase sph;
  __shared__ u32 sflag;
  __shared__ Gather<DevGrid> q;
  const DevGrid t;
  u64 scanned = phases(t, a, &sph, &sflag, &q);
  for (int o = 32; o > 0; o >>= 1) scanned += __shfl_xor(scanned, o, 64);
  if (scanned && (threadIdx.x & 63) == 0)
    __hip_atomic_fetch_add((u64 PBH_GLB*)&a.c->relax, scanned, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_nf_init(u64* dist, u32* nstamp, u32* fstamp, u64* done_at, u32 n, u32 src) {
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) {
    dist[i] = i == src ? 0ull : KINF;
    nstamp[i] = NONE;
    fstamp[i] = NONE;
    done_at[i] = KINF;
  }
}

// Maximum out-degree, edge-weight sum and CSR validity (one pass).
struct Scan {
  u64 bad, maxdeg, wsum;
};
__global__ void k_nf_scan(const u64* off, const u32* tg, const u32* wt, u32 n, u64 m, Scan* out) {
  u64 bad = 0, md = 0, ws = 0;
  const u64 stride = (u64)gridDim.x * blockDim.x, t0 = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  for (u64 u = t0; u < n; u += stride) {
    const u64 a = off[u], b = off[u + 1];
    if (b < a)
      bad = 1;
    else
      md = b - a > md ? b - a : md;
  }
  if (t0 == 0 && (off[0] != 0 || off[n] != m)) bad = 1;
  for (u64 e = t0; e < m; e += stride) {
    if (tg[e] >= n) bad = 1;
    ws += wt[e];
  }
  // one update per workgroup (updates of one word take about 10 ns each)
  __shared__ u64 sb[4], sm[4], sw[4];
  for (int o = 32; o > 0; o >>= 1) {
    const u64 m2 = __shfl_xor(md, o, 64);
    bad |= __shfl_xor(bad, o, 64);
    md = m2 > md ? m2 : md;
    ws += __shfl_xor(ws, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sb[threadIdx.x >> 6] = bad;
    sm[threadIdx.x >> 6] = md;
    sw[threadIdx.x >> 6] = ws;
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < 4; ++w) {
    bad |= sb[w];
    md = sm[w] > md ? sm[w] : md;
    ws += sw[w];
  }
  if (bad) atomicOr(&out->bad, 1ull);
  if (md) atomicMax(&out->maxdeg, md);
  if (ws) atomicAdd(&out->wsum, ws);
}

thread_local char g_nferr[256] = "";
std::mutex g_nf_mu;

int nf_fail(int code, const char* msg) {
  snprintf(g_nferr, sizeof g_nferr, "%s", msg);
  return code;
}

}  // namespace nf
}  // namespace bkt

using namespace bkt;
using namespace bkt::nf;

#define NFCHK(expr)                                                                            \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess) {                                                                    \
      snprintf(g_nferr, sizeof g_nferr, "%s: %s", #expr, hipGetErrorString(e_));               \
      rc = e_ == hipErrorOutOfMemory ? PBH_ENOMEM : PBH_EDEVICE;                               \
      goto out;                                                                                \
    }                                                                                          \
  } while (0)

extern "C" {

const char* sssp_nearfar_last_error(void) { return g_nferr; }

int sssp_nearfar(const uint64_t* offsets, const uint32_t* targets, const uint32_t* weights, uint32_t n,
                 uint64_t m, uint32_t source, uint64_t* dist_out, uint64_t delta, sssp_nearfar_stats* stats,
                 void* stream) {
  if (stats) std::memset(stats, 0, sizeof *stats);
  if (!offsets || !dist_out || (m > 0 && (!targets || !weights))) return nf_fail(PBH_EINVAL, "NULL array argument");
  if (n == 0 || source >= n) return nf_fail(PBH_EINVAL, "n == 0 or source >= n");
  hipStream_t s = (hipStream_t)stream;
  std::lock_guard<std::mutex> lock(g_nf_mu);
  int rc = PBH_OK;
  unsigned char* buf = nullptr;
  Scan sc{};
  Ctl ctl{};
  hipEvent_t e0 = nullptr, e1 = nullptr;
  const u64 cap = n;
  const u64 bytes = 256 + ((sizeof(Ctl) + 255) / 256) * 256 + 8ull * n + 4ull * (6 * cap + 2ull * n);
  Args a{};
  int dev = 0, cus = 0, occ = 0;
  float ms = 0.f;
  u64 avgdeg;
  NFCHK(hipMalloc(&buf, bytes));
  {
    Scan* dscan = reinterpret_cast<Scan*>(buf);
    Ctl* dctl = reinterpret_cast<Ctl*>(buf + 256);
    u32* q = reinterpret_cast<u32*>(buf + 256 + ((sizeof(Ctl) + 255) / 256) * 256);
    NFCHK(hipMemsetAsync(dscan, 0, sizeof(Scan), s));
    hipLaunchKernelGGL(k_nf_scan, dim3(std::min<u64>(1024, (std::max<u64>(n, m) + 255) / 256)), dim3(256), 0, s,
                       (const u64*)offsets, targets, weights, n, m, dscan);
    NFCHK(hipGetLastError());
    NFCHK(hipMemcpyAsync(&sc, dscan, sizeof sc, hipMemcpyDeviceToHost, s));
    NFCHK(hipStreamSynchronize(s));
    if (sc.bad) {
      rc = nf_fail(PBH_EINVAL, "malformed CSR (offsets or targets)");
      goto out;
    }
    avgdeg = m / n ? m / n : 1;
    if (delta == 0) {
      // Davidson et al.'s choice: mean weight x wavefront width / mean degree
      const u64 wmean = m ? (sc.wsum + m - 1) / m : 1;
      delta = std::max<u64>(1, wmean * 64 / avgdeg);
    }
    a.off = (const u64*)offsets;
    a.tg = targets;
    a.wt = weights;
    a.dist = (u64*)dist_out;
    a.n = n;
    a.delta = delta;
    a.glog = avgdeg <= 6 ? 2 : avgdeg <= 12 ? 3 : avgdeg <= 24 ? 4 : avgdeg <= 48 ? 5 : 6;
    a.done_at = reinterpret_cast<u64*>(q);
    q += 2ull * n;
    for (int i = 0; i < 2; ++i) {
      a.ql[i] = q + (u64)i * cap;
      a.qh[i] = q + (u64)(2 + i) * cap;
      a.far[i] = q + (u64)(4 + i) * cap;
    }
    a.nstamp = q + 6 * cap;
    a.fstamp = q + 6 * cap + n;
    a.cap = (u32)cap;
    a.heavy = sc.maxdeg > HEAVY ? 1u : 0u;
    // one step of one workgroup (groups of G lanes).  Measured with 0 / 1 / 4 /
    // 16 steps: ring of 100,003 53.5 / 51.8 / 55.2 / 85.9 ms, 4-grid of 930
    // vertices 0.59 / 0.45 / 0.45 / 0.46 ms.
    a.solo = NT >> a.glog;
    a.max_phases = (u32)std::min<u64>(0xFFFFFFF0ull, 64ull * n + (1ull << 20));
    a.c = dctl;
    hipLaunchKernelGGL(k_nf_init, dim3(std::min<u32>(4096, (n + 255) / 256)), dim3(256), 0, s, (u64*)dist_out,
                       a.nstamp, a.fstamp, a.done_at, n, source);
    NFCHK(hipGetLastError());
    // the source is the first near frontier (heavy if its degree is)
    u64 so[2];
    NFCHK(hipMemcpyAsync(so, offsets + source, sizeof so, hipMemcpyDeviceToHost, s));
    NFCHK(hipStreamSynchronize(s));
    const bool heavy = so[1] - so[0] > HEAVY;
    ctl.cl[0].w = heavy ? 0 : 1;
    ctl.ch[0].w = heavy ? 1 : 0;
    ctl.fmin[0] = ctl.fmin[1] = KINF;
    ctl.ph.mode = RELAX;
    ctl.ph.src = 0;
    ctl.ph.dst = 1;
    ctl.ph.nl = heavy ? 0 : 1;
    ctl.ph.nh = heavy ? 1 : 0;
    ctl.ph.fsrc = 1;
    ctl.ph.fdst = 0;
    ctl.ph.phase = 0;
    ctl.ph.epoch = 0;
    ctl.ph.T = delta;
    NFCHK(hipMemcpyAsync(dctl, &ctl, sizeof ctl, hipMemcpyHostToDevice, s));
    const u32 srcv = source;
    NFCHK(hipMemcpyAsync(heavy ? a.qh[0] : a.ql[0], &srcv, sizeof(u32), hipMemcpyHostToDevice, s));
    NFCHK(hipGetDevice(&dev));
    NFCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    NFCHK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_nearfar, NT, 0));
    if (occ < 1) {
      rc = nf_fail(PBH_EDEVICE, "the near-far kernel cannot be resident");
      goto out;
    }
    NFCHK(hipEventCreate(&e0));
    NFCHK(hipEventCreate(&e1));
    NFCHK(hipEventRecord(e0, s));
    {
      void* args[] = {&a};
      NFCHK(hipLaunchCooperativeKernel((const void*)k_nearfar, dim3(cus), dim3(NT), args, 0, s));
    }
    NFCHK(hipEventRecord(e1, s));
    NFCHK(hipMemcpyAsync(&ctl, dctl, sizeof ctl, hipMemcpyDeviceToHost, s));
    NFCHK(hipStreamSynchronize(s));
    NFCHK(hipEventElapsedTime(&ms, e0, e1));
    if (ctl.err.w) {
      rc = nf_fail(ctl.err.w & ERR_TIMEOUT ? PBH_ETIMEOUT : PBH_EINTERNAL,
                   ctl.err.w & ERR_TIMEOUT ? "a grid barrier wait ran out" :
                   ctl.err.w & ERR_OVERFLOW ? "a frontier queue overflowed" : "phase or time limit reached");
      goto out;
    }
    if (stats) {
      stats->relaxations = ctl.relax;
      stats->phases = ctl.phases;
      stats->splits = ctl.ph.epoch;
      stats->delta = delta;
      stats->workgroups = (uint32_t)cus;
      stats->kernel_ms = ms;
    }
  }
out:
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (buf) {
    (void)hipStreamSynchronize(s);
    (void)hipFree(buf);
  }
  return rc;
}

}  // extern "C"
