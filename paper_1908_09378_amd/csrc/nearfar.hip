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
#include "pbh_team.h"

namespace bkt {
namespace nf {

constexpr u64 KINF = ~0ull;
constexpr u32 NONE = ~0u;
constexpr int NT = 512;          // threads per workgroup
constexpr u32 HEAVY = 1024;      // out-degree above which a vertex is scanned by the whole grid
constexpr u32 PUSHES = 4096;     // near / far pushes gathered per workgroup before they are written out
constexpr u64 TIMEOUT_TICKS = 2000000000ull;  // 20 s of the 100 MHz real-time clock
constexpr u64 RUN_LIMIT_TICKS = 12000000000ull;  // 120 s: a run that long is stopped

enum { RELAX = 0, SPLIT = 1, DONE = 2 };
enum { ERR_TIMEOUT = 1, ERR_OVERFLOW = 2, ERR_PHASES = 4 };

// Phase descriptor, written by the barrier's leader.
struct Phase {
  u32 mode;
  u32 src, dst;     // near queues read (relax) and written
  u32 nl, nh;       // relax: light and heavy vertices in queue src
  u32 fsrc, fdst;   // far piles: split reads fsrc; relax and split append to fdst
  u32 nf;           // split: entries of fsrc
  u32 phase;        // stamp of near pushes in this phase
  u32 epoch;        // stamp of far pushes
  u64 T;            // threshold
  u64 t0;           // real-time clock at the first barrier
};

// Words that different workgroups update at the same time are lines apart.
struct alignas(128) Line {
  u32 w;
  u32 pad_[31];
};
struct Ctl {
  Line arrive[9], gen, err;  // arrivals at a barrier: per group of workgroups, then of the groups
  Line cl[2], ch[2];  // near queue sizes (light, heavy)
  Line cf[2];         // far pile sizes
  alignas(128) u64 fmin[2];  // smallest key filed in each far pile
  alignas(128) u64 relax;    // edges scanned
  alignas(128) u32 phases;   // phases ended (also a sign of life)
  Phase ph;
};

struct Args {
  const u64* off;
  const u32* tg;
  const u32* wt;
  u64* dist;
  u32 n;
  u64 delta;
  u32 glog;         // light vertices: groups of 2^glog lanes
  u32* ql[2];       // near queues, light vertices
  u32* qh[2];       // near queues, heavy vertices
  u32* far[2];      // far piles
  u32* nstamp;      // per vertex: phase of its last near push
  u32* fstamp;      // per vertex: epoch of its last far filing
  u64* done_at;     // per vertex: the distance at which its edges were last scanned
  u32 cap;          // capacity of every queue and pile
  u32 heavy;        // some vertex has more than HEAVY out-edges
  u32 solo;         // frontiers of at most this many vertices are one workgroup's
  u32 max_phases;
  Ctl* c;
};

__device__ __forceinline__ u32 ld32(const u32* p) {
  return __hip_atomic_load((const u32 PBH_GLB*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 ld64(const u64* p) {
  return __hip_atomic_load((const u64 PBH_GLB*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st32(u32* p, u32 v) {
  __hip_atomic_store((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st64(u64* p, u64 v) {
  __hip_atomic_store((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u32 xchg32(u32* p, u32 v) {
  return __hip_atomic_exchange((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 xchg64(u64* p, u64 v) {
  return __hip_atomic_exchange((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u32 add32(u32* p, u32 v) {
  return __hip_atomic_fetch_add((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 min64(u64* p, u64 v) {
  return __hip_atomic_fetch_min((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Pushes gathered in LDS: light near vertices from the front, far ones from
// the back, and the smallest far key (heavy vertices, rare, go out one by one).
struct Gather {
  u32 buf[PUSHES];
  u32 nn, nf, slot_n, slot_f;
  u64 fmin;
};

__device__ __forceinline__ void overflow(const Args& a) {
  __hip_atomic_fetch_or((u32 PBH_GLB*)&a.c->err.w, (u32)ERR_OVERFLOW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Writes the gathered pushes out (every thread of the workgroup calls it).
__device__ __forceinline__ void flush(const Args& a, const Phase& ph, Gather* q) {
  __syncthreads();
  const u32 nn = q->nn, nf = q->nf;
  if (nn + nf) {
    if (threadIdx.x == 0) {
      q->slot_n = nn ? add32(&a.c->cl[ph.dst].w, nn) : 0u;
      q->slot_f = nf ? add32(&a.c->cf[ph.fdst].w, nf) : 0u;
      if (nf) min64(&a.c->fmin[ph.fdst], q->fmin);
    }
    __syncthreads();
    const u32 sn = q->slot_n, sf = q->slot_f;
    for (u32 x = threadIdx.x; x < nn; x += NT) {
      if (sn + x < a.cap)
        st32(a.ql[ph.dst] + sn + x, q->buf[x]);
      else
        overflow(a);
    }
    for (u32 x = threadIdx.x; x < nf; x += NT) {
      if (sf + x < a.cap)
        st32(a.far[ph.fdst] + sf + x, q->buf[PUSHES - 1 - x]);
      else
        overflow(a);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      q->nn = q->nf = 0;
      q->fmin = KINF;
    }
  }
  __syncthreads();
}

// Files vertex v with key `key` (improved in this phase): near (below T) or
// far, each at most once per phase / epoch.  Between two flushes a workgroup
// files at most PUSHES vertices (room()).
__device__ __forceinline__ void file(const Args& a, const Phase& ph, Gather* q, bool imp, u32 v, u64 key) {
  const bool near = imp && key < ph.T;
  const bool fresh_near = near && xchg32(a.nstamp + v, ph.phase) != ph.phase;
  const bool fresh_far = imp && !near && xchg32(a.fstamp + v, ph.epoch) != ph.epoch;
  bool heavy = false;
  if (a.heavy && fresh_near) heavy = a.off[v + 1] - a.off[v] > HEAVY;
  if (heavy) {
    const u32 s = add32(&a.c->ch[ph.dst].w, 1u);
    if (s < a.cap)
      st32(a.qh[ph.dst] + s, v);
    else
      overflow(a);
  } else if (fresh_near) {
    q->buf[__hip_atomic_fetch_add((u32 PBH_LDS*)&q->nn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = v;
  }
  if (fresh_far) {
    q->buf[PUSHES - 1 -
           __hip_atomic_fetch_add((u32 PBH_LDS*)&q->nf, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = v;
    __hip_atomic_fetch_min((u64 PBH_LDS*)&q->fmin, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// Makes sure the next file() of every thread finds room (each files at most
// one vertex).  `left` counts the calls that are sure to fit; every thread of
// the workgroup has the same value and makes the same calls, so the barriers
// are only passed when it runs out, by all of them.
__device__ __forceinline__ void room(const Args& a, const Phase& ph, Gather* q, u32& left) {
  if (left == 0) {
    __syncthreads();
    const u32 used = q->nn + q->nf;
    __syncthreads();  // (no push before every thread has read it)
    if (used + NT > PUSHES) {
      flush(a, ph, q);
      left = PUSHES / NT;
    } else {
      left = (PUSHES - used) / NT;
    }
  }
  --left;
}

// Relaxes edge e out of a vertex at distance du; files an improved target.
__device__ __forceinline__ void relax_edge(const Args& a, const Phase& ph, Gather* q, bool in, u64 e, u64 du) {
  u32 v = 0;
  u64 cand = 0;
  bool imp = false;
  if (in) {
    v = a.tg[e];
    cand = du + (u64)a.wt[e];
    imp = cand < min64(a.dist + v, cand);
  }
  file(a, ph, q, imp, v, cand);
}

// Leader of a grid barrier: turns the queue sizes of the phase that ended
// into the next phase's descriptor (every other workgroup is waiting).
__device__ void lead(const Args& a, Phase& ph) {
  // The phase that ended tells where its results are, so everything read
  // here is read at once: one round trip.
  Ctl* c = a.c;
  const u32 d = ph.dst, f = ph.fdst;
  const u32 nl = ld32(&c->cl[d].w), nh = ld32(&c->ch[d].w), nf = ld32(&c->cf[f].w);
  const u64 fm = ld64(&c->fmin[f]);
  const u32 phases = ph.phase + 1;
  st32(&c->phases, phases);
  const u64 now = __builtin_amdgcn_s_memrealtime();
  if (ph.t0 == 0) ph.t0 = now;
  if (phases > a.max_phases || now - ph.t0 > RUN_LIMIT_TICKS) {
    __hip_atomic_fetch_or((u32 PBH_GLB*)&c->err.w, (u32)ERR_PHASES, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ph.mode = DONE;
    return;
  }
  ph.phase += 1;
  if (nl + nh > 0) {
    ph.mode = RELAX;
    ph.src = d;
    ph.dst = d ^ 1;
    ph.nl = nl < a.cap ? nl : a.cap;
    ph.nh = nh < a.cap ? nh : a.cap;
    st32(&c->cl[d ^ 1].w, 0u);
    st32(&c->ch[d ^ 1].w, 0u);
    return;
  }
  if (nf == 0) {
    ph.mode = DONE;
    return;
  }
  // Next threshold: one Delta further, or the first multiple of Delta past
  // the smallest key filed in the far pile if that is further.
  u64 t = ph.T + a.delta < ph.T ? KINF : ph.T + a.delta;
  if (fm != KINF) {
    const u64 j = (fm / a.delta + 1) * a.delta;
    const u64 jt = j < fm ? KINF : j;  // saturate
    t = jt > t ? jt : t;
  }
  ph.T = t;
  ph.mode = SPLIT;
  ph.dst = d;  // empty: the relax phase that ended filed nothing near
  ph.fsrc = f;
  ph.fdst = f ^ 1;
  ph.nf = nf < a.cap ? nf : a.cap;
  ph.epoch += 1;
  st32(&c->cf[f ^ 1].w, 0u);
  st64(&c->fmin[f ^ 1], KINF);
}

// One phase's work by `nwg` workgroups, this one being number `wg` of them.
__device__ __forceinline__ void do_phase(const Args& a, const Phase& ph, Gather* q, u32 wg, u32 nwg, u64& scanned) {
  const u32 G = 1u << a.glog;
  const u32 gtid = wg * NT + threadIdx.x;
  const u32 nthreads = nwg * NT;
  const u32 sub = gtid >> a.glog, nsub = nthreads >> a.glog, lig = threadIdx.x & (G - 1);
  u32 left = PUSHES / NT;  // the gather starts empty
  if (ph.mode == RELAX) {
    // light vertices: one group of G lanes per vertex, striding its edges
    const u32 rounds_l = (ph.nl + nsub - 1) / nsub;
    for (u32 r = 0; r < rounds_l; ++r) {
      const u32 j = r * nsub + sub;
      bool have = j < ph.nl;
      const u32 u = have ? ld32(a.ql[ph.src] + j) : 0u;
      // a vertex is in the queue once, so its last-scan mark is this group's
      // alone in this phase (no exchange needed)
      const u64 du = have ? ld64(a.dist + u) : 0ull, seen = have ? ld64(a.done_at + u) : 0ull;
      const u64 r0 = have ? a.off[u] : 0ull, r1 = have ? a.off[u + 1] : 0ull;
      have = have && seen != du;  // already scanned at this distance (filed twice): skipped
      if (have && lig == 0) st64(a.done_at + u, du);
      const u64 e0 = have ? r0 : 0ull, e1 = have ? r1 : 0ull;
      const u64 deg = e1 - e0;
      scanned += lig == 0 ? deg : 0;
      // every wavefront of the workgroup runs the same number of steps (the
      // largest degree in it): room() counts them
      u32 steps = (u32)((deg + G - 1) / G);
      for (int o = 32; o > 0; o >>= 1) {
        const u32 s2 = (u32)__shfl_xor((int)steps, o, 64);
        steps = s2 > steps ? s2 : steps;
      }
      __shared__ u32 ws[NT / 64];
      if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = steps;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) steps = ws[w] > steps ? ws[w] : steps;
      for (u32 s = 0; s < steps; ++s) {
        room(a, ph, q, left);
        const u64 e = e0 + (u64)s * G + lig;
        relax_edge(a, ph, q, e < e1, e, du);
      }
      __syncthreads();
    }
    // heavy vertices: every workgroup takes a share of each one's edges
    // (always scanned: every workgroup would have to agree on a skip)
    for (u32 h = 0; h < ph.nh; ++h) {
      const u32 u = ld32(a.qh[ph.src] + h);
      const u64 du = ld64(a.dist + u);
      const u64 e0 = a.off[u], e1 = a.off[u + 1];
      if (gtid == 0) scanned += e1 - e0;
      const u64 span = e1 - e0;
      const u64 steps = (span + nthreads - 1) / nthreads;
      for (u64 s = 0; s < steps; ++s) {
        room(a, ph, q, left);
        const u64 e = e0 + s * nthreads + gtid;
        relax_edge(a, ph, q, e < e1, e, du);
      }
    }
  } else {  // SPLIT: far vertices now below T become the near frontier
    const u32 rounds_f = (ph.nf + nthreads - 1) / nthreads;
    for (u32 r = 0; r < rounds_f; ++r) {
      room(a, ph, q, left);
      const u32 j = r * nthreads + gtid;
      const bool have = j < ph.nf;
      const u32 v = have ? ld32(a.far[ph.fsrc] + j) : 0u;
      const u64 dv = have ? ld64(a.dist + v) : KINF;
      file(a, ph, q, have, v, dv);
    }
  }
  flush(a, ph, q);
}

// Is the phase one workgroup's work?
__device__ __forceinline__ bool solo(const Args& a, const Phase& ph) {
  return ph.mode == RELAX ? ph.nh == 0 && ph.nl <= a.solo : ph.mode == SPLIT && ph.nf <= NT;
}

// Grid barrier.  Every thread first waits for its own memory operations;
// one arrival per workgroup; the last one runs lead(), then the small phases
// that follow, and bumps the generation the others spin on.  Returns false
// once the run has failed.
__device__ bool grid_sync(const Args& a, Phase& ph, Phase* sph, u32* sflag, Gather* q, u64& scanned) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  Ctl* c = a.c;
  if (threadIdx.x == 0) {
    const u32 g = ld32(&c->gen.w);
    // one word takes about 10 ns per arrival: eight groups, then their last
    // ones (workgroups go round the dies, so a group is a die's)
    const u32 grp = blockIdx.x & 7u, ngrp = gridDim.x < 8u ? gridDim.x : 8u;
    bool last = add32(&c->arrive[grp].w, 1u) == (gridDim.x - grp + 7u) / 8u - 1u;
    if (last) {
      st32(&c->arrive[grp].w, 0u);
      last = add32(&c->arrive[8].w, 1u) == ngrp - 1u;
    }
    if (last) {
      st32(&c->arrive[8].w, 0u);
      lead(a, ph);
      *sph = ph;
      *sflag = 2;
    } else {
      u64 t0 = __builtin_amdgcn_s_memrealtime();
      u32 at = ld32(&c->phases);
      while (ld32(&c->gen.w) == g) {
        if (ld32(&c->err.w)) break;
        if (__builtin_amdgcn_s_memrealtime() - t0 > TIMEOUT_TICKS) {
          // the last workgroup may be at small phases of its own: it is alive
          // while it counts them
          const u32 now = ld32(&c->phases);
          if (now != at) {
            at = now;
            t0 = __builtin_amdgcn_s_memrealtime();
            continue;
          }
          __hip_atomic_fetch_or((u32 PBH_GLB*)&c->err.w, (u32)ERR_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
      const u32* gp = reinterpret_cast<const u32*>(&c->ph);
      u32* d = reinterpret_cast<u32*>(&ph);
      for (u32 i = 0; i < sizeof(Phase) / 4; ++i) d[i] = ld32(gp + i);
      *sph = ph;
      *sflag = ld32(&c->err.w) ? 1 : 0;
    }
  }
  __syncthreads();
  ph = *sph;
  if (*sflag == 2) {
    u32 bad = 0;
    while (solo(a, ph)) {
      do_phase(a, ph, q, 0u, 1u, scanned);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (threadIdx.x == 0) {
        *sflag = ld32(&c->err.w);
        if (!*sflag) lead(a, ph);
        *sph = ph;
      }
      __syncthreads();
      ph = *sph;
      bad = *sflag;
      __syncthreads();
      if (bad) break;
    }
    if (threadIdx.x == 0) {
      u32* src = reinterpret_cast<u32*>(&ph);
      u32* dstp = reinterpret_cast<u32*>(&c->ph);
      for (u32 i = 0; i < sizeof(Phase) / 4; ++i) st32(dstp + i, src[i]);
      __builtin_amdgcn_s_waitcnt(0);
      st32(&c->gen.w, ld32(&c->gen.w) + 1u);
      *sflag = ld32(&c->err.w) ? 1 : 0;
    }
    __syncthreads();
  }
  return *sflag == 0;
}

__global__ __launch_bounds__(NT) void k_nearfar(Args a) {
  __shared__ Phase sph;
  __shared__ u32 sflag;
  __shared__ Gather q;
  Phase ph;
  if (threadIdx.x == 0) {
    const u32* gp = reinterpret_cast<const u32*>(&a.c->ph);
    u32* d = reinterpret_cast<u32*>(&sph);
    for (u32 i = 0; i < sizeof(Phase) / 4; ++i) d[i] = ld32(gp + i);
    q.nn = q.nf = 0;
    q.fmin = KINF;
  }
  __syncthreads();
  ph = sph;
  u64 scanned = 0;
  while (ph.mode != DONE) {
    do_phase(a, ph, &q, blockIdx.x, gridDim.x, scanned);
    if (!grid_sync(a, ph, &sph, &sflag, &q, scanned)) break;
  }
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
