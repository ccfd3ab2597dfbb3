// The phases of Near-Far and the grid barrier between them (nearfar.hip says
// what they do), written once against a grid of workgroups E: the GPU's, or one
// whose threads the CPU tests interleave at every memory access.
//
// E gives the sizes (NT threads a workgroup, wavefronts of W, HEAVY, PUSHES),
// the workgroup's place, its barrier (sync), the wait for a thread's own memory
// operations (wait_mem), the real-time clock, agent-scope relaxed loads, stores
// and atomics, and Word, a 32-bit word in LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define NF_INL __host__ __device__ __forceinline__

namespace bkt {

typedef unsigned long long u64;
typedef unsigned int u32;

namespace nf {

constexpr u64 KINF = ~0ull;
constexpr u32 NONE = ~0u;
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
  Line arrive[9], gen, err;  // arrivals at barriers so far: per group of workgroups, then of the groups
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

// Pushes gathered in LDS: light near vertices from the front, far ones from
// the back, and the smallest far key (heavy vertices, rare, go out one by one).
template <class E>
struct Gather {
  u32 buf[E::PUSHES];
  typename E::Word nn, nf, slot_n, slot_f;
  u64 fmin;
  u32 ws[E::NT / E::W];  // steps of each wavefront
};

template <class E>
NF_INL void overflow(const E& t, const Args& a) {
  t.or32(&a.c->err.w, ERR_OVERFLOW);
}

// Writes the gathered pushes out (every thread of the workgroup calls it).
template <class E>
NF_INL void flush(const E& t, const Args& a, const Phase& ph, Gather<E>* q) {
  t.sync();
  const u32 nn = q->nn, nf = q->nf;
  if (nn + nf) {
    if (t.tid() == 0) {
      q->slot_n = nn ? t.add32(&a.c->cl[ph.dst].w, nn) : 0u;
      q->slot_f = nf ? t.add32(&a.c->cf[ph.fdst].w, nf) : 0u;
      if (nf) t.min64(&a.c->fmin[ph.fdst], q->fmin);
    }
    t.sync();
    const u32 sn = q->slot_n, sf = q->slot_f;
    for (u32 x = t.tid(); x < nn; x += E::NT) {
      if (sn + x < a.cap)
        t.st32(a.ql[ph.dst] + sn + x, q->buf[x]);
      else
        overflow(t, a);
    }
    for (u32 x = t.tid(); x < nf; x += E::NT) {
      if (sf + x < a.cap)
        t.st32(a.far[ph.fdst] + sf + x, q->buf[E::PUSHES - 1 - x]);
      else
        overflow(t, a);
    }
    t.sync();
    if (t.tid() == 0) {
      q->nn = q->nf = 0;
      q->fmin = KINF;
    }
  }
  t.sync();
}

// Files vertex v with key `key` (improved in this phase): near (below T) or
// far, each at most once per phase / epoch.  Between two flushes a workgroup
// files at most PUSHES vertices (room()).
template <class E>
NF_INL void file(const E& t, const Args& a, const Phase& ph, Gather<E>* q, bool imp, u32 v, u64 key) {
  const bool near = imp && key < ph.T;
  const bool fresh_near = near && t.xchg32(a.nstamp + v, ph.phase) != ph.phase;
  const bool fresh_far = imp && !near && t.xchg32(a.fstamp + v, ph.epoch) != ph.epoch;
  bool heavy = false;
  if (a.heavy && fresh_near) heavy = a.off[v + 1] - a.off[v] > E::HEAVY;
  if (heavy) {
    const u32 s = t.add32(&a.c->ch[ph.dst].w, 1u);
    if (s < a.cap)
      t.st32(a.qh[ph.dst] + s, v);
    else
      overflow(t, a);
  } else if (fresh_near) {
    q->buf[t.lds_next(&q->nn)] = v;
  }
  if (fresh_far) {
    q->buf[E::PUSHES - 1 - t.lds_next(&q->nf)] = v;
    t.lds_min(&q->fmin, key);
  }
}

// Makes sure the next file() of every thread finds room (each files at most
// one vertex).  `left` counts the calls that are sure to fit; every thread of
// the workgroup has the same value and makes the same calls, so the barriers
// are only passed when it runs out, by all of them.
template <class E>
NF_INL void room(const E& t, const Args& a, const Phase& ph, Gather<E>* q, u32& left) {
  if (left == 0) {
    t.sync();
    const u32 used = q->nn + q->nf;
    t.sync();  // (no push before every thread has read it)
    if (used + E::NT > E::PUSHES) {
      flush(t, a, ph, q);
      left = E::PUSHES / E::NT;
    } else {
      left = (E::PUSHES - used) / E::NT;
    }
  }
  --left;
}

// Relaxes edge e out of a vertex at distance du; files an improved target.
template <class E>
NF_INL void relax_edge(const E& t, const Args& a, const Phase& ph, Gather<E>* q, bool in, u64 e, u64 du) {
  u32 v = 0;
  u64 cand = 0;
  bool imp = false;
  if (in) {
    v = a.tg[e];
    cand = du + (u64)a.wt[e];
    imp = cand < t.min64(a.dist + v, cand);
  }
  file(t, a, ph, q, imp, v, cand);
}

// Leader of a grid barrier: turns the queue sizes of the phase that ended
// into the next phase's descriptor (every other workgroup is waiting).
template <class E>
__host__ __device__ inline void lead(const E& t, const Args& a, Phase& ph) {
  // The phase that ended tells where its results are, so everything read
  // here is read at once: one round trip.
  Ctl* c = a.c;
  const u32 d = ph.dst, f = ph.fdst;
  const u32 nl = t.ld32(&c->cl[d].w), nh = t.ld32(&c->ch[d].w), nf = t.ld32(&c->cf[f].w);
  const u64 fm = t.ld64(&c->fmin[f]);
  const u32 phases = ph.phase + 1;
  t.st32(&c->phases, phases);
  const u64 now = t.clock();
  if (ph.t0 == 0) ph.t0 = now;
  if (phases > a.max_phases || now - ph.t0 > RUN_LIMIT_TICKS) {
    t.or32(&c->err.w, ERR_PHASES);
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
    t.st32(&c->cl[d ^ 1].w, 0u);
    t.st32(&c->ch[d ^ 1].w, 0u);
    return;
  }
  if (nf == 0) {
    ph.mode = DONE;
    return;
  }
  // Next threshold: one Delta further, or the first multiple of Delta past
  // the smallest key filed in the far pile if that is further.
  u64 next = ph.T + a.delta < ph.T ? KINF : ph.T + a.delta;
  if (fm != KINF) {
    const u64 j = (fm / a.delta + 1) * a.delta;
    const u64 jt = j < fm ? KINF : j;  // saturate
    next = jt > next ? jt : next;
  }
  ph.T = next;
  ph.mode = SPLIT;
  ph.dst = d;  // empty: the relax phase that ended filed nothing near
  ph.fsrc = f;
  ph.fdst = f ^ 1;
  ph.nf = nf < a.cap ? nf : a.cap;
  ph.epoch += 1;
  t.st32(&c->cf[f ^ 1].w, 0u);
  t.st64(&c->fmin[f ^ 1], KINF);
}

// One phase's work by `nwg` workgroups, this one being number `wg` of them.
template <class E>
NF_INL void do_phase(const E& t, const Args& a, const Phase& ph, Gather<E>* q, u32 wg, u32 nwg, u64& scanned) {
  const u32 G = 1u << a.glog;
  const u32 gtid = wg * E::NT + t.tid();
  const u32 nthreads = nwg * E::NT;
  const u32 sub = gtid >> a.glog, nsub = nthreads >> a.glog, lig = t.tid() & (G - 1);
  u32 left = E::PUSHES / E::NT;  // the gather starts empty
  if (ph.mode == RELAX) {
    // light vertices: one group of G lanes per vertex, striding its edges
    const u32 rounds_l = (ph.nl + nsub - 1) / nsub;
    for (u32 r = 0; r < rounds_l; ++r) {
      const u32 j = r * nsub + sub;
      bool have = j < ph.nl;
      const u32 u = have ? t.ld32(a.ql[ph.src] + j) : 0u;
      // a vertex is in the queue once, so its last-scan mark is this group's
      // alone in this phase (no exchange needed); its distance may fall
      // meanwhile, so the group goes by what its first lane has read
      u64 du = have ? t.ld64(a.dist + u) : 0ull, seen = have ? t.ld64(a.done_at + u) : 0ull;
      const u64 r0 = have ? a.off[u] : 0ull, r1 = have ? a.off[u + 1] : 0ull;
      du = t.from_lane(du, t.tid() & ~(G - 1));
      seen = t.from_lane(seen, t.tid() & ~(G - 1));
      have = have && seen != du;  // already scanned at this distance (filed twice): skipped
      if (have && lig == 0) t.st64(a.done_at + u, du);
      const u64 e0 = have ? r0 : 0ull, e1 = have ? r1 : 0ull;
      const u64 deg = e1 - e0;
      scanned += lig == 0 ? deg : 0;
      // every wavefront of the workgroup runs the same number of steps (the
      // largest degree in it): room() counts them
      u32 steps = (u32)((deg + G - 1) / G);
      steps = t.wave_max(steps);
      if (t.tid() % E::W == 0) q->ws[t.tid() / E::W] = steps;
      t.sync();
#pragma unroll
      for (int w = 0; w < E::NT / E::W; ++w) steps = q->ws[w] > steps ? q->ws[w] : steps;
      for (u32 s = 0; s < steps; ++s) {
        room(t, a, ph, q, left);
        const u64 e = e0 + (u64)s * G + lig;
        relax_edge(t, a, ph, q, e < e1, e, du);
      }
      t.sync();
    }
    // heavy vertices: every workgroup takes a share of each one's edges
    // (always scanned: every workgroup would have to agree on a skip)
    for (u32 h = 0; h < ph.nh; ++h) {
      const u32 u = t.ld32(a.qh[ph.src] + h);
      const u64 du = t.ld64(a.dist + u);
      const u64 e0 = a.off[u], e1 = a.off[u + 1];
      if (gtid == 0) scanned += e1 - e0;
      const u64 span = e1 - e0;
      const u64 steps = (span + nthreads - 1) / nthreads;
      for (u64 s = 0; s < steps; ++s) {
        room(t, a, ph, q, left);
        const u64 e = e0 + s * nthreads + gtid;
        relax_edge(t, a, ph, q, e < e1, e, du);
      }
    }
  } else {  // SPLIT: far vertices now below T become the near frontier
    const u32 rounds_f = (ph.nf + nthreads - 1) / nthreads;
    for (u32 r = 0; r < rounds_f; ++r) {
      room(t, a, ph, q, left);
      const u32 j = r * nthreads + gtid;
      const bool have = j < ph.nf;
      const u32 v = have ? t.ld32(a.far[ph.fsrc] + j) : 0u;
      const u64 dv = have ? t.ld64(a.dist + v) : KINF;
      file(t, a, ph, q, have, v, dv);
    }
  }
  flush(t, a, ph, q);
}

// Is the phase one workgroup's work?
template <class E>
NF_INL bool solo(const Args& a, const Phase& ph) {
  return ph.mode == RELAX ? ph.nh == 0 && ph.nl <= a.solo : ph.mode == SPLIT && ph.nf <= E::NT;
}

// Grid barrier, the `nth` of the run (from 0).  Every thread first waits for
// its own memory operations; one arrival per workgroup; the last one runs
// lead(), then the small phases that follow, and sets the generation that the
// others spin on to nth + 1.  The arrivals are counted on from barrier to
// barrier: a reset would have to reach memory before the next barrier's first
// arrival, and the thread that makes it is not the one that lets the others go.
// Returns false once the run has failed.
template <class E>
__host__ __device__ inline bool grid_sync(const E& t, const Args& a, Phase& ph, Phase* sph, typename E::Word* sflag,
                                          Gather<E>* q, u64& scanned, u32 nth) {
  t.wait_mem();
  t.sync();
  Ctl* c = a.c;
  if (t.tid() == 0) {
    // one word takes about 10 ns per arrival: eight groups, then their last
    // ones (workgroups go round the dies, so a group is a die's)
    const u32 grp = t.wg() & 7u, ngrp = t.nwg() < 8u ? t.nwg() : 8u;
    bool last = t.add32(&c->arrive[grp].w, 1u) + 1u == (nth + 1u) * ((t.nwg() - grp + 7u) / 8u);
    if (last) last = t.add32(&c->arrive[8].w, 1u) + 1u == (nth + 1u) * ngrp;
    if (last) {
      lead(t, a, ph);
      *sph = ph;
      *sflag = 2;
    } else {
      u64 t0 = t.clock();
      u32 at = t.ld32(&c->phases);
      while (t.ld32(&c->gen.w) == nth) {
        if (t.ld32(&c->err.w)) break;
        if (t.clock() - t0 > TIMEOUT_TICKS) {
          // the last workgroup may be at small phases of its own: it is alive
          // while it counts them
          const u32 now = t.ld32(&c->phases);
          if (now != at) {
            at = now;
            t0 = t.clock();
            continue;
          }
          t.or32(&c->err.w, ERR_TIMEOUT);
          break;
        }
        t.nap();
      }
      const u32* gp = reinterpret_cast<const u32*>(&c->ph);
      u32* d = reinterpret_cast<u32*>(&ph);
      for (u32 i = 0; i < sizeof(Phase) / 4; ++i) d[i] = t.ld32(gp + i);
      *sph = ph;
      *sflag = t.ld32(&c->err.w) ? 1 : 0;
    }
  }
  t.sync();
  ph = *sph;
  const u32 flag = *sflag;
  if (flag == 2) {
    // (every wavefront has read the flag before thread 0 writes it again: one
    // that read it late would pass by this block and its barriers)
    t.sync();
    u32 bad = 0;
    while (solo<E>(a, ph)) {
      do_phase(t, a, ph, q, 0u, 1u, scanned);
      t.wait_mem();
      t.sync();
      if (t.tid() == 0) {
        *sflag = t.ld32(&c->err.w);
        if (!*sflag) lead(t, a, ph);
        *sph = ph;
      }
      t.sync();
      ph = *sph;
      bad = *sflag;
      t.sync();
      if (bad) break;
    }
    if (t.tid() == 0) {
      u32* src = reinterpret_cast<u32*>(&ph);
      u32* dstp = reinterpret_cast<u32*>(&c->ph);
      for (u32 i = 0; i < sizeof(Phase) / 4; ++i) t.st32(dstp + i, src[i]);
      t.wait_mem();
      t.st32(&c->gen.w, nth + 1u);
      *sflag = t.ld32(&c->err.w) ? 1 : 0;
    }
    t.sync();
    return *sflag == 0;
  }
  return flag == 0;
}

// The run: phase after phase until the leader says DONE or the run has failed;
// returns the edges this thread scanned.
template <class E>
NF_INL u64 phases(const E& t, const Args& a, Phase* sph, typename E::Word* sflag, Gather<E>* q) {
  Phase ph;
  if (t.tid() == 0) {
    const u32* gp = reinterpret_cast<const u32*>(&a.c->ph);
    u32* d = reinterpret_cast<u32*>(sph);
    for (u32 i = 0; i < sizeof(Phase) / 4; ++i) d[i] = t.ld32(gp + i);
    q->nn = q->nf = 0;
    q->fmin = KINF;
  }
  t.sync();
  ph = *sph;
  u64 scanned = 0;
  for (u32 nth = 0; ph.mode != DONE; ++nth) {
    do_phase(t, a, ph, q, t.wg(), t.nwg(), scanned);
    if (!grid_sync(t, a, ph, sph, sflag, q, scanned, nth)) break;
  }
  return scanned;
}

}  // namespace nf
}  // namespace bkt
