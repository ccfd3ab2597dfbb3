// Near-Far's phases and grid barrier (nearfar_core.h) on the CPU, for tests:
// a few small workgroups whose threads are fibers, which give way at every
// access to memory that others see.  With `late_stores`, a store reaches other
// workgroups at any time up to its thread's next wait for its own operations,
// and not in the order of the thread's other operations; the thread itself and
// its workgroup see it at once.
#include <cstring>
#include <map>
#include <vector>

#include "../../paper_1908_09378_amd/csrc/nearfar_core.h"
#include "fibers.h"

using namespace bkt;
using namespace bkt::nf;

namespace {

struct Store {
  u32 thread;
  void* p;
  u64 v;
  int bytes;
};

struct Machine {
  fibers::Pool* pool;
  u32 nwg, nt, nw;
  bool late_stores;
  std::vector<fibers::Barrier> wgb, waveb;
  std::vector<Store> pending;      // in order of issue
  std::vector<u64> lane_value[2];  // exchanged between the lanes of a wavefront
  std::vector<u32> turn;           // of each thread, which of the two

  static void land(const Store& s) { std::memcpy(s.p, &s.v, (size_t)s.bytes); }
  // Lands thread t's stores (all of them).
  void drain(u32 t) {
    size_t k = 0;
    for (Store& s : pending)
      if (s.thread == t)
        land(s);
      else
        pending[k++] = s;
    pending.resize(k);
  }
  // An access to p by thread t: its workgroup's stores to p come first.
  void before(u32 t, const void* p) {
    pool->give_way();
    size_t k = 0;
    for (Store& s : pending)
      if (s.p == p && s.thread / nt == t / nt)
        land(s);
      else
        pending[k++] = s;
    pending.resize(k);
    if (!pending.empty() && pool->random() % 16 == 0) {  // one store lands (the oldest to its place)
      const void* at = pending[pool->random() % pending.size()].p;
      for (size_t i = 0; i < pending.size(); ++i)
        if (pending[i].p == at) {
          land(pending[i]);
          pending.erase(pending.begin() + (long)i);
          break;
        }
    }
  }
  void store(u32 t, void* p, u64 v, int bytes) {
    before(t, p);
    const Store s{t, p, v, bytes};
    if (late_stores)
      pending.push_back(s);
    else
      land(s);
  }
};
Machine* g_m;

// A word in LDS: every read and write gives way first.
struct LdsWord {
  u32 v;
  operator u32() const {
    g_m->pool->give_way();
    return v;
  }
  LdsWord& operator=(u32 x) {
    g_m->pool->give_way();
    v = x;
    return *this;
  }
  LdsWord& operator=(const LdsWord& o) { return *this = (u32)o; }
};

struct FiberGrid {
  static constexpr int NT = 4, W = 2;
  static constexpr u32 HEAVY = 6, PUSHES = 8;
  using Word = LdsWord;
  static u32 me() { return g_m->pool->current; }
  u32 tid() const { return me() % NT; }
  u32 wg() const { return me() / NT; }
  u32 nwg() const { return g_m->nwg; }
  void sync(int line = __builtin_LINE()) const { g_m->pool->wait(g_m->wgb[wg()], line); }
  void wait_mem() const { g_m->drain(me()); }
  void nap() const { g_m->pool->nap(); }
  u64 clock() const { return g_m->pool->steps; }
  u32 ld32(const u32* p) const { return g_m->before(me(), p), *p; }
  u64 ld64(const u64* p) const { return g_m->before(me(), p), *p; }
  void st32(u32* p, u32 v) const { g_m->store(me(), p, v, 4); }
  void st64(u64* p, u64 v) const { g_m->store(me(), p, v, 8); }
  u32 xchg32(u32* p, u32 v) const {
    const u32 o = ld32(p);
    *p = v;
    return o;
  }
  u32 add32(u32* p, u32 v) const {
    const u32 o = ld32(p);
    *p = o + v;
    return o;
  }
  u32 or32(u32* p, u32 v) const {
    const u32 o = ld32(p);
    *p = o | v;
    return o;
  }
  u64 min64(u64* p, u64 v) const {
    const u64 o = ld64(p);
    if (v < o) *p = v;
    return o;
  }
  u32 lds_next(LdsWord* p) const { return g_m->pool->give_way(), p->v++; }
  void lds_min(u64* p, u64 v) const {
    g_m->pool->give_way();
    if (v < *p) *p = v;
  }
  // Puts x where the wavefront's other lanes find it, once all have.
  const std::vector<u64>& exchange(u64 x, int line) const {
    const u32 t = me();
    std::vector<u64>& a = g_m->lane_value[g_m->turn[t]++ & 1];
    a[t] = x;
    g_m->pool->wait(g_m->waveb[t / W], line);
    return a;
  }
  u32 wave_max(u32 x, int line = __builtin_LINE()) const {
    const std::vector<u64>& a = exchange(x, line);
    for (u32 l = 0; l < W; ++l) x = a[me() / W * W + l] > x ? (u32)a[me() / W * W + l] : x;
    return x;
  }
  u64 from_lane(u64 x, u32 from, int line = __builtin_LINE()) const { return exchange(x, line)[wg() * NT + from]; }
};

}  // namespace

// A whole run from `src`, as sssp_nearfar sets it up.  Returns fibers::OK,
// MISMATCH or HANG, or the run's error word.
extern "C" int nfm_run(const u64* off, const u32* tg, const u32* wt, u32 n, u32 src, u64 delta, u32 glog, u32 nwg,
                       int policy, int late_stores, u64 seed, u64 max_steps, u64* dist) {
  const u32 nthreads = nwg * FiberGrid::NT;
  std::vector<u32> q(6ull * n), stamp(2ull * n, NONE);
  std::vector<u64> done(n, KINF);
  Ctl* c = new Ctl;
  std::memset(c, 0, sizeof *c);
  Args a{};
  a.off = off, a.tg = tg, a.wt = wt, a.dist = dist, a.n = n, a.delta = delta, a.glog = glog;
  for (u32 i = 0; i < 2; ++i) {
    a.ql[i] = q.data() + i * n;
    a.qh[i] = q.data() + (2 + i) * n;
    a.far[i] = q.data() + (4 + i) * n;
  }
  a.nstamp = stamp.data(), a.fstamp = stamp.data() + n, a.done_at = done.data(), a.cap = n, a.c = c;
  for (u32 v = 0; v < n; ++v) {
    dist[v] = v == src ? 0 : KINF;
    a.heavy |= off[v + 1] - off[v] > FiberGrid::HEAVY;
  }
  a.solo = FiberGrid::NT >> glog;
  a.max_phases = 64 * n + 1024;
  const bool heavy = off[src + 1] - off[src] > FiberGrid::HEAVY;
  (heavy ? a.qh : a.ql)[0][0] = src;
  c->cl[0].w = !heavy, c->ch[0].w = heavy;
  c->fmin[0] = c->fmin[1] = KINF;
  c->ph.mode = RELAX, c->ph.src = 0, c->ph.dst = 1, c->ph.nl = !heavy, c->ph.nh = heavy;
  c->ph.fsrc = 1, c->ph.fdst = 0, c->ph.T = delta;
  fibers::Pool pool(policy, seed, max_steps);
  Machine m;
  m.pool = &pool, m.nwg = nwg, m.nt = FiberGrid::NT, m.late_stores = late_stores != 0;
  m.wgb.resize(nwg);
  for (auto& b : m.wgb) b.size = FiberGrid::NT;
  m.waveb.resize(nthreads / FiberGrid::W);
  for (auto& b : m.waveb) b.size = FiberGrid::W;
  m.turn.assign(nthreads, 0);
  for (auto& v : m.lane_value) v.assign(nthreads, 0);
  struct Lds {
    Phase ph;
    LdsWord flag;
    Gather<FiberGrid> q;
  };
  std::vector<Lds> lds(nwg);
  g_m = &m;
  auto body = [&](u32 i) {
    Lds& s = lds[i / FiberGrid::NT];
    phases(FiberGrid(), a, &s.ph, &s.flag, &s.q);
  };
  int rc = pool.run(nthreads, body);
  if (rc == fibers::OK) rc = (int)c->err.w;
  delete c;
  return rc;
}
