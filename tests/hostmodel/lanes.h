// A team of wavefronts of 64 lanes on the CPU: each lane is a fiber (fibers.h)
// that runs up to the next operation in which lanes take part together.
#pragma once
#include <cstring>
#include <vector>

#include "../../paper_1908_09378_amd/csrc/pbh_core.h"
#include "fibers.h"

namespace bkt {

struct LaneMachine {
  fibers::Pool* pool = nullptr;
  int nt = 0;
  fibers::Barrier team;
  std::vector<fibers::Barrier> wave;
  // What the lanes put down for each other, in turn: slot [turn % 2] holds the
  // values, and what the first reader made of them.  (A slot is written again
  // two turns on, when every lane has read it.)
  struct Slot {
    std::vector<u64> a, b;
    u64 made = 0;  // 1 + the turn that ra, rb and the lists are of
    u64 ra = 0, rb = 0;
  };
  std::vector<Slot> wslot, tslot;
  std::vector<u64> wturn, tturn;

  LaneMachine(fibers::Pool* p, int threads) : pool(p), nt(threads) {
    const size_t nw = (size_t)threads / 64;
    team.size = (u32)threads;
    wave.resize(nw);
    for (auto& w : wave) w.size = 64;
    wslot.resize(2 * nw);
    for (auto& s : wslot) s.a.resize(64), s.b.resize(64);
    tslot.resize(2);
    for (auto& s : tslot) s.a.resize((size_t)threads), s.b.resize((size_t)threads);
    wturn.assign((size_t)threads, 0);
    tturn.assign((size_t)threads, 0);
  }
  // Puts (a, b) down for the lanes of the wavefront / the team and waits for
  // theirs; `make` is called once per exchange.
  template <class F>
  Slot& among_wave(u64 a, u64 b, int line, F make) {
    const u32 t = pool->current;
    const u64 turn = wturn[t]++;
    Slot& s = wslot[2 * (t / 64) + turn % 2];
    s.a[t % 64] = a, s.b[t % 64] = b;
    pool->wait(wave[t / 64], line);
    if (s.made != turn + 1) make(s), s.made = turn + 1;
    return s;
  }
  template <class F>
  Slot& among_team(u64 a, u64 b, int line, F make) {
    const u32 t = pool->current;
    const u64 turn = tturn[t]++;
    Slot& s = tslot[turn % 2];
    s.a[t] = a, s.b[t] = b;
    pool->wait(team, line);
    if (s.made != turn + 1) make(s), s.made = turn + 1;
    return s;
  }
};

#define LINE_ int line = __builtin_LINE()
template <int NT, bool STAGE>
struct LaneTeam {
  static constexpr int kNT = NT, kNW = NT / 64, kW = 64;
  static constexpr int kE = NT == 64 ? 8 : 4, kM = 4, kME = NT == 1024 ? 4 : 8;  // as DevTeam's
  static constexpr bool kStage = STAGE;
  static constexpr int kHeld = STAGE && NT == 256 ? 32 : 16;
  static constexpr int kRU = STAGE || NT >= 256 ? 4 : 1;
  static constexpr u32 prof = 0;
  TeamShared<kNW>* sh;
  LaneMachine* m;
  u64* stk = nullptr;
  u32* stv = nullptr;
  u32* stp = nullptr;

  using Slot = LaneMachine::Slot;
  static void nothing(Slot&) {}
  int tid() const { return (int)m->pool->current; }
  int lane() const { return tid() % 64; }
  int wave() const { return tid() / 64; }
  void sync(LINE_) const { m->pool->wait(m->team, line); }
  void wsync(LINE_) const { m->pool->wait(m->wave[(size_t)wave()], line); }
  u32 uni(u32 x) const { return x; }
  u64 uni64(u64 x) const { return x; }
  u64 lane_val64(u64 x, int l, LINE_) const { return m->among_wave(x, 0, line, nothing).a[(size_t)l]; }
  u32 lane_val(u32 x, int l, LINE_) const { return (u32)lane_val64(x, l, line); }
  u64 lane_get64(u64 x, u32 from, LINE_) const { return lane_val64(x, (int)from, line); }
  float wave_xor(float x, int o, LINE_) const {
    u32 u;
    std::memcpy(&u, &x, 4);
    u = lane_val(u, lane() ^ o, line);
    std::memcpy(&x, &u, 4);
    return x;
  }
  u64 ballot(bool p, LINE_) const {
    return m->among_wave(p, 0, line, [](Slot& s) {
              s.ra = 0;
              for (int l = 0; l < 64; ++l) s.ra |= s.a[(size_t)l] << l;
            }).ra;
  }
  u32 count_below(u64 mask) const { return (u32)__builtin_popcountll(mask & ((1ull << lane()) - 1)); }
  bool any_lane(bool p, LINE_) const { return ballot(p, line) != 0; }
  u32 wave_max32(u32 x, LINE_) const {
    return (u32)m->among_wave(x, 0, line, [](Slot& s) {
                   s.ra = 0;
                   for (u64 y : s.a) s.ra = y > s.ra ? y : s.ra;
                 }).ra;
  }
  u32 wave_or32(u32 x, LINE_) const {
    return (u32)m->among_wave(x, 0, line, [](Slot& s) {
                   s.ra = 0;
                   for (u64 y : s.a) s.ra |= y;
                 }).ra;
  }
  // Prefix sums: the values make way for the sums before them.
  static void sums(Slot& s) {
    u32 run = 0;
    for (size_t i = 0; i < s.a.size(); ++i) s.b[i] = run, run += (u32)s.a[i];
    s.ra = run;
  }
  u32 wave_scan(u32 x, LINE_) const { return (u32)m->among_wave(x, 0, line, sums).b[(size_t)lane()] + x; }
  void wave_sort(u32& a, u32& from, LINE_) const {
    Slot& s = m->among_wave(a, (u64)lane(), line, [](Slot& q) {
      for (size_t i = 1; i < 64; ++i)
        for (size_t j = i; j && q.a[j] < q.a[j - 1]; --j) {
          u64 t = q.a[j];
          q.a[j] = q.a[j - 1], q.a[j - 1] = t;
          t = q.b[j], q.b[j] = q.b[j - 1], q.b[j - 1] = t;
        }
    });
    a = (u32)s.a[(size_t)lane()];
    from = (u32)s.b[(size_t)lane()];
  }
  u32 scan_excl(u32 x, u32* total, LINE_) const {
    Slot& s = m->among_team(x, 0, line, sums);
    *total = (u32)s.ra;
    return (u32)s.b[(size_t)tid()];
  }
  u32 sum(u32 x, LINE_) const {
    u32 t;
    scan_excl(x, &t, line);
    return t;
  }
  bool any(bool p, LINE_) const { return sum(p ? 1u : 0u, line) != 0; }
  void minmax64(u64& lo, u64& hi, LINE_) const {
    Slot& s = m->among_team(lo, hi, line, [](Slot& q) {
      q.ra = ~0ull, q.rb = 0;
      for (u64 x : q.a) q.ra = x < q.ra ? x : q.ra;
      for (u64 x : q.b) q.rb = x > q.rb ? x : q.rb;
    });
    lo = s.ra, hi = s.rb;
  }
  void minkv(u64& k, u32& v, LINE_) const {
    Slot& s = m->among_team(k, v, line, [](Slot& q) {
      q.ra = q.a[0], q.rb = q.b[0];
      for (size_t i = 1; i < q.a.size(); ++i)
        if (q.a[i] < q.ra || (q.a[i] == q.ra && q.b[i] < q.rb)) q.ra = q.a[i], q.rb = q.b[i];
    });
    k = s.ra, v = (u32)s.rb;
  }
  void hist_add(u32* h, u32 b) const { h[b] += 1; }
  u32 hist_next(u32* p) const { return (*p)++; }
  u64 atomic_min(u64* p, u64 v) const {
    const u64 o = *p;
    if (v < o) *p = v;
    return o;
  }
  u32 atomic_or32(u32* p, u32 v) const {
    const u32 o = *p;
    *p = o | v;
    return o;
  }
  u32 atomic_add32(u32* p, u32 v) const {
    const u32 o = *p;
    *p = o + v;
    return o;
  }
  u64 atomic_exch(u64* p, u64 v) const {
    const u64 o = *p;
    *p = v;
    return o;
  }
  u64 load_cur(const u64* p) const { return *p; }
  u32 load32(const u32* p) const { return *p; }
  void store_cur(u64* p, u64 v) const { *p = v; }
  void fence() const {}
};
#undef LINE_

// How the lanes are scheduled between the operations that they take part in
// together: in turn (seed 0), or at random, so that what one lane writes and
// another reads without such an operation between them comes out differently.
static u64 g_lane_seed = 0;

// body(t) by every lane of a team (its shared memory and staging area as t's):
// 0, or fibers::MISMATCH or HANG.
template <int NT, bool STAGE, class F>
int run_team(const LaneTeam<NT, STAGE>& t, F&& body) {
  fibers::Pool pool(g_lane_seed ? fibers::PRIORITY : fibers::ROUND_ROBIN, g_lane_seed, ~0ull);
  LaneMachine m(&pool, NT);
  auto one = [&](u32) {
    LaneTeam<NT, STAGE> mine = t;
    mine.m = &m;
    body(mine);
  };
  return pool.run(NT, one);
}

}  // namespace bkt
