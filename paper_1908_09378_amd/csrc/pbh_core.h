// Parallel bucket heap (Section 2.2) and parDijkstra rounds (Section 4.1),
// written once against a "team" (pbh_team.h): every thread of the team runs the
// same control flow on team-uniform values; the data-parallel steps (Merge,
// DeleteDuplicates, Select, PrefixSums, the relaxation) are split across the
// team's threads.
//
// Elements are (key u64, id u32) in structure-of-arrays form, ordered by
// (key, id).  Level i has a bucket B_i and a signal buffer S_i, each kept
// sorted by id (Section 2.1), nominal sizes |B_i| = 2d*4^i and |S_i| = d*4^i
// (Section 2.2), and a pivot p_i with B_i <= p_i < every element deeper.
#pragma once
#include "pbh_team.h"

#define PBH_HD __host__ __device__
#define PBH_INL __host__ __device__ __forceinline__
#define PBH_NOINL __host__ __device__ __attribute__((noinline))

namespace bkt {

constexpr u64 KINF = ~0ull;
constexpr u32 VINF = ~0u;
constexpr int MAXL = 16;

enum { E_OK = 0, E_INVAL = -1, E_CAPACITY = -2, E_INTERNAL = -6 };

struct KV {
  u64 k;
  u32 v;
};
PBH_HD inline bool kv_less(KV a, KV b) { return a.k < b.k || (a.k == b.k && a.v < b.v); }
PBH_HD inline bool kv_le(KV a, KV b) { return !kv_less(b, a); }
PBH_HD inline KV kv_inf() { return KV{KINF, VINF}; }

// A view of an element array: keys and ids.  The pointer types carry the
// address space on the GPU (LDS levels -> ds_* instructions, HBM levels ->
// global_* instructions); the geometry hands out generic views (Arr) that are
// cast to the typed view of the level's placement.
template <class KP, class VP>
struct ArrT {
  KP k;
  VP v;
};
using Arr = ArrT<u64*, u32*>;
template <class A>
PBH_INL A as_arr(Arr a) {
  A r;
  r.k = (decltype(r.k))a.k;
  r.v = (decltype(r.v))a.v;
  return r;
}

// ---------------------------------------------------------------- geometry
// Nominal sizes from Section 2.2, and the allocated buffer sizes.  A level
// stores two B buffers (merge ping-pong, 4d*4^i each), one temporary T (4d*4^i)
// and two S buffers (2d*4^i each): 16d*4^i elements.  The allocated sizes
// leave room for what Algorithm 1 can hold between two Resolve(i): B_i may
// absorb elements of S_i that fall below p_i, and each Resolve(i-1) adds at
// most |S_{i-1}| + |B_{i-1}| to S_i.
PBH_HD inline u64 nomS(u32 d, int i) { return (u64)d << (2 * i); }
PBH_HD inline u64 nomB(u32 d, int i) { return (u64)d << (2 * i + 1); }
PBH_HD inline u64 capS(u32 d, int i) { return (u64)d << (2 * i + 1); }
PBH_HD inline u64 capB(u32 d, int i) { return (u64)d << (2 * i + 2); }
PBH_HD inline u64 lvl_size(u32 d, int i) { return (16ull * d) << (2 * i); }
// (4^i - 1) / 3 = 1 + 4 + ... + 4^(i-1)
PBH_HD inline u64 lvl_off(u32 d, int i) { return 16ull * d * (0x5555555555555555ull & ((1ull << (2 * i)) - 1ull)); }

struct Geom {
  u32 d;
  int q;     // levels allocated
  int qlds;  // levels 0..qlds-1 live in LDS
  u64* gk;   // global arena (level qlds at offset 0)
  u32* gv;
  u64* lk;   // LDS arena
  u32* lv;
};

// Buffer w of level i: 0/1 = B ping-pong, 2 = T, 3/4 = S ping-pong.
PBH_HD inline Arr lbuf(const Geom& g, int i, int w) {
  u64 cb = capB(g.d, i);
  u64 off = (w < 3) ? (u64)w * cb : 3ull * cb + (u64)(w - 3) * capS(g.d, i);
  if (i < g.qlds) {
    u64 b = lvl_off(g.d, i) + off;
    return Arr{g.lk + b, g.lv + b};
  }
  u64 b = lvl_off(g.d, i) - lvl_off(g.d, g.qlds) + off;
  return Arr{g.gk + b, g.gv + b};
}

struct Lvl {
  u32 nB, nS;    // sizes of B_i and S_i
  u32 bsel;      // which B buffer (0/1) holds B_i
  u32 ssel;      // which S buffer (0/1) holds S_i
  u64 pk;        // pivot p_i = (pk, pv); KINF = +infinity
  u32 pv;
  u32 cnt;       // Resolve(i) executions
};

// Time accounting of a profiled SSSP run (ticks of the device's constant
// real-time clock): prof[i] for i < MAXL is the time inside Resolve(i); the
// other slots split each round into its steps.
enum {
  PROF_DRIVE = MAXL,  // Resolve(0), the schedule and refills after each operation
  PROF_PIECE,         // moving the next piece of a round's update list into S_0
  PROF_PROPOSE,       // features and the MLP (learned rule)
  PROF_EXTRACT,       // choosing and removing the round's minima from B_0
  PROF_RELAX,         // scanning their out-edges (atomicMin on dist)
  PROF_INTAKE,        // the round's updates: filter, sort by id, deduplicate
  PROF_OTHER,
  PROF_WAIT,          // waiting for a deep-level worker (inside PROF_DRIVE)
  PROF_N
};

struct HeapState {
  Lvl L[MAXL];
  int ell;       // deepest non-empty level, -1 if the heap is empty
  int err;
  u32 d;
  int q;
  u64 elems;     // heap elements read + written by level operations
  u64 live;      // elements in the heap (queue size)
  u64 progress;  // resumable progress of a multi-piece operation
  u64 aux[5];
  // Levels resolved by their own workers (the deep-level service of the SSSP
  // kernel): this team's copies of their states are not kept up to date, so
  // the deepest level known to hold elements (-1: none) and the number of
  // elements in the worker levels stand in for them.
  int deep_floor;
  u64 deep_n;
  u64 prof_last;  // clock at the last lap mark
  u64 prof_res;   // clock at the start of the running Resolve
  u64 prof[PROF_N];
};

// The device's constant-rate real-time clock (0 on the host).
PBH_INL u64 pbh_clock() {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_s_memrealtime();
#else
  return 0;
#endif
}

// Lap mark of a profiled run: the time since the previous mark goes to `cat`.
// One thread keeps the books; marks sit after the team's barriers, so the
// time of a step includes its slowest wavefront.
template <class T, class SP>
PBH_INL void prof_lap(const T& t, SP st, int cat) {
  if (t.prof && t.tid() == 0) {
    const u64 now = pbh_clock();
    st->prof[cat] += now - st->prof_last;
    st->prof_last = now;
  }
}

template <class SP>
PBH_HD inline void state_init(SP st, u32 d, int q) {
  for (int i = 0; i < MAXL; ++i) {
    st->L[i].nB = st->L[i].nS = st->L[i].bsel = st->L[i].ssel = st->L[i].cnt = 0;
    st->L[i].pk = KINF;
    st->L[i].pv = VINF;
  }
  st->ell = -1;
  st->err = 0;
  st->d = d;
  st->q = q;
  st->elems = st->live = st->progress = 0;
  for (int i = 0; i < 5; ++i) st->aux[i] = 0;
  st->deep_floor = -1;
  st->deep_n = 0;
  st->prof_last = st->prof_res = 0;
  for (int i = 0; i < PROF_N; ++i) st->prof[i] = 0;
}

// Field-wise copies of a level's state (the state may live in LDS, whose
// objects have no implicit copy into generic memory).
template <class SP>
PBH_INL Lvl lvl_load(SP st, int i) {
  Lvl a;
  a.nB = st->L[i].nB;
  a.nS = st->L[i].nS;
  a.bsel = st->L[i].bsel;
  a.ssel = st->L[i].ssel;
  a.pk = st->L[i].pk;
  a.pv = st->L[i].pv;
  a.cnt = st->L[i].cnt;
  return a;
}
// The same for a team: the values are the same in every thread, and saying so
// keeps them in scalar registers, with scalar branches on them.
template <class T, class SP>
PBH_INL Lvl lvl_uni(const T& t, SP st, int i) {
  Lvl a = lvl_load(st, i);
  a.nB = t.uni(a.nB);
  a.nS = t.uni(a.nS);
  a.bsel = t.uni(a.bsel);
  a.ssel = t.uni(a.ssel);
  a.pk = t.uni64(a.pk);
  a.pv = t.uni(a.pv);
  a.cnt = t.uni(a.cnt);
  return a;
}
template <class SP>
PBH_INL void lvl_store(SP st, int i, const Lvl& a) {
  st->L[i].nB = a.nB;
  st->L[i].nS = a.nS;
  st->L[i].bsel = a.bsel;
  st->L[i].ssel = a.ssel;
  st->L[i].pk = a.pk;
  st->L[i].pv = a.pv;
  st->L[i].cnt = a.cnt;
}

// Host-side policy: every array and the state live in ordinary memory.  The
// GPU policy (kernels.hip) types LDS levels, HBM levels and the state with
// their address spaces.
struct HostPolicy {
  using L = Arr;
  using G = Arr;
  using SP = HeapState*;
  // called before (after = false) and after every Resolve(i); the CPU tests'
  // policy records the level sizes there, the others do nothing
  template <class SPP>
  PBH_INL static void on_resolve(const Geom&, SPP, int, bool) {}
};

// ---------------------------------------------------------------- primitives

// Where an array lives.
template <class A>
struct in_lds {
  static constexpr bool v = false;
};
template <>
struct in_lds<ArrT<u64 PBH_LDS*, u32 PBH_LDS*>> {
  static constexpr bool v = true;
};

template <class A, class B>
struct same_arr {
  static constexpr bool v = false;
};
template <class A>
struct same_arr<A, A> {
  static constexpr bool v = true;
};

// Merge-path split (Green, McColl, Bader 2012): how many of the first `diag`
// elements of merge(A, B) by id come from A (A first on equal ids).  QUAD: each
// step tests three split points, whose six reads are in flight together; the
// search is a chain of dependent reads, so half as many steps is half its time
// for one wavefront on LDS (about 60 ns a step, seven steps -> four on 128
// elements).  Where many lanes' scattered reads load the LDS or the L1, the
// plain search's fewer reads are faster.
template <bool QUAD, class VA, class VB>
PBH_INL u32 merge_path(VA av, u32 na, VB bv, u32 nb, u32 diag) {
  u32 lo = diag > nb ? diag - nb : 0u, hi = diag < na ? diag : na;
  if constexpr (QUAD) {
    while (lo < hi) {
      const u32 len = hi - lo;
      const u32 m1 = lo + (len >> 2), m2 = lo + (len >> 1), m3 = lo + ((3u * (len >> 1)) >> 1);
      const bool t1 = av[m1] <= bv[diag - 1 - m1], t2 = av[m2] <= bv[diag - 1 - m2],
                 t3 = av[m3] <= bv[diag - 1 - m3];
      // true on a prefix: t3 implies t2 implies t1
      lo = t3 ? m3 + 1 : (t2 ? m2 + 1 : (t1 ? m1 + 1 : lo));
      hi = t3 ? hi : (t2 ? m3 : (t1 ? m2 : m1));
    }
  } else {
    while (lo < hi) {
      const u32 mid = (lo + hi) >> 1;
      if (av[mid] <= bv[diag - 1 - mid])
        lo = mid + 1;
      else
        hi = mid;
    }
  }
  return lo;
}

// The same split by one wavefront: every step tests as many split points as it
// has lanes (the tests are true on a prefix, so their number narrows the range),
// two or three dependent reads of HBM instead of a dozen.
template <class T, class VA, class VB>
PBH_INL u32 merge_path_lanes(const T& t, VA av, u32 na, VB bv, u32 nb, u32 diag) {
  u32 lo = diag > nb ? diag - nb : 0u, hi = diag < na ? diag : na;
  while (lo < hi) {
    const u32 stride = (hi - lo + (u32)T::kW - 1) / (u32)T::kW, mid = lo + ((u32)t.lane() + 1u) * stride - 1u;
    bool afirst = false;
    if (mid < hi) afirst = av[mid] <= bv[diag - 1 - mid];
    lo += (u32)__builtin_popcountll(t.ballot(afirst)) * stride;
    hi = lo + stride - 1 < hi ? lo + stride - 1 : hi;
  }
  return lo < hi ? lo : hi;
}

// Merge + DeleteDuplicates (Algorithm 1; DeleteDuplicates by scan + prefix
// sums as in Lemma 2's proof).  A and B are sorted by id with unique ids; the
// output C (not aliasing A or B) is sorted by id with unique ids.  For a pair
// of copies of one id the one whose key equals cur[id] (the live one) is kept;
// if neither is live both are dropped; without cur the smaller key is kept
// (Section 2.1: duplicates keep the smaller priority).  With filterB, B
// elements that are not live are dropped as well.  (The heap's merges pass
// false, which folds it away: what moves up into B_0 is checked in the split
// before.  Without the parameter the compiler orders the speculative rounds'
// code differently and the learned ring lattice of 100,003 vertices takes 94 ms
// instead of 92; six spellings of it were measured.)
enum { PREFER_LIVE = 0, PREFER_A = 1, PREFER_B = 2 };

// The next E elements of A and of B from a thread's split, held in registers:
// all their reads are in flight together, and the walk over the outputs shifts
// the two windows instead of reading element by element (a chain of reads).
// walk() merges E outputs (`valid` of them), decides duplicates and liveness
// and returns the mask of kept outputs.  Which copy of a pair lives is looked
// up after the walk, for all of the thread's pairs at once.
template <int E>
struct MergeWin {
  // vectors, not arrays: a choice between two elements of an array becomes a
  // load from a chosen address, which puts the array into scratch memory
  typedef u64 VK __attribute__((ext_vector_type(E)));
  typedef u32 VV __attribute__((ext_vector_type(E)));
  VK ak, bk, ko;
  VV av, bv, vo;
  u32 prev;  // A's element before the window (VINF: none; ids are below VINF)

  // A[i, ...) of na elements, B[j, ...) of nb
  template <class AA, class AB>
  PBH_INL void load(AA A, u32 i, u32 na, AB B, u32 j, u32 nb) {
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const bool ia = i + s < na, ib = j + s < nb;
      av[s] = ia ? A.v[i + s] : VINF;
      bv[s] = ib ? B.v[j + s] : VINF;
      ak[s] = ia ? A.k[i + s] : 0ull;
      bk[s] = ib ? B.k[j + s] : 0ull;
    }
    prev = i > 0 ? A.v[i - 1] : VINF;
  }

  template <class T>
  PBH_INL u32 walk(const T& t, u32 valid, const u64* cur, bool filterB, int prefer) {
    u64 alt[E];  // the other copy's key where the current key decides
    u32 keep = 0, ask = 0, askb = 0;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const bool in = (u32)s < valid, takeA = av[0] <= bv[0], dup = av[0] == bv[0];
      const u64 ka = ak[0], kb = bk[0];
      u64 k = takeA ? ka : kb;
      bool kp = in;
      alt[s] = kb;
      if (takeA) {
        if (dup && ka != kb) {
          if (prefer == PREFER_B)
            k = kb;
          else if (prefer == PREFER_LIVE) {
            if (cur)
              ask |= (u32)in << s;
            else
              k = kb < ka ? kb : ka;
          }
        }
      } else {
        kp = in && prev != bv[0];
        if (filterB) askb |= (u32)kp << s;
      }
      ko[s] = k;
      vo[s] = takeA ? av[0] : bv[0];
      keep |= (u32)kp << s;
      prev = takeA ? av[0] : prev;
#pragma unroll
      for (int x = 0; x + 1 < E; ++x) {
        if (x + 1 >= E - s) continue;  // what no later output reads
        av[x] = takeA ? av[x + 1] : av[x];
        ak[x] = takeA ? ak[x + 1] : ak[x];
        bv[x] = takeA ? bv[x] : bv[x + 1];
        bk[x] = takeA ? bk[x] : bk[x + 1];
      }
    }
    if (ask | askb) {
      u64 c[E];
#pragma unroll
      for (int s = 0; s < E; ++s) c[s] = ((ask | askb) >> s) & 1u ? t.load_cur(cur + vo[s]) : 0ull;
#pragma unroll
      for (int s = 0; s < E; ++s) {
        const bool q = ((ask | askb) >> s) & 1u;
        const bool other = q && ko[s] != c[s];
        const bool second = other && ((ask >> s) & 1u) && alt[s] == c[s];
        ko[s] = second ? alt[s] : ko[s];
        if (other && !second) keep &= ~(1u << s);
      }
    }
    return keep;
  }
};

// What a merge counts of its outputs on the way: how many are <= p.
struct CountLe {
  KV p;
  u32 n;
};

// E outputs of a merge from A's window [i, ea) and B's [j, eb) of one area in
// LDS (A's begins at 0), with no branch but the one for pairs: a lone wavefront
// pays 16 cycles and more for each.  A step reads one id; the keys follow at
// the end, all at once.  The decisions are MergeWin's.
template <int E>
struct MergeArea {
  typedef u64 VK __attribute__((ext_vector_type(E)));
  typedef u32 VV __attribute__((ext_vector_type(E)));
  VK ko;
  VV vo;

  template <class T, class AS>
  PBH_INL u32 walk(const T& t, AS S, u32 i, u32 ea, u32 j, u32 eb, u32 valid, const u64* cur, bool filterB,
                   int prefer) {
    constexpr u32 LAST = (u32)T::kNT * E - 1;
    // (a device's area is followed by more of the team's LDS)
    auto in_area = [](u32 x) { return T::kW == 1 && x > LAST ? LAST : x; };
    VV src, oth;
    u32 keep = 0, pair = 0, askb = 0;
    const u32 pv = S.v[i > 0 ? i - 1 : 0], v0 = S.v[in_area(i)], v1 = S.v[in_area(j)];
    u32 prev = i > 0 ? pv : VINF, va = i < ea ? v0 : VINF, vb = j < eb ? v1 : VINF;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const bool in = (u32)s < valid, takeA = va <= vb, kp = in & (takeA | (prev != vb));
      src[s] = in_area(takeA ? i : j);
      oth[s] = in_area(j);
      vo[s] = takeA ? va : vb;
      keep |= (u32)kp << s;
      pair |= (u32)(in & (va == vb)) << s;
      askb |= (u32)(kp & !takeA) << s;
      prev = takeA ? va : prev;
      i += takeA ? 1u : 0u;
      j += takeA ? 0u : 1u;
      if (s + 1 == E) continue;
      const u32 x = takeA ? i : j, n = S.v[in_area(x)], nv = x < (takeA ? ea : eb) ? n : VINF;
      va = takeA ? nv : va;
      vb = takeA ? vb : nv;
    }
#pragma unroll
    for (int s = 0; s < E; ++s) ko[s] = S.k[src[s]];
    if (!filterB) askb = 0;
    if (prefer == PREFER_A) pair = 0;
    if (pair | askb) {
      VK alt, c;
#pragma unroll
      for (int s = 0; s < E; ++s) {
        alt[s] = S.k[oth[s]];
        if (alt[s] == ko[s]) pair &= ~(1u << s);
      }
      const bool by_cur = prefer == PREFER_LIVE && cur;
      if (!by_cur) {
#pragma unroll
        for (int s = 0; s < E; ++s) {
          const bool other = ((pair >> s) & 1u) & ((prefer == PREFER_B) | (alt[s] < ko[s]));
          ko[s] = other ? alt[s] : ko[s];
        }
        pair = 0;
      }
      if (pair | askb) {
#pragma unroll
        for (int s = 0; s < E; ++s) c[s] = t.load_cur(cur + (((pair | askb) >> s) & 1u ? vo[s] : 0u));
#pragma unroll
        for (int s = 0; s < E; ++s) {
          const bool other = (((pair | askb) >> s) & 1u) & (ko[s] != c[s]);
          const bool second = other & ((pair >> s) & 1u) & (alt[s] == c[s]);
          ko[s] = second ? alt[s] : ko[s];
          keep &= ~((u32)(other & !second) << s);
        }
      }
    }
    return keep;
  }
};

// A thread's kept outputs, and above them those of them that are <= le->p (a
// tile has at most 2^15 outputs).
template <int E, class W>
PBH_INL u32 merge_count(const W& w, u32 keep, const CountLe* le) {
  u32 x = (u32)__builtin_popcount(keep);
  if (le) {
    u32 c = 0;
#pragma unroll
    for (int s = 0; s < E; ++s) c += ((keep >> s) & 1u) & (u32)kv_le(KV{w.ko[s], w.vo[s]}, le->p);
    x |= c << 16;
  }
  return x;
}

// Places a thread's kept outputs (a prefix sum over the team) and counts those
// <= le->p; returns the tile's output count.
template <class T, int E, class AC>
PBH_INL u32 merge_store(const T& t, const MergeWin<E>& w, u32 keep, AC C, u32 out, CountLe* le) {
  u32 tot;
  u32 o = out + (t.scan_excl(merge_count<E>(w, keep, le), &tot) & 0xFFFFu);
#pragma unroll
  for (int s = 0; s < E; ++s)
    if ((keep >> s) & 1u) {
      C.k[o] = w.ko[s];
      C.v[o] = w.vo[s];
      ++o;
    }
  if (le) le->n += tot >> 16;
  return tot & 0xFFFFu;
}

template <class T, int E, class AA, class AB, class AC>
PBH_INL u32 merge_dedup_e(const T& t, AA A, u32 na, AB B, u32 nb, AC C, const u64* cur, bool filterB, int prefer,
                          CountLe* le) {
  const u32 total = na + nb;
  u32 out = 0;
  for (u32 base = 0; base < total; base += (u32)T::kNT * E) {
    u32 d0 = base + (u32)t.tid() * E;
    d0 = d0 < total ? d0 : total;
    const u32 i = merge_path<T::kNT == 64 && in_lds<AA>::v && in_lds<AB>::v>(A.v, na, B.v, nb, d0);
    MergeWin<E> w;
    w.load(A, i, na, B, d0 - i, nb);
    const u32 keep = w.walk(t, total - d0, cur, filterB, prefer);
    out += merge_store<T, E>(t, w, keep, C, out, le);
  }
  t.sync();
  return out;
}

// Bytes of the staging area of a team of NT threads walking E outputs each.
PBH_HD inline u64 stage_bytes(int nt, int e) {
  const u64 w = (u64)nt * (u64)e + 2u;
  return ((2u * w * 12u + ((u64)nt + 1u) * 4u) + 7u) & ~7ull;
}
// Carves the staging area out of `base` (8-byte aligned); !on: the team has
// none, also if an earlier query of its had one (this query's levels may lie
// there now).
template <class T, class BP>
PBH_INL void stage_setup(T& t, BP base, bool on) {
  const u64 w = (u64)T::kNT * T::kE + 2u;
  if (!on) {
    t.stk = nullptr;
    t.stv = nullptr;
    t.stp = nullptr;
    return;
  }
  t.stk = (decltype(t.stk))base;
  t.stv = (decltype(t.stv))(base + 2u * w * 8u);
  t.stp = (decltype(t.stp))(base + 2u * w * 12u);
}

// Merge + DeleteDuplicates of arrays in HBM through the team's LDS staging
// area, with the same result as merge_dedup_e.  The merge-path split of every
// tile boundary is found first (a batch of boundaries at a time: one per
// wavefront while they are few, one per thread otherwise); then each tile's
// inputs are loaded into LDS with coalesced reads, A's and B's one after the
// other, with A's element before them and the next one of each, which the
// duplicate checks look at; and the per-thread merge-path searches and walks
// run on LDS while the next tile's inputs are on their way.
// Bound by the chain of each tile's steps (one wavefront per SIMD, nothing to
// switch to), full or not.  256 threads take 8 outputs each rather than 4, so
// that a tile's search and barriers serve twice as many (4,000 elements 25,600
// -> 19,900 cycles), and a remainder of up to half a tile one of half the size;
// a tile's windows share one area, of the size two apart would have for half
// the tile.
//
// The outputs at merge positions [from, total) go to C from `out` on; the new
// end of C is returned.
template <int E, class T, class AA, class AB, class AC>
PBH_INL u32 merge_tiles(const T& t, AA A, u32 na, AB B, u32 nb, AC C, u32 from, u32 total, u32 out, const u64* cur,
                        bool filterB, int prefer, CountLe* le) {
  // (with the three neighbours the inputs are at most E elements per thread)
  constexpr u32 TILE = (u32)T::kNT * E - 4u;
  const auto sk = t.stk;
  const auto sv = t.stv;
  const auto sp = t.stp;
  u64 xk[E];
  u32 xv[E];
  for (u32 cbase = from; cbase < total; cbase += TILE * (u32)T::kNT) {
    u32 ntile = (total - cbase + TILE - 1) / TILE;
    ntile = ntile < (u32)T::kNT ? ntile : (u32)T::kNT;
    if (T::kW > 1 && ntile <= 4u * T::kNW) {
      for (u32 j = t.uni((u32)t.wave()); j <= ntile; j += T::kNW) {
        const u32 dg = total - cbase < j * TILE ? total : cbase + j * TILE;
        const u32 i = merge_path_lanes(t, A.v, na, B.v, nb, dg);
        if (t.lane() == 0) sp[j] = i;
      }
    } else {
      for (u32 j = (u32)t.tid(); j <= ntile; j += (u32)T::kNT) {
        const u64 dg = (u64)cbase + (u64)j * TILE;
        sp[j] = merge_path<false>(A.v, na, B.v, nb, dg < total ? (u32)dg : total);
      }
    }
    t.sync();
    // tile k: its inputs A[a0, a1) and B[b0, b1), and the window A[abase, abase
    // + la) and B[b0, b0 + lb)
    u32 d0, d1, a0, a1, b0, b1, abase, la, lb;
    auto tile = [&](u32 k) {
      d0 = cbase + k * TILE;
      d1 = total - d0 < TILE ? total : d0 + TILE;
      a0 = t.uni(sp[k]);
      a1 = t.uni(sp[k + 1]);
      b0 = d0 - a0;
      b1 = d1 - a1;
      abase = a0 > 0 ? a0 - 1 : 0;
      la = (a1 < na ? a1 + 1 : a1) - abase;
      lb = (b1 < nb ? b1 + 1 : b1) - b0;
      // (past the end, the last element again: no branches)
#pragma unroll
      for (int r = 0; r < E; ++r) {
        u32 x = (u32)t.tid() + (u32)r * (u32)T::kNT;
        x = x < la + lb ? x : la + lb - 1;
        const bool fa = x < la;
        const u32 y = fa ? abase + x : b0 + (x - la);
        xk[r] = (fa ? A.k : B.k)[y];
        xv[r] = (fa ? A.v : B.v)[y];
      }
    };
    tile(0);
    for (u32 k = 0; k < ntile; ++k) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const u32 x = (u32)t.tid() + (u32)r * (u32)T::kNT;
        sk[x] = xk[r];
        sv[x] = xv[r];
      }
      t.sync();
      const u32 n = d1 - d0, wa = a1 - a0, wb = b1 - b0, skip = a0 - abase, ea = la, eb = lb;
      if (k + 1 < ntile) tile(k + 1);
      // this thread's outputs of the tile, from e0
      u32 e0 = (u32)t.tid() * E;
      e0 = e0 < n ? e0 : n;
      const u32 i = merge_path<T::kNT == 64>(sv + skip, wa, sv + ea, wb, e0), j = e0 - i;
      MergeArea<E> w;
      const u32 keep = w.walk(t, ArrT<decltype(t.stk), decltype(t.stv)>{sk, sv}, skip + i, ea, ea + j, ea + eb, n - e0,
                              cur, filterB, prefer);
      // The outputs go to their places in the staging area (the scan's barrier
      // ends the walks) and from there out in rows: a thread's outputs are
      // consecutive, so stored from the registers each store would touch 64
      // lines.  Eight consecutive places are permuted by the eight they lie
      // in, or the threads' places would meet in a few banks.
      u32 tot, x = merge_count<E>(w, keep, le);
      u32 o = t.scan_excl(x, &tot) & 0xFFFFu;
      if (le) le->n += tot >> 16;
      tot &= 0xFFFFu;
      auto place = [](u32 o) { return o ^ ((o >> 3) & 7u); };
#pragma unroll
      for (int s = 0; s < E; ++s) {  // (a dropped one goes past the outputs)
        const u32 y = (keep >> s) & 1u ? place(o) : (u32)T::kNT * E;
        sk[y] = w.ko[s];
        sv[y] = w.vo[s];
        o += (keep >> s) & 1u;
      }
      t.sync();
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const u32 y = (u32)t.tid() + (u32)r * (u32)T::kNT;
        if ((u32)r * (u32)T::kNT < tot && y < tot) {
          C.k[out + y] = sk[place(y)];
          C.v[out + y] = sv[place(y)];
        }
      }
      out += tot;
      t.sync();  // the next tile overwrites the windows
    }
  }
  return out;
}
template <class T, class AA, class AB, class AC>
PBH_INL u32 merge_dedup_staged(const T& t, AA A, u32 na, AB B, u32 nb, AC C, const u64* cur, bool filterB,
                               int prefer, CountLe* le) {
  constexpr int E = T::kME, H = T::kNT == 1 ? E : E / 2;
  constexpr u32 TILE = (u32)T::kNT * E - 4u, HALF = (u32)T::kNT * H - 4u;
  const u32 total = na + nb, rest = total % TILE, cut = rest <= HALF ? total - rest : total;
  u32 out = 0;
  if (cut) out = merge_tiles<E>(t, A, na, B, nb, C, 0u, cut, out, cur, filterB, prefer, le);
  if (cut < total) out = merge_tiles<H>(t, A, na, B, nb, C, cut, total, out, cur, filterB, prefer, le);
  t.sync();
  return out;
}

// Merge + DeleteDuplicates of a short array P with an array Q of at most R * kW
// elements, by one wavefront in registers: P sits in the lanes (one element
// each), Q in rows of kW elements.  Each element of P in turn is compared with
// all rows: ballots count Q's ids below it (its place), the lanes count P's
// ids below theirs.  No search, no walk, and few instructions: one wavefront
// spends 5 to 8 cycles on each instruction, so their number is its time.  A
// pair of copies is decided at P's lane.  R = 1 covers arrays of up to one
// element per lane without loops over rows.
constexpr u32 SHORT = 16;
template <class T>
PBH_INL u32 small_rows(u32 na, u32 nb) {  // rows of the longer array, 0: too large for this form
  const u32 p = na < nb ? na : nb, q = na < nb ? nb : na;
  const u32 rows = (q + (u32)T::kW - 1) / (u32)T::kW;
  return p <= SHORT && p <= (u32)T::kW && rows <= 4u && p * rows <= 24u ? (rows ? rows : 1u) : 0u;
}

template <int R>
struct SmallMerge {
  u64 pk, qk[R];
  u32 pv, qv[R];
  u32 place;         // Q's ids below this lane's id of P
  u32 below[R];      // P's ids below each of this lane's ids of Q
  bool pin, qin[R];  // outputs: P's elements but dead pairs, Q's but copies
  u32 dups, deads;   // P's elements with a copy in Q / with no live copy
  u32 m;             // outputs

  template <class T, class AP, class AQ>
  PBH_INL void run(const T& t, AP P, u32 np, AQ Q, u32 nq, bool p_is_a, const u64* cur, int prefer) {
    constexpr u32 W = (u32)T::kW;
    const u32 lane = (u32)t.lane();
    // reads past the end are clamped to the last element, not branched around
    pin = lane < np;
    pk = 0;
    pv = VINF;
    if (np) {
      const u32 pi = pin ? lane : np - 1;
      pk = P.k[pi];
      const u32 v = P.v[pi];
      pv = pin ? v : VINF;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      qk[r] = 0;
      qv[r] = VINF;
      qin[r] = false;
      below[r] = 0;
      if ((u32)r * W >= nq) continue;
      const u32 x = (u32)r * W + lane, xi = x < nq ? x : nq - 1;
      qk[r] = Q.k[xi];
      const u32 v = Q.v[xi];
      qin[r] = x < nq;
      qv[r] = qin[r] ? v : VINF;
    }
    place = 0;
    dups = 0;
    u64 other = 0;  // the copy's key in Q
    for (u32 j = 0; j < np; ++j) {
      const u32 s = t.lane_val(pv, (int)j);
      u32 c = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r > 0 && (u32)r * W >= nq) continue;
        c += (u32)__builtin_popcountll(t.ballot(qv[r] < s));
        below[r] += qv[r] > s ? 1u : 0u;
        const u64 e = t.ballot(qv[r] == s);
        if (e) {
          dups |= 1u << j;
          qin[r] = qin[r] && qv[r] != s;
          const u64 ko = t.lane_val64(qk[r], __builtin_ctzll(e));
          other = lane == j ? ko : other;
        }
      }
      place = lane == j ? c : place;
    }
    deads = 0;
    if (dups && prefer != (p_is_a ? (int)PREFER_A : (int)PREFER_B)) {
      const bool dup = pin && ((dups >> (lane & 31u)) & 1u);
      if (prefer != PREFER_LIVE) {
        pk = dup ? other : pk;
      } else if (cur) {
        u64 c = pk;
        const bool ask = dup && pk != other;
        if (ask) c = t.load_cur(cur + pv);
        const bool second = ask && other == c, dead = ask && pk != c && other != c;
        pk = second ? other : pk;
        pin = pin && !dead;
        deads = (u32)t.ballot(dead);
      } else {
        pk = dup && other < pk ? other : pk;
      }
    }
    m = np + nq - (u32)__builtin_popcount(dups) - (u32)__builtin_popcount(deads);
  }

  // Outputs <= p.
  template <class T>
  PBH_INL u32 count_le(const T& t, KV p) const {
    u32 c = (u32)__builtin_popcountll(t.ballot(pin && kv_le(KV{pk, pv}, p)));
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r == 0 || t.any_lane(qin[r])) c += (u32)__builtin_popcountll(t.ballot(qin[r] && kv_le(KV{qk[r], qv[r]}, p)));
    return c;
  }

  template <class T, class AC>
  PBH_INL void store(const T& t, u32 nq, AC C) const {
    constexpr u32 W = (u32)T::kW;
    const u32 gone = dups | deads;
    u32 o = (u32)t.lane() + place;
    if (gone) o -= t.count_below(dups) + t.count_below(deads);
    if (pin) {
      C.k[o] = pk;
      C.v[o] = pv;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r > 0 && (u32)r * W >= nq) continue;
      u32 x = (u32)r * W + (u32)t.lane() + below[r];
      if (gone) {
        const u32 lo = (1u << below[r]) - 1u;  // below <= SHORT
        x -= (u32)__builtin_popcount(dups & lo) + (u32)__builtin_popcount(deads & lo);
      }
      if (qin[r]) {
        C.k[x] = qk[r];
        C.v[x] = qv[r];
      }
    }
  }

  // The r-th smallest output, by taking out the smallest (or, if the rank is
  // closer to the other end, the largest) one by one.
  template <class T>
  PBH_INL KV select(const T& t, u32 r) const {
    const bool top = m - r + 1 < r;
    const u64 fk = top ? KINF : 0ull;
    const u32 fv = top ? VINF : 0u;
    u64 bk = 0;
    u32 bv = 0;
    bool pl = pin, ql[R];
#pragma unroll
    for (int q = 0; q < R; ++q) ql[q] = qin[q];
    for (u32 it = top ? m - r + 1 : r;; --it) {
      bk = pl ? pk ^ fk : KINF;
      bv = pl ? pv ^ fv : VINF;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const u64 k = ql[q] ? qk[q] ^ fk : KINF;
        const u32 v = ql[q] ? qv[q] ^ fv : VINF;
        const bool lt = kv_less(KV{k, v}, KV{bk, bv});
        bk = lt ? k : bk;
        bv = lt ? v : bv;
      }
      t.minkv(bk, bv);
      bk ^= fk;
      bv ^= fv;
      if (it == 1) return KV{bk, bv};
      pl = pl && pv != bv;  // (ids are distinct)
#pragma unroll
      for (int q = 0; q < R; ++q) ql[q] = ql[q] && qv[q] != bv;
    }
  }

  // Stable three-way split of the outputs (as partition3).
  template <class T, class A0, class A1>
  PBH_INL void split(const T& t, KV p1, KV p2, A0 O0, A1 O1, A1 O2, const u64* live0, u32* n0, u32* n1,
                     u32* n2) const {
    constexpr u32 W = (u32)T::kW;
    const bool two = p2.k == KINF && p2.v == VINF;  // nothing above p2
    auto cls = [&](bool in, u64 k, u32 v) -> u32 {
      u32 c = kv_le(KV{k, v}, p1) ? 0u : 1u;
      if (!two) c = c && !kv_le(KV{k, v}, p2) ? 2u : c;
      if (live0) {
        u64 l = k;
        if (in && c == 0u) l = t.load_cur(live0 + v);
        c = l != k ? 3u : c;
      }
      return in ? c : 3u;
    };
    const u32 cp = cls(pin, pk, pv);
    const u32 p0 = (u32)t.ballot(cp == 0u), pb1 = (u32)t.ballot(cp == 1u), pb2 = two ? 0u : (u32)t.ballot(cp == 2u);
    u32 c0 = 0, c1 = 0, c2 = 0;  // Q's outputs of the rows before
    u32 of = t.count_below(cp == 0u ? p0 : (cp == 1u ? pb1 : pb2));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r > 0 && !t.any_lane(qin[r])) continue;
      const u32 c = cls(qin[r], qk[r], qv[r]);
      const u64 b0 = t.ballot(c == 0u), b1 = t.ballot(c == 1u), b2 = two ? 0ull : t.ballot(c == 2u);
      {
        const u32 lo = (1u << below[r]) - 1u;
        const u32 pm = c == 0u ? p0 : (c == 1u ? pb1 : pb2);
        const u32 o = (c == 0u ? c0 : (c == 1u ? c1 : c2)) + t.count_below(c == 0u ? b0 : (c == 1u ? b1 : b2)) +
                      (u32)__builtin_popcount(pm & lo);
        auto ok = c == 0u ? O0.k : (c == 1u ? O1.k : O2.k);
        auto ov = c == 0u ? O0.v : (c == 1u ? O1.v : O2.v);
        if (c < 3u) {
          ok[o] = qk[r];
          ov[o] = qv[r];
        }
      }
      {  // P's elements: Q's outputs of their class before their place
        const u64 bm = cp == 0u ? b0 : (cp == 1u ? b1 : b2);
        const u32 y = place > (u32)r * W ? place - (u32)r * W : 0u;
        of += (u32)__builtin_popcountll(y >= W ? bm : bm & ((1ull << y) - 1ull));
      }
      c0 += (u32)__builtin_popcountll(b0);
      c1 += (u32)__builtin_popcountll(b1);
      c2 += (u32)__builtin_popcountll(b2);
    }
    {
      auto ok = cp == 0u ? O0.k : (cp == 1u ? O1.k : O2.k);
      auto ov = cp == 0u ? O0.v : (cp == 1u ? O1.v : O2.v);
      if (cp < 3u) {
        ok[of] = pk;
        ov[of] = pv;
      }
    }
    *n0 = c0 + (u32)__builtin_popcount(p0);
    *n1 = c1 + (u32)__builtin_popcount(pb1);
    *n2 = c2 + (u32)__builtin_popcount(pb2);
  }
};

template <int R, class T, class AA, class AB, class AC>
PBH_INL u32 merge_small(const T& t, AA A, u32 na, AB B, u32 nb, AC C, const u64* cur, int prefer, CountLe* le) {
  SmallMerge<R> s;
  u32 nq = nb;
  if constexpr (same_arr<AA, AB>::v) {
    const bool pa = na <= nb;
    nq = pa ? nb : na;
    s.run(t, pa ? A : B, pa ? na : nb, pa ? B : A, nq, pa, cur, prefer);
  } else if (na <= nb) {
    s.run(t, A, na, B, nb, true, cur, prefer);
  } else {
    nq = na;
    s.run(t, B, nb, A, na, false, cur, prefer);
  }
  s.store(t, nq, C);
  if (le) le->n += s.count_le(t, le->p);
  t.sync();
  return s.m;
}

// Merge + DeleteDuplicates by whichever form suits the team and the sizes: one
// wavefront takes a short array into registers (SmallMerge); otherwise every
// thread walks from its merge-path split, for arrays in HBM of more than two
// elements per thread through the LDS staging area when the team has one (256
// threads: 500 elements 4,600 cycles as they are, 6,400 staged; 1,500 14,300
// and 10,000; 4,000 30,000 and 19,900).
template <class T, class AA, class AB, class AC>
PBH_INL u32 merge_dedup(const T& t, AA A, u32 na_, AB B, u32 nb_, AC C, const u64* cur, bool filterB,
                        int prefer = PREFER_LIVE, CountLe* le = nullptr) {
  const u32 na = t.uni(na_), nb = t.uni(nb_);
  if constexpr (T::kNW == 1) {
    const u32 rows = filterB ? 0u : small_rows<T>(na, nb);
    if (rows == 1) return merge_small<1>(t, A, na, B, nb, C, cur, prefer, le);
    if (rows) return merge_small<4>(t, A, na, B, nb, C, cur, prefer, le);
  }
  if constexpr (T::kStage && !in_lds<AA>::v && !in_lds<AB>::v) {
    if (t.stk && na + nb > 2u * (u32)T::kNT)
      return merge_dedup_staged(t, A, na, B, nb, C, cur, filterB, prefer, le);
  }
  if constexpr (T::kNT >= 256) {
    if (na + nb <= 2u * (u32)T::kNT) return merge_dedup_e<T, 2>(t, A, na, B, nb, C, cur, filterB, prefer, le);
  }
  return merge_dedup_e<T, T::kM>(t, A, na, B, nb, C, cur, filterB, prefer, le);
}

// Finds the histogram bin where the r-th element (1-based) falls.
template <class T>
PBH_INL void hist_pick(const T& t, u32 r, u32* D, u32* below, u32* cnt) {
  constexpr int BPT = (256 + T::kNT - 1) / T::kNT;
  u32 b0 = (u32)t.tid() * BPT;
  u32 loc = 0;
#pragma unroll
  for (int q = 0; q < BPT; ++q)
    if (b0 + q < 256) loc += t.sh->hist[b0 + q];
  u32 tot;
  u32 pre = t.scan_excl(loc, &tot);
#pragma unroll
  for (int q = 0; q < BPT; ++q) {
    u32 b = b0 + q;
    if (b < 256) {
      u32 h = t.sh->hist[b];
      if (pre < r && r <= pre + h) {
        t.sh->b32[0] = b;
        t.sh->b32[1] = pre;
        t.sh->b32[2] = h;
      }
      pre += h;
    }
  }
  t.sync();
  *D = t.sh->b32[0];
  *below = t.sh->b32[1];
  *cnt = t.sh->b32[2];
  t.sync();
}

// r-th smallest by repeated team minima (or the (n-r+1)-th largest by
// repeated maxima) over at most 8 elements per thread held in registers; for
// the small ranks that Resolve asks for when one element leaves B_0.
template <class T, class AA>
PBH_INL KV select_small(const T& t, AA A, u32 n_, u32 r_) {
  const u32 n = t.uni(n_), r = t.uni(r_);
  const bool top = (n - r + 1) < r;
  u32 it = top ? n - r + 1 : r;
  u64 kk[8];
  u32 vv[8];
  u32 live = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    u32 x = (u32)t.tid() + (u32)j * (u32)T::kNT;
    kk[j] = 0;
    vv[j] = 0;
    if ((u32)(j * T::kNT) < n && x < n) {
      kk[j] = top ? ~A.k[x] : A.k[x];
      vv[j] = top ? ~A.v[x] : A.v[x];
      live |= 1u << j;
    }
  }
  u64 bk = KINF;
  u32 bv = VINF;
  for (u32 s = 0; s < it; ++s) {
    bk = KINF;
    bv = VINF;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if ((u32)(j * T::kNT) < n && ((live >> j) & 1u)) {
        bool lt = kk[j] < bk || (kk[j] == bk && vv[j] < bv);
        bk = lt ? kk[j] : bk;
        bv = lt ? vv[j] : bv;
      }
    t.minkv(bk, bv);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if ((u32)(j * T::kNT) < n && ((live >> j) & 1u) && kk[j] == bk && vv[j] == bv) live &= ~(1u << j);
  }
  return top ? KV{~bk, ~bv} : KV{bk, bv};
}

// Select over at most Q elements per thread, read once into registers: one
// histogram of the eight bits below the highest one where the keys differ
// usually leaves a few candidates, which go to LDS and are ranked by counting,
// by every wavefront for itself.  More than SEL_FEW candidates go through
// another eight bits (ids after the keys).  Every wavefront finds the bin by
// itself (four bins per lane), so a pass has two barriers; 512 elements,
// 256 threads: 8,800 cycles for three passes of the radix form, about 2,500
// for this.
constexpr u32 SEL_FEW = 32;
template <int Q, class T, class AA>
PBH_INL KV select_hist(const T& t, AA A, u32 n, u32 r) {
  u64 k[Q];
  u32 v[Q], act = 0;
  const u64 k0 = A.k[0];
  u64 df = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const u32 x = (u32)t.tid() + (u32)q * (u32)T::kNT;
    k[q] = k0;
    v[q] = 0;
    if ((u32)q * (u32)T::kNT >= n) continue;
    const u32 xi = x < n ? x : n - 1;
    k[q] = A.k[xi];
    v[q] = A.v[xi];
    act |= x < n ? 1u << q : 0u;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) df |= k[q] ^ k0;
  u32 dh = t.wave_or32((u32)(df >> 32)), dl = t.wave_or32((u32)df);
  if constexpr (T::kNW > 1) {
    if (t.lane() == 0) t.sh->wk[t.wave()] = ((u64)dh << 32) | dl;
  }
  for (u32 b = (u32)t.tid(); b < 256; b += (u32)T::kNT) t.sh->hist[b] = 0;
  if (t.tid() == 0) t.sh->b32[0] = 0;
  t.sync();
  if constexpr (T::kNW > 1) {
    u64 d = 0;
#pragma unroll
    for (int w = 0; w < T::kNW; ++w) d |= t.sh->wk[w];
    dh = t.uni((u32)(d >> 32));
    dl = t.uni((u32)d);
  }
  // digits of the 96-bit value (key, id) from bit `lo` up: the ids' 32 bits,
  // then the key's
  const int top = dh ? 96 - __builtin_clz(dh) : (dl ? 64 - __builtin_clz(dl) : 32);
  int lo = top > 8 ? top - 8 : 0;
  auto digit = [&](u64 kk, u32 vv) -> u32 {
    const u64 w = lo >= 32 ? kk >> (lo - 32) : ((kk << 32) | vv) >> lo;
    return (u32)w & 255u;
  };
  u32 cnt;
  for (;;) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if ((u32)q * (u32)T::kNT < n && ((act >> q) & 1u)) t.hist_add(t.sh->hist, digit(k[q], v[q]));
    t.sync();
    // the bin of rank r: four bins per lane, scanned by every wavefront
    u32 D = 0, below = 0;
    cnt = 0;
    if constexpr (T::kW == 1) {
      for (u32 b = 0, run = 0; b < 256; run += t.sh->hist[b], ++b)
        if (run < r && r <= run + t.sh->hist[b]) D = b, below = run, cnt = t.sh->hist[b];
    } else {
      u32 h[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) h[b] = t.sh->hist[4 * t.lane() + b];
      const u32 s = h[0] + h[1] + h[2] + h[3], inc = t.wave_scan(s);
      const int l = __builtin_ctzll(t.ballot(inc >= r));  // the first lane that reaches the rank
      u32 run = t.lane_val(inc - s, l);
      bool found = false;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const u32 x = t.lane_val(h[b], l);
        if (!found && r <= run + x) {
          D = 4u * (u32)l + (u32)b;
          below = run;
          cnt = x;
          found = true;
        }
        run += x;
      }
    }
    r -= below;
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if ((u32)q * (u32)T::kNT < n && ((act >> q) & 1u) && digit(k[q], v[q]) != D) act &= ~(1u << q);
    if (cnt <= SEL_FEW || lo == 0) break;
    lo = lo > 8 ? lo - 8 : 0;
    t.sync();  // every wavefront has read the histogram
    for (u32 b = (u32)t.tid(); b < 256; b += (u32)T::kNT) t.sh->hist[b] = 0;
    t.sync();
  }
  // the candidates (the values are distinct: one is left at the last bits)
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if ((u32)q * (u32)T::kNT < n && ((act >> q) & 1u)) {
      const u32 o = t.hist_next(&t.sh->b32[0]);
      t.sh->ex0[o] = k[q];
      t.sh->exd[o] = v[q];
    }
  t.sync();
  KV e = kv_inf();
  if constexpr (T::kW == 1) {
    for (u32 x = 0; x < cnt; ++x) {
      u32 c = 0;
      for (u32 y = 0; y < cnt; ++y)
        c += kv_less(KV{t.sh->ex0[y], t.sh->exd[y]}, KV{t.sh->ex0[x], t.sh->exd[x]}) ? 1u : 0u;
      if (c + 1 == r) e = KV{t.sh->ex0[x], t.sh->exd[x]};
    }
  } else {
    const u32 x = (u32)t.lane() < cnt ? (u32)t.lane() : cnt - 1;
    const u64 ck = t.sh->ex0[x];
    const u32 cv = t.sh->exd[x];
    u32 c = 0;
    for (u32 y = 0; y < cnt; ++y)
      c += kv_less(KV{t.lane_val64(ck, (int)y), t.lane_val(cv, (int)y)}, KV{ck, cv}) ? 1u : 0u;
    const int l = __builtin_ctzll(t.ballot((u32)t.lane() < cnt && c + 1 == r));
    e = KV{t.lane_val64(ck, l), t.lane_val(cv, l)};
  }
  t.sync();  // the scratch is free again
  return e;
}

// Select(A, r): the r-th smallest (key, id) of A, 1 <= r <= n.  Radix select,
// most significant byte first, over key - min(key) (only the bytes the key
// range needs), then over the id among elements with the selected key.  The
// paper sorted with a radix sort to select (Section 4.1); a radix select reads
// the candidates once per byte and sorts nothing.  Ranks within two of either
// end of a small array use select_small; other ranks in arrays of at most four
// elements per thread use select_hist, in HBM of at most kHeld: 16, or 32 for
// the single queries of 256 threads that also run speculative rounds (learned,
// 200,000 vertices, d = 256: 597 ms; 613 with 16).  The registers for 32 cost
// every round of the kernels that run plain rounds only more than large Selects
// gain (DAGs of 3,382 and 8,000 vertices, d = 705 and 3,143: 80.0 and 284 ms; 77.1
// and 268 with 16), and of the batches (96 learned queries 15.0 ms; 14.7).
template <class T, class AA>
PBH_INL KV select_kth(const T& t, AA A, u32 n_, u32 r_) {
  const u32 n = t.uni(n_);
  u32 r = t.uni(r_);
  if (n <= 8u * (u32)T::kNT && (r <= 2 || n - r + 1 <= 2)) return select_small(t, A, n, r);
  if (n <= 4u * (u32)T::kNT) return select_hist<4>(t, A, n, r);
  if constexpr (!in_lds<AA>::v) {
    if (n <= 16u * (u32)T::kNT) return select_hist<16>(t, A, n, r);
    if constexpr (T::kHeld > 16) {
      if (n <= (u32)T::kHeld * (u32)T::kNT) return select_hist<T::kHeld>(t, A, n, r);
    }
  }
  u64 lo = KINF, hi = 0;
  for (u32 base = 0; base < n; base += (u32)T::kNT * T::kRU) {
    u64 k[T::kRU];
#pragma unroll
    for (int r = 0; r < T::kRU; ++r) {
      const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
      k[r] = x < n ? A.k[x] : KINF;
    }
#pragma unroll
    for (int r = 0; r < T::kRU; ++r) {
      const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
      lo = k[r] < lo ? k[r] : lo;
      hi = (x < n && k[r] > hi) ? k[r] : hi;
    }
  }
  t.minmax64(lo, hi);
  u64 span = hi - lo;
  int nb = span ? 64 - __builtin_clzll(span) : 0;
  int top = (nb + 7) & ~7;
  u64 prefix = 0;
  u32 cnt = n;
  for (int s = top - 8; s >= 0; s -= 8) {
    for (u32 b = (u32)t.tid(); b < 256; b += (u32)T::kNT) t.sh->hist[b] = 0;
    t.sync();
    for (u32 base = 0; base < n; base += (u32)T::kNT * T::kRU) {
      u64 k[T::kRU];
#pragma unroll
      for (int r = 0; r < T::kRU; ++r) {
        const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
        k[r] = x < n ? A.k[x] : 0;
      }
#pragma unroll
      for (int r = 0; r < T::kRU; ++r) {
        const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
        const u64 dk = k[r] - lo;
        const bool m = x < n && ((s + 8 >= 64) ? true : ((dk >> (s + 8)) == prefix));
        if (m) t.hist_add(t.sh->hist, (u32)(dk >> s) & 255u);
      }
    }
    t.sync();
    u32 D, below;
    hist_pick(t, r, &D, &below, &cnt);
    prefix = (prefix << 8) | D;
    r -= below;
  }
  const u64 K = lo + prefix;
  if (cnt == 1) {
    for (u32 base = 0; base < n; base += (u32)T::kNT * T::kRU) {
      u64 k[T::kRU];
#pragma unroll
      for (int r = 0; r < T::kRU; ++r) {
        const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
        k[r] = x < n ? A.k[x] : ~K;
      }
#pragma unroll
      for (int r = 0; r < T::kRU; ++r)
        if (k[r] == K) t.sh->b32[3] = A.v[base + (u32)r * (u32)T::kNT + (u32)t.tid()];
    }
    t.sync();
    u32 id = t.sh->b32[3];
    t.sync();
    return KV{K, id};
  }
  u32 idp = 0;
  for (int s = 24; s >= 0; s -= 8) {
    for (u32 b = (u32)t.tid(); b < 256; b += (u32)T::kNT) t.sh->hist[b] = 0;
    t.sync();
    for (u32 base = 0; base < n; base += (u32)T::kNT * T::kRU) {
      u64 k[T::kRU];
      u32 v[T::kRU];
#pragma unroll
      for (int r = 0; r < T::kRU; ++r) {
        const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
        k[r] = x < n ? A.k[x] : ~K;
        v[r] = x < n ? A.v[x] : 0u;
      }
#pragma unroll
      for (int r = 0; r < T::kRU; ++r)
        if (k[r] == K && (s == 24 || (v[r] >> (s + 8)) == idp)) t.hist_add(t.sh->hist, (v[r] >> s) & 255u);
    }
    t.sync();
    u32 D, below, c2;
    hist_pick(t, r, &D, &below, &c2);
    idp = (idp << 8) | D;
    r -= below;
  }
  return KV{K, idp};
}

// Stable three-way split of A (order by id is kept in each part):
// e <= p1 -> O0, p1 < e <= p2 -> O1, e > p2 -> O2.  With live0, class-0
// elements that are not live are dropped.
// A tile is E rows of one element per thread (consecutive threads read and
// write consecutive elements: no LDS bank conflicts, coalesced in HBM); places
// within a row come from ballots.  One wavefront adds up the rows in scalars;
// a larger team exchanges the rows' counts through LDS, one barrier per tile
// (two areas in turn), and every wavefront scans them by itself.  Rows past
// the end are skipped by scalar branches.
template <class T, class AA, class A0, class A1, class A2>
PBH_INL void partition3(const T& t, AA A, u32 n_, KV p1, KV p2, A0 O0, A1 O1, A2 O2, u32* n0, u32* n1,
                        u32* n2, const u64* live0 = nullptr) {
  // twice the elements per thread from HBM: more loads in flight per tile;
  // at most one count per lane of a wavefront
  constexpr int EW = ((T::kStage || T::kNT >= 256) && !in_lds<AA>::v) ? 2 * T::kE : T::kE;
  constexpr int E = (T::kNW > 1 && EW * T::kNW > 64) ? 64 / T::kNW : EW;
  const u32 n = t.uni(n_);
  const bool three = t.uni((u32)kv_less(p2, kv_inf())) != 0;  // (else nothing lies beyond p2)
  u32 c0 = 0, c1 = 0, c2 = 0;
  u32 par = 0;
  for (u32 base = 0; base < n; base += (u32)T::kNT * E, par ^= 128u) {
    u64 kk[E];
    u32 vv[E], cl[E], at[E];
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const u32 x = base + (u32)s * (u32)T::kNT + (u32)t.tid();
      kk[s] = 0;
      vv[s] = 0;
      if (base + (u32)s * (u32)T::kNT < n && x < n) {
        kk[s] = A.k[x];
        vv[s] = A.v[x];
      }
    }
    u64 cur[E];
    if (live0) {
#pragma unroll
      for (int s = 0; s < E; ++s) {
        const u32 x = base + (u32)s * (u32)T::kNT + (u32)t.tid();
        cur[s] = kk[s];
        if (x < n && kv_le(KV{kk[s], vv[s]}, p1)) cur[s] = t.load_cur(live0 + vv[s]);
      }
    }
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const u32 x = base + (u32)s * (u32)T::kNT + (u32)t.tid();
      const KV e{kk[s], vv[s]};
      cl[s] = 3u;
      at[s] = 0;
      if (base + (u32)s * (u32)T::kNT >= n) continue;
      cl[s] = kv_le(e, p1) ? 0u : 1u;
      if (three) cl[s] = cl[s] == 0u || kv_le(e, p2) ? cl[s] : 2u;
      if (live0 && cur[s] != kk[s]) cl[s] = 3u;
      if (x >= n) cl[s] = 3u;
      const u64 b0 = t.ballot(cl[s] == 0u), b1 = t.ballot(cl[s] == 1u);
      u32 q0 = (u32)__builtin_popcountll(b0), q1 = (u32)__builtin_popcountll(b1), q2 = 0;
      const u32 r0 = t.count_below(b0), r1 = t.count_below(b1);
      u32 r2 = 0;
      if (three) {
        const u64 b2 = t.ballot(cl[s] == 2u);
        r2 = t.count_below(b2);
        q2 = (u32)__builtin_popcountll(b2);
      }
      if constexpr (T::kNW == 1) {
        at[s] = cl[s] == 0u ? c0 + r0 : (cl[s] == 1u ? c1 + r1 : c2 + r2);
        c0 += q0;
        c1 += q1;
        c2 += q2;
      } else {
        at[s] = cl[s] == 0u ? r0 : (cl[s] == 1u ? r1 : r2);
        if (t.lane() == 0) t.sh->base[par + (u32)s * T::kNW + (u32)t.wave()] = q0 | q1 << 8 | q2 << 16;
      }
    }
    if constexpr (T::kNW > 1) {
      t.sync();
      const u32 wv = t.uni((u32)t.wave());
      const u32 rows = (n - base + (u32)T::kNT - 1) / (u32)T::kNT;  // rows of this tile that hold counts
      const u32 w = (u32)t.lane() < (u32)(E * T::kNW) && (u32)t.lane() < rows * (u32)T::kNW
                        ? t.sh->base[par + (u32)t.lane()]
                        : 0u;
      const u32 x01 = (w & 0xFFu) | (w & 0xFF00u) << 8, x2 = w >> 16;
      const u32 i01 = t.wave_scan(x01), i2 = t.wave_scan(x2);
      const u32 e01 = i01 - x01, e2 = i2 - x2;
#pragma unroll
      for (int s = 0; s < E; ++s) {
        if (base + (u32)s * (u32)T::kNT >= n) continue;
        const int l = s * T::kNW + (int)wv;
        const u32 o01 = t.lane_val(e01, l), o2 = t.lane_val(e2, l);
        at[s] += cl[s] == 0u ? c0 + (o01 & 0xFFFFu) : (cl[s] == 1u ? c1 + (o01 >> 16) : c2 + o2);
      }
      const u32 t01 = t.lane_val(i01, 63);
      c0 += t01 & 0xFFFFu;
      c1 += t01 >> 16;
      c2 += t.lane_val(i2, 63);
    }
#pragma unroll
    for (int s = 0; s < E; ++s) {
      if (base + (u32)s * (u32)T::kNT >= n) continue;
      if constexpr (same_arr<A0, A1>::v && same_arr<A0, A2>::v) {
        // one store for whichever array it goes to
        const auto pk = cl[s] == 0u ? O0.k : (cl[s] == 1u ? O1.k : O2.k);
        const auto pv = cl[s] == 0u ? O0.v : (cl[s] == 1u ? O1.v : O2.v);
        if (cl[s] < 3u) {
          pk[at[s]] = kk[s];
          pv[at[s]] = vv[s];
        }
        continue;
      }
      if (cl[s] == 0u) {
        O0.k[at[s]] = kk[s];
        O0.v[at[s]] = vv[s];
      } else if (cl[s] == 1u) {
        O1.k[at[s]] = kk[s];
        O1.v[at[s]] = vv[s];
      } else if (cl[s] == 2u) {
        O2.k[at[s]] = kk[s];
        O2.v[at[s]] = vv[s];
      }
    }
  }
  t.sync();
  *n0 = c0;
  *n1 = c1;
  *n2 = c2;
}

struct DigitId {
  int s;
  PBH_INL u32 operator()(u64, u32 v) const { return (v >> s) & 255u; }
};
struct DigitKey {
  int s;
  u64 lo;
  PBH_INL u32 operator()(u64 k, u32) const { return (u32)((k - lo) >> s) & 255u; }
};

// One stable counting-sort pass on an 8-bit digit (LSD radix sort).  Ranks
// among equal digits inside a wavefront come from ballots (peer masks), and
// across wavefronts from per-wave digit counts in LDS.
template <class T, class AS, class AD, class F>
PBH_INL void radix_pass(const T& t, AS src, AD dst, u32 n, F dig) {
  for (u32 b = (u32)t.tid(); b < 256; b += (u32)T::kNT) t.sh->hist[b] = 0;
  t.sync();
  for (u32 x = (u32)t.tid(); x < n; x += (u32)T::kNT) t.hist_add(t.sh->hist, dig(src.k[x], src.v[x]));
  t.sync();
  {
    constexpr int BPT = (256 + T::kNT - 1) / T::kNT;
    u32 b0 = (u32)t.tid() * BPT, loc = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q)
      if (b0 + q < 256) loc += t.sh->hist[b0 + q];
    u32 tot;
    u32 pre = t.scan_excl(loc, &tot);
#pragma unroll
    for (int q = 0; q < BPT; ++q)
      if (b0 + q < 256) {
        t.sh->base[b0 + q] = pre;
        pre += t.sh->hist[b0 + q];
      }
  }
  t.sync();
  for (u32 tb = 0; tb < n; tb += (u32)T::kNT) {
    u32 x = tb + (u32)t.tid();
    bool valid = x < n;
    u64 k = valid ? src.k[x] : 0;
    u32 v = valid ? src.v[x] : 0;
    u32 dg = valid ? dig(k, v) : 0;
    u64 m = t.ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      bool bit = (dg >> b) & 1u;
      u64 bb = t.ballot(valid && bit);
      m &= bit ? bb : ~bb;
    }
    u32 rank = t.count_below(m);
    u32 cnt = (u32)__builtin_popcountll(m);
    for (u32 z = (u32)t.tid(); z < (u32)T::kNW * 256; z += (u32)T::kNT) t.sh->wcnt[z >> 8][z & 255] = 0;
    t.sync();
    if (valid && rank == 0) t.sh->wcnt[t.wave()][dg] = cnt;
    t.sync();
    for (u32 gd = (u32)t.tid(); gd < 256; gd += (u32)T::kNT) {
      u32 run = t.sh->base[gd];
      for (int w = 0; w < T::kNW; ++w) {
        u32 c = t.sh->wcnt[w][gd];
        t.sh->wcnt[w][gd] = run;
        run += c;
      }
      t.sh->base[gd] = run;
    }
    t.sync();
    if (valid) {
      u32 pos = t.sh->wcnt[t.wave()][dg] + rank;
      dst.k[pos] = k;
      dst.v[pos] = v;
    }
    t.sync();
  }
}

// Sorts n elements by id (idbits significant bits).  Returns true when the
// result ended in tmp (false: in a).
template <class T, class A>
PBH_INL bool sort_by_id(const T& t, A a, A tmp, u32 n, int idbits) {
  bool in_tmp = false;
  for (int s = 0; s < idbits; s += 8) {
    if (in_tmp)
      radix_pass(t, tmp, a, n, DigitId{s});
    else
      radix_pass(t, a, tmp, n, DigitId{s});
    in_tmp = !in_tmp;
  }
  return in_tmp;
}

// Sorts n elements by (key, id); returns true when the result is in tmp.
template <class T, class A>
PBH_INL bool sort_kv(const T& t, A a, A tmp, u32 n, int idbits) {
  bool in_tmp = sort_by_id(t, a, tmp, n, idbits);
  if (n == 0) return in_tmp;
  A src = in_tmp ? tmp : a;
  u64 lo = KINF, hi = 0;
  for (u32 x = (u32)t.tid(); x < n; x += (u32)T::kNT) {
    u64 k = src.k[x];
    lo = k < lo ? k : lo;
    hi = k > hi ? k : hi;
  }
  t.minmax64(lo, hi);
  u64 span = hi - lo;
  int nb = span ? 64 - __builtin_clzll(span) : 0;
  for (int s = 0; s < nb; s += 8) {
    if (in_tmp)
      radix_pass(t, tmp, a, n, DigitKey{s, lo});
    else
      radix_pass(t, a, tmp, n, DigitKey{s, lo});
    in_tmp = !in_tmp;
  }
  return in_tmp;
}

template <class T, class AS, class AD>
PBH_INL void copy_arr(const T& t, AS src, AD dst, u32 n) {
  for (u32 x = (u32)t.tid(); x < n; x += (u32)T::kNT) {
    dst.k[x] = src.k[x];
    dst.v[x] = src.v[x];
  }
  t.sync();
}

// ---------------------------------------------------------------- the heap

// Recomputes ell (deepest non-empty level) and sets p_j = +inf for j >= ell:
// the deepest non-empty level has nothing below it to separate from.
// A deep_floor set by the deep-level service counts as a non-empty level.
template <class SP>
PBH_INL void fix_ell(SP st, int q) {
  int e = -1;
  for (int j = q - 1; j >= 0; --j)
    if (st->L[j].nB + st->L[j].nS) {
      e = j;
      break;
    }
  if (st->deep_floor > e) e = st->deep_floor;
  st->ell = e;
  for (int j = e < 0 ? 0 : e; j < MAXL; ++j) {
    st->L[j].pk = KINF;
    st->L[j].pv = VINF;
  }
}

// fix_ell by the team: one lane per level (the loop over the levels is a chain
// of LDS reads, 0.4 us a Resolve).  Every thread calls it; the first wavefront
// does the work, after its own thread 0 may have changed the state.
template <class T, class SP>
PBH_INL void fix_ell_team(const T& t, SP st, int q) {
  if constexpr (T::kW == 1) {
    fix_ell(st, q);
  } else if (t.wave() == 0) {
    t.wsync();
    const int l = t.lane();
    const u32 has = l < q ? (st->L[l].nB | st->L[l].nS) : 0u;
    const u64 m = t.ballot(has != 0);
    int e = m ? 63 - __builtin_clzll(m) : -1;
    if (st->deep_floor > e) e = st->deep_floor;
    if (l == 0) st->ell = e;
    if (l >= e && l < MAXL) {
      st->L[l].pk = KINF;
      st->L[l].pv = VINF;
    }
  }
}

// Algorithm 1, Resolve(i): empty S_i and fill B_i, with level i's arrays of
// type AI and level i+1's of type AN.
//   EMPTY: B_i <- DeleteDuplicates(Merge(S_i, B_i)); if more than 2d*4^i
//          elements are <= p_i, p_i <- Select(B_i, 2d*4^i); elements > p_i move
//          to S_{i+1} <- Merge(S_{i+1}, B'_i).
//   FILL (if |B_i| < 2d*4^i and i is not the deepest non-empty level):
//          B_{i+1} <- DeleteDuplicates(Merge(B_{i+1}, S_{i+1}));
//          p_i <- Select(B_{i+1}, 2d*4^i - |B_i|); elements <= p_i move up into
//          B_i <- Merge(B_i, B'_{i+1}); elements > p_{i+1} go back to S_{i+1}.
// Readings (documented with the others): EMPTY also runs when B_i holds more
// than 2d*4^i elements with S_i empty (B_i can absorb elements of S_i during
// FILL of level i-1); the new p_i in FILL never exceeds p_{i+1}, so nothing
// deeper than level i+1 can be smaller than an element moved up; the two
// splits at the end of FILL are one three-way split.
//
// Written as one loop over the four merges (EMPTY, the push down, FILL, the
// move up) around one merge, one Select and one split: the round loop runs
// through its code once per round, and every instance of these primitives
// that it passes has to come through the 64 KiB instruction cache (four merges
// and two of each other inlined: 286 KB for the smallest kernel, and a round
// was bound by instruction fetches).
template <class T, class P, class AI, class AN>
PBH_INL void resolve_t(T t, Geom g, typename P::SP st, const u64* cur, int i) {
  constexpr bool kSame = same_arr<AI, AN>::v;
  enum { EMPTY, PUSH, FILL, UP, END };
  Lvl a = lvl_uni(t, st, i);
  const bool nx = i + 1 < g.q;
  Lvl b = nx ? lvl_uni(t, st, i + 1) : Lvl{0, 0, 0, 0, KINF, VINF, 0};
  int ell = (int)t.uni((u32)st->ell);
  KV pi{a.pk, a.pv}, pn{b.pk, b.pv};
  const u32 cB = (u32)nomB(g.d, i);
  u64 touched = 0;
  int err = 0;
  u32 n1 = 0;          // elements pushed down / moved up, in X
  // arrays are named by level (i or i + 1) and buffer, and resolved where they
  // are used (pointers would be seven pairs of scalars to keep)
  constexpr u32 NXT = 8u, X = 2u;
  auto at = [&](u32 c) { return lbuf(g, i + (int)(c >> 3), (int)(c & 7u)); };
  // FILL is due once EMPTY (if due) is through
  auto fill_due = [&] { return a.nB < cB && i < ell && nx ? (int)FILL : (int)END; };
  int step = a.nS > 0 || a.nB > cB ? (int)EMPTY : fill_due();
  while (step != END) {
    // the merge of this step: B into A's order, output M
    u32 A, B, M;
    u32 na, nb, m;
    int prefer = PREFER_LIVE;
    bool merge = true;  // false: one side is empty, M is the other
    CountLe le{pi, 0};
    if (step == EMPTY) {
      A = 3 + a.ssel;
      B = a.bsel;
      M = a.bsel ^ 1;
      na = a.nS;
      nb = a.nB;
      // S_0 holds the latest updates, so at level 0 its copy of an id is the live one.
      if (i == 0) prefer = PREFER_A;
      if ((u64)na + nb > capB(g.d, i)) err = E_INTERNAL;
    } else if (step == PUSH) {
      A = NXT + (3 + b.ssel);
      B = X;
      M = NXT + (3 + (b.ssel ^ 1));
      na = b.nS;
      nb = n1;
      // (with S_{i+1} empty the split wrote to M, where both levels are of one kind)
      merge = !kSame || na > 0;
    } else if (step == FILL) {
      A = NXT + (b.bsel);
      B = NXT + (3 + b.ssel);
      M = NXT + (b.bsel ^ 1);
      na = b.nB;
      nb = b.nS;
      merge = nb > 0;
      if (!merge) M = A;
      if ((u64)na + nb > capB(g.d, i + 1)) err = E_INTERNAL;
    } else {
      A = a.bsel;
      B = X;
      M = a.bsel ^ 1;
      na = a.nB;
      nb = n1;
      if (i == 0 && cur != nullptr) prefer = PREFER_B;
    }
    if (err) break;
    m = na + nb;
    if (merge) {
      if constexpr (kSame)
        m = merge_dedup(t, as_arr<AI>(at(A)), na, as_arr<AI>(at(B)), nb, as_arr<AI>(at(M)), cur, false, prefer, &le);
      else if (step == PUSH)
        m = merge_dedup(t, as_arr<AN>(at(A)), na, as_arr<AI>(at(B)), nb, as_arr<AN>(at(M)), cur, false, prefer, &le);
      else if (step == FILL)
        m = merge_dedup(t, as_arr<AN>(at(A)), na, as_arr<AN>(at(B)), nb, as_arr<AN>(at(M)), cur, false, prefer, &le);
      else
        m = merge_dedup(t, as_arr<AI>(at(A)), na, as_arr<AI>(at(B)), nb, as_arr<AI>(at(M)), cur, false, prefer, &le);
    }
    touched += 2ull * ((u64)na + nb) + m;
    if (step == PUSH) {
      b.ssel ^= 1;
      b.nS = m;
      if (ell < i + 1) ell = i + 1;
      step = fill_due();
      continue;
    }
    if (step == UP) {
      a.bsel ^= 1;
      a.nB = m;
      step = END;
      continue;
    }
    // EMPTY and FILL: choose the pivot, split M at it
    u32 r = 0;  // rank of the pivot in M (0: no Select)
    KV p1 = pi, p2 = kv_inf();
    u32 O0, O1, O2;
    const u64* live = nullptr;
    if (step == EMPTY) {
      a.bsel ^= 1;
      a.nS = 0;
      a.ssel = 0;
      u32 num = le.n;
      if (num > cB) r = num = cB;
      if (num == m) {
        a.nB = m;
        step = fill_due();
        continue;
      }
      if (!nx) {
        err = E_CAPACITY;
        break;
      }
      if ((u64)b.nS + (m - num) > capS(g.d, i + 1)) {
        err = E_INTERNAL;
        break;
      }
      O0 = a.bsel ^ 1;
      O1 = kSame && b.nS == 0 ? NXT + 3 + (b.ssel ^ 1) : X;
      O2 = O1;
    } else {
      if (merge) b.bsel ^= 1;
      b.nS = 0;
      b.ssel = 0;
      b.nB = m;
      if (m == 0) {
        step = END;
        continue;
      }
      const u32 want = cB - a.nB;
      r = want < m ? want : 0u;
      p1 = kv_inf();
      p2 = pn;
      O0 = X;
      O1 = NXT + (b.bsel ^ 1);
      O2 = NXT + (3);
      // Elements moving up into B_0 are checked for liveness here, all at once.
      if (i == 0) live = cur;
    }
    if (r) {
      touched += m;
      if constexpr (kSame)
        p1 = select_kth(t, as_arr<AI>(at(M)), m, r);
      else if (step == EMPTY)
        p1 = select_kth(t, as_arr<AI>(at(M)), m, r);
      else
        p1 = select_kth(t, as_arr<AN>(at(M)), m, r);
    }
    if (step == FILL && kv_less(pn, p1)) p1 = pn;
    pi = p1;
    touched += 3ull * m;
    u32 n0, n2;
    if constexpr (kSame)
      partition3(t, as_arr<AI>(at(M)), m, p1, p2, as_arr<AI>(at(O0)), as_arr<AI>(at(O1)), as_arr<AI>(at(O2)), &n0, &n1, &n2, live);
    else if (step == EMPTY)
      partition3(t, as_arr<AI>(at(M)), m, p1, p2, as_arr<AI>(at(O0)), as_arr<AI>(at(O1)), as_arr<AI>(at(O2)), &n0, &n1, &n2);
    else
      partition3(t, as_arr<AN>(at(M)), m, p1, p2, as_arr<AI>(at(O0)), as_arr<AN>(at(O1)), as_arr<AN>(at(O2)), &n0, &n1, &n2, live);
    if (step == EMPTY) {
      a.bsel ^= 1;
      a.nB = n0;
      step = PUSH;
    } else {
      b.bsel ^= 1;
      b.nB = n1;
      b.nS = n2;
      n1 = n0;
      step = UP;
    }
  }
  t.sync();
  if (t.tid() == 0) {
    if (err) {
      st->err = err;
    } else {
      a.cnt++;
      a.pk = pi.k;
      a.pv = pi.v;
      if (touched) {
        lvl_store(st, i, a);
        if (nx) lvl_store(st, i + 1, b);
        st->elems += touched;
      } else {
        st->L[i].cnt = a.cnt;
      }
    }
  }
  if (!err) fix_ell_team(t, st, g.q);
  t.sync();
}

// Resolve(0) by one wavefront with levels 0 and 1 in LDS, while the arrays
// are small (small_rows): each of EMPTY and FILL is one pass in registers --
// merge, Select and split without the merged array in between -- and so are
// the push down and the move up.  The result is resolve_t's.  A round of the
// plain rule is bound by the instructions of its one wavefront (5 to 8 cycles
// each, whatever they do), and most of them were the general form's: places of
// buffers for any level and placement, loops over elements per thread, the
// merged array's way through LDS.  Returns false if resolve_t has to do (the
// rest of) the work; the state is then as if that part were still due.
template <class T, class P>
PBH_INL bool resolve0_wave(const T& t, const Geom& g, typename P::SP st, const u64* cur) {
  using AI = typename P::L;
  Lvl a = lvl_uni(t, st, 0), b = lvl_uni(t, st, 1);
  const u32 d = g.d, cB = 2u * d;
  int ell = (int)t.uni((u32)st->ell);
  auto arr = [&](u32 o) {  // by element offset: level 0 starts at 0, level 1 at 16 d
    AI x = as_arr<AI>(Arr{g.lk, g.lv});
    x.k += o;
    x.v += o;
    return x;
  };
  auto l1B = [&](u32 s) { return 16u * d + s * 16u * d; };
  auto l1S = [&](u32 s) { return 64u * d + s * 8u * d; };
  const u32 X = 8u * d;  // the level's temporary buffer
  u32 touched = 0, n0, n1, n2;
  KV pi{a.pk, a.pv};
  if (a.nS > 0 || a.nB > cB) {
    const u32 rows = small_rows<T>(a.nS, a.nB);
    if (rows == 0 || a.nS + a.nB > 4u * d) return false;  // (resolve_t reports what does not fit)
    u32 m = 0;
    KV p1 = pi;
    bool fit = true;
    auto empty = [&](auto& s) {
      const bool sa = a.nS <= a.nB;
      const u32 oS = 12u * d, oB = a.bsel * 4u * d;
      s.run(t, arr(sa ? oS : oB), sa ? a.nS : a.nB, arr(sa ? oB : oS), sa ? a.nB : a.nS, sa, cur, PREFER_A);
      m = s.m;
      u32 num = pi.k == KINF ? m : s.count_le(t, pi);
      const bool sel = num > cB;
      if (sel) num = cB;
      if (b.nS + (m - num) > 8u * d) {
        fit = false;
        return;
      }
      if (sel) {
        p1 = s.select(t, cB);
        touched += m;
      }
      s.split(t, p1, kv_inf(), arr((a.bsel ^ 1u) * 4u * d), arr(b.nS ? X : l1S(b.ssel ^ 1u)),
              arr(b.nS ? X : l1S(b.ssel ^ 1u)), nullptr, &n0, &n1, &n2);
    };
    if (rows == 1) {
      SmallMerge<1> s;
      empty(s);
    } else {
      SmallMerge<4> s;
      empty(s);
    }
    if (!fit) return false;
    touched += 2u * (a.nS + a.nB) + m;
    a.bsel ^= 1u;
    a.nB = n0;
    a.nS = 0;
    if (n1) {
      touched += 3u * m;
      pi = p1;
      t.sync();
      const u32 ns = b.nS;
      b.nS = ns ? merge_dedup(t, arr(l1S(b.ssel)), ns, arr(X), n1, arr(l1S(b.ssel ^ 1u)), cur, false) : n1;
      b.ssel ^= 1u;
      touched += 2u * (ns + n1) + b.nS;
      if (ell < 1) ell = 1;
    }
    t.sync();
  }
  bool whole = true;
  if (a.nB < cB && 0 < ell) {
    // (what does not fit B_1's buffers is left to resolve_t as well; asked for
    // as a scalar, the test costs a round nothing that can be measured, and
    // 0.7% folded into `rows`)
    const u32 rows = small_rows<T>(b.nB, b.nS);
    whole = rows != 0 && t.uni(b.nB + b.nS) <= t.uni(16u * d);
    if (whole) {
      u32 m = 0;
      KV p1 = kv_inf();
      const KV pn{b.pk, b.pv};
      auto fill = [&](auto& s) {
        const bool sb = b.nB <= b.nS;
        const u32 oB = l1B(b.bsel), oS = l1S(b.ssel);
        s.run(t, arr(sb ? oB : oS), sb ? b.nB : b.nS, arr(sb ? oS : oB), sb ? b.nS : b.nB, sb, cur, PREFER_LIVE);
        m = s.m;
        const u32 want = cB - a.nB;
        if (want < m) {
          p1 = s.select(t, want);
          touched += m;
        }
        if (kv_less(pn, p1)) p1 = pn;
        s.split(t, p1, pn, arr(X), arr(l1B(b.bsel ^ 1u)), arr(l1S(0)), cur, &n0, &n1, &n2);
      };
      if (rows == 1) {
        SmallMerge<1> s;
        fill(s);
      } else {
        SmallMerge<4> s;
        fill(s);
      }
      t.sync();
      touched += 2u * (b.nB + b.nS) + m;
      b.bsel ^= 1u;
      b.nB = n1;
      b.nS = n2;
      b.ssel = 0;
      if (m) {
        const u32 nb = a.nB;
        a.nB = merge_dedup(t, arr(a.bsel * 4u * d), nb, arr(X), n0, arr((a.bsel ^ 1u) * 4u * d), cur, false,
                           cur != nullptr ? PREFER_B : PREFER_LIVE);
        a.bsel ^= 1u;
        touched += 3u * m + 2u * (nb + n0) + a.nB;
        pi = p1;
      }
    }
  }
  if (t.tid() == 0) {
    a.cnt += whole ? 1u : 0u;
    a.pk = pi.k;
    a.pv = pi.v;
    lvl_store(st, 0, a);
    if (touched) lvl_store(st, 1, b);
    st->elems += touched;
    if (!whole) st->ell = ell;
  }
  if (whole) fix_ell_team(t, st, g.q);
  t.sync();
  return whole;
}

template <class T, class P>
PBH_INL void resolve(const T& t, const Geom& g, typename P::SP st, const u64* cur, int i) {
  P::on_resolve(g, st, i, false);
  if (t.prof && t.tid() == 0) st->prof_res = pbh_clock();
  bool done = false;
  if constexpr (T::kNW == 1) {
    if (i == 0 && g.qlds > 1) done = resolve0_wave<T, P>(t, g, st, cur);
  }
  if (done) {
    // nothing left
  } else if (i + 1 < g.qlds)
    resolve_t<T, P, typename P::L, typename P::L>(t, g, st, cur, i);
  else if (i < g.qlds)
    resolve_t<T, P, typename P::L, typename P::G>(t, g, st, cur, i);
  else
    resolve_t<T, P, typename P::G, typename P::G>(t, g, st, cur, i);
  if (t.prof && t.tid() == 0) st->prof[i] += pbh_clock() - st->prof_res;
  P::on_resolve(g, st, i, true);
}

// Can Resolve(j) move its worst case (all of S_j and B_j) into level j+1?
template <class SP>
PBH_INL bool room_below(const Geom& g, SP st, int j) {
  if (j + 1 >= g.q) return true;
  u64 push = (u64)st->L[j].nS + st->L[j].nB;
  u64 bS = st->L[j + 1].nS, bB = st->L[j + 1].nB;
  return bS + push <= capS(g.d, j + 1) && bB + bS + push <= capB(g.d, j + 1);
}

enum { DRIVE_AFTER = 1, DRIVE_ENSURE = 2 };

// The resolution schedule, as one loop with a single call of Resolve (so each
// placement variant of Resolve is instantiated once per kernel).  Requests:
//
// * DRIVE_AFTER -- after an operation: Resolve(0), then the schedule:
//     sched 0 = Theorem 1: Resolve(i+1) after every fourth Resolve(i);
//     sched 1 = on demand (as the sequential bucket heap of Section 2.1 does):
//               Resolve(i+1) only when the next Resolve(i) would otherwise
//               violate its preconditions on level i+1.
// * DRIVE_ENSURE -- then, while B_0 is empty and the heap is not (possible
//     when dead copies thin out the levels below: Resolve(0) drops the dead
//     ones among the elements it moves up), let j be the shallowest non-empty
//     level below 0 and resolve levels j, j-1, ..., 0 (Resolve(j) first, so
//     that S_j elements above p_j move down and B_j is filled).  A cascade
//     puts a live element into B_0 or drops dead ones at level 0; the loop
//     gives up with E_INTERNAL after (elements + 1) * (q + 1) cascades rather
//     than spin.
//
// Every requested Resolve(x) first resolves the levels below x that lack
// room for what Resolve(x) may push down: find the first j >= x whose next
// level can take all of S_j and B_j, then resolve j, j-1, ..., x.  After
// Resolve(j), level j has S_j empty and |B_j| <= 2d*4^j, which always leaves
// room for level j-1.
//
// `res(i)` performs Resolve(i) on `st`: the team's own Resolve in the kernels,
// or the device-wide engine driven from the host.
//
// With the deep-level service (levels >= lim resolved by their own workers,
// Section 2.2.1), this caller never resolves a level >= lim itself: when the
// Theorem 1 schedule reaches Resolve(lim), `post(lim)` hands it to level lim's
// worker and the schedule of this caller ends there (the worker continues
// it); levels lack room only up to lim - 1 here (res(lim - 1) makes room in
// level lim itself); and when B_0 must be refilled but every level below 0
// that this caller holds is empty, `ensure()` refills it from the worker
// levels and the drive ends.  lim >= q: no workers.
template <class T, class SP, class R, class PO, class EN>
PBH_INL void drive_with(const T& t, const Geom& g, SP st, int sched, int what, R&& res, int lim, PO&& post,
                        EN&& ensure) {
  int tgt = -1, chain = -1;  // pending chain: levels chain, chain-1, ..., tgt
  int stage = (what & DRIVE_AFTER) ? 0 : 2;
  int si = 0;                // schedule position
  int ek = -1;               // refill position
  u64 cascades = 0, climit = 0;
  for (;;) {
    // the words the common path looks at, read together
    const u32 err = (u32)st->err, ell0 = (u32)st->ell, nB0 = st->L[0].nB, nS0 = st->L[0].nS, cnt0 = st->L[0].cnt,
              nB1 = st->L[1].nB, nS1 = st->L[1].nS;
    if (t.uni(err)) break;
    int lvl = -1;
    if (stage == 0) {
      const u64 push = (u64)t.uni(nS0) + t.uni(nB0), bS = t.uni(nS1), bB = t.uni(nB1);
      if (g.q < 2 || (bS + push <= capS(g.d, 1) && bB + bS + push <= capB(g.d, 1)) || lim <= 1) {
        stage = 1;  // Resolve(0), with room below it
        tgt = lvl = 0;
        if constexpr (T::kW > 1) {
          // Nothing to empty and nothing to fill (half of the speculative
          // rounds' Resolves): only the count and an emptied level 0 show.
          const u32 nb = t.uni(nB0), ell = t.uni(ell0), cnt = t.uni(cnt0) + 1u;
          if (push == nb && nb <= (u32)nomB(g.d, 0) && ((int)ell < 1 || nb == (u32)nomB(g.d, 0))) {
            t.sync();
            if (t.tid() == 0) {
              st->L[0].cnt = cnt;
              if ((int)ell < 1) st->ell = nb ? 0 : -1;
            }
            t.sync();
            if (sched == 0 && ((int)ell < 1 || (cnt & 3u) != 0)) {
              stage = 2;
              if (!(what & DRIVE_ENSURE) || nb != 0 || (int)ell < 1) break;
            }
            lvl = -1;
            continue;
          }
        }
      }
    } else if (stage == 1 && chain < 0 && si == 0 && sched == 0 &&
               ((int)t.uni(ell0) < 1 || (t.uni(cnt0) & 3u) != 0)) {
      stage = 2;  // no Resolve(1) due
      if (!(what & DRIVE_ENSURE) || t.uni(nB0) != 0 || (int)t.uni(ell0) < 1) break;
    }
    if (lvl == 0) {
      // decided above
    } else if (chain >= 0) {
      lvl = chain;
      chain = chain > tgt ? chain - 1 : -1;
    } else {
      int x = -1;
      if (stage == 0) {
        x = 0;
        stage = 1;
        si = 0;
      } else if (stage == 1) {
        bool go = si + 1 < g.q && si + 1 <= st->ell;
        if (go) {
          if (sched == 0) {
            go = (st->L[si].cnt & 3u) == 0;
          } else {
            u64 bS = st->L[si + 1].nS, bB = st->L[si + 1].nB;
            go = bS > nomS(g.d, si + 1) - nomS(g.d, si) ||
                 (si + 1 < st->ell && bB < nomS(g.d, si + 1) + nomS(g.d, si));
          }
        }
        if (go && si + 1 >= lim) {
          post(si + 1);
          stage = 2;
        } else if (go) {
          x = si + 1;
          ++si;
        } else {
          stage = 2;
        }
      }
      if (x < 0 && stage == 2) {
        if (!(what & DRIVE_ENSURE)) break;
        if (ek < 0) {
          const int ell = st->ell;
          if (st->L[0].nB != 0 || ell < 1) break;
          int j = 1;
          u64 tot = 0;
          for (int l = 0; l <= ell; ++l) tot += (u64)st->L[l].nB + st->L[l].nS;
          while (j <= ell && j < lim && st->L[j].nB + st->L[j].nS == 0) ++j;
          if (j >= lim && j <= ell) {
            ensure();
            break;
          }
          if (cascades == 0) climit = (tot + 1) * (u64)(g.q + 1);
          if (j > ell || ++cascades > climit) {
            t.sync();
            if (t.tid() == 0) st->err = E_INTERNAL;
            t.sync();
            break;
          }
          ek = j;
        }
        x = ek--;
      }
      int j = x;
      while (j + 1 < g.q && j + 1 < lim && !room_below(g, st, j)) ++j;
      tgt = x;
      lvl = j;
      chain = j > x ? j - 1 : -1;
    }
    res(lvl);
  }
}

template <class T, class SP, class R>
PBH_INL void drive_with(const T& t, const Geom& g, SP st, int sched, int what, R&& res) {
  drive_with(t, g, st, sched, what, res, MAXL, [](int) {}, [] {});
}

template <class T, class P>
PBH_INL void drive(const T& t, const Geom& g, typename P::SP st, const u64* cur, int sched, int what) {
  drive_with(t, g, st, sched, what, [&](int lvl) { resolve<T, P>(t, g, st, cur, lvl); });
}

// ---------------------------------------------------------------- deep-level service
// Section 2.2.1 and Theorem 1: Resolve(i) only needs levels i and i+1, so
// Resolves of levels two apart can run at the same time.  The paper gives
// every level its own thread block (Section 4.1).  Here the team that runs the
// rounds (the "front") keeps levels 0 .. lim-1 -- among them every level in
// its LDS -- and each level i >= lim has a worker team of its own that runs
// Resolve(i) on request.  Level i+1's owner is idle whenever Resolve(i) runs:
//
//  * the owner of level i-1 (the front for i = lim) posts a request for
//    Resolve(i) after every fourth Resolve(i-1) (Theorem 1), and before each
//    Resolve(i-1) waits until every posted Resolve(i) is done;
//  * worker i, before each Resolve(i), waits until every posted Resolve(i+1)
//    is done; if level i+1 lacks room for what Resolve(i) can push down, it
//    posts an extra Resolve(i+1) and waits for it first.
//
// So Resolve(i) never overlaps Resolve(i-1) or Resolve(i+1), and the levels
// below lim leave the front's critical path: they run while the front goes on
// with its rounds.  A worker posts its own follow-up request (Theorem 1 again)
// before it reports its Resolve done, so "every level idle" is observed
// correctly by a scan from lim downwards.
//
// Whoever runs Resolve(i) sees real states of levels i and i+1 only.  Two
// facts stand in for the levels further down: deeper[j] = the number of
// elements in levels >= j (j >= lim; Resolve(i) moves elements between levels
// i and i+1 and drops dead ones, so it changes deeper[i+1] and lowers
// deeper[lim .. i]; a concurrent drop makes the value an upper bound), and
// HeapState::deep_floor, which makes the deepest-level computation (fix_ell)
// count "something below" as a non-empty level.  An upper bound is safe: a
// pivot stays finite (the last Select result) one Resolve longer than needed,
// which only moves elements down that could have stayed; a pivot never
// becomes +infinity while anything lies below it.
//
// Refilling an empty B_0 from the worker levels, which the schedule does not
// cover, is done by the front with every worker idle (it holds all levels and
// runs the one-team code), as are the final statistics.
struct DeepCtl {
  u32 req[MAXL];          // Resolve(i) requests posted
  u32 done[MAXL];         // Resolve(i) finished
  u64 deeper[MAXL + 1];   // elements in levels >= i, for i >= lim
  Lvl L[MAXL];            // states of the worker levels (level lim: also the front's, while worker lim is idle)
  u64 elems;              // heap elements touched by the workers' Resolves
  u64 busy[MAXL];         // clock ticks inside Resolve(i) of worker i (profiled runs)
  int err;                // first error of any team (E_*), 0 if none
  u32 exit;               // set by the front once every worker is idle at the end
  u32 beat;               // the front's round count, published every 1024 rounds (it is alive)
  u32 beat_pad;
};

enum { E_TIMEOUT = -5 };

template <class SP>
PBH_INL u64 lvl_count(SP st, int i) {
  return (u64)st->L[i].nB + st->L[i].nS;
}

// Worker i: one requested Resolve(i).  `sy` is the synchronisation layer
// (device spin waits and fences in the kernel, a deterministic scheduler in
// the CPU tests): wait_idle(t, j) returns once every posted Resolve(j) is done
// (false on an error), post(t, j) / done(t, j) count a request / completion
// after making this team's writes visible, get/put copy level states from /
// to the control block, deeper(t, j) reads deeper[j], account(...) applies a
// Resolve's changes to deeper[] and the element count.
template <class T, class P, class SY>
PBH_INL void deep_step(const T& t, const Geom& g, typename P::SP st, const u64* cur, int i, SY& sy) {
  const bool nx = i + 1 < g.q;
  if (nx && !sy.wait_idle(t, i + 1)) return;
  for (int tries = 0;; ++tries) {
    sy.get(t, st, i);
    if (nx) sy.get(t, st, i + 1);
    const u64 below = i + 2 < g.q ? sy.deeper(t, i + 2) : 0ull;
    if (t.tid() == 0) {
      st->deep_floor = below ? i + 2 : -1;
      fix_ell(st, g.q);
    }
    t.sync();
    if (!nx || room_below(g, st, i)) break;
    if (tries > 2 * MAXL) {
      sy.fail(t, E_INTERNAL);
      return;
    }
    sy.post(t, i + 1);  // an extra Resolve(i+1) makes room
    if (!sy.wait_idle(t, i + 1)) return;
  }
  const u64 c01 = lvl_count(st, i) + (nx ? lvl_count(st, i + 1) : 0ull);
  const u64 c1 = nx ? lvl_count(st, i + 1) : 0ull;
  const u64 e0 = st->elems;
  // worker levels are never in LDS: only the global placement is needed
  if (t.prof && t.tid() == 0) st->prof_res = pbh_clock();
  resolve_t<T, P, typename P::G, typename P::G>(t, g, st, cur, i);
  if (t.prof && t.tid() == 0) st->prof[i] += pbh_clock() - st->prof_res;
  if (st->err) {
    sy.fail(t, st->err);
    return;
  }
  const u64 n01 = lvl_count(st, i) + (nx ? lvl_count(st, i + 1) : 0ull);
  const u64 n1 = nx ? lvl_count(st, i + 1) : 0ull;
  sy.put(t, st, i);
  if (nx) sy.put(t, st, i + 1);
  sy.account(t, i, (long long)n01 - (long long)c01, (long long)n1 - (long long)c1, st->elems - e0,
             t.prof ? st->prof[i] : 0ull);
  if (nx && (st->L[i].cnt & 3u) == 0 && i + 1 <= st->ell) sy.post(t, i + 1);
  sy.done(t, i);
}

// The front's side of the service (levels 0 .. lim-1), handed to the round
// loop.  `sy` null: no workers, every level is the front's.
template <class T, class P, class SY>
struct DeepFront {
  SY* sy;
  int lim;
  bool hold;  // every worker idle and every level held by the front

  // Resolve(lvl) as the front runs it.  Resolve(lim - 1) shares level lim
  // with worker lim: wait until that worker is idle, take level lim's state,
  // make room in it if needed (an extra Resolve(lim) by the worker), and
  // hand the level back afterwards.  (One call of resolve() per kernel: each
  // placement variant of Resolve is instantiated once.)
  PBH_INL void res(const T& t, const Geom& g, typename P::SP st, const u64* cur, int lvl) {
    const bool shared = sy && !hold && lvl == lim - 1;
    u64 c = 0;
    if (shared) {
      if (!take_lim(t, g, st)) return;
      c = lvl_count(st, lim);
    }
    resolve<T, P>(t, g, st, cur, lvl);
    if (shared && !st->err) give_lim(t, g, st, c);
  }

  PBH_INL bool take_lim(const T& t, const Geom& g, typename P::SP st) {
    if (!sy->wait_idle(t, lim)) {
      fail(t, st);
      return false;
    }
    for (int tries = 0;; ++tries) {
      sy->get(t, st, lim);
      const u64 below = lim + 1 < g.q ? sy->deeper(t, lim + 1) : 0ull;
      if (t.tid() == 0) {
        st->deep_floor = below ? lim + 1 : -1;
        fix_ell(st, g.q);
      }
      t.sync();
      if (room_below(g, st, lim - 1)) return true;
      if (tries > 2 * MAXL) {
        sy->fail(t, E_INTERNAL);
        fail(t, st);
        return false;
      }
      sy->post(t, lim);
      if (!sy->wait_idle(t, lim)) {
        fail(t, st);
        return false;
      }
    }
  }

  // After Resolve(lim - 1): level lim (which held c elements) goes back to
  // its worker; the front keeps only the count of the worker levels.
  PBH_INL void give_lim(const T& t, const Geom& g, typename P::SP st, u64 c) {
    const u64 nc = lvl_count(st, lim);
    sy->put(t, st, lim);
    const u64 dn = sy->front_account(t, lim, (long long)nc - (long long)c);
    if (t.tid() == 0) {
      st->L[lim].nB = st->L[lim].nS = 0;
      st->deep_n = dn;
      st->deep_floor = dn ? lim : -1;
      fix_ell(st, g.q);
    }
    t.sync();
  }

  PBH_INL void fail(const T& t, typename P::SP st) {
    t.sync();
    if (t.tid() == 0 && st->err == 0) st->err = sy->error(t);
    t.sync();
  }

  // Every worker idle; the front takes every level's real state.
  PBH_INL bool hold_all(const T& t, const Geom& g, typename P::SP st) {
    for (int j = lim; j < g.q; ++j)
      if (!sy->wait_idle(t, j)) return false;
    for (int j = lim; j < g.q; ++j) sy->get(t, st, j);
    if (t.tid() == 0) {
      st->deep_floor = -1;
      st->deep_n = 0;
      fix_ell(st, g.q);
    }
    t.sync();
    hold = true;
    return true;
  }

  PBH_INL void release_all(const T& t, const Geom& g, typename P::SP st) {
    u64 tot = 0;
    for (int j = g.q - 1; j >= lim; --j) {
      tot += lvl_count(st, j);
      sy->put(t, st, j);
      sy->set_deeper(t, j, tot);
    }
    sy->publish(t);
    if (t.tid() == 0) {
      for (int j = lim; j < g.q; ++j) st->L[j].nB = st->L[j].nS = 0;
      st->deep_n = tot;
      st->deep_floor = tot ? lim : -1;
      fix_ell(st, g.q);
    }
    t.sync();
    hold = false;
  }

  // Resolve(0) and the schedule after an operation (and the refill of B_0).
  // A refill that needs the worker levels makes a second pass with every
  // level held (all workers idle): the one-team refill of drive_with.
  PBH_INL void drive(const T& t, const Geom& g, typename P::SP st, const u64* cur, int sched, int what) {
    if constexpr (!SY::kOn) {
      drive_with(t, g, st, sched, what, [&](int lvl) { resolve<T, P>(t, g, st, cur, lvl); });
    } else {
      int w = what;
      for (int pass = 0; pass < 2; ++pass) {
        bool refill = false;
        drive_with(
            t, g, st, sched, w, [&](int lvl) { res(t, g, st, cur, lvl); }, (sy && !hold) ? lim : MAXL,
            [&](int lvl) { sy->post(t, lvl); }, [&] { refill = true; });
        if (!refill || st->err) break;
        if (!hold_all(t, g, st)) {
          fail(t, st);
          break;
        }
        w = DRIVE_ENSURE;
      }
      if (hold) {
        if (!st->err) release_all(t, g, st);
        hold = false;
      }
    }
  }

  // Every 1024 rounds the front shows it is alive, so that a worker whose
  // level gets no request for a long time can tell that from a stopped front.
  PBH_INL void tick(const T& t, u64 rounds) {
    if constexpr (SY::kOn) {
      if (sy && (rounds & 1023u) == 0) sy->beat(t, (u32)rounds);
    }
  }

  // End of the run: every worker idle, their levels' Resolve counts and
  // element traffic merged into st, then the workers leave.
  PBH_INL void finish(const T& t, const Geom& g, typename P::SP st) {
    if constexpr (SY::kOn) {
      if (!sy) return;
      if (!st->err) {
        if (hold_all(t, g, st)) {
          sy->merge_stats(t, st, lim, g.q);
        } else {
          fail(t, st);
        }
      }
      sy->leave(t);
    }
  }
};

// No workers (every level is the front's).
struct NoDeepSync {
  static constexpr bool kOn = false;
};

// ---------------------------------------------------------------- parDijkstra

PBH_HD inline int bits_for(u32 n) {
  int b = 0;
  while (b < 32 && ((u64)1 << b) < (u64)n) ++b;
  return b < 1 ? 1 : b;
}

// U (relaxation output, n pairs in S) -> sorted by id with one pair per id.
// With rows sorted by target the pairs already are strictly increasing in id
// and nothing is done.  Otherwise each id keeps the pair whose key equals
// dist[id] (the minimum, since dist was lowered by atomicMin) and the rest is
// sorted by id.
template <class T, class A>
PBH_INL u32 intake(const T& t, A S, u32 n, A tmp, A tmp2, const u64* dist, int idbits) {
  if (n < 2) return n;
  bool bad = false;
  for (u32 x = (u32)t.tid() + 1; x < n; x += (u32)T::kNT) bad = bad || S.v[x - 1] >= S.v[x];
  if (!t.any(bad)) return n;
  u32 out = 0;
  for (u32 base = 0; base < n; base += (u32)T::kNT) {
    u32 x = base + (u32)t.tid();
    bool keep = x < n && t.load_cur(dist + S.v[x]) == S.k[x];
    u64 k = x < n ? S.k[x] : 0;
    u32 v = x < n ? S.v[x] : 0;
    u32 tot;
    u32 o = out + t.scan_excl(keep ? 1u : 0u, &tot);
    if (keep) {
      tmp.k[o] = k;
      tmp.v[o] = v;
    }
    out += tot;
  }
  t.sync();
  bool in2 = sort_by_id(t, tmp, tmp2, out, idbits);
  if (in2)
    copy_arr(t, tmp2, S, out);
  else
    copy_arr(t, tmp, S, out);
  return out;
}

// One parDijkstra round (Section 4.1) with level 0 of type A0: extract the
// minimum (key, id) of B_0 -- B_0 holds only live elements, so this is the
// closest unsettled vertex u -- relax all out-edges of u in parallel
// (atomicMin on dist) and compact the improved (dist, v) pairs with a prefix
// sum straight into S_0 (a BulkUpdate of at most d = max out-degree pairs).
// Returns false when the heap is empty.
// LONG: the forms for long rows and a large B_0 in HBM (the plain-rule-only
// kernel, whose registers have room for them; in the kernel that also runs
// speculative rounds they would change the register allocation of those).
template <class T, class P, class A0, bool LONG = false>
PBH_INL bool round_body(const T& t, const Geom& g, typename P::SP st, const u64* off, const u32* tg,
                        const u32* wt, u64* dist, int idbits, u64* relax, u64* upd, u32* order, u64 order_cap,
                        u64 nth) {
  const Lvl a0 = lvl_uni(t, st, 0);
  if (a0.nB == 0) return false;
  A0 B = as_arr<A0>(lbuf(g, 0, a0.bsel));
  // The minimum, U elements per thread in flight; then it is taken out in
  // place: B_0 is sorted by id, so the elements after it, and only those,
  // move down by one (every wavefront has read its elements by then: the
  // team's minimum is a barrier).  B_0 of more than U elements per thread is
  // read again for the move, tile by tile.
  constexpr int U = in_lds<A0>::v ? 4 : 8;
  u64 mk = KINF, k[U];
  u32 mv = VINF, v[U];
  for (u32 base = 0; base < a0.nB; base += (u32)T::kNT * U) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
      k[r] = x < a0.nB ? B.k[x] : KINF;
      v[r] = x < a0.nB ? B.v[x] : VINF;
    }
#pragma unroll
    for (int r = 0; r < U; ++r)
      if (k[r] < mk || (k[r] == mk && v[r] < mv)) {
        mk = k[r];
        mv = v[r];
      }
  }
  t.minkv(mk, mv);
  const u64 e0 = off[mv], e1 = off[mv + 1];
  if (order && nth < order_cap && t.tid() == 0) order[nth] = mv;  // the settle order, when asked for
  if (a0.nB <= (u32)T::kNT * U) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const u32 x = (u32)r * (u32)T::kNT + (u32)t.tid();
      if (x < a0.nB && v[r] > mv) {
        B.k[x - 1] = k[r];
        B.v[x - 1] = v[r];
      }
    }
  } else {
    for (u32 base = 0; base < a0.nB; base += (u32)T::kNT * U) {
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
        k[r] = x < a0.nB ? B.k[x] : KINF;
        v[r] = x < a0.nB ? B.v[x] : 0u;
      }
      t.sync();
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
        if (x < a0.nB && v[r] > mv) {
          B.k[x - 1] = k[r];
          B.v[x - 1] = v[r];
        }
      }
    }
  }
  const u32 n1 = a0.nB - 1;
  A0 T0 = as_arr<A0>(lbuf(g, 0, 2));
  prof_lap(t, st, PROF_EXTRACT);
  A0 S = as_arr<A0>(lbuf(g, 0, 3));
  u32 nu = 0;
  u64 eb = e0;
  // Long rows: four edges per thread per pass, their loads and atomics in
  // flight together (the scans place the improvements in edge order, edge
  // eb + r * NT + tid before those of r + 1).
  constexpr int RE = 4;
  for (; LONG && e1 - eb >= (u64)T::kNT * RE; eb += (u64)T::kNT * RE) {
    u64 cand[RE];
    u32 v[RE];
    bool imp[RE];
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      const u64 e = eb + (u64)r * T::kNT + (u64)t.tid();
      v[r] = tg[e];
      cand[r] = mk + (u64)wt[e];
    }
#pragma unroll
    for (int r = 0; r < RE; ++r) imp[r] = cand[r] < t.atomic_min(dist + v[r], cand[r]);
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      u32 tot;
      const u32 p = t.scan_excl(imp[r] ? 1u : 0u, &tot);
      if (imp[r]) {
        S.k[nu + p] = cand[r];
        S.v[nu + p] = v[r];
      }
      nu += tot;
    }
  }
  for (; eb < e1; eb += (u64)T::kNT) {
    u64 e = eb + (u64)t.tid();
    bool imp = false;
    u64 cand = 0;
    u32 v = 0;
    if (e < e1) {
      v = tg[e];
      cand = mk + (u64)wt[e];
      imp = cand < t.atomic_min(dist + v, cand);
    }
    u32 tot;
    u32 p = t.scan_excl(imp ? 1u : 0u, &tot);
    if (imp) {
      S.k[nu + p] = cand;
      S.v[nu + p] = v;
    }
    nu += tot;
  }
  t.sync();
  prof_lap(t, st, PROF_RELAX);
  nu = intake(t, S, nu, T0, as_arr<A0>(lbuf(g, 0, 4)), dist, idbits);
  if (t.tid() == 0) {
    st->L[0].nB = n1;
    st->L[0].nS = nu;
    st->L[0].ssel = 0;
    st->elems += 3ull * a0.nB + nu;
    if (st->ell < 0 && (n1 + nu) > 0) st->ell = 0;
  }
  t.sync();
  prof_lap(t, st, PROF_INTAKE);
  *relax += e1 - e0;
  *upd += nu;
  return true;
}

// ------------------------------------------------------------ speculative rounds
// A round may extract the k >= 1 smallest live elements of B_0 instead of one
// (the plain rule of Section 4.1 is k = 1).  All out-edges of the k vertices
// are relaxed; any vertex whose distance later improves is re-inserted into the
// heap and relaxed again, so the distances are exact for every choice of k.
// The k of each round comes from a rule: plain, fixed, a given sequence, or a
// small learned model (see mlp_forward).

constexpr int KMAX_ROUND = 256;  // cap on k per round (extracted vertices kept in LDS)
constexpr int TRACE_K = 32;      // key-ordered prefix of B_0 recorded per traced round
constexpr int NFEAT = 8;
constexpr int MLP_H = 64;
// MLP parameters (float32, weights already rounded to bfloat16), in order:
// W1[NFEAT][MLP_H] (input-major), b1[MLP_H], W2[MLP_H][MLP_H] (input-major),
// b2[MLP_H], w3[MLP_H], b3, then the feature normalisation mu[NFEAT],
// sd[NFEAT] and the output scale s (k = 2^(s * y)).
constexpr int MLP_PARAMS = NFEAT * MLP_H + MLP_H + MLP_H * MLP_H + MLP_H + MLP_H + 1;
constexpr int MLP_BLOB = MLP_PARAMS + 2 * NFEAT + 1;

struct SpecCfg {
  int rule;           // 0 plain, 1 fixed, 2 learned, 3 sequence
  u32 kfix, kmax;
  const u32* kseq;
  u32 kseq_len;
  const float* model;  // MLP_BLOB floats (learned rule)
  u64* uk;             // round update list (capacity kmax * d) and a temporary of the same size
  u32* uv;
  u64* tk;
  u32* tv;
  // training traces: every trace_every-th round records NFEAT features and the
  // TRACE_K smallest (key, id) of B_0 in key order
  float* trace_f;
  u64* trace_k;
  u32* trace_v;
  u32 trace_every, trace_cap;
  u32* trace_count;
  u32* trace_q;  // query index of each record
  u32 qid;
  // trial limits: no round starts once the heap's smallest key exceeds
  // stop_key (0 = none) or after max_rounds rounds (0 = none)
  u64 stop_key;
  u32 max_rounds;
  float kscale;  // learned rule: multiplies log2 k
  u32 kevery;    // learned rule: the model runs every kevery-th round (>= 1)
  // LDS room for the round's list after the LDS levels: two buffers of lcap
  // pairs (keys, then ids); 0 = the intake sorts in global memory
  u32 lcap;
  // extracted ids in extraction order (order[j] = the j-th extraction; a
  // round of k > 1 writes its k in id order), first order_cap of them
  u32* order;
  u64 order_cap;
};

struct SsspCounters {
  u64 rounds, relax, updates, extracted;
  u64 last_key;  // smallest key left in the heap when the rounds stopped (KINF: ran empty)
  u32 stopped;   // a trial limit ended the rounds
};

// Smallest key of B_0 (the heap's minimum once B_0 has been refilled).
template <class T, class P>
PBH_INL u64 b0_min_key(const T& t, const Geom& g, typename P::SP st) {
  const Lvl a0 = lvl_load(st, 0);
  Arr Bg = lbuf(g, 0, a0.bsel);
  u64 lo = KINF, hi = 0;
  if (g.qlds > 0) {
    typename P::L B = as_arr<typename P::L>(Bg);
    for (u32 x = (u32)t.tid(); x < a0.nB; x += (u32)T::kNT) lo = B.k[x] < lo ? B.k[x] : lo;
  } else {
    typename P::G B = as_arr<typename P::G>(Bg);
    for (u32 x = (u32)t.tid(); x < a0.nB; x += (u32)T::kNT) lo = B.k[x] < lo ? B.k[x] : lo;
  }
  t.minmax64(lo, hi);
  return lo;
}

struct RoundMemo {  // team-uniform facts about the previous round
  float avgdeg;
  u32 k;          // the last k the learned rule proposed
  bool resident;  // the round's update list is in S_0's array already
};

PBH_INL float flog2p1(float x) { return __builtin_log2f(1.0f + x); }

// The 8 model features, identical in plain and speculative runs: heap size,
// |B_0|, key spread of B_0, the pivots p_0 and p_1 relative to the minimum
// key (a quantile sketch of the queue: the level boundaries), the minimum key
// itself, the mean out-degree of the previous round's vertices, and d.
template <class T, class SP, class A0>
PBH_INL void round_features(const T& t, const Geom& g, SP st, A0 B, u32 nB, const RoundMemo& memo, float* f) {
  u64 lo = KINF, hi = 0;
  for (u32 x = (u32)t.tid(); x < nB; x += (u32)T::kNT) {
    u64 k = B.k[x];
    lo = k < lo ? k : lo;
    hi = k > hi ? k : hi;
  }
  t.minmax64(lo, hi);
  u64 tot = st->deep_n;
#pragma unroll
  for (int i = 0; i < MAXL; ++i) tot += i < g.q ? (u64)st->L[i].nB + st->L[i].nS : 0ull;
  const float spread = (float)(hi - lo);
  f[0] = flog2p1((float)tot);
  f[1] = flog2p1((float)nB);
  f[2] = flog2p1(spread);
  const u64 p0 = st->L[0].pk, p1 = st->L[1].pk;
  f[3] = p0 == KINF ? f[2] + 1.0f : flog2p1((float)(p0 - lo));
  f[4] = (g.q < 2 || p1 == KINF) ? f[3] + 1.0f : flog2p1((float)(p1 - lo));
  f[5] = flog2p1((float)lo) * 0.125f;
  f[6] = flog2p1(memo.avgdeg);
  f[7] = flog2p1((float)g.d);
}

// Rounds a float to bfloat16 (round to nearest even) and back: the model's
// weights are used at BF16 precision with FP32 accumulation.
PBH_INL float bf16r(float x) {
  u32 u = __builtin_bit_cast(u32, x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return __builtin_bit_cast(float, u & 0xFFFF0000u);
}

PBH_INL float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// A thread's share of the model's parameters, read before the features are
// known so that the reads (global memory) run beside that work: the first
// layer's column of this thread's hidden unit, and for teams of >= 256 threads
// its quarter of the second layer's column.
template <class T>
struct MlpRegs {
  static constexpr int kQ = T::kNT >= 256 ? MLP_H / 4 : 1;
  float w1[NFEAT], w2[kQ], b1, b2, w3, mu[NFEAT], sd[NFEAT];
  PBH_INL void load(const T& t, const float* m) {
    const int j = t.tid() & (MLP_H - 1);
    const float* W2 = m + NFEAT * MLP_H + MLP_H;
    const float* B2 = W2 + MLP_H * MLP_H;
    const float* mm = B2 + 2 * MLP_H + 1;
#pragma unroll
    for (int i = 0; i < NFEAT; ++i) {
      w1[i] = m[i * MLP_H + j];
      mu[i] = mm[i];
      sd[i] = mm[NFEAT + i];
    }
    b1 = m[NFEAT * MLP_H + j];
    b2 = B2[j];
    w3 = B2[MLP_H + j];
    if constexpr (T::kNT >= 256) {
      const int qtr = (t.tid() >> 6) & 3;
#pragma unroll
      for (int i = 0; i < kQ; ++i) w2[i] = W2[(qtr * kQ + i) * MLP_H + j];
    }
  }
};

// MLP 8 -> 64 -> 64 -> 1 with GELU (exact, x * Phi(x)); every parameter is
// used rounded to bfloat16, as in training; thread j computes hidden unit j of
// each layer (weights stored input-major, so the loads of
// one input row are contiguous), the output is reduced through LDS.  BF16
// weights, FP32 accumulation.  Returns y (k = 2^(s * y)).
template <class T>
PBH_INL float mlp_forward(const T& t, const float* m, const float* f, const MlpRegs<T>& r) {
  const float* W1 = m;
  const float* b1 = W1 + NFEAT * MLP_H;
  const float* W2 = b1 + MLP_H;
  const float* b2 = W2 + MLP_H * MLP_H;
  const float* w3 = b2 + MLP_H;
  const float* b3 = w3 + MLP_H;
  const float* sd = b3 + 1 + NFEAT;
  float x[NFEAT];
#pragma unroll
  for (int i = 0; i < NFEAT; ++i) x[i] = (f[i] - r.mu[i]) / r.sd[i];
  if constexpr (T::kNT >= MLP_H) {
    if (t.tid() < MLP_H) {
      float a = bf16r(r.b1);
#pragma unroll
      for (int i = 0; i < NFEAT; ++i) a += bf16r(r.w1[i]) * x[i];
      t.sh->mlp_h[t.tid()] = gelu(a);
    }
  } else {
    for (int j = t.tid(); j < MLP_H; j += T::kNT) {
      float a = bf16r(b1[j]);
#pragma unroll
      for (int i = 0; i < NFEAT; ++i) a += bf16r(W1[i * MLP_H + j]) * x[i];
      t.sh->mlp_h[j] = gelu(a);
    }
  }
  t.sync();
  if constexpr (T::kNT >= 256) {
    // four threads per hidden unit, each summing a quarter of the inputs
    if (t.tid() < 4 * MLP_H) {
      const int qtr = t.tid() >> 6;
      float a = 0.0f;
#pragma unroll
      for (int i = 0; i < MLP_H / 4; ++i) a += bf16r(r.w2[i]) * t.sh->mlp_h[qtr * (MLP_H / 4) + i];
      t.sh->mlp_p[t.tid()] = a;
    }
    t.sync();
    if (t.tid() < MLP_H) {
      float a = bf16r(r.b2);
      for (int q = 0; q < 4; ++q) a += t.sh->mlp_p[q * MLP_H + t.tid()];
      t.sh->mlp_z[t.tid()] = bf16r(r.w3) * gelu(a);
    }
  } else {
    for (int j = t.tid(); j < MLP_H; j += T::kNT) {
      float a = bf16r(b2[j]);
#pragma unroll 16
      for (int i = 0; i < MLP_H; ++i) a += bf16r(W2[i * MLP_H + j]) * t.sh->mlp_h[i];
      t.sh->mlp_z[j] = bf16r(w3[j]) * gelu(a);
    }
  }
  t.sync();
  float y = bf16r(b3[0]);
  if constexpr (T::kNT >= 64) {
    // every wavefront sums the 64 output terms with a butterfly of lane
    // exchanges (the same order in every lane), instead of each thread
    // reading all 64 from LDS one after another
    static_assert(MLP_H == 64, "one output term per lane");
    float z = t.sh->mlp_z[t.lane()];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) z += t.wave_xor(z, o);
    y += z;
  } else {
    for (int j = 0; j < MLP_H; ++j) y += t.sh->mlp_z[j];
  }
  t.sync();
  return y * sd[NFEAT];
}

template <class T, class SP, class A0>
PBH_INL u32 propose_k(const T& t, const Geom& g, SP st, const SpecCfg& sc, A0 B, u32 nB, u64 round,
                      RoundMemo& memo) {
  u32 k = 1;
  if (sc.rule == 1) {
    k = sc.kfix;
  } else if (sc.rule == 3) {
    k = sc.kseq[round % sc.kseq_len];
  } else if (sc.rule == 2 && sc.kevery > 1 && round % sc.kevery != 0) {
    k = memo.k;  // between model runs the last proposal stands
  } else if (sc.rule == 2) {
    float f[NFEAT];
    MlpRegs<T> r;
    r.load(t, sc.model);
    round_features(t, g, st, B, nB, memo, f);
    float y = mlp_forward(t, sc.model, f, r) * sc.kscale;
    // fall back to the plain rule on anything that is not a finite number
    if (y == y && y > -64.0f && y < 64.0f) {
      float kk = __builtin_exp2f(y);
      k = kk < 1.0f ? 1u : (kk > (float)sc.kmax ? sc.kmax : (u32)(kk + 0.5f));
    }
  }
  k = k < 1 ? 1 : k;
  k = k > sc.kmax ? sc.kmax : k;
  k = k > (u32)KMAX_ROUND ? (u32)KMAX_ROUND : k;
  memo.k = k;
  return k;
}

// Records one training trace: features and the TRACE_K smallest (key, id) of
// B_0 in key order (by repeated team minima; traced rounds are sparse).
template <class T, class SP, class A0>
PBH_INL void record_trace(const T& t, const Geom& g, SP st, const SpecCfg& sc, A0 B, u32 nB,
                          const RoundMemo& memo) {
  float f[NFEAT];
  round_features(t, g, st, B, nB, memo, f);
  u32 slot = 0;
  if (t.tid() == 0) slot = t.atomic_add32(sc.trace_count, 1u);
  slot = t.sum(slot);
  if (slot >= sc.trace_cap) return;
  if (t.tid() == 0) {
    for (int i = 0; i < NFEAT; ++i) sc.trace_f[(u64)slot * NFEAT + i] = f[i];
    if (sc.trace_q) sc.trace_q[slot] = sc.qid;
  }
  u64 lastk = 0;
  u32 lastv = 0;
  bool have = false;
  for (int r = 0; r < TRACE_K; ++r) {
    u64 bk = KINF;
    u32 bv = VINF;
    for (u32 x = (u32)t.tid(); x < nB; x += (u32)T::kNT) {
      u64 k = B.k[x];
      u32 v = B.v[x];
      bool after = !have || k > lastk || (k == lastk && v > lastv);
      if (after && (k < bk || (k == bk && v < bv))) {
        bk = k;
        bv = v;
      }
    }
    t.minkv(bk, bv);
    if (t.tid() == 0) {
      sc.trace_k[(u64)slot * TRACE_K + r] = bk;
      sc.trace_v[(u64)slot * TRACE_K + r] = bv;
    }
    lastk = bk;
    lastv = bv;
    have = true;
  }
  t.sync();
}

// The pairs of U (n of them, global) whose key equals dist[id], to W.  Each
// pair of a round's list lowered its distance (atomicMin returned a larger
// one), and later pairs of that id are smaller still, so exactly one pair per
// id is left: the sorted list needs no further pass for duplicates.
template <class T, class GA, class AW>
PBH_INL u32 filter_live(const T& t, GA U, u32 n, AW W, const u64* dist) {
  u32 out = 0;
  constexpr int RE = 4;  // elements per thread per pass, loads issued together
  for (u32 base = 0; base < n; base += (u32)T::kNT * RE) {
    u64 k[RE], c[RE];
    u32 v[RE];
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
      k[r] = x < n ? U.k[x] : 0;
      v[r] = x < n ? U.v[x] : 0;
    }
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      const u32 x = base + (u32)r * (u32)T::kNT + (u32)t.tid();
      c[r] = x < n ? t.load_cur(dist + v[r]) : ~k[r];
    }
    u32 cnt = 0;
#pragma unroll
    for (int r = 0; r < RE; ++r) cnt += c[r] == k[r] ? 1u : 0u;
    u32 tot;
    u32 o = out + t.scan_excl(cnt, &tot);
#pragma unroll
    for (int r = 0; r < RE; ++r)
      if (c[r] == k[r]) {
        W.k[o] = k[r];
        W.v[o] = v[r];
        ++o;
      }
    out += tot;
  }
  t.sync();
  return out;
}

// Round update list U (n pairs, global) -> one pair per id, sorted by id, in U
// (W: scratch of the same size).
template <class T, class GA>
PBH_INL u32 intake_list(const T& t, GA U, u32 n, GA W, const u64* dist, int idbits) {
  const u32 out = filter_live(t, U, n, W, dist);
  if (!sort_by_id(t, W, U, out, idbits)) copy_arr(t, W, U, out);
  return out;
}

// Sorts n <= RUNS * kW pairs of L1 by id into D (L2: scratch).  Each
// wavefront sorts runs of one element per lane in registers; an element's
// place is its place in its run plus, from a search in every other run, the
// elements there that come before it.  Two barriers in all, where the radix
// sort takes about six per 8-bit digit and 256 elements (256 pairs of 20-bit
// ids, 256 threads: about 1 us against 3).  Beyond RUNS runs the searches cost
// more than the radix passes.
constexpr u32 RUNS = 8;
template <class T, class LA, class AD>
PBH_INL void sort_runs(const T& t, LA L1, LA L2, u32 n, AD D) {
  constexpr u32 W = (u32)T::kW;
  constexpr int Q = (int)((RUNS + T::kNW - 1) / T::kNW);  // runs per wavefront
  u64 k[Q];
  u32 v[Q], rank[Q];
  const u32 nr = (n + W - 1) / W;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const u32 run = (u32)q * T::kNW + (u32)t.wave();
    if (run >= nr) continue;
    const u32 x = run * W + (u32)t.lane();
    const u64 kk = x < n ? L1.k[x] : 0ull;
    u32 from;
    v[q] = x < n ? L1.v[x] : VINF;
    t.wave_sort(v[q], from);
    k[q] = t.lane_get64(kk, from);
    L2.v[x] = v[q];
  }
  t.sync();
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const u32 run = (u32)q * T::kNW + (u32)t.wave();
    if (run >= nr) continue;
    rank[q] = 0;
#pragma unroll 4
    for (u32 c = 0; c < nr; ++c) {
      // the elements of run c below v (or equal, in an earlier run); all runs
      // hold W entries, the last one padded with VINF
      const u32 lim = c < run ? v[q] : v[q] - 1u;
      u32 lo = 0;
      if constexpr (W == 64) {
#pragma unroll
        for (u32 h = 16; h; h /= 4)
          lo += h * ((L2.v[c * W + lo + h - 1] <= lim ? 1u : 0u) + (L2.v[c * W + lo + 2 * h - 1] <= lim ? 1u : 0u) +
                     (L2.v[c * W + lo + 3 * h - 1] <= lim ? 1u : 0u));
      }
      lo += L2.v[c * W + lo] <= lim ? 1u : 0u;
      lo = c > run && v[q] == 0u ? 0u : lo;
      rank[q] += c == run ? (u32)t.lane() : lo;
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const u32 run = (u32)q * T::kNW + (u32)t.wave();
    if (run >= nr || v[q] == VINF) continue;
    D.k[rank[q]] = k[q];
    D.v[rank[q]] = v[q];
  }
  t.sync();
}

// The round's final pairs (n of them in L1, one per id; L1 and L2 hold lcap),
// sorted by id, to D.
template <class T, class LA, class AD>
PBH_INL void intake_sorted(const T& t, LA L1, LA L2, u32 lcap, u32 n, AD D, int idbits) {
  constexpr u32 W = (u32)T::kW;
  if (n <= RUNS * W && (n + W - 1) / W * W <= lcap)
    sort_runs(t, L1, L2, n, D);
  else if (sort_by_id(t, L1, L2, n, idbits))
    copy_arr(t, L2, D, n);
  else
    copy_arr(t, L1, D, n);
}

// One speculative round: extract the `k` smallest of B_0, relax every out-edge
// of them, collect the improved (dist, v) pairs in the global list U.
template <class T, class P, class A0>
PBH_INL bool round_spec(const T& t, const Geom& g, typename P::SP st, const u64* off, const u32* tg,
                        const u32* wt, u64* dist, int idbits, u32 k, const SpecCfg& sc, SsspCounters* c,
                        RoundMemo* memo, u32* ulen) {
  using G = typename P::G;
  const Lvl a0 = lvl_uni(t, st, 0);
  if (a0.nB == 0) return false;
  A0 B = as_arr<A0>(lbuf(g, 0, a0.bsel));
  const u32 take = k < a0.nB ? k : a0.nB;
  KV thr = take == a0.nB ? kv_inf() : select_kth(t, B, a0.nB, take);
  u32 n0, n1, n2;
  A0 X = as_arr<A0>(lbuf(g, 0, 2));
  partition3(t, B, a0.nB, thr, kv_inf(), X, as_arr<A0>(lbuf(g, 0, a0.bsel ^ 1)), X, &n0, &n1, &n2);
  if (sc.order)
    for (u32 j = (u32)t.tid(); j < take; j += (u32)T::kNT)
      if (c->extracted + j < sc.order_cap) sc.order[c->extracted + j] = X.v[j];
  prof_lap(t, st, PROF_EXTRACT);
  // the extracted vertices' rows: first edge and prefix sums of the out-degrees
  u32 E = 0, maxdeg = 0;
  for (u32 base = 0; base < take; base += (u32)T::kNT) {
    u32 j = base + (u32)t.tid();
    u64 e0 = 0, e1 = 0;
    if (j < take) {
      u32 v = X.v[j];
      e0 = off[v];
      e1 = off[v + 1];
      t.sh->ex0[j] = e0;
    }
    u32 tot;
    u32 p = E + t.scan_excl((u32)(e1 - e0), &tot);
    if (j < take) t.sh->exd[j] = p;
    E += tot;
    maxdeg = (u32)(e1 - e0) > maxdeg ? (u32)(e1 - e0) : maxdeg;
  }
  maxdeg = t.wave_max32(maxdeg);
  if (t.tid() == 0) t.sh->exd[take] = E;
  if constexpr (T::kNW > 1) {
    if (t.lane() == 0) t.sh->wv[t.wave()] = maxdeg;
  }
  t.sync();
  if constexpr (T::kNW > 1) {
#pragma unroll
    for (int w = 0; w < T::kNW; ++w) maxdeg = t.sh->wv[w] > maxdeg ? t.sh->wv[w] : maxdeg;
    maxdeg = t.uni(maxdeg);
  }
  // Which edge is whose.  With even degrees, by groups: 2^gl lanes (the mean
  // degree, rounded up) scan a vertex's edges in `per` steps; a row is a block
  // of vertices at one step, and two LDS reads give a thread its edge.  Where
  // that would leave more than a third of the threads without one (measured on
  // degrees around 24: slower than searching), an edge's vertex is the largest
  // j with exd[j] <= e.  The edges are then taken kW at a time by a wavefront:
  // the vertex of every kW-th edge is found first (one search per thread), and
  // an edge's own search runs over the few vertices of its wavefront's edges.
  u32 gl = 2;
  while (gl < 6 && ((u64)take << gl) < E) ++gl;
  if ((u32)T::kNT < 64u) gl = 0;
  const u32 per = (maxdeg + (1u << gl) - 1) >> gl, vpr = (u32)T::kNT >> gl;
  const u64 grows = (u64)((take + vpr - 1) / vpr) * per;
  const bool groups = 2ull * grows * T::kNT <= 3ull * E + 2ull * T::kNT;
  auto owner = [&](u32 e, u32 lo, u32 hi) -> u32 {
    while (hi - lo > 1) {
      const u32 mid = (lo + hi) >> 1;
      if (t.sh->exd[mid] <= e)
        lo = mid;
      else
        hi = mid;
    }
    return lo;
  };
  const u32 nch = (E + (u32)T::kW - 1) / (u32)T::kW;
  const u32 rows = groups ? (u32)grows : (E + (u32)T::kNT - 1) / (u32)T::kNT;
  const bool marked = !groups && T::kW > 1 && nch < 256u;
  if (marked) {
    for (u32 c = (u32)t.tid(); c <= nch; c += (u32)T::kNT)
      t.sh->hist[c] = owner(c * (u32)T::kW < E ? c * (u32)T::kW : E - 1, 0, take);
    t.sync();
  }
  G U{(decltype(G::k))sc.uk, (decltype(G::v))sc.uv};
  // the LDS after the levels, two lists of lcap pairs
  using L = typename P::L;
  unsigned char* lb = reinterpret_cast<unsigned char*>(g.lk) + lvl_off(g.d, g.qlds) * 12ull;
  L L1, L2;
  L1.k = (decltype(L1.k))reinterpret_cast<u64*>(lb);
  L2.k = (decltype(L2.k))reinterpret_cast<u64*>(lb + (u64)sc.lcap * 8u);
  L1.v = (decltype(L1.v))reinterpret_cast<u32*>(lb + (u64)sc.lcap * 16u);
  L2.v = (decltype(L2.v))reinterpret_cast<u32*>(lb + (u64)sc.lcap * 20u);
  u32 nu = 0, nl = 0;  // improved pairs in U / final pairs in L1
  // RE rows per pass: their CSR loads and atomics are all in flight before any
  // result is waited for; one scan places the improvements.
  constexpr int RE = 8;
  u32 blk = 0, stp = 0;  // block of vertices and step of the next row (groups)
  for (u32 rb = 0; rb < rows; rb += RE) {
    u64 cand[RE];
    u32 v[RE], w[RE];
    bool imp[RE];
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      imp[r] = false;
      cand[r] = 0;
      v[r] = w[r] = 0;
      if (rb + (u32)r >= rows) continue;
      u32 lo = 0, at;
      bool in;
      if (groups) {
        const u32 j = blk * vpr + ((u32)t.tid() >> gl);
        lo = j < take ? j : take - 1;
        at = (stp << gl) + ((u32)t.tid() & ((1u << gl) - 1u));
        in = j < take && at < t.sh->exd[lo + 1] - t.sh->exd[lo];
        if (++stp == per) {
          stp = 0;
          ++blk;
        }
      } else {
        const u32 e = (rb + (u32)r) * (u32)T::kNT + (u32)t.tid();
        u32 hi = take;
        in = e < E;
        if (marked) {
          const u32 c = (rb + (u32)r) * T::kNW + t.uni((u32)t.wave());
          if (c < nch) {
            lo = t.uni(t.sh->hist[c]);
            hi = t.uni(t.sh->hist[c + 1]) + 1u;
          }
        }
        lo = owner(in ? e : E - 1, lo, hi);
        at = e - t.sh->exd[lo];
      }
      const u64 ei = in ? t.sh->ex0[lo] + at : 0ull;
      imp[r] = in;  // (a thread without an edge reads the graph's first one)
      v[r] = tg[ei];
      w[r] = wt[ei];
      cand[r] = X.k[lo];
    }
    // Most edges improve nothing.  In a round of one pass the distances are
    // looked at first, and atomics go out only for what may improve them
    // (distances only fall: an old value lets a needless atomic through, no
    // more): ring of 100,003, 900 edges a round, 5.8 -> 4.9 us.  In larger
    // rounds a compute unit's time is the number of lines it asks for, which
    // the look would add to: 6,000 scattered edges, 31 us without, 34 with it.
    u64 now[RE];
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      now[r] = KINF;
      if (rows <= (u32)RE && (u32)r < rows) now[r] = t.load_cur(dist + v[r]);
    }
    u32 cnt = 0;
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      if (rb + (u32)r >= rows) continue;
      cand[r] += (u64)w[r];
      imp[r] = imp[r] && cand[r] < now[r];
    }
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      if (rb + (u32)r >= rows) continue;
      if (imp[r]) imp[r] = cand[r] < t.atomic_min(dist + v[r], cand[r]);
      cnt += imp[r] ? 1u : 0u;
    }
    u32 tot;
    if (sc.lcap != 0 && rows <= (u32)RE) {
      // The round's only pass: once every edge is relaxed (the barrier), a
      // pair whose key is the distance is final, so the filter works on the
      // registers and the list goes straight to LDS; U, its way through global
      // memory and its reads are left out.
      t.sync();
      prof_lap(t, st, PROF_RELAX);
      u64 c[RE];
#pragma unroll
      for (int r = 0; r < RE; ++r) c[r] = imp[r] ? t.load_cur(dist + v[r]) : 0ull;
      cnt = 0;
#pragma unroll
      for (int r = 0; r < RE; ++r) {
        imp[r] = imp[r] && c[r] == cand[r];
        cnt += imp[r] ? 1u : 0u;
      }
      u32 p = t.scan_excl(cnt, &tot);
      if (tot <= sc.lcap) {
#pragma unroll
        for (int r = 0; r < RE; ++r)
          if (imp[r]) {
            L1.k[p] = cand[r];
            L1.v[p] = v[r];
            ++p;
          }
        nl = tot;
        break;
      }
      cnt = 0;
#pragma unroll
      for (int r = 0; r < RE; ++r) cnt += imp[r] ? 1u : 0u;
    }
    u32 p = nu + t.scan_excl(cnt, &tot);
#pragma unroll
    for (int r = 0; r < RE; ++r)
      if (imp[r]) {
        U.k[p] = cand[r];
        U.v[p] = v[r];
        ++p;
      }
    nu += tot;
  }
  t.sync();
  prof_lap(t, st, PROF_RELAX);
  memo->resident = false;
  if (nu != 0 && sc.lcap != 0 && nu <= sc.lcap) nl = filter_live(t, U, nu, L1, dist);
  if (nl != 0 || nu == 0) {
    // the list is in the LDS after the levels: sort it there; if it is one
    // piece it goes to S_0's (empty) array at once
    nu = nl;
    memo->resident = nu <= g.d;
    if (memo->resident)
      intake_sorted(t, L1, L2, sc.lcap, nu, as_arr<A0>(lbuf(g, 0, 3)), idbits);
    else
      intake_sorted(t, L1, L2, sc.lcap, nu, U, idbits);
  } else {
    G Wt{(decltype(G::k))sc.tk, (decltype(G::v))sc.tv};
    nu = intake_list(t, U, nu, Wt, dist, idbits);
  }
  if (t.tid() == 0) {
    st->L[0].bsel = a0.bsel ^ 1;
    st->L[0].nB = n1;
    st->elems += 3ull * a0.nB + 3ull * nu;
    if (st->ell < 0 && n1 > 0) st->ell = 0;
  }
  t.sync();
  prof_lap(t, st, PROF_INTAKE);
  c->relax += E;
  c->updates += nu;
  c->extracted += take;
  memo->avgdeg = (float)E / (float)take;
  *ulen = nu;
  return true;
}

// parDijkstra: rounds until the heap is empty.  The extraction and the bulk
// update of a round share one Resolve(0) and the schedule: between them S_0 is
// empty and B_0 keeps at least d elements, so Algorithm 1's preconditions hold.
// Speculative rounds bulk-update their list U in pieces of at most d, each
// piece an operation followed by Resolve(0) and the schedule.
struct NoHook {
  template <class SP>
  PBH_INL void operator()(const Geom&, SP, const SsspCounters&) const {}
};

// `hook` sees the heap after every operation's Resolve schedule (the CPU
// tests use it to check invariants; the kernels pass NoHook).
// With `sy` (and lim < q), levels >= lim are resolved by their own workers
// (the deep-level service above).
// SPEC false: the plain rule only (one extraction per round, no traces) --
// the speculative rounds, the model and the update pieces are left out of
// the code, which lightens the kernel of plain runs.
template <class T, class P, class Hook = NoHook, class SY = NoDeepSync, bool SPEC = true>
PBH_INL void sssp_rounds(const T& t, const Geom& g, typename P::SP st, const u64* off, const u32* tg,
                         const u32* wt, u64* dist, u32 n, u32 src, int sched, const SpecCfg& sc, SsspCounters* cnt,
                         const Hook& hook = Hook(), SY* sy = nullptr, int lim = MAXL) {
  using G = typename P::G;
  DeepFront<T, P, SY> fr{sy, lim, false};
  const int idbits = bits_for(n);
  if (t.tid() == 0) {
    Arr S = lbuf(g, 0, 3);
    if (g.qlds > 0) {
      typename P::L s = as_arr<typename P::L>(S);
      s.k[0] = 0;
      s.v[0] = src;
    } else {
      typename P::G s = as_arr<typename P::G>(S);
      s.k[0] = 0;
      s.v[0] = src;
    }
    st->L[0].nS = 1;
    st->L[0].ssel = 0;
    st->ell = 0;
    st->prof_last = pbh_clock();
  }
  t.sync();
  SsspCounters c{0, 0, 1, 0, KINF, 0};
  RoundMemo memo{0.0f, 1u, false};
  u32 upos = 0, ulen = 0;
  for (;;) {
    // Resolve(0) and the schedule after the previous operation (the source's
    // insertion, a round's bulk update or a piece of it), then make sure B_0
    // holds the minimum if the heap is not empty.
    fr.drive(t, g, st, dist, sched, DRIVE_AFTER | DRIVE_ENSURE);
    prof_lap(t, st, PROF_DRIVE);
    if (st->err) break;
    hook(g, st, c);
    if (SPEC && upos < ulen) {  // next piece of the round's bulk update
      u32 len = ulen - upos < g.d ? ulen - upos : g.d;
      G U{(decltype(G::k))sc.uk, (decltype(G::v))sc.uv};
      if (memo.resident) {
        // nothing to move
      } else if (g.qlds > 0) {
        typename P::L S = as_arr<typename P::L>(lbuf(g, 0, 3));
        for (u32 x = (u32)t.tid(); x < len; x += (u32)T::kNT) {
          S.k[x] = U.k[upos + x];
          S.v[x] = U.v[upos + x];
        }
      } else {
        G S = as_arr<G>(lbuf(g, 0, 3));
        for (u32 x = (u32)t.tid(); x < len; x += (u32)T::kNT) {
          S.k[x] = U.k[upos + x];
          S.v[x] = U.v[upos + x];
        }
      }
      t.sync();
      if (t.tid() == 0) {
        st->L[0].nS = len;
        st->L[0].ssel = 0;
        if (st->ell < 0) st->ell = 0;
      }
      t.sync();
      prof_lap(t, st, PROF_PIECE);
      upos += len;
      continue;
    }
    if (sc.max_rounds || sc.stop_key) {
      const u64 mn = b0_min_key<T, P>(t, g, st);
      if ((sc.max_rounds && c.rounds >= sc.max_rounds) || (sc.stop_key && mn != KINF && mn > sc.stop_key)) {
        c.last_key = mn;
        c.stopped = 1;
        break;
      }
    }
    // Every extraction consumes one insertion and every insertion comes from
    // one scanned edge (or the source), so rounds <= 1 + relax always holds.
    if (c.rounds > c.relax + 1) {
      if (t.tid() == 0) st->err = E_INTERNAL;
      t.sync();
      break;
    }
    prof_lap(t, st, PROF_OTHER);
    bool more;
    if (!SPEC || (sc.rule == 0 && !sc.trace_f)) {
      more = g.qlds > 0
                 ? round_body<T, P, typename P::L, !SPEC>(t, g, st, off, tg, wt, dist, idbits, &c.relax, &c.updates,
                                                          sc.order, sc.order_cap, c.extracted)
                 : round_body<T, P, typename P::G, !SPEC>(t, g, st, off, tg, wt, dist, idbits, &c.relax, &c.updates,
                                                          sc.order, sc.order_cap, c.extracted);
      c.extracted += more ? 1 : 0;
    } else if constexpr (SPEC) {
      const Lvl a0 = lvl_load(st, 0);
      Arr Bg = lbuf(g, 0, a0.bsel);
      u32 k;
      if (g.qlds > 0) {
        typename P::L B = as_arr<typename P::L>(Bg);
        if (sc.trace_f && a0.nB && c.rounds % sc.trace_every == 0) record_trace(t, g, st, sc, B, a0.nB, memo);
        k = propose_k(t, g, st, sc, B, a0.nB, c.rounds, memo);
        prof_lap(t, st, PROF_PROPOSE);
        more = round_spec<T, P, typename P::L>(t, g, st, off, tg, wt, dist, idbits, k, sc, &c, &memo, &ulen);
      } else {
        G B = as_arr<G>(Bg);
        if (sc.trace_f && a0.nB && c.rounds % sc.trace_every == 0) record_trace(t, g, st, sc, B, a0.nB, memo);
        k = propose_k(t, g, st, sc, B, a0.nB, c.rounds, memo);
        prof_lap(t, st, PROF_PROPOSE);
        more = round_spec<T, P, G>(t, g, st, off, tg, wt, dist, idbits, k, sc, &c, &memo, &ulen);
      }
      upos = 0;
    }
    fr.tick(t, c.rounds);
    if (!more) {
      // B_0 is empty only once the heap is (the refill above guarantees it).
      if (st->ell >= 0) {
        t.sync();
        if (t.tid() == 0) st->err = E_INTERNAL;
        t.sync();
      }
      break;
    }
    ++c.rounds;
  }
  fr.finish(t, g, st);
  *cnt = c;
}

// ---------------------------------------------------------------- pbh_* calls
struct PbhParams {
  Geom g;
  HeapState* gst;  // heap state in device memory, loaded into LDS per kernel
  u64* cur;        // current key of every id
  u32* bitmap;     // one bit per id, all zero between calls
  u32 nwords;
  u32 id_cap;
  int sched;
  int idbits;
  // bulk update
  const u64* keys;
  const u32* ids;
  u64 count;
  u64* ukeys;  // compacted update list
  u32* uids;
  // extract
  u64 k;
  u64* okeys;
  u32* oids;
};

// Could the next operation push elements out of the deepest allocated level?
// Then the caller adds a level first (growing the arena keeps the offsets of
// the existing levels).
template <class SP>
PBH_INL bool need_grow(const Geom& g, SP st) {
  const int q = g.q;
  u64 have = (u64)st->L[q - 1].nB + st->L[q - 1].nS;
  u64 in = (q == 1) ? (u64)g.d : capB(g.d, q - 2) + capS(g.d, q - 2);
  return have + in > nomB(g.d, q - 1);
}

// BulkUpdate of one call.  First pass: cur[id] = min(cur[id], key) with
// atomicMin (duplicates in the batch: the smallest key wins), ids whose key
// dropped are marked in a bitmap; compacting the bitmap gives the changed ids
// in increasing id order with their new keys, i.e. U sorted by value as
// Section 2.2 requires.  Then pieces of at most d go into S_0, each followed
// by Resolve(0) and the schedule.  Resumable: st->aux[0] = list length,
// aux[1] = list built, aux[3] = stopped because a level must be added,
// progress = list position reached.  All levels are in HBM (type P::G).
template <class T, class P>
PBH_INL void pbh_update_body(const T& t, const Geom& g, typename P::SP st, const PbhParams& p) {
  using G = typename P::G;
  if (st->aux[1] == 0) {
    u32 newly = 0;
    for (u64 x = (u64)t.tid(); x < p.count; x += (u64)T::kNT) {
      u32 id = p.ids[x];
      u64 k = p.keys[x];
      u64 old = t.atomic_min(p.cur + id, k);
      if (k < old) {
        t.atomic_or32(p.bitmap + (id >> 5), 1u << (id & 31));
        newly += (old == KINF);
      }
    }
    newly = t.sum(newly);
    t.fence();
    t.sync();
    u64 nu = 0;
    for (u32 wb = 0; wb < p.nwords; wb += (u32)T::kNT) {
      u32 w = wb + (u32)t.tid();
      u32 bits = 0;
      if (w < p.nwords) {
        bits = t.load32(p.bitmap + w);
        if (bits) p.bitmap[w] = 0u;
      }
      u32 tot;
      u64 o = nu + t.scan_excl((u32)__builtin_popcount(bits), &tot);
      while (bits) {
        u32 b = (u32)__builtin_ctz(bits);
        bits &= bits - 1;
        u32 id = w * 32u + b;
        p.uids[o] = id;
        p.ukeys[o] = t.load_cur(p.cur + id);
        ++o;
      }
      nu += tot;
    }
    t.sync();
    if (t.tid() == 0) {
      st->aux[0] = nu;
      st->aux[1] = 1;
      st->live += newly;
      st->progress = 0;
    }
    t.sync();
  }
  const u64 nu = st->aux[0];
  if (t.tid() == 0) st->aux[3] = 0;
  t.sync();
  for (u64 c0 = st->progress; c0 < nu;) {
    if (need_grow(g, st)) {
      if (t.tid() == 0) st->aux[3] = 1;
      t.sync();
      break;
    }
    u32 len = (u32)((nu - c0) < g.d ? (nu - c0) : g.d);
    G S = as_arr<G>(lbuf(g, 0, 3));
    for (u32 x = (u32)t.tid(); x < len; x += (u32)T::kNT) {
      S.k[x] = p.ukeys[c0 + x];
      S.v[x] = p.uids[c0 + x];
    }
    t.sync();
    if (t.tid() == 0) {
      st->L[0].nS = len;
      st->L[0].ssel = 0;
      if (st->ell < 0) st->ell = 0;
      st->elems += 2ull * len;
    }
    t.sync();
    drive<T, P>(t, g, st, p.cur, p.sched, DRIVE_AFTER);
    if (st->err) break;
    c0 += len;
    if (t.tid() == 0) st->progress = c0;
    t.sync();
  }
}

// Delete(e) of one call (Section 1.2) for a batch of ids (absent ids: no-op).
// The paper sends a DEL priority down the levels that removes the matching
// elements when they meet in a merge.  Here the id's current key is set to
// "absent" (KINF) instead: every merge and every move into B_0 already drops
// copies whose key is not the current one (the duplicate reading used for
// updates), so copies in deeper levels leave when they next meet a merge or
// move up.  B_0 must hold only live elements, so it is filtered at once; then
// Resolve(0) and the schedule run, as after any operation.  Resumable like
// the update: aux[1] = ids marked and B_0 filtered, aux[3] = stopped because a
// level must be added.
template <class T, class P>
PBH_INL void pbh_delete_body(const T& t, const Geom& g, typename P::SP st, const PbhParams& p) {
  using G = typename P::G;
  if (st->aux[1] == 0) {
    u32 gone = 0;
    for (u64 x = (u64)t.tid(); x < p.count; x += (u64)T::kNT)
      gone += t.atomic_exch(p.cur + p.ids[x], KINF) != KINF ? 1u : 0u;
    gone = t.sum(gone);
    t.fence();
    t.sync();
    const Lvl a0 = lvl_load(st, 0);
    u32 n0 = 0, n1 = 0, n2 = 0;
    if (a0.nB) {
      G B = as_arr<G>(lbuf(g, 0, a0.bsel)), O = as_arr<G>(lbuf(g, 0, a0.bsel ^ 1)), X = as_arr<G>(lbuf(g, 0, 2));
      partition3(t, B, a0.nB, kv_inf(), kv_inf(), O, X, X, &n0, &n1, &n2, p.cur);
    }
    if (t.tid() == 0) {
      if (a0.nB) {
        st->L[0].bsel = a0.bsel ^ 1;
        st->L[0].nB = n0;
        st->elems += (u64)a0.nB + n0;
      }
      st->live -= gone;
      st->aux[1] = 1;
      fix_ell(st, g.q);
    }
    t.sync();
  }
  if (t.tid() == 0) st->aux[3] = 0;
  t.sync();
  if (need_grow(g, st)) {
    if (t.tid() == 0) st->aux[3] = 1;
    t.sync();
    return;
  }
  drive<T, P>(t, g, st, p.cur, p.sched, DRIVE_AFTER);
}

// Batched ExtractMin of one call: repeatedly take the smallest min(k_left,
// |B_0|) elements of B_0 (B_0 <= p_0 < everything else, and B_0 holds only
// live elements), output them sorted by (key, id), mark their ids absent, then
// Resolve(0) and the schedule.  Resumable: progress = elements written,
// aux[2] = an extraction awaits its Resolve(0), aux[3] = stopped for growth,
// aux[4] = heap ran empty.
template <class T, class P>
PBH_INL void pbh_extract_body(const T& t, const Geom& g, typename P::SP st, const PbhParams& p) {
  using G = typename P::G;
  if (t.tid() == 0) {
    st->aux[3] = 0;
    st->aux[4] = 0;
  }
  t.sync();
  for (;;) {
    const bool pending = st->aux[2] != 0;  // the last extraction still needs its Resolve(0)
    const u64 outpos = st->progress;
    if (!pending && outpos >= p.k) break;
    if (need_grow(g, st)) {
      if (t.tid() == 0) st->aux[3] = 1;
      t.sync();
      break;
    }
    drive<T, P>(t, g, st, p.cur, p.sched, (pending ? DRIVE_AFTER : 0) | (outpos < p.k ? DRIVE_ENSURE : 0));
    if (t.tid() == 0) st->aux[2] = 0;
    t.sync();
    if (st->err || outpos >= p.k) break;
    const Lvl a0 = lvl_load(st, 0);
    if (a0.nB == 0) {
      t.sync();
      if (t.tid() == 0) {
        if (st->ell >= 0)
          st->err = E_INTERNAL;  // the refill leaves B_0 empty only when the heap is
        else
          st->aux[4] = 1;
      }
      t.sync();
      break;
    }
    u32 take = (u32)((p.k - outpos) < a0.nB ? (p.k - outpos) : a0.nB);
    G B = as_arr<G>(lbuf(g, 0, a0.bsel));
    KV thr = (take == a0.nB) ? kv_inf() : select_kth(t, B, a0.nB, take);
    u32 n0, n1, n2;
    G X = as_arr<G>(lbuf(g, 0, 2));
    partition3(t, B, a0.nB, thr, kv_inf(), X, as_arr<G>(lbuf(g, 0, a0.bsel ^ 1)), X, &n0, &n1, &n2);
    G R = sort_kv(t, X, B, take, p.idbits) ? B : X;
    for (u32 x = (u32)t.tid(); x < take; x += (u32)T::kNT) {
      u32 id = R.v[x];
      p.okeys[outpos + x] = R.k[x];
      p.oids[outpos + x] = id;
      t.store_cur(p.cur + id, KINF);
    }
    t.fence();
    t.sync();
    if (t.tid() == 0) {
      st->L[0].bsel ^= 1;
      st->L[0].nB = n1;
      st->live -= take;
      st->progress = outpos + take;
      st->elems += 6ull * a0.nB;
      st->aux[2] = 1;
    }
    t.sync();
  }
}

}  // namespace bkt
