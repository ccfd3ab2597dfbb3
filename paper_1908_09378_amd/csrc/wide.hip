// Device-wide engine of the parallel bucket heap (see wide.h).
//
// Kernels (256 threads per workgroup, tiles of 2048 elements):
//   k_merge<false> / k_merge<true>
//       Merge of two id-sorted arrays with DeleteDuplicates (Section 2.1):
//       a counting pass (which also finds each tile's merge-path split
//       points and, where Resolve asks for it, counts the outputs <= a pivot)
//       and a writing pass; in both each thread walks 8 consecutive merge
//       positions from one merge-path search in LDS, and the writing pass
//       stores its outputs through an LDS transpose and notes their key range
//       (the start of Select).
//   k_part<false> / k_part<true>
//       Stable three-way split by two (key, id) pivots.
//   A counting pass adds its counts up as its workgroups end, 64 of them at a
//   time; a writing pass's workgroup sums what is before its tile itself.
//   k_sel_pass / k_sel_collect
//       Select: radix selection on the 96-bit (key, id) value, 8 bits per
//       pass from the first bit where the keys differ, until a few thousand
//       candidates remain; those are gathered, and the last workgroup of the
//       gather finishes among them.  The split that follows reads the result
//       on the device, so Select and split are one host step.
//   k_intake / k_bits<false> / k_bits<true>
//       BulkUpdate intake: atomicMin on the current keys, a mark byte per id
//       whose key dropped, and their compaction into U sorted by id.
//   k_rank, k_tsort / k_smerge
//       Sorting the extracted minima by (key, id): a few thousand by each
//       one's rank among all; more by tiles sorted in registers and LDS
//       (per-thread sort, then merge-path rounds), then merge passes.  The
//       kernel that writes them out also marks their ids absent.
//   k_delete
//       Marks deleted ids absent.
// The few results the host needs after a step are written into host-mapped
// memory as soon as they are known; the host goes on while the step's writing
// pass runs.
#include "wide.h"

#include <algorithm>
#include <chrono>
#include <cstddef>
#include <cstring>
#include <vector>

#include "pbh_team.h"

namespace bkt {
namespace {

using u8 = unsigned char;

constexpr int NT = 256;
constexpr int WE = 8;
constexpr u32 TILE = NT * WE;  // 2048
constexpr int SEL_BITS = 8;
constexpr int SEL_BINS = 1 << SEL_BITS;
constexpr int GRID_STRIDE = 2048;        // workgroups of the grid-stride kernels
constexpr int ST = 1024;                 // threads of the Select kernels
constexpr int GRID_SEL = 256;            // their workgroups: one per compute unit (each flushes its
                                         // histogram by atomics, about 10 ns a cache line)
constexpr u32 CANDMAX = 8192;            // candidates, finished in LDS (32,768 read from memory by the
                                         // last workgroup: 50 us more; another pass is at most 18)
constexpr u32 RANKED = 256;              // the last candidates, ranked by counting

// Device-side state of a selection (read and written by the Select kernels).
struct SelState {
  u64 pk;   // prefix: the leading nb bits of (key, id) fixed so far
  u32 pv;
  int nb;
  u32 rank; // rank still sought among the elements with that prefix
  u32 cnt;  // elements with that prefix
  int done; // few enough candidates: gather them
  int bad;  // no bin held the rank (never expected)
};
struct Ctl {
  SelState q;    // before the passes now running
  u32 sncand;
  u32 collected; // workgroups finished with the gather (the last one goes on)
  alignas(128) u32 shist[2][SEL_BINS];  // of the two passes
};

// What the host reads of a selection.  The Select kernels write it in device
// memory (the split reads it there) and then into host-mapped coherent memory,
// the step's sequence number last, which the host polls.
struct Mail {
  u64 rk;       // selected element
  u32 rv;
  int sfail;    // the selection needs more passes
  int sbad;     // the selection found no element of the rank (never expected)
  u32 npass;    // Select passes of the step that did work (the others returned at once)
  u32 seq;      // number of the last step published (host copy only)
};

__device__ __forceinline__ u64 atomic_min64(u64* p, u64 v) {
  return __hip_atomic_fetch_min((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 atomic_max64(u64* p, u64 v) {
  return __hip_atomic_fetch_max((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u32 atomic_add32(u32* p, u32 v) {
  return __hip_atomic_fetch_add((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Agent-scope atomic loads and stores: coherent across the XCDs' L2 caches
// within a launch, for words that workgroups of one launch hand to each
// other (a plain store can stay in one XCD's L2 until the kernel ends).
__device__ __forceinline__ u32 ld_a32(const u32* p) {
  return __hip_atomic_load((const u32 PBH_GLB*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 ld_a64(const u64* p) {
  return __hip_atomic_load((const u64 PBH_GLB*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_a32(u32* p, u32 v) {
  __hip_atomic_store((u32 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_a64(u64* p, u64 v) {
  __hip_atomic_store((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive scan over the workgroup (NTH threads); *total = the sum.
// sw: LDS scratch of NTH/64 words.
template <int NTH>
__device__ __forceinline__ u32 block_scan(u32 x, u32* total, u32* sw) {
  u32 inc = wave_incl(x);
  const int w = (int)(threadIdx.x >> 6);
  if ((threadIdx.x & 63) == 63) sw[w] = inc;
  __syncthreads();
  u32 pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < NTH / 64; ++k) {
    u32 s = sw[k];
    pre += k < w ? s : 0u;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + inc - x;
}
template <int NTH>
__device__ __forceinline__ u32 block_sum(u32 x, u32* sw) {
  u32 t;
  block_scan<NTH>(x, &t, sw);
  return t;
}
template <int NTH>
__device__ __forceinline__ void block_minmax(u64& lo, u64& hi, u64* swl, u64* swh) {
  wave_minmax64(lo, hi);
  const int w = (int)(threadIdx.x >> 6);
  if ((threadIdx.x & 63) == 0) {
    swl[w] = lo;
    swh[w] = hi;
  }
  __syncthreads();
  lo = swl[0];
  hi = swh[0];
#pragma unroll
  for (int k = 1; k < NTH / 64; ++k) {
    lo = swl[k] < lo ? swl[k] : lo;
    hi = swh[k] > hi ? swh[k] : hi;
  }
  __syncthreads();
}

// ------------------------------------------------------------------ counts
//
// A counting pass's workgroups leave their tiles' counts in memory and add
// them up in passing, per 64 tiles; the last of each 64 has their sums and
// posts them to the host.  A workgroup of the writing pass sums the counts
// before its tile itself, by one or two loads per lane of one wavefront.  (A
// scan kernel between the passes took 3 to 9 us and two gaps between
// launches.  One pass that counts and writes, each tile waiting for the counts
// of the tiles before it, was slower: 91-110 us for a merge of 8.4 million
// elements and 131 us for a split, 66-84 and 66 us in two passes, because
// every tile then waits with its LDS and registers held; and the host learns
// the sizes only at its end.)

__device__ __forceinline__ u64 atomic_add64(u64* p, u64 v) {
  return __hip_atomic_fetch_add((u64 PBH_GLB*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Up to three counts of 64 workgroups in one word: F fields of 57 / F bits,
// and above them how many of the workgroups have added theirs.
template <int F>
struct Field {
  static constexpr u32 bits = 57u / F;
  static constexpr u64 mask = (1ull << bits) - 1;
};
constexpr u64 ARRIVED = 1ull << 57;
constexpr u32 LINE = 16;  // words of 8 bytes in a cache line

// The end of workgroup t of nt, by one thread: the last of its 64 leaves their
// packed sums in gs[t / 64] (when set), where the writing pass reads them, and
// posts the full word to the host, which adds the groups up (one more stage on
// the device, over the groups' sums, took 3.7 us).  Atomics on one cache line
// take about 10 ns each, so each word has a line of its own.
__device__ __forceinline__ void arrive(u64* acc, u64* gs, u64* post, u32 t, u32 nt, u64 counts) {
  const u32 g = t >> 6;
  u64* w = acc + (u64)LINE * g;
  const u64 a = atomic_add64(w, ARRIVED + counts) + ARRIVED + counts;
  if ((u32)(a >> 57) != min(64u, nt - (g << 6))) return;
  st_a64(w, 0ull);
  if (gs) gs[g] = a & (ARRIVED - 1);
  __hip_atomic_store(post + g, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Key range of a merge's outputs, per 64 tiles: the writing pass's workgroups
// widen their group's by atomics.  (One range for all: 4096 workgroups took
// twice as long for it.)  A line each.
struct alignas(128) Range {
  u64 lo, hi;
};

// What a counting pass leaves and a writing pass reads.
struct Pass {
  u32* tc;     // tile counts, one array of `stride` per output stream
  u32 stride;
  u64* gs;     // sums of 64 tiles, packed
  u64* acc;    // arrival words, a line each
  u64* post;   // host-mapped: a word per 64 tiles
};
// The outputs before tile t in stream f of F, by one wavefront.
template <int F>
__device__ __forceinline__ u32 before_tile(const Pass& ps, u32 f, u32 t) {
  const u32 lane = threadIdx.x & 63u, g = t >> 6;
  u32 x = lane < (t & 63u) ? ps.tc[(u64)f * ps.stride + (g << 6) + lane] : 0u;
  for (u32 y = lane; y < g; y += 64u) x += (u32)((ps.gs[y] >> (f * Field<F>::bits)) & Field<F>::mask);
  return __builtin_amdgcn_readlane(wave_incl(x), 63);
}
// How many of the first `diag` elements of merge(A, B) come from A; ties go
// to A first.  ById compares ids, otherwise (key, id).
template <bool BYKV, class KP, class VP>
__device__ __forceinline__ u32 mpath(KP ak, VP av, u32 na, KP bk, VP bv, u32 nb, u32 diag) {
  u32 lo = diag > nb ? diag - nb : 0u, hi = diag < na ? diag : na;
  while (lo < hi) {
    u32 mid = (lo + hi) >> 1, jb = diag - 1 - mid;
    bool afirst;
    if constexpr (BYKV) {
      u64 ka = ak[mid], kb = bk[jb];
      afirst = ka < kb || (ka == kb && av[mid] <= bv[jb]);
    } else {
      afirst = av[mid] <= bv[jb];
    }
    if (afirst)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// The same split as mpath, found by one wavefront: each round every lane
// tests one of 64 evenly spaced probes and the ballot's popcount (the tests
// are true on a prefix) narrows the range 65-fold, so a split of arrays of
// millions costs about four dependent global loads instead of twenty-odd.
// All 64 lanes must call it with the same arguments.
template <bool BYKV, class KP, class VP>
__device__ __forceinline__ u32 mpath_wave(KP ak, VP av, u32 na, KP bk, VP bv, u32 nb, u32 diag) {
  const u32 lane = threadIdx.x & 63u;
  u32 lo = diag > nb ? diag - nb : 0u, hi = diag < na ? diag : na;
  while (lo < hi) {
    const u32 len = hi - lo;
    const bool small = len <= 64u;
    const u32 mid = small ? lo + lane : lo + (u32)(((u64)(lane + 1) * len) / 65u);
    bool afirst = false;
    if (!small || lane < len) {
      const u32 jb = diag - 1 - mid;
      if constexpr (BYKV) {
        const u64 ka = ak[mid], kb = bk[jb];
        afirst = ka < kb || (ka == kb && av[mid] <= bv[jb]);
      } else {
        afirst = av[mid] <= bv[jb];
      }
    }
    const u32 c = (u32)__popcll(__ballot(afirst));
    if (small) return lo + c;
    if (c == 0) {
      hi = lo + (u32)(len / 65u);
    } else {
      const u32 nlo = lo + (u32)(((u64)c * len) / 65u) + 1u;
      if (c < 64u) hi = lo + (u32)(((u64)(c + 1) * len) / 65u);
      lo = nlo;
    }
  }
  return lo;
}

// ------------------------------------------------------------------ merge by id

struct MArgs {
  const u64* ak;
  const u32* av;
  u32 na;
  const u64* bk;
  const u32* bv;
  u32 nb;
  u64* ck;
  u32* cv;
  const u64* cur;  // liveness for PREFER_LIVE (may be null)
  int prefer;
  Range* range;    // where the outputs' key range goes (may be null)
  u64 pk;          // outputs <= (pk, pv) are counted
  u32 pv;
};

// One tile of merge(A, B) by id with DeleteDuplicates: the outputs at merge
// positions [t*TILE, (t+1)*TILE), whose inputs are A[i0, i1) and B[j0, j1)
// (staged in LDS: ids, and keys in the writing pass).  Each thread takes WE
// consecutive merge positions: one merge-path search in LDS finds where they
// start, then a sequential walk merges them (ties: A first), so a copy of an
// id present in both inputs sits right after A's copy.  The pair is decided
// at A's slot and B's slot is dropped; a partner just outside the
// tile is A[i0-1] or B[j1].  Counting pass: the tile's kept outputs; with KEYS
// it also stages the keys and counts the outputs <= (pk, pv), which Resolve's
// EMPTY step needs before the writing pass.  Writing pass: a scan of the
// threads' kept counts gives each output its place in the tile's output
// range; the outputs are transposed through LDS (reusing the input staging,
// at index o + o/8 so that the threads' runs of WE spread over the banks) and
// stored coalesced.  Stored straight from the walk, each store instruction
// would touch 64 cache lines (a thread's outputs are consecutive), which
// measured 1.6x slower.  The key range goes into the group's Range by atomics,
// of which nearly all are spared by a look at the range so far.
template <bool WRITE, bool KEYS = WRITE>
__global__ __launch_bounds__(NT) void k_merge(MArgs a, u32* part, Pass ps) {
  static_assert(KEYS || !WRITE, "the writing pass stages keys");
  constexpr u32 NONE = 0xFFFFFFFFu;  // exhausted input (ids are < 2^32 - 1)
  constexpr u32 PAD = WRITE ? TILE / 8 : 0;  // room for the transposed index o + o/8
  __shared__ u32 sv[TILE + PAD];
  __shared__ u64 sk[KEYS ? TILE + PAD : 1];
  __shared__ u32 sw[NT / 64];
  __shared__ u32 s_base;
  __shared__ u64 swl[NT / 64], swh[NT / 64];
  const u32 t = blockIdx.x, total = a.na + a.nb;
  const u32 d0 = t * TILE, d1 = min(d0 + TILE, total);
  u32 i0, i1;
  if constexpr (!WRITE) {
    // The counting pass finds its tile's split points itself (wavefronts 0
    // and 1, one 65-way search each) and records them for the writing pass.
    __shared__ u32 ssplit[2];
    const u32 wv = threadIdx.x >> 6;
    if (wv < 2) {
      const u64 dg = (u64)(t + wv) * TILE;
      const u32 diag = (u32)(dg < total ? dg : total);
      const u32 i = mpath_wave<false>((const u64*)nullptr, a.av, a.na, (const u64*)nullptr, a.bv, a.nb, diag);
      if ((threadIdx.x & 63u) == 0) ssplit[wv] = i;
    }
    __syncthreads();
    i0 = ssplit[0];
    i1 = ssplit[1];
    if (threadIdx.x == 0) {
      part[t] = i0;
      if (t + 1 == gridDim.x) part[t + 1] = i1;
    }
  } else {
    i0 = part[t];
    i1 = part[t + 1];
    if (threadIdx.x < 64) {
      const u32 b = before_tile<2>(ps, 0, t);
      if (threadIdx.x == 0) s_base = b;
    }
  }
  const u32 j0 = d0 - i0, j1 = d1 - i1;
  const u32 nA = i1 - i0, nT = d1 - d0, nB = nT - nA;
  {
    u64 lk[WE];
    u32 lv[WE];
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      const u32 x = threadIdx.x + (u32)q * NT;
      const bool fromA = x < nA;
      const u32 g = fromA ? i0 + x : j0 + (x - nA);
      lv[q] = 0;
      lk[q] = 0;
      if (x < nT) {
        lv[q] = fromA ? a.av[g] : a.bv[g];
        if constexpr (KEYS) lk[q] = fromA ? a.ak[g] : a.bk[g];
      }
    }
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      const u32 x = threadIdx.x + (u32)q * NT;
      if (x < nT) {
        sv[x] = lv[q];
        if constexpr (KEYS) sk[x] = lk[q];
      }
    }
  }
  const bool hasPrev = i0 > 0, hasNext = j1 < a.nb;
  const u32 aprev = hasPrev ? a.av[i0 - 1] : 0u, bnext = hasNext ? a.bv[j1] : 0u;
  __syncthreads();
  const u32* sA = sv;
  const u32* sB = sv + nA;
  const u32 p0 = min((u32)threadIdx.x * WE, nT), p1 = min(p0 + WE, nT);
  u32 i = mpath<false>((const u64*)nullptr, sA, nA, (const u64*)nullptr, sB, nB, p0);
  u32 j = p0 - i;
  u32 va = i < nA ? sA[i] : NONE, vb = j < nB ? sB[j] : NONE;
  bool havePrevA = i > 0 || hasPrev;
  u32 prevA = i > 0 ? sA[i - 1] : aprev;
  u64 ko[WE];
  u32 vo[WE];
  u32 keep = 0, pair = 0, ia[WE];  // pairs of copies, and A's index of each
#pragma unroll
  for (int q = 0; q < WE; ++q) {
    ko[q] = 0;
    vo[q] = 0;
    ia[q] = i;
    if (p0 + (u32)q >= p1) continue;
    bool kp = true;
    if (va <= vb) {  // A's element (first on equal ids)
      const u32 v = va;
      const bool dup = j < nB ? vb == v : (hasNext && bnext == v);
      pair |= (u32)dup << q;
      vo[q] = v;
      ko[q] = KEYS ? sk[i] : 0ull;
      prevA = v;
      havePrevA = true;
      ++i;
      va = i < nA ? sA[i] : NONE;
    } else {  // B's element: dropped when A holds the id
      const u32 v = vb;
      const u64 k = KEYS ? sk[nA + j] : 0ull;
      kp = !(havePrevA && prevA == v);
      vo[q] = v;
      ko[q] = k;
      ++j;
      vb = j < nB ? sB[j] : NONE;
    }
    keep |= (u32)kp << q;
  }
  // The copy kept of each pair, all of the thread's pairs at once: one wait for
  // their keys and one for the current keys, where deciding each in the walk
  // cost two per pair (updates of a million keys that all have a copy:
  // writing pass 44.2 -> 39.8 us, counting pass 39.0 -> 35.0).
  if (pair && (a.prefer == PREFER_LIVE || (KEYS && a.prefer == PREFER_B))) {
    const bool by_cur = a.prefer == PREFER_LIVE && a.cur;
    u64 ka[WE], kb[WE], c[WE];
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      const u32 jb = p0 + (u32)q - ia[q];  // (B's copy may be the next tile's first)
      ka[q] = ko[q];
      kb[q] = 0;
      if ((pair >> q) & 1u) {
        if (!KEYS) ka[q] = a.ak[i0 + ia[q]];
        kb[q] = KEYS && jb < nB ? sk[nA + jb] : a.bk[j0 + jb];
      }
    }
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      c[q] = 0;
      if (by_cur && ((pair >> q) & 1u) && ka[q] != kb[q]) c[q] = a.cur[vo[q]];
    }
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      if (!((pair >> q) & 1u) || ka[q] == kb[q]) continue;
      const bool second = a.prefer == PREFER_B || (by_cur ? kb[q] == c[q] : kb[q] < ka[q]);
      ko[q] = second ? kb[q] : ka[q];
      if (by_cur && !second && ka[q] != c[q]) keep &= ~(1u << q);
    }
  }
  const u32 nk = (u32)__builtin_popcount(keep);
  if constexpr (!WRITE) {
    u32 nle = 0;
    if constexpr (KEYS) {
#pragma unroll
      for (int q = 0; q < WE; ++q) nle += ((keep >> q) & 1u) && kv_le(KV{ko[q], vo[q]}, KV{a.pk, a.pv});
    }
    const u32 tot = block_sum<NT>(nk | (nle << 16), sw);  // (a tile's counts fit 16 bits)
    if (threadIdx.x == 0) {
      const u32 kept = tot & 0xFFFFu;
      ps.tc[t] = kept;
      if (a.range && (t & 63u) == 0) a.range[t >> 6] = Range{KINF, 0};  // (for the writing pass)
      arrive(ps.acc, ps.gs, ps.post, t, gridDim.x, kept | ((u64)(tot >> 16) << Field<2>::bits));
    }
  } else {
    u32 tot;
    u32 o = block_scan<NT>(nk, &tot, sw);  // its barriers also end every walk's reads of sv / sk
    u64 lo = KINF, hi = 0;
#pragma unroll
    for (int q = 0; q < WE; ++q)
      if ((keep >> q) & 1u) {
        const u32 z = o + (o >> 3);
        sk[z] = ko[q];
        sv[z] = vo[q];
        ++o;
        lo = ko[q] < lo ? ko[q] : lo;
        hi = ko[q] > hi ? ko[q] : hi;
      }
    block_minmax<NT>(lo, hi, swl, swh);  // (its barriers also order the transpose)
    if (a.range && threadIdx.x == 0 && tot != 0) {
      Range* r = a.range + (t >> 6);
      const u64 clo = ld_a64(&r->lo), chi = ld_a64(&r->hi);
      if (lo < clo) atomic_min64(&r->lo, lo);
      if (hi > chi) atomic_max64(&r->hi, hi);
    }
    const u32 base = s_base;
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      const u32 x = threadIdx.x + (u32)q * NT;
      if (x < tot) {
        const u32 z = x + (x >> 3);
        a.ck[base + x] = sk[z];
        a.cv[base + x] = sv[z];
      }
    }
  }
}

// ------------------------------------------------------------------ three-way split

struct PArgs {
  const u64* k;
  const u32* v;
  u32 n;
  u64 p1k;
  u32 p1v;
  u64 p2k;
  u32 p2v;
  const u64* live;  // class-0 elements whose key is not live[id] are dropped
  u64* ok[3];
  u32* ov[3];
  // When set, the first pivot is min(the element Select published in this
  // box, (p1k, p1v)), and a failed Select (sfail / sbad) splits nothing.
  const Mail* sel;
};

// The first pivot: (p1k, p1v), or its minimum with the Select result; false:
// the Select failed, nothing is split.  (The arguments stay untouched: a
// modified copy of them, indexed by class, would live in scratch memory.)
__device__ __forceinline__ bool part_pivot(const PArgs& a, KV* p1) {
  *p1 = KV{a.p1k, a.p1v};
  if (!a.sel) return true;
  if (a.sel->sfail || a.sel->sbad) return false;
  const KV s{a.sel->rk, a.sel->rv};
  if (kv_less(s, *p1)) *p1 = s;
  return true;
}

__device__ __forceinline__ u32 pclass(const PArgs& a, KV p1, u64 k, u32 v) {
  KV e{k, v};
  u32 c = kv_le(e, p1) ? 0u : (kv_le(e, KV{a.p2k, a.p2v}) ? 1u : 2u);
  if (c == 0 && a.live && a.live[v] != k) c = 3;
  return c;
}

// Tile t = elements [t*TILE, (t+1)*TILE) in WE rounds of NT consecutive
// elements, so that each round's outputs are written in runs.  A ballot per
// class counts a wavefront's elements of a round; the tile's 32 counts (8
// rounds x 4 wavefronts, in order) are scanned by each wavefront, lane for
// lane, and three wavefronts sum what is before the tile, one per class.
// The counting pass reads the ids only where they decide.
template <bool WRITE>
__global__ __launch_bounds__(NT) void k_part(PArgs a, Pass ps) {
  constexpr int NW = NT / 64;
  static_assert(NW * WE <= 64, "one lane per round and wavefront");
  const u32 t = blockIdx.x;
  const u32 wv = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  KV p1;
  const u32 n = part_pivot(a, &p1) ? a.n : 0u;  // a failed Select: every element counts as dropped
  const u64 base = (u64)t * TILE;
  u64 kk[WE];
#pragma unroll
  for (int r = 0; r < WE; ++r) {
    const u64 x = base + (u64)r * NT + threadIdx.x;
    kk[r] = x < n ? a.k[x] : 0;
  }
  if constexpr (!WRITE) {
    __shared__ u32 sw[NT / 64];
    u32 c01 = 0, c2 = 0;
#pragma unroll
    for (int r = 0; r < WE; ++r) {
      const u64 x = base + (u64)r * NT + threadIdx.x;
      if (x >= n) continue;
      const u64 k = kk[r];
      const bool ids = k == p1.k || k == a.p2k || (a.live && k < p1.k);
      const u32 c = pclass(a, p1, k, ids ? a.v[x] : 0u);
      c01 += c == 0 ? 1u : (c == 1 ? 1u << 16 : 0u);
      c2 += c == 2;
    }
    c01 = block_sum<NT>(c01, sw);
    c2 = block_sum<NT>(c2, sw);
    if (threadIdx.x == 0) {
      const u32 c0 = c01 & 0xFFFFu, c1 = c01 >> 16;
      ps.tc[t] = c0;
      ps.tc[ps.stride + t] = c1;
      ps.tc[2 * ps.stride + t] = c2;
      arrive(ps.acc, ps.gs, ps.post, t, gridDim.x,
             c0 | ((u64)c1 << Field<3>::bits) | ((u64)c2 << (2 * Field<3>::bits)));
    }
  } else {
    __shared__ u32 s01[64], s2[64], s_base[3];
    u32 vv[WE], cls = 0, rank[WE];  // class, and place within the wavefront's round
#pragma unroll
    for (int r = 0; r < WE; ++r) {
      const u64 x = base + (u64)r * NT + threadIdx.x;
      vv[r] = x < n ? a.v[x] : 0;
    }
    if (wv < 3) {
      const u32 b = before_tile<3>(ps, wv, t);
      if (lane == 0) s_base[wv] = b;
    }
#pragma unroll
    for (int r = 0; r < WE; ++r) {
      const u64 x = base + (u64)r * NT + threadIdx.x;
      const u32 c = x < n ? pclass(a, p1, kk[r], vv[r]) : 3u;
      const u64 b0 = __ballot(c == 0), b1 = __ballot(c == 1), b2 = __ballot(c == 2);
      const u64 b = c == 0 ? b0 : (c == 1 ? b1 : b2);
      cls |= c << (2 * r);
      rank[r] = __builtin_amdgcn_mbcnt_hi((u32)(b >> 32), __builtin_amdgcn_mbcnt_lo((u32)b, 0u));
      if (lane == 0) {
        s01[r * NW + (int)wv] = (u32)__popcll(b0) | ((u32)__popcll(b1) << 16);
        s2[r * NW + (int)wv] = (u32)__popcll(b2);
      }
    }
    __syncthreads();
    const u32 m01 = lane < NW * WE ? s01[lane] : 0u, m2 = lane < NW * WE ? s2[lane] : 0u;
    const u32 e01 = wave_incl(m01) - m01, e2 = wave_incl(m2) - m2;
#pragma unroll
    for (int r = 0; r < WE; ++r) {
      const int l = r * NW + (int)__builtin_amdgcn_readfirstlane(wv);
      const u32 f01 = __builtin_amdgcn_readlane(e01, l), f2 = __builtin_amdgcn_readlane(e2, l);
      const u32 c = (cls >> (2 * r)) & 3u;
      if (c < 3) {
        const u32 pos = s_base[c] + rank[r] + (c == 0 ? f01 & 0xFFFFu : (c == 1 ? f01 >> 16 : f2));
        u64* ok = c == 0 ? a.ok[0] : (c == 1 ? a.ok[1] : a.ok[2]);
        u32* ov = c == 0 ? a.ov[0] : (c == 1 ? a.ov[1] : a.ov[2]);
        ok[pos] = kk[r];
        ov[pos] = vv[r];
      }
    }
  }
}

// ------------------------------------------------------------------ Select

__device__ __forceinline__ bool sel_match(u64 k, u32 v, u64 pk, u32 pv, int nb) {
  if (nb == 0) return true;
  if (nb <= 64) return (k >> (64 - nb)) == (pk >> (64 - nb));
  if (k != pk) return false;
  const int r = nb - 64;
  return (v >> (32 - r)) == (pv >> (32 - r));
}
// Bits [p, p + w) of the 96-bit value key * 2^32 + id.
__device__ __forceinline__ u32 sel_digit(u64 k, u32 v, int p, int w) {
  const u32 mask = (1u << w) - 1u;
  if (p >= 32) return (u32)(k >> (p - 32)) & mask;
  return (u32)(((k << 32) | v) >> p) & mask;
}

// Is this workgroup the last of the launch to get here?  Each thread first
// waits for its own memory operations (its atomics have then been performed),
// then one counter increment per workgroup; the last one sees gridDim.x - 1
// and resets the counter for the next launch.
__device__ __forceinline__ bool last_workgroup(u32* ctr, int* s_last) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    const u32 prev = __hip_atomic_fetch_add((u32 PBH_GLB*)ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_last = prev == gridDim.x - 1;
    if (*s_last) st_a32(ctr, 0u);
  }
  __syncthreads();
  return *s_last != 0;
}

// The Select kernels' state is worked out by every wavefront for itself: a
// barrier of 16 wavefronts costs about 0.4 us, and a gather that passed the
// state through LDS had some twenty of them.

// The start of a selection of rank r among n elements whose keys lie in the
// given ranges: the bits the keys share are the prefix.
__device__ __forceinline__ SelState sel_start(const Range* range, u32 nrange, u32 r, u32 n) {
  u64 lo = KINF, hi = 0;
  for (u32 x = threadIdx.x & 63u; x < nrange; x += 64u) {
    lo = range[x].lo < lo ? range[x].lo : lo;
    hi = range[x].hi > hi ? range[x].hi : hi;
  }
  wave_minmax64(lo, hi);
  SelState q;
  if (lo == hi) {
    q.nb = 64;
    q.pk = lo;
  } else {
    q.nb = __builtin_clzll(lo ^ hi);
    q.pk = q.nb ? (lo >> (64 - q.nb)) << (64 - q.nb) : 0ull;
  }
  q.pv = 0;
  q.rank = r;
  q.cnt = n;
  q.done = n <= CANDMAX;
  q.bad = 0;
  return q;
}
__device__ __forceinline__ int sel_width(const SelState& q) { return 96 - q.nb < SEL_BITS ? 96 - q.nb : SEL_BITS; }

// The state after a pass over q's elements that counted h[b] of them in bin b
// (four bins per lane): the bin that holds the rank goes into the prefix.
template <class H>
__device__ __forceinline__ SelState sel_pick(SelState q, H h, u32 limit) {
  static_assert(SEL_BINS == 256, "four bins per lane");
  const int w = sel_width(q), p = 96 - q.nb - w;
  const u32 lane = threadIdx.x & 63u;
  u32 c[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = h[4 * lane + j];
  const u32 sum = c[0] + c[1] + c[2] + c[3], inc = wave_incl(sum);
  const u64 m = __ballot(inc >= q.rank);
  if (q.rank == 0 || m == 0) {
    q.done = q.bad = 1;
    return q;
  }
  const int l = __builtin_ctzll(m);
  u32 b = 0, before = 0, cnt = 0, run = __builtin_amdgcn_readlane(inc - sum, l);
  bool found = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const u32 x = __builtin_amdgcn_readlane(c[j], l);
    if (!found && q.rank <= run + x) {
      b = 4u * (u32)l + (u32)j;
      before = run;
      cnt = x;
      found = true;
    }
    run += x;
  }
  if (p >= 32) {
    q.pk |= (u64)b << (p - 32);
  } else {
    u64 lo = ((q.pk & 0xFFFFFFFFull) << 32) | q.pv;
    lo |= (u64)b << p;
    q.pk = (q.pk & 0xFFFFFFFF00000000ull) | (lo >> 32);
    q.pv = (u32)lo;
  }
  q.nb += w;
  q.rank -= before;
  q.cnt = cnt;
  q.done = cnt <= limit || q.nb == 96;
  return q;
}

// The state after `passes` passes of this step.  Every wavefront works it out
// from the histograms (a pass whose last workgroup did so took 4 us more).
__device__ __forceinline__ SelState sel_after(const Ctl* c, SelState q, int passes, u32* npass) {
  *npass = 0;
  for (int p = 0; p < passes && !q.done; ++p) {
    q = sel_pick(q, &c->shist[p][0], CANDMAX);
    *npass += 1;
  }
  return q;
}

// One radix pass of Select (rank r among A[0, n)), number `pass` of its step:
// every workgroup histograms its share of the elements that match the prefix
// fixed so far (in four copies in LDS, then one atomic per non-empty bin).
// The first pass of a selection (nrange != 0) derives the starting prefix from
// the key range; the others read the state before the step.  A pass returns at
// once when the selection is done.  Bound by the read of the keys: 8 loads of
// 8 bytes in flight per thread and 16 wavefronts per compute unit (8.4 million
// keys: 17 us; with 4 loads and 8 wavefronts, 29).
__global__ __launch_bounds__(ST) void k_sel_pass(const u64* K, const u32* V, u32 n, Ctl* c, u32 r, int pass,
                                                 const Range* range, u32 nrange) {
  constexpr int CP = 4;
  __shared__ u32 h[CP][SEL_BINS];
  SelState q;
  if (nrange) {
    q = sel_start(range, nrange, r, n);
    if (blockIdx.x == 0 && threadIdx.x == 0) c->q = q;
  } else {
    u32 np;
    q = sel_after(c, c->q, pass, &np);
  }
  if (q.done) return;
  const int w = sel_width(q), p = 96 - q.nb - w;
  // the ids take part only once the prefix or this pass's digit reaches
  // them; until then the pass reads the keys alone
  const bool needv = q.nb > 64 || p < 32;
  for (u32 x = threadIdx.x; x < CP * SEL_BINS; x += ST) (&h[0][0])[x] = 0;
  __syncthreads();
  u32* mine = h[(threadIdx.x >> 6) % CP];
  const u64 step = (u64)gridDim.x * ST;
  for (u64 x0 = (u64)blockIdx.x * ST + threadIdx.x; x0 < n; x0 += WE * step) {
    u64 k[WE];
    u32 v[WE];
#pragma unroll
    for (int j = 0; j < WE; ++j) {
      const u64 x = x0 + j * step;
      k[j] = x < n ? K[x] : KINF;
      v[j] = needv && x < n ? V[x] : 0u;
    }
#pragma unroll
    for (int j = 0; j < WE; ++j)
      if (x0 + j * step < n && sel_match(k[j], v[j], q.pk, q.pv, q.nb)) atomicAdd(&mine[sel_digit(k[j], v[j], p, w)], 1u);
  }
  __syncthreads();
  if (threadIdx.x < SEL_BINS) {
    u32 sum = 0;
#pragma unroll
    for (int j = 0; j < CP; ++j) sum += h[j][threadIdx.x];
    if (sum) atomic_add32(&c->shist[pass][threadIdx.x], sum);
  }
}

// The end of a publication: this thread's stores to the mailbox become
// visible to the host before the number does.
__device__ __forceinline__ void publish(Mail* mail, u32 seq) {
  __threadfence_system();
  __hip_atomic_store(&mail->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Gathers the elements that match the prefix after the step's passes (at most
// CANDMAX), each workgroup through a list in LDS; the last workgroup to finish
// goes on with radix passes among them until at most RANKED are left and ranks
// those by counting: the one with exactly rank-1 smaller candidates is the
// answer.  Publishes the outcome to
// the box and to the host (sfail: the passes were not done, and the state is
// left for the next step; sbad: a consistency check failed).  nrange != 0: the
// selection starts here, without passes.
__global__ __launch_bounds__(ST) void k_sel_collect(const u64* K, const u32* V, u32 n, Ctl* c, u32 r, int passes,
                                                    const Range* range, u32 nrange, u64* ck, u32* cv, Mail* box,
                                                    Mail* mail, u32 seq) {
  __shared__ u64 sk[CANDMAX];
  __shared__ u32 sv[CANDMAX];
  __shared__ u32 h[SEL_BINS];
  __shared__ u32 s_n, s_base;
  __shared__ int s_last;
  u32 npass = 0;
  SelState q = nrange ? sel_start(range, nrange, r, n) : sel_after(c, c->q, passes, &npass);
  const bool go = q.done && !q.bad;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  if (go) {
    const u64 step = (u64)gridDim.x * ST;
    const bool needv = q.nb > 64;  // otherwise the match reads the keys alone, and a candidate's id is read when found
    for (u64 x0 = (u64)blockIdx.x * ST + threadIdx.x; x0 < n; x0 += WE * step) {
      u64 k[WE];
      u32 v[WE];
#pragma unroll
      for (int j = 0; j < WE; ++j) {
        const u64 x = x0 + j * step;
        k[j] = x < n ? K[x] : KINF;
        v[j] = needv && x < n ? V[x] : 0u;
      }
#pragma unroll
      for (int j = 0; j < WE; ++j) {
        const u64 x = x0 + j * step;
        if (x >= n || !sel_match(k[j], v[j], q.pk, q.pv, q.nb)) continue;
        const u32 id = needv ? v[j] : V[x], o = atomicAdd(&s_n, 1u);
        if (o < CANDMAX) {
          sk[o] = k[j];
          sv[o] = id;
        }
      }
    }
    __syncthreads();
    const u32 m = min(s_n, CANDMAX);  // (an excess shows in the sum)
    if (gridDim.x > 1) {
      if (threadIdx.x == 0) s_base = s_n ? atomic_add32(&c->sncand, s_n) : 0u;
      __syncthreads();
      for (u32 x = threadIdx.x; x < m; x += ST)
        if (s_base + x < CANDMAX) {
          st_a64(ck + s_base + x, sk[x]);
          st_a32(cv + s_base + x, sv[x]);
        }
    }
  }
  if (!last_workgroup(&c->collected, &s_last)) return;
  // every workgroup has read the state and the histograms
  if (threadIdx.x < SEL_BINS) c->shist[0][threadIdx.x] = c->shist[1][threadIdx.x] = 0;
  if (!q.done) {
    if (threadIdx.x == 0) {
      c->q = q;
      box->sfail = mail->sfail = 1;
      box->sbad = mail->sbad = 0;
      mail->npass = npass;
      publish(mail, seq);
    }
    return;
  }
  // (one workgroup's candidates never left LDS)
  const u32 found = gridDim.x == 1 ? s_n : ld_a32(&c->sncand), m = min(found, CANDMAX);
  bool bad = !go || found != q.cnt || m != found;
  __syncthreads();  // (s_n and sncand are read)
  if (gridDim.x > 1) {
    if (threadIdx.x == 0) st_a32(&c->sncand, 0u);
    for (u32 x = threadIdx.x; x < m; x += ST) {
      sk[x] = ld_a64(ck + x);
      sv[x] = ld_a32(cv + x);
    }
  }
  __syncthreads();
  while (!bad && q.cnt > RANKED && q.nb < 96) {
    const int w = sel_width(q), p = 96 - q.nb - w;
    if (threadIdx.x < SEL_BINS) h[threadIdx.x] = 0;
    __syncthreads();
    for (u32 x = threadIdx.x; x < m; x += ST) {
      const u64 k = sk[x];
      const u32 v = sv[x];
      if (sel_match(k, v, q.pk, q.pv, q.nb)) atomicAdd(&h[sel_digit(k, v, p, w)], 1u);
    }
    __syncthreads();
    q = sel_pick(q, &h[0], RANKED);
    bad = q.bad;
    __syncthreads();  // (every wavefront has read the histogram)
  }
  __shared__ u64 fk[RANKED];
  __shared__ u32 fv[RANKED];
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  if (!bad)
    for (u32 x = threadIdx.x; x < m; x += ST) {
      const u64 k = sk[x];
      const u32 v = sv[x];
      if (!sel_match(k, v, q.pk, q.pv, q.nb)) continue;
      const u32 o = atomicAdd(&s_n, 1u);
      if (o < RANKED) {
        fk[o] = k;
        fv[o] = v;
      }
    }
  __syncthreads();
  const u32 left = s_n;
  bad = bad || left != q.cnt || left > RANKED || q.rank == 0 || q.rank > left;
  if (!bad) {  // four threads per candidate
    constexpr u32 T = ST / RANKED;
    const u32 x = threadIdx.x / T;
    u32 below = 0;
    u64 k = 0;
    u32 v = 0;
    if (x < left) {
      k = fk[x];
      v = fv[x];
      for (u32 y = threadIdx.x % T; y < left; y += T) below += fk[y] < k || (fk[y] == k && fv[y] < v);
    }
#pragma unroll
    for (u32 d = 1; d < T; d *= 2) below += __shfl_xor(below, (int)d);
    if (x < left && threadIdx.x % T == 0 && below + 1 == q.rank) {
      box->rk = mail->rk = k;
      box->rv = mail->rv = v;
      __threadfence_system();
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    box->sfail = mail->sfail = 0;
    box->sbad = mail->sbad = bad;
    mail->npass = npass;
    publish(mail, seq);
  }
}

// ------------------------------------------------------------------ intake

// cur[id] = min(cur[id], key) for every pair (atomicMin); an id whose key
// dropped gets its mark byte set by a plain store (every writer stores the
// same 1, so no atomic is needed: a random atomic costs a round trip to the
// memory side, a byte store is merged in the L2).
__global__ __launch_bounds__(NT) void k_intake(const u64* keys, const u32* ids, u64 count, u64* cur, u8* marks,
                                               u64* acc, u64* post) {
  __shared__ u32 sw[NT / 64];
  u32 newly = 0;
  const u64 step = (u64)gridDim.x * NT;
  for (u64 x0 = (u64)blockIdx.x * NT + threadIdx.x; x0 < count; x0 += 4 * step) {
    u32 id[4];
    u64 k[4], old[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u64 x = x0 + q * step;
      id[q] = x < count ? ids[x] : 0u;
      k[q] = x < count ? keys[x] : KINF;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) old[q] = x0 + q * step < count ? atomic_min64(cur + id[q], k[q]) : KINF;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k[q] < old[q]) {
        marks[id[q]] = 1;
        newly += old[q] == KINF;
      }
  }
  newly = block_sum<NT>(newly, sw);
  if (threadIdx.x == 0) arrive(acc, nullptr, post, blockIdx.x, gridDim.x, newly);
}

// Mark compaction: marked ids in increasing order -> (cur[id], id); the
// marks are cleared.  Each thread takes 32 consecutive ids (two 16-byte loads)
// per round, turned into a 32-bit mask; a tile is BR rounds of NT * 32 ids (8
// rounds left 16 workgroups for a million ids: counting 6, writing 12 us).
// In the writing pass each round's marked ids are gathered in LDS in order (a
// scan of the masks' popcounts places them) and then written out coalesced,
// one output per thread, with cur[id] read alongside.
constexpr int BR = 2;
constexpr u32 BTILE = NT * BR;  // words of 32 ids
__device__ __forceinline__ u32 mark_mask(uint4 m) {
  const u32 w[4] = {m.x, m.y, m.z, m.w};
  u32 bits = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int b = 0; b < 4; ++b) bits |= (u32)(((w[j] >> (8 * b)) & 0xFFu) != 0u) << (4 * j + b);
  return bits;
}
template <bool WRITE>
__global__ __launch_bounds__(NT) void k_bits(u8* marks, u32 nwords, const u64* cur, u64* uk, u32* uv, Pass ps) {
  static_assert(BR == 2, "two counts of 16 bits");
  __shared__ u32 sw[NT / 64];
  __shared__ u32 sid[WRITE ? NT * 32 : 1];
  __shared__ u32 s_base;
  const u32 t = blockIdx.x;
  uint4* m4 = (uint4*)marks;
  u32 bitsr[BR], pc = 0;
#pragma unroll
  for (int r = 0; r < BR; ++r) {
    const u64 w = (u64)t * BTILE + (u64)r * NT + threadIdx.x;
    bitsr[r] = w < nwords ? mark_mask(m4[2 * w]) | (mark_mask(m4[2 * w + 1]) << 16) : 0u;
    pc |= (u32)__builtin_popcount(bitsr[r]) << (16 * r);
  }
  if constexpr (WRITE) {
    if (threadIdx.x < 64) {
      const u32 b = before_tile<1>(ps, 0, t);
      if (threadIdx.x == 0) s_base = b;
    }
  }
  u32 tot;
  const u32 ex = block_scan<NT>(pc, &tot, sw);
  const u32 t0 = tot & 0xFFFFu, t1 = tot >> 16;
  if constexpr (!WRITE) {
    if (threadIdx.x == 0) {
      ps.tc[t] = t0 + t1;
      arrive(ps.acc, ps.gs, ps.post, t, gridDim.x, t0 + t1);
    }
  } else {
#pragma unroll
    for (int r = 0; r < BR; ++r) {
      const u64 w = (u64)t * BTILE + (u64)r * NT + threadIdx.x;
      u32 bits = bitsr[r], o = r ? ex >> 16 : ex & 0xFFFFu;
      if (bits) {
        m4[2 * w] = make_uint4(0u, 0u, 0u, 0u);
        m4[2 * w + 1] = make_uint4(0u, 0u, 0u, 0u);
      }
      if (r) __syncthreads();  // (the round before read sid)
      while (bits) {
        const u32 b = (u32)__builtin_ctz(bits);
        bits &= bits - 1;
        sid[o++] = (u32)w * 32u + b;
      }
      __syncthreads();
      const u32 run = s_base + (r ? t0 : 0u), len = r ? t1 : t0;
      for (u32 x = threadIdx.x; x < len; x += NT) {
        const u32 id = sid[x];
        uv[run + x] = id;
        uk[run + x] = cur[id];
      }
    }
  }
}

// Delete of a batch of ids: cur[id] = KINF; each workgroup counts the ids
// that were present (the exchange returns the old key, so repeats in the
// batch count once).
__global__ __launch_bounds__(NT) void k_delete(const u32* ids, u64 count, u64* cur, u64* acc, u64* post) {
  __shared__ u32 sw[NT / 64];
  u32 gone = 0;
  for (u64 x = (u64)blockIdx.x * NT + threadIdx.x; x < count; x += (u64)gridDim.x * NT)
    gone += __hip_atomic_exchange((u64 PBH_GLB*)(cur + ids[x]), KINF, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) !=
                    KINF
                ? 1u
                : 0u;
  gone = block_sum<NT>(gone, sw);
  if (threadIdx.x == 0) arrive(acc, nullptr, post, blockIdx.x, gridDim.x, gone);
}

// ------------------------------------------------------------------ sort by (key, id)

// Compare-exchange by (key, id).
__device__ __forceinline__ void cx(u64& ka, u32& va, u64& kb, u32& vb) {
  if (ka > kb || (ka == kb && va > vb)) {
    const u64 tk = ka;
    const u32 tv = va;
    ka = kb;
    va = vb;
    kb = tk;
    vb = tv;
  }
}

// Sorts up to RANK_SORT pairs by counting, for each, the pairs below it, and
// marks their ids absent: 32 pairs per workgroup, each against all by 32
// threads, through tiles in LDS.  The work grows with the square, but it is
// one launch over the whole device, without a serial chain: 5,000 pairs 16 us
// (tiles of 2048 and two merge passes: 28 + 2 x 11 us, three workgroups at
// work); 12,000 pairs 41 us, 16,384 55 us, where a tile sort and two merge
// passes take 45.
constexpr u32 RANK_SORT = 12288;
constexpr u32 RW = 32, RTILE = 4096;
__global__ __launch_bounds__(1024) void k_rank(const u64* K, const u32* V, u32 n, u64* dk, u32* dv, u64* cur) {
  constexpr u32 SL = 1024 / RW;
  __shared__ u64 sk[RTILE];
  __shared__ u32 sv[RTILE];
  __shared__ u32 rank[RW];
  const u32 e = threadIdx.x % RW, sl = threadIdx.x / RW, x = blockIdx.x * RW + e;
  const u64 k = x < n ? K[x] : KINF;
  const u32 v = x < n ? V[x] : VINF;
  if (sl == 0) rank[e] = 0;
  u32 below = 0;
  for (u32 b = 0; b < n; b += RTILE) {
    const u32 m = min(n - b, RTILE);
    __syncthreads();
    for (u32 y = threadIdx.x; y < m; y += 1024) {
      sk[y] = K[b + y];
      sv[y] = V[b + y];
    }
    __syncthreads();
#pragma unroll 8
    for (u32 y = sl; y < m; y += SL) {
      const u64 o = sk[y];
      below += o < k || (o == k && sv[y] < v);
    }
  }
  atomicAdd(&rank[e], below);
  __syncthreads();
  if (sl == 0 && x < n) {
    const u32 r = rank[e];
    dk[r] = k;
    dv[r] = v;
    cur[v] = KINF;
  }
}

// Sorts each tile of STILE (key, id) pairs by (key, id): every thread sorts
// its SE consecutive elements in registers (odd-even transposition), then
// rounds merge the runs of SE, 2SE, ..., STILE/2 pairwise in LDS (ping-pong
// buffers), each thread producing its SE consecutive outputs after one
// merge-path search.  Padding (KINF, VINF) sorts last and is not written.
// Bound by the serial chain of the searches and walks, so the tile is spread
// over many threads (2048 pairs: 256 threads of 8 28 us, 512 of 4 20 us, 1024
// of 2 18 us), and it is as large as the LDS lets it be, which saves a merge
// pass of 8 to 10 us (4096 pairs by 1024 threads of 4: 27 us).
constexpr int SORT_T = 1024, SE = 4;
constexpr u32 STILE = SORT_T * SE;
__global__ __launch_bounds__(SORT_T) void k_tsort(const u64* sk_, const u32* sv_, u32 n, u64* dk, u32* dv) {
  __shared__ u64 bk[2][STILE];
  __shared__ u32 bv[2][STILE];
  const u64 base = (u64)blockIdx.x * STILE;
  {
    u64 lk[SE];
    u32 lv[SE];
#pragma unroll
    for (int q = 0; q < SE; ++q) {
      const u64 g = base + threadIdx.x + (u64)q * SORT_T;
      lk[q] = g < n ? sk_[g] : KINF;
      lv[q] = g < n ? sv_[g] : VINF;
    }
#pragma unroll
    for (int q = 0; q < SE; ++q) {
      bk[0][threadIdx.x + q * SORT_T] = lk[q];
      bv[0][threadIdx.x + q * SORT_T] = lv[q];
    }
  }
  __syncthreads();
  const u32 o0 = threadIdx.x * SE;
  u64 k[SE];
  u32 v[SE];
#pragma unroll
  for (int q = 0; q < SE; ++q) {
    k[q] = bk[0][o0 + q];
    v[q] = bv[0][o0 + q];
  }
#pragma unroll
  for (int r = 0; r < SE; ++r)
#pragma unroll
    for (int i = r & 1; i + 1 < SE; i += 2) cx(k[i], v[i], k[i + 1], v[i + 1]);
  int cur = 1;
  for (u32 L = SE; L < STILE; L *= 2, cur ^= 1) {
    // (buffer cur was last read two rounds ago, before the previous barrier)
#pragma unroll
    for (int q = 0; q < SE; ++q) {
      bk[cur][o0 + q] = k[q];
      bv[cur][o0 + q] = v[q];
    }
    __syncthreads();
    const u32 pb = (o0 / (2 * L)) * (2 * L), diag = o0 - pb;
    const u64* ak = bk[cur] + pb;
    const u32* av = bv[cur] + pb;
    const u64* bk2 = ak + L;
    const u32* bv2 = av + L;
    u32 i = mpath<true>(ak, av, L, bk2, bv2, L, diag), j = diag - i;
    u64 xa = i < L ? ak[i] : KINF, xb = j < L ? bk2[j] : KINF;
    u32 ya = i < L ? av[i] : VINF, yb = j < L ? bv2[j] : VINF;
#pragma unroll
    for (int q = 0; q < SE; ++q) {
      const bool ta = i < L && (j >= L || xa < xb || (xa == xb && ya <= yb));
      if (ta) {
        k[q] = xa;
        v[q] = ya;
        ++i;
        xa = i < L ? ak[i] : KINF;
        ya = i < L ? av[i] : VINF;
      } else {
        k[q] = xb;
        v[q] = yb;
        ++j;
        xb = j < L ? bk2[j] : KINF;
        yb = j < L ? bv2[j] : VINF;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < SE; ++q) {
    bk[cur][o0 + q] = k[q];
    bv[cur][o0 + q] = v[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < SE; ++q) {
    const u32 x = threadIdx.x + (u32)q * SORT_T;
    const u64 g = base + x;
    if (g < n) {
      dk[g] = bk[cur][x];
      dv[g] = bv[cur][x];
    }
  }
}

// Merge pass over sorted runs of length L (a multiple of TILE): runs 2p and
// 2p+1 are merged into [2pL, 2pL + 2L).  The last pass marks the ids absent (when set).
__device__ __forceinline__ void run_pair(u32 n, u32 L, u64 s, u32* base, u32* na, u32* nb) {
  const u64 b = (s / (2ull * L)) * 2ull * L;
  const u64 mid = b + L < n ? b + L : n, end = b + 2ull * L < n ? b + 2ull * L : n;
  *base = (u32)b;
  *na = (u32)(mid - b);
  *nb = (u32)(end - mid);
}

__global__ __launch_bounds__(NT) void k_smerge(const u64* K, const u32* V, u32 n, u32 L, u64* DK, u32* DV,
                                               u64* absent) {
  __shared__ u64 sk[TILE];
  __shared__ u32 sv[TILE];
  const u32 t = blockIdx.x;
  const u64 s = (u64)t * TILE;
  u32 b, na, nb;
  run_pair(n, L, s, &b, &na, &nb);
  const u32 d0 = (u32)(s - b);
  const u32 d1 = min(d0 + TILE, na + nb);
  __shared__ u32 ssplit[2];
  const u32 wv = threadIdx.x >> 6;
  if (wv < 2) {  // the tile's ends, one 65-way search each
    const u32 i = mpath_wave<true>(K + b, V + b, na, K + b + na, V + b + na, nb, wv ? d1 : d0);
    if ((threadIdx.x & 63u) == 0) ssplit[wv] = i;
  }
  __syncthreads();
  const u32 i0 = ssplit[0], i1 = ssplit[1];
  const u32 j0 = d0 - i0, j1 = d1 - i1;
  const u32 nA = i1 - i0, nT = d1 - d0, nB = j1 - j0;
  {
    u64 lk[WE];
    u32 lv[WE];
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      const u32 x = threadIdx.x + (u32)q * NT;
      const u32 g = x < nA ? b + i0 + x : b + na + j0 + (x - nA);
      lk[q] = x < nT ? K[g] : 0;
      lv[q] = x < nT ? V[g] : 0;
    }
#pragma unroll
    for (int q = 0; q < WE; ++q) {
      const u32 x = threadIdx.x + (u32)q * NT;
      if (x < nT) {
        sk[x] = lk[q];
        sv[x] = lv[q];
      }
    }
  }
  __syncthreads();
  const u32 dd0 = min((u32)threadIdx.x * WE, nT), dd1 = min(dd0 + WE, nT);
  u32 i = mpath<true>(sk, sv, nA, sk + nA, sv + nA, nB, dd0), j = dd0 - i;
  u64 ko[WE];
  u32 vo[WE];
#pragma unroll
  for (int q = 0; q < WE; ++q) {
    ko[q] = 0;
    vo[q] = 0;
    if (dd0 + q < dd1) {
      bool takeA = i < nA;
      if (takeA && j < nB) {
        const u64 ka = sk[i], kb = sk[nA + j];
        takeA = ka < kb || (ka == kb && sv[i] <= sv[nA + j]);
      }
      if (takeA) {
        ko[q] = sk[i];
        vo[q] = sv[i];
        ++i;
      } else {
        ko[q] = sk[nA + j];
        vo[q] = sv[nA + j];
        ++j;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < WE; ++q)
    if (dd0 + q < dd1) {
      sk[dd0 + q] = ko[q];
      sv[dd0 + q] = vo[q];
    }
  __syncthreads();
  for (u32 x = threadIdx.x; x < nT; x += NT) {
    DK[s + x] = sk[x];
    DV[s + x] = sv[x];
    if (absent) absent[sv[x]] = KINF;
  }
}

u32 cdiv(u64 a, u64 b) { return (u32)((a + b - 1) / b); }
u32 grid_for(u64 n) {
  u64 g = (n + NT - 1) / NT;
  return (u32)(g < 1 ? 1 : (g > GRID_STRIDE ? GRID_STRIDE : g));
}

}  // namespace

struct WideScratch {
  u32 d = 0;
  Ctl* ctl = nullptr;      // device
  Mail* box = nullptr;     // device: results of the current step
  Mail* mail_h = nullptr;  // host-mapped coherent mailbox (host view)
  Mail* mail_d = nullptr;  // its device address
  u32 seq = 0;             // steps published so far
  u8* marks = nullptr;     // one byte per id (32 per 32-id word), zero between calls
  u64 marks_n = 0;
  u32* part = nullptr;  // tile split points of a merge (maxtiles + 1)
  u32* tc = nullptr;    // tile counts, 3 arrays of maxtiles
  u64* gs = nullptr;    // their sums over 64 tiles, packed
  u64* acc = nullptr;   // arrival words (one per 64 workgroups; a line each)
  // Posts (host-mapped, a word per 64 workgroups) of a step and of the kernel
  // before it that counts ids (intake, delete).
  u64* post_h[2] = {nullptr, nullptr};
  u64* post_d[2] = {nullptr, nullptr};
  u32 npost[2] = {0, 0};  // workgroups of the launches that post
  // Key range of each level's B_i, per 64 tiles of the merge that last wrote
  // it (what was split off since only narrows it), and how many there are.
  Range* range[MAXL] = {};
  u32 nrange[MAXL] = {};
  u64* cand_k = nullptr;
  u32* cand_v = nullptr;
  u64* tmp_k = nullptr;  // sort scratch (4d elements)
  u32* tmp_v = nullptr;
  u32 maxtiles = 0;
  hipStream_t s = 0;
  // Profiling (off by default): HIP events around every kernel launch of
  // the engine, with the kernel's kind and algorithmic bytes; totalled per
  // kind when the operation ends.
  bool profile = false;
  struct Rec {
    int kind;
    u64 bytes;
  };
  std::vector<hipEvent_t> ev;  // event pairs, created as needed
  std::vector<Rec> rec;        // launches of the current operation
  WideKernelStat kst[WK_COUNT] = {};
};

namespace {

#define WCHK(x)                               \
  do {                                        \
    if ((x) != hipSuccess) return E_DEVICE;   \
  } while (0)

int launch_ok() { return hipGetLastError() == hipSuccess ? 0 : E_DEVICE; }

// Runs launch() -- one kernel launch -- bracketed by HIP events while
// profiling is on.  Returns the launch's record index (bytes can be patched
// once a step's results are known) or -1.
template <class F>
int plaunch(WideScratch* w, int kind, u64 bytes, F&& launch) {
  if (!w->profile) {
    launch();
    return -1;
  }
  const size_t i = w->rec.size();
  while (w->ev.size() < 2 * (i + 1)) {
    hipEvent_t e = nullptr;
    // timing-only events: without the system-scope fence a record does not
    // write back the L2 (which would slow the very step being timed)
    if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) {
      launch();
      return -1;
    }
    w->ev.push_back(e);
  }
  (void)hipEventRecord(w->ev[2 * i], w->s);
  launch();
  (void)hipEventRecord(w->ev[2 * i + 1], w->s);
  w->rec.push_back(WideScratch::Rec{kind, bytes});
  return (int)i;
}

void patch_bytes(WideScratch* w, int idx, u64 bytes) {
  if (idx >= 0) w->rec[(size_t)idx].bytes = bytes;
}
void patch_kind(WideScratch* w, int idx, int kind) {
  if (idx >= 0) w->rec[(size_t)idx].kind = kind;
}

// Totals the current operation's timed launches per kind (the operation's
// work has ended, so the events have passed).
int prof_collect(WideScratch* w) {
  if (w->rec.empty()) return 0;
  WCHK(hipEventSynchronize(w->ev[2 * w->rec.size() - 1]));
  for (size_t i = 0; i < w->rec.size(); ++i) {
    float ms = 0.f;
    WCHK(hipEventElapsedTime(&ms, w->ev[2 * i], w->ev[2 * i + 1]));
    WideKernelStat& k = w->kst[w->rec[i].kind];
    k.launches += 1;
    k.bytes += w->rec[i].bytes;
    k.ms += ms;
  }
  w->rec.clear();
  return 0;
}

// Waits until the host sees results in host-mapped memory, by polling it (a stream synchronisation would add the runtime's
// completion path and a system-scope cache write-back to every step).
// Should they not arrive within a second, the stream is synchronised, which
// also reports a failed kernel (E_DEVICE); a step whose kernels all ended
// without them gives E_TIMEOUT.
template <class Ready>
int wait_for(WideScratch* w, Ready&& ready) {
  const auto t0 = std::chrono::steady_clock::now();
  for (u32 spin = 1;; ++spin) {
    if (ready()) return 0;
    if ((spin & 4095u) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(1)) break;
  }
  WCHK(hipStreamSynchronize(w->s));
  return ready() ? 0 : E_TIMEOUT;
}
int wait_mail(WideScratch* w, u32 want) {
  return wait_for(w, [&] { return __atomic_load_n(&w->mail_h->seq, __ATOMIC_ACQUIRE) == want; });
}

// Clears the words in which the nt workgroups of the next launch post their
// counts, and returns their device address; read_posts waits for them and adds
// them up, F counts.
u64* open_posts(WideScratch* w, int which, u32 nt) {
  w->npost[which] = nt;
  for (u32 g = 0; g < cdiv(nt, 64); ++g) __atomic_store_n(w->post_h[which] + g, 0ull, __ATOMIC_RELAXED);
  return w->post_d[which];
}
template <int F>
int read_posts(WideScratch* w, int which, u64* sums) {
  for (int f = 0; f < F; ++f) sums[f] = 0;
  for (u32 g = 0; g < cdiv(w->npost[which], 64); ++g) {
    u64 x = 0;
    if (int rc = wait_for(w, [&] { return (x = __atomic_load_n(w->post_h[which] + g, __ATOMIC_ACQUIRE)) != 0; }))
      return rc;
    for (int f = 0; f < F; ++f) sums[f] += (x >> (f * Field<F>::bits)) & Field<F>::mask;
  }
  return 0;
}
Pass next_pass(WideScratch* w, u32 nt) {
  return Pass{w->tc, w->maxtiles, w->gs, w->acc, open_posts(w, 0, nt)};
}

// C = DeleteDuplicates(Merge(A, B)) by id; *num_le = outputs <= piv.  // With count_le the
// counting pass reads the keys too; level >= 0: the outputs become its B.
int wmerge(WideScratch* w, Arr A, u32 na, Arr B, u32 nb, Arr C, const u64* cur, int prefer, int level, bool count_le,
           KV piv, u32* m, u32* num_le) {
  const u64 total = (u64)na + nb;
  if (total == 0) {
    *m = 0;
    *num_le = 0;
    return 0;
  }
  const u32 nt = cdiv(total, TILE);
  if (nt > w->maxtiles) return E_INTERNAL;
  const MArgs a{A.k, A.v, na, B.k, B.v, nb, C.k, C.v, cur, prefer, level >= 0 ? w->range[level] : nullptr, piv.k, piv.v};
  if (level >= 0) w->nrange[level] = cdiv(nt, 64);
  const Pass ps = next_pass(w, nt);
  plaunch(w, WK_MERGE_COUNT, (count_le ? 12ull : 4ull) * total, [&] {
    if (count_le)
      hipLaunchKernelGGL((k_merge<false, true>), dim3(nt), dim3(NT), 0, w->s, a, w->part, ps);
    else
      hipLaunchKernelGGL((k_merge<false, false>), dim3(nt), dim3(NT), 0, w->s, a, w->part, ps);
  });
  const int iw = plaunch(w, WK_MERGE_WRITE, 12ull * total, [&] {
    hipLaunchKernelGGL((k_merge<true, true>), dim3(nt), dim3(NT), 0, w->s, a, w->part, ps);
  });
  if (int rc = launch_ok()) return rc;
  u64 sums[2];
  if (int rc = read_posts<2>(w, 0, sums)) return rc;
  *m = (u32)sums[0];
  *num_le = (u32)sums[1];
  patch_bytes(w, iw, 12ull * (total + *m));  // 12 B per input read + 12 B per output written
  return 0;
}

// Select(A, r) (rank r, 1-based) followed by the three-way split of A at
// (min(Select(A, r), cap), p2) into O0 / O1 / O2, as one host step: the
// split reads the selected element on the device.  *p1 = the split's first
// pivot.  A's keys lie in the range of level `level`.
int wpartition3_sel(WideScratch* w, Arr A, u32 n, KV p1, KV p2, Arr O0, Arr O1, Arr O2, const u64* live, u32* n0,
                    u32* n1, u32* n2, const Mail* sel);
int wselpart(WideScratch* w, Arr A, u32 n, u32 r, int level, KV cap, KV p2, Arr O0, Arr O1, Arr O2,
             const u64* live, KV* p1, u32* n0, u32* n1, u32* n2) {
  if (n == 0 || r == 0 || r > n) return E_INTERNAL;
  const u32 gs = std::min<u32>(cdiv(n, ST * 4), GRID_SEL);
  // Each pass fixes 8 more of the 96 bits, so 12 passes (6 steps of 2) always
  // finish; one or two typically do (two when the keys crowd at one end of
  // their range, as decreased keys do).  A pass after the last needed one
  // returns at once; few enough elements need none.
  for (int step = 0; step < 6; ++step) {
    const int passes = n <= CANDMAX ? 0 : 2;
    const auto first = [&](int p) { return step == 0 && p == 0 ? w->nrange[level] : 0u; };
    int ip[2];
    for (int p = 0; p < passes; ++p)
      ip[p] = plaunch(w, WK_SEL_PASS, 8ull * n, [&] {
        hipLaunchKernelGGL(k_sel_pass, dim3(gs), dim3(ST), 0, w->s, A.k, A.v, n, w->ctl, r, p, w->range[level], first(p));
      });
    const u32 want = ++w->seq;
    const int ic = plaunch(w, WK_SEL_GATHER, 8ull * n, [&] {
      hipLaunchKernelGGL(k_sel_collect, dim3(gs), dim3(ST), 0, w->s, A.k, A.v, n, w->ctl, r, passes, w->range[level],
                         first(passes), w->cand_k, w->cand_v, w->box, w->mail_d, want);
    });
    if (int rc = wpartition3_sel(w, A, n, cap, p2, O0, O1, O2, live, n0, n1, n2, w->box)) return rc;
    if (int rc = wait_mail(w, want)) return rc;
    // passes after the last needed one, and a gather before the passes were
    // done, returned at once: they read nothing
    for (int p = (int)w->mail_h->npass; p < passes; ++p) patch_kind(w, ip[p], WK_IDLE), patch_bytes(w, ip[p], 0);
    if (w->mail_h->sfail) patch_kind(w, ic, WK_IDLE), patch_bytes(w, ic, 0);
    if (w->mail_h->sbad) return E_INTERNAL;
    if (!w->mail_h->sfail) {
      *p1 = cap;
      const KV s{w->mail_h->rk, w->mail_h->rv};
      if (kv_less(s, cap)) *p1 = s;
      return 0;
    }
  }
  return E_INTERNAL;
}

int wpartition3_sel(WideScratch* w, Arr A, u32 n, KV p1, KV p2, Arr O0, Arr O1, Arr O2, const u64* live, u32* n0,
                    u32* n1, u32* n2, const Mail* sel) {
  if (n == 0) {
    *n0 = *n1 = *n2 = 0;
    return 0;
  }
  const u32 nt = cdiv(n, TILE);
  if (nt > w->maxtiles) return E_INTERNAL;
  const PArgs a{A.k, A.v, n, p1.k, p1.v, p2.k, p2.v, live, {O0.k, O1.k, O2.k}, {O0.v, O1.v, O2.v}, sel};
  const Pass ps = next_pass(w, nt);
  plaunch(w, WK_SPLIT_COUNT, 8ull * n, [&] { hipLaunchKernelGGL(k_part<false>, dim3(nt), dim3(NT), 0, w->s, a, ps); });
  plaunch(w, WK_SPLIT_WRITE, 24ull * n, [&] { hipLaunchKernelGGL(k_part<true>, dim3(nt), dim3(NT), 0, w->s, a, ps); });
  if (int rc = launch_ok()) return rc;
  u64 sums[3];
  if (int rc = read_posts<3>(w, 0, sums)) return rc;
  *n0 = (u32)sums[0];
  *n1 = (u32)sums[1];
  *n2 = (u32)sums[2];
  return 0;
}

int wpartition3(WideScratch* w, Arr A, u32 n, KV p1, KV p2, Arr O0, Arr O1, Arr O2, const u64* live, u32* n0,
                u32* n1, u32* n2) {
  return wpartition3_sel(w, A, n, p1, p2, O0, O1, O2, live, n0, n1, n2, nullptr);
}

// Sorts X[0, n) by (key, id) into D and marks the ids absent (n <= 4d; X is
// overwritten).
int wsort(WideScratch* w, Arr X, u32 n, u64* dk, u32* dv, u64* cur) {
  if (n == 0) return 0;
  if (n <= RANK_SORT) {
    plaunch(w, WK_SORT_TILE, 24ull * n, [&] {
      hipLaunchKernelGGL(k_rank, dim3(cdiv(n, RW)), dim3(1024), 0, w->s, X.k, X.v, n, dk, dv, cur);
    });
    return launch_ok();
  }
  const u32 nt = cdiv(n, TILE);
  int passes = 0;
  for (u64 L = STILE; L < n; L *= 2) ++passes;
  // ping-pong so that the last pass lands in D
  Arr bufs[2] = {X, Arr{w->tmp_k, w->tmp_v}};
  Arr src = bufs[passes & 1];
  plaunch(w, WK_SORT_TILE, 24ull * n,
          [&] { hipLaunchKernelGGL(k_tsort, dim3(cdiv(n, STILE)), dim3(SORT_T), 0, w->s, X.k, X.v, n, src.k, src.v); });
  u64 L = STILE;
  for (int p = 0; p < passes; ++p, L *= 2) {
    const bool last = p == passes - 1;
    Arr to = last ? Arr{dk, dv} : (src.k == bufs[0].k ? bufs[1] : bufs[0]);
    plaunch(w, WK_SORT_MERGE, 24ull * n, [&] {
      hipLaunchKernelGGL(k_smerge, dim3(nt), dim3(NT), 0, w->s, src.k, src.v, n, (u32)L, to.k, to.v,
                         last ? cur : nullptr);
    });
    src = to;
  }
  return launch_ok();
}

// Resolve(i) of Algorithm 1 with the device-wide steps; the control flow is
// the one-workgroup engine's (resolve_t), step for step.
int wresolve(WideScratch* w, const Geom& g, HeapState* st, const u64* cur, int i) {
  Lvl a = st->L[i];
  const bool nx = i + 1 < g.q;
  Lvl b = nx ? st->L[i + 1] : Lvl{0, 0, 0, 0, KINF, VINF, 0};
  int ell = st->ell;
  KV pi{a.pk, a.pv}, pn{b.pk, b.pv};
  const u32 cB = (u32)nomB(g.d, i);
  u64 touched = 0;
  int rc = 0;
  if (a.nS > 0 || a.nB > cB) {
    Arr S = lbuf(g, i, 3 + a.ssel), B = lbuf(g, i, a.bsel), M = lbuf(g, i, a.bsel ^ 1);
    if ((u64)a.nS + a.nB > capB(g.d, i)) return E_INTERNAL;
    u32 m, num;
    // S_0 holds the latest updates, so at level 0 its copy of an id is the live one.
    if ((rc = wmerge(w, S, a.nS, B, a.nB, M, cur, i == 0 ? PREFER_A : PREFER_LIVE, i, true, pi, &m, &num)))
      return rc;
    touched += 2ull * (a.nS + a.nB) + m;
    a.bsel ^= 1;
    a.nS = 0;
    a.ssel = 0;
    const bool sel = num > cB;
    if (sel) num = cB;
    if (num < m) {
      if (!nx) return E_CAPACITY;
      // (an empty S_{i+1} takes the upper part as it is)
      Arr Sn = lbuf(g, i + 1, 3 + b.ssel), Sn2 = lbuf(g, i + 1, 3 + (b.ssel ^ 1));
      Arr Lo = lbuf(g, i, a.bsel ^ 1), Hi = b.nS ? lbuf(g, i, 2) : Sn2;
      if (b.nS == 0 && m - std::min(num, m) > capS(g.d, i + 1)) return E_INTERNAL;
      u32 n0, n1, n2;
      if (sel) {  // p_i <- Select(B_i, 2d*4^i), and the split at it
        if ((rc = wselpart(w, M, m, cB, i, kv_inf(), kv_inf(), Lo, Hi, Hi, nullptr, &pi, &n0, &n1, &n2))) return rc;
        touched += m;
      } else if ((rc = wpartition3(w, M, m, pi, kv_inf(), Lo, Hi, Hi, nullptr, &n0, &n1, &n2))) {
        return rc;
      }
      touched += 3ull * m;
      a.bsel ^= 1;
      a.nB = n0;
      if ((u64)b.nS + n1 > capS(g.d, i + 1)) return E_INTERNAL;
      u32 ms = n1, dummy;
      if (b.nS && (rc = wmerge(w, Sn, b.nS, Hi, n1, Sn2, cur, PREFER_LIVE, -1, false, kv_inf(), &ms, &dummy)))
        return rc;
      touched += 2ull * (b.nS + n1) + ms;
      b.ssel ^= 1;
      b.nS = ms;
      if (ell < i + 1) ell = i + 1;
    } else {
      a.nB = m;
    }
  }
  if (a.nB < cB && i < ell && nx) {
    if ((u64)b.nB + b.nS > capB(g.d, i + 1)) return E_INTERNAL;
    u32 m2 = b.nB, dummy;
    if (b.nS) {  // (an empty one leaves B_{i+1} as it is)
      Arr Bn = lbuf(g, i + 1, b.bsel), Sn = lbuf(g, i + 1, 3 + b.ssel);
      if ((rc = wmerge(w, Bn, b.nB, Sn, b.nS, lbuf(g, i + 1, b.bsel ^ 1), cur, PREFER_LIVE, i + 1, false, kv_inf(),
                       &m2, &dummy)))
        return rc;
      b.bsel ^= 1;
    }
    touched += 2ull * (b.nB + b.nS) + m2;
    b.nS = 0;
    b.ssel = 0;
    b.nB = m2;
    if (m2 > 0) {
      const u32 r = cB - a.nB;
      Arr M2 = lbuf(g, i + 1, b.bsel), Bk = lbuf(g, i + 1, b.bsel ^ 1), Sk = lbuf(g, i + 1, 3);
      Arr Up = lbuf(g, i, 2);
      u32 nu, nb1, ns1;
      // p_i <- min(Select(B_{i+1}, r), p_{i+1}), and the split at (p_i,
      // p_{i+1}); elements moving up into B_0 are checked for liveness here,
      // all at once.
      KV pnew = pn;
      if (r < m2) {
        if ((rc = wselpart(w, M2, m2, r, i + 1, pn, pn, Up, Bk, Sk, i == 0 ? cur : nullptr, &pnew, &nu, &nb1, &ns1)))
          return rc;
        touched += m2;
      } else if ((rc = wpartition3(w, M2, m2, pnew, pn, Up, Bk, Sk, i == 0 ? cur : nullptr, &nu, &nb1, &ns1))) {
        return rc;
      }
      touched += 3ull * m2;
      b.bsel ^= 1;
      b.nB = nb1;
      b.nS = ns1;
      b.ssel = 0;
      Arr Bi = lbuf(g, i, a.bsel), Bi2 = lbuf(g, i, a.bsel ^ 1);
      u32 mb;
      if ((rc = wmerge(w, Bi, a.nB, Up, nu, Bi2, cur, i == 0 ? PREFER_B : PREFER_LIVE, i, false, kv_inf(), &mb,
                       &dummy)))
        return rc;
      touched += 2ull * (a.nB + nu) + mb;
      a.bsel ^= 1;
      a.nB = mb;
      pi = pnew;
    }
  }
  a.cnt++;
  a.pk = pi.k;
  a.pv = pi.v;
  st->L[i] = a;
  if (nx) st->L[i + 1] = b;
  st->elems += touched;
  fix_ell(st, g.q);
  return 0;
}

void wdrive(WideScratch* w, WideHeap* h, int what) {
  HostTeam t{nullptr};
  drive_with(t, h->g, h->st, h->sched, what, [&](int lvl) {
    int rc = wresolve(w, h->g, h->st, h->cur, lvl);
    if (rc) h->st->err = rc;
  });
}

int grow_if_needed(WideScratch* w, WideHeap* h) {
  while (need_grow(h->g, h->st)) {
    if (int rc = h->grow(h->ctx, &h->g)) return rc;
    if (int rc = wide_reserve(w, capB(h->g.d, h->g.q - 1))) return rc;
  }
  return 0;
}

}  // namespace

int wide_reserve(WideScratch* w, u64 elems) {
  u64 need = (elems + TILE - 1) / TILE + 2;
  if (need < (u64)GRID_STRIDE) need = GRID_STRIDE;
  if (need <= w->maxtiles) return 0;
  if (w->part) (void)hipFree(w->part);
  if (w->tc) (void)hipFree(w->tc);
  if (w->gs) (void)hipFree(w->gs);
  if (w->acc) (void)hipFree(w->acc);
  w->part = w->tc = nullptr;
  w->gs = w->acc = nullptr;
  w->maxtiles = 0;
  const u64 ng = need / 64 + 1;
  WCHK(hipMalloc(&w->part, (need + 1) * sizeof(u32)));
  WCHK(hipMalloc(&w->tc, 3 * need * sizeof(u32)));
  WCHK(hipMalloc(&w->gs, ng * sizeof(u64)));
  WCHK(hipMalloc(&w->acc, LINE * ng * sizeof(u64)));
  WCHK(hipMemset(w->acc, 0, LINE * ng * sizeof(u64)));
  for (int r = 0; r < 2; ++r) {
    if (w->post_h[r]) (void)hipHostFree(w->post_h[r]);
    w->post_h[r] = nullptr;
    WCHK(hipHostMalloc(&w->post_h[r], ng * sizeof(u64), hipHostMallocMapped | hipHostMallocCoherent));
    WCHK(hipHostGetDevicePointer((void**)&w->post_d[r], w->post_h[r], 0));
  }
  // the levels' ranges in one array; they outlive the growth of the heap
  Range* p = nullptr;
  WCHK(hipMalloc(&p, MAXL * ng * sizeof(Range)));
  Range* old = w->range[0];
  for (int i = 0; i < MAXL; ++i) {
    if (w->nrange[i])
      WCHK(hipMemcpy(p + i * ng, w->range[i], w->nrange[i] * sizeof(Range), hipMemcpyDeviceToDevice));
    w->range[i] = p + i * ng;
  }
  if (old) (void)hipFree(old);
  w->maxtiles = (u32)need;
  return 0;
}

int wide_create(WideScratch** out, u32 d) {
  WideScratch* w = new WideScratch;
  w->d = d;
  *out = w;
  WCHK(hipMalloc(&w->ctl, sizeof(Ctl)));
  WCHK(hipMalloc(&w->box, sizeof(Mail)));
  WCHK(hipMemset(w->box, 0, sizeof(Mail)));
  WCHK(hipHostMalloc(&w->mail_h, sizeof(Mail), hipHostMallocMapped | hipHostMallocCoherent));
  std::memset(w->mail_h, 0, sizeof(Mail));
  WCHK(hipHostGetDevicePointer((void**)&w->mail_d, w->mail_h, 0));
  WCHK(hipMalloc(&w->cand_k, CANDMAX * sizeof(u64)));
  WCHK(hipMalloc(&w->cand_v, CANDMAX * sizeof(u32)));
  WCHK(hipMalloc(&w->tmp_k, 4ull * d * sizeof(u64)));
  WCHK(hipMalloc(&w->tmp_v, 4ull * d * sizeof(u32)));
  WCHK(hipMemset(w->ctl, 0, sizeof(Ctl)));
  return wide_reserve(w, 4ull * d);
}

void wide_set_profiling(WideScratch* w, bool on) { w->profile = on; }

void wide_kernel_profile(const WideScratch* w, int kind, WideKernelStat* out) { *out = w->kst[kind]; }

const char* wide_kernel_name(int kind) {
  static const char* const names[WK_COUNT] = {
      "k_merge<true> (merge + DeleteDuplicates, writing pass)",
      "k_merge<false> (merge, counting pass)",
      "k_sel_pass (radix Select pass)",
      "k_sel_collect (Select gather and rank)",
      "k_part<false> (three-way split, counting pass)",
      "k_part<true> (three-way split, writing pass)",
      "k_intake (atomicMin on current keys + marks)",
      "k_bits<false> (mark compaction, counting pass)",
      "k_bits<true> (mark compaction, writing pass)",
      "k_rank / k_tsort (sort of the extracted minima)",
      "k_smerge (merge pass of the extracted minima)",
      "k_delete (ids marked absent)",
      "scans, reductions, result publishing",
      "Select passes and gathers that returned at once"};
  return kind >= 0 && kind < WK_COUNT ? names[kind] : nullptr;
}

void wide_destroy(WideScratch* w) {
  if (!w) return;
  (void)hipDeviceSynchronize();
  if (w->ctl) (void)hipFree(w->ctl);
  if (w->box) (void)hipFree(w->box);
  if (w->marks) (void)hipFree(w->marks);
  if (w->mail_h) (void)hipHostFree(w->mail_h);
  if (w->part) (void)hipFree(w->part);
  if (w->tc) (void)hipFree(w->tc);
  if (w->gs) (void)hipFree(w->gs);
  if (w->acc) (void)hipFree(w->acc);
  if (w->range[0]) (void)hipFree(w->range[0]);  // (all levels')
  for (u64* p : w->post_h)
    if (p) (void)hipHostFree(p);
  if (w->cand_k) (void)hipFree(w->cand_k);
  if (w->cand_v) (void)hipFree(w->cand_v);
  if (w->tmp_k) (void)hipFree(w->tmp_k);
  if (w->tmp_v) (void)hipFree(w->tmp_v);
  for (hipEvent_t e : w->ev) (void)hipEventDestroy(e);
  delete w;
}

// BulkUpdate (Section 2.2): cur[id] = min(cur[id], key) for every pair, the
// ids whose key dropped form U sorted by id; pieces of at most d go into S_0,
// each followed by Resolve(0) and the schedule.
int wide_bulk_update(WideScratch* w, WideHeap* h, const u64* keys, const u32* ids, u64 count) {
  HeapState* st = h->st;
  if (count == 0) return 0;
  // A batch of at most d pairs is one piece: the compaction writes it straight
  // into S_0 (empty between operations).
  const bool direct = count <= h->g.d;
  if (direct)
    if (int rc = grow_if_needed(w, h)) return rc;
  // (room for the tiles of the largest level and of the mark compaction)
  const u64 bits = (u64)h->nwords * TILE / BTILE;
  if (int rc = wide_reserve(w, std::max(capB(h->g.d, h->g.q - 1), bits))) return rc;
  if (w->marks_n < 32ull * h->nwords) {
    if (w->marks) (void)hipFree(w->marks);
    w->marks = nullptr;
    w->marks_n = 0;
    WCHK(hipMalloc(&w->marks, 32ull * h->nwords));
    WCHK(hipMemsetAsync(w->marks, 0, 32ull * h->nwords, w->s));
    w->marks_n = 32ull * h->nwords;
  }
  const u32 gi = grid_for(count);
  // per pair: the pair (12 B) and the atomicMin on its current key (8 B)
  u64* posts = open_posts(w, 1, gi);
  plaunch(w, WK_INTAKE, 20ull * count, [&] {
    hipLaunchKernelGGL(k_intake, dim3(gi), dim3(NT), 0, w->s, keys, ids, count, h->cur, w->marks, w->acc, posts);
  });
  const u32 nt = cdiv(h->nwords, BTILE);
  if (nt > w->maxtiles) return E_INTERNAL;
  const Arr S0 = lbuf(h->g, 0, 3);
  u64* uk = direct ? S0.k : h->ukeys;
  u32* uv = direct ? S0.v : h->uids;
  const u64 nmark = 32ull * h->nwords;  // one mark byte per id
  const Pass ps = next_pass(w, nt);
  plaunch(w, WK_BITS_COUNT, nmark, [&] {
    hipLaunchKernelGGL(k_bits<false>, dim3(nt), dim3(NT), 0, w->s, w->marks, h->nwords, (const u64*)h->cur, uk, uv, ps);
  });
  const int ib = plaunch(w, WK_BITS_WRITE, nmark, [&] {
    hipLaunchKernelGGL(k_bits<true>, dim3(nt), dim3(NT), 0, w->s, w->marks, h->nwords, (const u64*)h->cur, uk, uv, ps);
  });
  if (int rc = launch_ok()) return rc;
  u64 newly, nu;
  if (int rc = read_posts<1>(w, 1, &newly)) return rc;
  if (int rc = read_posts<1>(w, 0, &nu)) return rc;
  // marks read, plus per output its current key read (8 B) and the pair written (12 B)
  patch_bytes(w, ib, nmark + 20ull * nu);
  st->live += newly;
  for (u64 c0 = 0; c0 < nu;) {
    if (!direct)
      if (int rc = grow_if_needed(w, h)) return rc;
    const u32 len = (u32)((nu - c0) < h->g.d ? (nu - c0) : h->g.d);
    Arr S = lbuf(h->g, 0, 3);
    if (!direct) {
      WCHK(hipMemcpyAsync(S.k, h->ukeys + c0, len * sizeof(u64), hipMemcpyDeviceToDevice, w->s));
      WCHK(hipMemcpyAsync(S.v, h->uids + c0, len * sizeof(u32), hipMemcpyDeviceToDevice, w->s));
    }
    st->L[0].nS = len;
    st->L[0].ssel = 0;
    if (st->ell < 0) st->ell = 0;
    st->elems += 2ull * len;
    wdrive(w, h, DRIVE_AFTER);
    if (st->err) return st->err;
    c0 += len;
  }
  return prof_collect(w);
}

// Delete (Section 1.2) of a batch of ids: their current keys become absent,
// which every later merge and every move into B_0 treat as a dead copy; B_0
// is filtered at once (it holds only live elements), then Resolve(0) and the
// schedule.
int wide_delete(WideScratch* w, WideHeap* h, const u32* ids, u64 count) {
  HeapState* st = h->st;
  if (count == 0) return 0;
  if (int rc = wide_reserve(w, capB(h->g.d, h->g.q - 1))) return rc;
  const u32 gi = grid_for(count);
  u64* posts = open_posts(w, 1, gi);
  plaunch(w, WK_ABSENT, 12ull * count,
          [&] { hipLaunchKernelGGL(k_delete, dim3(gi), dim3(NT), 0, w->s, ids, count, h->cur, w->acc, posts); });
  if (int rc = launch_ok()) return rc;
  const Lvl a0 = st->L[0];
  if (a0.nB) {
    Arr B = lbuf(h->g, 0, a0.bsel), O = lbuf(h->g, 0, a0.bsel ^ 1), X = lbuf(h->g, 0, 2);
    u32 n0, n1, n2;
    if (int rc = wpartition3(w, B, a0.nB, kv_inf(), kv_inf(), O, X, X, h->cur, &n0, &n1, &n2)) return rc;
    st->L[0].bsel ^= 1;
    st->L[0].nB = n0;
    st->elems += (u64)a0.nB + n0;
  }
  u64 gone;
  if (int rc = read_posts<1>(w, 1, &gone)) return rc;
  st->live -= gone;
  fix_ell(st, h->g.q);
  if (int rc = grow_if_needed(w, h)) return rc;
  wdrive(w, h, DRIVE_AFTER);
  if (st->err) return st->err;
  return prof_collect(w);
}

// Batched ExtractMin: repeatedly the smallest min(k_left, |B_0|) elements of
// B_0 (B_0 <= p_0 < everything else and holds only live elements) are split
// off, sorted by (key, id), written out and marked absent; then Resolve(0)
// and the schedule.
int wide_extract_min(WideScratch* w, WideHeap* h, u64 k, u64* okeys, u32* oids, u64* count_out) {
  HeapState* st = h->st;
  *count_out = 0;
  u64 out = 0;
  bool pending = false;
  if (int rc = wide_reserve(w, capB(h->g.d, h->g.q - 1))) return rc;
  for (;;) {
    if (!pending && out >= k) break;
    if (int rc = grow_if_needed(w, h)) return rc;
    wdrive(w, h, (pending ? DRIVE_AFTER : 0) | (out < k ? DRIVE_ENSURE : 0));
    pending = false;
    if (st->err) return st->err;
    if (out >= k) break;
    const Lvl a0 = st->L[0];
    if (a0.nB == 0) {
      if (st->ell >= 0) return E_INTERNAL;  // the refill leaves B_0 empty only when the heap is
      break;
    }
    const u32 take = (u32)((k - out) < a0.nB ? (k - out) : a0.nB);
    Arr B = lbuf(h->g, 0, a0.bsel), X = lbuf(h->g, 0, 2);
    KV thr = kv_inf();
    u32 n0, n1, n2;
    if (take < a0.nB) {
      if (int rc = wselpart(w, B, a0.nB, take, 0, kv_inf(), kv_inf(), X, lbuf(h->g, 0, a0.bsel ^ 1), X, nullptr,
                            &thr, &n0, &n1, &n2))
        return rc;
    } else if (int rc = wpartition3(w, B, a0.nB, thr, kv_inf(), X, lbuf(h->g, 0, a0.bsel ^ 1), X, nullptr, &n0, &n1,
                                    &n2)) {
      return rc;
    }
    if (n0 != take) return E_INTERNAL;
    if (int rc = wsort(w, X, take, okeys + out, oids + out, h->cur)) return rc;
    st->L[0].bsel ^= 1;
    st->L[0].nB = n1;
    st->live -= take;
    st->elems += 6ull * a0.nB;
    out += take;
    pending = true;
  }
  WCHK(hipStreamSynchronize(w->s));
  *count_out = out;
  return prof_collect(w);
}

}  // namespace bkt
