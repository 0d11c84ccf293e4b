// Chunked parallel solve of a device-memory frame cache (HBFSim, arXiv
// 2609.09800, Sections "D5: Capacity" and "D6: Speculative Prefetcher";
// FIFO replacement and next-page prefetch as read in hbf_cache.hip).
//
// Within one chunk of accesses, suppose first that nothing is evicted.  The
// resident set then only grows, so:
//  - an access can fault only as the first access of its page q in the
//    chunk, at time A(q), and only if q was not resident when the chunk
//    began (q is then a candidate);
//  - a candidate q faults iff no candidate q - k (1 <= k <= d) faulted at
//    an earlier time A(q - k) < A(q) (such a fault inserted q, or found it
//    resident).  Along the page axis this is a recurrence of width d: one
//    wave walks each segment of candidates (a gap of more than d pages
//    separates two segments), 64 pages at a time;
//  - page r is inserted at tau(r), the earliest fault among r - d .. r, if
//    it was not resident when the chunk began.  A fault's insertions are
//    numbered in page order after those of every earlier fault (a prefix
//    sum over the chunk's accesses).
// The answer is the true one as long as every residency decision it took
// holds under FIFO: each hit's page, and each prefetch candidate found
// resident, must lie within the last F insertions at that moment.  Up to the
// first access whose decision fails the two processes insert the same pages
// in the same order, so the accesses before it are committed (hit flags,
// frame flags, evictions of prefetched pages never hit, counters), the
// insertions from it on are undone, and the next chunk begins there.  Nothing
// scales with the range: per-page state is tagged with the chunk's epoch.
//
// One launch serves a whole call: a group of workgroups per cache, with a
// barrier of the group between the steps of a chunk.  Nothing relies on all of
// them running at once (a captured call may be replayed beside another, and
// kernels of other streams hold CUs): a group is whoever has started when it
// closes (group_join).  Chunks
// are as long as their checks let them be: doubled while they pass, cut to
// twice what was committed when one does not, and where next to nothing is,
// one wave takes a stretch access by access.  What bounds a chunk is the chain
// of its eight steps -- a barrier of 256 workgroups is 9 us, of one workgroup
// nothing -- and the longest segment of its walk.  1.94 M accesses of the MoE
// stream, prefetch 7 (seven launches a chunk of 110 K accesses before, and a
// chunk that failed its check served access by access):
//   frames 1.77 M  1,600 -> 400 us     frames 300 K  8,330 -> 550 us
//   frames 1.0 M   2,580 -> 410 us     frames 4,000  9,200 -> 490 us
// and 64 accesses of a run 48 -> 50 us, scattered ones 79 -> 61.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "hbf_cache_run.h"
#include "hbf_group.h"
#include "hbf_internal.h"

namespace hbf {

namespace {

constexpr uint32_t NONE32 = 0xFFFFFFFFu;

// The thread's number, hidden from the compiler: what the steps derive from it
// would otherwise all be kept through a call's chunks (68 registers spilled, a
// third of the time of a call that runs access by access).
__device__ __forceinline__ uint32_t thread_id() {
  uint32_t t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ uint32_t lane_id() { return thread_id() & 63; }
__device__ __forceinline__ uint32_t rdl(uint32_t v, uint32_t l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}
__device__ __forceinline__ uint32_t ctz64(uint64_t m) { return (uint32_t)__builtin_ctzll(m); }
__device__ __forceinline__ uint32_t popc(uint64_t m) { return (uint32_t)__popcll(m); }

__device__ __forceinline__ int64_t wave_sum(int64_t v) {
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

struct Tags {
  uint64_t a, t;  // first access (~epoch), insertion time (epoch)
  __device__ explicit Tags(uint32_t epoch) : a((uint64_t)(~epoch) << 32), t((uint64_t)epoch << 32) {}
};
constexpr uint64_t HI = 0xFFFFFFFF00000000ull;


constexpr int CBLK = 1024;          // threads per workgroup
constexpr int CWAVES = CBLK / 64;
constexpr int64_t SCAN = CBLK;      // accesses per piece of the prefix sum, one per thread
constexpr uint32_t SPIN_MAX = 1u << 24;
// A chunk of which fewer accesses than this are committed costs more than
// taking them one after another (about 0.1 us each).
constexpr uint32_t SEQ_TRY = 1024;
// A chunk most of whose candidates lie within d pages of one first accessed
// later (7 of 16; half of them is the most there can be), more than DENSE_SEG
// of them a segment, is a scattered working set seen for the first time.  The
// groups of 64 pages of its segments cost 5 us each in turn; an eighth of it
// has short ones, and makes most of the rest resident: 200,000 accesses to
// 50,000 pages, prefetch 7, 4.3 ms whole and 0.61 ms so; 30,000 accesses,
// whose segments are short, 300 us so and 136 whole.  With fewer such candidates than
// DENSE_MIN the chunk is taken as it is.
constexpr uint32_t DENSE_MIN = 4096, DENSE_SEG = 512;
constexpr uint32_t SEQ_MIN = 4096, SEQ_MAX = 1u << 17;

// How long a group waits for its workgroups to start, in ticks of 10 ns: 100 us
// (starting 256 of them takes 10 or so), and, since fewer members take longer,
// 1 ns more for each access.
constexpr uint64_t PATIENCE = 10000, PATIENCE_PER = 10;

// One group as one of its workgroups sees it: its number, the members, and
// their barrier (a counter that only grows, zero at the launch).
struct Group {
  uint32_t b, nb;
  GroupWords *words;
  uint32_t target;
  int64_t *status;
  // Of at most `want` workgroups (group_join); false: this one is not a member.
  __device__ bool join(uint32_t want, uint64_t patience) {
    struct Words {
      GroupWords *w;
      uint64_t from, patience;
      __device__ uint32_t arrive() { return atomicAdd(&w->arrived, 1u); }
      __device__ uint32_t close() { return atomicOr(&w->arrived, GROUP_CLOSED); }
      __device__ uint32_t count() { return ld(&w->members); }
      __device__ void set_count(uint32_t n) { st(&w->members, n); }
      __device__ bool wait() {
        __builtin_amdgcn_s_sleep(1);
        return __builtin_amdgcn_s_memrealtime() - from < patience;
      }
    };
    __shared__ Member s_m;
    if (want > 1) {
      if (thread_id() == 0) {
        Words w = {words, __builtin_amdgcn_s_memrealtime(), patience};
        s_m = group_join(w, want);
      }
      __syncthreads();
      b = s_m.id;
      nb = s_m.count;
    } else {
      b = 0;
      nb = 1;
    }
    return nb != 0;
  }
  // Every store of the group before is visible to every load after.  False
  // (bounded wait, never expected) ends the kernel with HBF_EINTERNAL.
  __device__ bool sync() {
    __shared__ uint32_t s_ok;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    target += nb;
    if (nb == 1) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // atomics went past the L1
      return true;
    }
    if (thread_id() == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      uint32_t *bar = &words->bar;
      __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint32_t spin = 0;
      while (!counter_reached(__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), target) &&
             ++spin < SPIN_MAX)
        __builtin_amdgcn_s_sleep(1);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      s_ok = spin < SPIN_MAX;
      if (!s_ok) st(status, (int64_t)HBF_EINTERNAL);
    }
    __syncthreads();
    const bool ok = s_ok != 0;
    return ok;
  }
  // The group's threads over [0, n); consecutive waves' shares go to different
  // workgroups, since the faults, which cost, are often all in the first few.
  __device__ int64_t first() const {
    const uint32_t t = thread_id();
    return (int64_t)(t / 64 * nb + b) * 64 + (t & 63);
  }
  __device__ int64_t step() const { return (int64_t)nb * CBLK; }
};

// Tags of the chunk's first access per page; counts cleared.
__device__ __forceinline__ void chunk_tag(const Group &gr, const ChunkCfg &cc, const uint64_t *__restrict__ pages,
                                          int64_t L, uint32_t epoch, const Tags &tg) {
  for (int64_t j = gr.first(); j < L; j += gr.step()) {
    atomicMin((unsigned long long *)&cc.at[pages[j]], (unsigned long long)(tg.a | (uint64_t)j));
    cc.S[j] = 0;
    if (j % SCAN == 0) cc.bs[j / SCAN] = 0;
  }
  if (gr.b == 0 && thread_id() == 0) {
    cc.S[L] = 0;
    cc.ctl->nseg[epoch & 1] = 0;  // (the other ones may still be read)
    cc.ctl->loose[epoch & 1] = 0;
    cc.ctl->good = (uint32_t)L;
    cc.ctl->lost_old = 0;
  }
}

// Access j is a fault of `cnt` insertions: its word of the prefix sums
// (insertions << 32 | faults).
__device__ __forceinline__ void set_fault(const ChunkCfg &cc, uint32_t j, uint32_t cnt) {
  cc.S[j] = ((uint64_t)cnt << 32) | 1u;
}

// The page word of r, if the fault at access A inserted it: its rank, else -1.
__device__ __forceinline__ int owned_rank(uint64_t v, const Tags &tg, uint32_t A) {
  return (v & (HI | 0xFFFFFFull)) == (tg.t | A) ? (int)((v >> 24) & 63u) : -1;
}

// The d + 1 pages from each of some of a workgroup's accesses on, one per lane,
// as many accesses at a time as a wave's lanes hold.  Access i of them has page
// q[i], index j[i], x[i]; load(in, i, k), then body(in, i, k, what load gave):
// the lane (if `in`) has page k of access i; a wave's lanes call it together.
// Returns the thread's i; out[i] holds what body left there, `none` if nothing.
// Each wave takes its own, or (SHARE_D pages or more) all waves share them
// out: few of them often have them all, and one access is a round (64
// scattered ones at depth 63, one wave's: 183 -> 57 us a call; at depth 7
// sharing gains 12 of 62 there, but its barriers cost runs 5 us of 68).
constexpr uint32_t SHARE_D = 16;
struct PageLds {
  uint64_t q[CBLK];
  int64_t x[CBLK];
  uint32_t j[CBLK], out[CBLK];
  uint32_t n[CWAVES];
};
template <typename Load, typename Body>
__device__ __forceinline__ uint32_t access_pages(PageLds &P, uint32_t d, bool mine, uint64_t q, uint32_t j, int64_t x,
                                                 uint32_t none, Load load, Body body) {
  constexpr uint32_t FLY = 2;  // rounds whose loads are in flight (4: the same)
  const uint64_t am = __ballot(mine);
  const uint32_t lane = lane_id(), w = thread_id() >> 6;
  const uint32_t m = d + 1, at_once = 64 / m, own = lane / m, k = lane - own * m;
  const bool share = d >= SHARE_D;  // (the same for the whole workgroup)
  uint32_t at = popc(am & ((1ull << lane) - 1)), all = popc(am);
  uint32_t from = w * 64, step = at_once;
  if (share) {
    if (lane == 0) P.n[w] = all;
    __syncthreads();
    all = 0;
    for (uint32_t i = 0; i < CWAVES; i++) {
      if (i < w) at += P.n[i];
      all += P.n[i];
    }
    from = w * at_once;
    step = at_once * CWAVES;
  } else {
    at += from;
    all += from;
  }
  if (mine) {
    P.q[at] = q;
    P.x[at] = x;
    P.j[at] = j;
    P.out[at] = none;
  }
  if (share) __syncthreads();
  else wave_lds_order();
  for (uint32_t f = from; f < all; f += FLY * step) {
    decltype(load(false, 0u, 0u)) v[FLY];
#pragma unroll
    for (uint32_t u = 0; u < FLY; u++) {
      const uint32_t i = f + u * step + own;
      const bool in = own < at_once && i < all;
      v[u] = load(in, in ? i : 0u, k);
    }
#pragma unroll
    for (uint32_t u = 0; u < FLY; u++) {
      const uint32_t i = f + u * step + own;
      const bool in = own < at_once && i < all;
      if (f + u * step < all) body(in, in ? i : 0u, k, v[u]);
    }
  }
  if (share) __syncthreads();
  else wave_lds_order();
  return at;
}
// The lanes that have the same access as this one there.
__device__ __forceinline__ uint64_t access_lanes(uint32_t d) {
  const uint32_t m = d + 1;
  return (m == 64 ? ~0ull : (1ull << m) - 1) << (lane_id() / m * m);
}

// A run: accesses j0, j0 + 1, ... to candidate pages q0, q0 + 1, ... (a
// scan).  If no candidate lies within d pages below q0, its faults are every
// (d + 1)-th access, so the walk can begin again at any multiple of d + 1
// pages into it.  It does every split_pages(d) pages (a multiple of a wave's
// 64 as well), up to SPLIT_MAX of them, each entry an own segment: a segment
// holds its first page (26 bits) and its split's number.  Without them a
// chunk waits for its longest scan, 1.1 us per 64 pages.
constexpr uint32_t SPLIT_SHIFT = 26, SPLIT_MAX = 14;
static_assert(CHUNK_MAX_R <= uint64_t(1) << SPLIT_SHIFT && SPLIT_MAX < 64, "a segment entry is one word");
__device__ __forceinline__ uint32_t split_pages(uint32_t d) {
  uint32_t p = 64, m = d + 1;  // lcm(64, d + 1)
  while (p % m) p += 64;
  return p * ((511 + p) / p);
}

// Segment starts: candidates with no candidate among the d pages below (not
// resident at the chunk's start: pins < lim), and the splits of runs.  Each
// workgroup takes consecutive pieces of CBLK accesses; a run entering its
// first is followed back as far as its splits reach.  Without prefetch every candidate is a
// fault of its own and nothing is left to walk.
__device__ __forceinline__ void chunk_starts(const Group &gr, PageLds &P, const CacheCfg &c, const ChunkCfg &cc,
                                             const uint64_t *__restrict__ pages, int64_t L, uint64_t R, int64_t lim,
                                             uint32_t epoch, const Tags &tg) {
  __shared__ int s_brk[CWAVES];
  __shared__ uint32_t s_cnt[CWAVES], s_seg;
  __shared__ uint64_t s_seen[CWAVES];
  const uint32_t lane = lane_id(), w = thread_id() >> 6, d = c.d;
  auto candidate = [&](int64_t j, uint64_t p) { return cc.at[p] == (tg.a | (uint64_t)j) && c.pins[p] < lim; };
  if (d == 0) {
    for (int64_t j = gr.first(); j < L; j += gr.step()) {
      const uint64_t p = pages[j];
      const bool f = candidate(j, p);
      const uint64_t m = __ballot(f);
      if (f) {
        cc.tt[p] = tg.t | (uint64_t)j;
        cc.S[j] = (uint64_t(1) << 32) | 1u;
        if (lane == ctz64(m))  // (a wave's accesses lie in one piece)
          atomicAdd((unsigned long long *)&cc.bs[j / SCAN], (unsigned long long)(((uint64_t(1) << 32) | 1u) * popc(m)));
      }
    }
    return;
  }
  const uint64_t group = access_lanes(d);
  // of page q (of those threads that ask): the first access of the nearest
  // candidate among the d pages below (NONE32: none)
  struct Word {
    uint64_t a;
    int64_t x;
  };
  auto before = [&](bool ask, uint64_t q) {
    auto load = [&](bool in, uint32_t i, uint32_t k) {
      const uint64_t r = P.q[i] - k;
      in = in && k > 0 && r < R;  // (wraps below page 0)
      return Word{in ? cc.at[r] : 0, in ? c.pins[r] : INT64_MAX};
    };
    const uint32_t i = access_pages(P, d, ask, q, 0, 0, NONE32, load, [&](bool in, uint32_t i, uint32_t, Word v) {
      const uint64_t m = __ballot(in && (v.a & HI) == tg.a && v.x < lim) & group;
      if (m && lane == ctz64(m)) P.out[i] = (uint32_t)v.a;
    });
    return ask ? P.out[i] : NONE32;
  };
  // A segment start with no candidate among the d pages above either is a
  // segment of its own: resolved here (page q, access j), where scattered
  // accesses would keep a wave each busy.  Whether it is one.
  auto alone = [&](bool ask, uint64_t q, uint32_t j) {
    auto load = [&](bool in, uint32_t i, uint32_t k) {
      const uint64_t r = P.q[i] + k;
      in = in && r < R;
      return Word{in && k > 0 ? cc.at[r] : 0, in ? c.pins[r] : INT64_MAX};
    };
    const uint32_t i = access_pages(P, d, ask, q, j, 0, 0, load, [&](bool in, uint32_t i, uint32_t k, Word v) {
      const bool ins = in && v.x < lim;  // not resident
      const uint64_t im = __ballot(ins) & group, cm = __ballot(ins && (v.a & HI) == tg.a) & group;
      if (cm || !ins) return;
      cc.tt[P.q[i] + k] = tg.t | (uint64_t)popc(im & ((1ull << lane) - 1)) << 24 | P.j[i];
      if (k == 0) {
        set_fault(cc, P.j[i], popc(im));
        P.out[i] = 1;
      }
    });
    return ask && P.out[i] != 0;
  };
  // whether access j goes on from access j - 1 in a run
  auto linked = [&](int64_t j) {
    if (j <= 0 || j >= L) return false;
    const uint64_t p = pages[j], p1 = pages[j - 1];
    return p == p1 + 1 && candidate(j, p) && candidate(j - 1, p1);
  };
  // the last access of this piece's at or before the thread's that does not
  // go on from its predecessor (-1: none); all: the piece's last one
  auto last_break = [&](int64_t j, bool brk, int &all) {
    int x = brk ? (int)j : -1;
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o);
      if (lane >= (uint32_t)o) x = max(x, y);
    }
    if (lane == 63) s_brk[w] = x;
    __syncthreads();
    all = -1;
    for (int i = 0; i < CWAVES; i++) {
      if (i < (int)w) x = max(x, s_brk[i]);
      all = max(all, s_brk[i]);
    }
    __syncthreads();
    return x;
  };
  const uint32_t W = split_pages(d);
  const uint32_t splits = min(SPLIT_MAX, (uint32_t)(7 * CBLK) / W);  // a run is followed back 7 pieces
  const int64_t per = ((L + CBLK - 1) / CBLK + gr.nb - 1) / gr.nb * CBLK;
  const int64_t a0 = (int64_t)gr.b * per, a1 = min(L, a0 + per);
  uint64_t seen = 0;  // the wave's candidates outside runs (low word), those near one accessed later (high)
  int in = -1;  // start of the run that the piece's first access goes on from (-1: not known)
  for (int64_t c0 = a0; c0 < a1; c0 += CBLK) {
    const int64_t j = c0 + thread_id();
    const bool lk = linked(j);
    int all = -1;
    int run = last_break(j, !lk, all);
    if (c0 == a0 && __syncthreads_or(thread_id() == 0 && lk)) {
      int back = -1;
      for (int64_t b0 = c0 - CBLK; b0 >= 0 && b0 >= c0 - 7 * CBLK && back < 0; b0 -= CBLK)
        last_break(b0 + thread_id(), !linked(b0 + thread_id()), back);
      in = back;
    }
    if (run < 0) run = in;
    if (all >= 0) in = all;  // for the next piece
    bool ask = false, loose = false;
    uint64_t p = 0, q = 0;  // its page; the page whose neighbours say whether a segment starts
    uint32_t split = 0;
    if (j < L) {
      p = q = pages[j];
      if (lk) {
        const uint32_t o = run < 0 ? 1u : (uint32_t)((int)j - run);  // pages into the run
        ask = o % W == 0 && o / W <= splits;
        if (ask) {
          q = pages[run];
          split = o / W;
        }
      } else {
        ask = loose = candidate(j, p);
      }
    }
    const uint32_t near = before(ask, q);
    const bool late = loose && near != NONE32 && near > (uint32_t)j;
    bool start = ask && near == NONE32;
    if (alone(start && loose, p, (uint32_t)j)) start = false;
    const uint32_t entry = (uint32_t)p | split << SPLIT_SHIFT;
    // A place in the list for the piece's starts (all waves asking for theirs
    // one by one waited for each other: 200,000 accesses in runs of 16 pages 184
    // us, and 121 so).
    const uint64_t sm = __ballot(start);
    seen += (uint64_t)popc(__ballot(late)) << 32 | popc(__ballot(loose));
    if (lane == 0) s_cnt[w] = popc(sm);
    __syncthreads();
    uint32_t k = popc(sm & ((1ull << lane) - 1)), starts = 0;
    for (uint32_t i = 0; i < CWAVES; i++) {
      if (i < w) k += s_cnt[i];
      starts += s_cnt[i];
    }
    if (starts) {  // (the same for the whole workgroup)
      if (thread_id() == 0) s_seg = atomicAdd(&cc.ctl->nseg[epoch & 1], starts);
      __syncthreads();
      k += s_seg;
      if (start && k < cc.Lmax) cc.seg[k] = entry;
    }
  }
  if (lane == 0) s_seen[w] = seen;
  __syncthreads();
  if (thread_id() == 0) {
    for (uint32_t i = 1; i < CWAVES; i++) seen += s_seen[i];
    if (seen) atomicAdd((unsigned long long *)&cc.ctl->loose[epoch & 1], (unsigned long long)seen);
  }
}
}  // namespace

// One wave per segment: faults, insertion times, per-fault insertion
// counts and each insertion's rank within its fault, all written as plain
// stores (the tagged per-page word and the fault's count), so that the
// page state of the next four groups stays in flight while one is resolved.
namespace {
struct Walk {
  uint64_t lastc;   // last candidate of the segment so far
  uint32_t pa;      // previous group: this lane's first-access time
  uint64_t open;    // previous group: faults whose windows reach this group
  uint32_t pcnt;    // previous group: insertions so far of this lane's open fault
  uint32_t lastA;   // previous group: the largest first-access time among its candidates
  bool hasA;
};

// Resolve the 64 pages at `base`; returns true once the segment has ended.
//
// Where the candidates' first-access times increase along the pages (a
// scan) and at most one fault reaches in from the previous group, every
// earlier fault within d pages blocks a candidate, so the faults are the
// greedy choice of candidates more than d pages apart, each page lies in
// at most one fault's window, and insertion time, rank and per-fault
// counts follow per lane.  Other groups take the general path: the lowest
// candidate not blocked by an earlier fault of smaller time is a fault.
__device__ __forceinline__ bool walk_group(Walk &w, uint64_t base, uint64_t at_c, int64_t pin_c, uint64_t R,
                                           uint32_t d, int64_t lim, const Tags &tg, const ChunkCfg &cc) {
  const uint32_t lane = lane_id();
  const uint64_t lt = (1ull << lane) - 1;
  const uint64_t le = lane == 63 ? ~0ull : (2ull << lane) - 1;
  const uint64_t r = base + lane;
  const bool inR = r < R;
  const uint32_t a = inR && (at_c & HI) == tg.a ? (uint32_t)at_c : NONE32;
  const bool nonres = inR && pin_c < lim;
  const bool cand = a != NONE32 && nonres;
  const uint64_t cm = __ballot(cand);
  const uint32_t af0 = rdl(a, 0);
  if (cm == ~0ull && !__ballot(a != af0 + lane) && popc(w.open) <= 1 && !(w.hasA && w.lastA >= af0) &&
      base + 64 < R && base - w.lastc <= d) {
    // a scan's middle: every (d + 1)-th page is a fault, beginning after the
    // window of the one that reaches in
    const uint32_t m = d + 1;
    uint32_t x = 0, g = 0, ag = 0, c0 = 0;
    if (w.open) {
      g = ctz64(w.open);
      x = g + m - 64;
      ag = rdl(w.pa, g);
      c0 = rdl(w.pcnt, g);
    }
    const uint32_t q = (((lane - x) & 0xFFu) * (65536u / m + 1)) >> 16;  // (lane - x) / m from lane x on
    const uint32_t f = x + q * m;
    const bool in = lane >= x;
    if (x && lane == g) set_fault(cc, w.pa, c0 + x);
    const bool flt = in && lane == f, whole = lane + d < 64;
    if (flt && whole) set_fault(cc, a, m);
    cc.tt[r] = tg.t | ((uint64_t)(in ? lane - f : c0 + lane) << 24) | (in ? af0 + f : ag);
    w.open = __ballot(flt && !whole);
    w.pa = a;
    w.pcnt = 64 - lane;
    w.lastc = base + 63;
    w.lastA = af0 + 63;
    w.hasA = true;
    return false;
  }
  // the segment continues while candidates are at most d pages apart
  const uint64_t below = cm & lt;
  const uint64_t prevpos = below ? base + 63 - (uint64_t)__builtin_clzll(below) : w.lastc;
  const uint64_t brk = __ballot(cand && r - prevpos > d);
  const uint64_t segc = brk ? (cm & ((1ull << ctz64(brk)) - 1)) : cm;
  if (segc) w.lastc = base + 63 - (uint64_t)__builtin_clzll(segc);
  const bool in_ext = inR && r <= w.lastc + d;
  const bool last = !(w.lastc + d >= base + 64 && base + 64 < R);
  // do the candidates of this group and the one before it (none further away
  // matters, d < 64) have increasing first-access times?
  const bool sc = (segc >> lane) & 1;
  const uint64_t sbelow = segc & lt;
  const uint32_t apl = (uint32_t)__shfl((int)a, sbelow ? 63 - __builtin_clzll(sbelow) : lane);
  const bool viol = sc && (sbelow ? apl >= a : (w.hasA && w.lastA >= a));
  const bool mono = !__ballot(viol) && popc(w.open) <= 1;

  uint64_t fm = 0, nopen = 0;
  uint32_t tau = NONE32, rank = 0, cnt = 0, ncnt = 0;
  bool fin_prev = false, fin_cur = false, ins = false;
  if (mono) {
    uint64_t rem = segc;
    const uint32_t g = w.open ? ctz64(w.open) : 0;
    if (w.open) rem &= ~((2ull << (g + d - 64)) - 1);  // lanes within the open fault's window
    while (rem) {
      const uint32_t f = ctz64(rem);
      fm |= 1ull << f;
      rem = f + d >= 63 ? 0 : rem & ~((2ull << (f + d)) - 1);
    }
    const uint64_t fb = fm & le;
    const uint32_t fs = fb ? 63 - __builtin_clzll(fb) : lane;
    const uint32_t af = (uint32_t)__shfl((int)a, fs);
    const bool cov = fb && lane - fs <= d;
    const uint32_t ag = w.open ? rdl(w.pa, g) : NONE32;
    const uint32_t c0 = w.open ? rdl(w.pcnt, g) : 0;
    const bool cov_prev = !cov && w.open && lane + 64 - g <= d;
    tau = cov ? af : (cov_prev ? ag : NONE32);
    ins = in_ext && tau != NONE32 && nonres;
    const uint64_t im = __ballot(ins);
    rank = cov ? popc(im & lt & ~((1ull << fs) - 1)) : c0 + popc(im & lt);
    if (w.open && lane == g) {
      fin_prev = true;
      ncnt = c0 + popc(im & ((2ull << (g + d - 64)) - 1));
    }
    if ((fm >> lane) & 1) {
      const uint64_t win = (lane + d >= 63 ? ~0ull : (2ull << (lane + d)) - 1) & ~lt;
      cnt = popc(im & win);
      fin_cur = lane + d < 64 || last;
    }
    nopen = __ballot(((fm >> lane) & 1) && !fin_cur);
  } else {
    uint64_t rem = segc;
    for (uint64_t m = w.open; m; m &= m - 1) {
      const uint32_t g = ctz64(m);
      const uint32_t ag = rdl(w.pa, g);
      const bool near = lane + 64 - g <= d;
      rem &= ~__ballot(near && ag < a);
      if (near) tau = ag < tau ? ag : tau;
    }
    while (rem) {
      const uint32_t f = ctz64(rem);
      fm |= 1ull << f;
      const uint32_t af = rdl(a, f);
      rem &= ~(1ull << f);
      const bool near = lane >= f && lane - f <= d;
      rem &= ~__ballot(near && af < a);
      // insertion time: the earliest fault whose window holds this page
      if (near) tau = af < tau ? af : tau;
    }
    ins = in_ext && tau != NONE32 && nonres;
    for (uint64_t m = w.open; m; m &= m - 1) {  // windows that end in this group
      const uint32_t g = ctz64(m);
      const uint32_t ag = rdl(w.pa, g);
      const bool mine = ins && tau == ag;
      const uint64_t mm = __ballot(mine);
      const uint32_t c0 = rdl(w.pcnt, g);
      if (mine) rank = c0 + popc(mm & lt);
      if (lane == g) {
        fin_prev = true;
        ncnt = c0 + popc(mm);  // the count of the previous group's fault in this lane
      }
    }
    for (uint64_t m = fm; m; m &= m - 1) {
      const uint32_t f = ctz64(m);
      const uint32_t af = rdl(a, f);
      const bool mine = ins && tau == af;
      const uint64_t mm = __ballot(mine);
      if (mine) rank = popc(mm & lt);
      if (lane == f) cnt = popc(mm);
      if (f + d < 64 || last) {
        if (lane == f) fin_cur = true;
      } else {
        nopen |= 1ull << f;
      }
    }
  }
  // the largest first-access time among the group's candidates
  if (segc) {
    uint32_t mx = sc ? a : 0;
    if (mono) {
      mx = rdl(a, 63 - __builtin_clzll(segc));
    } else {
      for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t y = (uint32_t)__shfl_xor((int)mx, o);
        mx = y > mx ? y : mx;
      }
      mx = rdl(mx, 0);
    }
    w.lastA = mx;
    w.hasA = true;
  }
  // per-fault counts (packed: insertions << 32 | 1) and the page words
  if (fin_prev) set_fault(cc, w.pa, ncnt);
  if (fin_cur) set_fault(cc, a, cnt);
  if (ins) cc.tt[r] = tg.t | ((uint64_t)rank << 24) | tau;
  w.pa = a;
  w.open = nopen;
  w.pcnt = cnt;
  return last;
}
}  // namespace

namespace {
__device__ __forceinline__ void chunk_walk(const Group &gr, const CacheCfg &c, const ChunkCfg &cc, uint64_t R,
                                           int64_t lim, uint32_t epoch, const Tags &tg) {
  const uint32_t lane = lane_id(), d = c.d;
  const uint32_t nseg_all = ld(&cc.ctl->nseg[epoch & 1]);
  const uint32_t nseg = nseg_all < cc.Lmax ? nseg_all : cc.Lmax;
  const uint32_t W = split_pages(d), splits = min(SPLIT_MAX, (uint32_t)(7 * CBLK) / W);
  // page state, loaded unconditionally (addresses clamped into the range;
  // lanes past the end are masked when the group is resolved)
  const gptr<const uint64_t> atg = (gptr<const uint64_t>)cc.at;
  const gptr<const int64_t> ping = (gptr<const int64_t>)c.pins;
  auto at_of = [&](uint64_t base) { return atg[base + lane < R ? base + lane : R - 1]; };
  auto pin_of = [&](uint64_t base) { return ping[base + lane < R ? base + lane : R - 1]; };
  // (consecutive segments to different workgroups)
  for (uint32_t si = thread_id() / 64 * gr.nb + gr.b; si < nseg; si += gr.nb * CWAVES) {
    const uint32_t entry = ld(&cc.seg[si]), split = entry >> SPLIT_SHIFT;
    const uint64_t s = entry & ((1u << SPLIT_SHIFT) - 1);
    Walk w{s, NONE32, 0, 0, 0, false};
    uint32_t as = 0;                 // first access of page s
    bool run = split < splits;       // pages s .. so far are a run, which the next split may take on
    // the next four groups in flight
    uint64_t a0 = at_of(s), a1 = at_of(s + 64), a2 = at_of(s + 128), a3 = at_of(s + 192);
    int64_t p0 = pin_of(s), p1 = pin_of(s + 64), p2 = pin_of(s + 128), p3 = pin_of(s + 192);
    for (uint64_t base = s;; base += 64) {
      const uint64_t at_c = a0;
      const int64_t pin_c = p0;
      a0 = a1;
      p0 = p1;
      a1 = a2;
      p1 = p2;
      a2 = a3;
      p2 = p3;
      a3 = at_of(base + 256);
      p3 = pin_of(base + 256);
      const bool end = walk_group(w, base, at_c, pin_c, R, d, lim, tg, cc);
      if (end) break;
      if (run) {
        if (base == s) as = rdl((uint32_t)at_c, 0);
        const uint32_t o = (uint32_t)(base - s);
        run = !__ballot(!((at_c & HI) == tg.a && pin_c < lim && (uint32_t)at_c == as + o + lane));
        // (the split's page is the first of the next group)
        if (run && o + 64 == W) {
          if (__ballot(lane == 0 && (a0 & HI) == tg.a && p0 < lim && (uint32_t)a0 == as + W)) break;
          run = false;
        }
      }
    }
  }
}

// The sum of each piece's counts.  (Added up by atomics where the faults are
// found, a walk's loads wait behind them: a scan took 0.83 us and not 0.65
// per 64 pages.)
__device__ __forceinline__ void chunk_sums(const Group &gr, const ChunkCfg &cc, int64_t L) {
  __shared__ uint64_t part[CWAVES];
  for (int64_t q = gr.b; q * SCAN < L; q += gr.nb) {
    const int64_t j = q * SCAN + thread_id();
    uint64_t v = j < L ? cc.S[j] : 0;
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if (lane_id() == 0) part[thread_id() >> 6] = v;
    __syncthreads();
    if (thread_id() == 0) {
      uint64_t t = 0;
      for (int w = 0; w < CWAVES; w++) t += part[w];
      cc.bs[q] = t;
    }
    __syncthreads();
  }
}

// Exclusive scan of the packed per-access counts: each piece's own, offset by
// the sums of the pieces before it; then each fault in the piece (an access j whose page word names j
// itself, rank 0) numbers its insertions: I0 + insertions before j + rank.
__device__ __forceinline__ void chunk_scan(const Group &gr, PageLds &P, const CacheCfg &c, const ChunkCfg &cc,
                                           const uint64_t *__restrict__ pages, int64_t L, uint64_t R, int64_t I0,
                                           const Tags &tg) {
  __shared__ uint64_t part[CWAVES], before[CWAVES];
  const uint32_t lane = lane_id(), w = thread_id() >> 6;
  uint64_t pre = 0;  // the sums of the pieces before q
  int64_t done = 0;  // pieces in it
  for (int64_t q = gr.b; q * SCAN < L; q += gr.nb) {
    uint64_t p = 0;
    for (int64_t i = done + thread_id(); i < q; i += CBLK) p += cc.bs[i];
    for (int o = 32; o >= 1; o >>= 1) p += __shfl_xor(p, o);
    if (lane == 0) before[w] = p;
    const int64_t j = q * SCAN + thread_id();
    const uint64_t v = j < L ? cc.S[j] : 0;
    uint64_t x = v;  // inclusive scan within the wave
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t y = __shfl_up(x, o);
      if (lane >= (uint32_t)o) x += y;
    }
    if (lane == 63) part[w] = x;
    __syncthreads();
    for (int i = 0; i < CWAVES; i++) pre += before[i];
    uint64_t off = pre;
    for (uint32_t i = 0; i < w; i++) off += part[i];
    __syncthreads();
    done = q;
    const uint64_t sj = off + x - v;
    if (j < L) cc.S[j] = sj;
    if (j == L - 1) cc.S[L] = off + x;
    const bool fault = v != 0;
    const uint64_t pg = fault ? pages[j] : 0;
    const int64_t x0 = I0 + (int64_t)(sj >> 32);
    auto load = [&](bool in, uint32_t i, uint32_t k) {
      const uint64_t r = P.q[i] + k;
      return in && r < R ? cc.tt[r] : 0;
    };
    access_pages(P, c.d, fault, pg, (uint32_t)j, x0, 0, load, [&](bool, uint32_t i, uint32_t k, uint64_t t) {
      const int rk = owned_rank(t, tg, P.j[i]);
      if (rk >= 0) c.pins[P.q[i] + k] = P.x[i] + rk;
    });
  }
}

// The check: the first access whose decision does not hold -- a hit on a
// page, or a fault that found a prefetch candidate resident, not within the
// last F insertions at that moment -- into ctl->good.
__device__ __forceinline__ void chunk_check(const Group &gr, PageLds &P, const CacheCfg &c, const ChunkCfg &cc,
                                            const uint64_t *__restrict__ pages, int64_t L, uint64_t R, int64_t I0,
                                            const Tags &tg) {
  uint32_t bad = NONE32;
  const uint32_t lane = lane_id();
  const uint64_t group = access_lanes(c.d);
  struct Word {
    uint64_t t;
    int64_t x;
  };
  const int64_t first = gr.first();
  for (int64_t j0 = 0; j0 < L; j0 += gr.step()) {  // workgroups stay together
    const int64_t j = j0 + first;
    const uint64_t p = j < L ? pages[j] : 0;
    const int64_t low = j < L ? I0 + (int64_t)(cc.S[j] >> 32) - (int64_t)c.F : 0;  // resident at j: pins >= low
    const bool fault = j < L && cc.tt[p] == (tg.t | (uint64_t)j);
    if (j < L && !fault && c.pins[p] < low) bad = min(bad, (uint32_t)j);
    if (c.d == 0) continue;
    auto load = [&](bool in, uint32_t i, uint32_t k) {
      const uint64_t r = P.q[i] + k;
      in = in && r < R;
      return Word{in ? cc.tt[r] : 0, in ? c.pins[r] : INT64_MAX};  // (past the range: never a failure)
    };
    access_pages(P, c.d, fault, p, (uint32_t)j, low, 0, load, [&](bool in, uint32_t i, uint32_t, Word v) {
      const uint32_t jf = P.j[i];
      const bool own = in && owned_rank(v.t, tg, jf) >= 0;
      // the fault's insertions before this candidate
      const uint64_t before = __ballot(own) & group & ((1ull << lane) - 1);
      if (in && !own && v.x < P.x[i] + (int64_t)popc(before)) bad = min(bad, jf);
    });
  }
  for (int o = 32; o >= 1; o >>= 1) bad = min(bad, (uint32_t)__shfl_xor((int)bad, o));
  if (lane_id() == 0 && bad != NONE32) atomicMin(&cc.ctl->good, bad);
}

// Frames filled before the chunk and evicted by its first T accesses that
// hold a prefetched page never hit (read before any flag changes; a page
// resident at the start and accessed was hit before its eviction).
__device__ __forceinline__ void chunk_lost(const Group &gr, const CacheCfg &c, const ChunkCfg &cc,
                                           const uint64_t *__restrict__ pages, int64_t T, int64_t I0, int64_t I1,
                                           const Tags &tg) {
  const int64_t F = c.F;
  const int64_t ylo = I0 - F > 0 ? I0 - F : 0, yhi = I1 - F < I0 ? I1 - F : I0;
  if (yhi <= ylo) return;  // nothing of before is evicted
  int64_t lost = 0;
  for (int64_t j = gr.first(); j < T; j += gr.step()) {
    const uint64_t p = pages[j];
    if (cc.at[p] != (tg.a | (uint64_t)j)) continue;
    const int64_t x = c.pins[p];
    if (x >= ylo && x < yhi) {
      const uint64_t fr = (uint64_t)x % (uint64_t)F;
      lost -= (c.fpf[fr] && !c.fhit[fr]) ? 1 : 0;
    }
  }
  for (int64_t y = ylo + gr.first(); y < yhi; y += gr.step()) {
    const uint64_t fr = (uint64_t)y % (uint64_t)F;
    lost += (c.fpf[fr] && !c.fhit[fr]) ? 1 : 0;
  }
  lost = wave_sum(lost);
  if (lane_id() == 0 && lost) atomicAdd((unsigned long long *)&cc.ctl->lost_old, (unsigned long long)lost);
}

// Commit of the first T accesses: hit flags; a hit on a page resident at the
// start marks its frame; each fault's insertions still resident set their
// frame flags, those evicted meanwhile count as unused when prefetched and
// never hit, prefetch outputs; then the counters.  The insertions of later
// faults are undone (a page not resident at the start stays so).  The frames
// written here are distinct: they hold the last F insertions.
__device__ __forceinline__ void chunk_commit(const Group &gr, PageLds &P, const CacheCfg &c, const ChunkCfg &cc,
                                             const uint64_t *__restrict__ pages, int64_t c0, int64_t L, int64_t T,
                                             uint64_t R, int64_t I0, int64_t npf0, const Tags &tg, uint8_t *hit,
                                             uint64_t *pf_page, int64_t *pf_src, int64_t pf_cap, int64_t *n_pf) {
  const uint64_t tot = ld(&cc.S[T]);
  const int64_t F = c.F, nf = (uint32_t)tot, M = (int64_t)(tot >> 32), I1 = I0 + M;
  int64_t lost = 0;
  const int64_t first = gr.first();
  for (int64_t j0 = 0; j0 < L; j0 += gr.step()) {  // workgroups stay together
    const int64_t j = j0 + first;
    const uint64_t p = j < L ? pages[j] : 0;
    const bool fault = j < L && cc.tt[p] == (tg.t | (uint64_t)j), ok = j < T;
    if (ok && hit) hit[c0 + j] = fault ? 0 : 1;
    if (ok && !fault && cc.at[p] == (tg.a | (uint64_t)j)) {
      const int64_t x = c.pins[p];
      if (x >= I1 - F && x < I0) c.fhit[(uint64_t)x % (uint64_t)F] = 1;
    }
    const uint64_t sj = fault ? cc.S[j] : 0;
    const int64_t pf0 = npf0 + (int64_t)(sj >> 32) - (int64_t)(uint32_t)sj - 1;  // prefetch reads before, less 1
    struct Word {
      uint64_t t, a;
      int64_t x;
    };
    auto load = [&](bool in, uint32_t i, uint32_t k) {
      const uint64_t r = P.q[i] + k;
      in = in && r < R;
      return Word{in ? cc.tt[r] : 0, in ? cc.at[r] : 0, in ? c.pins[r] : 0};
    };
    access_pages(P, c.d, fault, p, (uint32_t)j, pf0, 0, load, [&](bool, uint32_t i, uint32_t k, Word v) {
      const uint64_t r = P.q[i] + k;
      const uint32_t jf = P.j[i];
      const int64_t q = P.x[i];
      const int rk = owned_rank(v.t, tg, jf);
      if (rk < 0) return;
      if ((int64_t)jf >= T) {
        c.pins[r] = PINS_NEVER;
        return;
      }
      // (a prefetched page is hit from its first access on)
      const bool used = rk > 0 && (v.a & HI) == tg.a && (int64_t)(uint32_t)v.a < T;
      const int64_t x = v.x;
      if (x >= I1 - F) {
        const uint64_t fr = (uint64_t)x % (uint64_t)F;
        c.fpf[fr] = rk > 0 ? 1 : 0;
        c.fhit[fr] = used ? 1 : 0;
      } else {
        lost += (rk > 0 && !used) ? 1 : 0;
      }
      if (pf_page && rk > 0 && q + rk < pf_cap) {
        pf_page[q + rk] = r;
        pf_src[q + rk] = c0 + (int64_t)jf;
      }
    });
  }
  lost = wave_sum(lost);
  if (gr.b == 0 && thread_id() == 0) {
    lost += ld(&cc.ctl->lost_old);
    c.ctl->count[0] += T - nf;
    c.ctl->count[1] += nf;
    c.ctl->count[2] += M - nf;
    c.ctl->ins = I1;
    c.ctl->head = (uint32_t)((uint64_t)I1 % (uint64_t)F);
    c.ctl->pend = 0;
    if (n_pf) *n_pf = npf0 + M - nf;
  }
  if (lane_id() == 0 && lost) atomicAdd((unsigned long long *)&c.ctl->count[4], (unsigned long long)lost);
}

__device__ __forceinline__ void chunk_clear(const Group &gr, const ChunkCfg &cc, uint64_t R) {
  for (uint64_t q = (uint64_t)gr.first(); q < R; q += (uint64_t)gr.step()) {
    cc.at[q] = ~0ull;
    cc.tt[q] = 0;
  }
}
}  // namespace

struct ChunkRun {
  const CacheCfg *cfgs;
  const ChunkCfg *ccs;
  const int *ids;
  int n_ids;
  uint32_t groups;
  uint64_t R;
  const uint64_t *pages;
  int64_t n;
  uint32_t chunk;  // accesses per chunk, 0: as many as pass
  uint8_t *hit;
  uint64_t *pf_page;
  int64_t *pf_src;
  int64_t pf_cap;
  int64_t *status, *n_pf;
  GroupWords *words;  // one entry per group
};

__global__ __launch_bounds__(CBLK) void k_chunk_run(ChunkRun A) {
  __shared__ union {  // a barrier lies between their uses
    RunLds run;
    PageLds pages;
  } S;
  // A page outside the range: nothing changes.  (One thread reads the word
  // for all: a barrier that runs out writes it during the launch.)
  __shared__ uint32_t s_go;
  if (threadIdx.x == 0) s_go = ld(A.status) == 0;
  __syncthreads();
  if (!s_go) return;
  const uint32_t want = gridDim.x / A.groups, grp = blockIdx.x / want;
  if (grp >= A.groups) return;
  Group gr = {0, 0, A.words + grp, 0, A.status};
  if (!gr.join(want, PATIENCE + (uint64_t)A.n / PATIENCE_PER)) return;
  for (int ci = (int)grp; ci < A.n_ids; ci += (int)A.groups) {
    const int id = A.ids[ci];
    CacheCfg c = A.cfgs[id];
    ChunkCfg cc = A.ccs[id];
    const bool first = ci == 0;
    uint64_t *pf_page = first ? A.pf_page : nullptr;
    int64_t *n_pf = first ? A.n_pf : nullptr;
    uint8_t *hit = A.hit;  // (a single cache's)
    const uint32_t most = A.chunk ? A.chunk : cc.Lmax;
    uint32_t len = A.chunk ? A.chunk : min(cc.Lmax, CHUNK_FIRST), seq = SEQ_MIN;
    uint32_t epoch = ld(&cc.ctl->epoch);
    int64_t pos = 0;
    // A barrier of the chunk.  Where it runs out the call ends, and later ones
    // begin past every tag in use (workgroups are at most one chunk apart).
    auto meet = [&]() {
      if (gr.sync()) return true;
      if (threadIdx.x == 0) atomicMax(&cc.ctl->epoch, epoch + 2);
      return false;
    };
    while (pos < A.n) {  // (all of it the same on every workgroup of the group)
      if (epoch >= 0xFFFFFF00u) {  // tags about to repeat
        chunk_clear(gr, cc, A.R);
        epoch = 0;
        if (!meet()) return;
      }
      const Tags tg(++epoch);
      const uint64_t *pages = A.pages + pos;
      const int64_t L = A.n - pos < (int64_t)len ? A.n - pos : (int64_t)len;
      const int64_t I0 = ld(&c.ctl->ins), lim = I0 - (int64_t)c.F, npf0 = n_pf ? ld(n_pf) : 0;
      chunk_tag(gr, cc, pages, L, epoch, tg);
      if (!meet()) return;
      chunk_starts(gr, S.pages, c, cc, pages, L, A.R, lim, epoch, tg);
      if (!meet()) return;
      const uint32_t nseg = ld(&cc.ctl->nseg[epoch & 1]);
      if (!A.chunk) {
        const uint64_t lw = ld(&cc.ctl->loose[epoch & 1]);
        const uint32_t loose = (uint32_t)lw, late = (uint32_t)(lw >> 32);
        if (loose >= DENSE_MIN && late > loose / 16 * 7 && nseg < loose / DENSE_SEG) {
          len = (uint32_t)(L / 8);  // begin again with less
          continue;
        }
      }
      if (c.d > 0) {
        if (nseg) {  // (scattered accesses are resolved already)
          chunk_walk(gr, c, cc, A.R, lim, epoch, tg);
          if (!meet()) return;
        }
        chunk_sums(gr, cc, L);
        if (!meet()) return;
      }
      chunk_scan(gr, S.pages, c, cc, pages, L, A.R, I0, tg);
      if (!meet()) return;
      chunk_check(gr, S.pages, c, cc, pages, L, A.R, I0, tg);
      if (!meet()) return;
      const int64_t T = ld(&cc.ctl->good);
      const int64_t I1 = I0 + (int64_t)(ld(&cc.S[T]) >> 32);
      if (I1 > (int64_t)c.F && I0 > 0) {  // frames of before are evicted
        chunk_lost(gr, c, cc, pages, T, I0, I1, tg);
        if (!meet()) return;
      }
      chunk_commit(gr, S.pages, c, cc, pages, pos, L, T, A.R, I0, npf0, tg, hit, pf_page, A.pf_src, A.pf_cap, n_pf);
      pos += T;
      if (pos >= A.n) break;  // nothing of this cache is read again
      if (!meet()) return;
      if (T == L) {
        len = min(len > most / 2 ? most : len * 2, most);
        seq = SEQ_MIN;
        continue;
      }
      len = (uint32_t)min((int64_t)most, max((int64_t)2 * T, (int64_t)SEQ_TRY));
      if (T >= SEQ_TRY) continue;
      const int64_t m = A.n - pos < (int64_t)seq ? A.n - pos : (int64_t)seq;
      if (gr.b == 0 && thread_id() < 64)
        cache_run_wave(c, S.run, A.R, A.pages + pos, m, hit ? hit + pos : nullptr, pf_page, A.pf_src, A.pf_cap, n_pf,
                       pos);
      {  // (read again, so as not to hold its registers through the run)
        int again = __builtin_amdgcn_readfirstlane(id);
        asm volatile("" : "+s"(again));
        c = A.cfgs[again];
        cc = A.ccs[again];
      }
      if (!meet()) return;
      pos += m;
      seq = min(seq * 2, SEQ_MAX);
      len = min(most, CHUNK_MIN);
    }
    if (gr.b == 0 && thread_id() == 0) cc.ctl->epoch = epoch;
  }
}

__global__ __launch_bounds__(256) void k_chunk_clear(const ChunkCfg *__restrict__ ccs, const int *ids, uint64_t R) {
  const ChunkCfg cc = ccs[ids[blockIdx.y]];
  for (uint64_t q = (uint64_t)blockIdx.x * 256 + thread_id(); q < R; q += (uint64_t)gridDim.x * 256) {
    cc.at[q] = ~0ull;
    cc.tt[q] = 0;
  }
  if (blockIdx.x == 0 && thread_id() == 0) cc.ctl->epoch = 0;
}

hipError_t launch_chunk_clear(const ChunkCfg *dev_ccfgs, const int *cfg_ids, int n_cfg, uint64_t R, hipStream_t s) {
  uint64_t b = (R + 255) / 256;
  if (b > 2048) b = 2048;
  hipLaunchKernelGGL(k_chunk_clear, dim3((uint32_t)b, (uint32_t)n_cfg), dim3(256), 0, s, dev_ccfgs, cfg_ids, R);
  return hipGetLastError();
}

// A workgroup for each 512 accesses, above 64 of them for each 2,048:
// scattered faults and short runs want waves, a barrier costs more the more
// workgroups meet.  10,000 accesses to 50,000 pages 115 us at one per 1,024, 94
// at one per 512; 200,000 of them 433 at one per 1,024, 358 at one per 2,048.
static int64_t chunk_share(int64_t n) {
  return std::max((n + 2 * CBLK - 1) / (2 * CBLK), std::min((n + CBLK / 2 - 1) / (CBLK / 2), (int64_t)64));
}

hipError_t launch_cache_chunks(const CacheCfg *cfgs, const ChunkCfg *ccs, const int *ids, int n_cfg, uint64_t R,
                               const uint64_t *pages, int64_t n, uint32_t chunk, uint8_t *hit, uint64_t *pf_page,
                               int64_t *pf_src, int64_t pf_cap, int64_t *status, int64_t *n_pf, GroupWords *words,
                               hipStream_t s) {
  // one workgroup per CU: a barrier's cost grows with them
  int dev = 0, blocks = 0;
  hipError_t e;
  if ((e = hipGetDevice(&dev)) != hipSuccess ||
      (e = hipDeviceGetAttribute(&blocks, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
    return e;
  ChunkRun A = {cfgs, ccs, ids, n_cfg, 0, R, pages, n, chunk, hit, pf_page, pf_src, pf_cap, status, n_pf, words};
  // no more workgroups than a short call, or its chunks, have work for
  const int64_t use = chunk_share(chunk ? std::min(n, (int64_t)chunk) : n) * n_cfg;
  if (use < blocks) blocks = (int)use;
  A.groups = (uint32_t)std::min(std::min(n_cfg, blocks), CHUNK_GROUPS);
  hipLaunchKernelGGL(k_chunk_run, dim3((uint32_t)blocks), dim3(CBLK), 0, s, A);
  return hipGetLastError();
}

}  // namespace hbf
