// One wave runs one device-memory frame cache, one access after another:
// shared by the sequential kernel and the chunked solve, which hands it the
// stretches it cannot take in parallel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hbf_internal.h"

namespace hbf {

__device__ __forceinline__ uint32_t lane_no() { return __lane_id(); }

// Device-memory accesses of the cache state, as global (not flat)
// instructions: a flat access also counts against the LDS wait counter, so
// every later LDS wait would wait for it too.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ T ld(const T *p) {
  return __hip_atomic_load((gptr<const T>)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st(T *p, T v) {
  __hip_atomic_store((gptr<T>)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ int64_t read_lane(int64_t v, uint32_t l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), (int)l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}


// ---- caches of more than CACHE_LDS_MAX frames: state in device memory
//
// With FIFO replacement the resident pages are exactly the last F pages
// inserted (a page is inserted only when absent, so those F are distinct):
// after I insertions, the page of insertion x is resident iff x >= I - F.
// The state is therefore the number of each page's latest insertion (pins,
// PINS_NEVER if none) and the counter I; insertion x fills frame x mod F,
// which keeps two flags (prefetched; hit since then), and eviction needs no
// bookkeeping of its own.  One wave runs one cache, 64 accesses per round:
//  - one gather of the pins of the round's pages; one of the candidates
//    (p+1 .. p+d) of the pages that miss at the start of the round; the
//    flags of the frames the round may refill, copied to LDS;
//  - the faults are then resolved in order inside the wave: a fault's
//    candidate k is inserted iff its latest insertion is below
//    I + c_k - F, with c_k the insertions of this fault before it (the
//    page itself first).  The condition is monotone in the set of
//    insertions, so iterating it from the candidates absent at the start
//    reaches the sequential answer in a few steps.  Later lanes and later
//    candidates see the round's insertions through a per-round list of
//    (page, first insertion, inserted-candidate mask);
//  - a page that becomes absent during the round (evicted by its own
//    round) loads its candidates when it faults.
// Evicting insertion x - F while inserting x counts a prefetched page
// evicted unused when its frame's flags say prefetched and not hit; the
// prefetched pages used are the prefetch reads minus those evicted unused
// minus those still resident and never hit (k_cache_pending).
constexpr int SNAP_CHUNK = 256;        // frame flags copied per chunk
constexpr int SNAP_MAX = 64 * 64;      // insertions in one round: 64 faults x (1 + 63 candidates)

// One wave runs one cache, and a wave's LDS operations execute in issue
// order, so between its own LDS writes and reads only the compiler must be
// kept from reordering or caching them (no wait is needed).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

struct RunLds {
  int64_t cand[64 * 64];   // [slot][k]: latest insertion of candidate k of the slot-th start miss
  int64_t page[64], cod[64];
  uint32_t mlane[64];
  int64_t fbase[64];
  uint64_t fmask[64];
  uint8_t snpf[SNAP_MAX], snhit[SNAP_MAX];
  uint8_t ipf[SNAP_MAX], ihit[SNAP_MAX];  // the round's own insertions I_rs + u
};

// One wave serves pages[0..n) on cache c, one access after another.  myhit:
// the accesses' hit flags (or null); pf_page / pf_src (or null): prefetch
// outputs from *n_pf_out on, naming access i_base + i.
__device__ __forceinline__ void cache_run_wave(const CacheCfg &c, RunLds &S, uint64_t R,
                                               const uint64_t *__restrict__ pages, int64_t n,
                                               uint8_t *__restrict__ myhit, uint64_t *__restrict__ pf_page,
                                               int64_t *__restrict__ pf_src, int64_t pf_cap, int64_t *n_pf_out,
                                               int64_t i_base) {
  int64_t *s_cand = S.cand, *s_page = S.page, *s_cod = S.cod, *s_fbase = S.fbase;
  uint32_t *s_mlane = S.mlane;
  uint64_t *s_fmask = S.fmask;
  uint8_t *s_snpf = S.snpf, *s_snhit = S.snhit, *s_ipf = S.ipf, *s_ihit = S.ihit;
  const uint32_t lane = lane_no(), d = c.d;
  const int64_t F = c.F;  // >= 64: an insertion offset within one fault (<= 63) is below F
  const bool keep_pf = pf_page != nullptr;
  // state left by earlier launches: coherent loads, never the scalar cache
  int64_t I = ld(&c.ctl->ins);
  int64_t Imod = (int64_t)((uint64_t)I % (uint64_t)F);
  int64_t hits = 0, faults = 0, pfr = 0, unused_l = 0;
  int64_t npf = n_pf_out ? ld(n_pf_out) : 0;  // prefetch outputs so far

  if (d == 0) {
    // No prefetch: a fault inserts only its own page, no frame is ever
    // prefetched, so only the insertion numbers matter.  Lane l of a round
    // faults iff no earlier lane of the round faulted on its page (such a
    // page stays resident for the rest of the round: a round inserts at most
    // 64 <= F pages) and its latest insertion is below I + c_l - F, with c_l
    // the faults of the lanes before it.  Each lane's outcome depends only
    // on those of the lanes before it, so the equations have one solution,
    // and iterating them from any guess reaches it after at most 64 steps
    // (after step k the first k lanes are settled); usually after 2.
    for (int64_t b0 = 0; b0 < n; b0 += 64) {
      const int64_t i = b0 + lane;
      const bool act = i < n;
      const uint32_t a = act ? (uint32_t)pages[i] : 0xFFFFFFFFu;
      const int64_t view = act ? ld(&c.pins[a]) : PINS_NEVER;
      // earlier lanes of the round with the same page
      uint64_t same = 0;
#pragma unroll
      for (uint32_t j = 0; j < 64; j++) {
        const uint32_t aj = (uint32_t)__builtin_amdgcn_readlane((int)a, (int)j);
        same |= aj == a ? (1ull << j) : 0ull;
      }
      same &= (1ull << lane) - 1;
      uint64_t fm = __ballot(act && view < I - F);
      for (int it = 0; it <= 64; it++) {
        const int64_t cl = (int64_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(fm >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)fm, 0u));
        const uint64_t nf = __ballot(act && !(same & fm) && view < I + cl - F);
        if (nf == fm) break;
        fm = nf;
      }
      const bool flt = (fm >> lane) & 1;
      if (flt) {
        const int64_t cl = (int64_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(fm >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)fm, 0u));
        st(&c.pins[a], I + cl);
      }
      if (act && myhit) myhit[i] = flt ? 0 : 1;
      const int64_t m = __popcll(fm);
      faults += m;
      hits += __popcll(__ballot(act)) - m;
      I += m;
    }
    if (lane == 0) {
      c.ctl->ins = I;
      c.ctl->head = (uint32_t)((uint64_t)I % (uint64_t)F);
      c.ctl->count[0] += hits;
      c.ctl->count[1] += faults;
      c.ctl->pend = 0;
    }
    return;
  }

  for (int64_t b0 = 0; b0 < n; b0 += 64) {
    const int64_t i = b0 + lane;
    const bool act = i < n;
    const int64_t a = act ? (int64_t)pages[i] : -1;
    int64_t view = act ? ld(&c.pins[a]) : PINS_NEVER;
    const int64_t I_rs = I, Imod_rs = Imod;
    // flags of the frames (Imod_rs + u) mod F, u < snap: they hold insertions
    // I_rs - F + u, which the round's insertions I_rs + u evict
    uint32_t snap = 0;
    auto load_snap = [&]() {
      uint8_t pf[SNAP_CHUNK / 64], hh[SNAP_CHUNK / 64];
#pragma unroll
      for (int u = 0; u < SNAP_CHUNK / 64; u++) {
        const int64_t fr = (int64_t)((uint32_t)(Imod_rs + (int64_t)(snap + u * 64 + lane)) % (uint32_t)F);
        pf[u] = ld(&c.fpf[fr]);
        hh[u] = ld(&c.fhit[fr]);
      }
#pragma unroll
      for (int u = 0; u < SNAP_CHUNK / 64; u++) {
        s_snpf[snap + u * 64 + lane] = pf[u];
        s_snhit[snap + u * 64 + lane] = hh[u];
      }
      snap += SNAP_CHUNK;
    };
    if (I_rs + 64 * (int64_t)(d + 1) > F) load_snap();  // the round may evict
    const uint64_t miss0 = __ballot(act && view < I_rs - F);
    int64_t fr = view >= 0 ? (int64_t)((uint64_t)view % (uint64_t)F) : 0;  // frame of this lane's page
    // candidates of the first pages missing at the start of the round, as
    // many as one 512-entry gather holds (the earliest misses are the
    // likeliest faults: later ones are often filled by an earlier fault's
    // prefetch); a fault beyond them reads its candidates when it happens
    const uint32_t n_pre = d > 0 ? min((uint32_t)__popcll(miss0), 512u / d) : 0u;
    if (n_pre > 0) {
      s_page[lane] = a;
      if ((miss0 >> lane) & 1) s_mlane[__builtin_amdgcn_mbcnt_hi((uint32_t)(miss0 >> 32),
                                       __builtin_amdgcn_mbcnt_lo((uint32_t)miss0, 0u))] = lane;
      lds_fence();
      const uint32_t total = n_pre * d;
      for (uint32_t e0 = 0; e0 < total; e0 += 512) {
        int64_t v[8];
        uint32_t at[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
          const uint32_t e = e0 + (uint32_t)u * 64 + lane;
          v[u] = PINS_NEVER;
          at[u] = 0xFFFFFFFFu;
          if (e < total) {
            const uint32_t sl = e / d, k = e - sl * d + 1;
            const int64_t q = s_page[s_mlane[sl]] + (int64_t)k;
            at[u] = sl * 64 + k;
            if ((uint64_t)q < R) v[u] = ld(&c.pins[q]);
          }
        }
#pragma unroll
        for (int u = 0; u < 8; u++)
          if (at[u] != 0xFFFFFFFFu) s_cand[at[u]] = v[u];
      }
      lds_fence();
    }

    uint32_t cursor = 0, J = 0;
    int64_t my_fpm = 0;  // page of the round's lane-th fault
    uint64_t hitmask = 0;
    while (true) {
      const bool later = act && lane >= cursor;
      const uint64_t mm = __ballot(later && view < I - F);
      const uint32_t f = mm ? (uint32_t)__builtin_ctzll(mm) : 64u;
      // the accesses before the next fault hit (their bookkeeping is done at
      // the end of the round: a lane's view no longer changes after its turn)
      const uint64_t hm = __ballot(later && lane < f);
      hitmask |= hm;
      hits += __popcll(hm);
      if (f == 64) break;
      faults++;
      const int64_t pm = read_lane(a, f);
      const int64_t im = b0 + f;
      // candidate k = lane (lane 0: the page itself)
      const bool cv = lane <= d && (uint64_t)(pm + (int64_t)lane) < R;
      int64_t L = PINS_NEVER;
      const uint32_t slot = (uint32_t)__popcll(miss0 & ((1ull << f) - 1));
      if (((miss0 >> f) & 1) && slot < n_pre) {
        if (lane >= 1 && cv) L = s_cand[slot * 64 + lane];
      } else {
        // not among the gathered misses: read the candidates now (through
        // LDS, so that only this branch waits for device memory)
        if (lane >= 1 && cv) s_cod[lane] = ld(&c.pins[pm + (int64_t)lane]);
        lds_fence();
        if (lane >= 1 && cv) L = s_cod[lane];
      }
      // an earlier fault of this round can have inserted pm + lane only if
      // its page lies in [pm + 1 - d, pm + d]
      // (lane j holds fault j's page: one ballot finds the few that do, where
      // a loop over them took 2 of a scattered fault's 2.9 us)
      uint64_t near = __ballot(lane < J && my_fpm <= pm + (int64_t)d && my_fpm + (int64_t)d >= pm + 1);
      for (; near; near &= near - 1) {  // the last of them wins
        const uint32_t j = (uint32_t)__builtin_ctzll(near);
        const int64_t off = pm + (int64_t)lane - read_lane(my_fpm, j);
        if (lane >= 1 && cv && off >= 0 && off <= (int64_t)d) {
          const uint64_t fm = s_fmask[j];
          if ((fm >> off) & 1) L = s_fbase[j] + __popcll(fm & ((1ull << off) - 1));
        }
      }
      // insertions: the least fixed point of ins_k = (L_k < I + c_k - F);
      // the first guess takes c_k = 1, which is exact for depth 1
      uint64_t msk = __ballot(cv && (lane == 0 || L < I + 1 - F));
      while (d > 1) {
        const int64_t ck = (int64_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(msk >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)msk, 0u));
        const uint64_t m2 = __ballot(cv && (lane == 0 || L < I + ck - F));
        if (m2 == msk) break;
        msk = m2;
      }
      const uint32_t m = (uint32_t)__popcll(msk);
      // the flags of the frames these insertions take must be in the copy
      // before any later hit of this round could touch them (counted at the
      // end of the round)
      if (I + (int64_t)m > F) {
        int64_t need = I + (int64_t)m - I_rs;
        if (need > F) need = F;  // beyond F the evicted insertions are the round's own
        if ((int64_t)snap < need) {
          while ((int64_t)snap < need) load_snap();
          lds_fence();
        }
      }
      if ((msk >> lane) & 1) {
        const uint32_t off = __builtin_amdgcn_mbcnt_hi((uint32_t)(msk >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)msk, 0u));
        const int64_t x = I + off;
        int64_t fx = Imod + off;
        if (fx >= F) fx -= F;
        s_ipf[x - I_rs] = lane > 0 ? 1 : 0;
        s_ihit[x - I_rs] = 0;
        const int64_t q = pm + (int64_t)lane;
        st(&c.pins[q], x);
        st(&c.fpf[fx], (uint8_t)(lane > 0 ? 1 : 0));
        st(&c.fhit[fx], (uint8_t)0);
        if (lane > 0 && keep_pf) {
          const int64_t j = npf + (int64_t)off - 1;
          if (j < pf_cap) {
            pf_page[j] = (uint64_t)q;
            pf_src[j] = i_base + im;
          }
        }
      }
      npf += m - 1;
      pfr += m - 1;
      if (d > 0) {
        if (lane == 0) {
          s_fbase[J] = I;
          s_fmask[J] = msk;
        }
        if (lane == J) my_fpm = pm;
      }
      // the later accesses see this fault's insertions
      {
        const int64_t off = a - pm;
        if (act && lane > f && off >= 0 && off <= (int64_t)d && ((msk >> off) & 1)) {
          const int64_t o = __popcll(msk & ((1ull << off) - 1));
          view = I + o;
          fr = Imod + o;
          if (fr >= F) fr -= F;
        }
      }
      J++;
      I += m;
      Imod += m;
      if (Imod >= F) Imod -= F;
      wave_lds_order();
      cursor = f + 1;
    }
    const bool hl = (hitmask >> lane) & 1;
    if (act && myhit) myhit[i] = hl ? 1 : 0;
    if (hl) {
      // mark the hit insertion in the round's records or the flag copy, and
      // in device memory if it is still resident (else its frame was refilled)
      if (view >= I_rs) {
        s_ihit[view - I_rs] = 1;
      } else {
        const int64_t u = view - (I_rs - F);
        if (u >= 0 && u < (int64_t)snap) s_snhit[u] = 1;
      }
      if (view >= I - F) st(&c.fhit[fr], (uint8_t)1);
    }
    wave_lds_order();
    // evictions of the round: its insertions I_rs + u with I_rs + u >= F took
    // the frames of insertions I_rs - F + u -- made before the round (their
    // flags are in the copy) or, when u >= F, by the round itself (in its
    // own records); every hit on an evicted insertion preceded its eviction
    {
      const int64_t lo = F - I_rs > 0 ? F - I_rs : 0, hi = I - I_rs;
      for (int64_t u = lo + lane; u < hi; u += 64) {
        const bool gone_unused = u >= F ? (s_ipf[u - F] && !s_ihit[u - F]) : (s_snpf[u] && !s_snhit[u]);
        unused_l += gone_unused ? 1 : 0;
      }
    }
    lds_fence();
  }
  int64_t unused = unused_l;
  for (int o = 32; o >= 1; o >>= 1) unused += __shfl_xor(unused, o);
  if (lane == 0) {
    c.ctl->ins = I;
    c.ctl->head = (uint32_t)Imod;
    c.ctl->count[0] += hits;
    c.ctl->count[1] += faults;
    c.ctl->count[2] += pfr;
    c.ctl->count[4] += unused;
    c.ctl->pend = 0;
    if (n_pf_out) *n_pf_out = npf;
  }
}

}  // namespace hbf
