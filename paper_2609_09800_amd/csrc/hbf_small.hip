// Small calls in one launch (HBFSim, arXiv 2609.09800, Section "Design": the
// online media model, a die-read queue then a channel-transfer queue, each
// FCFS).  A call of a few thousand requests is otherwise bound by its
// launches, not by its work.  Here one 1,024-thread workgroup does it all:
//   1. classify and validate, and rank each request among the call's
//      requests of its die queue (stable: index order);
//   2. stage the call in die order (queue-major) and take the Lindley form
//      of each die queue as one segmented prefix maximum:
//      die_done_r = (r+1)*tR + max(L, max over i <= r of issue_i - i*tR);
//   3. one wave per channel (several on one or two channels, each a stretch of
//      the channel's time; a share of a wave on more than 64) orders the
//      channel's die runs by (die-done, index) in registers (the lane merge of
//      hbf_device.h), takes the channel's Lindley form over the merged positions,
//      complete_r = (r+1)*xfer + max(F, max over i <= r of die_done_i - i*xfer),
//      and stores the completions; runs too long or too far apart for one
//      merge are taken in several steps;
//   4. new clocks, or, on any error, HBF_TIME_ERROR everywhere and the clocks
//      left as they were.
// It serves the plain two-stage model (no refresh quanta pending, no
// register blocking, not the vmem route) where its LDS fits.  The call is a
// chain of latencies on one CU (loads, ranks, two block scans, a merge): the
// kernel takes 13 us at 512 requests and 14 at 1,536 on 16 channels x 8
// dies, 23 at 4,096.  Searching each request's rank in every other run of
// its channel by LDS reads took 60, 69 and 100 us.  A call that crowds one
// of its channels serializes on that channel's wave, so one or two channels
// share the workgroup's waves between them (4,096 requests on 1 x 16: 39 us
// against 67 on one wave); from four channels on the second merge this
// takes costs more than it gives (4 x 4: 36 us against 26).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hbf_device.h"
#include "hbf_internal.h"

namespace hbf {

namespace {

constexpr int SM_THREADS = 1024;
constexpr int SM_WAVES = SM_THREADS / 64;
constexpr int SM_SLOTS = 8;  // requests per lane of a merge at most
constexpr uint32_t SM_SHARE = 4 * SM_WAVES;  // channels above which several share a wave

// LDS: ranges | wcnt[SM_WAVES][K] u16 | seg[K+1] u32 | cf[C] i64 | sdd[cap] i64 | sidx, skey [cap] u16,
// cap = requests the workgroup holds
struct SmallLayout {
  size_t wcnt, seg, cf, sdd, sidx, skey, total;
};
__host__ __device__ inline SmallLayout small_layout(uint32_t K, uint32_t C, uint32_t cap) {
  SmallLayout L;
  size_t o = (sizeof(LdsRanges) + 15) & ~size_t(15);
  L.wcnt = o; o += (size_t)SM_WAVES * K * 2;
  o = (o + 15) & ~size_t(15);
  L.seg = o;  o += (size_t)(K + 1) * 4;
  o = (o + 15) & ~size_t(15);
  L.cf = o;   o += (size_t)C * 8;
  L.sdd = o;  o += (size_t)cap * 8;
  L.sidx = o; o += (size_t)cap * 2;
  L.skey = o; o += (size_t)cap * 2;
  L.total = o;
  return L;
}

// Stable rank of each item among this wave's items with the same key (item,
// then lane order), and the wave's per-key counts in wcnt.  The lanes that
// share a key are found with one ballot per key bit (a small call's keys
// are few, so many lanes of a wave share one).
template <int ITEMS>
DEVI void wave_rank_bits(const uint32_t (&key)[ITEMS], uint32_t (&rank)[ITEMS], uint16_t *wcnt, uint32_t nbits) {
#pragma unroll
  for (int e = 0; e < ITEMS; e++) {
    const uint32_t k = key[e];
    const bool valid = k != KEY_NONE;
    uint64_t mask = __ballot(valid);
    for (uint32_t b = 0; b < nbits; b++) {
      const bool bit = (k >> b) & 1u;
      const uint64_t bb = __ballot(valid && bit);
      mask &= bit ? bb : ~bb;
    }
    const uint32_t below = mask_below(mask), cnt = (uint32_t)__popcll(mask);
    uint32_t prior = 0;
    if (valid) prior = wcnt[k];
    // all reads of this item happen before the group's first lane updates
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) wcnt[k] = (uint16_t)(prior + cnt);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    rank[e] = prior + below;
  }
}

// One merge of a wave: the `take` (at most SL << lp) requests of each run
// (lane d: run d) from staged position cur, all within 2^30 ns of tb; m in
// all, channel ranks from `rank`, entering term `gin`.  Returns the term
// after them and, with `emit`, stores their completions.
template <int SL>
DEVI int64_t small_merge(const int64_t *sdd, const uint16_t *sidx, uint32_t cur, uint32_t take, uint32_t lp,
                         int64_t tb, uint32_t m, int64_t rank, int64_t xfer, int64_t gin, bool emit,
                         int64_t *__restrict__ complete, uint32_t *errb) {
  const uint32_t lane = lane_id();
  const uint32_t d = lane >> lp, skip = (lane & ((1u << lp) - 1)) * SL;
  const uint32_t at = __shfl(cur, (int)d) + skip, have = __shfl(take, (int)d);
  const uint32_t cnt = have > skip ? have - skip : 0u;
  uint64_t a[SL];
#pragma unroll
  for (int i = 0; i < SL; i++) {
    a[i] = KEY_NONE64;
    if ((uint32_t)i < cnt) a[i] = KEY_TOP | (uint64_t)(sdd[at + i] - tb) << 31 | sidx[at + i];
  }
  merge_runs<SL>(a, lp);
  const uint32_t p0 = lane * SL, mine = m > p0 ? min(m - p0, (uint32_t)SL) : 0u;
  const int64_t cst = tb - rank * xfer;
  auto value = [&](int i) {  // of merged position p0 + i
    return cst + (int64_t)((a[i] >> 31) & 0x3FFFFFFFu) - (int64_t)mul32(p0 + i, (uint32_t)xfer);
  };
  int64_t loc = NEG;
#pragma unroll
  for (int i = 0; i < SL; i++)
    if ((uint32_t)i < mine) loc = imax(loc, value(i));
  const int64_t inc = wave_incl_max(loc);
  if (!emit) return imax(gin, lane63(inc));
  int64_t carry = __shfl_up(inc, 1);
  if (lane == 0) carry = NEG;
  carry = imax(carry, gin);
  const int64_t r0x = rank * xfer;
#pragma unroll
  for (int i = 0; i < SL; i++) {
    if ((uint32_t)i < mine) {
      carry = imax(carry, value(i));
      const int64_t cpl = r0x + (int64_t)mul32(p0 + i + 1, (uint32_t)xfer) + carry;
      if (cpl >= TIME_LIMIT) *errb |= ERR_OVERFLOW;
      complete[(uint32_t)a[i] & 0x7FFFFFFFu] = cpl;
    }
  }
  return imax(gin, lane63(inc));
}

// Several channels at once, 2^lw lanes each: a run has 2^lr of them, and the
// lane holds `len` (at most SL) of its requests from staged position `at`.  The
// group merges and completes its channel of m requests (0: none) as small_merge
// does with 64 lanes.  cfree: the channel's clock; returns its term after the
// call (on every lane).
template <int SL>
DEVI int64_t group_merge(const int64_t *sdd, const uint16_t *sidx, uint32_t at, uint32_t len, uint32_t lr,
                         uint32_t lw, int64_t tb, uint32_t m, int64_t xfer, int64_t cfree,
                         int64_t *__restrict__ complete, uint32_t *errb) {
  const uint32_t lane = lane_id(), W = 1u << lw, sub = lane & (W - 1);
  uint64_t a[SL];
#pragma unroll
  for (int i = 0; i < SL; i++) {
    a[i] = KEY_NONE64;
    if ((uint32_t)i < len) a[i] = KEY_TOP | (uint64_t)(sdd[at + i] - tb) << 31 | sidx[at + i];
  }
  if (lr <= 0 && lw >= 1) lane_merge<1, SL>(a);
  if (lr <= 1 && lw >= 2) lane_merge<2, SL>(a);
  if (lr <= 2 && lw >= 3) lane_merge<4, SL>(a);
  if (lr <= 3 && lw >= 4) lane_merge<8, SL>(a);
  if (lr <= 4 && lw >= 5) lane_merge<16, SL>(a);
  if (lr <= 5 && lw >= 6) lane_merge<32, SL>(a);
  const uint32_t p0 = sub * SL, mine = m > p0 ? min(m - p0, (uint32_t)SL) : 0u;
  auto value = [&](int i) {  // of merged position p0 + i
    return tb + (int64_t)((a[i] >> 31) & 0x3FFFFFFFu) - (int64_t)mul32(p0 + i, (uint32_t)xfer);
  };
  int64_t inc = NEG;
#pragma unroll
  for (int i = 0; i < SL; i++)
    if ((uint32_t)i < mine) inc = imax(inc, value(i));
  for (uint32_t o = 1; o < W; o <<= 1) {
    const int64_t y = __shfl_up(inc, o);
    if (sub >= o) inc = imax(inc, y);
  }
  int64_t carry = __shfl_up(inc, 1);
  carry = sub ? imax(carry, cfree) : cfree;
#pragma unroll
  for (int i = 0; i < SL; i++) {
    if ((uint32_t)i < mine) {
      carry = imax(carry, value(i));
      const int64_t cpl = (int64_t)mul32(p0 + i + 1, (uint32_t)xfer) + carry;
      if (cpl >= TIME_LIMIT) *errb |= ERR_OVERFLOW;
      complete[(uint32_t)a[i] & 0x7FFFFFFFu] = cpl;
    }
  }
  return imax(cfree, __shfl(inc, (int)(lane | (W - 1))));
}

}  // namespace

// ITEMS: requests per thread; the call has at most ITEMS * 1,024.  SHARE: more
// than SM_SHARE channels.
template <bool POW2, int ITEMS, bool SHARE>
__global__ __launch_bounds__(SM_THREADS) void k_small(const uint64_t *__restrict__ addr,
                                                      const int64_t *__restrict__ issue, uint32_t n,
                                                      int64_t *__restrict__ complete, Geo g, RangeTable rt,
                                                      DevState *st, CallCtl *ctl) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ uint32_t shsum[SM_WAVES];
  __shared__ SegMax shseg[SM_WAVES];
  __shared__ uint32_t s_err;
  __shared__ int64_t s_max, s_term[SM_WAVES];
  const uint32_t K = g.K, Dk = g.Dk, C = g.C;
  const SmallLayout SL = small_layout(K, C, ITEMS * SM_THREADS);
  LdsRanges *lr = (LdsRanges *)smem;
  uint16_t *wcnt = (uint16_t *)(smem + SL.wcnt);
  uint32_t *seg = (uint32_t *)(smem + SL.seg);
  int64_t *cf = (int64_t *)(smem + SL.cf);
  int64_t *sdd = (int64_t *)(smem + SL.sdd);
  uint16_t *sidx = (uint16_t *)(smem + SL.sidx);
  uint16_t *skey = (uint16_t *)(smem + SL.skey);
  const uint32_t t = threadIdx.x, lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t nw = (n + 64 * ITEMS - 1) / (64 * ITEMS);  // waves with requests
  const int64_t tR = g.tR, xfer = g.xfer;

  // item e of wave w: requests (w * ITEMS + e) * 64 + lane
  const uint32_t wb = w * 64 * ITEMS;
  int64_t iss[ITEMS], prev[ITEMS];
  uint64_t ad[ITEMS];
#pragma unroll
  for (int e = 0; e < ITEMS; e++) {
    const uint32_t i = wb + e * 64 + lane;
    iss[e] = i < n ? issue[i] : 0;
    ad[e] = i < n ? addr[i] : 0;
    prev[e] = lane == 0 && i > 0 && i < n ? issue[i - 1] : 0;
  }
  // (one range, the common case, needs no table in LDS)
  if (rt.n != 1) load_ranges(lr, rt);
  for (uint32_t q = t; q < nw * K; q += SM_THREADS) wcnt[q] = 0;
  if (t == 0) {
    s_err = 0;
    s_max = NEG;
  }
  __syncthreads();
  const RangeReg rr = {rt.n, rt.base[0], rt.bytes[0], rt.pbase[0]};
  uint32_t errb = 0;

  // 1. classify, validate, rank within the die queue
  uint32_t key[ITEMS], rank[ITEMS];
  int64_t df[ITEMS];  // the queue's clock, loaded ahead of the run's head
#pragma unroll
  for (int e = 0; e < ITEMS; e++) {
    const uint32_t i = wb + e * 64 + lane;
    const bool v = i < n;
    const int64_t x = iss[e];
    int64_t before = dpp64<DPP_WAVE_SHR1, 0xF>(x, x);  // lane l - 1's issue time
    if (lane == 0) before = i > 0 ? prev[e] : x;
    uint32_t k = KEY_NONE;
    df[e] = NEG;
    if (v) {
      if (x < 0 || x >= ISSUE_LIMIT) errb |= ERR_RANGE_TIME;
      if (x < before) errb |= ERR_UNSORTED;
      k = key_of<POW2>(g, lr, rr, ad[e]);
      if (k == KEY_NONE) complete[i] = x;  // native path: no modeled delay
      else df[e] = st->die_free[k];
    }
    key[e] = k;
  }
  uint32_t nbits = 0;
  while ((1u << nbits) < K) nbits++;
  if (w < nw) wave_rank_bits<ITEMS>(key, rank, wcnt + w * K, nbits);
  if (errb) atomicOr(&s_err, errb);
  // the failure: every completion HBF_TIME_ERROR, the clocks as they were
  auto fail = [&](uint32_t err) {
    for (uint32_t i = t; i < n; i += SM_THREADS) complete[i] = HBF_TIME_ERROR;
    if (t == 0) {
      atomicOr(&st->sticky, err);
      ctl->err = err;
      ctl->n_in = 0;
      ctl->max_cpl = NEG;
    }
  };
  __syncthreads();
  if (s_err) {  // (the steps below rely on valid, ascending issue times)
    fail(s_err);
    return;
  }
  {  // each wave's offset among the waves; each queue's run in die order
    const uint32_t per = (K + SM_THREADS - 1) / SM_THREADS;
    const uint32_t a0 = min(K, t * per), b0 = min(K, a0 + per);
    uint32_t sum = 0;
    for (uint32_t k = a0; k < b0; k++) {
      uint32_t run = 0;
      for (uint32_t v = 0; v < nw; v++) {
        const uint32_t c = wcnt[v * K + k];
        wcnt[v * K + k] = (uint16_t)run;
        run += c;
      }
      seg[k] = run;
      sum += run;
    }
    uint32_t ex;
    const uint32_t all = block_excl_sum<SM_WAVES>(sum, &ex, shsum);
    for (uint32_t k = a0; k < b0; k++) {
      const uint32_t c = seg[k];
      seg[k] = ex;
      ex += c;
    }
    if (t == 0) seg[K] = all;
  }
  __syncthreads();
  // 2. stage issue_r - r*tR in die order; a run's head also takes the die clock
#pragma unroll
  for (int e = 0; e < ITEMS; e++) {
    const uint32_t k = key[e];
    if (k != KEY_NONE) {
      const uint32_t rc = wcnt[w * K + k] + rank[e];
      const uint32_t P = seg[k] + rc;
      int64_t v = iss[e] - (int64_t)rc * tR;
      if (rc == 0) v = imax(v, df[e]);
      sdd[P] = v;
      sidx[P] = (uint16_t)(wb + e * 64 + lane);
      skey[P] = (uint16_t)k;
    }
  }
  __syncthreads();
  const uint32_t m = seg[K];
  {
    const uint32_t p0 = t * ITEMS;
    int64_t vals[ITEMS];
    uint32_t rk[ITEMS];
    SegMax agg = {0, NEG};
#pragma unroll
    for (int q = 0; q < ITEMS; q++) {
      const uint32_t p = p0 + q;
      vals[q] = NEG;
      rk[q] = 0;
      if (p < m) {
        vals[q] = sdd[p];
        rk[q] = p - seg[skey[p]];
        agg = seg_comb(agg, SegMax{rk[q] == 0, vals[q]});
      }
    }
    const SegMax ex = block_excl_segmax<SM_WAVES>(agg, shseg);
    int64_t run = ex.v;
#pragma unroll
    for (int q = 0; q < ITEMS; q++) {
      const uint32_t p = p0 + q;
      if (p < m) {
        run = rk[q] == 0 ? vals[q] : imax(run, vals[q]);
        const int64_t dd = (int64_t)(rk[q] + 1) * tR + run;
        if (dd >= TIME_LIMIT) errb |= ERR_OVERFLOW;
        sdd[p] = dd;
      }
    }
  }
  __syncthreads();
  // 3. merge, channel completions, channel clocks: a wave per channel or,
  // where there are fewer channels than waves, `parts` waves per channel,
  // each taking one stretch of its time: they find their stretches' terms,
  // then merge again with the terms entering them.
  const uint32_t lp = run_lanes_lg(Dk);
  const uint32_t most = (uint32_t)SM_SLOTS << lp;  // requests of a run per merge
  const uint32_t parts = !SHARE && C <= 2 ? SM_WAVES / C : 1u;
  // one channel (or, with `parts` above 1, the wave's stretch of it)
  auto channel = [&](uint32_t c, uint32_t part) {
    uint32_t lo = 0, hi = 0;
    int64_t rank = 0, term = NEG;
    if (c < C) {
      if (lane < Dk) {
        lo = seg[c * Dk + lane];
        hi = seg[c * Dk + lane + 1];
      }
      if (parts > 1) {
        // stretches between equally spaced requests of the longest run
        const uint32_t len = hi - lo, longest = wave_umax(len);
        const uint32_t d = (uint32_t)__builtin_ctzll(__ballot(len == longest));
        const uint32_t head = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)d);
        auto first = [&](uint32_t j) {  // of the lane's requests at or after stretch j's start
          if (j == 0) return lo;
          if (j == parts) return hi;
          const int64_t T = sdd[head + (uint32_t)((uint64_t)longest * j / parts)];
          uint32_t a = lo, b = hi;
          while (a < b) {
            const uint32_t mid = (a + b) >> 1;
            if (sdd[mid] < T) a = mid + 1;
            else b = mid;
          }
          return a;
        };
        if (longest) {
          const uint32_t a = first(part), b = first(part + 1);
          rank = wave_sum(a - lo);
          lo = a;
          hi = b;
        }
      }
    }
    for (int pass = parts > 1 ? 0 : 1; pass < 2; pass++) {
      const bool emit = pass == 1;
      if (c < C && emit) {
        term = st->chan_free[c];
        for (uint32_t j = 0; parts > 1 && j < part; j++) term = imax(term, s_term[w - part + j]);
      }
      uint32_t cur = lo;
      int64_t at = rank;
      while (c < C && __ballot(hi != cur) != 0) {
        const uint32_t rem = hi - cur;
        // the earliest die-done left, by a maximum of 2^62 - time, and the
        // first time this merge leaves out
        const int64_t tb = TIME_LIMIT - wave_max(rem ? TIME_LIMIT - sdd[cur] : NEG);
        int64_t te = tb + (int64_t(1) << 30);
        if (rem > most) te = imin(te, sdd[cur + most]);
        te = TIME_LIMIT - wave_max(TIME_LIMIT - te);
        uint32_t take = min(rem, most);
        if (rem && sdd[cur + take - 1] >= te) {  // (each run ascends)
          uint32_t a = 0, b = take - 1;
          while (a < b) {
            const uint32_t mid = (a + b) >> 1;
            if (sdd[cur + mid] < te) a = mid + 1;
            else b = mid;
          }
          take = a;
        }
        const uint32_t longest = wave_umax(take), mm = wave_sum(take);
        if (longest <= (2u << lp))
          term = small_merge<2>(sdd, sidx, cur, take, lp, tb, mm, at, xfer, term, emit, complete, &errb);
        else if (longest <= (4u << lp))
          term = small_merge<4>(sdd, sidx, cur, take, lp, tb, mm, at, xfer, term, emit, complete, &errb);
        else
          term = small_merge<SM_SLOTS>(sdd, sidx, cur, take, lp, tb, mm, at, xfer, term, emit, complete, &errb);
        cur += take;
        at += mm;
      }
      if (!emit) {
        if (lane == 0) s_term[w] = term;
        __syncthreads();
      } else if (c < C && part + 1 == parts && at > 0 && lane == 0) {
        cf[c] = at * xfer + term;  // the channel's last completion
        atomicMax((long long *)&s_max, (long long)cf[c]);
      }
    }
  };
  if constexpr (SHARE) {
    // Many channels: 2^(lp - lr) of them share a wave, each run on 2^lr lanes,
    // enough for twice the mean run.  A channel with a longer run, or with
    // requests 2^30 ns after its first, follows by itself.  2,048 requests on
    // 512 x 1: 22 us, 80 with every channel by itself.
    uint32_t lr = 0;
    while (lr < lp && (uint64_t)K * SM_SLOTS << lr < 2 * (uint64_t)m) lr++;
    const uint32_t lw = 6 - lp + lr, hold = (uint32_t)SM_SLOTS << lr;
    const uint32_t d = (lane & ((1u << lw) - 1)) >> lr, skip = (lane & ((1u << lr) - 1)) * SM_SLOTS;
    for (uint32_t c0 = w << (6 - lw); c0 < C; c0 += SM_WAVES << (6 - lw)) {
      const uint32_t c = c0 + (lane >> lw);
      const bool on = c < C && d < Dk;
      const uint32_t lo = on ? seg[c * Dk + d] : 0u, all = on ? seg[c * Dk + d + 1] - lo : 0u;
      if (__ballot(all != 0) == 0) continue;
      int64_t tb = all ? sdd[lo] : TIME_LIMIT;
      for (uint32_t o = 1u << lr; o < (1u << lw); o <<= 1) tb = imin(tb, __shfl_xor(tb, o));
      const uint64_t over = __ballot(all > hold || (all && sdd[lo + all - 1] - tb >= (int64_t(1) << 30)));
      const uint64_t group = (lw == 6 ? ~uint64_t(0) : (uint64_t(1) << (1u << lw)) - 1) << (lane >> lw << lw);
      const bool alone = (over & group) != 0;
      uint32_t len = alone || all <= skip ? 0u : min(all - skip, (uint32_t)SM_SLOTS), mm = len;
      for (uint32_t o = 1; o < (1u << lw); o <<= 1) mm += (uint32_t)__shfl_xor((int)mm, o);
      const uint32_t longest = wave_umax(len);
      if (longest) {
        const int64_t cfree = c < C ? st->chan_free[c] : NEG;
        const int64_t term = group_merge<SM_SLOTS>(sdd, sidx, lo + skip, len, lr, lw, tb, mm, xfer, cfree, complete,
                                                   &errb);
        if (mm && (lane & ((1u << lw) - 1)) == 0) {
          cf[c] = mm * xfer + term;  // the channel's last completion
          atomicMax((long long *)&s_max, (long long)cf[c]);
        }
      }
      for (uint64_t rest = __ballot(alone); rest;) {
        const uint32_t q = (uint32_t)__builtin_ctzll(rest) >> lw;
        channel(c0 + q, 0);
        rest &= ~((lw == 6 ? ~uint64_t(0) : (uint64_t(1) << (1u << lw)) - 1) << (q << lw));
      }
    }
  } else {
    for (uint32_t c0 = 0; c0 < C; c0 += SM_WAVES) channel(c0 + w / parts, w % parts);  // (parts > 1: one round)
  }
  if (errb) atomicOr(&s_err, errb);
  __syncthreads();
  // 4. clocks, or the failure
  if (s_err) {
    fail(s_err);
    return;
  }
  for (uint32_t k = t; k < K; k += SM_THREADS)
    if (seg[k + 1] > seg[k]) st->die_free[k] = sdd[seg[k + 1] - 1];
  for (uint32_t c = t; c < C; c += SM_THREADS)
    if (seg[(c + 1) * Dk] > seg[c * Dk]) st->chan_free[c] = cf[c];
  if (t == 0) {
    ctl->err = 0;
    ctl->n_in = m;
    ctl->max_cpl = s_max;
  }
}

// Requests per thread of a call of n requests.
static int small_items(int64_t n) { return n <= 2 * SM_THREADS ? 2 : 4; }

bool small_path_ok(const Geo &g, int64_t n, bool refresh) {
  return !refresh && !g.reg_block && !g.vmem && n > 0 && n <= SMALL_N &&
         small_layout(g.K, g.C, small_items(n) * SM_THREADS).total <= SMALL_LDS_MAX;
}

hipError_t launch_small(const Geo &g, const RangeTable &rt, DevState *st, CallCtl *ctl, const uint64_t *addr,
                        const int64_t *issue, int64_t n, int64_t *complete, hipStream_t s) {
  const int items = small_items(n);
  const size_t lds = small_layout(g.K, g.C, items * SM_THREADS).total;
  auto pick = [&](auto two, auto four) { return items == 2 ? two : four; };
  auto f = g.C > SM_SHARE ? (g.pow2 ? pick(k_small<true, 2, true>, k_small<true, 4, true>)
                                              : pick(k_small<false, 2, true>, k_small<false, 4, true>))
                                    : (g.pow2 ? pick(k_small<true, 2, false>, k_small<true, 4, false>)
                                              : pick(k_small<false, 2, false>, k_small<false, 4, false>));
  hipLaunchKernelGGL(f, dim3(1), dim3(SM_THREADS), lds, s, addr, issue, (uint32_t)n, complete, g, rt, st, ctl);
  return hipGetLastError();
}

// (the largest LDS any geometry on this path asks for)
hipError_t set_lds_small() {
  const void *f[] = {(const void *)k_small<true, 2, false>,  (const void *)k_small<true, 4, false>,
                     (const void *)k_small<false, 2, false>, (const void *)k_small<false, 4, false>,
                     (const void *)k_small<true, 2, true>,   (const void *)k_small<true, 4, true>,
                     (const void *)k_small<false, 2, true>,  (const void *)k_small<false, 4, true>};
  for (const void *k : f) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_LDS_MAX);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace hbf
