// HIP kernels (gfx950, wave64) of the HBF service-model hot path.
//
// hbf_time_requests computes, for every request, the completion of a
// die-read queue followed by a channel-transfer queue (the online media
// model of HBFSim, arXiv 2609.09800, Section "Design"; the two-stage reading
// of that model is documented in hbf.h).  Each stage is a first-come
// first-served single server with a constant service time S, whose
// departures obey the Lindley form
//
//     f_m = m*S + max(f_0, max_{i<=m} (a_i - (i-1)*S))          (m = 1, 2, ...)
//
// for arrivals a_1 <= ... in service order and a server free at f_0.  Both
// stages are therefore a rank computation plus a prefix maximum, done here
// with exact int64 arithmetic:
//
//   k_die_reduce   pass 1 over the requests: classify + map (Section D1),
//                  validate issue times, write complete = issue for the
//                  native path, and per (tile, die queue) the count and the
//                  departure of the tile's last request from an idle die.
//   k_tile_scan    per die queue, compose the tiles in order -> each tile's
//                  incoming die clock and rank offset; new die clocks; then
//                  die-queue segment offsets and the time-cell grid.
//   k_die_scatter  pass 2: exact die-done times, written in die-queue order
//                  (an LDS-staged stable multisplit) plus, per (channel,
//                  time cell, die), the first die rank in that cell.
//   k_cell_chan    per (time window, channel group), in window order: merge
//                  each cell's die runs by (die-done, index), publish the
//                  cell's channel term, take the term entering it by a
//                  decoupled look-back over earlier windows, and write
//                  complete[] in request order (staged by index in LDS
//                  where the window's requests cluster).
//   k_finalize     fail-closed error fill, or commit of the new clocks.
//
// A die emits at most one request per t_read_ns, so a time cell of width
// 2^shift <= T * t_read_ns holds at most T requests per die, and a bucket
// of width 2^floor(log2 t_read_ns) at most one: cells are bounded by
// construction and merge without searching.
#include <hip/hip_runtime.h>

#include <mutex>
#include <stdint.h>

#include "hbf_device.h"
#include "hbf_internal.h"

namespace hbf {

// ------------------------------------------------------------------ k_die_reduce


// Die time of the first g admissions of a die queue in one call when the
// first R of them each also carry a refresh quantum (Section D4): the sum of
// their services, g*tR + min(g, R)*tQ.  With R = 0 it is the plain g*tR.
DEVI int64_t svc_sum(uint32_t g, uint32_t R, int64_t tR, int64_t tQ) {
  return (int64_t)g * tR + (int64_t)min(g, R) * tQ;
}

// With refresh quanta pending (REF) the service of a die queue's request
// depends on its rank in the call, so the tile aggregate is kept in global
// form, max over the tile of issue - svc_sum(global rank), with the global
// ranks of the tile's first requests taken from a count pass (tin_base).
// LDS: ranges | amax[K] i64 | cmax[K] i64 | cnt[K] u32 | wcnt[DWAVES][K] u16 | tot[K] u16 | refp[K] u32 |
//      tag[DWAVES][K] u32
template <bool POW2, bool REF>
__global__ __launch_bounds__(DBLK) void k_die_reduce(const uint64_t *__restrict__ addr,
                                                    const int64_t *__restrict__ issue, int64_t n,
                                                    int64_t *__restrict__ complete, Geo g,
                                                    RangeTable rt, int64_t tile_elems,
                                                    uint32_t *__restrict__ agg_cnt,
                                                    int64_t *__restrict__ agg_A,
                                                    uint32_t *__restrict__ KR,
                                                    const uint32_t *__restrict__ tin_base, DevState *st) {
  extern __shared__ __align__(16) unsigned char smem[];
  LdsRanges *lr = (LdsRanges *)smem;
  const uint32_t K = g.K;
  int64_t *amax = (int64_t *)(smem + ((sizeof(LdsRanges) + 15) & ~size_t(15)));
  int64_t *cmax = amax + K;  // this chunk's max of issue - (rank in chunk)*tR, per key
  uint32_t *cnt = (uint32_t *)(cmax + K);
  uint16_t *wcnt = (uint16_t *)(cnt + K);
  uint16_t *tot = wcnt + DWAVES * K;
  // REF: pending quanta per key, read once per block (4-byte aligned: K may be odd)
  uint32_t *refp = (uint32_t *)(((uintptr_t)(tot + K) + 3) & ~(uintptr_t)3);
  uint32_t *tags = refp + K;

  // per-queue LDS state is indexed by the queue's LDS slot (lslot); global
  // per-queue arrays by the queue itself
  load_ranges(lr, rt);
  for (uint32_t li = threadIdx.x; li < K; li += DBLK) {
    const uint32_t k = lkey(g, li);
    // REF: cnt holds the call-wide rank of the tile's next request of k
    cnt[li] = REF ? tin_base[(size_t)blockIdx.x * K + k] : 0;
    amax[li] = NEG;
    cmax[li] = NEG;
    if (REF) refp[li] = st->ref_pend[k];
  }
  __syncthreads();
  const RangeReg rr = range_reg(lr);

  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * tile_elems;
  const int64_t t1 = imin(n, t0 + tile_elems);
  const int64_t tR = g.tR;
  uint32_t errb = 0;
  uint16_t *mycnt = wcnt + w * K;

  // the next chunk's requests are loaded while this one is ranked
  int64_t nx[DITEMS], nb = 0;
  uint64_t na[DITEMS];
  auto fetch = [&](int64_t cc) {
    const int64_t wb = cc + (int64_t)w * 64 * DITEMS;
#pragma unroll
    for (int e = 0; e < DITEMS; e++) {
      const int64_t i = wb + e * 64 + lane;
      const bool v = i < t1;
      nx[e] = v ? issue[i] : 0;
      na[e] = v ? addr[i] : 0;
    }
    nb = (lane == 0 && wb > 0 && wb < t1) ? issue[wb - 1] : 0;
  };
  if (t0 < t1) fetch(t0);
  for (int64_t c0 = t0; c0 < t1; c0 += CHUNK) {
    for (uint32_t k = lane; k < K; k += 64) mycnt[k] = 0;
    uint32_t key[DITEMS], rank[DITEMS];
    int64_t iss[DITEMS];
    int64_t cx[DITEMS];
    uint64_t ca[DITEMS];
#pragma unroll
    for (int e = 0; e < DITEMS; e++) {
      cx[e] = nx[e];
      ca[e] = na[e];
    }
    const int64_t before = nb;  // issue time preceding this wave's first request
    if (c0 + CHUNK < t1) fetch(c0 + CHUNK);
    int64_t carry_prev = 0;
    const int64_t wbase = c0 + (int64_t)w * 64 * DITEMS;
#pragma unroll
    for (int e = 0; e < DITEMS; e++) {
      const int64_t i = wbase + e * 64 + lane;
      const bool v = i < t1;
      const int64_t x = cx[e];
      const uint64_t a = ca[e];
      // previous request's issue time, for the order check
      int64_t prev = dpp64<DPP_WAVE_SHR1, 0xF>(x, x);  // lane l - 1's issue time
      int64_t last_of_prev_item = carry_prev;
      carry_prev = lane63(x);
      if (lane == 0) prev = (e > 0) ? last_of_prev_item : ((i > 0 && v) ? before : x);
      if (v) {
        if (x < 0 || x >= ISSUE_LIMIT) errb |= ERR_RANGE_TIME;
        if (i > 0 && x < prev) errb |= ERR_UNSORTED;
      }
      uint32_t k = v ? key_of<POW2>(g, lr, rr, a) : KEY_NONE;
      if (v && k == KEY_NONE) complete[i] = x;  // native path: no modeled delay
      key[e] = k == KEY_NONE ? KEY_NONE : lslot(g, k);
      iss[e] = x;
    }
    wave_rank(key, rank, mycnt, tags + w * K);
    __syncthreads();
    cross_wave_offsets(wcnt, tot, K);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < DITEMS; e++) {
      const uint32_t k = key[e];
      const int64_t i = wbase + e * 64 + lane;
      if (k != KEY_NONE) {
        const uint32_t rc = mycnt[k] + rank[e];  // rank among key k in the chunk
        if (REF)
          atomicMax((long long *)&amax[k],
                    (long long)(iss[e] - svc_sum(cnt[k] + rc, refp[k], tR, g.tQ)));
        else
          atomicMax((long long *)&cmax[k], (long long)(iss[e] - (int64_t)mul32(rc, (uint32_t)tR)));
        KR[i] = (k << 16) | rc;
      } else if (i < t1) {
        KR[i] = (uint32_t)KEY_NONE << 16;
      }
    }
    __syncthreads();
    // fold the chunk into the tile: ranks in the tile are cnt[k] + rank in chunk
    for (uint32_t k = threadIdx.x; k < K; k += DBLK) {
      const uint32_t t = tot[k];
      if (t) {
        if (!REF) {
          amax[k] = imax(amax[k], cmax[k] - (int64_t)mul32(cnt[k], (uint32_t)tR));
          cmax[k] = NEG;
        }
        cnt[k] += t;
      }
    }
    __syncthreads();
  }
  const size_t row = (size_t)blockIdx.x * K;
  for (uint32_t li = threadIdx.x; li < K; li += DBLK) {
    const uint32_t k = lkey(g, li);
    if (REF) {  // global form; the counts came from the count pass
      agg_A[row + k] = amax[li];
    } else {    // departure of the tile's last request of k from an idle die
      const uint32_t c = cnt[li];
      agg_cnt[row + k] = c;
      agg_A[row + k] = c ? (int64_t)c * tR + amax[li] : NEG;
    }
  }
  if (errb) atomicOr(&st->call_err, errb);
}

// Count pass of the refresh path: per tile, the in-range requests of each
// die queue (no ranks, no times).
template <bool POW2>
__global__ __launch_bounds__(DBLK) void k_die_count(const uint64_t *__restrict__ addr, int64_t n, Geo g,
                                                   RangeTable rt, int64_t tile_elems,
                                                   uint32_t *__restrict__ agg_cnt) {
  extern __shared__ __align__(16) unsigned char smem[];
  LdsRanges *lr = (LdsRanges *)smem;
  uint32_t *cnt = (uint32_t *)(smem + ((sizeof(LdsRanges) + 15) & ~size_t(15)));
  const uint32_t K = g.K;
  load_ranges(lr, rt);
  for (uint32_t k = threadIdx.x; k < K; k += DBLK) cnt[k] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * tile_elems;
  const int64_t t1 = imin(n, t0 + tile_elems);
  const RangeReg rr = range_reg(lr);
  for (int64_t i = t0 + threadIdx.x; i < t1; i += DBLK) {
    const uint32_t k = key_of<POW2>(g, lr, rr, addr[i]);
    if (k != KEY_NONE) atomicAdd(&cnt[lslot(g, k)], 1u);
  }
  __syncthreads();
  for (uint32_t li = threadIdx.x; li < K; li += DBLK) agg_cnt[(size_t)blockIdx.x * K + lkey(g, li)] = cnt[li];
}

// ------------------------------------------------------------------ tile scans

// Per die queue, the tiles in order: what enters each tile.  A block takes
// TQ consecutive die queues, thread (queue, group) a contiguous group of
// tiles, so a row of threads reads consecutive words of a tile's row; the
// group's values are loaded at once and kept, the groups are composed by lane
// moves within a wave and through LDS across waves, and each thread walks its
// group again.  Latency-bound: with one wave per queue, its lanes reading
// their tiles a row apart and twice, this took 9 us for 128 queues x 245
// tiles, 20 for 512 x 489 and 45 for 2,048 x 367 (and a launch of its own for
// the grid below); now 8, 9 and 12 with the grid.
//   TS_COUNT    refresh path, after the count pass: the call-wide rank of
//               each tile's first request and the queue's total;
//   TS_REFRESH  refresh path: the clock entering each tile from the
//               global-form tile maxima M_t: L = svc_sum(base) + max(f0, max
//               of M before);
//   TS_PLAIN    both at once: composition of (A, count) segments in order,
//               (A1, c1) then (A2, c2) = (max(A2, A1 + c2*tR), c1 + c2), A =
//               NEG when empty; a clock L entering a segment leaves as
//               max(A, L + c*tR).
// The last block of TS_PLAIN and TS_REFRESH then sets up the call's control
// block: die-queue segment starts, in-range count, time-cell grid.
enum { TS_COUNT, TS_PLAIN, TS_REFRESH };
constexpr int TSBLK = 1024;
constexpr int TQ = 16;              // die queues per block
constexpr int TG = TSBLK / TQ;      // tile groups per queue
constexpr int TPER = (TARGET_TILES + TG - 1) / TG;  // tiles per group at most

// Segment offsets and the time-cell grid, by one block; err: the call's
// errors so far.  totals and dfnew come from blocks of the same launch.
DEVI void key_scan(const uint32_t *totals, const int64_t *dfnew, uint32_t K, uint32_t *__restrict__ seg_start,
                   const int64_t *__restrict__ issue, uint32_t gmax, uint32_t s0, uint32_t err, CallCtl *ctl) {
  __shared__ uint32_t sh[TSBLK / 64];
  __shared__ int64_t s_dd;
  if (threadIdx.x == 0) s_dd = NEG;
  __syncthreads();
  const uint32_t per = (K + TSBLK - 1) / TSBLK;
  const uint32_t a = min(K, threadIdx.x * per), b = min(K, a + per);
  uint32_t sum = 0;
  int64_t dd = NEG;  // the latest die-done time of the call
  for (uint32_t k = a; k < b; k++) {
    const uint32_t t = agent_load32(&totals[k]);
    sum += t;
    if (t) dd = imax(dd, (int64_t)agent_load64((const uint64_t *)&dfnew[k]));
  }
  uint32_t ex;
  const uint32_t tot = block_excl_sum<TSBLK / 64>(sum, &ex, sh);
  for (uint32_t k = a; k < b; k++) {
    seg_start[k] = ex;
    ex += agent_load32(&totals[k]);
  }
  dd = wave_max(dd);
  if (lane_id() == 0) atomicMax((long long *)&s_dd, (long long)dd);
  __syncthreads();
  if (threadIdx.x == 0) {
    CallCtl c = {err, tot, 0, 0, s_dd, NEG, 0, 0, 0};
    if (s_dd >= TIME_LIMIT) c.err |= ERR_OVERFLOW;
    if (tot != 0) {
      c.cbase = issue[0];
      const int64_t span = s_dd - c.cbase + 1;  // > 0: every die-done > issue[0]
      uint32_t sh2 = s0;
      while (sh2 < 62 && ((span - 1) >> sh2) + 1 > (int64_t)gmax) sh2++;
      c.shift = sh2;
      c.G = (uint32_t)(((span - 1) >> sh2) + 1);
    }
    *ctl = c;
  }
}

template <int MODE>
__global__ __launch_bounds__(TSBLK) void k_tile_scan(const uint32_t *__restrict__ agg_cnt,
                                                     const int64_t *__restrict__ agg_A, uint32_t nt, Geo g,
                                                     DevState *st, int64_t *__restrict__ tin_L, uint32_t *tin_base,
                                                     uint32_t *totals, int64_t *dfnew,
                                                     uint32_t *__restrict__ seg_start,
                                                     const int64_t *__restrict__ issue, uint32_t gmax, uint32_t s0,
                                                     CallCtl *ctl) {
  __shared__ int64_t wA[TSBLK / 64][TQ];
  __shared__ uint32_t wC[TSBLK / 64][TQ];
  __shared__ uint32_t s_last;
  const uint32_t K = g.K, t = threadIdx.x, lane = lane_id(), w = t >> 6;
  const int64_t tR = g.tR;
  if (MODE != TS_COUNT) {
    const uint32_t err = st->call_err;  // of pass 1; the same for every block
    if (err) {
      if (blockIdx.x == 0 && t == 0) *ctl = CallCtl{err, 0, 0, 0, NEG, NEG, 0, 0, 0};
      return;
    }
  }
  const uint32_t k = blockIdx.x * TQ + (t & (TQ - 1)), grp = t / TQ;
  const bool on = k < K;
  const uint32_t per = (nt + TG - 1) / TG;  // at most TPER
  const uint32_t ta = min(nt, grp * per), tb = min(nt, ta + per);
  uint32_t c[TPER];
  int64_t v[TPER];
#pragma unroll
  for (int q = 0; q < TPER; q++) {
    const bool in = on && ta + q < tb;
    const size_t at = in ? (size_t)(ta + q) * K + k : 0;
    c[q] = in && MODE != TS_REFRESH ? agg_cnt[at] : 0u;
    v[q] = in && MODE != TS_COUNT ? agg_A[at] : NEG;
  }
  int64_t f0 = NEG;
  uint32_t R = 0;
  if (MODE != TS_COUNT && on) f0 = st->die_free[k];
  if (MODE == TS_REFRESH && on) R = st->ref_pend[k];
  // the group's (A, C); a tile without requests of k leaves A as it is
  int64_t A = NEG;
  uint32_t C = 0;
#pragma unroll
  for (int q = 0; q < TPER; q++) {
    if (MODE == TS_REFRESH) {
      A = imax(A, v[q]);
    } else if (c[q]) {
      if (MODE == TS_PLAIN) A = imax(v[q], A + (int64_t)c[q] * tR);
      C += c[q];
    }
  }
  const int64_t tS = MODE == TS_PLAIN ? tR : 0;
  // inclusive over the wave's groups of the same queue (16 lanes apart)
#pragma unroll
  for (int d = TQ; d < 64; d <<= 1) {
    const int64_t pA = __shfl_up(A, d);
    const uint32_t pC = __shfl_up(C, d);
    if (lane >= (uint32_t)d) {
      A = imax(A, pA + (int64_t)C * tS);
      C += pC;
    }
  }
  if (lane >= 64 - TQ) {
    wA[w][lane & (TQ - 1)] = A;
    wC[w][lane & (TQ - 1)] = C;
  }
  int64_t xA = __shfl_up(A, TQ);  // exclusive within the wave
  uint32_t xC = __shfl_up(C, TQ);
  if (lane < TQ) {
    xA = NEG;
    xC = 0;
  }
  __syncthreads();
  int64_t pA = NEG;
  uint32_t pC = 0;
  for (uint32_t q = 0; q < w; q++) {
    const uint32_t cq = wC[q][t & (TQ - 1)];
    pA = imax(wA[q][t & (TQ - 1)], pA + (int64_t)cq * tS);
    pC += cq;
  }
  const int64_t bA = imax(xA, pA + (int64_t)xC * tS);  // before the thread's group
  const uint32_t bC = pC + xC;
  if (on && t >= TSBLK - TQ) {  // the last group: the queue as a whole
    const int64_t eA = imax(A, pA + (int64_t)C * tS);
    const uint32_t eC = pC + C;
    uint32_t tot = eC;
    if (MODE == TS_REFRESH) tot = totals[k];
    else agent_store32(&totals[k], tot);
    if (MODE != TS_COUNT) {
      const int64_t end = MODE == TS_PLAIN ? imax(eA, f0 + (int64_t)tot * tR)
                                           : svc_sum(tot, R, tR, g.tQ) + imax(f0, eA);
      agent_store64((uint64_t *)&dfnew[k], (uint64_t)end);
    }
  }
  if (on) {
    int64_t L = MODE == TS_PLAIN ? imax(bA, f0 + (int64_t)bC * tR) : imax(f0, bA);
    uint32_t base = bC;
#pragma unroll
    for (int q = 0; q < TPER; q++) {
      if (ta + q >= tb) break;
      const size_t at = (size_t)(ta + q) * K + k;
      if (MODE == TS_REFRESH) {
        tin_L[at] = svc_sum(tin_base[at], R, tR, g.tQ) + L;
        L = imax(L, v[q]);
        continue;
      }
      tin_base[at] = base;
      base += c[q];
      if (MODE == TS_PLAIN) {
        tin_L[at] = L;
        if (c[q]) L = imax(v[q], L + (int64_t)c[q] * tR);
      }
    }
  }
  if (MODE == TS_COUNT) return;
  // the block that finishes last goes on (totals and dfnew were stored past
  // the caches above; each wave's stores have left it before the count)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (t == 0) s_last = atomicAdd(&st->scan_ctr, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  if (t == 0) st->scan_ctr = 0;
  key_scan(totals, dfnew, K, seg_start, issue, gmax, s0, 0, ctl);
}

// ------------------------------------------------------------------ k_die_scatter

// Pass 2 of the die stage.  Per chunk: stage the requests in (die queue,
// rank) order using the ranks pass 1 stored (LDS histogram + offsets, no
// re-ranking), compute exact die-done times with a segmented prefix max,
// and write them in die-queue order, filling the cell table on the way.
//
// Per die queue k the chunk needs a handful of numbers; they sit in two
// 16-byte records so that each phase reads one record per request (random
// k: one bank-conflicted access instead of several):
//   KA[k] = {koff: offset of k's run in the chunk, cnt: k's requests in the
//            tile before this chunk, L: die clock entering the chunk}
//   KW[k] = {rbase: die rank (within the call) of k's first request in the
//            chunk, pbase: its die-order position, lbo: k's column in the
//            cell table, tot: k's requests in the call}
// LDS: sval[CP] i64 | KA[K] | KW[K] | hist[K] u32 | (SC = 2) histA[K] u32 | refp[K] u32 |
//      skr [CP] u32 (key << 16 | rank in the step) | sloc [CP] u16, with CP = SC*CHUNK + SC*CHUNK/16
//
// SC pass-1 chunks are staged together (SC = 2 wherever its LDS fits: up to
// 954 die queues). A queue's run in die order then grows from one chunk's
// requests to two, so the die-order stores touch fewer partially written
// lines: measured 2.19 -> 1.83 ms on 2^28 requests over 512 queues.
template <int SC>
constexpr int chunk_pad() { return SC * CHUNK + SC * CHUNK / 16; }
// Pass 2 runs 1,024-thread blocks, 4 requests per thread per pass-1 chunk:
// with one chunk per step, measured 2.20 ms on 2^28 requests against
// 2.27 ms for two 512-thread blocks per CU.
constexpr int SBLK = 1024;
constexpr int SWAVES = SBLK / 64;
// Runs up to this length are scanned by one thread each; a chunk with a
// longer run (a hot die) takes the block-wide segmented scan.
constexpr uint32_t RUN_WALK_MAX = 64;

struct KeyA {
  uint32_t koff, cnt;
  int64_t L;
};
struct KeyW {
  uint32_t rbase, pbase, lbo, tot;
};

// REF (refresh quanta pending): the services depend on the call-wide rank,
// so the staged terms are issue - svc_sum(rank) and die_done =
// svc_sum(rank + 1) + prefix max; each admission that claims a quantum
// writes the quantum's completion (tR before its own read ends).
template <bool REF, int SC>
__global__ __launch_bounds__(SBLK) void k_die_scatter(
    const int64_t *__restrict__ issue, const uint32_t *__restrict__ KR, int64_t n, Geo g,
    int64_t tile_elems, const int64_t *__restrict__ tin_L, const uint32_t *__restrict__ tin_base,
    const uint32_t *__restrict__ seg_start, const uint32_t *__restrict__ totals,
    int64_t *__restrict__ DD, uint32_t *__restrict__ IX, uint32_t *__restrict__ LB, uint32_t gmax,
    CallCtl *ctl, const DevState *st, uint64_t *__restrict__ WST, int64_t *__restrict__ ISS) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ SegMax shseg[SWAVES];
  __shared__ uint32_t shsum[SWAVES];
  __shared__ uint32_t s_nvalid, s_longrun;
  if (agent_load32(&ctl->err)) return;
  const uint32_t K = g.K;
  int64_t *sval = (int64_t *)smem;
  constexpr int SCH = SC * CHUNK;     // requests staged per step
  constexpr int CP = chunk_pad<SC>();
  constexpr int SITEMS = SCH / SBLK;  // per thread; the first SITEMS / SC come from the first chunk
  KeyA *KA = (KeyA *)(sval + CP);
  KeyW *KW = (KeyW *)(KA + K);
  uint32_t *hist = (uint32_t *)(KW + K);
  uint32_t *histA = hist + K;  // SC = 2: requests of each key in the first of the two chunks
  uint32_t *refp = histA + (SC == 2 ? K : 0);  // REF: pending quanta per key, read once per block
  uint32_t *skr = refp + K;
  uint16_t *sloc = (uint16_t *)(skr + CP);

  const uint32_t Dk = g.Dk;
  const size_t row = (size_t)blockIdx.x * K;
  // per-queue LDS records by LDS slot (lslot), as in pass 1, whose ranks
  // carry the slot
  for (uint32_t li = threadIdx.x; li < K; li += SBLK) {
    const uint32_t k = lkey(g, li);
    const uint32_t base = tin_base[row + k];  // die rank of the tile's first request of k
    KA[li] = KeyA{0u, 0u, tin_L[row + k]};
    const uint32_t ch = k / Dk;
    KW[li] = KeyW{base, seg_start[k] + base, ch * (gmax + 1) * Dk + (k - ch * Dk), totals[k]};
    if (REF) refp[li] = st->ref_pend[k];
  }
  const int64_t cbase = ctl->cbase;
  const uint32_t shift = ctl->shift, G = ctl->G;
  const bool narrow = shift <= 32;
  if (G) {  // clear the fused channel stage's look-back words of this call's cells (channel-major)
    const size_t nw = (size_t)G * g.C, step = (size_t)gridDim.x * SBLK;
    for (size_t q = (size_t)blockIdx.x * SBLK + threadIdx.x; q < nw; q += step) {
      const size_t c = q / G, at = c * gmax + (q - c * G);
      WST[at] = 0;
      WST[(size_t)gmax * g.C + at] = 0;
    }
  }
  const uint64_t relmask = narrow ? (uint64_t(1) << shift) - 1 : 0;
  const int64_t t0 = (int64_t)blockIdx.x * tile_elems;
  const int64_t t1 = imin(n, t0 + tile_elems);
  const uint32_t tR = (uint32_t)g.tR;

  // a chunk's requests are loaded while the previous one is scanned and
  // written (they are only needed up to the staging step)
  int64_t iss[SITEMS];
  uint32_t kr[SITEMS];
  auto fetch = [&](int64_t cc) {
#pragma unroll
    for (int e = 0; e < SITEMS; e++) {
      const int64_t i = cc + e * SBLK + threadIdx.x;
      iss[e] = 0;
      kr[e] = (uint32_t)KEY_NONE << 16;
      if (i < t1) {
        iss[e] = issue[i];
        kr[e] = KR[i];
      }
    }
  };
  if (t0 < t1) fetch(t0);
  for (int64_t c0 = t0; c0 < t1; c0 += SCH) {
    for (uint32_t k = threadIdx.x; k < K; k += SBLK) {
      hist[k] = 0;
      if (SC == 2) histA[k] = 0;
    }
    if (threadIdx.x == 0) s_longrun = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < SITEMS; e++) {
      const uint32_t k = kr[e] >> 16;
      if (k != KEY_NONE) atomicAdd(SC == 2 && e < SITEMS / 2 ? &histA[k] : &hist[k], 1u);
    }
    __syncthreads();
    {  // chunk offsets of each key's run
      const uint32_t per = (K + SBLK - 1) / SBLK;
      const uint32_t a0 = threadIdx.x * per, b0 = min(K, a0 + per);
      uint32_t sum = 0;
      for (uint32_t k = a0; k < b0; k++) {
        if (SC == 2) hist[k] += histA[k];
        sum += hist[k];
      }
      uint32_t ex;
      const uint32_t all = block_excl_sum<SWAVES>(sum, &ex, shsum);
      uint32_t longest = 0;
      for (uint32_t k = a0; k < b0; k++) {
        KA[k].koff = ex;
        ex += hist[k];
        longest = max(longest, hist[k]);
      }
      if (threadIdx.x == 0) s_nvalid = all;
      if (longest > RUN_WALK_MAX) s_longrun = 1u;
    }
    __syncthreads();
    // stage v = issue - r0*tR in die order (r0 = rank of the request among
    // k's in the tile); a run's head also folds in the entering clock,
    // M_k = L_k - cnt_k*tR, so the segmented prefix max below is the whole
    // Lindley term: die_done = (r0+1)*tR + max(M_k, max of v over the run)
#pragma unroll
    for (int e = 0; e < SITEMS; e++) {
      const uint32_t k = kr[e] >> 16;
      if (k != KEY_NONE) {
        const KeyA ka = KA[k];
        // pass 1's rank is within its own chunk: the second chunk's requests
        // of k follow the first chunk's
        const uint32_t rc = (kr[e] & 0xFFFFu) + (SC == 2 && e >= SITEMS / 2 ? histA[k] : 0u);
        const uint32_t P = pad16(ka.koff + rc);
        int64_t v;
        if (REF) {
          const uint32_t R = refp[k], g0 = KW[k].rbase;
          v = iss[e] - svc_sum(g0 + rc, R, g.tR, g.tQ);
          if (rc == 0) v = imax(v, ka.L - svc_sum(g0, R, g.tR, g.tQ));
        } else {
          v = iss[e] - (int64_t)mul32(ka.cnt + rc, tR);
          if (rc == 0) v = imax(v, ka.L - (int64_t)mul32(ka.cnt, tR));
        }
        sval[P] = v;
        skr[P] = k << 16 | rc;
        sloc[P] = (uint16_t)(e * SBLK + threadIdx.x);
        if (ISS) {  // register blocking: the issue times in die order as well
          const uint32_t gp = KW[k].pbase + rc;
          if (gp < n) ISS[gp] = iss[e];
        }
      }
    }
    __syncthreads();
    if (c0 + SCH < t1) fetch(c0 + SCH);
    const uint32_t nv = s_nvalid;
    if (!s_longrun) {
      // one thread per die queue walks its run with a running maximum (the
      // run's head already holds the entering clock)
      for (uint32_t k = threadIdx.x; k < K; k += SBLK) {
        const uint32_t t = hist[k];
        if (!t) continue;
        const KeyA ka = KA[k];
        int64_t run = NEG;
        if (REF) {
          const uint32_t R = refp[k], g0 = KW[k].rbase;
          for (uint32_t q = 0; q < t; q++) {
            const uint32_t P = pad16(ka.koff + q);
            run = imax(run, sval[P]);
            sval[P] = svc_sum(g0 + q + 1, R, g.tR, g.tQ) + run;
          }
          continue;
        }
        for (uint32_t q = 0; q < t; q++) {
          const uint32_t P = pad16(ka.koff + q);
          run = imax(run, sval[P]);
          sval[P] = (int64_t)mul32(ka.cnt + q + 1, tR) + run;
        }
      }
    } else {  // a long run: segmented scan over the whole block
      const uint32_t p0 = threadIdx.x * SITEMS;
      int64_t vals[SITEMS];
      SegMax agg = {0, NEG};
#pragma unroll
      for (int q = 0; q < SITEMS; q++) {
        const uint32_t p = p0 + q;
        vals[q] = NEG;
        if (p < nv) {
          const int64_t v = sval[pad16(p)];
          vals[q] = v;
          agg = seg_comb(agg, SegMax{(skr[pad16(p)] & 0xFFFFu) == 0, v});
        }
      }
      SegMax ex = block_excl_segmax<SWAVES>(agg, shseg);
      int64_t run = ex.v;  // prefix of the segment continuing into this thread
#pragma unroll
      for (int q = 0; q < SITEMS; q++) {
        const uint32_t p = p0 + q;
        if (p < nv) {
          const uint32_t kr2 = skr[pad16(p)];
          const uint32_t rc = kr2 & 0xFFFFu;
          run = (rc == 0) ? vals[q] : imax(run, vals[q]);
          const uint32_t kk = kr2 >> 16;
          if (REF)
            sval[pad16(p)] = svc_sum(KW[kk].rbase + rc + 1, refp[kk], g.tR, g.tQ) + run;
          else
            sval[pad16(p)] = (int64_t)mul32(KA[kk].cnt + rc + 1, tR) + run;
        }
      }
    }
    __syncthreads();
    // write die-ordered (die_done, index); fill the cell table
    for (uint32_t p = threadIdx.x; p < nv; p += SBLK) {
      const uint32_t P = pad16(p);
      const uint32_t kr2 = skr[P];
      const uint32_t k = kr2 >> 16;
      const uint32_t rc = kr2 & 0xFFFFu;
      const KeyW kw = KW[k];
      const uint32_t r = kw.rbase + rc;  // die rank within this call
      const int64_t dd = sval[P];
      const uint32_t gpos = kw.pbase + rc;
      if (gpos < n) {
        const uint32_t ix = (uint32_t)(c0 + sloc[P]);
        if (narrow)  // one word: offset of die-done in its cell, request index
          reinterpret_cast<uint64_t *>(DD)[gpos] = ((uint64_t)(dd - cbase) & relmask) << 32 | ix;
        else {
          DD[gpos] = dd;
          IX[gpos] = ix;
        }
      }
      if (REF && r < refp[k]) {  // this admission claimed quantum r of its queue's pending ones
        const uint32_t kq = lkey(g, k);
        *st->ref_slot[st->ref_off[kq] + st->ref_head[kq] + r] = dd - g.tR;
      }
      // die-done of slot p - 1 (the same queue's previous request when rc > 0):
      // lane l - 1's value, or read back by lane 0
      int64_t pdd = dpp64<DPP_WAVE_SHR1, 0xF>(dd, dd);
      if (lane_id() == 0 && p > 0) pdd = sval[pad16(p - 1)];
      const int64_t prev = (rc > 0) ? pdd : KA[k].L;
      const int64_t cell = imin((dd - cbase) >> shift, (int64_t)G);
      const int64_t pcell = (r == 0) ? -1 : imin((prev - cbase) >> shift, (int64_t)G);
      uint32_t *lbrow = LB + kw.lbo;
      for (int64_t c = pcell + 1; c <= cell; c++) lbrow[(size_t)c * Dk] = r;
      if (r + 1 == kw.tot)
        for (int64_t c = cell + 1; c <= (int64_t)G; c++) lbrow[(size_t)c * Dk] = r + 1;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < K; k += SBLK) {
      const uint32_t t = hist[k];
      if (t) {
        KA[k].L = sval[pad16(KA[k].koff + t - 1)];
        KA[k].cnt += t;
        KW[k].rbase += t;
        KW[k].pbase += t;
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ channel stage

constexpr int SLOTS_MAX = 16;  // die runs per channel on the bucket path; requests per lane elsewhere
static_assert(SLOTS_MAX == LANE_SLOTS, "both orders keep their slots in Merged");

// Sort keys of the bucket path are integers below 2^51 held in the mantissa
// of a double in [1, 2) (exponent bits 0x3FF): there IEEE order is integer
// order, so one exact v_min_f64 / v_max_f64 pair is a whole compare-exchange.
constexpr uint64_t KEY_ONE = uint64_t(0x3FF) << 52;
constexpr uint64_t KEY_EMPTY = KEY_ONE | ((uint64_t(1) << 52) - 1);  // above every key

// Batcher's odd-even merge sort over SL registers (SL a power of two; 63
// compare-exchanges for 16), ascending.
template <int SL>
DEVI void sort_slots(uint64_t (&a)[SL]) {
#pragma unroll
  for (int p = 1; p < SL; p <<= 1) {
#pragma unroll
    for (int k = p; k >= 1; k >>= 1) {
#pragma unroll
      for (int j = k % p; j + k < SL; j += 2 * k) {
#pragma unroll
        for (int i = 0; i < k; i++) {
          if (i + j + k < SL && (i + j) / (2 * p) == (i + j + k) / (2 * p)) cx_key(a[i + j], a[i + j + k]);
        }
      }
    }
  }
}

// Channel stage.  With channel ranks k (1-based) and the channel free at f0
// before the call, complete_k = k*xfer + max(f0, max_{i<=k} (dd_(i) - (i-1)*xfer)).
// A cell knows its first rank from the cell table (the sum of its row), so
// its aggregate is one number, M_j = max over its requests of
// (dd - (rank-1)*xfer), and the term entering cell j is max(f0, M_j' for
// j' < j).  k_cell_chan orders each cell once, in registers, and finds the
// entering term by a look-back over earlier windows.  Two ways to order a
// cell, one wave each:
//   bucket merge  cells of at most 64 buckets of width 2^lg_tR <= tR, which
//                 hold at most one request per die: lane q gathers the
//                 requests of bucket q, sorts them in registers and owns
//                 merged positions boff..boff+cnt-1 (cell_merge);
//   lane merge    every other grid (cells wider than 64 buckets, because
//                 the stream is sparse, or more than 16 die queues per
//                 channel): the runs are cut into pieces of up to 16
//                 requests, one piece per lane, and merged by a bitonic
//                 network across the lanes (cell_sort).
// A cell's runs, lane d = die run d: die-order bounds [lo, hi) and the die
// rank r0 of the first one.
struct CellRuns {
  uint32_t lo, hi, r0;
};
DEVI CellRuns cell_runs(const uint32_t *__restrict__ LB, const uint32_t *__restrict__ seg_start,
                        const uint32_t *__restrict__ totals, uint32_t Dk, uint32_t gmax, uint32_t c,
                        uint32_t j) {
  CellRuns r = {0, 0, 0};
  const uint32_t lane = lane_id();
  if (lane < Dk) {
    const uint32_t k = c * Dk + lane;
    if (totals[k] != 0) {
      const uint32_t *lbrow = LB + (size_t)c * (gmax + 1) * Dk + lane;
      const uint32_t sg = seg_start[k];
      r.r0 = lbrow[(size_t)j * Dk];
      r.lo = r.r0 + sg;
      r.hi = lbrow[(size_t)(j + 1) * Dk] + sg;
    }
  }
  return r;
}

// The bucket path's loads: lane q < 64 reads entry q of every run (runs of
// bucketable cells hold at most 64), all in flight at once.
template <int SL>
DEVI void load_runs(const int64_t *__restrict__ DD, const CellRuns &cr, int R, uint64_t (&xv)[SL]) {
  const uint32_t lane = lane_id();
  const uint64_t *DX = reinterpret_cast<const uint64_t *>(DD);
  const uint32_t len = cr.hi - cr.lo;
#pragma unroll
  for (int d = 0; d < SL; d++) {
    const uint32_t lod = __builtin_amdgcn_readlane(cr.lo, d);
    const uint32_t lend = __builtin_amdgcn_readlane(len, d);
    xv[d] = 0;
    if (d < R && lane < lend) xv[d] = DX[lod + lane];
  }
}

// Whether the cell grid allows the bucket merge: buckets of width 2^lg_tR,
// at most 64 of them per cell, packed 32-bit cell offsets, and at most SL
// die runs per channel.
template <int SL>
DEVI bool grid_bucketable(const Geo &g, uint32_t shift) {
  return (shift - g.lg_tR <= 6) && shift <= 32 && g.lg_tR <= 20 && (int)g.Dk <= SL;
}

constexpr uint32_t CMIN_NONE = 0xFFFFFFFFu;

// ---- The stage's work is cut into units of up to 32 cells (16 with the lane
// merge, whose network needs the registers of the second cell): one time
// window of a group of 32 channels or, with fewer channels, as many windows
// of all channels as make 32 cells; units are claimed in (window, group) order from
// a counter of the call.  One 1,024-thread workgroup per unit:
//   1. each wave orders its one or two cells (kept in registers) and
//      publishes each cell's term M_j;
//   2. per channel, the term entering the cell, max(f0, M_j' for j' < j),
//      by a decoupled look-back over the earlier windows' published words:
//      the nearest inclusive term plus the aggregates in between;
//   3. it publishes the inclusive term max(entering, M_j);
//   4. it writes the completions.  Those of one window fall in a band of
//      request indices (each die queue serves its next requests), so each
//      completion is staged in LDS at its index's offset from the band start
//      as a 32-bit offset from a base, and the band is written in index
//      order (whole lines); completions outside the staged span, or whose
//      offset does not fit, are stored directly.
// A unit waits only for its own waves and for units claimed before it: all
// of them run and publish their aggregates without waiting, so every wait
// ends.
// The wait is bounded all the same; running past the bound fails the call
// with ERR_INTERNAL instead of hanging.  The published words are single
// 64-bit atomics that carry their own validity (0 = not yet), cleared by
// k_die_scatter for the cells of the call and laid out channel-major, so a
// half-wave polling 32 consecutive windows of one channel reads two lines.
constexpr int WIN_WAVES = 16;
constexpr int WIN_THREADS = WIN_WAVES * 64;
constexpr uint32_t WIN_SLOTS = 32768;
constexpr uint32_t WIN_EMPTY = 0xFFFFFFFFu;
constexpr uint32_t LOOKBACK_ROUNDS = 1u << 22;

struct WinLds {
  uint32_t stage[WIN_SLOTS];                         // completion - wbase at index lo + slot
  uint8_t tbl[WIN_WAVES][MAX_BUCKETS][SLOTS_MAX];   // per wave: 1 + position in run d of bucket q's entry
  uint32_t rmin[WIN_WAVES];
  int64_t rbase[WIN_WAVES];
  uint32_t top;                                      // staged slots in use
  uint32_t unit;
};

// Stage slot of band offset r.  One channel's requests often sit at a
// fixed stride in the index space (sequential streams stripe over the
// channels), so the offsets one store instruction writes can share their
// low bits; XOR-ing in the next six bits spreads them over the LDS banks,
// while each aligned group of 64 consecutive offsets stays a permutation of
// itself (the write-out reads them conflict-free).
DEVI uint32_t win_slot(uint32_t r) { return r ^ ((r >> 6) & 63u); }

// Look-back words: 0 = not yet published, else the value + 2^62 (every
// published value lies in [NEG, 2^62)).
DEVI uint64_t enc_time(int64_t x) { return (uint64_t)x + (uint64_t(1) << 62); }
DEVI int64_t dec_time(uint64_t w) { return (int64_t)(w - (uint64_t(1) << 62)); }
// Inclusive maximum within each half (32 lanes) of the wave: lanes 31 and
// 63 end up holding the two halves' maxima.
DEVI int64_t half_incl_max(int64_t x) {
  x = imax(x, dpp64<DPP_ROW_SHR1, 0xF>(NEG, x));
  x = imax(x, dpp64<DPP_ROW_SHR2, 0xF>(NEG, x));
  x = imax(x, dpp64<DPP_ROW_SHR4, 0xF>(NEG, x));
  x = imax(x, dpp64<DPP_ROW_SHR8, 0xF>(NEG, x));
  x = imax(x, dpp64<DPP_ROW_BCAST15, 0xA>(NEG, x));
  return x;
}
DEVI int64_t lane_i64(int64_t x, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The terms entering two cells, one per half-wave (lanes 0-31: window ja of
// channel ca, 32-63: window jb of channel cb; a channel >= C is skipped).  Lane s
// of a half inspects window base - s: its inclusive word, else its
// aggregate.  A round ends at the nearest inclusive word (or before window
// 0, where the term is the channel's clock f0) if no aggregate before it is
// missing; otherwise the half folds what precedes the first missing one and
// polls again from there.
DEVI void look_back2(const uint64_t *WAGG, const uint64_t *WINC, uint32_t C, uint32_t gmax, uint32_t ja,
                     uint32_t jb, uint32_t ca, uint32_t cb, int64_t f0a, int64_t f0b, int64_t &ga, int64_t &gb,
                     uint32_t *errb) {
  const uint32_t lane = lane_id(), s = lane & 31;
  const bool hi = lane >= 32;
  const uint32_t c = hi ? cb : ca;
  const int64_t f0 = hi ? f0b : f0a;
  int64_t acc0 = NEG, acc1 = NEG;
  int64_t base0 = (int64_t)ja - 1, base1 = (int64_t)jb - 1;
  bool done0 = ca >= C, done1 = cb >= C;
  uint32_t rounds = 0;
  while (!(done0 && done1)) {
    const bool mine_done = hi ? done1 : done0;
    const int64_t jj = (hi ? base1 : base0) - (int64_t)s;
    int stt = 2;  // 2: inclusive (or nothing left to fold), 1: aggregate, 0: not yet published
    int64_t v = NEG;
    if (!mine_done) {
      if (jj < 0) {
        v = f0;
      } else {
        const size_t at = (size_t)c * gmax + (size_t)jj;  // a half reads 32 consecutive words
        const uint64_t wi = agent_load64(&WINC[at]);
        if (wi) {
          v = dec_time(wi);
        } else {
          const uint64_t wa = agent_load64(&WAGG[at]);
          stt = wa ? 1 : 0;
          if (wa) v = dec_time(wa);
        }
      }
    }
    const uint64_t incl = __ballot(stt == 2), none = __ballot(stt == 0);
    const uint32_t bi0 = (uint32_t)incl, bi1 = (uint32_t)(incl >> 32);
    const uint32_t bn0 = (uint32_t)none, bn1 = (uint32_t)(none >> 32);
    const uint32_t fi0 = bi0 ? (uint32_t)__builtin_ctz(bi0) : 32u, fi1 = bi1 ? (uint32_t)__builtin_ctz(bi1) : 32u;
    const uint32_t fn0 = bn0 ? (uint32_t)__builtin_ctz(bn0) : 32u, fn1 = bn1 ? (uint32_t)__builtin_ctz(bn1) : 32u;
    // fold: through the inclusive word if it precedes every gap, else up to the gap
    const uint32_t fi = hi ? fi1 : fi0, fn = hi ? fn1 : fn0;
    const uint32_t lim = (fi < fn) ? fi + 1 : fn;
    const int64_t red = half_incl_max(s < lim ? v : NEG);
    bool stalled = false;
    if (!done0) {
      acc0 = imax(acc0, lane_i64(red, 31));
      if (fi0 < fn0) done0 = true;
      else {
        base0 -= fn0;
        stalled |= fn0 == 0;
      }
    }
    if (!done1) {
      acc1 = imax(acc1, lane_i64(red, 63));
      if (fi1 < fn1) done1 = true;
      else {
        base1 -= fn1;
        stalled |= fn1 == 0;
      }
    }
    if (stalled) {
      if (++rounds > LOOKBACK_ROUNDS) {
        *errb |= ERR_INTERNAL;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
  }
  ga = acc0;
  gb = acc1;
}

// An ordered cell, held in registers: each lane owns cnt consecutive merged
// positions from boff (slot, ascending); plus the cell's size, its smallest
// request index, the channel rank of its first request, and per lane the
// maximum of dd - (rank0 + position) * xfer over its entries.  big (uniform):
// a cell ordered in several steps, whose slots are not kept.
template <int SL>
struct Merged {
  uint64_t slot[SL];
  uint32_t cnt, boff;
  uint32_t m, head;
  int64_t rank0, loc;
  bool big;
};

// Merge one bucketable cell (lane q gathers bucket q's entries from the
// lanes that loaded them, sorts them, and takes merged positions
// boff..boff+cnt-1).  Its run of die d holds at most one entry per bucket.
template <int SL>
DEVI void cell_merge(uint8_t (*tbl)[SLOTS_MAX], const CellRuns &cr, const uint64_t (&xv)[SL], const Geo &g,
                     int64_t cstart, Merged<SL> &M, uint32_t *errb) {
  const uint32_t lane = lane_id();
  const int R = (int)g.Dk;
  const uint32_t lgt = g.lg_tR;
  const int64_t xfer = g.xfer;
  const uint32_t len = cr.hi - cr.lo;
  M.m = wave_sum(len);
  M.cnt = 0;
  M.boff = 0;
  M.head = CMIN_NONE;
  M.rank0 = 0;
  M.loc = NEG;
  M.big = false;
#pragma unroll
  for (int d = 0; d < SL; d++) M.slot[d] = KEY_EMPTY;
  if (M.m == 0) return;
  if (wave_umax(lane < (uint32_t)R ? len : 0u) > 64) {  // impossible on a bucketable grid
    *errb |= ERR_INTERNAL;
    M.m = 0;
    return;
  }
  M.rank0 = wave_sum(cr.r0);
  reinterpret_cast<uint4 *>(&tbl[0][0])[lane] = make_uint4(0, 0, 0, 0);
  wave_sync();
  // sort key of entry `lane` of run d: offset in its bucket (< 2^20) << 31 | index
  const uint64_t offmask = (uint64_t(1) << lgt) - 1;
  uint64_t key[SL];
  uint32_t head = CMIN_NONE;
#pragma unroll
  for (int d = 0; d < SL; d++) {
    const uint32_t lend = __builtin_amdgcn_readlane(len, d);
    const uint64_t rel = xv[d] >> 32;
    key[d] = KEY_ONE | (rel & offmask) << 31 | (xv[d] & 0xFFFFFFFFull);
    if (d < R && lane < lend) tbl[rel >> lgt][d] = (uint8_t)(lane + 1);
    // a run's first entry has its smallest index (die order is index order)
    const uint32_t ix0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)xv[d], 0);
    if (d < R && lend > 0) head = min(head, ix0);
  }
  M.head = head;
  wave_sync();
  {
    const uint4 row = reinterpret_cast<const uint4 *>(&tbl[0][0])[lane];
    const uint32_t rw[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
    for (int d = 0; d < SL; d++) {
      const uint32_t y = (rw[d >> 2] >> (8 * (d & 3))) & 0xFFu;
      const uint64_t v = __shfl(key[d], y ? (int)(y - 1) : 0);
      M.slot[d] = y ? v : KEY_EMPTY;
      M.cnt += y ? 1u : 0u;
    }
  }
  sort_slots<SL>(M.slot);
  M.boff = wave_excl_sum(M.cnt);
  const int64_t cst = cstart + ((int64_t)lane << lgt) - M.rank0 * xfer;
#pragma unroll
  for (int i = 0; i < SL; i++) {
    if ((uint32_t)i < M.cnt) {
      const int64_t v = cst + (int64_t)((M.slot[i] >> 31) & 0x1FFFFFu) - (int64_t)mul32(M.boff + i, (uint32_t)xfer);
      M.loc = imax(M.loc, v);
    }
  }
  wave_sync();  // tbl is reused by the wave's next cell
}

// ---- Cells of the lane merge.
// A cell is merged with the fewest slots per lane (2, 4, 8 or 16) that hold
// its longest run, and needs no search and no second pass: reducing every
// such cell, scanning and ordering it again by binary searches in LDS took
// 1,060 us of a 4 M-request call at 85 % channel load (32 channels x 16
// dies; the whole call 1,156 us, now 176) and 2,770 us of a 3 M-request call
// with 64 die queues per channel (2,890, now 245).
constexpr uint32_t SUB_LG_MAX = 30;  // offsets of a lane-merge key

// The die-order entries of a call: packed words (cells at most 2^32 ns wide)
// or die-done times and indices.
struct DieOrder {
  const int64_t *__restrict__ DD;
  const uint32_t *__restrict__ IX;
  bool narrow;
  DEVI int64_t time(uint32_t at, int64_t cstart) const {
    return narrow ? cstart + (int64_t)(reinterpret_cast<const uint64_t *>(DD)[at] >> 32) : DD[at];
  }
  DEVI uint32_t index(uint32_t at) const {
    return narrow ? (uint32_t)reinterpret_cast<const uint64_t *>(DD)[at] : IX[at];
  }
};

// Order at most 64 * SL requests: lane d holds run d's position `lo` and
// length `len`, base time tb (>= cstart, every request within 2^30 of it).
// Each run takes 2^lp neighbouring lanes (len at most SL << lp) or, with
// `pieces`, as many lanes as it needs (lp 0, run_pieces<SL>(len) at most 64).
template <int SL>
DEVI uint32_t run_pieces(uint32_t len) { return (len + SL - 1) / SL; }
template <int SL>
DEVI void sort_take(const DieOrder &D, uint32_t lo, uint32_t len, uint32_t lp, int64_t cstart, int64_t tb,
                    uint64_t (&slot)[SLOTS_MAX], bool pieces = false) {
  const uint32_t lane = lane_id();
  uint32_t d = lane >> lp, skip = (lane & ((1u << lp) - 1)) * SL;
  if (pieces) {  // the lane's run: the first whose pieces end past the lane
    const uint32_t end = wave_incl_sum(run_pieces<SL>(len));
    uint32_t a = 0, b = 63;
    for (int step = 0; step < 6; step++) {
      const uint32_t mid = (a + b) >> 1;
      if ((uint32_t)__shfl((int)end, (int)mid) > lane) b = mid;
      else a = mid + 1;
    }
    d = a;
    skip = (lane - ((uint32_t)__shfl((int)end, (int)d) - run_pieces<SL>((uint32_t)__shfl((int)len, (int)d)))) * SL;
  }
  const uint32_t at = __shfl(lo, (int)d) + skip, have = __shfl(len, (int)d);
  const uint32_t cnt = have > skip ? have - skip : 0u;
  uint64_t a[SL];
  if (D.narrow) {
    const uint64_t *DX = reinterpret_cast<const uint64_t *>(D.DD) + at;
    const uint32_t sub = (uint32_t)(tb - cstart);
#pragma unroll
    for (int i = 0; i < SL; i++) a[i] = (uint32_t)i < cnt ? DX[i] : 0;
#pragma unroll
    for (int i = 0; i < SL; i++)
      a[i] = (uint32_t)i < cnt
                 ? (KEY_TOP | (uint64_t)((uint32_t)(a[i] >> 32) - sub) << 31 | (uint32_t)a[i])
                 : KEY_NONE64;
  } else {
#pragma unroll
    for (int i = 0; i < SL; i++) {
      a[i] = KEY_NONE64;
      if ((uint32_t)i < cnt) a[i] = KEY_TOP | (uint64_t)(D.DD[at + i] - tb) << 31 | D.IX[at + i];
    }
  }
  merge_runs<SL>(a, lp);
#pragma unroll
  for (int i = 0; i < SLOTS_MAX; i++) slot[i] = i < SL ? a[i < SL ? i : 0] : KEY_NONE64;
}

// Offset from the base time held by a slot.
template <bool SORT>
DEVI int64_t slot_off(uint64_t slot) {
  return (int64_t)((slot >> 31) & (SORT ? 0x3FFFFFFFu : 0x1FFFFFu));
}

// Positions and Lindley terms of m ordered requests, per requests a lane.
DEVI void sorted_terms(Merged<SLOTS_MAX> &M, uint32_t m, uint32_t per, int64_t tb, int64_t rank, int64_t xfer) {
  M.boff = lane_id() * per;
  M.cnt = m > M.boff ? min(m - M.boff, per) : 0u;
  M.loc = NEG;
  const int64_t cst = tb - rank * xfer;
#pragma unroll
  for (int i = 0; i < SLOTS_MAX; i++)
    if ((uint32_t)i < M.cnt)
      M.loc = imax(M.loc, cst + slot_off<true>(M.slot[i]) - (int64_t)mul32(M.boff + i, (uint32_t)xfer));
}

// The next requests of a cell that one step cannot hold: up to the first one
// that the longest runs' lanes or the keys' offsets (2^30 from the earliest
// left) leave out.  cur/hi: lane d's run; returns the step's requests of the
// lane's run and its base time, or false at the end.  (One hot die queue in a
// sparse stream makes its cells big; steps of a fixed 2^15 ns then took them
// nearly a request at a time, 2.8 ms for 300,000 requests on 64 queues a
// channel.)
DEVI bool big_step(const DieOrder &D, uint32_t cur, uint32_t hi, uint32_t lp, int64_t cstart, int64_t &tb,
                   uint32_t &cnt) {
  const uint32_t rem = hi - cur, most = 16u << lp;
  if (__ballot(rem != 0) == 0) return false;
  // the wave's smallest time, by a maximum of 2^62 - time (0 where none)
  tb = TIME_LIMIT - wave_max(rem ? TIME_LIMIT - D.time(cur, cstart) : 0);
  int64_t te = tb + (int64_t(1) << SUB_LG_MAX);
  if (rem > most) te = imin(te, D.time(cur + most, cstart));
  te = TIME_LIMIT - wave_max(TIME_LIMIT - te);
  cnt = min(rem, most);
  if (cnt && D.time(cur + cnt - 1, cstart) >= te) {  // (each run ascends)
    uint32_t a = 0, b = cnt - 1;
    while (a < b) {
      const uint32_t mid = (a + b) >> 1;
      if (D.time(cur + mid, cstart) < te) a = mid + 1;
      else b = mid;
    }
    cnt = a;
  }
  return true;
}

// Order a cell by the lane merge.
DEVI void cell_sort(const DieOrder &D, const CellRuns &cr, const Geo &g, uint32_t lp, uint32_t shift,
                    int64_t cstart, Merged<SLOTS_MAX> &M) {
  const uint32_t len = cr.hi - cr.lo;
  M.m = wave_sum(len);
  M.cnt = 0;
  M.boff = 0;
  M.head = CMIN_NONE;
  M.rank0 = 0;
  M.loc = NEG;
  M.big = false;
  if (M.m == 0) return;
  M.rank0 = wave_sum(cr.r0);
  const uint32_t longest = wave_umax(len);
  M.head = ~wave_umax(len ? ~D.index(cr.lo) : 0u);  // a run's first entry has its smallest index
  M.big = longest > (16u << lp) || shift > SUB_LG_MAX;
  // A run or two longer than their lanes, in a cell whose requests fit the
  // wave: the lanes are dealt out by need (one hot die queue in a sparse
  // stream; a call of 9,000 requests on 8 x 64
  // queues 188 -> 63 us)
  if (M.big && shift <= SUB_LG_MAX) {
    uint32_t per = 0;
    if (wave_sum(run_pieces<4>(len)) <= 64) {
      per = 4;
      sort_take<4>(D, cr.lo, len, 0, cstart, cstart, M.slot, true);
    } else if (wave_sum(run_pieces<16>(len)) <= 64) {
      per = 16;
      sort_take<16>(D, cr.lo, len, 0, cstart, cstart, M.slot, true);
    }
    if (per) {
      M.big = false;
      sorted_terms(M, M.m, per, cstart, M.rank0, g.xfer);
      return;
    }
  }
  uint32_t cur = cr.lo, take = len, m = M.m;
  int64_t tb = cstart, rank = M.rank0, term = NEG;
  // one step, or as many as a big cell takes (only their terms are kept)
  while (!M.big || big_step(D, cur, cr.hi, lp, cstart, tb, take)) {
    const uint32_t most = M.big ? wave_umax(take) : longest;
    if (M.big) m = wave_sum(take);
    uint32_t per;
    if (most <= (2u << lp)) {
      per = 2;
      sort_take<2>(D, cur, take, lp, cstart, tb, M.slot);
    } else if (most <= (4u << lp)) {
      per = 4;
      sort_take<4>(D, cur, take, lp, cstart, tb, M.slot);
    } else if (most <= (8u << lp)) {
      per = 8;
      sort_take<8>(D, cur, take, lp, cstart, tb, M.slot);
    } else {
      per = 16;
      sort_take<16>(D, cur, take, lp, cstart, tb, M.slot);
    }
    sorted_terms(M, m, per, tb, rank, g.xfer);
    if (!M.big) return;
    term = imax(term, wave_max(M.loc));
    cur += take;
    rank += m;
  }
  M.loc = term;
  M.cnt = 0;
}

// Completions of an ordered cell given its entering term gin and the base
// time of its slots (bucket merge: of bucket 0): staged in the band when they
// fit, else stored directly.  mytop: staged span used.
template <bool SORT, int SL>
DEVI void cell_emit(const Merged<SL> &M, const Geo &g, int64_t tb, int64_t gin, uint32_t lo, int64_t wbase,
                    uint32_t *stage, int64_t *__restrict__ complete, uint32_t n, uint32_t *errb,
                    uint32_t &mytop) {
  if (M.m == 0) return;
  const uint32_t lane = lane_id();
  const int64_t xfer = g.xfer;
  const int64_t cst = tb + (SORT ? 0 : ((int64_t)lane << g.lg_tR)) - M.rank0 * xfer;
  int64_t carry = __shfl_up(wave_incl_max(M.loc), 1);
  if (lane == 0) carry = NEG;
  carry = imax(carry, gin);
  const int64_t r0x = M.rank0 * xfer;
#pragma unroll
  for (int i = 0; i < SL; i++) {
    if ((uint32_t)i < M.cnt) {
      const int64_t v = cst + slot_off<SORT>(M.slot[i]) - (int64_t)mul32(M.boff + i, (uint32_t)xfer);
      carry = imax(carry, v);
      const int64_t cpl = r0x + (int64_t)mul32(M.boff + i + 1, (uint32_t)xfer) + carry;
      if (cpl >= TIME_LIMIT) *errb |= ERR_OVERFLOW;
      const uint32_t ix = (uint32_t)M.slot[i] & 0x7FFFFFFFu;
      if (ix < n) {
        const uint32_t rel = ix - lo;
        const uint64_t off = (uint64_t)(cpl - wbase);
        if (ix >= lo && rel < WIN_SLOTS && off < WIN_EMPTY) {
          stage[win_slot(rel)] = (uint32_t)off;
          mytop = max(mytop, rel + 1);
        } else {
          complete[ix] = cpl;
        }
      }
    }
  }
}

// Completions of a cell of the lane merge; a big cell takes its steps again,
// now with the entering term.
DEVI void sort_emit(const DieOrder &D, const CellRuns &cr, Merged<SLOTS_MAX> &M, const Geo &g, uint32_t lp,
                    int64_t cstart, int64_t gin, uint32_t lo, int64_t wbase, uint32_t *stage,
                    int64_t *__restrict__ complete, uint32_t n, uint32_t *errb, uint32_t &mytop) {
  uint32_t cur = cr.lo, take = 0;
  int64_t tb = cstart;
  while (!M.big || big_step(D, cur, cr.hi, lp, cstart, tb, take)) {
    if (M.big) {
      M.m = wave_sum(take);
      sort_take<16>(D, cur, take, lp, cstart, tb, M.slot);
      sorted_terms(M, M.m, 16, tb, M.rank0, g.xfer);
    }
    cell_emit<true, SLOTS_MAX>(M, g, tb, gin, lo, wbase, stage, complete, n, errb, mytop);
    if (!M.big) return;
    gin = imax(gin, wave_max(M.loc));
    cur += take;
    M.rank0 += M.m;
  }
}

// Requests of channel c in the call (lanes < Dk read one die queue each).
DEVI uint32_t chan_total(const uint32_t *__restrict__ totals, uint32_t Dk, uint32_t c) {
  const uint32_t lane = lane_id();
  return wave_sum(lane < Dk ? totals[c * Dk + lane] : 0u);
}

// Units of the channel stage, cells ordered by the bucket merge or (SORT)
// the lane merge.
template <bool SORT, int SL>
DEVI void chan_units(WinLds &S, const DieOrder &D, const uint32_t *__restrict__ LB,
                     const uint32_t *__restrict__ seg_start, const uint32_t *__restrict__ totals, const Geo &g,
                     CallCtl *ctl, const DevState *st, uint64_t *WAGG, uint64_t *WINC,
                     int64_t *__restrict__ complete, int64_t *__restrict__ cfnew, uint32_t gmax, uint32_t n) {
  const uint32_t G = ctl->G, shift = ctl->shift, C = g.C;
  const int64_t cbase = ctl->cbase, xfer = g.xfer;
  const uint32_t t = threadIdx.x, lane = t & 63;
  const uint32_t w = __builtin_amdgcn_readfirstlane(t >> 6);  // uniform: the cells' bounds stay scalar
  // cells of a unit: fewer where the call has too few to give every
  // workgroup a full unit (1 M requests on 16 channels, 128 windows: 74 us a
  // call with 16 or 8 cells a unit, 80 with 32)
  uint32_t cells = SORT ? WIN_WAVES : 2 * WIN_WAVES;
  while (cells > WIN_WAVES / 2 && (uint64_t)G * C <= (uint64_t)gridDim.x * (cells / 2)) cells >>= 1;
  const uint32_t Cg = min(C, cells);                    // channels of a unit
  const uint32_t NG = (C + cells - 1) / cells;
  const uint32_t NW = cells / Cg;                       // windows of a unit (1 if there are several groups)
  const uint32_t U = (G + NW - 1) / NW * NG;
  const uint32_t lp = run_lanes_lg(g.Dk);
  for (uint32_t q = t; q < WIN_SLOTS; q += WIN_THREADS) S.stage[q] = WIN_EMPTY;
  uint32_t errb = 0;
  while (true) {
    if (t == 0) S.unit = atomicAdd(&ctl->wctr, 1u);
    __syncthreads();
    const uint32_t u = S.unit;
    if (u >= U) break;  // the same for the whole workgroup
    const uint32_t jw = u / NG, c0 = (u - jw * NG) * cells;
    // the wave's cells (channel C: none)
    uint32_t ca = C, cb = C, ja = 0, jb = 0;
    {
      const uint32_t qa = w / Cg, qb = (w + WIN_WAVES) / Cg;
      ja = jw * NW + qa;
      jb = jw * NW + qb;
      if (w < cells && qa < NW && ja < G) ca = min(C, c0 + w - qa * Cg);
      if (!SORT && w + WIN_WAVES < cells && qb < NW && jb < G) cb = min(C, c0 + w + WIN_WAVES - qb * Cg);
    }
    const int64_t sa = cbase + ((int64_t)ja << shift), sb = cbase + ((int64_t)jb << shift);
    Merged<SL> A, B;
    A.m = B.m = 0;
    CellRuns ra = {0, 0, 0};
    if constexpr (SORT) {
      if (ca < C) {
        ra = cell_runs(LB, seg_start, totals, g.Dk, gmax, ca, ja);
        cell_sort(D, ra, g, lp, shift, sa, A);
      }
    } else {
      if (ca < C) {
        const CellRuns cr = cell_runs(LB, seg_start, totals, g.Dk, gmax, ca, ja);
        uint64_t xv[SL];
        load_runs<SL>(D.DD, cr, (int)g.Dk, xv);
        cell_merge<SL>(S.tbl[w], cr, xv, g, sa, A, &errb);
      }
      if (cb < C) {
        const CellRuns cr = cell_runs(LB, seg_start, totals, g.Dk, gmax, cb, jb);
        uint64_t xv[SL];
        load_runs<SL>(D.DD, cr, (int)g.Dk, xv);
        cell_merge<SL>(S.tbl[w], cr, xv, g, sb, B, &errb);
      }
    }
    const int64_t ma = A.m ? wave_max(A.loc) : NEG, mb = B.m ? wave_max(B.loc) : NEG;
    if (lane == 0) {
      if (ca < C) agent_store64(&WAGG[(size_t)ca * gmax + ja], enc_time(ma));
      if (cb < C) agent_store64(&WAGG[(size_t)cb * gmax + jb], enc_time(mb));
    }
    int64_t ga = NEG, gb = NEG;
    look_back2(WAGG, WINC, C, gmax, ja, jb, ca, cb, ca < C ? st->chan_free[ca] : NEG,
               cb < C ? st->chan_free[cb] : NEG, ga, gb, &errb);
    const int64_t ia = imax(ga, ma), ib = imax(gb, mb);
    if (lane == 0) {
      if (ca < C) agent_store64(&WINC[(size_t)ca * gmax + ja], enc_time(ia));
      if (cb < C) agent_store64(&WINC[(size_t)cb * gmax + jb], enc_time(ib));
    }
    if (ca < C && ja == G - 1) {  // the channel's clock after the call
      const uint32_t ta = chan_total(totals, g.Dk, ca);
      if (lane == 0) {
        cfnew[ca] = (int64_t)ta * xfer + ia;
        if (ta) atomicMax((long long *)&ctl->max_cpl, (long long)((int64_t)ta * xfer + ia));
      }
    }
    if (cb < C && jb == G - 1) {
      const uint32_t tb = chan_total(totals, g.Dk, cb);
      if (lane == 0) {
        cfnew[cb] = (int64_t)tb * xfer + ib;
        if (tb) atomicMax((long long *)&ctl->max_cpl, (long long)((int64_t)tb * xfer + ib));
      }
    }
    // band start (smallest index of the unit's requests) and completion base
    // (a lower bound of every completion of the unit)
    uint32_t mn = min(A.m ? A.head : CMIN_NONE, B.m ? B.head : CMIN_NONE);
    int64_t bmin = INT64_MAX;
    if (A.m) bmin = imin(bmin, (A.rank0 + 1) * xfer + ga);
    if (B.m) bmin = imin(bmin, (B.rank0 + 1) * xfer + gb);
    if (lane == 0) {
      S.rmin[w] = mn;
      S.rbase[w] = bmin;
    }
    if (t == 0) S.top = 0;
    __syncthreads();
    uint32_t lo = CMIN_NONE;
    int64_t wbase = INT64_MAX;
#pragma unroll
    for (int k = 0; k < WIN_WAVES; k++) {
      lo = min(lo, S.rmin[k]);
      wbase = imin(wbase, S.rbase[k]);
    }
    if (lo != CMIN_NONE) {  // the same for the whole workgroup
      uint32_t top = 0;
      if constexpr (SORT) {
        sort_emit(D, ra, A, g, lp, sa, ga, lo, wbase, S.stage, complete, n, &errb, top);
      } else {
        cell_emit<false, SL>(A, g, sa, ga, lo, wbase, S.stage, complete, n, &errb, top);
        cell_emit<false, SL>(B, g, sb, gb, lo, wbase, S.stage, complete, n, &errb, top);
      }
      top = wave_umax(top);
      if (lane == 0 && top) atomicMax(&S.top, top);
      __syncthreads();
      const uint32_t used = S.top;
      for (uint32_t q = t; q < used; q += WIN_THREADS) {
        const uint32_t sq = win_slot(q);
        const uint32_t v = S.stage[sq];
        if (v != WIN_EMPTY) {
          complete[lo + q] = wbase + (int64_t)v;
          S.stage[sq] = WIN_EMPTY;
        }
      }
    }
    __syncthreads();
  }
  if (errb) atomicOr(&ctl->late, errb);
}

// SL: die runs per channel of the bucket merge; WHAT: the grids this kernel
// takes (it returns at once on others).  One kernel for both costs the bucket
// merge 17 spilled registers, 6.28 ms against 6.03 on 2^28 requests; two
// kernels cost a launch, 4 us.
constexpr int GRID_BUCKET = 1, GRID_LANE = 2;
template <int SL, int WHAT>
__global__ __launch_bounds__(WIN_THREADS) void k_cell_chan(
    const int64_t *__restrict__ DD, const uint32_t *__restrict__ IX, const uint32_t *__restrict__ LB,
    const uint32_t *__restrict__ seg_start, const uint32_t *__restrict__ totals, Geo g, CallCtl *ctl,
    const DevState *st, uint64_t *WAGG, uint64_t *WINC, int64_t *__restrict__ complete,
    int64_t *__restrict__ cfnew, uint32_t gmax, uint32_t n) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (agent_load32(&ctl->err) || ctl->G == 0) return;
  WinLds &S = *(WinLds *)smem;
  const DieOrder D = {DD, IX, ctl->shift <= 32};
  const bool bucket = grid_bucketable<SL>(g, ctl->shift);
  if constexpr ((WHAT & GRID_BUCKET) != 0)
    if (bucket)
      chan_units<false, SL>(S, D, LB, seg_start, totals, g, ctl, st, WAGG, WINC, complete, cfnew, gmax, n);
  if constexpr ((WHAT & GRID_LANE) != 0)
    if (!bucket)
      chan_units<true, SLOTS_MAX>(S, D, LB, seg_start, totals, g, ctl, st, WAGG, WINC, complete, cfnew, gmax, n);
}
// Calls of at least this many requests take a kernel per kind of grid.
constexpr int64_t CHAN_SPLIT = int64_t(1) << 22;

// ------------------------------------------------------------------ k_finalize

__global__ __launch_bounds__(BLK) void k_finalize(int64_t *__restrict__ complete, int64_t n,
                                                  CallCtl *ctl, DevState *st,
                                                  const int64_t *__restrict__ dfnew,
                                                  const uint32_t *__restrict__ totals,
                                                  const int64_t *__restrict__ cfnew, uint32_t K,
                                                  uint32_t C) {
  const uint32_t late = agent_load32(&ctl->late), err = agent_load32(&ctl->err) | late;
  if (err) {
    for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
      complete[i] = HBF_TIME_ERROR;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ctl->err = err;  // (`late` decides the same for workgroups that read this one)
      atomicOr(&st->sticky, err);
      st->call_err = 0;
    }
    return;
  }
  if (blockIdx.x != 0) return;
  for (uint32_t k = threadIdx.x; k < K; k += BLK)
    if (totals[k]) st->die_free[k] = dfnew[k];
  if (ctl->G)
    for (uint32_t c = threadIdx.x; c < C; c += BLK) st->chan_free[c] = cfnew[c];
}

// ------------------------------------------------------------------ classify + reset

template <bool POW2>
__global__ __launch_bounds__(BLK) void k_classify(const uint64_t *__restrict__ addr, int64_t n,
                                                  uint64_t *__restrict__ map, Geo g, RangeTable rt,
                                                  DevState *st) {
  __shared__ LdsRanges lr;
  load_ranges(&lr, rt);
  __syncthreads();
  uint32_t errb = 0;
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) {
    const uint64_t a = addr[i];
    const int r = find_range(&lr, a);
    uint64_t word = 0;
    if (r >= 0) {
      const Loc L = map_page<POW2>(g, dev_page<POW2>(g, &lr, r, a));
      if (L.page > 0xffffffffull) {
        errb |= ERR_MAP;
      } else {
        word = (uint64_t(1) << 63) | ((uint64_t)lr.rid[r] << 56) | ((uint64_t)L.plane << 50) |
               ((uint64_t)L.die << 42) | ((uint64_t)L.ch << 32) | L.page;
      }
    }
    map[i] = word;
  }
  if (errb) atomicOr(&st->sticky, errb);
}

__global__ void k_reset(DevState *st) {
  for (uint32_t k = threadIdx.x; k < MAX_KEYS; k += blockDim.x) {
    st->die_free[k] = NEG;
    st->ref_pend[k] = 0;  // pending refresh quanta are dropped
    st->ref_head[k] = 0;
  }
  for (uint32_t c = threadIdx.x; c < MAX_CHANNELS; c += blockDim.x) st->chan_free[c] = NEG;
  if (threadIdx.x == 0) {  // the vmem route: idle, no burst
    st->vfree = NEG;
    st->vlast = 0;
    st->vburst = 0;
    st->vhave = 0;
  }
}

// ------------------------------------------------------------------ refresh bookkeeping

// After a call on the refresh path: die queue k's first min(pending, its
// admissions) quanta were claimed.  Success retires them; a failed call
// claims nothing, so their completion cells go back to pending.
__global__ __launch_bounds__(BLK) void k_refresh_commit(const CallCtl *ctl, DevState *st,
                                                        const uint32_t *__restrict__ totals, uint32_t K) {
  const uint32_t err = agent_load32(&ctl->err);
  for (uint32_t k = blockIdx.x * BLK + threadIdx.x; k < K; k += gridDim.x * BLK) {
    const uint32_t R = st->ref_pend[k], used = min(R, totals[k]);
    if (!used) continue;
    if (err) {
      int64_t *const *q = st->ref_slot + st->ref_off[k] + st->ref_head[k];
      for (uint32_t r = 0; r < used; r++) *q[r] = REFRESH_PENDING;
    } else {
      st->ref_head[k] += used;
      st->ref_pend[k] = R - used;
    }
  }
}

// Idle-window drain: each die queue, oldest quantum first, starts the next
// one at max(its clock, t_from) while it ends by t_to.
__global__ __launch_bounds__(BLK) void k_refresh_drain(DevState *st, uint32_t K, int64_t tQ, int64_t t_from,
                                                       int64_t t_to) {
  const uint32_t k = blockIdx.x * BLK + threadIdx.x;
  if (k >= K) return;
  uint32_t R = st->ref_pend[k], h = st->ref_head[k];
  if (!R) return;
  int64_t t = imax(st->die_free[k], t_from);  // NEG (idle since -inf) -> t_from
  int64_t *const *q = st->ref_slot + st->ref_off[k];
  const uint32_t R0 = R;
  while (R && t + tQ <= t_to) {
    t += tQ;
    *q[h++] = t;
    R--;
  }
  if (R != R0) {
    st->die_free[k] = t;
    st->ref_head[k] = h;
    st->ref_pend[k] = R;
  }
}

__global__ __launch_bounds__(BLK) void k_fill(int64_t *__restrict__ p, int64_t n, int64_t v) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) p[i] = v;
}

// ------------------------------------------------------------------ launchers

const char *const kKernelNames[] = {"k_die_reduce", "k_tile_scan", "k_die_scatter", "k_cell_chan",
                                    "k_finalize", "k_small"};
const int kNumTimedKernels = 6;
constexpr int SMALL_SLOT = 5;  // k_small's timing slot

static size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

// LDS of pass 1: range table | amax[K], cmax[K] i64 | cnt[K] | wcnt[DWAVES][K] u16 | tot[K] u16 |
// refp[K] u32 | tag[DWAVES][K] u32
size_t lds_die_reduce(uint32_t K) {
  return align16(sizeof(LdsRanges)) + K * (8 + 8 + 4) + DWAVES * K * 2 + K * 2 + 4 + K * 4 + DWAVES * K * 4;
}
size_t lds_die_count(uint32_t K) { return align16(sizeof(LdsRanges)) + K * 4; }
static size_t lds_die_scatter_sc(uint32_t K, int SC) {
  const size_t cp = SC == 2 ? chunk_pad<2>() : chunk_pad<1>();
  return cp * 8 + (size_t)K * (sizeof(KeyA) + sizeof(KeyW) + 4 + 4 + (SC == 2 ? 4 : 0)) + cp * 6;
}
constexpr size_t LDS_MAX = 160 * 1024;
// two chunks per step where their LDS fits
static int die_scatter_sc(uint32_t K) { return lds_die_scatter_sc(K, 2) <= LDS_MAX ? 2 : 1; }
size_t lds_die_scatter(uint32_t K) { return lds_die_scatter_sc(K, die_scatter_sc(K)); }

hipError_t launch_time_requests(const Geo &g, const RangeTable &rt, const Layout &Lo, char *ws,
                                DevState *st, const uint64_t *addr, const int64_t *issue,
                                int64_t *complete, hipStream_t s, hipEvent_t *ev, int n_ev,
                                bool refresh) {
  if (g.vmem) return launch_vmem(g, rt, Lo, ws, st, addr, issue, complete, s);
  CallCtl *ctl = (CallCtl *)(ws + Lo.off_ctl);
  if (small_path_ok(g, Lo.n, refresh)) {  // one launch; timed in its own slot
    for (int i = 0; i <= SMALL_SLOT && ev && i < n_ev; i++) hipEventRecord(ev[i], s);
    const hipError_t es = launch_small(g, rt, st, ctl, addr, issue, Lo.n, complete, s);
    for (int i = SMALL_SLOT + 1; ev && i < n_ev; i++) hipEventRecord(ev[i], s);
    return es;
  }
  uint32_t *agg_cnt = (uint32_t *)(ws + Lo.off_agg_cnt);
  int64_t *agg_A = (int64_t *)(ws + Lo.off_agg_A);
  int64_t *tin_L = (int64_t *)(ws + Lo.off_tin_L);
  uint32_t *tin_base = (uint32_t *)(ws + Lo.off_tin_base);
  uint32_t *totals = (uint32_t *)(ws + Lo.off_totals);
  uint32_t *seg = (uint32_t *)(ws + Lo.off_seg);
  int64_t *dfnew = (int64_t *)(ws + Lo.off_dfnew);
  int64_t *cfnew = (int64_t *)(ws + Lo.off_cfnew);
  int64_t *DD = (int64_t *)(ws + Lo.off_dd);
  uint32_t *IX = (uint32_t *)(ws + Lo.off_ix);
  uint32_t *KR = (uint32_t *)(ws + Lo.off_kr);
  uint32_t *LB = (uint32_t *)(ws + Lo.off_lb);
  uint64_t *WST = (uint64_t *)(ws + Lo.off_wst);
  const bool p2 = g.pow2 != 0;
  int evi = 0;
  auto mark = [&]() {
    if (ev && evi < n_ev) hipEventRecord(ev[evi++], s);
  };
  hipError_t e;
  mark();
  // (the call's control block is set up by the tile scan; errors before it
  // go to the model's call_err, which is zero between calls)
  const dim3 tq((g.K + TQ - 1) / TQ);
  auto tile_scan = [&](auto kfn) {
    hipLaunchKernelGGL(kfn, tq, dim3(TSBLK), 0, s, agg_cnt, agg_A, Lo.nt, g, st, tin_L, tin_base, totals, dfnew, seg,
                       issue, Lo.gmax, Lo.s0, ctl);
    return hipGetLastError();
  };
  if (refresh) {
    // count pass and per-tile rank bases first (timed with pass 1)
    const size_t lds = lds_die_count(g.K);
    if (p2)
      hipLaunchKernelGGL(k_die_count<true>, dim3(Lo.nt), dim3(DBLK), lds, s, addr, Lo.n, g, rt, Lo.tile_elems,
                         agg_cnt);
    else
      hipLaunchKernelGGL(k_die_count<false>, dim3(Lo.nt), dim3(DBLK), lds, s, addr, Lo.n, g, rt,
                         Lo.tile_elems, agg_cnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = tile_scan(k_tile_scan<TS_COUNT>)) != hipSuccess) return e;
  }
  {
    const size_t lds = lds_die_reduce(g.K);
    auto kfn = p2 ? (refresh ? k_die_reduce<true, true> : k_die_reduce<true, false>)
                  : (refresh ? k_die_reduce<false, true> : k_die_reduce<false, false>);
    hipLaunchKernelGGL(kfn, dim3(Lo.nt), dim3(DBLK), lds, s, addr, issue, Lo.n, complete, g, rt, Lo.tile_elems,
                       agg_cnt, agg_A, KR, tin_base, st);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark();
  if ((e = refresh ? tile_scan(k_tile_scan<TS_REFRESH>) : tile_scan(k_tile_scan<TS_PLAIN>)) != hipSuccess) return e;
  mark();
  {
    const size_t lds = lds_die_scatter(g.K);
    const bool two = die_scatter_sc(g.K) == 2;
    hipLaunchKernelGGL(refresh ? (two ? k_die_scatter<true, 2> : k_die_scatter<true, 1>)
                               : (two ? k_die_scatter<false, 2> : k_die_scatter<false, 1>),
                       dim3(Lo.nt), dim3(SBLK), lds, s,
                       issue, KR, Lo.n, g, Lo.tile_elems, tin_L, tin_base, seg, totals, DD, IX, LB, Lo.gmax, ctl,
                       st, WST, g.reg_block ? (int64_t *)(ws + Lo.off_iss) : (int64_t *)nullptr);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark();
  if (g.reg_block) {
    // media variant: the channel stage simulated per channel in service
    // order (timed in the first channel-stage slot)
    if ((e = launch_regblock(g, (const uint64_t *)DD, IX, (const int64_t *)(ws + Lo.off_iss), seg, totals, st, ctl,
                             complete, dfnew, cfnew, refresh, s)) != hipSuccess)
      return e;
  } else {
    // channel stage: one 1,024-thread workgroup per CU (its LDS holds a
    // unit's band)
    int dev = 0, ncu = 256;
    hipGetDevice(&dev);
    hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    uint64_t *WAGG = WST, *WINC = WST + (size_t)Lo.gmax * g.C;
    auto chan = [&](auto kfn) {
      hipLaunchKernelGGL(kfn, dim3((uint32_t)ncu), dim3(WIN_THREADS), sizeof(WinLds), s, DD, IX, LB, seg, totals, g,
                         ctl, st, WAGG, WINC, complete, cfnew, Lo.gmax, (uint32_t)Lo.n);
      return hipGetLastError();
    };
    constexpr int BOTH = GRID_BUCKET | GRID_LANE;
    if (g.Dk > SLOTS_MAX) {
      e = chan(k_cell_chan<SLOTS_MAX, GRID_LANE>);
    } else if (Lo.n < CHAN_SPLIT) {
      e = chan(g.Dk <= 4 ? k_cell_chan<4, BOTH> : g.Dk <= 8 ? k_cell_chan<8, BOTH> : k_cell_chan<16, BOTH>);
    } else {
      e = chan(g.Dk <= 4   ? k_cell_chan<4, GRID_BUCKET>
               : g.Dk <= 8 ? k_cell_chan<8, GRID_BUCKET> : k_cell_chan<16, GRID_BUCKET>);
      if (e == hipSuccess) e = chan(k_cell_chan<SLOTS_MAX, GRID_LANE>);
    }
    if (e != hipSuccess) return e;
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark();
  {
    int64_t blocks = (Lo.n + BLK - 1) / BLK;  // (only a failed call needs more than one)
    if (blocks > 256) blocks = 256;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_finalize, dim3((uint32_t)blocks), dim3(BLK), 0, s, complete, Lo.n, ctl, st, dfnew,
                       totals, cfnew, g.K, g.C);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (refresh) {
    hipLaunchKernelGGL(k_refresh_commit, dim3((g.K + BLK - 1) / BLK), dim3(BLK), 0, s, ctl, st, totals, g.K);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  mark();
  while (ev && evi < n_ev) mark();  // the remaining slots (k_small's) take no time
  return hipSuccess;
}

hipError_t launch_classify(const Geo &g, const RangeTable &rt, DevState *st, const uint64_t *addr,
                           int64_t n, uint64_t *map, hipStream_t s) {
  // a large grid (a few requests per thread) keeps the most loads in flight:
  // measured 4.7 TB/s at 8,192 blocks against 5.5+ at 131,072 for this
  // read-8-write-8 stream
  int64_t blocks = (n + BLK - 1) / BLK;
  if (blocks > 131072) blocks = 131072;
  if (blocks < 1) blocks = 1;
  if (g.pow2)
    hipLaunchKernelGGL(k_classify<true>, dim3((uint32_t)blocks), dim3(BLK), 0, s, addr, n, map, g, rt, st);
  else
    hipLaunchKernelGGL(k_classify<false>, dim3((uint32_t)blocks), dim3(BLK), 0, s, addr, n, map, g, rt, st);
  return hipGetLastError();
}

hipError_t launch_reset(DevState *st, hipStream_t s) {
  hipLaunchKernelGGL(k_reset, dim3(1), dim3(BLK), 0, s, st);
  return hipGetLastError();
}

// ------------------------------------------------------------------ closed-loop layers

// Issue time of a layer: t_start for the first, else the previous layer's
// done time + compute_ns (an error value stays negative and fails the layer).
DEVI int64_t layer_time(const int64_t *prev_done, int64_t t_start, int64_t compute_ns) {
  return prev_done ? *prev_done + compute_ns : t_start;
}

__global__ __launch_bounds__(BLK) void k_layer_issue(int64_t *__restrict__ issue, int64_t count,
                                                     const int64_t *prev_done, int64_t t_start,
                                                     int64_t compute_ns) {
  const int64_t t = layer_time(prev_done, t_start, compute_ns);
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLK)
    issue[i] = t;
}

// done = max(t, every completion of the layer), or HBF_TIME_ERROR if the
// layer failed.  Its in-range completions end no later than the last one
// of each channel, which the channel scan recorded in the call's control
// block; native requests complete at t.
__global__ void k_layer_done(const CallCtl *ctl, int64_t count, const int64_t *prev_done, int64_t t_start,
                             int64_t compute_ns, int64_t *done) {
  if (threadIdx.x != 0) return;
  const int64_t t = layer_time(prev_done, t_start, compute_ns);
  int64_t d;
  if (t < 0)
    d = HBF_TIME_ERROR;
  else if (count == 0)
    d = t;
  else if (agent_load32(&ctl->err))
    d = HBF_TIME_ERROR;
  else
    d = imax(t, ctl->max_cpl);
  *done = d;
}

hipError_t launch_layer_issue(int64_t *issue, int64_t count, const int64_t *prev_done, int64_t t_start,
                              int64_t compute_ns, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  int64_t blocks = (count + BLK - 1) / BLK;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_layer_issue, dim3((uint32_t)blocks), dim3(BLK), 0, s, issue, count, prev_done, t_start,
                     compute_ns);
  return hipGetLastError();
}

hipError_t launch_layer_done(const CallCtl *ctl, int64_t count, const int64_t *prev_done, int64_t t_start,
                             int64_t compute_ns, int64_t *done, hipStream_t s) {
  hipLaunchKernelGGL(k_layer_done, dim3(1), dim3(64), 0, s, ctl, count, prev_done, t_start, compute_ns, done);
  return hipGetLastError();
}

hipError_t set_lds_limits(uint32_t K) {
  hipError_t e;
  const int a = (int)lds_die_reduce(K), b = (int)lds_die_scatter(K), c = (int)lds_die_count(K);
  const void *fa[] = {(const void *)k_die_reduce<true, false>, (const void *)k_die_reduce<false, false>,
                      (const void *)k_die_reduce<true, true>, (const void *)k_die_reduce<false, true>};
  for (const void *f : fa)
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, a)) != hipSuccess) return e;
  const void *fb[] = {(const void *)k_die_scatter<false, 1>, (const void *)k_die_scatter<true, 1>,
                      (const void *)k_die_scatter<false, 2>, (const void *)k_die_scatter<true, 2>};
  for (const void *f : fb)
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, b)) != hipSuccess) return e;
  const void *fc[] = {(const void *)k_die_count<true>, (const void *)k_die_count<false>};
  for (const void *f : fc)
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, c)) != hipSuccess) return e;
  if ((e = set_lds_small()) != hipSuccess) return e;
  constexpr int BOTH = GRID_BUCKET | GRID_LANE;
  const void *fw[] = {(const void *)k_cell_chan<4, BOTH>,        (const void *)k_cell_chan<8, BOTH>,
                      (const void *)k_cell_chan<16, BOTH>,       (const void *)k_cell_chan<4, GRID_BUCKET>,
                      (const void *)k_cell_chan<8, GRID_BUCKET>, (const void *)k_cell_chan<16, GRID_BUCKET>,
                      (const void *)k_cell_chan<16, GRID_LANE>};
  for (const void *f : fw)
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(WinLds))) != hipSuccess)
      return e;
  return hipSuccess;
}

hipError_t launch_refresh_drain(const Geo &g, DevState *st, int64_t t_from, int64_t t_to, hipStream_t s) {
  hipLaunchKernelGGL(k_refresh_drain, dim3((g.K + BLK - 1) / BLK), dim3(BLK), 0, s, st, g.K, g.tQ, t_from, t_to);
  return hipGetLastError();
}

// ------------------------------------------------------------------ static scratch

// Scratch of hbf_time_requests_noalloc: one array per GPU, held until the
// process ends.  In host code `scratch` names a host-side stand-in, not a
// device address; the device address comes from hipGetSymbolAddress, once
// per device, with that device current.
static __device__ __align__(256) char scratch[HBF_NOALLOC_SCRATCH_BYTES];
constexpr int SCRATCH_DEVICES = 64;

hipError_t noalloc_scratch(int dev, char **ptr) {
  static std::mutex mu;
  static char *addr[SCRATCH_DEVICES] = {};
  if (dev < 0 || dev >= SCRATCH_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || (uintptr_t)p % 256) return hipErrorInvalidValue;
    addr[dev] = (char *)p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_fill(int64_t *p, int64_t n, int64_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + BLK - 1) / BLK;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill, dim3((uint32_t)blocks), dim3(BLK), 0, s, p, n, v);
  return hipGetLastError();
}

}  // namespace hbf
