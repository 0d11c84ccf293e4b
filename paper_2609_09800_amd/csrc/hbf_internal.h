// Internal declarations shared by the HIP kernels and the C ABI host code.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "hbf.h"

namespace hbf {

// "Idle since minus infinity".  Every modeled time of a call lies in
// [0, 2^62); the prefix maxima of the Lindley form (time - rank * service)
// stay above -2^60, so -2^61 is below every value that can occur.
constexpr int64_t NEG = -(int64_t(1) << 61);
constexpr int64_t ISSUE_LIMIT = int64_t(1) << 61;
constexpr int64_t TIME_LIMIT = int64_t(1) << 62;
constexpr int64_t SERVICE_LIMIT = int64_t(1) << 29;
constexpr int64_t N_LIMIT = int64_t(1) << 31;
constexpr int MAX_RANGES = 64;
constexpr int MAX_KEYS = 2048;      // die queues
constexpr int MAX_CHANNELS = 1024;
constexpr uint16_t KEY_NONE = 0xFFFF;

// per-call / sticky device error bits
constexpr uint32_t ERR_RANGE_TIME = 1u;
constexpr uint32_t ERR_UNSORTED = 2u;
constexpr uint32_t ERR_OVERFLOW = 4u;
constexpr uint32_t ERR_MAP = 8u;
constexpr uint32_t ERR_INTERNAL = 16u;  // a bounded internal wait ran out (never expected)

constexpr int BLK = 256;            // threads per block of the small kernels
constexpr int DBLK = 512;           // threads per block of the two die-stage passes
constexpr int DWAVES = DBLK / 64;
constexpr int DITEMS = 8;           // requests per thread per chunk
constexpr int CHUNK = DBLK * DITEMS;  // 4096 requests staged per chunk
constexpr int TARGET_TILES = 512;   // die-stage tiles: two 512-thread blocks per CU

// Channel stage: a time cell of one channel of minimum width holds at most
// MCAP requests (one step of a wave), MAX_BUCKETS per die queue.  Time
// buckets of width 2^floor(log2 tR) hold at most one request per die.
constexpr int MCAP = 1024;
constexpr int MAX_BUCKETS = 64;
constexpr int MAX_RUNS = 64;        // die queues per channel (D, or D*P)
// Closed-loop layers in one launch: one workgroup per layer ranks each
// layer's requests, so layers are bounded; larger ones take a call per layer.
constexpr int64_t LAYERS_MAX_LAYER = int64_t(1) << 22;
constexpr int LAYERS_MAX_COUNT = 1 << 20;

// Snapshot of the registered ranges, sorted by base (passed by value).
struct RangeTable {
  uint64_t base[MAX_RANGES];
  uint64_t bytes[MAX_RANGES];
  uint64_t pbase[MAX_RANGES];     // first device page of the range
  uint32_t rid[MAX_RANGES];       // registration index
  int32_t n;
};

// Geometry and timing (passed by value).
struct Geo {
  uint32_t C, D, P;
  uint32_t Dk;        // die queues per channel (D, or D*P)
  uint32_t K;         // die queues (C * Dk)
  uint32_t page_bytes;
  uint32_t plane_parallel;
  uint32_t pow2;      // page_bytes, C, D, P all powers of two
  uint32_t lg_page, lg_C, lg_D, lg_P;
  uint32_t lg_tR;     // floor(log2(tR)): bucket width of the channel merge
  int64_t tR, xfer;
  int64_t tQ;         // die time of one refresh quantum (tR + tPROG), 0 if unset
  uint32_t reg_block; // media variant: die page-register blocking
  uint32_t vmem;      // timing source: the calibrated end-to-end vmem curve
  int64_t vknot[6];   // vmem burst cost T(L) at L = 1, 4, 16, 64, 256, 512 pages
};

// Persistent device state of a model.  Refresh quanta pending at die queue
// k are entries ref_off[k] + ref_head[k] .. + ref_pend[k] - 1 of ref_slot,
// oldest first; each entry points at the caller's cell that receives the
// quantum's completion time.
struct DevState {
  int64_t die_free[MAX_KEYS];     // NEG = idle
  int64_t chan_free[MAX_CHANNELS];
  uint32_t sticky;                // sticky error bits
  uint32_t call_err;              // errors of the call in progress, from pass 1 (zero between calls)
  uint32_t ref_pend[MAX_KEYS];
  uint32_t ref_head[MAX_KEYS];
  uint32_t ref_off[MAX_KEYS];
  int64_t **ref_slot;
  // Instrumented GEMV with delays: the time origin of the current call
  // (wall-clock ticks, read by the call's first kernel).
  uint64_t gemv_origin;
  // vmem route: its clock (NEG = idle), the device page of the last
  // in-range access and the length of the burst it ended (vhave = 0: none)
  int64_t vfree;
  uint64_t vlast;
  int64_t vburst;
  uint32_t vhave;
  uint32_t scan_ctr;              // finished blocks of the tile scan (zero between launches)
};

// Completion cell of a refresh quantum that has not been served.
constexpr int64_t REFRESH_PENDING = -1;

// Per-call control block (in the workspace).  The waves of a workgroup read
// `err` one by one and leave the call on it, so no kernel that does so may
// write it: what the channel stage finds goes to `late`, and k_finalize adds it.
struct CallCtl {
  uint32_t err;       // per-call error bits
  uint32_t n_in;      // in-range requests
  uint32_t G;         // time cells per channel
  uint32_t shift;     // log2(cell width in ns)
  int64_t max_dd;     // largest die-done time of the call
  int64_t max_cpl;    // largest in-range completion of the call (NEG if none)
  int64_t cbase;      // origin of the cell grid (= first issue time)
  uint32_t wctr;      // next unit of the channel stage
  uint32_t late;      // error bits found by the channel stage
};

// Workspace layout of one hbf_time_requests call.
struct Layout {
  int64_t n;
  uint32_t nt;            // die-stage tiles
  int64_t tile_elems;
  uint32_t gmax;          // cell budget per channel
  uint32_t s0;            // minimum cell shift
  size_t off_ctl, off_agg_cnt, off_agg_A, off_tin_L, off_tin_base;
  size_t off_totals, off_seg, off_dfnew, off_cfnew;
  size_t off_dd, off_ix, off_kr, off_lb;
  size_t off_wst;             // channel stage: published aggregate and inclusive term per cell
  size_t off_iss;             // register blocking: issue times in die order (n int64)
  // vmem route (tiles of VM_TILE requests): per tile its burst summary, the
  // summary of everything before it, its route-clock pair and entering
  // clock; per request its service (u32); the call's closing state
  size_t off_vsum, off_vin, off_vpair, off_vfin, off_vcost, off_vend;
  size_t off_vwsum, off_vwpair;  // the same summary and pair per wave span of a tile
  size_t total;
};

Layout make_layout(const Geo &g, int64_t n);

// Launchers (hbf_kernels.hip).  All enqueue on `s` and return the first
// launch error.
// refresh: quanta may be pending (the die stage then charges them to the
// admissions that claim them; a count pass comes first)
hipError_t launch_time_requests(const Geo &g, const RangeTable &rt, const Layout &L, char *ws,
                                DevState *st, const uint64_t *addr, const int64_t *issue,
                                int64_t *complete, hipStream_t s, hipEvent_t *ev, int n_ev,
                                bool refresh);
// Register-blocking channel stage (hbf_blocking.hip): one workgroup per channel.
hipError_t launch_regblock(const Geo &g, const uint64_t *DDw, const uint32_t *IX, const int64_t *issue_do,
                           const uint32_t *seg_start, const uint32_t *totals, DevState *st, CallCtl *ctl,
                           int64_t *complete, int64_t *dfnew, int64_t *cfnew, bool ref, hipStream_t s);
// Calibrated vmem curve (hbf_vmem.hip): the whole timing call on the vmem
// route (classification, burst lengths, route clock, complete[]).
constexpr int VM_THREADS = 256;
constexpr int VM_ITEMS = 16;
constexpr int64_t VM_TILE = VM_THREADS * VM_ITEMS;
hipError_t launch_vmem(const Geo &g, const RangeTable &rt, const Layout &L, char *ws, DevState *st,
                       const uint64_t *addr, const int64_t *issue, int64_t *complete, hipStream_t s);
// Closed-loop layers in one launch (hbf_layers.hip): whether a geometry can
// take it on this GPU (every channel's workgroup resident at once), its
// scratch for n requests in L layers, and the launch (host_ls: L + 1 layer
// starts on the host).
bool layers_fast_ok(const Geo &g, int ncu);
size_t layers_ws_bytes(const Geo &g, int64_t n, int L);
hipError_t launch_layers(const Geo &g, const RangeTable &rt, char *ws, DevState *st, const uint64_t *addr,
                         int64_t n, const int64_t *host_ls, int L, int64_t t_start, int64_t compute_ns,
                         int64_t *issue, int64_t *complete, int64_t *done, std::vector<unsigned char> &up,
                         hipEvent_t up_done, hipStream_t s);
hipError_t launch_refresh_drain(const Geo &g, DevState *st, int64_t t_from, int64_t t_to, hipStream_t s);
hipError_t launch_fill(int64_t *p, int64_t n, int64_t v, hipStream_t s);
// Device address of this GPU's static scratch of hbf_time_requests_noalloc
// (HBF_NOALLOC_SCRATCH_BYTES); `dev` must be the current device.
hipError_t noalloc_scratch(int dev, char **ptr);
// Small calls (hbf_small.hip): a whole timing call of at most SMALL_N
// requests by one workgroup, for the plain two-stage model where its LDS fits.
constexpr int64_t SMALL_N = 4096;
constexpr int SMALL_LDS_MAX = 156 * 1024;  // dynamic LDS; the kernel's static LDS fits beside it in 160 KB
bool small_path_ok(const Geo &g, int64_t n, bool refresh);
hipError_t launch_small(const Geo &g, const RangeTable &rt, DevState *st, CallCtl *ctl, const uint64_t *addr,
                        const int64_t *issue, int64_t n, int64_t *complete, hipStream_t s);
hipError_t set_lds_small();
hipError_t launch_classify(const Geo &g, const RangeTable &rt, DevState *st, const uint64_t *addr,
                           int64_t n, uint64_t *map, hipStream_t s);
hipError_t launch_reset(DevState *st, hipStream_t s);
// Closed-loop layers: write the issue times of one layer / reduce its done time.
hipError_t launch_layer_issue(int64_t *issue, int64_t count, const int64_t *prev_done, int64_t t_start,
                              int64_t compute_ns, hipStream_t s);
hipError_t launch_layer_done(const CallCtl *ctl, int64_t count, const int64_t *prev_done, int64_t t_start,
                             int64_t compute_ns, int64_t *done, hipStream_t s);
hipError_t launch_gemv(const uint16_t *W, int E, int K, int N, int page_bytes, const uint16_t *X,
                       int B, float *Y, const int64_t *pi, const int64_t *pc, int64_t *meas,
                       int64_t tick_ps, DevState *st, int ncu, hipStream_t s);
// Capacity-mode frame cache (hbf_cache.hip).  Caches of up to
// CACHE_LDS_MAX frames: the page held by each frame (-1 empty) and a
// prefetched-and-not-yet-hit flag per frame, loaded into LDS per call.
// Larger caches: the number of each page's latest insertion (PINS_NEVER if
// none) and, per frame, a prefetched flag and a hit-since-insertion flag.
// Both: the FIFO head, the counters (hits, faults, prefetch reads,
// prefetched used, evicted unused), the insertion count and the prefetched
// pages resident and unhit (device-memory caches, after each run).
struct CacheCtl {
  uint32_t head;
  uint32_t pad;
  int64_t count[5];
  int64_t ins;
  int64_t pend;
};
struct CacheCfg {
  int64_t *frame_page;
  uint32_t *frame_pf;
  int64_t *pins;
  uint8_t *fpf, *fhit;
  CacheCtl *ctl;
  uint32_t F, d;
};
constexpr int64_t PINS_NEVER = INT64_MIN / 4;
// Chunked solve of a device-memory cache (hbf_cache_chunk.hip).  Per page
// (R entries each, tagged with the chunk's epoch in the high 32 bits): the
// chunk's first access (tag ~epoch, kept by atomicMin) and, for a page
// inserted by the chunk, the time of the fault that inserted it (bits 0-23)
// and its rank among that fault's insertions (bits 24-29).  Per chunk: the
// per-access insertion/fault counts and their exclusive scan (S, Lmax + 1
// entries), the sums per 1,024 accesses and the segment starts.
struct ChunkCtl {
  uint32_t nseg[2];  // segments; odd or even tag
  uint32_t good;     // accesses of the chunk before the first decision that does not hold
  uint32_t epoch;    // last chunk tag used
  uint64_t loose[2];  // candidates outside runs (low word), those near one accessed later (high); odd or even tag
  int64_t lost_old;  // frames filled before the chunk, evicted within it holding a prefetched page never hit
};
struct ChunkCfg {
  uint64_t *at, *tt;
  uint64_t *S;
  uint64_t *bs;
  uint32_t *seg;
  ChunkCtl *ctl;
  uint32_t Lmax;
};
// The words by which the workgroups of one group meet, each in a line of its own.
struct GroupWords {
  uint32_t bar, pad0[31];      // arrivals at barriers
  uint32_t arrived, pad1[31];  // workgroups that have started (group_join)
  uint32_t members, pad2[31];
};
constexpr uint32_t CHUNK_MAX = 1u << 18;          // accesses per chunk that a caller can ask for
constexpr uint32_t CHUNK_LIMIT = 1u << 21;        // accesses per chunk (24 bits of a page's word hold a time)
constexpr uint32_t CHUNK_FIRST = 1u << 20;        // accesses of a call's first chunk
constexpr int CHUNK_GROUPS = 256;                 // caches served at the same time
constexpr uint64_t CHUNK_MAX_R = uint64_t(1) << 26;  // range pages with per-page chunk state
constexpr uint32_t CHUNK_MIN = 16384;            // default accesses per chunk, at least

constexpr uint32_t CACHE_MAX_PREFETCH = 63;  // one fault's candidates fit one wave
// Caches of up to this many frames run with their whole state in LDS (a
// hash of the resident pages); larger ones keep each page's latest
// insertion number in device memory, which needs at least 64 frames (a
// round of 64 accesses without prefetch then never evicts a page it
// inserted, and one fault's insertion offsets, at most 63, stay below F).
constexpr uint32_t CACHE_LDS_MAX = 63;
// Accesses per chunk that hbf_cache_get_chunk reports for a new cache of F
// frames (0: sequential only); unless a length is asked for, chunks are as
// long as their checks let them be, up to chunk_limit.
inline uint32_t chunk_default(uint32_t F, uint64_t R) {
  if (F <= CACHE_LDS_MAX || R > CHUNK_MAX_R) return 0;
  uint32_t c = F / 16;
  return c < CHUNK_MIN ? CHUNK_MIN : (c > CHUNK_MAX ? CHUNK_MAX : c);
}
// The length a cache whose setting is `accesses` (not 0) asks of the chunked
// solve: that one, or 0 (as long as the checks allow) where it is the one
// reported for a new cache, so that putting a saved setting back is no change.
inline uint32_t chunk_asked(uint32_t accesses, uint32_t F, uint64_t R) {
  return accesses == chunk_default(F, R) ? 0 : accesses;
}
// Accesses a chunk's state holds over R pages: the state per access stays
// below the state per page.
inline uint32_t chunk_limit(uint64_t R) {
  const uint64_t c = R / 2;
  return (uint32_t)(c < CHUNK_MIN ? CHUNK_MIN : (c > CHUNK_LIMIT ? CHUNK_LIMIT : c));
}
hipError_t launch_cache_clear(CacheCfg *dev_cfgs, int n_cfg, uint64_t R, uint32_t max_f, hipStream_t s);
// cfg_ids: the caches to run (device, n_cfg entries); every one of them has
// F <= CACHE_LDS_MAX when lds is set, else F > CACHE_LDS_MAX.  max_f: their
// largest frame count.
hipError_t launch_cache_run(const CacheCfg *dev_cfgs, const int *cfg_ids, int n_cfg, bool lds, uint32_t max_f,
                            uint64_t R, const uint64_t *pages, int64_t n, uint8_t *hit, uint64_t *pf_page,
                            int64_t *pf_src, int64_t pf_cap, int64_t *status, int64_t *n_pf_out, hipStream_t s);
hipError_t cache_set_lds_limit();
// Serve pages[0..n) on the caches ids[0..n_cfg) (all with chunk state): one
// launch.  chunk: accesses per chunk (0: as many as pass their check).  hit (n
// entries), pf_*, n_pf: the first cache's, or null.  groups: one entry per
// cache, at most CHUNK_GROUPS of them, zero.
hipError_t launch_cache_chunks(const CacheCfg *dev_cfgs, const ChunkCfg *dev_ccfgs, const int *cfg_ids, int n_cfg,
                               uint64_t R, const uint64_t *pages, int64_t n, uint32_t chunk, uint8_t *hit,
                               uint64_t *pf_page, int64_t *pf_src, int64_t pf_cap, int64_t *status, int64_t *n_pf,
                               GroupWords *groups, hipStream_t s);
hipError_t launch_cache_check(const uint64_t *pages, int64_t n, uint64_t R, int64_t *status, hipStream_t s);
hipError_t launch_cache_pending(const CacheCfg *dev_cfgs, const int *cfg_ids, int n_cfg, uint32_t max_f,
                                const int64_t *status, hipStream_t s);
hipError_t launch_chunk_clear(const ChunkCfg *dev_ccfgs, const int *cfg_ids, int n_cfg, uint64_t R, hipStream_t s);
hipError_t launch_cache_report(const CacheCfg *dev_cfgs, int n_cfg, const int64_t *n_pf, const int64_t *status,
                               int64_t *out, int per_cfg, hipStream_t s);

extern const char *const kKernelNames[];
extern const int kNumTimedKernels;

}  // namespace hbf
