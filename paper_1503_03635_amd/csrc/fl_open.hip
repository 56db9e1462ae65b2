// fl_open.hip -- the facility-opening loop (Alg. 4 with OpenFacilities,
// Alg. 5) on the GPU.
//
// Rung t uses alpha = a[t] (alpha grows before use).  For each unopened
// facility f the loop needs N(f, alpha): the HIP estimate of the unfrozen
// served clients within alpha of f, a predicated query over f's sketch
// (Sec. 4.5).  It is kept exactly as an integer in units of 2^-52 (split into
// two 64-bit words, fix52) over a "live list": the crossed sketch entries
// (distance <= alpha) whose client is still unfrozen, compacted in place at
// the front of f's sketch row.  Per rung:
//   light kernel  (thread per facility): when nothing crossed and no client
//                 froze in the previous rung, N is unchanged; update q and
//                 test the opening condition q >= c(f) directly.
//   heavy kernel  (16 lanes per facility): drop frozen clients from the live
//                 list when clients froze in the previous rung, append newly
//                 crossed entries, recompute N exactly, then update q with
//                 Eq. 2 (first rung, sequential sum in sketch order) or Eq. 3
//                 (eps * alpha * N) and test the opening condition.
//   distance to the open set: multi-source Bellman-Ford from the facilities
//                 opened in this rung.
//   freeze kernel (thread per vertex): unfrozen served clients within
//                 (1 + eps) alpha of an open facility freeze at this rung.
// Several graphs (a disjoint union) run the loop together: rung t is the same
// for every graph still running, alpha and the counters are per graph, and a
// graph leaves the loop when its own stopping rule holds.
//
// The loop's control is on the device (k_open_ctl): each graph's counts and
// flags, the rung, a window of the ladder, whether a look-ahead is due.  The
// host launches the kernels of several rungs at a time and reads back why they
// stopped; kernels of rungs after a stop exit at once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "fl_common.h"
#include "fl_frontier.h"
#include "fl_open.h"

namespace fl {

// status counters per graph: field f of graph g, stripe s at
// [((g * OC_NFIELD + f) * stripes + s) * sstride]; a single graph stripes
// its counters over 64 words on separate 128-byte lines, so that the blocks'
// atomics do not queue on one line
enum { OC_HEAVY = 0, OC_OPENED, OC_FROZEN, OC_FINITE, OC_NUF_DEC, OC_LIVE, OC_NFIELD };

constexpr uint32_t FF_WIN = 256;   // rungs of a look-ahead
constexpr uint32_t LAD_WIN = 2048; // ladder entries held on the device per graph
static_assert(LAD_WIN > 2 * FF_WIN, "a window covers several look-aheads");

// a graph in the loop
struct OpenG {
  uint32_t nF, nO;           // facilities, opened
  uint32_t nU, nUF;          // unfrozen served clients, unopened facilities among them
  uint32_t finite;           // unfrozen clients with a finite distance to the open set
  uint32_t frz_prev;         // some client froze in the previous rung
  uint32_t run, done;        // evaluates the current rung; has left the loop
  uint32_t stuck, gflag;     // the stall check runs; 1: stall guard
  uint32_t rungs;            // last rung evaluated
  int32_t rc;
  double a0, a1;             // first two ladder values
};
enum OpenStop : uint32_t {
  OS_RUN = 0,
  OS_DONE,   // no graph is left in the loop
  OS_STUCK,  // a stall check is due: k_stuck_scan, then this kernel again
  OS_SSSP    // the search of the current rung has not ended: the next rung's launches go on with it
};
struct OpenCtl {
  uint32_t stop;
  uint32_t pending;  // a rung was evaluated and is not closed yet
  uint32_t ff, t0;   // a look-ahead is due; its first rung
  uint32_t tev;      // the rung to evaluate (the first with an event)
  uint32_t base;     // rung of the ladder window's first entry
  uint32_t heavy_cnt, opened_cnt;
  uint32_t stalls;   // stall checks asked for so far
  uint32_t unseeded; // the facilities the rung opened are not labelled yet (see sssp_opened)
};

struct OpenArgs {
  uint32_t n, nF, cap;
  uint32_t stripes, sstride;
  const uint32_t *gid;        // graph of each vertex (nullptr: one graph)
  const SegInfo *seg;
  uint32_t G;
  double eps, one_eps;
  OpenG *og;                  // [G]
  OpenCtl *ctl;
  double *win;                // [G * LAD_WIN] ladder values from rung ctl->base on
  const uint32_t *fac_list;
  const uint32_t *fac_cost;   // vertex-indexed
  uint32_t *sk_rank;          // live region holds client ids
  uint32_t *sk_dist;
  uint32_t *thr;              // rows by facility index
  const uint32_t *cnt;
  const uint8_t *ceff;
  uint32_t *frz;              // vertex-indexed freeze rung
  uint64_t *live;             // bitmap of the served clients not frozen yet
  uint32_t *orung;            // vertex-indexed open rung
  double *q;
  uint64_t *shi, *slo;
  uint32_t *cursor, *nlive, *nxt;
  double *nhat;
  uint8_t *state;
  uint32_t *heavy;            // [nF]
  uint32_t *opened;           // [nF] vertex ids opened this rung
  uint32_t *ctr;              // [G * OC_NFIELD * stripes * sstride]
};

// ladder value of rung t
__device__ inline double lad_at(const OpenArgs &A, uint32_t g, uint32_t t) {
  return A.win[(size_t)g * LAD_WIN + (t - A.ctl->base)];
}

// Served and not frozen.  One bit per vertex: on R-MAT 2^22 the entries that
// facilities cross or rescan (some 10^9 lookups) then hit the L2, where a byte
// and a word per vertex (21 MB) did not: opening loop 53 -> 42 ms there, 16.8 ->
// 14.8 on R-MAT 2^20 directed, the smaller graphs unchanged.
__device__ inline bool is_live(const OpenArgs &A, uint32_t c) { return (A.live[c >> 6] >> (c & 63)) & 1u; }

__device__ inline void ctr_add(const OpenArgs &A, uint32_t g, int field, uint32_t v) {
  if (v) atomicAdd(&A.ctr[(((size_t)g * OC_NFIELD + field) * A.stripes + (blockIdx.x % A.stripes)) * A.sstride], v);
}

// Block-aggregated counter adds of a single graph (every thread of a
// 256-thread block calls it, in uniform control flow): for fields f0, f1 and
// f2 (-1: none), the number of the block's threads with v0, v1 or v2 set, one
// atomic per block and field.
__device__ inline void block_ctr(const OpenArgs &A, int f0, bool v0, int f1, bool v1, int f2, bool v2) {
  __shared__ uint32_t s_c[3][256 / WAVE];
  const int wv = threadIdx.x / WAVE;
  const uint32_t c0 = (uint32_t)__popcll(__ballot(v0));
  const uint32_t c1 = (uint32_t)__popcll(__ballot(v1));
  const uint32_t c2 = (uint32_t)__popcll(__ballot(v2));
  if (lane_id() == 0) {
    s_c[0][wv] = c0;
    s_c[1][wv] = c1;
    s_c[2][wv] = c2;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int i = (int)threadIdx.x;
    const int f = i == 0 ? f0 : (i == 1 ? f1 : f2);
    uint32_t tot = 0;
    for (int w = 0; w < 256 / WAVE; ++w) tot += s_c[i][w];
    if (f >= 0) ctr_add(A, 0, f, tot);
  }
  __syncthreads();  // s_c may be reused
}

// Block-aggregated append (every thread of a 256-thread block calls it, in
// uniform control flow): one global atomic per block.  Used where most waves
// append, so that the waves do not queue on one counter.
__device__ inline void block_append(uint32_t *list, uint32_t *count, bool want, uint32_t x) {
  __shared__ uint32_t s_off[256 / WAVE];
  __shared__ uint32_t s_base;
  const int lane = lane_id();
  const int wv = threadIdx.x / WAVE;
  const uint64_t m = __ballot(want);
  if (lane == 0) s_off[wv] = (uint32_t)__popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int i = 0; i < 256 / WAVE; ++i) {
      const uint32_t cw = s_off[i];
      s_off[i] = tot;
      tot += cw;
    }
    s_base = tot ? atomicAdd(count, tot) : 0u;
  }
  __syncthreads();
  if (want) list[s_base + s_off[wv] + lanes_below(m)] = x;
  __syncthreads();  // s_off and s_base may be reused
}

__global__ void k_fac_init(OpenArgs A) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.nF) return;
  A.q[i] = 0.0;
  A.shi[i] = 0;
  A.slo[i] = 0;
  A.cursor[i] = 0;
  A.nlive[i] = 0;
  A.nxt[i] = 0;  // entry 0 of every sketch is the facility itself, at distance 0
  A.nhat[i] = 0.0;
  A.state[i] = 0;
}

// a wave per word of the bitmap
__global__ __launch_bounds__(256) void k_live_init(OpenArgs A) {
  const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t m = __ballot(c < A.n && A.ceff[c] && A.frz[c] == FL_RUNG_NONE);
  if (c < A.n && lane_id() == 0) A.live[c >> 6] = m;
}

// the ladder window from its first two entries (a[t] = a[t-1] (1 + eps), one
// rounding each, as the host computes it)
__global__ void k_ladder_init(OpenArgs A) {
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= A.G) return;
  double a = A.og[g].a0;
  for (uint32_t i = 0; i < LAD_WIN; ++i) {
    A.win[(size_t)g * LAD_WIN + i] = a;
    a = a * A.one_eps;
  }
}

// Between two rungs, by one block: closes the rung that was evaluated (counts
// and stopping rule of each graph), then opens the next one.  stuck_done: the
// stall check this kernel asked for has run.
// With the control on the host a rung was three round trips and some ten small
// copies and fills, whatever its size (R-MAT 2^18, unit weights, eps 0.01: 118
// us a rung; opening loop 57 ms, now 27; ER 2,000: 2.3 -> 1.2 ms; a batch of
// 64 power-law graphs 114 -> 99 ms).
constexpr uint32_t CTL_T = 256;
__global__ __launch_bounds__(CTL_T) void k_open_ctl(OpenArgs A, int stuck_done) {
  __shared__ OpenCtl s;
  __shared__ uint32_t any_stuck, any_run, any_frz, any_inf, s_f[OC_NFIELD];
  const uint32_t tid = threadIdx.x;
  if (tid == 0) {
    s = *A.ctl;
    any_stuck = any_run = any_frz = any_inf = 0;
  }
  __syncthreads();
  if (s.stop != (stuck_done ? OS_STUCK : OS_RUN)) return;
  const uint32_t t0 = s.tev + 1;
  if (A.stripes > 1) {
    // one graph: a wave per field sums its stripes, a lane each
    for (int f = (int)(tid / WAVE); f < OC_NFIELD; f += CTL_T / WAVE) {
      const uint32_t i = (uint32_t)lane_id();
      const uint64_t v = wave_sum_u64(i < A.stripes ? A.ctr[((size_t)f * A.stripes + i) * A.sstride] : 0u);
      if (i == 0) s_f[f] = (uint32_t)v;
    }
    __syncthreads();
  }
  auto field = [&](uint32_t g, int f) -> uint32_t {
    return A.stripes > 1 ? s_f[f] : A.ctr[((size_t)g * OC_NFIELD + f) * A.sstride];
  };
  for (uint32_t g = tid; g < A.G; g += CTL_T) {
    OpenG &x = A.og[g];
    if (s.pending && x.run) {
      x.nO += field(g, OC_OPENED);
      x.nU -= field(g, OC_FROZEN);
      x.nUF -= field(g, OC_NUF_DEC);
      x.finite = field(g, OC_FINITE);
      x.frz_prev = field(g, OC_FROZEN) > 0;
      x.rungs = s.tev;
      x.run = 0;
      if (!(x.nO < x.nF && x.nU > 0)) x.done = 1;
    }
    if (stuck_done) {
      // stall guard: no unopened facility sees an unfrozen client
      if (x.stuck && field(g, OC_LIVE) == 0) {
        x.gflag |= 1;
        x.nU = 0;
        x.done = 1;
      }
      x.stuck = 0;
    } else {
      // nothing in reach: the stall check
      x.stuck = !x.done && x.finite == 0 && x.nUF == 0;
      if (x.stuck) any_stuck = 1;
    }
  }
  __syncthreads();
  const bool stuck = any_stuck != 0;
  if (!stuck) {
    // the ladder window holds rungs t0 .. t0 + FF_WIN + 1 (the next rung's t0)
    const bool shift = t0 + FF_WIN + 1 >= s.base + LAD_WIN;
    for (uint32_t g = tid; g < A.G; g += CTL_T) {
      OpenG &x = A.og[g];
      double *w = A.win + (size_t)g * LAD_WIN;
      if (shift) {
        double a = w[t0 - s.base];
        for (uint32_t i = 0; i < LAD_WIN; ++i) {
          w[i] = a;
          a = a * A.one_eps;
        }
      }
      if (x.done) continue;
      const uint32_t o = shift ? 0u : t0 - s.base;
      if (!isfinite(w[o])) {
        x.rc = FL_ERANGE;
        x.done = 1;
        continue;
      }
      x.run = 1;
      any_run = 1;
      if (x.frz_prev) any_frz = 1;
      if (!isfinite(w[o + FF_WIN])) any_inf = 1;
    }
    __syncthreads();
    if (tid == 0) {
      s.stop = OS_RUN;
      if (shift) s.base = t0;
      if (!any_run) {
        s.stop = OS_DONE;
      } else {
        // skip the quiet rungs before the next event (not the first rung, which
        // uses Eq. 2, and not right after a freeze, which changes N)
        s.ff = t0 > 1 && A.nF > 0 && !any_frz && !any_inf;
        s.t0 = t0;
        s.tev = s.ff ? t0 + FF_WIN : t0;
      }
    }
  } else if (tid == 0) {
    s.stop = OS_STUCK;
    ++s.stalls;
  }
  __syncthreads();
  for (uint32_t i = tid; i < A.G * (uint32_t)OC_NFIELD * A.stripes; i += CTL_T) A.ctr[(size_t)i * A.sstride] = 0;
  if (tid == 0) {
    s.pending = s.unseeded = s.stop == OS_RUN;
    s.heavy_cnt = s.opened_cnt = 0;
    *A.ctl = s;
  }
}

// opening test and bookkeeping of a facility that opens at rung t
__device__ inline bool try_open(const OpenArgs &A, uint32_t fi, uint32_t f, double qn, uint32_t t) {
  if (qn >= (double)A.fac_cost[f]) {
    A.state[fi] = 1;
    A.orung[f] = t;
    return true;
  }
  return false;
}

// live lists up to this long are rescanned by the light kernel (a thread per
// facility); longer ones, and facilities with newly crossed entries, take
// the heavy kernel (16 lanes per facility)
constexpr uint32_t LIGHT_RESCAN = 32;

// 256 threads per block (block_append)
__global__ __launch_bounds__(256) void k_open_light(OpenArgs A) {
  if (A.ctl->stop) return;
  const uint32_t t = A.ctl->tev, t0 = A.ctl->t0;
  const uint32_t fi = blockIdx.x * blockDim.x + threadIdx.x;
  bool heavy = false, opened = false, nuf = false;
  uint32_t f = 0, g = 0;
  if (fi < A.nF && !A.state[fi]) {
    f = A.fac_list[fi];
    g = seg_of(A.gid, f);
    const OpenG &x = A.og[g];
    if (x.run) {
      const double alpha = lad_at(A, g, t);
      double q0 = A.q[fi];
      if (t > t0) {
        // the quiet rungs t0 .. t - 1
        const double nh = A.nhat[fi];
        for (uint32_t i = t0; i < t; ++i) {
          const double ea = A.eps * lad_at(A, g, i);
          q0 = q0 + ea * nh;
        }
        A.q[fi] = q0;
      }
      const uint32_t nx = A.nxt[fi];
      const uint32_t nl = A.nlive[fi];
      const bool rescan = x.frz_prev && nl > 0;
      heavy = (nx != INF32 && (double)nx <= alpha) || (rescan && nl > LIGHT_RESCAN);
      if (!heavy) {
        double nh = A.nhat[fi];
        if (rescan) {
          // a short live list: drop the clients that froze, as the heavy
          // kernel does (exact subtraction, entries after the first gap move)
          const size_t base = (size_t)f * A.cap, trow = (size_t)fi * A.cap;
          uint64_t rhi = 0, rlo = 0;
          uint32_t wpos = 0;
          for (uint32_t i = 0; i < nl; ++i) {
            const uint32_t id = A.sk_rank[base + i];
            if (!is_live(A, id)) {
              const Fix52 x = fix52_of(hip_weight(A.thr[trow + i]));
              rhi += x.hi;
              rlo += x.lo;
            } else {
              if (wpos != i) {
                A.sk_rank[base + wpos] = id;
                A.thr[trow + wpos] = A.thr[trow + i];
                A.sk_dist[base + wpos] = A.sk_dist[base + i];
              }
              ++wpos;
            }
          }
          if (wpos != nl) {
            const uint64_t shi = A.shi[fi] - rhi, slo = A.slo[fi] - rlo;
            A.shi[fi] = shi;
            A.slo[fi] = slo;
            A.nlive[fi] = wpos;
            nh = fix52_to_double(shi, slo);
            A.nhat[fi] = nh;
          }
        }
        // Eq. 3 with the current estimate (0 when nothing is live; at the
        // first rung nothing is live on this path, and an empty Eq. 2 sum is
        // 0 as well)
        const double inc = (A.eps * alpha) * nh;
        const double qn = q0 + inc;
        A.q[fi] = qn;
        opened = try_open(A, fi, f, qn, t);
        nuf = opened && is_live(A, f);
      }
    }
  }
  // late rungs open facilities in most waves: block-level appends and counts
  block_append(A.heavy, &A.ctl->heavy_cnt, heavy, fi);
  block_append(A.opened, &A.ctl->opened_cnt, opened, f);
  if (A.gid) {
    if (opened) ctr_add(A, g, OC_OPENED, 1);
    if (nuf) ctr_add(A, g, OC_NUF_DEC, 1);
  } else {
    block_ctr(A, OC_OPENED, opened, OC_NUF_DEC, nuf, -1, false);
  }
}

// The heavy kernel gives each facility a group of OPEN_G lanes, so that a
// wave follows WAVE / OPEN_G facilities' chains of dependent loads (cursor,
// entries, the clients' freeze state, sums) at once.
constexpr int OPEN_G = 16;
static_assert(OPEN_G >= 2 && OPEN_G < 32 && (OPEN_G & (OPEN_G - 1)) == 0,
              "group masks are 32-bit: a power of two below 32 lanes");

// sum over the lane's OPEN_G-lane group (the group's lanes converged)
__device__ inline uint64_t group_sum_u64(uint64_t x) {
#pragma unroll
  for (int d = OPEN_G / 2; d >= 1; d >>= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)x, d, WAVE), hi = __shfl_xor((uint32_t)(x >> 32), d, WAVE);
    x += ((uint64_t)hi << 32) | lo;
  }
  return x;
}

__global__ __launch_bounds__(256) void k_open_heavy(OpenArgs A) {
  if (A.ctl->stop) return;
  const uint32_t t = A.ctl->tev;
  const int lane = lane_id();
  const int sub = lane % OPEN_G;
  const int lead = lane - sub;  // the group's first lane
  const uint32_t below = (1u << sub) - 1u;
  // lanes of this group with cond set, as OPEN_G group-relative bits
  auto gballot = [&](bool cond) -> uint32_t {
    return (uint32_t)(__ballot(cond) >> lead) & ((1u << OPEN_G) - 1u);
  };
  const uint32_t nh = A.ctl->heavy_cnt;
  constexpr uint32_t GPW = WAVE / OPEN_G;
  const uint64_t h0 = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE * GPW + (uint64_t)(lane / OPEN_G);
  const uint64_t ng = ((uint64_t)gridDim.x * blockDim.x) / WAVE * GPW;
  for (uint64_t h = h0; h < nh; h += ng) {
    const uint32_t fi = A.heavy[h];
    const uint32_t f = A.fac_list[fi];
    const uint32_t g = seg_of(A.gid, f);
    const OpenG &x = A.og[g];
    const RankMap rm = rank_map(A.seg[g]);
    const double alpha = lad_at(A, g, t);
    const uint32_t any_freeze_prev = x.frz_prev;
    const size_t base = (size_t)f * A.cap;
    const size_t trow = (size_t)fi * A.cap;
    const uint32_t c = A.cnt[f];
    uint32_t nl = A.nlive[fi];
    uint32_t cur = A.cursor[fi];
    uint64_t lhi = 0, llo = 0;  // weight added (crossed entries)
    uint64_t rhi = 0, rlo = 0;  // weight removed (clients that froze)
    const bool rescan = any_freeze_prev && nl > 0;
    if (rescan) {
      // drop the clients that froze: subtract their weights from the exact
      // sum and close the gaps (entries before the first gap stay in place)
      uint32_t wpos = 0;
      for (uint32_t b = 0; b < nl; b += OPEN_G) {
        const uint32_t i = b + sub;
        const bool valid = i < nl;
        const uint32_t id = valid ? A.sk_rank[base + i] : 0u;
        const bool gone = valid && !is_live(A, id);
        const bool keep = valid && !gone;
        const uint32_t mk = gballot(keep);
        const uint32_t p = wpos + (uint32_t)__popc(mk & below);
        const bool move = keep && p != i;
        uint32_t T = 0, d = 0;
        if (gone || move) T = A.thr[trow + i];
        if (move) d = A.sk_dist[base + i];
        if (gone) {
          const Fix52 x = fix52_of(hip_weight(T));
          rhi += x.hi;
          rlo += x.lo;
        }
        if (move) {
          A.sk_rank[base + p] = id;
          A.thr[trow + p] = T;
          A.sk_dist[base + p] = d;
        }
        wpos += (uint32_t)__popc(mk);
      }
      nl = wpos;
    }
    // cross entries with distance <= alpha (entries are sorted by distance)
    while (cur < c) {
      const uint32_t j = cur + sub;
      const bool valid = j < c;
      uint32_t d = INF32;
      if (valid) d = A.sk_dist[base + j];
      const bool cross = valid && (double)d <= alpha;
      const uint32_t ncross = (uint32_t)__popc(gballot(cross));
      if (ncross == 0) break;
      bool keep = false;
      uint32_t id = 0, T = 0;
      if (cross) {
        id = id_of(A.sk_rank[base + j], rm);
        T = A.thr[trow + j];
        keep = is_live(A, id);
      }
      const uint32_t mk = gballot(keep);
      if (keep) {
        const uint32_t p = nl + (uint32_t)__popc(mk & below);
        A.sk_rank[base + p] = id;
        A.thr[trow + p] = T;
        A.sk_dist[base + p] = d;
        const Fix52 x = fix52_of(hip_weight(T));
        lhi += x.hi;
        llo += x.lo;
      }
      nl += (uint32_t)__popc(mk);
      cur += ncross;
      if (ncross < (uint32_t)OPEN_G) break;
    }
    lhi = group_sum_u64(lhi);
    llo = group_sum_u64(llo);
    rhi = group_sum_u64(rhi);
    rlo = group_sum_u64(rlo);
    // each word is a sum over the live entries, so removing a subset keeps it
    // exact (no word goes below zero)
    uint64_t shi = A.shi[fi] - rhi + lhi;
    uint64_t slo = A.slo[fi] - rlo + llo;
    const double nh_ = fix52_to_double(shi, slo);
    if (sub == 0) {
      double inc;
      if (t == 1) {
        // Eq. 2: sum over the live entries, in sketch order, of
        // a_j ((1+eps) alpha - beta(d_j)); beta is a[0] or a[1] here
        const double ae = A.one_eps * alpha;
        double s = 0.0;
        for (uint32_t i = 0; i < nl; ++i) {
          const double dj = (double)A.sk_dist[base + i];
          const double b = dj <= x.a0 ? x.a0 : x.a1;
          s = s + hip_weight(A.thr[trow + i]) * (ae - b);
        }
        inc = s;
      } else {
        inc = (A.eps * alpha) * nh_;
      }
      A.shi[fi] = shi;
      A.slo[fi] = slo;
      A.nlive[fi] = nl;
      A.cursor[fi] = cur;
      A.nxt[fi] = cur < c ? A.sk_dist[base + cur] : INF32;
      A.nhat[fi] = nh_;
      const double qn = A.q[fi] + inc;
      A.q[fi] = qn;
      if (try_open(A, fi, f, qn, t)) {
        const uint32_t p = atomicAdd(&A.ctl->opened_cnt, 1u);
        A.opened[p] = f;
        ctr_add(A, g, OC_OPENED, 1);
        if (is_live(A, f)) ctr_add(A, g, OC_NUF_DEC, 1);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Quiet rungs.  When no client froze in the previous rung, a rung in which no
// facility crosses its next sketch entry, none reaches its cost and no client
// comes within (1 + eps) alpha of the open set changes nothing but q:
// q += (eps alpha_t) N for every unopened facility, with N fixed.  The next
// rung with an event is found on the device, and the quiet rungs before it
// are applied by that rung's light kernel, in the same floating-point order as
// rung by rung.
// ---------------------------------------------------------------------------
// rung i of graph g's look-ahead (i < FF_WIN): the first with d <= f * a[t0 + i],
// or FF_WIN (the ladder does not decrease)
__device__ inline uint32_t ff_first(const double *a, double d, double f, bool scaled) {
  uint32_t lo = 0, n = FF_WIN;
  while (n) {
    const uint32_t h = n / 2;
    if (d <= (scaled ? f * a[lo + h] : a[lo + h])) {
      n = h;
    } else {
      lo += h + 1;
      n -= h + 1;
    }
  }
  return lo;
}

// The look-ahead: blocks below fblocks take facilities, the others clients.
// Only the earliest event counts, so a facility stops adding at the earliest
// one found so far (read again every FF_CHECK rungs): with every facility
// going to its own event the scan took 80 us on R-MAT 2^18 and 0.9 ms on 2^22
// (unit weights).
constexpr uint32_t FF_CHECK = 8;
__global__ __launch_bounds__(256) void k_ff_scan(OpenArgs A, uint32_t fblocks, const uint64_t *dlab) {
  if (A.ctl->stop || !A.ctl->ff) return;
  const uint32_t t0 = A.ctl->t0;
  uint32_t *tev = &A.ctl->tev;
  uint32_t ev = FF_WIN;
  if (blockIdx.x < fblocks) {
    const uint32_t fi = blockIdx.x * blockDim.x + threadIdx.x;
    if (fi >= A.nF || A.state[fi]) return;
    const uint32_t f = A.fac_list[fi];
    const uint32_t g = seg_of(A.gid, f);
    if (!A.og[g].run) return;
    const double *a = A.win + (size_t)g * LAD_WIN + (t0 - A.ctl->base);
    const uint32_t nx = A.nxt[fi];
    if (nx != INF32) ev = ff_first(a, (double)nx, 0.0, false);
    double q = A.q[fi];
    const double nh = A.nhat[fi], c = (double)A.fac_cost[f];
    for (uint32_t i = 0; i < ev; ++i) {
      if (i % FF_CHECK == 0 && t0 + i >= __hip_atomic_load(tev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
      const double ea = A.eps * a[i];
      q = q + ea * nh;
      if (q >= c) {
        ev = i;
        break;
      }
    }
  } else {
    const uint64_t c = (uint64_t)(blockIdx.x - fblocks) * blockDim.x + threadIdx.x;
    if (c >= A.n || !is_live(A, (uint32_t)c)) return;
    const uint64_t L = dlab[c];
    if (L == INF64) return;
    const uint32_t g = seg_of(A.gid, (uint32_t)c);
    if (!A.og[g].run) return;
    const double *a = A.win + (size_t)g * LAD_WIN + (t0 - A.ctl->base);
    ev = ff_first(a, (double)(uint32_t)(L >> 32), A.one_eps, true);
  }
  if (ev < FF_WIN && t0 + ev < __hip_atomic_load(tev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMin(tev, t0 + ev);
}

// Opened facilities become sources at distance 0 (tie = own id) and the first
// frontier of the search, unless they are already; for rungs whose searches
// take wide iterations (the one-block kernel seeds itself otherwise, up to its
// limit).  The flag is cleared by the next launch (sssp_chain).
__global__ __launch_bounds__(256) void k_seed_opened(OpenArgs A, uint64_t *lab, SsspWork wk) {
  if (!A.ctl->unseeded) return;
  const uint32_t cnt = A.ctl->opened_cnt;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += stride) {
    const uint32_t f = A.opened[i];
    lab[f] = (uint64_t)f;
    wk.front[0][i] = f;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *wk.st = SsspState{cnt, 0u, wk.st->iter, 0u, 0u, wk.st->wide};
}

__global__ __launch_bounds__(256) void k_freeze(OpenArgs A, const uint64_t *dlab, const SsspState *sst,
                                                const uint32_t *fac_idx) {
  const uint32_t stop = A.ctl->stop;
  if (stop != OS_RUN && stop != OS_SSSP) return;
  // (a block that starts after block 0 has written reads the other of the two
  // and does the same)
  if (blockIdx.x == 0 && threadIdx.x == 0) A.ctl->stop = sst->nf ? OS_SSSP : OS_RUN;
  if (sst->nf) return;  // the search has not ended
  const uint32_t t = A.ctl->tev;
  const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool froze = false, finite = false, nuf = false;
  uint32_t g = 0;
  const bool live = c < A.n && is_live(A, (uint32_t)c);
  if (live && A.og[g = seg_of(A.gid, (uint32_t)c)].run) {
    const uint64_t L = dlab[c];
    if (L != INF64) {
      const uint32_t d = (uint32_t)(L >> 32);
      if ((double)d <= A.one_eps * lad_at(A, g, t)) {
        A.frz[c] = t;
        froze = true;
        const uint32_t fi = fac_idx[c];
        nuf = fi != INF32 && !A.state[fi];
      } else {
        finite = true;
      }
    }
  }
  // a wave per word of the bitmap
  const uint64_t left = __ballot(live && !froze);
  if (__ballot(froze) && lane_id() == 0) A.live[c >> 6] = left;
  if (A.gid) {
    const bool valid = c < A.n;
    if (valid) g = seg_of(A.gid, (uint32_t)c);
    seg_add32(A.ctr, valid, g, OC_FROZEN, OC_NFIELD, A.stripes, froze ? 1u : 0u);
    seg_add32(A.ctr, valid, g, OC_FINITE, OC_NFIELD, A.stripes, finite ? 1u : 0u);
    seg_add32(A.ctr, valid, g, OC_NUF_DEC, OC_NFIELD, A.stripes, nuf ? 1u : 0u);
  } else {
    block_ctr(A, OC_FROZEN, froze, OC_FINITE, finite, OC_NUF_DEC, nuf);
  }
}

// Does some unopened facility still have an unfrozen served client anywhere
// in its sketch?  (Stall check; due only when no unfrozen client can be
// reached by an open facility and no unopened facility is itself one.)  One
// such facility answers for its graph, so a wave skips the rest.
__global__ __launch_bounds__(256) void k_stuck_scan(OpenArgs A) {
  if (A.ctl->stop != OS_STUCK) return;
  const int lane = lane_id();
  const uint64_t nw = (uint64_t)gridDim.x * (blockDim.x / WAVE);
  for (uint64_t fi = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; fi < A.nF; fi += nw) {
    if (A.state[fi]) continue;
    const uint32_t f = A.fac_list[fi];
    const uint32_t g = seg_of(A.gid, f);
    if (!A.og[g].stuck) continue;
    uint32_t *found = &A.ctr[((size_t)g * OC_NFIELD + OC_LIVE) * A.stripes * A.sstride];
    if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) continue;
    const RankMap rm = rank_map(A.seg[g]);
    const size_t base = (size_t)f * A.cap;
    const uint32_t nl = A.nlive[fi], cur = A.cursor[fi], c = A.cnt[f];
    bool live = false;
    for (uint32_t i = lane; i < nl; i += WAVE) live |= is_live(A, A.sk_rank[base + i]);
    for (uint32_t j = cur + lane; j < c; j += WAVE) {
      const uint32_t id = id_of(A.sk_rank[base + j], rm);
      live |= is_live(A, id);
    }
    if (__ballot(live) && lane == 0) atomicAdd(found, 1u);
  }
}

// graphs flagged in gflag[g] & 1: stall guard; & 2: end phase
__global__ void k_guard(uint32_t n, const uint32_t *gid, const uint8_t *gflag, const uint8_t *ceff, uint32_t *frz,
                        uint32_t *orung, const uint64_t *gam) {
  const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n || !(gflag[seg_of(gid, (uint32_t)c)] & 1) || !ceff[c] || frz[c] != FL_RUNG_NONE) return;
  const uint32_t f = (uint32_t)(gam[c] & 0xFFFFFFFFu);
  orung[f] = FL_RUNG_GUARD;
  frz[c] = FL_RUNG_GUARD;
}

__global__ void k_endphase(uint32_t n, const uint32_t *gid, const uint8_t *gflag, const uint8_t *ceff,
                           uint32_t *frz) {
  const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < n && (gflag[seg_of(gid, (uint32_t)c)] & 2) && ceff[c] && frz[c] == FL_RUNG_NONE) frz[c] = FL_RUNG_END;
}

size_t open_graph_bytes() { return LAD_WIN * sizeof(double) + sizeof(OpenG) + OC_NFIELD * 4 + 1; }

int open_phase(Ctx &c, const OpenIn &in, OpenOut &out) {
  const Graph &g = *in.g;
  const uint32_t n = g.n, nF = in.nF, G = in.G;
  OpenArgs A{};
  A.n = n;
  A.nF = nF;
  A.cap = in.ads->cap;
  // one graph: 64 stripes, 32 words (128 B) apart; a union: one plain
  // counter per graph and field (seg_add32 indexes it unstrided)
  A.stripes = G == 1 ? (uint32_t)WAVE : 1;
  A.sstride = G == 1 ? 32 : 1;
  A.gid = in.gid;
  A.seg = in.seg;
  A.fac_list = in.fac_list;
  A.fac_cost = in.fac_cost;
  A.sk_rank = in.ads->sk_rank;
  A.sk_dist = in.ads->sk_dist;
  A.thr = in.ads->thr;
  A.cnt = in.ads->cnt;
  A.ceff = in.ceff;
  A.frz = out.frz;
  A.orung = out.orung;
  A.q = out.q;
  A.shi = c.arena->get<uint64_t>(nF);
  A.slo = c.arena->get<uint64_t>(nF);
  A.cursor = c.arena->get<uint32_t>(nF);
  A.nlive = c.arena->get<uint32_t>(nF);
  A.nxt = c.arena->get<uint32_t>(nF);
  A.nhat = c.arena->get<double>(nF);
  A.state = c.arena->get<uint8_t>(nF);
  A.heavy = c.arena->get<uint32_t>(nF);
  A.opened = c.arena->get<uint32_t>(nF);
  const size_t ctr_words = (size_t)G * OC_NFIELD * A.stripes * A.sstride;
  A.ctr = c.arena->get<uint32_t>(ctr_words);
  A.live = c.arena->get<uint64_t>(ceil_div(n, WAVE));
  A.G = G;
  A.eps = in.eps;
  A.one_eps = 1.0 + in.eps;
  A.og = c.arena->get<OpenG>(G);
  A.ctl = c.arena->get<OpenCtl>(1);
  A.win = c.arena->get<double>((size_t)G * LAD_WIN);
  uint8_t *d_gflag = c.arena->get<uint8_t>(G);
  uint64_t *dlab = c.arena->get<uint64_t>(n);
  fill_u64(c, dlab, n, INF64);
  fill_u32(c, out.frz, n, FL_RUNG_NONE);
  fill_u32(c, out.orung, n, FL_RUNG_NONE);
  k_live_init<<<(uint32_t)ceil_div(n, 256), 256, 0, c.s>>>(A);
  FL_LAUNCH_CHECK();
  if (nF) {
    k_fac_init<<<(uint32_t)ceil_div(nF, 256), 256, 0, c.s>>>(A);
    FL_LAUNCH_CHECK();
  }
  SsspWork wk;
  sssp_alloc(c, wk, n, g.m);

  std::vector<OpenG> og(G);
  for (uint32_t q = 0; q < G; ++q) {
    OpenG &x = og[q];
    x = OpenG{};
    x.nF = (uint32_t)in.nF_g[q];
    x.nU = (uint32_t)in.nCeff[q];
    x.nUF = (uint32_t)in.nUF0[q];
    x.done = !(x.nF > 0 && x.nU > 0);
    x.a0 = (*in.lad)[q][0];
    x.a1 = (*in.lad)[q][1];
  }
  FL_HIP(hipMemcpyAsync(A.og, og.data(), G * sizeof(OpenG), hipMemcpyHostToDevice, c.s));
  fill_u32(c, reinterpret_cast<uint32_t *>(A.ctl), sizeof(OpenCtl) / 4, 0);
  fill_u32(c, A.ctr, ctr_words, 0);
  k_ladder_init<<<(uint32_t)ceil_div(G, 64), 64, 0, c.s>>>(A);
  FL_LAUNCH_CHECK();
  const uint32_t fblocks = (uint32_t)ceil_div(nF ? nF : 1, 256);
  const uint32_t hblocks = (uint32_t)std::min<uint64_t>(ceil_div((uint64_t)(nF ? nF : 1) * OPEN_G, 256), 4096);
  const uint32_t vblocks = (uint32_t)ceil_div(n, 256);
  const uint32_t sblocks = (uint32_t)std::min<uint64_t>(ceil_div((uint64_t)(nF ? nF : 1) * WAVE, 256), 4096);
  auto ctl = [&](int stuck_done) {
    k_open_ctl<<<1, CTL_T, 0, c.s>>>(A, stuck_done);
    FL_LAUNCH_CHECK();
  };
  auto freeze = [&]() {
    k_freeze<<<vblocks, 256, 0, c.s>>>(A, dlab, wk.st, in.fac_idx);
    FL_LAUNCH_CHECK();
  };
  auto seed = [&]() {
    k_seed_opened<<<std::min<uint32_t>(fblocks, 256), 256, 0, c.s>>>(A, dlab, wk);
    FL_LAUNCH_CHECK();
  };
  // One rung.  stall: with the launches of a stall check (without them a check
  // that falls due stops the chunk).  wide: iterations of the search launched
  // for frontiers beyond one block; a search that needs more goes on in the
  // launches of the next rung, whose other kernels exit.
  auto rung = [&](bool stall, int wide) {
    ctl(0);
    if (stall) {
      k_stuck_scan<<<sblocks, 256, 0, c.s>>>(A);
      FL_LAUNCH_CHECK();
      ctl(1);
    }
    k_ff_scan<<<fblocks + vblocks, 256, 0, c.s>>>(A, fblocks, dlab);
    FL_LAUNCH_CHECK();
    k_open_light<<<fblocks, 256, 0, c.s>>>(A);
    FL_LAUNCH_CHECK();
    k_open_heavy<<<hblocks, 256, 0, c.s>>>(A);
    FL_LAUNCH_CHECK();
    if (wide) {
      seed();
      sssp_chain(c, g, dlab, &A.ctl->unseeded, wk, wide);
    } else {
      sssp_opened(c, g, dlab, A.opened, &A.ctl->opened_cnt, &A.ctl->unseeded, wk);
    }
    freeze();
  };
  // Rungs are launched up to OPEN_CHUNK at a time, with wide iterations as long
  // as a fair share of a chunk's rungs took some, or where a search has not
  // ended, and with stall checks where the chunk before had any due.  They are
  // due in every rung until a client is in finite reach of an open facility
  // where no facility is a client, and hardly ever elsewhere.
  // A search that has not ended by the end of a chunk runs on its own, and the
  // next chunk is half as long: the launches of a chunk's other rungs advance it
  // by OPEN_WIDE iterations in thirteen launches (a grid of 1,200 x 1,200, weights
  // 1..9, 1% facilities, 7,700 wide iterations: opening loop 226 to 260 ms with
  // them, 172 to 182 without).
  constexpr uint32_t OPEN_CHUNK = 8;
  constexpr int OPEN_WIDE = 2;
  OpenCtl st{};
  SsspState sst{};
  uint32_t wide_seen = 0, stalls_seen = 0, chunk = OPEN_CHUNK;
  int wide = nF > NARROW_V ? OPEN_WIDE : 0;
  bool stall = false;
  for (const OpenG &x : og) stall |= !x.done && x.nUF == 0;
  for (;;) {
    for (uint32_t r = 0; r < chunk; ++r) rung(stall, wide);
    FL_HIP(hipMemcpyAsync(c.h_status, A.ctl, sizeof(OpenCtl), hipMemcpyDeviceToHost, c.s));
    FL_HIP(hipMemcpyAsync(c.h_status + 64, wk.st, sizeof(SsspState), hipMemcpyDeviceToHost, c.s));
    c.sync();
    std::memcpy(&st, c.h_status, sizeof(OpenCtl));
    std::memcpy(&sst, c.h_status + 64, sizeof(SsspState));
    if (st.stop == OS_DONE) break;
    stall = st.stalls != stalls_seen;
    stalls_seen = st.stalls;
    wide = st.stop == OS_SSSP || sst.wide - wide_seen >= OPEN_CHUNK / 4 ? OPEN_WIDE : 0;
    wide_seen = sst.wide;
    if (st.stop == OS_SSSP) {
      seed();
      sssp_finish(c, g, dlab, &A.ctl->unseeded, wk);
      freeze();
      chunk = std::max(chunk / 2, 1u);
    } else {
      chunk = std::min(2 * chunk, OPEN_CHUNK);
    }
  }
  FL_HIP(hipMemcpyAsync(og.data(), A.og, G * sizeof(OpenG), hipMemcpyDeviceToHost, c.s));
  c.sync();
  out.rungs.resize(G);
  out.rc.resize(G);
  out.nO.resize(G);
  std::vector<uint8_t> gflag(G, 0);
  bool any_flag = false;
  for (uint32_t q = 0; q < G; ++q) {
    out.rungs[q] = og[q].rungs;
    out.rc[q] = og[q].rc;
    out.nO[q] = og[q].nO;
    gflag[q] = (uint8_t)og[q].gflag;
    // end phase
    if (og[q].nO == og[q].nF && og[q].nU > 0 && og[q].rc == FL_OK) gflag[q] |= 2;
    any_flag |= gflag[q] != 0;
    // the host's ladder reaches every rung evaluated (the radii of the selection)
    std::vector<double> &lad = (*in.lad)[q];
    while (lad.size() <= og[q].rungs) lad.push_back(lad.back() * A.one_eps);
  }
  if (any_flag) {
    FL_HIP(hipMemcpyAsync(d_gflag, gflag.data(), G, hipMemcpyHostToDevice, c.s));
    k_guard<<<vblocks, 256, 0, c.s>>>(n, in.gid, d_gflag, in.ceff, out.frz, out.orung, in.gam_lab);
    FL_LAUNCH_CHECK();
    k_endphase<<<vblocks, 256, 0, c.s>>>(n, in.gid, d_gflag, in.ceff, out.frz);
    FL_LAUNCH_CHECK();
    c.sync();  // gflag is read by the copy above
  }
  // q by vertex for the caller's diagnostics is scattered later
  return FL_OK;
}

}  // namespace fl
