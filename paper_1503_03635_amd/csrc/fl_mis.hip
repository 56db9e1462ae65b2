// fl_mis.hip -- facility selection: a maximal independent set of the
// conflict graph H-bar, per rung (Sec. 4.3, Alg. 6), without building H.
//
// A client c and a facility f are joined in H when both carry the same rung
// t (c froze at t, f opened at t) and d(c, f) <= (1 + eps) a[t]; facilities
// conflict when they share a client.  Priorities pi(f) are a seeded
// bijection, and each round of the fixed-priority algorithm is three bounded
// sweeps over the graph:
//   1. every client takes the smallest priority of the active facilities
//      within the radius (pi_min);
//   2. every active facility takes the smallest pi_min of the clients within
//      the radius; it joins S when that is its own priority (or when it has
//      no client);
//   3. active facilities within the radius of a client covered by a joined
//      facility (the client's pi_min is that facility's priority) retire.
// Rounds repeat until no facility is active; the result is the greedy MIS in
// priority order.  The radius is measured from client to facility, d(c, f):
// sweep 1 starts at facilities and pushes over the in-arcs, sweeps 2 and 3
// start at clients and push over the out-arcs (the same arcs when the graph
// is undirected).  In a union of several graphs, each graph walks through its
// own non-empty rungs: step i runs the i-th one of every graph at once (the
// graphs share no vertex, so their sweeps do not interact), each with its own
// radius and priorities.  A sweep computes, for every vertex x, the minimum label
// over sources within distance R of x.  It runs in distance order (round j
// settles labels at distance exactly j) with one pending-label array per
// distance slot modulo max_w + 1, so a label is forwarded only when it
// lowers a vertex's current minimum.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "fl_common.h"
#include "fl_frontier.h"
#include "fl_mis.h"

namespace fl {

// The phase's work on one step (the i-th non-empty rung of every graph) in
// order; rounds repeat from MP_ROUND until no facility is active.
enum MisPhase : uint32_t {
  MP_STEP = 0,  // the step's facilities (act) and clients (ct), the clients' bitmap
  MP_ROUND,     // priorities of the active facilities, their bitmap
  MP_SWEEP1,    // from act: smallest priority at the clients
  MP_TAKE,      // the clients' minima become their labels (src)
  MP_SWEEP2,    // from src: smallest of them at the facilities
  MP_JOIN,      // facilities that join, the rest (act2), covered clients (cov)
  MP_SWEEP3,    // from cov: facilities that retire
  MP_COLLECT,   // the facilities still active (act)
  MP_END        // the clients' bitmap is cleared
};
// Why the one-block kernel stopped.
enum MisGo : uint32_t {
  MG_DONE = 1,  // every step is done
  MG_WIDE,      // the sweep's next distance is too large for one block
  MG_LIST,      // the phase's lists are
  MG_ERROR      // more rounds than facilities
};
struct MisState {
  uint32_t go, phase;
  uint32_t j;       // the sweep's distance to settle next
  uint32_t start;   // it starts from the sources (distance 0)
  uint32_t cnt;     // vertices to settle there
  uint32_t step, round, stamp;             // round within the step; rounds in all
  uint32_t na, ncl, ns2, nr, ncov, nnew;   // lengths of act, ct, src, act2, cov, the new act
  uint32_t ntouched, nheavy;
};
struct SweepArgs {
  uint32_t n, NS;
  const uint32_t *gid;  // graph of each vertex (nullptr: one graph)
  const uint32_t *Rg;   // [G] radius of each graph in the current step
  const uint64_t *row_ptr;
  const uint32_t *col;
  const uint32_t *w;
  const uint32_t *cend;  // [n * C] arcs of a row in its first classes (nullptr: rows not in class order)
  uint32_t C;
  uint32_t *ml;       // [n] current minimum label (INF32 = none)
  uint32_t *pend;     // [NS * n] pending label per slot
  uint32_t *tl;       // [NS * n] vertices with a pending label per slot
  uint32_t *tl_cnt;   // [NS * CNT_PAD] list length of each slot, one per line
  uint32_t *touched;  // [n] vertices whose ml was set
  uint32_t *touched_cnt;
  uint64_t *heavy;    // pieces of the long rows queued in the current distance
  uint32_t *heavy_cnt;
  const uint32_t *tbits;  // bitmap of the vertices whose result is read
};

// One step's ranges, and one range: a graph's facilities and clients of the
// step's rung.
struct MisStep {
  uint32_t r0, r1;       // its ranges
  uint32_t nf, nc;       // facilities and clients in all
  uint32_t nf_max;       // most facilities of a range
};
struct MisRange {
  uint64_t f0, c0;       // in flist and clist
  uint32_t nf, nc, fdst, cdst;  // lengths, places in act and ct
  uint32_t q, R;         // graph and radius
};

// Device view of the whole phase.  Direction 0: from facilities over the
// in-arcs, to the clients of cbits; 1: from clients over the out-arcs, to the
// facilities of fbits.
struct MisArgs {
  SweepArgs S;  // row_ptr, col, w and tbits are set per direction
  const uint64_t *rp[2];
  const uint32_t *col[2], *w[2], *cend[2];
  uint32_t *bits[2];  // cbits, fbits
  MisState *st;
  const MisStep *steps;
  const MisRange *ranges;
  uint32_t nsteps, G, luby;
  const uint32_t *flist, *clist;  // facilities and clients by (graph, rung)
  uint32_t *act, *act2, *ct, *src, *cov;
  uint32_t *lab;     // [n] source labels
  uint32_t *Rg;      // [G] radius of each graph in the current step
  uint32_t *gstamp;  // [G] last round with an active facility
  uint32_t *rcount;  // [G] rounds
  const SegInfo *seg;
  uint8_t *open;
};
__device__ inline SweepArgs sweep_args(const MisArgs &A, uint32_t phase) {
  // both sides of each choice are loaded: an index that the compiler cannot
  // see would put the arrays in scratch memory
  const bool in = phase == MP_SWEEP1;
  SweepArgs S = A.S;
  S.row_ptr = in ? A.rp[0] : A.rp[1];
  S.col = in ? A.col[0] : A.col[1];
  S.w = in ? A.w[0] : A.w[1];
  S.cend = in ? A.cend[0] : A.cend[1];
  S.tbits = in ? A.bits[0] : A.bits[1];
  return S;
}

// ---- rows in weight-class order ---------------------------------------------
// A label settled at distance j uses the arcs of weight R - j at most, and of
// the arcs a sweep reads in a row's own order few are that light: 387 of the
// 4,650 million of the first sweeps on R-MAT 2^21 with weights 1..100, 53 of
// the 2,302 million of the second.  So a weighted graph's rows are copied once
// per call with their arcs ordered by weight class, and a push reads the
// classes up to that of R - j.  The copy reads and writes the arcs once each
// (2 ms there); MIS 137 -> 96 ms there, 23.7 -> 17.8 on a Chung-Lu graph of
// 50,000 vertices (weights 1..50), 62 -> 45 for a burst of twelve such graphs;
// with weights 1..4 on a grid or a few thousand vertices it saves or costs
// less than 0.1 ms, so every weighted graph takes it.
// Class of a weight: two per octave, so that the classes up to a weight's hold
// at most weights 1.5 times as large.  At most 16 for weights up to 255.
constexpr uint32_t MAX_CLASS = 16;
__host__ __device__ inline uint32_t weight_class(uint32_t w) {
  uint32_t e = 0;
  for (uint32_t s = 4; s >= 1; s >>= 1)  // floor(log2(w)) of a weight in 1..255
    if (w >> (e + s)) e += s;
  return e ? 2 * e + ((w >> (e - 1)) & 1u) : 0u;
}
static_assert(MAX_W < 256, "weight_class covers 8 bits");
// arcs of x, from its row's start, that a label with b >= 1 left of its radius can use
__device__ inline uint64_t sweep_degree(const SweepArgs &S, uint32_t x, uint64_t a0, uint32_t b) {
  if (S.cend) return S.cend[(size_t)x * S.C + weight_class(b < S.NS ? b : S.NS - 1)];
  return S.row_ptr[x + 1] - a0;
}

// Class order of every row (col, w -> ocol, ow; cend[x * C + c] arcs of x in
// classes 0..c): a wave per row, counted and placed by class ballots.  Rows
// above CLASS_ROW go to k_class_hubs, a block each: one wave would walk a hub
// of R-MAT 2^21 (some 10^5 arcs) alone while the chip idles.
constexpr uint32_t CLASS_ROW = 4096;
struct ClassArgs {
  uint32_t n, C;
  const uint64_t *row_ptr;
  const uint32_t *col, *w;
  uint32_t *ocol, *ow, *cend;
  uint32_t *hubs, *nhubs;
};
// this lane's count of class `lane` among 64 arcs of classes c (MAX_CLASS and
// above: no arc), and the lanes of its own arc's class
__device__ inline uint32_t class_count(uint32_t C, uint32_t c, uint64_t *same) {
  uint32_t cnt = 0;
  uint64_t sm = 0;
  for (uint32_t q = 0; q < C; ++q) {
    const uint64_t m = __ballot(c == q);
    if (c == q) sm = m;
    if ((uint32_t)lane_id() == q) cnt = (uint32_t)__popcll(m);
  }
  *same = sm;
  return cnt;
}
__device__ inline void class_place(const ClassArgs &A, uint64_t a0, uint64_t b0, uint64_t b1, uint32_t base) {
  const uint32_t lane = (uint32_t)lane_id();
  for (uint64_t b = b0; b < b1; b += WAVE) {
    const uint64_t a = b + lane;
    const bool have = a < b1;
    const uint32_t y = have ? A.col[a] : 0u, wt = have ? A.w[a] : 0u;
    const uint32_t c = have ? weight_class(wt) : MAX_CLASS;
    uint64_t same;
    const uint32_t cnt = class_count(A.C, c, &same);
    const uint32_t at = __shfl(base, (int)(have ? c : 0u), WAVE) + lanes_below(same);
    if (have) {
      A.ocol[a0 + at] = y;
      A.ow[a0 + at] = wt;
    }
    base += cnt;
  }
}
__device__ inline uint32_t class_counts(const ClassArgs &A, uint64_t b0, uint64_t b1) {
  uint32_t cnt = 0;
  uint64_t same;
  for (uint64_t b = b0; b < b1; b += WAVE) {
    const uint64_t a = b + (uint32_t)lane_id();
    cnt += class_count(A.C, a < b1 ? weight_class(A.w[a]) : MAX_CLASS, &same);
  }
  return cnt;
}
__global__ __launch_bounds__(256) void k_class_rows(ClassArgs A) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint64_t nw = (uint64_t)gridDim.x * (blockDim.x / WAVE);
  for (uint64_t x = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; x < A.n; x += nw) {
    const uint64_t a0 = A.row_ptr[x], a1 = A.row_ptr[x + 1];
    if (a1 - a0 > CLASS_ROW) {
      if (lane == 0) A.hubs[atomicAdd(A.nhubs, 1u)] = (uint32_t)x;
      continue;
    }
    const uint32_t cnt = class_counts(A, a0, a1);
    const uint32_t incl = wave_scan_incl(cnt);
    if (lane < A.C) A.cend[x * A.C + lane] = incl;
    class_place(A, a0, a0, a1, incl - cnt);
  }
}
constexpr uint32_t CLASS_HUB_T = 1024, CLASS_HUB_WAVES = CLASS_HUB_T / WAVE;
__global__ __launch_bounds__(CLASS_HUB_T) void k_class_hubs(ClassArgs A) {
  __shared__ uint32_t s_cnt[MAX_CLASS][CLASS_HUB_WAVES];
  const uint32_t lane = (uint32_t)lane_id(), wv = threadIdx.x / WAVE, nh = *A.nhubs;
  for (uint32_t h = blockIdx.x; h < nh; h += gridDim.x) {
    const uint32_t x = A.hubs[h];
    const uint64_t a0 = A.row_ptr[x], a1 = A.row_ptr[x + 1];
    const uint64_t part = (a1 - a0 + CLASS_HUB_T - 1) / CLASS_HUB_T * WAVE;  // arcs of a wave
    const uint64_t b0 = a0 + wv * part < a1 ? a0 + wv * part : a1, b1 = b0 + part < a1 ? b0 + part : a1;
    const uint32_t cnt = class_counts(A, b0, b1);
    if (lane < MAX_CLASS) s_cnt[lane][wv] = lane < A.C ? cnt : 0u;
    __syncthreads();
    if (wv == 0) {  // starts of every (class, wave), class-major: four per lane
      uint32_t *q = &s_cnt[0][0] + 4 * lane;
      const uint32_t v0 = q[0], v1 = q[1], v2 = q[2], v3 = q[3];
      const uint32_t end = wave_scan_incl(v0 + v1 + v2 + v3);
      const uint32_t at = end - (v0 + v1 + v2 + v3);
      q[0] = at;
      q[1] = at + v0;
      q[2] = at + v0 + v1;
      q[3] = at + v0 + v1 + v2;
      if (lane % 4 == 3 && lane / 4 < A.C) A.cend[(size_t)x * A.C + lane / 4] = end;
    }
    __syncthreads();
    class_place(A, a0, b0, b1, lane < MAX_CLASS ? s_cnt[lane][wv] : 0u);
    __syncthreads();
  }
}
static_assert(MAX_CLASS * CLASS_HUB_WAVES == 4 * WAVE && CLASS_HUB_WAVES == 16, "four starts per lane, a class in four lanes");

// the sources of a sweep
__device__ inline const uint32_t *sweep_sources(const MisArgs &A, const MisState &st, uint32_t phase, uint32_t *n) {
  *n = phase == MP_SWEEP1 ? st.na : phase == MP_SWEEP2 ? st.ns2 : st.ncov;
  return phase == MP_SWEEP1 ? A.act : phase == MP_SWEEP2 ? A.src : A.cov;
}

// Queue appends (vertex y to the list of slot s), staged per wave in LDS
// (2 WAVE entries) and written WAVE at a time with one atomic per distinct
// slot among them: with per-step atomics the waves of a large frontier queue
// on the slot's one count.
struct SlotQ {
  uint32_t *ys, *ss;  // this wave's LDS staging: vertices and their slots
  uint32_t *cs;       // this wave's count per slot (MAX_W + 1 words, zero between calls)
  uint32_t cnt;       // staged entries (wave-uniform, < WAVE between calls)
};

// Append y to the list of slot s on the lanes with have set: the lanes of a
// slot are counted in LDS, and one lane per distinct slot reserves room for
// all of them.  The reservations are one instruction, so a write waits for one
// atomic's return; a loop over the distinct slots (about 47 among 64 entries
// at weights 1..100) waited for one after another, and that wait was most of
// a wide step: with it and wave_share gone from 35 to 16 us a launch on a
// Chung-Lu graph of 50,000 vertices, half of the launches empty (MIS 43 -> 33 ms).
// With unit weights every entry of a step goes to the same slot.
__device__ inline void slotq_write(const SweepArgs &S, const SlotQ &q, bool have, uint32_t y, uint32_t s) {
  if (S.NS == 2) {
    const uint64_t m = __ballot(have);
    const int lead = __ffsll((long long)m) - 1;  // m != 0
    const uint32_t s0 = __shfl(s, lead, WAVE);
    wave_push(S.tl + (size_t)s0 * S.n, &S.tl_cnt[s0 * CNT_PAD], have, y);
    return;
  }
  uint32_t r = 0, v = 0;
  if (have) r = atomicAdd(&q.cs[s], 1u);
  wave_lds_sync();
  if (have) v = q.cs[s];
  wave_lds_sync();
  if (have && r == 0) q.cs[s] = atomicAdd(&S.tl_cnt[s * CNT_PAD], v);
  wave_lds_sync();
  if (have) v = q.cs[s];
  wave_lds_sync();
  if (have && r == 0) q.cs[s] = 0;
  wave_lds_sync();
  if (have) S.tl[(size_t)s * S.n + v + r] = y;
}

// every lane calls, converged
__device__ inline void slotq_push(const SweepArgs &S, SlotQ &q, bool add, uint32_t y, uint32_t s) {
  const int lane = lane_id();
  const uint64_t m = __ballot(add);
  if (!m) return;
  if (add) {
    q.ys[q.cnt + lanes_below(m)] = y;
    q.ss[q.cnt + lanes_below(m)] = s;
  }
  q.cnt += (uint32_t)__popcll(m);
  if (q.cnt < (uint32_t)WAVE) return;
  wave_lds_sync();
  slotq_write(S, q, true, q.ys[lane], q.ss[lane]);
  q.cnt -= WAVE;
  const bool more = (uint32_t)lane < q.cnt;
  const uint32_t ry = more ? q.ys[WAVE + lane] : 0u, rs = more ? q.ss[WAVE + lane] : 0u;
  wave_lds_sync();
  if (more) {
    q.ys[lane] = ry;
    q.ss[lane] = rs;
  }
  wave_lds_sync();
}

// the staged remainder (every lane calls, converged, before the wave exits)
__device__ inline void slotq_flush(const SweepArgs &S, SlotQ &q) {
  if (!q.cnt) return;
  const int lane = lane_id();
  wave_lds_sync();
  const bool have = (uint32_t)lane < q.cnt;
  slotq_write(S, q, have, have ? q.ys[lane] : 0u, have ? q.ss[lane] : 0u);
  q.cnt = 0;
}

// LDS staging for the 256 / WAVE waves of a block
#define SLOTQ_DECL(q)                                                                                   \
  __shared__ uint32_t q##_ys[256 / WAVE][2 * WAVE];                                                     \
  __shared__ uint32_t q##_ss[256 / WAVE][2 * WAVE];                                                     \
  __shared__ uint32_t q##_cs[256 / WAVE][MAX_W + 1];                                                    \
  SlotQ q{q##_ys[threadIdx.x / WAVE], q##_ss[threadIdx.x / WAVE], q##_cs[threadIdx.x / WAVE], 0u};      \
  for (uint32_t i_ = (uint32_t)lane_id(); i_ < S.NS; i_ += WAVE) q.cs[i_] = 0;                          \
  wave_lds_sync()

// Two arc steps of a push (every lane calls, converged; a lane with v0 or v1
// false has no arc in that group): per arc, lower the pending label of the
// head at distance j + w when that is within R, and queue the head once per
// slot.  Both groups' columns, weights and head minima are loaded before
// either group is tested, so a wave keeps two chains of dependent reads in
// flight instead of one (on the large weighted workload MIS went 1.17 ->
// 1.11 s from the long rows, then 1.106 -> 1.095 s from the short rows).
// A head whose settled minimum is already at most the label is skipped: it
// reached that minimum at a smaller distance, so the push could never settle
// (a concurrent settle only lowers ml, which keeps the test safe).  A label
// landing at distance exactly R goes no further, so there it is kept only at
// the sweep's targets, the vertices whose minimum is read afterwards.
__device__ inline void sweep_arcs2(const SweepArgs &S, SlotQ &q, uint32_t j, bool v0, uint64_t i0, uint32_t lab0,
                                   uint32_t R0, bool v1, uint64_t i1, uint32_t lab1, uint32_t R1) {
  const uint32_t y0 = v0 ? S.col[i0] : 0u, y1 = v1 ? S.col[i1] : 0u;
  const uint32_t w0 = v0 ? (S.w ? S.w[i0] : 1u) : 0u, w1 = v1 ? (S.w ? S.w[i1] : 1u) : 0u;
  const uint64_t d0 = (uint64_t)j + w0, d1 = (uint64_t)j + w1;
  const bool k0 = v0 && (d0 < R0 || (d0 == R0 && ((S.tbits[y0 >> 5] >> (y0 & 31)) & 1u)));
  const bool k1 = v1 && (d1 < R1 || (d1 == R1 && ((S.tbits[y1 >> 5] >> (y1 & 31)) & 1u)));
  const uint32_t m0 = k0 ? __hip_atomic_load(&S.ml[y0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
  const uint32_t m1 = k1 ? __hip_atomic_load(&S.ml[y1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
  bool add0 = false, add1 = false;
  uint32_t s0 = 0, s1 = 0;
  if (k0 && lab0 < m0) {
    s0 = (j + w0) % S.NS;
    uint32_t *p = &S.pend[(size_t)s0 * S.n + y0];
    if (lab0 < __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) add0 = atomicMin(p, lab0) == INF32;
  }
  if (k1 && lab1 < m1) {
    s1 = (j + w1) % S.NS;
    uint32_t *p = &S.pend[(size_t)s1 * S.n + y1];
    if (lab1 < __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) add1 = atomicMin(p, lab1) == INF32;
  }
  slotq_push(S, q, add0, y0, s0);
  slotq_push(S, q, add1, y1, s1);
}

// The short rows of the lanes flattened over the wave, two steps of 64 arcs
// per call of f(v0, arc0, owner0, v1, arc1, owner1) (every lane calls,
// converged): arc c*64 + lane of the concatenated rows is found by a binary
// search over the running degree sum, as in flat_arcs.
template <class F>
__device__ inline void flat_arcs2(bool light, uint64_t a0, uint64_t deg, F &&f) {
  const int lane = lane_id();
  const uint32_t d = light ? (uint32_t)deg : 0u;
  const uint32_t incl = wave_scan_incl(d);
  const uint32_t total = __shfl(incl, WAVE - 1, WAVE);
  const uint32_t excl = incl - d;
  auto locate = [&](uint32_t idx, bool &valid, uint64_t &arc, int &own) {
    uint32_t pos = 0;  // first lane whose inclusive sum exceeds idx
#pragma unroll
    for (uint32_t s = 32; s >= 1; s >>= 1) {
      const uint32_t val = __shfl(incl, (int)(pos + s - 1), WAVE);
      if (val <= idx) pos += s;
    }
    valid = idx < total;
    own = valid ? (int)pos : 0;
    arc = shfl_u64(a0, own) + (idx - __shfl(excl, own, WAVE));
  };
  for (uint32_t c0 = 0; c0 < total; c0 += 2 * WAVE) {
    bool v0, v1;
    uint64_t x0, x1;
    int o0, o1;
    locate(c0 + (uint32_t)lane, v0, x0, o0);
    locate(c0 + WAVE + (uint32_t)lane, v1, x1, o1);
    f(v0, x0, o0, v1, x1, o1);
  }
}

// Rows of a sweep flattened over the wave: at most this many arcs (half the
// other frontier kernels' FLAT_MAX).  Longer rows go to k_sweep_heavy, whose
// waves keep more reads in flight than a flattened step: MIS 0.898 -> 0.835 s
// on the large weighted workload against 256, timed on one box, identical
// results.
constexpr uint32_t SWEEP_FLAT_MAX = 128;

// Push the labels of the lanes' vertices (want) from distance j: short rows
// flattened over the wave, long rows queued for k_sweep_heavy.
__device__ inline void sweep_push_lanes(const SweepArgs &S, SlotQ &q, bool want, uint32_t x, uint32_t lab,
                                        uint32_t j) {
  uint64_t a0 = 0, deg = 0;
  uint32_t R = 0;
  if (want) {
    R = S.Rg[seg_of(S.gid, x)];
    want = j < R;  // arcs weigh at least 1: a label settled at distance R goes no further
  }
  if (want) {
    a0 = S.row_ptr[x];
    deg = sweep_degree(S, x, a0, R - j);
  }
  const bool heavy = want && deg > SWEEP_FLAT_MAX;
  push_pieces(S.heavy, S.heavy_cnt, heavy, x, deg);
  flat_arcs2(want && !heavy, a0, deg, [&](bool v0, uint64_t x0, int o0, bool v1, uint64_t x1, int o1) {
    sweep_arcs2(S, q, j, v0, x0, __shfl(lab, o0, WAVE), __shfl(R, o0, WAVE), v1, x1, __shfl(lab, o1, WAVE),
                __shfl(R, o1, WAVE));
  });
}

// vertices whose ml was set for the first time -> touched (one atomic per wave)
__device__ inline void touch(const SweepArgs &S, bool first, uint32_t x) {
  wave_push(S.touched, S.touched_cnt, first, x);
}

// Wide step, first launch: settle the labels pending at distance st->j, or the
// sources' (a lane per vertex).  Nothing to do unless a wide step is due.
__global__ __launch_bounds__(256) void k_sweep_wide(MisArgs A) {
  if (A.st->go != MG_WIDE) return;
  const uint32_t phase = A.st->phase, j = A.st->j;
  const SweepArgs S = sweep_args(A, phase);
  SLOTQ_DECL(q);
  const uint32_t slot = j % S.NS;
  const bool start = A.st->start != 0;
  uint32_t cnt = 0;
  const uint32_t *list = sweep_sources(A, *A.st, phase, &cnt);
  if (!start) {
    list = S.tl + (size_t)slot * S.n;
    cnt = S.tl_cnt[slot * CNT_PAD];
  }
  const uint32_t vw = wave_share(cnt), lane = (uint32_t)lane_id();
  const uint64_t stride = (uint64_t)gridDim.x * (blockDim.x / WAVE) * vw;
  for (uint64_t b = ((uint64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE) * vw; b < cnt; b += stride) {
    const uint64_t i = b + lane;
    bool want = false, first = false;
    uint32_t y = 0, v = INF32;
    if (lane < vw && i < cnt) {
      y = list[i];
      uint32_t cur = INF32;
      if (start) {
        v = A.lab[y];
      } else {
        v = S.pend[(size_t)slot * S.n + y];
        cur = S.ml[y];
        S.pend[(size_t)slot * S.n + y] = INF32;
      }
      if (v < cur) {
        S.ml[y] = v;
        want = true;
        first = cur == INF32;
      }
    }
    touch(S, first, y);
    sweep_push_lanes(S, q, want, y, v, j);
  }
  slotq_flush(S, q);
}

// Wide step, second launch: the pieces of long rows queued at distance st->j,
// one wave per piece; the label is the vertex's own (settled at this
// distance, unchanged until the next).
__global__ __launch_bounds__(256) void k_sweep_heavy(MisArgs A) {
  if (A.st->go != MG_WIDE) return;
  const uint32_t cnt = A.st->nheavy, j = A.st->j;
  if (blockIdx.x * (blockDim.x / WAVE) >= cnt) return;
  const SweepArgs S = sweep_args(A, A.st->phase);
  SLOTQ_DECL(q);
  const int lane = lane_id();
  const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) / WAVE;
  for (uint64_t i = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; i < cnt; i += nw) {
    uint64_t a0, a1;
    const uint32_t x = piece_arcs(S.heavy[i], S.row_ptr, &a0, &a1);
    const uint32_t lab = S.ml[x];
    const uint32_t R = S.Rg[seg_of(S.gid, x)];
    if (S.cend) {  // the piece ends where the classes do
      const uint64_t r0 = S.row_ptr[x], end = r0 + sweep_degree(S, x, r0, R - j);
      a1 = a1 < end ? a1 : end;
    }
    for (uint64_t b = a0; b < a1; b += 2 * WAVE) {
      const uint64_t i0 = b + lane, i1 = b + WAVE + lane;
      sweep_arcs2(S, q, j, i0 < a1, i0, lab, R, i1 < a1, i1, lab, R);
    }
  }
  slotq_flush(S, q);
}

__global__ void k_sweep_reset(SweepArgs S) {
  const uint32_t cnt = *S.touched_cnt;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt;
       i += (uint64_t)gridDim.x * blockDim.x)
    S.ml[S.touched[i]] = INF32;
}

// ---- small per-round kernels -------------------------------------------------
// Priority of facility f: the fixed one (luby_round == 0), or for Luby's
// variant the one drawn for round r of the rung, a bijection keyed by
// SplitMix64(seed ^ (3 + 256 r)).
__device__ inline PermKey priority_key(const SegInfo &sg, uint32_t luby_round) {
  return luby_round ? perm_key(sg.seed, 3ull + 256ull * luby_round) : sg.pk;
}
__device__ inline uint32_t priority_of(uint32_t f, const uint32_t *gid, const SegInfo *seg, uint32_t luby_round) {
  const SegInfo &sg = seg[seg_of(gid, f)];
  return perm_fwd(f - sg.base, priority_key(sg, luby_round));
}
__global__ void k_set_key_labels(const uint32_t *list, uint32_t cnt, uint32_t *lab, const uint32_t *gid,
                                 const SegInfo *seg, uint32_t luby_round) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) lab[list[i]] = priority_of(list[i], gid, seg, luby_round);
}
// clients of the rung: their pi_min (ml[c]) becomes their label; sources for
// sweep 2 are those with a value
__global__ void k_take_pmin(const uint32_t *cl, uint32_t ncl, const uint32_t *ml, uint32_t *lab,
                            uint32_t *src, uint32_t *nsrc) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool want = false;
  uint32_t c = 0;
  if (i < ncl) {
    c = cl[i];
    const uint32_t v = ml[c];
    if (v != INF32) {
      lab[c] = v;
      want = true;
    }
  }
  const uint64_t m = __ballot(want);
  if (m) {
    const int lead = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane_id() == lead) base = atomicAdd(nsrc, (uint32_t)__popcll(m));
    base = __shfl(base, lead, WAVE);
    if (want) src[base + lanes_below(m)] = c;
  }
}
// Facility f joins iff it has no client (its minimum m is INF32) or m == pi(f).
__device__ inline bool joins(uint32_t m, uint32_t f, const uint32_t *gid, const SegInfo *seg, uint32_t luby_round) {
  return m == INF32 || m >= priority_of(f, gid, seg, luby_round);
}
// A client with label pi_min is covered iff the facility with that priority
// joined: a facility joins when its priority is the smallest pi_min around it,
// so it is pi_min at every client it has.  (An active facility is open only if
// it joined this round.)
__device__ inline bool covered(uint32_t c, const uint32_t *gid, const SegInfo *seg, uint32_t luby_round,
                               const uint8_t *open, const uint32_t *lab) {
  const SegInfo &sg = seg[seg_of(gid, c)];
  const uint32_t f = perm_inv(lab[c], priority_key(sg, luby_round)) + sg.base;
  return __hip_atomic_load(&open[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
__global__ void k_join(const uint32_t *act, uint32_t na, const uint32_t *ml, const uint32_t *gid,
                       const SegInfo *seg, uint32_t luby_round, uint8_t *open, uint32_t *rest, uint32_t *nr) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool r = false;
  uint32_t f = 0;
  if (i < na) {
    f = act[i];
    r = !joins(ml[f], f, gid, seg, luby_round);
    if (!r) open[f] = 1;
  }
  wave_push(rest, nr, r, f);
}
// the covered clients of src; their labels become 0, for sweep 3
__global__ void k_covered(const uint32_t *src, uint32_t cnt, const uint32_t *gid, const SegInfo *seg,
                          uint32_t luby_round, const uint8_t *open, uint32_t *lab, uint32_t *cov, uint32_t *ncov) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool hit = false;
  uint32_t x = 0;
  if (i < cnt) {
    x = src[i];
    hit = covered(x, gid, seg, luby_round, open, lab);
    if (hit) lab[x] = 0;
  }
  wave_push(cov, ncov, hit, x);
}
// facilities of the list not reached by a label (ml != 0) -> list
__global__ void k_collect_alive(const uint32_t *list, uint32_t cnt, const uint32_t *ml, uint32_t *out,
                                uint32_t *nout) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t x = i < cnt ? list[i] : 0u;
  wave_push(out, nout, i < cnt && ml[x] != 0, x);
}

// ---- the phase in one block --------------------------------------------------
// Lists of up to LIST_MAX entries, and up to TOUCH_MAX minima to clear, are
// handled by the block; 1,024 threads take some 1-2 us per 1,024 entries, a
// separate launch with the host's round trip 30 us or more.  A step's ranges
// (one per graph of a union) are flattened, their starts in LDS: up to
// RANGE_MAX of them.  Walked one after another, 2,000 ranges were 2,000
// dependent reads a step (batches of ER graphs of 40 vertices, MIS of a worker:
// 2,000 graphs 12.2 -> 5.4 ms, 667 4.2 -> 2.35, 100 1.45 -> 1.2, 10 unchanged).
constexpr uint32_t LIST_MAX = 16384, TOUCH_MAX = 65536, RANGE_MAX = NARROW_V;
enum MisEntry : int { ME_START = 0, ME_CLOSE, ME_LISTED };

// Runs the phase (every step, round and sweep) until a sweep's distance or a
// list is too large for one block, which then stops with the reason in
// st->go; the host launches the wide form of that piece and this kernel again:
// ME_CLOSE after a wide step (a no-op if none was due), ME_LISTED after the
// wide form of the phase's lists.
//
// Narrow steps of a sweep (see fl_frontier.h): the distances with pending
// labels in increasing order, empty ones skipped.  The slot counts live in LDS
// meanwhile, so appends take LDS atomics.  Pending labels, minima and bitmaps
// are read and changed at the device's L2 (agent scope); lists and source
// labels are written and read by this block only, a barrier apart.  While the
// block runs, every wide counter is zero.
//
// Bound by latency: a step is the chain list -> row, label and minimum ->
// column -> minimum -> atomic minimum -> list, some 5 us.  Against two
// launches per distance, empty ones included, 8 distances per host check, and
// a fourth sweep per round (MIS of R-MAT 2^18, unit weights, eps 0.01: 120 ms;
// of a Chung-Lu graph of 50,000 vertices, weights 1..50: 81 ms; of R-MAT 2^21,
// weights 1..100: 204 ms): one block per sweep 64, 33 and 144 ms; one block
// for the whole phase 14, 24 and 137.
__global__ __launch_bounds__(NARROW_T) void k_mis_narrow(MisArgs A, int entry) {
  __shared__ uint64_t s_a0[NARROW_V];
  __shared__ uint32_t s_excl[NARROW_V], s_lab[NARROW_V], s_R[NARROW_V], s_cnt[MAX_W + 1], s_tmp[NARROW_WAVES];
  __shared__ uint32_t s_next;
  __shared__ MisState s;
  const uint32_t tid = threadIdx.x, NS = A.S.NS;
  if (entry == ME_CLOSE && A.st->go != MG_WIDE) return;  // no wide step was due
  if (tid == 0) {
    s = *A.st;
    s_next = INF32;
  }
  __syncthreads();
  uint32_t phase = s.phase, go = 0;
  bool closing = entry == ME_CLOSE, listed = entry == ME_LISTED;
  if (tid < NS) s_cnt[tid] = closing && tid != s.j % NS ? A.S.tl_cnt[tid * CNT_PAD] : 0u;
  __syncthreads();
  // f(i, valid) for every entry of a list, by all threads, whole waves at a time
  auto for_list = [&](uint32_t cnt, auto &&f) {
    for (uint32_t b = 0; b < cnt; b += NARROW_T) f(b + tid, b + tid < cnt);
  };
  auto clear_minima = [&]() { for_list(s.ntouched, [&](uint32_t i, bool v) { if (v) A.S.ml[A.S.touched[i]] = INF32; }); };
  auto minimum = [&](uint32_t x) -> uint32_t {
    return __hip_atomic_load(&A.S.ml[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto set_bit = [&](uint32_t *bits, uint32_t x) { atomicOr(&bits[x >> 5], 1u << (x & 31)); };
  auto clear_bit = [&](uint32_t *bits, uint32_t x) { atomicAnd(&bits[x >> 5], ~(1u << (x & 31))); };
  // one phase per turn; every condition is the same in all threads, and the
  // state is changed between two barriers
  for (;;) {
    __syncthreads();
    const uint32_t luby_round = A.luby ? s.round : 0u;
    if (phase == MP_STEP) {
      if (s.step == A.nsteps) {
        go = MG_DONE;
        break;
      }
      const MisStep st = A.steps[s.step];
      if (!listed) {
        for (uint32_t r = st.r0 + tid; r < st.r1; r += NARROW_T) A.Rg[A.ranges[r].q] = A.ranges[r].R;
        const uint32_t nr = st.r1 - st.r0;
        if (st.nf > LIST_MAX || st.nc > LIST_MAX || nr > RANGE_MAX) {
          go = MG_LIST;
          break;
        }
        // f(i, where entry i of all ranges' is) for every entry of the
        // facilities (or clients); places past the last range hold the total
        const uint32_t half = narrow_half(nr);
        auto for_ranges = [&](bool fac, uint32_t total, auto &&f) {
          for (uint32_t p = tid; p < NARROW_V; p += NARROW_T) {
            const MisRange *x = A.ranges + st.r0 + p;
            s_excl[p] = p < nr ? (fac ? x->fdst : x->cdst) : total;
            if (p < nr) s_a0[p] = fac ? x->f0 : x->c0;
          }
          __syncthreads();
          for (uint32_t i = tid; i < total; i += NARROW_T) {
            const uint32_t p = narrow_owner(s_excl, i, half);
            f(i, s_a0[p] + (i - s_excl[p]));
          }
          __syncthreads();
        };
        for_ranges(true, st.nf, [&](uint32_t i, uint64_t at) { A.act[i] = A.flist[at]; });
        for_ranges(false, st.nc, [&](uint32_t i, uint64_t at) {
          const uint32_t c = A.clist[at];
          A.ct[i] = c;
          set_bit(A.bits[0], c);
        });
      }
      listed = false;
      if (tid == 0) {
        s.na = st.nf;
        s.ncl = st.nc;
        s.round = 0;
      }
      phase = MP_ROUND;
    } else if (phase == MP_ROUND) {
      if (s.na == 0) {
        phase = MP_END;
        continue;
      }
      if (!listed) {
        // the active facility of smallest priority of each graph joins every round
        const bool over = s.round > A.steps[s.step].nf_max;
        __syncthreads();
        if (tid == 0) {
          ++s.round;
          ++s.stamp;
        }
        __syncthreads();
        if (over || s.na > LIST_MAX) {
          go = over ? MG_ERROR : MG_LIST;
          break;
        }
        for_list(s.na, [&](uint32_t i, bool v) {
          if (!v) return;
          const uint32_t f = A.act[i];
          A.lab[f] = priority_of(f, A.S.gid, A.seg, A.luby ? s.round : 0u);
          set_bit(A.bits[1], f);
          if (A.G > 1) A.gstamp[A.S.gid[f]] = s.stamp;
        });
        __syncthreads();
      }
      listed = false;
      for (uint32_t g = tid; g < A.G; g += NARROW_T)
        if (A.G == 1 || A.gstamp[g] == s.stamp) A.rcount[g] += 1;
      if (tid == 0) {
        s.j = 0;
        s.start = 1;
      }
      phase = MP_SWEEP1;
    } else if (phase == MP_SWEEP1 || phase == MP_SWEEP2 || phase == MP_SWEEP3) {
      const SweepArgs S = sweep_args(A, phase);
      uint32_t nsrc = 0;
      const uint32_t *src = sweep_sources(A, s, phase, &nsrc);
      uint32_t j = s.j, cnt = 0;
      bool start = s.start && !closing, done = false;
      closing = false;
      __syncthreads();
      if (start && tid == 0) s.ntouched = 0;
      for (;;) {
        if (start) {
          cnt = nsrc;
        } else {
          // the next distance with a pending label (slots j + 1 .. j + NS - 1)
          if (tid + 1 < NS && s_cnt[(j + 1 + tid) % NS]) atomicMin(&s_next, tid);
          __syncthreads();
          const uint32_t d = s_next;
          __syncthreads();
          if (d == INF32) {
            done = true;
            break;
          }
          j += 1 + d;
          cnt = s_cnt[j % NS];
          if (tid == 0) s_next = INF32;
        }
        if (cnt > NARROW_V) break;
        const uint32_t slot = j % NS;
        uint32_t x[2] = {0, 0}, lv[2] = {INF32, INF32}, cur[2] = {INF32, INF32}, R[2] = {0, 0}, deg[2] = {0, 0}, ex[2];
        uint64_t a0[2] = {0, 0};
        bool set[2] = {false, false};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t p = tid + h * NARROW_T;
          if (p < cnt) {
            x[h] = start ? src[p] : S.tl[(size_t)slot * S.n + p];
            if (start) {
              lv[h] = A.lab[x[h]];
            } else {
              lv[h] =
                  __hip_atomic_load(&S.pend[(size_t)slot * S.n + x[h]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              cur[h] = minimum(x[h]);
            }
            R[h] = S.Rg[seg_of(S.gid, x[h])];
            a0[h] = S.row_ptr[x[h]];
            const uint64_t d = j < R[h] ? sweep_degree(S, x[h], a0[h], R[h] - j) : 0u;
            set[h] = lv[h] < cur[h];
            // arcs weigh at least 1: a label settled at distance R goes no further
            if (set[h]) deg[h] = d > NARROW_ARCS ? NARROW_ARCS + 1 : (uint32_t)d;
          }
        }
        uint32_t t0, t1 = 0;
        ex[0] = narrow_scan_excl(deg[0], s_tmp, &t0);
        ex[1] = t0;
        if (cnt > NARROW_T) ex[1] = t0 + narrow_scan_excl(deg[1], s_tmp, &t1);
        const uint32_t total = t0 + t1;
        if (total > NARROW_ARCS) break;  // a wide step takes this distance (nothing is settled yet)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t p = tid + h * NARROW_T;
          if (!start && p < cnt) S.pend[(size_t)slot * S.n + x[h]] = INF32;
          if (set[h]) S.ml[x[h]] = lv[h];
          wave_push(S.touched, &s.ntouched, set[h] && cur[h] == INF32, x[h]);
          s_excl[p] = p < cnt ? ex[h] : total;
          s_a0[p] = a0[h];
          s_lab[p] = lv[h];
          s_R[p] = R[h];
        }
        if (tid == 0 && !start) s_cnt[slot] = 0;
        __syncthreads();
        const uint32_t half = narrow_half(cnt);
        for (uint32_t b = 0; b < total; b += NARROW_T) {
          const uint32_t idx = b + tid;
          bool add = false;
          uint32_t y = 0, sl = 0;
          if (idx < total) {
            const uint32_t p = narrow_owner(s_excl, idx, half);
            const uint64_t a = s_a0[p] + (idx - s_excl[p]);
            const uint32_t l = s_lab[p], Rp = s_R[p];
            y = S.col[a];
            const uint32_t w = S.w ? S.w[a] : 1u;
            const uint64_t d = (uint64_t)j + w;
            // the conditions of sweep_arcs2
            bool keep = d < Rp;
            if (d == Rp)
              keep = (__hip_atomic_load(&S.tbits[y >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (y & 31)) & 1u;
            if (keep && l < minimum(y)) {
              sl = (j + w) % NS;
              add = atomicMin(&S.pend[(size_t)sl * S.n + y], l) == INF32;
            }
          }
          if (NS == 2) {
            wave_push(S.tl + (size_t)((j + 1) & 1) * S.n, &s_cnt[(j + 1) & 1], add, y);  // one slot: one atomic per wave
          } else if (add) {
            S.tl[(size_t)sl * S.n + atomicAdd(&s_cnt[sl], 1u)] = y;
          }
        }
        __syncthreads();
        start = false;
      }
      __syncthreads();
      if (tid == 0) {
        s.j = j;
        s.start = start ? 1u : 0u;
        s.cnt = cnt;
      }
      if (!done) {
        go = MG_WIDE;
        break;
      }
      phase += 1;
    } else if (phase == MP_TAKE) {
      if (!listed) {
        if (tid == 0) s.ns2 = 0;
        __syncthreads();
        if (s.ncl > LIST_MAX || s.ntouched > TOUCH_MAX) {
          go = MG_LIST;
          break;
        }
        for_list(s.ncl, [&](uint32_t i, bool v) {
          const uint32_t c = v ? A.ct[i] : 0u;
          const uint32_t m = v ? minimum(c) : INF32;
          if (m != INF32) A.lab[c] = m;
          wave_push(A.src, &s.ns2, m != INF32, c);
        });
        __syncthreads();
        clear_minima();
      }
      listed = false;
      if (tid == 0) {
        s.j = 0;
        s.start = 1;
      }
      phase = MP_SWEEP2;
    } else if (phase == MP_JOIN) {
      if (!listed) {
        if (tid == 0) s.nr = s.ncov = 0;
        __syncthreads();
        if (s.na > LIST_MAX || s.ns2 > LIST_MAX || s.ntouched > TOUCH_MAX) {
          go = MG_LIST;
          break;
        }
        for_list(s.na, [&](uint32_t i, bool v) {
          const uint32_t f = v ? A.act[i] : 0u;
          const bool rest = v && !joins(minimum(f), f, A.S.gid, A.seg, luby_round);
          if (v && !rest) A.open[f] = 1;
          wave_push(A.act2, &s.nr, rest, f);
        });
        __syncthreads();
        clear_minima();
        for_list(s.ns2, [&](uint32_t i, bool v) {
          const uint32_t c = v ? A.src[i] : 0u;
          const bool hit = v && covered(c, A.S.gid, A.seg, luby_round, A.open, A.lab);
          if (hit) A.lab[c] = 0;
          wave_push(A.cov, &s.ncov, hit, c);
        });
        __syncthreads();
      }
      listed = false;
      phase = s.nr ? MP_SWEEP3 : MP_COLLECT;
      __syncthreads();
      if (tid == 0) {
        s.j = 0;
        s.start = 1;
        s.ntouched = 0;
      }
    } else if (phase == MP_COLLECT) {
      if (!listed) {
        if (tid == 0) s.nnew = 0;
        __syncthreads();
        if (s.na > LIST_MAX || s.ntouched > TOUCH_MAX) {
          go = MG_LIST;
          break;
        }
        for_list(s.na, [&](uint32_t i, bool v) { if (v) clear_bit(A.bits[1], A.act[i]); });
        __syncthreads();
        for_list(s.nr, [&](uint32_t i, bool v) {
          const uint32_t f = v ? A.act2[i] : 0u;
          wave_push(A.act, &s.nnew, v && minimum(f) != 0, f);
        });
        __syncthreads();
        clear_minima();
      }
      listed = false;
      __syncthreads();
      if (tid == 0) s.na = s.nnew;
      phase = MP_ROUND;
    } else {  // MP_END
      if (!listed) {
        if (s.ncl > LIST_MAX) {
          go = MG_LIST;
          break;
        }
        for_list(s.ncl, [&](uint32_t i, bool v) { if (v) clear_bit(A.bits[0], A.ct[i]); });
      }
      listed = false;
      __syncthreads();
      if (tid == 0) ++s.step;
      phase = MP_STEP;
    }
  }
  __syncthreads();
  if (tid < NS) A.S.tl_cnt[tid * CNT_PAD] = s_cnt[tid];
  if (tid == 0) {
    s.go = go;
    s.phase = phase;
    s.nheavy = 0;
    *A.st = s;
  }
}

// per-(graph, rung) lists: counting sort by key koff[g] + t - 1 (t in 1..T[g])
__device__ inline bool rung_key(uint32_t v, const uint32_t *rung, const uint32_t *gid, const uint32_t *koff,
                                const uint32_t *Tg, uint32_t *key) {
  const uint32_t t = rung[v];
  const uint32_t g = seg_of(gid, v);
  if (t < 1 || t > Tg[g]) return false;
  *key = koff[g] + t - 1;
  return true;
}
// With few keys (K <= RK_LDS) a block counts in LDS first and adds one
// global atomic per key it saw: the per-rung counters are otherwise hit by
// every vertex of the rung.
constexpr uint32_t RK_LDS = 4096;
constexpr uint32_t RK_ITEMS = 16;  // vertices per thread in the LDS path
__global__ __launch_bounds__(256) void k_rung_count(uint32_t n, const uint32_t *rung, const uint32_t *gid,
                                                    const uint32_t *koff, const uint32_t *Tg, uint32_t K,
                                                    uint32_t *cnt) {
  __shared__ uint32_t lc[RK_LDS];
  uint32_t key;
  if (K > RK_LDS) {
    const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n && rung_key((uint32_t)v, rung, gid, koff, Tg, &key)) atomicAdd(&cnt[key], 1u);
    return;
  }
  for (uint32_t i = threadIdx.x; i < K; i += blockDim.x) lc[i] = 0;
  __syncthreads();
  const uint64_t v0 = (uint64_t)blockIdx.x * blockDim.x * RK_ITEMS;
  for (uint32_t it = 0; it < RK_ITEMS; ++it) {
    const uint64_t v = v0 + (uint64_t)it * blockDim.x + threadIdx.x;
    if (v < n && rung_key((uint32_t)v, rung, gid, koff, Tg, &key)) atomicAdd(&lc[key], 1u);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < K; i += blockDim.x)
    if (lc[i]) atomicAdd(&cnt[i], lc[i]);
}
__global__ __launch_bounds__(256) void k_rung_scatter(uint32_t n, const uint32_t *rung, const uint32_t *gid,
                                                      const uint32_t *koff, const uint32_t *Tg, uint32_t K,
                                                      const uint64_t *off, uint32_t *cur, uint32_t *out) {
  __shared__ uint32_t lc[RK_LDS];
  uint32_t key;
  if (K > RK_LDS) {
    const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n && rung_key((uint32_t)v, rung, gid, koff, Tg, &key))
      out[off[key] + atomicAdd(&cur[key], 1u)] = (uint32_t)v;
    return;
  }
  // local positions, then one reservation per key, then the writes
  for (uint32_t i = threadIdx.x; i < K; i += blockDim.x) lc[i] = 0;
  __syncthreads();
  const uint64_t v0 = (uint64_t)blockIdx.x * blockDim.x * RK_ITEMS;
  uint32_t lpos[RK_ITEMS], keys[RK_ITEMS];
  for (uint32_t it = 0; it < RK_ITEMS; ++it) {
    const uint64_t v = v0 + (uint64_t)it * blockDim.x + threadIdx.x;
    keys[it] = INF32;
    if (v < n && rung_key((uint32_t)v, rung, gid, koff, Tg, &key)) {
      keys[it] = key;
      lpos[it] = atomicAdd(&lc[key], 1u);
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < K; i += blockDim.x)
    if (lc[i]) lc[i] = atomicAdd(&cur[i], lc[i]);
  __syncthreads();
  for (uint32_t it = 0; it < RK_ITEMS; ++it) {
    const uint64_t v = v0 + (uint64_t)it * blockDim.x + threadIdx.x;
    if (keys[it] != INF32) out[off[keys[it]] + lc[keys[it]] + lpos[it]] = (uint32_t)v;
  }
}
// a step's facilities and clients; blockIdx.x picks the range, the blocks
// along y split it
__global__ void k_gather_step(MisArgs A, uint32_t r0) {
  const MisRange x = A.ranges[r0 + blockIdx.x];
  const uint32_t i0 = blockIdx.y * blockDim.x + threadIdx.x, stride = gridDim.y * blockDim.x;
  for (uint64_t i = i0; i < x.nf; i += stride) A.act[x.fdst + i] = A.flist[x.f0 + i];
  for (uint64_t i = i0; i < x.nc; i += stride) A.ct[x.cdst + i] = A.clist[x.c0 + i];
}
// graphs whose facility of list[i] is active this round
__global__ void k_mark_graphs(const uint32_t *list, uint32_t cnt, const uint32_t *gid, uint32_t *gstamp,
                              uint32_t stamp) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) gstamp[gid[list[i]]] = stamp;
}
__global__ void k_guard_open(uint32_t n, const uint32_t *orung, uint8_t *open) {
  const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) open[v] = orung[v] == FL_RUNG_GUARD ? 1 : 0;
}
// bitmap membership of the vertices of a list (set or clear)
__global__ void k_mark_bits(const uint32_t *list, uint32_t cnt, uint32_t *bits, int set) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  const uint32_t x = list[i];
  if (set) atomicOr(&bits[x >> 5], 1u << (x & 31));
  else atomicAnd(&bits[x >> 5], ~(1u << (x & 31)));
}
static void mark_bits(Ctx &c, const uint32_t *list, uint32_t cnt, uint32_t *bits, int set) {
  if (!cnt) return;
  k_mark_bits<<<(uint32_t)ceil_div(cnt, 256), 256, 0, c.s>>>(list, cnt, bits, set);
  FL_LAUNCH_CHECK();
}
// facilities alone in their graph's rung join at once: at[i] are their places
__global__ void k_open_singles(const uint32_t *flist, const uint32_t *at, uint32_t cnt, uint8_t *open) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) open[flist[at[i]]] = 1;
}

static void by_rung(Ctx &c, uint32_t n, const uint32_t *rung, const uint32_t *gid, const uint32_t *koff,
                    const uint32_t *Tg, uint32_t K, uint32_t *list, std::vector<uint64_t> &hoff) {
  uint32_t *cnt = c.arena->get<uint32_t>((size_t)K + 1);
  uint32_t *cur = c.arena->get<uint32_t>((size_t)K + 1);
  uint64_t *off = c.arena->get<uint64_t>((size_t)K + 2);
  fill_u32(c, cnt, K + 1, 0);
  fill_u32(c, cur, K + 1, 0);
  const uint32_t vb = (uint32_t)(K > RK_LDS ? ceil_div(n, 256) : ceil_div(n, 256 * RK_ITEMS));
  k_rung_count<<<vb, 256, 0, c.s>>>(n, rung, gid, koff, Tg, K, cnt);
  FL_LAUNCH_CHECK();
  scan_u32_to_u64(c, cnt, off, K);
  k_rung_scatter<<<vb, 256, 0, c.s>>>(n, rung, gid, koff, Tg, K, off, cur, list);
  FL_LAUNCH_CHECK();
  hoff.resize((size_t)K + 1);
  FL_HIP(hipMemcpyAsync(hoff.data(), off, hoff.size() * 8, hipMemcpyDeviceToHost, c.s));
  c.sync();
}

// blocks of a long-row sweep launch: twice the other frontier kernels'
// HEAVY_BLOCKS, 32 waves per CU on 256 CUs.  A hub piece keeps two groups of
// reads in flight per wave, and the extra waves add more: MIS 1.080 -> 0.954 s
// on the large weighted workload, timed on one box, identical results (four
// times gave the same)
constexpr uint32_t SWEEP_HEAVY_BLOCKS = 2 * HEAVY_BLOCKS;

// Copies of a weighted graph's rows in class order, for both directions, if
// what the call reserved has room for them: a call that only just fits its
// workspace runs the sweeps on the rows as they are.  The reservation does not
// count the copies; the sketch rounds before need more than the sweeps do, and
// what they leave holds them: always on undirected graphs of 4 to 32 arcs per
// vertex; on directed ones, whose two copies are larger, below a million
// vertices or from weights of about 10 on (32 arcs per vertex, every vertex a
// facility).  Room that an earlier, larger call left in the cached arena does
// not count: the same call takes the same sweeps every time.  Small weights
// lose nothing by it: 1..4 on a directed graph of 60,000 rows of 640 arcs, MIS
// 2.05 ms without the copies, 2.35 with them.
static void class_rows(Ctx &c, const Graph &g, MisArgs &A) {
  const uint32_t n = g.n, C = weight_class(g.max_w) + 1;
  const bool one = g.in_ptr == g.row_ptr && g.in_col == g.col && g.in_w == g.w;
  const uint32_t dirs = one ? 1 : 2;
  const size_t need = dirs * ((size_t)g.m * 8 + (size_t)n * C * 4) + (size_t)n * 4 + 4096;
  if (c.arena->used() + need > std::min(c.budget, c.arena->capacity())) return;
  A.S.C = C;
  uint32_t *hubs = c.arena->get<uint32_t>(n);
  uint32_t *nhubs = c.arena->get<uint32_t>(2);
  fill_u32(c, nhubs, 2, 0);
  for (uint32_t d = 0; d < dirs; ++d) {
    ClassArgs K{n, C, A.rp[d], A.col[d], A.w[d], c.arena->get<uint32_t>(g.m), c.arena->get<uint32_t>(g.m),
                c.arena->get<uint32_t>((size_t)n * C), hubs, nhubs + d};
    k_class_rows<<<(uint32_t)std::min<uint64_t>(ceil_div(n, 256 / WAVE), 8192), 256, 0, c.s>>>(K);
    FL_LAUNCH_CHECK();
    k_class_hubs<<<(uint32_t)std::min<uint64_t>(g.m / CLASS_ROW + 1, 512), CLASS_HUB_T, 0, c.s>>>(K);
    FL_LAUNCH_CHECK();
    A.col[d] = K.ocol;
    A.w[d] = K.ow;
    A.cend[d] = K.cend;
  }
  if (one) {
    A.col[1] = A.col[0];
    A.w[1] = A.w[0];
    A.cend[1] = A.cend[0];
  }
}

int mis_phase(Ctx &c, const MisIn &in, uint8_t *open, std::vector<uint32_t> &rounds_out) {
  const Graph &g = *in.g;
  const uint32_t n = g.n, G = in.G;
  const uint32_t NS = (g.w ? g.max_w : 1u) + 1;
  k_guard_open<<<(uint32_t)ceil_div(n, 256), 256, 0, c.s>>>(n, in.orung, open);
  FL_LAUNCH_CHECK();
  rounds_out.assign(G, 0);
  // keys (graph, rung) -> koff[g] + t - 1
  std::vector<uint32_t> hkoff(G), hT(G);
  uint64_t K64 = 0;
  for (uint32_t q = 0; q < G; ++q) {
    hkoff[q] = (uint32_t)K64;
    hT[q] = in.rungs[q];
    K64 += in.rungs[q];
  }
  if (K64 == 0) return FL_OK;
  if (K64 >= 0xFFFFFFF0ull) return FL_ENOMEM;
  const uint32_t K = (uint32_t)K64;
  uint32_t *koff = c.arena->get<uint32_t>(G);
  uint32_t *Tg = c.arena->get<uint32_t>(G);
  FL_HIP(hipMemcpyAsync(koff, hkoff.data(), G * 4, hipMemcpyHostToDevice, c.s));
  FL_HIP(hipMemcpyAsync(Tg, hT.data(), G * 4, hipMemcpyHostToDevice, c.s));
  uint32_t *flist = c.arena->get<uint32_t>(n);
  uint32_t *clist = c.arena->get<uint32_t>(n);
  std::vector<uint64_t> foff, coff;
  by_rung(c, n, in.orung, in.gid, koff, Tg, K, flist, foff);
  by_rung(c, n, in.frz, in.gid, koff, Tg, K, clist, coff);

  MisArgs A{};
  A.S.n = n;
  A.S.NS = NS;
  A.S.gid = in.gid;
  A.Rg = c.arena->get<uint32_t>(G);
  A.S.Rg = A.Rg;
  A.S.ml = c.arena->get<uint32_t>(n);
  A.S.pend = c.arena->get<uint32_t>((size_t)NS * n);
  A.S.tl = c.arena->get<uint32_t>((size_t)NS * n);
  A.S.tl_cnt = c.arena->get<uint32_t>((size_t)NS * CNT_PAD);
  A.S.touched = c.arena->get<uint32_t>(n);
  A.S.heavy = c.arena->get<uint64_t>(piece_capacity(n, g.m));
  A.st = c.arena->get<MisState>(1);
  A.S.touched_cnt = &A.st->ntouched;
  A.S.heavy_cnt = &A.st->nheavy;
  A.rp[0] = g.in_ptr;
  A.col[0] = g.in_col;
  A.w[0] = g.in_w;
  A.rp[1] = g.row_ptr;
  A.col[1] = g.col;
  A.w[1] = g.w;
  const size_t nwords = ((size_t)n + 31) / 32;
  A.bits[0] = c.arena->get<uint32_t>(nwords);
  A.bits[1] = c.arena->get<uint32_t>(nwords);
  A.G = G;
  A.luby = in.luby ? 1u : 0u;
  A.flist = flist;
  A.clist = clist;
  A.act = c.arena->get<uint32_t>(n);
  A.act2 = c.arena->get<uint32_t>(n);
  A.ct = c.arena->get<uint32_t>(n);
  A.src = c.arena->get<uint32_t>(n);
  A.cov = c.arena->get<uint32_t>(n);
  A.lab = c.arena->get<uint32_t>(n);
  A.gstamp = c.arena->get<uint32_t>(G);
  A.rcount = c.arena->get<uint32_t>(G);
  A.seg = in.seg;
  A.open = open;

  // Each graph's non-empty rungs, in order; step i takes the i-th of every
  // graph.  A facility alone in its rung conflicts with nothing: it joins.
  const double one_eps = 1.0 + in.eps;
  std::vector<std::vector<uint32_t>> lists(G);
  size_t nlists = 0;
  for (uint32_t q = 0; q < G; ++q) {
    for (uint32_t t = 1; t <= hT[q]; ++t) {
      const uint32_t key = hkoff[q] + t - 1;
      if (foff[key + 1] > foff[key]) lists[q].push_back(t);
    }
    nlists = std::max(nlists, lists[q].size());
  }
  std::vector<MisStep> steps;
  std::vector<MisRange> ranges;
  std::vector<uint32_t> singles;
  for (size_t i = 0; i < nlists; ++i) {
    MisStep st{(uint32_t)ranges.size(), 0, 0, 0, 0};
    for (uint32_t q = 0; q < G; ++q) {
      if (i >= lists[q].size()) continue;
      const uint32_t t = lists[q][i];
      const uint32_t key = hkoff[q] + t - 1;
      const uint32_t nf = (uint32_t)(foff[key + 1] - foff[key]);
      if (nf == 1) {
        singles.push_back((uint32_t)foff[key]);
        rounds_out[q] += 1;
        continue;
      }
      const uint32_t nc = (uint32_t)(coff[key + 1] - coff[key]);
      const double rho = one_eps * (*in.lad)[q][t];
      // integer radius: d <= rho  <=>  d <= floor(rho)
      const uint32_t R = rho >= 4294967295.0 ? 0xFFFFFFFEu : (uint32_t)std::floor(rho);
      ranges.push_back(MisRange{foff[key], coff[key], nf, nc, st.nf, st.nc, q, R});
      st.nf += nf;
      st.nc += nc;
      st.nf_max = std::max(st.nf_max, nf);
    }
    st.r1 = (uint32_t)ranges.size();
    if (st.r1 > st.r0) steps.push_back(st);
  }
  if (!singles.empty()) {
    uint32_t *d = c.arena->get<uint32_t>(singles.size());
    FL_HIP(hipMemcpyAsync(d, singles.data(), singles.size() * 4, hipMemcpyHostToDevice, c.s));
    const uint32_t ns1 = (uint32_t)singles.size();
    k_open_singles<<<(uint32_t)ceil_div(ns1, 256), 256, 0, c.s>>>(flist, d, ns1, open);
    FL_LAUNCH_CHECK();
  }
  if (steps.empty()) {
    c.sync();  // singles is read by the copy above
    return FL_OK;
  }
  MisStep *d_steps = c.arena->get<MisStep>(steps.size());
  MisRange *d_ranges = c.arena->get<MisRange>(ranges.size());
  FL_HIP(hipMemcpyAsync(d_steps, steps.data(), steps.size() * sizeof(MisStep), hipMemcpyHostToDevice, c.s));
  FL_HIP(hipMemcpyAsync(d_ranges, ranges.data(), ranges.size() * sizeof(MisRange), hipMemcpyHostToDevice, c.s));
  A.steps = d_steps;
  A.ranges = d_ranges;
  A.nsteps = (uint32_t)steps.size();
  if (g.w && g.m) class_rows(c, g, A);
  fill_u32(c, A.S.ml, n, INF32);
  fill_u32(c, A.S.pend, (size_t)NS * n, INF32);
  fill_u32(c, A.S.tl_cnt, (size_t)NS * CNT_PAD, 0);
  fill_u32(c, reinterpret_cast<uint32_t *>(A.st), sizeof(MisState) / 4, 0);
  fill_u32(c, A.bits[0], nwords, 0);
  fill_u32(c, A.bits[1], nwords, 0);
  fill_u32(c, A.gstamp, G, 0);
  fill_u32(c, A.rcount, G, 0);

  MisState st{};
  auto narrow = [&](MisEntry e) {
    k_mis_narrow<<<1, NARROW_T, 0, c.s>>>(A, e);
    FL_LAUNCH_CHECK();
  };
  // A wide step is two launches and the one-block kernel, which closes it and
  // goes on.  One that finds no wide step due exits at once.  A frontier can
  // grow from a handful of vertices to most of the graph, so every launch
  // gets a grid for any frontier (the kernel strides over the count).
  auto wide = [&](uint64_t want) {
    k_sweep_wide<<<wide_blocks(n, want), 256, 0, c.s>>>(A);
    FL_LAUNCH_CHECK();
    k_sweep_heavy<<<SWEEP_HEAVY_BLOCKS, 256, 0, c.s>>>(A);
    FL_LAUNCH_CHECK();
    narrow(ME_CLOSE);
  };
  auto check = [&]() {
    c.fetch(A.st, sizeof(MisState));
    std::memcpy(&st, c.h_status, sizeof(MisState));
  };
  auto blocks = [](uint32_t cnt) { return (uint32_t)ceil_div(cnt ? cnt : 1, 256); };
  auto clear_minima = [&]() {
    k_sweep_reset<<<1024, 256, 0, c.s>>>(A.S);
    FL_LAUNCH_CHECK();
  };
  // the wide form of a phase's lists
  auto lists_of = [&](uint32_t phase) {
    const uint32_t luby_round = in.luby ? st.round : 0u;
    if (phase == MP_STEP) {
      const MisStep &ms = steps[st.step];
      uint32_t longest = 1;
      for (uint32_t r = ms.r0; r < ms.r1; ++r) longest = std::max({longest, ranges[r].nf, ranges[r].nc});
      const uint32_t cy = (uint32_t)std::min<uint64_t>(ceil_div(longest, 1024), 1024);
      k_gather_step<<<dim3(ms.r1 - ms.r0, cy), 256, 0, c.s>>>(A, ms.r0);
      FL_LAUNCH_CHECK();
      mark_bits(c, A.ct, ms.nc, A.bits[0], 1);
    } else if (phase == MP_ROUND) {
      k_set_key_labels<<<blocks(st.na), 256, 0, c.s>>>(A.act, st.na, A.lab, in.gid, in.seg, luby_round);
      FL_LAUNCH_CHECK();
      mark_bits(c, A.act, st.na, A.bits[1], 1);
      if (G > 1) {
        k_mark_graphs<<<blocks(st.na), 256, 0, c.s>>>(A.act, st.na, in.gid, A.gstamp, st.stamp);
        FL_LAUNCH_CHECK();
      }
    } else if (phase == MP_TAKE) {
      k_take_pmin<<<blocks(st.ncl), 256, 0, c.s>>>(A.ct, st.ncl, A.S.ml, A.lab, A.src, &A.st->ns2);
      FL_LAUNCH_CHECK();
      clear_minima();
    } else if (phase == MP_JOIN) {
      k_join<<<blocks(st.na), 256, 0, c.s>>>(A.act, st.na, A.S.ml, in.gid, in.seg, luby_round, open, A.act2,
                                             &A.st->nr);
      FL_LAUNCH_CHECK();
      clear_minima();
      k_covered<<<blocks(st.ns2), 256, 0, c.s>>>(A.src, st.ns2, in.gid, in.seg, luby_round, open, A.lab, A.cov,
                                                 &A.st->ncov);
      FL_LAUNCH_CHECK();
    } else if (phase == MP_COLLECT) {
      mark_bits(c, A.act, st.na, A.bits[1], 0);  // before act is rewritten
      k_collect_alive<<<blocks(st.nr), 256, 0, c.s>>>(A.act2, st.nr, A.S.ml, A.act, &A.st->nnew);
      FL_LAUNCH_CHECK();
      clear_minima();
    } else {
      mark_bits(c, A.ct, st.ncl, A.bits[0], 0);
    }
  };
  narrow(ME_START);
  check();
  while (st.go != MG_DONE) {
    if (st.go == MG_WIDE) {
      wide((uint64_t)st.cnt * 2);
      wide(0);
    } else if (st.go == MG_LIST) {
      // large lists are mostly a large sweep's sources
      lists_of(st.phase);
      narrow(ME_LISTED);
      wide(0);
    } else {
      return FL_EHIP;  // more rounds than facilities: a bug
    }
    check();
  }
  std::vector<uint32_t> hr(G);
  FL_HIP(hipMemcpyAsync(hr.data(), A.rcount, G * 4, hipMemcpyDeviceToHost, c.s));
  c.sync();
  for (uint32_t q = 0; q < G; ++q) rounds_out[q] += hr[q];
  return FL_OK;
}

}  // namespace fl
