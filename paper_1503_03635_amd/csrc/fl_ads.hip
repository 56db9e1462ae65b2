// fl_ads.hip -- bottom-k all-distances sketches (ADS, Sec. 3.3) by rounds of
// edge relaxation on the GPU.
//
// Schedule.  Round D settles every sketch entry at distance exactly D (integer
// weights >= 1).  A candidate (r, D) reaches u from an in-neighbour v over an
// arc v -> u of weight w only if v inserted r in round D - w, so all entries at smaller
// distances are final when round D runs: sketches grow append-only, already in
// (distance, id) order, and no entry is ever evicted (the CleanUp of Alg. 2 is
// never needed).  With unit weights this is the superstep order of Alg. 2.
// Entries move along arcs, so on a directed graph the sketch of u holds the
// vertices that reach u, at d(v, u) (an undirected graph is read as both arcs).
//
// Work items.  A vertex with at most TASK_ARCS arcs (TASK_ARCS_SPARSE in
// rounds run from marks) is one task; a larger one is split into tasks of
// that many arcs.  Each task (one wave64) streams the
// entries its neighbours inserted at distance D - w (pull), drops those whose
// rank is not below T_u (the k-th smallest rank of u's sketch so far: k
// entries that all come first have a smaller rank) and those already in u's
// bottom-k set, and prunes the rest.  A split vertex's tasks leave their kept
// sets in scratch; a merge wave prunes their union (the prune is associative
// and idempotent, so the split does not change the result).
//
// Level records and marks.  The level a vertex commits at distance D is
// described in slot D % NS of its record ring (start, count and its two
// smallest ranks), so a level of one or two entries needs no further read and
// a level whose smallest rank fails the reader's threshold is skipped whole.
// In rounds run from marks, the committing vertex sets, for each arc out of it,
// the bit of the arc's position in the head's in-arc row in the bit plane of
// the round the level reaches the head; that round's tasks are the vertices
// with a bit in their row, and a task reads only the arcs whose bits are set.
//
// Level prune.  A candidate of level D is accepted iff fewer than k ranks
// below its own belong to entries that come first: the sketch so far, or
// level-D candidates with a smaller vertex id (ties in distance go by id).
// Candidates are counting-sorted into id buckets; buckets are walked in id
// order, filtered in parallel against the running k-th smallest rank, and
// the survivors of a bucket are decided 64 at a time by one parallel count
// (set elements below + earlier candidates of the chunk below < k).
// Levels are stored in increasing rank order while the rounds run (a
// neighbour reads one only up to its threshold); the rows that need the
// canonical order (those with a HIP-threshold row) also receive each level in
// id order, in their threshold row, at commit.  A last pass moves that order
// into the sketch row and computes the HIP thresholds T_j (k-th smallest
// rank before entry j) in its place.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "fl_ads.h"
#include "fl_common.h"

namespace fl {

constexpr int TASK_WPB = 1;         // waves per block of the round kernels: a block's LDS is
                                    // freed when its own task ends (task lengths vary widely)
// Survivor buffer of a level (ids per wave): ADS_SB for k <= 64, twice that
// for k <= 128.  A level accepts about k (1 + ln(N / k)) of its N candidates
// (453 for k = 32 and N = 2^24), so k <= 32 starts with half the buffer: the
// round kernel then fits 5 waves per SIMD instead of 4.  A level that
// overflows it anyway restarts the build with the full buffer.
constexpr uint32_t ADS_SB = 1024;
static_assert((ADS_SB & (ADS_SB - 1)) == 0, "wave_sort_lds pads to a power of two inside the buffer");
inline uint32_t ads_full_sb(uint32_t k) { return k > 64 ? 2 * ADS_SB : ADS_SB; }
constexpr uint32_t TASK_ARCS = 1024;  // arcs per task of a split vertex in dense rounds (the fewest)
// Sparse rounds (run from marks) cut only longer rows: there a hub is active in
// most rounds but few of its arcs bring candidates, and every split costs a
// merge that prunes the tasks' kept sets again.  Results do not depend on the
// cut (a candidate accepted over all arcs is accepted within its piece, and
// the merge prunes the union exactly).
constexpr uint32_t TASK_ARCS_SPARSE = 2048;
static_assert(TASK_ARCS_SPARSE >= TASK_ARCS, "scratch slots are sized for TASK_ARCS");
// With marks by arc a task reads only the arcs that carry a level, so its cost
// follows those, not its length: rows are cut far less often.
constexpr uint32_t TASK_ARCS_FLAGGED = 8192;
static_assert(TASK_ARCS_FLAGGED >= TASK_ARCS, "scratch slots are sized for TASK_ARCS");
// A vertex that is new to u at this level arrives over every arc whose tail
// holds it, hundreds of times for the lowest ranks, and until the next prune
// each copy passes the offer's other filters.  The last rank buffered under
// each low-bits key is kept (no atomics: a lost entry only lets a copy pass).
// Round kernels of R-MAT 2^22 (unit, k = 64): 514 ms without, 467 with 128 keys,
// 440 with 256, 467 with 512 (LDS for fewer waves then); 2^18 at k = 128: 85, 78
// with 128 keys, 82 with 256.  (The two-task kernel's levels are small: there 64
// keys per task cost 224 -> 248 ms on R-MAT 2^21, weights 1..100, and are not
// kept.)
constexpr uint32_t seen_keys(int KR) { return KR == 1 ? 256 : 128; }
constexpr uint32_t level_words(int KR) { return (2 + KR) * WAVE + seen_keys(KR); }  // s_cnt of the round kernels
constexpr uint32_t LONG_LIST = 64;  // entry lists at least this long are streamed one arc at a time

// Statistics counters of the sketch rounds, cumulative over a build: one
// 128-byte line per stripe holds every field, and a block adds into stripe
// blockIdx.x % CTR_STRIPES (a field striped over consecutive words would put
// ~16 blocks on each line).
constexpr uint32_t CTR_STRIPES = 256, CTR_FIELDS = 16;
enum CtrField : uint32_t {
  CF_EXAMINED = 0,  // relaxations executed
  CF_COMMITS,       // levels committed (vertices that changed)
  CF_SURVIVORS,     // candidates kept after the offer filters
  CF_PRUNES,        // level prunes
  CF_SCANNED,       // arcs scanned (dbg)
  CF_MATCHED,       // level records matched (dbg)
  CF_REACH,         // largest distance any arc was marked for (a maximum)
  CF_COUNT
};
struct AdsArgs {
  uint32_t n, k, cap, NS;
  const uint32_t *gid;  // graph of each vertex (nullptr: one graph)
  const SegInfo *seg;   // per-graph rank keys, base, bucket shift
  // entries travel along arcs: a vertex gathers over its in-arcs and, when
  // its sketch changes, marks the heads of its out-arcs (one CSR twice when
  // the graph is undirected)
  const uint64_t *row_ptr;  // in-arcs
  const uint32_t *col;
  const uint32_t *w;
  const uint64_t *out_ptr;  // out-arcs
  const uint32_t *out_col;
  const uint32_t *out_w;
  uint32_t *sk_rank;
  uint32_t *sk_dist;
  uint32_t *bk;
  uint32_t *cnt;
  uint4 *lvl;          // [NS * n] level records, slot (D % NS) of each vertex
  // Marks of the rounds to come, in planes of pw words, plane D % NS for round
  // D.  With by_arc, bit p of a plane says that a level reaches in-arc position
  // p in that round; otherwise (arc positions do not fit 32 bits) bit u says
  // that some level reaches vertex u, and a task scans all its in-arcs.
  uint32_t *plane;
  uint64_t pw;
  uint32_t by_arc;
  const uint32_t *out_to_in;  // [m] out-arc -> in-arc position (by_arc)
  uint32_t *reach;            // [1] CF_REACH as of the start of the current round
  uint32_t *kept;      // [slots * sb] kept ids of split tasks (sb: the survivor buffer of the build)
  uint32_t *kept_cnt;  // [slots]
  uint64_t *ctr;       // [CTR_STRIPES * CTR_FIELDS] cumulative counters, see CtrField
  uint32_t dbg;
  uint32_t *status;    // [0] capacity overflow, [1] survivor-buffer overflow
  uint32_t *thr;             // [rows * cap] threshold rows: canonical-order ranks until the last pass
  const uint32_t *thr_idx;   // [n] threshold row of each vertex (INF32 = none); nullptr = row u
};

__device__ inline uint32_t thr_row(const AdsArgs &P, uint32_t u) {
  return P.thr ? (P.thr_idx ? P.thr_idx[u] : u) : INF32;
}

__device__ inline void ctr_add(const AdsArgs &P, CtrField f, uint64_t v) {
  atomicAdd((unsigned long long *)&P.ctr[(blockIdx.x % CTR_STRIPES) * CTR_FIELDS + f], (unsigned long long)v);
}

// The level a vertex committed at distance D stays in slot D % NS until the
// level at D + NS reuses it: {D, its smallest rank, its second smallest rank
// (INF32 for a single entry), start | count << 16}.  A level is stored in
// increasing rank order, so a reader whose threshold is at most the smallest
// rank skips it whole, and a level of one or two entries is read from the
// record alone.
__device__ inline uint4 level_record(uint32_t D, uint32_t r0, uint32_t r1, uint32_t start, uint32_t count) {
  return make_uint4(D, r0, r1, start | (count << 16));
}

// The out-arc a leads to a level in round D + w: set its bit in that round's
// plane (Dm = D % NS), with no wait.  A larger distance than any marked before
// goes to the block's stripe of CF_REACH (few arcs: from the first rounds on
// only the heaviest exceed what earlier rounds reached; with unit weights
// every arc of a round reaches as far, and one lane speaks for the wave).
template <bool UNITW>
__device__ inline void mark_arc(const AdsArgs &P, uint64_t a, uint32_t D, uint32_t Dm, uint32_t seen) {
  const uint32_t wv = UNITW ? 1u : P.out_w[a];
  uint32_t s = Dm + wv;
  if (s >= P.NS) s -= P.NS;
  uint32_t *pl = P.plane + (size_t)s * P.pw;
  if (P.by_arc) {
    const uint32_t p = P.out_to_in[a];
    atomicOr(&pl[p >> 5], 1u << (p & 31));
  } else {
    const uint32_t y = P.out_col[a];
    const uint32_t bit = 1u << (y & 31);
    if (!(__hip_atomic_load(&pl[y >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) atomicOr(&pl[y >> 5], bit);
  }
  if (D + wv > seen && (!UNITW || lane_id() == __ffsll((long long)__ballot(1)) - 1))
    atomicMax((unsigned long long *)&P.ctr[(blockIdx.x % CTR_STRIPES) * CTR_FIELDS + CF_REACH],
              (unsigned long long)(D + wv));
}

// u committed a level at distance D: mark the arcs out of u.  Several waves
// can share a long row: wave `part` of `parts` takes every parts-th group of
// 64 arcs.
template <bool UNITW>
__device__ inline void mark_neighbours(const AdsArgs &P, uint32_t u, uint32_t D, uint32_t part = 0,
                                       uint32_t parts = 1) {
  const int lane = lane_id();
  const uint64_t a0 = P.out_ptr[u], a1 = P.out_ptr[u + 1];
  const uint32_t Dm = D % P.NS, seen = *P.reach;
  for (uint64_t a = a0 + (uint64_t)part * WAVE + lane; a < a1; a += (uint64_t)parts * WAVE)
    mark_arc<UNITW>(P, a, D, Dm, seen);
}

// Round 0: every vertex holds (r(v), 0).  One wave per vertex.
template <bool UNITW>
__global__ __launch_bounds__(256) void k_ads_init(AdsArgs P, int mark) {
  const int lane = lane_id();
  const uint64_t u64 = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  if (u64 >= P.n) return;
  const uint32_t u = (uint32_t)u64;
  const uint32_t r = rank_of(u, rank_map(P.seg[seg_of(P.gid, u)]));
  if (lane == 0) {
    P.sk_rank[(size_t)u * P.cap] = r;
    P.sk_dist[(size_t)u * P.cap] = 0;
    const uint32_t tr = thr_row(P, u);
    if (tr != INF32) P.thr[(size_t)tr * P.cap] = r;
    P.bk[(size_t)u * P.k] = r;
    P.cnt[u] = 1;
    P.lvl[u] = level_record(0, r, INF32, 0, 1);  // slot 0
  }
  if (mark) mark_neighbours<UNITW>(P, u, 0);
}

// ---------------------------------------------------------------------------
// sorting helpers
// ---------------------------------------------------------------------------
// Sort s[0..n) ascending in LDS (bitonic over the next power of two; the
// caller guarantees that many slots).
__device__ inline void wave_sort_lds(uint32_t *s, uint32_t n) {
  const int lane = lane_id();
  uint32_t p2 = 2;
  while (p2 < n) p2 <<= 1;
  for (uint32_t i = n + lane; i < p2; i += WAVE) s[i] = INF32;
  wave_lds_sync();
  for (uint32_t k2 = 2; k2 <= p2; k2 <<= 1) {
    for (uint32_t j = k2 >> 1; j > 0; j >>= 1) {
      for (uint32_t i = lane; i < p2; i += WAVE) {
        const uint32_t ixj = i ^ j;
        if (ixj > i) {
          const uint32_t a = s[i], b = s[ixj];
          if ((a > b) == ((i & k2) == 0)) {
            s[i] = b;
            s[ixj] = a;
          }
        }
      }
      wave_lds_sync();
    }
  }
}

// Sort the distinct ranks s[0..n), none above `most`, ascending in place (tmp:
// n words, s_b: WAVE words).  A counting sort into 64 buckets, four to each
// octave below `most`, then each rank's place among its bucket's.  A level's
// accepted ranks are about as many in every octave above the bottom-k's, so a
// bucket holds some ten of a few hundred: a tenth of the instructions of a
// bitonic network over LDS, and a few waits instead of 45 (levels of more than
// 64 ids, 314 on average on R-MAT 2^22, unit, k = 64: with the copies dropped
// from large buckets, round kernels 540 -> 514 ms).
__device__ inline void wave_sort_ranks(uint32_t *s, uint32_t *tmp, uint32_t n, uint32_t most, uint32_t *s_b) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t z0 = (uint32_t)__clz((int)(most | 1u));
  auto bucket = [&](uint32_t r) -> uint32_t {
    const uint32_t x = r | 1u, z = (uint32_t)__clz((int)x);
    const uint32_t o = z - z0;  // octaves below `most`
    return o > 15u ? 0u : 60u - 4u * o + ((x << z) >> 29 & 3u);
  };
  s_b[lane] = 0;
  wave_lds_sync();
  for (uint32_t i = lane; i < n; i += WAVE) atomicAdd(&s_b[bucket(s[i])], 1u);
  wave_lds_sync();
  const uint32_t c = s_b[lane];
  const uint32_t st = wave_scan_incl(c) - c;
  wave_lds_sync();
  s_b[lane] = st;
  wave_lds_sync();
  for (uint32_t i = lane; i < n; i += WAVE) {
    const uint32_t r = s[i];
    tmp[atomicAdd(&s_b[bucket(r)], 1u)] = r;
  }
  wave_lds_sync();
  for (uint32_t i = lane; i < n; i += WAVE) {
    const uint32_t r = tmp[i], b = bucket(r);
    const uint32_t b0 = b ? s_b[b - 1] : 0u, b1 = s_b[b];  // s_b[b] is the bucket's end now
    uint32_t at = b0;
    for (uint32_t j = b0; j < b1; ++j) at += tmp[j] < r ? 1u : 0u;
    s[at] = r;
  }
  wave_lds_sync();
}

// Sort one value per lane ascending across the wave (bitonic network).
__device__ inline uint32_t wave_sort_reg(uint32_t x) {
  const int lane = lane_id();
#pragma unroll
  for (int k2 = 2; k2 <= WAVE; k2 <<= 1) {
#pragma unroll
    for (int j = k2 >> 1; j > 0; j >>= 1) {
      const uint32_t y = __shfl_xor(x, j, WAVE);
      const bool keep_min = ((lane & k2) == 0) == ((lane & j) == 0);
      x = keep_min ? (x < y ? x : y) : (x > y ? x : y);
    }
  }
  return x;
}

// Values of lanes 0..n-1 (n <= 64; lanes from n on hold INF32) sorted
// ascending onto lanes 0..n-1, INF32 above.  Each lane counts the staged
// values that come before its own (smaller, or equal on a lower lane), four
// per LDS read, and writes its value there: for a few values this is cheaper
// than the 21 exchange steps of the bitonic network.  s_r: 64 words, 16-byte
// aligned, free on entry and on return.
constexpr uint32_t COUNT_SORT_MAX = 16;
__device__ inline uint32_t wave_sort_few(uint32_t x, uint32_t n, uint32_t *s_r) {
  const uint32_t lane = (uint32_t)lane_id();
  s_r[lane] = x;
  wave_lds_sync();
  uint32_t pos = 0;
  for (uint32_t j4 = 0; j4 < n; j4 += 4) {
    const uint4 v = *reinterpret_cast<const uint4 *>(&s_r[j4]);
    pos += (v.x < x || (v.x == x && j4 + 0 < lane)) ? 1u : 0u;
    pos += (v.y < x || (v.y == x && j4 + 1 < lane)) ? 1u : 0u;
    pos += (v.z < x || (v.z == x && j4 + 2 < lane)) ? 1u : 0u;
    pos += (v.w < x || (v.w == x && j4 + 3 < lane)) ? 1u : 0u;
  }
  wave_lds_sync();
  if (lane < n) s_r[pos] = x;
  wave_lds_sync();
  const uint32_t y = lane < n ? s_r[lane] : INF32;
  wave_lds_sync();
  return y;
}

// Merge of a bitonic sequence held one value per lane into ascending
// (desc = false) or descending order.
__device__ inline uint32_t wave_bitonic_merge(uint32_t x, bool desc) {
  const int lane = lane_id();
#pragma unroll
  for (int j = 32; j >= 1; j >>= 1) {
    const uint32_t y = __shfl_xor(x, j, WAVE);
    const bool lo = ((lane & j) == 0) != desc;
    x = lo ? (x < y ? x : y) : (x > y ? x : y);
  }
  return x;
}

// Two ascending sequences a and b, one value per lane: lo receives the 64
// smallest of both, hi the 64 largest, each ascending (the first step of a
// bitonic merge splits them into two bitonic halves).
__device__ inline void wave_merge2(uint32_t a, uint32_t b, uint32_t &lo, uint32_t &hi) {
  const uint32_t br = __shfl(b, WAVE - 1 - lane_id(), WAVE);
  lo = wave_bitonic_merge(a < br ? a : br, false);
  hi = wave_bitonic_merge(a < br ? br : a, false);
}

// The running bottom-k set of a level: ascending, element i in register
// i / 64 at lane i % 64, INF32 above its size.  One register holds k <= 64,
// two hold k <= 128.
template <int KR>
struct KSet {
  uint32_t v[KR];
};

// element i of the set (i per lane, below 64 KR)
template <int KR>
__device__ inline uint32_t kset_at(const KSet<KR> &s, uint32_t i) {
  if (KR == 1) return __shfl(s.v[0], (int)i, WAVE);
  const uint32_t a = __shfl(s.v[0], (int)(i & 63u), WAVE);
  const uint32_t b = __shfl(s.v[KR - 1], (int)(i & 63u), WAVE);
  return i < 64u ? a : b;
}

// the set becomes the k smallest of itself and the ascending chunk x
// (INF32-padded)
template <int KR>
__device__ inline void kset_merge(KSet<KR> &s, uint32_t x, uint32_t k) {
  const uint32_t lane = (uint32_t)lane_id();
  if (KR == 1) {
    const uint32_t y = __shfl(x, WAVE - 1 - (int)lane, WAVE);
    uint32_t mm = s.v[0] < y ? s.v[0] : y;  // bitonic, holds the 64 smallest of both
    mm = wave_bitonic_merge(mm, false);
    s.v[0] = lane < k ? mm : INF32;
  } else {
    // the 64 smallest of everything lie in the lower half and the chunk; the
    // next 64 in what is left of those and the upper half
    uint32_t lo1, hi1, lo2, hi2;
    wave_merge2(s.v[0], x, lo1, hi1);
    wave_merge2(hi1, s.v[KR - 1], lo2, hi2);
    s.v[0] = lane < k ? lo1 : INF32;
    s.v[KR - 1] = 64u + lane < k ? lo2 : INF32;
  }
}

// number of values below r in a set held one value per lane, ascending, with
// INF32 above its size (per-lane r; every lane runs the shuffles)
__device__ inline uint32_t set_count_below(uint32_t setv, uint32_t r) {
  uint32_t q = 0;
#pragma unroll
  for (uint32_t s = 32; s >= 1; s >>= 1) {
    const uint32_t val = __shfl(setv, (int)(q + s - 1), WAVE);
    if (val < r) q += s;
  }
  const uint32_t atq = __shfl(setv, (int)q, WAVE);
  if (atq < r) ++q;  // all 64 values below r
  return q;
}

// number of elements of the set below r (per-lane r)
template <int KR>
__device__ inline uint32_t kset_below(const KSet<KR> &s, uint32_t r) {
  const uint32_t q = set_count_below(s.v[0], r);
  if (KR == 1) return q;
  const uint32_t q2 = set_count_below(s.v[KR - 1], r);
  return q == 64u ? 64u + q2 : q;
}

// The lanes (of vm, those with valid set) with a smaller rank than this one.
// The ranks of the valid lanes are distinct and at most `most`.  They are
// compared bit by bit from the highest that can differ: eq holds the lanes
// equal so far, and a ballot of each bit splits it, until every eq is a single
// lane (after some 13 bits for 64 random ranks, 10 instructions each).
// Comparing all pairs out of LDS took 13 instructions per 4 candidates and
// then a sort of the accepted ranks, which here have their places: round
// kernels of R-MAT 2^22 (unit, k = 64) 576 -> 547 ms with it for every chunk,
// also small ones (700 -> 668 ms when first used, for more than 24).
__device__ inline uint64_t wave_smaller(uint32_t r, bool valid, uint64_t vm, uint32_t most) {
  uint32_t el = valid ? (uint32_t)vm : 0u, eh = valid ? (uint32_t)(vm >> 32) : 0u, ll = 0, lh = 0;
  for (int b = most ? 31 - __clz(most) : 0; b >= 0; b -= 4) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if (b < d) break;
      const uint32_t bm = (uint32_t)__builtin_amdgcn_sbfe((int)r, (uint32_t)(b - d), 1u);
      const uint64_t B = __ballot(bm != 0);
      const uint32_t bl = (uint32_t)B, bh = (uint32_t)(B >> 32);
      ll |= el & ~bl & bm;
      lh |= eh & ~bh & bm;
      el &= ~(bl ^ bm);
      eh &= ~(bh ^ bm);
    }
    if (!__ballot((el & (el - 1)) | (eh & (eh - 1)) | (el && eh ? 1u : 0u))) break;
  }
  return ((uint64_t)lh << 32) | ll;
}

// One chunk of candidates, one id per lane in ascending lane order (INF32 =
// empty slot at the end); duplicates are adjacent; `prev` is the last id of
// the previous chunk of this level.  Candidate i is accepted iff
//   #(running set below r_i) + #(earlier distinct candidates of the chunk below r_i) < k.
// The running set becomes the k smallest ranks of itself and the chunk.
// Returns the mask of accepted lanes.
template <int KR>
__device__ inline uint64_t chunk_accept(uint32_t id, uint32_t k, const RankMap &rm, KSet<KR> &set,
                                        uint32_t &nset, uint32_t &prev, uint32_t *s_r) {
  const int lane = lane_id();
  uint32_t left = __shfl_up(id, 1, WAVE);
  if (lane == 0) left = prev;
  bool valid = id != INF32 && id != left;
  const uint32_t r = valid ? rank_of(id, rm) : INF32;
  const uint32_t q = kset_below(set, r);
  // (none is in the set at the level's start, the offers saw to that, and a
  // repeated id is next to its first)
  // one with k set elements below it is rejected, and so is any it could count
  // for: only those below the set's k-th rank remain
  if (q >= k) valid = false;
  const uint64_t vm = __ballot(valid);
  const uint32_t kth = nset < k ? INF32 : __builtin_amdgcn_readfirstlane(kset_at(set, k - 1));
  const uint64_t lt = wave_smaller(r, valid, vm, kth);
  const bool acc = valid && q + lanes_below(lt) < k;
  const uint64_t am = __ballot(acc);
  const uint32_t na = (uint32_t)__popcll(am);
  if (na) {
    // the running set becomes the k smallest of (set, accepted ranks), which
    // each lane puts in its place (rejected candidates have k smaller ranks
    // before them and never enter it)
    if (acc) s_r[__popcll(lt & am)] = r;
    wave_lds_sync();
    const uint32_t x = (uint32_t)lane < na ? s_r[lane] : INF32;
    wave_lds_sync();
    kset_merge(set, x, k);
  }
  const uint32_t tot = nset + na;
  nset = tot < k ? tot : k;
  const uint64_t real = __ballot(id != INF32);
  if (real) prev = __shfl(id, 63 - __clzll(real), WAVE);
  return am;
}

// Prune of one distance level.  s_id[0..ns) holds candidate ranks (unsorted,
// duplicates allowed); set/nset the running set.  Accepted ids end in
// s_tmp[0..m) in increasing id order; returns m.  s_id is clobbered.
// s_cnt holds level_words(KR) words: [0, WAVE) bucket offsets, then the
// pending chunk; [WAVE, (1 + KR) WAVE) belongs to the caller; the next WAVE
// hold chunk ranks, the rest is the caller's.
// With tbk, lane b of *tbk receives a rank bound for id bucket b: the running
// k-th smallest rank when the bucket was reached, which no later candidate of
// that bucket can beat.
template <int KR>
__device__ inline uint32_t prune_level(uint32_t *s_id, uint32_t *s_tmp, uint32_t *s_cnt, uint32_t ns,
                                       uint32_t k, const RankMap &rm, KSet<KR> &set, uint32_t &nset,
                                       uint32_t *tbk = nullptr) {
  const int lane = lane_id();
  uint32_t *s_pend = s_cnt;
  uint32_t *s_r = s_cnt + (1 + KR) * WAVE;
  uint32_t m = 0, prev = INF32;
  if (ns <= (uint32_t)WAVE && !tbk) {
    uint32_t x = (uint32_t)lane < ns ? id_of(s_id[lane], rm) : INF32;
    x = ns <= COUNT_SORT_MAX ? wave_sort_few(x, ns, s_r) : wave_sort_reg(x);
    const uint64_t am = chunk_accept(x, k, rm, set, nset, prev, s_r);
    if ((am >> lane) & 1) s_tmp[lanes_below(am)] = x;
    wave_lds_sync();
    return (uint32_t)__popcll(am);
  }
  // counting sort by id bucket (bucket order is id order)
  s_cnt[lane] = 0;
  wave_lds_sync();
  for (uint32_t i = lane; i < ns; i += WAVE) {
    const uint32_t id = id_of(s_id[i], rm);
    s_id[i] = id;
    atomicAdd(&s_cnt[bucket_of(id, rm)], 1u);
  }
  wave_lds_sync();
  const uint32_t bc = s_cnt[lane];
  const uint32_t bstart = wave_scan_incl(bc) - bc;
  wave_lds_sync();
  s_cnt[lane] = bstart;
  wave_lds_sync();
  for (uint32_t i = lane; i < ns; i += WAVE) {
    const uint32_t id = s_id[i];
    s_tmp[atomicAdd(&s_cnt[bucket_of(id, rm)], 1u)] = id;
  }
  wave_lds_sync();
  // Buckets are walked in id order, in windows: the whole buckets among the
  // next WAVE ids, one id per lane.  A window's ids are filtered against the
  // running threshold and gathered in one pending chunk of at most WAVE ids,
  // which is decided when the next window does not fit; accepted ids are
  // written back to s_tmp[m..), which never reaches a bucket not yet read
  // (accepted ones are a subset of the buckets already read).  A bucket of
  // more than WAVE ids is filtered in place first, and if it is still larger,
  // sorted into s_id (free now) and taken from there.
  // With one bucket per step (some 15 ids each, and a rank, a threshold and a
  // compaction for every one) the walk was a quarter of the prune.
  const uint32_t bend = bstart + bc;
  uint64_t nonempty = __ballot(bc != 0);
  uint32_t tb = INF32;
  int done_b = -1;
  uint32_t npend = 0;
  uint32_t w0 = 0, wn = 0;  // the rest of a large bucket, sorted, in s_id
  auto threshold = [&]() -> uint32_t { return nset < k ? INF32 : kset_at(set, k - 1); };
  for (;;) {
    const bool end = !wn && !nonempty;
    bool fresh = false, wait = false;  // the window starts at a new bucket; it waits for the pending chunk
    int b = 0, last = 0;
    uint32_t cnt = 0;
    const uint32_t *win = s_tmp;
    bool open = nset < k;
    uint32_t T = threshold();
    if (wn) {
      cnt = wn < (uint32_t)WAVE ? wn : (uint32_t)WAVE;
      win = s_id + w0;
      w0 += cnt;
      wn -= cnt;
    } else if (nonempty) {
      b = __ffsll((long long)nonempty) - 1;
      const uint32_t sb = __builtin_amdgcn_readlane(bstart, b);
      const uint64_t fit = __ballot(bend - sb <= (uint32_t)WAVE) & nonempty;
      win = s_tmp + sb;
      if (fit) {
        last = 63 - __clzll(fit);
        cnt = __builtin_amdgcn_readlane(bend, last) - sb;
        nonempty &= ~fit;
        fresh = true;
      } else if (npend) {
        wait = true;
      } else {
        // the running threshold bounds every bucket up to b
        if (lane > done_b && lane <= b) tb = T;
        done_b = b;
        nonempty &= nonempty - 1;
        const uint32_t cb = __builtin_amdgcn_readlane(bc, b);
        for (uint32_t j0 = 0; j0 < cb; j0 += WAVE) {
          const uint32_t id = j0 + lane < cb ? s_tmp[sb + j0 + lane] : INF32;
          const bool pass = j0 + lane < cb && (open || rank_of(id, rm) < T);
          // most of a large bucket are copies of a few ids (a vertex reaches u
          // over many arcs): each 64 keep one of each
          const uint32_t x = wave_sort_reg(pass ? id : INF32);
          const uint32_t left = __shfl_up(x, 1, WAVE);
          const bool keep = x != INF32 && (lane == 0 || x != left);
          const uint64_t pm = __ballot(keep);
          if (keep) s_tmp[sb + cnt + lanes_below(pm)] = x;
          cnt += (uint32_t)__popcll(pm);
        }
        wave_lds_sync();
        if (cnt > (uint32_t)WAVE) {
          for (uint32_t i = lane; i < cnt; i += WAVE) s_id[i] = s_tmp[sb + i];
          wave_sort_lds(s_id, cnt);
          w0 = 0;
          wn = cnt;
          continue;
        }
      }
    }
    const uint32_t id = (uint32_t)lane < cnt ? win[lane] : INF32;
    const uint32_t r = rank_of(id, rm);
    bool pass = (uint32_t)lane < cnt && (open || r < T);
    uint64_t pm = __ballot(pass);
    uint32_t np = (uint32_t)__popcll(pm);
    if (npend && (end || wait || npend + np > (uint32_t)WAVE)) {
      uint32_t x = (uint32_t)lane < npend ? s_pend[lane] : INF32;
      x = npend <= COUNT_SORT_MAX ? wave_sort_few(x, npend, s_r) : wave_sort_reg(x);
      const uint64_t am = chunk_accept(x, k, rm, set, nset, prev, s_r);
      if ((am >> lane) & 1) s_tmp[m + lanes_below(am)] = x;
      m += (uint32_t)__popcll(am);
      npend = 0;
      wave_lds_sync();
      // every earlier candidate is decided: the threshold is exact for the window
      open = nset < k;
      T = threshold();
      pass = pass && (open || r < T);
      pm = __ballot(pass);
      np = (uint32_t)__popcll(pm);
    }
    if (end) break;
    if (fresh) {
      if (lane > done_b && lane <= last) tb = T;
      done_b = last;
    }
    if (pass) s_pend[npend + lanes_below(pm)] = id;
    npend += np;
    wave_lds_sync();
  }
  if (tbk) {
    const uint32_t Tend = nset < k ? INF32 : kset_at(set, k - 1);
    if (lane > done_b) tb = Tend;
    *tbk = tb;
  }
  return m;
}

// ---------------------------------------------------------------------------
// per-wave level state: candidate intake with filtering and buffering
// ---------------------------------------------------------------------------
template <int KR>
struct Level {
  KSet<KR> set0;         // u's bottom-k set at the start of the level
  uint32_t nset0;
  uint32_t T0;           // its k-th smallest rank (INF32 while fewer than k)
  bool full0;
  uint32_t cu;           // entries of u so far
  uint32_t ns;           // buffered candidates
  uint32_t tb;           // lane b: rank bound for candidates of id bucket b
  RankMap rm;            // ranks and id buckets of u's graph
  bool overflow;
  uint32_t nsurv, nprune;  // statistics
  uint32_t nmatch;         // level records found (per lane; with dbg only)
};

template <int KR>
__device__ inline void level_init(const AdsArgs &P, uint32_t u, Level<KR> &L, uint32_t *s_cnt) {
  const int lane = lane_id();
  const uint32_t k = P.k;
  L.rm = rank_map(P.seg[seg_of(P.gid, u)]);
  L.cu = __builtin_amdgcn_readfirstlane(P.cnt[u]);
  L.nset0 = L.cu < k ? L.cu : k;
#pragma unroll
  for (int g = 0; g < KR; ++g) {
    const uint32_t e = (uint32_t)(64 * g + lane);
    L.set0.v[g] = e < L.nset0 ? P.bk[(size_t)u * k + e] : INF32;
    s_cnt[WAVE + e] = L.set0.v[g];
  }
  for (uint32_t i = lane; i < seen_keys(KR); i += WAVE) s_cnt[(2 + KR) * WAVE + i] = INF32;
  wave_lds_sync();
  L.full0 = L.nset0 == k;
  L.T0 = L.full0 ? __builtin_amdgcn_readfirstlane(kset_at(L.set0, k - 1)) : INF32;
  L.ns = 0;
  L.tb = L.T0;
  L.overflow = false;
  L.nsurv = L.nprune = L.nmatch = 0;
}

// One candidate per lane (valid, rank r): keep it if its rank is
// below T0 and it is not already in the set; buffer kept ids, shrinking the
// buffer by a prune against the set when full.
template <int KR, uint32_t SB>
__device__ inline void level_offer(const AdsArgs &P, Level<KR> &L, bool valid, uint32_t r, uint32_t *s_id,
                                   uint32_t *s_tmp, uint32_t *s_cnt) {
  const uint32_t *s_set0 = s_cnt + WAVE;  // LDS copy of the set at the level start
  uint32_t *s_seen = s_cnt + (2 + KR) * WAVE;
  const int lane = lane_id();
  bool pass = valid && (!L.full0 || r < L.T0);
  if (!__ballot(pass)) return;
  {
    // already in the set (same vertex at a shorter distance)?  A search of
    // fixed length over the padded set, without branches: a loop that each
    // lane leaves at its own step cost more (round kernels of R-MAT 2^22, k =
    // 64: 743 -> 703 ms)
    const uint32_t seen = s_seen[r % seen_keys(KR)];
    uint32_t lo = 0;
#pragma unroll
    for (uint32_t s = 32 * KR; s >= 1; s >>= 1)
      if (s_set0[lo + s - 1] < r) lo += s;
    if (lo < L.nset0 && s_set0[lo] == r) pass = false;
    if (seen == r && r != INF32) pass = false;  // buffered in this level already
  }
  // Bucket bound from the last prune: all candidates of earlier id buckets
  // come first, and k of them (or of the set) already rank below it.  Until
  // there has been one the bound is T0, and the candidate's id is not needed:
  // the buffer holds ranks, and a prune turns all of them into ids, 64 at a
  // time, where an offer would do so for the 20 or so lanes that pass (round
  // kernels of R-MAT 2^22, unit, k = 64: 545 -> 540 ms).
  uint32_t bkt = 0;
  if (L.nprune) {
    bkt = bucket_of(pass ? id_of(r, L.rm) : L.rm.base, L.rm);
    const uint32_t bnd = __shfl(L.tb, (int)bkt, WAVE);
    if (pass && r >= bnd) pass = false;
  }
  uint64_t msk = __ballot(pass);
  if (!msk) return;
  uint32_t np = (uint32_t)__popcll(msk);
  if (L.ns + np > SB) {
    KSet<KR> tv = L.set0;
    uint32_t tn = L.nset0;
    if (!L.nprune) bkt = bucket_of(pass ? id_of(r, L.rm) : L.rm.base, L.rm);
    ++L.nprune;
    L.ns = prune_level(s_id, s_tmp, s_cnt, L.ns, P.k, L.rm, tv, tn, &L.tb);
    for (uint32_t i = lane; i < L.ns; i += WAVE) s_id[i] = rank_of(s_tmp[i], L.rm);
    wave_lds_sync();
    // the new bounds may reject some of this chunk too
    const uint32_t bnd2 = __shfl(L.tb, (int)bkt, WAVE);
    if (pass && r >= bnd2) pass = false;
    msk = __ballot(pass);
    np = (uint32_t)__popcll(msk);
    if (L.ns + np > SB) {
      L.overflow = true;
      return;
    }
  }
  if (pass) {
    s_id[L.ns + lanes_below(msk)] = r;
    s_seen[r % seen_keys(KR)] = r;
  }
  L.ns += np;
  L.nsurv += np;
  wave_lds_sync();
}

// One in-arc per lane (arc index a, valid): the level each arc's tail
// committed at distance D - w is offered to u's level D.  Levels of one or
// two entries come from the record; longer ones from the tail's sketch row,
// the whole wave on one list at a time when it is long (a level is stored in
// increasing rank order, so once a rank reaches T0 the rest cannot enter).
template <bool UNITW, int KR, uint32_t SB>
__device__ inline uint64_t gather_batch(const AdsArgs &P, uint32_t D, uint64_t a, bool valid, Level<KR> &L,
                                        uint32_t *s_id, uint32_t *s_tmp, uint32_t *s_cnt) {
  const int lane = lane_id();
  const uint32_t Dm = D % P.NS;
  uint64_t examined = 0;
  {
    uint32_t v = 0, st = 0, cn = 0, r0 = INF32, r1 = INF32;
    if (valid) {
      v = P.col[a];
      const uint32_t wv = UNITW ? 1u : P.w[a];
      if (wv <= D) {
        const uint32_t src = D - wv;
        const uint32_t sl = Dm >= wv ? Dm - wv : Dm + P.NS - wv;
        const uint4 rec = P.lvl[(size_t)sl * P.n + v];
        // a level whose smallest rank is not below T0 has nothing for u
        if (P.dbg && rec.x == src) ++L.nmatch;
        if (rec.x == src && (!L.full0 || rec.y < L.T0)) {
          r0 = rec.y;
          r1 = rec.z;
          st = rec.w & 0xFFFFu;
          // (one whose second smallest is not has one entry for u)
          cn = L.full0 && r1 >= L.T0 ? 1u : rec.w >> 16;
        }
      }
    }
    // Long lists: one arc at a time, the whole wave on its list, four loads in
    // flight (r0 is offered while r1, r2 and r3 arrive).  A level is stored in
    // increasing rank order, so once a rank reaches T0 the rest of the list
    // cannot enter u's sketch.  (A block past the stop test is loaded, not
    // counted.)  The filter and prune of an offer are a few thousand
    // instructions inlined, so there is one offer for long lists and one for
    // short ones; seven copies cost instruction fetches and scalar registers.
    uint64_t lm = __ballot(cn >= LONG_LIST);
    while (lm && !L.overflow) {
      const int j = __ffsll((long long)lm) - 1;
      lm &= lm - 1;
      const uint32_t vj = __builtin_amdgcn_readlane(v, j);
      const uint32_t stj = __builtin_amdgcn_readlane(st, j);
      const uint32_t cnj = __builtin_amdgcn_readlane(cn, j);
      const uint32_t *src = P.sk_rank + (size_t)vj * P.cap + stj;
      auto load = [&](uint32_t i) -> uint32_t { return i < cnj ? src[i] : INF32; };
      uint32_t q0 = load(lane), q1 = load(lane + WAVE), q2 = load(lane + 2 * WAVE), q3 = load(lane + 3 * WAVE);
      for (uint32_t c0 = 0; c0 < cnj && !L.overflow; c0 += WAVE) {
        const bool in = c0 + lane < cnj;
        const uint32_t r = q0;
        q0 = q1;
        q1 = q2;
        q2 = q3;
        q3 = load(c0 + lane + 4 * WAVE);
        examined += cnj - c0 < WAVE ? cnj - c0 : WAVE;
        level_offer<KR, SB>(P, L, in, r, s_id, s_tmp, s_cnt);
        if (L.full0 && __ballot(in && r >= L.T0)) break;
      }
    }
    // Short lists: flattened over the wave, the owner lane of an entry found by
    // binary search.  A level of one or two entries has its ranks in the
    // record.
    const uint32_t cs = cn < LONG_LIST ? cn : 0u;
    const uint32_t incl = wave_scan_incl(cs);
    const uint32_t total = __builtin_amdgcn_readlane(incl, WAVE - 1);
    const uint32_t excl = incl - cs;
    examined += total;
    for (uint32_t c0 = 0; c0 < total && !L.overflow; c0 += WAVE) {
      const uint32_t idx = c0 + lane;
      uint32_t pos = 0;  // owner lane: first lane whose inclusive count exceeds idx
#pragma unroll
      for (uint32_t s = 32; s >= 1; s >>= 1) {
        const uint32_t val = __shfl(incl, (int)(pos + s - 1), WAVE);
        if (val <= idx) pos += s;
      }
      const bool in = idx < total;
      const uint32_t ov = __shfl(v, (int)pos, WAVE);
      const uint32_t ost = __shfl(st, (int)pos, WAVE);
      const uint32_t ocn = __shfl(cs, (int)pos, WAVE);
      const uint32_t i = idx - __shfl(excl, (int)pos, WAVE);
      const uint32_t o0 = __shfl(r0, (int)pos, WAVE), o1 = __shfl(r1, (int)pos, WAVE);
      uint32_t r = i == 0 ? o0 : o1;
      if (in && ocn > 2) r = P.sk_rank[(size_t)ov * P.cap + ost + i];
      level_offer<KR, SB>(P, L, in, r, s_id, s_tmp, s_cnt);
    }
  }
  return examined;
}

// Stream the candidates of arcs [a0, a1) of u for level D (every in-arc is
// looked at: rounds run over the dense vertex list).
template <bool UNITW, int KR, uint32_t SB>
__device__ inline uint64_t gather_arcs(const AdsArgs &P, uint32_t D, uint64_t a0, uint64_t a1, Level<KR> &L,
                                       uint32_t *s_id, uint32_t *s_tmp, uint32_t *s_cnt) {
  const int lane = lane_id();
  uint64_t examined = 0;
  for (uint64_t b = a0; b < a1 && !L.overflow; b += WAVE)
    examined += gather_batch<UNITW, KR, SB>(P, D, b + lane, b + lane < a1, L, s_id, s_tmp, s_cnt);
  return examined;
}

// Rounds run from marks: a tail that committed a level set the bit of
// each arc it marked, at the arc's position in the in-arc rows, in the plane
// of the round the level reaches the head.  Only those arcs of [a0, a1) are
// read: 64 plane words per step, their set bits compacted over the wave.
template <bool UNITW, int KR, uint32_t SB>
__device__ inline uint64_t gather_flagged(const AdsArgs &P, uint32_t D, uint64_t a0, uint64_t a1, Level<KR> &L,
                                          uint32_t *s_id, uint32_t *s_tmp, uint32_t *s_cnt) {
  const int lane = lane_id();
  const uint32_t *plane = P.plane + (size_t)(D % P.NS) * P.pw;
  const uint64_t w0 = a0 >> 5, w1 = (a1 + 31) >> 5;
  uint64_t examined = 0;
  for (uint64_t wb = w0; wb < w1 && !L.overflow; wb += WAVE) {
    const uint64_t wi = wb + lane;
    uint32_t bits = 0;
    if (wi < w1) {
      bits = plane[wi];
      const uint64_t base = wi << 5;  // arcs [base, base + 32) of this word
      if (base < a0) bits &= ~0u << (uint32_t)(a0 - base);
      if (a1 - base < 32) bits &= (1u << (uint32_t)(a1 - base)) - 1u;
    }
    const uint32_t nb = (uint32_t)__popc(bits);
    const uint32_t incl = wave_scan_incl(nb);
    const uint32_t total = __shfl(incl, WAVE - 1, WAVE);
    for (uint32_t c0 = 0; c0 < total && !L.overflow; c0 += WAVE) {
      const uint32_t idx = c0 + lane;
      uint32_t pos = 0;  // word (lane) holding set bit idx: first lane whose inclusive count exceeds idx
#pragma unroll
      for (uint32_t sh = 32; sh >= 1; sh >>= 1) {
        const uint32_t val = __shfl(incl, (int)(pos + sh - 1), WAVE);
        if (val <= idx) pos += sh;
      }
      const bool valid = idx < total;
      const uint32_t src = valid ? pos : 0u;
      uint32_t x = __shfl(bits, (int)src, WAVE);
      uint32_t kth = idx - (__shfl(incl, (int)src, WAVE) - (uint32_t)__popc(x));
      uint32_t bit = 0;  // position of the kth set bit of x
#pragma unroll
      for (uint32_t sh = 16; sh >= 1; sh >>= 1) {
        const uint32_t cnt = (uint32_t)__popc(x & ((1u << sh) - 1u));
        if (kth >= cnt) {
          kth -= cnt;
          x >>= sh;
          bit += sh;
        }
      }
      const uint64_t a = ((wb + src) << 5) + bit;
      examined += gather_batch<UNITW, KR, SB>(P, D, a, valid, L, s_id, s_tmp, s_cnt);
    }
  }
  return examined;
}

// Final prune of u's level-D candidates and the append of the accepted ones.
template <bool UNITW, int KR>
__device__ inline bool level_commit(const AdsArgs &P, uint32_t u, uint32_t D, Level<KR> &L, int mark, uint32_t *s_id,
                                    uint32_t *s_tmp, uint32_t *s_cnt) {
  const int lane = lane_id();
  if (L.ns == 0) return false;
  KSet<KR> set = L.set0;
  uint32_t nset = L.nset0;
  const uint32_t m = prune_level(s_id, s_tmp, s_cnt, L.ns, P.k, L.rm, set, nset);
  if (m == 0) return false;
  const uint32_t cu = L.cu;
  if (cu + m > P.cap) {
    if (lane == 0) atomicOr(&P.status[0], 1u);
    return false;
  }
  // The level is stored in increasing rank order, so that a neighbour reads
  // it only up to its own threshold.  A row with a threshold row also gets the
  // level in id order (the order of s_tmp) there, for the last pass.
  const uint32_t tr = thr_row(P, u);
  if (tr != INF32) {
    uint32_t *trow = P.thr + (size_t)tr * P.cap + cu;
    for (uint32_t i = lane; i < m; i += WAVE) trow[i] = rank_of(s_tmp[i], L.rm);
  }
  const size_t base = (size_t)u * P.cap + cu;
  uint32_t x0, x1;  // the two smallest ranks of the level, for its record
  if (m <= (uint32_t)WAVE) {
    uint32_t *s_r = s_cnt + (1 + KR) * WAVE;
    const bool in = (uint32_t)lane < m;
    uint32_t x = in ? rank_of(s_tmp[lane], L.rm) : INF32;
    const uint64_t lt = wave_smaller(x, in, m < (uint32_t)WAVE ? (1ull << m) - 1 : ~0ull, L.T0);
    if (in) s_r[__popcll(lt)] = x;
    wave_lds_sync();
    x = in ? s_r[lane] : INF32;
    wave_lds_sync();
    if ((uint32_t)lane < m) {
      P.sk_rank[base + lane] = x;
      P.sk_dist[base + lane] = D;
    }
    x0 = __shfl(x, 0, WAVE);
    x1 = __shfl(x, 1, WAVE);
  } else {
    for (uint32_t i = lane; i < m; i += WAVE) s_id[i] = rank_of(s_tmp[i], L.rm);
    wave_lds_sync();
    wave_sort_ranks(s_id, s_tmp, m, L.T0, s_cnt);
    for (uint32_t i = lane; i < m; i += WAVE) {
      P.sk_rank[base + i] = s_id[i];
      P.sk_dist[base + i] = D;
    }
    x0 = s_id[0];
    x1 = s_id[1];
  }
#pragma unroll
  for (int g = 0; g < KR; ++g)
    if ((uint32_t)(64 * g + lane) < nset) P.bk[(size_t)u * P.k + 64 * g + lane] = set.v[g];
  if (lane == 0) {
    P.cnt[u] = cu + m;
    P.lvl[(size_t)(D % P.NS) * P.n + u] = level_record(D, x0, x1, cu, m);
    ctr_add(P, CF_COMMITS, 1);
  }
  if (mark) mark_neighbours<UNITW>(P, u, D);
  return true;
}

// One task, by one wave.  slot == INF32: the task is the whole vertex and
// commits; otherwise it leaves its kept set in scratch slot `slot`.
// What is the same in every lane (its count and threshold, the list a wave
// walks, in the five-wave instance for unit weights the task itself) is read
// into scalar registers.  As vector registers it made the five-wave instances
// (k <= 32) spill 29 of them, 5.6 KB of scratch traffic a task; 3 now (7 with
// weights): sketches of ER 1,000,000 (unit, average degree 4, k = 8) 44.4 -> 28.4
// ms, ER 300,000 11.6 -> 8.5, R-MAT 2^18 (unit, k = 32) 15.5 -> 13.5.  The others did
// not spill but do less work per lane: R-MAT 2^22 (unit, k = 64) 489 -> 465, 2^18 at
// k = 128 75 -> 70.  A scalar task costs them 2% in rounds run from marks (k = 64:
// R-MAT 2^20, weights 1..100, 255 -> 262 ms; a grid of 150 x 220, unit, 21.8 -> 22.2)
// and gives nothing in dense ones; without it ER 1,000,000 above takes 31.6.
template <bool UNITW, int KR, uint32_t SB>
__device__ inline void ads_task(const AdsArgs &P, uint32_t D, uint32_t u, uint32_t sub, uint32_t slot,
                                uint32_t task_arcs, int sparse, int mark, uint32_t *s_id, uint32_t *s_tmp,
                                uint32_t *s_cnt) {
  const int lane = lane_id();
  if (UNITW && SB <= ADS_SB / 2) {
    u = __builtin_amdgcn_readfirstlane(u);
    sub = __builtin_amdgcn_readfirstlane(sub);
    slot = __builtin_amdgcn_readfirstlane(slot);
  }
  Level<KR> L;
  level_init(P, u, L, s_cnt);
  const uint64_t r0 = P.row_ptr[u], r1 = P.row_ptr[u + 1];
  uint64_t a0 = r0, a1 = r1;
  if (slot != INF32) {
    a0 = r0 + (uint64_t)sub * task_arcs;
    a1 = a0 + task_arcs < r1 ? a0 + task_arcs : r1;
  }
  const uint64_t examined = sparse && P.by_arc ? gather_flagged<UNITW, KR, SB>(P, D, a0, a1, L, s_id, s_tmp, s_cnt)
                                               : gather_arcs<UNITW, KR, SB>(P, D, a0, a1, L, s_id, s_tmp, s_cnt);
  if (lane == 0) {
    ctr_add(P, CF_EXAMINED, examined);
    ctr_add(P, CF_SURVIVORS, L.nsurv);
    ctr_add(P, CF_PRUNES, L.nprune);
  }
  if (P.dbg) {
    const uint64_t nm = wave_sum_u64(L.nmatch);
    if (lane == 0) {
      ctr_add(P, CF_SCANNED, a1 - a0);
      ctr_add(P, CF_MATCHED, nm);
    }
  }
  if (L.overflow) {
    if (lane == 0) atomicOr(&P.status[1], 1u);
    return;
  }
  if (slot == INF32) {
    level_commit<UNITW, KR>(P, u, D, L, mark, s_id, s_tmp, s_cnt);
  } else {
    uint32_t m = 0;
    if (L.ns) {
      KSet<KR> set = L.set0;
      uint32_t nset = L.nset0;
      m = prune_level(s_id, s_tmp, s_cnt, L.ns, P.k, L.rm, set, nset);
      for (uint32_t i = lane; i < m; i += WAVE) P.kept[(size_t)slot * SB + i] = s_tmp[i];
    }
    if (lane == 0) P.kept_cnt[slot] = m;
  }
}

// ---------------------------------------------------------------------------
// Two small tasks per wave (k <= 32, rounds run from marks).  Lanes
// 0..31 run one task and lanes 32..63 the next; every step works within the
// lane's half (shuffles of width 32, ballots cut to the half), so the fixed
// per-task instructions are shared by two tasks.  A task the halves cannot
// finish -- a slice of a split vertex, a row of more than PAIR_ROW_MAX arcs,
// more than 64 survivors in its level -- is left, before it has written
// anything, to the one-wave kernel, which runs after this one in the same
// round on the list of tasks left.  Tasks of a round are independent and
// the prune does not depend on how candidates are grouped, so both kernels
// give the same levels.
// ---------------------------------------------------------------------------
// Device totals of one round run from marks.
struct RoundTot {
  unsigned long long tasks, slots, splits;  // task list, kept slots, split vertices
  unsigned long long left;                  // tasks the two-task kernel left
};
constexpr uint32_t HALF = 32;
// Rows longer than this go to the one-wave kernel too: a wave runs two
// unrelated tasks, and a long row would keep its partner half idle (2,048
// and 1,024 measured equal on the large weighted workload, 4,096 and no limit
// 2-4% slower).
constexpr uint64_t PAIR_ROW_MAX = 2048;
__device__ inline uint32_t half_lane() { return (uint32_t)lane_id() & (HALF - 1); }
__device__ inline uint32_t half_ballot(bool p) { return (uint32_t)(__ballot(p) >> ((uint32_t)lane_id() & HALF)); }
__device__ inline uint32_t half_below(uint32_t m) { return (uint32_t)__popc(m & ((1u << half_lane()) - 1u)); }
__device__ inline uint32_t half_shfl(uint32_t x, uint32_t src) { return __shfl(x, (int)src, HALF); }
__device__ inline uint32_t half_scan_incl(uint32_t x) {
  const uint32_t l = half_lane();
#pragma unroll
  for (int d = 1; d < (int)HALF; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, HALF);
    if (l >= (uint32_t)d) x += y;
  }
  return x;
}
// ascending sort of one value per lane within each half (bitonic network)
__device__ inline uint32_t half_sort(uint32_t x) {
  const uint32_t l = half_lane();
#pragma unroll
  for (uint32_t k2 = 2; k2 <= HALF; k2 <<= 1) {
#pragma unroll
    for (uint32_t j = k2 >> 1; j > 0; j >>= 1) {
      const uint32_t y = __shfl_xor(x, (int)j, HALF);
      const bool keep_min = ((l & k2) == 0) == ((l & j) == 0);
      x = keep_min ? (x < y ? x : y) : (x > y ? x : y);
    }
  }
  return x;
}
// a bitonic sequence within each half, ascending
__device__ inline uint32_t half_bitonic_merge(uint32_t x) {
  const uint32_t l = half_lane();
#pragma unroll
  for (uint32_t j = HALF / 2; j >= 1; j >>= 1) {
    const uint32_t y = __shfl_xor(x, (int)j, HALF);
    x = (l & j) == 0 ? (x < y ? x : y) : (x > y ? x : y);
  }
  return x;
}
// values below r (per lane) in the half's ascending set (INF32 above its size)
__device__ inline uint32_t half_count_below(uint32_t setv, uint32_t r) {
  uint32_t q = 0;
#pragma unroll
  for (uint32_t s = HALF / 2; s >= 1; s >>= 1) {
    const uint32_t val = half_shfl(setv, q + s - 1);
    if (val < r) q += s;
  }
  if (half_shfl(setv, q) < r) ++q;  // all 32 below r
  return q;
}

// Levels of at most this many survivors in both halves are decided by
// comparing all pairs instead of sorting (a level has 4 survivors on average
// on the large weighted workload, and most have none).
constexpr uint32_t PAIR_FEW = 12;
static_assert(PAIR_FEW <= HALF, "one survivor per lane");
// 6 waves per SIMD (80 registers, a few spilled) measured 2% faster than 5 on
// the large weighted workload; 8 (64 registers) slower
template <bool UNITW>
__global__ __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(6, 8)))
void k_ads_pairs(AdsArgs P, uint32_t D, const uint32_t *task_u, const uint32_t *task_sub, const uint32_t *task_slot,
                 RoundTot *tot, uint32_t *left, uint64_t *ts) {
  __shared__ __align__(16) uint32_t s_id[2][2 * HALF];  // survivors of the level (ranks, then ids)
  __shared__ uint32_t s_acc[2][2 * HALF];           // accepted ids, in id order
  __shared__ uint32_t s_set[2][HALF];               // the set at the level start
  __shared__ __align__(16) uint32_t s_r[2][HALF];   // chunk ranks
  const uint32_t lane = (uint32_t)lane_id(), h = lane >> 5, hl = lane & (HALF - 1);
  const uint32_t k = P.k;
  const uint64_t total = tot->tasks;
  const uint32_t Dm = D % P.NS, seen = *P.reach;
  if (ts && blockIdx.x == 0 && lane == 0) *ts = wall_clock64();
  for (uint64_t pi = blockIdx.x; 2 * pi < total; pi += gridDim.x) {
    const uint64_t t = 2 * pi + h;
    const bool live = t < total;
    uint32_t u = 0, slot = INF32;
    if (live) {
      u = task_u[t];
      slot = task_slot[t];
    }
    bool defer = live && slot != INF32;  // a slice of a split vertex
    bool act = live && !defer;           // half-uniform from here on
    // the task's row, set and count are loaded together: one wait
    const RankMap rm = rank_map(P.seg[seg_of(P.gid, u)]);
    const uint32_t cu = act ? P.cnt[u] : 0u;
    const uint32_t bkv = act && hl < k ? P.bk[(size_t)u * k + hl] : INF32;
    uint64_t a0 = 0, a1 = 0;
    if (act) {
      a0 = P.row_ptr[u];
      a1 = P.row_ptr[u + 1];
    }
    const uint32_t nset0 = cu < k ? cu : k;
    const uint32_t setv = hl < nset0 ? bkv : INF32;
    s_set[h][hl] = setv;
    wave_lds_sync();
    const bool full0 = nset0 == k;
    const uint32_t set_kth = half_shfl(setv, k - 1);
    const uint32_t T0 = full0 ? set_kth : INF32;
    uint32_t ns = 0;
    uint64_t examined = 0;
    // one candidate per lane: kept if below T0 and not in the start set
    auto offer = [&](bool valid, uint32_t r) {
      bool pass = act && valid && (!full0 || r < T0);
      if (!__ballot(pass)) return;
      // already in the set?  A search of fixed length over the padded set,
      // without branches (the lanes would leave a loop at different steps)
      uint32_t lo = 0;
#pragma unroll
      for (uint32_t s = HALF / 2; s >= 1; s >>= 1)
        if (s_set[h][lo + s - 1] < r) lo += s;
      if (lo < nset0 && s_set[h][lo] == r) pass = false;
      const uint32_t m = half_ballot(pass);
      const uint32_t np = (uint32_t)__popc(m);
      if (ns + np > 2 * HALF) {
        defer = true;  // more survivors than one chunk: the one-wave kernel
        act = false;
      } else {
        if (pass) s_id[h][ns + half_below(m)] = r;
        ns += np;
      }
      wave_lds_sync();
    };
    // one in-arc per lane: the level its tail committed at D - w
    auto batch = [&](bool valid, uint64_t a) {
      uint32_t v = 0, st = 0, cn = 0, r0 = INF32, r1 = INF32;
      if (act && valid) {
        v = P.col[a];
        const uint32_t wv = UNITW ? 1u : P.w[a];
        if (wv <= D) {
          const uint32_t src = D - wv;
          const uint32_t sl = Dm >= wv ? Dm - wv : Dm + P.NS - wv;
          const uint4 rec = P.lvl[(size_t)sl * P.n + v];
          if (rec.x == src && (!full0 || rec.y < T0)) {
            r0 = rec.y;
            r1 = rec.z;
            st = rec.w & 0xFFFFu;
            cn = full0 && r1 >= T0 ? 1u : rec.w >> 16;  // a second entry not below T0 ends the list
          }
        }
      }
      // long lists: one at a time per half, 32 entries per step; a level is
      // stored in increasing rank order, so once a rank reaches T0 the rest
      // of the list cannot enter
      uint32_t lm = half_ballot(act && cn >= LONG_LIST);
      while (__ballot(lm != 0)) {
        const bool has = lm != 0;
        const uint32_t j = has ? (uint32_t)(__ffs(lm) - 1) : 0u;
        if (has) lm &= lm - 1;
        const uint32_t vj = half_shfl(v, j), stj = half_shfl(st, j);
        uint32_t cnj = half_shfl(cn, j);
        if (!has) cnj = 0;
        const uint32_t *lst = P.sk_rank + (size_t)vj * P.cap + stj;
        bool go = has;
        for (uint32_t c0 = 0;; c0 += HALF) {
          const bool step = go && act && c0 < cnj;
          if (!__ballot(step)) break;
          const uint32_t i = c0 + hl;
          const bool ok = step && i < cnj;
          const uint32_t r = ok ? lst[i] : INF32;
          if (step) examined += cnj - c0 < HALF ? cnj - c0 : HALF;
          offer(ok, r);
          if (full0 && half_ballot(ok && r >= T0)) go = false;
        }
      }
      // short lists: flattened over the half, the owner lane of an entry found
      // by binary search; a level of one or two entries has its ranks in the
      // record
      const uint32_t cs = (act && cn < LONG_LIST) ? cn : 0u;
      const uint32_t incl = half_scan_incl(cs);
      const uint32_t tot = half_shfl(incl, HALF - 1);
      const uint32_t excl = incl - cs;
      examined += tot;
      for (uint32_t c0 = 0;; c0 += HALF) {
        const bool cm = act && c0 < tot;
        if (!__ballot(cm)) break;
        const uint32_t idx = c0 + hl;
        uint32_t pos = 0;  // owner lane: first lane whose inclusive count exceeds idx
#pragma unroll
        for (uint32_t s = HALF / 2; s >= 1; s >>= 1) {
          const uint32_t val = half_shfl(incl, pos + s - 1);
          if (val <= idx) pos += s;
        }
        const bool ok = cm && idx < tot;
        const uint32_t ov = half_shfl(v, pos), ost = half_shfl(st, pos), ocn = half_shfl(cs, pos);
        const uint32_t i = idx - half_shfl(excl, pos);
        const uint32_t o0 = half_shfl(r0, pos), o1 = half_shfl(r1, pos);
        uint32_t r = i == 0 ? o0 : o1;
        if (ok && ocn > 2) r = P.sk_rank[(size_t)ov * P.cap + ost + i];
        offer(ok, r);
      }
    };
    if (act && a1 - a0 > PAIR_ROW_MAX) {
      defer = true;  // a long row: the one-wave kernel
      act = false;
    }
    if (P.by_arc) {
      // only the arcs marked in this round's plane
      const uint32_t *plane = P.plane + (size_t)Dm * P.pw;
      const uint64_t w0 = a0 >> 5, w1 = (a1 + 31) >> 5;
      for (uint64_t wb = w0;; wb += HALF) {
        const bool more = act && wb < w1;
        if (!__ballot(more)) break;
        const uint64_t wi = wb + hl;
        uint32_t bits = 0;
        if (more && wi < w1) {
          bits = plane[wi];
          const uint64_t base = wi << 5;
          if (base < a0) bits &= ~0u << (uint32_t)(a0 - base);
          if (a1 - base < 32) bits &= (1u << (uint32_t)(a1 - base)) - 1u;
        }
        const uint32_t incl = half_scan_incl((uint32_t)__popc(bits));
        const uint32_t tot = half_shfl(incl, HALF - 1);
        for (uint32_t c0 = 0;; c0 += HALF) {
          const bool cm = act && more && c0 < tot;
          if (!__ballot(cm)) break;
          const uint32_t idx = c0 + hl;
          uint32_t pos = 0;  // word (lane) holding set bit idx
#pragma unroll
          for (uint32_t s = HALF / 2; s >= 1; s >>= 1) {
            const uint32_t val = half_shfl(incl, pos + s - 1);
            if (val <= idx) pos += s;
          }
          const bool ok = cm && idx < tot;
          const uint32_t src = ok ? pos : 0u;
          uint32_t x = half_shfl(bits, src);
          uint32_t kth = idx - (half_shfl(incl, src) - (uint32_t)__popc(x));
          uint32_t bit = 0;
#pragma unroll
          for (uint32_t sh = 16; sh >= 1; sh >>= 1) {
            const uint32_t cnt = (uint32_t)__popc(x & ((1u << sh) - 1u));
            if (kth >= cnt) {
              kth -= cnt;
              x >>= sh;
              bit += sh;
            }
          }
          batch(ok, ((wb + src) << 5) + bit);
        }
      }
    } else {
      for (uint64_t b = a0;; b += HALF) {
        const bool more = act && b < a1;
        if (!__ballot(more)) break;
        batch(more && b + hl < a1, b + hl);
      }
    }
    // The level's accepted ids (s_acc, in id order), their ranks ascending (ra,
    // then rb) and number (m), and the set they leave (set1, nset1).  nmax, the
    // larger half's survivors, picks the way; it is the same in every lane.
    uint32_t m = 0, nset1 = nset0, set1 = setv, ra = INF32, rb = INF32, x0 = INF32, x1 = INF32;
    uint32_t nmax = act ? ns : 0u;
    {
      const uint32_t o = __shfl_xor(nmax, (int)HALF, WAVE);
      nmax = __builtin_amdgcn_readfirstlane(nmax > o ? nmax : o);
    }
    if (nmax && nmax <= PAIR_FEW) {
      // Few survivors: every lane compares its own with the half's, four per
      // LDS read, instead of sorting.  A repeated id keeps its lowest lane.
      const uint32_t nc = act ? ns : 0u;
      uint32_t r = hl < nc ? s_id[h][hl] : INF32;
      wave_lds_sync();
      uint32_t x = hl < nc ? id_of(r, rm) : INF32;
      s_r[h][hl] = r;
      wave_lds_sync();
      bool dup = false;
      for (uint32_t j4 = 0; j4 < nmax; j4 += 4) {
        const uint4 v = *reinterpret_cast<const uint4 *>(&s_r[h][j4]);
        dup |= (v.x == r && j4 + 0 < hl) || (v.y == r && j4 + 1 < hl) || (v.z == r && j4 + 2 < hl) ||
               (v.w == r && j4 + 3 < hl);
      }
      wave_lds_sync();
      if (dup) x = r = INF32;
      s_r[h][hl] = r;
      s_id[h][hl] = x;
      wave_lds_sync();
      // accepted: fewer than k ranks below its own in the set or among the
      // candidates with a smaller id (none is in the set: the offers checked)
      const uint32_t q = half_count_below(setv, r);
      uint32_t cb = 0;
      for (uint32_t j4 = 0; j4 < nmax; j4 += 4) {
        const uint4 v = *reinterpret_cast<const uint4 *>(&s_r[h][j4]);
        const uint4 w = *reinterpret_cast<const uint4 *>(&s_id[h][j4]);
        cb += (v.x < r && w.x < x) ? 1u : 0u;
        cb += (v.y < r && w.y < x) ? 1u : 0u;
        cb += (v.z < r && w.z < x) ? 1u : 0u;
        cb += (v.w < r && w.w < x) ? 1u : 0u;
      }
      wave_lds_sync();
      const bool acc = x != INF32 && q + cb < k;
      m = (uint32_t)__popc(half_ballot(acc));
      if (!acc) x = r = INF32;
      s_r[h][hl] = r;
      s_id[h][hl] = x;
      wave_lds_sync();
      // each accepted one's place by id and by rank, and how many rank below
      // this lane's set element
      uint32_t pi = 0, pr = 0, add = 0;
      for (uint32_t j4 = 0; j4 < nmax; j4 += 4) {
        const uint4 v = *reinterpret_cast<const uint4 *>(&s_r[h][j4]);
        const uint4 w = *reinterpret_cast<const uint4 *>(&s_id[h][j4]);
        pi += (w.x < x ? 1u : 0u) + (w.y < x ? 1u : 0u) + (w.z < x ? 1u : 0u) + (w.w < x ? 1u : 0u);
        pr += (v.x < r ? 1u : 0u) + (v.y < r ? 1u : 0u) + (v.z < r ? 1u : 0u) + (v.w < r ? 1u : 0u);
        add += (v.x < setv ? 1u : 0u) + (v.y < setv ? 1u : 0u) + (v.z < setv ? 1u : 0u) + (v.w < setv ? 1u : 0u);
      }
      wave_lds_sync();
      if (acc) {
        s_acc[h][pi] = x;
        s_r[h][pr] = r;
        if (q + pr < k) s_set[h][q + pr] = r;
      }
      if (hl < nset0 && hl + add < k) s_set[h][hl + add] = setv;
      wave_lds_sync();
      nset1 = nset0 + m < k ? nset0 + m : k;
      set1 = hl < nset1 ? s_set[h][hl] : INF32;
      ra = hl < m ? s_r[h][hl] : INF32;
    } else if (nmax) {
    // Up to 64 survivors, sorted by id and decided in chunks of 32: each id
    // is accepted if fewer than k ranks below its own are in the set (which
    // by the second chunk holds the first chunk's accepted ranks) or among
    // the chunk's earlier candidates.  (Every shuffle here runs on all lanes:
    // a lane reads another only while that lane is active.)
    const bool two = nmax > HALF;  // some half has a second chunk
    uint32_t lo = half_sort((act && hl < ns) ? id_of(s_id[h][hl], rm) : INF32), hi = INF32;
    if (two) {
      const uint32_t xb = half_sort((act && HALF + hl < ns) ? id_of(s_id[h][HALF + hl], rm) : INF32);
      const uint32_t xbr = half_shfl(xb, HALF - 1 - hl);
      const uint32_t l2 = lo < xbr ? lo : xbr, h2 = lo < xbr ? xbr : lo;
      lo = half_bitonic_merge(l2);  // the 32 smallest ids
      hi = half_bitonic_merge(h2);  // the next 32
    }
    // one chunk against the set (setc, nsetc); prevx: the id before the chunk
    auto decide = [&](uint32_t x, uint32_t prevx, uint32_t setc, uint32_t nsetc, uint32_t &r_out) -> bool {
      uint32_t left = __shfl_up(x, 1, HALF);
      if (hl == 0) left = prevx;
      bool valid = act && x != INF32 && x != left;
      const uint32_t r = valid ? rank_of(x, rm) : INF32;
      const uint32_t q = half_count_below(setc, r);
      const uint32_t atq = half_shfl(setc, q < HALF - 1 ? q : HALF - 1);
      if (q < nsetc && atq == r) valid = false;
      const uint32_t vm = half_ballot(valid);
      s_r[h][hl] = valid ? r : INF32;
      wave_lds_sync();
      uint32_t top = vm ? 32u - (uint32_t)__clz(vm) : 0u;
      const uint32_t top2 = __shfl_xor(top, (int)HALF, WAVE);
      top = top > top2 ? top : top2;
      uint32_t cp = 0;
      for (uint32_t j4 = 0; j4 < top; j4 += 4) {
        const uint4 vv = *reinterpret_cast<const uint4 *>(&s_r[h][j4]);
        cp += (j4 + 0 < hl && vv.x < r) ? 1u : 0u;
        cp += (j4 + 1 < hl && vv.y < r) ? 1u : 0u;
        cp += (j4 + 2 < hl && vv.z < r) ? 1u : 0u;
        cp += (j4 + 3 < hl && vv.w < r) ? 1u : 0u;
      }
      wave_lds_sync();  // s_r is rewritten by the next chunk
      r_out = r;
      return valid && q + cp < k;
    };
    // the set after a chunk: the k smallest of the set and the chunk's
    // accepted ranks (xs, ascending)
    auto merge_set = [&](uint32_t setc, uint32_t xs) -> uint32_t {
      const uint32_t xrev = half_shfl(xs, HALF - 1 - hl);
      const uint32_t mm = half_bitonic_merge(setc < xrev ? setc : xrev);
      return hl < k ? mm : INF32;
    };
    uint32_t r1 = INF32;
    const bool acc1 = decide(lo, INF32, setv, nset0, r1);
    const uint32_t am1 = half_ballot(acc1);
    const uint32_t m1 = (uint32_t)__popc(am1);
    if (acc1) s_acc[h][half_below(am1)] = lo;
    const uint32_t xs1 = half_sort(acc1 ? r1 : INF32);
    set1 = merge_set(setv, xs1);
    nset1 = nset0 + m1 < k ? nset0 + m1 : k;
    ra = xs1;
    m = m1;
    if (two) {
      const uint32_t prevx = half_shfl(lo, HALF - 1);  // the first chunk is full when there is a second
      uint32_t r2 = INF32;
      const bool acc2 = decide(hi, prevx, set1, nset1, r2);
      const uint32_t am2 = half_ballot(acc2);
      const uint32_t m2 = (uint32_t)__popc(am2);
      if (acc2) s_acc[h][m1 + half_below(am2)] = hi;
      const uint32_t xs2 = half_sort(acc2 ? r2 : INF32);
      set1 = merge_set(set1, xs2);
      nset1 = nset1 + m2 < k ? nset1 + m2 : k;
      const uint32_t x2r = half_shfl(xs2, HALF - 1 - hl);
      const uint32_t l2 = xs1 < x2r ? xs1 : x2r, h2 = xs1 < x2r ? x2r : xs1;
      ra = half_bitonic_merge(l2);
      rb = half_bitonic_merge(h2);
      m = m1 + m2;
    }
    wave_lds_sync();  // s_acc is read below
    }
    x0 = half_shfl(ra, 0);
    x1 = half_shfl(ra, 1);
    bool committed = false;
    if (act && m) {
      if (cu + m > P.cap) {
        if (hl == 0) atomicOr(&P.status[0], 1u);
      } else {
        committed = true;
        const uint32_t tr = thr_row(P, u);
        if (tr != INF32) {
          uint32_t *trow = P.thr + (size_t)tr * P.cap + cu;
          if (hl < m) trow[hl] = rank_of(s_acc[h][hl], rm);
          if (HALF + hl < m) trow[HALF + hl] = rank_of(s_acc[h][HALF + hl], rm);
        }
        const size_t base = (size_t)u * P.cap + cu;
        if (hl < m) {
          P.sk_rank[base + hl] = ra;
          P.sk_dist[base + hl] = D;
        }
        if (HALF + hl < m) {
          P.sk_rank[base + HALF + hl] = rb;
          P.sk_dist[base + HALF + hl] = D;
        }
        if (hl < nset1) P.bk[(size_t)u * k + hl] = set1;
        if (hl == 0) {
          P.cnt[u] = cu + m;
          P.lvl[(size_t)(D % P.NS) * P.n + u] = level_record(D, x0, x1, cu, m);
        }
      }
    }
    // u's out-arcs are marked for round D + w
    if (committed) {
      // (an undirected graph's out-arcs are its in-arcs)
      const bool same = P.out_ptr == P.row_ptr;
      const uint64_t b0 = same ? a0 : P.out_ptr[u], b1 = same ? a1 : P.out_ptr[u + 1];
      for (uint64_t a = b0 + hl; a < b1; a += HALF) mark_arc<UNITW>(P, a, D, Dm, seen);
    }
    // tasks left to the one-wave kernel
    const bool lv = live && hl == 0 && defer;
    const uint64_t lm = __ballot(lv);
    if (lm) {
      uint32_t p0 = 0;
      if (lane == 0) p0 = (uint32_t)atomicAdd(&tot->left, (unsigned long long)__popcll(lm));
      p0 = __shfl(p0, 0, WAVE);
      if (lv) left[p0 + lanes_below(lm)] = (uint32_t)t;
    }
    if (live && hl == 0 && !defer) {
      ctr_add(P, CF_EXAMINED, examined);
      ctr_add(P, CF_SURVIVORS, ns);
      if (committed) ctr_add(P, CF_COMMITS, 1);
    }
    wave_lds_sync();  // the half buffers are rewritten by the next pair
  }
}

// One wave per task.  task_slot == INF32: the task is the whole vertex and
// commits; otherwise it leaves its kept set in scratch slot task_slot.  With
// tot (device) the grid strides over its task count (the host does not know
// it); otherwise one wave per task.  With `left`, just the tasks of that list
// (those the two-task kernel left).
template <bool UNITW, int KR, uint32_t SB>
__global__ __launch_bounds__(TASK_WPB * WAVE) __attribute__((amdgpu_waves_per_eu(SB <= ADS_SB / 2 ? 5 : 4)))
void k_ads_tasks(AdsArgs P, uint32_t D, const uint32_t *task_u, const uint32_t *task_sub, const uint32_t *task_slot,
                 uint32_t ntasks, const RoundTot *tot, uint32_t task_arcs, int sparse, int mark,
                 const uint32_t *left, uint64_t *ts) {
  __shared__ uint32_t lds_id[TASK_WPB][SB];
  __shared__ uint32_t lds_tmp[TASK_WPB][SB];
  __shared__ __align__(16) uint32_t lds_cnt[TASK_WPB][level_words(KR)];
  const int wv = threadIdx.x / WAVE;
  const uint64_t total = tot ? (left ? tot->left : tot->tasks) : ntasks;
  if (ts && blockIdx.x == 0 && threadIdx.x == 0) *ts = wall_clock64();
  for (uint64_t i = (uint64_t)blockIdx.x * TASK_WPB + wv; i < total; i += (uint64_t)gridDim.x * TASK_WPB) {
    const uint64_t item = left ? left[i] : i;
    ads_task<UNITW, KR, SB>(P, D, task_u[item], task_sub[item], task_slot[item], task_arcs, sparse, mark, lds_id[wv],
                            lds_tmp[wv], lds_cnt[wv]);
  }
}

// One block per split vertex: MERGE_WPB - 1 waves each prune the union of a
// strided share of its tasks' kept sets into a partial set in LDS, then the
// first wave prunes the union of the partial sets and commits.  The prune is
// associative and idempotent, so the grouping does not change the result;
// it shortens the chain of dependent work per hub, which bounds a round.
constexpr int MERGE_WPB = 8;
template <bool UNITW, int KR, uint32_t SB>
__global__ __launch_bounds__(MERGE_WPB * WAVE) void k_ads_merge(AdsArgs P, uint32_t D, const uint32_t *split_u,
                                                                const uint32_t *split_first,
                                                                const uint32_t *split_nt, uint32_t nsplit,
                                                                const RoundTot *tot, int mark, uint64_t *ts) {
  constexpr uint32_t NW = MERGE_WPB - 1;  // waves that build partial sets
  __shared__ uint32_t lds_id[MERGE_WPB][SB];
  __shared__ uint32_t lds_tmp[MERGE_WPB][SB];
  __shared__ __align__(16) uint32_t lds_cnt[MERGE_WPB][level_words(KR)];
  __shared__ uint32_t part_n[MERGE_WPB];
  __shared__ uint32_t s_mark;  // the item committed a level: its out-arcs are marked
  const int lane = lane_id();
  const int wv = threadIdx.x / WAVE;
  uint32_t *s_id = lds_id[wv];
  uint32_t *s_tmp = lds_tmp[wv];
  uint32_t *s_cnt = lds_cnt[wv];
  // the block's split vertices (uniform over the block): every wave reaches
  // both barriers of every item
  const uint64_t total = tot ? tot->splits : nsplit;
  if (ts && blockIdx.x == 0 && threadIdx.x == 0) *ts = wall_clock64();
  for (uint64_t item = blockIdx.x; item < total; item += gridDim.x) {
    const uint32_t u = split_u[item];
    const uint32_t first = split_first[item];
    const uint32_t nt = split_nt[item];
    Level<KR> L;
    level_init(P, u, L, s_cnt);
    if (wv > 0) {
      // tasks wv - 1, wv - 1 + NW, ...: a virtual list of `mine` tasks
      const uint32_t t0 = (uint32_t)wv - 1;
      const uint32_t mine = nt > t0 ? (nt - t0 + NW - 1) / NW : 0u;
      for (uint32_t g0 = 0; g0 < mine && !L.overflow; g0 += WAVE) {
        const uint32_t task = first + t0 + (g0 + lane) * NW;
        const uint32_t cn = g0 + lane < mine ? P.kept_cnt[task] : 0u;
        const uint32_t incl = wave_scan_incl(cn);
        const uint32_t tot = __shfl(incl, WAVE - 1, WAVE);
        const uint32_t excl = incl - cn;
        for (uint32_t c0 = 0; c0 < tot && !L.overflow; c0 += WAVE) {
          const uint32_t idx = c0 + lane;
          uint32_t pos = 0;
#pragma unroll
          for (uint32_t sh = 32; sh >= 1; sh >>= 1) {
            const uint32_t val = __shfl(incl, (int)(pos + sh - 1), WAVE);
            if (val <= idx) pos += sh;
          }
          const bool valid = idx < tot;
          const uint32_t oex = __shfl(excl, (int)pos, WAVE);
          const uint32_t otask = __shfl(task, (int)pos, WAVE);
          const uint32_t r = valid ? rank_of(P.kept[(size_t)otask * SB + (idx - oex)], L.rm) : INF32;
          level_offer<KR, SB>(P, L, valid, r, s_id, s_tmp, s_cnt);
        }
      }
      uint32_t m = 0;
      if (!L.overflow && L.ns) {
        KSet<KR> set = L.set0;
        uint32_t nset = L.nset0;
        m = prune_level(s_id, s_tmp, s_cnt, L.ns, P.k, L.rm, set, nset);  // partial set in s_tmp[0..m)
      }
      if (lane == 0) part_n[wv] = L.overflow ? INF32 : m;
    }
    __syncthreads();
    if (wv == 0) {
      for (int w = 1; w < MERGE_WPB && !L.overflow; ++w) {
        const uint32_t pn = part_n[w];
        if (pn == INF32) {
          L.overflow = true;
          break;
        }
        const uint32_t *part = lds_tmp[w];
        for (uint32_t c0 = 0; c0 < pn && !L.overflow; c0 += WAVE) {
          const bool valid = c0 + lane < pn;
          const uint32_t r = valid ? rank_of(part[c0 + lane], L.rm) : INF32;
          level_offer<KR, SB>(P, L, valid, r, s_id, s_tmp, s_cnt);
        }
      }
      bool committed = false;
      if (L.overflow) {
        if (lane == 0) atomicOr(&P.status[1], 1u);
      } else {
        committed = level_commit<UNITW, KR>(P, u, D, L, 0, s_id, s_tmp, s_cnt);
      }
      if (lane == 0) s_mark = committed && mark ? 1u : 0u;
    }
    // the partial sets are read before the next item rebuilds them; s_mark is
    // read by every wave before wave 0 passes the next item's first barrier
    __syncthreads();
    // a split vertex is a hub: every wave of the block marks a share of its out-arcs
    if (s_mark) mark_neighbours<UNITW>(P, u, D, (uint32_t)wv, MERGE_WPB);
  }
}

// Last pass over the rows with a threshold row (one wave per row): the row
// holds the sketch in canonical (distance, id) order (written at commit); it
// is copied into the sketch row, and entry j of the threshold row becomes
// T_j = the k-th smallest rank of entries 0..j-1 (0 for j < k, meaning 2^32).
// Every later entry ranks below its T_j (that is what membership of the
// sketch means), so each one enters the running bottom-k set and evicts its
// maximum, and no later entry is above that maximum.  Hence for a chunk C of
// up to 64 entries after a full set S, the threshold of the chunk's i-th
// entry is the (i+1)-th largest of S and C together, and the next S is the k
// smallest of them: one sort and a few bitonic merges per chunk.  The set is
// held in KR registers per lane (k <= 64 KR).
template <int KR>
__global__ __launch_bounds__(256) void k_hip_thresholds(uint32_t rows, const uint32_t *row_vertex, uint32_t cap,
                                                        uint32_t k, const uint32_t *cnt, uint32_t *sk_rank,
                                                        uint32_t *thr) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint64_t row = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  if (row >= rows) return;
  const uint32_t u = row_vertex ? row_vertex[row] : (uint32_t)row;
  const uint32_t c = cnt[u];
  uint32_t *rk = sk_rank + (size_t)u * cap;
  uint32_t *out = thr + (size_t)row * cap;  // canonical ranks in, thresholds out (each lane its own slots)
  const uint32_t k0 = c < k ? c : k;
  uint32_t first[KR];
#pragma unroll
  for (int g = 0; g < KR; ++g) {
    const uint32_t e = 64u * g + lane;
    first[g] = e < k0 ? out[e] : INF32;
    if (e < k0) {
      rk[e] = first[g];
      out[e] = 0;
    }
  }
  if (c <= k) return;
  // S: the first k entries, ascending, INF32 above k
  KSet<KR> S;
  if (KR == 1) {
    S.v[0] = wave_sort_reg(first[0]);
  } else {
    uint32_t hi;
    wave_merge2(wave_sort_reg(first[0]), wave_sort_reg(first[KR - 1]), S.v[0], hi);
    S.v[KR - 1] = hi;
  }
  for (uint32_t j0 = k; j0 < c; j0 += WAVE) {
    const uint32_t m = c - j0 < (uint32_t)WAVE ? c - j0 : (uint32_t)WAVE;
    const uint32_t mine = lane < m ? out[j0 + lane] : INF32;
    if (lane < m) rk[j0 + lane] = mine;
    const uint32_t ca = wave_sort_reg(mine);  // chunk ascending, INF32 above m
    // the 64 largest: S descending (0 past its size) against C ascending (0 below 64 - m)
    const uint32_t sd = kset_at(S, lane < k ? k - 1 - lane : 0u);
    const uint32_t cs = __shfl(ca, (int)(lane >= WAVE - m ? lane - (WAVE - m) : 0), WAVE);
    uint32_t top = (lane < k ? sd : 0u) > (lane >= WAVE - m ? cs : 0u) ? (lane < k ? sd : 0u)
                                                                        : (lane >= WAVE - m ? cs : 0u);
    top = wave_bitonic_merge(top, true);  // lane i: the (i+1)-th largest
    if (lane < m) out[j0 + lane] = top;
    kset_merge(S, ca, k);  // the k smallest of S and C
  }
}

// ---------------------------------------------------------------------------
// task lists
// ---------------------------------------------------------------------------
__global__ void k_task_count(const uint32_t *list, uint32_t count, const uint64_t *row_ptr, uint32_t task_arcs,
                             uint32_t *ntask, uint32_t *nslot, uint32_t *isplit) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t u = list[i];
  const uint64_t d = row_ptr[u + 1] - row_ptr[u];
  const uint32_t nt = d <= task_arcs ? 1u : (uint32_t)((d + task_arcs - 1) / task_arcs);
  ntask[i] = nt;
  nslot[i] = nt > 1 ? nt : 0u;
  isplit[i] = nt > 1 ? 1u : 0u;
}

__global__ void k_task_fill(const uint32_t *list, uint32_t count, const uint32_t *ntask, const uint64_t *task_off,
                            const uint64_t *slot_off, const uint64_t *split_off, uint32_t *task_u,
                            uint32_t *task_sub, uint32_t *task_slot, uint32_t *split_u, uint32_t *split_first,
                            uint32_t *split_nt) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t u = list[i];
  const uint32_t nt = ntask[i];
  const uint64_t t0 = task_off[i];
  for (uint32_t j = 0; j < nt; ++j) {
    task_u[t0 + j] = u;
    task_sub[t0 + j] = j;
    task_slot[t0 + j] = nt > 1 ? (uint32_t)(slot_off[i] + j) : INF32;
  }
  if (nt > 1) {
    const uint64_t s = split_off[i];
    split_u[s] = u;
    split_first[s] = (uint32_t)slot_off[i];
    split_nt[s] = nt;
  }
}

struct TaskList {
  uint32_t *task_u, *task_sub, *task_slot;
  uint32_t *split_u, *split_first, *split_nt;
  uint32_t ntasks = 0, nsplit = 0, nslots = 0;
  uint32_t task_arcs = TASK_ARCS;  // arcs per task of a split vertex
};

// scratch of build_tasks: 3 count arrays + 3 offset arrays
struct TaskScratch {
  uint32_t *ntask, *nslot, *isplit;
  uint64_t *toff, *soff, *poff;
};

// Start of a round run from marks: the task list of the vertices with a mark
// in plane D % NS.  A thread takes `ITEMS` vertices; rows of up to
// SCAN_WORDS words of the plane are read by their thread, longer ones by the
// wave, 512 words at a time up to the first mark.  Each block reserves the
// tile's tasks, kept slots and split records with one atomic per counter (the
// order of the tasks does not matter: the prune does not depend on it).
// The launch also clears the plane of round D - 1, which the marks of this
// round may reuse, and block 0 takes the reach of the earlier rounds.
//
// Reading every row pointer and one plane a round (8 B per vertex + 1 bit per
// arc, tens of us at 2^21 vertices and 65M arcs) replaced worklists, which
// every mark paid for: a read of the head's flag, and for a first mark two
// dependent atomics, the second on the slot's one count.  On a grid with
// weights 1..4 those counts bounded the round: 57 -> 17 us a round of the
// two-task kernel; on R-MAT 2^21 (weights 1..100) 708 -> 608 us.
// tot: this round's totals, zero before the launch.
constexpr uint32_t SCAN_WORDS = 8;
constexpr uint32_t BEGIN_T = 256;  // threads of a block: small blocks start sooner beside other streams' kernels
template <uint32_t ITEMS>
__global__ __launch_bounds__(BEGIN_T) void k_round_begin(AdsArgs P, uint32_t D, uint32_t task_arcs, RoundTot *tot,
                                                     uint32_t *task_u, uint32_t *task_sub, uint32_t *task_slot,
                                                     uint32_t *split_u, uint32_t *split_first, uint32_t *split_nt,
                                                     uint64_t *ts) {
  __shared__ uint32_t wsum[3][BEGIN_T / WAVE];
  __shared__ uint64_t base[3];
  __shared__ uint32_t s_reach[4];
  const uint32_t lane = (uint32_t)lane_id(), wv = threadIdx.x / WAVE;
  if (blockIdx.x == 0) {
    if (ts && threadIdx.x == 0) *ts = wall_clock64();
    static_assert(CTR_STRIPES == 4 * WAVE, "one stripe per thread of the first four waves");
    if (wv < 4) {
      const uint32_t r = wave_max_u32((uint32_t)P.ctr[(size_t)threadIdx.x * CTR_FIELDS + CF_REACH]);
      if (lane == 0) s_reach[wv] = r;
    }
    __syncthreads();
    if (threadIdx.x == 0)
      *P.reach = max(max(s_reach[0], s_reach[1]), max(s_reach[2], s_reach[3]));
  }
  const uint32_t *plane = P.plane + (size_t)(D % P.NS) * P.pw;
  {
    uint4 *old = reinterpret_cast<uint4 *>(P.plane + (size_t)((D - 1) % P.NS) * P.pw);  // pw is a multiple of 4
    const uint64_t nq = P.pw / 4, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq; i += stride)
      old[i] = make_uint4(0, 0, 0, 0);
  }
  constexpr uint32_t TILE = BEGIN_T * ITEMS;
  for (uint64_t b = (uint64_t)blockIdx.x * TILE; b < P.n; b += (uint64_t)gridDim.x * TILE) {
    uint64_t a0[ITEMS], a1[ITEMS];
    uint32_t nt[ITEMS], any[ITEMS];
    uint32_t c[3] = {0, 0, 0};
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      const uint64_t u = b + (uint64_t)j * BEGIN_T + threadIdx.x;
      a0[j] = u < P.n ? P.row_ptr[u] : 0;
      a1[j] = u < P.n ? P.row_ptr[u + 1] : 0;
    }
    // bits of the row [r0, r1) in its i-th word
    auto row_bits = [&](uint32_t i, uint64_t r0, uint64_t r1) -> uint32_t {
      const uint64_t p = ((r0 >> 5) + i) << 5;
      uint32_t x = plane[(r0 >> 5) + i];
      if (p < r0) x &= ~0u << (uint32_t)(r0 - p);
      if (r1 - p < 32) x &= (1u << (uint32_t)(r1 - p)) - 1u;
      return x;
    };
    auto row_words = [&](uint64_t r0, uint64_t r1) -> uint32_t {
      return r1 > r0 ? (uint32_t)(((r1 - 1) >> 5) - (r0 >> 5)) + 1u : 0u;
    };
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      any[j] = 0;
      if (!P.by_arc) {
        const uint64_t u = b + (uint64_t)j * BEGIN_T + threadIdx.x;
        any[j] = a1[j] > a0[j] ? (plane[u >> 5] >> (u & 31)) & 1u : 0u;
      } else {
        // every lane loads SCAN_WORDS words, its row's last one again past the
        // row's end: without branches the loads are in flight together
        const uint32_t nw = row_words(a0[j], a1[j]);
        const uint32_t last = nw ? nw - 1 : 0u;
        uint32_t x[SCAN_WORDS];
#pragma unroll
        for (uint32_t i = 0; i < SCAN_WORDS; ++i) x[i] = plane[(a0[j] >> 5) + (i < last ? i : last)];
        const uint32_t mf = ~0u << (uint32_t)(a0[j] & 31), ml = ~0u >> (uint32_t)((32 - (a1[j] & 31)) & 31);
#pragma unroll
        for (uint32_t i = 0; i < SCAN_WORDS; ++i) {
          if (i == 0) x[i] &= mf;
          if (i == last) x[i] &= ml;
          if (i <= last) any[j] |= x[i];
        }
        if (nw == 0) any[j] = 0;
      }
    }
    if (P.by_arc) {
#pragma unroll
      for (uint32_t j = 0; j < ITEMS; ++j) {
        uint64_t lm = __ballot(row_words(a0[j], a1[j]) > SCAN_WORDS);
        while (lm) {
          const int o = __ffsll((long long)lm) - 1;
          lm &= lm - 1;
          const uint64_t r0 = shfl_u64(a0[j], o), r1 = shfl_u64(a1[j], o);
          const uint32_t rw = row_words(r0, r1);
          uint64_t hit = 0;
          // 8 words per lane and step: an unmarked hub's row is read to its end
          for (uint32_t i0 = 0; i0 < rw && !hit; i0 += 8 * WAVE) {
            uint32_t x = 0;
#pragma unroll
            for (uint32_t q = 0; q < 8; ++q) {
              const uint32_t i = i0 + q * WAVE + lane;
              if (i < rw) x |= row_bits(i, r0, r1);
            }
            hit = __ballot(x != 0);
          }
          if ((int)lane == o) any[j] = hit != 0;
        }
      }
    }
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      const uint64_t d = a1[j] - a0[j];
      nt[j] = !any[j] ? 0u : d <= task_arcs ? 1u : (uint32_t)((d + task_arcs - 1) / task_arcs);
      c[0] += nt[j];
      c[1] += nt[j] > 1 ? nt[j] : 0u;
      c[2] += nt[j] > 1 ? 1u : 0u;
    }
    uint32_t incl[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      incl[q] = wave_scan_incl(c[q]);
      if (lane == WAVE - 1) wsum[q][wv] = incl[q];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
      const uint32_t q = threadIdx.x;
      uint32_t t = 0;
      for (uint32_t w = 0; w < BEGIN_T / WAVE; ++w) t += wsum[q][w];
      unsigned long long *dst = q == 0 ? &tot->tasks : (q == 1 ? &tot->slots : &tot->splits);
      base[q] = t ? atomicAdd(dst, (unsigned long long)t) : 0ull;
    }
    __syncthreads();
    uint64_t off[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      uint64_t o = base[q] + (incl[q] - c[q]);
      for (uint32_t w = 0; w < wv; ++w) o += wsum[q][w];
      off[q] = o;
    }
    __syncthreads();  // wsum and base are rewritten by the next tile
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      const uint32_t u = (uint32_t)(b + (uint64_t)j * BEGIN_T + threadIdx.x);
      for (uint32_t t = 0; t < nt[j]; ++t) {
        task_u[off[0] + t] = u;
        task_sub[off[0] + t] = t;
        task_slot[off[0] + t] = nt[j] > 1 ? (uint32_t)(off[1] + t) : INF32;
      }
      if (nt[j] > 1) {
        split_u[off[2]] = u;
        split_first[off[2]] = (uint32_t)off[1];
        split_nt[off[2]] = nt[j];
        off[1] += nt[j];
        off[2] += 1;
      }
      off[0] += nt[j];
    }
  }
}

// After a round, or a chunk of them: what the host reads back.
struct RoundInfo {
  uint64_t examined, commits, reach;  // cumulative counters
  uint64_t ts;                        // clock at the end
  uint32_t cap_over, buf_over;        // status bits
};
__global__ __launch_bounds__(256) void k_round_end(AdsArgs P, RoundInfo *out) {
  __shared__ uint64_t s_e[4], s_c[4];
  __shared__ uint32_t s_r[4];
  const uint64_t *f = P.ctr + (size_t)threadIdx.x * CTR_FIELDS;
  const uint64_t e = wave_sum_u64(f[CF_EXAMINED]), c = wave_sum_u64(f[CF_COMMITS]);
  const uint32_t r = wave_max_u32((uint32_t)f[CF_REACH]);
  const uint32_t wv = threadIdx.x / WAVE;
  if (lane_id() == 0) {
    s_e[wv] = e;
    s_c[wv] = c;
    s_r[wv] = r;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    *out = RoundInfo{s_e[0] + s_e[1] + s_e[2] + s_e[3], s_c[0] + s_c[1] + s_c[2] + s_c[3],
                     max(max(s_r[0], s_r[1]), max(s_r[2], s_r[3])), (uint64_t)wall_clock64(), P.status[0],
                     P.status[1]};
}

// in-degrees: out[0] scratch slots of the vertices a dense round splits,
// out[1] the largest (both zero before the launch)
__global__ __launch_bounds__(256) void k_degrees(uint32_t n, const uint64_t *row_ptr, unsigned long long *out) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t slots = 0, mx = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint64_t d = row_ptr[i + 1] - row_ptr[i];
    if (d > TASK_ARCS) slots += (d + TASK_ARCS - 1) / TASK_ARCS;
    mx = d > mx ? d : mx;
  }
  slots = wave_sum_u64(slots);
  mx = wave_max_u32((uint32_t)mx);  // a simple graph's degree is below n
  if (lane_id() == 0) {
    if (slots) atomicAdd(&out[0], (unsigned long long)slots);
    if (mx) atomicMax(&out[1], (unsigned long long)mx);
  }
}

// task_arcs >= TASK_ARCS: the scratch slots are sized for TASK_ARCS
static void build_tasks(Ctx &c, const Graph &g, const uint32_t *list, uint32_t count, uint32_t task_arcs,
                        TaskScratch &ts, TaskList &tl) {
  tl.ntasks = tl.nsplit = tl.nslots = 0;
  tl.task_arcs = task_arcs;
  if (count == 0) return;
  const uint32_t blocks = (uint32_t)ceil_div(count, 256);
  k_task_count<<<blocks, 256, 0, c.s>>>(list, count, g.in_ptr, task_arcs, ts.ntask, ts.nslot, ts.isplit);
  FL_LAUNCH_CHECK();
  scan_u32_to_u64(c, ts.ntask, ts.toff, count);
  scan_u32_to_u64(c, ts.nslot, ts.soff, count);
  scan_u32_to_u64(c, ts.isplit, ts.poff, count);
  k_task_fill<<<blocks, 256, 0, c.s>>>(list, count, ts.ntask, ts.toff, ts.soff, ts.poff, tl.task_u, tl.task_sub,
                                       tl.task_slot, tl.split_u, tl.split_first, tl.split_nt);
  FL_LAUNCH_CHECK();
  uint64_t h[3];
  FL_HIP(hipMemcpyAsync(&h[0], ts.toff + count, 8, hipMemcpyDeviceToHost, c.s));
  FL_HIP(hipMemcpyAsync(&h[1], ts.soff + count, 8, hipMemcpyDeviceToHost, c.s));
  FL_HIP(hipMemcpyAsync(&h[2], ts.poff + count, 8, hipMemcpyDeviceToHost, c.s));
  c.sync();
  tl.ntasks = (uint32_t)h[0];
  tl.nslots = (uint32_t)h[1];
  tl.nsplit = (uint32_t)h[2];
}

// Undirected graph: the position of the reverse (y, u) of each arc (u, y)
// (rows are sorted and free of repeats, validated).  The end with the larger
// degree (ties: the larger id) searches the other's row and writes both
// directions: half the searches of one per arc, each in the shorter row, and
// the tails come with the walk (R-MAT 2^22 13.3 -> 8 ms, 2^21 5.9 -> 3).
__global__ __launch_bounds__(256) void k_reverse_arcs(uint32_t n, uint64_t m, const uint64_t *row_ptr,
                                                      const uint32_t *col, uint32_t *out_to_in) {
  uint64_t b0, b1;
  wave_range(m, &b0, &b1);
  wave_arcs(n, row_ptr, b0, b1, [&](bool valid, uint64_t a, uint32_t u) {
    if (!valid) return;
    const uint64_t du = row_ptr[u + 1] - row_ptr[u];
    const uint32_t y = col[a];
    uint64_t lo = row_ptr[y], hi = row_ptr[y + 1];
    if (hi - lo > du || (hi - lo == du && y > u)) return;
    while (lo < hi) {  // u is there
      const uint64_t mid = lo + ((hi - lo) >> 1);
      if (col[mid] < u) lo = mid + 1;
      else hi = mid;
    }
    out_to_in[a] = (uint32_t)lo;
    out_to_in[lo] = (uint32_t)a;
  });
}

// list of vertices with at least one in-arc
__global__ void k_nonisolated_flags(uint32_t n, const uint64_t *row_ptr, uint32_t *flag) {
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) flag[i] = row_ptr[i + 1] > row_ptr[i] ? 1u : 0u;
}
__global__ void k_compact(uint32_t n, const uint32_t *flag, const uint64_t *pos, uint32_t *out) {
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && flag[i]) out[pos[i]] = (uint32_t)i;
}
// Compact the per-vertex sketches into CSR (one wave per vertex).
__global__ __launch_bounds__(256) void k_ads_export(uint32_t n, uint32_t cap, const uint32_t *cnt,
                                                    const uint64_t *off, const uint32_t *sk_rank,
                                                    const uint32_t *sk_dist, const uint32_t *thr,
                                                    uint32_t *o_rank, uint32_t *o_dist, uint32_t *o_thr) {
  const uint64_t u = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  if (u >= n) return;
  const uint32_t c = cnt[u];
  const uint64_t o = off[u];
  for (uint32_t i = lane_id(); i < c; i += WAVE) {
    o_rank[o + i] = sk_rank[u * cap + i];
    o_dist[o + i] = sk_dist[u * cap + i];
    o_thr[o + i] = thr[u * cap + i];
  }
}

uint32_t ads_capacity(uint32_t n, uint32_t k) {
  double lnr = std::log((double)n / (double)k);
  if (lnr < 0) lnr = 0;
  double mean = (double)k * (1.0 + lnr);
  double sd = std::sqrt((double)k * lnr + 1.0);
  double cap = std::ceil(mean + 8.0 * sd + 16.0);
  uint64_t c = ((uint64_t)cap + 15) & ~15ull;
  if (c > n) c = n;
  if (c < 1) c = 1;
  return (uint32_t)c;
}

size_t ads_scratch_bytes(uint32_t n, uint64_t m, uint32_t k, uint32_t NS) {
  const uint64_t slots = 2 * (m / TASK_ARCS) + 2;  // >= sum of ceil(deg/TASK_ARCS) over vertices with deg > TASK_ARCS
  const uint64_t tasks = (uint64_t)n + m / TASK_ARCS + 64;
  size_t b = 0;
  b += (size_t)n * k * 4;                  // bottom-k sets
  b += (size_t)NS * n * 16;                // per-slot level records
  b += (size_t)m * 4 + (size_t)NS * (m / 32 + n / 32 + 8) * 4;  // reverse-arc positions, planes (arcs or vertices)
  b += (size_t)slots * (ADS_SB * (k > 64 ? 2 : 1) + 1) * 4;   // kept sets of split tasks
  // two task lists, task scratch, the dense list: builds with weights hold one
  // list and nothing else of these; what they leave is room for the ordered
  // rows of the selection
  b += (size_t)tasks * 4 * 3 * 2 + (size_t)n * 4 * 3 * 2;
  b += (size_t)n * (4 * 3 + 8 * 3) + (size_t)n * 24;
  b += (size_t)tasks * 4;                  // tasks left by the two-task kernel
  b += (size_t)8 << 20;
  return b;
}

// Builds the sketches.  Returns FL_OK, or FL_ENOMEM / FL_ENOTIMPL.  The
// caller provides cap; on capacity overflow the call reports *need_more.
// Launches of the round kernels: the instance is picked by unit weights, the
// set registers of k and the survivor buffer of the build.
static void launch_tasks(hipStream_t s, uint32_t grid, bool unit, uint32_t k, uint32_t sb, const AdsArgs &P,
                         uint32_t D, const uint32_t *tu, const uint32_t *tsub, const uint32_t *tslot, uint32_t nt,
                         const RoundTot *tot, uint32_t task_arcs, int sparse, int mark, const uint32_t *left,
                         uint64_t *ts) {
#define FL_TASKS(U, K, S)                                                                                          \
  k_ads_tasks<U, K, S><<<grid, TASK_WPB * WAVE, 0, s>>>(P, D, tu, tsub, tslot, nt, tot, task_arcs, sparse, mark, \
                                                        left, ts)
  if (k > 64) {
    if (unit) FL_TASKS(true, 2, 2 * ADS_SB);
    else FL_TASKS(false, 2, 2 * ADS_SB);
  } else if (sb < ADS_SB) {
    if (unit) FL_TASKS(true, 1, ADS_SB / 2);
    else FL_TASKS(false, 1, ADS_SB / 2);
  } else {
    if (unit) FL_TASKS(true, 1, ADS_SB);
    else FL_TASKS(false, 1, ADS_SB);
  }
#undef FL_TASKS
}
static void launch_merge(hipStream_t s, uint32_t grid, bool unit, uint32_t k, uint32_t sb, const AdsArgs &P,
                         uint32_t D, const uint32_t *su, const uint32_t *sfirst, const uint32_t *snt, uint32_t ns,
                         const RoundTot *tot, int mark, uint64_t *ts) {
#define FL_MERGE(U, K, S) \
  k_ads_merge<U, K, S><<<grid, MERGE_WPB * WAVE, 0, s>>>(P, D, su, sfirst, snt, ns, tot, mark, ts)
  if (k > 64) {
    if (unit) FL_MERGE(true, 2, 2 * ADS_SB);
    else FL_MERGE(false, 2, 2 * ADS_SB);
  } else if (sb < ADS_SB) {
    if (unit) FL_MERGE(true, 1, ADS_SB / 2);
    else FL_MERGE(false, 1, ADS_SB / 2);
  } else {
    if (unit) FL_MERGE(true, 1, ADS_SB);
    else FL_MERGE(false, 1, ADS_SB);
  }
#undef FL_MERGE
}

// sb: survivor buffer (ADS_SB / 2 or ads_full_sb(k)).  *buf_over: a level
// overflowed it (the caller restarts with a larger one).
static int ads_run(Ctx &c, const Graph &g, const AdsConfig &cfg, AdsOut &o, bool *need_more, uint32_t sb,
                   bool *buf_over) {
  const uint32_t n = g.n, k = cfg.k, cap = o.cap;
  const uint32_t W = g.w ? g.max_w : 1u;
  const uint32_t NS = W + 1;
  const bool unit = g.w == nullptr;
  *need_more = false;
  *buf_over = false;

  AdsArgs P{};
  P.n = n;
  P.k = k;
  P.cap = cap;
  P.NS = NS;
  P.gid = cfg.gid;
  P.seg = cfg.seg;
  P.row_ptr = g.in_ptr;
  P.col = g.in_col;
  P.w = g.in_w;
  P.out_ptr = g.row_ptr;
  P.out_col = g.col;
  P.out_w = g.w;
  P.sk_rank = o.sk_rank;
  P.sk_dist = o.sk_dist;
  P.bk = c.arena->get<uint32_t>((size_t)n * k);
  P.cnt = o.cnt;
  P.lvl = c.arena->get<uint4>((size_t)NS * n);
  P.ctr = c.arena->get<uint64_t>((size_t)CTR_STRIPES * CTR_FIELDS);
  P.dbg = std::getenv("FL_DEBUG") ? 1u : 0u;
  P.thr = o.thr;
  P.thr_idx = o.thr ? cfg.thr_idx : nullptr;
  // marks by arc where arc positions fit 32 bits, by vertex otherwise
  // (FL_TEST_MARK_VERTICES: always by vertex, so that the tests run both)
  P.by_arc = g.m < 0xFFFFFFFFull && !std::getenv("FL_TEST_MARK_VERTICES") ? 1u : 0u;
  P.pw = (((P.by_arc ? g.m : (uint64_t)n) / 32 + 2) + 3) & ~3ull;
  P.plane = c.arena->get<uint32_t>((size_t)NS * P.pw);
  fill_u32(c, P.plane, (size_t)NS * P.pw, 0);
  P.out_to_in = nullptr;
  if (P.by_arc && g.m) {
    if (g.out_to_in) {
      P.out_to_in = g.out_to_in;
    } else {
      uint32_t *o2i = c.arena->get<uint32_t>(g.m);
      const uint32_t blocks = (uint32_t)std::min<uint64_t>(ceil_div(g.m, 256), 4096);
      k_reverse_arcs<<<blocks, 256, 0, c.s>>>(n, g.m, g.row_ptr, g.col, o2i);
      FL_LAUNCH_CHECK();
      P.out_to_in = o2i;
    }
  }
  fill_u64(c, reinterpret_cast<uint64_t *>(P.lvl), (size_t)NS * n * 2, INF64);  // no level anywhere
  // small device state of the rounds, zeroed together: counters, status, the
  // totals of a chunk's rounds, clocks, what the host reads back
  constexpr uint32_t RCHUNK = 16;
  struct RoundState {
    RoundTot tot[RCHUNK];
    uint64_t ts[RCHUNK][3];  // clocks at the start of a round, of its kernels, of its merge
    RoundInfo info;
    uint64_t deg[2];
    uint32_t status[2], reach, pad;
  };
  RoundState *rs = c.arena->get<RoundState>(1);
  fill_u64(c, P.ctr, (size_t)CTR_STRIPES * CTR_FIELDS, 0);
  fill_u32(c, reinterpret_cast<uint32_t *>(rs), sizeof(RoundState) / 4, 0);
  P.status = rs->status;
  P.reach = &rs->reach;
  // Round 0 marks every arc: the farthest mark is the largest weight.  With
  // the dense list the rounds end when nothing changed; the reach is not kept
  // (no mark exceeds INF32).
  const bool dense_ok = unit && !(cfg.flags & FL_FLAG_NO_DENSE);
  if (g.m) {
    fill_u64(c, P.ctr + CF_REACH, 1, dense_ok ? INF32 : W);
    fill_u32(c, P.reach, 1, dense_ok ? INF32 : W);
  }

  // scratch slots: enough for every vertex split at once
  uint64_t max_deg = 0;
  {
    k_degrees<<<(uint32_t)std::min<uint64_t>(ceil_div(n, 256), 1024), 256, 0, c.s>>>(
        n, g.in_ptr, reinterpret_cast<unsigned long long *>(rs->deg));
    FL_LAUNCH_CHECK();
    c.fetch(rs->deg, sizeof(rs->deg));
    const uint64_t slots = c.h_status[0] + 1;
    max_deg = c.h_status[1];
    P.kept = c.arena->get<uint32_t>(slots * sb);
    P.kept_cnt = c.arena->get<uint32_t>(slots);
  }
  // task lists (sized for a list of all vertices) and the dense list's scratch
  const uint64_t max_tasks = (uint64_t)n + g.m / TASK_ARCS + 64;
  TaskScratch ts{};
  if (dense_ok) {
    ts.ntask = c.arena->get<uint32_t>(n);
    ts.nslot = c.arena->get<uint32_t>(n);
    ts.isplit = c.arena->get<uint32_t>(n);
    ts.toff = c.arena->get<uint64_t>((size_t)n + 1);
    ts.soff = c.arena->get<uint64_t>((size_t)n + 1);
    ts.poff = c.arena->get<uint64_t>((size_t)n + 1);
  }
  TaskList tl_dense, tl;
  auto alloc_list = [&](TaskList &t) {
    t.task_u = c.arena->get<uint32_t>(max_tasks);
    t.task_sub = c.arena->get<uint32_t>(max_tasks);
    t.task_slot = c.arena->get<uint32_t>(max_tasks);
    t.split_u = c.arena->get<uint32_t>(n);
    t.split_first = c.arena->get<uint32_t>(n);
    t.split_nt = c.arena->get<uint32_t>(n);
  };
  alloc_list(tl);

  // dense list: vertices with at least one arc, and its static task list
  uint32_t n_dense = 0;
  if (dense_ok) {
    uint32_t *fl = c.arena->get<uint32_t>(n);
    uint64_t *pos = c.arena->get<uint64_t>((size_t)n + 1);
    uint32_t *dense = c.arena->get<uint32_t>(n);
    k_nonisolated_flags<<<(uint32_t)ceil_div(n, 256), 256, 0, c.s>>>(n, g.in_ptr, fl);
    FL_LAUNCH_CHECK();
    scan_u32_to_u64(c, fl, pos, n);
    k_compact<<<(uint32_t)ceil_div(n, 256), 256, 0, c.s>>>(n, fl, pos, dense);
    FL_LAUNCH_CHECK();
    FL_HIP(hipMemcpyAsync(c.h_status, pos + n, 8, hipMemcpyDeviceToHost, c.s));
    c.sync();
    n_dense = (uint32_t)c.h_status[0];
    alloc_list(tl_dense);
    build_tasks(c, g, dense, n_dense, TASK_ARCS, ts, tl_dense);
  }
  // a round marks (so that the next one runs from marks) once the previous
  // round changed at most a quarter of the dense list
  const uint64_t dense_threshold = (uint64_t)n_dense / 4;

  // round 0
  bool mark = !dense_ok || n_dense <= dense_threshold;
  {
    uint64_t blocks = ceil_div((uint64_t)n * WAVE, 256);
    if (unit) k_ads_init<true><<<(uint32_t)blocks, 256, 0, c.s>>>(P, mark ? 1 : 0);
    else k_ads_init<false><<<(uint32_t)blocks, 256, 0, c.s>>>(P, mark ? 1 : 0);
    FL_LAUNCH_CHECK();
  }
  bool sparse = mark;  // mode of round 1
  o.kernel_ms = 0.0;
  o.merge_ms = 0.0;
  o.launches = 0;
  double ms_per_tick = 0.0;  // of the clock the kernels read
  if (c.timing) {
    int dev = 0, khz = 0;
    FL_HIP(hipGetDevice(&dev));
    FL_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    ms_per_tick = khz > 0 ? 1.0 / khz : 0.0;
  }
  const bool pairs = k <= HALF && !dense_ok;  // the set of a level fits one half of a wave
  const uint32_t sparse_arcs = P.by_arc ? TASK_ARCS_FLAGGED : TASK_ARCS_SPARSE;
  const bool splits = max_deg > sparse_arcs;  // some row is split in rounds run from marks
  const uint32_t GT = (uint32_t)std::min<uint64_t>(max_tasks, 65536);  // one-wave blocks striding over tasks
  const uint32_t GL = (uint32_t)std::min<uint64_t>(max_tasks, 8192);   // the same over the tasks left
  const uint32_t GM = (uint32_t)std::min<uint64_t>(n, 2048);           // merge blocks striding over hubs
  const uint32_t GP = (uint32_t)std::min<uint64_t>(ceil_div(max_tasks, 2), 65536);  // two-task waves
  uint32_t *left = pairs ? c.arena->get<uint32_t>(max_tasks) : nullptr;
  // one round run from marks; r: its place in the chunk
  auto sparse_round = [&](uint32_t D, uint32_t r, int marks) {
    RoundTot *tot = &rs->tot[r];
    uint64_t *ts = c.timing ? rs->ts[r] : nullptr;
    auto tsp = [&](int i) { return ts ? ts + i : nullptr; };
#define FL_BEGIN(ITEMS)                                                                                       \
  k_round_begin<ITEMS><<<(uint32_t)std::min<uint64_t>(ceil_div(n, BEGIN_T * ITEMS), 2048), BEGIN_T, 0, c.s>>>( \
      P, D, sparse_arcs, tot, tl.task_u, tl.task_sub, tl.task_slot, tl.split_u, tl.split_first, tl.split_nt, \
      tsp(0))
    if (n >= (1u << 18)) FL_BEGIN(4);
    else FL_BEGIN(1);
#undef FL_BEGIN
    FL_LAUNCH_CHECK();
    if (pairs) {
      // k <= 32: two small tasks per wave first, then the one-wave kernel on the rest
      if (unit)
        k_ads_pairs<true><<<GP, WAVE, 0, c.s>>>(P, D, tl.task_u, tl.task_sub, tl.task_slot, tot, left, tsp(1));
      else
        k_ads_pairs<false><<<GP, WAVE, 0, c.s>>>(P, D, tl.task_u, tl.task_sub, tl.task_slot, tot, left, tsp(1));
      FL_LAUNCH_CHECK();
    }
    launch_tasks(c.s, pairs ? GL : GT, unit, k, sb, P, D, tl.task_u, tl.task_sub, tl.task_slot, 0, tot, sparse_arcs, 1,
                 marks, left, pairs ? nullptr : tsp(1));
    FL_LAUNCH_CHECK();
    if (splits) {
      launch_merge(c.s, GM, unit, k, sb, P, D, tl.split_u, tl.split_first, tl.split_nt, 0, tot, marks, tsp(2));
      FL_LAUNCH_CHECK();
    }
  };
  // host copy of the rounds' state (waits)
  std::vector<uint64_t> hbuf(sizeof(RoundState) / 8);
  const RoundState &h = *reinterpret_cast<const RoundState *>(hbuf.data());
  auto round_end = [&]() {
    k_round_end<<<1, CTR_STRIPES, 0, c.s>>>(P, &rs->info);
    FL_LAUNCH_CHECK();
    c.fetch(rs, sizeof(RoundState));
    std::memcpy(hbuf.data(), c.h_status, sizeof(RoundState));
  };
  // device time of round r's kernels and merge (next: clock at the next start)
  auto add_times = [&](uint32_t r, uint64_t next, bool merged) {
    o.launches += 1;
    if (!c.timing) return;
    const uint64_t kend = merged ? h.ts[r][2] : next;
    o.kernel_ms += (double)(kend - h.ts[r][1]) * ms_per_tick;
    if (merged) o.merge_ms += (double)(next - kend) * ms_per_tick;
  };
  static_assert(sizeof(RoundState) <= 4096 * 8, "fits the host status words");
  uint32_t rounds = 0;
  if (!dense_ok) {
    // Every round runs from marks.  Rounds are launched RCHUNK at a time
    // with their task lists built on the device (nothing goes to the host in
    // between); the round kernels stride over the device-side totals.  Rounds
    // after the last one with a mark find no task and change nothing.
    for (uint32_t D0 = 1;; D0 += RCHUNK) {
      if (D0 > 1) fill_u32(c, reinterpret_cast<uint32_t *>(rs->tot), sizeof(rs->tot) / 4, 0);
      for (uint32_t r = 0; r < RCHUNK; ++r) sparse_round(D0 + r, r, 1);
      round_end();
      if (h.info.cap_over) {
        *need_more = true;
        return FL_OK;
      }
      if (h.info.buf_over) {
        *buf_over = true;
        return FL_OK;
      }
      // every round of the chunk launched the round kernel (those past the
      // last one with work exit at once): all are counted and timed, as a
      // kernel trace sees them
      for (uint32_t r = 0; r < RCHUNK; ++r) {
        add_times(r, r + 1 < RCHUNK ? h.ts[r + 1][0] : h.info.ts, splits);
        if (h.tot[r].tasks) rounds = D0 + r;  // every vertex with a mark makes a task
      }
      if (rounds == 0) rounds = 1;
      if (std::getenv("FL_DEBUG"))
        std::fprintf(stderr, "[fl] rounds %u-%u: tasks of the first %llu, left to the one-wave kernel %llu, reach %llu\n",
                     D0, D0 + RCHUNK - 1, h.tot[0].tasks, h.tot[0].left, (unsigned long long)h.info.reach);
      if (h.info.reach < (uint64_t)D0 + RCHUNK) break;  // no mark beyond this chunk
      // a settled entry is at most (n-1) max_w away, and its vertex marks its
      // neighbours once more: marks beyond n max_w mean a bug
      if ((uint64_t)D0 > (uint64_t)n * W) return FL_EHIP;
    }
  }
  uint64_t active_prev = n;
  uint64_t commits_prev = 0;  // commits counted before this round
  bool was_sparse = false;
  for (uint32_t D = 1; dense_ok; ++D) {
    // marking decision for this round (decides the mode of the next one)
    mark = active_prev <= dense_threshold;
    bool merged = sparse && splits;
    if (sparse) {
      fill_u32(c, reinterpret_cast<uint32_t *>(rs->tot), sizeof(RoundTot) / 4, 0);
      sparse_round(D, 0, mark ? 1 : 0);
    } else if (tl_dense.ntasks) {
      const TaskList &T = tl_dense;
      // the marks of a round run from them, which this round's may join
      if (was_sparse) fill_u32(c, P.plane + (size_t)((D - 1) % NS) * P.pw, P.pw, 0);
      launch_tasks(c.s, (uint32_t)ceil_div(T.ntasks, TASK_WPB), unit, k, sb, P, D, T.task_u, T.task_sub, T.task_slot,
                   T.ntasks, nullptr, T.task_arcs, 0, mark ? 1 : 0, nullptr, c.timing ? &rs->ts[0][1] : nullptr);
      FL_LAUNCH_CHECK();
      if (T.nsplit) {
        merged = true;
        // one block of MERGE_WPB waves per split vertex
        launch_merge(c.s, T.nsplit, unit, k, sb, P, D, T.split_u, T.split_first, T.split_nt, T.nsplit, nullptr,
                     mark ? 1 : 0, c.timing ? &rs->ts[0][2] : nullptr);
        FL_LAUNCH_CHECK();
      }
    }
    ++rounds;
    round_end();
    if (h.info.cap_over) {
      *need_more = true;
      return FL_OK;
    }
    if (h.info.buf_over) {
      *buf_over = true;
      return FL_OK;
    }
    if (sparse ? h.tot[0].tasks != 0 : tl_dense.ntasks != 0) add_times(0, h.info.ts, merged);
    const uint64_t active = h.info.commits - commits_prev;  // vertices that changed this round
    commits_prev = h.info.commits;
    if (std::getenv("FL_DEBUG"))
      std::fprintf(stderr, "[fl] round %u: %s, %llu tasks, %llu changed, examined(cum) %.3fG\n", D,
                   sparse ? "sparse" : "dense", sparse ? h.tot[0].tasks : (unsigned long long)tl_dense.ntasks,
                   (unsigned long long)active, h.info.examined / 1e9);
    if (active == 0) break;
    active_prev = active;
    was_sparse = sparse;
    sparse = mark;
    // a settled entry is at most (n-1) max_w away: more rounds mean a bug
    if ((uint64_t)D > (uint64_t)(n - 1) * W + 2) return FL_EHIP;
  }
  o.rounds = rounds;
  o.relax_exec = h.info.examined;
  return FL_OK;
}

int ads_build(Ctx &c, const Graph &g, const AdsConfig &cfg, AdsOut &o) {
  if (cfg.k == 0) return FL_EINVAL;
  if (cfg.k > MAX_K) return FL_ENOTIMPL;
  if (g.w && g.max_w > MAX_W) return FL_ENOTIMPL;
  if (!g.in_ptr) return FL_EINVAL;  // the in-arc view is set by set_in_arcs
  uint32_t cap = ads_capacity(cfg.n_cap ? cfg.n_cap : g.n, cfg.k);
  // half the survivor buffer for k <= 32 (FL_TEST_SMALL_SURVIVOR_BUFFER: for
  // k <= 64 too, so that tests reach the restart below on small graphs)
  const uint32_t small_k = std::getenv("FL_TEST_SMALL_SURVIVOR_BUFFER") ? 64u : 32u;
  uint32_t sb = cfg.k <= small_k ? ADS_SB / 2 : ads_full_sb(cfg.k);
  for (int attempt = 0; attempt < 7; ++attempt) {
    if (cap > MAX_CAP) return FL_ENOTIMPL;
    const size_t mark = c.arena->used();
    o.cap = cap;
    o.sk_rank = c.arena->get<uint32_t>((size_t)g.n * cap);
    o.sk_dist = c.arena->get<uint32_t>((size_t)g.n * cap);
    o.cnt = c.arena->get<uint32_t>(g.n);
    const uint32_t thr_rows = cfg.thr_rows;
    o.thr = thr_rows ? c.arena->get<uint32_t>((size_t)thr_rows * cap) : nullptr;
    o.thr_idx = cfg.thr_idx;
    const size_t after_out = c.arena->used();
    bool more = false, buf_over = false;
    int rc = ads_run(c, g, cfg, o, &more, sb, &buf_over);
    if (rc != FL_OK) return rc;
    c.arena->rewind(after_out);
    if (buf_over) {
      // a level overflowed the survivor buffer: again with the full one
      if (sb >= ads_full_sb(cfg.k)) return FL_ENOMEM;
      if (std::getenv("FL_DEBUG")) std::fprintf(stderr, "[fl] sketches: survivor buffer %u overflowed\n", sb);
      sb = ads_full_sb(cfg.k);
      c.arena->rewind(mark);
      continue;
    }
    if (std::getenv("FL_DEBUG"))
      std::fprintf(stderr, "[fl] sketches: cap %u rounds %u overflow %d\n", cap, o.rounds, (int)more);
    if (!more) {
      // rows without a threshold row keep rank order within a level: only
      // the rows of facilities (every row for fl_ads_build) are read later
      if (o.thr && thr_rows) {
        const uint32_t tgrid = (uint32_t)ceil_div((uint64_t)thr_rows * WAVE, 256);
        if (cfg.k <= 64)
          k_hip_thresholds<1><<<tgrid, 256, 0, c.s>>>(thr_rows, cfg.thr_rows_vertex, cap, cfg.k, o.cnt, o.sk_rank, o.thr);
        else
          k_hip_thresholds<2><<<tgrid, 256, 0, c.s>>>(thr_rows, cfg.thr_rows_vertex, cap, cfg.k, o.cnt, o.sk_rank, o.thr);
        FL_LAUNCH_CHECK();
      }
      return FL_OK;
    }
    uint64_t nc = (uint64_t)cap * 3 / 2 + 16;
    const uint32_t nmax = cfg.n_cap ? cfg.n_cap : g.n;
    if (nc > nmax) nc = nmax;
    if (nc == cap) return FL_ENOMEM;
    c.arena->rewind(mark);
    cap = (uint32_t)nc;
  }
  return FL_ENOMEM;
}

int ads_export(Ctx &c, const Graph &g, const AdsOut &o, uint64_t *off, uint32_t *rank, uint32_t *dist,
               uint32_t *thr) {
  k_ads_export<<<(uint32_t)ceil_div((uint64_t)g.n * WAVE, 256), 256, 0, c.s>>>(
      g.n, o.cap, o.cnt, off, o.sk_rank, o.sk_dist, o.thr, rank, dist, thr);
  FL_LAUNCH_CHECK();
  return FL_OK;
}

}  // namespace fl
