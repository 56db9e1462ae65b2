// fl_graph.hip -- graph-level kernels: input validation, fills, scans,
// reductions, and the frontier Bellman-Ford used for the multi-source
// shortest-path sweeps (gamma, distance to the open set, assignment).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "fl_common.h"
#include "fl_frontier.h"

namespace fl {

// ---------------------------------------------------------------------------
// fills
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_fill(T *p, uint64_t n, T v) {
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}
template <class T>
static void fill_t(Ctx &c, T *p, uint64_t n, T v) {
  if (n == 0) return;
  uint64_t blocks = ceil_div(n, 256);
  if (blocks > 65536) blocks = 65536;
  k_fill<T><<<(uint32_t)blocks, 256, 0, c.s>>>(p, n, v);
  FL_LAUNCH_CHECK();
}
void fill_u32(Ctx &c, uint32_t *p, uint64_t n, uint32_t v) { fill_t(c, p, n, v); }
void fill_u64(Ctx &c, uint64_t *p, uint64_t n, uint64_t v) { fill_t(c, p, n, v); }
void fill_u8(Ctx &c, uint8_t *p, uint64_t n, uint8_t v) { fill_t(c, p, n, v); }
void fill_f64(Ctx &c, double *p, uint64_t n, double v) { fill_t(c, p, n, v); }

// ---------------------------------------------------------------------------
// Validation (a simple undirected graph as a symmetric CSR, Sec. 3.1; a
// directed graph gives its out-arcs and skips the symmetry test).  A lane per
// arc, equal ranges of arcs to every wave; row bounds and costs by a lane per
// vertex.  Bound by the reads of the searches (row bounds and columns of the
// other end): R-MAT 2^22, 127 million arcs, 8.0 ms; a wave per vertex, which
// ends with one wave in the longest row, 19.4 (R-MAT 2^21 11.2 -> 4.4, 2^18 1.6 ->
// 0.37, 64 graphs of 500 to 200,000 vertices 3.5 -> 1.3).  err bits: 1 =
// structural error.  Also reduces max weight and max facility
// cost.  Each block reduces its waves' results in LDS and adds them to
// stripe blockIdx.x % stripes, one 128-byte line per stripe: v32[32 s + 0]
// error bits, [32 s + 1] max weight, [32 s + 2] max cost; lt[16 s + 0]
// leading arcs, [16 s + 1] trailing arcs.
//
// Symmetry: an arc u -> v is "leading" when u has the larger degree (ties:
// the larger id).  Only leading arcs look up their reverse, by binary search
// in the row of the smaller end, and must find it with the same weight; the
// leading and trailing arcs are counted.  The reverse of a leading arc is a
// trailing arc, distinct arcs have distinct reverses, so equal counts mean
// every trailing arc is the reverse of a leading one: the arc set is
// symmetric with equal weights.
// ---------------------------------------------------------------------------
__device__ inline bool find_arc(const uint64_t *row_ptr, const uint32_t *col, uint64_t m, uint32_t u,
                                uint32_t v, uint64_t *pos) {
  uint64_t lo = row_ptr[u], hi = row_ptr[u + 1];
  const uint64_t end = hi;
  if (hi > m || lo > hi) return false;  // malformed row: never read past col[m-1]
  while (lo < hi) {
    uint64_t mid = lo + ((hi - lo) >> 1);
    if (col[mid] < v) lo = mid + 1;
    else hi = mid;
  }
  *pos = lo;
  return lo < end && col[lo] == v;
}

constexpr uint32_t VAL_STRIDE32 = 32, VAL_STRIDE64 = 16;  // one 128-byte line per stripe
constexpr uint32_t VAL_BLOCKS = 4096;                      // grid of a validation launch (at most)
__global__ __launch_bounds__(256) void k_validate(uint32_t n, uint64_t m, const uint64_t *row_ptr,
                                                  const uint32_t *col, const uint32_t *w,
                                                  const uint32_t *fac_cost, uint32_t *v32, uint32_t stripes,
                                                  uint32_t directed, unsigned long long *lt) {
  __shared__ uint32_t sh_bad[256 / WAVE], sh_mw[256 / WAVE], sh_mc[256 / WAVE];
  __shared__ unsigned long long sh_lead[256 / WAVE], sh_trail[256 / WAVE];
  const int lane = lane_id();
  const uint32_t wv = threadIdx.x / WAVE;
  uint32_t bad = 0, mw = 0, mc = 0;
  uint64_t nlead = 0, ntrail = 0;
  for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t a0 = row_ptr[u], a1 = row_ptr[u + 1];
    if (a1 < a0 || a1 > m) bad = 1;
    if (fac_cost) {
      const uint32_t cst = fac_cost[u];
      if (cst != FL_NOT_FACILITY && cst > mc) mc = cst;
    }
  }
  uint64_t b0, b1;
  wave_range(m, &b0, &b1);
  wave_arcs(n, row_ptr, b0, b1, [&](bool valid, uint64_t a, uint32_t u) {
    if (!valid) return;
    const uint64_t a0 = row_ptr[u], du = row_ptr[u + 1] - a0;
    const uint32_t v = col[a];
    const uint32_t wa = w ? w[a] : 1u;
    if (v >= n || v == u || wa == 0) { bad = 1; return; }
    if (a > a0 && col[a - 1] >= v) { bad = 1; return; }
    if (!directed) {
      const uint64_t r0 = row_ptr[v], r1 = row_ptr[v + 1];
      if (r1 < r0 || r1 > m) { bad = 1; return; }
      const uint64_t dv = r1 - r0;
      if (du > dv || (du == dv && u > v)) {
        ++nlead;
        uint64_t back;
        if (!find_arc(row_ptr, col, m, v, u, &back)) { bad = 1; return; }
        if ((w ? w[back] : 1u) != wa) bad = 1;
      } else {
        ++ntrail;
      }
    }
    mw = wa > mw ? wa : mw;
  });
  const uint64_t anybad = __ballot(bad != 0);
  mw = ~wave_min_u32(~mw);  // wave max
  mc = ~wave_min_u32(~mc);
  const uint64_t lead = wave_sum_u64(nlead), trail = wave_sum_u64(ntrail);
  if (lane == 0) {
    sh_bad[wv] = anybad ? 1u : 0u;
    sh_mw[wv] = mw;
    sh_mc[wv] = mc;
    sh_lead[wv] = lead;
    sh_trail[wv] = trail;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t b = 0, x = 0, c = 0;
    unsigned long long l = 0, t = 0;
    for (uint32_t i = 0; i < blockDim.x / WAVE; ++i) {
      b |= sh_bad[i];
      x = sh_mw[i] > x ? sh_mw[i] : x;
      c = sh_mc[i] > c ? sh_mc[i] : c;
      l += sh_lead[i];
      t += sh_trail[i];
    }
    const uint32_t st = blockIdx.x % stripes;
    uint32_t *q = v32 + (size_t)st * VAL_STRIDE32;
    unsigned long long *r = lt + (size_t)st * VAL_STRIDE64;
    if (b) atomicOr(&q[0], 1u);
    if (x) atomicMax(&q[1], x);
    if (c) atomicMax(&q[2], c);
    if (l) atomicAdd(&r[0], l);
    if (t) atomicAdd(&r[1], t);
  }
}

static uint32_t validate_blocks(uint32_t n, uint64_t m) {
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(ceil_div(std::max<uint64_t>(n, m), 256), VAL_BLOCKS));
}

int validate_graph(Ctx &c, const fl_problem *p, bool directed, uint32_t *max_w_out, uint32_t *max_cost_out) {
  const uint32_t n = p->n;
  // row_ptr[0] and row_ptr[n]
  uint64_t ends[2];
  FL_HIP(hipMemcpyAsync(&ends[0], p->row_ptr, 8, hipMemcpyDeviceToHost, c.s));
  FL_HIP(hipMemcpyAsync(&ends[1], p->row_ptr + n, 8, hipMemcpyDeviceToHost, c.s));
  c.sync();
  if (ends[0] != 0 || ends[1] != p->n_arcs) return FL_EINVAL;
  constexpr uint32_t S = 64;  // stripes
  uint32_t *d = c.arena->get<uint32_t>((size_t)S * VAL_STRIDE32);
  uint64_t *lt = c.arena->get<uint64_t>((size_t)S * VAL_STRIDE64);
  fill_u32(c, d, (size_t)S * VAL_STRIDE32, 0);
  fill_u64(c, lt, (size_t)S * VAL_STRIDE64, 0);
  k_validate<<<validate_blocks(n, p->n_arcs), 256, 0, c.s>>>(n, p->n_arcs, p->row_ptr, p->col, p->w, p->fac_cost, d, S,
                                                  directed ? 1u : 0u, reinterpret_cast<unsigned long long *>(lt));
  FL_LAUNCH_CHECK();
  std::vector<uint32_t> h((size_t)S * VAL_STRIDE32);
  std::vector<uint64_t> hl((size_t)S * VAL_STRIDE64);
  FL_HIP(hipMemcpyAsync(h.data(), d, h.size() * 4, hipMemcpyDeviceToHost, c.s));
  FL_HIP(hipMemcpyAsync(hl.data(), lt, hl.size() * 8, hipMemcpyDeviceToHost, c.s));
  c.sync();
  uint32_t err = 0, mw = 1, mc = 0;
  uint64_t lead = 0, trail = 0;
  for (uint32_t i = 0; i < S; ++i) {
    const uint32_t *q = &h[(size_t)i * VAL_STRIDE32];
    err |= q[0];
    mw = q[1] > mw ? q[1] : mw;
    mc = q[2] > mc ? q[2] : mc;
    lead += hl[(size_t)i * VAL_STRIDE64];
    trail += hl[(size_t)i * VAL_STRIDE64 + 1];
  }
  if (err || lead != trail) return FL_EINVAL;
  *max_w_out = mw;
  *max_cost_out = mc;
  return FL_OK;
}

// row_ptr[0] == 0 and row_ptr[n] == n_arcs of each graph
struct EndsDesc {
  const uint64_t *row_ptr;
  uint32_t n;
  uint64_t m;
};
__global__ void k_check_ends(const EndsDesc *d, uint32_t G, uint32_t *err) {
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < G && (d[g].row_ptr[0] != 0 || d[g].row_ptr[d[g].n] != d[g].m)) err[(size_t)g * VAL_STRIDE32] |= 2u;
}

void validate_graphs(Ctx &c, const fl_problem *const *ps, uint32_t G, bool directed, std::vector<int> &rc,
                     std::vector<uint32_t> &max_w, std::vector<uint32_t> &max_cost) {
  // one stripe (a 128-byte line of counters) per graph
  uint32_t *d = c.arena->get<uint32_t>((size_t)VAL_STRIDE32 * G);
  uint64_t *lt = c.arena->get<uint64_t>((size_t)VAL_STRIDE64 * G);
  fill_u64(c, lt, (size_t)VAL_STRIDE64 * G, 0);
  EndsDesc *ed = c.arena->get<EndsDesc>(G);
  std::vector<EndsDesc> hd(G);
  for (uint32_t g = 0; g < G; ++g) hd[g] = EndsDesc{ps[g]->row_ptr, ps[g]->n, ps[g]->n_arcs};
  fill_u32(c, d, (size_t)VAL_STRIDE32 * G, 0);
  FL_HIP(hipMemcpyAsync(ed, hd.data(), G * sizeof(EndsDesc), hipMemcpyHostToDevice, c.s));
  k_check_ends<<<(uint32_t)ceil_div(G, 256), 256, 0, c.s>>>(ed, G, d);
  FL_LAUNCH_CHECK();
  // the row checks read row_ptr only inside [0, n_arcs], whatever its values
  for (uint32_t g = 0; g < G; ++g) {
    const fl_problem *p = ps[g];
    k_validate<<<validate_blocks(p->n, p->n_arcs), 256, 0, c.s>>>(p->n, p->n_arcs, p->row_ptr, p->col, p->w, p->fac_cost,
                                                       d + (size_t)VAL_STRIDE32 * g, 1, directed ? 1u : 0u,
                                                       reinterpret_cast<unsigned long long *>(lt) +
                                                           (size_t)VAL_STRIDE64 * g);
    FL_LAUNCH_CHECK();
  }
  std::vector<uint32_t> h((size_t)VAL_STRIDE32 * G);
  std::vector<uint64_t> hl((size_t)VAL_STRIDE64 * G);
  FL_HIP(hipMemcpyAsync(h.data(), d, h.size() * 4, hipMemcpyDeviceToHost, c.s));
  FL_HIP(hipMemcpyAsync(hl.data(), lt, hl.size() * 8, hipMemcpyDeviceToHost, c.s));
  c.sync();
  rc.assign(G, FL_OK);
  max_w.assign(G, 1);
  max_cost.assign(G, 0);
  for (uint32_t g = 0; g < G; ++g) {
    const uint32_t *q = &h[(size_t)VAL_STRIDE32 * g];
    const uint64_t *r = &hl[(size_t)VAL_STRIDE64 * g];
    if (q[0] || r[0] != r[1]) rc[g] = FL_EINVAL;
    max_w[g] = q[1] > 1 ? q[1] : 1u;
    max_cost[g] = q[2];
  }
}

std::vector<uint64_t> read_seg_ctr(Ctx &c, const uint64_t *d, uint32_t G, uint32_t nf, uint32_t stripes,
                                   bool max_last) {
  std::vector<uint64_t> h((size_t)G * nf * stripes);
  FL_HIP(hipMemcpyAsync(h.data(), d, h.size() * 8, hipMemcpyDeviceToHost, c.s));
  c.sync();
  std::vector<uint64_t> out((size_t)G * nf, 0);
  for (size_t i = 0; i < out.size(); ++i) {
    const bool mx = max_last && (i % nf) == nf - 1;
    for (uint32_t s = 0; s < stripes; ++s) {
      const uint64_t x = h[i * stripes + s];
      out[i] = mx ? (x > out[i] ? x : out[i]) : out[i] + x;
    }
  }
  return out;
}

// ---------------------------------------------------------------------------
// Exclusive scan u32 -> u64 (n+1 outputs).  Three passes: per-block sums,
// one block scans the block sums, blocks add their prefix.
// ---------------------------------------------------------------------------
constexpr int SCAN_BLOCK = 1024;
constexpr int SCAN_ITEMS = 4;
constexpr uint32_t SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

__device__ inline uint64_t block_scan_excl_u64(uint64_t x, uint64_t *tmp, uint64_t *total) {
  // wave-level inclusive scan then block combine
  const int lane = lane_id(), wv = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  uint64_t inc = x;
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    uint64_t y = __shfl_up(inc, d, WAVE);
    if (lane >= d) inc += y;
  }
  if (lane == WAVE - 1) tmp[wv] = inc;
  __syncthreads();
  if (wv == 0) {
    uint64_t t = lane < nw ? tmp[lane] : 0;
    uint64_t ti = t;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
      uint64_t y = __shfl_up(ti, d, WAVE);
      if (lane >= d) ti += y;
    }
    if (lane < nw) tmp[lane] = ti - t;
    if (lane == nw - 1) tmp[WAVE] = ti;
  }
  __syncthreads();
  uint64_t r = tmp[wv] + inc - x;
  *total = tmp[WAVE];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_tiles(const uint32_t *in, uint32_t n, uint64_t *out,
                                                          uint64_t *tile_sums) {
  __shared__ uint64_t tmp[WAVE + 1];
  const uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_ITEMS;
  uint32_t v[SCAN_ITEMS];
  uint64_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    v[i] = base + i < n ? in[base + i] : 0u;
    s += v[i];
  }
  uint64_t total;
  uint64_t pre = block_scan_excl_u64(s, tmp, &total);
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    if (base + i < n) out[base + i] = pre;
    pre += v[i];
  }
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_sums(uint64_t *sums, uint32_t count, uint64_t *grand) {
  __shared__ uint64_t tmp[WAVE + 1];
  uint64_t carry = 0;
  for (uint32_t base = 0; base < count; base += SCAN_BLOCK) {
    uint32_t i = base + threadIdx.x;
    uint64_t x = i < count ? sums[i] : 0;
    uint64_t total;
    uint64_t pre = block_scan_excl_u64(x, tmp, &total);
    if (i < count) sums[i] = pre + carry;
    carry += total;
  }
  if (threadIdx.x == 0) *grand = carry;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_add(uint64_t *out, uint32_t n, const uint64_t *sums) {
  const uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_ITEMS;
  const uint64_t add = sums[blockIdx.x];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i)
    if (base + i < n) out[base + i] += add;
}

size_t scan_sums_count(uint32_t n) { return ceil_div(n ? n : 1, SCAN_TILE) + 1; }

void scan_u32_to_u64(Ctx &c, const uint32_t *in, uint64_t *out, uint32_t n, uint64_t *sums) {
  uint32_t tiles = (uint32_t)ceil_div(n ? n : 1, SCAN_TILE);
  if (!sums) sums = c.arena->get<uint64_t>(tiles + 1);
  k_scan_tiles<<<tiles, SCAN_BLOCK, 0, c.s>>>(in, n, out, sums);
  FL_LAUNCH_CHECK();
  k_scan_sums<<<1, SCAN_BLOCK, 0, c.s>>>(sums, tiles, out + n);
  FL_LAUNCH_CHECK();
  k_scan_add<<<tiles, SCAN_BLOCK, 0, c.s>>>(out, n, sums);
  FL_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// In-arcs of a directed graph (Sec. 3.1 admits directed graphs): a counting
// sort of the arcs by head.  Within a row the order is that of the atomic
// cursor; nothing downstream depends on it (sketches, labels and sweeps are
// minima over the row).
// ---------------------------------------------------------------------------
__global__ void k_in_degree(uint64_t m, const uint32_t *col, uint32_t *deg) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; a < m; a += stride) atomicAdd(&deg[col[a]], 1u);
}

// row_ptr is validated: row_ptr[0] = 0, non-decreasing, row_ptr[n] = m, and
// every col < n, so the tail search stays in [0, n) and p < in_ptr[v + 1].
__global__ void k_in_scatter(uint32_t n, uint64_t m, const uint64_t *row_ptr, const uint32_t *col,
                             const uint32_t *w, const uint64_t *in_ptr, uint32_t *cur, uint32_t *in_col,
                             uint32_t *in_w, uint32_t *out_to_in) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; a < m; a += stride) {
    uint32_t lo = 0, hi = n;  // row_ptr[lo] <= a < row_ptr[hi]
    while (hi - lo > 1) {
      const uint32_t mid = lo + ((hi - lo) >> 1);
      if (row_ptr[mid] <= a) lo = mid;
      else hi = mid;
    }
    const uint32_t v = col[a];
    const uint64_t p = in_ptr[v] + atomicAdd(&cur[v], 1u);
    in_col[p] = lo;
    if (w) in_w[p] = w[a];
    if (out_to_in) out_to_in[a] = (uint32_t)p;
  }
}

size_t transpose_bytes(uint32_t n, uint64_t m, bool weighted) {
  return (size_t)(n + 1) * 8 + (size_t)n * 4 + (size_t)m * (weighted ? 12 : 8) + ((size_t)1 << 20);
}

void set_in_arcs(Ctx &c, Graph &g, bool directed) {
  if (!directed) {
    g.in_ptr = g.row_ptr;
    g.in_col = g.col;
    g.in_w = g.w;
    return;
  }
  const uint32_t n = g.n;
  const uint64_t m = g.m;
  uint32_t *deg = c.arena->get<uint32_t>(n);
  uint64_t *ip = c.arena->get<uint64_t>((size_t)n + 1);
  uint32_t *ic = c.arena->get<uint32_t>(m ? m : 1);
  uint32_t *iw = g.w ? c.arena->get<uint32_t>(m ? m : 1) : nullptr;
  // arc positions fit 32 bits below 2^32 arcs; beyond, the sketch rounds scan every in-arc
  uint32_t *o2i = m < 0xFFFFFFFFull ? c.arena->get<uint32_t>(m ? m : 1) : nullptr;
  fill_u32(c, deg, n, 0);
  const uint32_t blocks = (uint32_t)std::min<uint64_t>(ceil_div(m ? m : 1, 256), 16384);
  if (m) {
    k_in_degree<<<blocks, 256, 0, c.s>>>(m, g.col, deg);
    FL_LAUNCH_CHECK();
  }
  scan_u32_to_u64(c, deg, ip, n);
  fill_u32(c, deg, n, 0);  // now the per-row cursor
  if (m) {
    k_in_scatter<<<blocks, 256, 0, c.s>>>(n, m, g.row_ptr, g.col, g.w, ip, deg, ic, iw, o2i);
    FL_LAUNCH_CHECK();
  }
  g.in_ptr = ip;
  g.in_col = ic;
  g.in_w = iw;
  g.out_to_in = o2i;
}

// ---------------------------------------------------------------------------
// sum_v cnt[v] * deg(v) and sum_v cnt[v]
// ---------------------------------------------------------------------------
__global__ void k_ads_totals(uint32_t n, const uint64_t *row_ptr, const uint32_t *cnt, const uint32_t *gid,
                             uint64_t *ctr, uint32_t stripes) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = i < n;
  uint64_t r = 0, e = 0;
  uint32_t g = 0;
  if (valid) {
    e = cnt[i];
    r = e * (row_ptr[i + 1] - row_ptr[i]);
    g = seg_of(gid, (uint32_t)i);
  }
  seg_add((unsigned long long *)ctr, valid, g, 0, 2, stripes, r);
  seg_add((unsigned long long *)ctr, valid, g, 1, 2, stripes, e);
}

void ads_totals(Ctx &c, const Graph &g, const uint32_t *gid, uint32_t G, const uint32_t *cnt,
                std::vector<uint64_t> &relax_alg, std::vector<uint64_t> &entries) {
  const uint32_t stripes = G == 1 ? 64 : 1;
  uint64_t *ctr = c.arena->get<uint64_t>((size_t)2 * G * stripes);
  fill_u64(c, ctr, (size_t)2 * G * stripes, 0);
  k_ads_totals<<<(uint32_t)ceil_div(g.n, 256), 256, 0, c.s>>>(g.n, g.row_ptr, cnt, gid, ctr, stripes);
  FL_LAUNCH_CHECK();
  const std::vector<uint64_t> h = read_seg_ctr(c, ctr, G, 2, stripes);
  relax_alg.resize(G);
  entries.resize(G);
  for (uint32_t q = 0; q < G; ++q) {
    relax_alg[q] = h[2 * q];
    entries[q] = h[2 * q + 1];
  }
}

// ---------------------------------------------------------------------------
// Frontier Bellman-Ford on packed labels (value << 32 | tie): a label moves
// along an arc of weight w as label + (w << 32).  Each vertex of the current
// frontier pushes its label to all neighbours with 64-bit atomicMin; a
// neighbour whose label dropped joins the next frontier once (stamped with
// the iteration number).  The fixed point is the lexicographic minimum over
// sources of (init value + distance, tie).
// ---------------------------------------------------------------------------
// Appends to the next frontier, staged per wave in LDS (2 WAVE entries) and
// written WAVE at a time with one atomic: every wave of a large frontier
// appends at nearly every step, and per-step atomics queue on the one count.
struct WaveQ {
  uint32_t *buf;  // this wave's LDS staging area
  uint32_t cnt;   // staged entries (wave-uniform, < WAVE between calls)
  uint32_t *next, *nnext;
};

// every lane calls, converged
__device__ inline void wq_push(WaveQ &q, bool add, uint32_t y) {
  const int lane = lane_id();
  const uint64_t m = __ballot(add);
  if (!m) return;
  if (add) q.buf[q.cnt + lanes_below(m)] = y;
  q.cnt += (uint32_t)__popcll(m);
  if (q.cnt < (uint32_t)WAVE) return;
  wave_lds_sync();
  uint32_t base = 0;
  if (lane == 0) base = atomicAdd(q.nnext, (uint32_t)WAVE);
  base = __shfl(base, 0, WAVE);
  q.next[base + lane] = q.buf[lane];
  q.cnt -= WAVE;
  const uint32_t rest = (uint32_t)lane < q.cnt ? q.buf[WAVE + lane] : 0u;
  wave_lds_sync();
  if ((uint32_t)lane < q.cnt) q.buf[lane] = rest;
  wave_lds_sync();
}

// The staged remainders of a block's 4 waves (every thread of the block calls,
// once, before it exits): one atomic on the count for all of them.  A frontier
// of some thousand vertices of low degree is spread over 2,048 waves of 4
// vertices, each with a handful of appends; with an atomic per wave they queued
// on the one count (opening loop of a grid of 1,200 x 1,200, weights 1..9, 320 ->
// 226 to 255 ms; assignment on 600 x 600 2.8 -> 2.0; R-MAT 2^20 directed, weights
// 1..100, gamma 1.5 -> 1.2, opening loop 28.7 -> 27.5).
__device__ inline void wq_flush(WaveQ &q) {
  __shared__ uint32_t s_n[256 / WAVE], s_base;
  const uint32_t lane = (uint32_t)lane_id(), wv = threadIdx.x / WAVE;
  if (lane == 0) s_n[wv] = q.cnt;
  __syncthreads();
  uint32_t at = 0, tot = 0;
#pragma unroll
  for (uint32_t i = 0; i < 256 / WAVE; ++i) {
    at += i < wv ? s_n[i] : 0u;
    tot += s_n[i];
  }
  if (threadIdx.x == 0 && tot) s_base = atomicAdd(q.nnext, tot);
  __syncthreads();
  if (lane < q.cnt) q.next[s_base + at + lane] = q.buf[lane];
}

// one arc step (every lane calls, converged): relax arc a with label L
__device__ inline void sssp_arc(const uint32_t *col, const uint32_t *w, uint64_t *labels, bool valid, uint64_t a,
                                uint64_t L, WaveQ &q, uint32_t *stamp, uint32_t iter) {
  bool add = false;
  uint32_t y = 0;
  if (valid) {
    y = col[a];
    const uint64_t nl = L + ((uint64_t)(w ? w[a] : 1u) << 32);
    if (nl < __hip_atomic_load(&labels[y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      const uint64_t old = atomicMin((unsigned long long *)&labels[y], (unsigned long long)nl);
      if (nl < old) add = atomicMax(&stamp[y], iter) < iter;
    }
  }
  wq_push(q, add, y);
}

// One search over the arcs, its two frontier lists and its device state.
struct SsspArgs {
  const uint64_t *row_ptr;
  const uint32_t *col, *w;
  uint64_t *labels;
  uint32_t *front[2];
  uint32_t *stamp;
  uint64_t *heavy;
  SsspState *st;
};

// Wide iteration, first launch: one lane per frontier vertex; short rows
// flattened over the wave, long rows queued for k_sssp_heavy (one wave per
// row).  Nothing to do when the search has ended.
__global__ __launch_bounds__(256) void k_sssp_push(SsspArgs S) {
  __shared__ uint32_t s_q[256 / WAVE][2 * WAVE];
  const uint32_t nf = S.st->nf, cur = S.st->cur, iter = S.st->iter + 1;
  WaveQ q{s_q[threadIdx.x / WAVE], 0u, S.front[cur ^ 1], &S.st->nnext};
  const uint32_t *front = S.front[cur];
  const uint32_t vw = wave_share(nf), lane = (uint32_t)lane_id();
  const uint64_t stride = (uint64_t)gridDim.x * (blockDim.x / WAVE) * vw;
  for (uint64_t b = ((uint64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE) * vw; b < nf; b += stride) {
    const uint64_t i = b + lane;
    const bool want = lane < vw && i < nf;
    uint32_t v = 0;
    uint64_t a0 = 0, deg = 0, L = 0;
    if (want) {
      v = front[i];
      L = __hip_atomic_load(&S.labels[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      a0 = S.row_ptr[v];
      deg = S.row_ptr[v + 1] - a0;
    }
    const bool hv = want && deg > FLAT_MAX;
    push_pieces(S.heavy, &S.st->nheavy, hv, v, deg);
    flat_arcs(want && !hv, a0, deg, [&](bool valid, uint64_t a, int o) {
      sssp_arc(S.col, S.w, S.labels, valid, a, shfl_u64(L, o), q, S.stamp, iter);
    });
  }
  wq_flush(q);
}

// Wide iteration, second launch: the queued pieces, one wave per piece.
__global__ __launch_bounds__(256) void k_sssp_heavy(SsspArgs S) {
  __shared__ uint32_t s_q[256 / WAVE][2 * WAVE];
  const uint32_t cnt = S.st->nheavy, iter = S.st->iter + 1;
  WaveQ q{s_q[threadIdx.x / WAVE], 0u, S.front[S.st->cur ^ 1], &S.st->nnext};
  const int lane = lane_id();
  const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) / WAVE;
  for (uint64_t i = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; i < cnt; i += nw) {
    uint64_t a0, a1;
    const uint32_t v = piece_arcs(S.heavy[i], S.row_ptr, &a0, &a1);
    const uint64_t L = __hip_atomic_load(&S.labels[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (uint64_t c = a0; c < a1; c += WAVE)
      sssp_arc(S.col, S.w, S.labels, c + lane < a1, c + lane, L, q, S.stamp, iter);
  }
  wq_flush(q);
}

// Narrow iterations (see fl_frontier.h), by one block, until the frontier is
// empty or too large.  SE_SEEDS: start from the nseeds <= NARROW_V vertices of
// seeds; SE_WIDE: first close the wide iteration that ran before (its frontier
// is the list it appended to); SE_STATE: go on from the state (and clear
// *unseeded); SE_OPENED: if *unseeded, start from the *d_nseeds vertices of
// seeds, label them and clear the flag (more than NARROW_V are left as they
// are, the flag set).  Labels are read and lowered at the
// device's L2 (agent scope); the frontier lists are written and read by this
// block only, a barrier apart.
// Bound by latency: an iteration is the chain list -> row and label ->
// column -> label -> atomic minimum -> stamp -> list.  Opening loop of R-MAT
// 2^18 (unit weights, eps 0.01, 476 searches): 86 -> 60 ms, of a Chung-Lu
// graph of 50,000 vertices 20 -> 13 ms, against 8 wide iterations per check.
enum SsspEntry : int { SE_SEEDS = 0, SE_WIDE, SE_STATE, SE_OPENED };
__global__ __launch_bounds__(NARROW_T) void k_sssp_narrow(SsspArgs S, const uint32_t *seeds, uint32_t nseeds,
                                                          int entry, const uint32_t *d_nseeds, uint32_t *unseeded) {
  __shared__ uint64_t s_a0[NARROW_V], s_L[NARROW_V];
  __shared__ uint32_t s_excl[NARROW_V], s_tmp[NARROW_WAVES], s_nn;
  const uint32_t tid = threadIdx.x;
  uint32_t nf = nseeds, cur = S.st->cur, iter = S.st->iter, wide = S.st->wide;
  const uint32_t *list = seeds;
  if (entry == SE_WIDE || entry == SE_STATE) {
    if (entry == SE_STATE && tid == 0) *unseeded = 0;
    nf = S.st->nf;
    if (nf == 0) return;  // the search had ended before the wide launches
    if (entry == SE_WIDE) {
      nf = S.st->nnext;
      cur ^= 1;
      ++iter;
      ++wide;
    }
    list = S.front[cur];
  } else if (entry == SE_OPENED) {
    if (!*unseeded) return;
    nf = *d_nseeds;
    if (nf <= NARROW_V)
      for (uint32_t p = tid; p < nf; p += NARROW_T) S.labels[seeds[p]] = (uint64_t)seeds[p];
  }
  __syncthreads();  // every thread has read the state and the flag before they are rewritten
  if (entry == SE_OPENED && nf <= NARROW_V && tid == 0) *unseeded = 0;
  while (nf && nf <= NARROW_V) {
    uint32_t v[2] = {0, 0}, deg[2] = {0, 0}, ex[2];
    uint64_t a0[2] = {0, 0}, L[2] = {0, 0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t p = tid + h * NARROW_T;
      if (p < nf) {
        v[h] = list[p];
        L[h] = __hip_atomic_load(&S.labels[v[h]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a0[h] = S.row_ptr[v[h]];
        const uint64_t d = S.row_ptr[v[h] + 1] - a0[h];
        deg[h] = d > NARROW_ARCS ? NARROW_ARCS + 1 : (uint32_t)d;  // sums stay far below 2^32
      }
    }
    uint32_t t0, t1 = 0;
    ex[0] = narrow_scan_excl(deg[0], s_tmp, &t0);
    ex[1] = t0;
    if (nf > NARROW_T) ex[1] = t0 + narrow_scan_excl(deg[1], s_tmp, &t1);
    const uint32_t total = t0 + t1;
    if (total > NARROW_ARCS) break;  // a wide iteration takes this frontier
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t p = tid + h * NARROW_T;
      s_excl[p] = p < nf ? ex[h] : total;
      s_a0[p] = a0[h];
      s_L[p] = L[h];
    }
    if (tid == 0) s_nn = 0;
    __syncthreads();
    ++iter;
    uint32_t *next = S.front[cur ^ 1];
    const uint32_t half = narrow_half(nf);
    for (uint32_t b = 0; b < total; b += NARROW_T) {
      const uint32_t idx = b + tid;
      bool add = false;
      uint32_t y = 0;
      if (idx < total) {
        const uint32_t p = narrow_owner(s_excl, idx, half);
        const uint64_t a = s_a0[p] + (idx - s_excl[p]);
        y = S.col[a];
        const uint64_t nl = s_L[p] + ((uint64_t)(S.w ? S.w[a] : 1u) << 32);
        if (nl < __hip_atomic_load(&S.labels[y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          const uint64_t old = atomicMin((unsigned long long *)&S.labels[y], (unsigned long long)nl);
          if (nl < old) add = atomicMax(&S.stamp[y], iter) < iter;
        }
      }
      wave_push(next, &s_nn, add, y);
    }
    __syncthreads();
    nf = s_nn;
    cur ^= 1;
    list = S.front[cur];
    __syncthreads();  // s_nn is cleared and the LDS arrays are rewritten by the next iteration
  }
  if (nf && nf <= NARROW_V && list == seeds) {
    // the first iteration is a wide one: it reads the frontier list
    for (uint32_t p = tid; p < nf; p += NARROW_T) S.front[cur][p] = seeds[p];
  }
  if (tid == 0) *S.st = SsspState{nf, cur, iter, 0u, 0u, wide};
}

// a search that starts with a wide iteration over front[0]
__global__ void k_sssp_start(SsspState *st, uint32_t nf) { *st = SsspState{nf, 0u, st->iter, 0u, 0u, st->wide}; }

void sssp_alloc(Ctx &c, SsspWork &wk, uint32_t n, uint64_t m) {
  wk.front[0] = c.arena->get<uint32_t>(n + 1);
  wk.front[1] = c.arena->get<uint32_t>(n + 1);
  wk.flag = c.arena->get<uint32_t>(n);
  wk.heavy = c.arena->get<uint64_t>(piece_capacity(n, m));
  wk.st = c.arena->get<SsspState>(1);
  fill_u32(c, wk.flag, n, 0);
  fill_u32(c, reinterpret_cast<uint32_t *>(wk.st), sizeof(SsspState) / 4, 0);
}

// Runs to the fixed point.  Stamps grow monotonically across the calls on one
// workspace.  Labels travel against the arcs (over the in-arcs), so each
// vertex ends with the best label of the seeds it can reach: distances from
// every vertex TO the seed set.
//
// Narrow iterations run in one launch until the frontier is empty or too
// large; a wide iteration is two launches and the narrow one that closes it
// (and goes on if what is left is narrow).  WIDE_CHAIN wide iterations are
// launched before the first host check, twice as many before each next one up
// to WIDE_CHAIN_MAX; those that find the search ended exit at once.  Most
// searches take a few; on a grid of 600 x 600 (weights 1..4, distances of
// hundreds) two per check made the assignment 2.0 ms, 1.8 with this.
constexpr int WIDE_CHAIN = 2, WIDE_CHAIN_MAX = 16;
static SsspArgs sssp_args(const Graph &g, uint64_t *labels, const SsspWork &wk) {
  return SsspArgs{g.in_ptr, g.in_col, g.in_w, labels, {wk.front[0], wk.front[1]}, wk.flag, wk.heavy, wk.st};
}
static void sssp_narrow(Ctx &c, const SsspArgs &S, const uint32_t *seeds, uint32_t nseeds, SsspEntry e,
                        const uint32_t *d_nseeds = nullptr, uint32_t *unseeded = nullptr) {
  k_sssp_narrow<<<1, NARROW_T, 0, c.s>>>(S, seeds, nseeds, e, d_nseeds, unseeded);
  FL_LAUNCH_CHECK();
}
// a frontier can grow by orders of magnitude within a chain: every launch gets
// a grid for any frontier (blocks past the count exit)
static void sssp_wide(Ctx &c, const Graph &g, const SsspArgs &S, uint32_t nf) {
  k_sssp_push<<<wide_blocks(g.n, nf), 256, 0, c.s>>>(S);
  FL_LAUNCH_CHECK();
  k_sssp_heavy<<<HEAVY_BLOCKS, 256, 0, c.s>>>(S);
  FL_LAUNCH_CHECK();
  sssp_narrow(c, S, nullptr, 0, SE_WIDE);
}
static uint32_t sssp_check(Ctx &c, const SsspWork &wk) {
  c.fetch(wk.st, sizeof(uint32_t));
  return (uint32_t)(c.h_status[0] & 0xFFFFFFFFu);
}
static void sssp_loop(Ctx &c, const Graph &g, const SsspArgs &S, const SsspWork &wk, uint32_t nf) {
  for (int chain = WIDE_CHAIN; nf; chain = std::min(2 * chain, WIDE_CHAIN_MAX)) {
    for (int b = 0; b < chain; ++b) sssp_wide(c, g, S, b == 0 ? nf : 0u);
    nf = sssp_check(c, wk);
  }
}

void sssp_run(Ctx &c, const Graph &g, uint64_t *labels, const uint32_t *seeds, uint32_t nseeds, SsspWork &wk) {
  if (nseeds == 0) return;
  const SsspArgs S = sssp_args(g, labels, wk);
  uint32_t nf = nseeds;
  if (nseeds <= NARROW_V) {
    sssp_narrow(c, S, seeds, nseeds, SE_SEEDS);
    nf = sssp_check(c, wk);
  } else {
    FL_HIP(hipMemcpyAsync(wk.front[0], seeds, (size_t)nseeds * 4, hipMemcpyDeviceToDevice, c.s));
    k_sssp_start<<<1, 1, 0, c.s>>>(wk.st, nseeds);
    FL_LAUNCH_CHECK();
  }
  sssp_loop(c, g, S, wk, nf);
}

void sssp_opened(Ctx &c, const Graph &g, uint64_t *labels, const uint32_t *seeds, const uint32_t *d_nseeds,
                 uint32_t *unseeded, SsspWork &wk) {
  sssp_narrow(c, sssp_args(g, labels, wk), seeds, 0, SE_OPENED, d_nseeds, unseeded);
}

void sssp_chain(Ctx &c, const Graph &g, uint64_t *labels, uint32_t *unseeded, SsspWork &wk, int wide) {
  const SsspArgs S = sssp_args(g, labels, wk);
  sssp_narrow(c, S, nullptr, 0, SE_STATE, nullptr, unseeded);
  for (int b = 0; b < wide; ++b) sssp_wide(c, g, S, 0);
}

void sssp_finish(Ctx &c, const Graph &g, uint64_t *labels, uint32_t *unseeded, SsspWork &wk) {
  const SsspArgs S = sssp_args(g, labels, wk);
  sssp_narrow(c, S, nullptr, 0, SE_STATE, nullptr, unseeded);
  sssp_loop(c, g, S, wk, sssp_check(c, wk));
}

}  // namespace fl
