// fl_frontier.h -- expansion of a frontier's rows, in two forms.
//
// Wide steps (many blocks): a frontier kernel flattens short rows over the
// wave (flat_arcs) and queues each long row as pieces of HCHUNK arcs; a second
// kernel walks the queue with one wave per piece, so the arcs of a hub are
// spread over many waves.
//
// Narrow steps (one block): a frontier of at most NARROW_V vertices with at
// most NARROW_ARCS arcs is expanded by a single block of 1,024 threads, which
// flattens all its rows over the block.  The block runs step after step with
// nothing but __syncthreads() between them and stops at the first step that
// exceeds the limits, which a wide step then takes.  Most steps are narrow:
// on graphs of 2,000 to 2^18 vertices 85-100% of the steps of the sweeps and
// of the Bellman-Ford searches have fewer than 1,024 vertices.  Such a step
// is a chain of about seven dependent memory round trips (some 5 us in one
// block); as two launches of many blocks it took 10-20 us and the gaps
// between the launches, whatever its size.
#pragma once

#include <algorithm>

#include "fl_common.h"

namespace fl {

// arcs per queued piece: hubs split finely enough to keep the long-row
// kernels' waves busy (MIS 0.935 -> 0.907 s on the large weighted workload
// against 2,048-arc pieces, timed on one box, identical results)
constexpr uint32_t HCHUNK = 512;
// blocks (of 256 threads) of a long-row kernel: it walks a device-side count
// with one wave per piece, so it needs many waves per CU to hide the random
// accesses of hub rows (16 per CU on 256 CUs); idle blocks exit at once
constexpr uint32_t HEAVY_BLOCKS = 1024;

// queue entries needed for n vertices and m arcs at most
inline uint64_t piece_capacity(uint64_t n, uint64_t m) { return n + m / HCHUNK + 64; }

// Every lane calls.  Lanes with heavy == true queue their row as pieces:
// entry = piece << 32 | vertex.
__device__ inline void push_pieces(uint64_t *q, uint32_t *qcnt, bool heavy, uint32_t x, uint64_t deg) {
  const uint32_t np = heavy ? (uint32_t)((deg + HCHUNK - 1) / HCHUNK) : 0u;
  const uint32_t incl = wave_scan_incl(np);
  const uint32_t tot = __shfl(incl, WAVE - 1, WAVE);
  if (!tot) return;
  uint32_t base = 0;
  if (lane_id() == 0) base = atomicAdd(qcnt, tot);
  base = __shfl(base, 0, WAVE);
  for (uint32_t p = 0; p < np; ++p) q[base + incl - np + p] = ((uint64_t)p << 32) | x;
}

// arcs [*b0, *b1) of queue entry e
__device__ inline uint32_t piece_arcs(uint64_t e, const uint64_t *row_ptr, uint64_t *b0, uint64_t *b1) {
  const uint32_t x = (uint32_t)e;
  const uint64_t p = e >> 32;
  const uint64_t a0 = row_ptr[x], a1 = row_ptr[x + 1];
  *b0 = a0 + p * HCHUNK;
  *b1 = *b0 + HCHUNK < a1 ? *b0 + HCHUNK : a1;
  return x;
}

// Frontier vertices per wave of a wide step: a full wave of 64, or fewer (a
// power of two, at least 4) while that keeps the launch at SHARE_WAVES busy
// waves or fewer, so that a frontier of some thousand vertices is spread over
// the chip.  A wave walks its rows' arcs 64 or 128 at a time, one dependent
// chain after another: with 64 vertices of average degree 12 that is six
// chains, with 4 it is one.  More waves than that cost more in appends (each
// wave reserves room per distinct slot) than they hide: with 8,192 the MIS
// of R-MAT 2^21 (weights 1..100) took 164 ms, with 2,048 144 ms; with one
// vertex per lane throughout 152 ms.
constexpr uint32_t SHARE_WAVES = 2048;
__device__ inline uint32_t wave_share(uint32_t cnt) {
  const uint64_t all = (uint64_t)gridDim.x * (blockDim.x / WAVE);
  const uint64_t nw = all < SHARE_WAVES ? all : SHARE_WAVES;
  uint32_t vw = WAVE;
  while (vw > 4 && nw * (vw / 2) >= cnt) vw /= 2;
  return vw;
}
// Blocks of a wide step over n vertices: 2,048 (32 waves per CU on 256 CUs)
// for any frontier that may arise, fewer where n cannot fill them, more for a
// frontier known to be larger (`want` vertices).
inline uint32_t wide_blocks(uint32_t n, uint64_t want) {
  const uint64_t any = std::min<uint64_t>(ceil_div(n, 16), 2048);
  return (uint32_t)std::min<uint64_t>(std::max<uint64_t>(any, ceil_div(want, 256)), 8192);
}

// ---------------------------------------------------------------------------
// narrow steps
// ---------------------------------------------------------------------------
constexpr uint32_t NARROW_T = 1024;            // threads of the block
constexpr uint32_t NARROW_V = 2 * NARROW_T;    // frontier vertices of a step: two per thread
// Arcs of a step: the block relaxes 2,048 arcs per 2-3 us, so beyond this a
// wide step is the faster one.
constexpr uint32_t NARROW_ARCS = 16384;
constexpr uint32_t NARROW_WAVES = NARROW_T / WAVE;

// Exclusive prefix of x over the block and its total (every thread calls;
// tmp: NARROW_WAVES words of LDS, free on entry and on return).
__device__ inline uint32_t narrow_scan_excl(uint32_t x, uint32_t *tmp, uint32_t *total) {
  const uint32_t wv = threadIdx.x / WAVE;
  const uint32_t incl = wave_scan_incl(x);
  if (lane_id() == WAVE - 1) tmp[wv] = incl;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (uint32_t i = 0; i < NARROW_WAVES; ++i) {
    const uint32_t t = tmp[i];
    pre += i < wv ? t : 0u;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return pre + incl - x;
}

// The row of arc idx: the last position p with excl[p] <= idx, for NARROW_V
// exclusive sums padded with the total (rows without arcs are skipped).  The
// search covers the first 2 * half positions.
__device__ inline uint32_t narrow_owner(const uint32_t *excl, uint32_t idx, uint32_t half) {
  uint32_t pos = 0;
  for (uint32_t s = half; s >= 1; s >>= 1)
    if (excl[pos + s] <= idx) pos += s;
  return pos;
}
// half of the smallest power of two that holds cnt positions
__device__ inline uint32_t narrow_half(uint32_t cnt) {
  return cnt <= 1 ? 0u : 1u << (31 - __clz(cnt - 1));
}

}  // namespace fl
