// plan_device.hip -- the plan of one expert-stage run, built on the GPU (gfx950).
//
// The host builder (plan.cpp) walks the routing serially.  Here the same plan -- layout,
// schedule, work queues and combine plan (paper Section 3.2, Algorithm 1; segment
// composition of Section 3.3.2) -- comes from four kernels in stream order:
//
//   rows    grid over dispatched rows: validates the routing and records, per (expert, source
//           rank), the run of rows it occupies (a histogram by run bounds: the dispatch order
//           keeps each source rank's rows of an expert contiguous); a hash set of (rank, slot)
//           catches duplicates.
//   layout  one workgroup: per expert, the owner groups in rank order (remote ranks ascending,
//           then the local rank) with band padding, prefix sums into tile rows and groups, the
//           remote-first schedule (experts by remote band count, descending), the tail split,
//           each schedule position's row group and the per-XCD queue bounds -- all closed forms
//           of the host's greedy walks.
//   fill    grid: every work item straight to its queue slot; the row tables; per tile row, the
//           logical rows where transfer segments start and end, compacted into short lists.
//   segs    one workgroup: prefix sums of the per-tile-row counts pair the k-th start with the
//           k-th end; each segment's fields and ready position; then a stable counting sort by
//           ready position (the order the consumer claims them in).
//
// Plans of a small capacity take one kernel instead, which also resets the run (small_plan).
//
// Every step reproduces the host's tables exactly for routing in dispatch order.  The
// single-workgroup kernels keep their tables in LDS when they fit, and need only workgroup
// barriers between phases: every wave of a workgroup shares one compute unit, whose vector
// cache is coherent for it, so no device-scope fence (an L2 write-back on this chip) is paid.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/moe_stage.h"
#include "init_device.hpp"
#include "plan_device.hpp"

namespace moe {
namespace {

constexpr int kWg = 1024;   // threads of the single-workgroup kernels
constexpr int kBlk = 256;   // threads of the grid kernels; one logical row each in a tile row
static_assert(kBlk == kTileM, "the fill and segment kernels give each tile row one workgroup");

__device__ __forceinline__ int32_t round_up_i(int32_t v, int32_t m) { return (v + m - 1) / m * m; }

// Inclusive prefix sum of x over a workgroup of kThreads threads: a shuffle scan within each
// 64-lane wave, then one over the wave totals.  `sh` holds kThreads / 64 ints of LDS; *total
// gets the workgroup's sum.  Every thread must call it.
template <int kThreads>
__device__ __forceinline__ int32_t wg_incl_scan(int32_t x, int32_t* sh, int32_t* total) {
  constexpr int kWaves = kThreads / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) sh[wv] = x;
  __syncthreads();
  if (wv == 0) {
    int32_t t = lane < kWaves ? sh[lane] : 0;
    for (int d = 1; d < kWaves; d <<= 1) {
      const int32_t y = __shfl_up(t, d, 64);
      if (lane >= d) t += y;
    }
    if (lane < kWaves) sh[lane] = t;
  }
  __syncthreads();
  const int32_t r = x + (wv ? sh[wv - 1] : 0);
  *total = sh[kWaves - 1];
  __syncthreads();  // sh may be reused at once
  return r;
}

// Exclusive prefix sum of v[0, n) in place by one workgroup of kThreads threads (v in LDS or
// global memory); returns the total, the same in every thread.
// kAtomicIn: v was last written by atomics; read it with device-coherent loads.
template <int kThreads, bool kAtomicIn = false>
__device__ int32_t wg_scan(int32_t* v, int32_t n, int32_t* sh) {
  const int tid = threadIdx.x;
  int32_t carry = 0;
  for (int32_t c0 = 0; c0 < n; c0 += kThreads) {
    const int32_t i = c0 + tid;
    int32_t x = 0;
    if (i < n) x = kAtomicIn ? __hip_atomic_load(&v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : v[i];
    int32_t tot;
    const int32_t incl = wg_incl_scan<kThreads>(x, sh, &tot);
    if (i < n) v[i] = carry + incl - x;
    carry += tot;
  }
  __syncthreads();
  return carry;
}

// Largest e in [0, n) with begin[e] <= i, for non-decreasing begin[] with begin[0] <= i: the
// expert (or owner) whose range holds i when empty ranges share their successor's start.
__device__ __forceinline__ int32_t range_of(const int32_t* begin, int32_t n, int32_t i) {
  int32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (begin[mid] <= i)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Inserts key into the open-addressing set; true if it was there already.  The set holds at
// most half its capacity, so a free entry is always found.
__device__ bool seen_insert(uint64_t* set, int64_t cap, uint64_t key) {
  uint64_t h = key * 0x9E3779B97F4A7C15ull;
  h ^= h >> 29;
  const uint64_t mask = (uint64_t)cap - 1;
  h &= mask;
  for (int64_t probe = 0; probe < cap; ++probe) {
    const unsigned long long prev = atomicCAS((unsigned long long*)&set[h], ~0ull, (unsigned long long)key);
    if (prev == ~0ull) return false;
    if (prev == key) return true;
    h = (h + 1) & mask;
  }
  return true;
}

// Rank order of the layout (Section 3.2.1): remote ranks ascending, the local rank last.
__device__ __forceinline__ int32_t rank_at(int32_t j, int32_t R, int32_t self) {
  return j == R - 1 ? self : (j < self ? j : j + 1);
}

__device__ void write_empty(const DevPlanArgs& a) {
  if (threadIdx.x < 2 * (kXcds + 1)) a.queues[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    PlanHeader* H = a.hdr;
    H->n_tile_rows = H->n_groups = H->n_gu = H->n_down = H->n_segs = 0;
    H->tail_split = 1;
    H->n_split_rows = H->n_partials = H->down_qmax = H->n_groups_all = 0;
    H->n_valid = H->n_lrows = H->n_band_pad = H->n_remote = 0;
  }
}

// ---------------------------------------------------------------------------------------------
// rows: validation and the per-(expert, rank) runs.
// ---------------------------------------------------------------------------------------------
constexpr int kLdsOffsets = 4096;  // expert offsets staged in LDS up to this many experts
constexpr int kLdsRanks = 1024;    // receive-buffer sizes staged in LDS up to this many ranks

__global__ __launch_bounds__(kBlk) void plan_rows_kernel(DevPlanArgs a) {
  __shared__ int32_t off_lds[kLdsOffsets + 1];
  __shared__ int64_t rr_lds[kLdsRanks];
  const bool in_lds = !a.no_lds && a.E_l <= kLdsOffsets;
  const bool rr_in_lds = !a.no_lds && a.R <= kLdsRanks;
  const int32_t* off = in_lds ? off_lds : a.off;
  const int64_t* rrows = rr_in_lds ? rr_lds : a.return_rows;
  int bad_off = 0;
  for (int e = threadIdx.x; e <= a.E_l; e += kBlk) {
    const int32_t v = a.off[e];
    if (in_lds) off_lds[e] = v;
    if (e < a.E_l) bad_off |= v > a.off[e + 1];
  }
  if (rr_in_lds)
    for (int r = threadIdx.x; r < a.R; r += kBlk) rr_lds[r] = a.return_rows[r];
  bad_off = __syncthreads_or(bad_off);
  const int32_t rows = off[a.E_l];
  int32_t code = 0;
  if (rows < 0)
    code = MOE_EROUTING;
  else if (rows > a.max_rows)
    code = MOE_ECAPACITY;
  else if (off[0] != 0 || bad_off)
    code = MOE_EROUTING;
  if (code) {
    if (blockIdx.x == 0 && threadIdx.x == 0) a.hdr->status = code;
    return;
  }
  const int32_t R = a.R;
  for (int32_t i = blockIdx.x * kBlk + threadIdx.x; i < rows; i += gridDim.x * kBlk) {
    // Neighbours are loaded with the row itself (clamped indices), so one round trip serves all.
    const int32_t ip = i > 0 ? i - 1 : i, in = i + 1 < rows ? i + 1 : i;
    const int32_t r = a.src[i], s = a.slot[i], r_prev = a.src[ip], r_next = a.src[in], s_prev = a.slot[ip];
    const int32_t e = range_of(off, a.E_l, i);
    const int32_t lo = off[e], hi = off[e + 1];
    bool bad = r < 0 || r >= R || s < 0 || (int64_t)s >= rrows[r];
    if (!bad) {
      const bool first = i == lo || r_prev != r;
      const bool last = i == hi - 1 || r_next != r;
      if (!first && s_prev >= s) bad = true;  // slots ascend within a rank's run
      if (first && atomicCAS(&a.ws.run_lo[e * R + r], -1, i) != -1) bad = true;  // a second run
      if (last) a.ws.run_hi[e * R + r] = i + 1;
      if (seen_insert(a.ws.seen, a.ws.seen_cap, ((uint64_t)r << 32) | (uint32_t)s)) bad = true;
    }
    if (bad) {
      atomicMin(&a.hdr->bad_row, i);
      a.hdr->status = MOE_EROUTING;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// layout: one workgroup.
// ---------------------------------------------------------------------------------------------
constexpr int kLdsExperts = 1024;  // per-expert tables in LDS up to this many experts,
constexpr int kLdsGroups = 2048;   // run and group tables up to this many (expert, rank) pairs
constexpr int kLayoutLds = kWg + 7 * kLdsExperts + 5 * kLdsGroups;  // ints

// kLds: the per-expert, run and group tables in LDS (`lds` holds kLayoutLds ints), else in the
// global scratch.  The bound of this phase is its chain of dependent reads, so the runs come into
// LDS in one round trip: read where they are used, one rank after the other, they were 2R of
// them and twice over: 18.9 us with 32 experts and 8 ranks, 15.7 so (2 experts, 4 ranks: 11.1, 9.3).
template <bool kLds>
__device__ __forceinline__ void layout_phase(const DevPlanArgs& a, int32_t* lds) {
  __shared__ unsigned long long s_pad, s_remote;
  int32_t* sh = lds;
  PlanHeader* H = a.hdr;
  const int tid = threadIdx.x;
  const int32_t E_l = a.E_l, R = a.R, self = a.self;
  const int32_t tb = a.overlapped ? a.tb : 1;
  const DevPlanWs& w = a.ws;
  int32_t* ex = lds + kWg;
  int32_t* gr = ex + 7 * kLdsExperts;
  int32_t* ex_ntr = kLds ? ex : w.ex_ntr;
  int32_t* ex_ng = kLds ? ex + kLdsExperts : w.ex_ng;
  int32_t* ex_hr = kLds ? ex + 2 * kLdsExperts : w.ex_hr;
  int32_t* ex_bands = kLds ? ex + 3 * kLdsExperts : w.ex_bands;
  int32_t* ex_roff = kLds ? ex + 4 * kLdsExperts : w.ex_roff;
  int32_t* ex_loff = kLds ? ex + 5 * kLdsExperts : w.ex_loff;
  int32_t* tmp = kLds ? ex + 6 * kLdsExperts : w.tmp;
  int32_t* gl_lrow0 = kLds ? gr : w.g_lrow0;
  int32_t* gl_rows = kLds ? gr + kLdsGroups : w.g_rows;
  int32_t* gl_dst = kLds ? gr + 2 * kLdsGroups : w.g_dst;
  int32_t* run_lo = kLds ? gr + 3 * kLdsGroups : w.run_lo;
  int32_t* run_hi = kLds ? gr + 4 * kLdsGroups : w.run_hi;
  if constexpr (kLds)
    for (int32_t i = tid; i < E_l * R; i += kWg) {
      run_lo[i] = w.run_lo[i];
      run_hi[i] = w.run_hi[i];
    }
  if (tid == 0) s_pad = s_remote = 0;
  if (H->status != 0) {
    write_empty(a);
    return;
  }
  __syncthreads();

  // Per expert: its owner groups in rank order, band padding after each remote group (only
  // in the overlapped layout), its extent in tile rows, and its schedule key.
  for (int32_t e = tid; e < E_l; e += kWg) {
    int32_t pos = 0, bands = 0, ng = 0, remote_end = 0;
    int64_t pad_e = 0, remote_e = 0;
    for (int32_t j = 0; j < R; ++j) {
      const int32_t r = rank_at(j, R, self);
      const int32_t lo = run_lo[e * R + r];
      if (lo < 0) continue;
      const int32_t n = run_hi[e * R + r] - lo;
      ++ng;
      pos += n;
      if (r != self) {
        remote_e += n;
        bands += (n + tb - 1) / tb;
        remote_end = pos;
        if (a.overlapped) {
          const int32_t p = round_up_i(pos, tb) - pos;
          pad_e += p;
          pos += p;
        }
      }
    }
    ex_ntr[e] = round_up_i(pos, kTileM) / kTileM;
    // Remote rows precede local ones, and padding never fills a whole tile row, so the tile
    // rows holding remote rows are the expert's first ones, through the last remote row's.
    ex_hr[e] = remote_end > 0 ? (remote_end - 1) / kTileM + 1 : 0;
    ex_bands[e] = bands;
    ex_ng[e] = ng;
    if (pad_e) atomicAdd(&s_pad, (unsigned long long)pad_e);
    if (remote_e) atomicAdd(&s_remote, (unsigned long long)remote_e);
  }
  __syncthreads();
  const int32_t n_tr = wg_scan<kWg>(ex_ntr, E_l, sh);   // ex_ntr: first tile row of each expert
  const int32_t n_grp = wg_scan<kWg>(ex_ng, E_l, sh);   // ex_ng: first group of each expert
  if (n_tr > a.max_tile_rows || n_tr >= kMaxTileRows) {
    if (tid == 0) H->status = MOE_ECAPACITY;
    write_empty(a);
    return;
  }

  // Remote-first schedule (Section 3.2.2): experts by remote band count, descending, ties by
  // id, each contributing its remote tile rows; then every expert's local-only tile rows in
  // expert order.  tmp[rank] takes each expert's remote tile-row count for the prefix sum.
  for (int32_t e = tid; e < E_l; e += kWg) {
    const int32_t b = ex_bands[e];
    int32_t rank = 0;
    for (int32_t f = 0; f < E_l; ++f) {
      const int32_t c = ex_bands[f];
      rank += (c > b) || (c == b && f < e);
    }
    tmp[rank] = ex_hr[e];
    ex_roff[e] = rank;
    const int32_t ntr_e = (e + 1 < E_l ? ex_ntr[e + 1] : n_tr) - ex_ntr[e];
    ex_loff[e] = ntr_e - ex_hr[e];
  }
  __syncthreads();
  const int32_t n_hr = wg_scan<kWg>(tmp, E_l, sh);
  wg_scan<kWg>(ex_loff, E_l, sh);  // + n_hr: first local-only position of each expert
  for (int32_t e = tid; e < E_l; e += kWg) ex_roff[e] = tmp[ex_roff[e]];

  // Owner groups with their places in the padded layout (the fill kernel reads the global
  // copies of the group table and of each expert's first group).
  for (int32_t e = tid; e < E_l; e += kWg) {
    const int32_t base = ex_ntr[e] * kTileM;
    int32_t g = ex_ng[e], pos = base;
    if constexpr (kLds) w.ex_ng[e] = g;
    for (int32_t j = 0; j < R; ++j) {
      const int32_t r = rank_at(j, R, self);
      const int32_t lo = run_lo[e * R + r];
      if (lo < 0) continue;
      const int32_t n = run_hi[e * R + r] - lo;
      w.g_lrow0[g] = pos;
      w.g_rows[g] = n;
      w.g_dst[g] = r;
      w.g_src0[g] = lo;
      if constexpr (kLds) {
        gl_lrow0[g] = pos;
        gl_rows[g] = n;
        gl_dst[g] = r;
      }
      if (a.overlapped) a.groups[g] = Group{e, pos, n, r};
      ++g;
      pos += n;
      if (a.overlapped && r != self) pos = base + round_up_i(pos - base, tb);
    }
  }

  // K parts of the down tiles: an explicit split_k splits every tile row; by default the tile
  // rows holding the last, partly filled round of kRoundTiles down tiles are split into as
  // many parts as fill that round.
  const int32_t dpr = a.down_per_row, gpr = a.gu_per_row;
  int32_t S = 1, n_split = 0;
  if (a.split_k > 0) {
    S = a.split_k;
    n_split = a.split_k > 1 ? n_tr : 0;
  } else if (n_tr > 0) {
    const int64_t rem = ((int64_t)n_tr * dpr) % kRoundTiles;
    if (rem > 0) {
      const int32_t rows = (int32_t)((rem + dpr - 1) / dpr);
      const int64_t s = kRoundTiles / ((int64_t)rows * dpr);
      const int32_t s2 = (int32_t)min(min(s, (int64_t)kMaxSplitK), (int64_t)a.nk);
      if (s2 > 1) {
        S = s2;
        n_split = rows;
      }
    }
  }
  const int32_t n_whole = n_tr - n_split;
  __syncthreads();

  // Tile rows, their schedule positions and row groups.  A position's class run [cs, ce) is
  // its expert's remote (or local-only) tile rows, consecutive in the schedule; the host's
  // greedy grouping in closed form: within the run, clipped to the range [a0, a1) being
  // grouped, groups of g positions start at max(cs, a0).
  const int32_t ggu = max(a.gu_group, 1), gdn = max(a.down_group, 1);
  for (int32_t t = tid; t < n_tr; t += kWg) {
    const int32_t e = range_of(ex_ntr, E_l, t);
    const int32_t j = t - ex_ntr[e], hr = ex_hr[e];
    const int32_t ntr_e = (e + 1 < E_l ? ex_ntr[e + 1] : n_tr) - ex_ntr[e];
    const int32_t t0 = t * kTileM;
    int32_t nvalid = 0, has_remote = 0;
    const int32_t g1 = e + 1 < E_l ? ex_ng[e + 1] : n_grp;
    for (int32_t g = ex_ng[e]; g < g1; ++g) {
      const int32_t L0 = gl_lrow0[g];
      const int32_t lo = max(t0, L0), hi = min(t0 + kTileM, L0 + gl_rows[g]);
      if (hi > lo) {
        nvalid += hi - lo;
        if (gl_dst[g] != self) has_remote = 1;
      }
    }
    int32_t cs, ce, q;
    if (j < hr) {
      cs = ex_roff[e];
      ce = cs + hr;
      q = cs + j;
    } else {
      cs = n_hr + ex_loff[e];
      ce = cs + (ntr_e - hr);
      q = cs + (j - hr);
    }
    w.order[q] = t;
    {
      const int32_t A = cs + (q - cs) / ggu * ggu;
      w.ga_gu[q] = A;
      w.gb_gu[q] = min(A + ggu, ce);
    }
    {
      const int32_t a0 = q < n_whole ? 0 : n_whole, a1 = q < n_whole ? n_whole : n_tr;
      const int32_t base = max(cs, a0);
      const int32_t A = base + (q - base) / gdn * gdn;
      w.ga_dn[q] = A;
      w.gb_dn[q] = min(A + gdn, min(ce, a1));
    }
    const bool split = q >= n_whole;
    a.tile_rows[t] = TileRow{e, t0, nvalid, has_remote, split ? S : 1, split ? (q - n_whole) * dpr * S : -1};
    if (split && a.split_k == 0) a.tail_rows[q - n_whole] = t;
    for (int32_t n = 0; n < dpr; ++n) w.pos_of_down[t * dpr + n] = -1;
  }

  // Queue bounds: each launch's item sequence dealt round-robin to the XCD queues in chunks of
  // kQueueChunk items (queue x holds chunks x, x + kXcds, ...).  Absolute item indices.
  const int32_t n_gu = n_tr * gpr;
  const int32_t n_down = n_whole * dpr + n_split * dpr * S;
  if (tid < 2) {
    const int32_t N = tid == 0 ? n_gu : n_down, base = tid == 0 ? 0 : n_gu;
    const int32_t nf = N / kQueueChunk, part = N % kQueueChunk;
    int32_t acc = 0, qmax = 0;
    for (int x = 0; x < kXcds; ++x) {
      a.queues[tid * (kXcds + 1) + x] = base + acc;
      int32_t L = (nf > x ? (nf - x + kXcds - 1) / kXcds : 0) * kQueueChunk;
      if (part && nf % kXcds == x) L += part;
      acc += L;
      qmax = max(qmax, L);
    }
    a.queues[tid * (kXcds + 1) + kXcds] = base + acc;
    if (tid == 1) H->down_qmax = qmax;
  }
  if (tid == 0) {
    H->n_tile_rows = n_tr;
    H->n_groups = a.overlapped ? n_grp : 0;
    H->n_groups_all = n_grp;
    H->n_gu = n_gu;
    H->n_down = n_down;
    H->n_segs = 0;
    H->tail_split = S;
    H->n_split_rows = n_split;
    H->n_partials = n_split * dpr * S;
    H->n_valid = a.off[E_l];
    H->n_lrows = (int64_t)n_tr * kTileM;
    H->n_band_pad = (int64_t)s_pad;
    H->n_remote = (int64_t)s_remote;
  }
}

__device__ __forceinline__ bool layout_in_lds(const DevPlanArgs& a) {
  return !a.no_lds && a.E_l <= kLdsExperts && (int64_t)a.E_l * a.R <= kLdsGroups;
}

__global__ __launch_bounds__(kWg) void plan_layout_kernel(DevPlanArgs a) {
  __shared__ int32_t lds[kLayoutLds];
  if (layout_in_lds(a))
    layout_phase<true>(a, lds);
  else
    layout_phase<false>(a, lds);
}

// ---------------------------------------------------------------------------------------------
// fill: work items, row tables, segment boundaries.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlk) void plan_fill_kernel(DevPlanArgs a) {
  __shared__ int32_t sh[kBlk];
  const PlanHeader* H = a.hdr;
  if (H->status != 0) return;
  const DevPlanWs& w = a.ws;
  const int32_t n_tr = H->n_tile_rows, n_gu = H->n_gu, n_down = H->n_down;
  const int32_t S = H->tail_split, n_whole = n_tr - H->n_split_rows, n_grp = H->n_groups_all;
  const int32_t gpr = a.gu_per_row, dpr = a.down_per_row;
  const int32_t gid = blockIdx.x * kBlk + threadIdx.x, gsz = gridDim.x * kBlk;

  // A sequence index s of a launch lies in the row group [A, B) of the schedule position
  // s / cols (every group of a range has the same columns), column-major within the group.
  for (int32_t s = gid; s < n_gu; s += gsz) {
    const int32_t p = s / gpr, A = w.ga_gu[p], m = w.gb_gu[p] - A, loc = s - A * gpr;
    const int32_t c = loc / m, q = A + loc % m;
    const int32_t ch = s / kQueueChunk, x = ch % kXcds;
    const int32_t pos = ch / kXcds * kQueueChunk + s % kQueueChunk;
    a.items[a.queues[x] + pos] = ((uint32_t)w.order[q] << kItemRowShift) | (uint32_t)c;
  }
  const int32_t n_wd = n_whole * dpr;
  for (int32_t s = gid; s < n_down; s += gsz) {
    int32_t p, A, loc;
    if (s < n_wd) {
      p = s / dpr;
      A = w.ga_dn[p];
      loc = s - A * dpr;
    } else {
      const int32_t cols = dpr * S, s2 = s - n_wd;
      p = n_whole + s2 / cols;
      A = w.ga_dn[p];
      loc = s2 - (A - n_whole) * cols;
    }
    const int32_t m = w.gb_dn[p] - A;
    const int32_t pc = loc / m, q = A + loc % m, t = w.order[q];
    const int32_t part = pc / dpr, n = pc % dpr;  // (part, column) pairs, part-major
    const int32_t ch = s / kQueueChunk, x = ch % kXcds;
    const int32_t pos = ch / kXcds * kQueueChunk + s % kQueueChunk;
    a.items[a.queues[kXcds + 1 + x] + pos] =
        kItemDown | ((uint32_t)t << kItemRowShift) | ((uint32_t)n << kDownColShift) | (uint32_t)part;
    atomicMax(&w.pos_of_down[t * dpr + n], pos);
  }

  // Logical rows, one tile row per workgroup pass.  A transfer group (Section 3.3.2) is cut at
  // tile-row boundaries into k pieces; its first and last pieces are one chunk each and the
  // middle ones coalesce mid_pieces at a time; a slot gap also starts a segment.
  const int32_t xm = max(a.mid_pieces, 1);
  const int tid = threadIdx.x;
  for (int32_t t = blockIdx.x; t < n_tr; t += gridDim.x) {
    const int32_t q = t * kTileM + tid;
    const int32_t e = a.tile_rows[t].expert;
    const int32_t g1 = e + 1 < a.E_l ? w.ex_ng[e + 1] : n_grp;
    int32_t g = -1;
    for (int32_t k = w.ex_ng[e]; k < g1; ++k)
      if (q >= w.g_lrow0[k] && q < w.g_lrow0[k] + w.g_rows[k]) {
        g = k;
        break;
      }
    int32_t start = 0, end = 0, np = 1;
    if (g >= 0) {
      const int32_t L0 = w.g_lrow0[g], L1 = L0 + w.g_rows[g];
      const int32_t i = w.g_src0[g] + (q - L0);
      const int32_t r = w.g_dst[g], sl = a.slot[i];
      a.row_x[q] = i;
      a.row_rank[q] = r;
      a.row_slot[q] = sl;
      if (a.overlapped && (r != a.self || !a.local_direct)) {
        const int32_t first_t = L0 / kTileM, k = (L1 - 1) / kTileM - first_t + 1, b = t - first_t;
        auto chunk_start = [&](int32_t pb) { return pb == 0 || k <= 2 || pb == k - 1 || (pb - 1) % xm == 0; };
        start = q == L0 || (q % kTileM == 0 && chunk_start(b)) || (int64_t)a.slot[i - 1] + 1 != sl;
        end = q == L1 - 1 || ((q + 1) % kTileM == 0 && chunk_start(b + 1)) ||
              (int64_t)a.slot[i + 1] != (int64_t)sl + 1;
        if (k > 2 && b > 0 && b < k - 1) {
          const int32_t cb = 1 + (b - 1) / xm * xm;
          np = min(cb + xm, k - 1) - cb;
        }
      }
    } else {
      a.row_x[q] = a.off[e];
      a.row_rank[q] = -1;
      a.row_slot[q] = -1;
    }
    // Compact this tile row's segment starts and ends (counts packed in one scan).
    const int32_t v = start | (end << 16);
    int32_t tot;
    const int32_t ex = wg_incl_scan<kBlk>(v, sh, &tot) - v;
    if (start) {
      w.start_q[t * kTileM + (ex & 0xFFFF)] = q;
      w.start_np[t * kTileM + (ex & 0xFFFF)] = np;
    }
    if (end) w.end_q[t * kTileM + (ex >> 16)] = q + 1;
    if (tid == 0) {
      w.cnt_s[t] = tot & 0xFFFF;
      w.cnt_e[t] = tot >> 16;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// segs: one workgroup pairs starts with ends, finishes each segment, and orders them by ready
// position, stably.
// ---------------------------------------------------------------------------------------------
constexpr int kLdsTileRows = 4096;  // per-tile-row counts in LDS up to this many tile rows
constexpr int kLdsHist = 8192;      // ready-position histogram in LDS up to this many positions

__global__ __launch_bounds__(kWg) void plan_segs_kernel(DevPlanArgs a) {
  __shared__ int32_t sh[kWg];
  __shared__ int32_t cnt_lds[2 * kLdsTileRows];
  __shared__ int32_t hist_lds[kLdsHist];
  PlanHeader* H = a.hdr;
  if (H->status != 0) return;
  const DevPlanWs& w = a.ws;
  const int32_t n_tr = H->n_tile_rows, K = H->down_qmax, dpr = a.down_per_row;
  const int tid = threadIdx.x;
  const bool c_in_lds = !a.no_lds && n_tr <= kLdsTileRows;
  int32_t* cs = c_in_lds ? cnt_lds : w.cnt_s;
  int32_t* ce = c_in_lds ? cnt_lds + kLdsTileRows : w.cnt_e;
  if (c_in_lds)
    for (int32_t t = tid; t < n_tr; t += kWg) {
      cs[t] = w.cnt_s[t];
      ce[t] = w.cnt_e[t];
    }
  __syncthreads();
  const int32_t n = wg_scan<kWg>(cs, n_tr, sh);
  wg_scan<kWg>(ce, n_tr, sh);  // the k-th end closes the k-th start's segment
  if (tid == 0) H->n_segs = n;
  if (n == 0) return;
  int32_t* hist = !a.no_lds && K <= kLdsHist ? hist_lds : w.hist;
  for (int32_t i = tid; i < K; i += kWg) hist[i] = 0;
  __syncthreads();
  for (int32_t k = tid; k < n; k += kWg) {
    const int32_t ts = range_of(cs, n_tr, k), te = range_of(ce, n_tr, k);
    const int32_t js = ts * kTileM + (k - cs[ts]);
    const int32_t q0 = w.start_q[js], q1 = w.end_q[te * kTileM + (k - ce[te])];
    Segment sg;
    sg.dst_rank = a.row_rank[q0];
    sg.rows = q1 - q0;
    sg.y_row0 = q0;
    sg.slot0 = a.row_slot[q0];
    const int32_t t0 = q0 / kTileM, t1 = (q1 - 1) / kTileM;
    sg.flag_begin = t0 * dpr;
    sg.flag_count = (t1 - t0 + 1) * dpr;
    int32_t rp = 0;
    for (int32_t f = sg.flag_begin; f < sg.flag_begin + sg.flag_count; ++f) rp = max(rp, w.pos_of_down[f]);
    sg.ready_pos = rp;
    sg.npieces = w.start_np[js];
    w.seg_tmp[k] = sg;
    w.seg_key[k] = rp;
    atomicAdd(&hist[rp], 1);
  }
  __syncthreads();
  wg_scan<kWg, true>(hist, K, sh);
  // Stable placement, kWg segments at a time: a segment goes after every earlier one with
  // the same ready position.
  for (int32_t c0 = 0; c0 < n; c0 += kWg) {
    const int32_t i = c0 + tid;
    const int32_t k = i < n ? w.seg_key[i] : -1;
    sh[tid] = k;
    __syncthreads();
    int32_t dest = 0;
    if (i < n) {
      int32_t rank = 0;
      for (int j = 0; j < tid; ++j) rank += sh[j] == k;
      dest = __hip_atomic_load(&hist[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + rank;
    }
    __syncthreads();
    if (i < n) {
      a.segs[dest] = w.seg_tmp[i];
      atomicAdd(&hist[k], 1);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Small plans: the run's reset and all four phases in one workgroup, every intermediate table in
// LDS.  A small plan's time is launches, cold instruction fetches and round trips to memory (each
// kernel re-reads what the one before it wrote, from beyond its XCD's L2), so this one reads the
// routing once, writes the tables once, and is short: the layout phase needs one wave, its scans
// shuffles.  Reset to plan ready, this kernel against init and the four kernels: 110 rows in 2 experts
// 18 against 30 us (overlapped plan 20, 36), 227 rows in 32 experts 27 against 39 (31, 52).
// The limits are where its tables fill the LDS; up to them it was the faster one everywhere (1774 rows
// in 32 experts 30 against 41, 1839 in 64 experts 36 against 39).
// ---------------------------------------------------------------------------------------------
constexpr int kSmallExperts = 64;     // one lane each
constexpr int kSmallGroups = 1024;    // (expert, rank) pairs
constexpr int kSmallRows = 2048;
constexpr int kSmallTileRows = 160;
constexpr int kSmallTiles = 8192;     // down tiles
constexpr int kSmallItems = 8192;
constexpr int kSmallSeen = 2 * kSmallRows;
constexpr int kSmallRowBits = 11;     // a segment's place in layout order, in the sort key below its ready position
static_assert((1 << kSmallRowBits) >= kSmallRows && kSmallItems < (1 << (30 - kSmallRowBits)), "segment sort key");

__device__ __forceinline__ int32_t wave_incl_scan(int32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

// A workgroup barrier for LDS alone: nothing this kernel writes to memory is read back in it, so its
// stores need not complete first (a plain barrier waits for them, about a microsecond each time).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__global__ __launch_bounds__(kWg) void plan_small_kernel(DevPlanArgs a, InitArgs ia) {
  __shared__ unsigned long long seen[kSmallSeen];
  __shared__ int32_t src[kSmallRows], slot[kSmallRows + 1], off[kSmallExperts + 1];
  __shared__ int64_t rrows[kSmallGroups];
  __shared__ int32_t run_lo[kSmallGroups], run_hi[kSmallGroups];
  __shared__ int32_t g_lrow0[kSmallGroups], g_rows[kSmallGroups], g_dst[kSmallGroups], g_src0[kSmallGroups], g_c0[kSmallGroups];
  __shared__ int32_t ex_ntr[kSmallExperts + 1], ex_ng[kSmallExperts + 1], ex_hr[kSmallExperts], ex_roff[kSmallExperts],
      ex_loff[kSmallExperts], ex_tmp[kSmallExperts];
  __shared__ int32_t tr_e[kSmallTileRows], order[kSmallTileRows], ga_gu[kSmallTileRows], gb_gu[kSmallTileRows],
      ga_dn[kSmallTileRows], gb_dn[kSmallTileRows];
  __shared__ int32_t pos_of_down[kSmallTiles];
  __shared__ int32_t start_q[kSmallRows], start_np[kSmallRows], end_q[kSmallRows];
  __shared__ __attribute__((aligned(16))) int32_t key[kSmallRows + 16];
  __shared__ int32_t queues[2 * (kXcds + 1)], sh[kWg / 64];
  __shared__ int32_t s_code, s_bad, s_pad, s_remote, s_qmax;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int32_t E_l = a.E_l, R = a.R, self = a.self;
  if (ia.ctr) reset_run(ia, tid, kWg);

  // Routing into LDS; the checks of the rows kernel.
  for (int i = tid; i < kSmallSeen; i += kWg) seen[i] = ~0ull;
  for (int i = tid; i < E_l * R; i += kWg) run_lo[i] = -1;
  if (tid == 0) s_code = s_pad = s_remote = 0, s_bad = INT_MAX;
  if (tid <= E_l) off[tid] = a.off[tid];
  for (int r = tid; r < R; r += kWg) rrows[r] = ia.n_ret ? ia.ret_rows[r] : a.return_rows[r];
  lds_barrier();
  const int32_t rows = off[E_l];
  if (tid < E_l && off[tid] > off[tid + 1]) s_code = MOE_EROUTING;
  if (tid == 0 && off[0] != 0) s_code = MOE_EROUTING;
  lds_barrier();
  int32_t code = rows < 0 ? MOE_EROUTING : rows > a.max_rows ? MOE_ECAPACITY : s_code;
  if (code == 0) {
    for (int i = tid; i < rows; i += kWg) {
      src[i] = a.src[i];
      slot[i] = a.slot[i];
    }
    lds_barrier();
    for (int i = tid; i < rows; i += kWg) {
      const int32_t r = src[i], s = slot[i];
      const int32_t e = range_of(off, E_l, i);
      bool bad = r < 0 || r >= R || s < 0 || (int64_t)s >= rrows[r < 0 || r >= R ? 0 : r];
      if (!bad) {
        const bool first = i == off[e] || src[i - 1] != r;
        const bool last = i == off[e + 1] - 1 || src[i + 1] != r;
        if (!first && slot[i - 1] >= s) bad = true;                          // slots ascend within a rank's run
        if (first && atomicCAS(&run_lo[e * R + r], -1, i) != -1) bad = true;  // a second run
        if (last) run_hi[e * R + r] = i + 1;
        if (seen_insert((uint64_t*)seen, kSmallSeen, ((uint64_t)r << 32) | (uint32_t)s)) bad = true;
      }
      if (bad) {
        atomicMin(&s_bad, i);
        s_code = MOE_EROUTING;
      }
    }
    lds_barrier();
    code = s_code;
  }

  // Layout: lane e of wave 0 takes expert e (see the layout kernel for each closed form).
  const int32_t tb = a.overlapped ? a.tb : 1, tb_shift = 31 - __clz(tb);  // a power of two
  int32_t ntr = 0, ng = 0, hr = 0, bands = 0;
  if (code == 0 && wv == 0) {
    int32_t pos = 0, remote_end = 0, pad = 0, remote = 0;
    if (lane < E_l) {
#pragma unroll 4
      for (int32_t j = 0; j < R; ++j) {
        const int32_t r = rank_at(j, R, self), lo = run_lo[lane * R + r], hi = run_hi[lane * R + r];
        const int32_t n = lo < 0 ? 0 : hi - lo;
        ng += n > 0;
        pos += n;
        if (r != self && n > 0) {
          remote += n;
          bands += (n + tb - 1) >> tb_shift;
          remote_end = pos;
          const int32_t p = -pos & (tb - 1);  // none in the baseline's layout (tb = 1)
          pad += p;
          pos += p;
        }
      }
      ntr = round_up_i(pos, kTileM) / kTileM;
      hr = remote_end > 0 ? (remote_end - 1) / kTileM + 1 : 0;
      if (pad) atomicAdd(&s_pad, pad);
      if (remote) atomicAdd(&s_remote, remote);
    }
    const int32_t it = wave_incl_scan(ntr), ig = wave_incl_scan(ng);
    ex_ntr[lane + 1] = it;
    ex_ng[lane + 1] = ig;
    if (lane == 0) ex_ntr[0] = ex_ng[0] = 0;
    // Schedule position of each expert's remote tile rows: experts by bands, descending, ties by id.
    int32_t rank = 0;
#pragma unroll 1
    for (int f = 0; f < E_l; ++f) {
      const int32_t c = __builtin_amdgcn_readlane(bands, f);
      rank += c > bands || (c == bands && f < lane);
    }
    if (lane < E_l) {
      ex_hr[lane] = hr;
      ex_tmp[rank] = hr;
    }
    __builtin_amdgcn_wave_barrier();
    const int32_t h = lane < E_l ? ex_tmp[lane] : 0;
    const int32_t ih = wave_incl_scan(h), n_hr = __shfl(ih, 63, 64);
    __builtin_amdgcn_wave_barrier();
    if (lane < E_l) ex_tmp[lane] = ih - h;
    __builtin_amdgcn_wave_barrier();
    const int32_t local = ntr - hr, il = wave_incl_scan(local);
    if (lane < E_l) {
      ex_roff[lane] = ex_tmp[rank];
      ex_loff[lane] = n_hr + il - local;
      // Owner groups with their places in the padded layout.
      const int32_t base = (it - ntr) * kTileM;
      int32_t g = ig - ng, p = base, c = off[lane];
#pragma unroll 2
      for (int32_t j = 0; j < R; ++j) {
        const int32_t r = rank_at(j, R, self), lo = run_lo[lane * R + r], hi = run_hi[lane * R + r];
        if (lo < 0) continue;
        const int32_t n = hi - lo;
        g_lrow0[g] = p;
        g_rows[g] = n;
        g_dst[g] = r;
        g_src0[g] = lo;
        g_c0[g] = c;
        c += n;
        if (a.overlapped) a.groups[g] = Group{lane, p, n, r};
        ++g;
        p += n;
        if (r != self) p += -(p - base) & (tb - 1);
      }
    }
  }
  lds_barrier();
  const int32_t n_tr = code == 0 ? ex_ntr[E_l] : 0, n_grp = code == 0 ? ex_ng[E_l] : 0;
  if (code == 0 && n_tr > a.max_tile_rows) code = MOE_ECAPACITY;
  if (code) {
    if (tid == 0) {
      a.hdr->status = code;
      a.hdr->bad_row = s_bad;
    }
    write_empty(a);
    return;
  }

  // K parts, tile rows, schedule positions and row groups, queue bounds.
  const uint32_t dpr = (uint32_t)a.down_per_row, gpr = (uint32_t)a.gu_per_row;
  int32_t S = 1, n_split = 0;
  if (a.split_k > 0) {
    S = a.split_k;
    n_split = a.split_k > 1 ? n_tr : 0;
  } else {
    const uint32_t rem = (uint32_t)n_tr * dpr % (uint32_t)kRoundTiles;
    if (rem > 0) {
      const uint32_t r = (rem + dpr - 1) / dpr;
      const int32_t s2 = min(min((int32_t)((uint32_t)kRoundTiles / (r * dpr)), kMaxSplitK), a.nk);
      if (s2 > 1) S = s2, n_split = (int32_t)r;
    }
  }
  const int32_t n_whole = n_tr - n_split;
  const int32_t n_gu = n_tr * (int32_t)gpr, n_down = n_whole * (int32_t)dpr + n_split * (int32_t)dpr * S;
  if (tid < n_tr) {
    const int32_t t = tid, e = range_of(ex_ntr, E_l, t);
    const int32_t j = t - ex_ntr[e], ehr = ex_hr[e], t0 = t * kTileM;
    int32_t nvalid = 0, has_remote = 0;
#pragma unroll 1
    for (int32_t g = ex_ng[e]; g < ex_ng[e + 1]; ++g) {
      const int32_t lo = max(t0, g_lrow0[g]), hi = min(t0 + kTileM, g_lrow0[g] + g_rows[g]);
      if (hi > lo) {
        nvalid += hi - lo;
        if (g_dst[g] != self) has_remote = 1;
      }
    }
    const bool rem = j < ehr;
    const int32_t cs = rem ? ex_roff[e] : ex_loff[e];
    const int32_t ce = cs + (rem ? ehr : ex_ntr[e + 1] - ex_ntr[e] - ehr);
    const int32_t q = cs + (rem ? j : j - ehr);
    const int32_t ggu = max(a.gu_group, 1), gdn = max(a.down_group, 1);
    tr_e[t] = e;
    order[q] = t;
    const int32_t A = cs + (int32_t)((uint32_t)(q - cs) / (uint32_t)ggu) * ggu;
    ga_gu[q] = A;
    gb_gu[q] = min(A + ggu, ce);
    const bool split = q >= n_whole;
    const int32_t a0 = split ? n_whole : 0, a1 = split ? n_tr : n_whole, base = max(cs, a0);
    const int32_t D = base + (int32_t)((uint32_t)(q - base) / (uint32_t)gdn) * gdn;
    ga_dn[q] = D;
    gb_dn[q] = min(D + gdn, min(ce, a1));
    a.tile_rows[t] = TileRow{e, t0, nvalid, has_remote, split ? S : 1, split ? (q - n_whole) * (int32_t)dpr * S : -1};
    if (split && a.split_k == 0) a.tail_rows[q - n_whole] = t;
  }
  for (int i = tid; i < n_tr * (int32_t)dpr; i += kWg) pos_of_down[i] = -1;
  if (wv == kWg / 64 - 1 && lane < 2) {  // a wave of its own: one lane per launch
    const int32_t N = lane == 0 ? n_gu : n_down;
    const int32_t nf = N / kQueueChunk, part = N % kQueueChunk;
    int32_t acc = lane == 0 ? 0 : n_gu, qmax = 0;
#pragma unroll 1
    for (int x = 0; x <= kXcds; ++x) {
      queues[lane * (kXcds + 1) + x] = acc;
      a.queues[lane * (kXcds + 1) + x] = acc;
      int32_t L = (nf > x ? (nf - x + kXcds - 1) / kXcds : 0) * kQueueChunk;
      if (part && nf % kXcds == x) L += part;
      if (x < kXcds) acc += L, qmax = max(qmax, L);
    }
    if (lane == 1) s_qmax = qmax;
  }
  lds_barrier();

  // Work items, to their queue slots: one loop over both launches.
  for (int32_t i = tid; i < n_gu + n_down; i += kWg) {
    const bool down = i >= n_gu;
    const uint32_t s = (uint32_t)(down ? i - n_gu : i), n_wd = (uint32_t)n_whole * dpr;
    const bool tail = down && s >= n_wd;
    const uint32_t cols = !down ? gpr : tail ? dpr * (uint32_t)S : dpr;
    const uint32_t p0 = tail ? (uint32_t)n_whole : 0u, s2 = tail ? s - n_wd : s;
    const uint32_t p = p0 + s2 / cols;
    const uint32_t A = (uint32_t)(down ? ga_dn[p] : ga_gu[p]), m = (uint32_t)(down ? gb_dn[p] : gb_gu[p]) - A;
    const uint32_t loc = s2 - (A - p0) * cols, c = loc / m, q = A + (loc - c * m);
    const uint32_t t = (uint32_t)order[q];
    const uint32_t ch = s / kQueueChunk, x = ch % kXcds, pos = ch / kXcds * kQueueChunk + s % kQueueChunk;
    uint32_t item = (t << kItemRowShift) | c;
    if (down) {
      const uint32_t part = c / dpr, n = c - part * dpr;  // (part, column) pairs, part-major
      item = kItemDown | (t << kItemRowShift) | (n << kDownColShift) | part;
      atomicMax(&pos_of_down[t * dpr + n], (int32_t)pos);
    }
    a.items[queues[(down ? kXcds + 1 : 0) + x] + (int32_t)pos] = item;
  }

  // Row tables.
#pragma unroll 1
  for (int32_t q = tid; q < n_tr * kTileM; q += kWg) {
    const int32_t e = tr_e[q / kTileM], g0 = ex_ng[e];
    const int32_t g = g0 + range_of(g_lrow0 + g0, ex_ng[e + 1] - g0, q), d = q - g_lrow0[g];
    const bool routed = d < g_rows[g];
    const int32_t row = routed ? g_src0[g] + d : off[e];
    a.row_x[q] = row;
    a.row_rank[q] = routed ? g_dst[g] : -1;
    a.row_slot[q] = routed ? slot[row] : -1;
  }

  // Segment boundaries, kWg routed rows at a time in logical order (group by group); the running
  // counts pair the k-th start with the k-th end.
  const int32_t xm = max(a.mid_pieces, 1);
  int32_t n_seg = 0, n_end = 0;
#pragma unroll 1
  for (int32_t c0 = 0; a.overlapped && c0 < rows; c0 += kWg) {
    const int32_t c = c0 + tid;
    int32_t start = 0, end = 0, np = 1, q = 0;
    if (c < rows) {
      const int32_t g = range_of(g_c0, n_grp, c), d = c - g_c0[g];
      const int32_t L0 = g_lrow0[g], n = g_rows[g], row = g_src0[g] + d, sl = slot[row];
      q = L0 + d;
      if (g_dst[g] != self || !a.local_direct) {
        const int32_t L1 = L0 + n, t = q / kTileM;
        const int32_t first_t = L0 / kTileM, k = (L1 - 1) / kTileM - first_t + 1, b = t - first_t;
        auto chunk_start = [&](int32_t pb) {
          return pb == 0 || k <= 2 || pb == k - 1 || (uint32_t)(pb - 1) % (uint32_t)xm == 0;
        };
        start = d == 0 || (q % kTileM == 0 && chunk_start(b)) || (int64_t)slot[row - 1] + 1 != sl;
        end = d == n - 1 || ((q + 1) % kTileM == 0 && chunk_start(b + 1)) ||
              (int64_t)slot[row + 1] != (int64_t)sl + 1;
        if (k > 2 && b > 0 && b < k - 1) {
          const int32_t cb = 1 + (int32_t)((uint32_t)(b - 1) / (uint32_t)xm) * xm;
          np = min(cb + xm, k - 1) - cb;
        }
      }
    }
    // Starts and ends counted together, 16 bits each (at most kWg a pass): by ballot in a wave, and
    // every wave scans the waves' counts for itself.
    const uint64_t ms = __ballot(start), me = __ballot(end), below = (1ull << lane) - 1;
    if (lane == 0) sh[wv] = __popcll(ms) | (__popcll(me) << 16);
    lds_barrier();
    int32_t upto = lane < kWg / 64 ? sh[lane] : 0;
#pragma unroll
    for (int d = 1; d < kWg / 64; d <<= 1) {
      const int32_t y = __shfl_up(upto, d, 64);
      if (lane >= d) upto += y;
    }
    const int32_t total = __builtin_amdgcn_readlane(upto, kWg / 64 - 1);
    const int32_t ex = (wv ? __shfl(upto, wv - 1, 64) : 0) + (__popcll(ms & below) | (__popcll(me & below) << 16));
    if (start) {
      start_q[n_seg + (ex & 0xFFFF)] = q;
      start_np[n_seg + (ex & 0xFFFF)] = np;
    }
    if (end) end_q[n_end + (ex >> 16)] = q + 1;
    n_seg += total & 0xFFFF;
    n_end += total >> 16;
    lds_barrier();
  }
  lds_barrier();

  // Segments in layout order, then each to its place in ready order: after every segment ready
  // before it and every earlier one ready with it.
  auto ready = [&](int32_t q0, int32_t q1) {
    const int32_t f1 = ((q1 - 1) / kTileM + 1) * (int32_t)dpr;
    int32_t rp = 0;
#pragma unroll 4
    for (int32_t f = q0 / kTileM * (int32_t)dpr; f < f1; ++f) rp = max(rp, pos_of_down[f]);
    return rp;
  };
  for (int32_t k = tid; k < n_seg; k += kWg) key[k] = (ready(start_q[k], end_q[k]) << kSmallRowBits) | k;
  if (tid < 16) key[n_seg + tid] = INT_MAX;
  lds_barrier();
#pragma unroll 1
  for (int32_t k = tid; k < n_seg; k += kWg) {
    const int32_t mine = key[k];
    int32_t dest = 0;
#pragma unroll 4
    for (int32_t j = 0; j < n_seg; j += 4) {
      const int4 v = *(const int4*)&key[j];
      dest += (v.x < mine) + (v.y < mine) + (v.z < mine) + (v.w < mine);
    }
    const int32_t q0 = start_q[k], q1 = end_q[k], t0 = q0 / kTileM, t1 = (q1 - 1) / kTileM;
    const int32_t e = tr_e[t0];
    const int32_t g = ex_ng[e] + range_of(g_lrow0 + ex_ng[e], ex_ng[e + 1] - ex_ng[e], q0);
    Segment sg;
    sg.dst_rank = g_dst[g];
    sg.rows = q1 - q0;
    sg.y_row0 = q0;
    sg.slot0 = slot[g_src0[g] + (q0 - g_lrow0[g])];
    sg.flag_begin = t0 * (int32_t)dpr;
    sg.flag_count = (t1 - t0 + 1) * (int32_t)dpr;
    sg.ready_pos = mine >> kSmallRowBits;
    sg.npieces = start_np[k];
    a.segs[dest] = sg;
  }
  if (tid == 0) {
    PlanHeader h{};
    h.bad_row = INT_MAX;
    h.n_tile_rows = n_tr;
    h.n_groups = a.overlapped ? n_grp : 0;
    h.n_groups_all = n_grp;
    h.n_gu = n_gu;
    h.n_down = n_down;
    h.n_segs = n_seg;
    h.tail_split = S;
    h.n_split_rows = n_split;
    h.n_partials = n_split * (int32_t)dpr * S;
    h.down_qmax = s_qmax;
    h.n_valid = rows;
    h.n_lrows = (int64_t)n_tr * kTileM;
    h.n_band_pad = s_pad;
    h.n_remote = s_remote;
    *a.hdr = h;
  }
}

// Plans the single-workgroup planner takes, by capacity (the host does not know the routing).
bool small_plan(const DevPlanArgs& a, int64_t max_items) {
  return !a.no_lds && a.E_l <= kSmallExperts && (int64_t)a.E_l * a.R <= kSmallGroups && a.max_rows <= kSmallRows &&
         a.max_tile_rows <= kSmallTileRows && (int64_t)a.max_tile_rows * a.down_per_row <= kSmallTiles &&
         max_items <= kSmallItems;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct WsLayout {
  size_t run_lo, run_hi, seen, ex, g, order, ga, pod, lists, cnt, seg_tmp, seg_key, hist, total;
  int64_t seen_cap;
};

WsLayout ws_layout(int32_t E_l, int32_t R, int32_t max_rows, int32_t max_tile_rows, int32_t dpr,
                   int64_t max_lrows, int64_t max_items) {
  WsLayout L{};
  int64_t cap = 64;
  while (cap < 2 * (int64_t)max_rows) cap <<= 1;
  L.seen_cap = cap;
  const size_t er = (size_t)E_l * R;
  size_t o = 0;
  // run_lo, run_hi and seen are contiguous (one all-ones fill); seen is 8-byte aligned.
  L.run_lo = o;   o += 4 * er;
  L.run_hi = o;   o += 4 * er;
  o = (o + 7) & ~(size_t)7;
  L.seen = o;     o += 8 * (size_t)cap;
  o = align256(o);
  L.ex = o;       o = align256(o + 4 * 7 * (size_t)E_l);
  L.g = o;        o = align256(o + 4 * 4 * er);
  L.order = o;    o = align256(o + 4 * (size_t)max_tile_rows);
  L.ga = o;       o = align256(o + 4 * 4 * (size_t)max_tile_rows);
  L.pod = o;      o = align256(o + 4 * (size_t)max_tile_rows * dpr);
  L.lists = o;    o = align256(o + 4 * 3 * (size_t)max_lrows);
  L.cnt = o;      o = align256(o + 4 * 2 * (size_t)max_tile_rows);
  L.seg_tmp = o;  o = align256(o + sizeof(Segment) * (size_t)max_lrows);
  L.seg_key = o;  o = align256(o + 4 * (size_t)max_lrows);
  L.hist = o;     o = align256(o + 4 * (size_t)(max_items + 1));
  L.total = o;
  return L;
}

}  // namespace

size_t devplan_ws_bytes(int32_t E_l, int32_t R, int32_t max_rows, int32_t max_tile_rows,
                        int32_t down_per_row, int64_t max_lrows, int64_t max_items) {
  return ws_layout(E_l, R, max_rows, max_tile_rows, down_per_row, max_lrows, max_items).total;
}

DevPlanWs devplan_ws_carve(void* base_, int32_t E_l, int32_t R, int32_t max_rows, int32_t max_tile_rows,
                           int32_t down_per_row, int64_t max_lrows, int64_t max_items) {
  const WsLayout L = ws_layout(E_l, R, max_rows, max_tile_rows, down_per_row, max_lrows, max_items);
  uint8_t* b = (uint8_t*)base_;
  DevPlanWs w{};
  w.run_lo = (int32_t*)(b + L.run_lo);
  w.run_hi = (int32_t*)(b + L.run_hi);
  w.seen = (uint64_t*)(b + L.seen);
  w.seen_cap = L.seen_cap;
  w.fill_words = (int64_t)((L.seen + 8 * (size_t)L.seen_cap - L.run_lo) / 4);
  int32_t* ex = (int32_t*)(b + L.ex);
  w.ex_ntr = ex;
  w.ex_ng = ex + E_l;
  w.ex_hr = ex + 2 * E_l;
  w.ex_bands = ex + 3 * E_l;
  w.ex_roff = ex + 4 * E_l;
  w.ex_loff = ex + 5 * E_l;
  w.tmp = ex + 6 * E_l;
  const size_t er = (size_t)E_l * R;
  int32_t* g = (int32_t*)(b + L.g);
  w.g_lrow0 = g;
  w.g_rows = g + er;
  w.g_dst = g + 2 * er;
  w.g_src0 = g + 3 * er;
  w.order = (int32_t*)(b + L.order);
  int32_t* ga = (int32_t*)(b + L.ga);
  w.ga_gu = ga;
  w.gb_gu = ga + max_tile_rows;
  w.ga_dn = ga + 2 * (size_t)max_tile_rows;
  w.gb_dn = ga + 3 * (size_t)max_tile_rows;
  w.pos_of_down = (int32_t*)(b + L.pod);
  int32_t* lists = (int32_t*)(b + L.lists);
  w.start_q = lists;
  w.start_np = lists + max_lrows;
  w.end_q = lists + 2 * max_lrows;
  w.cnt_s = (int32_t*)(b + L.cnt);
  w.cnt_e = w.cnt_s + max_tile_rows;
  w.seg_tmp = (Segment*)(b + L.seg_tmp);
  w.seg_key = (int32_t*)(b + L.seg_key);
  w.hist = (int32_t*)(b + L.hist);
  return w;
}

hipError_t launch_devplan(const DevPlanArgs& a, const InitArgs& init, int64_t max_items, int num_cus, hipStream_t s) {
  if (small_plan(a, max_items)) {
    // One workgroup resets the run too, but for what only testing and timing flags ask for (fills as
    // large as the staged output).
    InitArgs ia = init;
    ia.fill_ones = nullptr;
    ia.plan_hdr = nullptr;
    if (init.poison || init.wcount || init.tile_ready || init.publish) {
      const hipError_t e = launch_init(ia, s);
      if (e != hipSuccess) return e;
      ia.ctr = nullptr;
    }
    hipLaunchKernelGGL(plan_small_kernel, dim3(1), dim3(kWg), 0, s, a, ia);
    return hipGetLastError();
  }
  const hipError_t e = launch_init(init, s);
  if (e != hipSuccess) return e;
  const int64_t wide = (int64_t)std::max(num_cus, 1) * 4;
  const int rows_grid = (int)std::max<int64_t>(1, std::min<int64_t>(wide, ((int64_t)a.max_rows + kBlk - 1) / kBlk));
  // The fill kernel: a workgroup per tile row, and enough threads for the work items.
  const int fill_grid = (int)std::max<int64_t>(
      1, std::min<int64_t>(wide, std::max<int64_t>(a.max_tile_rows, (max_items + kBlk - 1) / kBlk)));
  hipLaunchKernelGGL(plan_rows_kernel, dim3(rows_grid), dim3(kBlk), 0, s, a);
  hipLaunchKernelGGL(plan_layout_kernel, dim3(1), dim3(kWg), 0, s, a);
  hipLaunchKernelGGL(plan_fill_kernel, dim3(fill_grid), dim3(kBlk), 0, s, a);
  if (a.overlapped) hipLaunchKernelGGL(plan_segs_kernel, dim3(1), dim3(kWg), 0, s, a);
  return hipGetLastError();
}

}  // namespace moe
