// init_device.hpp -- the reset that precedes every run, as a device function: a kernel of its own,
// or the first phase of the single-workgroup planner.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stddef.h>
#include <stdint.h>

#include "kernels.hpp"

namespace moe {

// Thread i of `stride` threads resets its share of the run's state.
__device__ __forceinline__ void reset_run(const InitArgs& a, int64_t i, int64_t stride) {
  // The counters word by word: all zero but prod_t0 (all ones, a minimum is taken), and the sticky
  // watchdog reports and the epoch left alone.
  constexpr int64_t kCtrWords = offsetof(RunCounters, pad_) / 4;
  for (int64_t j = i; j < kCtrWords; j += stride) {
    if (j >= (int64_t)offsetof(RunCounters, timeouts) / 4 && j <= (int64_t)offsetof(RunCounters, timeout_seg) / 4) continue;
    if (j >= (int64_t)offsetof(RunCounters, go) / 4 && j < (int64_t)offsetof(RunCounters, units_pub) / 4) continue;
    const bool t0 = j == (int64_t)offsetof(RunCounters, prod_t0) / 4 || j == (int64_t)offsetof(RunCounters, prod_t0) / 4 + 1;
    ((uint32_t*)a.ctr)[j] = t0 ? ~0u : 0u;
  }
  // The upload of a host-built plan: read over the host link by the kernel that has to run anyway
  // (a copy before it is an engine of its own to start and to wait for: 49000 rows in 16 experts, stage
  // 658 -> 639 us; with the table below, 227 rows in 32 experts 534 -> 508, 110 rows in two 36 -> 32).
  if (a.up_src) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    for (int64_t j = i; j < a.up_n16; j += stride) ((u32x4*)a.up_dst)[j] = ((const u32x4*)a.up_src)[j];
  }
  if (i < a.n_ret) {
    a.ret_dst[i] = a.ret[i];
    a.ret_rows_dst[i] = a.ret_rows[i];
  }
  if (i == 0 && a.plan_hdr) {
    a.plan_hdr->status = 0;
    a.plan_hdr->bad_row = INT_MAX;
  }
  if (a.fill_ones)
    for (int64_t j = i; j < a.n_fill_ones; j += stride) a.fill_ones[j] = ~0u;
  for (int64_t j = i; j < a.n_arrivals; j += stride) a.arrivals[j] = 0;
  if (a.wcount)
    for (int64_t j = i; j < a.n_wcount; j += stride) a.wcount[j] = 0;
  if (a.tile_ready)
    for (int64_t j = i; j < a.n_arrivals; j += stride) a.tile_ready[j] = 0;
  if (a.simd_waves)
    for (int64_t j = i; j < kWaveCounters; j += stride) a.simd_waves[j] = 0;
  // Published flags are stored as the producer raises them (relaxed, agent scope): a plain store
  // would sit in this XCD's L2, and the consumer's polls on other XCDs would not see it until the
  // line is written back.
  if (a.publish)
    for (int64_t j = i; j < a.n_publish; j += stride)
      __hip_atomic_store(&a.publish[j], a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (a.poison) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 nan = {0x7FC07FC0u, 0x7FC07FC0u, 0x7FC07FC0u, 0x7FC07FC0u};
    for (int64_t j = i; j < a.poison_elems / 8; j += stride) ((u32x4*)a.poison)[j] = nan;
  }
}
static_assert(offsetof(RunCounters, timeout_where) == offsetof(RunCounters, timeouts) + 4 &&
                  offsetof(RunCounters, timeout_seg) == offsetof(RunCounters, timeouts) + 8,
              "the sticky reports are adjacent");

}  // namespace moe
