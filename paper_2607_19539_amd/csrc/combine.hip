// combine.hip -- gfx950 kernel of the weighted combine on a source rank (paper Section 2.1,
// step 5): each token's k returned expert rows, weighted by the router's gate values, summed
// in fp32 and rounded to bf16.  HBM-bound gather: every row is read once with 16-byte
// vector loads and the output row is written once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.hpp"

namespace moe {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 g_u32x4;
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two floats -> two bf16, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t to_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Up to this many workgroups a call leaves compute units idle and its time is a chain of loads
// (slots, rows, the next batch's): then one vector per thread, so a token spreads over more
// workgroups, and with over four choices eight rows in flight instead of four.
constexpr int64_t kFewWorkgroups = 512;

// out[t] = bf16(sum_j gate[t, j] * recv[slot[t, j]]).
// A workgroup covers kVec * 256 16-byte vectors of one token's row; each thread keeps
// kVec * 8 fp32 sums.  The k choices are taken kBatch at a time: the rows of a batch are
// loaded together, then added in choice order as separately rounded products and sums
// (contraction off), so the result does not depend on the batching.  Out-of-range
// slots are skipped and counted.
template <int kVec, int kBatch>
__device__ __forceinline__ void combine_rows(const CombineArgs& a) {
#pragma clang fp contract(off)
  const int64_t nvec = a.H / 8;
  const int64_t spans = (nvec + 256 * kVec - 1) / (256 * kVec);
  const int64_t work = a.tokens * spans;
  for (int64_t w = blockIdx.x; w < work; w += gridDim.x) {
    const int64_t t = w / spans;
    const int64_t span = w - t * spans;
    const int64_t v0 = span * (256 * kVec) + threadIdx.x;
    float acc[kVec][8];
#pragma unroll
    for (int u = 0; u < kVec; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[u][e] = 0.0f;
    for (int j0 = 0; j0 < a.k; j0 += kBatch) {
      u32x4 v[kBatch][kVec];
      float g[kBatch];
      bool ok[kBatch];
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        const int j = j0 + jj;
        const int32_t s = j < a.k ? a.slot[t * a.k + j] : -1;
        ok[jj] = s >= 0 && (int64_t)s < a.recv_rows;
        if (j < a.k && !ok[jj] && span == 0 && threadIdx.x == 0 && a.bad_slots)
          atomicAdd(a.bad_slots, 1u);
        g[jj] = ok[jj] ? a.gate[t * a.k + j] : 0.0f;
        const u32x4* row = (const u32x4*)(a.recv + (int64_t)(ok[jj] ? s : 0) * a.H);
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
          const int64_t i = v0 + u * 256;
          v[jj][u] = (ok[jj] && i < nvec) ? row[i] : u32x4{0u, 0u, 0u, 0u};
        }
      }
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        if (!ok[jj]) continue;
#pragma unroll
        for (int u = 0; u < kVec; ++u)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t word = v[jj][u][q];
            const float lo = __uint_as_float(word << 16), hi = __uint_as_float(word & 0xFFFF0000u);
            acc[u][2 * q] = acc[u][2 * q] + g[jj] * lo;
            acc[u][2 * q + 1] = acc[u][2 * q + 1] + g[jj] * hi;
          }
      }
    }
    g_u32x4* dst = (g_u32x4*)(a.out + t * a.H);
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const int64_t i = v0 + u * 256;
      if (i < nvec) {
        u32x4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = to_bf16x2(acc[u][2 * q], acc[u][2 * q + 1]);
        dst[i] = o;
      }
    }
  }
}

// Eight choices a batch where few workgroups run: 48 tokens of 8 rows of 14 KiB 6.2 -> 4.1 us, 16 of 6
// rows of 4 KiB 3.6 -> 3.5; with four or fewer choices, or many workgroups (4096 tokens of 6 rows of
// 4 KiB 19.1 -> 20.2), the wider batch only costs registers.
// It rides on the two-vector kernel, whose registers it fits, so the one-vector kernel keeps its own.
template <int kVec>
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a) {
  if (kVec == 2 && a.few)
    combine_rows<1, 8>(a);
  else
    combine_rows<kVec, 4>(a);
}

hipError_t launch_combine(const CombineArgs& args, hipStream_t s) {
  if (args.tokens <= 0) return hipSuccess;
  CombineArgs a = args;
  const int64_t nvec = a.H / 8;
  int vec = nvec <= 256 ? 1 : nvec <= 512 ? 2 : 4;
  // With four or fewer choices one batch holds them, and the spread costs more than it gives
  // (16 tokens of 2 rows of 8 KiB 2.85 -> 2.92 us).
  a.few = a.k > 4 && a.tokens * ((nvec + 256 * vec - 1) / (256 * vec)) < kFewWorkgroups;
  const int width = a.few ? 256 : 256 * vec;
  const int64_t spans = (nvec + width - 1) / width;
  const int grid = (int)std::min<int64_t>(a.tokens * spans, 65536);
  if (a.few || vec == 2)
    hipLaunchKernelGGL(combine_kernel<2>, dim3(grid), dim3(256), 0, s, a);
  else if (vec == 1)
    hipLaunchKernelGGL(combine_kernel<1>, dim3(grid), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(combine_kernel<4>, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace moe
