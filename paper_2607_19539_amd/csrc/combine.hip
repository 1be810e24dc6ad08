// combine.hip -- gfx950 kernel of the weighted combine on a source rank (paper Section 2.1,
// step 5): each token's k returned expert rows, weighted by the router's gate values, summed
// in fp32 and rounded to bf16.  Every row is read once with 16-byte vector loads and the output row is
// written once.  Many tokens are bound by memory (4096 of 2 rows of 8 KiB 15.8 us, 6.4 TB/s); few by the
// chain from slots to rows, so a batch's rows have to be in flight together.  With the slots loaded as
// vectors each waited for the row loads before it, one row at a time: 48 tokens of 8 rows of 14 KiB took
// 4.0 us, 3.1 now, 300 of 5 of 4 KiB 3.7 and 3.2, 8192 of 2 of 512 bytes 11.4 and 9.6 (the division of
// 64-bit workgroup numbers by the parts of a row went with it).
// Over 669 shapes (rows of 512 bytes to 16 KiB, 1 to 8192 tokens, 1 to 12 choices, in a graph) the median is 1.18 times as
// quick so; slower are 4096 of 12 of 4 KiB, 32.5 and 34.1 us, and by 1-4 % eight more of many rows (1024 of 9 of 8 KiB
// 14.7 and 15.2).  Without the wait behind a batch these gain what they lost, but other large calls of several
// batches lose up to 8 %, and no rule on sizes parts them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "combine_split.hpp"
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

// A load through the scalar cache (the arrays are written before the launch): it counts on lgkmcnt,
// so the wait for it is not a wait for the row loads before it.
template <class T>
__device__ __forceinline__ T load_scalar(const T* p) {
  return *(const __attribute__((address_space(4))) T*)p;
}

// out[t] = bf16(sum_j gate[t, j] * recv[slot[t, j]]).
// A workgroup covers kVec * 256 16-byte vectors of one token's row (blockIdx.y, then every gridDim.y-th
// token; blockIdx.x which part of the row); each thread keeps kVec * 8 fp32 sums.  The k choices are
// taken four at a time: a batch's slots come through the scalar cache, its rows are then loaded
// together and added in choice order as separately rounded products and sums (contraction off), so the
// result does not depend on the batching.  Out-of-range slots are skipped and counted.
template <int kVec>
__global__ __launch_bounds__(kCombineThreads) void combine_kernel(CombineArgs a) {
#pragma clang fp contract(off)
  constexpr int kBatch = 4;
  const uint32_t nvec = (uint32_t)a.H / 8;
  const uint32_t v0 = blockIdx.x * (kCombineThreads * kVec) + threadIdx.x;
  for (int64_t t = blockIdx.y; t < a.tokens; t += gridDim.y) {
    const int32_t* slots = a.slot + t * a.k;
    const float* gates = a.gate + t * a.k;
    float acc[kVec][8];
#pragma unroll
    for (int u = 0; u < kVec; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[u][e] = 0.0f;
    for (int j0 = 0; j0 < a.k; j0 += kBatch) {
      u32x4 v[kBatch][kVec];
      int32_t slot[kBatch];
      float g[kBatch];
      bool ok[kBatch];
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        const bool have = j0 + jj < a.k;
        slot[jj] = have ? load_scalar(slots + j0 + jj) : -1;
        g[jj] = have ? load_scalar(gates + j0 + jj) : 0.0f;
      }
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        ok[jj] = slot[jj] >= 0 && slot[jj] < a.recv_rows;
        if (!ok[jj]) continue;
        const g_u32x4* row = (const g_u32x4*)(a.recv + (int64_t)slot[jj] * a.H);
#pragma unroll
        for (int u = 0; u < kVec; ++u)
          if (v0 + u * kCombineThreads < nvec) v[jj][u] = row[v0 + u * kCombineThreads];
      }
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        if (!ok[jj]) {
          if (j0 + jj < a.k && blockIdx.x == 0 && threadIdx.x == 0 && a.bad_slots) atomicAdd(a.bad_slots, 1u);
          continue;
        }
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
      // Every load has been added by now.  Said once for all paths, or the compiler waits before each
      // load of the next batch in case a skipped choice had left its registers to an older one.
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    }
    g_u32x4* dst = (g_u32x4*)(a.out + t * a.H);
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      if (v0 + u * kCombineThreads >= nvec) continue;
      u32x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = to_bf16x2(acc[u][2 * q], acc[u][2 * q + 1]);
      dst[v0 + u * kCombineThreads] = o;
    }
  }
}

template <int kVec>
hipError_t launch(const CombineArgs& a, hipStream_t s) {
  const dim3 grid((uint32_t)combine_spans(a.H, kVec), (uint32_t)std::min<int64_t>(a.tokens, 65535));
  hipLaunchKernelGGL((combine_kernel<kVec>), grid, dim3(kCombineThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_combine(const CombineArgs& a, hipStream_t s) {
  if (a.tokens <= 0) return hipSuccess;
  const int vec = combine_vec(a.tokens, a.k, a.H);
  return vec == 1 ? launch<1>(a, s) : vec == 2 ? launch<2>(a, s) : launch<4>(a, s);
}

}  // namespace moe
