// combine_split.hpp -- how a combine call is divided among workgroups (host side, plain C++).
#pragma once
#include <stdint.h>

namespace moe {

constexpr int kCombineThreads = 256;

// Workgroups that a token's row of H bf16 values takes at `vec` 16-byte vectors per thread.
inline int64_t combine_spans(int32_t H, int vec) {
  const int64_t width = (int64_t)kCombineThreads * vec;
  return (H / 8 + width - 1) / width;
}

// 16-byte vectors per thread: 1, 2 or 4.  Longer rows take more, so that many tokens need few
// workgroups; as long as those would not even give each of the 256 compute units one (at four vectors and
// eight choices or more, the longest ones, two) a token spreads over more workgroups instead, one vector
// per thread.  Unspread against spread, in a graph:
//   48 tokens of 8 rows of 14 KiB 4.65 -> 3.13 us, 511 of 8 of 14 KiB 11.3 -> 9.1,
//   256 of 6 of 8 KiB 3.69 -> 3.53, 256 of 2 of 4112 bytes 2.49 -> 2.56 and of 14 KiB 3.25 -> 3.41;
//   past the line 511 of 2 of 14 KiB 4.02 -> 4.68, 300 of 2 of 8 KiB 2.74 -> 2.94,
//   511 of 8 of 4112 bytes 4.10 -> 4.97, 511 of 6 of 8 KiB 4.66 -> 4.65.
inline int combine_vec(int64_t tokens, int32_t k, int32_t H) {
  const int64_t nvec = H / 8;
  const int vec = nvec <= 256 ? 1 : nvec <= 512 ? 2 : 4;
  return tokens * combine_spans(H, vec) <= (vec == 4 && k >= 8 ? 512 : 256) ? 1 : vec;
}

}  // namespace moe
