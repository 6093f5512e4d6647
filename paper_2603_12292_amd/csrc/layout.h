// Ranges of programs in the packed layout.
#pragma once

#include "kernels.h"

namespace bgl {

// Token range of program p when it lies within the token array (else
// false: the program is rejected by the layout checks of the decoder).
__device__ __forceinline__ bool tok_range(const PrepareArgs& a, int p, int64_t& off, int32_t& L) {
  off = a.tok_offset[p];
  L = a.tok_len[p];
  return L >= 0 && L <= MAX_LEN && off >= 0 && off + L <= a.n_tokens;
}

__device__ __forceinline__ bool const_range(const PrepareArgs& a, int p, int64_t& off, int32_t& n) {
  off = a.const_offset[p];
  n = a.const_count[p];
  return n >= 0 && (n == 0 || (off >= 0 && off + n <= a.n_consts));
}

// Whether program q's token range (or, for the adjoint, its constant range)
// holds a slot of [off, off + L) (of [coff, coff + cc)).
__device__ __forceinline__ bool overlaps(const PrepareArgs& a, int q, int64_t off, int32_t L, int64_t coff, int32_t cc) {
  int64_t o;
  int32_t n;
  if (tok_range(a, q, o, n) && n > 0 && L > 0 && o < off + L && off < o + n) return true;
  return a.adjoint && const_range(a, q, o, n) && n > 0 && cc > 0 && o < coff + cc && coff < o + n;
}

// Whether no lower-indexed program's range meets program p's: the whole wave
// looks through them, four of its rounds at a time (a round is one latency:
// 4000 programs in shuffled order, 62 rounds, ~10 us).  A thread by itself would
// take 64 times as long, so the kernels that decode with one have the owner
// arrays.
__device__ __forceinline__ bool wave_alone(const PrepareArgs& a, int p, int64_t off, int32_t L, int64_t coff,
                                           int32_t cc) {
  const int lane = int(threadIdx.x & 63u);
  for (int q0 = 0; q0 < p; q0 += 256) {
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = q0 + r * 64 + lane;
      bad |= q < p && overlaps(a, q, off, L, coff, cc);
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0) return false;
  }
  return true;
}

}  // namespace bgl
