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

}  // namespace bgl
