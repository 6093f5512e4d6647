// Distribution of work items over the waves of a persistent grid.
#pragma once

#include "kernels.h"

namespace bgl {

// Work items [0, items) of a persistent grid's waves.  A short list (at most
// four items per wave) is walked statically (wave w takes items w, w + W, ...:
// no atomics); a longer one through a shared counter, in claims that shrink
// towards the list's end: long claims at the end leave waves idle, but
// same-address atomics serialise at the counter (~10 ns each), so that items
// of one tile are never claimed one by one (2^20 of them: 3.9 ms with single
// claims over the last 4 %, 2.6 ms with eight).
// The loop around next() must stay free of divergent branches: a lane-0-only
// branch around the atomic lets the compiler restructure it so that after
// the first item only lane 0 goes back to the atomic.  So every lane takes
// part in the atomic (lane 0 adds the claim, the others 0) and the result is
// read from lane 0 explicitly.
struct WaveItems {
  int64_t item, end, items, step;
  int64_t waves;
  unsigned long long* work;
  int64_t least;  // items of one claim at least
  bool claimed;
  __device__ __forceinline__ WaveItems(int64_t items_, unsigned long long* work_, int64_t least_)
      : items(items_), work(work_), least(least_) {
    const int per = int(blockDim.x >> 6);
    waves = int64_t(gridDim.x) * per;
    claimed = items > 4 * waves;
    const int64_t id = __builtin_amdgcn_readfirstlane(int(blockIdx.x) * per + int(threadIdx.x >> 6));
    item = claimed ? 0 : id;
    end = claimed ? 0 : items;
    step = claimed ? 1 : waves;
  }
  // the next item, or -1
  __device__ __forceinline__ int64_t next() {
    if (item >= end) {
      if (!claimed) return -1;
      // (`end` is where this wave's last claim stood: a lower bound of the
      // counter, so the claim is at most 1/8 of a wave's share of the rest)
      const int64_t left = (items - end) / (8 * waves);
      const int64_t n = left > CLAIM_MAX ? CLAIM_MAX : left < least ? least : left;
      const unsigned long long it = atomicAdd(work, (threadIdx.x & 63u) == 0 ? (unsigned long long)n : 0ull);
      const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(it), 0);
      const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(it >> 32), 0);
      const int64_t first = int64_t((uint64_t(hi) << 32) | lo);
      if (first >= items) return -1;
      item = first;
      end = first + n < items ? first + n : items;
    }
    const int64_t r = item;
    item += step;
    return r;
  }
};

// items of one claim at least, by an evaluation item's cases
__device__ __forceinline__ int64_t claim_least(int64_t cases) {
  return cases >= 8 * TILE ? 1 : cases >= 4 * TILE ? 2 : cases >= 2 * TILE ? 4 : 8;
}

}  // namespace bgl
