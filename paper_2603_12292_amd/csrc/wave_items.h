// Distribution of work items over the waves of a persistent grid.
#pragma once

#include "kernels.h"

namespace bgl {

// Work items [0, items) of a persistent grid's waves.  A short list (at most
// four items per wave) is walked statically (of every W items a wave takes one,
// in each round another place on, so that a wave does not meet the same program
// in chunk after chunk where W is a multiple of the programs: 24 programs x 8
// 10^6 cases took as long as the longest of them; no atomics); a longer one
// through shared counters, in claims that shrink towards the list's end: long
// claims at the end leave waves idle.
// Atomics on one address serialise (12 ns each, whatever the number of
// waves): with one counter, the first claim of 6144 waves takes 75 us, the
// last, which finds nothing, as much again, and 300 000 one-tile items of
// eight to a claim 450 us in all (3..12 tokens x 512 cases: 640 us, now 350).
// So a long list has 2^shift counters, each on a line of its own (1.0 ns per
// claim over 16 counters, no less over 32 or 64).  Counter s hands out items
// s, s + 2^shift, ... in order, to the workgroups of its own only: the counters'
// shares are alike, and waves sent on from a counter that has run out to one
// that has not all met at the last one (100 us).
// The loop around next() must stay free of divergent branches: a lane-0-only
// branch around the atomic lets the compiler restructure it so that after
// the first item only lane 0 goes back to the atomic.  So every lane takes
// part in the atomic (lane 0 adds the claim, the others 0) and the result is
// read from lane 0 explicitly.
struct WaveItems {
  int64_t item, items;  // the next item of this wave's claim; all items
  unsigned long long* work;
  int rest, stride;  // items left of the claim, and between them
  int counter;       // -1: a static walk, `stride` items a round, `rest` the place in it
  __device__ __forceinline__ WaveItems(int64_t items_, unsigned long long* work_, int shift)
      : items(items_), work(work_) {
    const int per = int(blockDim.x >> 6), waves = int(gridDim.x) * per;
    const int id = __builtin_amdgcn_readfirstlane(int(blockIdx.x) * per + int(threadIdx.x >> 6));
    if (items > 4 * int64_t(waves)) {
      // (every counter needs a workgroup)
      while ((1u << shift) > gridDim.x) --shift;
      // (the workgroups of one counter share an XCD)
      stride = 1 << shift;
      counter = int(blockIdx.x) & (stride - 1);
      item = counter;
      rest = 0;
    } else {
      counter = -1;
      item = 0;
      rest = id;
      stride = waves;
    }
  }
  __device__ __forceinline__ bool claim(int least) {
    // (`item` is where this wave's last claim ended: a lower bound of its
    // counter, so a claim is at most 1/8 of a wave's share of the rest)
    const float share = 0.125f / float(gridDim.x * (blockDim.x >> 6));
    const int left = __builtin_amdgcn_readfirstlane(int(float(items - item) * share));
    const int n = left > CLAIM_MAX ? CLAIM_MAX : left < least ? least : left;
    const unsigned long long it =
        atomicAdd(work + counter * COUNTER_STRIDE, (threadIdx.x & 63u) == 0 ? (unsigned long long)n : 0ull);
    const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(it), 0);
    const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(it >> 32), 0);
    const int64_t first = int64_t((uint64_t(hi) << 32) | lo);
    const int64_t all = (items - counter + stride - 1) >> __builtin_ctz(stride);
    if (first >= all) return false;
    item = first * stride + counter;
    rest = first + n < all ? n : int(all - first);
    return true;
  }
  // the next item, or -1; claims are of at least `least` items
  __device__ __forceinline__ int64_t next(int least) {
    if (counter < 0) {
      const int64_t r = item + rest;
      item += stride;
      rest += int(0.38f * float(stride)) | 1;
      if (rest >= stride) rest -= stride;
      return r < items ? r : -1;
    }
    if (rest == 0 && !claim(least)) return -1;
    --rest;
    const int64_t r = item;
    item += stride;
    return r;
  }
};

// items of one claim at least: whole programs of a resident table by their
// cases (a short program's one tile takes about as long as a claim)
__device__ __forceinline__ int claim_least(int64_t cases) {
  return cases >= 8 * TILE ? 1 : cases >= 2 * TILE ? 4 : 8;
}

}  // namespace bgl
