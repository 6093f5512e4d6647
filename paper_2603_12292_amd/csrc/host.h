// Host-side internals shared by the C ABI files: the context, error
// reporting, workspace management, argument checks and the tile-width tuner.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/beagle.h"
#include "kernels.h"

namespace bgl {
namespace host {

// Problem-shape bucket of the tile-width tuner: (kind, D, round(log2 M),
// round(log2 mean program length)).
using TuneKey = std::tuple<int, int, int, int>;

// A captured batched launch sequence and what it was captured for.
struct BatchGraph {
  std::string key;  // bytes of the problem table + kind + workspace address
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  uint64_t last_use = 0;
};

}  // namespace host
}  // namespace bgl

struct beagle_ctx {
  int device = 0;
  size_t cap = 0;       // 0 = unlimited
  char* ws = nullptr;   // device workspace
  size_t ws_size = 0;
  bool timing = false;  // record events around the main evaluation kernel
  std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
  int tuning = BEAGLE_TUNE_AUTO;
  int decoder = BEAGLE_DECODE_WAVE;  // decoder of programs of at most 64 tokens
  // side stream of the target statistics (beside the decoding), created on
  // first use, with its fork and join events
  hipStream_t side = nullptr;
  hipEvent_t side_fork = nullptr, side_join = nullptr;
  std::map<bgl::host::TuneKey, int> tuned;  // bucket -> tile variant (0 wide, 1 narrow)
  std::string tune_file;                    // BEAGLE_AUTOTUNE_CACHE at creation ("" = none)
  // batched evaluation
  size_t refused = 0;  // bytes of the smallest workspace that could not be allocated (0: none)
  std::vector<bgl::host::BatchGraph> graphs;
  hipStream_t capture_stream = nullptr;  // graphs are captured here, launched on the caller's stream
  std::vector<bgl::BatchProblem> table;  // host copy of the last uploaded problem table
  hipEvent_t table_copied = nullptr;     // the last table upload has read `table`
  uint64_t use_clock = 0;
  int64_t graph_captures = 0, graph_replays = 0;
};

namespace bgl {
namespace host {

beagle_status fail(beagle_status s, const std::string& msg);
beagle_status hip_fail(hipError_t e, const char* where);
void clear_error();
const char* last_error();

// Makes ctx->device current for the duration of a call.
struct DeviceGuard {
  int prev = -1;
  hipError_t err = hipSuccess;
  explicit DeviceGuard(int dev) {
    err = hipGetDevice(&prev);
    if (err == hipSuccess && prev != dev) err = hipSetDevice(dev);
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

// Bump allocator over the context workspace (256-byte aligned pieces).
struct Carve {
  size_t used = 0;
  template <class T>
  size_t take(size_t count) {
    const size_t at = (used + 255) & ~size_t(255);
    used = at + count * sizeof(T);
    return at;
  }
};

// Grows the workspace to `bytes` (synchronises the device and drops the
// captured graphs when it moves).
beagle_status reserve(beagle_ctx* ctx, size_t bytes);
// How much workspace a call is laid out with: all that speed wants; without
// derived rows and folded programs (the same values, bit for bit); or the least,
// with few case chunks too (sums in another order).
enum Level { LEVEL_FULL, LEVEL_BARE, LEVEL_LEAST, N_LEVELS };
// Reserves the first of the layouts that the cap allows and the device has
// memory for; layout(level) makes one and returns its bytes.
template <class F>
beagle_status reserve_first(beagle_ctx* ctx, F layout) {
  for (int level = LEVEL_FULL;; ++level) {
    const size_t bytes = layout(level);
    if (level != LEVEL_LEAST) {
      if (ctx->cap && bytes > ctx->cap) continue;
      if (ctx->refused && bytes >= ctx->refused && bytes > ctx->ws_size) continue;
    }
    const beagle_status st = reserve(ctx, bytes);
    if (st != BEAGLE_E_NOMEM || level == LEVEL_LEAST) return st;
  }
}
beagle_status check_programs(const beagle_programs* p);
beagle_status check_data(const beagle_dataset* d, int kind);
int64_t round_up(int64_t v, int64_t m);
// Case chunks of one call: at most max_chunk_cases cases each (rounded up to
// a multiple of unit, the cases one kernel iteration covers), more when the
// population alone gives too few work items.
void choose_chunks(int64_t M, int64_t N, int64_t* chunk, int32_t* n_chunks, int64_t max_chunk_cases, int64_t unit,
                   int64_t target_blocks = 4096);
// The evaluation's chunks (see CHUNK_CASES, CHUNK_ITEMS).
void eval_chunks(int64_t M, int64_t N, int64_t* chunk, int32_t* n_chunks, int level = LEVEL_FULL);
// Whether an evaluation of N programs on M cases stages derived input rows:
// their computing and writing is 5 D rows' work per case, and every program
// saves about a quarter of its own.  D = 5, 5..64 tokens: 16 programs x 10^5
// cases 47 us (without 43), 40 x 10^5 63 (61), 64 x 10^5 72 (73), 200 x 10^5 146
// (171).  Rows that don't stay in the caches are read from memory as well: 24
// programs x 8 10^6 cases 1270 us (1060), 64 x 2 10^6 690 (710); D = 9, 100 x 10^6
// 986 (857), 200 x 10^6 equal.
inline bool use_derived(int64_t N, int64_t M, int32_t D) {
  const bool cached = int64_t(bgl::stage_rows(D, 1)) * M * 4 <= int64_t(64) << 20;
  return N >= 16 && N >= (cached ? 8 : 12) * int64_t(D);
}
// Program-cases from which a population for the resident kernels does: copying
// the derived rows into every compute unit takes longer than they save.  7596
// programs of 16 operators x 310 cases 98 against 94 us, 20 000 programs 211
// against 227.
constexpr int64_t DERIVED_MIN_RESIDENT = int64_t(1) << 22;
// Mean program length (of the token array: slots count whole) from which a
// population gives up the resident table, which the derived rows would not fit,
// for them: a short program's start is not repaid by what they save.  65 000
// programs x 1500 cases, D = 9, table against streamed rows with derived ones:
// 3..12 tokens 210 and 250 us, 3..32 325 and 325, 5..64 555 and 515; x 2048, D = 5:
// 240 and 260, 411 and 386, 750 and 650.  Over more tiles it is: x 4096, D = 5,
// 3..12 tokens 440 and 390.
constexpr int64_t DERIVED_MIN_LENGTH = 12;
void zero_i32(int32_t* p, int64_t n, hipStream_t s);

// Tile variant of class 0 for a problem (0 wide, 1 narrow).  Under
// BEAGLE_TUNE_AUTO a bucket met for the first time is measured: `run(kv)`
// must enqueue one evaluation of the problem with that variant on `s`
// between the two events it is given.
using TuneRun = hipError_t (*)(void* user, int kv, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
beagle_status tile_variant(beagle_ctx* ctx, int kind, int D, int64_t M, int64_t N, double mean_len, hipStream_t s,
                           TuneRun run, void* user, int* kv);
// The variant without measuring: false when it is AUTO's to measure and the
// bucket has not yet been met.
bool known_tile_variant(const beagle_ctx* ctx, int kind, int D, int64_t M, int64_t N, double mean_len, int* kv);
void load_tune_file(beagle_ctx* ctx);
void release_graphs(beagle_ctx* ctx);

}  // namespace host
}  // namespace bgl
