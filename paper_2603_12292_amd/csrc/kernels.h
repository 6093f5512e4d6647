// Kernel argument blocks and host-side launchers of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/beagle.h"
#include "beagle_device.h"

namespace bgl {

struct PrepareArgs {
  const uint16_t* tokens;
  int64_t n_tokens;
  const int64_t* tok_offset;
  const int32_t* tok_len;
  const float* consts;
  int64_t n_consts;
  const int64_t* const_offset;
  const int32_t* const_count;
  int32_t n_programs;
  int32_t D;
  uint32_t* code;      // [n_tokens] decoded words
  uint32_t* aux;       // [n_tokens] adjoint operands per decoded word
  float* cval;         // [n_tokens] CONST values by output position
  uint8_t* vrow;       // [n_tokens] input rows of the VAR words, in word order
  // nonzero: the staged cases hold the base operators' values of every
  // variable as rows of their own (see derived_row), and "unary operator of a
  // variable" decodes to a VAR word of such a row
  int32_t derived;
  int32_t max_words;   // decoded words allowed (longer -> BEAGLE_PROG_TOO_LONG)
  uint16_t* scr;  // [3 * n_tokens] scratch of the programs longer than 128 tokens
  ProgMeta* meta;      // [n_programs]
  int8_t* status_out;  // [n_programs] or null
  int32_t* class_count;  // [N_CLASSES] programs per register-need class
  int32_t* class_list;   // [N_CLASSES][n_programs] program indices per class
  int32_t* len_count;    // [5] adjoint lists (see k_prepare)
  int32_t* len_list;     // [5][n_programs]
  int32_t short_words;
  // nonzero: also write the adjoint's per-word operands (aux) and its
  // program lists (an evaluation without gradients needs neither)
  int32_t adjoint;
  // programs k_prepare leaves to k_prepare_long (count zero at launch)
  int32_t* long_count;
  int32_t* long_list;  // [n_programs]
  // Disjoint ranges: every program is decoded in place of its tokens, so the
  // token ranges of different programs (and, for the adjoint, whose gradient
  // output has the constants' layout, the constant ranges) must not overlap.
  // layout[0], layout[1] (zero at launch): set by k_stage_and_check when the
  // token / constant ranges are not sorted and disjoint by program index;
  // then owner / cowner hold, per token / constant slot, the lowest index of
  // a program whose range covers it, and a program finding another index in
  // its range gets BEAGLE_PROG_BAD_LAYOUT.
  // On few programs (OWNER_MIN_PROGRAMS) owner and cowner are null where a wave
  // decodes or folds a program, and it looks through the lower-indexed ones itself.
  int32_t* layout;
  int32_t* owner;   // [n_tokens]
  int32_t* cowner;  // [n_consts] (adjoint only)
  // programs each wave of k_prepare_wave decodes (1..64)
  int32_t wave_programs;
};

// Folding of constant subtrees (fold.hip): the rewritten programs, at their
// own token offsets, and their constants behind room for the caller's (copied
// for the programs that are kept as they are).
struct FoldArgs {
  PrepareArgs in;         // the caller's programs and the ranges check's results
  int32_t first;          // (set by launch_fold) the launch's first program
  uint16_t* tokens;       // [n_tokens]
  int32_t* tok_len;       // [n_programs]; -1: the ranges check failed
  float* consts;          // [n_consts + n_tokens]
  int64_t* const_offset;  // [n_programs]
  int32_t* const_count;   // [n_programs]
  // adjoint: per program, map_n entries at its token offset, one per CONST
  // token: original slot | folded slot << 8, and the derivative (map_n = 0:
  // a program kept as it is)
  int32_t* map_n;
  uint16_t* map_slots;
  double* map_der;
};
void launch_fold(const FoldArgs& f, hipStream_t s);

// Staged cases: tiles of TILE cases, row-major within a tile (`rows` rows of
// TILE cases: the D variables, the derived rows when there are any, the
// targets last), so that a row of a tile is one run of 2 KB and a tile's rows
// lie together.
constexpr int TILE = 512;
// offset of a case of row 0 in floats
__host__ __device__ constexpr int64_t case_offset(int64_t i, int32_t rows) {
  return (i / TILE) * (int64_t(rows) * TILE) + i % TILE;
}
// Derived rows: base unary operator u (SIN .. SQRT: 0..4) of variable d.
// Of the arithmetic of random programs a quarter is an operator of the base
// set applied to a variable itself; computing those 5 D rows once per call and
// reading them costs a few programs' work.
__host__ __device__ constexpr int derived_row(int u, int d, int D) { return D + u * D + d; }
constexpr int DERIVED_OPS = 5;
__host__ __device__ constexpr int32_t stage_rows(int32_t D, int derived) {
  return (derived ? (1 + DERIVED_OPS) * D : D) + 1;
}
static_assert((1 + DERIVED_OPS) * MAX_D <= 256, "rows are bytes");

struct StageArgs {
  const float* X;
  const float* y;
  int64_t M;
  int64_t Mp;  // padded to whole tiles
  int32_t D;
  int32_t derived;
  float* Xt;  // [Mp / TILE][rows][TILE]
};

// Evaluation without a fitness: every case's output is written (beside the
// library's fitness kinds).
constexpr int KIND_OUTPUTS = 4;

// Partial sums per (chunk, program) of each fitness kind (the evaluator's
// epilogue: MSE 1, CORR 3, the paper's POINT score 1, its R4 score 7).
__host__ __device__ constexpr int kind_sums(int kind) {
  return kind == BEAGLE_FIT_MSE ? 1 : kind == BEAGLE_FIT_CORR ? 3 : kind == BEAGLE_FIT_POINT ? 1 : 7;
}
constexpr int MAX_SUMS = 8;

struct EvalArgs {
  const uint32_t* code;
  const float* cval;
  const uint8_t* vrow;
  const int64_t* tok_offset;
  const ProgMeta* meta;
  const float* Xt;  // staged cases
  int32_t rows;     // rows per tile
  int64_t M;
  int32_t n_programs;
  int32_t n_chunks;
  int64_t chunk;          // cases per chunk, a multiple of CHUNK_UNIT
  double* part;           // [n_sums][n_chunks][n_programs]
  const double* stats;    // target statistics (correlation fitness)
  const int32_t* class_count;       // [N_CLASSES]
  const int32_t* class_list;        // [N_CLASSES][n_total] global program indices
  unsigned long long* work;         // [N_CLASSES] lists' work counters, zero at launch
  int32_t work_shift;               // ... 2^work_shift each (counter_shift)
  int32_t n_total;                  // programs in the whole population
  int32_t prog_begin;               // first program of this launch (slice-local index 0)
  double smax = 0.0;                // the paper's scores: maximum score S
  float* out = nullptr;             // KIND_OUTPUTS: [n_programs][M]
  // correlation and Eq. 2 in one chunk: the kernels take each program's shift
  // from their own first tile and store it here (the same array as meta)
  ProgMeta* meta_shift = nullptr;
};

struct FinalizeArgs {
  const ProgMeta* meta;
  const double* part;
  const double* stats;
  int64_t M;
  int32_t n_programs;
  int32_t n_chunks;
  int32_t kind;
  double* fitness;
  // correlation fitness only, or null: per program (alpha, beta, mu) of the
  // gradient seed dF/dyhat_i = alpha (w_i - mean w) + beta (yhat_i - mu)
  double* coef = nullptr;
  double smax = 0.0;  // the paper's scores: maximum score S
};

struct ValuesArgs {
  const uint32_t* code;
  const float* cval;
  const int64_t* tok_offset;
  ProgMeta* meta;
  const float* Xt;
  int32_t rows;
};

// A prediction of few program-cases, or of few cases: a wave per program and 64
// of them, one per lane, in one launch (see k_outputs_small).
constexpr int64_t SMALL_OUTPUTS = int64_t(1) << 20;
inline bool small_outputs(int64_t n_programs, int64_t M) {
  return n_programs * M <= SMALL_OUTPUTS || (M <= 128 && n_programs < (int64_t(1) << 26));
}

// One problem of a batched evaluation: an entry of the device problem table.
// Every pointer (the caller's arrays and this problem's share of the
// workspace) is resolved on the host before the table is uploaded.
struct BatchProblem {
  PrepareArgs prep;  // programs, decode targets, class lists, status output
  const float* X;    // [M x D] caller's cases
  const float* y;    // [M]
  float* Xt;         // staged cases
  int32_t rows;      // rows per tile
  double* stats;     // [4] target statistics
  double* part;      // [n_sums][n_chunks][n_programs]
  double* fitness;   // [n_programs] caller's output
  int64_t M;
  int64_t Mp;
  int64_t chunk;
  int32_t n_chunks;
  int32_t kv;          // tile variant of class 0 for this problem
  int64_t prog_begin;  // first program of this problem in the batch-wide program index
  int64_t case_begin;  // first padded case of this problem in the batch-wide case index
};

// Work lists of a batched evaluation: class 0 wide tile, class 0 narrow
// tile, class 1, class 2.
constexpr int N_LISTS = 4;

struct BatchArgs {
  const BatchProblem* table;
  int32_t n_problems;
  int32_t kind;
  int64_t n_programs;          // over the whole table
  int64_t n_cases;             // padded cases over the whole table
  int64_t* item_off;           // [N_LISTS][n_problems + 1] first work item of each problem per list
  unsigned long long* work;    // [N_LISTS] lists' work counters, zero at launch
  int32_t work_shift;          // ... 2^work_shift each (counter_shift)
};

// The problem holding batch-wide index x of a prefix field (prog_begin or
// case_begin): the last q with field(q) <= x.
template <class F>
__device__ __forceinline__ int batch_find(const BatchArgs& b, int64_t x, F field) {
  int lo = 0, hi = b.n_problems;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (field(b.table[mid]) <= x)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// programs from which the owner arrays are filled: two launches, for a check that
// otherwise reads every lower-indexed header only where a layout is flagged.  Below
// it the waves of k_prepare_wave and k_fold read them (PrepareArgs::layout).  A
// decoder with a thread per program has the arrays, in a batch from
// OWNER_MIN_BATCH programs of a problem on: 64 headers take a thread about as
// long as the launches (two problems of 32 programs in order 155 -> 151 us)
constexpr int32_t OWNER_MIN_PROGRAMS = 4097;
constexpr int32_t OWNER_MIN_BATCH = 65;
constexpr int EVAL_WAVES = 4;
// rows a wave keeps in flight: two are enough behind the other waves of a
// SIMD, and four cost the fifth of them (the workgroup's 32 KB leave room for
// four): 1.67 against 1.83 ms on 4096 programs x 10^5 cases
constexpr int RING = 2;
// Case chunks: a wave takes one program on one chunk.  At most CHUNK_CASES
// cases (eight tiles: long enough that a work item's start is a few per cent of
// it, short enough that the last items end together and that a chunk's rows
// stay in an XCD's L2), a multiple of CHUNK_UNIT (a narrow tile).
constexpr int64_t CHUNK_CASES = 4096;
constexpr int64_t CHUNK_UNIT = 256;
// Work items that a population of few programs is split into: four for each
// of the 6144 waves of the 8-case kernel (six per SIMD), which walk them
// without claims.  With 4096, less than a wave's worth each, the longest
// programs decided the time: 4096 programs x 4096 cases 245 us (now 120), 1000
// x 20 000 with the further operators 280 (190), 100 x 10^5 175 (94); with
// 65 536 an item's start counts (2000 x 10^4: 140 -> 148 us).
constexpr int64_t CHUNK_ITEMS = 24576;
// Chunks whose partial sums a wave adds, 64 at a time, instead of a thread, one
// after the other (10 programs x 10^5 cases in 391 chunks: correlation 112
// us, now 75).
constexpr int32_t WIDE_FINALIZE_CHUNKS = 16;
// The resident-inputs evaluator (small case sets, register-need classes 0
// and 1): staged rows of at most this many bytes, populations of at least this
// many programs.
constexpr size_t RESIDENT_MAX_BYTES = 158 * 1024;
constexpr int32_t RESIDENT_MIN_PROGRAMS = 4096;
inline size_t resident_bytes(int64_t M, int32_t rows) {
  return size_t((M + TILE - 1) / TILE) * size_t(rows) * size_t(TILE) * sizeof(float);
}
inline bool resident_call(int64_t n_programs, int32_t n_chunks, int64_t M, int32_t rows) {
  return n_chunks == 1 && n_programs >= RESIDENT_MIN_PROGRAMS && resident_bytes(M, rows) <= RESIDENT_MAX_BYTES;
}
// Cases from which constant subtrees are folded: the fold costs a program a
// few hundred instructions, and saves about a hundred per 512 cases of an
// evaluation, three times that of a gradient.
constexpr int64_t FOLD_MIN_CASES = 2048;
constexpr int64_t FOLD_MIN_WORK = int64_t(1) << 26;  // programs x cases that repay its launch
constexpr int64_t FOLD_MIN_CASES_ADJOINT = 512;
// Work items of one narrow tile up to which one launch runs all register-need
// classes: two launches fewer count for more there than the three waves per
// SIMD that its registers allow (400 items 32 -> 27 us, 3000 37 -> 33, 4000
// within 1 us either way; 5..64 tokens).  Items of several tiles need the
// class kernels' waves (100 programs x 10^5 cases in 40 chunks: 175 against 109
// us).  It has one tile width: nothing to tune.
constexpr int64_t MIXED_MAX_ITEMS = 4096;
inline bool mixed_launch(int64_t n_programs, int64_t n_chunks, int64_t chunk) {
  return n_programs * n_chunks <= MIXED_MAX_ITEMS && chunk <= CHUNK_UNIT;
}
constexpr int CLAIM_MAX = 16;  // work items of one claim at most
// Work counters of a list (see WaveItems): 2^shift of them, a line apart; the
// lists' counters follow one another.  One counter where every grid walks the
// list without claims, or nearly so.
constexpr int COUNTER_SHIFT = 4;
constexpr int COUNTER_STRIDE = 16;  // 64-bit words: 128 bytes
inline int counter_shift(int64_t items) { return items > 4096 ? COUNTER_SHIFT : 0; }
__host__ __device__ constexpr int counter_words(int shift) { return shift ? COUNTER_STRIDE << shift : 1; }
__host__ __device__ constexpr int class_k(int c, int kv) { return c == 0 ? (kv == 0 ? 8 : 4) : 4; }

// decoding: programs of at most 64 tokens in k_prepare_wave (a wave per
// program) or k_prepare (a thread per program, narrow LDS scratch), the
// longer ones they list for k_prepare_long
// the disjoint-ranges check before decoding (see PrepareArgs::layout):
// neighbour comparison, then (only when that found unsorted or overlapping
// ranges) the owner arrays filled and marked
__global__ void k_layout_fill(PrepareArgs a);
__global__ void k_layout_mark(PrepareArgs a);
__global__ void k_layout_check_batch(BatchArgs b);
__global__ void k_layout_fill_batch(BatchArgs b);
__global__ void k_layout_mark_batch(BatchArgs b);
__global__ void k_prepare(PrepareArgs a);
// ADJ: also the adjoint's per-word operands and lists (PrepareArgs::adjoint)
template <bool ADJ>
__global__ void k_prepare_wave(PrepareArgs a);
__global__ void k_prepare_long(PrepareArgs a);
__global__ void k_stage_and_check(StageArgs sa, PrepareArgs pa, uint32_t stage_blocks);
__global__ void k_prepare_batch(BatchArgs b);
__global__ void k_stage_batch(BatchArgs b);
__global__ void k_target_stats_batch(BatchArgs b);
__global__ void k_shifts_batch(BatchArgs b);
__global__ void k_batch_items(BatchArgs b);
__global__ void k_finalize_batch(BatchArgs b);
__global__ void k_target_stats(const float* __restrict__ y, int64_t M, double* __restrict__ stats);
// (more than WIDE_FINALIZE_CHUNKS chunks: a wave per program, else a thread)
void launch_finalize(const FinalizeArgs& a, hipStream_t s);
__global__ void k_shifts(ValuesArgs a);
// Programs from which class 1 of a prediction takes the resident table, which
// leaves its kernel few waves; below, its programs are cut by tiles and streamed.
// 16 operators: 20 000 programs x 1000 cases 291 us, streamed 228 (a wave per
// program and 64 cases 257); x 300 177 and 149; 100 000 x 300 417 and 465.
constexpr int64_t RESIDENT_MIN_DEEP_OUTPUTS = 65536;
// Tiles of a prediction below which its classes 1 and 2 are cut by half tiles: their
// kernels hold 4096 waves, and little more than that in whole tiles ends in a round
// that is nearly empty.  1000 programs x 3000 cases 71 us, in half tiles 65; 5000 x
// 500 83 and 76; 1000 x 10 000 (20 000 tiles) 127 and 145.
constexpr int64_t HALF_TILE_DEEP_OUTPUTS = 12288;
__global__ void k_outputs_small(ValuesArgs a, int64_t M, int32_t D, float* out);
// NaN rows of the invalid programs of a prediction (a workgroup per program, and
// the programs a grid apart)
__global__ void k_nan_rows(const ProgMeta* meta, int32_t n_programs, int64_t M, float* out);
// host launchers of the templated evaluation kernels (eval.hip)
// ev0/ev1 (may be null) are recorded on `s` right before and after the
// fast-path kernel.
// kv selects the tile variant of class 0.
// counters_clear: a.work is known to be zero (else it is cleared first).
// kind: a fitness kind or KIND_OUTPUTS.
hipError_t launch_eval(int kind, int kv, const EvalArgs& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                       bool counters_clear = false);
// The work-list kernels of a batched evaluation; lists with has_items[v] == 0
// are skipped.
hipError_t launch_eval_batch(int kind, const BatchArgs& b, const int* has_items, hipStream_t s);
// Runs the occupancy queries of those launches (before a stream capture).
void prime_eval_batch(int kind);

}  // namespace bgl
