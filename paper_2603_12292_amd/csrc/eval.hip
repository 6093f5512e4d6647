// Population evaluation: the stack interpreter, per-case fitness terms,
// in-block reductions and the cross-chunk finalize.
//
// Work decomposition.  A wave evaluates ONE program on one chunk of fitness
// cases; it walks the chunk in tiles of 64 lanes x K cases, so every token of
// the program is decoded once per tile (a wave-uniform scalar branch on the
// handler byte) and applied to K cases per lane.  All lanes of a wave run the
// same program on different cases, the mapping the paper's kernel uses to
// avoid divergence (section 2.1.2), but with no cap on the number of cases.
//
// The decoded program stays in a VGPR per 64 tokens (one word per lane,
// fetched with v_readlane); constants come from a side table read the same
// way.  The operand stack lives in registers with compile-time names: the
// handler byte fixes the stack size at which a token runs.  Input rows stream
// through a ring of slots in LDS, in the order the program reads them (see
// RowRing).
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "beagle_device.h"
#include "kernels.h"
#include "per_device.h"
#include "trig.h"
#include "wave_items.h"

namespace bgl {

// The 4-case class-0 variant is held to CLASS0_NARROW_WAVES waves per SIMD.
#ifndef CLASS0_NARROW_WAVES
#define CLASS0_NARROW_WAVES 7
#endif
#ifndef RESIDENT_WAVES
#define RESIDENT_WAVES 6
#endif
#ifndef CLASS0_WIDE_WAVES
#define CLASS0_WIDE_WAVES 6
#endif
#ifndef BATCH_WIDE_WAVES
#define BATCH_WIDE_WAVES 5
#endif

template <uint32_t O>
__device__ __forceinline__ float binop(float a, float b) {
  if constexpr (O == B_ADD) return a + b;
  if constexpr (O == B_SUB) return a - b;
  if constexpr (O == B_MUL) return a * b;
  if constexpr (O == B_DIV) return op_div(a, b);
  if constexpr (O == B_RSUB) return b - a;
  if constexpr (O == B_RDIV) return op_div(b, a);
  return 0.0f;
}

// r[k] = a[k] op b[k] on the K cases of a lane; the protected division
// (and its reversed form) through div_tile, one check per wave
template <uint32_t O, int K>
__device__ __forceinline__ void binop_tile(const float (&a)[K], const float (&b)[K], float (&r)[K]) {
  if constexpr (O == B_DIV) {
    div_tile<K>(a, b, r);
  } else if constexpr (O == B_RDIV) {
    div_tile<K>(b, a, r);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) r[k] = binop<O>(a[k], b[k]);
  }
}

// Input rows of one wave, in the order in which its program reads them.  A
// program reads a row for every VAR word (about ten of ~25 words) and the
// targets after its last word; those reads are known in advance (the
// decoder's list of rows), so the wave keeps the next RING of them in flight:
// each fetch waits for the oldest row, reads its K values per lane from LDS
// and has the row RING reads further on loaded into the slot just freed,
// straight from global memory.  Nothing is staged per tile, the LDS of a wave
// is RING rows whatever the number of variables (a tile of all of them held
// occupancy down from D = 6 on), and the latency of a load is covered by the
// words between RING reads.  K = 4: a row of 256 cases, one 16-byte load per
// lane; K = 8: 512 cases, two.
template <int K>
struct RowRing {
  static constexpr int LOADS = K / 4;
  uint32_t at;        // LDS byte address of this lane's 16 bytes of slot 0
  float* ring;        // the wave's slots
  const float* tile;  // row 0 of the tile the look-ahead is in (uniform)
  const float* last;  // ... of the chunk's last tile: the look-ahead stays there
  uint32_t rows_f;    // floats per tile of the layout: rows x TILE
  uint32_t half;      // K = 4: floats from a tile's first to its second half
  const uint8_t* list;
  int n, i, lane;     // reads per tile (at least one), look-ahead position in them
  int nv, yrow;       // VAR words; the targets' row
  int stop;           // where the look-ahead position next wraps or needs another block of rows
  int vt;             // rows of 64 reads, one per lane
  uint32_t slot;      // byte offset of the slot of the next read
  static constexpr uint32_t SLOT = K * 256u;  // bytes

  __device__ __forceinline__ int block(int b) const {
    const int j = b + lane;
    return j < nv ? int(list[j]) : yrow;
  }
  // The same in the middle of a tile (programs of 64 or more VAR words only).
  // A load whose wait the compiler placed would be waited for on the common
  // path as well, and with it every load in flight.
  __device__ __forceinline__ int block_now(int b) const {
    const int j = b + lane;
    const uint8_t* at_j = list + (j < nv ? j : 0);
    int v;
    asm volatile("global_load_ubyte %0, %1, off\n\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(at_j) : "memory");
    return j < nv ? v : yrow;
  }
  // the look-ahead row into `slot`
  __device__ __forceinline__ void issue() {
    const uint32_t row = __builtin_amdgcn_readlane(uint32_t(vt), i & 63);
    const char* src = (reinterpret_cast<const char*>(tile) + row * uint32_t(TILE * sizeof(float))) + uint32_t(lane) * 16u;
    char* dst = reinterpret_cast<char*>(ring) + slot;
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
    if constexpr (LOADS == 2) __builtin_amdgcn_global_load_lds(src, dst, 16, 1024, 0);
    slot = slot + SLOT == RING * SLOT ? 0u : slot + SLOT;
    if (__builtin_expect(++i == stop, 0)) turn();
  }
  __device__ __forceinline__ void turn() {
    if (i == n) {
      i = 0;
      if constexpr (K == 8) {
        tile = tile == last ? last : tile + rows_f;
      } else {
        // the other half of the tile, or the next tile's first
        tile = tile == last ? last : tile + half;
        half = rows_f - half;
      }
    }
    if (n > 64) vt = block_now(i);
    stop = i + 64 < n ? i + 64 : n;
  }
  // starts at case `c0` (a multiple of the tile) of the chunk ending at `c1`;
  // the targets are read after the last word or not at all
  __device__ __forceinline__ void start(const EvalArgs& a, float* ring_, const uint8_t* list_, int nv_, bool targets,
                                        int64_t c0, int64_t c1) {
    lane = int(threadIdx.x & 63u);
    ring = ring_;
    at = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)ring_)) + uint32_t(lane) * 16u;
    rows_f = uint32_t(a.rows) * TILE;
    list = list_;
    nv = nv_;
    n = targets || nv == 0 ? nv + 1 : nv;
    yrow = a.rows - 1;
    tile = a.Xt + (c0 / TILE) * int64_t(rows_f);
    const int64_t cl = c1 - 1;
    last = a.Xt + (cl / TILE) * int64_t(rows_f);
    half = rows_f;
    if constexpr (K == 4) {
      // (tile pointers name half tiles: 256 cases)
      tile += c0 % TILE;
      last += cl % TILE / 256 * 256;
      half = c0 % TILE ? rows_f - 256u : 256u;
    }
    i = 0;
    stop = n < 64 ? n : 64;
    vt = block(0);
    slot = 0;
#pragma unroll
    for (int r = 0; r < RING; ++r) issue();
  }
  // The next read's K values per lane.  The wait leaves only the younger
  // reads' loads in flight (loads complete in order; other memory operations
  // among them make it wait longer, never shorter).
  __device__ __forceinline__ void fetch(float (&x)[K]) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    const uint32_t addr = at + slot;
    if constexpr (K == 8) {
      v4 p, q;
      asm volatile(
          "s_waitcnt vmcnt(%3)\n\t"
          "ds_read_b128 %0, %2\n\t"
          "ds_read_b128 %1, %2 offset:1024\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(p), "=&v"(q)
          : "v"(addr), "n"((RING - 1) * LOADS)
          : "memory");
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        x[k] = p[k];
        x[4 + k] = q[k];
      }
    } else {
      v4 p;
      asm volatile(
          "s_waitcnt vmcnt(%2)\n\t"
          "ds_read_b128 %0, %1\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(p)
          : "v"(addr), "n"((RING - 1) * LOADS)
          : "memory");
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = p[k];
    }
    issue();
  }
  __device__ __forceinline__ void row(uint32_t, float (&x)[K]) { fetch(x); }
  __device__ __forceinline__ void targets(float (&x)[K]) { fetch(x); }
  __device__ __forceinline__ void next_tile() {}
};

// Input rows of a whole case set held in LDS (the resident kernels), in the
// staged layout.
template <int K>
struct TableRows {
  const float* x;  // this lane's cases of row 0 of the current tile
  uint32_t rows_f, half;
  __device__ __forceinline__ void start(const EvalArgs& a, const float* table) {
    x = table + (threadIdx.x & 63u) * 4u;
    rows_f = uint32_t(a.rows) * TILE;
    half = K == 4 ? 256u : 0u;
  }
  __device__ __forceinline__ void row(uint32_t r, float (&v)[K]) const {
#pragma unroll
    for (int g = 0; g < K / 4; ++g) {
      const float4 q = *reinterpret_cast<const float4*>(x + r * uint32_t(TILE) + g * 256);
      v[4 * g + 0] = q.x;
      v[4 * g + 1] = q.y;
      v[4 * g + 2] = q.z;
      v[4 * g + 3] = q.w;
    }
  }
  __device__ __forceinline__ void targets(float (&v)[K]) const { row(rows_f / TILE - 1, v); }
  __device__ __forceinline__ void next_tile() {
    if constexpr (K == 8) {
      x += rows_f;
    } else {
      // the other half of the tile, or the next tile's first
      x += half;
      half = rows_f - half;
    }
  }
};

// Rows of one case per lane in LDS, 64 of a row together (k_outputs_small).
struct LaneRows {
  const float* x;
  __device__ __forceinline__ void row(uint32_t r, float (&v)[1]) const { v[0] = x[r * 64u]; }
};

// Rows of case 0, read straight from global memory (the shifts).
struct DirectRows {
  const float* x;
  __device__ __forceinline__ void row(uint32_t r, float (&v)[1]) const { v[0] = x[r * uint32_t(TILE)]; }
};

// A word and a constant per lane, loaded and waited for in one place: the
// wait for an ordinary load would be placed where its path joins the common
// one and hold up every tile.
__device__ __forceinline__ void load_now(const uint32_t* w, const float* v, uint32_t& word, float& value) {
  asm volatile(
      "global_load_dword %0, %2, off\n\t"
      "global_load_dword %1, %3, off\n\t"
      "s_waitcnt vmcnt(0)"
      : "=&v"(word), "=&v"(value)
      : "v"(w), "v"(v)
      : "memory");
}

// The stack interpreter for one program on K cases per lane.
//   vc0/vv0: instruction words / constant values of tokens 0..63 (one per
//   lane); longer programs read later tokens from memory, 64 at a time.  rows
//   gives the input rows of VAR words.
template <int K, int S, class Rows>
__device__ __forceinline__ void interpret(uint32_t vc0, float vv0, const uint32_t* __restrict__ code,
                                          const float* __restrict__ cval,
                                          int L, int lane, Rows& rows, float (&top)[K]) {
  // S slots: the unconditional store of a token at stack size n = S lands in
  // slot S-1, above the S-1 live values
  // (at S = 16 an array per case: one of all cases would be too large to be
  // indexed in registers; at S = 8 one array is a third faster)
  static_assert(K <= 4, "at most four cases per lane");
  constexpr bool ONE = S <= 8;
  float all[ONE ? K : 1][S];
  float s0[ONE ? 1 : S], s1[ONE ? 1 : S], s2[ONE ? 1 : S], s3[ONE ? 1 : S];
  float* const stk[4] = {ONE ? all[0] : s0, ONE ? all[K > 1 ? 1 : 0] : s1, ONE ? all[K > 2 ? 2 : 0] : s2,
                         ONE ? all[K > 3 ? 3 : 0] : s3};
#pragma unroll
  for (int k = 0; k < K; ++k) {
    top[k] = 0.0f;
#pragma unroll
    for (int j = 0; j < S; ++j) stk[k][j] = 0.0f;
  }
  for (int base = 0; base < L; base += 64) {
    uint32_t vc = vc0;
    float vv = vv0;
    if (base != 0) {
      const int i = base + lane < L ? base + lane : L - 1;
      load_now(code + i, cval + i, vc, vv);
    }
    const int n = __builtin_amdgcn_readfirstlane(L - base < 64 ? L - base : 64);
    for (int t = 0; t < n; ++t) {
      const uint32_t w = __builtin_amdgcn_readlane(vc, t);
      const uint32_t arg = (w >> 8) & 0xFFu;
      const uint32_t ws = (w >> 16) & 0xFu;
#pragma unroll
      for (int k = 0; k < K; ++k) stk[k][ws] = top[k];
      switch (w & 0xFFu) {
        case H_VAR: {
          rows.row(arg, top);
          break;
        }
        case H_CONST: {
          const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vv), t));
#pragma unroll
          for (int k = 0; k < K; ++k) top[k] = v;
          break;
        }
#define BGL_BIN(O, N)                                                          \
  case H_BIN + 15 * O + (N - 2):                                               \
    if constexpr (N <= S) {                                                    \
      float a_[K], t_[K];                                                      \
      _Pragma("unroll") for (int k = 0; k < K; ++k) {                          \
        a_[k] = stk[k][N <= S ? N - 2 : 0];                                    \
        t_[k] = top[k];                                                        \
      }                                                                        \
      binop_tile<O, K>(a_, t_, top);                                           \
    }                                                                          \
    break;
#define BGL_BIN_ALL(O)                                                          \
  BGL_BIN(O, 2) BGL_BIN(O, 3) BGL_BIN(O, 4) BGL_BIN(O, 5) BGL_BIN(O, 6) BGL_BIN(O, 7) \
  BGL_BIN(O, 8) BGL_BIN(O, 9) BGL_BIN(O, 10) BGL_BIN(O, 11) BGL_BIN(O, 12)     \
  BGL_BIN(O, 13) BGL_BIN(O, 14) BGL_BIN(O, 15) BGL_BIN(O, 16)
        BGL_BIN_ALL(B_ADD)
        BGL_BIN_ALL(B_SUB)
        BGL_BIN_ALL(B_MUL)
        BGL_BIN_ALL(B_DIV)
        BGL_BIN_ALL(B_RSUB)
        BGL_BIN_ALL(B_RDIV)
#undef BGL_BIN
#undef BGL_BIN_ALL
#define BGL_FUSED(O)                                                           \
  case H_FUSED + O: {                                                          \
    float x_[K], t_[K];                                                        \
    rows.row(arg, x_);                                                         \
    _Pragma("unroll") for (int k = 0; k < K; ++k) t_[k] = top[k];              \
    binop_tile<O, K>(t_, x_, top);                                             \
    break;                                                                     \
  }                                                                            \
  case H_FUSED + 6 + O: {                                                      \
    const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vv), t)); \
    float t_[K], c_[K];                                                        \
    _Pragma("unroll") for (int k = 0; k < K; ++k) {                            \
      t_[k] = top[k];                                                          \
      c_[k] = v;                                                               \
    }                                                                          \
    binop_tile<O, K>(t_, c_, top);                                             \
    break;                                                                     \
  }
        BGL_FUSED(B_ADD)
        BGL_FUSED(B_SUB)
        BGL_FUSED(B_MUL)
        BGL_FUSED(B_DIV)
        BGL_FUSED(B_RSUB)
        BGL_FUSED(B_RDIV)
#undef BGL_FUSED
        case H_UN + 0:
          trig_tile<false, K>(top);
          break;
        case H_UN + 1:
          trig_tile<true, K>(top);
          break;
        case H_UN + 2:
          exp_tile<K>(top);
          break;
        case H_UN + 3:
          log_tile<K>(top);
          break;
        case H_UN + 4:
          sqrt_tile<K>(top);
          break;
#define BGL_EXT(U)                                                             \
  case H_UN + U:                                                               \
    _Pragma("unroll") for (int k = 0; k < K; ++k) top[k] = op_ext<U>(top[k]);  \
    break;
        BGL_EXT(5) BGL_EXT(6) BGL_EXT(7) BGL_EXT(8) BGL_EXT(9) BGL_EXT(10) BGL_EXT(11)
#undef BGL_EXT
        default:
          break;
      }
    }
  }
}

// The small-stack interpreter (programs of register need <= 4): no cached
// top; the handler index i0 (word bits 24..31) names the stack size, so each
// handler reads and rewrites its slots in place and no word moves values
// between registers.  st[k][j] is stack slot j of case k; the result is slot 0.
template <int K, class Rows>
__device__ __forceinline__ void interpret_small(uint32_t vc0, float vv0, const uint32_t* __restrict__ code,
                                                const float* __restrict__ cval,
                                                int L, int lane, Rows& rows, float (&res)[K]) {
  constexpr int S = 4;
  float st[K][S];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int j = 0; j < S; ++j) st[k][j] = 0.0f;
  for (int base = 0; base < L; base += 64) {
    uint32_t vc = vc0;
    float vv = vv0;
    if (base != 0) {
      const int i = base + lane < L ? base + lane : L - 1;
      load_now(code + i, cval + i, vc, vv);
    }
    const int n = __builtin_amdgcn_readfirstlane(L - base < 64 ? L - base : 64);
    for (int t = 0; t < n; ++t) {
      const uint32_t w = __builtin_amdgcn_readlane(vc, t);
      const uint32_t arg = (w >> 8) & 0xFFu;
      switch (w >> 24) {
#define BGL_S_PUSH(N)                                                           \
  case I0_PUSH_VAR + N: {                                                       \
    float x_[K];                                                                \
    rows.row(arg, x_);                                                          \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N] = x_[k];             \
    break;                                                                      \
  }                                                                             \
  case I0_PUSH_CONST + N: {                                                     \
    const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vv), t)); \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N] = v;                 \
    break;                                                                      \
  }
        BGL_S_PUSH(0) BGL_S_PUSH(1) BGL_S_PUSH(2) BGL_S_PUSH(3)
#undef BGL_S_PUSH
#define BGL_S_BIN(O, N)                                                         \
  case I0_BIN + 3 * O + (N - 2): {                                              \
    float a_[K], b_[K], r_[K];                                                  \
    _Pragma("unroll") for (int k = 0; k < K; ++k) {                             \
      a_[k] = st[k][N - 2];                                                     \
      b_[k] = st[k][N - 1];                                                     \
    }                                                                           \
    binop_tile<O, K>(a_, b_, r_);                                               \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 2] = r_[k];         \
    break;                                                                      \
  }
#define BGL_S_BIN3(O) BGL_S_BIN(O, 2) BGL_S_BIN(O, 3) BGL_S_BIN(O, 4)
        BGL_S_BIN3(B_ADD) BGL_S_BIN3(B_SUB) BGL_S_BIN3(B_MUL) BGL_S_BIN3(B_DIV) BGL_S_BIN3(B_RSUB) BGL_S_BIN3(B_RDIV)
#undef BGL_S_BIN3
#undef BGL_S_BIN
#define BGL_S_UN(N)                                                             \
  case I0_UN + 0 * 4 + (N - 1): {                                               \
    float c[K];                                                                 \
    _Pragma("unroll") for (int k = 0; k < K; ++k) c[k] = st[k][N - 1];          \
    trig_tile<false, K>(c);                                                     \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = c[k];          \
    break;                                                                      \
  }                                                                             \
  case I0_UN + 1 * 4 + (N - 1): {                                               \
    float c[K];                                                                 \
    _Pragma("unroll") for (int k = 0; k < K; ++k) c[k] = st[k][N - 1];          \
    trig_tile<true, K>(c);                                                      \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = c[k];          \
    break;                                                                      \
  }                                                                             \
  case I0_UN + 2 * 4 + (N - 1): {                                               \
    float c[K];                                                                 \
    _Pragma("unroll") for (int k = 0; k < K; ++k) c[k] = st[k][N - 1];          \
    exp_tile<K>(c);                                                             \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = c[k];          \
    break;                                                                      \
  }                                                                             \
  case I0_UN + 3 * 4 + (N - 1): {                                               \
    float c[K];                                                                 \
    _Pragma("unroll") for (int k = 0; k < K; ++k) c[k] = st[k][N - 1];          \
    log_tile<K>(c);                                                             \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = c[k];          \
    break;                                                                      \
  }                                                                             \
  case I0_UN + 4 * 4 + (N - 1): {                                               \
    float c[K];                                                                 \
    _Pragma("unroll") for (int k = 0; k < K; ++k) c[k] = st[k][N - 1];          \
    sqrt_tile<K>(c);                                                            \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = c[k];          \
    break;                                                                      \
  }
        BGL_S_UN(1) BGL_S_UN(2) BGL_S_UN(3) BGL_S_UN(4)
#undef BGL_S_UN
#define BGL_S_FUSED(O, N)                                                       \
  case I0_FUSED + 3 * O + (N - 1): {                                            \
    float x_[K], a_[K], r_[K];                                                  \
    rows.row(arg, x_);                                                          \
    _Pragma("unroll") for (int k = 0; k < K; ++k) a_[k] = st[k][N - 1];         \
    binop_tile<O, K>(a_, x_, r_);                                               \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = r_[k];         \
    break;                                                                      \
  }                                                                             \
  case I0_FUSED + 3 * (6 + O) + (N - 1): {                                      \
    const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vv), t)); \
    float a_[K], c_[K], r_[K];                                                  \
    _Pragma("unroll") for (int k = 0; k < K; ++k) {                             \
      a_[k] = st[k][N - 1];                                                     \
      c_[k] = v;                                                                \
    }                                                                           \
    binop_tile<O, K>(a_, c_, r_);                                               \
    _Pragma("unroll") for (int k = 0; k < K; ++k) st[k][N - 1] = r_[k];         \
    break;                                                                      \
  }
#define BGL_S_FUSED3(O) BGL_S_FUSED(O, 1) BGL_S_FUSED(O, 2) BGL_S_FUSED(O, 3)
        BGL_S_FUSED3(B_ADD) BGL_S_FUSED3(B_SUB) BGL_S_FUSED3(B_MUL) BGL_S_FUSED3(B_DIV) BGL_S_FUSED3(B_RSUB)
        BGL_S_FUSED3(B_RDIV)
#undef BGL_S_FUSED3
#undef BGL_S_FUSED
        default:
          break;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) res[k] = st[k][0];
}

// Eq. 3 for one case (the paper's point-to-point score, see beagle.h): the
// products and differences rounded separately (no contraction), so that the
// rounding decision is the one a plain binary64 evaluation takes.
__device__ __forceinline__ double point_case(float yh, float y, double smax, double s11) {
  const bool vh = isfinite(yh), vy = isfinite(y);
  if (!(vh && vy)) return vh == vy ? smax : -smax;
  const double a = fabs(double(yh)), b = fabs(double(y));
  const double hi = a > b ? a : b, lo = a > b ? b : a;
  if (hi == 0.0) return smax;
  double t = __dmul_rn(smax, lo / hi);
  if ((yh < 0.0f && y > 0.0f) || (yh > 0.0f && y < 0.0f)) t = __dsub_rn(t, s11);
  return __builtin_rint(t);
}

// Per-lane accumulators of one fitness kind over the cases a lane adds, and
// their wave sums in partial order (see eval_block).
template <int KIND>
struct Acc {
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0;
  uint32_t n1 = 0u, n2 = 0u;
  __device__ __forceinline__ void add(float yh, float yt, bool valid, double shift, double ybar, double smax,
                                      double s11) {
    // masks act on the terms' inputs and every product is an explicit FMA,
    // so a case adds the same bits whether its tile is masked or not
    if constexpr (KIND == BEAGLE_FIT_MSE) {
      const double d = valid ? double(yh) - double(yt) : 0.0;
      s0 = __builtin_fma(d, d, s0);
    } else if constexpr (KIND == BEAGLE_FIT_CORR) {
      const double u = valid ? double(yh) - shift : 0.0;
      const double w = valid ? double(yt) - ybar : 0.0;
      s0 += u;
      s1 = __builtin_fma(u, u, s1);
      s2 = __builtin_fma(u, w, s2);
    } else if constexpr (KIND == BEAGLE_FIT_POINT) {
      s0 += valid ? point_case(yh, yt, smax, s11) : 0.0;
    } else {
      const bool vh = isfinite(yh), vy = isfinite(yt);
      const bool both = valid && vh && vy;
      n1 += valid && vh != vy ? 1u : 0u;
      n2 += valid && !vh && !vy ? 1u : 0u;
      const double u = both ? double(yh) - shift : 0.0;
      const double w = both ? double(yt) - ybar : 0.0;
      s0 += u;
      s1 = __builtin_fma(u, u, s1);
      s2 = __builtin_fma(u, w, s2);
      s3 += w;
      s4 = __builtin_fma(w, w, s4);
    }
  }
  // the wave's sums in partial order: MSE, POINT {s0}; CORR {s0, s1, s2};
  // R4 {c1, c2, s0, s1, s2, s3, s4}
  __device__ __forceinline__ void wave_sums(double (&v)[MAX_SUMS]) const {
    if constexpr (KIND == BEAGLE_FIT_R4) {
      v[0] = wave_sum(double(n1));
      v[1] = wave_sum(double(n2));
      v[2] = wave_sum(s0);
      v[3] = wave_sum(s1);
      v[4] = wave_sum(s2);
      v[5] = wave_sum(s3);
      v[6] = wave_sum(s4);
    } else {
      v[0] = wave_sum(s0);
      if constexpr (KIND == BEAGLE_FIT_CORR) {
        v[1] = wave_sum(s1);
        v[2] = wave_sum(s2);
      }
    }
  }
};

// One wave: program p on case chunk c.  Writes the chunk's partial sums
//   MSE  : part[0][c][p] = sum (yhat - y)^2
//   CORR : part[j][c][p] = sum u, sum u^2, sum u*w   (u = yhat - shift_p,
//          w = y - ybar), all in binary64
//   POINT: part[0][c][p] = sum of the Eq. 3 case scores (integers, exact)
//   R4   : part[j][c][p] = c1, c2 (cases with one / two invalid values), and
//          over the cases where both are valid sum u, sum u^2, sum u*w,
//          sum w, sum w^2.
// Case order: lane l holds cases 4l .. 4l+3 of every 256 (a tile with K = 8
// is two such runs), and adds its cases in increasing order, so the tile
// width changes no result bit.
// RESIDENT: `lds` is the table of the whole case set (one chunk), else the
// wave's ring.
template <int KIND, int K, int S, bool RESIDENT>
__device__ __forceinline__ void eval_wave(const EvalArgs& a, int p, int c, float* lds) {
  const ProgMeta m = a.meta[p];
  const int lane = threadIdx.x & 63;
  const int64_t off = a.tok_offset[p];
  const uint32_t* code = a.code + off;
  const float* cval = a.cval + off;
  const int L = __builtin_amdgcn_readfirstlane(m.len);
  const int64_t c0 = int64_t(c) * a.chunk;
  const int64_t c1 = c0 + a.chunk < a.M ? c0 + a.chunk : a.M;
  std::conditional_t<RESIDENT, TableRows<K>, RowRing<K>> rows;
  if constexpr (RESIDENT)
    rows.start(a, lds);
  else
    rows.start(a, lds, a.vrow + off, __builtin_amdgcn_readfirstlane(m.nv), KIND != KIND_OUTPUTS, c0, c1);
  const uint32_t vc0 = lane < L ? code[lane] : 0u;
  const float vv0 = lane < L ? cval[lane] : 0.0f;
  constexpr bool SHIFTED = KIND == BEAGLE_FIT_CORR || KIND == BEAGLE_FIT_R4;
  double shift = double(m.shift);
  const double ybar = SHIFTED ? a.stats[0] : 0.0;
  const double smax = a.smax, s11 = a.smax / 11.0;
  Acc<KIND> acc;
  for (int64_t base = c0; base < c1; base += 64 * K) {
    float top[K], yk[K];
    if constexpr (S == 4)
      interpret_small<K>(vc0, vv0, code, cval, L, lane, rows, top);
    else
      interpret<K, S>(vc0, vv0, code, cval, L, lane, rows, top);
    if constexpr (KIND == KIND_OUTPUTS) {
      rows.next_tile();
      const int64_t i = base + 4 * lane;
      float* out = a.out + int64_t(p) * a.M + i;
      // (four cases of a lane are one 16-byte store where a program's outputs
      // start on 16 bytes)
      const bool quads = (reinterpret_cast<uintptr_t>(a.out) & 15u) == 0 && (a.M & 3) == 0;
#pragma unroll
      for (int g = 0; g < K / 4; ++g) {
        if (quads) {
          if (i + g * 256 < c1)
            *reinterpret_cast<float4*>(out + g * 256) =
                make_float4(top[4 * g], top[4 * g + 1], top[4 * g + 2], top[4 * g + 3]);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (i + g * 256 + k < c1) out[g * 256 + k] = top[4 * g + k];
        }
      }
      continue;
    }
    rows.targets(yk);
    rows.next_tile();
    if (SHIFTED && a.meta_shift && base == c0) {
      // (one chunk) the shift is the output at case 0 (lane 0, first case)
      // when finite
      const float y0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(top[0]), 0));
      const float sh = isfinite(y0) ? y0 : 0.0f;
      if (lane == 0) a.meta_shift[p].shift = sh;
      shift = double(sh);
    }
    // a tile wholly inside the chunk (every tile but the last) adds without
    // per-case validity masks
    if (base + 64 * K <= c1) {
#pragma unroll
      for (int k = 0; k < K; ++k) acc.add(top[k], yk[k], true, shift, ybar, smax, s11);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool valid = base + (k / 4) * 256 + 4 * lane + (k % 4) < c1;
        acc.add(top[k], yk[k], valid, shift, ybar, smax, s11);
      }
    }
  }
  if constexpr (KIND != KIND_OUTPUTS) {
    double v[MAX_SUMS];
    acc.wave_sums(v);
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < kind_sums(KIND); ++j) a.part[(int64_t(j) * a.n_chunks + c) * a.n_programs + p] = v[j];
    }
  }
  // the look-ahead's last loads land before another item's are issued
  if constexpr (!RESIDENT) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
}

// One register-need class: a persistent grid's waves take (chunk, program)
// work items, chunk-major so that the waves running at any moment share one
// chunk of cases in L2.  Which wave takes which item does not change any
// result: each item writes its own partial.
template <int KIND, int CLS, int KV>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CLS == 0 ? (KV == 1 ? CLASS0_NARROW_WAVES : CLASS0_WIDE_WAVES) : CLS == 1 ? 4 : 1)))
k_eval_class(EvalArgs a) {
  constexpr int S = class_stack(CLS);
  constexpr int K = class_k(CLS, KV);
  __shared__ __align__(16) float rings[EVAL_WAVES][RING * K * 64];
  const int32_t count = __builtin_amdgcn_readfirstlane(a.class_count[CLS]);
  const int64_t items = int64_t(count) * a.n_chunks;
  const int32_t* list = a.class_list + int64_t(CLS) * a.n_total;
  // workgroups beyond the items leave at once
  if (int64_t(blockIdx.x) * EVAL_WAVES >= items) return;
  float* ring = rings[__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6))];
  WaveItems work(items, a.work + CLS * counter_words(a.work_shift), a.work_shift);
  for (;;) {
    const int64_t it = work.next(CLS == 0 && a.chunk < 2 * TILE ? 2 : 1);
    if (it < 0) break;
    const int c = a.n_chunks == 1 ? 0 : int(it / count);
    const int p = __builtin_amdgcn_readfirstlane(list[it - int64_t(c) * count] - a.prog_begin);
    // (else a program of another slice)
    if (p >= 0 && p < a.n_programs) eval_wave<KIND, K, S, false>(a, p, c, ring);
  }
}

// All register-need classes in one launch, for few work items.
template <int KIND>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1))) k_eval_mixed(EvalArgs a) {
  __shared__ __align__(16) float rings[EVAL_WAVES][RING * 4 * 64];
  const int32_t n0 = __builtin_amdgcn_readfirstlane(a.class_count[0]);
  const int32_t n01 = n0 + __builtin_amdgcn_readfirstlane(a.class_count[1]);
  const int32_t count = n01 + __builtin_amdgcn_readfirstlane(a.class_count[2]);
  const int64_t items = int64_t(count) * a.n_chunks;
  if (int64_t(blockIdx.x) * EVAL_WAVES >= items) return;
  float* ring = rings[__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6))];
  WaveItems work(items, a.work, a.work_shift);
  for (;;) {
    const int64_t it = work.next(1);
    if (it < 0) break;
    const int c = int(it / count), i = int(it - int64_t(c) * count);
    const int cls = i < n0 ? 0 : i < n01 ? 1 : 2;
    const int p = __builtin_amdgcn_readfirstlane(
        a.class_list[int64_t(cls) * a.n_total + i - (cls == 0 ? 0 : cls == 1 ? n0 : n01)] - a.prog_begin);
    if (p < 0 || p >= a.n_programs) continue;  // a program of another slice
    if (cls == 0)
      eval_wave<KIND, 4, 4, false>(a, p, c, ring);
    else if (cls == 1)
      eval_wave<KIND, 4, 8, false>(a, p, c, ring);
    else
      eval_wave<KIND, 4, 16, false>(a, p, c, ring);
  }
}

// Small case sets (one chunk whose staged rows fit a compute unit's LDS):
// every workgroup copies all of them once, and each wave then takes whole
// programs, reading rows where it needs them: no look-ahead, no list of rows,
// and a program's start (a few thousand cycles behind the ring's first loads
// where a program has one tile) costs only its header.  The waves of a
// workgroup are as many as let the workgroups that fit fill the SIMDs (see
// resident_shape).
template <int KIND, int K, int CLS>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 1024), amdgpu_waves_per_eu(CLS == 0 ? RESIDENT_WAVES : 4)))
k_eval_resident(EvalArgs a) {
  extern __shared__ __align__(16) float table[];
  const int32_t count = __builtin_amdgcn_readfirstlane(a.class_count[CLS]);
  const int32_t* list = a.class_list + int64_t(CLS) * a.n_total;
  // workgroups whose waves would find nothing leave before copying
  if (int64_t(blockIdx.x) * int(blockDim.x >> 6) >= count) return;
  const int n4 = int((a.M + TILE - 1) / TILE) * a.rows * (TILE / 4);
  for (int i = threadIdx.x; i < n4; i += blockDim.x)
    reinterpret_cast<float4*>(table)[i] = reinterpret_cast<const float4*>(a.Xt)[i];
  __syncthreads();
  WaveItems work(count, a.work + CLS * counter_words(a.work_shift), a.work_shift);
  for (;;) {
    const int64_t it = work.next(claim_least(a.M));
    if (it < 0) break;
    const int p = __builtin_amdgcn_readfirstlane(list[it] - a.prog_begin);
    if (p >= 0 && p < a.n_programs) eval_wave<KIND, K, class_stack(CLS), true>(a, p, 0, table);  // else another slice's
  }
}

// One work list of a batched evaluation (a class and tile variant): the
// same persistent scheme over the (problem, chunk, program) items of the
// table's problems in that list, problem by problem in table order and
// chunk-major within a problem.  Items are claimed in increasing order, so a
// wave's next item lies in its previous item's problem or a later one: the
// problem is found by stepping forward from there when it is near, by
// bisection otherwise.
template <int KIND, int CLS, int KV>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CLS == 0 ? (KV == 1 ? CLASS0_NARROW_WAVES : BATCH_WIDE_WAVES) : CLS == 1 ? 4 : 1)))
k_eval_batch(BatchArgs b, int vl) {
  constexpr int S = class_stack(CLS);
  constexpr int K = class_k(CLS, KV);
  __shared__ __align__(16) float rings[EVAL_WAVES][RING * K * 64];
  const int64_t* off = b.item_off + int64_t(vl) * (b.n_problems + 1);
  const int64_t items = off[b.n_problems];
  if (int64_t(blockIdx.x) * EVAL_WAVES >= items) return;  // (as in k_eval_class)
  float* ring = rings[__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6))];
  WaveItems work(items, b.work + vl * counter_words(b.work_shift), b.work_shift);
  int lo = 0;  // the problem of the previous item (a lower bound for the next)
  for (;;) {
    const int64_t it = work.next(2);
    if (it < 0) break;
    // the last problem q >= lo with off[q] <= it (problems without items in
    // this list have empty ranges and are stepped over)
    int steps = 0;
    while (steps < 4 && lo + 1 < b.n_problems && off[lo + 1] <= it) {
      ++lo;
      ++steps;
    }
    if (steps == 4) {
      int hi = b.n_problems;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= it)
          lo = mid;
        else
          hi = mid;
      }
    }
    const BatchProblem& P = b.table[lo];
    const int32_t count = P.prep.class_count[CLS];
    const int64_t local = it - off[lo];
    const int c = int(local / count);
    const int p = __builtin_amdgcn_readfirstlane(P.prep.class_list[int64_t(CLS) * P.prep.n_programs + local % count]);
    EvalArgs a;
    a.code = P.prep.code;
    a.cval = P.prep.cval;
    a.vrow = P.prep.vrow;
    a.tok_offset = P.prep.tok_offset;
    a.meta = P.prep.meta;
    a.Xt = P.Xt;
    a.rows = P.rows;
    a.M = P.M;
    a.n_programs = P.prep.n_programs;
    a.n_chunks = P.n_chunks;
    a.chunk = P.chunk;
    a.part = P.part;
    a.stats = P.stats;
    a.class_count = nullptr;
    a.class_list = nullptr;
    a.work = nullptr;
    a.work_shift = 0;
    a.n_total = P.prep.n_programs;
    a.prog_begin = 0;
    a.meta_shift = P.n_chunks == 1 ? P.prep.meta : nullptr;
    eval_wave<KIND, K, S, false>(a, p, c, ring);
  }
}

// Every program's output at case 0, where finite, as the shift of its
// correlation sums (a non-finite one is either the whole fitness, NaN, or an
// invalid pair of the paper's scores): one wave per program.
__device__ static void shift_program(const ValuesArgs& a, int p) {
  const int lane = threadIdx.x;
  const ProgMeta m = a.meta[p];
  if (m.status != BEAGLE_PROG_OK) return;
  const int64_t off = a.tok_offset[p];
  const uint32_t* code = a.code + off;
  const float* cval = a.cval + off;
  const int L = m.len;
  const uint32_t vc0 = lane < L ? code[lane] : 0u;
  const float vv0 = lane < L ? cval[lane] : 0.0f;
  DirectRows rows{a.Xt};
  float top[1];
  interpret<1, MAX_STACK>(vc0, vv0, code, cval, L, lane, rows, top);
  if (lane == 0) a.meta[p].shift = isfinite(top[0]) ? top[0] : 0.0f;
}

__global__ void __launch_bounds__(64) k_shifts(ValuesArgs a) { shift_program(a, blockIdx.x); }

// Correlation shifts of every program of the table's problems of more than
// one chunk (one wave per program; the evaluator finds the others').
__global__ void __launch_bounds__(64) k_shifts_batch(BatchArgs b) {
  const int64_t g = blockIdx.x;
  const int q = batch_find(b, g, [](const BatchProblem& t) { return t.prog_begin; });
  const BatchProblem& P = b.table[q];
  if (P.n_chunks == 1) return;
  ValuesArgs a;
  a.code = P.prep.code;
  a.cval = P.prep.cval;
  a.tok_offset = P.prep.tok_offset;
  a.meta = P.prep.meta;
  a.Xt = P.Xt;
  a.rows = P.rows;
  shift_program(a, int(g - P.prog_begin));
}

// Outputs of one program on 64 cases, a case per lane: four times the waves of
// the narrow tile, which is what counts with few of them, and nothing computed
// for cases that aren't there (100 000 programs x 64 cases: 190 us, with the
// narrow tile 280; 5000 x 64 45 and 60; 300 x 3000 with the further operators 35 and
// 40).  Invalid programs' rows are NaN.
__global__ void __launch_bounds__(64) k_outputs_small(ValuesArgs a, int64_t M, int32_t D, float* out) {
  __shared__ float x[MAX_D * 64];
  const int p = blockIdx.x, lane = threadIdx.x;
  const int64_t i = int64_t(blockIdx.y) * 64 + lane;
  const ProgMeta m = a.meta[p];
  float top[1] = {__int_as_float(0x7FC00000)};
  if (m.status == BEAGLE_PROG_OK) {
    const int64_t off = a.tok_offset[p];
    const uint32_t* code = a.code + off;
    const float* cval = a.cval + off;
    const int L = m.len;
    const uint32_t vc0 = lane < L ? code[lane] : 0u;
    const float vv0 = lane < L ? cval[lane] : 0.0f;
    const float* xt = a.Xt + case_offset(i, a.rows);
    for (int d = 0; d < D; ++d)
      if ((m.vmask >> d) & 1u) x[d * 64 + lane] = xt[d * TILE];
    __syncthreads();
    LaneRows rows{x + lane};
    interpret<1, MAX_STACK>(vc0, vv0, code, cval, L, lane, rows, top);
  }
  if (i < M) out[int64_t(p) * M + i] = top[0];
}

__global__ void __launch_bounds__(256) k_nan_rows(const ProgMeta* meta, int32_t n_programs, int64_t M,
                                                  float* out) {
  for (int64_t p = blockIdx.x; p < n_programs; p += gridDim.x) {
    if (meta[p].status == BEAGLE_PROG_OK) continue;
    for (int64_t i = threadIdx.x; i < M; i += 256) out[p * M + i] = __int_as_float(0x7FC00000);
  }
}

// Fitness of every program from its chunk partials.  Up to
// WIDE_FINALIZE_CHUNKS a thread adds them in chunk order, eight loaded ahead of
// their additions; more (WIDE) a wave, lane l chunks l, l + 64, ... and then the
// lanes' sums: one load after the other, the 73 chunks of a problem took 55 us.
template <bool WIDE>
__device__ static double chunk_sum(const FinalizeArgs& a, int j, int p) {
  const double* part = a.part + int64_t(j) * a.n_chunks * a.n_programs + p;
  double s = 0.0;
  if constexpr (WIDE) {
#pragma unroll 4
    for (int c = threadIdx.x & 63; c < a.n_chunks; c += 64) s += part[int64_t(c) * a.n_programs];
    return wave_sum(s);
  }
  int c = 0;
  for (; c + 8 <= a.n_chunks; c += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[int64_t(c + u) * a.n_programs];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; c < a.n_chunks; ++c) s += part[int64_t(c) * a.n_programs];
  return s;
}

// (WIDE: every lane of the wave, with the same p)
template <bool WIDE>
__device__ static void finalize_program(const FinalizeArgs& a, int p) {
  const ProgMeta m = a.meta[p];
  const bool one = !WIDE || (threadIdx.x & 63) == 0;
  const double nan = __longlong_as_double(0x7FF8000000000000LL);
  double F;
  if (m.status != BEAGLE_PROG_OK) {
    F = nan;
  } else if (a.kind == BEAGLE_FIT_MSE) {
    F = chunk_sum<WIDE>(a, 0, p) / double(a.M);
  } else if (a.kind == BEAGLE_FIT_POINT) {
    F = chunk_sum<WIDE>(a, 0, p);
  } else if (a.kind == BEAGLE_FIT_R4) {
    double s[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) s[j] = chunk_sum<WIDE>(a, j, p);
    const double c1 = s[0], c2 = s[1], n = double(a.M) - c1 - c2;
    double r = 0.0;
    if (n >= 2.0) {
      const double sxx = s[3] - s[2] * s[2] / n;
      const double syy = s[6] - s[5] * s[5] / n;
      const double sxy = s[4] - s[2] * s[5] / n;
      if (sxx > 0.0 && syy > 0.0) r = sxy / sqrt(sxx * syy);
    }
    const double r2 = r * r;
    F = a.smax * (r2 * r2) * n - a.smax * (c1 - c2);
  } else {
    double s[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) s[j] = chunk_sum<WIDE>(a, j, p);
    const double Md = double(a.M);
    const double syy = a.stats[2], sw = a.stats[1];
    // gradient seed (1 - r^2 differentiated, unclamped; zero for a constant
    // output, NaN for a NaN fitness): with u = yhat - shift and w = y - ybar,
    // Sxx = sum u^2 - (sum u)^2 / M, Sxy = sum u w - sum u sum w / M, so
    // dSxx/dyhat_i = 2 (yhat_i - mu), dSxy/dyhat_i = w_i - mean w and
    // dF/dyhat_i = -2 r (dSxy/dyhat_i / sqrt(Sxx Syy) - r (yhat_i - mu) / Sxx)
    double alpha = nan, beta = nan, mu = nan;
    if (!isfinite(s[0]) || !isfinite(s[1]) || !isfinite(s[2])) {
      F = nan;
    } else if (!(syy > 0.0)) {
      F = nan;
    } else {
      const double sxx = s[1] - s[0] * s[0] / Md;
      const double sxy = s[2] - s[0] * sw / Md;
      mu = double(m.shift) + s[0] / Md;
      if (!(sxx > 0.0)) {
        F = 1.0;
        alpha = beta = 0.0;
      } else {
        const double q = sqrt(sxx * syy);
        const double r = sxy / q;
        F = 1.0 - r * r;
        F = F < 0.0 ? 0.0 : (F > 1.0 ? 1.0 : F);
        alpha = -2.0 * r / q;
        beta = 2.0 * r * r / sxx;
      }
    }
    if (a.coef && one) {
      a.coef[3 * int64_t(p)] = alpha;
      a.coef[3 * int64_t(p) + 1] = beta;
      a.coef[3 * int64_t(p) + 2] = mu;
    }
  }
  if (one) a.fitness[p] = F;
}

__global__ void __launch_bounds__(64) k_finalize(FinalizeArgs a) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < a.n_programs) finalize_program<false>(a, p);
}

__global__ void __launch_bounds__(256) k_finalize_wide(FinalizeArgs a) {
  for (int64_t p = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6); p < a.n_programs; p += int64_t(gridDim.x) * 4)
    finalize_program<true>(a, int(p));
}

void launch_finalize(const FinalizeArgs& a, hipStream_t s) {
  if (a.n_chunks > WIDE_FINALIZE_CHUNKS)
    hipLaunchKernelGGL(k_finalize_wide, dim3(std::min((a.n_programs + 3) / 4, 1 << 20)), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_finalize, dim3((a.n_programs + 63) / 64), dim3(64), 0, s, a);
}

// One wave per program of every problem of the table.
__global__ void __launch_bounds__(256) k_finalize_batch(BatchArgs b) {
  for (int64_t g = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6); g < b.n_programs; g += int64_t(gridDim.x) * 4) {
    const int q = batch_find(b, g, [](const BatchProblem& t) { return t.prog_begin; });
    const BatchProblem& P = b.table[q];
    FinalizeArgs a;
    a.meta = P.prep.meta;
    a.part = P.part;
    a.stats = P.stats;
    a.M = P.M;
    a.n_programs = P.prep.n_programs;
    a.n_chunks = P.n_chunks;
    a.kind = b.kind;
    a.fitness = P.fitness;
    a.coef = nullptr;
    const int p = int(g - P.prog_begin);
    if (P.n_chunks > WIDE_FINALIZE_CHUNKS)
      finalize_program<true>(a, p);
    else if ((threadIdx.x & 63) == 0)
      finalize_program<false>(a, p);
  }
}

// First work item of every problem in each work list (exclusive prefix sums
// in table order), from the class counts that k_prepare_batch produced.
__global__ void k_batch_items(BatchArgs b) {
  const int v = threadIdx.x;
  if (v >= N_LISTS) return;
  const int cls = v == 0 ? 0 : v - 1;
  int64_t* off = b.item_off + int64_t(v) * (b.n_problems + 1);
  int64_t acc = 0;
  for (int q = 0; q < b.n_problems; ++q) {
    off[q] = acc;
    const BatchProblem& P = b.table[q];
    if (v >= 2 || P.kv == v) acc += int64_t(P.prep.class_count[cls]) * P.n_chunks;
  }
  off[b.n_problems] = acc;
}

__global__ void k_zero_u64(unsigned long long* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0ull;
}

static int cu_count() {
  static int n = 0;
  if (!n) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 1;
  }
  return n;
}

// Persistent grid of a class kernel: resident workgroups per CU, times the CUs.
template <int KIND, int CLS, int KV>
static int class_grid() {
  static int cached = 0;
  if (!cached) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_eval_class<KIND, CLS, KV>, 256, 0) != hipSuccess || nb < 1)
      nb = 1;
    cached = nb * cu_count();
  }
  return cached;
}

template <int KIND, int CLS, int KV>
static hipError_t launch_class(const EvalArgs& a, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr) {
  // (never more waves than programs x chunks)
  const int64_t most = (int64_t(a.n_total) * a.n_chunks + EVAL_WAVES - 1) / EVAL_WAVES;
  const int grid = int(std::min<int64_t>(class_grid<KIND, CLS, KV>(), std::max<int64_t>(most, 1)));
  // timing events, when asked for, are taken by the dispatch itself
  if (ev0 || ev1)
    hipExtLaunchKernelGGL((k_eval_class<KIND, CLS, KV>), dim3(grid), dim3(256), 0, s, ev0, ev1, 0u, a);
  else
    hipLaunchKernelGGL((k_eval_class<KIND, CLS, KV>), dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int KIND, int K, int CLS>
static hipError_t launch_resident(const EvalArgs& a, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr) {
  // (the limit of a kernel's LDS is the current device's)
  static PerDevice<hipError_t> limit_raised;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = limit_raised.get(dev, [] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k_eval_resident<KIND, K, CLS>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, int(RESIDENT_MAX_BYTES));
  });
  if (e != hipSuccess) return e;
  const size_t lds = resident_bytes(a.M, a.rows);
  // Workgroups per CU, of those that fit, and waves of each: together the
  // waves that the registers allow (RESIDENT_WAVES per SIMD, 4 for the deeper
  // class; the narrow tile's registers allow more, which took longer: 16 000
  // programs x 256 cases 45 against 41 us), at most 16 in one workgroup and a
  // multiple of four (a wave of each workgroup more on one SIMD than on another
  // would keep the next workgroup out).  The most that fit are not always the
  // most waves: four tables of 35 KB leave 16 waves, three 24 (20 000 programs of
  // 3..12 tokens x 512 cases, D = 16: 100 and 60 us).
  const int want = 4 * (CLS == 0 ? RESIDENT_WAVES : 4);
  int fit = 1, waves = std::min(16, want);
  for (int f = 2; f <= std::min(want / 4, int(RESIDENT_MAX_BYTES / lds)); ++f) {
    const int w = std::min(16, want / f / 4 * 4);
    if (f * w >= fit * waves) fit = f, waves = w;
  }
  const int grid = fit * cu_count();
  if (ev0 || ev1)
    hipExtLaunchKernelGGL((k_eval_resident<KIND, K, CLS>), dim3(grid), dim3(waves * 64), uint32_t(lds), s, ev0, ev1, 0u,
                          a);
  else
    hipLaunchKernelGGL((k_eval_resident<KIND, K, CLS>), dim3(grid), dim3(waves * 64), lds, s, a);
  return hipGetLastError();
}

template <int KIND>
static hipError_t launch_kind(int kv, const EvalArgs& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                              bool counters_clear) {
  if (!counters_clear)
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(256), 0, s, a.work, N_CLASSES * counter_words(a.work_shift));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // (a chunk of half a tile: only the narrow tile starts inside a tile)
  const bool wide = kv == 0 && a.chunk % TILE == 0;
  // The resident kernels take the call when there is one chunk whose rows fit
  // and enough programs to repay the copies; both give the same bits (a wave
  // adds a program's cases in the same order).
  const bool resident = resident_call(a.n_total, a.n_chunks, a.M, a.rows);
  // the classes 1 and 2 of a prediction, whose outputs don't depend on the chunks
  EvalArgs d = a;
  const int64_t tiles = (a.M + TILE - 1) / TILE;
  const bool halves = a.n_total * tiles < HALF_TILE_DEEP_OUTPUTS;
  const bool cut = KIND == KIND_OUTPUTS && (resident ? a.n_total < RESIDENT_MIN_DEEP_OUTPUTS : halves);
  if (cut) {
    d.chunk = halves ? CHUNK_UNIT : TILE;
    d.n_chunks = int32_t((a.M + d.chunk - 1) / d.chunk);
  }
  if (resident) {
    e = wide ? launch_resident<KIND, 8, 0>(a, s, ev0, ev1) : launch_resident<KIND, 4, 0>(a, s, ev0, ev1);
    if (e != hipSuccess) return e;
    e = cut ? launch_class<KIND, 1, 0>(d, s) : launch_resident<KIND, 4, 1>(a, s);
    return e != hipSuccess ? e : launch_class<KIND, 2, 0>(d, s);
  }
  if (mixed_launch(a.n_total, a.n_chunks, a.chunk)) {
    const int grid = int((int64_t(a.n_total) * a.n_chunks + EVAL_WAVES - 1) / EVAL_WAVES);
    if (ev0 || ev1)
      hipExtLaunchKernelGGL(k_eval_mixed<KIND>, dim3(grid), dim3(256), 0, s, ev0, ev1, 0u, a);
    else
      hipLaunchKernelGGL(k_eval_mixed<KIND>, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  e = wide ? launch_class<KIND, 0, 0>(a, s, ev0, ev1) : launch_class<KIND, 0, 1>(a, s, ev0, ev1);
  if (e != hipSuccess) return e;
  e = launch_class<KIND, 1, 0>(d, s);
  if (e != hipSuccess) return e;
  return launch_class<KIND, 2, 0>(d, s);
}

hipError_t launch_eval(int kind, int kv, const EvalArgs& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                       bool counters_clear) {
  switch (kind) {
    case BEAGLE_FIT_MSE:
      return launch_kind<BEAGLE_FIT_MSE>(kv, a, s, ev0, ev1, counters_clear);
    case BEAGLE_FIT_CORR:
      return launch_kind<BEAGLE_FIT_CORR>(kv, a, s, ev0, ev1, counters_clear);
    case BEAGLE_FIT_POINT:
      return launch_kind<BEAGLE_FIT_POINT>(kv, a, s, ev0, ev1, counters_clear);
    case KIND_OUTPUTS:
      return launch_kind<KIND_OUTPUTS>(kv, a, s, ev0, ev1, counters_clear);
    default:
      return launch_kind<BEAGLE_FIT_R4>(kv, a, s, ev0, ev1, counters_clear);
  }
}

// Persistent grid of a work-list kernel (the occupancy queries all happen
// before a graph capture: prime_eval_batch).
template <int KIND, int CLS, int KV>
static int list_grid() {
  static int cached = 0;
  if (!cached) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_eval_batch<KIND, CLS, KV>, 256, 0) != hipSuccess || nb < 1)
      nb = 1;
    cached = nb * cu_count();
  }
  return cached;
}

template <int KIND, int CLS, int KV>
static hipError_t launch_list(const BatchArgs& b, int v, const int* has, hipStream_t s) {
  if (!has[v]) return hipSuccess;
  hipLaunchKernelGGL((k_eval_batch<KIND, CLS, KV>), dim3(list_grid<KIND, CLS, KV>()), dim3(256), 0, s, b, v);
  return hipGetLastError();
}

template <int KIND>
static void prime_kind() {
  (void)list_grid<KIND, 0, 0>();
  (void)list_grid<KIND, 0, 1>();
  (void)list_grid<KIND, 1, 0>();
  (void)list_grid<KIND, 2, 0>();
}

void prime_eval_batch(int kind) {
  if (kind == BEAGLE_FIT_MSE)
    prime_kind<BEAGLE_FIT_MSE>();
  else
    prime_kind<BEAGLE_FIT_CORR>();
}

template <int KIND>
static hipError_t launch_batch_kind(const BatchArgs& b, const int* has, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(256), 0, s, b.work, N_LISTS * counter_words(b.work_shift));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = launch_list<KIND, 0, 0>(b, 0, has, s)) != hipSuccess) return e;
  if ((e = launch_list<KIND, 0, 1>(b, 1, has, s)) != hipSuccess) return e;
  if ((e = launch_list<KIND, 1, 0>(b, 2, has, s)) != hipSuccess) return e;
  return launch_list<KIND, 2, 0>(b, 3, has, s);
}

hipError_t launch_eval_batch(int kind, const BatchArgs& b, const int* has_items, hipStream_t s) {
  return kind == BEAGLE_FIT_MSE ? launch_batch_kind<BEAGLE_FIT_MSE>(b, has_items, s)
                                : launch_batch_kind<BEAGLE_FIT_CORR>(b, has_items, s);
}

}  // namespace bgl
