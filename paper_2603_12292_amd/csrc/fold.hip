// Folding of constant subtrees, before decoding.
//
// A subtree whose leaves are all constants has one value for every case (and
// the partial derivative of that value by each of its constants is one number
// too), but the interpreter and the adjoint sweeps would recompute it for
// each.  This pass rewrites every valid program of at most 64 tokens with
// each maximal constant subtree as one CONST token, its value computed by the
// interpreter's own functions (so the outputs keep their bits), into the
// workspace; the decoders read the rewritten programs.  For the adjoint it
// also lists, per CONST token of the original program, its slot, the slot of
// the constant it was folded into and the derivative of that constant's value:
// the gradient of a slot is the sum of (gradient of the folded constant) x
// (derivative), taken once after the cases are summed.  For that
// an operator is folded only if every product of derivatives from it down to
// a constant is at most 1 in magnitude: an adjoint that reaches the constant
// as a binary32 product then overflows nowhere on its way, and the gradient is
// infinite or NaN exactly where the sum over the cases is.
//
// One wave per program, a token per lane.  In postfix order the operands of an
// operator whose operands are single CONST tokens stand directly before it, so
// a round folds every "CONST, unary" and "CONST, CONST, binary" at once and
// closes the gaps; a constant subtree of height h takes h rounds.  Programs
// that are not valid, longer, or whose folded constants would need more slots
// than they have, keep their tokens.  The pass also does the ownership
// check of overlapping ranges on the original arrays (the rewritten ranges are
// shorter) and hands its verdict on as a negative length.
#include "beagle_device.h"
#include "deriv.h"
#include "kernels.h"
#include "layout.h"

namespace bgl {

namespace {

__device__ __forceinline__ int lane_read(int v, int src) { return __builtin_amdgcn_ds_bpermute(src << 2, v); }
__device__ __forceinline__ float lane_readf(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src << 2, __float_as_int(v)));
}
// v of the lane before (0 in lane 0)
__device__ __forceinline__ float lane_before(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, true);
}
__device__ __forceinline__ int prefix_sum(int v) {
  v = dpp_add<0x111, 0xF>(v);
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);
  v = dpp_add<0x143, 0xC>(v);
  return v;
}
// token flag: an operator that is not folded
constexpr uint32_t KEPT = 0x80000000u;

__device__ __forceinline__ int rank_in(uint64_t m) {
  return int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)));
}

// value and partial derivatives of binary operator O where mask m has the lane
template <uint32_t O, bool ADJ>
__device__ __forceinline__ void fold_binary(uint64_t m, float a, float b, float& v, float& da, float& db) {
  if (m == 0) return;
  const bool on = __builtin_amdgcn_inverse_ballot_w64(m);
  const float r = gbinop<O>(a, b);
  v = on ? r : v;
  if constexpr (ADJ) {
    float pa, pb;
    dbinop<O>(a, b, pa, pb);
    da = on ? pa : da;
    db = on ? pb : db;
  }
}

template <uint32_t U, bool ADJ>
__device__ __forceinline__ void fold_unary(uint64_t m, float x, float& v, float& db) {
  if (m == 0) return;
  const bool on = __builtin_amdgcn_inverse_ballot_w64(m);
  float r;
  if constexpr (U == 0) r = trig1<false>(x);
  else if constexpr (U == 1) r = trig1<true>(x);
  else if constexpr (U == 2) r = op_exp(x);
  else if constexpr (U == 3) r = op_log(x);
  else if constexpr (U == 4) r = op_sqrt(x);
  else r = op_ext<U>(x);
  v = on ? r : v;
  if constexpr (ADJ) {
    const float p = dunary(U, x, r);
    db = on ? p : db;
  }
}

}  // namespace

template <bool ADJ>
__global__ void __launch_bounds__(256) k_fold(FoldArgs f) {
  __shared__ uint32_t lds_t[4][64];
  __shared__ float lds_v[4][64];
  __shared__ unsigned long long lds_keep[4];
  const PrepareArgs& a = f.in;
  const int lane = int(threadIdx.x & 63u), w = int(threadIdx.x >> 6);
  const int p = __builtin_amdgcn_readfirstlane(f.first + int(blockIdx.x) * 4 + w);
  if (p >= a.n_programs) return;  // (no barrier below)
  uint32_t* st = lds_t[w];
  float* sv = lds_v[w];
  const int64_t off = a.tok_offset[p], coff = a.const_offset[p];
  const int32_t L0 = a.tok_len[p], cc = a.const_count[p];
  int32_t L = L0;
  const bool range = L0 >= 0 && off >= 0 && off + L0 <= a.n_tokens && cc >= 0 &&
                     (cc == 0 || (coff >= 0 && coff + cc <= a.n_consts));
  int32_t out_len = L0, out_cc = cc;
  int64_t out_coff = coff;
  int n_map = 0;
  if (L0 > MAX_LEN) {
    // (kept as it is: too long)
  } else if (!range) {
    out_len = L0 == 0 ? 0 : -1;
  } else {
    // ownership of the ranges where they are not sorted and disjoint
    bool mine = true;
    if (!a.owner) {
      if (a.layout[0] | a.layout[1]) mine = wave_alone(a, p, off, L0, coff, cc);
    } else if (a.layout[0])
      for (int32_t j0 = 0; j0 < L0 && mine; j0 += 64)
        mine = __builtin_amdgcn_ballot_w64(j0 + lane < L0 && a.owner[off + j0 + lane] != p) == 0;
    if (ADJ && a.owner && mine && a.layout[1])
      for (int32_t j0 = 0; j0 < cc && mine; j0 += 64)
        mine = __builtin_amdgcn_ballot_w64(j0 + lane < cc && a.cowner[coff + j0 + lane] != p) == 0;
    if (!mine && L0 > 0) out_len = -1;
    if (mine && L0 > 64)
      for (int32_t j = lane; j < L0; j += 64) f.tokens[off + j] = a.tokens[off + j];
    if (mine && L0 >= 1 && L0 <= 64) {
      bool act = lane < L;
      uint64_t actm = L >= 64 ? ~0ull : (1ull << L) - 1ull;
      uint32_t t = act ? uint32_t(a.tokens[off + lane]) : 0xFFu;
      const uint32_t t0 = t;
      uint32_t op = t & 0xFFu;
      const uint32_t arg = t >> 8;
      // a valid program: every opcode, variable and slot in range, no
      // underflow, one value left
      constexpr uint64_t ARITY = 0x5554155AAull;  // 2 bits per opcode, as in the decoders
      const int ar = op < N_OPCODES ? int((ARITY >> (2u * op)) & 3u) : 0;
      const int d = prefix_sum(act ? 1 - ar : 0);
      const bool bad = act && (op >= uint32_t(N_OPCODES) || (op == OP_VAR && int(arg) >= a.D) ||
                               (op == OP_CONST && int(arg) >= cc) || d < 1);
      const bool valid = (__builtin_amdgcn_ballot_w64(bad) == 0) && __builtin_amdgcn_readlane(d, L - 1) == 1;
      const uint64_t cm0 = __builtin_amdgcn_ballot_w64(act && op == OP_CONST);
      if (valid && cm0 != 0) {
        float v = 0.0f;
        if (act && op == OP_CONST) v = a.consts[coff + arg];
        // lane i holds a CONST token of the original program: its constant is
        // now the token at `root`, whose value has derivative `der` by it
        int root = lane;
        double der = 1.0;
        double way = 0.0;  // the largest |product| of derivatives from the root down
        for (;;) {
          const uint64_t cm = __builtin_amdgcn_ballot_w64(op == OP_CONST);
          auto has = [&](uint32_t o) { return __builtin_amdgcn_ballot_w64(op == o); };
          const uint64_t one = (cm << 1) & actm, two = one & (cm << 2);
          const uint64_t open = ADJ ? __builtin_amdgcn_ballot_w64((t & KEPT) == 0u) : ~0ull;
          uint64_t bm = __builtin_amdgcn_ballot_w64(op < 4u) & two & open;
          uint64_t um =
              __builtin_amdgcn_ballot_w64(op - uint32_t(OP_SIN) < 5u || op - uint32_t(OP_SQUARE) < 7u) & one & open;
          uint64_t fm = bm | um;
          if (fm == 0) break;
          const float y = lane_before(v), x = lane_before(y);  // the top operand, the one below
          float r = v, da = 0.0f, db = 0.0f;
          if (bm) {
            fold_binary<B_ADD, ADJ>(has(OP_ADD) & bm, x, y, r, da, db);
            fold_binary<B_SUB, ADJ>(has(OP_SUB) & bm, x, y, r, da, db);
            fold_binary<B_MUL, ADJ>(has(OP_MUL) & bm, x, y, r, da, db);
            fold_binary<B_DIV, ADJ>(has(OP_DIV) & bm, x, y, r, da, db);
          }
          if (um) {
            fold_unary<0, ADJ>(has(OP_SIN) & um, y, r, db);
            fold_unary<1, ADJ>(has(OP_COS) & um, y, r, db);
            fold_unary<2, ADJ>(has(OP_EXP) & um, y, r, db);
            fold_unary<3, ADJ>(has(OP_LOG) & um, y, r, db);
            fold_unary<4, ADJ>(has(OP_SQRT) & um, y, r, db);
            if (um & __builtin_amdgcn_ballot_w64(op > uint32_t(OP_CONST))) {
              fold_unary<5, ADJ>(has(OP_SQUARE) & um, y, r, db);
              fold_unary<6, ADJ>(has(OP_RECIP) & um, y, r, db);
              fold_unary<7, ADJ>(has(OP_TAN) & um, y, r, db);
              fold_unary<8, ADJ>(has(OP_ASIN) & um, y, r, db);
              fold_unary<9, ADJ>(has(OP_ACOS) & um, y, r, db);
              fold_unary<10, ADJ>(has(OP_ATAN) & um, y, r, db);
              fold_unary<11, ADJ>(has(OP_TANH) & um, y, r, db);
            }
          }
          if constexpr (ADJ) {
            // operators with a product of derivatives above 1 (or a NaN) stay
            const bool in_top = ((fm >> 1) >> root) & 1u, in_below = ((bm >> 2) >> root) & 1u;
            const int parent = root + (in_top ? 1 : in_below ? 2 : 0);
            const float mt = lane_readf(db, parent & 63), mb = lane_readf(da, parent & 63);
            const double m = fabs(double(in_top ? mt : mb));
            const bool on = __builtin_amdgcn_inverse_ballot_w64(cm0) && (in_top || in_below);
            const bool large = on && !(m <= 1.0 && m * way <= 1.0);
            if (__builtin_amdgcn_ballot_w64(large) != 0) {
              if (lane == 0) lds_keep[w] = 0ull;
              __builtin_amdgcn_wave_barrier();
              if (large) __hip_atomic_fetch_or(&lds_keep[w], 1ull << parent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
              __builtin_amdgcn_wave_barrier();
              const uint64_t keep = lds_keep[w];
              const uint64_t km = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(keep >> 32)))) << 32) |
                                  uint32_t(__builtin_amdgcn_readfirstlane(int(keep)));
              __builtin_amdgcn_wave_barrier();
              t = __builtin_amdgcn_inverse_ballot_w64(km) ? t | KEPT : t;
              bm &= ~km;
              um &= ~km;
              fm &= ~km;
              if (fm == 0) continue;
            }
          }
          const bool folded = __builtin_amdgcn_inverse_ballot_w64(fm);
          t = folded ? uint32_t(OP_CONST) : t;
          v = folded ? r : v;
          const uint64_t top = fm >> 1, below = bm >> 2;  // consumed operands
          const uint64_t alive = actm & ~(top | below);
          const int pos = rank_in(alive);
          if constexpr (ADJ) {
            // follow the constants into the operator that consumed them
            const bool in_top = (top >> root) & 1u, in_below = (below >> root) & 1u;
            const int parent = root + (in_top ? 1 : in_below ? 2 : 0);
            const float mt = lane_readf(db, parent & 63), mb = lane_readf(da, parent & 63);
            if (in_top || in_below) {
              const double m = in_top ? mt : mb;
              der *= m;
              way = fabs(m) > fabs(m) * way ? fabs(m) : fabs(m) * way;
            }
            root = lane_read(pos, parent & 63);
          }
          if (__builtin_amdgcn_inverse_ballot_w64(alive)) {
            st[pos] = t;
            sv[pos] = v;
          }
          __builtin_amdgcn_wave_barrier();
          L = __popcll(alive);
          actm = (1ull << L) - 1ull;  // (a round removes at least one token)
          act = lane < L;
          t = act ? st[lane] : 0xFFu;
          v = act ? sv[lane] : 0.0f;
          __builtin_amdgcn_wave_barrier();
          op = t & 0xFFu;
        }
        const uint64_t cm = __builtin_amdgcn_ballot_w64(op == OP_CONST);
        const int n = __popcll(cm), slot = rank_in(cm);
        // (the adjoint's partial gradients have the constants' layout: no
        // more folded constants than slots)
        if (!ADJ || n <= cc) {
          if (op == OP_CONST) {
            t = uint32_t(OP_CONST) | (uint32_t(slot) << 8);
            f.consts[a.n_consts + off + slot] = v;
          }
          if (act) f.tokens[off + lane] = uint16_t(t);
          if constexpr (ADJ) {
            const int s = lane_read(slot, root & 63);
            const int e = rank_in(cm0);
            if (__builtin_amdgcn_inverse_ballot_w64(cm0)) {
              f.map_slots[off + e] = uint16_t((t0 >> 8) | (uint32_t(s) << 8));
              f.map_der[off + e] = der;
            }
            n_map = __popcll(cm0);
          }
          out_len = L;
          out_cc = n;
          out_coff = a.n_consts + off;
        } else if (lane < L0) {
          f.tokens[off + lane] = uint16_t(t0);
        }
      } else if (act) {
        f.tokens[off + lane] = uint16_t(t0);
      }
    }
  }
  // a program kept as it is reads its constants where they were: those that its
  // tokens can name, a byte's worth (4096 programs that share a table of 20 000
  // constants x 20 000 cases: 526 us with all of it copied for each)
  if (out_coff == coff && out_len > 0 && out_len <= MAX_LEN)
    for (int32_t j = lane; j < min(cc, 256); j += 64) f.consts[coff + j] = a.consts[coff + j];
  if (lane == 0) {
    f.tok_len[p] = out_len;
    f.const_offset[p] = out_coff;
    f.const_count[p] = out_cc;
    if (ADJ) f.map_n[p] = n_map;
  }
}

void launch_fold(const FoldArgs& f, hipStream_t s) {
  // (a grid has fewer than 2^32 threads, and a program takes 64)
  constexpr int32_t LAUNCH = 1 << 24;
  FoldArgs g = f;
  for (int64_t first = 0; first < f.in.n_programs; first += LAUNCH) {
    g.first = int32_t(first);
    const uint32_t grid = uint32_t((std::min<int64_t>(f.in.n_programs - first, LAUNCH) + 3) / 4);
    if (f.in.adjoint)
      hipLaunchKernelGGL(k_fold<true>, dim3(grid), dim3(256), 0, s, g);
    else
      hipLaunchKernelGGL(k_fold<false>, dim3(grid), dim3(256), 0, s, g);
  }
}

}  // namespace bgl
