// Generation step on the device: ramped half-and-half initialisation,
// tournament selection, subtree crossover and point mutation on postfix
// programs, driven by the Philox4x32-10 counter-based generator.
//
// Child c's random words come from Philox with key =
// seed and counter (c, generation, block, tag); word j of the child's stream
// is word j % 4 of block j / 4, so every draw has a fixed position whatever
// operator the child ends up using, and children are independent of the
// order in which threads run.
#include "beagle_device.h"
#include "gen.h"

namespace bgl {

// ---- Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) ---------------------
struct U4 {
  uint32_t v[4];
};

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                            uint32_t k1) {
  constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u;  // round multipliers
  constexpr uint32_t kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;  // key schedule (Weyl) increments
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += kW0;
      k1 += kW1;
    }
    const uint32_t hi0 = __umulhi(kM0, c0), lo0 = kM0 * c0;
    const uint32_t hi1 = __umulhi(kM1, c2), lo1 = kM1 * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  U4 o;
  o.v[0] = c0;
  o.v[1] = c1;
  o.v[2] = c2;
  o.v[3] = c3;
  return o;
}

// word j of the stream of (seed, index, gen, tag)
struct Stream {
  uint32_t k0, k1, index, gen, tag;
  int blk = -1;
  U4 words;
  __device__ Stream(uint64_t seed, uint32_t index_, uint32_t gen_, uint32_t tag_)
      : k0(uint32_t(seed)), k1(uint32_t(seed >> 32)), index(index_), gen(gen_), tag(tag_) {}
  __device__ uint32_t draw(int j) {
    const int b = j >> 2;
    if (b != blk) {
      words = philox4x32_10(index, gen, uint32_t(b), tag, k0, k1);
      blk = b;
    }
    // (selected, not indexed: an indexed array would be moved to LDS, 40 KB
    // of it per 64 threads, and cost the kernel its occupancy)
    const uint32_t lo = (j & 1) ? words.v[1] : words.v[0], hi = (j & 1) ? words.v[3] : words.v[2];
    return (j & 2) ? hi : lo;
  }
};

// integer in [0, n): multiply-high; unit float: 24 high bits
__device__ __forceinline__ uint32_t below(uint32_t u, uint32_t n) { return __umulhi(u, n); }
__device__ __forceinline__ double unit01(uint32_t u) { return double(u >> 8) * (1.0 / 16777216.0); }

// fp32(lo + (hi - lo) * unit), every step rounded in binary64 (no contraction)
__device__ __noinline__ float const_value(uint32_t u, float lo, float hi) {
#pragma clang fp contract(off)
  const double span = double(hi) - double(lo);
  const double prod = span * unit01(u);
  return float(double(lo) + prod);
}

// Zeroes elements [from, to) of a child slot with `lanes` threads (this one
// number l): element stores up to the first 16-byte boundary, then 16-byte
// stores, then the tail.
template <class T>
__device__ __forceinline__ void zero_fill(T* base, int from, int to, int l, int lanes) {
  constexpr int PER = 16 / int(sizeof(T));
  const int off = int((reinterpret_cast<uintptr_t>(base + from) & 15u) / sizeof(T));
  const int head = off == 0 ? from : from + (PER - off) < to ? from + (PER - off) : to;
  for (int i = from + l; i < head; i += lanes) base[i] = T(0);
  const int vecs = (to - head) / PER;
  for (int v = l; v < vecs; v += lanes) *reinterpret_cast<uint4*>(base + head + v * PER) = make_uint4(0u, 0u, 0u, 0u);
  for (int i = head + vecs * PER + l; i < to; i += lanes) base[i] = T(0);
}

// opcode of unary index u (0..4: SIN..SQRT, 5..11: SQUARE..TANH)
__device__ __forceinline__ uint32_t unary_opcode(uint32_t u) { return u < 5u ? OP_SIN + u : OP_SQUARE + (u - 5u); }

__device__ __forceinline__ bool better(double fa, int ia, double fb, int ib) {
  // lower fitness wins; NaN loses to everything; ties -> lower index
  const bool na = isnan(fa), nb = isnan(fb);
  if (na != nb) return nb;
  if (!na && fa != fb) return fa < fb;
  return ia < ib;
}

// The winner of entrants first_draw .. first_draw + t - 1; four draws and
// their fitness loads are made before the first comparison.
__device__ __forceinline__ int tournament(Stream& s, int first_draw, int t, const double* fit, uint32_t N) {
  int best = 0x7FFFFFFF;
  double fb = __longlong_as_double(0x7FF8000000000000LL);  // loses to every entrant
  for (int k = 0; k < t; k += 4) {
    int e[4];
    double f[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      // (a repeated last entrant changes nothing)
      e[u] = int(below(s.draw(first_draw + (k + u < t ? k + u : t - 1)), N));
      f[u] = fit[e[u]];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (better(f[u], e[u], fb, best)) {
        best = e[u];
        fb = f[u];
      }
    }
  }
  return best;
}

// Children in two phases.  First every lane (of the first `per_wave`) draws
// one child's random words and parents and reads the parents' headers; then
// the wave writes its children, GEN_GROUP lanes each, eight at a time: a
// group walks the child's token positions GEN_GROUP at a time, so that
// parents are read and children written in runs of lanes, and the constants
// are numbered by ballots.  Bound by the reads of random parents (a token
// slot, a constant row and two header entries, a memory line each) and the
// child writes.  One thread per child walked its tokens one by one, each
// lane in another line, behind 40 KB of LDS per wave: 572 us for 10^6
// children of slots of 64 tokens (microcosm selection), 128 us for 16 384 of
// 128 tokens (tournaments of four and crossover).
constexpr int GEN_GROUP = 8;
constexpr int GEN_GROUPS = 64 / GEN_GROUP;

// The start of the subtree that ends at position i of tok, found by every
// group for itself: GEN_GROUP positions a step backwards from i, the open
// operand count by prefix sums over the group's lanes (0 for a malformed
// parent; parents must be valid).  Groups with `on` false leave at once; every
// lane of the wave takes part.
__device__ __forceinline__ int subtree_start(const uint16_t* tok, int i, bool on, int gl, int gb) {
  int need = 1, start = 0;
  bool open = on;
  for (int j0 = i; __builtin_amdgcn_ballot_w64(open) != 0; j0 -= GEN_GROUP) {
    const int j = j0 - gl;
    int v = open && j >= 0 ? arity(tok[j] & 0xFFu) - 1 : 0;
#pragma unroll
    for (int d = 1; d < GEN_GROUP; d <<= 1) {
      const int w = __builtin_amdgcn_ds_bpermute((gb + (gl >= d ? gl - d : gl)) << 2, v);
      v += gl >= d ? w : 0;
    }
    const uint32_t closed = uint32_t(__builtin_amdgcn_ballot_w64(open && j >= 0 && need + v == 0) >> gb) &
                            ((1u << GEN_GROUP) - 1u);
    const int last = __builtin_amdgcn_ds_bpermute((gb + GEN_GROUP - 1) << 2, v);
    if (open && closed != 0) {
      start = j0 - (__ffs(closed) - 1);
      open = false;
    }
    need += last;
    if (j0 - GEN_GROUP < 0) open = false;
  }
  return start;
}

__global__ void __launch_bounds__(256) k_generation(GenStepArgs a) {
  const int lane = int(threadIdx.x & 63u);
  const int64_t c0 = (int64_t(blockIdx.x) * 4 + int64_t(threadIdx.x >> 6)) * a.per_wave;
  if (c0 >= a.n) return;
  const int here = int(a.n - c0 < a.per_wave ? a.n - c0 : a.per_wave);
  // ---- phase 1: lane j draws child c0 + j
  const int t = a.tournament;
  const uint32_t N = uint32_t(a.n_parents);
  int kind = 0;  // 0 empty, 1 copy of A, 2 mutant of A, 3 crossover
  int LA = 0, LB = 0, ca = 0, cb = 0, xa = 0, xb = 0, mpos = 0;
  int64_t oa = 0, ob = 0, coa = 0, cob = 0;
  uint32_t msym = 0, mconst = 0;
  if (lane < here) {
    Stream s(a.seed, uint32_t(c0 + lane), a.generation, a.tag);
    const double choice = unit01(s.draw(0));
    int ia, ib;
    if (a.surv) {
      const int S = *a.n_surv;
      const uint32_t ua = below(s.draw(1), uint32_t(S > 0 ? S : N));
      const uint32_t ub = below(s.draw(1 + t), uint32_t(S > 0 ? S : N));
      ia = S > 0 ? a.surv[ua] : int(ua);
      ib = S > 0 ? a.surv[ub] : int(ub);
    } else {
      ia = tournament(s, 1, t, a.fitness, N);
      ib = tournament(s, 1 + t, t, a.fitness, N);
    }
    const bool cross = choice < double(a.t_cross);
    // a parent outside its arrays, empty or longer than a child slot gives an
    // empty child (parents are meant to be valid programs)
    auto usable = [&](int64_t o, int L, int64_t co, int cc) {
      return L > 0 && L <= a.max_len && o >= 0 && o + L <= a.n_tokens && cc >= 0 &&
             (cc == 0 || (co >= 0 && co + cc <= a.n_consts));
    };
    // (a regular layout gives the offsets without reading them)
    const bool reg = a.slots && a.slots[0] != 0;
    oa = reg ? a.slots[1] + int64_t(ia) * a.slots[2] : a.tok_offset[ia];
    coa = reg ? a.slots[3] + int64_t(ia) * a.slots[4] : a.const_offset[ia];
    LA = a.tok_len[ia];
    ca = a.const_count[ia];
    bool okB = false;
    if (cross) {  // (only crossover reads parent B)
      ob = reg ? a.slots[1] + int64_t(ib) * a.slots[2] : a.tok_offset[ib];
      cob = reg ? a.slots[3] + int64_t(ib) * a.slots[4] : a.const_offset[ib];
      LB = a.tok_len[ib];
      cb = a.const_count[ib];
      okB = usable(ob, LB, cob, cb);
    }
    const bool okA = usable(oa, LA, coa, ca);
    kind = !okA || (cross && !okB) ? 0 : cross ? 3 : choice < double(a.t_mut) ? 2 : 1;
    xa = int(below(s.draw(2 * t + 1), uint32_t(okA ? LA : 0)));
    xb = int(below(s.draw(2 * t + 2), uint32_t(okB ? LB : 0)));
    mpos = int(below(s.draw(2 * t + 3), uint32_t(okA ? LA : 0)));
    msym = s.draw(2 * t + 4);
    mconst = s.draw(2 * t + 5);
    if (kind == 0) LA = LB = ca = cb = 0, oa = ob = coa = cob = 0;
  }
  // ---- phase 2: the wave's groups write the children
  const int gl = lane & (GEN_GROUP - 1), gb = lane & ~(GEN_GROUP - 1);
  auto of = [](int v, int src) { return __builtin_amdgcn_ds_bpermute(src << 2, v); };
  auto of64 = [&](int64_t v, int src) {
    const uint32_t lo = uint32_t(of(int(uint32_t(uint64_t(v))), src));
    const uint32_t hi = uint32_t(of(int(uint32_t(uint64_t(v) >> 32)), src));
    return int64_t((uint64_t(hi) << 32) | lo);
  };
  for (int j0 = 0; j0 < here; j0 += GEN_GROUPS) {
    const int j = j0 + (lane / GEN_GROUP);
    const bool live = j < here;
    const int sj = live ? j : 0;
    // (every lane takes part in the reads across lanes)
    int k = of(kind, sj);
    if (!live) k = 0;
    const int la = of(LA, sj), pa = of(ca, sj), pb = of(cb, sj), ma = of(mpos, sj);
    const int ya = of(xa, sj), yb = of(xb, sj);
    const uint16_t* A = a.tokens + of64(oa, sj);
    const uint16_t* B = a.tokens + of64(ob, sj);
    const float* Ac = a.consts + of64(coa, sj);
    const float* Bc = a.consts + of64(cob, sj);
    const uint32_t ms = uint32_t(of(int(msym), sj)), mc = uint32_t(of(int(mconst), sj));
    // crossover: A[0, sa) B[sb, yb] A[ya + 1, la)
    int sa = 0x7FFFFFFF, nb = 0, sb = 0, len = k == 0 ? 0 : la;
    if (__builtin_amdgcn_ballot_w64(k == 3) != 0) {
      const int s0 = subtree_start(A, ya, k == 3, gl, gb);
      const int s1 = subtree_start(B, yb, k == 3, gl, gb);
      const int l = la - (ya - s0 + 1) + (yb - s1 + 1);
      if (k == 3 && l <= a.max_len) {  // (a longer child: a copy of A)
        sa = s0;
        sb = s1;
        nb = yb - s1 + 1;
        len = l;
      }
    }
    // mutation: the new symbol of position ma
    uint32_t repl = 0;
    float rval = 0.0f;
    bool need_count = false;
    if (k == 2) {
      const uint32_t old = A[ma] & 0xFFu;
      const int ar = arity(old);
      if (ar == 2) {
        repl = below(ms, 4);  // ADD, SUB, MUL, DIV
      } else if (ar == 1) {
        repl = unary_opcode(below(ms, uint32_t(a.n_unary)));
      } else {
        const uint32_t sym = below(ms, uint32_t(a.D + 1));
        need_count = int(sym) >= a.D;
        repl = need_count ? uint32_t(OP_CONST) : OP_VAR | (sym << 8);
      }
    }
    if (__builtin_amdgcn_ballot_w64(need_count) != 0) {
      // a new constant only if the parent's others leave it a slot
      int others = 0;
      for (int i0 = 0; __builtin_amdgcn_ballot_w64(need_count && i0 < la) != 0; i0 += GEN_GROUP) {
        const int i = i0 + gl;
        const bool cst = need_count && i < la && i != ma && (A[i] & 0xFFu) == OP_CONST;
        others += __popc(uint32_t(__builtin_amdgcn_ballot_w64(cst) >> gb) & ((1u << GEN_GROUP) - 1u));
      }
      if (need_count) {
        if (others < a.max_consts)
          rval = const_value(mc, a.const_lo, a.const_hi);
        else
          repl = OP_VAR;
      }
    }
    const int64_t c = c0 + j;
    uint16_t* out = a.child_tokens + (live ? c : 0) * a.max_len;
    float* outc = a.child_consts + (live ? c : 0) * a.max_consts;
    int ncst = 0;
    for (int i0 = 0; __builtin_amdgcn_ballot_w64(i0 < len) != 0; i0 += GEN_GROUP) {
      const int i = i0 + gl;
      const bool on = i < len;
      const bool inb = i >= sa && i < sa + nb;
      uint32_t tk = 0;
      if (on) tk = inb ? B[sb + i - sa] : A[i < sa ? i : ya + 1 + (i - sa - nb)];
      const bool mut = k == 2 && i == ma;
      if (mut) tk = repl;
      const bool cst = on && (tk & 0xFFu) == OP_CONST;
      const uint32_t m = uint32_t(__builtin_amdgcn_ballot_w64(cst) >> gb) & ((1u << GEN_GROUP) - 1u);
      if (cst) {
        const int slot = ncst + __popc(m & ((1u << gl) - 1u));
        const int arg = int(tk >> 8);
        float v = rval;
        if (!mut) v = arg < (inb ? pb : pa) ? (inb ? Bc : Ac)[arg] : 0.0f;
        if (slot < a.max_consts) {
          tk = OP_CONST | (uint32_t(slot) << 8);
          outc[slot] = v;
        } else {
          tk = OP_VAR;
        }
      }
      if (on) out[i] = uint16_t(tk);
      ncst += __popc(m);
    }
    ncst = ncst < a.max_consts ? ncst : a.max_consts;
    if (live) {
      zero_fill(out, len, a.max_len, gl, GEN_GROUP);
      zero_fill(outc, ncst, a.max_consts, gl, GEN_GROUP);
      if (gl == 0) {
        a.child_len[c] = len;
        a.child_const_count[c] = ncst;
      }
    }
  }
}

// Children per wave: 32 (64 left the second phase's last waves alone: 6 % longer
// for 10^6 children, 250 us), fewer (not below the GEN_GROUPS that the second
// phase writes at a time) where that would leave under 8192 waves, eight per
// SIMD: the phases are chains of dependent reads, which only other waves hide.
void launch_generation(GenStepArgs a, hipStream_t s) {
  int per = 32;
  while (per > GEN_GROUPS && int64_t(a.n) < int64_t(8192) * per) per >>= 1;
  a.per_wave = per;
  const int64_t waves = (int64_t(a.n) + per - 1) / per;
  hipLaunchKernelGGL(k_generation, dim3(uint32_t((waves + 3) / 4)), dim3(256), 0, s, a);
}

// ---- microcosm selection ----------------------------------------------------
// A random sample of the population, ranked in one workgroup, gives the
// fitness threshold at the keep quantile; every individual at least that
// good survives, compacted in index order (per-block counts, one scan, a
// scatter), and the children draw their parents uniformly from the
// survivors.  Sort order of the sample: lower fitness first, NaN last, ties
// by draw position; survival: fitness not NaN and <= tau (every non-NaN
// individual when tau is NaN).

__device__ __forceinline__ bool survives(double f, double tau) { return !isnan(f) && (isnan(tau) || f <= tau); }

// blockDim.x == MICRO_MAX_SAMPLE, one workgroup
__global__ void __launch_bounds__(MICRO_MAX_SAMPLE) k_micro_threshold(MicroArgs a) {
  __shared__ double f[MICRO_MAX_SAMPLE];
  const int j = threadIdx.x;
  if (j == 0 && a.slots) {
    // the layout of parents 0 and 1, tested on every parent by k_micro_count
    const int64_t t0 = a.tok_offset[0], c0 = a.const_offset[0];
    a.slots[0] = 1;
    a.slots[1] = t0;
    a.slots[2] = a.n > 1 ? a.tok_offset[1] - t0 : 0;
    a.slots[3] = c0;
    a.slots[4] = a.n > 1 ? a.const_offset[1] - c0 : 0;
  }
  if (j < a.sample) {
    Stream s(a.seed, MICRO_INDEX, a.generation, a.tag);
    f[j] = a.fitness[below(s.draw(j), uint32_t(a.n))];
  }
  __syncthreads();
  if (j >= a.sample) return;
  const double fj = f[j];
  const bool nj = isnan(fj);
  int rank = 0;
  for (int i = 0; i < a.sample; ++i) {
    const double fi = f[i];
    const bool ni = isnan(fi);
    const bool less = ni != nj ? nj : (!ni && fi != fj ? fi < fj : i < j);
    rank += less ? 1 : 0;
  }
  if (rank == a.k) *a.tau = fj;  // ranks are a permutation: exactly one writer
}

// survivors of block b (MICRO_BLOCK consecutive individuals), MICRO_BLOCK threads
__global__ void __launch_bounds__(MICRO_BLOCK) k_micro_count(MicroArgs a) {
  __shared__ int wave_n[MICRO_BLOCK / 64];
  const int64_t i = int64_t(blockIdx.x) * MICRO_BLOCK + threadIdx.x;
  const double tau = *a.tau;
  const bool keep = i < a.n && survives(a.fitness[i], tau);
  if (a.slots && i < a.n &&
      (a.tok_offset[i] != a.slots[1] + i * a.slots[2] || a.const_offset[i] != a.slots[3] + i * a.slots[4]))
    a.slots[0] = 0;  // (every writer stores the same value)
  const int n = __popcll(__builtin_amdgcn_ballot_w64(keep));
  if ((threadIdx.x & 63) == 0) wave_n[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < MICRO_BLOCK / 64; ++w) t += wave_n[w];
    a.block_off[blockIdx.x] = t;
  }
}

// exclusive prefix sums of the block counts in place, and the total; one
// workgroup of 1024 threads walking the counts 1024 at a time
__global__ void __launch_bounds__(1024) k_micro_scan(MicroArgs a) {
  __shared__ int wave_tot[16];
  __shared__ int carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int base = 0; base < a.n_blocks; base += 1024) {
    const int b = base + int(threadIdx.x);
    const int v = b < a.n_blocks ? a.block_off[b] : 0;
    // inclusive scan inside the wave
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wave_tot[w] = x;
    __syncthreads();
    const int carry = carry_s;
    int before = 0;
    for (int q = 0; q < w; ++q) before += wave_tot[q];
    if (b < a.n_blocks) a.block_off[b] = carry + before + x - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry_s = carry + before + x;
    __syncthreads();
  }
  if (threadIdx.x == 0) *a.n_surv = carry_s;
}

__global__ void __launch_bounds__(MICRO_BLOCK) k_micro_scatter(MicroArgs a) {
  __shared__ int wave_n[MICRO_BLOCK / 64];
  const int64_t i = int64_t(blockIdx.x) * MICRO_BLOCK + threadIdx.x;
  const double tau = *a.tau;
  const bool keep = i < a.n && survives(a.fitness[i], tau);
  if (a.slots && i < a.n &&
      (a.tok_offset[i] != a.slots[1] + i * a.slots[2] || a.const_offset[i] != a.slots[3] + i * a.slots[4]))
    a.slots[0] = 0;  // (every writer stores the same value)
  const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
  if ((threadIdx.x & 63) == 0) wave_n[threadIdx.x >> 6] = __popcll(m);
  __syncthreads();
  int at = a.block_off[blockIdx.x];
  for (int w = 0; w < int(threadIdx.x >> 6); ++w) at += wave_n[w];
  at += __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
  if (keep) a.surv[at] = int32_t(i);
}

__global__ void k_init_population(InitArgs a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= a.n) return;
  const int n_depths = a.depth_max - a.depth_min + 1;
  const int depth = a.depth_min + c % n_depths;
  const bool full = ((c / n_depths) % 2) == 0;
  Stream s(a.seed, uint32_t(c), 0u, a.tag);
  int cursor = 0;
  uint16_t* out = a.tokens + int64_t(c) * a.max_len;
  float* outc = a.consts + int64_t(c) * a.max_consts;
  int len = 0, ncst = 0;
  // pre-order generation, post-order emission: frames of open functions
  struct Frame {
    uint8_t op, left, level;
  };
  Frame fr[MAX_INIT_DEPTH + 1];
  int sp = 0;
  int level = 0;
  const uint32_t n_fun = 4u + uint32_t(a.n_unary);
  for (;;) {
    bool term;
    uint32_t sym;
    if (level == depth) {
      term = true;
      sym = below(s.draw(cursor++), uint32_t(a.D + 1));
    } else if (full) {
      term = false;
      sym = below(s.draw(cursor++), n_fun);
    } else {
      const uint32_t v = below(s.draw(cursor++), n_fun + uint32_t(a.D + 1));
      term = v >= n_fun;
      sym = term ? v - n_fun : v;
    }
    if (!term) {
      // functions in the order ADD SUB MUL DIV, then the unary ones
      fr[sp].op = uint8_t(sym < 4u ? sym : unary_opcode(sym - 4u));
      fr[sp].left = uint8_t(arity(fr[sp].op));
      fr[sp].level = uint8_t(level);
      ++sp;
      ++level;
      continue;
    }
    if (int(sym) < a.D) {
      out[len++] = uint16_t(OP_VAR | (sym << 8));
    } else if (ncst < a.max_consts) {
      out[len++] = uint16_t(OP_CONST | (uint32_t(ncst) << 8));
      outc[ncst++] = const_value(s.draw(cursor++), a.const_lo, a.const_hi);
    } else {
      out[len++] = uint16_t(OP_VAR);
    }
    while (sp > 0) {
      Frame& f = fr[sp - 1];
      if (--f.left > 0) break;
      out[len++] = uint16_t(f.op);
      --sp;
    }
    if (sp == 0) break;
    level = fr[sp - 1].level + 1;
  }
  zero_fill(out, len, a.max_len, 0, 1);
  zero_fill(outc, ncst, a.max_consts, 0, 1);
  a.len[c] = len;
  a.const_count[c] = ncst;
}

}  // namespace bgl
