// Beam step (gfx950, wave64): the K best of an utterance's K * V totals, in order, with the state gather by parent
// (Alg. 1 Stage 3: hyps_expansion_score, prune_expanded, S[t]).
//
// One workgroup per utterance.  Neither the rows nor the survivors are sorted:
//
//  * The beams' rows are spread over up to 16 waves.  Every lane forms the totals of its tokens (base boosts in
//    registers; tokens that an arc of the failure chain overrides are marked in LDS by the first wave of the beam,
//    which evaluates the arcs one per lane) and keeps their maximum.
//  * Bound.  The maxima of the lanes meet in 64 slots; the K-th largest of these, which is no larger than the K-th best
//    total, is bounded from below (joint_bound).
//  * Totals that reach the bound -- K and a few more -- go to a list in LDS, and their ranks come from counting: a
//    thread per entry compares it with all others by (total descending, k * V + v ascending).
//  * A list that overflows (rows that are flat, or tie: more totals reach the bound than it holds) is itself a sample of
//    the totals: the K-th best of its entries, by the same order, is a higher bound, and the totals are collected again
//    until they fit (raised_bound).
//  * An utterance of dead beams (hypothesis scores of -inf: a finished one in a batch, mostly) has only totals of -inf, so
//    its survivors are the first K flat indices; the rows are not looked at (put_dead).
//
// U x K, V: 32 x 4, 1024 7.0 -> 5.9 us (graph replay) against a kernel with a wave per beam and K rounds of arg-max in
// each; against the workgroup-per-utterance row build (launch_beam) 16 x 8, 1025, a table of trees 35.9 -> 8.2, 32 x 8,
// 8192 81.9 -> 17.0, 16 x 16, 50000 1130 -> 93.  With one dead utterance among 32 a step takes what it takes without
// (32 x 8, 8192: 17 us; K rounds of arg-max over its rows took 182), with constant rows everywhere about twice that (38;
// rounds 187).
//
// A few beams over aligned narrow rows keep the wave-per-beam kernel (see wave_beams).
//
// Rows whose share of a wave fits its registers are read once (beam_regs_kernel); longer ones are streamed, with the
// maximum of every chunk kept, and only the chunks that reach the bound are read again (beam_stream_kernel).
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "pb_chunk.hpp"
#include "pb_kernels.hpp"
#include "pb_wave.hpp"

namespace pb {

namespace {

using namespace wv;

constexpr int kBeamMax = 32;     // beams of an utterance at most
constexpr int kBeamWaves = 16;   // waves of a workgroup at most
constexpr unsigned kKeyNegInf = 0x007fffffu;  // ukey(-inf)

struct BeamOut {
  int32_t *tokens, *parents, *states;
  float* scores;
  __device__ __forceinline__ void put(int slot, int tok, int parent, int state, float score) const {
    tokens[slot] = tok;
    parents[slot] = parent;
    states[slot] = state;
    scores[slot] = score;
  }
};

// (total, flat index) as one number that is larger for the better candidate.
__device__ __forceinline__ u64 cand_key(float total, int flat) {
  return (static_cast<u64>(ukey(__fadd_rn(total, 0.0f))) << 32) | static_cast<unsigned>(~flat);  // (-0 ties with +0)
}

struct Small {  // the fixed part of the workgroup's LDS
  unsigned lane_best[64];
  int child[kBeamMax];  // put_dead: the arcs of a beam's first tokens
  int count;
};
struct Shared {  // the list of survivors (the first part of the dynamic LDS) and the fixed part
  u64* key;
  int4* entry;  // bits of the total, token, beam, next state of an arc's candidate (-1 for a base candidate)
  int cap;
  Small* s;
};
// Entries of the list: 64 per wave of the workgroup, at least 128 (a multiple of what reaches the bound).  The list is
// part of what limits the utterances a CU holds at once: with room for 1024 entries in every workgroup 8192 utterances
// of one beam (V = 1024) took 20.5 us instead of 14.
__host__ __device__ constexpr int list_cap(int waves) { return waves <= 2 ? 128 : 64 * waves; }
__host__ __device__ constexpr size_t list_bytes(int waves) { return static_cast<size_t>(list_cap(waves)) * 24; }
__device__ __forceinline__ Shared shared_at(char* lds, Small* s, int nwaves) {
  const int cap = list_cap(nwaves);
  int4* entry = reinterpret_cast<int4*>(lds);
  return Shared{reinterpret_cast<u64*>(entry + cap), entry, cap, s};
}

// Adds a candidate to the list (called by the lanes that have one).
__device__ __forceinline__ void push(const Shared& sh, float total, int k, int v, int V, int child) {
  const int i = atomicAdd(&sh.s->count, 1);
  if (i < sh.cap) {
    sh.key[i] = cand_key(total, k * V + v);
    sh.entry[i] = make_int4(__float_as_int(total), v, k, child);
  }
}

__device__ __forceinline__ bool overflowed(const Shared& sh) {
  return __hip_atomic_load(&sh.s->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > sh.cap;
}
// Of a list of n >= 64 entries (a barrier lies behind the last push): a key that at least K of them reach and that is
// higher than most of them: the K-th largest of the maxima of 64 disjoint parts of the list.
__device__ __forceinline__ u64 raised_bound(const Shared& sh, int lane, int n, int K) {
  u64 best = 0;
  for (int i = lane; i < n; i += 64) best = sh.key[i] > best ? sh.key[i] : best;
  int rank = 0;  // (the keys are all different)
#pragma unroll 8
  for (int l = 0; l < 64; ++l) {
    const u64 o = (static_cast<u64>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(best >> 32), l))) << 32) |
                  static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(best), l));
    rank += o > best ? 1 : 0;
  }
  const int from = first_lane(__ballot(rank == K - 1));
  return (static_cast<u64>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(best >> 32), from))) << 32) |
         static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(best), from));
}
__device__ __forceinline__ float key_total(u64 key) { return ukey_val(static_cast<unsigned>(key >> 32)); }

// The bound.  The lanes' maxima are collected in 64 slots (as keys, zero before the barrier that precedes post_lane; the
// lanes of a wave are rotated against those of the others, so that rows too short for all lanes still fill the slots).
// Every slot that is not empty holds the total of a candidate of its own, so the K-th largest slot is no larger than the
// K-th best total.  It is approached from below: the smallest of a few distances from the best slot within which at
// least K slots lie, counted side by side, first in powers of two, then in eighths.  A binary search over the keys, the
// other way, is a chain of ballots (16 of them took 1700 cycles of the 13000 of a step); it is left for slots that lie
// further apart.
__device__ __forceinline__ void post_lane(const Shared& sh, int lane, int wave, int nwaves, float m) {
  atomicMax(&sh.s->lane_best[(lane + wave * (64 / nwaves)) & 63], ukey(m));
}
__device__ __forceinline__ float joint_bound(const Shared& sh, int lane, int K) {  // after the barrier that follows
  const unsigned key = max(sh.s->lane_best[lane], kKeyNegInf);  // (keys below that of -inf are no numbers)
  const unsigned top = wave_max_u(key);
  const float v = ukey_val(key), M = ukey_val(top);
  if (K == 1 || top == kKeyNegInf) return M;
  auto reach = [&](float d) { return static_cast<int>(__popcll(__ballot(v >= M - d))) >= K; };
  float d = 0.0f;
#pragma unroll
  for (int e = 7; e >= -3; --e) {
    const float step = e >= 0 ? static_cast<float>(1 << e) : 1.0f / static_cast<float>(1 << -e);
    d = reach(step) ? step : d;
  }
  if (d > 0.0f) {
    const float e0 = d, e1 = 0.875f * d, e2 = 0.75f * d, e3 = 0.625f * d;
    d = reach(e3) ? e3 : reach(e2) ? e2 : reach(e1) ? e1 : e0;
    return M - d;
  }
  unsigned T = 0;
#pragma unroll 1
  for (int bit = 31; bit >= 12; --bit) {
    const unsigned c = T | (1u << bit);
    if (static_cast<int>(__popcll(__ballot(key >= c))) >= K) T = c;
  }
  return ukey_val(T < kKeyNegInf ? kKeyNegInf : T);
}

// What a beam's row needs besides its log-probs.
struct Beam {
  int k, s;
  float hyp, p_root, eos_boost;
};
__device__ __forceinline__ Beam beam_at(const TreeView& t, int k, int s, float hyp) {
  Beam b{k, s, hyp, t.p_root[s], 0.0f};
  if (t.eos >= 0) b.eos_boost = t.eos_score[s];
  return b;
}

// Walks the failure chain of the beam, deepest state first, one arc per lane, marking tokens as it goes (the marks are
// clear before): `use(total, token, child)` for every arc that no deeper state shadows.  LDS operations of one wave
// execute in order, and the tokens of one state are distinct, so marks need no barrier inside the wave.  The first arcs
// of a state and of the one behind its failure link, which share a record, are requested together.
template <typename Use>
__device__ __forceinline__ void walk_mark(const TreeView& t, const Beam& b, const float* __restrict__ row, float alpha,
                                          unsigned* marks, int lane, Use&& use) {
  float p = 0.0f;
  auto one = [&](const ArcRec& a, float xv, float back, int child) {
    const int pos = token_pos<false>(t, a.token);
    if (!tag_test(marks, pos)) {
      tag_set(marks, pos);
      use(__fadd_rn(b.hyp, __fadd_rn(xv, __fmul_rn(alpha, __fadd_rn(back, a.score)))), a.token, child);
    }
  };
  auto rest = [&](const Rec& r, float back) {
#pragma unroll 1
    for (int j = 64 + lane; j < r.count; j += 64) {
      const ArcRec a = t.arc[r.begin + j];
      one(a, row[a.token], back, r.begin + j + 1);
    }
  };
#pragma unroll 1
  for (int x = b.s; x != 0;) {
    const Rec2 r = load_rec2(t, x);
    const bool two = r.a.fail != 0, has0 = lane < r.a.count, has1 = two && lane < r.b.count;
    const ArcRec a0 = t.arc[r.a.begin + max(0, min(lane, r.a.count - 1))];
    ArcRec a1 = a0;
    if (two) a1 = t.arc[r.b.begin + max(0, min(lane, r.b.count - 1))];
    const float x0 = row[has0 ? a0.token : 0], x1 = row[has1 ? a1.token : 0];
    if (has0) one(a0, x0, p, r.a.begin + lane + 1);
    rest(r.a, p);
    if (!two) return;
    p = __fadd_rn(p, r.a.backoff);
    if (has1) one(a1, x1, p, r.b.begin + lane + 1);
    rest(r.b, p);
    p = __fadd_rn(p, r.b.backoff);
    x = uniform_i(r.b.fail);
  }
}

// The same walk again, clearing the marks the first one has left: an arc whose mark is gone already is shadowed.
template <typename Use>
__device__ __forceinline__ void walk_clear(const TreeView& t, const Beam& b, const float* __restrict__ row, float alpha,
                                           unsigned* marks, int lane, Use&& use) {
  float p = 0.0f;
#pragma unroll 1
  for (int x = b.s; x != 0;) {
    const Rec r = load_rec(t, x);
#pragma unroll 1
    for (int j = lane; j < r.count; j += 64) {
      const ArcRec a = t.arc[r.begin + j];
      const int pos = token_pos<false>(t, a.token);
      if (tag_test(marks, pos)) {
        atomicAnd(&marks[pos >> 5], ~(1u << (pos & 31)));
        use(__fadd_rn(b.hyp, __fadd_rn(row[a.token], __fmul_rn(alpha, __fadd_rn(p, a.score)))), a.token, r.begin + j + 1);
      }
    }
    p = __fadd_rn(p, r.backoff);
    x = uniform_i(r.fail);
  }
}

// Totals of the lane's NS positions from `cb` on, from their log-probs and root scores, in place of the log-probs: the
// blank boosts by 0, the EOS token by the value tabulated for the state; copies behind the end become NaN.
template <int NS>
__device__ __forceinline__ void piece_totals(const TreeView& t, const Beam& b, int cb, float alpha, int lane,
                                             const float (&rw)[NS], float (&x)[NS]) {
  const int blank = (t.blank >= 0 ? token_pos<false>(t, t.blank) : -1) - cb;
  const int eos = (t.eos >= 0 ? token_pos<false>(t, t.eos) : -1) - cb;
  float bo[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) bo[j] = __fmul_rn(alpha, __fadd_rn(b.p_root, rw[j]));
  const bool has_blank = static_cast<unsigned>(blank) < 64u * NS, has_eos = static_cast<unsigned>(eos) < 64u * NS;
  if (has_blank || has_eos || cb + 64 * NS > t.V) {  // uniform, and false for most pieces
    const int ln = opaque(lane);
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      if (has_blank && slot_is(j, ln, blank)) bo[j] = __fmul_rn(alpha, 0.0f);
      if (has_eos && slot_is(j, ln, eos)) bo[j] = __fmul_rn(alpha, b.eos_boost);
      const int u = cb + 256 * (j >> 2) + 4 * ln;
      if ((j & 3) < u - min(u, t.V - 4)) bo[j] = NAN;
    }
  }
#pragma unroll
  for (int j = 0; j < NS; ++j) x[j] = __fadd_rn(b.hyp, __fadd_rn(x[j], bo[j]));
}

// NaN into the totals of marked positions.
template <int NS>
__device__ __forceinline__ void drop_marked(const unsigned* marks, int cb, int lane, float (&x)[NS]) {
#pragma unroll
  for (int i = 0; i < NS / 4; ++i) {
    const int pos = cb + 256 * i + 4 * lane;
    const unsigned bits = marks[pos >> 5] >> (pos & 31);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[4 * i + k] = (bits >> k) & 1u ? NAN : x[4 * i + k];
  }
}

template <int NS>
__device__ __forceinline__ float piece_max(const float (&x)[NS]) {  // (NaN entries are passed over; all NaN: -inf)
  float g[NS / 4];
  return max2(group_maxima(x, g), -INFINITY);
}

// Puts the survivors of a piece (pmax: the lane's largest total of it) on the list: a bit per slot, then a turn of a
// loop per slot that has any.  (The push written out for every slot made 13 to 34 KB of code per kernel, and a step of
// few utterances waits for its instructions, too; a loop over all slots took 0.5 us longer.)  MAY_STOP: once the list has
// overflowed the rest is left out.  (Not the first time: looking at the count costs a step of 16 beams 1.5 %.)
template <bool MAY_STOP, int NS>
__device__ __forceinline__ void push_hits(const Shared& sh, const TreeView& t, int k, int cb, int lane, unsigned hits,
                                          const float (&x)[NS]) {
  float y[NS];  // (a copy: indexed by a number that is not a constant, it must not take the whole row out of registers)
#pragma unroll
  for (int j = 0; j < NS; ++j) y[j] = x[j];
  for (u64 left = __ballot(hits != 0); left != 0; left = __ballot(hits != 0)) {
    const int j = __builtin_ctz(__builtin_amdgcn_readlane(static_cast<int>(hits), first_lane(left)));
    if ((hits >> j) & 1u) push(sh, y[j], k, pos_token<false>(t, cb + tok_of(j, lane)), t.V, -1);
    hits &= ~(1u << j);
    if (MAY_STOP && overflowed(sh)) break;
  }
}
template <int NS>
__device__ __forceinline__ void push_piece(const Shared& sh, const TreeView& t, int k, int cb, int lane, float bound,
                                           float pmax, const float (&x)[NS]) {
  if (__ballot(pmax >= bound) == 0) return;
  unsigned hits = 0;
#pragma unroll
  for (int j = 0; j < NS; ++j) hits |= x[j] >= bound ? 1u << j : 0u;
  push_hits<false>(sh, t, k, cb, lane, hits, x);
}
// The same for a bound on (total, flat index).
template <int NS>
__device__ __forceinline__ void push_piece(const Shared& sh, const TreeView& t, int k, int cb, int lane, u64 bound,
                                           float pmax, const float (&x)[NS]) {
  const float total = key_total(bound);
  if (__ballot(pmax >= total) == 0 || overflowed(sh)) return;
  unsigned hits = 0;
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const u64 key = cand_key(x[j], k * t.V + pos_token<false>(t, cb + tok_of(j, lane)));
    hits |= x[j] >= total && key >= bound ? 1u << j : 0u;
  }
  push_hits<true>(sh, t, k, cb, lane, hits, x);
}

// The arcs of a wave's beams: every lane keeps its best and the value of its second best, so that a second walk is
// needed only where a lane holds two survivors.
struct ArcBest {
  float best = -INFINITY, second = -INFINITY;
  int k = 0, tok = 0, child = -1;  // (child < 0: none)
  __device__ __forceinline__ void add(float total, int beam, int token, int c) {
    const bool up = total > best || child < 0;
    second = up ? (child < 0 ? second : best) : max2(second, total);
    best = up ? total : best;
    k = up ? beam : k;
    tok = up ? token : tok;
    child = up ? c : child;
  }
};

// A long list costs in ranks what it has saved in passes (1024 entries: 20 us): it is cut above a raised bound first.
constexpr int kRankMost = 192;
__device__ __forceinline__ int shorten(const Shared& sh, int lane, int n, int K) {
  const int i = threadIdx.x;  // (a list that is long has no more entries than the workgroup has threads)
  const u64 bound = raised_bound(sh, lane, n, K), key = i < n ? sh.key[i] : 0;
  const int4 e = i < n ? sh.entry[i] : make_int4(0, 0, 0, 0);
  __syncthreads();
  if (threadIdx.x == 0) sh.s->count = 0;
  __syncthreads();
  if (key >= bound) {
    const int at = atomicAdd(&sh.s->count, 1);
    sh.key[at] = key;
    sh.entry[at] = e;
  }
  __syncthreads();
  return sh.s->count;
}

// The list is complete with n entries (a barrier lies behind the last push): rank every entry by counting and write the
// first K.
__device__ __forceinline__ void write_ranked(const Shared& sh, const TreeView& t, int u, int n, int K,
                                             const int32_t* states_in, const BeamOut& out) {
  if (n > kRankMost) n = shorten(sh, threadIdx.x & 63, n, K);  // (uniform)
#pragma unroll 1
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const u64 key = sh.key[i];
    const int4 e = sh.entry[i];
    const int v = e.y, k = e.z, child = e.w;
    int next = child;
    if (child < 0) next = v == t.blank || v == t.eos ? states_in[u * K + k] : t.root_next[v];  // (in flight below)
    int rank = 0;
#pragma unroll 4
    for (int q = 0; q < n; ++q) rank += sh.key[q] > key ? 1 : 0;
    if (rank < K) out.put(u * K + rank, v, k, next, __int_as_float(e.x));
  }
  for (int r = n + static_cast<int>(threadIdx.x); r < K; r += blockDim.x) out.put(u * K + r, -1, -1, -1, NAN);  // (NaN rows)
}

// An overflowed list is collected again above a raised bound, until it fits: `again(bound)` pushes every candidate that
// reaches the bound (by key) and may stop once the list overflows.  Called by all threads, after the barrier behind the
// last push; ends with one and returns the number of entries.
template <typename Again>
__device__ __forceinline__ int collect_again(const Shared& sh, int lane, int K, Again&& again) {
  int n;
  while ((n = sh.s->count) > sh.cap) {  // (uniform)
    const u64 bound = raised_bound(sh, lane, sh.cap, K);
    __syncthreads();  // every wave has read the list
    if (threadIdx.x == 0) sh.s->count = 0;
    __syncthreads();
    again(bound);
    __syncthreads();
  }
  return n;
}

// Survivors of an utterance whose hypothesis scores are all -inf: flat indices 0 .. K - 1, with totals of -inf.  One wave.
// The arcs of a state ascend by token, so those on the first n tokens are among its first n.
__device__ __forceinline__ void put_dead(const Shared& sh, const TreeView& t, int u, int K, const int32_t* states_in, int lane,
                                         const BeamOut& out) {
#pragma unroll 1
  for (int k = 0; k * t.V < K; ++k) {
    const int s = uniform_i(states_in[u * K + k]), n = min(t.V, K - k * t.V);
    if (lane < n) sh.s->child[lane] = -1;
#pragma unroll 1
    for (int x = s; x != 0;) {  // deepest state first
      const Rec r = load_rec(t, x);
      if (lane < min(r.count, n)) {
        const int v = t.arc[r.begin + lane].token;
        if (v < n && sh.s->child[v] < 0) sh.s->child[v] = r.begin + lane + 1;
      }
      x = uniform_i(r.fail);
    }
    if (lane < n) {
      int next = sh.s->child[lane];
      if (next < 0) next = lane == t.blank || lane == t.eos ? s : t.root_next[lane];
      out.put(u * K + k * t.V + lane, lane, k, next, -INFINITY);
    }
  }
}

// The tree and the validity of an utterance (uniform over the workgroup); an utterance with an invalid state or tree
// is marked as a whole.
__device__ __forceinline__ bool utterance_ok(const TreePick& pick, DeviceTree& mine, const int32_t* states_in, int u, int K,
                                             int lane, const BeamOut& out) {
  const bool tree_ok = pick_tree(pick, u, mine);
  const int s = states_in[u * K + min(lane, K - 1)];
  const bool ok = tree_ok && __ballot(static_cast<unsigned>(s) >= static_cast<unsigned>(mine.num_states)) == 0;
  const int slot = threadIdx.x;
  if (!ok && slot < K) out.put(u * K + slot, -1, -1, -1, NAN);
  return ok;
}

// ---- rows held in registers ---------------------------------------------------------------------------------------------
// A beam has `parts` waves, each with 64 * NS positions of its row.  ONE: a single beam in a single wave.  A step is
// latency-bound, so the requests go out in the order of the single greedy step: root scores, row, states and hypothesis
// score before the first wait (with a table of trees the root scores follow the table), and an utterance with an invalid
// state is decoded from the root and marked at the end, so that no early exit separates the wave start from the requests.
template <bool FOREST, int NS, bool ONE>
__global__ void __launch_bounds__(64 * kBeamWaves) beam_regs_kernel(
    const float* __restrict__ logp, int64_t row_stride, const float* hyp,
    const int32_t* __restrict__ states_in, const float* __restrict__ root_score, float alpha, int K, int parts, int words,
    int32_t* __restrict__ tokens, int32_t* __restrict__ parents, int32_t* __restrict__ states_out,
    float* scores_out, DeviceTree dt, TreePick pick) {
  constexpr int PS = NS < 16 ? NS : 16, NP = NS / PS;  // positions per lane of a piece, pieces
  // Whether the totals stay in registers for a list that overflows: with 16 positions that costs every step registers
  // (96 instead of 68, U x K, V = 4096 x 8, 1024 60 us instead of 49).
  constexpr bool KEPT = NS <= 8;
  extern __shared__ __align__(16) char lds[];
  __shared__ Small small;
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int u = blockIdx.x, k = wave / parts, part = wave - k * parts, P0 = part * 64 * NS, V = dt.vocab_size;
  const float* row = logp + static_cast<size_t>(u * K + k) * row_stride;
  float x[NP][PS], rw[PS];
  if constexpr (!FOREST) load_row<false>(root_score, P0, V, lane, rw);
#pragma unroll
  for (int c = 0; c < NP; ++c) load_row<false>(row, P0 + c * 64 * PS, V, lane, x[c]);
  const int sk = states_in[u * K + min(lane, K - 1)];  // every wave sees all K states
  const float hk = hyp[u * K + min(lane, K - 1)];    // ... and hypothesis scores
  __builtin_amdgcn_sched_barrier(0);  // (all of the above is in flight before the first wait)
  const Shared sh = shared_at(lds, &small, nwaves);
  unsigned* marks = reinterpret_cast<unsigned*>(lds + (ONE ? 0 : list_bytes(nwaves)));
  const BeamOut out{tokens, parents, states_out, scores_out};
  const int slot = threadIdx.x;
  DeviceTree mine = dt;
  if constexpr (FOREST) {
    if (!pick_tree(pick, u, mine)) {  // (uniform over the workgroup)
      if (slot < K) out.put(u * K + slot, -1, -1, -1, NAN);
      return;
    }
  }
  const TreeView t = make_view(mine);
  if constexpr (FOREST) load_row<false>(t.root_score, P0, V, lane, rw);
  if (slot == 0) sh.s->count = 0;
  if (slot < 64) sh.s->lane_best[slot] = 0;
  unsigned* m = marks + k * words;
  const bool bad = __ballot(!valid_state(t, sk)) != 0;
  if (!bad && __ballot(hk != -INFINITY) == 0) {  // (a wave that reads `hyp` after this has overwritten it sees the same)
    if (wave == 0) put_dead(sh, t, u, K, states_in, lane, out);
    return;
  }
  const Beam b = beam_at(t, k, bad ? 0 : __builtin_amdgcn_readlane(sk, k),
                         __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hk), k)));
  ArcBest arcs;
  if (part == 0 && b.s != 0) {
    tags_clear_n(m, words, lane);
    walk_mark(t, b, row, alpha, m, lane,
                          [&](float total, int tok, int child) { arcs.add(total, k, tok, child); });
  }
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    if (c > 0) load_row<false>(t.root_score, P0 + c * 64 * PS, V, lane, rw);
    piece_totals(t, b, P0 + c * 64 * PS, alpha, lane, rw, x[c]);
  }
  __syncthreads();  // the marks are set
  float top = max2(arcs.best, -INFINITY), pmax[NP];
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    if (b.s != 0) drop_marked(m, P0 + c * 64 * PS, lane, x[c]);
    pmax[c] = piece_max(x[c]);
    top = max2(top, pmax[c]);
  }
  if constexpr (ONE) {
    // the best total itself, of which only the lowest token is wanted: no list
    const float bound = ukey_val(wave_max_u(ukey(top)));
    int flat = arcs.child >= 0 && arcs.best == bound ? arcs.tok : INT_MAX, child = arcs.child;
    if (b.s != 0 && __ballot(arcs.second >= bound) != 0) {
      walk_clear(t, b, row, alpha, m, lane, [&](float total, int tok, int c) {
        if (total == bound && tok < flat) {
          flat = tok;
          child = c;
        }
      });
    }
#pragma unroll
    for (int c = NP - 1; c >= 0; --c)
#pragma unroll
      for (int j = PS - 1; j >= 0; --j) {
        const int v = pos_token<false>(t, P0 + c * 64 * PS + tok_of(j, lane));
        if (x[c][j] == bound && v < flat) {
          flat = v;
          child = -1;
        }
      }
    const int v = wave_min_nn(flat);
    if (bad || v == INT_MAX) {
      if (lane == 0) out.put(u, -1, -1, -1, NAN);  // (no number in the row, for one)
    } else if (flat == v) {
      out.put(u, v, 0, child >= 0 ? child : v == t.blank || v == t.eos ? b.s : t.root_next[v], bound);
    }
    return;
  }
  post_lane(sh, lane, wave, nwaves, top);
  __syncthreads();
  const float bound = joint_bound(sh, lane, K);
  if (__ballot(top >= bound) != 0) {
#pragma unroll
    for (int c = 0; c < NP; ++c) push_piece(sh, t, k, P0 + c * 64 * PS, lane, bound, pmax[c], x[c]);
    if (part == 0 && b.s != 0 && __ballot(arcs.second >= bound) != 0) {
      walk_clear(t, b, row, alpha, m, lane, [&](float total, int tok, int child) {
        if (total >= bound) push(sh, total, k, tok, t.V, child);
      });
    } else if (arcs.child >= 0 && arcs.best >= bound) {
      push(sh, arcs.best, arcs.k, arcs.tok, t.V, arcs.child);
    }
  }
  __syncthreads();
  if (bad) {
    if (slot < K) out.put(u * K + slot, -1, -1, -1, NAN);
    return;
  }
  const int n = collect_again(sh, lane, K, [&](u64 floor) {
    const float total = key_total(floor);
    if (part == 0 && b.s != 0 && (!KEPT || __ballot(arcs.second >= total) != 0)) {
      tags_clear_n(m, words, lane);
      walk_mark(t, b, row, alpha, m, lane, [&](float v, int tok, int child) {
        if (v >= total && cand_key(v, k * V + tok) >= floor) push(sh, v, k, tok, V, child);
      });
    } else if (arcs.child >= 0 && arcs.best >= total && cand_key(arcs.best, k * V + arcs.tok) >= floor) {
      push(sh, arcs.best, k, arcs.tok, V, arcs.child);
    }
    if constexpr (KEPT) {
      push_piece(sh, t, k, P0, lane, floor, pmax[0], x[0]);
    } else {  // from memory again, 256 positions at a time
      __syncthreads();  // the marks are set
#pragma unroll 1
      for (int p0 = P0; p0 < P0 + 64 * NS; p0 += 256) {
        float y[4], ry[4];
        load_row<false>(row, p0, V, lane, y);
        load_row<false>(t.root_score, p0, V, lane, ry);
        piece_totals(t, b, p0, alpha, lane, ry, y);
        if (b.s != 0) drop_marked(m, p0, lane, y);
        push_piece(sh, t, k, p0, lane, floor, piece_max(y), y);
      }
    }
  });
  write_ranked(sh, t, u, n, K, states_in, out);
}

// ---- rows streamed -------------------------------------------------------------------------------------------------------
// Beam k has max(1, nwaves / K) waves, which take its chunks in turn; with more beams than waves a wave has several.
__global__ void __launch_bounds__(64 * kBeamWaves) beam_stream_kernel(
    const float* __restrict__ logp, int64_t row_stride, const float* hyp,
    const int32_t* __restrict__ states_in, float alpha, int K, int32_t* __restrict__ tokens,
    int32_t* __restrict__ parents, int32_t* __restrict__ states_out, float* scores_out, DeviceTree dt,
    TreePick pick) {
  extern __shared__ __align__(16) char lds[];
  __shared__ Small small;
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const Shared sh = shared_at(lds, &small, nwaves);
  unsigned* marks = reinterpret_cast<unsigned*>(lds + list_bytes(nwaves));
  const int u = blockIdx.x;
  const BeamOut out{tokens, parents, states_out, scores_out};
  DeviceTree mine = dt;
  if (!utterance_ok(pick, mine, states_in, u, K, lane, out)) return;
  const TreeView t = make_view(mine);
  if (__ballot(hyp[u * K + min(lane, K - 1)] != -INFINITY) == 0) {
    if (wave == 0) put_dead(sh, t, u, K, states_in, lane, out);
    return;
  }
  const int nch = (t.V + kChunk - 1) / kChunk, words = nch * kTagWords, last_ch = nch - 1;
  float* cmax = reinterpret_cast<float*>(marks + static_cast<size_t>(K) * words);  // [K][nch]
  const int parts = K < nwaves ? nwaves / K : 1, k0 = wave / parts, part = wave - k0 * parts;
  auto beam = [&](int k) { return beam_at(t, k, uniform_i(states_in[u * K + k]), uniform_f(hyp[u * K + k])); };
  auto row_of = [&](int k) { return logp + static_cast<size_t>(u * K + k) * row_stride; };
  const int slot = threadIdx.x;
  if (slot == 0) sh.s->count = 0;
  if (slot < 64) sh.s->lane_best[slot] = 0;
  ArcBest arcs;
  if (part == 0) {
    for (int k = k0; k < K; k += nwaves) {
      const Beam b = beam(k);
      unsigned* m = marks + static_cast<size_t>(k) * words;
      tags_clear_n(m, words, lane);
      walk_mark(t, b, row_of(k), alpha, m, lane,
                            [&](float total, int tok, int child) { arcs.add(total, k, tok, child); });
    }
  }
  __syncthreads();  // the marks are set
  float top = max2(arcs.best, -INFINITY);
  for (int k = k0; k < K; k += nwaves) {
    const Beam b = beam(k);
    const float* row = row_of(k);
    const unsigned* m = marks + static_cast<size_t>(k) * words;
    float x[2][16], rw[2][16];
    load_row<false>(row, min(part, last_ch) * kChunk, t.V, lane, x[0]);
    load_row<false>(t.root_score, min(part, last_ch) * kChunk, t.V, lane, rw[0]);
    for (int ch0 = part; ch0 < nch; ch0 += 2 * parts) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int ch = ch0 + q * parts, nx = min(ch + parts, last_ch) * kChunk;
        load_row<false>(row, nx, t.V, lane, x[(q + 1) % 2]);  // (without a condition: behind the end the last one again)
        load_row<false>(t.root_score, nx, t.V, lane, rw[(q + 1) % 2]);
        if (ch < nch) {
          piece_totals(t, b, ch * kChunk, alpha, lane, rw[q], x[q]);
          if (b.s != 0) drop_marked(m, ch * kChunk, lane, x[q]);
          const float cm = piece_max(x[q]);
          top = max2(top, cm);
          const float wm = ukey_val(wave_max_u(ukey(cm)));
          if (lane == 0) cmax[k * nch + ch] = wm;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  post_lane(sh, lane, wave, nwaves, top);
  __syncthreads();
  const float bound = joint_bound(sh, lane, K);
  auto push_rows = [&](auto floor, float least) {  // what reaches `floor`, of the chunks whose best total is not below `least`
    for (int k = k0; k < K; k += nwaves) {
      const Beam b = beam(k);
      const unsigned* m = marks + static_cast<size_t>(k) * words;
#pragma unroll 1
      for (int ch = part; ch < nch; ch += parts) {
        if (uniform_f(cmax[k * nch + ch]) >= least) {
          float x[16], rw[16];
          load_row<false>(row_of(k), ch * kChunk, t.V, lane, x);
          load_row<false>(t.root_score, ch * kChunk, t.V, lane, rw);
          piece_totals(t, b, ch * kChunk, alpha, lane, rw, x);
          if (b.s != 0) drop_marked(m, ch * kChunk, lane, x);
          push_piece(sh, t, k, ch * kChunk, lane, floor, piece_max(x), x);
          if (sizeof(floor) == sizeof(u64) && overflowed(sh)) return;
        }
      }
    }
  };
  push_rows(bound, bound);
  __syncthreads();  // (the second walk clears marks that the other waves of the beam have read until here)
  if (part == 0 && __ballot(arcs.second >= bound) != 0) {
    for (int k = k0; k < K; k += nwaves)
      walk_clear(t, beam(k), row_of(k), alpha, marks + static_cast<size_t>(k) * words, lane,
                             [&](float total, int tok, int child) {
                               if (total >= bound) push(sh, total, k, tok, t.V, child);
                             });
  } else if (arcs.child >= 0 && arcs.best >= bound) {
    push(sh, arcs.best, arcs.k, arcs.tok, t.V, arcs.child);
  }
  __syncthreads();
  const int n = collect_again(sh, lane, K, [&](u64 floor) {
    if (part == 0) {
      for (int k = k0; k < K; k += nwaves) {
        unsigned* m = marks + static_cast<size_t>(k) * words;
        tags_clear_n(m, words, lane);
        walk_mark(t, beam(k), row_of(k), alpha, m, lane, [&](float v, int tok, int child) {
          if (v >= key_total(floor) && cand_key(v, k * t.V + tok) >= floor) push(sh, v, k, tok, t.V, child);
        });
      }
    }
    __syncthreads();  // the marks are set
    push_rows(floor, key_total(floor));
  });
  write_ranked(sh, t, u, n, K, states_in, out);
}

// ---- few beams over aligned rows of 516 .. 1024 tokens ---------------------------------------------------------------------
// A wave per beam.  It keeps the raw row in LDS, where the arcs of the failure chain (one per lane, deepest state first)
// find their log-probs and leave their fused values and children; the beam's K best totals are taken in K rounds of
// arg-max (a taken entry becomes NaN, which no maximum or equality test selects), and wave 0 merges the K * K.  For one to
// three beams that is less than a bound and a list (see wave_beams).
constexpr int kWaveBeams = 3;
constexpr int kWaveLdsFloats = 2 * kChunk + kTagWords;  // row and values, children, marks
constexpr int kWaveCands = 16;                           // candidates (a multiple of four: the rows behind them are aligned)
static_assert(kWaveBeams * kWaveBeams <= kWaveCands, "the merge holds every wave's best");
constexpr size_t wave_beam_lds(int K) { return (3 * kWaveCands + static_cast<size_t>(K) * kWaveLdsFloats) * sizeof(float); }

template <int FORM>
__global__ void __launch_bounds__(64 * kWaveBeams) beam_wave_kernel(
    const float* __restrict__ logp, int64_t row_stride, const float* hyp, const int32_t* __restrict__ states_in,
    const float* __restrict__ root_score, float alpha, int K, int32_t* __restrict__ tokens, int32_t* __restrict__ parents,
    int32_t* __restrict__ states_out, float* scores_out, DeviceTree dt) {
  extern __shared__ __align__(16) char lds_bytes[];
  float* lds = reinterpret_cast<float*>(lds_bytes);
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6);
  const int u = blockIdx.x, h = u * K + wave;
  const TreeView t = make_view(dt);
  const int V = t.V;
  const float* lrow = logp + static_cast<size_t>(h) * row_stride;
  float x[16], c[16];
  load_row<FORM>(root_score, 0, V, lane, c, 0.0f);  // (the tree's array, as a leading argument: in registers at the start)
  load_row<FORM>(lrow, 0, V, lane, x);
  const int sk = states_in[u * K + min(lane, K - 1)];  // every wave sees all K states
  const float hs_in = hyp[h];
  __builtin_amdgcn_sched_barrier(0);  // (all of the above is in flight before the first wait)
  // per-slot multiplier of the boost (alpha; 0 in the blank's slot), formed while the states are on their way
  float am[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    am[j] = slot_is(j, lane, t.blank) ? 0.0f : alpha;
    asm volatile("" : "+v"(am[j]));  // (formed here, not where it is used)
  }
  __builtin_amdgcn_sched_barrier(0);
  float* cand_val = lds;  // [K * K], then the flat indices and the children
  int* cand_idx = reinterpret_cast<int*>(lds + kWaveCands);
  int* cand_nxt = cand_idx + kWaveCands;
  float* ov = lds + 3 * kWaveCands + wave * kWaveLdsFloats;
  int* ov_next = reinterpret_cast<int*>(ov + kChunk);
  unsigned* tags = reinterpret_cast<unsigned*>(ov + 2 * kChunk);
  const bool bad = __ballot(!valid_state(t, sk)) != 0;  // (marked as a whole at the end)
  const int s = bad ? 0 : __builtin_amdgcn_readlane(sk, wave);
  const float hs = uniform_f(hs_in);
  const Cursor cur = cursor_at(t, s);
  __builtin_amdgcn_sched_barrier(0);  // (the parts of the cursor are requested together)
#pragma unroll
  for (int j = 0; j < 16; ++j) c[j] = __fmul_rn(am[j], __fadd_rn(cur.p_root, c[j]));  // base boosts, in place
  tags_clear(tags, lane);
  store_row_lds(ov, lane, x);
  {
    float p = 0.0f;
    for (int xs = s; xs != 0;) {
      const Rec r = load_rec(t, xs);
      for (int j = lane; j < r.count; j += 64) {
        const ArcRec a = t.arc[r.begin + j];
        if (!tag_test(tags, a.token)) {  // tokens of one state are distinct: no lane races for an entry
          tag_set(tags, a.token);
          ov[a.token] = __fadd_rn(ov[a.token], __fmul_rn(alpha, __fadd_rn(p, a.score)));
          ov_next[a.token] = r.begin + j + 1;
        }
      }
      p = __fadd_rn(p, r.backoff);
      xs = uniform_i(r.fail);
    }
  }
  float tv[16];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int v0 = 256 * i + 4 * lane;
    const unsigned bits = tags[v0 >> 5] >> (v0 & 31);
    const float4 o = *reinterpret_cast<const float4*>(ov + v0);
    const float oa[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float expansion = ((bits >> k) & 1u) ? oa[k] : __fadd_rn(x[4 * i + k], c[4 * i + k]);
      // positions past V hold -inf: the real tokens, which come first, are taken before them
      tv[4 * i + k] = (FORM == kWhole || v0 + k < V) ? __fadd_rn(hs, expansion) : -INFINITY;
    }
  }
  if (t.eos >= 0) {  // EOS rule (Sec. II-C): boosted by the value tabulated for the state; no arc carries the token
    const float ce = __fmul_rn(alpha, cur.eos_boost);
    const int ln = opaque(lane);
#pragma unroll
    for (int j = 0; j < 16; ++j) tv[j] = slot_is(j, ln, t.eos) ? __fadd_rn(hs, __fadd_rn(x[j], ce)) : tv[j];
  }
  for (int r = 0; r < K; ++r) {
    float g[4];
    const float M = ukey_val(wave_max_u(ukey(group_maxima(tv, g))));
    const int v = uniform_i(pos_token<FORM>(t, first_pos_equal(tv, g, M, lane)));
    int nx = s;  // the blank and the EOS keep the state
    if (v != t.blank && v != t.eos) nx = tag_test(tags, v) ? ov_next[v] : t.root_next[v];
    if (lane == 0) {
      cand_val[wave * K + r] = M;
      cand_idx[wave * K + r] = wave * V + v;
      cand_nxt[wave * K + r] = nx;
    }
    const int taken = slot_in_lane(opaque(lane), v);
#pragma unroll
    for (int j = 0; j < 16; ++j) tv[j] = taken == j ? NAN : tv[j];
  }
  __syncthreads();
  if (wave != 0) return;
  const int n = K * K;
  const bool have = lane < n;
  const float val = have ? cand_val[lane] : 0.0f;
  const int idx = have ? cand_idx[lane] : INT_MAX, nxt = have ? cand_nxt[lane] : 0;
  bool live = have;
  for (int j = 0; j < K; ++j) {
    const float M = ukey_val(wave_max_u(live ? ukey(val) : 0u));
    const int best = wave_min_nn((live && val == M) ? idx : INT_MAX);
    if (live && idx == best) {
      tokens[u * K + j] = bad ? -1 : idx % V;
      parents[u * K + j] = bad ? -1 : idx / V;
      states_out[u * K + j] = bad ? -1 : nxt;
      scores_out[u * K + j] = bad ? NAN : val;
      live = false;
    }
  }
}

// Which calls the wave-per-beam kernel is for: one tree, aligned rows of more than 512 tokens (up to there the other kernel
// holds fewer positions per lane and is faster), one beam until the chip is full several times over, two or three where
// the chip is about full (us, this kernel / the other one):
//   V = 1024, K = 1: U = 1 3.64/3.71, 1024 5.13/5.41, 4096 6.43/7.31, 16384 19.5/19.9; V = 640: 4096 6.95/7.34, 16384 19.3/18.6
//   V = 1024, K = 2: U = 512 5.95/5.91, 768 6.19/7.23, 2048 7.46/8.68, 3072 10.4/10.2, 16384 40.3/38.7; V = 640: 2048 7.64/8.51
//   V = 1024, K = 3: U = 256 6.52/5.76, 768 7.39/7.85, 1536 9.11/9.74, 2048 12.6/11.1; V = 640: 1536 9.34/9.35
bool wave_beams(const DeviceTree& t, const TreePick& pick, const float* logp, int64_t row_stride, int K, int64_t U) {
  auto aligned16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  if (pick.table != nullptr || K > kWaveBeams || t.vocab_size <= 512 || t.vocab_size > kChunk || t.vocab_size % 4 != 0 ||
      row_stride % 4 != 0 || !aligned16(logp) || !aligned16(t.root_score))
    return false;
  return K == 1 ? U <= 8192 : U * K > 1024 && U * K <= 4608;
}

int g_beam_max_lds = 48 * 1024;  // dynamic LDS the device allows these kernels, set once

struct BeamPlan {
  int ns, parts, waves;  // ns == 0: streamed
  int words;             // marks of a beam
  size_t lds;
  bool one() const { return waves == 1 && ns >= 4 && ns <= 16; }  // (K == 1, a row of up to 1024 tokens)
};
// Positions per lane: the fewest that spread a beam's row over as many waves as the workgroup takes -- a step of few
// utterances is latency-bound, so it wants little to do in each wave -- but no more than kBeamFill waves over all
// utterances: past that a row cut finer only brings more barriers, bounds and lists.  (V = 1024, K = 4: U = 128 7.1 us
// with 8 positions, 7.7 with 16; U = 1024 9.8 us with 16, 12.5 with 8, 21.5 with 4.  V = 4096, K = 4, U = 512: 11.8 us
// with 32, 17.3 with 16.)  A single beam stays in one wave where 16 positions hold it.  Rows that do not fit at 64 positions are streamed.
constexpr int kBeamFill = 4096;
BeamPlan plan_beam(int V, int K, int64_t U) {
  const int nch = (V + kChunk - 1) / kChunk;
  BeamPlan p{0, 0, kBeamWaves, nch * kTagWords, 0};
  for (const int ns : {4, 8, 16, 32, 64}) {
    const int parts = (V + 64 * ns - 1) / (64 * ns);
    if (K * parts > kBeamWaves || (ns == 64 && p.ns == 32)) continue;
    const int words = parts * 2 * ns > nch * kTagWords ? parts * 2 * ns : nch * kTagWords;
    p = BeamPlan{ns, parts, K * parts, words, 0};
    if (parts == 1 || (U * K * parts <= kBeamFill && (K > 1 || ns >= 16))) break;
  }
  // (streamed: the maxima of a beam's chunks behind the marks)
  p.lds = (p.one() ? 0 : list_bytes(p.waves)) + static_cast<size_t>(K) * (p.words + (p.ns ? 0 : nch)) * sizeof(unsigned);
  return p;
}

}  // namespace

bool beam_wave_ok(const DeviceTree& t, int32_t U, int32_t K) {
  return t.p_root != nullptr && t.vocab_size >= 4 && plan_beam(t.vocab_size, K, U).lds <= static_cast<size_t>(g_beam_max_lds);
}

int launch_beam_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride, const float* d_hyp,
                     const int32_t* d_states_in, float alpha, int32_t U, int32_t K, int32_t* d_tokens,
                     int32_t* d_parents, int32_t* d_states_out, float* d_scores_out, hipStream_t stream) {
  const int V = t.vocab_size;
  if (wave_beams(t, pick, d_logp, row_stride, K, U)) {
#define PB_WAVE(FORM)                                                                                                     \
  hipLaunchKernelGGL(beam_wave_kernel<FORM>, dim3(static_cast<unsigned>(U)), dim3(static_cast<unsigned>(64 * K)),         \
                     wave_beam_lds(K), stream, d_logp, row_stride, d_hyp, d_states_in, t.root_score, alpha, K, d_tokens,  \
                     d_parents, d_states_out, d_scores_out, t)
    if (V == kChunk) {
      PB_WAVE(kWhole);
    } else {
      PB_WAVE(kGroups);
    }
#undef PB_WAVE
    return hipGetLastError() == hipSuccess ? PB_OK : PB_EHIP;
  }
  const BeamPlan p = plan_beam(V, K, U);
  const dim3 grid(static_cast<unsigned>(U)), block(static_cast<unsigned>(64 * p.waves));
  const bool forest = pick.table != nullptr;
#define PB_REGS(FOREST, NS, ONE)                                                                                     \
  hipLaunchKernelGGL((beam_regs_kernel<FOREST, NS, ONE>), grid, block, p.lds, stream, d_logp, row_stride, d_hyp,     \
                     d_states_in, t.root_score, alpha, K, p.parts, p.words, d_tokens, d_parents, d_states_out,       \
                     d_scores_out, t, pick)
#define PB_SHAPE(NS, ONE)     \
  if (forest) {               \
    PB_REGS(true, NS, ONE);   \
  } else {                    \
    PB_REGS(false, NS, ONE);  \
  }
  switch (p.ns + (p.one() ? 1 : 0)) {
    case 5: PB_SHAPE(4, true) break;
    case 9: PB_SHAPE(8, true) break;
    case 17: PB_SHAPE(16, true) break;
    case 4: PB_SHAPE(4, false) break;
    case 8: PB_SHAPE(8, false) break;
    case 16: PB_SHAPE(16, false) break;
    case 32: PB_SHAPE(32, false) break;
    case 64: PB_SHAPE(64, false) break;
    default:
      hipLaunchKernelGGL(beam_stream_kernel, grid, block, p.lds, stream, d_logp, row_stride, d_hyp, d_states_in, alpha, K,
                         d_tokens, d_parents, d_states_out, d_scores_out, t, pick);
  }
#undef PB_SHAPE
#undef PB_REGS
  return hipGetLastError() == hipSuccess ? PB_OK : PB_EHIP;
}

int prepare_beam_kernels(int max_lds_bytes) {
  constexpr int kStatic = sizeof(Small) + 1024;
  const int bytes = max_lds_bytes - kStatic;
  int limit = 64 * 1024 - kStatic;
  if (bytes > limit) {
    const hipFuncAttribute attr = hipFuncAttributeMaxDynamicSharedMemorySize;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(beam_stream_kernel), attr, bytes) == hipSuccess)
      limit = bytes;
    else
      (void)hipGetLastError();
  }
  g_beam_max_lds = limit;
  return PB_OK;
}

}  // namespace pb
