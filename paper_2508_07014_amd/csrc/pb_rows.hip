// Multi-frame greedy decoding in two passes (gfx950, wave64): all rows at once, then the automaton.
//
// The segment decoders (pb_narrow.hpp, pb_wide.hip) stream the rows of a hypothesis in the order of its frames, so
// they fill the chip only where there are frames enough for some thousand segments, and a boundary guessed wrong
// means rows streamed again.  Here what a frame costs in bytes does not depend on the state at all:
//
//  * Pass 1 (rows_narrow_kernel, rows_wide_kernel; every row on its own, no order) finds the winner w of the row
//    under root-state boosts, and the raw arg-max for the two-stage rules.  In a state with total backoff p a token
//    without an arc on the chain has the fused value logp[v] + alpha * (p + root_score[v]): p moves all of them by
//    the same amount, so w is the base winner in every state -- up to rounding.  The rounding is bounded: with u =
//    2^-24, S >= |p + root_score| (DeviceTree::reach) and M the winner's value, a computed fused value is off by less
//    than u * (2.01 |alpha| S + 1.01 |value|), in the root and in the state, for either of two tokens.  A token whose
//    value under root boosts lies more than u * (10.1 |alpha| S + 4.1 |M|) below M therefore loses in every state.
//    A row with another token within that band (near_band: 12 and 6, the slack covers the band's own rounding) is
//    marked, and its frame decided by a plain pass over the row -- unless log-prob and root score are the winner's
//    own, as they are for most exact ties: equal operands give equal values in every state, and the lower token wins.
//  * Pass 2 (walk_kernel; one workgroup per hypothesis) runs the automaton on the winners, a frame per lane.  The states
//    that the winners alone lead to come first: every lane carries the state of the frame before it over its own winner,
//    again until nothing changes, so a spoken phrase of n tokens takes n turns, all phrases side by side, and a turn is one
//    access to the table of arcs by (state, token).  Then all frames are decided from those states at once, their arcs
//    shared out over the lanes.  A frame that comes out differently sends the ones behind it round again, once side by side,
//    then one frame after the other where they are few, until every frame was decided from what the frame before it led to;
//    the waves hand on their ends between barriers.  Frames that the winners do not settle (near ties, a base winner shadowed
//    by a weaker arc, a barred label under the CTC rule) take passes over their rows, a wave or a few to each.
//
// What bounds pass 2 is how many scattered lines one CU takes in (a frame's winners, root scores, records, arcs and their
// log-probs: about 8 cycles a line), then the chain of dependent accesses, and where most frames surprise the winners the
// instructions of one wave that follows them (about 4000 cycles a frame).  Against deciding frames one after the other inside
// a phrase, in segments (medians of a trace): 500 frames x 32, V = 1025, CTC rule 62.6 -> 43.3 us; 100 x 16, V = 32001
// 32.4 -> 21.4.
//
// Between the passes the winners travel in the call's own outputs (put_winners), so the outputs must not overlap what pass 2
// reads (frames_apart).
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

// Values below M by more than this lose to the winner in every state (see above); the last term covers denormals.
__device__ __forceinline__ float near_band(float alpha, float reach, float M) {
  return 1.1920929e-7f * (6.0f * fabsf(alpha) * reach + 3.0f * fabsf(M)) + 1e-36f;
}

// The token that says where the frame leads under root-state boosts: the blank (single-stage rule: boost 0) or w.
__device__ __forceinline__ int root_choice(const TreeView& t, float alpha, float x_blank, float M, int w) {
  const float fb = __fadd_rn(x_blank, __fmul_rn(alpha, 0.0f));
  return t.blank >= 0 && (fb > M || (fb == M && t.blank < w)) ? t.blank : w;
}

// The winners of a row between the passes: w, v0 and the mark in one word where the vocabulary allows it (the words of a
// hypothesis lie B apart, a cache line each, and what pass 2 waits for is lines).
constexpr int kPackedV = 1 << 15;
__device__ __forceinline__ void put_winners(int V, size_t o, int w, int v0, bool marked, int32_t* tokens, int32_t* states) {
  if (V <= kPackedV) {
    tokens[o] = w | v0 << 15 | (marked ? 1 << 30 : 0);
  } else {
    tokens[o] = marked ? ~w : w;
    states[o] = v0;
  }
}
__device__ __forceinline__ void get_winners(int V, int word, int word2, int& w, int& v0, bool& marked) {
  const bool packed = V <= kPackedV;
  marked = packed ? (word >> 30 & 1) != 0 : word < 0;
  w = packed ? word & (kPackedV - 1) : word < 0 ? ~word : word;
  v0 = packed ? word >> 15 & (kPackedV - 1) : word2;
}

// ---- pass 1, rows of up to 64 * NS positions: a wave per row, root scores kept in registers -------------------------
// A wave takes frames s, s + strips, ... of hypothesis b, the next row requested while one is looked at.
template <int NS, int SEL>
__global__ void __launch_bounds__(256) rows_narrow_kernel(DeviceTree dt, TreePick pick, const float* __restrict__ logp,
                                                          int64_t frame_stride, int64_t row_stride, float alpha, int T,
                                                          int B, int strips, int32_t* __restrict__ tokens,
                                                          int32_t* __restrict__ states) {
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6);
  const int g = blockIdx.x * (blockDim.x >> 6) + wave;
  const int s = g / B, b = g - s * B;
  if (s >= strips) return;
  DeviceTree mine = dt;
  if (!pick_tree(pick, b, mine)) return;  // (pass 2 marks every frame of the hypothesis)
  const TreeView t = make_view(mine);
  const int V = t.V;
  const float* rp = logp + static_cast<size_t>(b) * row_stride;
  float x[NS], rw[NS], c[NS];
  load_row<false>(t.root_score, 0, V, lane, rw);
  load_row<false>(rp + static_cast<size_t>(s) * frame_stride, 0, V, lane, x);
#pragma unroll
  for (int i = 0; i < NS / 4; ++i) {
    const float4 q = mask_special<false>(t, 256 * i + 4 * lane, make_float4(rw[4 * i], rw[4 * i + 1], rw[4 * i + 2], rw[4 * i + 3]));
    rw[4 * i + 0] = q.x; rw[4 * i + 1] = q.y; rw[4 * i + 2] = q.z; rw[4 * i + 3] = q.w;
  }
#pragma unroll
  for (int j = 0; j < NS; ++j) c[j] = __fmul_rn(alpha, rw[j]);
  const int bcol = t.blank >= 0 ? t.blank : 0;
  for (int f = s; f < T; f += strips) {
    const float* row = rp + static_cast<size_t>(f) * frame_stride;
    const int fn = f + strips < T ? f + strips : f;
    float xn[NS];
    const float x_blank = SEL == 0 ? row[bcol] : 0.0f;
    load_row<false>(rp + static_cast<size_t>(fn) * frame_stride, 0, V, lane, xn);
    float v[NS], gm[NS / 4];
#pragma unroll
    for (int j = 0; j < NS; ++j) v[j] = __fadd_rn(x[j], c[j]);
    const float m = max2(group_maxima(v, gm), -INFINITY);  // (a lane that holds nothing but masked columns)
    const float M = ukey_val(wave_max_u(ukey(m)));
    const int wpos = first_pos_equal(v, gm, M, lane);
    int w = pos_token<false>(t, wpos);
    const float thr = M - near_band(alpha, mine.reach, M);
    const int own = lane == ((wpos >> 2) & 63) ? (((wpos >> 8) << 2) | (wpos & 3)) : -1;
    bool near = false;
#pragma unroll
    for (int j = 0; j < NS; ++j) near = near || (v[j] >= thr && j != own);
    bool marked = M == -INFINITY;
    if (!marked && __ballot(near) != 0) {
      const float xw = row[w], rww = t.root_score[w];
      near = false;
#pragma unroll
      for (int j = 0; j < NS; ++j) near = near || (v[j] >= thr && !(x[j] == xw && rw[j] == rww));
      marked = __ballot(near) != 0;
    }
    int v0 = w;
    if (SEL != 0) {
      float M0;
      plain_argmax<false>(t, x, lane, M0, v0);
    } else {
      v0 = root_choice(t, alpha, x_blank, M, w);
    }
    if (lane == 0) put_winners(V, static_cast<size_t>(f) * B + b, w, v0, marked, tokens, states);
#pragma unroll
    for (int j = 0; j < NS; ++j) x[j] = xn[j];
  }
}

// ---- pass 1, wider rows: a workgroup per row, its waves taking the chunks in turn -------------------------------------
struct RowPart {
  float M, M0;
  int w, v0;
};

template <int SEL>
__global__ void __launch_bounds__(1024) rows_wide_kernel(DeviceTree dt, TreePick pick, const float* __restrict__ logp,
                                                         int64_t frame_stride, int64_t row_stride, float alpha, int B,
                                                         int32_t* __restrict__ tokens, int32_t* __restrict__ states) {
  __shared__ RowPart part[16];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int f = blockIdx.x / B, b = blockIdx.x - f * B;
  DeviceTree mine = dt;
  if (!pick_tree(pick, b, mine)) return;  // (pass 2 marks every frame of the hypothesis; the whole workgroup leaves)
  const TreeView t = make_view(mine);
  const int V = t.V, nch = (V + kChunk - 1) / kChunk;
  const float* row = logp + static_cast<size_t>(f) * frame_stride + static_cast<size_t>(b) * row_stride;
  const int bpos = t.blank >= 0 ? token_pos<false>(t, t.blank) : -1, epos = t.eos >= 0 ? token_pos<false>(t, t.eos) : -1;
  // root scores of chunk ch with the special columns and the copies behind the end out of the way
  auto mask = [&](int ch, float (&rw)[16]) {
    const int cb = ch * kChunk;
    const bool special = static_cast<unsigned>(bpos - cb) < static_cast<unsigned>(kChunk) ||
                         static_cast<unsigned>(epos - cb) < static_cast<unsigned>(kChunk) || cb + kChunk > V;
    if (special) {  // uniform, and false for most chunks
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 q = mask_special<false>(t, cb + 256 * i + 4 * opaque(lane),
                                             make_float4(rw[4 * i], rw[4 * i + 1], rw[4 * i + 2], rw[4 * i + 3]));
        rw[4 * i + 0] = q.x; rw[4 * i + 1] = q.y; rw[4 * i + 2] = q.z; rw[4 * i + 3] = q.w;
      }
    }
  };
  LaneBest fb = lane_best_init(), rb = lane_best_init();
  float second = -INFINITY;  // the lane's second largest fused value
  float x[2][16], rw[2][16];
  const int last_ch = nch - 1;
  load_row<false>(row, min(wave, last_ch) * kChunk, V, lane, x[0]);
  load_row<false>(t.root_score, min(wave, last_ch) * kChunk, V, lane, rw[0]);
  const float x_blank = SEL == 0 && t.blank >= 0 ? row[t.blank] : 0.0f;
  for (int ch0 = wave; ch0 < nch; ch0 += 2 * nwaves) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ch = ch0 + u * nwaves;
      // the next chunk is requested without a condition (behind the end: the last one again, from cache)
      load_row<false>(row, min(ch + nwaves, last_ch) * kChunk, V, lane, x[(u + 1) % 2]);
      load_row<false>(t.root_score, min(ch + nwaves, last_ch) * kChunk, V, lane, rw[(u + 1) % 2]);
      if (ch < nch) {
        mask(ch, rw[u]);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const float v = __fadd_rn(x[u][j], __fmul_rn(alpha, rw[u][j]));
          second = __builtin_amdgcn_fmed3f(v, fb.m, second);  // (second <= m; a NaN leaves it as it is)
          const bool up = v > fb.m;
          fb.m = up ? v : fb.m;
          fb.code = up ? 16 * ch + j : fb.code;
        }
        if constexpr (SEL != 0) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const bool up = x[u][j] > rb.m;
            rb.m = up ? x[u][j] : rb.m;
            rb.code = up ? 16 * ch + j : rb.code;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  RowPart mine_part{0.0f, 0.0f, 0, 0};
  wave_pick<false>(t, fb, lane, mine_part.M, mine_part.w);
  if (SEL != 0) wave_pick<false>(t, rb, lane, mine_part.M0, mine_part.v0);
  if (lane == 0) part[wave] = mine_part;
  __syncthreads();
  const bool have = lane < nwaves;
  const RowPart q = part[have ? lane : 0];
  const float M = ukey_val(wave_max_u(have ? ukey(q.M) : 0u));
  const int w = wave_min_nn(have && q.M == M ? q.w : INT_MAX);
  int v0 = w;
  if (SEL != 0) {
    const float M0 = ukey_val(wave_max_u(have ? ukey(q.M0) : 0u));
    v0 = wave_min_nn(have && q.M0 == M0 ? q.v0 : INT_MAX);
  } else {
    v0 = root_choice(t, alpha, x_blank, M, w);
  }
  bool marked = M == -INFINITY;
  const float thr = M - near_band(alpha, mine.reach, M);
  const bool own = fb.m == M && pos_token<false>(t, code_pos(fb.code, lane)) == w;
  const bool near = second >= thr || (fb.m >= thr && !own);
  if (__syncthreads_or(!marked && near)) {  // (M is the same in every wave: all of them or none get here)
    const float xw = row[w], rww = t.root_score[w];
    bool differs = false;
    for (int ch = wave; ch < nch; ch += nwaves) {
      load_row<false>(row, ch * kChunk, V, lane, x[0]);
      load_row<false>(t.root_score, ch * kChunk, V, lane, rw[0]);
      mask(ch, rw[0]);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float v = __fadd_rn(x[0][j], __fmul_rn(alpha, rw[0][j]));
        differs = differs || (v >= thr && !(x[0][j] == xw && rw[0][j] == rww));
      }
    }
    marked = __syncthreads_or(differs) != 0;
  }
  if (threadIdx.x == 0) put_winners(V, static_cast<size_t>(f) * B + b, w, v0, marked, tokens, states);
}

// ---- pass 2 --------------------------------------------------------------------------------------------------------------
constexpr int kWalkPairs = 256;  // (frame, arc) pairs looked at together: four a lane

// The order of a frame's arcs: by value, then the lower token, then the level of the chain, deepest state first (11 bits;
// levels past the last one counted are told apart by a pass over the row).
constexpr int kLevelBits = 11, kLastLevel = (1 << kLevelBits) - 1, kMaxWalkV = 1 << (32 - kLevelBits);
static_assert(kMaxWalkV >= kMaxTableV);
__device__ __forceinline__ u64 arc_key(float value, int token, int level) {
  const unsigned low = static_cast<unsigned>(token) << kLevelBits | static_cast<unsigned>(min(level, kLastLevel));
  return static_cast<u64>(ukey(value)) << 32 | ~low;
}

// What the lanes of a wave tell each other about their frames while they share out the arcs.
struct alignas(16) WalkMeta {
  int start, c0, c1, c2;    // first pair of the frame; arcs on the first of four levels of the chain, first two, first three
  int o0, o1, o2, o3;       // arc of pair j of the frame: j + the offset of its level
  float p0, p1, p2, p3;     // backoff paid before the levels
};
struct WalkLds {  // of a wave
  WalkMeta meta[64];
  u64 best[64];        // largest (value, lowest token, deepest state) of the frame's arcs, see arc_key
  unsigned flag[64];   // 1: an arc overrides the base winner, 2: an arc of value -0.0
  int owner[kWalkPairs];
};
struct WalkJob {  // a frame of the block that needs a pass over its row, from state s, token excl barred (-1: none)
  int s, frame, excl;
};
// Frames of a wave that do not fit: up to this many are decided one after the other.  (1500 drawn calls against deciding
// them all side by side: 3 and 6 frames 0.99, log-depth weights at alpha = 1 0.82; one call in 80 is slower with 6, by up to
// 1.3 times where most frames are blanks, with 3 by up to 1.1.)
constexpr int kWalkFollow = 3;
constexpr int kWalkJobs = 64;  // listed at a time
struct WalkBest {  // of a wave's share of such a row
  float val;
  int tok, child;
};
struct WalkShared {  // of the workgroup
  int hard[16];  // frames of every wave that need a pass over their row
  WalkJob job[kWalkJobs];
  WalkBest part[16];
  int end[16], end_label[16];  // state and label every wave's frames end in
};

// A frame, one per lane: what pass 1 knows of its row, the state and label it is taken to start from, and its outcome.
struct WalkFrame {
  int w, v0, target;           // winner, raw arg-max (single-stage rule: see root_choice), where w leads from the root
  bool marked;
  float xw, x0, xe, rsw;       // log-probs of w, v0 (single-stage rule: the blank) and the EOS; root score of w
  int s, label;                // start
  int tok, next, moving;       // outcome: token, state after it; the token the frame emits when it moves the state
  bool moves, decided;         // the token moves the state; the outcome is the rule's (else: assumed)
  bool hard;                   // the outcome waits for a pass over the row (it is only likely until then)
  float val;
};

// (Known to lie in device memory: the accesses through pointers of a tree out of a table are flat ones otherwise, which
// LDS accesses wait for.)
#define PB_AS1 __attribute__((address_space(1)))
typedef int v2i __attribute__((ext_vector_type(2)));

// The table of arcs: the first aligned address behind the other sub-arrays (256 bytes, as all of them are aligned).
__device__ __forceinline__ const v4i PB_AS1* arc_table_of(const DeviceTree& t) {
  const uintptr_t end = t.eos_score != nullptr ? reinterpret_cast<uintptr_t>(t.eos_score + t.num_states)
                                               : reinterpret_cast<uintptr_t>(t.root_rec + t.vocab_size);
  return (const v4i PB_AS1*)((end + 255) & ~static_cast<uintptr_t>(255));
}

template <int SEL>
struct Walker {
  TreeView t;
  const v4i PB_AS1* states;  // StateRec, two to a state
  const v2i PB_AS1* arc;     // ArcRec: token, score bits
  const v4i PB_AS1* slots;   // ArcSlot
  unsigned slot_mask;
  const int PB_AS1* root_next;
  const RootRec* root_rec;
  const float PB_AS1 *p_root, *eos_score, *root_score;
  const float* hyp;  // logp of the frame of lane 0
  int64_t frame_stride;
  float alpha;
  WalkLds& L;
  int lane;

  // The lanes go on from here together.  Needed (a) between what they write and read of each other in LDS: the operations
  // of one wave are executed in order, but without the fences the compiler hands a lane what it has written itself; (b) at
  // the end of a loop body whose last branch differs from lane to lane: the lanes that take it and those that do not get a
  // way back of their own otherwise, the compiler makes two nested loops of the two, and the inner one runs its ballots and
  // shuffles with half of the lanes.  (No instruction comes of it.)
  __device__ __forceinline__ static void together() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // The state that the arc of state s on token v leads to, 0 if there is none (per lane).
  __device__ __forceinline__ int child(int s, int v) const {
#pragma unroll 1
    for (unsigned at = arc_hash(s, v);; ++at) {
      const v4i q = slots[at & slot_mask];
      if (q.x == s && q.y == v) return q.z;
      if (q.x < 0) return 0;
    }
  }
  // The state after token v in state s (per lane); target: where v leads from the root.
  __device__ __forceinline__ int step_to(int s, int v, int target) const {
#pragma unroll 1
    while (s != 0) {
      const int fail = states[2 * static_cast<size_t>(s)].z;
      const int next = child(s, v);
      if (next > 0) return next;
      s = fail;
    }
    return target;
  }

  // The state and label that the outcomes before a lane's frame lead to.  Frames lo .. hi - 1; the first starts from (from,
  // from_label).
  __device__ __forceinline__ void start_of(const WalkFrame& f, int lo, int hi, int from, int from_label, int& s, int& label) const {
    const u64 before = __ballot(f.moves && lane >= lo && lane < hi) & ((1ull << lane) - 1);
    const int got = __shfl(f.next, before ? 63 - __builtin_clzll(before) : 0);
    s = before ? got : from;
    label = -1;
    if (SEL == 2) {
      label = __shfl_up(f.tok, 1);
      label = lane == lo ? from_label : label;
    }
  }
  // The frames that were not decided from there, and where they start.
  __device__ __forceinline__ u64 misfits(const WalkFrame& f, int lo, int hi, int from, int from_label, int& s, int& label) const {
    start_of(f, lo, hi, from, from_label, s, label);
    return __ballot(lane >= lo && lane < hi && (!f.decided || s != f.s || (SEL == 2 && label != f.label)));
  }

  // Carries the outcomes of the frames to the starts of those behind them until nothing changes.  A frame whose start
  // has changed is undecided again and taken to emit what it did.  (At most 64 turns; a phrase takes as many as it has
  // tokens, side by side with all others.)  Frames lo .. hi - 1; the first starts from (from, from_label).
  __device__ __forceinline__ void settle_starts(WalkFrame& f, int lo, int hi, int from, int from_label) const {
    const bool mine = lane >= lo && lane < hi;
    bool any;
#pragma unroll 1
    do {
      int s, label;
      start_of(f, lo, hi, from, from_label, s, label);
      const bool changed = mine && (s != f.s || (SEL == 2 && label != f.label));
      any = __ballot(changed) != 0;
      if (changed) {
        f.s = s;
        f.label = label;
        f.decided = false;
        f.hard = false;
        if (SEL != 0) {
          f.moves = f.v0 != t.blank && (SEL != 2 || f.v0 != label);
          f.tok = f.moves ? f.moving : f.v0;
        }
        f.next = s;
        if (f.moves) f.next = step_to(s, f.tok, f.tok == f.w ? f.target : root_next[f.tok]);
      }
      together();
    } while (any);
  }

  // Decides the frames of `need` from their starts.
  __device__ __forceinline__ void decide_frames(WalkFrame& f, u64 need) const {
    const bool mine = (need >> lane) & 1;
    const bool kept = SEL != 0 && (f.v0 == t.blank || (SEL == 2 && f.v0 == f.label));
    // ---- the best arc of every frame: four levels of every frame's chain as one list of arcs, deepest state first, shared
    // out over the lanes ---------------------------------------------------------------------------------------------------
    // (One loop of little code: the same with the arcs of a frame on the lanes, eight frames unrolled, spent its time on
    // fetching instructions that no wave had run before.)
    float pr = 0.0f, eb = 0.0f;  // pr: the backoffs in chain order, at last what p_root holds
    int x = 0;                   // the next state of the chain
    bool hard = f.marked;
    if (mine && !kept && !hard) {
      if (t.eos >= 0) eb = eos_score[f.s];
      x = f.s;
    }
    L.best[lane] = 0;
    L.flag[lane] = 0;
#pragma unroll 1
    for (int level = 0; __ballot(x != 0) != 0; level += 4) {  // (a second turn for chains of more than four states)
      int c0 = 0, c1 = 0, c2 = 0, total = 0, o0 = 0, o1 = 0, o2 = 0, o3 = 0;
      const float p0 = pr;
      float p1 = 0.0f, p2 = 0.0f, p3 = 0.0f;
      if (x != 0) {
        const v4i q = states[2 * static_cast<size_t>(x)], q1 = states[2 * static_cast<size_t>(x) + 1];
        c0 = q.y;
        pr = p1 = __fadd_rn(p0, __int_as_float(q.w));
        o0 = q.x;
        c1 = c2 = total = c0;
        x = q.z;
        if (x != 0) {
          x = q1.z;
          pr = p2 = __fadd_rn(p1, __int_as_float(q1.w));
          o1 = q1.x - c0;
          c1 = c2 = total = c0 + q1.y;
          if (x != 0) {
            const v4i z = states[2 * static_cast<size_t>(x)], z1 = states[2 * static_cast<size_t>(x) + 1];
            x = z.z;
            pr = p3 = __fadd_rn(p2, __int_as_float(z.w));
            o2 = z.x - c1;
            c2 = total = c1 + z.y;
            if (x != 0) {
              x = z1.z;
              pr = __fadd_rn(p3, __int_as_float(z1.w));
              o3 = z1.x - c2;
              total = c2 + z1.y;
            }
          }
        }
      }
      const int end = prefix_sum(total);
      const int start = end - total, pairs = lane_i(end, 63);
      L.meta[lane] = WalkMeta{start, c0, c1, c2, o0, o1, o2, o3, p0, p1, p2, p3};
      together();
#pragma unroll 1
      for (int base = 0; base < pairs; base += kWalkPairs) {
#pragma unroll
        for (int k = 0; k < 4; ++k) L.owner[64 * k + lane] = 0;
        together();
        if (total > 0 && end > base && start < base + kWalkPairs) L.owner[max(start - base, 0)] = lane + 1;
        together();
        int fr[4], lv[4];
        float p[4], xa[4];
        v2i a[4];
        int before = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) fr[k] = L.owner[64 * k + lane];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          fr[k] = max(before, prefix_max(fr[k]));
          before = lane_i(fr[k], 63);
          fr[k] -= 1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const WalkMeta m = L.meta[fr[k]];
          const int j = min(base + 64 * k + lane, pairs - 1) - m.start;
          int off = m.o0;
          p[k] = m.p0;
          lv[k] = 0;
          if (j >= m.c0) { off = m.o1; p[k] = m.p1; lv[k] = 1; }
          if (j >= m.c1) { off = m.o2; p[k] = m.p2; lv[k] = 2; }
          if (j >= m.c2) { off = m.o3; p[k] = m.p3; lv[k] = 3; }
          a[k] = arc[j + off];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) xa[k] = hyp[static_cast<int64_t>(fr[k]) * frame_stride + a[k].x];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float v = __fadd_rn(xa[k], __fmul_rn(alpha, __fadd_rn(p[k], __int_as_float(a[k].y))));
          const int w = __shfl(f.w, fr[k]);
          if (base + 64 * k + lane < pairs) {
            atomicMax(&L.best[fr[k]], arc_key(v, a[k].x, level + lv[k]));
            const unsigned say = (a[k].x == w ? 1u : 0u) | (__float_as_uint(v) == 0x80000000u ? 2u : 0u);
            if (say != 0) atomicOr(&L.flag[fr[k]], say);
          }
        }
        together();
      }
    }
    together();
    const float M = __fadd_rn(f.xw, __fmul_rn(alpha, __fadd_rn(pr, f.rsw)));
    hard = hard || M == -INFINITY;
    const unsigned flag = L.flag[lane];
    const u64 key = L.best[lane];
    const unsigned low = ~static_cast<unsigned>(key);
    const bool overridden = (flag & 1u) != 0;
    float am = key != 0 ? ukey_val(static_cast<unsigned>(key >> 32)) : -INFINITY;
    int at = key != 0 ? static_cast<int>(low >> kLevelBits) : INT_MAX;
    bool by_arc = key != 0;
    // (the order tells -0.0 from 0.0, which are equal values: the lower token may be the other one's)
    hard = hard || ((flag & 2u) != 0 && am == 0.0f);
    // ---- the frames' decisions, one per lane ----------------------------------------------------------------------------
    auto special = [&](int token, float fv) {
      const bool take = fv > am || (fv == am && token < at);
      am = take ? fv : am;
      at = take ? token : at;
      by_arc = by_arc && !take;
    };
    if (SEL == 0 && t.blank >= 0) special(t.blank, __fadd_rn(f.x0, __fmul_rn(alpha, 0.0f)));
    if (t.eos >= 0) special(t.eos, __fadd_rn(f.xe, __fmul_rn(alpha, eb)));
    // (at == w: the winner's own arc has the base value, as it does after a whole phrase; the other tokens of that value
    // are higher ones)
    const bool take = at != INT_MAX && (am > M || (am == M && at <= f.w));
    hard = hard || (overridden && !take);  // the base winner is shadowed by an arc that does not beat it
    // A token belongs to the deepest state that has it.  Where that is another one than the winning arc's, its value there
    // is a lower one (of equal ones the deepest is taken), and another token may win.  (A shadowed arc that does not win
    // changes nothing.)
    int next = f.target;
    by_arc = by_arc && take;
    if (mine && !kept && !hard && by_arc) {
      const int level = static_cast<int>(low) & kLastLevel;
      int l = 0, c = f.s;
#pragma unroll 1
      for (;; ++l) {
        next = child(c, at);
        if (next > 0 || c == 0) break;  // (some state of the chain has it)
        c = states[2 * static_cast<size_t>(c)].z;
      }
      hard = l != level || level == kLastLevel;
    }
    const int dtok = take ? at : f.w;
    const bool barred = SEL == 2 && !hard && dtok == f.label;  // the rule bars the previous label
    if (mine) {
      f.decided = true;
      f.hard = !kept && (hard || barred);
      f.tok = kept ? f.v0 : dtok;
      f.val = kept ? f.x0 : take ? am : M;
      f.moves = !kept && (!take || by_arc);
      f.next = f.moves ? next : f.s;
      if (f.moves) f.moving = dtok;
    }
  }

  // Decides frames one after the other, the arcs of one on the lanes: the first of `wrong` (see misfits, `starts` and
  // `labels` are what it says) and those behind it until one was already decided from where this leads, then the next of
  // those that still do not fit.  Two dependent accesses a frame of up to 64 arcs, about 1.5 us, where carrying the starts
  // on and deciding them side by side takes about ten, however few they are: this is for the few.  Bounded by the
  // instructions of one wave: requesting several turns of arcs together made it slower.  Returns the frame that it stops at
  // because its chain has more than four states, a bit, or 0.
  __device__ __forceinline__ u64 follow(WalkFrame& f, u64 wrong, int starts, int labels, int lo, int hi, int from,
                                        int from_label) const {
    // (the records of where the winners lead from the root)
    const v4i *rec0 = reinterpret_cast<const v4i*>(root_rec + f.w);
    const v4i ra = ((const v4i PB_AS1*)rec0)[0], rb = ((const v4i PB_AS1*)rec0)[1];
    int l = first_lane(wrong);
    int s = lane_i(starts, l), label = lane_i(labels, l);
    Cursor cur = cursor_at(t, s);
#pragma unroll 1
    for (;;) {
      const int w = lane_i(f.w, l), v0 = lane_i(f.v0, l), target = lane_i(f.target, l);
      const float x0 = lane_f(f.x0, l);
      const bool kept = SEL != 0 && (v0 == t.blank || (SEL == 2 && v0 == label));
      int tok = v0, next = s, from_arc = -1;
      bool moves = false, hard = false, by_root = false;
      float val = x0;
      v4i k0 = {0, 0, 0, 0}, k1 = k0;  // the record of the state that this lane's first arc leads to
      float kp = 0.0f, ke = 0.0f;
      int kid = 0;
      if (!kept) {
        const float M = __fadd_rn(lane_f(f.xw, l), __fmul_rn(alpha, __fadd_rn(cur.p_root, lane_f(f.rsw, l))));
        hard = lane_i(f.marked ? 1 : 0, l) != 0 || M == -INFINITY;
        float am = -INFINITY;
        int at = INT_MAX;
        bool overridden = false, by_arc = false;
        if (!hard && s != 0) {
          // ---- four levels of the chain, deepest state first ----------------------------------------------------------
          const Rec none{0, 0, 0, 0.0f};
          const Rec r1 = cur.rec.fail != 0 ? cur.rec1 : none;
          Rec2 r{none, none};
          if (r1.fail != 0) r = load_rec2(t, r1.fail);
          if (r.a.fail == 0) r.b = none;
          const int c0 = cur.rec.count, c1 = c0 + r1.count, c2 = c1 + r.a.count, total = c2 + r.b.count;
          if (r.b.fail != 0) {  // (a longer chain)
            if (lane == l) {
              f.s = s;
              f.label = label;
              f.decided = false;
            }
            return 1ull << l;
          }
          const float p1 = __fadd_rn(0.0f, cur.rec.backoff), p2 = __fadd_rn(p1, r1.backoff), p3 = __fadd_rn(p2, r.a.backoff);
          int low = INT_MAX, to = 0, a_tok = -1, a_lv = 0;  // this lane's best: token and level, target; its first arc
          float v = -INFINITY;
          bool hit = false;
#pragma unroll 1
          for (int j0 = 0; j0 < total; j0 += 64) {
            const int j = j0 + lane;
            const int lv = (j >= c0 ? 1 : 0) + (j >= c1 ? 1 : 0) + (j >= c2 ? 1 : 0);
            if (j < total) {
              const int i = lv == 0 ? cur.rec.begin + j : lv == 1 ? r1.begin + j - c0 : lv == 2 ? r.a.begin + j - c1 : r.b.begin + j - c2;
              const float p = lv == 0 ? 0.0f : lv == 1 ? p1 : lv == 2 ? p2 : p3;
              const v2i a = arc[i];
              const float xa = hyp[static_cast<int64_t>(l) * frame_stride + a.x];
              if (j0 == 0) {
                k0 = states[2 * static_cast<size_t>(i + 1)];
                k1 = states[2 * static_cast<size_t>(i + 1) + 1];
                kp = p_root[i + 1];
                if (t.eos >= 0) ke = eos_score[i + 1];
                kid = i + 1;
                a_tok = a.x;
                a_lv = lv;
              }
              const float fa = __fadd_rn(xa, __fmul_rn(alpha, __fadd_rn(p, __int_as_float(a.y))));
              const int code = a.x << 2 | lv;
              const bool up = fa > v || (fa == v && code < low);
              v = up ? fa : v;
              low = up ? code : low;
              to = up ? i + 1 : to;
              hit = hit || a.x == w;
            }
            together();
          }
          // the largest value, the lowest token of that, its deepest state
          const float top = ukey_val(wave_max_u(low != INT_MAX ? ukey(v) : 0u));
          const bool best = low != INT_MAX && v == top;
          const int first = wave_min_nn(best ? low : INT_MAX);
          const u64 who = __ballot(best && low == first);
          overridden = __ballot(hit) != 0;
          if (who != 0) {
            from_arc = first_lane(who);
            am = lane_f(v, from_arc);
            at = first >> 2;
            by_arc = true;
            next = lane_i(to, from_arc);
            // (a deeper state has the token too, with a lower value: another token may win)
            const int lv = first & 3;
            hard = __ballot(a_tok == at && a_lv < lv) != 0;
            if (total > 64 && lv > 0)
              hard = hard || child(s, at) != 0 || (lv > 1 && child(cur.rec.fail, at) != 0) || (lv > 2 && child(r1.fail, at) != 0);
          }
        }
        auto special = [&](int token, float fv) {
          if (fv > am || (fv == am && token < at)) {
            am = fv;
            at = token;
            by_arc = false;
          }
        };
        if (SEL == 0 && t.blank >= 0) special(t.blank, __fadd_rn(x0, __fmul_rn(alpha, 0.0f)));
        if (t.eos >= 0) special(t.eos, __fadd_rn(lane_f(f.xe, l), __fmul_rn(alpha, cur.eos_boost)));
        const bool take = at != INT_MAX && (am > M || (am == M && at <= w));
        by_arc = by_arc && take;
        by_root = !take;
        hard = hard || (overridden && !take);
        tok = take ? at : w;
        hard = hard || (SEL == 2 && tok == label);
        val = take ? am : M;
        moves = by_root || by_arc;
        next = by_arc ? next : by_root ? target : s;
        if (!by_arc) from_arc = -1;
      }
      if (lane == l) {
        f.s = s;
        f.label = label;
        f.decided = true;
        f.hard = hard;
        f.tok = tok;
        f.val = val;
        f.moves = moves;
        f.next = next;
        if (moves) f.moving = tok;
      }
      together();
      // ---- on to the next frame ----------------------------------------------------------------------------------------
      s = next;
      label = tok;
      if (++l >= hi) return 0;
      const bool fits = lane_i(f.decided ? 1 : 0, l) != 0 && lane_i(f.s, l) == s && (SEL != 2 || lane_i(f.label, l) == label);
      if (fits) {
        wrong = misfits(f, lo, hi, from, from_label, starts, labels);
        if (wrong == 0) return 0;
        l = first_lane(wrong);
        s = lane_i(starts, l);
        label = lane_i(labels, l);
        cur = cursor_at(t, s);
      } else if (from_arc >= 0 && lane_i(kid, from_arc) != s) {
        cur = cursor_at(t, s);
      } else if (from_arc >= 0) {
        cur = Cursor{s, Rec{lane_i(k0.x, from_arc), lane_i(k0.y, from_arc), lane_i(k0.z, from_arc), __int_as_float(lane_i(k0.w, from_arc))},
                     Rec{lane_i(k1.x, from_arc), lane_i(k1.y, from_arc), lane_i(k1.z, from_arc), __int_as_float(lane_i(k1.w, from_arc))},
                     lane_f(kp, from_arc), lane_f(ke, from_arc)};
      } else if (by_root) {
        const int q = l - 1;
        cur = Cursor{s, Rec{lane_i(ra.y, q), lane_i(ra.z, q), lane_i(ra.w, q), __int_as_float(lane_i(rb.x, q))}, Rec{0, 0, 0, 0.0f},
                     __int_as_float(lane_i(rb.y, q)), __int_as_float(lane_i(rb.z, q))};
      }
    }
  }

  // A frame from state q.s by a pass over its row, any case, a share of it: part of `parts` waves.  Tokens that a chain
  // state has an arc on are marked, deepest state first, by wave 0 of them, the others follow with their base boosts.
  // Every wave of the workgroup gets here as often, with or without a row: several waves meet at barriers.
  __device__ __forceinline__ WalkBest row_pass(const WalkJob& q, const float* row, unsigned* tags, bool active, int part,
                                               int parts) const {
    WalkBest o{-INFINITY, INT_MAX, -1};
    auto offer = [&](int tk, float v, int next) {
      const bool take = v > o.val || (v == o.val && tk < o.tok);
      o.val = take ? v : o.val;
      o.tok = take ? tk : o.tok;
      o.child = take ? next : o.child;
    };
    auto meet = [&]() {
      if (parts > 1)
        __syncthreads();
      else
        together();
    };
    if (active)
      for (int i = 64 * part + lane; i < (t.V + 31) / 32; i += 64 * parts) tags[i] = 0u;
    meet();
    if (active && part == 0) {
      float p = 0.0f;
#pragma unroll 1
      for (int x = q.s; x != 0;) {
        const Rec r = load_rec(t, x);
#pragma unroll 1
        for (int j = lane; j < r.count; j += 64) {  // (tokens of one state are distinct: no two lanes meet on a mark)
          const v2i a = arc[r.begin + j];
          if (!tag_test(tags, a.x)) {
            tag_set(tags, a.x);
            if (SEL != 2 || a.x != q.excl)
              offer(a.x, __fadd_rn(row[a.x], __fmul_rn(alpha, __fadd_rn(p, __int_as_float(a.y)))), r.begin + j + 1);
          }
        }
        p = __fadd_rn(p, r.backoff);
        x = uniform_i(r.fail);
        together();
      }
      // the blank (single-stage rule: boost 0, state kept) and the EOS token (boost tabulated per state, state kept)
      if (SEL == 0 && t.blank >= 0 && lane == 0) offer(t.blank, __fadd_rn(row[t.blank], __fmul_rn(alpha, 0.0f)), -1);
      if (t.eos >= 0 && lane == 0 && (SEL != 2 || t.eos != q.excl))
        offer(t.eos, __fadd_rn(row[t.eos], __fmul_rn(alpha, t.eos_score[q.s])), -1);
    }
    meet();
    if (active) {
      const float pr = t.p_root[q.s];
      constexpr int kAhead = 4;
#pragma unroll 1
      for (int v0 = 64 * kAhead * part; v0 < t.V; v0 += 64 * kAhead * parts) {
        float x[kAhead], rs[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
          const int v = min(v0 + 64 * i + lane, t.V - 1);
          x[i] = row[v];
          rs[i] = root_score[v];
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
          const int v = v0 + 64 * i + lane;
          const bool in = v < t.V && v != t.blank && v != t.eos && (SEL != 2 || v != q.excl) && !tag_test(tags, min(v, t.V - 1));
          if (in) offer(v, __fadd_rn(x[i], __fmul_rn(alpha, __fadd_rn(pr, rs[i]))), -1);
        }
        together();
      }
      o = best_of(o);
    }
    return o;
  }
  // The best of the lanes' candidates (tok == INT_MAX: none), in every lane.
  __device__ __forceinline__ static WalkBest best_of(const WalkBest& o) {
    const float best = ukey_val(wave_max_u(o.tok != INT_MAX ? ukey(o.val) : 0u));
    const bool mine = o.tok != INT_MAX && o.val == best;  // (zeros of both signs are equal)
    const int tok = wave_min_nn(mine ? o.tok : INT_MAX);
    const u64 who = __ballot(mine && o.tok == tok);
    const int from = who != 0 ? first_lane(who) : 0;
    return WalkBest{lane_f(o.val, from), tok, lane_i(o.child, from)};
  }

  template <int CTRL, int ROWS>
  __device__ __forceinline__ static int from_lane(int v) {  // 0 where there is no such lane
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
  }
  // Sum of the lanes up to this one.
  __device__ __forceinline__ static int prefix_sum(int v) {
    v += from_lane<0x111, 0xf>(v);  // row_shr:1
    v += from_lane<0x112, 0xf>(v);  // row_shr:2
    v += from_lane<0x114, 0xf>(v);  // row_shr:4
    v += from_lane<0x118, 0xf>(v);  // row_shr:8
    v += from_lane<0x142, 0xa>(v);  // row_bcast:15
    v += from_lane<0x143, 0xc>(v);  // row_bcast:31
    return v;
  }
  // Largest value of the lanes up to this one (values >= 0).
  __device__ __forceinline__ static int prefix_max(int v) {
    v = max(v, from_lane<0x111, 0xf>(v));
    v = max(v, from_lane<0x112, 0xf>(v));
    v = max(v, from_lane<0x114, 0xf>(v));
    v = max(v, from_lane<0x118, 0xf>(v));
    v = max(v, from_lane<0x142, 0xa>(v));
    v = max(v, from_lane<0x143, 0xc>(v));
    return v;
  }
  __device__ __forceinline__ static int lane_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
  __device__ __forceinline__ static float lane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
  }
};

// The first frame that the lanes of a wave with frames f0 .. f1 - 1 hold: the last few before f0 tell what state those start
// in.
constexpr int kWalkLook = 16;
__device__ __forceinline__ int first_held(int f0, int f1) { return max(max(f0 - kWalkLook, f1 - 64), 0); }

template <int SEL>
__global__ void __launch_bounds__(1024) walk_kernel(DeviceTree dt, TreePick pick, const float* __restrict__ logp,
                                                    int64_t frame_stride, int64_t row_stride,
                                                    const int32_t* __restrict__ states0,
                                                    const int32_t* __restrict__ last0, float alpha, int T, int B, int side,
                                                    int32_t* tokens, int32_t* states, float* __restrict__ scores) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int b = blockIdx.x;
  DeviceTree mine = dt;
  const bool tree_ok = pick_tree(pick, b, mine);
  const TreeView t = make_view(mine);
  // (the frames of the first block are requested with the state, not behind it)
  const int wave_end = static_cast<int>(static_cast<int64_t>(wave + 1) * min(64 * nwaves, T) / nwaves);
  const int my_frame = first_held(static_cast<int>(static_cast<int64_t>(wave) * min(64 * nwaves, T) / nwaves), wave_end) + lane;
  int w_first = 0, v0_first = 0;
  if (my_frame < wave_end) {
    w_first = tokens[static_cast<size_t>(my_frame) * B + b];
    if (t.V > kPackedV) v0_first = states[static_cast<size_t>(my_frame) * B + b];
  }
  int s = tree_ok ? uniform_i(states0[b]) : -1;  // an unknown tree marks the hypothesis like an invalid state
  int last = SEL == 2 && last0 != nullptr ? uniform_i(last0[b]) : -1;
  if (!tree_ok || !valid_state(t, s)) {
    for (int f = threadIdx.x; f < T; f += blockDim.x) {
      const size_t o = static_cast<size_t>(f) * B + b;
      tokens[o] = -1;
      states[o] = -1;
      scores[o] = NAN;
    }
    return;
  }
  WalkLds* shared = reinterpret_cast<WalkLds*>(lds);
  WalkShared& W = *reinterpret_cast<WalkShared*>(shared + nwaves);
  const int tag_words = (t.V + 31) / 32;
  unsigned* tags = reinterpret_cast<unsigned*>(&W + 1);  // a bit per token, for each of `side` rows
  for (int F0 = 0; F0 < T; F0 += 64 * nwaves) {
    // A wave's frames f0 .. f1 - 1 are its last lanes; those before hold the frames before, from which the state that
    // its own start in is found.
    const int count = min(64 * nwaves, T - F0);
    const int f0 = static_cast<int>(static_cast<int64_t>(wave) * count / nwaves);
    const int f1 = static_cast<int>(static_cast<int64_t>(wave + 1) * count / nwaves);
    const int base = first_held(f0, f1), lo = f0 - base, hi = f1 - base, fr = base + lane;
    const Walker<SEL> walk{t, (const v4i PB_AS1*)mine.state, (const v2i PB_AS1*)mine.arc,
                           arc_table_of(mine), arc_slots(mine.num_states) - 1,
                           (const int PB_AS1*)mine.root_next, mine.root_rec,
                           (const float PB_AS1*)mine.p_root, (const float PB_AS1*)mine.eos_score, (const float PB_AS1*)mine.root_score,
                           logp + static_cast<int64_t>(F0 + base) * frame_stride + static_cast<int64_t>(b) * row_stride,
                           frame_stride, alpha, shared[wave], lane};
    WalkFrame f{};
    const size_t o = static_cast<size_t>(F0 + fr) * B + b;
    if (lane < hi) {
      int word = w_first, word2 = v0_first;
      if (F0 > 0) {
        word = tokens[o];
        word2 = t.V > kPackedV ? states[o] : 0;
      }
      get_winners(t.V, word, word2, f.w, f.v0, f.marked);
      f.moves = f.v0 != t.blank;
      if (SEL == 0 || f.moves) f.target = walk.root_next[f.w];
      if (lane >= lo) {
        const float* row = walk.hyp + static_cast<int64_t>(lane) * frame_stride;
        if (SEL == 0 || f.moves) {
          f.xw = row[f.w];
          f.rsw = walk.root_score[f.w];
        }
        f.x0 = SEL != 0 ? row[f.v0] : (t.blank >= 0 ? row[t.blank] : 0.0f);
        f.xe = t.eos >= 0 ? row[t.eos] : 0.0f;
      }
      f.s = -1;
      f.tok = f.moves ? f.w : f.v0;
      f.moving = f.w;
      f.next = f.target;
    }
    // First the states that the winners alone lead to, then the frames' decisions from there.  What does not fit then is
    // carried on and decided again once -- behind a surprise the winners are mostly right again -- and after that, where it
    // is few frames, one after the other: where most frames surprise the winners (log-depth weights, alpha = 1, phrases
    // without blanks) carrying on further was 1.6 .. 2.7 times as slow (V = 1025, 250 x 16, CTC rule 221 -> 116 us; V = 512,
    // 250 x 8 194 -> 89), without the second turn runs inside phrases of few tokens were (V = 1024, 500 x 4 52 -> 87).
    int from = base == 0 ? s : 0, from_label = base == 0 ? last : -1;
    for (int carries = 0;;) {
      int starts = 0, labels = 0;
      const u64 wrong = carries > 0 ? walk.misfits(f, lo, hi, from, from_label, starts, labels) : ~0ull;
      if (wrong != 0) {
        u64 need;
        if (carries < 2 || __builtin_popcountll(wrong) > kWalkFollow) {
          walk.settle_starts(f, carries > 0 ? lo : 0, hi, from, from_label);
          if (carries == 0 && lo > 0) {
            from = Walker<SEL>::lane_i(f.next, lo - 1);
            from_label = Walker<SEL>::lane_i(f.tok, lo - 1);
          }
          ++carries;
          need = __ballot(lane >= lo && lane < hi && !f.decided);
        } else {
          need = walk.follow(f, wrong, starts, labels, lo, hi, from, from_label);
        }
        if (need != 0) walk.decide_frames(f, need);
        continue;
      }
      int end = Walker<SEL>::lane_i(f.next, max(hi - 1, 0)), end_label = Walker<SEL>::lane_i(f.tok, max(hi - 1, 0));
      if (lo == hi) {
        end = from;
        end_label = from_label;
      }
      const u64 hard = __ballot(lane >= lo && lane < hi && f.hard);
      if (lane == 0) {
        W.end[wave] = end;
        W.end_label[wave] = end_label;
        W.hard[wave] = __builtin_popcountll(hard);
      }
      __syncthreads();
      bool changed = false;
      if (wave > 0) {
        const int have = uniform_i(W.end[wave - 1]), have_label = uniform_i(W.end_label[wave - 1]);
        changed = have != from || (SEL == 2 && have_label != from_label);
        from = have;
        from_label = have_label;
      }
      const int upto = Walker<SEL>::prefix_sum(lane < nwaves ? W.hard[lane] : 0);
      const int total = Walker<SEL>::lane_i(upto, 63), own = wave > 0 ? Walker<SEL>::lane_i(upto, wave - 1) : 0;
      if (__syncthreads_or(changed)) continue;  // (wave k starts where it should after k rounds at the latest)
      if (total == 0) break;  // (frames that need their row wait until the starts agree)
      // ---- what the winners do not settle: passes over the rows, in the order of the frames, several side by side -------
      // (The label is barred from the start: where it would not win, barring it changes nothing.)
      const int at = own + __builtin_popcountll(hard & ((1ull << lane) - 1));
      const bool listed = ((hard >> lane) & 1) && at < kWalkJobs;
      if (listed) W.job[at] = WalkJob{f.s, fr, SEL == 2 ? f.label : -1};
      __syncthreads();
      const int jobs = min(total, kWalkJobs);
#pragma unroll 1
      for (int i = 0; i < jobs; i += side) {
        const int n = min(jobs - i, side), parts = nwaves / n, which = wave / parts;
        WalkJob q = W.job[i + min(which, n - 1)];
        q.s = uniform_i(q.s);
        q.frame = uniform_i(q.frame);
        q.excl = uniform_i(q.excl);
        const WalkBest o = walk.row_pass(q, walk.hyp + static_cast<int64_t>(q.frame - base) * frame_stride,
                                         tags + min(which, n - 1) * tag_words, which < n, wave - which * parts, parts);
        if (lane == 0) W.part[wave] = o;
        __syncthreads();
        if (listed && at >= i && at < i + n) {
          WalkBest best = W.part[(at - i) * parts];
#pragma unroll 1
          for (int k = 1; k < parts; ++k) {
            const WalkBest p = W.part[(at - i) * parts + k];
            if (p.tok != INT_MAX && (best.tok == INT_MAX || p.val > best.val || (p.val == best.val && p.tok < best.tok))) best = p;
          }
          if (best.tok == INT_MAX) best = WalkBest{0.0f, 0, -1};  // (a row of NaN, a precondition violation: stay in range)
          const bool stays = best.child < 0 && (best.tok == t.blank || best.tok == t.eos);
          f.hard = false;
          f.tok = best.tok;
          f.val = best.val;
          f.moves = !stays;
          f.next = best.child >= 0 ? best.child : stays ? f.s : walk.root_next[best.tok];
          if (!stays) f.moving = best.tok;
        }
        __syncthreads();  // (the next ones' marks and parts take the place of these)
      }
    }
    s = uniform_i(W.end[nwaves - 1]);
    last = uniform_i(W.end_label[nwaves - 1]);
    if (lane >= lo && lane < hi) {
      tokens[o] = f.tok;
      states[o] = f.next;
      scores[o] = f.val;
    }
    if (F0 + count < T) __syncthreads();  // (the next block's ends take the place of these)
  }
}

int g_walk_max_lds = 63 * 1024;  // dynamic LDS the device allows the walk kernel, set once

size_t walk_lds_bytes(int V, int waves, int side) {
  return static_cast<size_t>(waves) * sizeof(WalkLds) + sizeof(WalkShared) + side * sizeof(unsigned) * ((static_cast<size_t>(V) + 31) / 32);
}

}  // namespace

bool frames_rows_ok(const DeviceTree& t, int32_t T, int32_t B, int sel) {
  return t.p_root != nullptr && t.root_rec != nullptr && rows_pay(t.vocab_size, T, B, sel, t.num_states) &&
         walk_lds_bytes(t.vocab_size, 1, 1) <= static_cast<size_t>(g_walk_max_lds);
}

int launch_frames_rows(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                       int64_t row_stride, const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T,
                       int32_t B, int sel, int32_t* d_tokens, int32_t* d_states, float* d_scores, hipStream_t stream) {
  const int V = t.vocab_size;
  const int64_t rows = static_cast<int64_t>(T) * B;
  if (V <= kNarrowMaxV) {
    int64_t strips = (8192 + B - 1) / B;  // waves per hypothesis: two rounds of what the chip holds
    if (strips > T) strips = T;
    const int64_t blocks = (strips * B + 3) / 4;
#define PB_ROWS(NS, SEL)                                                                                                   \
  hipLaunchKernelGGL((rows_narrow_kernel<NS, SEL>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, t, pick,    \
                     d_logp, frame_stride, row_stride, alpha, T, B, static_cast<int>(strips), d_tokens, d_states)
#define PB_ROWS_SEL(NS) \
  if (sel == 0) {       \
    PB_ROWS(NS, 0);     \
  } else {              \
    PB_ROWS(NS, 1);     \
  }
    if (V <= 256) {
      PB_ROWS(4, 1);  // (CTC rule only)
    } else if (V <= 512) {
      PB_ROWS_SEL(8)
    } else if (V <= 1024) {
      PB_ROWS_SEL(16)
    } else {
      PB_ROWS_SEL(20)
    }
#undef PB_ROWS_SEL
#undef PB_ROWS
  } else {
    // Waves per row: one per eight chunks where the rows alone fill the chip, up to one per chunk where they do not.
    const int nch = (V + kChunk - 1) / kChunk;
    int waves = static_cast<int>((8192 + rows - 1) / rows);
    if (waves < (nch + 7) / 8) waves = (nch + 7) / 8;
    if (waves > nch) waves = nch;
    if (waves > 16) waves = 16;
    if (sel == 0)
      hipLaunchKernelGGL(rows_wide_kernel<0>, dim3(static_cast<unsigned>(rows)), dim3(64 * waves), 0, stream, t, pick, d_logp,
                         frame_stride, row_stride, alpha, B, d_tokens, d_states);
    else
      hipLaunchKernelGGL(rows_wide_kernel<1>, dim3(static_cast<unsigned>(rows)), dim3(64 * waves), 0, stream, t, pick, d_logp,
                         frame_stride, row_stride, alpha, B, d_tokens, d_states);
  }
  if (hipGetLastError() != hipSuccess) return PB_EHIP;
  // A wave takes 16 frames or more (those that it looks back over are read once more: 40 frames x 1 with 16 / 4 waves 13.0 /
  // 11.3 us, 60 x 48 21.9 / 18.2, V = 1025), at most 64 (1000 x 16 with 16 / 8 waves 42 / 56 us).
  int waves = T >= 256 ? 16 : (T + 15) / 16;
  const size_t room = static_cast<size_t>(g_walk_max_lds);
  while (waves > 1 && walk_lds_bytes(V, waves, 1) > room) --waves;
  // Rows that are passed over side by side: a wave each up to 4096 tokens, more waves to wider ones (V = 4096, 250 x 8,
  // log-probs of bf16 logits: one wave a row 45.9 us, four 48.2, all waves to one row after the other 49.8; V = 32001,
  // 100 x 16, CTC rule, where 7 waves take one row: 96 us and 100 with a wave each).
  int side = static_cast<int>(static_cast<int64_t>(waves) * 4096 / V);
  side = side < 1 ? 1 : side > waves ? waves : side;
  while (side > 1 && walk_lds_bytes(V, waves, side) > room) --side;
  const size_t lds = walk_lds_bytes(V, waves, side);
#define PB_WALK(SEL)                                                                                                     \
  hipLaunchKernelGGL(walk_kernel<SEL>, dim3(static_cast<unsigned>(B)), dim3(64 * waves), lds, stream, t, pick, d_logp,   \
                     frame_stride, row_stride, d_states0, d_last0, alpha, T, B, side, d_tokens, d_states, d_scores)
  if (sel == 0) {
    PB_WALK(0);
  } else if (sel == 1) {
    PB_WALK(1);
  } else {
    PB_WALK(2);
  }
#undef PB_WALK
  return hipGetLastError() == hipSuccess ? PB_OK : PB_EHIP;
}

int prepare_rows_kernels(int max_lds_bytes) {
  constexpr int kPlainLimit = 63 * 1024;  // static LDS of the kernel included
  int limit = kPlainLimit;
  if (max_lds_bytes > kPlainLimit + 1024) {
    const int bytes = max_lds_bytes - 1024;
    const hipFuncAttribute attr = hipFuncAttributeMaxDynamicSharedMemorySize;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(walk_kernel<0>), attr, bytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(walk_kernel<1>), attr, bytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(walk_kernel<2>), attr, bytes) == hipSuccess)
      limit = bytes;
    else
      (void)hipGetLastError();
  }
  g_walk_max_lds = limit;
  return PB_OK;
}

}  // namespace pb
