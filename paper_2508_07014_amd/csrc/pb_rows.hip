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
//  * Pass 2 (walk_kernel; one workgroup per hypothesis) runs the automaton on the winners: a wave per segment, from
//    the state the last winner before it leads to.  A frame gathers a handful of log-probs (winner, blank, the arcs
//    of the chain) instead of a row, and those of sixteen frames are requested at once for the states the winners lead
//    to.  Runs of frames whose outcomes fit together are taken over whole, the others -- inside a spoken phrase,
//    mostly -- are decided one after the other.  The outcomes sit in LDS; segments that started from a wrong guess are decoded again until they meet what
//    is there (equal state and label: equal future), in rounds between barriers.
//
// Between the passes the winners travel in the call's own outputs: tokens holds w (~w for a marked row), states the
// raw arg-max (single-stage rule: the blank where it wins under root boosts, else w), so the outputs must not overlap
// what pass 2 reads (frames_apart).
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

// ---- pass 1, rows of 1025 .. 64 * NS positions: a wave per row, root scores kept in registers -------------------------
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
    if (lane == 0) {
      const size_t o = static_cast<size_t>(f) * B + b;
      tokens[o] = marked ? ~w : w;
      states[o] = v0;
    }
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
  if (threadIdx.x == 0) {
    const size_t o = static_cast<size_t>(f) * B + b;
    tokens[o] = marked ? ~w : w;
    states[o] = v0;
  }
}

// ---- pass 2 --------------------------------------------------------------------------------------------------------------
constexpr int kWalkBlock = 1024;  // frames whose winners and outcomes sit in LDS at a time
constexpr int kWalkGroup = 16;    // frames whose arcs and log-probs are requested together
constexpr int kWalkLook = 64;     // frames a segment's guess may look back over (one per lane)

struct WalkLds {  // per block of frames; `tags` is this wave's
  int *w, *v0, *st, *tok;
  float* sc;
  unsigned* tags;
};

template <int SEL>
struct Walker {
  TreeView t;
  const float* hyp;  // logp of frame 0 of the block
  int64_t frame_stride;
  float alpha;
  WalkLds L;
  int tag_words, nch, lane;

  // The state and label a segment that begins at frame f0 > 0 is guessed to start from: the last winner that moves
  // the state (block_s: the state the block starts in, for a block that only keeps it).
  __device__ __forceinline__ void guess(int f0, int block_s, int& s, int& label) const {
    const int f = f0 - 1 - lane;
    const int v0 = f >= 0 ? L.v0[f] : 0, wm = f >= 0 ? L.w[f] : 0, w = wm < 0 ? ~wm : wm;
    bool moves = f >= 0 && v0 != t.blank;
    if (SEL == 2 && f >= 1) {  // a repeat of the label before it keeps the state
      const int pm = L.w[f - 1], pv = L.v0[f - 1];
      moves = moves && v0 != (pv == t.blank ? pv : (pm < 0 ? ~pm : pm)) && v0 != pv;
    }
    const u64 mask = __ballot(moves);
    if (mask != 0) {
      s = uniform_i(t.root_next[__builtin_amdgcn_readlane(SEL == 0 ? v0 : w, first_lane(mask))]);
    } else {
      s = f0 <= kWalkLook ? block_s : 0;
    }
    label = __builtin_amdgcn_readlane(SEL == 0 || !(mask & 1) ? v0 : w, 0);
  }

  // Decodes frames [f0, f1) of the block from (s, last).  COMPARE: stops at the frame that meets the stored outcome
  // and returns true; false when the end was reached.
  //   Frames are first decided side by side, a lane holding one, from the states the winners before them lead to; then
  //   runs of frames whose outcome is the state the next one was decided from are taken over whole, and what lies
  //   between them -- mostly inside a spoken phrase -- is decided frame by frame.  (Frame by frame throughout took
  //   about 1 us a frame, a chain of dependent reductions.)
  template <bool COMPARE>
  __device__ __forceinline__ bool run(int f0, int f1, int s, int last) const {
    Cursor cur = cursor_at(t, s);
#pragma unroll 1
    for (int fb = f0; fb < f1; fb += 64) {
      const int n = min(64, f1 - fb);
      // ---- one frame per lane: its winner and what the winner's value and target need --------------------------
      const int lf = fb + min(lane, n - 1);
      const float* lrow = hyp + static_cast<int64_t>(lf) * frame_stride;
      const int wm = L.w[lf], w = wm < 0 ? ~wm : wm, v0 = L.v0[lf];
      const int old_st = COMPARE ? L.st[lf] : 0, old_tok = COMPARE ? L.tok[lf] : 0;
      const float xw = lrow[w];
      const float x0 = SEL != 0 ? lrow[v0] : (t.blank >= 0 ? lrow[t.blank] : 0.0f);
      const float xe = t.eos >= 0 ? lrow[t.eos] : 0.0f;
      const float rsw = t.root_score[w];
      const v8i rr = reinterpret_cast<const v8i*>(root_rec)[w];
      int out_st = 0, out_tok = 0;
      float out_sc = 0.0f;
      Ahead g{};
      if constexpr (!COMPARE) g = decide_ahead(cur, last, fb, n, wm, w, v0, xw, x0, xe, rsw, rr);
      int met = -1;
#pragma unroll 1
      for (int l = 0; l < n && met < 0;) {
        if (!COMPARE && ((g.settled >> l) & 1) && cur.s == __builtin_amdgcn_readlane(g.s, l) &&
            (SEL != 2 || last == __builtin_amdgcn_readlane(g.label, l))) {
          const int e = min(n - 1, l + __builtin_ctzll(~(g.linked >> l)));  // (linked has no bit for the last lane)
          const bool in = lane >= l && lane <= e;
          out_st = in ? g.next : out_st;
          out_tok = in ? g.tok : out_tok;
          out_sc = in ? g.val : out_sc;
          const int kind = __builtin_amdgcn_readlane(g.kind, e);
          if (kind == kByArc) {
            cur = cursor_at(t, __builtin_amdgcn_readlane(g.next, e));
          } else if (kind == kByRoot) {
            cur = cursor_from_root_rec(lane_rec(rr, e));
          } else {
            cur = Cursor{__builtin_amdgcn_readlane(g.s, e), Rec{__builtin_amdgcn_readlane(g.begin, e),
                         __builtin_amdgcn_readlane(g.count, e), 0, 0.0f}, Rec{0, 0, 0, 0.0f}, lane_f(g.p_root, e),
                         lane_f(g.eos_boost, e)};
          }
          last = __builtin_amdgcn_readlane(g.tok, e);
          l = e + 1;
          continue;
        }
        const float* row = hyp + static_cast<int64_t>(fb + l) * frame_stride;
        const int fw = __builtin_amdgcn_readlane(w, l), fv0 = __builtin_amdgcn_readlane(v0, l);
        const float fx0 = lane_f(x0, l);
        FrameOut o{fx0, fv0, false, 0};
        if (SEL == 0 || (fv0 != t.blank && (SEL != 2 || fv0 != last))) {
          const bool marked = __builtin_amdgcn_readlane(wm, l) < 0;
          const float M = __fadd_rn(lane_f(xw, l), __fmul_rn(alpha, __fadd_rn(cur.p_root, lane_f(rsw, l))));
          Cursor child;
          bool child_known;
          o = decide(cur, row, M, fw, marked, fx0, lane_f(xe, l), last, child, child_known);
          if (o.arc) {
            cur = child_known ? child : cursor_at(t, o.child);
          } else if (o.tok == fw && fw != t.blank && fw != t.eos) {
            cur = cursor_from_root_rec(lane_rec(rr, l));
          } else if (o.tok != t.blank && o.tok != t.eos) {
            const v8i r = t.root_rec[o.tok];
            cur = cursor_from_root_rec(r);
          }
        }
        if (lane == l) {
          out_st = cur.s;
          out_tok = o.tok;
          out_sc = o.val;
        }
        last = o.tok;
        if (COMPARE && __builtin_amdgcn_readlane(old_st, l) == cur.s &&
            (SEL != 2 || __builtin_amdgcn_readlane(old_tok, l) == o.tok))
          met = l;  // (this frame is written too, its score may differ; the rest stands)
        ++l;
      }
      if (lane < (met >= 0 ? met + 1 : n)) {
        L.st[fb + lane] = out_st;
        L.tok[fb + lane] = out_tok;
        L.sc[fb + lane] = out_sc;
      }
      if (met >= 0) return true;
    }
    return false;
  }

  // Outcomes of a batch of frames, one per lane, each decided from the state the winners before it lead to.
  enum Kind { kKeep = 0, kByArc = 1, kByRoot = 2 };
  struct Ahead {
    u64 settled, linked;            // decided; and: the next frame is decided, from this frame's outcome
    int s, begin, count;            // the state it was decided from
    float p_root, eos_boost;
    int label;                      // ... and the label before it (CTC rule)
    int tok, next, kind;
    float val;
  };
  __device__ __forceinline__ Ahead decide_ahead(const Cursor& cur, int last, int fb, int n, int wm, int w, int v0, float xw,
                                                float x0, float xe, float rsw, const v8i& rr) const {
    Ahead g;
    // ---- where each frame starts: in the state the last moving frame before it leads to, else in the batch's own ----
    bool moves = v0 != t.blank;
    const int pv = __shfl_up(v0, 1), pw = __shfl_up(w, 1);
    if (SEL == 2) moves = moves && (lane == 0 ? v0 != last : v0 != pv && v0 != pw);
    const u64 before = __ballot(moves) & ((1ull << lane) - 1);
    const int src = before ? 63 - __builtin_clzll(before) : 0;
    g.s = __shfl(rr.s0, src);
    g.begin = __shfl(rr.s1, src);
    g.count = __shfl(rr.s2, src);
    g.p_root = __int_as_float(__shfl(rr.s5, src));
    g.eos_boost = __int_as_float(__shfl(rr.s6, src));
    bool settled = wm >= 0 && lane < n;
    if (!before) {
      g.s = cur.s;
      g.begin = cur.rec.begin;
      g.count = cur.rec.count;
      g.p_root = cur.p_root;
      g.eos_boost = cur.eos_boost;
      settled = settled && (cur.s == 0 || cur.rec.fail == 0);  // (one level of arcs: all that is looked at here)
    }
    if (g.s == 0) g.count = 0;  // (the root's arcs are the root row)
    // ---- the best arc of every frame's state: the arcs of a frame on the lanes, kWalkGroup frames at a time -----------
    float am = -INFINITY;
    int at = INT_MAX, ac = -1;
    bool overridden = false;
    const u64 with_arcs = __ballot(g.count > 0 && lane < n);
#pragma unroll 1
    for (int l0 = 0; l0 < n; l0 += kWalkGroup) {
      if (((with_arcs >> l0) & ((1ull << kWalkGroup) - 1)) == 0) continue;
      ArcRec arcs[kWalkGroup];
      float xa[kWalkGroup];
#pragma unroll
      for (int i = 0; i < kWalkGroup; ++i) {
        const int gb = __builtin_amdgcn_readlane(g.begin, l0 + i), gc = __builtin_amdgcn_readlane(g.count, l0 + i);
        arcs[i] = t.arc[gb + max(0, min(lane, gc - 1))];
      }
#pragma unroll
      for (int i = 0; i < kWalkGroup; ++i) {
        const int gc = __builtin_amdgcn_readlane(g.count, l0 + i);
        const float* row = hyp + static_cast<int64_t>(fb + min(l0 + i, n - 1)) * frame_stride;
        xa[i] = row[lane < gc ? arcs[i].token : 0];
      }
#pragma unroll
      for (int i = 0; i < kWalkGroup; ++i) {
        const int l = l0 + i, gb = __builtin_amdgcn_readlane(g.begin, l), gc = __builtin_amdgcn_readlane(g.count, l);
        const int fw = __builtin_amdgcn_readlane(w, l);
        float best = lane < gc ? __fadd_rn(xa[i], __fmul_rn(alpha, __fadd_rn(0.0f, arcs[i].score))) : -INFINITY;
        int tok = lane < gc ? arcs[i].token : INT_MAX, child = gb + lane + 1;
        bool hit = tok == fw;
        if (gc > 64) {  // uniform
          const float* row = hyp + static_cast<int64_t>(fb + min(l, n - 1)) * frame_stride;
#pragma unroll 1
          for (int j = 64 + lane; j < gc; j += 64) {
            const ArcRec a = t.arc[gb + j];
            hit = hit || a.token == fw;
            const float fa = __fadd_rn(row[a.token], __fmul_rn(alpha, __fadd_rn(0.0f, a.score)));
            if (fa > best) {  // (tokens ascend with j: an equal one stays behind)
              best = fa;
              tok = a.token;
              child = gb + j + 1;
            }
          }
        }
        const float top = ukey_val(wave_max_u(ukey(best)));
        u64 who = __ballot(best == top && tok != INT_MAX);
        if (gc > 64 && (who & (who - 1)) != 0) {  // equal ones in two lanes: the lower token need not be in the lower lane
          const int low = wave_min_nn(best == top ? tok : INT_MAX);
          who = __ballot(best == top && tok == low);
        }
        const int from = who != 0 ? first_lane(who) : 0;
        const bool any_hit = __ballot(hit) != 0;
        const int wtok = __builtin_amdgcn_readlane(tok, from), wchild = __builtin_amdgcn_readlane(child, from);
        if (lane == l && who != 0) {
          am = top;
          at = wtok;
          ac = wchild;
          overridden = any_hit;
        }
      }
    }
    // ---- the frames' decisions, as in decide(), one per lane ------------------------------------------------------------
    const float M = __fadd_rn(xw, __fmul_rn(alpha, __fadd_rn(g.p_root, rsw)));
    settled = settled && M != -INFINITY;
    auto special = [&](int token, float fv) {
      const bool take = fv > am || (fv == am && token < at);
      am = take ? fv : am;
      at = take ? token : at;
      ac = take ? -1 : ac;
    };
    if (SEL == 0 && t.blank >= 0) special(t.blank, __fadd_rn(x0, __fmul_rn(alpha, 0.0f)));
    if (t.eos >= 0) special(t.eos, __fadd_rn(xe, __fmul_rn(alpha, g.eos_boost)));
    const bool take = at != INT_MAX && (am > M || (!overridden && am == M && at < w));
    settled = settled && !(overridden && !take);
    const int dtok = take ? at : w;
    bool kept = false;
    g.tok = dtok;
    g.label = -1;
    if (SEL != 0) {
      kept = v0 == t.blank;
      g.tok = kept ? v0 : dtok;
      if (SEL == 2) {
        // repeats depend on the labels before them: taken from the outcomes without repeats, then checked
        int prev = __shfl_up(g.tok, 1);
        prev = lane == 0 ? last : prev;
        const bool repeat = v0 == prev;
        g.tok = kept || repeat ? v0 : dtok;
        prev = __shfl_up(g.tok, 1);
        g.label = lane == 0 ? last : prev;
        const bool blank_frame = kept;
        kept = kept || repeat;
        // (a frame whose repeat this gets wrong, or whose token the rule bars, is decided frame by frame)
        settled = kept ? lane < n && (blank_frame || repeat == (v0 == g.label))
                       : settled && v0 != g.label && dtok != g.label;
      } else if (kept) {
        settled = lane < n;
      }
    }
    g.val = kept ? x0 : take ? am : M;
    g.kind = kept ? kKeep : take ? (ac >= 0 ? kByArc : kKeep) : kByRoot;
    g.next = g.kind == kByArc ? ac : g.kind == kByRoot ? rr.s0 : g.s;
    if (kept && !before && cur.s != 0 && cur.rec.fail != 0) settled = false;  // (its record is not a single level)
    g.settled = __ballot(settled);
    const int next_s = __shfl_down(g.s, 1);
    g.linked = __ballot(g.next == next_s && lane + 1 < n) & (g.settled >> 1);
    return g;
  }

  const RootRec* root_rec;  // (of the tree, for accesses that differ from lane to lane)
  const StateRec* states;
  const float *p_root, *eos_score;

  __device__ __forceinline__ static Rec lane_half(const v4i& r, int l) {
    return Rec{__builtin_amdgcn_readlane(r.x, l), __builtin_amdgcn_readlane(r.y, l), __builtin_amdgcn_readlane(r.z, l),
               __int_as_float(__builtin_amdgcn_readlane(r.w, l))};
  }
  __device__ __forceinline__ static float lane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
  }
  __device__ __forceinline__ static v8i lane_rec(const v8i& r, int l) {
    v8i o;
    o.s0 = __builtin_amdgcn_readlane(r.s0, l);
    o.s1 = __builtin_amdgcn_readlane(r.s1, l);
    o.s2 = __builtin_amdgcn_readlane(r.s2, l);
    o.s3 = __builtin_amdgcn_readlane(r.s3, l);
    o.s4 = __builtin_amdgcn_readlane(r.s4, l);
    o.s5 = __builtin_amdgcn_readlane(r.s5, l);
    o.s6 = __builtin_amdgcn_readlane(r.s6, l);
    o.s7 = 0;
    return o;
  }

  // One frame from state cur whose base winner is w with value M (marked: not certain, see near_band).
  //   x_blank, x_eos: log-probs of those columns
  //   An arc's target comes back in `child` when `child_known` (o.arc): its record is requested with the log-probs of
  //   the arcs, so that following a phrase costs no access of its own.
  __device__ __forceinline__ FrameOut decide(const Cursor& cur, const float* row, float M, int w, bool marked, float x_blank,
                                             float x_eos, int last, Cursor& child, bool& child_known) const {
    const Rec rec0 = cur.rec;
    const bool chain = cur.s != 0, multi = chain && rec0.fail != 0;
    float bf = -INFINITY;
    int btok = INT_MAX, bchild = 0;
    bool hit = false;
    bool settled = !marked && M != -INFINITY;
    v4i kid0 = {0, 0, 0, 0}, kid1 = kid0;  // the record of this lane's first arc's target
    float kid_p = 0.0f, kid_e = 0.0f;
    int kid = -1;
    if (settled && chain) {
      // The first four levels of the chain (two records) as one list of arcs, deepest state first: their arcs and
      // their log-probs are two accesses, however many levels there are.
      const Rec none{0, 0, 0, 0.0f};
      const Rec r1 = multi ? cur.rec1 : none;
      Rec2 r23{none, none};
      if (multi && r1.fail != 0) r23 = load_rec2(t, r1.fail);
      if (r23.a.fail == 0) r23.b = none;
      const int c0 = rec0.count, c1 = c0 + r1.count, c2 = c1 + r23.a.count, total = c2 + r23.b.count;
      const float p1 = __fadd_rn(0.0f, rec0.backoff), p2 = __fadd_rn(p1, r1.backoff), p3 = __fadd_rn(p2, r23.a.backoff);
      auto consider = [&](int tk, float score, float xv, float p, int next, bool valid, bool shadowed) {
        hit = hit || (valid && tk == w);
        const float fa = __fadd_rn(xv, __fmul_rn(alpha, __fadd_rn(p, score)));
        const bool take = valid && !shadowed && (fa > bf || (fa == bf && tk < btok));
        bf = take ? fa : bf;
        btok = take ? tk : btok;
        bchild = take ? next : bchild;
      };
#pragma unroll 1
      for (int j0 = 0; j0 < total; j0 += 64) {
        const int i = j0 + lane;
        const bool valid = i < total;
        const int lv = (i >= c0 ? 1 : 0) + (i >= c1 ? 1 : 0) + (i >= c2 ? 1 : 0);
        const int at = i < c0 ? rec0.begin + i : i < c1 ? r1.begin + i - c0 : i < c2 ? r23.a.begin + i - c1 : r23.b.begin + i - c2;
        const ArcRec a = t.arc[valid ? at : rec0.begin];
        const int tk = valid ? a.token : 0;  // an unused entry may hold anything: keep the indices in range
        const float xv = row[tk];
        if (j0 == 0) {
          kid = valid ? at + 1 : 0;
          const StateRec* k = states + kid;
          kid0 = reinterpret_cast<const v4i*>(k)[0];
          kid1 = reinterpret_cast<const v4i*>(k)[1];
          kid_p = p_root[kid];
          if (t.eos >= 0) kid_e = eos_score[kid];
        }
        bool shadowed = false;
        if (multi) {  // a deeper chain state owns its tokens (the marks are all clear between frames)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (valid && lv == q) {
              if (q > 0) shadowed = tag_test(L.tags, tk);
              tag_set(L.tags, tk);
            }
          }
        }
        consider(tk, a.score, xv, lv == 0 ? 0.0f : lv == 1 ? p1 : lv == 2 ? p2 : p3, at + 1, valid, shadowed);
      }
      float p = __fadd_rn(p3, r23.b.backoff);
#pragma unroll 1
      for (int x = r23.b.fail; x != 0;) {  // longer chains, level by level
        const Rec r = load_rec(t, x);
#pragma unroll 1
        for (int j = lane; j < r.count; j += 64) {
          const ArcRec a = t.arc[r.begin + j];
          const bool shadowed = tag_test(L.tags, a.token);
          tag_set(L.tags, a.token);
          consider(a.token, a.score, row[a.token], p, r.begin + j + 1, true, shadowed);
        }
        p = __fadd_rn(p, r.backoff);
        x = uniform_i(r.fail);
      }
      if (multi) tags_clear_n(L.tags, tag_words, lane);
    }
    child_known = false;
    // the blank (single-stage rule: boost 0, state kept) and the EOS token (boost tabulated per state, state kept)
    if (SEL == 0 && t.blank >= 0 && lane == 63) {
      const float fv = __fadd_rn(x_blank, __fmul_rn(alpha, 0.0f));
      const bool take = fv > bf || (fv == bf && t.blank < btok);
      bf = take ? fv : bf;
      btok = take ? t.blank : btok;
      bchild = take ? -1 : bchild;
    }
    if (t.eos >= 0 && lane == 62) {
      const float fv = __fadd_rn(x_eos, __fmul_rn(alpha, cur.eos_boost));
      const bool take = fv > bf || (fv == bf && t.eos < btok);
      bf = take ? fv : bf;
      btok = take ? t.eos : btok;
      bchild = take ? -1 : bchild;
    }
    FrameOut o{M, w, false, 0};
    const bool mine0 = btok != INT_MAX;
    if (settled && __ballot(mine0) != 0) {
      const float MA = ukey_val(wave_max_u(mine0 ? ukey(bf) : 0u));
      const bool overridden = __ballot(hit) != 0;
      if (overridden || MA >= M) {
        const bool mine = mine0 && bf == MA;
        const int va = wave_min_nn(mine ? btok : INT_MAX);
        const int next = __builtin_amdgcn_readlane(bchild, first_lane(__ballot(mine && btok == va)));
        if (MA > M || (!overridden && MA == M && va < w)) {
          o = FrameOut{MA, va, next >= 0, next};
          const u64 holds = __ballot(kid == next && next > 0);
          if (holds != 0) {
            const int q = first_lane(holds);
            child = Cursor{next, lane_half(kid0, q), lane_half(kid1, q), lane_f(kid_p, q), lane_f(kid_e, q)};
            child_known = true;
          }
        } else if (overridden) {
          settled = false;  // the base winner is shadowed by an arc that does not beat it
        }
      }
    }
    if (settled && SEL == 2 && o.tok == last) settled = false;  // the CTC rule bars the previous label
    if (!settled) {
      child_known = false;
      // (CTC: first without the exclusion -- the label may not even win -- then, if it does win, without the label)
      o = slow_frame<false, SEL>(t, cur, row, alpha, -1, L.tags, tag_words, nch, lane);
      if (SEL == 2 && o.tok == last) o = slow_frame<false, SEL>(t, cur, row, alpha, last, L.tags, tag_words, nch, lane);
      tags_clear_n(L.tags, tag_words, lane);
    }
    o.val = uniform_f(o.val);
    o.tok = uniform_i(o.tok);
    o.child = uniform_i(o.child);
    return o;
  }
};

template <int SEL>
__global__ void __launch_bounds__(1024) walk_kernel(DeviceTree dt, TreePick pick, const float* __restrict__ logp,
                                                    int64_t frame_stride, int64_t row_stride,
                                                    const int32_t* __restrict__ states0,
                                                    const int32_t* __restrict__ last0, float alpha, int T, int B,
                                                    int32_t* tokens, int32_t* states, float* __restrict__ scores) {
  extern __shared__ int lds[];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int b = blockIdx.x;
  DeviceTree mine = dt;
  const bool tree_ok = pick_tree(pick, b, mine);
  const TreeView t = make_view(mine);
  const RootRec* root_rec = mine.root_rec;
  const StateRec* state_recs = mine.state;
  const float *p_root = mine.p_root, *eos_score = mine.eos_score;
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
  const int nch = (t.V + kChunk - 1) / kChunk, tag_words = nch * kTagWords, cap = min(T, kWalkBlock);
  WalkLds L;
  L.w = lds;
  L.v0 = lds + cap;
  L.st = lds + 2 * cap;
  L.tok = lds + 3 * cap;
  L.sc = reinterpret_cast<float*>(lds + 4 * cap);
  L.tags = reinterpret_cast<unsigned*>(lds + 5 * cap) + wave * tag_words;
  tags_clear_n(L.tags, tag_words, lane);
  for (int F0 = 0; F0 < T; F0 += kWalkBlock) {
    const int n = min(kWalkBlock, T - F0);
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const size_t o = static_cast<size_t>(F0 + i) * B + b;
      L.w[i] = tokens[o];
      L.v0[i] = states[o];
    }
    __syncthreads();
    const Walker<SEL> walk{t, logp + static_cast<int64_t>(F0) * frame_stride + static_cast<int64_t>(b) * row_stride,
                           frame_stride, alpha, L, tag_words, nch, lane, root_rec, state_recs, p_root, eos_score};
    const int f0 = static_cast<int>(static_cast<int64_t>(wave) * n / nwaves);
    const int f1 = static_cast<int>(static_cast<int64_t>(wave + 1) * n / nwaves);
    int from = s, from_tok = last;
    if (f0 > 0) walk.guess(f0, s, from, from_tok);
    if (f0 < f1) walk.template run<false>(f0, f1, from, from_tok);
    __syncthreads();
    for (;;) {  // (segment k is final after k rounds at the latest: the one before it then is)
      bool dirty = false;
      int have = from, have_tok = from_tok;
      if (f0 > 0 && f0 < f1) {
        have = uniform_i(L.st[f0 - 1]);
        have_tok = uniform_i(L.tok[f0 - 1]);
      }
      __syncthreads();  // (every outcome is read before any segment is decoded again)
      if (have != from || (SEL == 2 && have_tok != from_tok)) {
        from = have;
        from_tok = have_tok;
        dirty = !walk.template run<true>(f0, f1, from, from_tok);
      }
      if (!__syncthreads_or(dirty)) break;
    }
    s = uniform_i(L.st[n - 1]);
    last = uniform_i(L.tok[n - 1]);
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const size_t o = static_cast<size_t>(F0 + i) * B + b;
      tokens[o] = L.tok[i];
      states[o] = L.st[i];
      scores[o] = L.sc[i];
    }
    __syncthreads();  // (the next block overwrites what has just been read)
  }
}

int g_walk_max_lds = 63 * 1024;  // dynamic LDS the device allows the walk kernel, set once

size_t walk_lds_bytes(int V, int T, int waves) {
  const int cap = T < kWalkBlock ? T : kWalkBlock;
  return sizeof(int) * (static_cast<size_t>(5) * cap + static_cast<size_t>(waves) * ((V + kChunk - 1) / kChunk) * kTagWords);
}

}  // namespace

// Which calls the two passes are for.  Pass 1 reads the rows at the chip's rate whatever T and B are; pass 2 costs about
// 10 us and 0.5 to 1 us for every 16 frames of a hypothesis.  The segment decoders need some thousand segments for that
// rate and read again what a wrong guess has spoilt, but have no second pass over the frames.  Measured: time of the two
// passes over that of the segment decoder, mean over vocabularies, rules and kinds of rows (random; a fifth of the frames
// inside listed phrases; the same with half of the frames blank), 4365 calls in all.
//   V = 1025 .. 1280     T <= 128, T * B <= 2048 / more   129 .. 256, <= 2048 / more   257 .. 512, <= 64K   513 ..
//     single-stage       0.98 / 1.12                      1.00 / 1.20                  1.45                 1.7
//     two-stage          0.87 / 1.01                      0.93 / 1.09                  1.29                 1.6
//     CTC                0.79 / 0.75                      0.66 / 0.77                  0.90                 1.1
//   (500 frames x 32 / 33 / 64 / 128 under the CTC rule, V = 1025: 0.90, 0.83, 0.97, 0.84; 750 x 16: 1.15)
//   V = 1281 .. 16384    T <= 128, T * B <= 8192 / 16384   T <= V / 16, <= 8192 / 16384   V / 16 .. V / 8, B < 12 / more
//     1281 .. 2048       0.90 / 0.95                       - / -                          0.90 / 1.01
//     2500, 3000         0.82 / 0.95                       0.86 / 0.99                    0.86 / 0.98
//     4096, 6000         0.66 / 0.89                       0.83 / 0.91                    0.85 / 1.05
//     8192, 10000        0.48 / 0.94                       0.73 / 0.96                    0.65 / 1.11
//     12288 .. 16384     0.39 / 0.91                       0.72 / 0.97                    0.59 / 1.08
//   The third column past 8192 rows: 0.92 to 1.03 under the single-stage rule, 0.92 to 1.04 under the CTC rule, with single
//   calls up to 1.33; 0.88 to 0.93 under the two-stage rule.  Past V / 8: 1.03 to 1.4 up to 3000 tokens; for one to four
//   hypotheses 1.04 at 4096, 0.83 at 6000, 0.4 to 0.6 above.
//   V > 16384 (no segment decoder): 32001, 100 frames x 16: 3340 -> 75 us.
// These are means: a call loses where one hypothesis speaks many phrases, whose frames the second pass takes one by one
// (CTC rule: V = 6000, 200 x 32 1.4, V = 16384, 250 x 32 1.2), and gains as much where none does.
static bool rows_pay(int V, int32_t T, int32_t B, int sel) {
  const int64_t rows = static_cast<int64_t>(T) * B;
  if (V > kWideMaxV) return rows <= kMaxWorkgroups;
  if (V <= 1024) return false;
  if (V <= kNarrowMaxV) {
    if (sel == 2) return T <= 512 && rows <= 65536;
    return T <= (sel == 0 ? 128 : 256) && rows <= 2048;
  }
  if (rows > 16384) return false;
  if (V >= 4096 && B <= 4) return true;
  const int longest = V / (B < 12 ? 8 : 16);
  return T <= 128 || (T <= longest && (sel == 1 || rows <= 8192));
}

bool frames_rows_ok(const DeviceTree& t, int32_t T, int32_t B, int sel) {
  return t.p_root != nullptr && t.root_rec != nullptr && rows_pay(t.vocab_size, T, B, sel) &&
         walk_lds_bytes(t.vocab_size, T, 1) <= static_cast<size_t>(g_walk_max_lds);
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
#define PB_ROWS(SEL)                                                                                                      \
  hipLaunchKernelGGL((rows_narrow_kernel<kNarrowMaxV / 64, SEL>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, \
                     t, pick, d_logp, frame_stride, row_stride, alpha, T, B, static_cast<int>(strips), d_tokens, d_states)
    if (sel == 0) {
      PB_ROWS(0);
    } else {
      PB_ROWS(1);
    }
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
  int waves = 16;
  while (waves > 1 && (waves * 2 > T || walk_lds_bytes(V, T, waves) > static_cast<size_t>(g_walk_max_lds))) --waves;
  const size_t lds = walk_lds_bytes(V, T, waves);
#define PB_WALK(SEL)                                                                                                     \
  hipLaunchKernelGGL(walk_kernel<SEL>, dim3(static_cast<unsigned>(B)), dim3(64 * waves), lds, stream, t, pick, d_logp,   \
                     frame_stride, row_stride, d_states0, d_last0, alpha, T, B, d_tokens, d_states, d_scores)
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
