// Wave kernels for rows wider than 1280 tokens (gfx950, wave64): the multi-frame greedy decoder and the
// single greedy step with their selection rules (Alg. 1 Stage 3, Eq. 1; Sec. II-C).
//
//  * A row is consumed in chunks of 1024 tokens in the 16-tokens-per-lane layout of the narrow kernels.  In
//    the multi-frame decoder one wave owns a hypothesis segment and streams its rows through a ring of two to four
//    register buffers (ring_of) that runs across frame boundaries: while a frame is being decided the first chunks of
//    the next one are already in flight.  The root scores of the row sit in LDS, shared by the workgroup.
//  * Base candidates.  Every lane keeps a running maximum of logp[v] + alpha * (p_root + root_score[v])
//    over its tokens in ascending order (strictly greater replaces, so the lowest token among equal values
//    stays); one wave reduction per frame yields the row maximum and its lowest token.  The two-stage rules
//    keep a second running maximum of the raw row in the same pass.
//  * Arc candidates.  After the pass the arcs of the failure chain are evaluated one per lane, their
//    log-probs gathered from the row in memory (it has just been read, so the gathers hit in cache); chains
//    with more than one state mark tokens in an LDS bit set so that an arc shadowed by a deeper chain state
//    is skipped.  The frame is decided as in the narrow kernels: the best arc against the base winner.
//    The rare cases that this cannot settle -- the base winner is itself overridden by an arc that does not
//    beat it, the CTC rule bars the winner, or every candidate is -inf -- take a plain second pass over the
//    row with all overridden tokens marked.
//  * The single step spreads one row (up to 65536 tokens) over a workgroup, one to four chunks per wave, so that
//    the whole row is requested at once; the waves' partial winners meet in LDS and wave 0 evaluates the arcs and decides.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "pb_chunk.hpp"
#include "pb_kernels.hpp"
#include "pb_wave.hpp"

namespace pb {

namespace {

using namespace wv;

#ifndef PB_WIDE_WAVES_EU
#define PB_WIDE_WAVES_EU 2
#endif
// RING: chunks in flight or in use per wave.  A row is padded to whole turns of the ring, so the launch picks the
// ring that pads it least: four buffers, three (5, 6 and 9 chunks), or two (rows of two chunks).
constexpr int ring_of(int nch) { return nch == 2 ? 2 : (nch + 2) / 3 * 3 < (nch + 3) / 4 * 4 ? 3 : 4; }

// Decides a frame whose base winner (M, vb) over all tokens is known: the arcs of the failure chain against it.
//   early: arc number `lane` of the state (clamped into its arc range), requested before the row pass, and
//   early_x: the log-prob of that arc's token, gathered during the pass
//   last:  label of the previous frame (SEL == 2; any value outside [0, V) = none)
template <int FORM, int SEL>
__device__ __forceinline__ FrameOut decide_wide(const TreeView& t, const Cursor& cur, const float* __restrict__ rowp,
                                                float alpha, float M, int vb, const ArcRec& early, float early_x, int last,
                                                unsigned* tags, int tag_words, int nch, int lane) {
  const Rec rec0 = cur.rec;
  const bool chain = cur.s != 0;
  const bool multi = chain && rec0.fail != 0;
  float bf = -INFINITY;
  int btok = INT_MAX, bchild = 0;
  bool hit_vb = false;
  if (chain) {
    if (multi) tags_clear_n(tags, tag_words, lane);
    Rec r = rec0;
    float p = 0.0f;
    for (int level = 0;; ++level) {
      for (int j0 = 0; j0 < r.count; j0 += 64) {
        const int j = j0 + lane;
        const bool valid = j < r.count;
        ArcRec a = early;
        float xv = early_x;
        const bool first = level == 0 && j0 == 0;
        if (!first) a = t.arc[r.begin + min(j, r.count - 1)];
        const int tk = valid ? a.token : 0;  // an unused entry may hold anything: keep the indices in range
        if (!first) xv = rowp[tk];
        bool shadowed = !valid;
        if (multi) {
          if (level > 0) shadowed = shadowed || tag_test(tags, tk);  // a deeper chain state owns this token
          if (valid) tag_set(tags, tk);
        }
        hit_vb = hit_vb || (valid && tk == vb);
        const float fa = __fadd_rn(xv, __fmul_rn(alpha, __fadd_rn(p, a.score)));
        const bool take = !shadowed && (fa > bf || (fa == bf && tk < btok));
        bf = take ? fa : bf;
        btok = take ? tk : btok;
        bchild = take ? r.begin + j + 1 : bchild;
      }
      p = __fadd_rn(p, r.backoff);
      if (r.fail == 0) break;
      r = load_rec(t, r.fail);
    }
  }
  if ((SEL == 0 && t.blank >= 0) || t.eos >= 0) {  // the blank and the EOS token, kept out of the base pass
    int tk;
    float fv;
    if (special_candidate<SEL>(t, rowp, alpha, __fmul_rn(alpha, cur.eos_boost), true, lane, tk, fv)) {
      const bool take = fv > bf || (fv == bf && tk < btok);
      bf = take ? fv : bf;
      btok = take ? tk : btok;
      bchild = take ? -1 : bchild;  // no arc: the state stays
    }
  }
  bool settled = M != -INFINITY;
  FrameOut o{M, vb, false, 0};
  const bool mine0 = btok != INT_MAX;
  if (settled && __ballot(mine0) != 0) {
    const float MA = ukey_val(wave_max_u(mine0 ? ukey(bf) : 0u));
    const bool vb_overridden = __ballot(hit_vb) != 0;
    if (vb_overridden || MA >= M) {
      const bool mine = mine0 && bf == MA;
      const int va = wave_min_nn(mine ? btok : INT_MAX);
      const int achild = __builtin_amdgcn_readlane(bchild, first_lane(__ballot(mine && btok == va)));
      if (MA > M || (!vb_overridden && MA == M && va < vb)) {
        o = FrameOut{MA, va, achild >= 0, achild};
      } else if (vb_overridden) {
        settled = false;  // the base winner is shadowed by an arc that does not beat it
      }
    }
  }
  if (settled && SEL == 2 && o.tok == last) settled = false;  // the CTC rule bars the previous label
  if (!settled) {
    int excl = -1;
    if (SEL == 2) {
      // first without the exclusion (the label may not even win), then, if it does win, without the label
      o = slow_frame<FORM, SEL>(t, cur, rowp, alpha, -1, tags, tag_words, nch, lane);
      if (o.tok != last) return o;
      excl = last;
    }
    o = slow_frame<FORM, SEL>(t, cur, rowp, alpha, excl, tags, tag_words, nch, lane);
    return o;
  }
  o.val = uniform_f(o.val);
  o.tok = uniform_i(o.tok);
  o.child = uniform_i(o.child);
  return o;
}

// The state after a frame decided as `o` (need_record: false when only the id is wanted).
__device__ __forceinline__ void advance(const TreeView& t, Cursor& cur, const FrameOut& o, bool need_record) {
  if (o.arc) {
    if (need_record) {
      cur = cursor_at(t, o.child);
    } else {
      cur.s = o.child;
    }
  } else if (o.tok != t.blank && o.tok != t.eos) {  // the blank and the EOS keep the state
    const v8i rr = t.root_rec[o.tok];
    cur = cursor_from_root_rec(rr);
  }
  cur.s = uniform_i(cur.s);
  cur.rec.begin = uniform_i(cur.rec.begin);
  cur.rec.count = uniform_i(cur.rec.count);
  cur.rec.fail = uniform_i(cur.rec.fail);
  cur.rec.backoff = uniform_f(cur.rec.backoff);
  cur.p_root = uniform_f(cur.p_root);
  cur.eos_boost = uniform_f(cur.eos_boost);
}

// Winner under root-state boosts from the lanes' running maxima `gb`; under the single-stage rule the blank
// (kept out of the pass) competes with boost 0.
template <int FORM, int SEL>
__device__ __forceinline__ int root_winner(const TreeView& t, const LaneBest& gb, const float* __restrict__ rowp,
                                           float alpha, int lane) {
  float M;
  int w;
  wave_pick<FORM>(t, gb, lane, M, w);
  w = uniform_i(w);
  if (SEL == 0 && t.blank >= 0) {
    const float fb = __fadd_rn(uniform_f(rowp[t.blank]), __fmul_rn(alpha, 0.0f));
    if (fb > M || (fb == M && t.blank < w)) w = t.blank;
  }
  return w;
}

// Raw arg-max v0 (two-stage rules) and winner w under root-state boosts of one row, by a plain pass.
template <int FORM, int SEL>
__device__ __forceinline__ void row_winners(const TreeView& t, const float* __restrict__ rowp, float alpha,
                                            const float* rs, int nch, int lane, int& v0, int& w) {
  LaneBest fb = lane_best_init(), rb = lane_best_init(), gb = lane_best_init();
  float x[2][16];
  load_chunk<FORM>(rowp, 0, t.V, lane, x[0]);
  for (int ch0 = 0; ch0 < nch; ch0 += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ch = ch0 + u;
      if (ch < nch) {
        if (ch + 1 < nch) load_chunk<FORM>(rowp, (ch + 1) * kChunk, t.V, lane, x[(u + 1) % 2]);
        float rw[16];
        read_rs_lds(rs, ch * kChunk, lane, rw);
        wide_chunk<SEL, true>(x[u], rw, ch, 0.0f, alpha, fb, rb, gb);
      }
    }
  }
  w = root_winner<FORM, SEL>(t, gb, rowp, alpha, lane);
  v0 = -1;
  if (SEL != 0) {
    float M;
    wave_pick<FORM>(t, rb, lane, M, v0);
    v0 = uniform_i(v0);
  }
}

// Boundary guess for wide rows, the scheme of the narrow kernels: (v0, w) are the winners of frame f, the one
// before the boundary; frames that keep the state are skipped going back, up to kLookBack frames or the start
// of the call.  Both neighbours of a boundary compute it from the same rows with the same arithmetic.
template <int FORM, int SEL>
__device__ __forceinline__ void guess_boundary_wide(const TreeView& t, int v0, int w, const float* __restrict__ rowp,
                                                    int64_t frame_stride, int f, const int32_t* __restrict__ states0,
                                                    int b, float alpha, const float* rs, int nch, int lane, int& state,
                                                    int& label) {
  label = -1;
  for (int k = 0;; ++k) {
    bool keep = false;
    int win = w;
    if (SEL != 0) {
      keep = v0 == t.blank;
      if (keep) win = v0;
    }
    if (!keep) keep = win == t.blank || win == t.eos;
    if (k == 0) label = win;
    if (!keep) {
      state = uniform_i(t.root_next[win]);
      return;
    }
    if (f - k == 0) {  // nothing since the start of the call has moved the state
      const int s0 = uniform_i(states0[b]);
      state = valid_state(t, s0) ? s0 : 0;
      return;
    }
    if (k + 1 >= kLookBack) {
      state = 0;
      return;
    }
    rowp -= frame_stride;
    row_winners<FORM, SEL>(t, rowp, alpha, rs, nch, lane, v0, w);
  }
}

// Decodes frames [f0, f1) of hypothesis b, as run_frames_1k does for narrow rows (same arguments and rules).
//   rs: root scores of the row in LDS, for the positions of nchp chunks; tags: this wave's token marks (32 * nchp words)
//   nchp: chunks per row rounded up to a whole turn of the ring (chunks past the row hold copies of its end)
template <bool COMPARE, bool FORM, int RING, int SEL, bool EDGE>
__device__ __forceinline__ bool run_frames_wide(const TreeView& t, const float* __restrict__ logp, int64_t frame_stride,
                                                int64_t row_stride, float alpha, int B, int b, int f0, int f1, int s_in,
                                                int last_in, int T, const int32_t* __restrict__ states0,
                                                int32_t* __restrict__ tokens, int32_t* __restrict__ states,
                                                float* __restrict__ scores, const float* rs, unsigned* tags, int nchp,
                                                int lane) {
  if (f0 >= f1) return true;
  constexpr bool GUESS = EDGE && !COMPARE;
  const int V = t.V;
  const int nch = (V + kChunk - 1) / kChunk;
  const int tag_words = nchp * kTagWords;
  const float* rp = logp + static_cast<size_t>(b) * row_stride + static_cast<size_t>(f0) * frame_stride;
  // The ring: buffer u holds chunk ch with ch % RING == u.  A chunk is requested RING - 1 chunks ahead, into
  // the buffer the chunk before the current one has just left, at the start of a chunk's turn.
  float xb[RING][16];
#pragma unroll
  for (int u = 0; u + 1 < RING; ++u) load_chunk<FORM>(rp, u * kChunk, V, lane, xb[u]);
  StoredLane<SEL == 2> stored;
  if (COMPARE) stored.fetch(lane, f0, f1, B, b, tokens, states);
  int s = uniform_i(s_in);
  int last = -1;
  if (SEL == 2) last = uniform_i(last_in);
  const bool guessable = GUESS && t.num_states < kGuessOk;
  if (guessable && f0 > 0 && s == 0) {  // (an invalid start state, e.g. of an unknown tree, is left as it is)
    int v0, w, label;
    row_winners<FORM, SEL>(t, rp - frame_stride, alpha, rs, nch, lane, v0, w);
    guess_boundary_wide<FORM, SEL>(t, v0, w, rp - frame_stride, frame_stride, f0 - 1, states0, b, alpha, rs, nch, lane,
                                   s, label);
    if (SEL == 2) last = label;
  }
  if (!valid_state(t, s)) {
    fill_invalid(B, b, f0, f1, tokens, states, scores, lane);
    return false;
  }
  Cursor cur = cursor_at(t, s);
  LaneOut out{f0, 0, 0, 0.0f};
  for (int f = f0; f < f1; ++f) {
    if (GUESS) set_wave_priority(min(3, 4 * (f1 - f) / (f1 - f0)));  // (pass 1: the more is left, the higher)
    const bool more = f + 1 < f1;
    const bool track = guessable && !more && f1 < T;  // last frame of the range: also its root-state winner
    // the first arcs of the state, requested before the pass over the row (unconditionally; the index is
    // clamped into the state's arc range, see the narrow kernels)
    const ArcRec early = t.arc[cur.rec.begin + max(0, min(lane, cur.rec.count - 1))];
    LaneBest fb = lane_best_init(), rb = lane_best_init(), gb = lane_best_init();
    const float* rpn = more ? rp + frame_stride : rp;
    float early_x = 0.0f;  // log-prob of the early arc's token: gathered after the first turn of the ring, when the arc is there
    auto pass = [&](auto track_c) {
      constexpr bool TRACK = decltype(track_c)::value;
      auto turn = [&](int g) {  // one turn of the ring: RING chunks, straight-line code
#pragma unroll
        for (int u = 0; u < RING; ++u) {
          const int ch = g + u;
          // Request the chunk RING - 1 ahead, of this row or of the next, without a condition (after the last
          // frame of the range the row in hand is asked for again, from cache): straight-line code lets the
          // compiler wait for exactly the chunk it needs and keep the others in flight.
          const int nx = ch + RING - 1;
          const bool wrap = nx >= nchp;
          load_chunk<FORM>(wrap ? rpn : rp, (wrap ? nx - nchp : nx) * kChunk, V, lane, xb[(u + RING - 1) % RING]);
          float rw[16];
          read_rs_lds(rs, ch * kChunk, lane, rw);
          wide_chunk<SEL, TRACK>(xb[u], rw, ch, cur.p_root, alpha, fb, rb, gb);
          __builtin_amdgcn_sched_barrier(0);  // (the four turns would otherwise be interleaved and run out of registers)
        }
      };
      turn(0);
      // the early arc is there by now: the log-prob of its token is gathered while the rest of the row streams
      early_x = rp[lane < cur.rec.count ? early.token : 0];
      for (int g = RING; g < nchp; g += RING) turn(g);
    };
    if (track) {
      pass(std::integral_constant<bool, true>{});
    } else {
      pass(std::integral_constant<bool, false>{});
    }
    float M;
    int vb;
    wave_pick<FORM>(t, fb, lane, M, vb);
    int v0 = -1;
    FrameOut o;
    bool stage1 = false;
    if (SEL != 0) {  // stage 1: selection without boosting; a blank (or a CTC repeat) is emitted as it is
      float M0;
      wave_pick<FORM>(t, rb, lane, M0, v0);
      v0 = uniform_i(v0);
      if (v0 == t.blank || (SEL == 2 && v0 == last)) {
        o = FrameOut{uniform_f(M0), v0, false, 0};
        stage1 = true;
      }
    }
    if (!stage1) {
      o = decide_wide<FORM, SEL>(t, cur, rp, alpha, M, uniform_i(vb), early, early_x, last, tags, tag_words, nch, lane);
      advance(t, cur, o, more);
    }
    const int word = cur.s;
    const int slot = f - out.base;
    out.put(lane, f, o.tok, word, o.val);
    if (COMPARE) {
      // met the stored trajectory: this frame is written too (its score may differ), the rest stands
      if (stored.state_at(slot) == word && (SEL != 2 || stored.token_at(slot) == o.tok)) {
        out.template flush<true>(lane, slot + 1, B, b, tokens, states, scores);
        return true;
      }
    }
    if (track) {
      // the guess the next range starts from, made from the same rows; if it is what this range really ends
      // in, the last state word says so
      int g, glabel;
      const int w = root_winner<FORM, SEL>(t, gb, rp, alpha, lane);
      guess_boundary_wide<FORM, SEL>(t, v0, w, rp, frame_stride, f, states0, b, alpha, rs, nch, lane, g, glabel);
      if (g == cur.s && (SEL != 2 || glabel == o.tok)) {
        if (lane == slot) out.st |= kGuessOk;
      }
    }
    if (slot == 63 && more) {  // (the last group is written at the end)
      out.template flush<COMPARE>(lane, 64, B, b, tokens, states, scores);
      out.base = f + 1;
      if (COMPARE) stored.fetch(lane, f + 1, f1, B, b, tokens, states);
    }
    if (SEL == 2) last = o.tok;
    rp += frame_stride;
  }
  out.template flush<COMPARE>(lane, f1 - out.base, B, b, tokens, states, scores);
  return false;  // (a re-run: the end of the range was reached without meeting the stored trajectory)
}

template <int FORM>
__device__ __forceinline__ float4 staged_root_scores(const TreeView& t, int i) {
  const float* p = t.root_score + min(i, t.V - 4);
  return mask_special<FORM>(t, i, make_float4(p[0], p[1], p[2], p[3]));
}

// The same into LDS for a whole row, by the whole workgroup; ends with a barrier.
template <int FORM>
__device__ __forceinline__ void stage_root_scores(const TreeView& t, float* rs, int nchp) {
  const int n = nchp * kChunk;
  for (int i = 4 * static_cast<int>(threadIdx.x); i < n; i += 4 * static_cast<int>(blockDim.x))
    *reinterpret_cast<float4*>(rs + i) = staged_root_scores<FORM>(t, i);
  __syncthreads();
}

// Pass 1 (see frames_spec_kernel of the narrow rows).  With a table of trees the workgroup's waves may use
// different trees, so each wave then keeps its own copy of the root scores.
template <int FORM, int RING, int SEL, bool FOREST>
__global__ void __launch_bounds__(256, PB_WIDE_WAVES_EU) wide_spec_kernel(DeviceTree dt, TreePick pick, const float* __restrict__ logp,
                                                         int64_t frame_stride, int64_t row_stride,
                                                         const int32_t* __restrict__ states0,
                                                         const int32_t* __restrict__ last0, float alpha, int T, int B,
                                                         int seg_len, int nseg, int nchp, int32_t* __restrict__ tokens,
                                                         int32_t* __restrict__ states, float* __restrict__ scores) {
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int chain = blockIdx.x * nwaves + wave;
  const bool live = chain < B * nseg;
  const int j = live ? chain / B : 0, b = live ? chain - j * B : 0;
  DeviceTree mine = dt;
  bool tree_ok = true;
  if constexpr (FOREST) tree_ok = pick_tree(pick, b, mine);
  const TreeView t = make_view(mine);
  const int row_floats = nchp * kChunk;
  float* rs = lds;
  unsigned* tags;
  if constexpr (FOREST) {
    rs = lds + wave * (row_floats + nchp * kTagWords);
    tags = reinterpret_cast<unsigned*>(rs + row_floats);
    if (tree_ok) {
      for (int i = 4 * lane; i < row_floats; i += 256) *reinterpret_cast<float4*>(rs + i) = staged_root_scores<FORM>(t, i);
    }
  } else {
    tags = reinterpret_cast<unsigned*>(lds + row_floats) + wave * nchp * kTagWords;
    stage_root_scores<FORM>(t, rs, nchp);
  }
  if (!live) return;
  const int f0 = seg_begin(j, T, nseg), f1 = seg_begin(j + 1, T, nseg);
  int s = 0, last = -1;
  if (j == 0) {
    s = states0[b];
    if (SEL == 2 && last0 != nullptr) last = last0[b];
  }
  if (!tree_ok) s = -1;  // an unknown tree marks every frame of the hypothesis like an invalid state
  run_frames_wide<false, FORM, RING, SEL, true>(t, logp, frame_stride, row_stride, alpha, B, b, f0, f1, s, last, T, states0,
                                          tokens, states, scores, rs, tags, nchp, lane);
}

// Pass 2: one workgroup per hypothesis (one tree, so the root scores are shared).
template <int FORM, int RING, int SEL, bool FOREST>
__global__ void __launch_bounds__(512) wide_fix_kernel(DeviceTree dt, TreePick pick, const float* __restrict__ logp,
                                                        int64_t frame_stride, int64_t row_stride, float alpha, int T,
                                                        int B, int seg_len, int nseg, int nchp,
                                                        int32_t* __restrict__ tokens, int32_t* __restrict__ states,
                                                        float* __restrict__ scores) {
  extern __shared__ float lds[];
  __shared__ int assumed[64], assumed_tok[64];
  __shared__ unsigned bad_words[2];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int b = blockIdx.x;
  DeviceTree mine = dt;
  if constexpr (FOREST) {
    if (!pick_tree(pick, b, mine)) return;  // pass 1 has marked every frame of this hypothesis (the whole workgroup leaves)
  }
  const TreeView t = make_view(mine);
  float* rs = lds;
  unsigned* tags = reinterpret_cast<unsigned*>(lds + nchp * kChunk) + wave * nchp * kTagWords;
  stage_root_scores<FORM>(t, rs, nchp);
  fix_segments<SEL == 2>(T, B, b, seg_len, nseg, tokens, states, scores, nullptr, assumed, assumed_tok, bad_words, lane,
                         wave, nwaves,
                         [&](int seg, int s, int last) {
                           const int f0 = seg_begin(seg, T, nseg), f1 = seg_begin(seg + 1, T, nseg);
                           return run_frames_wide<true, FORM, RING, SEL, false>(t, logp, frame_stride, row_stride, alpha, B, b, f0, f1,
                                                                   s, last, T, nullptr, tokens, states, scores, rs, tags,
                                                                   nchp, lane);
                         });
}

// Single step: one workgroup per hypothesis, CPW chunks per wave (one up to 16384 tokens, four up to 65536), so that
// the whole row is requested at once; only the root scores of a wave's later chunks, which sit in a cache, follow chunk
// by chunk (two rows of four chunks do not fit the 128 registers of a 16-wave workgroup).  V = 50000, B = 16: 12.3 us
// per step against 26.5 with the row build in LDS it replaces; what is left is one CU taking 200 KB of row and as much
// of root scores.
// The waves' winners meet in LDS; wave 0 evaluates the arcs and decides.
struct StepPart {
  float M, M0;
  int vb, v0;
};

// (The order of the requests is what a single step costs: the root scores, which sit in a cache, and the row go out
// first, with the state id, before anything is waited for.  LEAN: one tree for all rows; the leading arguments,
// the root-score array among them, are then in registers when the wave starts, and an invalid state is decoded as
// the root and marked at the end, so that no early exit stands between the wave start and the requests.  The outputs come
// last: arguments that are there from the start would hold scalar registers until the end.)
template <int FORM, int CPW, int SEL, bool LEAN>
__global__ void __launch_bounds__(1024) step_wide_kernel(
    const float* __restrict__ logp, int64_t row_stride, const int32_t* __restrict__ states_in,
    const float* __restrict__ root_score, const int32_t* __restrict__ last_in, float alpha, DeviceTree dt, TreePick pick,
    int32_t* __restrict__ tokens, int32_t* __restrict__ states_out, float* __restrict__ scores) {
  extern __shared__ float lds[];  // wave 0's token marks
  __shared__ StepPart part[16];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const int b = blockIdx.x;
  DeviceTree mine = dt;
  bool tree_ok = true;
  if constexpr (!LEAN) tree_ok = pick_tree(pick, b, mine);
  const TreeView t = make_view(mine);
  const int nch = nwaves * CPW;  // (chunks behind the end of the row hold copies)
  const float* rowp = logp + static_cast<size_t>(b) * row_stride;
  const float* rsp = LEAN ? root_score : t.root_score;
  float x[CPW][16], rw[16];
  load_chunk<FORM>(rsp, wave * CPW * kChunk, t.V, lane, rw, 0.0f);
#pragma unroll
  for (int c = 0; c < CPW; ++c) load_chunk<FORM>(rowp, (wave * CPW + c) * kChunk, t.V, lane, x[c]);
  int s = tree_ok ? states_in[b] : -1;  // an unknown tree marks the hypothesis like an invalid state
  __builtin_amdgcn_sched_barrier(0);
  s = uniform_i(s);
  const bool ok = valid_state(t, s);  // uniform over the workgroup
  if (!LEAN && !ok) {
    if (threadIdx.x == 0) {
      tokens[b] = -1;
      states_out[b] = -1;
      scores[b] = NAN;
    }
    return;
  }
  if (!ok) s = 0;
  auto mask_row = [&](int ch) {  // NaN in the blank and EOS columns: those two are candidates of their own
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 q = mask_special<FORM>(t, ch * kChunk + 256 * i + 4 * lane,
                                          make_float4(rw[4 * i], rw[4 * i + 1], rw[4 * i + 2], rw[4 * i + 3]));
      rw[4 * i + 0] = q.x; rw[4 * i + 1] = q.y; rw[4 * i + 2] = q.z; rw[4 * i + 3] = q.w;
    }
  };
  mask_row(wave * CPW);
  Cursor cur;
  ArcRec early = ArcRec{0, 0.0f};
  float p_root;
  if (wave == 0) {
    cur = cursor_at(t, s);
    early = t.arc[cur.rec.begin + max(0, min(lane, cur.rec.count - 1))];
    p_root = cur.p_root;
  } else {
    p_root = t.p_root[s];
  }
  float early_x = 0.0f;  // (wave 0: the log-prob of its early arc's token, requested before the row is looked at)
  if (wave == 0) early_x = rowp[lane < cur.rec.count ? early.token : 0];
  LaneBest fb = lane_best_init(), rb = lane_best_init(), gb = lane_best_init();
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    float next_rw[16];
    if (c + 1 < CPW) load_chunk<FORM>(rsp, (wave * CPW + c + 1) * kChunk, t.V, lane, next_rw, 0.0f);
    wide_chunk<SEL, false>(x[c], rw, wave * CPW + c, p_root, alpha, fb, rb, gb);
    if (c + 1 < CPW) {
#pragma unroll
      for (int j = 0; j < 16; ++j) rw[j] = next_rw[j];
      mask_row(wave * CPW + c + 1);
    }
  }
  StepPart mine_part{0.0f, 0.0f, 0, 0};
  wave_pick<FORM>(t, fb, lane, mine_part.M, mine_part.vb);
  if (SEL != 0) wave_pick<FORM>(t, rb, lane, mine_part.M0, mine_part.v0);
  if (lane == 0) part[wave] = mine_part;
  __syncthreads();
  if (wave != 0) return;
  // chunks ascend with the wave index, so among equal maxima the lowest wave holds the lowest token
  const bool have = lane < nwaves;
  const StepPart q = part[have ? lane : 0];
  const float M = ukey_val(wave_max_u(have ? ukey(q.M) : 0u));
  const int vb = __builtin_amdgcn_readlane(q.vb, first_lane(__ballot(have && q.M == M)));
  const int vb_next = t.root_next[vb];  // where the base winner leads, requested before the arcs are evaluated
  int last = -1;
  if (SEL == 2 && last_in != nullptr) last = uniform_i(last_in[b]);
  FrameOut o;
  bool stage1 = false;
  if (SEL != 0) {
    const float M0 = ukey_val(wave_max_u(have ? ukey(q.M0) : 0u));
    const int v0 = __builtin_amdgcn_readlane(q.v0, first_lane(__ballot(have && q.M0 == M0)));
    if (v0 == t.blank || (SEL == 2 && v0 == last)) {
      o = FrameOut{M0, v0, false, 0};
      stage1 = true;
    }
  }
  if (!stage1) {
    unsigned* tags = reinterpret_cast<unsigned*>(lds);
    o = decide_wide<FORM, SEL>(t, cur, rowp, alpha, M, vb, early, early_x, last, tags, nch * kTagWords, nch, lane);
    if (!o.arc && o.tok == vb && vb != t.blank && vb != t.eos) {
      cur.s = uniform_i(vb_next);  // only the state id leaves the kernel
    } else {
      advance(t, cur, o, false);
    }
  }
  if (lane == 0) {
    tokens[b] = ok ? o.tok : -1;
    states_out[b] = ok ? cur.s : -1;
    scores[b] = ok ? o.val : NAN;
  }
}

int g_wide_fix_waves = 8;   // waves per fix-up workgroup the device's LDS allows for the widest row, set once
int g_wide_max_lds = 64 * 1024;

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

// Expands to one launch per (row kind, selection rule) pair.  Kinds of the multi-frame kernels: 0 = whole ring turns of
// full chunks in 16-byte aligned rows, 1 .. 3 = any row through a ring of four, three or two buffers.
#define PB_DISPATCH(kind, sel, LAUNCH)     \
  switch (3 * (kind) + (sel)) {            \
    case 0: LAUNCH(kWhole, 4, 0); break;     \
    case 1: LAUNCH(kWhole, 4, 1); break;     \
    case 2: LAUNCH(kWhole, 4, 2); break;     \
    case 3: LAUNCH(kAny, 4, 0); break;    \
    case 4: LAUNCH(kAny, 4, 1); break;    \
    case 5: LAUNCH(kAny, 4, 2); break;    \
    case 6: LAUNCH(kAny, 3, 0); break;    \
    case 7: LAUNCH(kAny, 3, 1); break;    \
    case 8: LAUNCH(kAny, 3, 2); break;    \
    case 9: LAUNCH(kAny, 2, 0); break;    \
    case 10: LAUNCH(kAny, 2, 1); break;   \
    default: LAUNCH(kAny, 2, 2); break;   \
  }

int launch_step_wide(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride,
                     const int32_t* d_states_in, const int32_t* d_last, float alpha, int32_t B, int sel,
                     int32_t* d_tokens, int32_t* d_states_out, float* d_scores, hipStream_t stream) {
  const int V = t.vocab_size;
  const int nch = (V + kChunk - 1) / kChunk;  // <= 64 (kStepMaxV)
  // Chunks per wave: the fewest that leave at most 16 waves, a workgroup of 1024 threads.
  const int cpw = (nch + 15) / 16, waves = (nch + cpw - 1) / cpw;
  const bool aligned = V % 4 == 0 && row_stride % 4 == 0 && aligned16(d_logp) && aligned16(t.root_score);
  const size_t lds = static_cast<size_t>(waves) * cpw * kTagWords * sizeof(unsigned);
  const dim3 grid(static_cast<unsigned>(B)), block(static_cast<unsigned>(64 * waves));
  const bool lean = pick.table == nullptr;
#define PB_STEP(FORM, CPW, SEL, LEAN)                                                                              \
  hipLaunchKernelGGL((step_wide_kernel<FORM, CPW, SEL, LEAN>), grid, block, lds, stream, d_logp, row_stride,       \
                     d_states_in, t.root_score, d_last, alpha, t, pick, d_tokens, d_states_out, d_scores)
#define PB_LAUNCH(FORM, CPW, SEL)   \
  if (lean) {                       \
    PB_STEP(FORM, CPW, SEL, true);  \
  } else {                          \
    PB_STEP(FORM, CPW, SEL, false); \
  }
#define PB_SELECTION(FORM, CPW)               \
  switch (sel) {                              \
    case 0: PB_LAUNCH(FORM, CPW, 0); break;   \
    case 1: PB_LAUNCH(FORM, CPW, 1); break;   \
    default: PB_LAUNCH(FORM, CPW, 2); break;  \
  }
  // (aligned rows that end inside a chunk: V = 10000, B = 4096 37.8 to 42.8 us by rule, 39.9 to 47.2 with the clamped form,
  // whose registers leave room for one workgroup fewer; more than one chunk per wave: the clamped form only -- the row no
  // longer fits one load per lane and what the clamps cost disappears behind it)
  switch (cpw) {
    case 1:
      if (aligned && V % kChunk == 0) {
        PB_SELECTION(kWhole, 1)
      } else if (aligned) {
        PB_SELECTION(kGroups, 1)
      } else {
        PB_SELECTION(kAny, 1)
      }
      break;
    case 2: PB_SELECTION(kAny, 2) break;
    case 3: PB_SELECTION(kAny, 3) break;
    default: PB_SELECTION(kAny, 4) break;
  }
#undef PB_SELECTION
#undef PB_LAUNCH
#undef PB_STEP
  return hipGetLastError() == hipSuccess ? PB_OK : PB_EHIP;
}

int launch_frames_wide(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                       int64_t row_stride, const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T,
                       int32_t B, int sel, int32_t* d_tokens, int32_t* d_states, float* d_scores, hipStream_t stream) {
  const int V = t.vocab_size;
  const int nch = (V + kChunk - 1) / kChunk, ring = ring_of(nch), nchp = (nch + ring - 1) / ring * ring;
  const bool full = V % (4 * kChunk) == 0 && row_stride % 4 == 0 && frame_stride % 4 == 0 && aligned16(d_logp) &&
                    aligned16(t.root_score);
  const int kind = full ? 0 : 5 - ring;
  const bool forest = pick.table != nullptr;
  const size_t row_bytes = static_cast<size_t>(nchp) * kChunk * sizeof(float);
  const size_t tag_bytes = static_cast<size_t>(nchp) * kTagWords * sizeof(unsigned);
  // pass 1: four waves per workgroup share the root scores (a forest: one copy per wave, fewer waves if LDS is short)
  int waves = 4;
  size_t lds = row_bytes + waves * tag_bytes;
  if (forest) {
    while (waves > 1 && waves * (row_bytes + tag_bytes) > static_cast<size_t>(g_wide_max_lds)) waves /= 2;
    lds = waves * (row_bytes + tag_bytes);
  }
  if (lds > static_cast<size_t>(g_wide_max_lds)) return PB_EUNSUPPORTED;
  const SegPlan plan = plan_segments(T, B, kWideTargetChains);
  const int nseg = plan.nseg, seg_len = plan.seg_len;
  const int64_t chains = static_cast<int64_t>(B) * nseg;
  const int64_t blocks = (chains + waves - 1) / waves;
  if (!grid_fits(blocks, 64 * waves)) return PB_EUNSUPPORTED;
#define PB_SPEC(FORM, RING, SEL, FOREST)                                                                                 \
  hipLaunchKernelGGL((wide_spec_kernel<FORM, RING, SEL, FOREST>), dim3(static_cast<unsigned>(blocks)), dim3(64 * waves), \
                     lds, stream, t, pick, d_logp, frame_stride, row_stride, d_states0, d_last0, alpha, T, B,      \
                     seg_len, nseg, nchp, d_tokens, d_states, d_scores)
#define PB_LAUNCH(FORM, RING, SEL) PB_SPEC(FORM, RING, SEL, false)
#define PB_LAUNCH_F(FORM, RING, SEL) PB_SPEC(FORM, RING, SEL, true)
  if (forest) {
    PB_DISPATCH(kind, sel, PB_LAUNCH_F)
  } else {
    PB_DISPATCH(kind, sel, PB_LAUNCH)
  }
#undef PB_LAUNCH
#undef PB_LAUNCH_F
#undef PB_SPEC
  if (hipGetLastError() != hipSuccess) return PB_EHIP;
  if (nseg > 1) {
    int fw = nseg - 1 < g_wide_fix_waves ? nseg - 1 : g_wide_fix_waves;
    while (fw > 1 && row_bytes + fw * tag_bytes > static_cast<size_t>(g_wide_max_lds)) --fw;
    const size_t lds2 = row_bytes + fw * tag_bytes;
    if (lds2 > static_cast<size_t>(g_wide_max_lds)) return PB_EUNSUPPORTED;
#define PB_FIX(FORM, RING, SEL, FOREST)                                                                                   \
  hipLaunchKernelGGL((wide_fix_kernel<FORM, RING, SEL, FOREST>), dim3(static_cast<unsigned>(B)), dim3(64 * fw), lds2,     \
                     stream, t, pick, d_logp, frame_stride, row_stride, alpha, T, B, seg_len, nseg, nchp, d_tokens, \
                     d_states, d_scores)
#define PB_LAUNCH(FORM, RING, SEL) PB_FIX(FORM, RING, SEL, false)
#define PB_LAUNCH_F(FORM, RING, SEL) PB_FIX(FORM, RING, SEL, true)
    if (forest) {
      PB_DISPATCH(kind, sel, PB_LAUNCH_F)
    } else {
      PB_DISPATCH(kind, sel, PB_LAUNCH)
    }
#undef PB_LAUNCH
#undef PB_LAUNCH_F
#undef PB_FIX
    if (hipGetLastError() != hipSuccess) return PB_EHIP;
  }
  return PB_OK;
}

int prepare_wide_kernels(int max_lds_bytes) {
  // The widest row needs 64 KiB of root scores plus the waves' token marks: past 64 KiB of dynamic LDS the
  // limit of each kernel must be raised.
  constexpr int kPlainLimit = 64 * 1024 - 1024;  // static LDS of the kernels included
  const int want = ((kWideMaxV / kChunk) * kChunk + 8 * (kWideMaxV / kChunk) * kTagWords) * 4 + 1024;
  int limit = kPlainLimit;
  if (max_lds_bytes > kPlainLimit) {
    const int bytes = (want < max_lds_bytes ? want : max_lds_bytes) - 1024;
    const hipFuncAttribute attr = hipFuncAttributeMaxDynamicSharedMemorySize;
    bool ok = true;
#define PB_SET(FORM, RING, SEL)                                                                                               \
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void*>(wide_fix_kernel<FORM, RING, SEL, false>), attr, bytes) == hipSuccess && \
       hipFuncSetAttribute(reinterpret_cast<const void*>(wide_fix_kernel<FORM, RING, SEL, true>), attr, bytes) == hipSuccess &&        \
       hipFuncSetAttribute(reinterpret_cast<const void*>(wide_spec_kernel<FORM, RING, SEL, false>), attr, bytes) == hipSuccess &&      \
       hipFuncSetAttribute(reinterpret_cast<const void*>(wide_spec_kernel<FORM, RING, SEL, true>), attr, bytes) == hipSuccess
    for (int ms = 0; ms < 12; ++ms) PB_DISPATCH(ms / 3, ms % 3, PB_SET)
#undef PB_SET
    if (ok) {
      limit = bytes;
    } else {
      (void)hipGetLastError();
    }
  }
  g_wide_max_lds = limit;
  g_wide_fix_waves = 8;
  return PB_OK;
}

}  // namespace pb
