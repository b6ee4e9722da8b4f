// Device helpers of the kernels that take a row chunk by chunk (gfx950, wave64): running maxima per lane, the masks of
// the columns that are candidates of their own, and the decision of a frame by a plain second pass over its row.
#pragma once
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "pb_wave.hpp"

namespace pb {
namespace wv {

// load_row for the kernels that take a row in chunks.  (Plain vectors where the chunks tile the row: with float4 the
// decoder of V = 4096 took 5 to 7 % longer under the two-stage rules, with vectors that of V = 1024 4 %.)
template <int FORM, int NS>
__device__ __forceinline__ void load_chunk(const float* __restrict__ base, int cb, int V, int lane, float (&x)[NS],
                                           float fill = -INFINITY) {
  if constexpr (FORM == kWhole) {
    typedef float vf4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < NS / 4; ++i) {
      const vf4 q = *reinterpret_cast<const vf4*>(base + cb + 256 * i + 4 * lane);
      x[4 * i + 0] = q.x; x[4 * i + 1] = q.y; x[4 * i + 2] = q.z; x[4 * i + 3] = q.w;
    }
  } else {
    load_row<FORM>(base, cb, V, lane, x, fill);
  }
}

// Running arg-max of a lane over its tokens of a row; code = 16 * chunk + slot of the lane's token.
struct LaneBest {
  float m;
  int code;
};
__device__ __forceinline__ LaneBest lane_best_init() { return LaneBest{-INFINITY, 0}; }
__device__ __forceinline__ int code_pos(int code, int lane) { return (code >> 4) * kChunk + tok_of(code & 15, lane); }

// Row maximum and its lowest token from the lanes' running maxima.  A row whose candidates are all -inf (or
// excluded) comes back as M == -inf with a token that means nothing: the caller takes the second pass then.
template <int FORM>
__device__ __forceinline__ void wave_pick(const TreeView& t, const LaneBest& lb, int lane, float& M, int& tok) {
  M = ukey_val(wave_max_u(ukey(lb.m)));
  tok = pos_token<FORM>(t, wave_min_nn(lb.m == M ? code_pos(lb.code, lane) : INT_MAX));
}

// Boosts alpha * (p_root + root_score[v]) of the lane's 16 tokens of chunk `cb`; the blank boosts by 0
// (SEL == 0) or is excluded (NaN), the EOS token by `ce` = alpha * (EOS boost of the state) when `ce_on`.
template <int FORM, int SEL>
__device__ __forceinline__ void chunk_boosts(const TreeView& t, int cb, int lane, float p_root, float alpha, bool ce_on,
                                             float ce, const float (&rw)[16], float (&bo)[16]) {
#pragma unroll
  for (int j = 0; j < 16; ++j) bo[j] = __fmul_rn(alpha, __fadd_rn(p_root, rw[j]));
  const int blank = token_pos<FORM>(t, t.blank) - cb, eos = token_pos<FORM>(t, t.eos) - cb;
  const bool has_blank = static_cast<unsigned>(blank) < static_cast<unsigned>(kChunk);
  const bool has_eos = ce_on && static_cast<unsigned>(eos) < static_cast<unsigned>(kChunk);
  if (has_blank || has_eos) {  // uniform, and false for most chunks
    const int ln = opaque(lane);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (has_blank && slot_is(j, ln, blank)) bo[j] = SEL == 0 ? __fmul_rn(alpha, 0.0f) : NAN;
      if (has_eos && slot_is(j, ln, eos)) bo[j] = ce;
    }
  }
}

// One chunk of a row into the running maxima: `fb` fused under the state's boosts, `rb` the raw row
// (two-stage rules), `gb` fused under root-state boosts (TRACK: what a boundary guess needs).
// `rw` are the root scores of the chunk with NaN in the blank and EOS columns: those two tokens never enter
// the running maxima of the fused values; `special_candidates` adds them to the arc candidates instead.
template <int SEL, bool TRACK>
__device__ __forceinline__ void wide_chunk(const float (&x)[16], const float (&rw)[16], int ch, float p_root,
                                           float alpha, LaneBest& fb, LaneBest& rb, LaneBest& gb) {
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const float f = __fadd_rn(x[j], __fmul_rn(alpha, __fadd_rn(p_root, rw[j])));
    const bool up = f > fb.m;
    fb.m = up ? f : fb.m;
    fb.code = up ? 16 * ch + j : fb.code;
  }
  if constexpr (SEL != 0) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const bool up = x[j] > rb.m;
      rb.m = up ? x[j] : rb.m;
      rb.code = up ? 16 * ch + j : rb.code;
    }
  }
  if constexpr (TRACK) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float f = __fadd_rn(x[j], __fmul_rn(alpha, __fadd_rn(0.0f, rw[j])));
      const bool up = f > gb.m;
      gb.m = up ? f : gb.m;
      gb.code = up ? 16 * ch + j : gb.code;
    }
  }
}

// The blank (single-stage rule: boost 0, state kept) and the EOS token (boost tabulated per state, state kept;
// Sec. II-C) as candidates of their own: lane 63 takes the blank, lane 62 the EOS.  `ce` = alpha * (EOS boost).
// Returns whether the lane holds one, with its token and fused value.
template <int SEL>
__device__ __forceinline__ bool special_candidate(const TreeView& t, const float* __restrict__ rowp, float alpha,
                                                  float ce, bool with_eos, int lane, int& tok, float& val) {
  const bool is_blank = SEL == 0 && t.blank >= 0 && lane == 63;
  const bool is_eos = with_eos && t.eos >= 0 && lane == 62;
  tok = is_blank ? t.blank : t.eos;
  val = 0.0f;
  if (is_blank || is_eos) val = __fadd_rn(rowp[tok], is_blank ? __fmul_rn(alpha, 0.0f) : ce);
  return is_blank || is_eos;
}

__device__ __forceinline__ void read_rs_lds(const float* rs, int cb, int lane, float (&rw)[16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float4 q = *reinterpret_cast<const float4*>(rs + cb + 256 * i + 4 * lane);
    rw[4 * i + 0] = q.x; rw[4 * i + 1] = q.y; rw[4 * i + 2] = q.z; rw[4 * i + 3] = q.w;
  }
}

__device__ __forceinline__ void tags_clear_n(unsigned* bits, int words, int lane) {
  for (int i = lane; i < words; i += 64) bits[i] = 0u;
}

struct FrameOut {  // wave-uniform outcome of one frame
  float val;
  int tok;
  bool arc;    // the winner is an arc of the failure chain: the next state is `child`
  int child;
};

// The whole decision of a frame by a plain second pass (any case, no speculation): every token that some
// chain state overrides is marked, the arcs are evaluated deepest state first, and the base arg-max runs
// over the unmarked tokens only.  `excl` (CTC rule): a token barred from the selection, or -1.
template <int FORM, int SEL>
__device__ __forceinline__ FrameOut slow_frame(const TreeView& t, const Cursor& cur, const float* __restrict__ rowp,
                                               float alpha, int excl, unsigned* tags, int tag_words, int nch, int lane) {
  tags_clear_n(tags, tag_words, lane);
  float bf = 0.0f;
  int btok = INT_MAX, bchild = 0;
  {
    float p = 0.0f;
    for (int xs = cur.s; xs != 0;) {
      const Rec r = load_rec(t, xs);
      for (int j = lane; j < r.count; j += 64) {  // tokens of one state are distinct: no two lanes meet on a mark
        const ArcRec a = t.arc[r.begin + j];
        if (!tag_test(tags, a.token)) {
          tag_set(tags, a.token);
          if (SEL != 2 || a.token != excl) {
            const float fa = __fadd_rn(rowp[a.token], __fmul_rn(alpha, __fadd_rn(p, a.score)));
            if (btok == INT_MAX || fa > bf || (fa == bf && a.token < btok)) {
              bf = fa;
              btok = a.token;
              bchild = r.begin + j + 1;
            }
          }
        }
      }
      p = __fadd_rn(p, r.backoff);
      xs = uniform_i(r.fail);
    }
  }
  bool has = false;
  float m = 0.0f;
  int mtok = INT_MAX;
  const float ce = __fmul_rn(alpha, cur.eos_boost);
  for (int ch = 0; ch < nch; ++ch) {
    const int cb = ch * kChunk;
    float x[16], rw[16], bo[16];
    load_chunk<FORM>(rowp, cb, t.V, lane, x);
    load_chunk<FORM>(t.root_score, cb, t.V, lane, rw, 0.0f);
    chunk_boosts<FORM, SEL>(t, cb, lane, cur.p_root, alpha, t.eos >= 0, ce, rw, bo);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int q = cb + tok_of(j, lane), first = q & ~3, held = FORM != kAny ? 0 : first - min(first, t.V - 4);
      const int v = min(q - held, t.V - 1);
      const float f = __fadd_rn(x[j], bo[j]);
      // (the token has a position of its own before this one, or there is none here)
      const bool copy = FORM == kAny ? (j & 3) < held : FORM == kGroups && q >= t.V;
      const bool out = copy || f != f || (SEL == 2 && v == excl) || tag_test(tags, v);
      if (!out && (!has || f > m)) {
        has = true;
        m = f;
        mtok = v;
      }
    }
  }
  FrameOut o{0.0f, 0, false, 0};
  const bool any_base = __ballot(has) != 0;
  float Mb = 0.0f;
  int vbase = INT_MAX;
  if (any_base) {
    Mb = ukey_val(wave_max_u(has ? ukey(m) : 0u));
    vbase = wave_min_nn((has && m == Mb) ? mtok : INT_MAX);
  }
  const bool mine0 = btok != INT_MAX;
  const bool any_arc = __ballot(mine0) != 0;
  float MA = 0.0f;
  int va = INT_MAX, achild = 0;
  if (any_arc) {
    MA = ukey_val(wave_max_u(mine0 ? ukey(bf) : 0u));
    const bool mine = mine0 && bf == MA;
    va = wave_min_nn(mine ? btok : INT_MAX);
    achild = __builtin_amdgcn_readlane(bchild, first_lane(__ballot(mine && btok == va)));
  }
  if (any_arc && (!any_base || MA > Mb || (MA == Mb && va < vbase))) {
    o = FrameOut{MA, va, true, achild};
  } else if (any_base) {
    o = FrameOut{Mb, vbase, false, 0};
  }  // (no candidate at all: only with NaN rows, a precondition violation; token 0 keeps the result in range)
  o.val = uniform_f(o.val);
  o.tok = uniform_i(o.tok);
  o.child = uniform_i(o.child);
  return o;
}

// Root scores of four positions (from i, a multiple of 4) for the pass over a row: NaN in the blank and EOS columns
// (those two tokens are candidates of their own, see special_candidate) and in the copies behind the end of the row.
template <int FORM>
__device__ __forceinline__ float4 mask_special(const TreeView& t, int i, float4 q) {
  const int first = FORM != kAny ? i : min(i, t.V - 4);
  float e[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (first + k == t.blank || first + k == t.eos || (FORM == kAny && k < i - first)) e[k] = NAN;
  return make_float4(e[0], e[1], e[2], e[3]);
}

}  // namespace wv
}  // namespace pb
