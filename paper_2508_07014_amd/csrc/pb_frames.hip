// Dispatch of the greedy step and the multi-frame decoder to the row shapes, the segment plan, and the beam step
// for rows of up to 1024 tokens (one wave per beam).
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstdint>
#include <random>

#include "pb_kernels.hpp"
#include "pb_wave.hpp"

namespace pb {

namespace {

using namespace wv;

// ------------------------------------------------------------------------------------------------
// Beam step, one wave per hypothesis row (V <= 1024, K <= kBeamWaveMaxK): the workgroup of an utterance
// has K waves.  Every wave forms the fused row of its beam -- base candidates in registers, the arcs
// of the failure chain scattered into an LDS overlay (value and child state per overridden token,
// deepest chain state first, later ones skipped through the token marks) -- adds the hypothesis
// score and extracts its K best totals in order by repeated wave arg-max (a taken entry becomes
// NaN, which no maximum or equality test selects).  The K*K survivors meet in LDS, and wave 0
// picks the utterance's K best by (total descending, flat index k*V+v ascending).
// A step is latency-bound, so the requests go out in the order of the single greedy step: root scores, row,
// states and hypothesis score before the first wait; an utterance with an invalid state is decoded from the
// root and marked at the end, so that no early exit separates the wave start from the requests.  The raw row
// goes into the overlay first: an arc then finds its log-prob in LDS instead of in memory.
constexpr int kBeamWaveMaxK = 8;
constexpr int kBeamWaveLdsFloats = 2 * kChunk + kTagWords;                   // overlay values, overlay children, marks
constexpr size_t kBeamCandBytes = kBeamWaveMaxK * kBeamWaveMaxK * 3 * sizeof(int);  // value, flat index, child

template <bool FULL>
__global__ void __launch_bounds__(64 * kBeamWaveMaxK) beam_wave_kernel(
    const float* __restrict__ logp, int64_t row_stride, const float* __restrict__ hyp,
    const int32_t* __restrict__ states_in, const float* __restrict__ root_score, float alpha, int K,
    int32_t* __restrict__ tokens, int32_t* __restrict__ parents, int32_t* __restrict__ states_out,
    float* __restrict__ scores_out, DeviceTree dt) {
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6);
  const int u = blockIdx.x, h = u * K + wave;
  const TreeView t = make_view(dt);
  const int V = t.V;
  const float* lrow = logp + static_cast<size_t>(h) * row_stride;
  float x[16], c[16];
  load_row<FULL>(root_score, 0, V, lane, c);  // (the tree's array, as a leading argument: in registers at the start)
  load_row<FULL>(lrow, 0, V, lane, x);
  const int sk = states_in[u * K + min(lane, K - 1)];  // every wave sees all K states
  const float hs_in = hyp[h];
  __builtin_amdgcn_sched_barrier(0);  // (all of the above is in flight before the first wait)
  // per-slot multiplier of the boost (alpha; 0 in the blank's slot), formed while the states are on their way:
  // what follows the arrival of the state's record is then two instructions per slot (see step_wave_kernel)
  float am[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    am[j] = slot_is(j, lane, t.blank) ? 0.0f : alpha;
    asm volatile("" : "+v"(am[j]));  // (formed here, not where it is used)
  }
  __builtin_amdgcn_sched_barrier(0);
  float* cand_val = lds;  // [K*K], then the flat indices and the children
  int* cand_idx = reinterpret_cast<int*>(lds + kBeamWaveMaxK * kBeamWaveMaxK);
  int* cand_nxt = cand_idx + kBeamWaveMaxK * kBeamWaveMaxK;
  float* ov = lds + 3 * kBeamWaveMaxK * kBeamWaveMaxK + wave * kBeamWaveLdsFloats;
  int* ov_next = reinterpret_cast<int*>(ov + kChunk);
  unsigned* tags = reinterpret_cast<unsigned*>(ov + 2 * kChunk);

  // an utterance with an invalid state is marked as a whole (at the end)
  const bool bad = __ballot(!valid_state(t, sk)) != 0;
  const int s = bad ? 0 : __builtin_amdgcn_readlane(sk, wave);
  const float hs = uniform_f(hs_in);
  const Cursor cur = cursor_at(t, s);
  __builtin_amdgcn_sched_barrier(0);  // (the parts of the cursor are requested together)
#pragma unroll
  for (int j = 0; j < 16; ++j) c[j] = __fmul_rn(am[j], __fadd_rn(cur.p_root, c[j]));  // base boosts, in place
  tags_clear(tags, lane);
  store_row_lds(ov, lane, x);  // the raw row: an arc reads its log-prob here and puts its fused value in its place
  // ---- overlay: arcs of the failure chain, deepest state first ------------------------------------
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
  // ---- totals of the lane's 16 tokens -------------------------------------------------------------
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
      // positions past V hold -inf: with at most V rounds the real tokens, which come first, are taken before them
      tv[4 * i + k] = (FULL || v0 + k < V) ? __fadd_rn(hs, expansion) : -INFINITY;
    }
  }
  if (t.eos >= 0) {  // EOS rule (Sec. II-C): boosted by the value tabulated for the state; no arc carries the token
    const float ce = __fmul_rn(alpha, cur.eos_boost);
    const int ln = opaque(lane);
#pragma unroll
    for (int j = 0; j < 16; ++j) tv[j] = slot_is(j, ln, t.eos) ? __fadd_rn(hs, __fadd_rn(x[j], ce)) : tv[j];
  }
  // ---- the row's best totals, in order ---------------------------------------------------------------
  const int rounds = min(K, V);
  for (int r = 0; r < rounds; ++r) {
    float g[4];
    const float M = ukey_val(wave_max_u(ukey(group_maxima(tv, g))));
    const int v = uniform_i(first_pos_equal(tv, g, M, lane));
    int nx = s;  // the blank and the EOS keep the state
    if (v != t.blank && v != t.eos) nx = tag_test(tags, v) ? ov_next[v] : t.root_next[v];
    if (lane == 0) {  // `rounds` entries per wave, packed
      cand_val[wave * rounds + r] = M;
      cand_idx[wave * rounds + r] = wave * V + v;
      cand_nxt[wave * rounds + r] = nx;
    }
    const int taken = slot_in_lane(opaque(lane), v);
#pragma unroll
    for (int j = 0; j < 16; ++j) tv[j] = taken == j ? NAN : tv[j];
  }
  __syncthreads();
  if (wave != 0) return;
  // ---- merge: one candidate per lane ------------------------------------------------------------------
  const int n = K * rounds;
  const bool have = lane < n;
  float val = have ? cand_val[lane] : 0.0f;
  const int idx = have ? cand_idx[lane] : INT_MAX;
  const int nxt = have ? cand_nxt[lane] : 0;
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

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

bool wave_path_ok(const DeviceTree& t) {
  return t.p_root != nullptr && t.root_rec != nullptr && t.vocab_size >= 4 && t.vocab_size <= kWideMaxV;
}

bool step_wave_ok(const DeviceTree& t) {
  return t.p_root != nullptr && t.root_rec != nullptr && t.vocab_size >= 4 && t.vocab_size <= kStepMaxV;
}

SegPlan plan_segments(int32_t T, int32_t B, int target_chains) {
  // Segments: enough concurrent chains to cover the memory latency, at most kMaxSegments per
  // hypothesis, at least kMinSegLen frames long.
  int nseg = (target_chains + B - 1) / B;
  nseg = nseg < 1 ? 1 : (nseg > kMaxSegments ? kMaxSegments : nseg);
  int seg_len = (T + nseg - 1) / nseg;
  if (seg_len < kMinSegLen) seg_len = kMinSegLen;
  nseg = (T + seg_len - 1) / seg_len;
  return SegPlan{nseg, seg_len};
}

// Row shape of a narrow row (see pb_narrow.hpp).  Aligned rows of 1024 tokens keep the form without clamps and copies;
// everything else runs the clamped form with as many positions per lane as it needs (V = 193, B = 804, a table of
// trees: 6.2 us with four, 7.1 with sixteen, 6.6 with the workgroup-per-row kernel it replaces; V = 1025: a step of
// B = 128 8.0 -> 4.8 us, 500 frames x 32 utterances under the CTC rule 1880 -> 119 us).
static int narrow_shape(const DeviceTree& t, const float* d_logp, int64_t frame_stride, int64_t row_stride) {
  if (t.vocab_size <= 512) return t.vocab_size <= 256 ? 3 : 4;
  if (t.vocab_size > 1024) return 2;
  return t.vocab_size == 1024 && row_stride % 4 == 0 && frame_stride % 4 == 0 && aligned16(d_logp) && aligned16(t.root_score) ? 0 : 1;
}

int launch_step_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride,
                     const int32_t* d_states_in, const int32_t* d_last, float alpha, int32_t B, int sel, int32_t* d_tokens,
                     int32_t* d_states_out, float* d_scores, hipStream_t stream) {
  if (t.vocab_size > kNarrowMaxV)
    return launch_step_wide(t, pick, d_logp, row_stride, d_states_in, d_last, alpha, B, sel, d_tokens, d_states_out,
                            d_scores, stream);
  const int row = narrow_shape(t, d_logp, 0, row_stride);
  constexpr decltype(&launch_step_row<0>) by_shape[] = {launch_step_row<0>, launch_step_row<1>, launch_step_row<2>,
                                                        launch_step_row<3>, launch_step_row<4>};
  return by_shape[row](t, pick, d_logp, row_stride, d_states_in, d_last, alpha, B, sel, d_tokens, d_states_out, d_scores, stream);
}

// A number that no earlier call of this process has used: a counter from a random 64-bit start.
uint64_t next_call_tag() {
  static std::atomic<uint64_t> counter{[] {
    std::random_device rd;
    const uint64_t a = rd(), b = rd();
    return (a << 32) ^ b ^ static_cast<uint64_t>(std::chrono::steady_clock::now().time_since_epoch().count());
  }()};
  return counter.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);  // (odd step: all 2^64 values in turn)
}

int64_t frames_workspace_bytes(const DeviceTree& t, int32_t T, int32_t B) {
  if (t.vocab_size > 1024) return 0;  // (wider rows repair wrong guesses in pass 2)
  const SegPlan plan = plan_segments(T, B, kTargetChains);
  return static_cast<int64_t>(plan.nseg - 1) * B * (kPatchInts + kStartInts) * static_cast<int64_t>(sizeof(int32_t));
}

int launch_frames_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                       int64_t row_stride,
                       const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T, int32_t B, int sel,
                       int32_t* d_tokens, int32_t* d_states, float* d_scores, int32_t* d_patches, hipStream_t stream) {
  if (t.vocab_size > kNarrowMaxV)
    return launch_frames_wide(t, pick, d_logp, frame_stride, row_stride, d_states0, d_last0, alpha, T, B, sel, d_tokens,
                              d_states, d_scores, stream);
  const unsigned tag_lo = static_cast<unsigned>(next_call_tag());  // marks the start records of this call (see kStartInts)
  const int row = narrow_shape(t, d_logp, frame_stride, row_stride);
  constexpr decltype(&launch_frames_row<0>) by_shape[] = {launch_frames_row<0>, launch_frames_row<1>, launch_frames_row<2>,
                                                          launch_frames_row<3>, launch_frames_row<4>};
  return by_shape[row](t, pick, d_logp, frame_stride, row_stride, d_states0, d_last0, alpha, T, B, sel, tag_lo, d_tokens,
                       d_states, d_scores, d_patches, stream);
}

int g_beam_wave_max_k = 7;  // widest beam the wave kernel's LDS allows on the device, set once

bool beam_wave_ok(const DeviceTree& t, const float* d_logp, int64_t row_stride, int32_t K) {
  return wave_path_ok(t) && t.vocab_size % 4 == 0 && row_stride % 4 == 0 && aligned16(d_logp) && aligned16(t.root_score) &&
         t.vocab_size <= kChunk && K <= g_beam_wave_max_k;
}

int launch_beam_wave(const DeviceTree& t, const float* d_logp, int64_t row_stride, const float* d_hyp,
                     const int32_t* d_states_in, float alpha, int32_t U, int32_t K, int32_t* d_tokens,
                     int32_t* d_parents, int32_t* d_states_out, float* d_scores_out, hipStream_t stream) {
  const size_t lds = kBeamCandBytes + static_cast<size_t>(K) * kBeamWaveLdsFloats * sizeof(float);
  const dim3 grid(static_cast<unsigned>(U)), block(static_cast<unsigned>(64 * K));
  if (t.vocab_size == kChunk)
    hipLaunchKernelGGL(beam_wave_kernel<true>, grid, block, lds, stream, d_logp, row_stride, d_hyp, d_states_in,
                       t.root_score, alpha, K, d_tokens, d_parents, d_states_out, d_scores_out, t);
  else
    hipLaunchKernelGGL(beam_wave_kernel<false>, grid, block, lds, stream, d_logp, row_stride, d_hyp, d_states_in,
                       t.root_score, alpha, K, d_tokens, d_parents, d_states_out, d_scores_out, t);
  return hipGetLastError() == hipSuccess ? PB_OK : PB_EHIP;
}

int prepare_wave_kernels() {
  int dev = 0, max_lds = 0;
  if (hipGetDevice(&dev) != hipSuccess) return PB_EHIP;
  if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return PB_EHIP;
  constexpr int kPlainLimit = 64 * 1024 - 1024;  // static LDS of the kernel included
  // The beam kernel with kBeamWaveMaxK waves needs a little more than 64 KiB.
  const int beam_bytes = static_cast<int>(kBeamCandBytes + kBeamWaveMaxK * kBeamWaveLdsFloats * sizeof(float));
  g_beam_wave_max_k = static_cast<int>((kPlainLimit - kBeamCandBytes) / (kBeamWaveLdsFloats * sizeof(float)));
  if (beam_bytes <= max_lds) {
    const hipFuncAttribute attr = hipFuncAttributeMaxDynamicSharedMemorySize;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(beam_wave_kernel<true>), attr, beam_bytes) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(beam_wave_kernel<false>), attr, beam_bytes) == hipSuccess)
      g_beam_wave_max_k = kBeamWaveMaxK;
    else
      (void)hipGetLastError();
  }
  const int rc = prepare_wide_kernels(max_lds);
  return rc == PB_OK ? prepare_rows_kernels(max_lds) : rc;
}

}  // namespace pb
