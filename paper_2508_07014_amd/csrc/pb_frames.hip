// Dispatch of the greedy step and the multi-frame decoder to the row shapes, and the segment plan.
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

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

bool wave_path_ok(const DeviceTree& t) {
  return t.p_root != nullptr && t.root_rec != nullptr && t.vocab_size >= 4 && t.vocab_size <= kWideMaxV;
}

bool step_wave_ok(const DeviceTree& t) {
  return t.p_root != nullptr && t.root_rec != nullptr && t.vocab_size >= 4 && t.vocab_size <= kStepMaxV;
}

bool frames_apart(const TreePick& pick, const int32_t* d_states0, const int32_t* d_last0, int32_t T, int32_t B,
                  const int32_t* d_tokens, const int32_t* d_states, const float* d_scores) {
  struct Range {
    uintptr_t at;
    size_t bytes;
  };
  auto range = [](const void* p, size_t n) { return Range{reinterpret_cast<uintptr_t>(p), p != nullptr ? n * 4 : 0}; };
  const size_t n = static_cast<size_t>(T) * static_cast<size_t>(B), rows = static_cast<size_t>(B);
  const Range out[] = {range(d_tokens, n), range(d_states, n), range(d_scores, n)};
  const Range in[] = {range(d_states0, rows), range(d_last0, rows), range(pick.ids, rows)};
  auto apart = [](const Range& a, const Range& b) {
    return a.bytes == 0 || b.bytes == 0 || a.at + a.bytes <= b.at || b.at + b.bytes <= a.at;
  };
  bool ok = apart(out[0], out[1]) && apart(out[0], out[2]) && apart(out[1], out[2]);
  for (const Range& o : out)
    for (const Range& i : in) ok = ok && apart(o, i);
  return ok;
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

// Row shape of a narrow row (see pb_narrow.hpp).  Aligned rows of 513 .. 1024 tokens keep the forms without clamps and
// copies (the clamped one spills in the multi-frame decoder: V = 1000, 1000 frames x 128 128 us against 109, under the CTC
// rule 205 against 127); everything else runs the clamped form with as many positions per lane as it needs (V = 193, B = 804, a table of
// trees: 6.2 us with four, 7.1 with sixteen, 6.6 with the workgroup-per-row kernel it replaces; V = 1025: a step of
// B = 128 8.0 -> 4.8 us, 500 frames x 32 utterances under the CTC rule 1880 -> 119 us).
static int narrow_shape(const DeviceTree& t, const float* d_logp, int64_t frame_stride, int64_t row_stride) {
  if (t.vocab_size <= 512) return t.vocab_size <= 256 ? 3 : 4;
  if (t.vocab_size > 1024) return 2;
  const bool aligned = t.vocab_size % 4 == 0 && row_stride % 4 == 0 && frame_stride % 4 == 0 && aligned16(d_logp) && aligned16(t.root_score);
  return !aligned ? 1 : t.vocab_size == 1024 ? 0 : 5;
}

int launch_step_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride,
                     const int32_t* d_states_in, const int32_t* d_last, float alpha, int32_t B, int sel, int32_t* d_tokens,
                     int32_t* d_states_out, float* d_scores, hipStream_t stream) {
  if (t.vocab_size > kNarrowMaxV)
    return launch_step_wide(t, pick, d_logp, row_stride, d_states_in, d_last, alpha, B, sel, d_tokens, d_states_out,
                            d_scores, stream);
  const int row = narrow_shape(t, d_logp, 0, row_stride);
  constexpr decltype(&launch_step_row<0>) by_shape[] = {launch_step_row<0>, launch_step_row<1>, launch_step_row<2>,
                                                        launch_step_row<3>, launch_step_row<4>, launch_step_row<5>};
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
                                                          launch_frames_row<3>, launch_frames_row<4>, launch_frames_row<5>};
  return by_shape[row](t, pick, d_logp, frame_stride, row_stride, d_states0, d_last0, alpha, T, B, sel, tag_lo, d_tokens,
                       d_states, d_scores, d_patches, stream);
}

int prepare_wave_kernels() {
  int dev = 0, max_lds = 0;
  if (hipGetDevice(&dev) != hipSuccess) return PB_EHIP;
  if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return PB_EHIP;
  int rc = prepare_wide_kernels(max_lds);
  if (rc == PB_OK) rc = prepare_rows_kernels(max_lds);
  if (rc == PB_OK) rc = prepare_beam_kernels(max_lds);
  return rc;
}

}  // namespace pb
