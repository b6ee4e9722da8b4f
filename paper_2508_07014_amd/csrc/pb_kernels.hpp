// Launch wrappers of the HIP kernels (defined in pb_kernels.hip).  Each returns a pb_status.
#pragma once
#include <hip/hip_runtime.h>

#include "pb_lines.hpp"
#include "pb_tree.hpp"

namespace pb {

// The tree of row i: `t` as passed, or table[ids[i]] when a table is given.  False for an id outside the table.
__device__ __forceinline__ bool pick_tree(const TreePick& p, int i, DeviceTree& t) {
  if (p.table == nullptr) return true;
  const int32_t id = p.ids[i];
  if (static_cast<uint32_t>(id) >= static_cast<uint32_t>(p.count)) return false;
  t = p.table[id];
  return true;
}

constexpr int kMaxChunk = 8192;   // tokens per LDS pass of the fused kernels (64 KiB of 8-byte entries)
#ifndef PB_SCORE_TILE
#define PB_SCORE_TILE 2048
#endif
constexpr int kScoreTile = PB_SCORE_TILE;  // tokens per workgroup of the score kernel (16 KiB of LDS)

int launch_score(const DeviceTree& t, const TreePick& pick, const int32_t* d_states, int32_t B, float* d_scores,
                 int32_t* d_next, hipStream_t stream);

// T == 1 with frame_stride == 0 is the single step.  sel is an enum pb_select_mode value; d_last0 (previous
// labels, CTC rule only) may be null.
int launch_fuse(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride, int64_t row_stride,
                const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T, int32_t B, int sel,
                int32_t* d_tokens, int32_t* d_states, float* d_scores, hipStream_t stream);

// Wave-per-hypothesis greedy kernels (pb_frames.hip, pb_narrow.hpp, pb_wide.hip).
#ifndef PB_TARGET_CHAINS
#define PB_TARGET_CHAINS 4096
#endif
constexpr int kTargetChains = PB_TARGET_CHAINS;  // concurrent decode chains aimed for by the multi-frame decoder
constexpr int kMinSegLen = 8;        // shortest speculative segment, in frames
constexpr int kMaxSegments = 64;     // segments per hypothesis (one lane each in the validation pass)

constexpr int kStepMaxV = 65536;     // widest row of the single step that one workgroup holds in registers
#ifndef PB_WIDE_TARGET_CHAINS
#define PB_WIDE_TARGET_CHAINS 1024
#endif
constexpr int kWideTargetChains = PB_WIDE_TARGET_CHAINS;  // the same for rows wider than kNarrowMaxV (one wave per SIMD:
                                                          // a wave keeps three 4-KiB chunks of its rows in flight)

struct SegPlan {
  int nseg, seg_len;  // segments per hypothesis and their nominal length
};
// First frame of segment j of nseg (j == nseg: T).  The frames are split evenly, then tapered: the first segment is
// 1/kSegTaper longer than the mean, the last one as much shorter, linearly in between.  The chains of a call are
// launched in segment order and a SIMD serves older waves first -- measured, the waves launched first run about 5 %
// faster than those launched last -- so equal segments would end the kernel with the youngest waves alone on the chip.
#ifndef PB_SEG_TAPER
#define PB_SEG_TAPER 20
#endif
constexpr int kSegTaper = PB_SEG_TAPER;
__host__ __device__ inline int seg_begin(int j, int T, int nseg) {
  const long long even = static_cast<long long>(j) * T / nseg;
  const long long bulge = kSegTaper > 0 ? static_cast<long long>(T) * j * (nseg - j) / (static_cast<long long>(kSegTaper) * nseg * nseg) : 0;
  return static_cast<int>(even + bulge);
}
SegPlan plan_segments(int32_t T, int32_t B, int target_chains);
// The chains aimed for by vocabulary size: what the chip holds at the kernels' waves per SIMD.
inline int narrow_target_chains(int V) { return V <= 1024 ? kTargetChains : kTargetChains / 2; }
inline int target_chains(int V) { return V <= kNarrowMaxV ? narrow_target_chains(V) : kWideTargetChains; }

// Rows of any stride and alignment, for vocabularies of 4 .. kWideMaxV (single step: kStepMaxV) tokens.
bool wave_path_ok(const DeviceTree& t);
bool step_wave_ok(const DeviceTree& t);
// Rows wider than kNarrowMaxV tokens (pb_wide.hip); same arguments as the calls below, which forward to them.
int prepare_wide_kernels(int max_lds_bytes);
int launch_step_wide(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride,
                     const int32_t* d_states_in, const int32_t* d_last, float alpha, int32_t B, int sel,
                     int32_t* d_tokens, int32_t* d_states_out, float* d_scores, hipStream_t stream);
int launch_frames_wide(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                       int64_t row_stride, const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T,
                       int32_t B, int sel, int32_t* d_tokens, int32_t* d_states, float* d_scores, hipStream_t stream);
int prepare_wave_kernels();  // once per device, after the device has been made current
int launch_step_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride,
                     const int32_t* d_states_in,
                     const int32_t* d_last, float alpha, int32_t B, int sel, int32_t* d_tokens, int32_t* d_states_out,
                     float* d_scores, hipStream_t stream);
// The narrow kernels, one instantiation per row shape (pb_narrow.hpp).
template <int ROW>
int launch_step_row(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride,
                    const int32_t* d_states_in, const int32_t* d_last, float alpha, int32_t B, int sel,
                    int32_t* d_tokens, int32_t* d_states_out, float* d_scores, hipStream_t stream);
template <int ROW>
int launch_frames_row(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                      int64_t row_stride, const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T,
                      int32_t B, int sel, unsigned tag_lo, int32_t* d_tokens, int32_t* d_states, float* d_scores,
                      int32_t* d_patches, hipStream_t stream);
// d_patches: optional workspace of frames_workspace_bytes(t, T, B) bytes (null: wrong boundary guesses are
// repaired by re-runs in pass 2 instead of patches from pass 1).
int64_t frames_workspace_bytes(const DeviceTree& t, int32_t T, int32_t B);
int launch_frames_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                       int64_t row_stride,
                       const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T, int32_t B, int sel,
                       int32_t* d_tokens, int32_t* d_states, float* d_scores, int32_t* d_patches, hipStream_t stream);

// A grid counts its threads in 32 bits, and a larger one is cut without an error: the workgroups behind the cut never
// run.  kMaxWorkgroups of any size fit; steps, beam steps and dense rows of more rows go out in slices, and the
// multi-frame kernels, whose outputs interleave the hypotheses, check (grid_fits).
inline bool grid_fits(int64_t groups, int64_t threads) { return groups <= kMaxThreads / threads; }

// Whether the outputs of a multi-frame call lie apart from its start states, previous labels and tree ids and from each
// other.  Those that do not go to launch_fuse, whose workgroups read what they start from before they write: the others
// decode a hypothesis in several waves, which write later frames while the first one, or a boundary guess, may still
// have the start states to read.
bool frames_apart(const TreePick& pick, const int32_t* d_states0, const int32_t* d_last0, int32_t T, int32_t B,
                  const int32_t* d_tokens, const int32_t* d_states, const float* d_scores);

// Multi-frame decoding in two passes, all rows and then the automaton (pb_rows.hip): whether a call takes it, and the
// launch.  The outputs hold the rows' winners in between: calls with frames_apart only.
int prepare_rows_kernels(int max_lds_bytes);
bool frames_rows_ok(const DeviceTree& t, int32_t T, int32_t B, int sel);
int launch_frames_rows(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t frame_stride,
                       int64_t row_stride, const int32_t* d_states0, const int32_t* d_last0, float alpha, int32_t T,
                       int32_t B, int sel, int32_t* d_tokens, int32_t* d_states, float* d_scores, hipStream_t stream);

// Beam step on waves (pb_beam.hip): rows of any stride and alignment, vocabularies of 4 tokens up to what the token
// marks of the beams leave room for in LDS; launch_beam takes the rest.
int prepare_beam_kernels(int max_lds_bytes);
bool beam_wave_ok(const DeviceTree& t, int32_t U, int32_t K);
int launch_beam_wave(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride, const float* d_hyp,
                     const int32_t* d_states_in, float alpha, int32_t U, int32_t K, int32_t* d_tokens,
                     int32_t* d_parents, int32_t* d_states_out, float* d_scores_out, hipStream_t stream);

int launch_beam(const DeviceTree& t, const TreePick& pick, const float* d_logp, int64_t row_stride, const float* d_hyp,
                const int32_t* d_states_in, float alpha, int32_t U, int32_t K, int32_t* d_tokens, int32_t* d_parents,
                int32_t* d_states_out, float* d_scores_out, hipStream_t stream);

}  // namespace pb
