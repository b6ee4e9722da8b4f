// Internal layout of a compiled boosting tree: host arrays plus their device mirror.
#pragma once
#include <cstdint>
#include <vector>

#include "pb.h"

namespace pb {

// One 32-byte record per state: everything a failure-chain hop needs, for the state and for the state its
// failure link leads to, so that one load serves two levels of the chain (kernels that walk level by level
// read the first half).
struct alignas(32) StateRec {
  int32_t arc_begin;  // first arc of the state in the (from_state, token)-sorted arc table
  int32_t arc_count;  // arcs leaving the state
  int32_t fail;       // failure link
  float backoff;      // backoff score paid when the state is abandoned
  int32_t f_arc_begin;  // the same four fields of state `fail`
  int32_t f_arc_count;
  int32_t f_fail;
  float f_backoff;
};

// One 8-byte record per arc; the arc with index j leads to state j + 1.
struct alignas(8) ArcRec {
  int32_t token;
  float score;
};

// One 32-byte record per token: where the root row sends the token (a depth-1 state, or the root
// itself for the c_unk self-loop) together with that state's record, so that following a root arc
// costs one load.
struct alignas(32) RootRec {
  int32_t next;       // target state
  int32_t arc_begin;  // StateRec of the target ...
  int32_t arc_count;
  int32_t fail;
  float backoff;
  float p_root;       // ... and its total backoff down to the root
  float eos_score;    // ... and its EOS boost (0 without an EOS rule)
  int32_t pad;
};

// One 16-byte slot of the table of arcs by (state, token), the root's aside: open addressing, linear probing, at most
// half full; state == -1 in an empty slot.  A deep state has few arcs and they could be searched, but the walk over a
// phrase (pb_rows.hip) follows one arc after the other, and the table makes that one access each instead of two or more.
// It lies behind the other sub-arrays on the device and its size follows from the number of states, so that DeviceTree, which
// every kernel takes by value or out of a table, has no field for it.  Only the two-pass decoder reads it: a tree of a
// vocabulary that never gets there has none, nor has one for which there is no memory, and its calls take the other decoders.
struct alignas(16) ArcSlot {
  int32_t state, token, next, pad;
};
// Slots: a power of two, at least 16 (256 bytes: what sub-arrays are aligned to); none where 32 bits do not count them.
constexpr int32_t kMaxTableStates = 1 << 30;
constexpr uint32_t arc_slots(int32_t num_states) {
  return num_states <= 8 ? 16u : num_states > kMaxTableStates ? 0u : 1u << (33 - __builtin_clz(static_cast<uint32_t>(num_states - 1)));
}
constexpr uint32_t arc_hash(int32_t state, int32_t token) {
  uint32_t h = static_cast<uint32_t>(state) * 0x9E3779B1u ^ static_cast<uint32_t>(token) * 0x85EBCA6Bu;
  h ^= h >> 15;
  return h * 0xC2B2AE35u >> 3;
}

// Whether calls on a tree of this vocabulary may take the two passes (see rows_pay and arc_key in pb_rows.hip).
constexpr int32_t kMinTableV = 128, kMaxTableV = 1 << 21;
constexpr bool wants_arc_table(int32_t vocab_size) { return vocab_size >= kMinTableV && vocab_size <= kMaxTableV; }

// Device mirror (one allocation, sub-arrays aligned to 256 bytes).
struct DeviceTree {
  const StateRec* state = nullptr;  // [N]
  const ArcRec* arc = nullptr;      // [N-1]
  const float* root_score = nullptr;  // [V]
  const int32_t* root_next = nullptr;  // [V]
  const float* p_root = nullptr;       // [N] backoff accumulated from the state down to the root (fp32, chain order)
  const RootRec* root_rec = nullptr;   // [V]
  const float* eos_score = nullptr;    // [N] boost of the EOS token in every state (Sec. II-C: largest score of the other
                                       // tokens plus the final weight of an end-of-phrase state); null without an EOS rule
  int32_t num_states = 0;
  int32_t vocab_size = 0;
  int32_t blank_id = -1;
  int32_t eos_id = -1;
  float reach = 0.0f;  // bound of |p_root + root_score| over all states and tokens (largest |p_root| plus largest |root_score|)
};

// Per-row choice among several trees (a different context list per hypothesis or utterance): row i uses
// table[ids[i]].  A null table means "the one tree passed beside it".
struct TreePick {
  const DeviceTree* table = nullptr;  // device array of `count` trees
  const int32_t* ids = nullptr;       // device array, one id per hypothesis (beam step: per utterance)
  int32_t count = 0;
};

struct HostTree {
  int32_t vocab_size = 0, blank_id = -1, eos_id = -1;
  int32_t max_depth = 0, max_fail_chain = 0, root_degree = 0;
  std::vector<StateRec> state;
  std::vector<ArcRec> arc;
  std::vector<RootRec> root_rec;
  std::vector<int32_t> arc_begin, arc_count, fail, depth, parent, arc_token, root_next;
  std::vector<float> backoff, arc_score, root_score, p_root, final_score, eos_score;
  std::vector<uint8_t> is_final;
  std::vector<double> acc;
};

// Alg. 1 Stages 1-2 on the host.  Returns a pb_status.
int compile_tree(const int32_t* tokens, const int64_t* offsets, int64_t n_phrases, const float* weights,
                 const pb_build_opts& opts, HostTree& out);
// The table of arcs by (state, token); empty where there is no memory for it or more states than 32 bits count slots for.
std::vector<ArcSlot> build_arc_table(const HostTree& tree);
// The state an arc of state s on token v leads to, 0 if there is none: what the kernel does.
int32_t find_arc(const std::vector<ArcSlot>& slots, int32_t s, int32_t v);
// Every arc but the root's is found where it leads, nothing else is in the table, and at least half of it is empty (so that
// every search ends).
bool arc_table_ok(const HostTree& tree, const std::vector<ArcSlot>& slots);

}  // namespace pb

struct pb_forest {
  pb::DeviceTree* d_table = nullptr;  // device copy of the members' DeviceTree records
  pb::DeviceTree proto;               // vocabulary size and blank id common to all members
  bool has_table = false;             // every member has its table of arcs
  int32_t count = 0;
  int device = -1;
};

struct pb_tree {
  pb::HostTree host;
  pb::DeviceTree dev;
  void* slab = nullptr;  // device allocation backing `dev`
  bool has_table = false;  // ... with the table of arcs
  int64_t device_bytes = 0;
  int device = -1;
};
