// The wave-per-hypothesis kernels for rows of 516 .. 1020 tokens, a multiple of 4, 16-byte aligned (see pb_narrow.hpp).
#include "pb_narrow.hpp"

namespace pb {
template int launch_step_row<5>(const DeviceTree&, const TreePick&, const float*, int64_t, const int32_t*,
                                const int32_t*, float, int32_t, int, int32_t*, int32_t*, float*, hipStream_t);
template int launch_frames_row<5>(const DeviceTree&, const TreePick&, const float*, int64_t, int64_t, const int32_t*,
                                  const int32_t*, float, int32_t, int32_t, int, unsigned, int32_t*, int32_t*, float*,
                                  int32_t*, hipStream_t);
}  // namespace pb
