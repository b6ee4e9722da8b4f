// Which multi-frame calls go to which decoder, as far as sizes decide it (host code without HIP: the tests of the
// dispatch compile it by itself).
#pragma once
#include <cstdint>

namespace pb {

constexpr int kNarrowMaxV = 1280;    // widest row that one wave holds in registers
constexpr int kWideMaxV = 16384;     // widest row of the multi-frame wave kernels (the root scores of a row live in LDS)
constexpr int64_t kMaxThreads = 0xffffffffll;  // of a grid
constexpr int64_t kMaxWorkgroups = kMaxThreads / 1024;

// Which calls the two passes are for.  Pass 1 reads the rows at the chip's rate whatever T and B are; pass 2 has one
// workgroup per hypothesis, so its time grows with T, and past some ten thousand rows with their number, and with the arcs
// of the states that the frames sit in.  The segment decoders read the rows once and in order, but need some thousand
// segments for that rate and read again what a wrong guess has spoilt.
// Inside the lines, time of the two passes over that of the decoder that took the call before them, geometric means over 3450
// drawn calls (up to 128 hypotheses, lists of 100 .. 20000 phrases, uniform or log-depth weights, alpha 0.3 .. 1, random
// rows, phrases on 20 % of the frames or none, 60 % blanks or none), by the number of states (up to 16384 / 49152 / more):
//   T up to                  128              256              512              1024
//   single-     V <= 384     .71 .68
//   and two-         767     .63 .70 .68      .64 .72 .74
//   stage            1024    .60 .75 .74      .71 .69 .73      .61 .84 .95
//                    1280    .70 .68 .54      .66 .67 .72      .66 .81 .78      .59 .68 .80
//                    4095    .67 .59 .56      .66 .65 .68      .61 .62 .56      .54 .66 .68
//                    16384   .70 .64 .71      .75 .69 .71      .73 .69 .64      .65 .63 .68
//   CTC         V <= 256     .70 .63 .90      .75 .63 .98 (T <= 160)
//                    384     .63 .63          .60 .70 .73      .64 .67 .75
//                    767     .51 .59 .63      .59 .62 .69      .65 .61 .71
//                    1024    .49 .52          .62 .53 .59      .57 .57 .62
//                    1280    .67 .60          .66 .62 .56      .70 .68 .54      .53 .69 .62
//                    4095    .68 .63 .50      .63 .67 .59      .67 .64 .64      .57 .66 .72
//                    16384   .67 .61 .66      .65 .65          .64 .59 .58      .60 .56 .71
// One in a hundred is slower by more than 4 %, most of them log-depth weights at alpha = 1 on rows without blanks under the
// CTC rule, where nearly every frame surprises the winners (1.1 .. 1.7).  Past 1024 frames long lists lose (phrases, random
// rows and bf16 logits, 6000 / 20000 of them: V = 1152, 2000 x 1, single-stage 1.58 / 2.13, V = 1025, 2000 x 8, CTC rule 1.10 /
// 1.30, V = 2000, 2000 x 1 1.24 / 1.47) and at V <= 1280 outside the CTC rule short ones too (2000 of them 1.14), but not past
// 4096 tokens (V = 4096, 2000 x 1 .54 .58 .61).  Outside the lines single-stage calls of many rows lose (V = 1024,
// 1000 x 16 1.0 .. 1.3; V = 1025, 1000 x 128, phrases 1.3); at V <= 1024 more than 512 frames gain in part (1000 x 1: V = 768
// .59 .. .79, V = 512 .73 .. 1.3, V = 1024 .56 .. 1.2) and stay with the segment decoders.  Vocabularies past 16384 have none
// (32001, 100 x 16, two-stage: 3340 us with a workgroup per hypothesis, 65).
inline bool rows_pay(int V, int32_t T, int32_t B, int sel, int32_t num_states) {
  const int64_t rows = static_cast<int64_t>(T) * B;
  const bool ctc = sel == 2, long_list = num_states > 16384;
  if (V > kWideMaxV) return rows <= kMaxWorkgroups;
  if (V < 128 || T > 2048) return false;
  if (V <= 1024) {
    if (T > 512) return false;
    if (ctc) return rows <= (V >= 768 ? 12800 : V > 256 || T <= 160 ? 4096 : 0);
    return rows <= (V >= 768 ? 4096 : V > 384 && T <= 256 ? 2048 : V > 256 && T <= 128 ? 512 : 0);
  }
  if (T > 1024 && V < 4096 && (long_list || (V <= kNarrowMaxV && !ctc))) return false;
  if (V <= kNarrowMaxV) return rows <= (ctc ? 131072 : 4096);
  return rows <= (ctc || V >= 4096 || T <= 128 ? 20480 : 8192);
}

}  // namespace pb
