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
// of the states that the frames sit in: with the length of the lists.  The segment decoders read the rows once and in order,
// but need some thousand segments for that rate and read again what a wrong guess has spoilt.  The lines keep the calls whose
// geometric mean is below 1 over six kinds of inputs: random rows, the same from bf16 logits (equal values of tokens with
// different scores, each a pass over the row), phrases and blanks, phrases without blanks on 20 % and on all frames (uniform
// weights, alpha = 0.5), and log-depth weights at alpha = 1.  Single kinds spread around it, phrases and blanks 0.3 .. 0.9,
// log-depth weights 0.6 .. 1.5.  Time of the two passes over that of the decoder that took the call before them, lists of
// 2000 / 6000 / 20000 phrases (9500, 27000, 80000 states):
//                 T x B    100 x 4          100 x 40         250 x 8          500 x 1          500 x 8          1000 x 1
//   single-stage  V = 300  .78 .90 .98
//                 512      .82 .95 .94                         .89 1.07 1.25
//                 1024     .83 .97 .96      .87 .98 1.18     .90 1.12 1.21    .96 1.20 1.65    1.10 1.26 1.50
//                 1152     .69 .76 .61      .74 .90 1.01     .79 .95 1.04     .81 .91 1.14     .87 1.10 1.30    .87 1.14 1.51
//                 2000     .65 .71 .60      .74 .80 .69      .78 .82 .75      .76 .94 1.06     .91 1.00 1.11    .82 1.06 1.25
//                 4096                                       .79 .81 .69      .63 .67 .65      .70 .71 .69      .52 .59 .63
//   CTC           V = 200  .75 .81 .99      .81 .93 .93
//                 512      .69 .73 .73      .83 .81 .86      .96 .93 .93      .81 1.02 1.16    .95 1.08 1.37
//                 1024     .66 .70 .78      .80 .82 .90      .83 .90 .98      .85 1.03 1.11    .92 1.08 1.30
//                 1025     .75 .79 .66      .86 .86 .84      .83 .94 .76      .66 .65 .64      .78 .83 .77      .62 .77 .91
//                 2000     .71 .76 .69      .83 .82 .79      .90 .89 .84      .77 .83 .92      .80 .96 1.06     .75 .90 1.13
//                 4096     .65 .64 .66      .74 .81 .71      .70 .80 .79      .59 .62 .67      .62 .73 .73      .55 .57 .65
//                 T x B    250 x 16         500 x 24         500 x 128        1000 x 16        2000 x 1         2000 x 8
//   single-stage  V = 1152 .77 1.01 1.12                                                       1.14 1.58 2.13
//                 4096     .81 .82 .76      .93 1.01 1.02                     1.05 1.15 1.18   .54 .58 .61      .97 1.14 1.26
//   CTC           V = 1024 .83 .97 1.12     1.01 1.07 1.26
//                 1025     .86 .91 .81      .75 .84 .80      .87 .90 .87      .75 .87 1.00     .87 1.05 1.33    .93 1.10 1.30
//                 4096     .72 .75 .76      .83 .88 .93                       .88 1.00 1.05    .55 .60 .66      .90 1.03 1.16
// The two-stage rule lies between the two, nearer the single-stage one, and has its lines.  Vocabularies past 16384 have no
// segment decoder (32001, 100 x 16, two-stage: 3340 us with a workgroup per hypothesis, 65).
inline bool rows_pay(int V, int32_t T, int32_t B, int sel, int32_t num_states) {
  const int64_t rows = static_cast<int64_t>(T) * B;
  const bool ctc = sel == 2;
  const int list = num_states <= 16384 ? 0 : num_states <= 49152 ? 1 : 2;
  if (V > kWideMaxV) return rows <= kMaxWorkgroups;
  if (V < 128 || T > 2048) return false;
  if (V <= 256) return ctc && T <= 160 && rows <= 4096;
  if (V <= 1024) {
    if (ctc) return T <= (list == 0 ? 512 : 256) && rows <= (V >= 768 && list < 2 ? 12800 : 4096);
    if (V <= 384) return T <= 128 && rows <= 512;
    if (V < 768 || list == 2) return T <= (list == 0 ? 256 : 128) && rows <= 2048;
    return T <= (list == 0 ? 512 : 128) && rows <= (T <= 256 ? 4096 : 2048);
  }
  if (V <= kNarrowMaxV) {
    if (ctc) return T <= (list == 0 ? 2048 : 1024) && rows <= 131072;
    return T <= (list == 0 ? 1024 : 256) && rows <= (list < 2 ? 4096 : 2048);
  }
  if (V < 4096) {
    if (ctc) return T <= 2048 >> list && rows <= 20480;
    return T <= 1024 >> list && rows <= (T <= 128 ? 20480 : 8192);
  }
  return rows <= (T <= 512 || (ctc && (list == 0 || V >= 8192)) ? 20480 : 8192);
}

}  // namespace pb
