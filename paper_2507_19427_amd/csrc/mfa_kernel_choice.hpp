// Which kernel an attention call over an 8-bit or 4-bit cache takes, from what the host knows.  Plain C++: a test checks it without a device.
#pragma once

#include <cstdint>

namespace mfa {

// short_lowbit_kernel below so many 64-token tiles per workgroup, counted at the length of the hint, else decode_lowbit_kernel.  The lines lie where lengths
// drawn from 1 .. hint, half the hint on average, no longer lose more than 1 %; lengths equal to the hint would have them lower.  us per call, short / decode, 50 sequences of the length of the hint and drawn:
//                                12 tiles                16 tiles                20 tiles                24 tiles                30 tiles
//   8 bit, one token    40.2/37.8  30.9/30.2    42.8/41.7  33.6/34.4    48.9/46.9  37.1/37.7    53.9/52.2  38.2/38.4    64.2/59.9  43.5/42.0
//   4 bit, one token    35.8/34.8  28.1/28.3    41.0/40.0  32.6/31.9    44.5/43.0  34.9/35.0    49.3/46.5  36.5/36.3    56.8/50.5  41.6/40.2
//   8 bit, two tokens   52.1/47.2  39.8/37.9    62.1/54.5  45.6/42.2    71.7/63.9  50.9/45.9    80.6/72.4  53.3/48.3    94.6/84.5  63.1/55.8
//   4 bit, two tokens   46.7/44.9  35.5/36.4    53.8/50.0  40.8/40.2    61.9/56.3  45.0/43.4    69.2/62.3  46.4/45.1    82.3/72.3  54.5/51.2
// and 64 sequences all of half, a quarter and 32 .. 64 tokens of the hint:
//                                12 tiles                16 tiles                20 tiles                24 tiles
//   4 bit, one token    22.0/21.7 17.9/19.7 13.7/15.8   24.6/23.6 18.9/19.7 13.8/15.9   26.8/25.7 20.5/21.1 13.8/15.9   28.7/28.2 22.2/21.6 13.8/16.0
//   8 bit, two tokens   34.4/33.6 27.8/29.2 17.3/20.6   39.8/36.8 30.2/31.1 17.4/20.6   43.4/40.7 32.1/33.5 17.3/20.5   46.9/43.4 34.3/33.6 17.3/20.6
//   4 bit, two tokens   30.8/34.3 25.1/26.0 16.6/20.2   34.6/36.4 27.2/28.2 16.7/20.3   38.9/37.1 29.3/30.7 16.7/20.4   43.7/40.2 31.1/32.9 16.7/20.4
// (4 bit, two tokens, 16 tiles: 36.4 against 34.6 under a hint of twice the lengths, 45.1 against 49.9 under a tight one.)
// The host knows no lengths: under a hint of four times the lengths and more, decode_lowbit_kernel costs up to a tenth, and 2 to 3.7 us at the shortest,
// whatever the size of the hint beyond the lines (at 32768: 8 bit, one token 15.4/16.7, two 18.0/21.1; 4 bit 15.0/16.8 and 17.7/20.9).  A hint near the longest
// length avoids it.  Asking only for the stages that a short segment has, instead of its last one again, changes nothing of it.
//
// Sequences of fewer than 12 tiles fill a workgroup with many segments, and decode_lowbit_kernel pays more for the start and end of each.  Lengths drawn from
// 1 .. hint, decode / short, 150 .. 4000 sequences: 5 tiles 1.03 .. 1.21, 10 tiles .96 .. 1.14, 16 tiles .92 .. 1.06; equal lengths .92 .. 1.10, the gains at
// much work and 8 bit (300 x 900, 15 tiles, two tokens: equal 71.3/75.9, drawn 55.3/54.1).  They change over later: at 48 tiles per workgroup (4 bit) and 30 (8 bit).
constexpr bool takes_short_lowbit_kernel(bool four_bit, bool one_token, int64_t tiles_per_workgroup, int64_t tiles_per_sequence)
{
    const int64_t line = one_token ? (four_bit ? 20 : 30) : (four_bit ? 16 : 12), short_sequences_line = four_bit ? 48 : 30;
    return tiles_per_workgroup < (tiles_per_sequence < 12 ? short_sequences_line : line);
}

}  // namespace mfa
