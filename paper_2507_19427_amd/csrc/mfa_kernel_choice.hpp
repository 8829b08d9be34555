// Which kernel an attention call takes, from what the host knows.  Plain C++: a test checks it without a device.
#pragma once

#include <cstdint>

namespace mfa {

// Short contexts: into how many workgroups brief_attn_kernel cuts a row (a query token of a sequence), or 0 where the kernels that cut the cache
// are ahead.  As many as leave a workgroup per compute unit, 16 at most: each part reads all keys of its row.
//
// The lines, in tokens of the hint, lie where equal lengths and lengths drawn from 1 .. hint gain, and one sequence of the hint's length among others of 32 tokens loses little (7 % at the very
// most, mostly nothing): uncut, a long row has its fixed share of the chip, where the balanced schedule gives it most of it.  us per call, the other kernels (streaming kernel and merge) / this one;
// in brackets what lies beyond a line.  Equal and drawn lengths:
//   bf16, one token    2 x 256  9.8/6.6     2 x 1024  11.6/11.0 11.7/10.9    (3 x 1280  12.4/12.6 12.2/12.3)    (6 x 1536  17.2/13.8 15.9/13.5    16 x 1536  18.3/16.5 19.1/14.1: runs, below)
//                      47 x 960  23.0/17.6 19.1/17.8    64 x 896  24.3/16.9 21.9/16.8    (64 x 960  24.5/18.2 21.8/18.0    64 x 1152  26.9/20.6 23.1/20.2    64 x 1536  30.0/24.2 25.5/22.9)
//                      128 x 384  23.5/17.6 22.4/18.2    (66 x 512  20.7/18.1 19.7/18.6    128 x 512  26.1/20.2 24.2/20.3    128 x 768  31.1/24.8 27.1/24.6)
//   8 bit, one token   2 x 256  10.9/6.2    1 x 1280  12.3/11.6     (1 x 1536  12.5/12.9)    18 x 2048  20.3/18.3 18.0/17.4    47 x 1536  23.4/18.8 19.4/18.0    64 x 1408  25.7/19.1 21.5/17.2
//                      (48 x 2048  28.4/22.5 22.0/22.1    64 x 1536  24.0/19.1 21.6/18.6    64 x 1792  26.1/21.6 22.0/20.7)    (99 x 512  23.3/17.8 20.8/18.2    128 x 640  24.2/20.8 23.7/21.0)
//   4 bit, one token   1 x 1536  12.3/11.9    (1 x 1792  12.3/13.1)    32 x 2048  20.5/17.9 17.6/16.1    34 x 1536  20.2/17.0 17.0/15.4    64 x 1792  23.1/19.1 20.6/18.8    (64 x 2048  24.3/21.3 21.6/20.9)
//                      128 x 512  21.5/17.0 21.7/17.2    (128 x 768  23.7/21.0 23.2/21.2)
//   two tokens within 1 us of twice the sequences
// One sequence of the hint's length, the others of 32 tokens, contiguous and paged:
//   bf16               16 x 1152  16.9/11.3 16.0/11.2    32 x 1536  17.5/17.5 16.8/16.7    47 x 960  16.7/16.4 15.6/15.8    64 x 896  16.7/15.3 15.7/14.6    (64 x 960  16.7/17.0 15.7/16.8    64 x 1152  17.3/18.8    64 x 1536  18.1/22.1)
//                      71 x 384  15.4/14.8 14.8/14.7    128 x 384  17.1/16.6 16.0/15.8    (66 x 512  15.9/16.9    128 x 448  16.7/18.5    128 x 768  17.4/23.0)
//   8 bit              32 x 2048  17.8/17.6 18.3/17.3    47 x 1536  16.8/17.3 17.3/16.8    64 x 1408  16.9/16.4 17.4/15.7    (64 x 1536  17.0/18.2 17.4/17.5    64 x 1792  17.5/19.5)    71 x 384  15.2/13.9 15.6/14.1
//                      128 x 384  16.0/15.1 16.4/15.2    (72 x 512  15.1/16.2 15.5/16.8    128 x 640  16.8/19.0)
//   4 bit              32 x 2048  17.6/16.0 18.1/16.2    64 x 1792  17.5/17.5 17.8/17.5    (64 x 2048  17.9/19.0)    71 x 512  14.9/15.3 15.4/15.4    128 x 512  15.8/16.0 16.2/15.9    (128 x 768  16.4/19.3)
//   two tokens         bf16 17 x 960  16.2/16.2 15.2/16.0    32 x 896  19.2/15.8 18.2/15.5    33 x 384  15.2/15.3 14.6/15.6   8 bit 32 x 1408  19.5/16.4 19.7/16.3
//   three and four     bf16, four 16 x 1536  26.5/22.7 26.6/22.5    24 x 768  25.0/23.2 25.1/22.8    17 x 512  20.9/18.1 21.1/17.9    (17 x 768  21.4/22.8 21.8/23.5)    three 24 x 768  22.0/22.5 22.0/22.4    33 x 768  22.7/23.3 22.7/22.9
//                      8 bit, four 16 x 6144  56.0/51.4 56.5/51.4    32 x 1792  39.1/39.2 39.9/39.8    (32 x 2048  40.6/43.4)    4 bit, four 32 x 2048  39.5/39.3 40.5/40.4
// Three and four tokens: the other kernels have more to merge (bf16) or take two passes (8 and 4 bit).  (With weights rounded to bf16 and rolled loads, up to a tenth slower
// than now; equal and drawn lengths:)
//   bf16, four   1 x 2048  20.7/17.9    8 x 2048  34.8/22.7 31.7/22.1    16 x 1536  36.3/25.9 33.4/25.0    64 x 256  36.9/29.0 31.8/26.7      three  33 x 768  31.7/25.6 28.1/25.3
//   8 bit, four  1 x 4096  31.7/27.5    (1 x 6144  36.9/38.7)    4 x 6144  46.7/41.0 48.9/38.6    8 x 6144  52.4/43.9 50.5/43.2    16 x 6144  66.0/54.8 55.5/53.1    32 x 1792  54.4/40.5 47.9/39.9    (32 x 2048  54.8/44.8 45.7/43.7)
//                64 x 1024  60.6/53.7 54.7/48.2
//   4 bit, four  1 x 4096  30.9/24.6    4 x 6144  45.4/38.1 47.9/36.7    8 x 6144  49.2/39.8 49.2/39.3    16 x 6144  60.6/47.1 52.1/46.3    32 x 2048  54.2/39.9 42.9/38.8    (64 x 2048  72.4/76.8 60.9/68.6)
//   8 bit, three  128 x 256  53.6/37.1 54.1/35.9
// Up to 32 rows the lines lie lower than these figures would have them, where brief_runs (below) has something better.
constexpr int kBriefBands = 11;
constexpr int kBriefRows[kBriefBands] = {4, 16, 21, 32, 47, 64, 71, 99, 128, 256, 384};
constexpr int kBriefParts[kBriefBands] = {16, 16, 8, 8, 4, 4, 2, 2, 2, 2, 2};
constexpr int kBriefLines[2][3][kBriefBands] = {                        // [three or four tokens][16, 8, 4 bits]
    {{768, 1152, 1280, 1536, 960, 896, 384, 384, 384, 0, 0}, {896, 1280, 1536, 2048, 1536, 1408, 384, 384, 384, 0, 0}, {1024, 1280, 1536, 2048, 1536, 1792, 512, 512, 512, 0, 0}},
    {{768, 1152, 1280, 2048, 1536, 1536, 512, 768, 768, 256, 0}, {896, 1280, 1536, 2048, 6144, 6144, 1792, 1792, 1792, 1024, 256}, {1024, 1280, 1536, 2048, 6144, 6144, 2048, 2048, 2048, 1024, 256}}};
constexpr int brief_parts(int bits, int q_len, int64_t rows, int64_t hint)
{
    for (int band = 0; band < kBriefBands; ++band)
        if (rows <= kBriefRows[band]) return hint <= kBriefLines[q_len >= 3][bits == 16 ? 0 : bits == 8 ? 1 : 2][band] ? kBriefParts[band] : 0;
    return 0;
}

// Beyond those lines, up to 32 rows (21 with one token, or two of longer contexts): into how many runs brief_attn_kernel cuts a row, or 0 where the other kernels are ahead.  A run takes
// kBriefCutParts workgroups; the runs of all rows fill the compute units once (a second round is a loss: 2 x 8192 with 32 runs 13.2, with 48 19.2), but with no
// less than 64 tokens each, 128 from three rows on (5 x 1536, of 12/9/6 runs 11.8/12.2/11.9 us, drawn 11.5/11.7/11.9; 8 x 2048, of 8/6/4 13.1/13.8/14.8; 3 x 1024, of 16/8 bf16 9.8/10.0, 8 bit
// 9.7/9.6).  Each compute unit reads rows * hint / 64 tokens' keys and values
// whole, through its own 107 GB/s: that is what the limits on rows * hint are.  us per call, uncut / the other kernels / runs, equal and drawn lengths:
//   bf16, one token    1 x 512 8.2/10.5/8.5   1 x 1024 10.9/11.4/9.2   1 x 1536 13.5/11.5/9.0   1 x 4096 -/12.7/10.8   1 x 32768 -/22.0/16.5   2 x 8192 -/18.1/13.7 -/18.9/13.7   4 x 768 10.1/12.4/10.2
//                      4 x 16384 -/25.1/22.3 -/22.5/21.9   (4 x 32768 -/34.6/37.2 -/27.7/32.5)   5 x 1536 13.9/16.2/11.9 13.4/14.1/12.0   8 x 8192 -/25.4/22.1 -/22.2/21.5   (8 x 16384 -/35.2/37.0)
//                      12 x 1024 12.6/17.1/13.2 11.2/15.8/12.8   12 x 2048 19.3/18.9/15.3 17.7/18.3/14.9   (16 x 4096 -/25.0/21.7 -/21.5/21.1, 16 x 8192 -/34.5/37.7 -/26.1/31.7)   20 x 2048 21.9/21.3/18.6
//                      20.5/19.8/17.6   (drawn: 10 x 6500 -/21.3/21.6   19 x 3400 -/21.3/22.6)   (24 x 2048, two runs 21.8/23.3/21.5 20.7/20.6/20.9)
//   8 bit, one token   1 x 32768 -/22.3/15.0   4 x 2048 16.0/17.2/11.7 15.5/14.4/11.3   16 x 2048 17.6/20.2/14.7 15.9/19.2/14.5   16 x 4096 -/22.2/18.5 -/20.1/18.3   (16 x 8192 -/27.9/26.3 -/22.9/25.9)
//   two tokens         bf16 2 x 8192 -/22.8/16.4 -/22.0/16.2   8 x 4096 -/24.2/22.0 -/24.7/21.2   8 bit 8 x 4096 -/24.5/18.4 -/23.7/18.4   11 x 2700 -/25.3/20.6 -/23.3/20.2   16 x 2700 -/26.0/21.8 -/22.7/20.7
//                      (12 x 3400 -/25.4/24.7 -/22.7/24.0)   bf16 16 x 2048 22.9/25.8/23.4 21.2/24.2/21.5   (16 x 3072 -/27.8/29.2 -/25.0/26.6)
//   four tokens        bf16 1 x 32768 -/39.8/32.4   2 x 16384 -/38.9/32.3 -/37.5/32.2   4 x 8192 -/40.0/32.3 -/35.6/31.6   (4 x 16384 -/46.4/55.0)   (8 x 4096 -/38.7/33.0 -/39.3/32.2)   three (10 x 4300, drawn -/32.0/33.5)
//                      8 bit 1 x 8192 -/41.0/15.5   2 x 32768 -/64.6/41.6 -/60.1/41.0   4 x 16384 -/57.2/41.3 -/55.9/40.4   8 x 8192 -/55.4/42.3 -/55.8/40.9
// One sequence of the hint's length, the others of 32 tokens, the other kernels before several waves merged / runs: bf16 2 x 8192 28.8/12.4   8 x 8000 29.5/20.4   16 x 3500 21.0/18.6   20 x 2400 19.0/18.2   8 bit 21 x 3000 19.4/16.7
//   two tokens bf16 16 x 2048 20.6/20.2   8 bit 16 x 2816 21.7/19.7   four tokens bf16 4 x 8192 40.6/30.7   8 bit 8 x 8000 63.0/39.6
// The units of a row are dealt out to its runs, so shorter lengths than the hint cost less: 1 x 4096 under a hint of 32768 15.9/11.9, 16 x 512 under 4096 18.0/11.5.
constexpr int kBriefCutParts = 4;
constexpr int kMostBriefRuns = 64;                                      // of all rows: 256 compute units
constexpr int brief_runs(int bits, int q_len, int64_t rows, int64_t hint)
{
    const bool many = q_len >= 3;                                       // (the other kernels have more to merge, or take two passes)
    const int64_t most = bits != 16 ? (many ? 262144 : 65536) : rows > 16 ? (many ? 114688 : 49152) : rows > 8 && !many ? 57344 : many ? 131072 : 65536;
    const bool two = q_len == 2 && rows > 21 && hint <= (bits == 16 ? 2048 : 2816);
    if (rows > (many || two ? 32 : 21) || (!two && rows * hint > most)) return 0;
    const int64_t fill = kMostBriefRuns / rows, by_length = hint / (rows <= 2 ? 64 : 128);
    return (int)(by_length < fill ? by_length : fill);
}

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
