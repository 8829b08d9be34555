// Which form of merge_splits_kernel a call takes, and which rows (sequence * query tokens of the launch + query token) its blocks take.  Plain C++: the host sizes the grid
// from it, the kernel finds its row by it, and a test checks it without a device.
//
// Sixteen blocks per row.  Consecutive block indices go to consecutive dies (each with its own L2), and the streaming kernel has numbered its ranges so that
// a die holds consecutive ranges (range_index), i.e. with lengths that are about equal the partial results of the sequences lie on the dies in order: the
// blocks of a die take the rows whose middle, (row + 1/2) * 8 / rows, falls to it.  With fewer than eight sequences the query tokens of one are
// spread over the dies that it covers.
#pragma once

namespace mfa {

constexpr int kMergeBlocksPerRow = 16;

// The first row of a die (die 8: all rows)
constexpr int first_row_of_die(int die, int rows) { return (int)((2u * (unsigned)die * (unsigned)rows + 7u) >> 4); }

// The row of a block, or -1: a die has room for ceil(rows / 8) rows and may have one less.  The block's place among the row's sixteen: (block >> 3) & 15.
constexpr int merge_row(unsigned block, int rows, int blocks_per_row = kMergeBlocksPerRow)
{
    const int die = (int)(block & 7u), row = first_row_of_die(die, rows) + (int)((block >> 3) / (unsigned)blocks_per_row);
    return row < first_row_of_die(die + 1, rows) ? row : -1;
}

constexpr unsigned merge_blocks_by_die(int rows, int blocks_per_row = kMergeBlocksPerRow) { return (unsigned)blocks_per_row * (unsigned)((rows + 7) / 8 * 8); }

// Few rows have many partial results each, and a thread that takes them four at a time is a chain of round trips (1 x 32768: 256 of them, 29 us); then a
// block takes a quarter as many positions, and each of its waves a run of the partial results, eight at a time.  us per call, one wave / this: 1 x 32768 43.8/21.8,
// 2 x 8000 28.3/16.9, 4 x 4096 21.5/16.8, 6 x 6000 ragged 25.4/22.0, 8 bit, two tokens 2 x 8000 30.9/21.8, four tokens 1 x 16000 53.6/34.4, 3 x 8000 ragged 40.3/32.6;
// 12 x 8000 ragged 25.8/24.3, two tokens 8 x 4000 25.5/24.6; from there on one wave is ahead (16 x 4096 24.7/25.1, 20 x 8000 38.9/40, 32 x 4096 33.9/36.3, 128 x 8192 ragged 110/119), and with few
// partial results per row (16 x 256, four 10.3/12.0; 2 x 512, eight 10.5/11.1; 4 x 1024, sixteen 13.0/12.4).
//
// Nine to sixteen rows whose batch is no multiple of eight: one wave by die / four by die / four in order / eight in order, equal lengths, drawn ones, one of full length and others of 500 tokens
//   one token    9 x 12000 bf16 32.7/32.1/31.7/32.5 28.8/25.7/25.3/25.8 36.8/26.4/22.4/21.8   11 37.5/37.5/37.3/37.7 28.2/27.9/26.0/25.8 35.5/26.7/23.3/22.4   15 42.9/42.9/43.1/44.3 29.9/29.1/28.4/29.6 33.5/26.1/22.9/23.7
//                9 x 12000 8 bit 25.4/24.9/24.8/25.6 24.4/21.3/21.3/21.8 35.3/24.9/22.3/21.7   13 28.2/28.1/28.7/29.6 23.8/23.2/22.9/23.8 30.7/24.2/23.2/23.6 (equal lengths, 13 and 14: 1.5 % slower in order)
//   two tokens   5 x 12000 bf16 29.5/29.5/28.7/28.5 32.0/26.8/26.2/26.9 38.2/28.2/24.1/23.7   6 30.7/31.2/30.9/30.6 30.4/30.6/27.5/27.2 39.9/37.4/24.2/23.7   7 33.5/34.3/34.6/33.9 30.4/30.4/28.7/28.0 40.0/37.4/24.7/24.9
//                7 x 12000 8 bit 31.9/32.8/33.1/32.4 28.3/28.2/26.7/26.0   4 bit 29.6/30.5/30.9/30.1 27.1/27.0/25.4/24.8   (seven of equal length: 1 .. 3 % slower than by one wave)
//   two passes (four tokens, 4 bit)   5 x 20000 65.1/65.1/66.9/66.6 65.0/56.8/59.2/57.2   6 67.1/67.5/70.6/70.1 63.0/60.5/57.3/58.3   7 69.8/71.0/75.9/74.6 62.7/58.7/57.7/59.7; one long 6 x 19000 81.3/77.1/53.1
//                by die in spite of that last one: in order, equal lengths are up to a tenth slower than by one wave
//   three sequences of three or four tokens (bf16)   32000 52.0/51.4/50.9/51.4 52.0/49.9/41.4/41.1
constexpr int merge_waves(int B, int n_here, int q_len, int pieces)
{
    const int rows = B * n_here;
    if (rows > 16 || pieces < (rows <= 8 ? 12 : 17)) return 1;
    return rows <= 8 || (q_len == 2 && (B & 7) != 0) ? 8 : 4;
}
// The runs of brief_attn_kernel, 64 at most, one / four / eight waves: 1 x 4096, 64 of them 16.3/11.2/10.8, 24 13.0/11.1/11.7; 4 x 1536, sixteen 11.8/10.8/11.4;
// 5 x 1536, nine 12.2/12.4/13.2; 8 x 4096, eight 16.2/16.6/17.6.
constexpr int merge_waves_of_runs(int runs) { return runs < 12 ? 1 : runs < 48 ? 4 : 8; }

// Whether the blocks of a die take the rows of that die.  us per call so / with rows in order:
//   one token   23 x 4096 28.4/33.0   30 x 6000 ragged 31.9/36.0   8 bit, ragged 23 x 20011 35.3/39.2   bf16 127 x 4000 44.0/45.1
//   several waves a block  5 x 8000 21.3/21.5   6 x 3000 ragged 17.9/19.1   8 bit, two tokens, 4 x 8000 24.4/24.7   16 x 4096 24.7/25.2
// Not where it would leave dies idle or give some of them twice the rows of others: 1 x 32768 30.2/21.7, 3 x 8000 20.8/19.1, 4 x 16000 ragged 25.9/23.5, 12 x 8000 ragged 24.7/24.1, four
// tokens 3 x 8000 ragged 38.1/32.4, and those above.  Looked up in the records, which is exact for ragged
// lengths, with what a die has beyond its share given to others: the same for most, but 122.2 against 120.5 at 128 x 8192 ragged and 24.8 against 22.6 at 128 x 400.
// Not by die with less than a tile for every compute unit, where a sequence's many one-tile pieces lie on several dies anyway (5 x 1500
// ragged: 16.7, in order 16.2), unless the batch divides evenly.
constexpr bool merge_by_die(int B, int n_here, int q_len, int n_wgs, int waves)
{
    const int rows = B * n_here;
    if (waves > 1 && (rows <= 4 || (rows > 8 && (B & 7) != 0 && q_len == n_here))) return false;
    return n_wgs > 0 && (n_wgs & 7) == 0 && (n_wgs >= 256 || (B & 7) == 0);
}

}  // namespace mfa
