// Which rows (sequence * query tokens of the launch + query token) the blocks of merge_splits_kernel take.  Plain C++: the host sizes the grid
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

}  // namespace mfa
