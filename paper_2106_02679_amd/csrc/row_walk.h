// The rows that a wavefront of a four-wavefront workgroup takes, one after the other, where a launch deals `rows` rows to fewer
// wavefronts - for row counts that leave room for one step more in an int; the kernels with a row per workgroup take the others, in 64 bits.
// (In 64 bits here the narrow fp32 LayerNorm took 3 % longer, with the index in scalar registers the 16-bit one 2 - 4 % at 131072 x 768.)
// No HIP in here, so that a host program can walk the same sequence.
#pragma once
#include <climits>

namespace lga {

constexpr int kWavesPerBlock = 4, kMostWalkBlocks = 2048;
constexpr bool row_walk_takes(int rows) { return rows <= INT_MAX - kWavesPerBlock * kMostWalkBlocks; }
// Workgroups for `rows` rows, at most `most` <= kMostWalkBlocks
constexpr int row_walk_blocks(int rows, int most) {
    const int all = (rows + kWavesPerBlock - 1) / kWavesPerBlock;
    return all < most ? all : most;
}
struct RowWalk {
    int row, step, rows;
    constexpr RowWalk(unsigned block, unsigned blocks, unsigned wave, int n) : row(block * kWavesPerBlock + wave), step(blocks * kWavesPerBlock), rows(n) {}
    constexpr bool valid() const { return row < rows; }
    constexpr int next() const { return row + step; }
    constexpr bool has_next() const { return next() < rows; }
    constexpr void advance() { row = next(); }
};

}  // namespace lga
