// How the MLP kernels (mlp.hip) cut their work into workgroups, in plain C++ so
// that the CPU tests walk the same code.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace nbsgd {

// Grid of the gradient kernel: entries (x) by shares of their feature blocks (y).
// From 21 mini-batches on the entries are rounded up to whole rounds of XCDs, so that
// an entry's workgroups share an L2; with fewer that leaves XCDs idle, and the
// workgroups follow each other over all of them (1 of 24576x512: 144.5 us rounded up,
// 114.5 not; 3072x512: 9 42.1 and 39.2, 20 57.9 and 54.5, 23 58.9 and 60.7, 41 84.5
// and 86.8).
constexpr int kBackRound = 21;
inline int back_entries(int count) { return count < kBackRound ? count : (count + 7) / 8 * 8; }

// Feature blocks that a workgroup of that kernel takes, of the `blocks` of each of
// `entries` entries: as few as keep the launch within one workgroup per CU, since the
// head costs each of them 10 us, but at most six (8 x 4 mini-batches 3072x512: 62.6 us
// so, 64.1 with two workgroups per CU; 12 x 8 of 1408x512 79.9 and 82.5; 16 x 16 373.4
// and 371.2 with at most four).
constexpr int kBackGrid = 256, kBackBlocks = 6;
inline int back_blocks(int blocks, int entries) {
  return (int)std::min<int64_t>(kBackBlocks, ((int64_t)blocks * entries + kBackGrid - 1) / kBackGrid);
}

}  // namespace nbsgd
