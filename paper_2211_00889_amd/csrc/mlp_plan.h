// How the MLP kernels (mlp.hip) cut their work into workgroups, and the order in which
// the forward takes the chunks of d_in, in plain C++ so that the CPU tests walk the
// same code.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "mlp_shape.h"

#ifndef NBSGD_HD
#ifdef __HIPCC__
#define NBSGD_HD __host__ __device__ __forceinline__
#else
#define NBSGD_HD inline
#endif
#endif

namespace nbsgd {

// Forward: d_in is T = d_in / 64 chunks (T is even), cut into leaves, eight or T if
// that is fewer, as equal as they go; leaf i is chunks leaf(i) .. leaf(i + 1) - 1.
// Leaves 2 p and 2 p + 1 are part p.  A pre-activation is the same sum, bit for bit,
// however many slices a launch cuts d_in into, so that a mini-batch's results do not
// depend on which others are in its call: a leaf's products in increasing k, a part
// its two leaves, the parts p0 + p1, (p0 + p1) + p2 or (p0 + p1) + (p2 + p3).  A slice
// is 1 / S of the parts, in pairs: k_mlp_fwd adds the leaves and the pairs of a slice,
// k_mlp_back the slices.
constexpr int kFwKc = 64;

// One pair of parts of a slice, or a part alone: the two halves of a workgroup's waves
// take one side each, a part of the pair or a leaf of the part.
struct FwdPair {
  int end;                // the part after it
  int first[2], n[2];     // chunks of each side (n: one more or less than the other's)
  int cut[2];             // chunks of the side's first leaf (0 where it is one leaf)
  NBSGD_HD int steps() const { return n[0] > n[1] ? n[0] : n[1]; }
};

struct FwdChunks {
  int T;
  NBSGD_HD int leaf(int i) const { return i * (T < 8 ? 8 : T) >> 3; }
  NBSGD_HD int parts() const { return (T < 8 ? T : 8) / 2; }
  // The pair from part p on in a slice that ends before part `end`.
  NBSGD_HD FwdPair pair(int p, int end) const {
    const int m = end - p < 2 ? 1 : 2;  // leaves of a side
    FwdPair g;
    g.end = p + m;
    for (int h = 0; h < 2; ++h) {
      const int i = 2 * p + m * h;
      g.first[h] = leaf(i);
      g.n[h] = leaf(i + m) - g.first[h];
      g.cut[h] = m == 2 ? leaf(i + 1) - g.first[h] : 0;
    }
    return g;
  }
};

// A step of a slice: chunk c of either side of a pair.  Past a side's end its last
// chunk stands in (loaded, never multiplied); past the slice's last step the position
// stays.
struct FwdPos {
  FwdPair g;
  int c;
  NBSGD_HD int chunk(int h) const {
    const int first = h ? g.first[1] : g.first[0], n = h ? g.n[1] : g.n[0];
    return first + (c < n ? c : n - 1);
  }
  NBSGD_HD void next(FwdChunks k, int end) {
    if (c + 1 < g.steps()) ++c;
    else if (g.end < end) g = k.pair(g.end, end), c = 0;
  }
};

// The pipeline of side h (0 and 1 run side by side) over parts p .. end - 1: W1's
// chunks of both sides go to one of two buffers, a step ahead of their use and loaded
// another step ahead; the side's own samples are loaded a step ahead and staged (by
// each wave for itself) where they are used.  first_leaf multiplies into the sums of
// the first of a side's two leaves, leaf into those of the other or only one (sums of
// their own, so that no step has to move them); add(first, last) ends a pair, the
// first and the last of the slice.  The loads are unconditional.  PAIRS is the slice's
// fwd_pairs: 0 for a part alone, 1 for a pair, 2 for a pair and one part or pair more;
// known at compile time since the sums of a second leaf take 64 registers of 256.
// ROLLED: a second pair runs the first one's code (512 x 3072x512 with W1 packed 129.3
// us so, 132.8 with code of its own; where W1 is not packed the loop spills and loses:
// 200 x 640x448 39.5 and 38.0).
constexpr int fwd_pairs(int parts) { return parts < 3 ? parts - 1 : 2; }
template <int PAIRS, bool ROLLED, class LoadW, class LoadA, class StageW, class StageA, class FirstLeaf,
          class Leaf, class Barrier, class Add>
NBSGD_HD void fwd_walk(FwdChunks k, int p, int end, int h, LoadW load_w, LoadA load_a, StageW stage_w,
                       StageA stage_a, FirstLeaf first_leaf, Leaf leaf, Barrier barrier, Add add) {
  FwdPos w = {k.pair(p, end), 0}, a = w;  // the steps last loaded
  load_w(w.chunk(0), w.chunk(1));
  load_a(a.chunk(h));
  stage_w(0);
  w.next(k, end);
  load_w(w.chunk(0), w.chunk(1));
  barrier();
  int buf = 0;
  auto step = [&](auto multiply, bool own, bool more) {
    if (own) stage_a();
    a.next(k, end);
    load_a(a.chunk(h));
    if (own) multiply(buf);
    if (more) {
      stage_w(buf ^ 1);
      w.next(k, end);
      load_w(w.chunk(0), w.chunk(1));
    }
    barrier();
    buf ^= 1;
  };
  auto pair = [&](bool first, bool last) {
    const FwdPair g = k.pair(p, end);
    const int n = h ? g.n[1] : g.n[0], other = h ? g.n[0] : g.n[1], cut = h ? g.cut[1] : g.cut[0];
    const int both = n < other ? n : other;
    p = g.end;
    if constexpr (PAIRS > 0)
      for (int c = 0; c < cut; ++c) step(first_leaf, true, true);
    for (int c = cut; c < both; ++c) step(leaf, true, !last || c + 1 < g.steps());
    if (n != other) step(leaf, n > other, !last);
    add(first, last);
  };
  if constexpr (PAIRS == 2 && ROLLED) {
#ifdef __clang__
#pragma clang loop unroll(disable)
#endif
    for (int q = 0; q < 2; ++q) pair(q == 0, q == 1);
  } else {
    pair(true, PAIRS < 2);
    if constexpr (PAIRS == 2) pair(false, true);
  }
}

// Chunk steps of the longest of S slices (S divides the parts).
inline int fwd_slice_steps(FwdChunks k, int S) {
  const int per = k.parts() / S;
  int most = 0;
  for (int s = 0; s < S; ++s) {
    int n = 0;
    for (int p = s * per; p < (s + 1) * per;) {
      const FwdPair g = k.pair(p, (s + 1) * per);
      n += g.steps();
      p = g.end;
    }
    most = std::max(most, n);
  }
  return most;
}

// Slices of d_in for `tiles` 128 x 128 output tiles: of the counts that divide the
// parts, the one that makes rounds of workgroups (one fits a CU, 256 a round) times
// chunk steps and four the least, the fewer slices on a tie.  A round's first chunks
// and its exchange of sums take as long as four steps, and every slice adds a plane of
// partial sums that is written and read.  Losses of 32-sample batches of 3072x512 in
// 1, 2 and 4 slices: 40 50.7, 31.9, 24.9 us; 64 53.4, 36.1, 30.8; 68 54.7, 36.6, 41.7;
// 128 55.1, 41.9, 50.6; 160 58.6, 66.1, 67.3; 300 114, 105, 113; 400 122, 135, 150.
// 86 of 384x512 in 1 and 3 slices 22.8 and 25.2; 300 of 256x512 in 1 and 2 35.8, 41.4.
// *steps: the chunk steps that a CU makes.
constexpr int kFwRound = 4;
inline int fwd_slices(int d_in, int tiles, int* steps) {
  const FwdChunks k = {d_in / kFwKc};
  int best = 0;
  int64_t least = 0;
  for (int q = 1; q <= kSkMaxSlices && q <= k.parts(); ++q) {
    if (k.parts() % q) continue;
    const int64_t rounds = ((int64_t)tiles * q + 255) / 256, n = fwd_slice_steps(k, q);
    if (best && rounds * (n + kFwRound) >= least) continue;
    best = q;
    least = rounds * (n + kFwRound);
    *steps = (int)(rounds * n);
  }
  return best;
}

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
