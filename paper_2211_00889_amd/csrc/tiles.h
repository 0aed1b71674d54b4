// How the step kernels cut the P columns of their rows into workgroups (step.hip),
// in plain C++ so that the CPU tests walk the same code.
//
// Every kernel of step.hip has two forms.  EVEN: P is a multiple of 4 and rows
// start on 128-byte lines (or on 16 bytes, where a step moves few rows: even_step);
// every lane takes four columns.  Otherwise rows may start on any float: whole tiles of 4 * LANES columns still move 16 bytes a
// lane (float-aligned), and the columns after them are taken one float a lane
// by tiles of LANES.  Measured (n = 8, m = 8, ring step, contiguous rows) against
// float lanes for odd P and float2 lanes for twice-odd P: P = 11,181,641 987 ->
// 635 us (5.3 TB/s), P = 11,181,642 776 -> 621 us, P = 262,143 26.7 -> 18.5 us.
// The even form is kept because the choice at the kernel's start costs it 0.5%
// (ResNet-18-sized step 549.8 against 546.9 us) and the neighbouring tiles
// below up to 4% (1.58M-parameter step 82.7 -> 85.4 us).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define NBSGD_HD __host__ __device__ __forceinline__
#else
#define NBSGD_HD inline
#endif

namespace nbsgd {

// The EVEN form, for rows ld floats apart.
inline bool even_rows(int64_t P, int64_t ld) { return P % 4 == 0 && ld % 32 == 0; }

// The form of a fused step that moves `rows` rows (reads and writes), the server's or
// the replicas'.  Rows off the lines but whole in 16 bytes lose by the neighbouring
// tiles where few rows are moved, and gain where many are; the line lies between,
// and for the server, which writes half as many of its rows, farther up.  EVEN against
// the other form: replicas, 22 rows (n = 2, P = 4,000,004) 86.8 and 94.0 us, 28 (n = 4,
// 4,383,948) 104.6 and 109.4, 41 (n = 8) 148.4 and 149.2, 36 (n = 1) 132.2 and 127.6, 42
// (n = 4) 141.9 and 132.7, 80 (n = 8, 1,578,508) 99.6 and 90.7; server, 66 (n = 8,
// 1,578,508) 80.3 and 87.5, 94 (n = 8, 2,000,004) 146.7 and 151.5, 113 (n = 4) 173.3 and
// 179.2, 129 (n = 16) 207.3 and 198.2, 153 (n = 8) 242.4 and 232.0.
inline bool even_step(int64_t P, int64_t ld, int64_t rows, bool server) {
  return even_rows(P, ld) || (P % 4 == 0 && ld % 4 == 0 && rows < (server ? 124 : 36));
}

// Column tile of workgroup b of `tiles`: where rows do not start on lines, XCD x
// (workgroups b % 8 == x) takes kNear neighbouring tiles in a row, so that a
// line shared by two tiles is mostly read and merged in one L2 (P = 11,181,641:
// 681 us with 1 tile, 638 with 2, 632 with 4, 622 with 8, but 8 slow the 17.2M
// sixteen-mini-batch step by 1% more than 4 do); the last tiles that fill no
// whole round of 8 * kNear keep their order.
constexpr uint32_t kNear = 4;
template <bool EVEN>
NBSGD_HD uint32_t tile_of(uint32_t b, uint32_t tiles) {
  constexpr uint32_t kRound = 8 * kNear;
  if (EVEN || tiles - b / kRound * kRound < kRound) return b;
  return b / kRound * kRound + b % 8 * kNear + b / 8 % kNear;
}

// First column of a lane in a tile, and whether it takes four columns (the same
// in all lanes of a tile) or one; a lane's columns are all below P or all beyond.
struct Cols {
  int64_t col;
  bool vec4;
};
template <bool EVEN, int LANES>
NBSGD_HD Cols columns(uint32_t tile, int lane, int64_t P) {
  const int64_t full = EVEN ? 0 : P / (4 * LANES);
  if (EVEN || tile < full) return {(int64_t)tile * (4 * LANES) + 4 * lane, true};
  return {full * (4 * LANES) + (tile - full) * LANES + lane, false};
}

// Tiles that columns<EVEN, LANES> covers P columns with.
template <int LANES>
inline int64_t tiles(int64_t P, bool even) {
  const int64_t full = P / (4 * LANES), rest = P % (4 * LANES);
  return full + (even ? (rest > 0) : (rest + LANES - 1) / LANES);
}

}  // namespace nbsgd
