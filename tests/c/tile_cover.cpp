// Walks the column tiles of the step kernels (csrc/tiles.h) on the CPU: for many
// column counts and both forms, every column is taken exactly once, by lanes whose
// columns are all below P, and tile_of is a permutation of the tiles.
#include <cstdio>
#include <vector>

#include "tiles.h"

using namespace nbsgd;

template <bool EVEN, int LANES>
static bool walk(int64_t P) {
  const int64_t T = tiles<LANES>(P, EVEN);
  std::vector<unsigned char> seen(P, 0), tile(T, 0);
  for (int64_t b = 0; b < T; ++b) {
    const uint32_t t = tile_of<EVEN>((uint32_t)b, (uint32_t)T);
    if (t >= T || tile[t]++) return std::printf("P=%lld: tile %u twice or beyond\n", (long long)P, t), false;
    for (int lane = 0; lane < LANES; ++lane) {
      const Cols c = columns<EVEN, LANES>(t, lane, P);
      if (c.vec4 != columns<EVEN, LANES>(t, 0, P).vec4) return std::printf("P=%lld: mixed tile\n", (long long)P), false;
      if (c.col >= P) continue;
      for (int k = 0; k < (c.vec4 ? 4 : 1); ++k)
        if (c.col + k >= P || seen[c.col + k]++)
          return std::printf("P=%lld: column %lld twice or beyond\n", (long long)P, (long long)(c.col + k)), false;
    }
  }
  for (int64_t k = 0; k < P; ++k)
    if (!seen[k]) return std::printf("P=%lld: column %lld missed\n", (long long)P, (long long)k), false;
  return true;
}

int main() {
  std::vector<int64_t> sizes;
  for (int64_t P = 1; P <= 2100; ++P) sizes.push_back(P);
  for (int64_t base : {8 * 4 * 256, 16 * 4 * 256, 32 * 1024, 50 * 1024})
    for (int64_t d = -260; d <= 260; d += 13) sizes.push_back(base + d);
  for (int64_t P : sizes) {
    if (!walk<false, 64>(P) || !walk<false, 256>(P)) return 1;
    if (P % 4 == 0 && (!walk<true, 64>(P) || !walk<true, 256>(P))) return 1;
    if (even_rows(P, P) && P % 32) return std::printf("even rows of %lld\n", (long long)P), 1;
  }
  if (even_rows(6, 32) || even_rows(8, 9) || !even_rows(8, 32)) return std::printf("even_rows\n"), 1;
  // the form of a step: 16-byte rows off the lines by the rows it moves, odd ones never
  for (int64_t rows : {5, 35, 36, 123, 124, 400})
    for (bool server : {false, true}) {
      const bool few = rows < (server ? 124 : 36);
      if (even_step(1578508, 1578508, rows, server) != few || even_step(1000, 1004, rows, server) != few ||
          !even_step(1000, 1024, rows, server) || even_step(1578506, 1578508, rows, server) ||
          even_step(1000, 1001, rows, server))
        return std::printf("form of a step of %lld rows\n", (long long)rows), 1;
    }
  std::puts("ok");
  return 0;
}
