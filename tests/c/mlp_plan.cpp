// Checks the work splitting of the MLP kernels (csrc/mlp_plan.h) on the CPU.
#include <cstdio>

#include "mlp_plan.h"

using namespace nbsgd;

// The gradient kernel's workgroups: no more than one per CU unless each takes the
// most blocks, and those with work spread over the XCDs (workgroup b runs on XCD
// b % 8), so that none has more than twice its share of them.
static bool back_grid() {
  for (int blocks = 1; blocks <= 400; ++blocks)
    for (int count = 1; count <= 896; ++count) {
      const int entries = back_entries(count), each = back_blocks(blocks, entries), y = (blocks + each - 1) / each;
      if (entries < count || each < 1 || each > kBackBlocks)
        return std::printf("%d x %d: %d entries, %d blocks each\n", blocks, count, entries, each), false;
      if (each < kBackBlocks && (int64_t)blocks * entries > (int64_t)kBackGrid * each)
        return std::printf("%d blocks of %d mini-batches: more than a workgroup per CU\n", blocks, count), false;
      if (count > 64 || y > 400) continue;
      int on[8] = {0}, most = 0;
      for (int b = 0; b < entries * y; ++b) on[b % 8] += b % entries < count;
      for (int x : on) most = std::max(most, x);
      if (count * y >= 64 && 8 * most > 2 * count * y)
        return std::printf("%d blocks of %d mini-batches: %d of %d workgroups on one XCD\n", blocks, count, most, count * y), false;
    }
  return true;
}

int main() {
  if (!back_grid()) return 1;
  std::puts("ok");
  return 0;
}
