// Walks the work splitting of the MLP kernels (csrc/mlp_plan.h) on the CPU: the grid
// of the gradient kernel, and the forward's pipeline over the chunks of d_in, the code
// the kernel runs, for every slice of every number of chunks up to 200 and some
// larger: each side's leaves multiplied whole and in order, from the buffer and the
// samples of the same chunk, no buffer read and restaged between two barriers, both
// sides at the same barriers, every chunk once.  Planted mistakes must fail it.
#include <cstdio>
#include <map>
#include <vector>

#include "mlp_plan.h"

using namespace nbsgd;

// Mistakes that the walk must report.
enum Mistake { kNone, kStageRead, kNoBarrier, kShortLeaf, kStaleSamples, kNoFold };

// What one half of a workgroup's waves does, by the barriers it has passed (its epoch).
struct Half {
  int epoch = 0;
  int w[2] = {-1, -1}, a = -1;           // loaded chunks: W1 of both halves, own samples
  int buf[2][2] = {{-1, -1}, {-1, -1}};  // staged W1 chunks
  int staged[2] = {-1, -1};              // epoch of the staging
  int samples = -1;                      // staged own samples
  int written = -1, read = -1;           // last epochs in which add used the exchange
  std::vector<int> leaf, leaf2, order;   // the chunks of the leaves at hand, and all of them
  std::vector<std::vector<int>> side;    // the leaves of the pair at hand
  std::vector<int> ends;                 // epoch in which each pair ended
  std::map<int, int> buf_reads, buf_writes;  // per epoch, a bit per buffer
};

template <int PAIRS, bool ROLLED>
static bool run_pairs(FwdChunks k, int p0, int p1, int h, Mistake m, Half* out) {
  Half s;
  bool ok = true;
  auto bad = [&](const char* what) {
    if (ok && m == kNone) std::printf("T=%d parts %d..%d half %d: %s\n", k.T, p0, p1, h, what);
    ok = false;
  };
  int barriers = 0, p = p0;
  auto barrier = [&] {
    if (m == kNoBarrier && ++barriers == 2) return;
    ++s.epoch;
  };
  auto read = [&](int b) {
    if (s.staged[b] < 0 || s.staged[b] >= s.epoch) bad("a buffer is read before the barrier after its staging");
    if (s.buf[b][h] != s.samples) bad("W1 and samples of different chunks");
    s.buf_reads[s.epoch] |= 1 << b;
  };
  fwd_walk<PAIRS, ROLLED>(
      k, p0, p1, h, [&](int k0, int k1) { s.w[0] = k0, s.w[1] = k1; }, [&](int c) { s.a = c; },
      [&](int b) {
        if (m == kStageRead) b ^= 1;
        if (s.w[0] < 0) bad("staged before it was loaded");
        s.buf[b][0] = s.w[0], s.buf[b][1] = s.w[1], s.staged[b] = s.epoch;
        s.buf_writes[s.epoch] |= 1 << b;
        s.w[0] = s.w[1] = -1;
      },
      [&] {
        if (m != kStaleSamples || s.samples < 0) s.samples = s.a;
      },
      [&](int b) {
        read(b);
        s.leaf.push_back(s.samples);
      },
      [&](int b) {
        read(b);
        (m == kNoFold ? s.leaf : s.leaf2).push_back(s.samples);
      },
      barrier,
      [&](bool first, bool last) {
        if (!s.leaf.empty()) s.side.push_back(s.leaf);
        s.side.push_back(s.leaf2);
        s.leaf.clear();
        s.leaf2.clear();
        if (first != (p == p0)) bad("first");
        // a pair is two parts as long as the slice has them; a side is half of it
        const int leaves = p1 - p >= 2 ? 2 : 1;
        if ((int)s.side.size() != leaves) bad("a side has not the leaves it should");
        for (int q = 0; q < (int)s.side.size(); ++q) {
          const int at = 2 * p + leaves * h + q, c0 = k.leaf(at), n = k.leaf(at + 1) - c0 - (m == kShortLeaf);
          if ((int)s.side[q].size() != n) bad("a leaf's chunks are not multiplied once each");
          for (int c = 0; c < (int)s.side[q].size(); ++c)
            if (s.side[q][c] != c0 + c) bad("a leaf's chunks are out of order");
          s.order.insert(s.order.end(), s.side[q].begin(), s.side[q].end());
        }
        s.side.clear();
        p += leaves;
        if (last != (p == p1)) bad("last");
        if (s.written == s.epoch || s.read == s.epoch) bad("the exchange is written again before a barrier");
        if (!first) barrier();  // after the first pair's sum is read from where the partner writes
        s.written = s.epoch;
        barrier();
        s.read = s.epoch;
        s.ends.push_back(s.epoch);
      });
  if (!s.leaf.empty() || !s.leaf2.empty() || p != p1) bad("chunks after the last pair's end");
  *out = s;
  return ok;
}

static bool run(FwdChunks k, int p0, int p1, int h, Mistake m, Half* out) {
  switch (fwd_pairs(p1 - p0)) {
    case 0: return run_pairs<0, false>(k, p0, p1, h, m, out);
    case 1: return run_pairs<1, false>(k, p0, p1, h, m, out);
  }
  return run_pairs<2, true>(k, p0, p1, h, m, out) && run_pairs<2, false>(k, p0, p1, h, m, out);
}

// Both halves of a slice side by side, and what they cover.
static bool slice(FwdChunks k, int p0, int p1, Mistake m, std::vector<int>* seen) {
  Half s[2];
  for (int h = 0; h < 2; ++h)
    if (!run(k, p0, p1, h, h ? kNone : m, &s[h])) return false;
  // as many barriers, pairs ending at the same ones, or the workgroup would hang
  if (s[0].epoch != s[1].epoch || s[0].ends != s[1].ends) return false;
  for (int e = 0; e <= s[0].epoch; ++e)
    if ((s[0].buf_reads[e] | s[1].buf_reads[e]) & (s[0].buf_writes[e] | s[1].buf_writes[e])) return false;
  for (const Half& q : s)
    for (int c : q.order) ++(*seen)[c];
  return true;
}

static bool forward(int T, Mistake m = kNone) {
  const FwdChunks k = {T};
  const int parts = k.parts();
  if (k.leaf(0) != 0 || k.leaf(2 * parts) != T) return false;
  for (int i = 0; i < 2 * parts; ++i)
    if (k.leaf(i) >= k.leaf(i + 1)) return false;
  for (int p = 0; p < parts; ++p)
    for (int end = p + 1; end <= parts; ++end) {
      const FwdPair g = k.pair(p, end);
      if (std::abs(g.n[0] - g.n[1]) > 1) return std::printf("T=%d: sides of %d and %d chunks\n", T, g.n[0], g.n[1]), false;
    }
  for (int S = 1; S <= parts; ++S) {
    if (parts % S) continue;
    std::vector<int> seen(T, 0);
    for (int s = 0; s < S; ++s)
      if (!slice(k, s * (parts / S), (s + 1) * (parts / S), m, &seen)) {
        if (m == kNone) std::printf("T=%d S=%d slice %d\n", T, S, s);
        return false;
      }
    for (int c = 0; c < T; ++c)
      if (seen[c] != 1) return m == kNone && std::printf("T=%d S=%d: chunk %d %d times\n", T, S, c, seen[c]), false;
  }
  return true;
}

// The slices chosen divide the parts, so that every launch adds the same sums.
static bool slices() {
  for (int T = 2; T <= 400; T += 2)
    for (int tiles = 1; tiles <= 1200; tiles = tiles * 21 / 20 + 1) {
      int steps = 0;
      const int S = fwd_slices(kFwKc * T, tiles, &steps), parts = FwdChunks{T}.parts();
      if (S < 1 || S > kSkMaxSlices || parts % S || steps < 1)
        return std::printf("T=%d tiles=%d: %d slices\n", T, tiles, S), false;
    }
  return true;
}

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
  for (int T = 2; T <= 200; T += 2)
    if (!forward(T)) return 1;
  for (int T : {384, 1026, 65534})
    if (!forward(T)) return 1;
  for (Mistake m : {kStageRead, kNoBarrier, kShortLeaf, kStaleSamples, kNoFold})
    for (int T : {4, 8, 26, 48})
      if (!(m == kStaleSamples && T < 8) && forward(T, m)) return std::printf("mistake %d passes at T=%d\n", m, T), 1;
  if (!slices()) return 1;
  if (!back_grid()) return 1;
  std::puts("ok");
  return 0;
}
