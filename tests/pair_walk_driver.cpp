// Walks the (sequence, tile) pairs of per-sequence launches as the kernel's workgroups do, by the launch's own plan: every pair
// is met once, by a grid that keeps the caller's budget.  Built by tests/test_pair_walk.py with sanitizers on the host code;
// touches no GPU.
#include <cstdio>
#include <vector>

#include "../paper_2512_23353_amd/csrc/kernels.h"
#include "../paper_2512_23353_amd/csrc/pair_walk.h"

using namespace isopo;

static int failures = 0, seen_plans[3], seen_alone;
#define EXPECT(cond)                                                                                                       \
  do {                                                                                                                     \
    if (!(cond)) { std::printf("FAIL %s: tile %d, %dx%d, %zu sequences, budget %d\n", #cond, tile, d_in, rows, len.size(), \
                               budget); ++failures; return; }                                                              \
  } while (0)

static unsigned long long state = 88172645463325252ULL;
static int rnd(int lo, int hi) {                           // xorshift64: fixed, portable sequence
  state ^= state << 13; state ^= state >> 7; state ^= state << 17;
  return lo + (int)(state % (unsigned)(hi - lo + 1));
}

static void walk(int tile, int rows, int d_in, const std::vector<int>& len, int budget) {
  std::vector<int32_t> off(1, 0);
  for (int l : len) off.push_back(off.back() + l);
  const int n = (int)len.size(), tiles = ((rows + tile - 1) / tile) * ((d_in + tile - 1) / tile);
  std::vector<unsigned short> order((size_t)n);
  const WalkPlan p = plan_walk(tile, rows, d_in, n, off.data(), budget, order.data());
  ++seen_plans[p.kind];
  const long long pairs = (long long)tiles * n;
  EXPECT(p.per_xcd >= 1 && p.per_xcd <= pairs);
  const int resident = budget ? budget / 8 : (tile == 256 ? 32 : 64);
  EXPECT(p.kind == kSingle ? tile == 128 && pairs <= 512 : p.per_xcd <= resident);
  std::vector<char> seen((size_t)n, 0), met((size_t)pairs, 0);
  for (int k = 0; p.kind != kSingle && k < n; ++k) {
    EXPECT(order[k] < n && !seen[order[k]]);
    seen[order[k]] = 1;
    EXPECT(k == 0 || len[order[k - 1]] >= len[order[k]]);
  }
  // one workgroup's list: how long it is, -1 where it meets a pair that is none or that was met
  auto list = [&](auto w) {
    int count = 0;
    for (; w.more(); w.next(), ++count) {
      if (w.i < 0 || w.tile() < 0 || w.tile() >= tiles) return -1;
      char& m = met[(size_t)w.i * tiles + w.tile()];
      if (m) return -1;
      m = 1;
    }
    return count;
  };
  for (int b = 0; b < 8 * p.per_xcd; ++b) {
    const int x = b & 7, first = p.first[x], end = p.first[x + 1], alone = p.alone[x];
    const TileDiv by = tile_div_by((unsigned)tiles);
    const int count = p.kind == kDealt    ? list(PairWalk<kDealt>(b, p.per_xcd, tiles, n, by, first, end, alone))
                      : p.kind == kRanges ? list(PairWalk<kRanges>(b, p.per_xcd, tiles, n, by, first, end, alone))
                                          : list(PairWalk<kSingle>(b, p.per_xcd, tiles, n, by, first, end, alone));
    EXPECT(count >= 0 && alone >= 0 && alone < (p.kind == kSingle ? 1 : p.per_xcd));
    EXPECT((p.kind != kSingle && b >> 3 >= alone) || count <= 1);
    seen_alone += b >> 3 < alone;
  }
  for (char m : met) EXPECT(m);
}

int main() {
  const int budgets[] = {0, 8, 9, 64, 100, 224, 255, 256};
  for (int tile : {128, 256})
    for (int tiles_n : {1, 2, 3, 7, 8, 9, 11, 16, 33})                  // every remainder of eight, strips and their ends
      for (int tiles_m : {1, 2, 3, 5, 8})
        for (int n : {1, 2, 7, 8, 9, 40, 255, 256, 257, 300, 1024}) {
          if ((long long)tiles_n * tiles_m * n > 60000) continue;
          std::vector<int> len((size_t)n);
          const int kind = rnd(0, 3);
          for (int& l : len) l = kind == 0 ? 0 : (kind == 1 ? 500 : rnd(0, 900));
          if (kind == 3) len[(size_t)rnd(0, n - 1)] = 16000;
          walk(tile, tiles_m * tile - rnd(0, tile / 8 - 1) * 8, tiles_n * tile - rnd(0, tile / 8 - 1) * 8, len,
               tile == 256 ? budgets[rnd(0, 7)] : 0);
        }
  for (int budget : budgets) walk(256, 1536, 1536, std::vector<int>(80, 300), budget);
  walk(256, 14336, 28672, std::vector<int>(32, 100), 0);                // more pairs than are simulated
  walk(256, 2816, 1280, std::vector<int>(700, 60), 64);
  std::printf("done failures=%d dealt=%d ranges=%d single=%d alone=%d\n", failures, seen_plans[0], seen_plans[1], seen_plans[2], seen_alone);
  return failures != 0;
}
