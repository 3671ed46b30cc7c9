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
  ++seen_plans[p.one_each ? 2 : (p.ranges ? 1 : 0)];
  const long long pairs = (long long)tiles * n;
  EXPECT(p.per_xcd >= 1 && p.per_xcd <= pairs);
  const int resident = budget ? budget / 8 : (tile == 256 ? 32 : 64);
  EXPECT(p.one_each ? budget == 0 : p.per_xcd <= resident);
  std::vector<char> seen(p.sorted ? n : 0, 0), met((size_t)pairs, 0);
  for (int k = 0; p.sorted && k < n; ++k) {
    EXPECT(order[k] < n && !seen[order[k]]);
    seen[order[k]] = 1;
    EXPECT(k == 0 || len[order[k - 1]] >= len[order[k]]);
  }
  for (int b = 0; b < 8 * p.per_xcd; ++b) {
    int count = 0;
    const int first = p.ranges ? p.first[b & 7] : 0;
    for (PairWalk<true> w(b, p.per_xcd, tiles, n, tile_div_by((unsigned)tiles), p.ranges, first, p.first[(b & 7) + 1],
                          p.alone[b & 7]); w.more(); w.next()) {
      EXPECT(w.i >= 0 && w.tile() >= 0 && w.tile() < tiles);
      const size_t id = (size_t)w.i * tiles + w.tile();
      EXPECT(!met[id]);
      met[id] = 1;
      ++count;
    }
    EXPECT(p.alone[b & 7] >= 0 && p.alone[b & 7] < (p.one_each ? 1 : p.per_xcd));
    EXPECT((!p.one_each && b >> 3 >= p.alone[b & 7]) || count <= 1);
    seen_alone += !p.one_each && b >> 3 < p.alone[b & 7];
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
