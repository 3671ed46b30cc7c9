// Host-side launch plan of the streaming bf16 contraction (per-sequence gradients G_i = Delta_i^T X_i of
// both hook listings, and the sums over all tokens): tile size, token split, and which (item, tile) pairs
// each of the eight XCDs and its workgroups take.  Pure host arithmetic, no HIP calls, so that it can be
// tested without a GPU.
#include "kernels.h"
#include "pair_walk.h"

#include <algorithm>
#include <functional>

namespace isopo {

// Row-major per-sequence launches whose widths are no multiples of 256 (others may keep the stash in tile order, whose
// tile is part of a layout): 128x128 tiles where they are modelled faster by 10 %, over stashes that the last-level cache
// takes (beyond it they lose: 2984x560, 101 sequences of 71 tokens, 337 MB: 145 / 157 us).  A compute unit takes
//   256: ceil(items / 256) whole items of  27 ns per token + 8 us   (one workgroup at a time)
//   128: items / 256 items of 9.8 ns per token + 1.5 us             (two at a time)
// and neither is faster than the stash is written (3.2 TB/s).  Measured, 256 against 128: 264x1280, 106 sequences of 260
// tokens 63 / 44 us; 2048x1032, 8 of 780: 50 / 41; 512x2056, 40 of 200: 42 / 36; 1000x2728, 24 of 420: 94 / 97; 648x3600,
// 60 of 1750: 585 / 770.  Of 36 random layers this side of the line 28 gained, by 1.2x on average and 1.8x at most; 384x10504,
// 26 of 374, lost most (169 / 175).
static bool small_tiles_win(int rows, int d_in, int n_tokens, int n_seq) {
  auto tiles = [&](int t) { return (double)((rows + t - 1) / t) * ((d_in + t - 1) / t) * n_seq; };
  const double len = (double)n_tokens / n_seq, write = (double)rows * d_in * n_seq * 2.0 / 3.2e12;
  const double items = tiles(256);
  double big = (double)(long long)((items + 255.0) / 256.0) * (len * 27e-9 + 8e-6);
  double small = tiles(128) / 256.0 * (len * 9.8e-9 + 1.5e-6);
  if (big < write) big = write;
  if (small < write) small = write;
  return small < 0.9 * big && 2.0 * rows * d_in * n_seq <= 256.0 * (1 << 20);
}

static ContractionPlan plan_with_tile(int rows, int d_in, int n_tokens, int n_seq, const int32_t* off_host, bool per_sequence,
                                      bool big);

// What a (sequence, tile) pair costs besides its tokens, in tokens, where the list is cut into ranges of equal work.
constexpr int kPairTokens = 192;

// The item-major list of (item, tile) pairs cut into eight contiguous ranges of equal work, weight(i) per pair of item i: range x
// opens at the first pair that starts at or beyond x eighths of the total.
template <class Weight>
static void cut_pairs(long long tiles, int n_items, Weight&& weight, int* first) {
  long long total = 0, cum = 0;
  for (int i = 0; i < n_items; ++i) total += weight(i) * tiles;
  int i = 0;
  first[0] = 0;
  for (int x = 1; x < 8; ++x) {
    const long long target = (x * total + 7) / 8;
    while (i < n_items && cum + tiles * weight(i) <= target) cum += tiles * weight(i++);
    first[x] = (int)(i == n_items ? tiles * n_items : i * tiles + (target - cum + weight(i) - 1) / weight(i));
  }
  first[8] = (int)(tiles * n_items);
}

ContractionPlan plan_contraction(int rows, int d_in, int n_tokens, int n_seq, const int32_t* off_host,
                                 bool per_sequence, bool weighted, bool budget) {
  const long long big_tiles = (long long)((rows + 255) / 256) * ((d_in + 255) / 256);
  // 256x256 tiles (one workgroup per CU) when they alone fill the chip, else 128x128 (two per CU).  In the
  // sum-over-all-tokens mode the token split supplies parallelism too.
  const long long par = per_sequence ? n_seq : (n_tokens / 1024 > 1 ? n_tokens / 1024 : 1);
  bool big = rows >= 256 && d_in >= 256 && big_tiles * par >= 256;
  // only the launch over 256x256 tiles keeps a budget of compute units, so a caller who gives one keeps those tiles
  if (big && per_sequence && !budget && (rows % 256 || d_in % 256) && small_tiles_win(rows, d_in, n_tokens, n_seq)) big = false;
  ContractionPlan pl = plan_with_tile(rows, d_in, n_tokens, n_seq, off_host, per_sequence, big);
  // A weighted sum cut into token chunks, of few tiles and with operands that stay in the last-level cache: 128x128 tiles,
  // whose four times as many workgroups need fewer chunks, are 5 - 25 % faster (1536x1536, 10^4 tokens: 87 -> 67 us; 2048x2048,
  // 1.4 10^4: 137 -> 122; 1024x4096, 1.2 10^4: 120 -> 106).  With more tiles or tokens their twice as many reads cost more
  // (2048x2304, 1.2 10^4: 132 -> 159; 1536x2560, 2.1 10^4: 173 -> 183, and 8.9 10^4: 556 -> 1020), and the plain sum is
  // faster on the large ones (1024x1024, 4.9 10^4: 118 -> 141), as is either one uncut (1536x8960: 221 -> 276).
  if (weighted && !per_sequence && big && pl.n_chunks > 1 && big_tiles <= 64 &&
      2LL * n_tokens * (rows + d_in) <= 128LL << 20)
    pl = plan_with_tile(rows, d_in, n_tokens, n_seq, off_host, per_sequence, false);
  return pl;
}

static ContractionPlan plan_with_tile(int rows, int d_in, int n_tokens, int n_seq, const int32_t* off_host, bool per_sequence,
                                      bool big) {
  ContractionPlan pl;
  constexpr int kBlockTokens = 32;
  pl.tile = big ? 256 : 128;
  pl.occupancy = big ? 1 : 2;
  pl.tiles_m = (rows + pl.tile - 1) / pl.tile;
  pl.tiles_n = (d_in + pl.tile - 1) / pl.tile;
  const long long tiles = (long long)pl.tiles_m * pl.tiles_n;
  pl.n_chunks = 1;
  pl.chunk_tokens = n_tokens;
  pl.whole_tiles = 0;
  for (int x = 0; x <= 8; ++x) pl.xcd_start[x] = 0;
  if (!per_sequence && big && tiles > 256 && tiles % 256 != 0 && tiles <= 0x3fffffffLL) {
    // More tiles than compute units, and the last round of one tile per compute unit would be partly idle:
    // the tiles of the full rounds stay whole (direct stores), the `rest` tiles of the last round are cut
    // into w token chunks that fill it (fp32 atomics on those tiles only).  Modelled time of the last round
    //   ceil(N / w) * t_token  +  (w > 1) * w * rest * tile outputs * t_atomic,
    // t_token a workgroup's time per token row, t_atomic the chip's time per fp32 atomic add; the split has
    // to win 5 %.  Workgroups are dispatched in id order, whole tiles first, so a compute unit takes a chunk
    // when it has finished its whole tiles.
    const long long rest = tiles % 256;
    const double t_token = 2.0e-8, t_atomic = 5.0e-12;
    long long most = 256 / rest;
    if (most > n_tokens / 512) most = n_tokens / 512;
    if (most > 64) most = 64;
    long long want = 1;
    double best = 0.95 * (double)n_tokens * t_token;
    for (long long w = 2; w <= most; ++w) {
      const double t = (double)((n_tokens + w - 1) / w) * t_token + (double)w * rest * 65536.0 * t_atomic;
      if (t < best) { best = t; want = w; }
    }
    if (want > 1) {
      pl.whole_tiles = (int)(tiles - rest);
      pl.chunk_tokens = (int)(((n_tokens + want - 1) / want + kBlockTokens - 1) / kBlockTokens * kBlockTokens);
      pl.n_chunks = (n_tokens + pl.chunk_tokens - 1) / pl.chunk_tokens;
      pl.blocks = 8LL * (pl.whole_tiles / 8 + (rest * pl.n_chunks + 7) / 8);
      return pl;
    }
  }
  if (!per_sequence) {
    // Number of token chunks: the count with the smallest modelled time
    //   rounds(w) * ceil(N / w) * t_token  +  (w > 1) * w * outputs * t_atomic,
    // rounds(w) = passes an XCD's 32 CUs make over its eighth of the tiles * w workgroups.  t_token is a
    // workgroup's time per token row, t_atomic the chip's time per fp32 atomic add (about 0.8 TB/s), both
    // measured; without the second term more chunks always look better, and the adds then cost more than
    // the idle CUs did.
    const long long slots = 32LL * pl.occupancy;                     // per XCD
    const double t_token = 2.0e-8 * (double)(pl.tile * pl.tile) / 65536.0 * pl.occupancy, t_atomic = 5.0e-12;
    const double outputs = (double)rows * d_in;
    const long long most = n_tokens / 512 > 1 ? n_tokens / 512 : 1;
    long long want = 1;
    double best = 0.0;
    for (long long w = 1; w <= most && w <= 64; ++w) {
      const long long rounds = ((tiles * w + 7) / 8 + slots - 1) / slots;
      const double t = (double)rounds * (double)((n_tokens + w - 1) / w) * t_token + (w > 1 ? w * outputs * t_atomic : 0.0);
      if (w == 1) best = 0.9 * t;                                    // a split has to win by a margin
      else if (t < best) { best = t; want = w; }
    }
    if (want > 1) {
      pl.chunk_tokens = (int)(((n_tokens + want - 1) / want + kBlockTokens - 1) / kBlockTokens * kBlockTokens);
      pl.n_chunks = (n_tokens + pl.chunk_tokens - 1) / pl.chunk_tokens;
    }
  }
  const bool mapped = per_sequence || pl.n_chunks > 1;
  const int n_items = per_sequence ? n_seq : pl.n_chunks;
  pl.blocks = mapped ? 8LL * n_items * ((tiles + 7) / 8) : tiles;
  // Per-sequence mode with a tile count that is a multiple of eight: XCD x takes the x-th eighth of the
  // tiles of every sequence (xcd_start stays zero).  Otherwise the item-major list of (item, tile) pairs is
  // cut into eight contiguous ranges of equal work.
  if (mapped && (!per_sequence || tiles % 8 != 0) && tiles * n_items <= 0x7fffffffLL) {
    // Work of item i: its tokens plus a fixed charge for the workgroup's prologue and epilogue.
    auto weight = [&](int i) -> long long {
      if (per_sequence) return (off_host ? off_host[i + 1] - off_host[i] : 1024) + kPairTokens;
      const long long t0 = (long long)i * pl.chunk_tokens;
      const long long t1 = t0 + pl.chunk_tokens < n_tokens ? t0 + pl.chunk_tokens : n_tokens;
      return (t1 - t0) + 64;
    };
    cut_pairs(tiles, n_items, weight, pl.xcd_start);
    int most = 0;
    for (int k = 0; k < 8; ++k) most = pl.xcd_start[k + 1] - pl.xcd_start[k] > most ? pl.xcd_start[k + 1] - pl.xcd_start[k] : most;
    pl.blocks = 8LL * most;
  }
  return pl;
}

// The per-sequence launch's walk.  Where every pair of 128x128 tiles has a workgroup at once, a workgroup takes one pair of the list
// as it comes, cut into an equal-work range per XCD.  Else as many workgroups as are resident share the list, longest sequences
// first, in the one of two arrangements with the smaller modelled time:
//   dealt   every sequence's tiles over all XCDs: the more even one, and every XCD reads every sequence
//   ranges  an equal-work range of the list per XCD: few XCDs read a sequence, and those with the long ones may have an uneven
//           number of pairs per workgroup
// t, the longest walk, and u, the bytes, overlap for the most part: max(t, u) + 0.6 min(t, u).  A walk is `block` per 32 tokens and,
// for what is not hidden of a pair's first operands and of its stores, `around` blocks per pair; operands arrive at 8 TB/s, the
// stash leaves at 4.5.  The operands are counted up to 24 tiles of 256x256, 40 of 128x128 (of more, neighbouring tiles on an XCD
// share what it reads); another arrangement than dealt (than ranges, of up to 40 128x128 tiles) has to win by a margin.
// Of 400 random layers, 1 to 512 sequences of 0 to 16384 tokens, against always dealt: 256x256 tiles 0.96x on average (1 slower by
// more than 5 %), 128x128 tiles 0.91x (5).  768x384, 28 sequences of 0 to 4460 tokens: 59.7 -> 47.9 us; 288x216, 267 of 1470: 225 ->
// 132; 768x1024, 400 of 4 to 8192: 521 -> 323; 1536x1536, one of 8000 and 31 of 100: 169 -> 154; 2048x2048, the same on a budget of 128
// workgroups: 209 -> 146.
WalkPlan plan_walk(int tile, int rows, int d_in, int n_seq, const int32_t* off_host, int max_workgroups, unsigned short* order) {
  constexpr int kXcds = 8;
  constexpr double kMargin = 1.05;
  WalkPlan plan{};
  const bool big = tile == 256;
  const int tiles_m = (rows + tile - 1) / tile, tiles_n = (d_in + tile - 1) / tile, tiles = tiles_m * tiles_n, rest = tiles % kXcds;
  const long long pairs = (long long)tiles * n_seq;
  const int resident = max_workgroups > 0 ? max_workgroups / kXcds : (big ? 32 : 64);
  auto length = [&](int i) { return off_host ? off_host[i + 1] - off_host[i] : 1024; };
  auto most_of = [&](const int* first) {
    int most = 0;
    for (int x = 0; x < kXcds; ++x) most = std::max(most, first[x + 1] - first[x]);
    return most;
  };
  if (!big && pairs <= kXcds * resident) {
    plan.kind = kSingle;
    cut_pairs(tiles, n_seq, [&](int i) { return length(i) + kPairTokens; }, plan.first);
    plan.per_xcd = most_of(plan.first);
    return plan;
  }

  unsigned long long keys[1024];                                    // longest first, then as they come
  for (int i = 0; i < n_seq; ++i) keys[i] = (unsigned long long)length(i) << 10 | (unsigned)(1023 - i);
  std::sort(keys, keys + n_seq, std::greater<unsigned long long>());
  for (int k = 0; k < n_seq; ++k) order[k] = (unsigned short)(1023 - (int)(keys[k] & 1023));
  const double around = big ? 4.0 : 3.0, block = big ? 0.6e-6 : 0.35e-6;
  double weight[1024], total = 0.0;
  long long tokens = 0;
  for (int k = 0; k < n_seq; ++k) {
    const int len = length(order[k]);
    tokens += len;
    weight[k] = (len > 32 ? (len + 31) / 32 : 1) + around;
    total += tiles * weight[k];
  }
  int first[kXcds + 1], alone[2][kXcds] = {};
  cut_pairs(tiles, n_seq, [&](int k) { return length(order[k]) + kPairTokens; }, first);
  const int of_dealt = (int)std::min<long long>((pairs + kXcds - 1) / kXcds, resident), of_ranges = std::min(most_of(first), resident);
  const double even = total / (kXcds * resident);
  double t_dealt = even, t_ranges = even;
  // The longest walk over W workgroups of the pairs that run(k, count) is called for, `count` of sequence k.  Those of the first
  // sequences that outlast the rest's even share stay alone.
  auto share_out = [&](auto&& runs, int W, int& ones) {
    double left = 0.0, longest = 0.0, load[64] = {};
    runs([&](int k, int count) { left += weight[k] * count; return true; });
    ones = 0;
    runs([&](int k, int count) {
      if (ones + count >= W || weight[k] * (W - ones) < left) return false;
      ones += count;
      left -= weight[k] * count;
      return true;
    });
    const int n = W - ones;
    int skip = ones, at = 0, step = 1;
    runs([&](int k, int count) {
      if (skip > 0) {
        longest = std::max(longest, weight[k]);
        skip -= count;
        return true;
      }
      for (int c = 0; c < count; ++c) {                             // to and fro, as PairWalk goes
        load[at] += weight[k];
        if (at + step < 0 || at + step == n) step = -step; else at += step;
      }
      return true;
    });
    return std::max(longest, *std::max_element(load, load + n));
  };
  if (weight[0] > even / 16.0) {                                    // else shares are even in either arrangement
    for (int x = 0; x < kXcds; ++x) {
      const double walk = share_out([&](auto&& run) {
        for (int id = first[x]; id < first[x + 1];) {
          const int k = id / tiles, upto = std::min((k + 1) * tiles, first[x + 1]);
          if (!run(k, upto - id)) break;
          id = upto;
        }
      }, of_ranges, alone[1][x]);
      t_ranges = std::max(t_ranges, walk);
    }
    auto share = [&](int x, int k) { return tiles / kXcds + (((x - k * rest) & 7) < rest ? 1 : 0); };
    int ones = 0;
    t_dealt = share_out([&](auto&& run) {                           // XCD 0; the others have the same but for odd tiles
      for (int k = 0; k < n_seq; ++k)
        if (!run(k, share(0, k))) break;
    }, of_dealt, ones);
    for (int x = 0; x < kXcds; ++x)
      for (int k = 0, at = 0; at < ones && k < n_seq; at += share(0, k), ++k)
        if (alone[0][x] + share(x, k) < of_dealt) alone[0][x] += share(x, k);
  }
  // operands: panels of a tile's width, a sequence's whole on one XCD, or on every XCD those of its eighth of the tiles
  const int whole = tiles_m + tiles_n, strip = tiles_n < 8 ? tiles_n : 8, eighth = (tiles + 7) / 8;
  int dealt = 2 * tiles;
  if (tiles > kXcds) dealt = kXcds * (std::min(eighth, strip) + (eighth + strip - 1) / strip);
  dealt = std::min(std::max(dealt, whole), kXcds * whole);
  const bool counted = tiles <= (big ? 24 : 40);
  const double panel = counted ? (double)tokens * tile * 2.0 / 8.0e12 : 0.0;
  auto time = [&](double walk, int panels) {
    const double t = walk * block, u = panels * panel + (double)n_seq * rows * d_in * 2.0 / 4.5e12;
    return std::max(t, u) + 0.6 * std::min(t, u);
  };
  t_dealt = time(t_dealt, dealt);
  t_ranges = time(t_ranges, whole);
  (counted && !big ? t_ranges : t_dealt) /= kMargin;
  const bool ranges = t_ranges < t_dealt;
  plan.kind = ranges ? kRanges : kDealt;
  plan.per_xcd = ranges ? of_ranges : of_dealt;
  std::copy(alone[ranges], alone[ranges] + kXcds, plan.alone);
  if (ranges) std::copy(first, first + kXcds + 1, plan.first);
  return plan;
}

// The fp32 contraction's launch: tile side, groups of four waves per tile, and for the sum over all tokens the number of
// token chunks, by the smallest modelled time
//   max( lone * steps_max + fixed,                                   the longest workgroup's walk, alone on its unit
//        (max(work, adds) + epilogues) / 256 units ) + (split) beta pass
// with `steps` the groups * 16 token steps of a workgroup, work = sum of steps * busy, adds = chunks * outputs * 3 ps (fp32
// atomics drain while others multiply).  Per shape, measured: `lone` the time of a step where a workgroup has its compute
// unit to itself, `busy` a step's share of a full unit, `epilogue` what a workgroup costs besides its steps:
//   128, 1 group   1536x1536, 16 sequences of 256 .. 1024: 276 us (64, 1 group: 340; 64, 4 groups: 602)
//   64, 1 group    768x768, 8 sequences of 30 .. 200: 18.5 us (128: 22.6; 64, 2 groups: 22.7)
//   64, 2 groups   1024x256, 8 sequences of 400 .. 1500: 45 us (64, 1 group: 48; 128: 80)
//   64, 4 groups   256x1280, 2 sequences, 3159 tokens: 41 us (64, 1 group: 66; 128: 123)
SplitContractionPlan plan_split_contraction(int rows, int d_in, int n_tokens, int n_seq, const int32_t* off_host,
                                            bool per_sequence) {
  struct Shape { int tile, groups; double lone, busy, epilogue, fixed; };
  static const Shape shapes[] = {{128, 1, 1.1e-6, 0.785e-6, 3.9e-6, 5.0e-6},
                                 {64, 1, 0.58e-6, 0.24e-6, 1.25e-6, 4.5e-6},
                                 {64, 2, 0.87e-6, 0.56e-6, 1.5e-6, 5.5e-6},
                                 {64, 4, 1.6e-6, 1.7e-6, 2.5e-6, 7.0e-6}};
  constexpr double kBeta = 6.0e-6, kAdd = 3.0e-12, kUnits = 256.0;
  constexpr int kBlock = 16;
  SplitContractionPlan pl{128, 1, 1, n_tokens > 0 ? n_tokens : 1, 0};
  // 16-token blocks in all and of the longest sequence (every sequence ends in a block of its own)
  long long blocks = 0, longest = 0;
  for (int i = 0; i < n_seq; ++i) {
    const long long len = off_host ? off_host[i + 1] - off_host[i] : n_tokens / n_seq;
    blocks += (len + kBlock - 1) / kBlock;
    if (len > longest) longest = len;
  }
  const double outputs = (double)rows * d_in;
  double best = 0.0;
  bool first = true;
  for (const Shape& sh : shapes) {
    const double tiles = (double)((rows + sh.tile - 1) / sh.tile) * ((d_in + sh.tile - 1) / sh.tile);
    const int step = sh.groups * kBlock;
    for (int w = 1; w <= (per_sequence ? 1 : 64); ++w) {
      if (w > 1 && n_tokens / w < step) break;
      const double items = per_sequence ? n_seq : w;
      const double steps = (double)blocks / sh.groups / items;
      const double steps_max = per_sequence ? (double)((longest + step - 1) / step) : steps;
      double work = tiles * items * steps * sh.busy;
      const double adds = w > 1 ? w * outputs * kAdd * kUnits : 0.0;
      if (adds > work) work = adds;
      const double full = (work + tiles * items * sh.epilogue) / kUnits, alone = steps_max * sh.lone + sh.fixed;
      const double t = (full > alone ? full : alone) + (w > 1 ? kBeta : 0.0);
      if (first || t < best) {
        best = t;
        first = false;
        pl.tile = sh.tile;
        pl.groups = sh.groups;
        pl.n_chunks = w;
      }
    }
  }
  if (pl.n_chunks > 1) {
    pl.chunk_tokens = ((n_tokens + pl.n_chunks - 1) / pl.n_chunks + kBlock - 1) / kBlock * kBlock;
    pl.n_chunks = (n_tokens + pl.chunk_tokens - 1) / pl.chunk_tokens;
  }
  // Longest first where the launch has more workgroups than are resident at a time (three per compute unit; from one per unit
  // on it would pay as well) and the longest sequence outlasts the mean by more than it takes every workgroup to find its
  // sequence (n_seq steps, a lane of a wave per sequence).  804x860, 22 sequences of 195 tokens on average and 370 at most: 58.9
  // -> 50.5 us; 988x388, 34 of 440 and 895: 118 -> 99; of 33 random layers this side of the line 31 gained, 0.89x on average.
  // Past it up to half was lost: 1508x152, 62 of 22 and 39: 21.0 -> 33.4; 484x2420, 32 of 90 and 150: 60.9 -> 66.2; 256x284,
  // 52 of 158 each: 18.5 -> 21.0.
  const double tiles = (double)((rows + pl.tile - 1) / pl.tile) * ((d_in + pl.tile - 1) / pl.tile);
  pl.longest_first = per_sequence && n_seq <= 64 && tiles * n_seq > 768.0 && longest - n_tokens / n_seq >= 128;
  return pl;
}

int stash_tile_order_ok(int d_out, int d_in, int n_tokens, int n_seq, const int32_t* off_host) {
  // multiples of the larger tile, so that a band of output rows may pick either tile size
  if (d_out % 256 || d_in % 256) return 0;
  return plan_contraction(d_out, d_in, n_tokens, n_seq, off_host, true).tile;
}

}  // namespace isopo
