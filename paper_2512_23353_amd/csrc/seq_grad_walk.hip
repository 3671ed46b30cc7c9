// Streaming bf16 contraction, workgroups that walk a list of work: the per-sequence gradients G_i = Delta_i^T X_i
// (`grad_out.T @ act_in` of both hook listings), row-major and in tile order, and the sums over all tokens (dW = Delta^T X,
// dW = Delta^T diag(c_tok) X) whose tokens are not cut into chunks.
//
// Tiles, LDS ring, swizzle and transposing fragment reads are those of seq_grad_stream.hip.  Two things bound a launch besides
// the matrix cores and the board's power:
//  * what a work item costs besides its tokens.  A workgroup per item waits for its first operands with idle matrix cores, and
//    again for the stores of its tile (5 us per 256x256 tile, 18 us for the fp32 tile of a sum, against 0.55 us per block of 32
//    tokens).  Here a workgroup's items are one stream of token blocks: the loads run on into the next item while the last
//    blocks of this one are multiplied and its tile is stored, no barrier or wait stands between two items, and the only
//    pipeline to fill is the first.  Which items those are is fixed at launch (plan_walk, PairWalk in pair_walk.h): no counters
//    to clear and to wait for.
//  * what a wave issues.  One wave per SIMD has time for about three instructions beside each MFMA.  A token block of 64 MFMAs
//    is 160 instructions, about 30 fewer than with a load's address formed by itself and the buffer descriptors copied and
//    clamped per block.
// 14336x4096, 32 sequences, 70429 tokens: 6.43 -> 6.19 ms (1.34 PFLOP/s); 1024x4096, the same tokens: 520 -> 485 us; 8960x1536,
// 256 sequences, 85229: 2.88 -> 2.56 ms (HBM: 7 GB of stash); 1536x1536, 16 sequences, 10685: 60.5 -> 56 us; the weighted sum
// 27648x5120 over 1279 tokens of 8 sequences: 490 -> 405 us.  Tried and level: loads issued half a block earlier (the ring has
// room for it, since a block's stage is free at its barrier), the XCDs set off against each other in time so that their
// stores do not meet.
#include "pair_walk.h"
#include "seq_grad_stream.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace isopo {
namespace {

enum { kSeq, kSum, kWeighted };          // per-sequence gradients; sum over all tokens, plain and weighted

// f(0) .. f(N - 1), the index a constant
template <class F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

struct WalkParams {
  const u16* X;
  const u16* Delta;
  const int32_t* off;
  const float* c;                        // weighted sum: one coefficient per sequence
  void* out;
  int d_in, d_out, n_seq, n_tokens;
  int row0, row_end, out_row0;
  long long out_seq_stride;
  float beta;
  TileGrid grid;
  TileDiv by_tiles;                      // of the grid
  int per_xcd;                           // workgroups
  struct { int first, end, alone, unused; } xcd[8];                   // per-sequence launch: see PairWalk
  unsigned* queue;                       // a caller's scratch, cleared
};
struct OrderedWalkParams : WalkParams {
  unsigned short order[1024];            // of the sequences in the list, longest first
};

// T: side of the output tile.  NW: waves per workgroup, a 2 x NW/2 arrangement of wave tiles; four on the per-sequence launch
// (on the 256x256 tile one wave per SIMD with its 256 accumulators per lane pinned to the AGPRs), eight on the sums (two waves
// per SIMD, 128 accumulators per lane in VGPRs), as in seq_grad_stream.hip.  THROUGH: a row-major stash goes past the L2s at once.
template <int T, int KIND, int WALK, bool TILED, int NW, bool THROUGH, class Params>
__device__ __forceinline__ void seq_grad_walk_body(const Params& p_) {
  static_assert(KIND == kSeq || !TILED, "tile order is a layout of the per-sequence stash");
  static_assert(NW == 4 || NW == 8, "waves per workgroup");
  constexpr bool SEQ = KIND == kSeq, WTD = KIND == kWeighted;
  constexpr bool TABLE = SEQ && WALK != kSingle;               // a workgroup of one pair reads its sequence's offsets itself
  // The transposed products (rows of X's features, columns of Delta's): a lane then holds runs of a row of the result and
  // stores 16 bytes at a time, a row-major bf16 tile without a trip through LDS, an fp32 tile in a quarter of the stores.  Tile
  // order is defined by the plain ones.
  constexpr bool SWAP = !TILED;
  constexpr bool PAIRED = SEQ && SWAP;                         // bf16: two fragments' runs of four make one of eight
  constexpr int WNC = NW / 2, NT = 64 * NW;                    // waves along the tile's columns; threads
  constexpr int WM = T / 2, WN = T / WNC;
  constexpr unsigned P = T * 2;                                // LDS row pitch, bytes (no padding: swizzled)
  constexpr unsigned HALF = BK * P, STAGE = 2 * HALF;          // Delta's rows, then X's
  constexpr int LH = HALF / 1024 / NW, LPT = 2 * LH;           // 1 KiB wave-loads per wave: of an operand, of a block
  constexpr int RPL = 1024 / P;                                // tile rows per wave-load
  constexpr int FM = WM / 16, FN = WN / 16, RB = FM / 2, H = RB * FN;   // fragments; rows and MFMAs of half a block
  constexpr bool AGPR = FM * FN * 4 > 128;
  constexpr int STORES = SEQ ? FM * FN / 2 : FM * FN;          // of a finished tile, per wave
  constexpr int MIN_BLOCKS = WTD ? 2 : 1;                      // a segment's first block and its last are two
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned smem_base = (unsigned)(size_t)(lds_void_ptr)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  auto uniform = [](int a) { return __builtin_amdgcn_readfirstlane(a); };
  const int wave = uniform(tid >> 6), wm = wave / WNC, wn = wave % WNC;
  // The parameters that the walk needs, fetched together and kept: left to itself the compiler fetches each where it is first
  // used, one trip to memory after the other ahead of the first operand load, and again where a walk comes to its next pair.
  // 256x64, 76 sequences of 17 tokens: 5.7 -> 4.7 us.
  WalkParams p = p_;
  int first = 0, end = 0, alone = 0;
  if constexpr (SEQ) {
    first = p_.xcd[blockIdx.x & 7].first;
    end = p_.xcd[blockIdx.x & 7].end;
    alone = p_.xcd[blockIdx.x & 7].alone;
  }
  asm volatile("" : "+s"(p.X), "+s"(p.Delta), "+s"(p.d_in), "+s"(p.d_out), "+s"(p.n_seq), "+s"(p.row0), "+s"(p.per_xcd));
  if constexpr (SEQ)
    asm volatile("" : "+s"(p.grid.m), "+s"(p.grid.n), "+s"(p.grid.strip.d), "+s"(p.grid.strip.mul), "+s"(p.grid.last.d),
                      "+s"(p.grid.last.mul), "+s"(p.grid.width), "+s"(p.grid.across.d), "+s"(p.grid.across.mul));
  if constexpr (SEQ)
    asm volatile("" : "+s"(p.by_tiles.d), "+s"(p.by_tiles.mul), "+s"(first), "+s"(end), "+s"(alone));

  // ---- the ranges of tokens: the sequences in the order they are walked in, or the segments of the weighted sum ----
  // Weighted sum: the tokens are walked segment by segment (a segment: a sequence that has tokens and a non-zero
  // coefficient), each in token blocks of its own, so that no block mixes two sequences (rows past a segment's end arrive as
  // zeros).  The accumulators hold the sum in units of the current segment's coefficient: tokens enter the MFMAs unscaled, and
  // where a new segment opens the accumulators are multiplied once by c_previous / c_new.  The epilogue multiplies by the last
  // segment's coefficient.  No operand is scaled or rounded.
  constexpr int kMaxSeq = 1024;            // the library's limit on sequences per layer
  __shared__ int sh_tok[TABLE || WTD ? kMaxSeq : 1], sh_len[TABLE || WTD ? kMaxSeq : 1];
  __shared__ float sh_ratio[WTD ? kMaxSeq : 1];
  __shared__ short sh_seq[TABLE ? kMaxSeq : 1];
  __shared__ int sh_count;
  __shared__ float sh_last_c;
  [[maybe_unused]] int n_seg = 0;
  [[maybe_unused]] float last_c = 0.f;
  [[maybe_unused]] auto offset = [&](int k) {
    return ((const __attribute__((address_space(4))) int32_t*)p.off)[uniform(k)];
  };
  if constexpr (TABLE) {
    for (int k = tid; k < p.n_seq; k += NT) {
      const int s = p_.order[k], o = p.off[s];
      sh_tok[k] = o;
      sh_len[k] = p.off[s + 1] - o;
      sh_seq[k] = (short)s;
    }
    __syncthreads();
  }
  if constexpr (WTD) {
    if (tid < 64) {
      int count = 0;
      for (int at = 0; at < p.n_seq; at += 64) {
        const int sq = at + lane;
        int a = 0, b = 0;
        float cs = 0.f;
        if (sq < p.n_seq) { a = p.off[sq]; b = p.off[sq + 1]; cs = p.c[sq]; }
        const bool valid = b > a && cs != 0.f;                 // a NaN coefficient is kept and spreads
        const unsigned long long mask = __ballot(valid);
        const int pos = count + __popcll(mask & ((1ull << lane) - 1ull));
        if (valid) { sh_tok[pos] = a; sh_len[pos] = b - a; sh_ratio[pos] = cs; }
        count += __popcll(mask);
      }
      if (lane == 0) sh_count = count;
    }
    __syncthreads();
    n_seg = uniform(sh_count);
    // coefficient -> ratio to the segment before (1 for the first), in place
    float ratio[kMaxSeq / NT];
#pragma unroll
    for (int q = 0; q < kMaxSeq / NT; ++q) {
      const int k = tid + NT * q;
      ratio[q] = (k > 0 && k < n_seg) ? sh_ratio[k - 1] / sh_ratio[k] : 1.f;
    }
    if (tid == 0) sh_last_c = n_seg > 0 ? sh_ratio[n_seg - 1] : 0.f;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kMaxSeq / NT; ++q) {
      const int k = tid + NT * q;
      if (k < n_seg) sh_ratio[k] = ratio[q];
    }
    __syncthreads();
    last_c = __builtin_bit_cast(float, uniform(__builtin_bit_cast(int, sh_last_c)));
  }
  auto blocks_of = [](int len) {
    const int n = (len + BK - 1) / BK;
    return n > MIN_BLOCKS ? n : MIN_BLOCKS;
  };

  // ---- loads ----
  // The loads' cursor is the two buffer descriptors of the next token block, of Delta's and of X's panel of the tile: address of
  // its first row, bytes to the end of its last valid row, so that rows past the end of a range arrive as zeros.  It moves on by
  // two 64-bit additions; all else is behind one branch, taken where a block is the last of its range or the range is through.
  const unsigned rbA = (unsigned)p.d_out * 2u, rbB = (unsigned)p.d_in * 2u;
  const int tiles = p.grid.m * p.grid.n;
  PairWalk<WALK> ahead((int)blockIdx.x, p.per_xcd, tiles, SEQ ? p.n_seq : 1, p.by_tiles, first, end, alone);   // of the loads
  PairWalk<WALK> walk = ahead;                                 // of the products
  v4i da, db;
  int cut_a = 0, cut_b = 0;                                    // bytes of a row ahead of the panels
  int rem = 0;                                                 // rows left of the range at the cursor
  [[maybe_unused]] int seg = 0, range_end = 0;                 // weighted sum: the segment; rem at its end
  // `left` rows, at most `most` and at least none: scalar instructions (the compiler's clamp is a vector one)
  auto rows_within = [](int left, auto most) {
    int rows;
    asm("s_max_i32 %0, %1, 0\n\ts_min_i32 %0, %0, %2" : "=s"(rows) : "s"(left), "n"(decltype(most)::value) : "scc");
    return rows;
  };
  auto set_rows = [&]() __attribute__((always_inline)) {
    const int rows = rows_within(rem, std::integral_constant<int, BK>{});
    int na = rows * (int)rbA - cut_a, nb = rows * (int)rbB - cut_b;
    asm("s_max_i32 %0, %0, 0\n\ts_max_i32 %1, %1, 0" : "+s"(na), "+s"(nb) : : "scc");
    da[2] = na;
    db[2] = nb;
  };
  auto set_address = [&](v4i& d, unsigned long long at) __attribute__((always_inline)) {
    d[0] = uniform((int)(unsigned)at);
    d[1] = uniform((int)(unsigned)(at >> 32));                 // device addresses have no bits where the stride lies
  };
  auto range_open = [&](int tok, int rows) __attribute__((always_inline)) {
    set_address(da, (unsigned long long)(p.Delta + (size_t)tok * p.d_out) + (unsigned)cut_a);
    set_address(db, (unsigned long long)(p.X + (size_t)tok * p.d_in) + (unsigned)cut_b);
    rem = rows;
    if constexpr (WTD) range_end = rows > BK ? 0 : -BK;
  };
  // the first range of the pair that `ahead` has come to
  auto pair_open = [&]() __attribute__((always_inline)) {
    rem = 0;                                                   // past the last pair: all-zero blocks
    if (ahead.more() && !(WTD && n_seg == 0)) {
      int tile_m, tile_n;
      tile_coords<SEQ ? 0 : kStrip>(ahead.tile(), p.grid, tile_m, tile_n);
      cut_a = uniform(p.row0 + tile_m * T) * 2;
      cut_b = uniform(tile_n * T) * 2;
      const int k = SEQ ? ahead.i : 0;
      if constexpr (KIND == kSum) {
        range_open(0, p.n_tokens);
      } else if constexpr (SEQ && !TABLE) {
        const int o = offset(k);
        range_open(o, offset(k + 1) - o);
      } else {
        range_open(uniform(sh_tok[k]), uniform(sh_len[k]));
      }
    }
  };
  auto cursor_add = [&]() __attribute__((always_inline)) {
    asm("s_add_u32 %0, %0, %4\n\ts_addc_u32 %1, %1, 0\n\ts_add_u32 %2, %2, %5\n\ts_addc_u32 %3, %3, 0"
        : "+s"(da[0]), "+s"(da[1]), "+s"(db[0]), "+s"(db[1]) : "s"(BK * rbA), "s"(BK * rbB) : "scc");
    rem -= BK;
  };
  auto cursor_step = [&]() __attribute__((always_inline)) {
    if (__builtin_expect(rem < BK, 0)) {
      if (rem <= (WTD ? range_end : 0)) {
        if (WTD && ++seg < n_seg) {
          range_open(uniform(sh_tok[seg]), uniform(sh_len[seg]));
        } else {
          seg = 0;
          ahead.next();
          pair_open();
        }
      }
      set_rows();
    }
  };
  da[0] = da[1] = db[0] = db[1] = 0;
  da[3] = db[3] = 0x00020000;
  pair_open();
  set_rows();

  // 16-byte column swizzle of token row r (fragments are read by lane groups whose rows lie 8 apart).
  auto swz = [](int r) { return ((r & 3) << 2) ^ (r & 2) ^ (((r >> 3) & 1) << 1); };
  unsigned offA[LH], offB[LH];
#pragma unroll
  for (int q = 0; q < LH; ++q) {
    const int r = (wave * LH + q) * RPL + lane / (64 / RPL);
    const int g = (lane % (64 / RPL)) ^ swz(r);
    offA[q] = (unsigned)r * rbA + (unsigned)(g * 16);
    offB[q] = (unsigned)r * rbB + (unsigned)(g * 16);
  }
  const unsigned dma_base = smem_base + (unsigned)(wave * LH) * 1024;

  // ---- the token block: one K = 32 step of the 16x16x32 MFMA, FM + FN fragments (16 features x 32 tokens each), FM x FN
  // MFMAs in two halves of FM / 2 rows, column by column.  Fragments are replaced in place as the MFMAs are done with them, so
  // that the fragment reads spread over the whole block and any number of blocks can follow each other: behind the second half
  // go the next block's first A rows and first B columns, behind the first half of that block the rest of both.
  typedef float f32x4v __attribute__((ext_vector_type(4)));
  constexpr int NB2 = FN == 8 ? 4 : (FM == 8 ? 2 : FN);        // B columns read in the second half
  unsigned adA[FM], adB[FN];
  {
    // lane (l, g4): token rows 8 g4 + l / 4 (+ 4 for the second read), features 4 (l % 4) ..+3 of the
    // fragment's 16; the transposing read leaves lane l with tokens 8 g4 ..+7 of feature l.  PAIRED: fragments 2q and 2q + 1
    // take features 8 (l % 4) ..+3 and +4 ..+7 of their 32, for l % 4 = 2 and 3 the other way round: the swizzle puts rows 8 apart
    // into the same four 16-byte columns, two apart, so that they meet in opposite halves.  (In the same halves every read
    // took three cycles of the LDS where it takes two.)
    const int l = lane & 15, g4 = lane >> 4;
    const int kr = 8 * g4 + (l >> 2);
    const int f = swz(kr);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int ca = wm * WM + i * 16 + 4 * (l & 3);
      adA[i] = smem_base + (unsigned)kr * P + (unsigned)(((ca >> 3) ^ f) << 4) + (unsigned)((ca & 7) * 2);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int cb = wn * WN + (PAIRED ? (j >> 1) * 32 + 8 * (l & 3) + 4 * ((j ^ (l >> 1)) & 1) : j * 16 + 4 * (l & 3));
      adB[j] = smem_base + HALF + (unsigned)kr * P + (unsigned)(((cb >> 3) ^ f) << 4) + (unsigned)((cb & 7) * 2);
    }
  }
  auto frag = [&](unsigned a) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(a));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(a + 4 * P));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  f32x4v acc[FM][FN];
  bf16x8 fa[FM], fb[FN];
  unsigned at = 0;                                             // of this block in the ring, bytes
  int since = 2;                                               // blocks since a tile was last stored
  // The MFMAs are asm, so that every accumulator stays where it is (left to itself the register allocator shuttles them
  // between AGPRs and VGPRs) and the fragment reads and loads stay between the MFMAs they are written behind.  One wave per
  // SIMD issues three instructions beside each MFMA in the time the MFMA takes, and every instruction more is time lost: a load
  // is the MFMA's two neighbours, its LDS address ahead of it and the load behind it (the one instruction that has to lie
  // between them).  The weighted sum, whose accumulators ordinary instructions multiply, takes the builtin, which knows how
  // long to wait between the two, and pins the rest to its place.
#define ISOPO_MFMA "v_mfma_f32_16x16x32_bf16 %0, %1, %2, "
#define ISOPO_M0 "s_add_u32 m0, %3, %4\n\t"
#define ISOPO_DMA "\n\tbuffer_load_dwordx4 %5, %6, 0 offen lds"
  auto mfma = [&](auto first_c, f32x4v& d, bf16x8 l, bf16x8 r) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_c)::value;
    if constexpr (WTD) d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, r, d, 0, 0, 0);
    else if constexpr (AGPR && FIRST) asm volatile(ISOPO_MFMA "0" : "=a"(d) : "v"(l), "v"(r));
    else if constexpr (AGPR) asm volatile(ISOPO_MFMA "%0" : "+a"(d) : "v"(l), "v"(r));
    else if constexpr (FIRST) asm volatile(ISOPO_MFMA "0" : "=&v"(d) : "v"(l), "v"(r));
    else asm volatile(ISOPO_MFMA "%0" : "+v"(d) : "v"(l), "v"(r));
  };
  auto mfma_load = [&](auto first_c, f32x4v& d, bf16x8 l, bf16x8 r, unsigned lds, auto imm, unsigned voff, v4i rsrc)
                       __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_c)::value;
    constexpr int IMM = decltype(imm)::value;
    if constexpr (WTD) {
      mfma(first_c, d, l, r);
      __builtin_amdgcn_sched_barrier(0);
      load_lds16(rsrc, lds + IMM, voff);
    }
    else if constexpr (AGPR && FIRST)
      asm volatile(ISOPO_M0 ISOPO_MFMA "0" ISOPO_DMA : "=a"(d) : "v"(l), "v"(r), "s"(lds), "n"(IMM), "v"(voff), "s"(rsrc) : "memory", "scc");
    else if constexpr (AGPR)
      asm volatile(ISOPO_M0 "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" ISOPO_DMA : "+a"(d) : "v"(l), "v"(r), "s"(lds), "n"(IMM), "v"(voff), "s"(rsrc) : "memory", "scc");
    else if constexpr (FIRST)
      asm volatile(ISOPO_M0 ISOPO_MFMA "0" ISOPO_DMA : "=&v"(d) : "v"(l), "v"(r), "s"(lds), "n"(IMM), "v"(voff), "s"(rsrc) : "memory", "scc");
    else
      asm volatile(ISOPO_M0 "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" ISOPO_DMA : "+v"(d) : "v"(l), "v"(r), "s"(lds), "n"(IMM), "v"(voff), "s"(rsrc) : "memory", "scc");
  };
#undef ISOPO_MFMA
#undef ISOPO_M0
#undef ISOPO_DMA
  auto pin = [] { if constexpr (WTD) __builtin_amdgcn_sched_barrier(0); };
  // FIRST: the tile's first block, which starts the sums.
  // SCALE (weighted sum only): 1 in a segment's first block, 2 in its last.  The accumulators change their
  // unit from the previous segment's coefficient to this one's by a factor r; those of the first RB rows
  // take it in the last block of the segment before, behind the MFMAs of the other rows, the others in
  // this segment's first block, behind the MFMAs of the first RB rows: every accumulator is multiplied
  // once between its last MFMA of one segment and its first of the next, and the matrix pipes never wait
  // for the multiplications.
  auto token_block = [&](auto first_c, auto scale_c, [[maybe_unused]] float r) __attribute__((always_inline)) {
    constexpr int SCALE = decltype(scale_c)::value;
    static_assert(SCALE == 0 || WTD, "only the weighted sum has units");
    const unsigned next = (at + STAGE) & (NSTAGE * STAGE - 1);
    // the block AHEAD ahead goes where the block before this one was, whose last reads ended before its barrier
    const unsigned dma = dma_base + ((at - STAGE) & (NSTAGE * STAGE - 1));
    constexpr int N1 = FN - NB2 + FM - RB;                     // fragments read in the first half: the B ones, then the A ones
    constexpr int STEP = FN == 8 ? 3 : (FM == 8 ? 2 : 1);
    static_assert((N1 - 1) * STEP < H && LPT <= H, "the first half's MFMAs carry its fragment reads and the loads");
    unrolled([&](auto idx_c) __attribute__((always_inline)) {
      constexpr int idx = decltype(idx_c)::value, j = idx / RB, i = idx % RB, load = (idx + 1) * LPT / H - 1;
      const bf16x8 l = SWAP ? fb[j] : fa[i], r8 = SWAP ? fa[i] : fb[j];
      if constexpr (load < idx * LPT / H) mfma(first_c, acc[i][j], l, r8);
      else if constexpr (load < LH) mfma_load(first_c, acc[i][j], l, r8, dma, std::integral_constant<int, load * 1024>{}, offA[load], da);
      else mfma_load(first_c, acc[i][j], l, r8, dma, std::integral_constant<int, (int)HALF + (load - LH) * 1024>{}, offB[load - LH], db);
      if constexpr (SCALE == 1) acc[RB + idx / FN][idx % FN] = acc[RB + idx / FN][idx % FN] * r;
      if constexpr (idx % STEP == 0 && idx / STEP < N1) {
        constexpr int q = idx / STEP;
        pin();
        if constexpr (q < FN - NB2) fb[NB2 + q] = frag(at + adB[NB2 + q]);
        else fa[RB + q - (FN - NB2)] = frag(at + adA[RB + q - (FN - NB2)]);
      }
    }, std::make_integer_sequence<int, H>{});
    // Block it + 1 has landed (this wave's part; the barrier makes it everyone's), and this wave has what it wanted of block
    // it.  In flight behind it: blocks it + 2 and it + 3, and in the two blocks after a tile's end that tile's stores, which
    // went out between them.
    asm volatile("s_cmp_lt_u32 %0, 2\n\ts_cbranch_scc1 .Lisopo_relaxed%=\n\ts_waitcnt vmcnt(%1)\n.Lisopo_relaxed%=:\n\t"
                 "s_waitcnt vmcnt(%2) lgkmcnt(0)\n\ts_barrier"
                 : : "s"(since), "n"((AHEAD - 1) * LPT), "n"((AHEAD - 1) * LPT + STORES < 63 ? (AHEAD - 1) * LPT + STORES : 63)
                 : "memory", "scc");
    cursor_add();
    unrolled([&](auto idx_c) __attribute__((always_inline)) {
      constexpr int idx = decltype(idx_c)::value, j = idx / RB, i = RB + idx % RB;
      mfma(first_c, acc[i][j], SWAP ? fb[j] : fa[i], SWAP ? fa[i] : fb[j]);
      if constexpr (SCALE == 2) acc[idx / FN][idx % FN] = acc[idx / FN][idx % FN] * r;
      // A row a behind MFMA 0, 2, 6 or 7, 10 or 11; B column b once its MFMAs are through
#pragma unroll
      for (int a = 0; a < RB; ++a)
        if (idx == (a < 2 ? 2 * a : (FN == 8 ? 7 : 6) + 4 * (a - 2))) { pin(); fa[a] = frag(next + adA[a]); }
#pragma unroll
      for (int b = 0; b < NB2; ++b)
        if (idx == RB * (b + 1) - 1 + (FN == 8 ? 2 : (FM == 8 ? 1 : 0))) { pin(); fb[b] = frag(next + adB[b]); }
    }, std::make_integer_sequence<int, H>{});
    at = next;
    ++since;
    asm volatile("" : : : "memory");                           // the fragment reads stay in their block
    cursor_step();
  };

#pragma unroll
  for (int s = 0; s < AHEAD; ++s) {
#pragma unroll
    for (int q = 0; q < LPT; ++q) {
      const unsigned lds = dma_base + (unsigned)s * STAGE + (q < LH ? q * 1024 : HALF + (q - LH) * 1024);
      load_lds16(q < LH ? da : db, lds, q < LH ? offA[q] : offB[q - LH]);
    }
    cursor_add();
    cursor_step();
  }
  __builtin_amdgcn_s_waitcnt(0x0f70 | (((AHEAD - 1) * LPT) & 15) | ((((AHEAD - 1) * LPT) >> 4) << 14));
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < RB; ++i) fa[i] = frag(adA[i]);
#pragma unroll
  for (int j = 0; j < NB2; ++j) fb[j] = frag(adB[j]);

  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  [[maybe_unused]] constexpr std::integral_constant<int, 2> c2{};
  [[maybe_unused]] auto rd = [](float a) {
    if constexpr (AGPR) return acc_read(a); else return a;
  };
  while (walk.more()) {
    // ---- the tile's sums ----
    [[maybe_unused]] int seq = 0;
    if constexpr (WTD) {
      // segment by segment: the first block and the last carry the change of unit (ratio 1 after the last segment)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
      auto ratio_of = [&](int k) { return __builtin_bit_cast(float, uniform(__builtin_bit_cast(int, sh_ratio[k]))); };
      float r_in = 1.f;
      for (int k = 0; k < n_seg; ++k) {
        const int blocks = blocks_of(uniform(sh_len[k]));
        const float r_out = k + 1 < n_seg ? ratio_of(k + 1) : 1.f;
        token_block(c0, c1, r_in);
        for (int b = 2; b < blocks; ++b) token_block(c0, c0, 0.f);
        token_block(c0, c2, r_out);
        r_in = r_out;
      }
    } else {
      int tokens = p.n_tokens;
      if constexpr (TABLE) tokens = uniform(sh_len[walk.i]);
      else if constexpr (SEQ) tokens = offset(walk.i + 1) - offset(walk.i);
      const int blocks = blocks_of(tokens);
      token_block(c1, c0, 0.f);
      int b = 1;
      for (; b + 1 < blocks; b += 2) {
        token_block(c0, c0, 0.f);
        token_block(c0, c0, 0.f);
      }
      for (; b < blocks; ++b) token_block(c0, c0, 0.f);
    }
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");         // the last MFMAs have retired
    // The compiler sees no MFMA in asm, and the wait above does not hold back instructions on registers alone: where ordinary ones
    // read the accumulators they get them from here.  (AGPRs are read by volatile asm; the builtin's results it waits for itself.)
    if constexpr (!AGPR && !WTD) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));
    }

    // ---- epilogue: lane l holds, of block (i, j), rows 4 (l / 16) ..+3 of column l % 16 (SWAP: the transpose).  Nothing is
    // waited for: the next pair's operands are on their way, and as many stores go out on every way through here.
    if constexpr (TABLE) seq = uniform(sh_seq[walk.i]);
    else if constexpr (SEQ) seq = walk.i;
    int tile_m, tile_n;
    tile_coords<SEQ ? 0 : kStrip>(walk.tile(), p.grid, tile_m, tile_n);
    tile_m = uniform(tile_m);
    tile_n = uniform(tile_n);
    const int m0 = p.row0 + tile_m * T, n0 = tile_n * T;
    if constexpr (TILED) {
      // Tile order: two blocks side by side make the lane's 16 bytes; a piece (two blocks, 512 elements) is
      // one 1 KiB store of the wave.
      const int tile_row = (m0 - p.out_row0) / T;
      // the wave's quadrant of the tile, and inside each 16-row strip of the quadrant the wave's pieces (all of
      // them with four waves, the left or the right half with eight)
      constexpr int QP = (T / 2) / 32;                         // pieces per strip of a quadrant
      const int quad = wm * 2 + wn / (WNC / 2), piece0 = (wn % (WNC / 2)) * (FN / 2);
      u16* const tb = static_cast<u16*>(p.out) + (size_t)seq * p.out_seq_stride +
                      ((size_t)tile_row * p.grid.n + tile_n) * (T * T) + (size_t)quad * ((T / 2) * (T / 2));
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(tb, 0, (T / 2) * (T / 2) * 2, 0x00020000);
      constexpr int kNonTemporal = 2, kSc1 = 16;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int jp = 0; jp < FN / 2; ++jp) {
          u32x4 pk;
          pk[0] = pack_bf16(rd(acc[i][2 * jp][0]), rd(acc[i][2 * jp][1]));
          pk[1] = pack_bf16(rd(acc[i][2 * jp][2]), rd(acc[i][2 * jp][3]));
          pk[2] = pack_bf16(rd(acc[i][2 * jp + 1][0]), rd(acc[i][2 * jp + 1][1]));
          pk[3] = pack_bf16(rd(acc[i][2 * jp + 1][2]), rd(acc[i][2 * jp + 1][3]));
          // written once and read after the launch: non-temporal, so the stash does not push the operand panels out of the L2,
          // and past the L2 at once (sc1), which leaves nothing to be written back behind the launch: 1536x8960, 256 sequences
          // 2537 -> 2508 us; 512x512, 9 of 122 tokens 4.5 -> 4.2; 24 random layers 0.987x, the slowest 1.01x
          __builtin_amdgcn_raw_buffer_store_b128(pk, rs, (unsigned)lane * 16u, (i * QP + piece0 + jp) * 1024, kNonTemporal | kSc1);
        }
    } else {
      // Row-major: sixteen rows at a time through a buffer descriptor of their own, which ends with the last row that is
      // there; columns past the end of a row are sent out of its range.
      constexpr int ES = SEQ ? 2 : 4, LANE = 16 / ES, RUN = 4 * LANE, PER = SEQ ? 2 : 1;   // a lane's run, a row's, its blocks
      const size_t pitch = (size_t)p.d_in * ES;
      char* const tb = static_cast<char*>(p.out) + ((size_t)seq * p.out_seq_stride + (size_t)(m0 - p.out_row0) * p.d_in) * ES;
      unsigned voff[FN / PER];
#pragma unroll
      for (int j = 0; j < FN / PER; ++j) {
        const int n = n0 + wn * WN + j * RUN + (lane >> 4) * LANE;
        voff[j] = n < p.d_in ? (unsigned)(lane & 15) * (unsigned)pitch + (unsigned)(n * ES) : 0x80000000u;
      }
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int r0 = wm * WM + i * 16, rows = rows_within(p.row_end - m0 - r0, std::integral_constant<int, 16>{});
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(tb + (size_t)r0 * pitch, 0, rows * (int)pitch, 0x00020000);
        if constexpr (SEQ) {
#pragma unroll
          for (int j = 0; j < FN / 2; ++j) {
            const unsigned p0 = pack_bf16(rd(acc[i][2 * j][0]), rd(acc[i][2 * j][1]));
            const unsigned p1 = pack_bf16(rd(acc[i][2 * j][2]), rd(acc[i][2 * j][3]));
            const unsigned p2 = pack_bf16(rd(acc[i][2 * j + 1][0]), rd(acc[i][2 * j + 1][1]));
            const unsigned p3 = pack_bf16(rd(acc[i][2 * j + 1][2]), rd(acc[i][2 * j + 1][3]));
            const u32x4 pk = lane < 32 ? u32x4{p0, p1, p2, p3} : u32x4{p2, p3, p0, p1};
            // Half a line, of a row that starts anywhere in a line.  Left to the L2 the halves meet there; stored
            // non-temporally each goes to memory by itself: 2216x632, 83 sequences of 41 tokens: 57 us against 158;
            // 3256x2560, 28 of 346: 291 against 367; 568x1104, 79 of 213: 46 against 64.  Widths whose rows start at lines
            // are level on average (256x1536, 85 of 750: 83 against 74; 512x3328, 40 of 24: 40 against 50).
            constexpr int kSc1 = 16;
            __builtin_amdgcn_raw_buffer_store_b128(pk, rs, voff[j], 0, THROUGH ? kSc1 : 0);
          }
        } else {
          f32x4v old[FN];
          if (p.beta != 0.f) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
              old[j] = p.beta * __builtin_bit_cast(f32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, voff[j], 0, 0));
          } else {
#pragma unroll
            for (int j = 0; j < FN; ++j) old[j] = f32x4v{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            f32x4v o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = old[j][v] + (WTD ? last_c * rd(acc[i][j][v]) : rd(acc[i][j][v]));
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rs, voff[j], 0, 0);
          }
        }
      }
    }
    since = 0;
    walk.next();
  }
  if (SEQ && p.queue && blockIdx.x == 0 && tid < 8) p.queue[tid] = 0u;
  __builtin_amdgcn_s_waitcnt(0x0f70);                          // loads into the LDS of a workgroup that is gone
}

template <int T, int OCC, int WALK, bool TILED, bool THROUGH, class Params>
__global__ __launch_bounds__(256, OCC) void seq_grad_walk_kernel(Params p) {
  seq_grad_walk_body<T, kSeq, WALK, TILED, 4, THROUGH>(p);
}

template <int T, int OCC, int KIND>
__global__ __launch_bounds__(512, OCC) void seq_grad_walk_waves8_kernel(WalkParams p) {
  seq_grad_walk_body<T, KIND, kDealt, false, 8, false>(p);
}

template <int T, int OCC, int KIND, int WALK, bool TILED, int NW, bool THROUGH, class Params>
hipError_t launch_walk(const Params& p, hipStream_t s) {
  constexpr size_t smem = (size_t)NSTAGE * BK * T * 2 * 2;
  auto kern = [] {
    if constexpr (NW == 8) return &seq_grad_walk_waves8_kernel<T, OCC, KIND>;
    else return &seq_grad_walk_kernel<T, OCC, WALK, TILED, THROUGH, Params>;
  }();
  // once per process (static initialisation is thread-safe); a failure is returned by every call
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(8u * (unsigned)p.per_xcd), dim3(64 * NW), smem, s, p);
  return hipGetLastError();
}

// Columns of a strip of tiles.  An XCD's workgroups take neighbouring tiles, and what bounds a launch beside the power limit is
// what they read from beyond their L2: with 32 tiles of an item at a time, eight columns by four rows are 12 operand panels; of the
// fewer that an XCD takes of a sequence of up to 160 tiles, four columns make the more compact block.  Per-sequence launches, 8
// against 4 columns, 256x256 tiles: 4x16 tiles, 32 sequences of 512 .. 4096 tokens 484 / 468 us; 11x7, 92 of 86 175 / 167; 8x8, 40 of
// 87 69 / 66; 6x17, 12 of 481 86 / 83; 30 random ones 0.988x on average, the slowest 1.02x (2x17, 76 of 3568).  Per-sequence launches
// of more tiles: level or slower with 4 (56x16, 32 sequences 0.997x; 35x6, 256 sequences 2535 / 2580), few columns (up to 6): level or
// slower cut.  Sums are not part of the rule, their width is known to the compiler: of eleven uncut ones nine are level with 4,
// two would gain (108x20 tiles, 1238 tokens 448 / 438; 16x56, 8000 tokens 785 / 755).
int strip_width(const ContractionPlan& pl, bool per_sequence) {
  return per_sequence && pl.tiles_n >= 7 && (long long)pl.tiles_m * pl.tiles_n <= 160 ? 4 : kStrip;
}

// False: nothing to do, or (status) too much of it.
bool fill_params(const SeqGradArgs& a, const ContractionPlan& pl, WalkParams& p, hipError_t& status) {
  const long long tiles = (long long)pl.tiles_m * pl.tiles_n, pairs = tiles * (a.per_sequence ? a.n_seq : 1);
  status = pairs > 0x3fffffffLL ? hipErrorInvalidValue : hipSuccess;
  if (pairs <= 0 || status != hipSuccess) return false;
  p.X = static_cast<const u16*>(a.X); p.Delta = static_cast<const u16*>(a.Delta); p.off = a.off; p.c = a.c; p.out = a.out;
  p.d_in = a.d_in; p.d_out = a.d_out; p.n_seq = a.n_seq; p.n_tokens = a.n_tokens;
  p.row0 = a.row0; p.row_end = a.row0 + a.rows; p.out_row0 = a.out_row0;
  p.out_seq_stride = a.out_seq_stride; p.beta = a.beta;
  p.grid = tile_grid(pl.tiles_m, pl.tiles_n, strip_width(pl, a.per_sequence));
  p.by_tiles = tile_div_by((unsigned)tiles);
  p.queue = nullptr;
  return true;
}

template <int KIND>
hipError_t launch_sum(const SeqGradArgs& a, const ContractionPlan& pl, hipStream_t s) {
  WalkParams p;
  hipError_t status;
  if (!fill_params(a, pl, p, status)) return status;
  p.per_xcd = std::min((pl.tiles_m * pl.tiles_n + 7) / 8, 32);
  return launch_walk<256, 1, KIND, kDealt, false, 8, false>(p, s);
}

template <int T, int OCC, bool TILED, bool THROUGH>
hipError_t launch_sequences(const SeqGradArgs& a, const ContractionPlan& pl, hipStream_t s) {
  OrderedWalkParams p;
  hipError_t status;
  if (!fill_params(a, pl, p, status)) return status;
  const int budget = T == 256 ? a.max_workgroups : 0;
  const WalkPlan w = plan_walk(T, a.rows, a.d_in, a.n_seq, a.off_host, budget, p.order);
  p.per_xcd = w.per_xcd;
  if (budget > 0) p.queue = a.queue;
  for (int x = 0; x < 8; ++x) p.xcd[x] = {w.first[x], w.first[x + 1], w.alone[x], 0};
  if constexpr (T == 128)
    if (w.kind == kSingle) return launch_walk<T, OCC, kSeq, kSingle, TILED, 4, THROUGH>(static_cast<const WalkParams&>(p), s);
  return w.kind == kRanges ? launch_walk<T, OCC, kSeq, kRanges, TILED, 4, THROUGH>(p, s)
                           : launch_walk<T, OCC, kSeq, kDealt, TILED, 4, THROUGH>(p, s);
}

}  // namespace

hipError_t launch_seq_grad_walk(const SeqGradArgs& a, const ContractionPlan& pl, hipStream_t s) {
  const bool big = pl.tile == 256;
  if (a.per_sequence) {
    if (a.tile_order) {
      // the caller has checked stash_tile_order_ok; anything else would scatter the stores
      if (a.rows % pl.tile || a.d_in % pl.tile || a.row0 % pl.tile || a.out_row0 % pl.tile) return hipErrorInvalidValue;
      return big ? launch_sequences<256, 1, true, false>(a, pl, s) : launch_sequences<128, 2, true, false>(a, pl, s);
    }
    // Row by row, where rows start at lines and the last-level cache (256 MiB) takes the stash: past the L2s at once, as in tile order.
    // Whole steps, us through the L2 and past it: 1448x256, 7 sequences of 512 tokens 26.9 / 25.5; 248x4800, 10 of 24 38.0 / 36.4;
    // 1488x1792, 9 of 745 61.2 / 59.9; 24 random ones 0.985x, the slowest 1.003x.  Larger stashes lose (1280x2944, 126 of 126, 950 MB
    // 634 / 668), and rows that start within lines up to a third (264x824, 201 of 88 90 / 119).
    if (a.d_in % 64 == 0 && 2LL * a.n_seq * a.rows * a.d_in <= 256LL << 20)
      return big ? launch_sequences<256, 1, false, true>(a, pl, s) : launch_sequences<128, 2, false, true>(a, pl, s);
    return big ? launch_sequences<256, 1, false, false>(a, pl, s) : launch_sequences<128, 2, false, false>(a, pl, s);
  }
  if (!big || pl.n_chunks > 1) return hipErrorInvalidValue;
  return a.c != nullptr ? launch_sum<kWeighted>(a, pl, s) : launch_sum<kSum>(a, pl, s);
}

}  // namespace isopo
