// Token-reduction contraction on the matrix cores, fp32 inputs:
//     out[o][k] = sum_t scale(t) * Delta[t][o] * X[t][k]
// which is the per-sequence log-probability gradient G_i = Delta_i^T X_i of both
// hook listings (`grad_out.T @ act_in`) when t runs over one sequence, and the
// weighted contraction dW = Delta^T diag(c_tok) X (`grad += advantages[i] *
// scale_i * seq_logprob_grad`) when t runs over all tokens.  (bf16 inputs, the
// benchmark's case, take the streaming kernel in seq_grad_stream.hip.)
//
// What bounds it: the matrix cores.  The fp32 MFMA is a sixteenth of the bf16 MFMA's rate, so every fp32 value
// enters as the sum of three bf16 values, x = h + m + l with h = bf16(x), m = bf16(x - h), l = x - h - m
// (8 + 8 + 8 significant bits: exact from 2^-110 on, where the last bit of l is the last one bf16 has), and a product is
// formed from the six partial products hh, hm, mh, mm, hl, lh.  The three left out are at most 2^-24 of the product, half
// an ulp of the fp32 product itself; and six accumulations per sixteen tokens round the fp32 accumulator less often than
// one per two tokens did.  Against 64-bit sums over 34 layers of 32 .. 2048 by 32 .. 4096 the error of dW is 0.52 of the plain
// fp32 MFMA form's and that of K, with the Gram pass's own sums, 0.47 (geometric means; neither larger on any layer).
// 1536x1536, 16 sequences, 10685 tokens: 286 us per-sequence (176 TFLOP/s of fp32 products, 1.06 PFLOP/s of bf16 at the clock
// the power limit leaves) against 593 us (85 TFLOP/s) for 64x64 fp32 MFMA tiles; the weighted sum 304 against 677.
//
// A tile whose result is not finite (an infinity or NaN among the inputs, a value that bf16 rounds to infinity) or among
// whose inputs is a nonzero value below 2^-110 (in the weighted sum: a Delta times its coefficient) is formed again with
// fp32 MFMAs, the operands staged as they are in the same LDS (1536x1536, 16 sequences, 9499 tokens: 270 us, every tile formed
// twice 580; the second time from global memory, token by token: 835).  The operands are what has to be looked at, not the
// result: a small one may meet a large one, or stand beside ordinary ones.  The look costs a fifth of the staging's
// instructions, under 2 % of a launch.  Subnormal parts and sums are kept by the bf16 MFMA as by the fp32 one.
//
// Both operands are token-major: the reduction index is the slow index of X and of Delta.  A thread loads two
// features of eight consecutive tokens, splits them in registers and stores 16 bytes (one feature, eight tokens)
// per part to LDS, which is the bf16 MFMA's operand layout: the multiplying waves read their fragments with plain
// 16-byte reads.  Two LDS stages of sixteen tokens (24 KiB each), one barrier per stage.
//
// Work item = (sequence, 128x128 tile of the [d_out, d_in] output) or (token chunk, tile); four waves, 64x64 each.
// The walk over the tokens goes sequence by sequence, sixteen rows at a time; the last block of a sequence is
// zero-filled, so ragged lengths need no host-side padding.
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace isopo {
namespace {

constexpr int kBK = 16;                              // tokens per stage
constexpr int kParts = 3;                            // bf16 parts of an fp32 value
constexpr int kUnit = 16;                            // bytes: eight tokens of one feature and part
// one part of a stage, [operand][token half][feature], and the two stages of a group of four waves
constexpr int plane_bytes(int bt) { return 2 * 2 * bt * kUnit; }
constexpr int group_lds(int bt) { return 2 * kParts * plane_bytes(bt); }
// Sequences of so few tokens are formed with fp32 MFMAs at once: a single product would be rounded more than once and lack
// what is left out (off by 1.5e-7 of itself at most, 6e-8 here; of the sum of magnitudes for two tokens 1.6e-7 and 1.1e-7).
// From three on the parts' sums are the closer ones.
constexpr int kFewTokens = 2;
// The parts of a nonzero value below 2^-110 may not hold all of it.  As 2 bits - 1, the sign shifted out: zero is the largest.
constexpr unsigned kLossy = 2u * 0x08800000u - 1u;

struct SeqGradParams {
  const float* X;
  const float* Delta;
  const int32_t* off;
  const float* c;
  float* out;
  int d_in, d_out, n_seq, n_tokens;
  int row0, row_end;
  int out_row0;
  long long out_seq_stride;
  float beta;
  int tiles_n, tiles;
  int chunk_tokens;                                  // sum over all tokens: tokens per chunk
  int atomic;                                        // ... whose partial tiles are added to `out`
  int few_tokens;                                    // sum over all tokens: kFewTokens or fewer per block of tokens
  int longest_first;                                 // per sequence: item i is the i-th longest sequence (n_seq <= 64)
};

// The features' 16-byte units of a stage swap places in pairs in half of all groups of eight, so that the writes of two
// neighbouring features per lane (32 bytes apart from lane to lane) cover all banks, and the reads of 32
// consecutive features still do.
__device__ __forceinline__ int unit_pos(int f) { return f ^ (((f >> 3) ^ (f >> 4)) & 1); }

// Two fp32 values -> their three bf16 parts, packed low half first.
__device__ __forceinline__ unsigned pack_bf16(float x0, float x1) {
  unsigned r;                                        // the compiler converts each half by itself and packs them after
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(x0), "v"(x1));
  return r;
}
__device__ __forceinline__ void split2(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  h = pack_bf16(x0, x1);
  x0 -= __builtin_bit_cast(float, h << 16);
  x1 -= __builtin_bit_cast(float, h & 0xffff0000u);
  m = pack_bf16(x0, x1);
  x0 -= __builtin_bit_cast(float, m << 16);
  x1 -= __builtin_bit_cast(float, m & 0xffff0000u);
  l = pack_bf16(x0, x1);
}

// The token ranges a work item walks: one sequence, or the parts of the sequences inside a chunk of tokens with
// their coefficients (one range for the whole chunk where nothing is weighted).
template <bool WEIGHTED>
struct TokenWalk {
  const SeqGradParams& p;
  int seq, t, t_end, chunk_end;
  float scale = 1.f;
  __device__ __forceinline__ TokenWalk(const SeqGradParams& prm, int item) : p(prm) {
    if constexpr (!WEIGHTED) {
      t = p.off[item];
      t_end = p.off[item + 1];
    } else {
      t = item * p.chunk_tokens;
      chunk_end = p.n_tokens - t < p.chunk_tokens ? p.n_tokens : t + p.chunk_tokens;
      if (!p.c) {
        t_end = chunk_end;
      } else {
        int lo = 0, hi = p.n_seq;                    // largest seq with off[seq] <= t
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (p.off[mid] <= t) lo = mid; else hi = mid;
        }
        seq = lo;
        enter();
      }
    }
  }
  __device__ __forceinline__ void enter() {
    const int e = p.off[seq + 1];
    t_end = e < chunk_end ? e : chunk_end;
    scale = p.c[seq];
  }
  // The next block of at most `step` tokens: [b0, b1) with its coefficient.  Uniform over the workgroup.
  __device__ __forceinline__ bool next(int step, int& b0, int& b1, float& s) {
    if constexpr (WEIGHTED) {
      if (p.c)
        while (t >= t_end && t < chunk_end) { ++seq; enter(); }
    }
    if (t >= t_end) return false;
    b0 = t;
    b1 = t_end - t < step ? t_end : t + step;
    s = scale;
    t = b1;
    return true;
  }
};

// The sequence with `rank` longer ones (ties by index), n_seq <= 64: every wave finds it by itself, lane = sequence.
__device__ __forceinline__ int sequence_by_length(const int32_t* off, int n_seq, int rank, int lane) {
  const int len = lane < n_seq ? off[lane + 1] - off[lane] : -1;
  int longer = 0;
  for (int j = 0; j < n_seq; ++j) {
    const int lj = __builtin_amdgcn_readlane(len, j);
    longer += lj > len || (lj == len && j < lane) ? 1 : 0;
  }
  return __ffsll((long long)__ballot(lane < n_seq && longer == rank)) - 1;
}

// WT: side of a wave's square of outputs (64 or 32); a tile is 2 WT on a side.  KG groups of four waves share a
// tile: group g takes every KG-th block of tokens, the groups' sums meet in LDS.  THROUGH: the stash goes past the L2s at once.
template <int WT, int KG, bool WEIGHTED, bool THROUGH>
__global__ __launch_bounds__(256 * KG, WT == 64 ? 3 : (KG == 1 ? 6 : KG)) void seq_grad_kernel(SeqGradParams p) {
  constexpr int BT = 2 * WT, NB = WT / 32;           // NB x NB MFMA blocks of 32x32 per wave
  constexpr int FPL = BT / 64;                       // features a lane stages
  constexpr int PLANE = plane_bytes(BT), STAGE = kParts * PLANE;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave_id >> 2, wave = wave_id & 3;
  const int wm = wave >> 1, wn = wave & 1;
  unsigned char* lds = smem + group * group_lds(BT);

  // XCD x walks the x-th eighth of every item's tiles
  int item = blockIdx.x / p.tiles;
  const int tile = (int)xcd_contiguous(blockIdx.x % p.tiles, p.tiles);
  if (!WEIGHTED && p.longest_first) item = sequence_by_length(p.off, p.n_seq, item, lane);
  const int m0 = p.row0 + (tile / p.tiles_n) * BT;   // first output row (index into d_out)
  const int n0 = (tile % p.tiles_n) * BT;            // first output column (index into d_in)

  // staging: waves 0, 1 take Delta, waves 2, 3 X; even waves tokens 0..7 of a block, odd waves 8..15; lane l the
  // features FPL l ..
  const bool is_x = wave >= 2;
  const int half = wave & 1;
  const int pitch = is_x ? p.d_in : p.d_out;
  const int f0 = is_x ? n0 : m0, f_end = is_x ? p.d_in : p.row_end;
  const float* src = (is_x ? p.X : p.Delta) + f0;
  const int f_bytes = (f_end - f0 < BT ? f_end - f0 : BT) * 4;
  float r[2][8][FPL];                                // two stages in flight
  // one buffer descriptor per token row, empty for a row past the block's end: what lies outside arrives as zeros,
  // without a branch between the loads and the MFMAs they are meant to run under
  auto gload = [&](float (&d)[8][FPL], int b0, int b1) {
    const float* rowp = src + (size_t)(b0 + 8 * half) * pitch;
    const int rows = b1 - b0 - 8 * half;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const __amdgpu_buffer_rsrc_t row =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(rowp), 0, i < rows ? f_bytes : 0, 0x00020000);
      if constexpr (FPL == 2) {
        const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(row, lane * 8, 0, 0));
        d[i][0] = v.x; d[i][1] = v.y;
      } else {
        d[i][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(row, lane * 4, 0, 0));
      }
      rowp += pitch;
    }
  };
  unsigned least = ~0u;                              // of 2 bits - 1 of the values this lane staged
  // SPLIT: the three parts of each value; else fp32 rows, [operand][token][feature].  `rows`: the tokens the block has (what
  // lies past them is zero and stays it, whatever the coefficient)
  auto sstore = [&](auto split, float (&d)[8][FPL], int buf, float scale, int rows) {
    if constexpr (WEIGHTED) {
      if (!is_x) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int f = 0; f < FPL; ++f) d[i][f] *= split || 8 * half + i < rows ? scale : 0.f;
      }
    }
    if constexpr (split) {
      unsigned char* const o = lds + buf * STAGE + ((is_x ? 2 : 0) + half) * BT * kUnit;
#pragma unroll
      for (int f = 0; f < FPL; ++f) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const unsigned b = 2u * __builtin_bit_cast(unsigned, d[i][f]) - 1u;
          least = b < least ? b : least;
        }
        unsigned h[4], m[4], l[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split2(d[2 * q][f], d[2 * q + 1][f], h[q], m[q], l[q]);
        unsigned char* const of = o + unit_pos(FPL * lane + f) * kUnit;
        *reinterpret_cast<uint4*>(of) = make_uint4(h[0], h[1], h[2], h[3]);
        *reinterpret_cast<uint4*>(of + PLANE) = make_uint4(m[0], m[1], m[2], m[3]);
        *reinterpret_cast<uint4*>(of + 2 * PLANE) = make_uint4(l[0], l[1], l[2], l[3]);
      }
    } else {
      float* const o = reinterpret_cast<float*>(lds + buf * STAGE) + ((is_x ? kBK : 0) + 8 * half) * BT + FPL * lane;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int f = 0; f < FPL; ++f) o[i * BT + f] = d[i][f];
    }
  };

  f32x16 acc[NB][NB];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  };

  const int mw = m0 + wm * WT, nw = n0 + wn * WT;
  const bool live = mw < p.row_end && nw < p.d_in;   // edge tiles: this wave has outputs
  const unsigned char* const at = lds + (lane >> 5) * BT * kUnit + unit_pos(wm * WT + (lane & 31)) * kUnit;
  const unsigned char* const bt = lds + (2 + (lane >> 5)) * BT * kUnit + unit_pos(wn * WT + (lane & 31)) * kUnit;
  auto compute = [&](auto split, int buf, int tokens) {
    if constexpr (split) {
      // small products first: lh, hl, mm, mh, hm, hh
      constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
      bf16x8 a[NB][kParts], b[NB][kParts];
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int s = 0; s < kParts; ++s) {
          a[i][s] = *reinterpret_cast<const bf16x8*>(at + buf * STAGE + s * PLANE + i * 32 * kUnit);
          b[i][s] = *reinterpret_cast<const bf16x8*>(bt + buf * STAGE + s * PLANE + i * 32 * kUnit);
        }
#pragma unroll
      for (int s = 0; s < 6; ++s)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][pa[s]], b[j][pb[s]], acc[i][j], 0, 0, 0);
    } else {
      const float* const rows = reinterpret_cast<const float*>(lds + buf * STAGE) + (lane >> 5) * BT + (lane & 31);
      auto two = [&](int t) {
        float a[NB], b[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          a[i] = rows[t * BT + wm * WT + i * 32];
          b[i] = rows[(kBK + t) * BT + wn * WT + i * 32];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
      };
      two(0);
      if (tokens > 2) {
#pragma unroll
        for (int t = 2; t < kBK; t += 2) two(t);
      }
    }
  };

  auto pass = [&](auto split) {
    TokenWalk<WEIGHTED> walk(p, item);
    // A step is KG blocks of tokens, one per group; a group without one in the last step loads zeros.  Step s is
    // multiplied from LDS while step s + 1 is in registers and step s + 2 on its way there.
    auto fetch = [&](float (&d)[8][FPL], float& scale, int& rows) -> bool {
      int b0 = 0, b1 = 0;
      bool any = false;
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        int q0 = 0, q1 = 0;
        float qs = 1.f;
        const bool got = walk.next(kBK, q0, q1, qs);
        if (g == 0) any = got;
        if (g == group && got) { b0 = q0; b1 = q1; scale = qs; }
      }
      gload(d, b0, b1);
      rows = b1 - b0;
      return any;
    };
    float s0 = 1.f, s1 = 1.f;
    int n0, n1, in0, in1;                            // tokens of the two steps in registers, and of those in LDS
    clear();
    bool have0 = fetch(r[0], s0, n0), have1 = fetch(r[1], s1, n1);
    if (have0) { sstore(split, r[0], 0, s0, n0); in0 = n0; }
    __syncthreads();
    // The step in LDS buffer `buf` multiplied and the next one, `d`, split and stored in the other: one straight run of code, five
    // of the splitting's instructions behind each MFMA.  (A step that is none any more arrives as zeros and is read by nobody; a wave
    // without outputs multiplies zeros.)  One after the other, each behind a branch, the two took 3 % more: 2048x2048, 16 sequences,
    // 9345 tokens 435 -> 421 us; 36x1400, 20 of 480 35.8 -> 33.1; the weighted sum 3072x768, 4394 tokens 135 -> 131.  Four or six and
    // more between: 1 to 2 % of that lost.
    auto step = [&](int buf, int tokens, float (&d)[8][FPL], float scale, int rows) __attribute__((always_inline)) {
      compute(split, buf, tokens);
      sstore(split, d, buf ^ 1, scale, rows);
      if constexpr (split) {
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * NB * kParts, 0);         // LDS reads
#pragma unroll
        for (int q = 0; q < 6 * NB * NB; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                       // MFMA
          __builtin_amdgcn_sched_group_barrier(0x2, 5, 0);                       // VALU
        }
      }
    };
    while (have0) {
      const bool have2 = fetch(r[0], s0, n0);
      step(0, in0, r[1], s1, n1);
      in1 = n1;
      __syncthreads();
      if (!have1) break;
      have1 = fetch(r[1], s1, n1);
      step(1, in1, r[0], s0, n0);
      in0 = n0;
      __syncthreads();
      have0 = have2;
    }
  };

  bool fp32 = WEIGHTED ? p.few_tokens : p.off[item + 1] - p.off[item] <= kFewTokens;      // uniform
  if (!fp32) {
    pass(std::true_type{});
    unsigned top = 0;                                // largest magnitude, as bits (zero outside the layer)
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const unsigned bits = __builtin_bit_cast(unsigned, (float)acc[i][j][v]) & 0x7fffffffu;
          top = bits > top ? bits : top;
        }
    fp32 = __syncthreads_or(least < kLossy || top >= 0x7f800000u);
  }
  if (fp32) pass(std::false_type{});

  if constexpr (KG > 1) {
    // the groups' sums, added in group order (every stage has been read: the loop ends with a barrier)
    float* red = reinterpret_cast<float*>(smem);     // [group - 1][value][thread of the group]
    const int tg = wave * 64 + lane;
    if (group > 0) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) red[((group - 1) * NB * NB * 16 + (i * NB + j) * 16 + v) * 256 + tg] = acc[i][j][v];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] += red[(g * NB * NB * 16 + (i * NB + j) * 16 + v) * 256 + tg];
          __builtin_amdgcn_sched_barrier(0);         // sixteen reads in flight, not all at once: no spills
        }
  }
  if (!live) return;

  // Lane l holds column l%32 and rows acc_row(v, l) of each block.
  const int col = lane & 31;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = nw + j * 32 + col;
      if (n >= p.d_in) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = mw + i * 32 + acc_row(v, lane);
        if (m >= p.row_end) continue;
        const size_t idx = (size_t)(m - p.out_row0) * p.d_in + n;
        if constexpr (WEIGHTED) {
          float* o = p.out + idx;
          if (p.atomic) atomicAdd(o, acc[i][j][v]);
          else *o = (p.beta != 0.f ? p.beta * *o : 0.f) + acc[i][j][v];
        } else {
          float* const o = p.out + (size_t)item * p.out_seq_stride + idx;
          if constexpr (THROUGH) __hip_atomic_store(o, (float)acc[i][j][v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // sc1
          else *o = acc[i][j][v];
        }
      }
    }
  }
}

template <int WT, int KG, bool WEIGHTED, bool THROUGH>
hipError_t launch_cfg(SeqGradParams p, int rows, long long items, hipStream_t s) {
  constexpr int BT = 2 * WT;
  p.tiles_n = (p.d_in + BT - 1) / BT;
  const long long tiles = (long long)((rows + BT - 1) / BT) * p.tiles_n, blocks = items * tiles;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  p.tiles = (int)tiles;
  constexpr size_t smem = (size_t)KG * group_lds(BT);
  static_assert(smem >= (size_t)(KG - 1) * WT * WT * 4 * sizeof(float), "the groups' sums meet in LDS");
  auto kern = seq_grad_kernel<WT, KG, WEIGHTED, THROUGH>;
  // once per process and instantiation (static initialisation is thread-safe); a failure is returned by every call
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256 * KG), smem, s, p);
  return hipGetLastError();
}

template <bool WEIGHTED, bool THROUGH>
hipError_t launch_plan(const SeqGradParams& p, const SplitContractionPlan& pl, int rows, long long items, hipStream_t s) {
  if (pl.tile == 128) return launch_cfg<64, 1, WEIGHTED, THROUGH>(p, rows, items, s);
  if (pl.groups == 1) return launch_cfg<32, 1, WEIGHTED, THROUGH>(p, rows, items, s);
  return pl.groups == 2 ? launch_cfg<32, 2, WEIGHTED, THROUGH>(p, rows, items, s) : launch_cfg<32, 4, WEIGHTED, THROUGH>(p, rows, items, s);
}

}  // namespace

hipError_t launch_seq_grad(const SeqGradArgs& a, hipStream_t s) {
  if (a.bf16) return launch_seq_grad_stream(a, s);
  SeqGradParams p;
  p.X = static_cast<const float*>(a.X); p.Delta = static_cast<const float*>(a.Delta); p.off = a.off; p.c = a.c;
  p.out = static_cast<float*>(a.out);
  p.d_in = a.d_in; p.d_out = a.d_out; p.n_seq = a.n_seq; p.n_tokens = a.n_tokens;
  p.row0 = a.row0; p.row_end = a.row0 + a.rows; p.out_row0 = a.out_row0;
  p.out_seq_stride = a.out_seq_stride; p.beta = a.beta;
  p.chunk_tokens = 1;
  p.atomic = 0;
  long long blocks = (a.n_tokens + kBK - 1) / kBK;   // of tokens; in the weighted sum a sequence ends one
  if (a.c && a.off_host) {
    blocks = 0;
    for (int i = 0; i < a.n_seq; ++i) blocks += (a.off_host[i + 1] - a.off_host[i] + kBK - 1) / kBK;
  }
  p.few_tokens = a.n_tokens <= kFewTokens * blocks;
  const SplitContractionPlan pl = plan_split_contraction(a.rows, a.d_in, a.n_tokens, a.n_seq, a.off_host, a.per_sequence);
  p.longest_first = pl.longest_first;
  if (a.per_sequence) {
    // Stores past the L2s leave nothing to be written back behind the launch: whole calls 892x256, 19 sequences of 57 tokens 37.3 -> 35.3
    // us; 336x512, 7 of 28 23.1 -> 21.8; 1536x1536, 16 of 668 328 -> 325.  A row that does not start at a line leaves pieces of lines,
    // which then go to memory one by one instead of meeting in the L2: 1220x300, 40 of 147 (58 MB) 87.5 -> 89.8, so those only where the
    // L2s (32 MiB) hold the stash (2652x440, 6 of 41 45.2 -> 44.1; 768x468, 3 of 39 24.1 -> 23.3).
    if (a.d_in % 32 == 0 || (long long)a.n_seq * a.rows * a.d_in * 4 <= 32LL << 20) return launch_plan<false, true>(p, pl, a.rows, a.n_seq, s);
    return launch_plan<false, false>(p, pl, a.rows, a.n_seq, s);
  }
  p.chunk_tokens = pl.chunk_tokens;
  if (pl.n_chunks > 1) {
    p.atomic = 1;
    const hipError_t e = launch_apply_beta(p.out + (size_t)(a.row0 - a.out_row0) * a.d_in, (long long)a.rows * a.d_in, a.beta, s);
    if (e != hipSuccess) return e;
  }
  return launch_plan<true, false>(p, pl, a.rows, pl.n_chunks, s);
}

}  // namespace isopo
