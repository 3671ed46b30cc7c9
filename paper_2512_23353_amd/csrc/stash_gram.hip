// Gram matrix and weighted sum over the stash of per-sequence gradients.
//
//   K_ij = sum_p S[i][p] * S[j][p]          (interacting listing: ntk[i, j] =
//                                            sum(seq_grads[i] * seq_grads[j]))
//   dW[p] = beta dW[p] + sum_i c_i S[i][p]  (stack(seq_grads, -1) @ coefficients)
//
// Both read the stash once and are bound by HBM.  The products of the Gram matrix are formed by the kernels of
// stash_gram_stream.hip, which leave partial sums in fixed slots; here are the finishing kernel, which adds the slots
// in a fixed tree (K is bit-reproducible and exactly symmetric), and the weighted sum.
#include "common.h"
#include "gram_finish.h"
#include "kernels.h"

namespace isopo {
namespace {

constexpr int kGramSlots = 256;             // at most: one partial slot per workgroup of the streaming kernel

constexpr int tri(int nb) { return nb * (nb + 1) / 2; }

__global__ __launch_bounds__(kFinishThreads) void stash_gram_finish_kernel(GramFinish f) { gram_finish<false>(f); }

// The weighted sum: a thread takes VPT 16-byte vectors of every sequence, kSumThreads apart, so a workgroup reads VPT runs of 4 KiB
// side by side and VPT * 8 loads of a thread are in flight.  Bound by HBM; which VPT where: launch_stash_weighted_sum's rule.
constexpr int kSumThreads = 256;

// Past the last-level cache many times over nothing of dW would stay there: non-temporal.
template <int VPT, class V>
__device__ __forceinline__ void store_result(V* o, V v) {
  if constexpr (VPT == 4) __builtin_nontemporal_store(v, o); else *o = v;
}

// acc[q][e] += sum_i c_i * element e of vector q (at src + at[q] in sequence i)
template <bool BF16, int VPT>
__device__ __forceinline__ void sum_vectors(const char* __restrict__ src, size_t seq_bytes, const long long (&at)[VPT], int n_seq,
                                            const float* __restrict__ c, float (&acc)[VPT][BF16 ? 8 : 4]) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int q = 0; q < VPT; ++q)
#pragma unroll
    for (int e = 0; e < (BF16 ? 8 : 4); ++e) acc[q][e] = 0.f;
#pragma unroll 8
  for (int i = 0; i < n_seq; ++i) {
    const float ci = c[i];
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      // read once: non-temporal
      const u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + (size_t)i * seq_bytes + at[q]));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (BF16) {
          acc[q][2 * e] += ci * __builtin_bit_cast(float, w[e] << 16);
          acc[q][2 * e + 1] += ci * __builtin_bit_cast(float, w[e] & 0xffff0000u);
        } else {
          const unsigned bits = w[e];
          acc[q][e] += ci * __builtin_bit_cast(float, bits);
        }
      }
    }
  }
}

template <bool BF16, bool OUTB, int VPT>
__global__ __launch_bounds__(kSumThreads) void stash_weighted_sum_kernel(const void* __restrict__ stash, long long seq_stride,
                                                                         long long n_vec, int n_seq,
                                                                         const float* __restrict__ c, float beta,
                                                                         void* __restrict__ dW_out) {
  constexpr int kV = BF16 ? 8 : 4;
  for (long long v0 = (long long)blockIdx.x * (kSumThreads * VPT) + threadIdx.x; v0 < n_vec;
       v0 += (long long)gridDim.x * (kSumThreads * VPT)) {
    float acc[VPT][kV];
    long long at[VPT];
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      const long long v = v0 + q * kSumThreads;
      at[q] = (v < n_vec ? v : v0) * 16;
    }
    sum_vectors<BF16, VPT>(static_cast<const char*>(stash), (size_t)seq_stride * (BF16 ? 2 : 4), at, n_seq, c, acc);
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      const long long vi = v0 + q * kSumThreads;
      if (vi >= n_vec) break;
      const float (&s)[kV] = acc[q];
      if constexpr (OUTB) {
        // bf16 dW (bf16 stash only): the thread's eight values are one 16-byte vector
        static_assert(!OUTB || BF16, "a bf16 dW is formed from a bf16 stash");
        uint4* o = static_cast<uint4*>(dW_out) + vi;
        unsigned w[4] = {0u, 0u, 0u, 0u};
        if (beta != 0.f) {
          const uint4 old = *o;
          w[0] = old.x; w[1] = old.y; w[2] = old.z; w[3] = old.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = s[2 * e] + beta * __builtin_bit_cast(float, w[e] << 16);
          const float hi = s[2 * e + 1] + beta * __builtin_bit_cast(float, w[e] & 0xffff0000u);
          w[e] = (unsigned)f32_to_bf16_bits(lo) | ((unsigned)f32_to_bf16_bits(hi) << 16);
        }
        *o = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
        float* o = static_cast<float*>(dW_out) + vi * kV;
#pragma unroll
        for (int e = 0; e < kV; e += 4) {
          float4 r = make_float4(s[e], s[e + 1], s[e + 2], s[e + 3]);
          if (beta != 0.f) {
            const float4 old = *reinterpret_cast<const float4*>(o + e);
            r.x += beta * old.x; r.y += beta * old.y; r.z += beta * old.z; r.w += beta * old.w;
          }
          store_result<VPT>(reinterpret_cast<f32x4*>(o + e), f32x4{r.x, r.y, r.z, r.w});
        }
      }
    }
  }
}

// The same from a stash in tile order (see stash_tile_order_ok): a thread's eight values are four rows of
// two columns of dW, 16 apart; a wave stores, per value, four rows' runs of 16 consecutive floats, and the
// values q and q + 4 complete each other's 128-byte lines.
template <int T, bool OUTB, int VPT>
__global__ __launch_bounds__(kSumThreads) void stash_weighted_sum_tiled_kernel(const void* __restrict__ stash, long long seq_stride,
                                                                       long long n_vec, int n_seq,
                                                                       const float* __restrict__ c, float beta,
                                                                       void* __restrict__ dW_out, int d_in, int tiles_n) {
  constexpr int NP = T / 64;                       // 16x32 pieces per 16-row strip of a quadrant
  constexpr int QV = (T / 2) * (T / 2) / 8;        // 16-byte vectors per quadrant
  constexpr int TV = T * T / 8;                    // ... per tile
  static_assert(TV % (kSumThreads * VPT) == 0, "a workgroup's vectors are there");
  for (long long v0 = (long long)blockIdx.x * (kSumThreads * VPT) + threadIdx.x; v0 < n_vec;
       v0 += (long long)gridDim.x * (kSumThreads * VPT)) {
    float acc[VPT][8];
    long long at[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) at[u] = (v0 + u * kSumThreads) * 16;
    sum_vectors<true, VPT>(static_cast<const char*>(stash), (size_t)seq_stride * 2, at, n_seq, c, acc);
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const long long vi = v0 + u * kSumThreads;
      const float (&s)[8] = acc[u];
      const long long tile = vi / TV;
      const int r = (int)(vi % TV), quad = r / QV, r2 = r % QV, piece = r2 / 64, lane = r2 % 64;
      const int strip = piece / NP, jp = piece % NP;
      const int tile_m = (int)(tile / tiles_n), tile_n = (int)(tile % tiles_n);
      const int n0 = tile_n * T + (quad & 1) * (T / 2) + jp * 32 + (lane & 15);
      const int m0 = tile_m * T + (quad >> 1) * (T / 2) + strip * 16 + 4 * (lane >> 4);
      if constexpr (OUTB) {
        // bf16 dW: neighbouring lanes hold neighbouring columns; the even lane takes its neighbour's values of
        // the left 16 columns and stores pairs there, the odd lane does the same for the right 16 columns
        // (n_vec is a multiple of 64 for a stash in tile order, so every lane of a wave is here)
        __bf16* dW = static_cast<__bf16*>(dW_out);
        const bool odd = lane & 1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float got = __shfl_xor(odd ? s[q] : s[q + 4], 1, kWave);
          float lo = odd ? got : s[q], hi = odd ? s[q + 4] : got;
          unsigned* o = reinterpret_cast<unsigned*>(dW + (size_t)(m0 + q) * d_in + (n0 & ~1) + (odd ? 16 : 0));
          if (beta != 0.f) {
            const unsigned old = *o;
            lo += beta * __builtin_bit_cast(float, old << 16);
            hi += beta * __builtin_bit_cast(float, old & 0xffff0000u);
          }
          *o = (unsigned)f32_to_bf16_bits(lo) | ((unsigned)f32_to_bf16_bits(hi) << 16);
        }
      } else {
        float* dW = static_cast<float*>(dW_out);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          float* o = dW + (size_t)(m0 + (q & 3)) * d_in + n0 + 16 * (q >> 2);
          store_result<VPT>(o, (beta != 0.f ? beta * *o : 0.f) + s[q]);
        }
      }
    }
  }
}

}  // namespace

static int block_side(int n_seq, bool bf16) { return bf16 && n_seq > 16 ? 32 : 16; }

size_t stash_gram_slot_floats(int n_seq, bool bf16) {
  const int mb = block_side(n_seq, bf16);
  return (size_t)tri((n_seq + mb - 1) / mb) * mb * mb;
}

size_t stash_gram_partial_bytes(int n_seq, bool bf16) {
  if (n_seq > 128)
    return bf16 ? (size_t)stash_gram_large_slots(n_seq) * stash_gram_large_slot_floats(n_seq) * sizeof(float) : 0;
  return (size_t)kGramSlots * stash_gram_slot_floats(n_seq, bf16) * sizeof(float);
}

int stash_gram_slots(int n_seq, bool bf16, long long n_elem) {
  return n_seq > 128 ? stash_gram_large_slots(n_seq) : stash_gram_stream_slots(n_seq, bf16, n_elem);
}

hipError_t launch_stash_gram(const StashGramArgs& a, hipStream_t s) {
  if (a.n_seq > 128) return a.bf16 ? launch_stash_gram_large(a, s) : hipErrorInvalidValue;
  return launch_stash_gram_stream(a, s);
}

hipError_t launch_stash_gram_finish(const float* partials, bool bf16, int slots, int n_seq, float* K, hipStream_t s) {
  if (n_seq > 128) return bf16 ? launch_stash_gram_large_finish(partials, n_seq, K, s) : hipErrorInvalidValue;
  const GramFinish f = gram_finish_of(partials, bf16, slots, n_seq, K);
  hipLaunchKernelGGL(stash_gram_finish_kernel, dim3((unsigned)(f.slot_floats / 64)), dim3(kFinishThreads), 0, s, f);
  return hipGetLastError();
}

GramFinish gram_finish_of(const float* partials, bool bf16, int slots, int n_seq, float* K) {
  return {partials, slots, (long long)stash_gram_slot_floats(n_seq, bf16), n_seq, block_side(n_seq, bf16), K};
}

// Vectors per thread.  Four (and non-temporal stores) over stashes of 2 GiB and up of wide sequences: in tile order 4096x14336, 32
// sequences 751 -> 632 us (6.3 TB/s), 1536x8960, 256 1229 -> 1070, 5120x13824, 16 496 -> 455; of 13 random ones of n_vec from 1.5 M on
// 12 were level or gained (0.86 .. 1.02 of one vector; 2.1 M, 65 sequences 1.05), narrower ones lose to two.  Row by row only fp32
// from 3 M (4.2 M, 90 sequences 1039 -> 893): eleven below and in bf16 took 0.99 .. 1.21 of one vector's time where two take 0.90 .. 0.98.
// Two from four workgroups per compute unit on: 4096x1024, 32 sequences 54.5 -> 45.5 us; 2048x4096, 16 55.1 -> 48.8; of 90 random ones
// 0.79 .. 1.06 of one vector's time.  Below that row by row they lose, whatever the remainder (2.7 .. 3.6 per unit 1.03 .. 1.38, fewer up
// to four times the time: 2816x1024, 32 31 / 42 us; 460x3328 fp32, 53 50 / 61); in tile order they gain (0.87 .. 0.95, 1024x2048, 64
// 52.6 -> 45.2) where the units get like numbers of workgroups, the fullest no more than an eighth above the mean, else not (0.99 .. 1.11).
static int sum_vectors_per_thread(long long n_vec, int n_seq, bool bf16, bool tiled) {
  if (n_vec * n_seq >= (2LL << 30) / 16 && (tiled ? n_vec >= 3 << 19 : !bf16 && n_vec >= 3 << 20)) return 4;
  const long long blocks = (n_vec + 2 * kSumThreads - 1) / (2 * kSumThreads), fullest = (blocks + 255) / 256;
  return blocks >= 1024 || (tiled && blocks >= 512 && fullest * 256 * 8 <= blocks * 9) ? 2 : 1;
}

static unsigned sum_blocks(long long n_vec, int vpt) {
  // (the kernels' loops stride over the rest of a stash beyond 2^39 elements)
  const long long blocks = (n_vec + kSumThreads * vpt - 1) / (kSumThreads * vpt);
  return (unsigned)(blocks > 0x7fffffffLL ? 0x7fffffffLL : blocks);
}

template <bool BF16, bool OUTB>
static hipError_t launch_rows_t(const void* stash, long long seq_stride, long long n_vec, int n_seq, const float* c, float beta,
                                void* dW, hipStream_t s) {
  const int vpt = sum_vectors_per_thread(n_vec, n_seq, BF16, false);
  auto kern = vpt == 4   ? stash_weighted_sum_kernel<BF16, OUTB, 4>
              : vpt == 2 ? stash_weighted_sum_kernel<BF16, OUTB, 2>
                         : stash_weighted_sum_kernel<BF16, OUTB, 1>;
  hipLaunchKernelGGL(kern, dim3(sum_blocks(n_vec, vpt)), dim3(kSumThreads), 0, s, stash, seq_stride, n_vec, n_seq, c, beta, dW);
  return hipGetLastError();
}

hipError_t launch_stash_weighted_sum(const void* stash, bool bf16, long long seq_stride, long long n_elem, int n_seq,
                                     const float* c, float beta, void* dW, bool dw_bf16, hipStream_t s) {
  const long long n_vec = n_elem / (bf16 ? 8 : 4);
  if (n_vec <= 0) return hipSuccess;
  if (dw_bf16 && !bf16) return hipErrorInvalidValue;
  if (!bf16) return launch_rows_t<false, false>(stash, seq_stride, n_vec, n_seq, c, beta, dW, s);
  return dw_bf16 ? launch_rows_t<true, true>(stash, seq_stride, n_vec, n_seq, c, beta, dW, s)
                 : launch_rows_t<true, false>(stash, seq_stride, n_vec, n_seq, c, beta, dW, s);
}

template <int T, bool OUTB>
static hipError_t launch_tiled_t(const void* stash, long long D, long long n_vec, int n_seq, const float* c, float beta,
                                 void* dW, int d_in, hipStream_t s) {
  const int vpt = sum_vectors_per_thread(n_vec, n_seq, true, true);
  auto kern = vpt == 4   ? stash_weighted_sum_tiled_kernel<T, OUTB, 4>
              : vpt == 2 ? stash_weighted_sum_tiled_kernel<T, OUTB, 2>
                         : stash_weighted_sum_tiled_kernel<T, OUTB, 1>;
  hipLaunchKernelGGL(kern, dim3(sum_blocks(n_vec, vpt)), dim3(kSumThreads), 0, s, stash, D, n_vec, n_seq, c, beta, dW, d_in,
                     d_in / T);
  return hipGetLastError();
}

hipError_t launch_stash_weighted_sum_tiled(const void* stash, int tile, int d_out, int d_in, int n_seq, const float* c,
                                           float beta, void* dW, bool dw_bf16, hipStream_t s) {
  if ((tile != 256 && tile != 128) || d_out % tile || d_in % tile) return hipErrorInvalidValue;
  const long long D = (long long)d_out * d_in, n_vec = D / 8;
  if (n_vec <= 0) return hipSuccess;
  if (tile == 256)
    return dw_bf16 ? launch_tiled_t<256, true>(stash, D, n_vec, n_seq, c, beta, dW, d_in, s)
                   : launch_tiled_t<256, false>(stash, D, n_vec, n_seq, c, beta, dW, d_in, s);
  return dw_bf16 ? launch_tiled_t<128, true>(stash, D, n_vec, n_seq, c, beta, dW, d_in, s)
                 : launch_tiled_t<128, false>(stash, D, n_vec, n_seq, c, beta, dW, d_in, s);
}

}  // namespace isopo
