// Gram matrix of a stash, streaming variants (n_seq <= 128, bf16 and fp32, first; larger bf16 batches further down):
//     K_ij = sum_p S[i][p] * S[j][p]        (interacting listing:
//                                            ntk[i, j] = sum(seq_grads[i] * seq_grads[j]))
// One pass over the stash, bound by HBM.  The stash rows are 10^7..10^8 elements
// apart, so fragment-shaped loads (one row per lane) touch 32 cache lines per
// instruction and use 32 bytes of each.  Here the loads are row-contiguous
// instead: global_load_lds moves 16 bytes per lane straight into LDS, a wave
// covering whole 1 KiB / 512 B / 256 B runs of a row, into a ring of 32 KiB
// stages (all rows x KW elements).  Each wave then reads MFMA fragments for its
// share of the stage's 16-element steps with ds_read_b128 (16-byte column index
// XOR-swizzled with the row, so the row-per-lane reads do not pile on one bank)
// and issues mfma(a_i, a_j) for every row-block pair i <= j; the A and B
// fragments of K = S S^T are the same registers.  Up to 16 sequences the stage holds 16 rows and the products are
// 16x16: 32 rows would stage every byte twice (16 sequences of 1536x1536 in bf16, 75 MB: 17.8 us with 32 rows, 15.7 us
// with 16).  fp32 stashes take fp32 MFMAs, one per element of a lane's 16-byte vector; the accumulators are emptied into
// a second set of registers every few stages, so that no chain of matrix-core sums is longer than 64 (which of four
// waves multiplied 1/4096 or 1/1024 of the elements then does not show in K's error).  16 sequences of
// 1536x1536 in fp32, 151 MB: 31 us (4.9 TB/s; fragment-shaped loads by 1024 workgroups: 71 us); 40 of 300x1220, 59 MB: 22 us (40 us).
//
// Deterministic: fixed p -> workgroup -> wave assignment, waves added in order
// through LDS into the workgroup's partial slot, slots added in a fixed tree by
// the finishing kernel.
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace isopo {
namespace {

typedef unsigned short u16;
typedef void __attribute__((address_space(3)))* lds_void_ptr;
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef v4u __attribute__((address_space(3)))* lds_v4u_ptr;

constexpr int kBlocks = 256;           // persistent workgroups, one per CU
constexpr int kStageBytes = 32768;
constexpr int kStages = 4;

__host__ __device__ constexpr int tri(int nb) { return nb * (nb + 1) / 2; }
__host__ __device__ constexpr int pair_index(int bi, int bj, int nb) { return bi * nb - bi * (bi - 1) / 2 + (bj - bi); }

struct Params {
  const void* stash;
  long long seq_stride, p0, p1;
  int n_seq, first;
  float* partials;
  long long slot_floats;
  int32_t* clear;
};

// 16 bytes per lane, global -> LDS (lane l lands at lds_addr + 16*l).  Inline asm keeps the compiler's
// LDS-DMA tracking from waiting on every outstanding load before each LDS read.
__device__ __forceinline__ void load_lds16(const void* gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(gptr) : "memory");
}
// The same with the non-temporal cache policy, for the one-pass kernels (up to 256 sequences) on stashes that the last-level
// cache does not hold: every byte is read once, and keeping it out of the caches' replacement order is worth 13 % of the pass
// for up to 128 sequences (6.2 -> 7.05 TB/s on a 3.8 GB stash) and 3 % for 129..256 (72 GB stash).  The super-block
// pair kernel reads a row once per pair and keeps the default policy.
__device__ __forceinline__ void load_lds16_nt(const void* gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" : : "s"(lds_addr), "v"(gptr) : "memory");
}

// MB   side of an MFMA block, 32 or 16 (fp32, and n_seq <= 16)
// NB   MB-row blocks that carry sequences (pairs are formed among these)
// NBL  row blocks of the LDS layout: 1, 2, 4 or 8 (NBL >= NB); stage = MB*NBL rows x KW elements
// ONCE load with the non-temporal policy
template <bool BF16, int MB, int NB, int NBL, bool ONCE>
__global__ __launch_bounds__(256, 1) void stash_gram_stream_kernel(Params p) {
  static_assert(BF16 || MB == 16, "fp32 products are formed in 16x16 blocks");
  constexpr int ES = BF16 ? 2 : 4, EPV = 16 / ES;   // bytes per element, elements per 16-byte vector
  constexpr int ROWS = MB * NBL;
  constexpr int RB = kStageBytes / ROWS;            // bytes per row and stage: 2048 (MB 16), 1024, 512, 256
  constexpr int KW = RB / ES;                       // elements per row and stage
  constexpr int VPR = RB / 16;                      // 16-byte vectors per row: 128, 64, 32, 16
  constexpr int LPW = kStageBytes / 1024 / 4;       // wave-loads per wave and stage: 8
  constexpr int LV = 64 / MB;                       // vectors of a row that one step's lanes hold: 2 or 4
  constexpr int STEPS = VPR / LV / 4;               // steps per wave and stage: 8, 8, 4, 2
  constexpr int AV = MB * MB / 64;                  // accumulator registers per block: 16 or 4
  constexpr int FLUSH = BF16 ? 1 : 64 / (STEPS * EPV);   // fp32: stages per chain of 64 sums
  typedef typename std::conditional<MB == 32, f32x16, f32x4>::type acc_t;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned smem_base = (unsigned)(size_t)(lds_void_ptr)smem;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);

  if (p.clear && blockIdx.x == 0 && threadIdx.x == 0) *p.clear = 0;

  const long long n_elems = p.p1 - p.p0;
  const long long n_super = (n_elems + KW - 1) / KW;
  const long long my_first = blockIdx.x;
  const long long my_count = my_first < n_super ? (n_super - my_first + gridDim.x - 1) / gridDim.x : 0;

  // DMA addressing: wave-load q of this wave covers bytes (wave*LPW + q) * 1024 .. of the stage
  const char* src[LPW];
  int vec_off[LPW];
#pragma unroll
  for (int q = 0; q < LPW; ++q) {
    const int slot = (wave * LPW + q) * 64 + lane;
    const int row = slot / VPR, pos = slot % VPR;
    const int g = pos ^ (row & (VPR - 1) & 31);                 // global vector this LDS slot holds
    const int r = row < p.n_seq ? row : p.n_seq - 1;            // padded rows re-read a real row; their K entries are dropped
    src[q] = static_cast<const char*>(p.stash) + ((size_t)r * p.seq_stride + p.p0) * ES;
    vec_off[q] = g * 16;
  }
  auto issue = [&](long long k) {     // k-th super step of this workgroup -> ring stage k % kStages
    const long long u = my_first + k * gridDim.x;
    const long long e0 = u * KW;                                     // element offset of the stage within [p0, p1)
    const unsigned stage = smem_base + (unsigned)(k % kStages) * kStageBytes;
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      long long byte = e0 * ES + vec_off[q];
      const long long last = (n_elems - EPV) * ES;
      if (byte > last) byte = last;                               // tail: stays inside the row, zeroed at read time
      if (k >= my_count) byte = 0;                                // look-ahead past the end: harmless re-read
      if constexpr (ONCE) load_lds16_nt(src[q] + byte, stage + (unsigned)(wave_s * LPW + q) * 1024);
      else load_lds16(src[q] + byte, stage + (unsigned)(wave_s * LPW + q) * 1024);
    }
  };

  acc_t acc[tri(NB)], sum[BF16 ? 1 : tri(NB)];
#pragma unroll
  for (int q = 0; q < tri(NB); ++q)
#pragma unroll
    for (int v = 0; v < AV; ++v) {
      acc[q][v] = 0.f;
      if constexpr (!BF16) sum[q][v] = 0.f;
    }

  // fragment addressing: lane (row = lane % MB, quarter = lane / MB) of row block b, step s of this wave
  const int frow = lane % MB, part = lane / MB;

#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) issue(s);

  for (long long k = 0; k < my_count; ++k) {
    // this wave's part of stage k landed, then everyone's; the stage of step k-1 is free after the barrier
    __builtin_amdgcn_s_waitcnt(0x0f70 | (((kStages - 2) * LPW) & 15) | ((((kStages - 2) * LPW) >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    issue(k + kStages - 1);
    const unsigned sb = smem_base + (unsigned)(k % kStages) * kStageBytes;
    const long long u = my_first + k * gridDim.x;
    const long long valid = n_elems - u * KW;                    // elements of this stage inside [p0, p1)
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int vec = (wave * STEPS + s) * LV + part;            // 16-byte vector within the row
      v4u frag[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int row = b * MB + frow;
        const unsigned a = sb + (unsigned)row * RB + (unsigned)((vec ^ (row & (VPR - 1) & 31)) * 16);
        frag[b] = *(lds_v4u_ptr)(a);
        if (valid < KW && (long long)vec * EPV >= valid) frag[b] = v4u{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int e = 0; e < (BF16 ? 1 : 4); ++e)
#pragma unroll
        for (int bi = 0; bi < NB; ++bi)
#pragma unroll
          for (int bj = bi; bj < NB; ++bj) {
            acc_t& a = acc[pair_index(bi, bj, NB)];
            if constexpr (BF16 && MB == 32)
              a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, frag[bi]),
                                                          __builtin_bit_cast(bf16x8, frag[bj]), a, 0, 0, 0);
            else if constexpr (BF16)
              a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, frag[bi]),
                                                          __builtin_bit_cast(bf16x8, frag[bj]), a, 0, 0, 0);
            else
              a = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f32x4, frag[bi])[e],
                                                       __builtin_bit_cast(f32x4, frag[bj])[e], a, 0, 0, 0);
          }
    }
    if constexpr (!BF16) {
      if (k % FLUSH == FLUSH - 1) {
#pragma unroll
        for (int q = 0; q < tri(NB); ++q)
#pragma unroll
          for (int v = 0; v < AV; ++v) { sum[q][v] += acc[q][v]; acc[q][v] = 0.f; }
      }
    }
  }
  if constexpr (!BF16) {
#pragma unroll
    for (int q = 0; q < tri(NB); ++q)
#pragma unroll
      for (int v = 0; v < AV; ++v) acc[q][v] += sum[q][v];
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);      // drain the look-ahead loads before LDS is reused / released
  __builtin_amdgcn_s_barrier();

  // waves 0..3 added in order through LDS (reusing the ring); slot layout [pair][v][lane]
  float* red = reinterpret_cast<float*>(smem);
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int q = 0; q < tri(NB); ++q)
#pragma unroll
        for (int v = 0; v < AV; ++v) {
          float* o = red + (q * AV + v) * 64 + lane;
          *o = (w == 0 ? 0.f : *o) + acc[q][v];
        }
    }
    __syncthreads();
  }
  float* out = p.partials + (long long)blockIdx.x * p.slot_floats;
  for (int e = threadIdx.x; e < tri(NB) * AV * 64; e += 256) out[e] = (p.first ? 0.f : out[e]) + red[e];
}

template <bool BF16, int MB, int NB, int NBL, bool ONCE>
hipError_t launch(const Params& p, int blocks, hipStream_t s) {
  constexpr size_t smem = (size_t)kStages * kStageBytes;
  static_assert((size_t)tri(NB) * MB * MB * 4 <= smem, "reduction scratch fits the ring");
  auto kern = stash_gram_stream_kernel<BF16, MB, NB, NBL, ONCE>;
  // once per process (static initialisation is thread-safe); a failure is returned by every call
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), smem, s, p);
  return hipGetLastError();
}

// fp32: 16x16 blocks throughout.  The fp32 MFMA's rate is the same for either shape, and of 32x32 blocks more lies below
// the diagonal or past the last sequence (40 sequences: 6 of 16x16 against 3 of 32x32, half the MFMA cycles).
template <bool ONCE>
hipError_t launch_f32(const Params& p, int blocks, hipStream_t s) {
  switch ((p.n_seq + 15) / 16) {
    case 1: return launch<false, 16, 1, 1, ONCE>(p, blocks, s);
    case 2: return launch<false, 16, 2, 2, ONCE>(p, blocks, s);
    case 3: return launch<false, 16, 3, 4, ONCE>(p, blocks, s);
    case 4: return launch<false, 16, 4, 4, ONCE>(p, blocks, s);
    case 5: return launch<false, 16, 5, 8, ONCE>(p, blocks, s);
    case 6: return launch<false, 16, 6, 8, ONCE>(p, blocks, s);
    case 7: return launch<false, 16, 7, 8, ONCE>(p, blocks, s);
    default: return launch<false, 16, 8, 8, ONCE>(p, blocks, s);
  }
}

template <bool ONCE>
hipError_t launch_bf16(const Params& p, int blocks, hipStream_t s) {
  if (p.n_seq <= 16) return launch<true, 16, 1, 1, ONCE>(p, blocks, s);
  switch ((p.n_seq + 31) / 32) {
    case 1: return launch<true, 32, 1, 1, ONCE>(p, blocks, s);
    case 2: return launch<true, 32, 2, 2, ONCE>(p, blocks, s);
    case 3: return launch<true, 32, 3, 4, ONCE>(p, blocks, s);
    default: return launch<true, 32, 4, 4, ONCE>(p, blocks, s);
  }
}


// ---- more than 128 sequences --------------------------------------------------------------------
// K is cut into 128x128 super blocks; one launch row (blockIdx.y) per super-block pair (I <= J).  A
// workgroup streams the 128 (I == J) or 256 (I < J) rows of its pair through the same kind of LDS ring
// and wave w forms the four 32x32 blocks (4I + w, 4J + 0..3).  Off-diagonal pairs read both row groups,
// so the stash is read (number of super blocks + 1)/2 times on average; this path serves the large-batch
// stress shape, where the contraction dominates anyway.  Partials: [gridDim.x][nbp*nbp blocks][16][64].
struct LargeParams {
  const u16* stash;
  long long seq_stride, p0, p1;
  int n_seq, first, nsb, nbp;       // super blocks, padded 32-row blocks per side (4 * nsb)
  float* partials;
  long long slot_floats;
};

template <bool DIAG>
__global__ __launch_bounds__(256) void stash_gram_pair_kernel(LargeParams p) {
  constexpr int ROWS = DIAG ? 128 : 256;
  constexpr int RB = kStageBytes / ROWS;            // 256 or 128 bytes per row and stage
  constexpr int KW = RB / 2;
  constexpr int VPR = RB / 16;                       // 16 or 8
  constexpr int RPL = 1024 / RB;                     // 4 or 8 rows per wave-load
  constexpr int LPW = kStageBytes / 1024 / 4;        // 8
  constexpr int STEPS = KW / 16;                     // every wave walks all steps of a stage
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned smem_base = (unsigned)(size_t)(lds_void_ptr)smem;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);

  // blockIdx.y enumerates the pairs of its kind: DIAG -> I = J = y; else the y-th pair with I < J
  int I, J;
  if (DIAG) {
    I = J = blockIdx.y;
  } else {
    int rem = blockIdx.y;
    I = 0;
    while (rem >= p.nsb - 1 - I) { rem -= p.nsb - 1 - I; ++I; }
    J = I + 1 + rem;
  }

  const long long n_elems = p.p1 - p.p0;
  const long long n_super = (n_elems + KW - 1) / KW;
  const long long my_first = blockIdx.x;
  const long long my_count = my_first < n_super ? (n_super - my_first + gridDim.x - 1) / gridDim.x : 0;

  const char* src[LPW];
  int vec_off[LPW];
#pragma unroll
  for (int q = 0; q < LPW; ++q) {
    const int row = (wave * LPW + q) * RPL + lane / VPR;               // row of the stage
    const int pos = lane % VPR;
    const int g = pos ^ (row & (VPR - 1));
    int seq = (row < 128 ? I * 128 + row : J * 128 + (row - 128));
    if (seq >= p.n_seq) seq = p.n_seq - 1;                             // padded rows: entries never written
    src[q] = reinterpret_cast<const char*>(p.stash + (size_t)seq * p.seq_stride + p.p0);
    vec_off[q] = g * 16;
  }
  auto issue = [&](long long k) {
    const long long e0 = (my_first + k * gridDim.x) * KW;
    const unsigned stage = smem_base + (unsigned)(k % kStages) * kStageBytes;
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      long long byte = e0 * 2 + vec_off[q];
      const long long last = (n_elems - 8) * 2;
      if (byte > last) byte = last;
      if (k >= my_count) byte = 0;
      load_lds16(src[q] + byte, stage + (unsigned)(wave_s * LPW + q) * 1024);
    }
  };

  f32x16 acc[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
  const int frow = lane & 31, half = lane >> 5;

#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) issue(s);
  for (long long k = 0; k < my_count; ++k) {
    __builtin_amdgcn_s_waitcnt(0x0f70 | (((kStages - 2) * LPW) & 15) | ((((kStages - 2) * LPW) >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    issue(k + kStages - 1);
    const unsigned sb = smem_base + (unsigned)(k % kStages) * kStageBytes;
    const long long valid = n_elems - (my_first + k * gridDim.x) * KW;
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      const int vec = st * 2 + half;
      const bool dead = valid < KW && (long long)vec * 8 >= valid;
      const int ra = wave * 32 + frow;
      v4u fa = *(lds_v4u_ptr)(sb + (unsigned)ra * RB + (unsigned)((vec ^ (ra & (VPR - 1))) * 16));
      if (dead) fa = v4u{0u, 0u, 0u, 0u};
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int rb = (DIAG ? 0 : 128) + b * 32 + frow;
        v4u fb = *(lds_v4u_ptr)(sb + (unsigned)rb * RB + (unsigned)((vec ^ (rb & (VPR - 1))) * 16));
        if (dead) fb = v4u{0u, 0u, 0u, 0u};
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa), __builtin_bit_cast(bf16x8, fb),
                                                         acc[b], 0, 0, 0);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);

  float* out = p.partials + (long long)blockIdx.x * p.slot_floats;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int bi = 4 * I + wave, bj = 4 * J + b;
    float* o = out + ((long long)(bi * p.nbp + bj) * 16) * 64 + lane;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v * 64] = (p.first ? 0.f : o[v * 64]) + acc[b][v];
  }
}

// ---- 129..256 sequences in one pass ---------------------------------------------------------------
// A 128-element slice of all 256 rows is two 32 KiB half-stages (rows 0..127 and 128..255, 256 bytes
// per row: shorter runs per row stream noticeably slower from HBM).  LDS holds a ring of five
// half-stages: two are multiplied while three are in flight.  Eight waves share the loads and
// the products (four, nine products each: 1536x8960, 256 sequences 1250 us against 1225; 1000x2728, 255 258 / 244;
// 4096x1024, 160 330 / 314).  The 36 upper-triangle 32x32 blocks of the 8x8 block grid are dealt to them four or five each
// so that no wave needs more row blocks than it has products: it reads their fragments per 16-element step.
// Every wave walks every step.
// The fragments of step s + 1 are read between the MFMAs of step s (two register sets), so no MFMA
// waits for the LDS.  A slice that is not whole (only the last one of [p0, p1) can be) takes a plain
// masking loop after the main one.  The stash is read exactly once; partials have the large path's layout.
constexpr int kWideHalves = 5;
constexpr int kWideWaves = 8;
struct WideBlocks {
  int n, bi[5], bj[5];                               // a wave's blocks
  constexpr bool reads(int b) const {
    for (int q = 0; q < n; ++q)
      if (bi[q] == b || bj[q] == b) return true;
    return false;
  }
  constexpr int rows() const {
    int r = 0;
    for (int b = 0; b < 8; ++b) r += reads(b) ? 1 : 0;
    return r;
  }
};
constexpr WideBlocks kWide[kWideWaves] = {
    {4, {0, 0, 0, 0, 0}, {0, 1, 2, 3, 0}}, {5, {0, 0, 0, 0, 7}, {4, 5, 6, 7, 7}},
    {4, {1, 1, 1, 1, 0}, {1, 2, 3, 4, 0}}, {5, {1, 1, 1, 6, 6}, {5, 6, 7, 6, 7}},
    {4, {2, 2, 2, 2, 0}, {2, 3, 4, 5, 0}}, {5, {2, 2, 5, 5, 5}, {6, 7, 5, 6, 7}},
    {5, {3, 3, 3, 3, 3}, {3, 4, 5, 6, 7}}, {4, {4, 4, 4, 4, 0}, {4, 5, 6, 7, 0}}};
constexpr bool wide_blocks_once() {
  for (int i = 0; i < 8; ++i)
    for (int j = i; j < 8; ++j) {
      int seen = 0;
      for (const WideBlocks& w : kWide)
        for (int q = 0; q < w.n; ++q) seen += w.bi[q] == i && w.bj[q] == j ? 1 : 0;
      if (seen != 1) return false;
    }
  return true;
}
static_assert(wide_blocks_once(), "every block on or above the diagonal has one wave");
// Row blocks that hold no sequence are neither loaded nor multiplied: a slice of 256 rows takes as long whether they are read
// from memory or are all the last one again.  4096x1024, 160 sequences 314 -> 243 us; 512x3072, 130 127 -> 104; 2048x4096, 192
// 726 -> 593 (with four waves before); 2048x3072, 224 582 -> 511.
constexpr WideBlocks wide_blocks(int wave, int row_blocks) {
  WideBlocks w{0, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}};
  for (int q = 0; q < kWide[wave].n; ++q)
    if (kWide[wave].bj[q] < row_blocks) {
      w.bi[w.n] = kWide[wave].bi[q];
      w.bj[w.n] = kWide[wave].bj[q];
      ++w.n;
    }
  return w;
}

template <int W, int RBLOCKS, bool ONCE>
__device__ __forceinline__ void wide_body(const LargeParams& p, unsigned smem_base, int lane, int wave_s,
                                          const char* const (&src)[2][4], const int (&vec_off)[4],
                                          long long n_elems, long long my_first, long long my_count) {
  constexpr int RB = 256, KW = 128, VPR = 16, LPW = 32 / kWideWaves, STEPS = 8;
  constexpr WideBlocks mine = wide_blocks(W, RBLOCKS);
  constexpr int NB = mine.n, ROWS = mine.rows();
  constexpr bool LOADS1 = 4 + W / 2 < RBLOCKS;       // a wave's loads of the second half are of half a row block
  auto issue = [&](long long j) {                    // half-stage j = 2 * slice + half
    const long long e0 = (my_first + (j >> 1)) * KW;
    const unsigned stage = smem_base + (unsigned)(j % kWideHalves) * kStageBytes;
    const int h = (int)(j & 1);
    if (h && !LOADS1) return;                        // the waits below count the first half's loads only
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      long long byte = e0 * 2 + vec_off[q];
      const long long last = (n_elems - 8) * 2;
      if (byte > last) byte = last;
      if ((j >> 1) >= my_count) byte = 0;
      const char* const from = (h ? src[1][q] : src[0][q]) + byte;
      if constexpr (ONCE) load_lds16_nt(from, stage + (unsigned)(wave_s * LPW + q) * 1024);
      else load_lds16(from, stage + (unsigned)(wave_s * LPW + q) * 1024);
    }
  };
  f32x16 acc[NB > 0 ? NB : 1];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
  const int frow = lane & 31, half = lane >> 5;
  // the products of one 16-element step
  auto multiply = [&](const v4u (&frag)[8]) {
#pragma unroll
    for (int q = 0; q < NB; ++q)
      acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, frag[mine.bi[q]]),
                                                       __builtin_bit_cast(bf16x8, frag[mine.bj[q]]), acc[q], 0, 0, 0);
  };
  auto read_step = [&](v4u (&frag)[8], unsigned sb0, unsigned sb1, int st) {
    const int vec = st * 2 + half;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (!mine.reads(b)) continue;
      const int row = (b & 3) * 32 + frow;
      frag[b] = *(lds_v4u_ptr)((b < 4 ? sb0 : sb1) + (unsigned)row * RB + (unsigned)((vec ^ (row & (VPR - 1))) * 16));
    }
  };

  // Only the very last slice of [p0, p1) can be short; it goes through the masking loop below.
  const bool short_tail = (n_elems % KW) != 0 && my_first + my_count == (n_elems + KW - 1) / KW;
  const long long n_whole = my_count - (short_tail ? 1 : 0);

  issue(0); issue(1); issue(2);
  for (long long k = 0; k < n_whole; ++k) {
    // half-stages 2k and 2k+1 landed (only 2k+2 may still be out), then everyone's; the two half-stages of
    // slice k-1 are free after the barrier and take 2k+3 and 2k+4
    __builtin_amdgcn_s_waitcnt(0x0f70 | LPW);
    __builtin_amdgcn_s_barrier();
    issue(2 * k + 3);
    issue(2 * k + 4);
    const unsigned sb0 = smem_base + (unsigned)((2 * k) % kWideHalves) * kStageBytes;
    const unsigned sb1 = smem_base + (unsigned)((2 * k + 1) % kWideHalves) * kStageBytes;
    // Two fragment sets: the reads of step st + 1 go out between the MFMAs of step st, one read behind each
    // of the first MFMAs, so that no MFMA waits for the LDS and the four waves' reads are spread out.
    v4u frag[2][8];
    read_step(frag[0], sb0, sb1, 0);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st + 1 < STEPS) read_step(frag[(st + 1) & 1], sb0, sb1, st + 1);
      multiply(frag[st & 1]);
      if (st == 0) __builtin_amdgcn_sched_group_barrier(0x100, ROWS, 0);        // step 0's own reads first
      if (st + 1 < STEPS) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          if (r < NB) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NB > ROWS ? NB - ROWS : 0, 0);
      } else {
        __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
      }
    }
  }
  if (short_tail) {
    const long long k = n_whole;
    __builtin_amdgcn_s_waitcnt(0x0f70 | LPW);
    __builtin_amdgcn_s_barrier();
    issue(2 * k + 3);
    issue(2 * k + 4);
    const unsigned sb0 = smem_base + (unsigned)((2 * k) % kWideHalves) * kStageBytes;
    const unsigned sb1 = smem_base + (unsigned)((2 * k + 1) % kWideHalves) * kStageBytes;
    const long long valid = n_elems - (my_first + k) * KW;
#pragma unroll 1
    for (int st = 0; st < STEPS; ++st) {
      const int vec = st * 2 + half;
      const bool dead = (long long)vec * 8 >= valid;
      v4u frag[8];
      read_step(frag, sb0, sb1, st);
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (mine.reads(b) && dead) frag[b] = v4u{0u, 0u, 0u, 0u};
      multiply(frag);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);

  float* out = p.partials + (long long)blockIdx.x * p.slot_floats;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    float* o = out + ((long long)(mine.bi[q] * 8 + mine.bj[q]) * 16) * 64 + lane;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v * 64] = (p.first ? 0.f : o[v * 64]) + acc[q][v];
  }
}

template <int RBLOCKS, bool ONCE>
__global__ __launch_bounds__(64 * kWideWaves) void stash_gram_wide_kernel(LargeParams p) {
  constexpr int KW = 128, VPR = 16, RPL = 4, LPW = 32 / kWideWaves;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned smem_base = (unsigned)(size_t)(lds_void_ptr)smem;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const long long n_elems = p.p1 - p.p0;
  const long long n_super = (n_elems + KW - 1) / KW;
  // a contiguous run of slices per workgroup: each of its 256 row streams walks consecutive cache lines
  const long long my_first = n_super * blockIdx.x / gridDim.x;
  const long long my_count = n_super * (blockIdx.x + 1) / gridDim.x - my_first;
  const char* src[2][LPW];
  int vec_off[LPW];
#pragma unroll
  for (int q = 0; q < LPW; ++q) {
    const int row = (wave * LPW + q) * RPL + lane / VPR;                // row within a half-stage, 0..127
    const int pos = lane % VPR;
    vec_off[q] = (pos ^ (row & (VPR - 1))) * 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = h * 128 + row;
      const int seq = r < p.n_seq ? r : p.n_seq - 1;                    // padded rows: entries never written
      src[h][q] = reinterpret_cast<const char*>(p.stash + (size_t)seq * p.seq_stride + p.p0);
    }
  }
  // every wave runs the same loop (same barriers), specialised on its block rows
  switch (wave_s) {
    case 0: wide_body<0, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    case 1: wide_body<1, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    case 2: wide_body<2, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    case 3: wide_body<3, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    case 4: wide_body<4, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    case 5: wide_body<5, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    case 6: wide_body<6, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
    default: wide_body<7, RBLOCKS, ONCE>(p, smem_base, lane, wave_s, src, vec_off, n_elems, my_first, my_count); break;
  }
}

// grid: one 1024-thread block per (block bi <= bj, v); 16 waves add the slots, then wave order.
__global__ __launch_bounds__(1024) void stash_gram_large_finish_kernel(const float* __restrict__ partials, int n_slots,
                                                                       long long slot_floats, int n_seq, int nbp,
                                                                       float* __restrict__ K) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int blk = blockIdx.x >> 4, v = blockIdx.x & 15;
  const int bi = blk / nbp, bj = blk % nbp;
  if (bi > bj || bi * 32 >= n_seq || bj * 32 >= n_seq) return;
  const long long e = ((long long)blk * 16 + v) * 64 + lane;
  float s = 0.f;
#pragma unroll 8
  for (int w = wave; w < n_slots; w += 16) s += partials[(long long)w * slot_floats + e];
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0) return;
  s = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) s += red[w][lane];
  const int i = bi * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), j = bj * 32 + (lane & 31);
  if (i < n_seq && j < n_seq && i <= j) {
    K[(size_t)i * n_seq + j] = s;
    K[(size_t)j * n_seq + i] = s;
  }
}

template <int RBLOCKS, bool ONCE>
hipError_t launch_wide_t(const LargeParams& p, int gx, hipStream_t s) {
  constexpr size_t smem = (size_t)kWideHalves * kStageBytes;          // 160 KiB: the whole LDS of a CU
  // once per process (static initialisation is thread-safe); a failure is returned by every call
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(stash_gram_wide_kernel<RBLOCKS, ONCE>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((stash_gram_wide_kernel<RBLOCKS, ONCE>), dim3(gx), dim3(64 * kWideWaves), smem, s, p);
  return hipGetLastError();
}
template <int RBLOCKS>
hipError_t launch_wide(const LargeParams& p, int gx, bool once, hipStream_t s) {
  return once ? launch_wide_t<RBLOCKS, true>(p, gx, s) : launch_wide_t<RBLOCKS, false>(p, gx, s);
}

// What the last-level cache holds (256 MiB) is left in it for the weighted sum that follows, and is there from the contraction
// before; larger stashes are read non-temporally.  Whole calls, non-temporal / default: 1000x2728 bf16, 24 sequences (131 MB) 136.6
// / 130.7 us, 40 (218 MB) 160.9 / 150.0, 80 (436 MB) 305.8 / 324.2; 4096x1024 bf16, 32 (268 MB) 181.0 / 179.4, 48 (403 MB) 271.4 /
// 275.4; of 39 random stashes of 16 to 250 MB 0.86 .. 1.00 with the default.  129 to 256 sequences: 824x72, 199 (24 MB) 58.9 / 52.4;
// 640x1208, 135 (209 MB) 130.9 / 122.9; 1600x408, 204 (266 MB) 262.8 / 263.1; 416x2152, 219 (392 MB) 232.1 / 247.6; 368x5200, 132
// (505 MB) 288 / 322.
bool read_once(long long elems, int n_seq, bool bf16) { return elems * n_seq * (bf16 ? 2 : 4) > 256LL << 20; }

template <bool DIAG>
hipError_t launch_pair(const LargeParams& p, int gx, int n_pairs, hipStream_t s) {
  if (n_pairs <= 0) return hipSuccess;
  constexpr size_t smem = (size_t)kStages * kStageBytes;
  auto kern = stash_gram_pair_kernel<DIAG>;
  // once per process (static initialisation is thread-safe); a failure is returned by every call
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(gx, n_pairs), dim3(256), smem, s, p);
  return hipGetLastError();
}

}  // namespace

// One workgroup per compute unit, fewer where the stash has fewer stages than that: a short stash's finish pass then
// adds only slots that hold something.
int stash_gram_stream_slots(int n_seq, bool bf16, long long n_elem) {
  const int rows = n_seq <= 16 ? 16 : (n_seq <= 32 ? 32 : (n_seq <= 64 ? 64 : 128));
  const long long kw = kStageBytes / rows / (bf16 ? 2 : 4), stages = (n_elem + kw - 1) / kw;
  return stages < kBlocks ? (int)(stages > 0 ? stages : 1) : kBlocks;
}

// Large batches (n_seq > 128).
int stash_gram_large_slots(int n_seq) {
  if (n_seq <= 256) return kBlocks;          // one-pass kernel: one persistent workgroup per CU
  const int nsb = (n_seq + 127) / 128;
  const int pairs = nsb * (nsb + 1) / 2;
  int gx = 512 / pairs;
  return gx < 16 ? 16 : (gx > 128 ? 128 : gx);
}
size_t stash_gram_large_slot_floats(int n_seq) {
  const int nbp = 4 * ((n_seq + 127) / 128);
  return (size_t)nbp * nbp * 1024;
}
hipError_t launch_stash_gram_large(const StashGramArgs& a, hipStream_t s) {
  if (!a.bf16 || a.n_seq <= 128) return hipErrorInvalidValue;
  LargeParams p;
  p.stash = static_cast<const u16*>(a.stash); p.seq_stride = a.seq_stride; p.p0 = a.p0; p.p1 = a.p1;
  p.n_seq = a.n_seq; p.first = a.first ? 1 : 0; p.partials = a.partials;
  p.nsb = (a.n_seq + 127) / 128; p.nbp = 4 * p.nsb;
  p.slot_floats = (long long)stash_gram_large_slot_floats(a.n_seq);
  const int gx = stash_gram_large_slots(a.n_seq);
  const bool once = read_once(a.p1 - a.p0, a.n_seq, true);
  if (a.n_seq <= 160) return launch_wide<5>(p, gx, once, s);
  if (a.n_seq <= 192) return launch_wide<6>(p, gx, once, s);
  if (a.n_seq <= 224) return launch_wide<7>(p, gx, once, s);
  if (a.n_seq <= 256) return launch_wide<8>(p, gx, once, s);
  hipError_t e = launch_pair<true>(p, gx, p.nsb, s);
  if (e != hipSuccess) return e;
  return launch_pair<false>(p, gx, p.nsb * (p.nsb - 1) / 2, s);
}
hipError_t launch_stash_gram_large_finish(const float* partials, int n_seq, float* K, hipStream_t s) {
  const int nbp = 4 * ((n_seq + 127) / 128);
  hipLaunchKernelGGL(stash_gram_large_finish_kernel, dim3((unsigned)(nbp * nbp * 16)), dim3(1024), 0, s, partials,
                     stash_gram_large_slots(n_seq), (long long)stash_gram_large_slot_floats(n_seq), n_seq, nbp, K);
  return hipGetLastError();
}

hipError_t launch_stash_gram_stream(const StashGramArgs& a, hipStream_t s) {
  if (a.n_seq < 1 || a.n_seq > 128) return hipErrorInvalidValue;
  Params p;
  p.stash = a.stash; p.seq_stride = a.seq_stride; p.p0 = a.p0; p.p1 = a.p1;
  p.n_seq = a.n_seq; p.first = a.first ? 1 : 0; p.partials = a.partials; p.clear = a.clear;
  p.slot_floats = (long long)stash_gram_slot_floats(a.n_seq, a.bf16);
  const bool once = read_once(a.p1 - a.p0, a.n_seq, a.bf16);
  if (a.bf16) return once ? launch_bf16<true>(p, a.slots, s) : launch_bf16<false>(p, a.slots, s);
  return once ? launch_f32<true>(p, a.slots, s) : launch_f32<false>(p, a.slots, s);
}

}  // namespace isopo
