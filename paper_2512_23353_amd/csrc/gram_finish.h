// The Gram matrix of up to 128 sequences from the partial slots of stash_gram_stream.hip: used by the finish kernel
// (stash_gram.hip) and by the one that goes on to the coefficients (transform.hip).
#pragma once

#include "common.h"

namespace isopo {

struct GramFinish {
  const float* partials;                 // [slots][slot_floats]
  int slots;
  long long slot_floats;
  int n_seq, mb;                         // mb: side of a block
  float* K;
};

constexpr int kFinishThreads = 1024;

// What one workgroup of a launch writes and another reads: past the L2s, which the accelerator dies do not share (sc1).
template <bool SHARED>
__device__ __forceinline__ void put_shared(float* p, float v) {
  if constexpr (SHARED) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); else *p = v;
}
template <bool SHARED>
__device__ __forceinline__ float get_shared(const float* p) {
  if constexpr (SHARED) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); else return *p;
}

// One 1024-thread block per 64 consecutive slot elements: wave w adds slots w, w+16, ... in order (eight loads in flight:
// a load per turn of the loop cost 0.4 us each), the 16 waves are added in wave order, in 64 bits; only entries with
// i <= j are written, mirrored, by wave 0.  256 slots of 32 sequences: 6.5 us before, 4.9 us now;
// an fp32 stash's 1024 slots: 20.7 us before, its 256 slots 5.0 us, 2.3 us where it has 16 stages.
template <bool SHARED>
__device__ __forceinline__ void gram_finish(const GramFinish& f) {
  __shared__ double red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long e = (long long)blockIdx.x * 64 + lane;      // element of the slot layout [pair][v][lane]
  double s = 0.0;
#pragma unroll 8
  for (int w = wave; w < f.slots; w += 16) s += (double)f.partials[(long long)w * f.slot_floats + e];
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0) return;
  s = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) s += red[w][lane];
  // blocks of mb x mb above the diagonal, row by row, each [v][lane] as the MFMA's accumulators hold it
  const int mb = f.mb, per = mb * mb, nb = (f.n_seq + mb - 1) / mb;
  const int v = (int)(e % per) >> 6;
  int bi = 0, rem = (int)(e / per);
  while (rem >= nb - bi) { rem -= nb - bi; ++bi; }
  const int i = bi * mb + (mb == 16 ? 4 * (lane >> 4) + v : 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3));
  const int j = (bi + rem) * mb + lane % mb;
  if (i < f.n_seq && j < f.n_seq && i <= j) {
    put_shared<SHARED>(f.K + (size_t)i * f.n_seq + j, (float)s);
    put_shared<SHARED>(f.K + (size_t)j * f.n_seq + i, (float)s);
  }
}

}  // namespace isopo
