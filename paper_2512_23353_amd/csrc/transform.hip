// Per-sequence coefficients from the layer's Gram matrix K and the advantages A.
//
//   FISHER       c_i = A_i / sqrt(||g_i||_F^2 + reg),  ||g_i||_F^2 = (1/m) sum_j K_ij^2
//                (non-interacting update u_l, with the Fisher norm of eq.
//                F-norm-basic taken over the batch's reduced gradients, j = i
//                included)
//   INTERACTING  c = (K + reg I)^-1 A          (v = J^T (K + cI)^-1 A)
//
// reg = lambda, or lambda times this batch's typical value of the quantity reg is
// added to, or lambda times the trailing mean over minibatches of that value.  For
// INTERACTING the value is tr(K)/m (the interacting experiment's regulariser,
// factor * E[mean(D)]: the mean eigenvalue is the trace over m, so no
// decomposition is needed for it); for FISHER it is mean_i ||g_i||_F^2 (the
// non-interacting derivation compares reg_l with the typical ||.||_F^2).
// The m x m problem is tiny next to the contractions around it, so one
// workgroup per problem works in fp64: a
// right-looking Cholesky factorisation in panels and two triangular solves.  The
// matrix lives in LDS (m <= 128) or in a caller-provided global scratch (larger
// m); the panel being factored is in LDS, column-major, and one wave factors its
// first 64 rows in registers (no barrier per column); A rides along as one more
// row of the matrix, which makes the forward solve part of the factorisation, and
// the backward solve runs panel by panel as well.  The result is the unique
// solution; the eigendecomposition the interacting listing uses reaches the same
// vector.  A non-positive pivot is reported, never clamped.
#include "common.h"
#include "kernels.h"

namespace isopo {
namespace {

constexpr int ISOPO_MAX_SEQ_TRANSFORM = 1024;     // the header's ISOPO_MAX_SEQ

template <int kThreads>
__device__ double block_sum(double x, double* red /* [kThreads/64] */) {
  x = wave_sum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) s += red[w];
  return s;
}

// The value lane `src` (the same for all lanes) holds.
__device__ __forceinline__ double lane_value(double x, int src) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), src);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), src);
  return __hiloint2double(hi, lo);
}

// x, as a value that the compiler knows nothing about: comparisons with it are made where they stand.  (Hoisted out of the
// panels' loop, a mask for each of 32 columns fills the scalar registers several times over.)
template <class T>
__device__ __forceinline__ T fresh(T x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Panel rows in LDS: one padding element after every 32 rows of a column, so that the trailing update's
// lanes, which read groups of four consecutive rows 32 bytes apart, spread over all banks.
__device__ __forceinline__ int panel_pos(int lr) { return lr + (lr >> 5); }
__host__ __device__ constexpr int panel_stride(int m) { return ((m + 1) + ((m + 1) >> 5) + 1 + 3) & ~3; }

// Doubles ahead of the matrix and the panel in LDS: the pivots' inverse roots and a copy of the panel's diagonal block.
__host__ __device__ constexpr int transform_panel(int m) { return m > kTransformLdsMax && m <= kTransformWidePanelMax ? 32 : 16; }
__host__ __device__ constexpr int transform_front(int m) { return m + transform_panel(m) * (transform_panel(m) + 1); }

// (K + reg I) c = A: M [m + 1, m] fp64 in LDS or global memory (row m holds A, then y), the panel of NB columns
// in LDS as PT[column][row - k0] with row stride RS.  c is left in cs.
//
// Panel step: every wave holds the NB rows of the panel's diagonal block and 64 - NB rows below it, one per lane, in
// registers, and factors the NB columns by itself (the diagonal block again in every wave): the pivot and a column's entries
// of the diagonal block's rows come from their lanes (v_readlane), so that a column is one reciprocal square root and a
// chain of multiply-adds, without an LDS round trip or a barrier (one of each per column, and a 64-bit division and
// square root in every thread, made a column 0.8 us).  Sequences, us before and now: 16, 11.4 and 7.8; 32, 23 and 13; 64, 49 and
// 25; 128, 112 and 57; 256, 328 and 186 (230 to 270 right after the Gram pass of a stash of many GB); 1024, 8980 and 5080 (of which
// launch and regulariser 6).  With the matrix in global memory the kernel spills 10 scalar registers, and at 1024 threads, whose
// cap is 128 vector registers, 8 and 16 vector ones.  The upper triangle of the diagonal block is carried along and never read.
// The trailing matrix (rows up to and including the row of A) then takes the rank-NB update in
// 16 x 16 blocks, a wave each, on the matrix cores, whose factors come from the panel in LDS: a lane reads two values for
// sixteen multiply-adds of its own (register blocks of 4 x 4, a lane each, read eight and were bound by the LDS: 256 sequences
// 225 us, 130 98 against 73).
template <int kThreads, int NB>
__device__ bool cholesky_solve(const float* __restrict__ K, const float* __restrict__ A, int m, double reg,
                               double* __restrict__ M, double* cs /* LDS [m] */, double* inv_diag /* LDS [m] */,
                               double* PT /* LDS */, int* fail /* LDS */, int* fail_col) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int RS = panel_stride(m);
  double* const diag = inv_diag + m;                     // [NB][NB + 1]
  // the whole square, so that every later read is of a defined value; the upper triangle never enters a result
  // (a wave per row, four rows of loads in flight)
  for (int q = lane; q < m; q += kWave) {
#pragma unroll 4
    for (int r = tid / kWave; r < m; r += kThreads / kWave)
      M[(size_t)r * m + q] = (double)K[(size_t)r * m + q] + (r == q ? reg : 0.0);
  }
  for (int i = tid; i < m; i += kThreads) M[(size_t)m * m + i] = (double)A[i];
  if (tid == 0) *fail = -1;
  __syncthreads();

  for (int k0 = 0; k0 < m; k0 += NB) {
    const int nbk = m - k0 < NB ? m - k0 : NB;
    const int nrows = m + 1 - k0;                        // rows k0 .. m
    // panel -> LDS (a wave reads NB-element pieces of rows), its diagonal block a second time
#pragma unroll 4
    for (int e = tid; e < nrows * NB; e += kThreads) {
      const int lr = e / NB, kk = e % NB;
      if (kk < nbk) {
        const double x = M[(size_t)(k0 + lr) * m + k0 + kk];
        PT[kk * RS + panel_pos(lr)] = x;
        if (lr < NB) diag[kk * (NB + 1) + lr] = x;
      }
    }
    __syncthreads();
    // lanes < NB: the diagonal block's rows, the others NB + base + lane - NB.  Rows and columns from nbk on are the
    // identity's, so that the columns are one straight run of code; what the row of A makes of them is never read.  A pivot
    // that is not positive leaves NaN or infinity in all that follows; the first one is found at the end.
    constexpr int kRowsPerWave = kWave - NB, kRowsPerPass = kRowsPerWave * (kThreads / kWave);
    for (int base = (tid / kWave) * kRowsPerWave; base == 0 || base < nrows - NB; base += kRowsPerPass) {
      const int lr = lane < NB ? lane : base + lane;
      const bool has = lr < nrows;
      double row[NB], pivot = 1.0, inv = 0.0;
      // (read whether wanted or not: a branch per entry costs more, and what its masks take of the scalar registers)
      const double* const from = lane < NB ? diag + lane : PT + panel_pos(has ? lr : 0);
      const int pitch = lane < NB ? NB + 1 : RS, wanted = has ? nbk : 0;
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const double x = from[q * pitch];
        row[q] = q < fresh(wanted) ? x : (fresh(lane) == q ? 1.0 : 0.0);
      }
#pragma unroll
      for (int kk = 0; kk < NB; ++kk) {
        if (fresh(lane) == kk) { pivot = row[kk]; inv = rsqrt(row[kk]); }
        row[kk] *= lane_value(inv, kk);                  // the entry of L; the pivot's own lane: d / sqrt(d)
#pragma unroll
        for (int q0 = kk + 1; q0 < NB; q0 += 8) {
          // eight entries at a time: more, fetched ahead, would not fit the scalar registers
          const double x = fresh(row[kk]);
#pragma unroll
          for (int q = q0; q < q0 + 8 && q < NB; ++q) row[q] = fresh(row[q] - row[kk] * lane_value(x, q));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (has && (lane >= NB || base == 0)) {
#pragma unroll
        for (int q = 0; q < NB; ++q) PT[q * RS + panel_pos(lr)] = row[q];      // columns from nbk on: read by nobody
      }
      if (base == 0) {
        if (lane < nbk) inv_diag[k0 + lane] = inv;
        const unsigned long long bad = __ballot(lane < nbk && !(pivot > 0.0));
        if (bad && lane == 0) *fail = k0 + __ffsll((long long)bad) - 1;
      }
    }
    __syncthreads();
    if (*fail >= 0) { *fail_col = *fail; return false; }           // every thread reads the same value
    for (int e = tid; e < nrows * NB; e += kThreads) {
      const int lr = e / NB, kk = e % NB;
      if (kk < nbk) M[(size_t)(k0 + lr) * m + k0 + kk] = PT[kk * RS + panel_pos(lr)];
    }
    // trailing update: rows t0 .. m (the row of A included), columns t0 .. min(row, m - 1), in 16x16 blocks on and below the
    // diagonal, row by row (nbr is nbq, or nbq + 1 where the row of A opens a block row).  Lane l supplies row l % 16, column
    // l / 16 of a step of the left factor and the same of the right one, and holds rows 4 q + l / 16 of column l % 16.
    const int t0 = k0 + nbk;
    const int nbr = (m + 1 - t0 + 15) / 16, nbq = (m - t0 + 15) / 16;
    const int below = nbq * (nbq + 1) / 2, blocks = below + (nbr - nbq) * nbq;
    const int l16 = lane & 15, l4 = lane >> 4;
    constexpr int kWaves = kThreads / kWave;
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    f64x4 next = {0.0, 0.0, 0.0, 0.0};
    int next_r0 = t0, next_q0 = t0;
    // a block's entries, fetched while the one before is multiplied
    auto fetch = [&](int e) {
      if (e >= blocks) return;
      int br, bq;
      if (e < below) {
        br = (int)((sqrtf(8.f * (float)e + 1.f) - 1.f) * 0.5f);
        if (br * (br + 1) / 2 > e) --br;
        if ((br + 1) * (br + 2) / 2 <= e) ++br;
        bq = e - br * (br + 1) / 2;
      } else {
        br = nbq;
        bq = e - below;
      }
      next_r0 = t0 + 16 * br;
      next_q0 = t0 + 16 * bq;
      const int q = next_q0 + l16 < m ? next_q0 + l16 : m - 1;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = next_r0 + 4 * v + l4;
        next[v] = M[(size_t)(r <= m ? r : m) * m + q];
      }
    };
    const int first_block = __builtin_amdgcn_readfirstlane(tid / kWave);
    fetch(first_block);
    for (int e = first_block; e < blocks; e += kWaves) {
      f64x4 cur = next;
      const int r0 = next_r0, q0 = next_q0;
      fetch(e + kWaves);
      const int lr = panel_pos((r0 + l16 <= m ? r0 + l16 : m) - k0), lq = panel_pos((q0 + l16 < m ? q0 + l16 : m - 1) - k0);
      double a[NB / 4], b[NB / 4];
#pragma unroll
      for (int step = 0; step < NB / 4; ++step) {
        const int kk = 4 * step + l4;
        const bool live = kk < nbk;                       // of a last panel, which has only the row of A below it
        a[step] = live ? -PT[(live ? kk : 0) * RS + lr] : 0.0;
        b[step] = live ? PT[(live ? kk : 0) * RS + lq] : 0.0;
      }
#pragma unroll
      for (int step = 0; step < NB / 4; ++step) cur = __builtin_amdgcn_mfma_f64_16x16x4f64(a[step], b[step], cur, 0, 0, 0);
      const int q = q0 + l16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + 4 * v + l4;
        if (r <= m && q < m && q <= r) M[(size_t)r * m + q] = cur[v];
      }
    }
    __syncthreads();
  }

  // backward: L^T c = y (y is row m of M), last panel first.  The sums over the rows below a panel are split
  // over kThreads / NB row groups and met in LDS; wave 0 then solves the panel's triangle, lane = column, with the
  // triangle's rows in registers.
  constexpr int RG = kThreads / NB;
  double* red = PT;                                       // [RG][NB + 1]
  double* tri = PT + RG * (NB + 1);                       // [NB][NB + 1]: the panel's diagonal block of L
  const int kk = tid % NB, rg = tid / NB;
  for (int k0 = ((m - 1) / NB) * NB; k0 >= 0; k0 -= NB) {
    const int nbk = m - k0 < NB ? m - k0 : NB;
    const int t0 = k0 + nbk;
    double acc = 0.0;
    if (kk < nbk)
#pragma unroll 4
      for (int r = t0 + rg; r < m; r += RG) acc += M[(size_t)r * m + k0 + kk] * cs[r];
    red[rg * (NB + 1) + kk] = acc;
    for (int e = tid; e < NB * NB; e += kThreads) {
      const int r = e / NB, q = e % NB;
      tri[r * (NB + 1) + q] = r < nbk && q < r ? M[(size_t)(k0 + r) * m + k0 + q] : 0.0;
    }
    __syncthreads();
    if (tid < kWave) {
      const bool has = lane < nbk;
      double t[NB], v = 0.0;
#pragma unroll
      for (int j = 0; j < NB; ++j) t[j] = tri[j * (NB + 1) + (lane < NB ? lane : 0)];
      if (has) {
        double sum = 0.0;
#pragma unroll 8
        for (int g = 0; g < RG; ++g) sum += red[g * (NB + 1) + lane];
        v = M[(size_t)m * m + k0 + lane] - sum;
      }
      const double inv = has ? inv_diag[k0 + lane] : 0.0;
#pragma unroll
      for (int j = NB - 1; j >= 0; --j) v -= t[j] * lane_value(v * inv, j);     // rows from nbk on: zeros
      if (has) cs[k0 + lane] = v * inv;
    }
    __syncthreads();
  }
  return true;
}

template <int kThreads, bool GLOBAL>
__global__ __launch_bounds__(kThreads) void transform_kernel(const float* __restrict__ Kb, const float* __restrict__ Ab,
                                                             int m, int variant, int reg_mode, float lambda,
                                                             float* __restrict__ cb, int32_t* __restrict__ info,
                                                             double* __restrict__ gws, float* __restrict__ ema_state,
                                                             float ema_decay) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ double red[kThreads / 64];
  const int prob = blockIdx.x, tid = threadIdx.x;
  const float* K = Kb + (size_t)prob * m * m;
  const float* A = Ab + (size_t)prob * m;
  float* c = cb + (size_t)prob * m;

  // FISHER: the norms first; the relative regulariser is measured against their mean
  __shared__ double f2s[ISOPO_MAX_SEQ_TRANSFORM];
  __shared__ int fail;
  if (variant == 0) {
    for (int i = tid / kWave; i < m; i += kThreads / kWave) {             // a wave per row
      double s = 0.0;
      for (int j = tid % kWave; j < m; j += kWave) {
        const double k = (double)K[(size_t)i * m + j];
        s += k * k;
      }
      s = wave_sum(s);
      if (tid % kWave == 0) f2s[i] = s / (double)m;
    }
    __syncthreads();
  }

  double reg = (double)lambda;
  if (reg_mode != 0) {
    // this batch's typical value of what reg is added to: the mean eigenvalue tr(K)/m of K (INTERACTING),
    // the mean of the Fisher norms (FISHER)
    double part = 0.0;
    for (int i = tid; i < m; i += kThreads) part += variant == 0 ? f2s[i] : (double)K[(size_t)i * m + i];
    double scale = block_sum<kThreads>(part, red) / (double)m;
    if (reg_mode == 2) {
      // trailing mean over minibatches, this one included; every thread forms the same value from the
      // state as it was, then one thread stores the new state
      float* st = ema_state + (size_t)prob * 2;
      const double prev = (double)st[0];
      const bool first = st[1] == 0.f;
      scale = first ? scale : (double)ema_decay * prev + (1.0 - (double)ema_decay) * scale;
      __syncthreads();                                                  // everyone has read the old state
      if (tid == 0) { st[0] = (float)scale; st[1] = st[1] + 1.f; }
    }
    reg = (double)lambda * scale;
  }

  if (variant == 0) {
    for (int i = tid; i < m; i += kThreads) {
      const double den = f2s[i] + reg;
      c[i] = den > 0.0 ? (float)((double)A[i] / sqrt(den)) : 0.f;
    }
    if (info && tid == 0) info[prob] = 0;
    return;
  }

  {
    if constexpr (GLOBAL) {
      double* Mg = gws + (size_t)prob * ((size_t)m * m + m);
      double* inv_diag = reinterpret_cast<double*>(smem);
      double* PT = inv_diag + transform_front(m);
      int fail_col = 0;
      const bool ok = m <= kTransformWidePanelMax ? cholesky_solve<kThreads, 32>(K, A, m, reg, Mg, f2s, inv_diag, PT, &fail, &fail_col)
                                                  : cholesky_solve<kThreads, 16>(K, A, m, reg, Mg, f2s, inv_diag, PT, &fail, &fail_col);
      for (int i = tid; i < m; i += kThreads) c[i] = ok ? (float)f2s[i] : __builtin_nanf("");
      if (info && tid == 0) info[prob] = ok ? 0 : fail_col + 1;
    } else {
      // the matrix in LDS as well, panels of 16 columns
      double* inv_diag = reinterpret_cast<double*>(smem);
      double* Ml = inv_diag + transform_front(m);
      int fail_col = 0;
      const bool ok = cholesky_solve<kThreads, 16>(K, A, m, reg, Ml, f2s, inv_diag, Ml + (size_t)(m + 1) * m, &fail, &fail_col);
      for (int i = tid; i < m; i += kThreads) c[i] = ok ? (float)f2s[i] : __builtin_nanf("");
      if (info && tid == 0) info[prob] = ok ? 0 : fail_col + 1;
    }
  }
}

}  // namespace

// Dynamic LDS of the INTERACTING transform: the panel (32 columns up to kTransformWidePanelMax sequences in
// global scratch, else 16) or what the backward solve keeps there instead (at most 1024 / 16 + 16 rows of 17),
// up to kTransformLdsMax sequences the matrix with the row of A in front of it, and what stands ahead of both.
constexpr size_t transform_lds_bytes(int m) {
  const bool lds = m <= kTransformLdsMax;
  const int nb = transform_panel(m);
  size_t panel = (size_t)nb * panel_stride(m);
  const size_t backward = nb == 32 ? (size_t)(32 + 32) * 33 : (size_t)(64 + 16) * 17;
  if (panel < backward) panel = backward;
  return (transform_front(m) + (lds ? (size_t)(m + 1) * m : 0) + panel) * sizeof(double);
}

template <int THREADS, bool GLOBAL>
hipError_t launch_transform_t(const TransformArgs& a, size_t smem, double* gws, hipStream_t s) {
  auto kern = transform_kernel<THREADS, GLOBAL>;
  // once per process and instantiation (static initialisation is thread-safe); a failure is returned by every call
  constexpr int max_smem = (int)transform_lds_bytes(kTransformLdsMax) > (int)transform_lds_bytes(kTransformWidePanelMax)
                               ? (int)transform_lds_bytes(kTransformLdsMax) : (int)transform_lds_bytes(kTransformWidePanelMax);
  static_assert(transform_lds_bytes(ISOPO_MAX_SEQ_TRANSFORM) <= (size_t)max_smem && max_smem + 8704 <= 160 * 1024, "LDS budget");
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, max_smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(a.batch), dim3(THREADS), smem, s, a.K, a.A, a.n_seq, a.variant, a.reg_mode, a.lambda,
                     a.c, a.info, gws, a.ema_state, a.ema_decay);
  return hipGetLastError();
}

hipError_t launch_transform(const TransformArgs& a, hipStream_t s) {
  const bool lds = a.n_seq <= kTransformLdsMax;
  const size_t smem = a.variant == 1 ? transform_lds_bytes(a.n_seq) : 0;
  double* gws = (a.variant == 1 && !lds) ? a.workspace : nullptr;
  // the matrix in global memory: 512 threads have the registers for panels of 32 columns (256 sequences, with register blocks
  // for the trailing update: 229 us against 309 with 1024, 328 before), 1024 the loads in flight for the larger ones (1024 sequences: 6.0 ms against 6.8 and 9.0)
  if (!lds) return a.variant == 1 && a.n_seq <= kTransformWidePanelMax ? launch_transform_t<512, true>(a, smem, gws, s)
                                                                       : launch_transform_t<1024, true>(a, smem, gws, s);
  // more threads for the larger problems' trailing updates
  if (a.n_seq <= 48) return launch_transform_t<256, false>(a, smem, gws, s);
  return launch_transform_t<512, false>(a, smem, gws, s);
}

}  // namespace isopo
