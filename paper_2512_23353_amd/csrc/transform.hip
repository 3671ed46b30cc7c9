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
// The m x m problem is tiny next to the contractions around it, so one workgroup per problem works in fp64: a right-looking
// Cholesky factorisation with A as one more row or column of the matrix, which makes the forward solve part of the factorisation,
// and a backward solve block by block.  Up to 256 sequences the matrix lives in the registers of the workgroup's waves
// (transform_regs_kernel); larger ones in a caller-provided global scratch, with the panel being factored in LDS, column-major
// (transform_kernel).  The result is the unique solution; the eigendecomposition the interacting listing uses reaches the same
// vector.  A non-positive pivot is reported, never clamped.
#include "common.h"
#include "gram_finish.h"
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
__host__ __device__ constexpr int transform_panel(int m) { return m <= kTransformWidePanelMax ? 32 : 16; }
__host__ __device__ constexpr int transform_front(int m) { return m + transform_panel(m) * (transform_panel(m) + 1); }

// (K + reg I) c = A: M [m + 1, m] fp64 in global memory (row m holds A, then y), the panel of NB columns
// in LDS as PT[column][row - k0] with row stride RS.  c is left in cs.
//
// Panel step: every wave holds the NB rows of the panel's diagonal block and 64 - NB rows below it, one per lane, in
// registers, and factors the NB columns by itself (the diagonal block again in every wave): the pivot and a column's entries
// of the diagonal block's rows come from their lanes (v_readlane), so that a column is one reciprocal square root and a
// chain of multiply-adds, without an LDS round trip or a barrier (one of each per column, and a 64-bit division and
// square root in every thread, made a column 0.8 us).  1024 sequences: 8980 us before, 5080 now.  The kernel spills 6 scalar
// registers, and at 1024 threads, whose cap is 128 vector registers, 4 and 14 vector ones.  The upper triangle of the diagonal
// block is carried along and never read.
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

// ---- up to kTransformRegsMax sequences: the matrix in registers ----
//
// M = U^T U by blocks of 16 x 16 of the upper triangle, with A as one more block column, every block four 64-bit values per lane of
// one wave (the fp64 MFMA's result: value v of lane l is row 4 v + l / 16 of column l % 16).  Those registers are at once the MFMA's
// right operand B and, as a left one, B^T, so that neither U_ki^T U_kj nor L^-1 M_kj ever turns a block round; blocks meet through
// LDS as they lie.  What is held is N = -M, so that the trailing update is the MFMA's own sum.  Per block row k:
//   factor   the wave with the diagonal block, four columns at a time with a row per lane, the other columns by one MFMA after
//            each four; the identity's rows ride along, which leaves the transpose of L^-1
//   solve    U_kj = L^-1 M_kj, the waves with the blocks of the row;  barrier
//   update   N_ij += U_ki^T U_kj, all waves; the wave with the next diagonal block starts with that and factors it at once;  barrier
// The backward solve goes column by column the other way, c_j = L_j^-T v_j by every wave for itself and v_k -= U_kj c_j by the wave
// with the block, a barrier per column.  Blocks of a row lie in different waves.
//
// What bounds it: the instructions of the chain of sixteen pivots per block row (about 2 us a row in all: at 64 sequences 8 of 12.7,
// the rest launch, loads and the backward solve), and past some 128 sequences the fp64 MFMAs of the update as well (at 256 half).
// With the matrix in LDS or in global memory and a panel of columns staged in LDS, as transform_kernel has it, every block goes
// through memory once per panel: us before and now, 16 sequences 7.3 and 5.0; 32, 12.5 and 7.3; 64, 24.4 and 12.7; 128, 56.9 and
// 27.9; 192, 113 and 58; 256, 187 and 89.  Tried: a row per lane for all sixteen columns, without the MFMA between (64: 15.3; 256:
// 123); the four pivots from their 4 x 4 block alone, in every lane (64: 13.1); eight waves at 256 (95).  Sixteen waves have 128
// registers each, of which the blocks take 80: ten words a lane go to scratch, and 85 scalar registers into lanes of vector ones (25 with
// eight waves, 32 where K is finished first, none with four).
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kBlk = 16, kBlkPitch = kBlk + 1;

struct Regulariser {
  int mode;
  float lambda;
  float* ema_state;
  float ema_decay;
};
// reg from the sum over the batch of what it is added to (the same in all threads)
template <class Barrier>
__device__ __forceinline__ double regulariser(const Regulariser& r, double sum, int m, int prob, Barrier&& barrier) {
  if (r.mode == 0) return (double)r.lambda;
  // this batch's typical value of what reg is added to: the mean eigenvalue tr(K)/m of K (INTERACTING),
  // the mean of the Fisher norms (FISHER)
  double scale = sum / (double)m;
  if (r.mode == 2) {
    // trailing mean over minibatches, this one included; every thread forms the same value from the
    // state as it was, then one thread stores the new state
    float* st = r.ema_state + (size_t)prob * 2;
    const double prev = (double)st[0];
    const bool first = st[1] == 0.f;
    scale = first ? scale : (double)r.ema_decay * prev + (1.0 - (double)r.ema_decay) * scale;
    barrier();                                                          // everyone has read the old state
    if (threadIdx.x == 0) { st[0] = (float)scale; st[1] = st[1] + 1.f; }
  }
  return (double)r.lambda * scale;
}

// Sum over the sixteen lanes of a row, in all of them.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
  return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double x) {
  x = dpp_add<0xb1>(x);                                  // quad_perm [1,0,3,2]
  x = dpp_add<0x4e>(x);                                  // quad_perm [2,3,0,1]
  x = dpp_add<0x141>(x);                                 // row_half_mirror
  return dpp_add<0x140>(x);                              // row_mirror
}

// The four rows of sixteen lanes of x, each in all four: r[g] of lane l is x of lane 16 g + l % 16.
__device__ __forceinline__ void four_rows(double x, double (&r)[4]) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  unsigned half[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned a = h ? (unsigned)__double2hiint(x) : (unsigned)__double2loint(x);
    const u32x2 p = __builtin_amdgcn_permlane32_swap(a, a, false, false);           // rows 0 1 0 1, 2 3 2 3
    const u32x2 lo = __builtin_amdgcn_permlane16_swap(p[0], p[0], false, false), hi = __builtin_amdgcn_permlane16_swap(p[1], p[1], false, false);
    half[h][0] = lo[0]; half[h][1] = lo[1]; half[h][2] = hi[0]; half[h][3] = hi[1];
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) r[g] = __hiloint2double((int)half[1][g], (int)half[0][g]);
}

// 1 / sqrt(p), p a positive number: the instruction's estimate y, and one third-order step, y (1 + e / 2 + 3 e^2 / 8) with
// e = 1 - p y^2.  NaN for zero and infinity (no pivot is infinite: kInfinite).
__device__ __forceinline__ double inverse_root(double p) {
  const double y = __builtin_amdgcn_rsq(p), e = fma(-p * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// An infinite diagonal entry as the factorisation holds it (K's finite ones are below 2^128, reg below 2^257): the root of its pivot
// divides that sequence's coefficient, and its part in the others', down to nothing.  (Infinity itself would be inf * 0 in
// inverse_root; a comparison there cost 2 % of the solve.)
constexpr double kInfinite = 0x1p1000;

// Doubles of dynamic LDS: the blocks of a row of U, every block row's -L^-1, transposed, and v.
__host__ __device__ constexpr int transform_blocks(int m) { return (m + kBlk - 1) / kBlk; }
constexpr size_t transform_regs_lds(int m) {
  const int nb = transform_blocks(m);
  return ((size_t)(nb + 1) * kBlk * kBlk + (size_t)nb * kBlk * kBlkPitch + nb * kBlk) * sizeof(double);
}

// W waves, the workgroup's first ones (the others have returned); S blocks off the diagonal and DN on it per wave.
template <int W, int S, int DN, bool SHARED>
__device__ __forceinline__ void transform_regs(const float* K, const float* A, int m, const Regulariser& prm, int prob, float* c,
                                               int32_t* info, unsigned char* smem) {
  __shared__ double red[W];
  __shared__ int fail;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = transform_blocks(m);
  double* const ubuf = reinterpret_cast<double*>(smem);  // [block column][value pair][lane][2]
  double* const xbuf = ubuf + (nb + 1) * kBlk * kBlk;    // [block row][i][kBlkPitch]: -(L^-1)^T
  double* const vec = xbuf + nb * kBlk * kBlkPitch;      // [nb * 16]

  // ---- the blocks: diagonal ones dealt to the waves in order, the others row by row ----
  int bk[S], bj[S];                                      // block row (-1: none) and column of a slot
  {
    int k = 0, at = wave;                                // place in row k, which has blocks k + 1 .. nb
#pragma unroll
    for (int s = 0; s < S; ++s) {
      while (k < nb && at >= nb - k) { at -= nb - k; ++k; }
      bk[s] = k < nb ? k : -1;
      bj[s] = k < nb ? k + 1 + at : 0;
      at += W;
    }
  }
  if (tid == 0) fail = -1;
  // entry (r, q), r <= q, is K's (q, r): the lower triangle is what is read
  float diag_in[DN][4], in[S][4];
#pragma unroll
  for (int d = 0; d < DN; ++d) {
    const int k = wave + d * W;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = kBlk * k + 4 * v + l4, q = kBlk * k + l16, lo = r < q ? r : q, hi = r < q ? q : r;
      const bool there = k < nb && hi < m;
      const float x = get_shared<SHARED>(K + (there ? (size_t)hi * m + lo : 0));
      diag_in[d][v] = there ? x : 0.f;
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const bool rhs = bj[s] == nb;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = kBlk * bk[s] + 4 * v + l4, q = rhs ? m : kBlk * bj[s] + l16;
      const bool there = bk[s] >= 0 && r < m && (rhs ? l16 == 0 : q < m);
      const float* const from = rhs ? A + r : K + (size_t)q * m + r;
      const float x = get_shared<SHARED>(there ? from : K);
      in[s][v] = there ? x : 0.f;
    }
  }
  double reg = (double)prm.lambda;
  if (prm.mode != 0) {
    const double part = wave_sum(tid < m ? (double)get_shared<SHARED>(K + (size_t)tid * m + tid) : 0.0);   // m <= 64 W
    if (lane == 0) red[wave] = part;
    __syncthreads();
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) sum += red[w];
    reg = regulariser(prm, sum, m, prob, [] { __syncthreads(); });
  }
  f64x4 D[DN], N[S];
#pragma unroll
  for (int d = 0; d < DN; ++d)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 4 * v + l4;
      const bool padded = kBlk * (wave + d * W) + r >= m;           // the identity's rows
      const double x = (double)diag_in[d][v] + (r == l16 ? (padded ? 1.0 : reg) : 0.0);
      D[d][v] = r == l16 && x > kInfinite ? -kInfinite : -x;
    }
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int v = 0; v < 4; ++v) N[s][v] = -(double)in[s][v];

  // One wave: block row k's diagonal block factored, -(L^-1)^T left in xbuf.
  auto factor = [&](const f64x4& n, int k) {
    f64x4 M = -n, X;                                     // X: rows of the identity; transposed, as the symmetric M is
#pragma unroll
    for (int v = 0; v < 4; ++v) X[v] = 4 * v + l4 == l16 ? 1.0 : 0.0;
    int first_bad = m;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // columns 4 s .. 4 s + 3 of row l % 16, in all lanes
      double w[4], x[4];
      four_rows(M[s], w);
      four_rows(X[s], x);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int at = 4 * s + j;
        const double p = lane_value(w[j], at);           // a pivot that is not positive leaves NaN or infinity in all that follows
        if (!(p > 0.0) && kBlk * k + at < first_bad) first_bad = kBlk * k + at;
        const double inv = inverse_root(p);
        w[j] *= inv;
        x[j] *= inv;
#pragma unroll
        for (int q = j + 1; q < 4; ++q) {
          const double f = lane_value(w[j], 4 * s + q);
          w[q] -= w[j] * f;
          x[q] -= x[j] * f;
        }
      }
      const double wk = l4 < 2 ? (l4 == 0 ? w[0] : w[1]) : (l4 == 2 ? w[2] : w[3]);
      const double xk = l4 < 2 ? (l4 == 0 ? x[0] : x[1]) : (l4 == 2 ? x[2] : x[3]);
      if (s < 3) {
        M = __builtin_amdgcn_mfma_f64_16x16x4f64(-wk, wk, M, 0, 0, 0);
        X = __builtin_amdgcn_mfma_f64_16x16x4f64(-wk, xk, X, 0, 0, 0);
      }
      xbuf[(k * kBlk + l16) * kBlkPitch + 4 * s + l4] = -xk;
    }
    if (first_bad < m && lane == 0) fail = first_bad;
  };
  auto put = [&](int j, const f64x4& u) {
    double2* const to = reinterpret_cast<double2*>(ubuf + j * kBlk * kBlk) + lane;
    to[0] = make_double2(u[0], u[1]);
    to[64] = make_double2(u[2], u[3]);
  };
  auto get = [&](int j) {
    const double2* const from = reinterpret_cast<const double2*>(ubuf + j * kBlk * kBlk) + lane;
    const double2 a = from[0], b = from[64];
    return f64x4{a.x, a.y, b.x, b.y};
  };
  auto product = [](const f64x4& a, const f64x4& b, f64x4 sum) {
#pragma unroll
    for (int s = 0; s < 4; ++s) sum = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], sum, 0, 0, 0);
    return sum;
  };

  if (wave == 0) factor(D[0], 0);
  for (int k = 0; k < nb; ++k) {
    __syncthreads();
    if (fail >= 0) break;                                // every thread reads the same value
    f64x4 left;                                          // -L^-1
#pragma unroll
    for (int s = 0; s < 4; ++s) left[s] = xbuf[(k * kBlk + 4 * s + l4) * kBlkPitch + l16];
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (bk[s] == k) {
        N[s] = product(left, N[s], f64x4{0.0, 0.0, 0.0, 0.0});
        put(bj[s], N[s]);
      }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < DN; ++d) {
      const int j = wave + d * W;
      if (j > k && j < nb) {
        const f64x4 u = get(j);
        D[d] = product(u, u, D[d]);
        if (j == k + 1) factor(D[d], j);
      }
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (bk[s] > k) N[s] = product(get(bk[s]), get(bj[s]), N[s]);
  }
  const int failed = fail;                               // read after a barrier: the last block row has no factor behind it
  if (failed >= 0) {
    for (int i = tid; i < m; i += 64 * W) c[i] = __builtin_nanf("");
    if (info && tid == 0) *info = failed + 1;
    return;
  }
  if (info && tid == 0) *info = 0;

  // backward: v starts as y
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (bk[s] >= 0 && bj[s] == nb && l16 == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) vec[kBlk * bk[s] + 4 * v + l4] = N[s][v];
    }
  for (int j = nb - 1; j >= 0; --j) {
    __syncthreads();
    double x = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) x -= xbuf[(j * kBlk + l16) * kBlkPitch + 4 * l4 + t] * vec[kBlk * j + 4 * l4 + t];
    x += __shfl_xor(x, 16, kWave);
    x += __shfl_xor(x, 32, kWave);
    if (wave == j % W && lane < kBlk && kBlk * j + lane < m) c[kBlk * j + lane] = (float)x;
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (bk[s] >= 0 && bj[s] == j) {
        double t[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) t[v] = row_sum(N[s][v] * x);
        if (l16 == 0) {
#pragma unroll
          for (int v = 0; v < 4; ++v) vec[kBlk * bk[s] + 4 * v + l4] -= t[v];
        }
      }
  }
}

// FISHER: the norms first; the relative regulariser is measured against their mean.
template <int THREADS, int ROWS, bool SHARED>
__device__ __forceinline__ void fisher_transform(const float* K, const float* A, int m, const Regulariser& prm, int prob, float* c,
                                                 int32_t* info) {
  constexpr int kWaves = THREADS / kWave;
  __shared__ double red[kWaves];
  __shared__ double f2s[ISOPO_MAX_SEQ_TRANSFORM];
  const int tid = threadIdx.x;
  // a wave takes ROWS rows at a time
  for (int i = tid / kWave * ROWS; i < m; i += kWaves * ROWS) {
    double s[ROWS] = {};
    if constexpr (ROWS == 1) {
      // 128 columns on their way together (below, the lanes whose trips are fewer wait for their last one by themselves: 96 sequences 6.7
      // us, and 6.3 so; four rows at a time, 256 sequences 16.3, and 17.2 so)
      for (int j0 = 0; j0 < m; j0 += 2 * kWave) {
        float k[2] = {0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int j = j0 + u * kWave + tid % kWave;
          if (j < m) k[u] = get_shared<SHARED>(K + (size_t)i * m + j);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) s[0] += (double)k[u] * (double)k[u];
      }
    } else {
#pragma unroll 2
      for (int j = tid % kWave; j < m; j += kWave)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          const double k = (double)get_shared<SHARED>(K + (size_t)(i + r < m ? i + r : m - 1) * m + j);
          s[r] += k * k;
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      s[r] = wave_sum(s[r]);
      if (tid % kWave == 0 && i + r < m) f2s[i + r] = s[r] / (double)m;
    }
  }
  __syncthreads();
  double part = 0.0;
  if (prm.mode != 0)
    for (int i = tid; i < m; i += THREADS) part += f2s[i];
  const double reg = regulariser(prm, prm.mode != 0 ? block_sum<THREADS>(part, red) : 0.0, m, prob, [] { __syncthreads(); });
  for (int i = tid; i < m; i += THREADS) {
    const double den = f2s[i] + reg;
    c[i] = den > 0.0 ? (float)((double)A[i] / sqrt(den)) : 0.f;
  }
  if (info && tid == 0) *info = 0;
}

template <int W, int S, int DN>
__global__ __launch_bounds__(64 * W) void transform_regs_kernel(const float* __restrict__ K, const float* __restrict__ A, int m,
                                                                Regulariser prm, float* __restrict__ c, int32_t* __restrict__ info) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int prob = blockIdx.x;
  transform_regs<W, S, DN, false>(K + (size_t)prob * m * m, A + (size_t)prob * m, m, prm, prob, c + (size_t)prob * m,
                           info ? info + prob : nullptr, smem);
}

template <int THREADS, int ROWS>
__global__ __launch_bounds__(THREADS) void fisher_transform_kernel(const float* __restrict__ K, const float* __restrict__ A, int m,
                                                                   Regulariser prm, float* __restrict__ c, int32_t* __restrict__ info) {
  const int prob = blockIdx.x;
  fisher_transform<THREADS, ROWS, false>(K + (size_t)prob * m * m, A + (size_t)prob * m, m, prm, prob, c + (size_t)prob * m,
                                  info ? info + prob : nullptr);
}

// The Gram matrix from its slots, and by the workgroup that finds itself the last one to have written its part of it the
// coefficients: a launch and the wait between two fewer.  `arrived` counts the workgroups, from zero.
// 16 sequences 8.9 us against 4.8 and 6.1 in two launches.  K's entries pass the L2s on their way out and back in, so that no
// workgroup has to write its L2 back or to drop it: with such fences the two launches were the faster ones (whole calls of 94 us
// 2 us slower).
template <int W, int S>
__global__ __launch_bounds__(kFinishThreads) void finish_transform_kernel(GramFinish f, int32_t* arrived, const float* __restrict__ A,
                                                                          int variant, Regulariser prm, float* __restrict__ c,
                                                                          int32_t* info) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int last;
  gram_finish<true>(f);
  if (threadIdx.x < kWave) {                             // the wave that has written: its part is there before it counts
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0) last = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  if (variant == 0) {
    fisher_transform<kFinishThreads, 1, true>(f.K, A, f.n_seq, prm, 0, c, info);
    return;
  }
  if (threadIdx.x >= 64 * W) return;
  transform_regs<W, S, 1, true>(f.K, A, f.n_seq, prm, 0, c, info, smem);
}

// INTERACTING, the matrix in global memory.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void transform_kernel(const float* __restrict__ Kb, const float* __restrict__ Ab, int m,
                                                             Regulariser prm, float* __restrict__ cb, int32_t* __restrict__ info,
                                                             double* __restrict__ gws) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ double red[kThreads / 64];
  __shared__ double cs[ISOPO_MAX_SEQ_TRANSFORM];
  __shared__ int fail;
  const int prob = blockIdx.x, tid = threadIdx.x;
  const float* K = Kb + (size_t)prob * m * m;
  const float* A = Ab + (size_t)prob * m;
  float* c = cb + (size_t)prob * m;
  double part = 0.0;
  if (prm.mode != 0)
    for (int i = tid; i < m; i += kThreads) part += (double)K[(size_t)i * m + i];
  const double reg = regulariser(prm, prm.mode != 0 ? block_sum<kThreads>(part, red) : 0.0, m, prob, [] { __syncthreads(); });
  double* Mg = gws + (size_t)prob * ((size_t)m * m + m);
  double* inv_diag = reinterpret_cast<double*>(smem);
  double* PT = inv_diag + transform_front(m);
  int fail_col = 0;
  const bool ok = m <= kTransformWidePanelMax ? cholesky_solve<kThreads, 32>(K, A, m, reg, Mg, cs, inv_diag, PT, &fail, &fail_col)
                                              : cholesky_solve<kThreads, 16>(K, A, m, reg, Mg, cs, inv_diag, PT, &fail, &fail_col);
  for (int i = tid; i < m; i += kThreads) c[i] = ok ? (float)cs[i] : __builtin_nanf("");
  if (info && tid == 0) info[prob] = ok ? 0 : fail_col + 1;
}

// Dynamic LDS of transform_kernel: the panel (32 columns up to kTransformWidePanelMax sequences, else 16) or what the backward
// solve keeps there instead (at most 1024 / 16 + 16 rows of 17), and what stands ahead of it.
constexpr size_t transform_lds_bytes(int m) {
  const int nb = transform_panel(m);
  size_t panel = (size_t)nb * panel_stride(m);
  const size_t backward = nb == 32 ? (size_t)(32 + 32) * 33 : (size_t)(64 + 16) * 17;
  if (panel < backward) panel = backward;
  return (transform_front(m) + panel) * sizeof(double);
}

// kern's dynamic LDS limit raised once per process (static initialisation is thread-safe); a failure is returned by every call
template <auto KERN, int BYTES>
hipError_t lds_limit() {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, BYTES);
  return attr;
}

template <int THREADS>
hipError_t launch_global(const TransformArgs& a, const Regulariser& reg, hipStream_t s) {
  constexpr int most = (int)transform_lds_bytes(kTransformWidePanelMax);
  static_assert(transform_lds_bytes(ISOPO_MAX_SEQ_TRANSFORM) <= (size_t)most && most + 8704 <= 160 * 1024, "LDS budget");
  if (const hipError_t e = lds_limit<&transform_kernel<THREADS>, most>(); e != hipSuccess) return e;
  hipLaunchKernelGGL(transform_kernel<THREADS>, dim3(a.batch), dim3(THREADS), transform_lds_bytes(a.n_seq), s, a.K, a.A, a.n_seq, reg, a.c,
                     a.info, a.workspace);
  return hipGetLastError();
}

template <int W, int S, int DN>
hipError_t launch_regs(const TransformArgs& a, const Regulariser& reg, hipStream_t s) {
  constexpr int blocks = W * DN, most = (int)transform_regs_lds(16 * blocks);
  static_assert(blocks * (blocks + 1) / 2 <= W * S && 16 * blocks <= 64 * W && most <= 150 * 1024, "slots for every block, a thread per row");
  if (const hipError_t e = lds_limit<&transform_regs_kernel<W, S, DN>, most>(); e != hipSuccess) return e;
  hipLaunchKernelGGL((transform_regs_kernel<W, S, DN>), dim3(a.batch), dim3(64 * W), transform_regs_lds(a.n_seq), s, a.K, a.A, a.n_seq, reg,
                     a.c, a.info);
  return hipGetLastError();
}

// K from the token products' 64-bit sums, and the coefficients, in one workgroup: a launch less.  With the chain's preparation in the
// launch of the products (ghost_gram.hip) Gram matrix and transform of ten random layers 0.89x (1024x3072, 7 sequences, 504 tokens 35.7
// -> 29.9 us); 5120x27648, 8 sequences of 64 to 256 tokens 517 -> 511 us a layer step.
template <int W, int S>
__global__ __launch_bounds__(kFinishThreads) void ghost_finish_transform_kernel(const double* __restrict__ K64, float* K, int m,
                                                                                const float* __restrict__ A, int variant,
                                                                                Regulariser prm, float* __restrict__ c, int32_t* info) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  for (int e = threadIdx.x; e < m * m; e += kFinishThreads) {
    const int i = e / m, j = e % m;
    if (i <= j) {
      const float v = (float)K64[e];
      K[(size_t)i * m + j] = v;
      K[(size_t)j * m + i] = v;
    }
  }
  __syncthreads();
  if (variant == 0) {
    fisher_transform<kFinishThreads, 1, false>(K, A, m, prm, 0, c, info);
    return;
  }
  if (threadIdx.x >= 64 * W) return;
  transform_regs<W, S, 1, false>(K, A, m, prm, 0, c, info, smem);
}

template <int W, int S>
hipError_t launch_finish(const GramFinish& f, int32_t* arrived, const TransformArgs& a, const Regulariser& reg, hipStream_t s) {
  static_assert(transform_regs_lds(16 * W) + sizeof(double) * (1024 + ISOPO_MAX_SEQ_TRANSFORM) <= 60 * 1024, "LDS without a limit raised");
  hipLaunchKernelGGL((finish_transform_kernel<W, S>), dim3((unsigned)(f.slot_floats / 64)), dim3(kFinishThreads),
                     transform_regs_lds(f.n_seq), s, f, arrived, a.A, a.variant, reg, a.c, a.info);
  return hipGetLastError();
}

template <int W, int S>
hipError_t launch_ghost_finish(const double* K64, float* K, const TransformArgs& a, const Regulariser& reg, hipStream_t s) {
  hipLaunchKernelGGL((ghost_finish_transform_kernel<W, S>), dim3(1), dim3(kFinishThreads), transform_regs_lds(a.n_seq), s, K64, K, a.n_seq,
                     a.A, a.variant, reg, a.c, a.info);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ghost_finish_transform(const double* K64, float* K, const TransformArgs& a, hipStream_t s) {
  const Regulariser reg{a.reg_mode, a.lambda, a.ema_state, a.ema_decay};
  if (a.n_seq > kTransformFinishMax || a.batch != 1) return hipErrorInvalidValue;
  return a.n_seq <= 64 ? launch_ghost_finish<4, 3>(K64, K, a, reg, s) : launch_ghost_finish<8, 5>(K64, K, a, reg, s);
}

hipError_t launch_finish_transform(const GramFinish& f, int32_t* arrived, const TransformArgs& a, hipStream_t s) {
  const Regulariser reg{a.reg_mode, a.lambda, a.ema_state, a.ema_decay};
  if (f.n_seq > kTransformFinishMax || !arrived || a.batch != 1) return hipErrorInvalidValue;
  return f.n_seq <= 64 ? launch_finish<4, 3>(f, arrived, a, reg, s) : launch_finish<8, 5>(f, arrived, a, reg, s);
}

hipError_t launch_transform(const TransformArgs& a, hipStream_t s) {
  const Regulariser reg{a.reg_mode, a.lambda, a.ema_state, a.ema_decay};
  if (a.variant == 0) {
    // What it waits for is memory, so as many rows are on their way as there are, but a wave more or a second sum costs too.  us with
    // 256 threads and a row per wave, 1024 and one, 1024 and four: 4 sequences 2.8, 3.1, 3.4; 16 3.9, 3.5, 3.7; 64 -, 5.3, 5.4;
    // 128 -, 8.0, 8.0; 224 -, 15.5, 12.1; 1024 -, 92, 71 (220 with one load in flight).  More problems than compute units (256) wait for
    // each other's waves, of which the smaller ones then take fewer: 16 sequences, 1000 problems 8.5 with 1024 threads, 6.2 with 512, 5.7
    // with 256; 33, 400 6.6, 5.8, 7.0; 64, 1000 15.2, 13.4, 13.2; 97, 400 11.6, 10.9, -.
    auto launch = [&](auto kern, int threads) {
      hipLaunchKernelGGL(kern, dim3(a.batch), dim3(threads), 0, s, a.K, a.A, a.n_seq, reg, a.c, a.info);
      return hipGetLastError();
    };
    if (a.n_seq <= 8 || (a.n_seq <= 48 && a.batch > 512)) return launch(fisher_transform_kernel<256, 1>, 256);
    if (a.n_seq <= 104 && a.batch > 256) return launch(fisher_transform_kernel<512, 1>, 512);
    return a.n_seq <= 96 ? launch(fisher_transform_kernel<1024, 1>, 1024) : launch(fisher_transform_kernel<1024, 4>, 1024);
  }
  if (a.n_seq <= 64) return launch_regs<4, 3, 1>(a, reg, s);
  if (a.n_seq <= 128) return launch_regs<8, 5, 1>(a, reg, s);
  if (a.n_seq <= kTransformRegsMax) return launch_regs<16, 9, 1>(a, reg, s);
  // the matrix in global memory: 512 threads have the registers for panels of 32 columns, 1024 the loads in flight for the larger
  // ones (1024 sequences: 6.0 ms against 6.8)
  return a.n_seq <= kTransformWidePanelMax ? launch_global<512>(a, reg, s) : launch_global<1024>(a, reg, s);
}

}  // namespace isopo
