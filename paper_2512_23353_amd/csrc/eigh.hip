// Eigendecomposition route of the interacting variant (interacting listing:
// D, U = eigh(ntk); c = U ((1 / (D + regularization)) * (U^T A))).
//
// One decomposition serves any number of regularisers, so a sweep over lambda
// costs one factorisation instead of one Cholesky per value.  K is m x m with
// m the number of sequences (tens to a few hundred), so one workgroup per problem
// (a block's projections go in one launch) runs the classical dense route in fp64:
// Householder tridiagonalisation, then divide and conquer on the tridiagonal matrix.
// Eigenvalues come out ascending, eigenvectors as columns.
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace isopo {
namespace {

template <int THREADS>
__device__ double block_sum(double x, double* red) {
  x = wave_sum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) s += red[w];
  return s;
}

// K = H T H^T with H a product of n - 2 reflectors H_k = I - tau_k v_k v_k^T and T tridiagonal; T = Q^T diag(D) Q by
// Cuppen's divide and conquer with Gu and Eisenstat's stable eigenvectors (SIAM J. Matrix Anal. Appl. 16, 1995);
// U = H Q^T.
// One workgroup per problem, fp64 throughout: bound by the latency of its dependent steps and, with sixteen waves on four
// vector units, by what each of them issues, so that sums run over sixteen lanes where sixteen rows wait side by side.
// 16 / 32 / 64 / 96 / 128 / 256 / 512 / 1024 sequences: 0.04 / 0.07 / 0.14 / 0.32 / 0.55 / 5.5 / 45 / 380 ms, where a Jacobi
// iteration (two barriers per round of n/2 rotations, up to 94 sequences) and implicit QL (a sequential chain of about 25
// dependent operations per plane rotation) took 0.09 / 0.26 / 1.19 ms at 16 / 32 / 64 and 5.5 / 22 / 100 / 630 from 128 on; errors
// of D, U^T U and U D U^T 2e-16 .. 1e-14 of the largest eigenvalue, a fifth of the Jacobi iteration's.
// K is scaled by a power of two so that its largest entry lies in [1, 2) (exact; D is scaled back at the end).
//   A (n x n, kept bit-symmetric; LDS up to 128 sequences, else U's own memory): rows k+1.. of the trailing block are
//     updated as A -= v w^T + w v^T; row k then holds v_k for the back-transformation
//   Qt (n x n, two of them; LDS up to 64 sequences, else global scratch): row i is eigenvector i of the blocks solved so
//     far; a merge writes the other one
//
// The tree's leaves are single indices (every off-diagonal entry is torn out as |e| (1, s)(1, s)^T), the first level's pairs
// are solved directly.  All merges of a level are alike and run in step, an index's block given by its position: at the level with nb blocks, block s holds
// indices [s n / nb, (s + 1) n / nb).  A merge of blocks with eigenvalues d and coupling vector z (the last row of
// the left, s times the first row of the right eigenvectors, over sqrt 2; rho = 2 |e|):
//   rank      d sorted within the block, one thread per index
//   deflation components with negligible rho |z|, and pairs close enough that a rotation clears one; the scan is sequential,
//             so it only runs in blocks where some neighbouring pair or component calls for it
//   roots     of 1 + rho sum z_i^2 / (d_i - x), sixteen lanes per root, as an offset from the nearer pole: the rational
//             interpolation through both neighbouring poles, kept inside a bracket that every step narrows
//   zh        the vector for which the computed roots are exact (products of differences): the eigenvectors formed from
//             it are orthogonal to rounding however close the roots are
//   vectors   columns zh_i / (d_i - x_j), normalised, times the old eigenvectors; a wave per four new vectors
constexpr double kUlp = 1.1102230246251565e-16;      // 2^-53
// Sums of squares below this, of a matrix whose largest entry is 1 to 2, count as zero: entries of 2^-450, where K's own
// reach down to 2^-277.  Where sequences are copies of each other the trailing block can shrink by 10^16 with every few
// columns, to where squares and their reciprocals leave the range of fp64.
constexpr double kNoSquare = 0x1p-900;

// Sums over the 16 lanes of a row, in all of them, and over the wave, in all lanes: lane permutations inside the vector
// unit instead of LDS round trips.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, false);
  return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double x) {
  x = dpp_add<0xB1, 0xf>(x);                         // lanes xor 1
  x = dpp_add<0x4E, 0xf>(x);                         // lanes xor 2
  x = dpp_add<0x141, 0xf>(x);                        // mirrored within eight
  return dpp_add<0x140, 0xf>(x);                     // mirrored within sixteen
}
__device__ __forceinline__ double quad_sum(double x) { return dpp_add<0x4E, 0xf>(dpp_add<0xB1, 0xf>(x)); }
__device__ __forceinline__ double oct_sum(double x) { return dpp_add<0x141, 0xf>(quad_sum(x)); }
__device__ __forceinline__ int row_count(int x) {    // the same for counts
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false);
  return x + __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ double dpp_mul(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false);
  return x * __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_product(double x) {
  return dpp_mul<0x140>(dpp_mul<0x141>(dpp_mul<0x4E>(dpp_mul<0xB1>(x))));
}
__device__ __forceinline__ double lane_value(double x, int src) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), src);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), src);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double x) {
  x = row_sum(x);
  x = dpp_add<0x142, 0xa>(x);                        // rows 1 and 3 += the row before
  x = dpp_add<0x143, 0xc>(x);                        // rows 2 and 3 += rows 0 and 1
  return lane_value(x, 63);
}

// 1/x and sqrt(x) to a unit or so in the last place (x of normal size), without the full division's and root's long
// dependent chains.
__device__ __forceinline__ double quick_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double quick_sqrt(double x) { return x > 0.0 ? x * rsqrt(x) : 0.0; }

// Root j of 1 + rho sum_i z_i^2 / (d_i - x) over the k poles d (ascending, distinct), as d[org] + tau; LPR lanes (4, 8 or 16,
// lane `sub` of them): the interpolation is repeated in every one of them, so few lanes where there are few poles.  Up to
// PER poles a lane are held in registers, a step's terms are then independent of each other and of the LDS; PER = 0: any
// number, read at every step.  False where `limit` steps did not get there.
template <int LPR, int PER>
__device__ __forceinline__ bool secular_root(const double* d, const double* z, int k, double rho, int j, int sub, int limit,
                                             int& org, double& tau) {
  auto lanes_sum = [](double x) { return LPR == 4 ? quad_sum(x) : (LPR == 8 ? oct_sum(x) : row_sum(x)); };
  const bool last = j == k - 1;
  double zz = 0.0;
  if (last) {
    for (int i = sub; i < k; i += LPR) zz += z[i] * z[i];
    zz = lanes_sum(zz);
  }
  const double gap = last ? rho * zz : d[j + 1] - d[j];
  // which half of the interval
  double mid = 0.0;
#pragma unroll 4
  for (int i = sub; i < k; i += LPR) mid += z[i] * z[i] * quick_rcp((d[i] - d[j]) - 0.5 * gap);
  mid = 1.0 + rho * lanes_sum(mid);
  double lo, hi;
  org = j;
  if (mid >= 0.0) { lo = 0.0; hi = 0.5 * gap; }
  else if (last) { lo = 0.5 * gap; hi = gap * (1.0 + 8.0 * kUlp); }
  else { org = j + 1; lo = -0.5 * gap; hi = 0.0; }
  tau = 0.5 * (lo + hi);
  const double near = 4.0 * kUlp * quick_sqrt((double)k);
  const double dorg = d[org], dj = d[j] - dorg, dj1 = last ? 0.0 : d[j + 1] - dorg;
  [[maybe_unused]] double pole[PER > 0 ? PER : 1], before[PER > 0 ? PER : 1], behind[PER > 0 ? PER : 1];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int i = sub + LPR * t;
    pole[t] = i < k ? d[i] - dorg : 1e300;                       // none there: nothing of the sums
    const double rzz = i < k ? rho * z[i] * z[i] : 0.0;
    before[t] = i <= j ? rzz : 0.0;
    behind[t] = i <= j ? 0.0 : rzz;
  }
  for (int it = 0; it < limit; ++it) {
    double psi = 0.0, dpsi = 0.0, phi = 0.0, dphi = 0.0;         // poles up to j, and after it
    auto term = [&](double from_org, double before, double behind) __attribute__((always_inline)) {
      const double inv = quick_rcp(from_org - tau), inv2 = inv * inv;
      psi = fma(before, inv, psi); dpsi = fma(before, inv2, dpsi);
      phi = fma(behind, inv, phi); dphi = fma(behind, inv2, dphi);
    };
    if constexpr (PER > 0) {
#pragma unroll
      for (int t = 0; t < PER; ++t) term(pole[t], before[t], behind[t]);
    } else {
#pragma unroll 2
      for (int i = sub; i < k; i += LPR) {
        const double rzz = rho * z[i] * z[i];
        term(d[i] - dorg, i <= j ? rzz : 0.0, i <= j ? 0.0 : rzz);
      }
    }
    psi = lanes_sum(psi); dpsi = lanes_sum(dpsi); phi = lanes_sum(phi); dphi = lanes_sum(dphi);
    const double w = 1.0 + psi + phi;
    if (fabs(w) <= near * (1.0 + fabs(psi) + fabs(phi))) return true;
    if (w < 0.0) lo = tau; else hi = tau;
    const double dp = dj - tau;
    double eta;
    if (last) {
      eta = dp + dpsi * dp * dp * quick_rcp(w - dpsi * dp);      // one pole and a constant
    } else {
      const double dq = dj1 - tau;
      const double c = w - dpsi * dp - dphi * dq, b = (dp + dq) * w - dp * dq * (dpsi + dphi), a = w * dp * dq;
      const double s = quick_sqrt(b * b - 4.0 * a * c);
      eta = b > 0.0 ? 2.0 * a * quick_rcp(b + s) : (b - s) * quick_rcp(2.0 * c);
    }
    double next = tau + eta;
    if (!(next > lo && next < hi)) next = 0.5 * (lo + hi);       // also where the interpolation gave no number
    if (next == tau || next == lo || next == hi) return true;    // the bracket's ends are never taken: one may be a pole
    tau = next;
  }
  return false;
}

// Row pitch of a matrix in LDS: an odd multiple of sixteen doubles, so that the four rows a wave works on at a time lie in
// different banks, where that fits.
__host__ __device__ constexpr int eigh_pitch(int m) {
  const int p = (m + 15) / 16 * 16, odd = p % 32 ? p : p + 16;
  return (m <= 64 || m * odd <= 128 * 128) ? odd : m;
}

// The reduction of up to 16 NE rows to tridiagonal form with the matrix in registers and one barrier per column.  Sixteen
// lanes hold a row (lane `sub` its elements sub + 16 t) and a lane RN rows, so WV waves hold them all; zeros stand beyond n.
// What a column costs is the chain of its dependent steps (row, norm, v, A v, barrier, w) and what the waves of a vector unit
// issue.  So every sixteen lanes form the next column's reflector by themselves, from the row that its owner put into LDS
// ahead of the update together with A v: no barrier stands between the update and the next product, and with four waves
// (one per vector unit) saying it sixteen times over costs what saying it once does.  The waves past WV wait at the barriers.
// Columns that are through are left out sixteen at a time.  Seven problems of 16 / 32 / 64 / 72 / 96 / 128 sequences, against
// the matrix in LDS with two barriers per column: 65 / 118 / 248 / 365 / 525 / 856 us -> 57 / 93 / 177 / 300 / 380 / 656,
// with the merges as they were then.
//   pbuf, rbuf (two of 16 NE each, by the column's parity): tau A v, and row k + 1 as column k finds it
//   A: row k receives v_k, which the updates read by row and the back-transformation later
// Rounding: v_i w_j + w_i v_j is formed from two rounded products, so (i, j) and (j, i) stay the same bits, and so do the
// copies of a row that different lanes form.
template <int NE, int RN, int WV>
__device__ __forceinline__ void tridiagonalise(double* A, int lda, int n, double* d, double* e, double* htau, double* pbuf,
                                               double* rbuf) {
  constexpr int M = 16 * NE, GR = 4 * WV;                    // rows in all; rows held side by side
  static_assert(NE <= 8 && GR * RN == M, "the waves hold the matrix");
  const int tid = threadIdx.x, sub = tid & 15, g = tid >> 4;
  const bool worker = __builtin_amdgcn_readfirstlane(tid >> 6) < WV;
  double x[RN][NE], v[NE];
  double tk = 0.0, v0 = 0.0;
  // v, tau and v's first element of column k, 16 T0 <= k < 16 T0 + 16, from row k
  auto reflector = [&](auto t0_c, const double (&a)[NE], int k) __attribute__((always_inline)) {
    constexpr int T0 = decltype(t0_c)::value;
    double sig = 0.0;
#pragma unroll
    for (int t = T0; t < NE; ++t) sig += sub + 16 * t > k + 1 ? a[t] * a[t] : 0.0;
    const double diag = lane_value(a[T0], k & 15);
    double x0 = lane_value(a[T0], (k + 1) & 15);
    if constexpr (T0 + 1 < NE) {
      const double y = lane_value(a[T0 + 1], 0);             // not left to an index into the row's registers
      x0 = (k & 15) == 15 ? y : x0;
    }
    sig = row_sum(sig);
    const bool reduced = sig < kNoSquare;                    // column already reduced
    const double nrm = quick_sqrt(x0 * x0 + sig);
    const double alpha = x0 > 0.0 ? -nrm : nrm;
    v0 = reduced ? 0.0 : x0 - alpha;
    tk = reduced ? 0.0 : 2.0 * quick_rcp(v0 * v0 + sig);
#pragma unroll
    for (int t = T0; t < NE; ++t) {
      const int j = sub + 16 * t;
      v[t] = j < k + 1 || reduced ? 0.0 : (j == k + 1 ? v0 : a[t]);
    }
    if (g == 0) {
      if (sub == 0) { d[k] = diag; e[k] = reduced ? x0 : alpha; htau[k] = tk; }
#pragma unroll
      for (int t = T0; t < NE; ++t)
        if (sub + 16 * t < n) A[(size_t)k * lda + sub + 16 * t] = v[t];
    }
  };
  if (worker) {
#pragma unroll
    for (int t = 0; t < NE; ++t) {
      const int j = sub + 16 * t;
      v[t] = j < n ? A[j] : 0.0;
#pragma unroll
      for (int r = 0; r < RN; ++r) x[r][t] = j < n && g + GR * r < n ? A[(size_t)(g + GR * r) * lda + j] : 0.0;
    }
  }
  __syncthreads();
  if (worker) {
    double a[NE];
#pragma unroll
    for (int t = 0; t < NE; ++t) a[t] = v[t];
    reflector(std::integral_constant<int, 0>{}, a, 0);
  }
  auto columns = [&](auto t0_c) __attribute__((always_inline)) {
    constexpr int T0 = decltype(t0_c)::value, R0 = 16 * T0 / GR;
    const int last = 16 * T0 + 14 < n - 3 ? 16 * T0 + 14 : n - 3;
    for (int k = T0 > 0 ? 16 * T0 - 1 : 0; k <= last; ++k) {  // columns k + 1 and up are live, so elements 16 T0 and up
      double* p = pbuf + (k & 1) * M;
      double* row = rbuf + (k & 1) * M;
      if (worker) {
#pragma unroll
        for (int r = R0; r < RN; ++r) {
          const int i = g + GR * r;
          double acc = 0.0;
#pragma unroll
          for (int t = T0; t < NE; ++t) acc += x[r][t] * v[t];
          acc = row_sum(acc);
          if (sub == 0) p[i] = i > k ? tk * acc : 0.0;        // rows that are through hold no more than numbers
          if (i == k + 1) {
#pragma unroll
            for (int t = T0; t < NE; ++t) row[sub + 16 * t] = x[r][t];
          }
        }
      }
      __syncthreads();
      if (worker) {
        double wj[NE], a[NE], kk = 0.0;
#pragma unroll
        for (int t = T0; t < NE; ++t) { wj[t] = p[sub + 16 * t]; a[t] = row[sub + 16 * t]; }
        double vi[RN], wi[RN];
#pragma unroll
        for (int r = R0; r < RN; ++r) {
          const int i = g + GR * r;
          wi[r] = p[i];
          vi[r] = i > k && i < n ? A[(size_t)k * lda + i] : 0.0;      // rows beyond n stay zeros
        }
        double w1 = p[k + 1];
        const double v1 = v0;
#pragma unroll
        for (int t = T0; t < NE; ++t) kk += wj[t] * v[t];
        kk = 0.5 * tk * row_sum(kk);
        w1 = __dsub_rn(w1, __dmul_rn(kk, v1));
        double vj[NE];
#pragma unroll
        for (int t = T0; t < NE; ++t) {
          vj[t] = v[t];
          wj[t] = __dsub_rn(wj[t], __dmul_rn(kk, vj[t]));
          a[t] = __dsub_rn(a[t], __dadd_rn(__dmul_rn(v1, wj[t]), __dmul_rn(w1, vj[t])));
        }
#pragma unroll
        for (int r = R0; r < RN; ++r) {
          const double w = __dsub_rn(wi[r], __dmul_rn(kk, vi[r]));
#pragma unroll
          for (int t = T0; t < NE; ++t)
            x[r][t] = __dsub_rn(x[r][t], __dadd_rn(__dmul_rn(vi[r], wj[t]), __dmul_rn(w, vj[t])));
        }
        reflector(t0_c, a, k + 1);                            // of the last two rows: nothing to clear
      }
    }
  };
  columns(std::integral_constant<int, 0>{});
  if constexpr (NE > 1) columns(std::integral_constant<int, 1>{});
  if constexpr (NE > 2) columns(std::integral_constant<int, 2>{});
  if constexpr (NE > 3) columns(std::integral_constant<int, 3>{});
  if constexpr (NE > 4) columns(std::integral_constant<int, 4>{});
  if constexpr (NE > 5) columns(std::integral_constant<int, 5>{});
  if constexpr (NE > 6) columns(std::integral_constant<int, 6>{});
  if constexpr (NE > 7) columns(std::integral_constant<int, 7>{});
  // the last row's diagonal element
  if (worker) {
#pragma unroll
    for (int r = 0; r < RN; ++r)
#pragma unroll
      for (int t = 0; t < NE; ++t)
        if (g + GR * r == n - 1 && sub + 16 * t == n - 1) d[n - 1] = x[r][t];
  }
  __syncthreads();
}

// Four waves per vector unit: with the 144 registers that 512 threads would be given a compute unit holds one workgroup, and a batch of
// more problems than units takes two rounds (300 of 16 / 32 sequences 82 / 134 us against 51 / 87).  1024 threads have 128 either way,
// of which 16 .. 28 bytes a lane go to scratch.
template <int THREADS, int MAXN, bool LDS, bool QLDS>
__global__ __launch_bounds__(THREADS, 4) void divide_eigh_kernel(const float* __restrict__ Kb, int m,
                                                              double* __restrict__ Db, double* __restrict__ Ub,
                                                              int32_t* __restrict__ infob, double* __restrict__ wsb,
                                                              size_t ws_stride, int root_steps) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ double d[MAXN], e[MAXN], htau[MAXN], v[2 * MAXN], w[MAXN];      // v: this column's and the next one's
  __shared__ double ds[MAXN], zs[MAXN], dk[MAXN], zk[MAXN], zh[MAXN], rtau[MAXN];
  __shared__ short perm[MAXN], list[MAXN], org[MAXN], rot_a[MAXN], rot_b[MAXN];
  __shared__ short n_live[MAXN], n_rot[MAXN], scan[MAXN];       // per block, at its first index
  __shared__ double red[THREADS / 64];
  __shared__ double tri_rows[LDS ? 2 * MAXN : 1];
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid & 15;
  constexpr int WAVES = THREADS / 64;
  const size_t prob = blockIdx.x;        // one problem per workgroup
  const float* K = Kb + prob * m * m;
  double* D = Db + prob * m;
  double* U = Ub + prob * m * m;
  int32_t* info = infob ? infob + prob : nullptr;
  const int n = m;
  const int lda = LDS ? eigh_pitch(m) : m, ldq = QLDS ? lda : m;
  double* A = LDS ? reinterpret_cast<double*>(smem_raw) : U;
  double* Qt = QLDS ? A + (size_t)m * lda : wsb + prob * ws_stride;
  double* Qnext = Qt + (size_t)m * ldq;
  const int group = tid >> 4;            // sixteen lanes, which work on a row of a matrix together
  constexpr int GROUPS = THREADS / 16;

  // symmetrised, scaled copy
  double amax = 0.0;
  for (int j = lane; j < n; j += 64)
#pragma unroll 4
    for (int i = wave; i < n; i += WAVES) {
      const double a = 0.5 * ((double)K[(size_t)i * n + j] + (double)K[(size_t)j * n + i]);
      A[(size_t)i * lda + j] = a;
      Qt[(size_t)i * ldq + j] = i == j ? 1.0 : 0.0;
      Qnext[(size_t)i * ldq + j] = 0.0;  // elements outside a vector's block are never written
      const double aa = fabs(a);
      amax = aa > amax ? aa : amax;      // a NaN never wins; it is found in the tridiagonal matrix
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { const double t = __shfl_xor(amax, o); amax = t > amax ? t : amax; }
  if (lane == 0) red[wave] = amax;
  if (tid == 0) bad = 0;
  __syncthreads();
  amax = 0.0;
#pragma unroll
  for (int q = 0; q < WAVES; ++q) amax = red[q] > amax ? red[q] : amax;
  int expo = 0;
  if (amax > 0.0 && amax < 1.7e308) (void)frexp(amax, &expo);
  const double down = scalbn(1.0, 1 - expo), up = scalbn(1.0, expo - 1);
  for (int i = wave; i < n; i += WAVES)
    for (int j = lane; j < n; j += 64) A[(size_t)i * lda + j] *= down;      // the elements this thread wrote
  __syncthreads();

  if constexpr (LDS) {
    // four waves, up to 96 sequences eight; past them a lane's registers hold eight elements of two rows, so sixteen
    if constexpr (THREADS == 512) tridiagonalise<2, 2, 4>(A, lda, n, d, e, htau, v, tri_rows);        // up to 32 sequences
    else if constexpr (MAXN == 64) tridiagonalise<4, 4, 4>(A, lda, n, d, e, htau, v, tri_rows);
    else if (n <= 96) tridiagonalise<6, 3, 8>(A, lda, n, d, e, htau, v, tri_rows);
    else tridiagonalise<8, 2, 16>(A, lda, n, d, e, htau, v, tri_rows);
  } else {
    // ---- tridiagonalisation: two barriers per column, sixteen lanes per row ----
    // The reflector of column k from row k of the (symmetric) matrix, by the sixteen lanes that hold the row (lane `sub` its
    // elements k + sub + 16 t): sig the sum of squares behind element k + 1, x0 that element, diag element k.
    auto reflector = [&](int k, double sig, double x0, double diag) {
      double* vk = v + (k & 1) * MAXN;
      if (sub == 0) d[k] = diag;
      if (sig < kNoSquare) {                                    // column already reduced
        if (sub == 0) { e[k] = x0; htau[k] = 0.0; }
        return;
      }
      const double nrm = quick_sqrt(x0 * x0 + sig);
      const double alpha = x0 > 0.0 ? -nrm : nrm;
      const double v0 = x0 - alpha;
      if (sub == 0) { e[k] = alpha; htau[k] = 2.0 * quick_rcp(v0 * v0 + sig); }
      for (int j = k + sub; j < n; j += 16) {
        if (j == k) continue;
        double* a = A + (size_t)k * lda + j;                    // kept there for the back-transformation
        const double vj = j == k + 1 ? v0 : *a;
        vk[j] = vj;
        *a = vj;
      }
    };
    if (group == 0 && n > 2) {
      double sig = 0.0, x0 = 0.0, diag = 0.0;
      for (int j = sub; j < n; j += 16) {
        const double x = A[j];
        if (j == 0) diag = x;
        else if (j == 1) x0 = x;
        else sig += x * x;
      }
      reflector(0, row_sum(sig), __shfl(x0, 1, 16), diag);
    }
    __syncthreads();
    for (int k = 0; k + 2 < n; ++k) {
      const double tk = htau[k];
      const double* vk = v + (k & 1) * MAXN;
      if (tk != 0.0) {                                          // uniform
        // p = tau A22 v
        for (int i = k + 1 + group; i < n; i += GROUPS) {
          const double* row = A + (size_t)i * lda;
          double acc = 0.0;
  #pragma unroll 4
          for (int j = k + 1 + sub; j < n; j += 16) acc += row[j] * vk[j];
          acc = row_sum(acc);
          if (sub == 0) w[i] = tk * acc;
        }
      }
      __syncthreads();
      // every sixteen lanes form p.v by themselves (the same sum in the same order: the same bits), then
      // A22 -= v w^T + w v^T with w = p - (tau/2)(p.v) v formed where it is used; the two products are added
      // before they are subtracted, so (i, j) and (j, i) get the same bits
      double kk = 0.0;
      if (tk != 0.0) {
  #pragma unroll 4
        for (int j = k + 1 + sub; j < n; j += 16) kk += w[j] * vk[j];
        kk = 0.5 * tk * row_sum(kk);
      }
      for (int i = k + 1 + group; i < n; i += GROUPS) {
        const bool next_row = i == k + 1;                       // whose lanes form the next reflector
        if (tk == 0.0 && !next_row) continue;
        const double vi = tk != 0.0 ? vk[i] : 0.0, wi = tk != 0.0 ? __dsub_rn(w[i], __dmul_rn(kk, vi)) : 0.0;
        double* row = A + (size_t)i * lda;
        double sig = 0.0, x0 = 0.0, diag = 0.0;
  #pragma unroll 4
        for (int j = k + 1 + sub; j < n; j += 16) {
          double x = row[j];
          if (tk != 0.0) {
            const double vj = vk[j], wj = __dsub_rn(w[j], __dmul_rn(kk, vj));
            const double p1 = __dmul_rn(vi, wj), p2 = __dmul_rn(wi, vj);
            x = __dsub_rn(x, __dadd_rn(p1, p2));
            row[j] = x;
          }
          if (j == i) diag = x;
          else if (j == i + 1) x0 = x;
          else sig += x * x;                                    // of use in the next row only
        }
        if (next_row && k + 3 < n) reflector(k + 1, row_sum(sig), __shfl(x0, 1, 16), diag);
      }
      __syncthreads();
    }
    if (tid == 0) {
      if (n >= 2) { d[n - 2] = A[(size_t)(n - 2) * lda + n - 2]; e[n - 2] = A[(size_t)(n - 2) * lda + n - 1]; }
      d[n - 1] = A[(size_t)(n - 1) * lda + n - 1];
    }
    __syncthreads();
  }
  double size = 0.0;                                          // of the tridiagonal matrix: largest sum of a row's magnitudes
#pragma unroll 4
  for (int i = lane; i < n; i += 64) {
    const double x = fabs(d[i]) + (i + 1 < n ? fabs(e[i]) : 0.0) + (i > 0 ? fabs(e[i - 1]) : 0.0);
    if (!(x < 1.7e308)) bad = 1;                              // NaN or infinity among the entries of K
    size = fmax(size, x);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) size = fmax(size, __shfl_xor(size, o));
  const double tol = 8.0 * kUlp * size;                       // what the merges may neglect
  __syncthreads();
  if (bad) {                                                  // uniform
    for (int i = tid; i < n; i += THREADS) D[i] = __builtin_nan("");
    for (int el = tid; el < n * n; el += THREADS) U[el] = __builtin_nan("");
    if (info && tid == 0) *info = 1;
    return;
  }

  // ---- divide and conquer ----
  int levels = 0;
  while ((1 << levels) < n) ++levels;
  // Tear the off-diagonal entries between the first level's pairs out, d_i -= |e| on both sides, and solve the pairs (some
  // are single indices) by one rotation each.
  const int pairs = 1 << (levels > 0 ? levels - 1 : 0);
  for (int s = tid; s < pairs; s += THREADS) {
    const int b0 = (int)((long long)s * n / pairs), b2 = (int)((long long)(s + 1) * n / pairs);
    if (b0 == b2) continue;
    double d0 = d[b0] - (b0 > 0 ? fabs(e[b0 - 1]) : 0.0);
    double d1 = d[b2 - 1];
    if (b2 < n) { if (b2 - b0 == 1) d0 -= fabs(e[b2 - 1]); else d1 -= fabs(e[b2 - 1]); }
    if (b2 - b0 == 2) {
      const double x = e[b0];
      if (x != 0.0) {
        // tan of the angle that clears x: the smaller root of t^2 + 2 q t - 1, q = (d1 - d0) / (2 x)
        const double q = (d1 - d0) / (2.0 * x);
        const double t = (q >= 0.0 ? 1.0 : -1.0) / (fabs(q) + sqrt(1.0 + q * q));
        const double c = 1.0 / sqrt(1.0 + t * t), sn = t * c;
        d0 -= t * x;
        d1 += t * x;
        Qt[(size_t)b0 * ldq + b0] = c;        Qt[(size_t)b0 * ldq + b0 + 1] = -sn;
        Qt[(size_t)(b0 + 1) * ldq + b0] = sn; Qt[(size_t)(b0 + 1) * ldq + b0 + 1] = c;
      }
      d[b0 + 1] = d1;
    }
    d[b0] = d0;
  }
  double* const rot_c = v;                                    // the reflectors' vectors are done with
  double* const rot_s = w;
  const float inv_n = 1.0f / (float)n;
  __syncthreads();
  for (int lev = 1; lev < levels; ++lev) {
    // Blocks before the merges of this level.  Their bounds are asked for in every step: by shifts, where 64-bit divisions were
    // a third of a merge.
    const int sh = levels - lev, nb = 1 << sh;
    auto block_of = [&](int i, int& b0, int& b1, int& b2) {
      int s = (int)((float)(i * (nb >> 1)) * inv_n);          // or next to it
      while (((2 * s + 2) * n >> sh) <= i) ++s;
      while ((2 * s * n >> sh) > i) --s;
      b0 = 2 * s * n >> sh;
      b1 = (2 * s + 1) * n >> sh;
      b2 = (2 * s + 2) * n >> sh;
    };
    // z, into sorted order; no scan asked for yet
    for (int i = group; i < n; i += GROUPS) {
      int b0, b1, b2;
      block_of(i, b0, b1, b2);
      const double di = d[i];
      int rank = 0;
      for (int j = b0 + sub; j < b2; j += 16) {
        const double dj = d[j];
        rank += (dj < di || (dj == di && j < i)) ? 1 : 0;
      }
      rank = row_count(rank);
      if (sub == 0) {
        double z = 0.0;
        if (b0 < b1 && b1 < b2)
          z = 0.70710678118654752440 *
              (i < b1 ? Qt[(size_t)i * ldq + b1 - 1] : (e[b1 - 1] < 0.0 ? -1.0 : 1.0) * Qt[(size_t)i * ldq + b1]);
        ds[b0 + rank] = di;
        zs[b0 + rank] = z;
        perm[b0 + rank] = (short)i;
        scan[i] = 0;
        n_rot[i] = 0;
      }
    }
    __syncthreads();
    for (int i = tid; i < n; i += THREADS) {                  // i: a sorted position
      int b0, b1, b2;
      block_of(i, b0, b1, b2);
      const double rho = b0 < b1 && b1 < b2 ? 2.0 * fabs(e[b1 - 1]) : 0.0;
      const double z0 = zs[i];
      bool want = rho * fabs(z0) <= tol;
      if (i + 1 < b2) {
        const double z1 = zs[i + 1];
        want = want || fabs((ds[i + 1] - ds[i]) * z0 * z1) <= tol * (z0 * z0 + z1 * z1);
      }
      if (want) scan[b0] = 1;
      list[i] = (short)i;                                     // nothing deflated
      if (i == b0) n_live[b0] = (short)(b2 - b0);
    }
    __syncthreads();
    for (int i = tid; i < n; i += THREADS) {
      int b0, b1, b2;
      block_of(i, b0, b1, b2);
      if (i != b0 || !scan[b0]) continue;
      const double rho = b0 < b1 && b1 < b2 ? 2.0 * fabs(e[b1 - 1]) : 0.0;
      int live = 0, gone = 0, turns = 0, pend = -1;
      double dp = 0.0, zp = 0.0;                              // the pending position's values
      double dnext = ds[b0], znext = zs[b0];                  // one position ahead
      for (int r = b0; r < b2; ++r) {
        const double dr = dnext, zr = znext;
        if (r + 1 < b2) { dnext = ds[r + 1]; znext = zs[r + 1]; }
        if (rho * fabs(zr) <= tol) { list[b2 - 1 - gone++] = (short)r; continue; }
        if (pend >= 0) {
          const double r2 = zr * zr + zp * zp, t = dr - dp;
          if (fabs(t * zr * zp) <= tol * r2) {
            const double h = sqrt(r2), c = zr / h, s = -zp / h;
            rot_a[b0 + turns] = perm[pend]; rot_b[b0 + turns] = perm[r];
            rot_c[b0 + turns] = c; rot_s[b0 + turns] = s;
            ++turns;
            ds[pend] = dp * c * c + dr * s * s;
            const double moved = dp * s * s + dr * c * c;
            ds[r] = moved; zs[r] = h; zs[pend] = 0.0;
            list[b2 - 1 - gone++] = (short)pend;
            pend = r; dp = moved; zp = h;
            continue;
          }
          list[b0 + live++] = (short)pend;
        }
        pend = r; dp = dr; zp = zr;
      }
      if (pend >= 0) list[b0 + live++] = (short)pend;
      n_live[b0] = (short)live;
      n_rot[b0] = (short)turns;
    }
    __syncthreads();
    // the rotations, in order, thread = element of the vectors; the poles that are left, side by side
    for (int i = tid; i < n; i += THREADS) {
      int b0, b1, b2;
      block_of(i, b0, b1, b2);
      for (int t = 0; t < n_rot[b0]; ++t) {
        double* qa = Qt + (size_t)rot_a[b0 + t] * ldq + i;
        double* qb = Qt + (size_t)rot_b[b0 + t] * ldq + i;
        const double c = rot_c[b0 + t], s = rot_s[b0 + t], xa = *qa, xb = *qb;
        *qa = c * xa + s * xb;
        *qb = c * xb - s * xa;
      }
      dk[i] = ds[list[i]];                                    // deflated ones too, behind the others
      zk[i] = zs[list[i]];
      list[i] = perm[list[i]];                                // from here on: the old vector at sorted position i
    }
    __syncthreads();
    auto roots = [&](auto lanes_c, auto per_c) __attribute__((always_inline)) {
      constexpr int LPR = decltype(lanes_c)::value, PER = decltype(per_c)::value;
      for (int i = tid / LPR; i < n; i += THREADS / LPR) {
        int b0, b1, b2;
        block_of(i, b0, b1, b2);
        const int k = n_live[b0], j = i - b0;
        if (j < k) {
          int o;
          double t;
          if (!secular_root<LPR, PER>(dk + b0, zk + b0, k, 2.0 * fabs(e[b1 - 1]), j, tid % LPR, root_steps, o, t)) bad = 1;
          if (tid % LPR == 0) { org[i] = (short)o; rtau[i] = t; }
        }
      }
    };
    // A merged block holds at most 2 << lev indices.  Few lanes a root, so that every vector unit has one wave or two: what all
    // lanes of a root repeat is issued least often.  64 sequences with this, the bounds by shifts, vectors fetched a step early and
    // U written by way of the LDS: 177 -> 141 us for seven problems, 128: 656 -> 547, 16: 57 -> 43.
    constexpr std::integral_constant<int, 4> c4{};
    constexpr std::integral_constant<int, 8> c8{};
    if constexpr (MAXN > 128) roots(std::integral_constant<int, 16>{}, std::integral_constant<int, 0>{});
    else if (2 << lev <= 16) roots(c4, c4);
    else if (2 << lev <= 32) roots(c4, c8);
    else if (MAXN == 64 || 2 << lev <= 64) roots(c8, c8);
    else roots(c4, std::integral_constant<int, 0>{});
    __syncthreads();
    for (int i = group; i < n; i += GROUPS) {
      int b0, b1, b2;
      block_of(i, b0, b1, b2);
      const int k = n_live[b0], q = i - b0;
      if (q >= k) continue;                                   // uniform over the sixteen lanes
      const double di = dk[i];
      const double* dd = dk + b0;
      double p = 1.0;
      for (int j = sub; j < k; j += 16) {
        const double diff = (dd[org[b0 + j]] - di) + rtau[b0 + j];           // root j - pole q
        p *= j == k - 1 ? diff : diff * quick_rcp((j < q ? dd[j] : dd[j + 1]) - di);
      }
      p = row_product(p);
      if (sub == 0) zh[i] = copysign(sqrt(fabs(p)), zk[i]);
    }
    __syncthreads();
    // New vectors, as a product of matrices in 16x16 tiles: rows u_j (zeros outside j's block, the unit vector for a
    // deflated position) times the old vectors in sorted order.  Lane l supplies row l % 16, column l / 16 of a step of
    // the left factor, which it forms itself, and row l / 16, column l % 16 of the right one.
    {
      typedef double f64x4 __attribute__((ext_vector_type(4)));
      const int nt = (n + 15) / 16, l16 = lane & 15, l4 = lane >> 4;
      for (int tt = wave; tt < nt * nt; tt += WAVES) {
        const int jt = tt / nt * 16, rt = tt % nt * 16;
        int lo, mid, hi, unused;
        block_of(jt, lo, mid, unused);
        block_of(jt + 15 < n ? jt + 15 : n - 1, unused, mid, hi);
        if (rt + 16 <= lo || rt >= hi) continue;
        const int j = jt + l16 < n ? jt + l16 : n - 1, r = rt + l16 < n ? rt + l16 : n - 1;
        int b0, b1, b2;
        block_of(j, b0, b1, b2);
        const int k = n_live[b0];
        const bool live = j - b0 < k;
        const double dorg = live ? dk[b0 + org[j]] : 0.0, t = live ? rtau[j] : 0.0;
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        double s = 0.0;
        // what a step reads is fetched one step early
        double x_next, dk_next, zh_next;
        auto fetch = [&](int i) {
          const int ic = i < n ? i : n - 1;
          x_next = Qt[(size_t)list[ic] * ldq + r];
          dk_next = dk[ic];
          zh_next = zh[ic];
        };
        fetch(lo + l4);
        for (int i0 = lo; i0 < hi; i0 += 4) {
          const int i = i0 + l4;
          const double x = x_next, dki = dk_next, zhi = zh_next;
          fetch(i + 4);
          double u = 0.0;
          if (live) {
            if (i >= b0 && i < b0 + k) u = zhi * quick_rcp((dki - dorg) - t);
          } else {
            u = i == j ? 1.0 : 0.0;
          }
          s += u * u;
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(u, x, acc, 0, 0, 0);
        }
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        const double norm = rsqrt(s);
#pragma unroll
        for (int q = 0; q < 4; ++q) {                         // lane holds rows 4 q + l / 16, column l % 16 of the tile
          const int row = 4 * q + l4;
          const double scale = __shfl(norm, row, 64);
          if (jt + row < n && rt + l16 < n) Qnext[(size_t)(jt + row) * ldq + rt + l16] = acc[q] * scale;
        }
      }
      for (int i = tid; i < n; i += THREADS) {
        int b0, b1, b2;
        block_of(i, b0, b1, b2);
        d[i] = i - b0 < n_live[b0] ? dk[b0 + org[i]] + rtau[i] : dk[i];
      }
    }
    __syncthreads();
    double* const swap = Qt; Qt = Qnext; Qnext = swap;
  }

  // ascending order by rank (ties broken by index)
  for (int i = group; i < n; i += GROUPS) {
    const double di = d[i];
    int rank = 0;
    for (int j = sub; j < n; j += 16) {
      const double dj = d[j];
      rank += (dj < di || (dj == di && j < i)) ? 1 : 0;
    }
    rank = row_count(rank);
    if (sub == 0) {
      D[rank] = di * up;
      perm[rank] = (short)i;
      list[i] = (short)rank;
    }
  }

  // ---- U = H_0 ... H_{n-3} Q^T: sixteen lanes (a wave, past 256 elements) per vector, its elements in registers; past 64
  // sequences two vectors at a time, which share the reflectors' reads (128: with the output below 618 us against 664 for seven problems) ----
  constexpr int VL = MAXN <= 256 ? 16 : 64, NE = MAXN / VL, NV = MAXN == 128 ? 2 : 1, VS = THREADS / VL;
  const int vl = tid % VL;
  for (int i = tid / VL; i < n; i += VS * NV) {
    double x[NV][NE], ahead[NE];                              // ahead: the next reflector's vector, fetched one step early
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
      for (int t = 0; t < NE; ++t)
        x[u][t] = t * VL + vl < n && i + VS * u < n ? Qt[(size_t)(i + VS * u) * ldq + t * VL + vl] : 0.0;
    auto fetch = [&](int k) {
#pragma unroll
      for (int t = 0; t < NE; ++t) {
        const int r = t * VL + vl;
        ahead[t] = k >= 0 && r > k && r < n ? A[(size_t)k * lda + r] : 0.0;
      }
    };
    fetch(n - 3);
    for (int k = n - 3; k >= 0; --k) {
      const double tk = htau[k];
      double vk[NE];
#pragma unroll
      for (int t = 0; t < NE; ++t) vk[t] = ahead[t];
      fetch(k - 1);
      if (tk == 0.0) continue;                                // uniform
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        double dot = 0.0;
#pragma unroll
        for (int t = 0; t < NE; ++t) dot += vk[t] * x[u][t];
        dot = tk * (VL == 16 ? row_sum(dot) : wave_total(dot));
#pragma unroll
        for (int t = 0; t < NE; ++t) x[u][t] -= dot * vk[t];
      }
    }
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
      for (int t = 0; t < NE; ++t)
        if (t * VL + vl < n && i + VS * u < n) Qt[(size_t)(i + VS * u) * ldq + t * VL + vl] = x[u][t];
  }
  __syncthreads();
  // eigenvectors as columns of U, by rank
  if constexpr (LDS) {
    // by way of A's memory, whose reflectors are done with: vectors are read and U is written along rows.  Rows lie n apart,
    // turned by their index where n is even, so that a column's elements lie in different banks.
    auto at = [&](int r, int c) { const int x = c + r; return (size_t)r * n + (n & 1 ? c : (x < n ? x : x - n)); };
    for (int i = wave; i < n; i += WAVES) {
      const int c = list[i];
      for (int r = lane; r < n; r += 64) A[at(r, c)] = Qt[(size_t)i * ldq + r];
    }
    __syncthreads();
#pragma unroll 4
    for (int r = wave; r < n; r += WAVES)
      for (int c = lane; c < n; c += 64) U[(size_t)r * n + c] = A[at(r, c)];
  } else {
    for (int c = lane; c < n; c += 64) {
      const double* q = Qt + (size_t)perm[c] * ldq;
#pragma unroll 4
      for (int r = wave; r < n; r += WAVES) U[(size_t)r * n + c] = q[r];
    }
  }
  if (info && tid == 0) *info = bad;
}

constexpr int kSolveThreads = 1024;

// c[l] = U ((U^T A) / (D + reg_l)) for each regulariser of the sweep.  Latency-bound: every pass over U is spread over the
// waves by rows (a thread that walked a column, and then a row, by itself waited for one load after the other: 48 us at 64
// sequences and three regularisers, 17 now).
__global__ __launch_bounds__(kSolveThreads) void eigh_solve_kernel(EighSolveArgs a) {
  constexpr int WAVES = kSolveThreads / 64;
  __shared__ double y[kEighMaxSeq], f[kEighMaxSeq];
  __shared__ double part[WAVES][64];
  __shared__ double red[WAVES];
  __shared__ double sh_scale;
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = a.n_seq;
  const size_t prob = blockIdx.x;        // one problem per workgroup
  const double* const D = a.D + prob * m;
  const double* const U = a.U + prob * m * m;
  const float* const A = a.A + prob * m;
  float* const c = a.c + prob * a.n_lambda * m;
  float* const ema_state = a.ema_state ? a.ema_state + prob * 2 : nullptr;
  double tr = 0.0;
  for (int j = tid; j < m; j += kSolveThreads) tr += D[j];
  if (tid == 0) bad = 0;
  // y = U^T A: a wave takes every sixteenth row, lanes along the row
  for (int j0 = 0; j0 < m; j0 += 64) {
    const int j = j0 + lane < m ? j0 + lane : m - 1;
    double s = 0.0;
#pragma unroll 4
    for (int i = wave; i < m; i += WAVES) s += U[(size_t)i * m + j] * (double)A[i];
    part[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && j0 + lane < m) {
      s = 0.0;
#pragma unroll
      for (int q = 0; q < WAVES; ++q) s += part[q][lane];
      y[j] = s;
    }
    __syncthreads();
  }
  const double mean_d = block_sum<kSolveThreads>(tr, red) / (double)m;
  if (tid == 0) {
    double scale = 1.0;                                   // ABSOLUTE
    if (a.reg_mode == 1) scale = mean_d;                  // this batch's mean eigenvalue
    if (a.reg_mode == 2) {                                // trailing mean over minibatches, this one included
      const double prev = (double)ema_state[0];
      const bool first = ema_state[1] == 0.f;
      scale = first ? mean_d : (double)a.ema_decay * prev + (1.0 - (double)a.ema_decay) * mean_d;
      ema_state[0] = (float)scale;
      ema_state[1] = ema_state[1] + 1.f;
    }
    sh_scale = scale;
  }
  __syncthreads();
  const double scale = sh_scale;
  for (int l = 0; l < a.n_lambda; ++l) {
    const double reg = (double)a.lambdas[l] * scale;
    for (int j = tid; j < m; j += kSolveThreads) {
      const double den = D[j] + reg;
      f[j] = den > 0.0 ? y[j] / den : 0.0;
      if (!(den > 0.0)) atomicAdd(&bad, 1);
    }
    __syncthreads();
    // a wave takes four rows at a time
    for (int i0 = wave * 4; i0 < m; i0 += WAVES * 4) {
      double s[4] = {0.0, 0.0, 0.0, 0.0};
      for (int j = lane; j < m; j += 64) {
        const double fj = f[j];
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] += U[(size_t)(i0 + q < m ? i0 + q : m - 1) * m + j] * fj;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double t = wave_total(s[q]);
        if (lane == 0 && i0 + q < m) c[(size_t)l * m + i0 + q] = (float)t;
      }
    }
    __syncthreads();
  }
  if (a.info && tid == 0) a.info[prob] = bad;
}

}  // namespace

size_t eigh_workspace(int m) {
  const int n = (m + 1) & ~1;
  return 2 * (size_t)n * (n + 1) * sizeof(double);
}

template <int THREADS, int MAXN, bool LDS, bool QLDS>
hipError_t launch_divide(const float* K, int m, int batch, double* D, double* U, int32_t* info, double* ws,
                         size_t ws_stride, int root_steps, hipStream_t s) {
  auto kern = divide_eigh_kernel<THREADS, MAXN, LDS, QLDS>;
  constexpr int matrices = LDS ? (QLDS ? 3 : 1) : 0;
  // eigh_pitch lets no single matrix grow past 128 x 128; 64 x 80 is the largest of three
  constexpr size_t most = (size_t)(QLDS ? matrices * 64 * 80 : matrices * 128 * 128) * sizeof(double);
  // once per process (static initialisation is thread-safe); a failure is returned by every call
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(batch), dim3(THREADS), (size_t)matrices * m * eigh_pitch(m) * sizeof(double), s, K, m, D, U, info, ws,
                     ws_stride, root_steps);
  return hipGetLastError();
}

hipError_t launch_ntk_eigh(const float* K, int m, int batch, double* D, double* U, int32_t* info, void* workspace,
                           hipStream_t s, int root_steps) {
  double* ws = static_cast<double*>(workspace);
  const size_t ws_stride = eigh_workspace(m) / sizeof(double);      // doubles per problem
  // where the matrices lie follows from what fits the LDS; 512 threads up to 32 sequences, 1024 above (64: 243 us against 289)
  if (m <= 32) return launch_divide<512, 64, true, true>(K, m, batch, D, U, info, ws, ws_stride, root_steps, s);
  if (m <= 64) return launch_divide<1024, 64, true, true>(K, m, batch, D, U, info, ws, ws_stride, root_steps, s);
  if (m <= 128) return launch_divide<1024, 128, true, false>(K, m, batch, D, U, info, ws, ws_stride, root_steps, s);
  if (m <= 256) return launch_divide<1024, 256, false, false>(K, m, batch, D, U, info, ws, ws_stride, root_steps, s);
  return launch_divide<1024, kEighMaxSeq, false, false>(K, m, batch, D, U, info, ws, ws_stride, root_steps, s);
}

hipError_t launch_eigh_solve(const EighSolveArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(eigh_solve_kernel, dim3(a.batch), dim3(kSolveThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace isopo
