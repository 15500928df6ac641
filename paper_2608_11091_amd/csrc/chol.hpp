// Right-looking Cholesky steps of a symmetric matrix of order m <= 64: eight
// waves hold the rows in registers, a ninth reduces the panels.
#pragma once

#include "common.hpp"

namespace tk {

constexpr int kCholPanel = 8;               // rows of a panel, and waves that hold rows
constexpr int kCholWaves = kCholPanel + 1;  // waves that call chol_rows
constexpr int kCholRows = kWave / kCholPanel;

template <typename T>
struct CholShared {
  T in[kCholPanel][kWave];      // the rows of the next panel
  T row[2][kCholPanel][kWave];  // a reduced panel and its rows / pivot
  T f[2][kCholPanel][kWave];
  int stop;
};

// Wave w < 8 holds the rows w, w + 8, .. (a[r] = entry (w + 8 r, lane)); entries
// left of the diagonal are not used.  Step k reads row k and updates every
// later row i:
//   A[i][j] -= A[k][i] (A[k][j] / pivot).
// scale(k, A[k][k], A[k][j], f), called by the ninth wave, sets f to A[k][j] /
// pivot (0: a dead column, nothing is updated) and returns whether to go on;
// chol_rows returns false in every thread when it was told not to.  retire(k, a)
// gets row k in wave k % 8.  All nine waves call it; other waves
// must have left the kernel.
//
// A serial chain of m divisions, so what counts is what else is on it.  The
// ninth wave reduces a panel of eight rows by itself (0.1 us a step: pivot
// through a scalar register, division, multiply-add) and leaves it in LDS; the
// others apply its eight steps to the row of theirs that the next panel needs,
// hand that over, and update the rest beside the next panel.  Every entry sees
// the same operations in the same order as one step at a time.  At order 53, FP64:
// 9.2 us (17.5 us with the panel reduced by every wave for itself and one
// barrier a panel, whose eight copies share the SIMDs).
template <typename T, typename Scale, typename Retire>
__device__ __forceinline__ bool chol_rows(T (&a)[kCholRows], int m, int lane, int w, CholShared<T>& sh,
                                          Scale&& scale, Retire&& retire) {
  constexpr int W = kCholPanel;
  if (w < W) sh.in[w][lane] = a[0];
  if (w == W && lane == 0) sh.stop = 0;
  __syncthreads();
  for (int k0 = 0, buf = 0; k0 < m; k0 += W, buf ^= 1) {
    if (w == W) {
      T r[W];
#pragma unroll
      for (int p = 0; p < W; ++p) r[p] = sh.in[p][lane];
      bool stop = false;
#pragma unroll
      for (int q = 0; q < W; ++q) {
        const int k = k0 + q;
        if (k < m) {
          const T pv = rdlane(r[q], k);
          T s[W];
#pragma unroll
          for (int p = 0; p < W; ++p)
            if (p > q) s[p] = rdlane(r[q], k0 + p);
          T f;
          stop |= !scale(k, pv, r[q], f);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int p = 0; p < W; ++p)
            if (p > q) r[p] = fma(-s[p], f, r[p]);
          sh.row[buf][q][lane] = r[q];
          sh.f[buf][q][lane] = f;
        }
      }
      if (stop && lane == 0) sh.stop = 1;
    }
    __syncthreads();
    if (sh.stop != 0) return false;
    if (w < W) {
      const int np = min(W, m - k0);
      if (w < np) retire(k0 + w, sh.row[buf][w][lane]);
#pragma unroll
      for (int i = 0; i + 1 < kCholRows; ++i) a[i] = a[i + 1];
    }
    if (k0 + W >= m) break;
    // a whole panel is behind (only the last can be short)
    T f[W];
    if (w < W) {
      T s[W];
#pragma unroll
      for (int q = 0; q < W; ++q) {
        f[q] = sh.f[buf][q][lane];
        s[q] = sh.row[buf][q][k0 + W + w];
      }
#pragma unroll
      for (int q = 0; q < W; ++q) a[0] = fma(-s[q], f[q], a[0]);
      sh.in[w][lane] = a[0];
    }
    __syncthreads();
    if (w < W) {
      const int live = (m - k0 - W - w + W - 1) / W;  // rows k0 + 8 + w + 8 i below m
#pragma unroll
      for (int i = 1; i < kCholRows; ++i)
        if (i < live) {
          T s[W];
#pragma unroll
          for (int q = 0; q < W; ++q) s[q] = sh.row[buf][q][k0 + W + w + W * i];
#pragma unroll
          for (int q = 0; q < W; ++q) a[i] = fma(-s[q], f[q], a[i]);
        }
    }
  }
  return true;
}

}  // namespace tk
