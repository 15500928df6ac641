// Right-looking Cholesky steps of a symmetric matrix of order m <= 64 held in
// the registers of eight waves.
#pragma once

#include "common.hpp"

namespace tk {

constexpr int kCholWaves = 8;
constexpr int kCholRows = kWave / kCholWaves;  // rows of a wave

// Wave w holds the rows w, w + W, .. (W waves; a[r] = entry (w + W r, lane));
// entries left of the diagonal are not used.  Step k reads row k and updates
// every later row i:
//   A[i][j] -= A[k][i] (A[k][j] / pivot).
// pivot(k, A[k][k]) says what to do: > 0 update, 0 skip the update (a dead
// column), < 0 stop (the same in every thread; chol_rows then returns false).
// retire(k, a) gets row k in its wave.  row_s: LDS for two panels.  All W waves
// call it; other waves must have left the kernel.
//
// A serial chain of m divisions.  The W rows of a panel are published at once
// and every wave reduces them for itself, so there is one LDS exchange and one
// barrier a panel; each wave then applies the panel's steps to its own rows.
// Every entry sees the same operations in the same order as one step at a
// time.  The multipliers A[k][i] come from the row's lanes through scalar
// registers, read ahead of their uses.  At order 48 a step takes
// 0.31 us (0.35 us with an exchange a step, 0.66 us with the matrix in
// LDS and 4 waves, whose update read two operands and wrote one there for
// every multiply-add).
template <typename Pivot, typename Retire>
__device__ __forceinline__ bool chol_rows(double (&a)[kCholRows], int m, int lane, int w,
                                          double (*row_s)[kCholWaves][kWave], Pivot&& pivot, Retire&& retire) {
  constexpr int W = kCholWaves;
  for (int k0 = 0, buf = 0; k0 < m; k0 += W, buf ^= 1) {
    row_s[buf][w][lane] = a[0];
    __syncthreads();
    double r[W], f[W];
#pragma unroll
    for (int p = 0; p < W; ++p) r[p] = row_s[buf][p][lane];
    int acts = 0;  // steps that update
#pragma unroll
    for (int q = 0; q < W; ++q) {
      const int k = k0 + q;
      if (k < m) {
        const double pv = rdlane(r[q], k);
        const int act = pivot(k, pv);
        if (act < 0) return false;
        if (w == q) retire(k, r[q]);
        if (act) {
          acts |= 1 << q;
          double s[W];
#pragma unroll
          for (int p = 0; p < W; ++p)
            if (p > q) s[p] = rdlane(r[q], k0 + p);
          f[q] = r[q] / pv;
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int p = 0; p < W; ++p)
            if (p > q) r[p] = fma(-s[p], f[q], r[p]);
        }
      }
    }
    const int live = (m - k0 - w + W - 1) / W;  // rows k0 + w + W i below m
#pragma unroll
    for (int q = 0; q < W; ++q) {
      if (!(acts >> q & 1)) continue;
#pragma unroll
      for (int g = 1; g < kCholRows; g += 4) {
        if (g >= live) continue;
        double s[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (g + u < kCholRows) s[u] = rdlane(r[q], k0 + w + W * (g + u));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (g + u < kCholRows) a[g + u] = fma(-s[u], f[q], a[g + u]);
      }
    }
#pragma unroll
    for (int i = 0; i + 1 < kCholRows; ++i) a[i] = a[i + 1];
  }
  return true;
}

}  // namespace tk
