// Small dense factorisations of the hot path, one workgroup per matrix:
// Householder QR (plain and column-pivoted with a rank cut) of tall-skinny
// FP64 matrices, the Cholesky factor of a small Gram, and the row-wise
// triangular solve that turns a Gram's Cholesky factor into a basis.
// Everything is deterministic: no atomics, fixed reduction orders.
#include <algorithm>
#include <cfloat>

#include "chol.hpp"
#include "kernels.hpp"

namespace tk {

namespace {

// ---------------------------------------------------------------- Householder QR
// Lane c of every wave owns column c (c < 64) and wave w holds rows
// [RS w, RS w + RS) of it in registers.  The pivot column's entries on a
// wave's rows are read across lanes (v_readlane) into scalar registers and
// enter the dot products and the updates as scalar operands, so a reflector
// never goes through LDS; it stays unscaled, v = (1, scal * x), and the scale
// is folded into the coefficients.  Before step j, row j of all columns leaves
// the registers for LDS (zeros take its place), where it becomes row j of R;
// in columns chosen earlier it holds their reflectors' entries.  Dot products,
// updates and norms then run over all rows of the registers without a test on
// the diagonal.  Sums over rows are in-thread plus one fixed-order pass over
// the waves' partials in LDS; every wave derives the pivot and the reflector
// from the same partials, so a factorisation step needs two barriers and a Q
// step one.
//
// Bound by latency: one dependent chain a step, at about 6 cycles an
// instruction where one wave has a SIMD to itself, so the rows are spread
// over four waves first (16 or 32 rows each) and over eight above 128 rows.
// Measured, three matrices a launch (in brackets the form that handed the
// reflector over through LDS and tested every row against the diagonal):
// pivoted 96 x 48 with Q 123 us (205), plain 48 x 48 with Q 78 (176); averages
// over solves, whose first iterations have lower ranks: R only 256 x 32 58 (79),
// R only 512 x 48 140 (172), pivoted 512 x 48 with Q 290 (771).
constexpr int QC_MAXROWS = 512;
constexpr int QC_V = 16;  // rows per register vector (indexed at run time by the retired row)
typedef double QcVec __attribute__((ext_vector_type(QC_V)));

struct QrJob {
  const double* Y;
  const double* ref;
  double* Q;
  double* R;
  double* Rt;
  int* rank_out;
  int m;
};
__device__ __forceinline__ QrJob job_of(const QrTask& t, int cap, const int* m_dev) {
  QrJob j{t.Y, nullptr, t.Q, t.R, nullptr, nullptr, 0};
  j.m = t.m ? *t.m : (m_dev ? *m_dev : cap);
  return j;
}
__device__ __forceinline__ QrJob job_of(const QrPivTask& t, int cap, const int*) {
  QrJob j{t.Y, t.ref, t.Q, t.R, t.Rt, t.rank_out, 0};
  j.m = t.m ? *t.m : cap;
  return j;
}

// Sum of part[q][c] over the NW waves in fixed order (every wave gets the
// same result).
template <int NW>
__device__ __forceinline__ double wave_partials_sum(const double (*part)[kWave], int c) {
  double s0 = part[0][c], s1 = part[1][c];
#pragma unroll
  for (int q = 2; q < NW; q += 2) {
    s0 += part[q][c];
    s1 += part[q + 1][c];
  }
  return s0 + s1;
}

// Householder vector of a column with leading entry alpha, squared norm xx
// (over the rows from the diagonal down) and squared norm `below` of the part
// below the diagonal: beta = -sign(alpha) ||x||, tau = (beta - alpha) / beta,
// v = (1, scal * x_below); tau = scal = 0 where nothing stands below the
// diagonal.  (Whether xx exceeds alpha^2 does not tell: a part of up to 1e-8
// of the diagonal is lost in the sum.)
struct Reflector {
  double beta, tau, scal;
};
__device__ __forceinline__ Reflector reflector(double alpha, double xx, double below) {
  const bool some = below > 0.0;
  const double aa = fabs(alpha);
  const double nrm = sqrt(some ? xx : 1.0);
  Reflector r;
  r.beta = some ? -copysign(nrm, alpha) : alpha;
  r.tau = some ? 1.0 + aa / nrm : 0.0;
  r.scal = some ? copysign(1.0 / (aa + nrm), alpha) : 0.0;
  return r;
}

// PIV = false: plain Householder QR of the leading m columns (m from the task,
// else m_dev, else cap).  PIV = true: column pivoting by the largest remaining
// norm relative to the column's reference norm (or to the largest input
// column when the task has no reference; the largest to 17 bits, ties to the
// lowest column) and a stop once that ratio is at or below drop_tol; R[j][c]
// is then the coefficient of input column c on basis column j.  NW waves of RS
// rows cover n.
template <bool PIV, typename Task, int RS, int NW>
__global__ __launch_bounds__(NW* kWave) void qr_cols_kernel(const Task* __restrict__ tasks, int n, int cap,
                                                             double drop_tol, const int* __restrict__ m_dev) {
  static_assert(NW * RS <= QC_MAXROWS && RS % QC_V == 0 && RS <= 4 * QC_V && NW % 2 == 0, "row blocks");
  constexpr int NV = RS / QC_V;
  __shared__ double rows[kWave + 1][kWave];  // retired rows: R, and reflector entries of columns chosen earlier
  __shared__ double pn1[NW][kWave];          // per-wave sums of squares over the rows in registers
  __shared__ double pw[2][NW][kWave];        // per-wave partials of x^T A
  __shared__ double tau_s[kWave], scal_s[kWave];
  __shared__ int piv_s[kWave];
  __shared__ int step_of[kWave];
  const QrJob jb = job_of(tasks[blockIdx.x], cap, m_dev);
  const int tid = threadIdx.x;
  const int c = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform: row tests stay scalar
  const int r0 = w * RS;
  const int m = __builtin_amdgcn_readfirstlane(max(0, min(jb.m, cap)));
  const int kmax = min(m, n);

  // unconditional loads at clamped indices (always inside the n x cap input),
  // masked afterwards: no per-row branches whose conditions stay live
  const int cl = min(c, cap - 1);
  const bool colin = c < m;
  QcVec a[NV];
  double sref = 0.0;  // this thread's share of the squared reference norm
  {
    const GPtr<double> gy = (GPtr<double>)jb.Y + (size_t)cl * n;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
#pragma unroll
      for (int i = 0; i < QC_V; ++i) a[v][i] = gy[min(r0 + v * QC_V + i, n - 1)];
    }
    const double one = colin ? 1.0 : 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int i = 0; i < QC_V; ++i) a[v][i] = r0 + v * QC_V + i < n ? (one != 0.0 ? a[v][i] : 0.0) : 0.0;
  }
  if (PIV) {
    if (jb.ref == nullptr) {
      // global cut: the reference columns are the input itself
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int i = 0; i < QC_V; ++i) sref = fma(a[v][i], a[v][i], sref);
    } else {
      // reference columns read a part at a time, so that their loads do not
      // all hold registers beside the input's
      const GPtr<double> gr = (GPtr<double>)jb.ref + (size_t)cl * n;
#pragma unroll
      for (int q = 0; q < RS; q += 8) {
#pragma unroll
        for (int i = q; i < q + 8; ++i) {
          const double v = gr[min(r0 + i, n - 1)];
          sref += (colin && r0 + i < n) ? v * v : 0.0;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // Replaces row `row` x of the registers by next(x) in the wave that holds it.
  // The register index is a run-time scalar; every wave writes some register
  // back (control flow around such a write copies the whole vector).
  auto swap_row = [&](int row, auto next) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int t = row - r0 - v * QC_V;
      const bool in = t >= 0 && t < QC_V;
      const int i = in ? t : 0;
      const double x = a[v][i];
      a[v][i] = in ? next(x) : x;
    }
  };
  auto retire = [&](int row) {
    double x = 0.0;
    swap_row(row, [&](double out) {
      x = out;
      return 0.0;
    });
    if (row >= r0 && row < r0 + RS) rows[row][c] = x;
  };
  auto norm_partial = [&]() {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int i = 0; i < QC_V; i += 2) {
        s0 = fma(a[v][i], a[v][i], s0);
        s1 = fma(a[v][i + 1], a[v][i + 1], s1);
      }
    pn1[w][c] = s0 + s1;
  };
  // the pivot column's entries, all reads before their uses (a read right
  // before its use stalls)
  auto column = [&](int v, int p, double (&x)[QC_V]) {
#pragma unroll
    for (int i = 0; i < QC_V; ++i) x[i] = rdlane(a[v][i], p);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto column_dot = [&](int p) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double x[QC_V];
      column(v, p, x);
#pragma unroll
      for (int i = 0; i < QC_V; i += 2) {
        s0 = fma(x[i], a[v][i], s0);
        s1 = fma(x[i + 1], a[v][i + 1], s1);
      }
    }
    return s0 + s1;
  };
  // The update reads the column again where, kept from the dot product, it
  // would not fit the scalar registers.
  auto reread = [&](int p) {
    if (RS > QC_V) asm volatile("" : "+s"(p));
    return p;
  };
  if (PIV) pw[1][w][c] = sref;
  if (tid < kWave) step_of[tid] = -1;
  retire(0);
  norm_partial();
  __syncthreads();
  double iref = 1.0;  // 1 / squared reference norm (0: the column is never chosen)
  if (PIV) {
    double t = wave_partials_sum<NW>(pw[1], c);
    if (jb.ref == nullptr) t = wave_max(t);  // global cut: against the largest input column
    iref = t > 0.0 ? 1.0 / t : 0.0;
  }

  // ---------------- factorisation
  bool alive = colin;  // this lane's column is still unchosen
  int nlive = 0;
  int nret = 1;        // retired rows
  for (int j = 0; j < kmax; ++j) {
    const double rj = rows[j][c];
    const double below = wave_partials_sum<NW>(pn1, c);
    const double n1 = fma(rj, rj, below);
    int p = j;
    if (PIV) {
      const double rel = n1 * iref;
      // false for NaN as well: every wave takes the same decision
      const bool cand = alive && rel > 0.0;
      const unsigned bits = __float_as_uint(fminf(float(rel), FLT_MAX));
      const unsigned key = wave_umax(cand ? 0x80000000u | (bits & ~63u) | unsigned(63 - c) : 0u);
      p = 63 - int(key & 63u);
      if (key == 0u || !(rdlane(rel, p) > drop_tol * drop_tol)) break;
    }
    pw[0][w][c] = column_dot(p);
    const Reflector rf = reflector(rdlane(rj, p), rdlane(n1, p), rdlane(below, p));
    if (tid == 0) {
      tau_s[j] = rf.tau;
      scal_s[j] = rf.scal;
      piv_s[j] = p;
    }
    alive = alive && c != p;
    __syncthreads();
    // w_c = v^T a_c; the other columns take a - tau w_c v
    const double wc = fma(rf.scal, wave_partials_sum<NW>(pw[0], c), rj);
    const double tw = alive ? rf.tau * wc : 0.0;
    const double mul = -tw * rf.scal;
    if (w == 0) rows[j][c] = c == p ? rf.beta : rj - tw;
    const int pu = reread(p);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double x[QC_V];
      column(v, pu, x);
#pragma unroll
      for (int i = 0; i < QC_V; ++i) a[v][i] = fma(mul, x[i], a[v][i]);
    }
    nlive = j + 1;
    if (j + 1 < kmax) {
      retire(j + 1);
      nret = j + 2;
    }
    norm_partial();
    __syncthreads();
  }
  nlive = __builtin_amdgcn_readfirstlane(nlive);
  nret = __builtin_amdgcn_readfirstlane(nret);
  if (tid < nlive) step_of[piv_s[tid]] = tid;
  __syncthreads();
  const int jj = step_of[c];

  // ---------------- R (and its transpose)
  if (jb.R != nullptr || jb.Rt != nullptr) {
    for (int row = w; row < cap; row += NW) {
      if (c < cap) {
        const bool ok = row < nlive && c < m && (PIV ? (jj < 0 || jj >= row) : c >= row);
        const double val = ok ? rows[ok ? row : 0][c] : 0.0;
        if (jb.R) jb.R[row + (size_t)c * cap] = val;
        if (jb.Rt) jb.Rt[c + (size_t)row * cap] = val;
      }
    }
  }
  if (jb.rank_out != nullptr && tid == 0) *jb.rank_out = nlive;

  // ---------------- Q by backward accumulation; basis column j sits in column piv[j]
  if (jb.Q == nullptr) return;  // R only (uniform over the block)
  // the reflectors' entries on the retired rows come back, zeros from the
  // diagonal up
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int i = 0; i < QC_V; ++i) {
      const int row = r0 + v * QC_V + i;
      if (row < nret) {
        const double x = rows[row][c];
        a[v][i] = (jj >= 0 && jj < row) ? x : 0.0;
      }
    }
  bool later = false;  // this lane's column already holds a finished basis column
  for (int j = nlive - 1; j >= 0; --j) {
    const int p = __builtin_amdgcn_readfirstlane(piv_s[j]);
    const double tau = tau_s[j], scal = scal_s[j];
    const int b = j & 1;
    pw[b][w][c] = column_dot(p);
    __syncthreads();
    // column p becomes basis column j: 0 above row j, 1 - tau at row j,
    // -tau v below; the finished columns, zero at row j, take a - tau w_c v
    const bool own = c == p;
    const double tw = later ? tau * (scal * wave_partials_sum<NW>(pw[b], c)) : 0.0;
    const double mul = (own ? -tau : -tw) * scal;
    const double keep = own ? 0.0 : 1.0;
    const int pu = reread(p);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double x[QC_V];
      column(v, pu, x);
#pragma unroll
      for (int i = 0; i < QC_V; ++i) a[v][i] = fma(mul, x[i], keep * a[v][i]);
    }
    swap_row(j, [&](double out) { return own ? 1.0 - tau : (later ? -tw : out); });
    later = later || own;
  }
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int i = 0; i < QC_V; ++i) {
      const int row = r0 + v * QC_V + i;
      if (row < n) {
        if (jj >= 0) jb.Q[row + (size_t)jj * n] = a[v][i];
        if (c >= nlive && c < cap) jb.Q[row + (size_t)c * n] = 0.0;
      }
    }
}

// One launch of the kernel with the row blocks that cover n.
template <bool PIV, typename Task>
void qr_launch(const Task* tasks_d, int ntasks, int n, int cap, double drop_tol, const int* m_dev, hipStream_t st) {
#define TK_QR_CASE(RS, NW)                                                                                       \
  hipLaunchKernelGGL((qr_cols_kernel<PIV, Task, RS, NW>), dim3(ntasks), dim3(NW * kWave), 0, st, tasks_d, n, cap, \
                     drop_tol, m_dev)
  if (n <= 64)
    TK_QR_CASE(16, 4);
  else if (n <= 128)
    TK_QR_CASE(32, 4);
  else if (n <= 256)
    TK_QR_CASE(32, 8);
  else
    TK_QR_CASE(64, 8);
#undef TK_QR_CASE
}

constexpr int CH_NT = 1024;  // 16 waves load the Gram, kCholWaves factor it
constexpr int CH_MAX = 64;

// Cholesky factor of one small Gram per workgroup.  The load is bound by one
// CU's bandwidth (the upper triangle of every split-K partial), the
// factorisation by its serial chain (chol_rows); row k of R is row k of the
// reduced matrix / sqrt(pivot).  A pivot that is not above max(dead_rel tr,
// dead_abs) marks a dead column: its row of R is zero and it updates nothing.
// Three Grams of order 53 from 8 partials each: 18.5 us (28.4 us with the matrix
// in LDS, 16 waves updating it and a barrier a step).
__global__ __launch_bounds__(CH_NT) void chol_kernel(const CholTask* __restrict__ tasks, int cap,
                                                     const int* __restrict__ m_dev, double dead_rel,
                                                     double dead_abs) {
  constexpr int NW = CH_NT / kWave;
  __shared__ double G[CH_MAX][CH_MAX + 1];
  __shared__ CholShared<double> chs;
  __shared__ double rk_s[CH_MAX];
  const CholTask tk_ = tasks[blockIdx.x];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  int m = m_dev ? *m_dev : cap;
  m = __builtin_amdgcn_readfirstlane(min(m, cap));
  const int last = max(m - 1, 0);
  // row i from column i of the symmetric Gram: contiguous over the lanes
  constexpr int RW = CH_MAX / NW;  // rows of a wave
  double g[RW];
  if (tk_.part) {  // the Gram's split-K partials, summed in split order (32 loads in flight)
    GPtr<double> pp[RW];
#pragma unroll
    for (int u = 0; u < RW; ++u) {
      const int i = min(wave + u * NW, last);
      pp[u] = (GPtr<double>)(tk_.part + min(max(lane, i), last) + (size_t)i * cap);
      g[u] = 0.0;
    }
    for (int sp = 0; sp < tk_.splits; sp += 8) {
      double v[RW][8];
#pragma unroll
      for (int u = 0; u < RW; ++u)
#pragma unroll
        for (int x = 0; x < 8; ++x) v[u][x] = pp[u][min(sp + x, tk_.splits - 1) * tk_.pstride];
#pragma unroll
      for (int u = 0; u < RW; ++u)
#pragma unroll
        for (int x = 0; x < 8; ++x) g[u] += sp + x < tk_.splits ? v[u][x] : 0.0;
    }
  } else {
#pragma unroll
    for (int u = 0; u < RW; ++u) {
      const int i = min(wave + u * NW, last);
      g[u] = ((GPtr<double>)tk_.G)[min(max(lane, i), last) + (size_t)i * cap];
    }
  }
#pragma unroll
  for (int u = 0; u < RW; ++u) {
    const int i = wave + u * NW;
    if (i < m) G[i][lane] = lane >= i && lane < m ? g[u] : 0.0;
  }
  __syncthreads();
  if (wave >= kCholWaves) return;  // a barrier waits for the waves that are left
  const double tr = wave_sum(lane < m ? G[lane][lane] : 0.0);
  const double s = tk_.shift * tr;
  const double dtol = fmax(dead_rel * tr, dead_abs);
  double a[kCholRows];
#pragma unroll
  for (int r = 0; r < kCholRows; ++r) {
    const int i = wave + kCholPanel * r;
    a[r] = i < m ? G[i][lane] : 0.0;
    if (lane == i) a[r] += s;
  }
  chol_rows(
      a, m, lane, wave, chs,
      [&](int k, double pv, double row, double& f) {
        const bool dead = !(pv > dtol);
        if (lane == 0) rk_s[k] = dead ? 0.0 : pv;
        f = dead ? 0.0 : row / pv;
        return true;
      },
      [&](int i, double v) { G[i][lane] = v; });
  __syncthreads();
  const double rk = sqrt(lane < m ? rk_s[lane] : 0.0);
  for (int j = wave; j < cap; j += kCholWaves) {
    double r = 0.0;
    if (lane < m && j < m && lane <= j && rk != 0.0) r = lane == j ? rk : G[lane][j] / rk;
    if (lane < cap) tk_.R[lane + (size_t)j * cap] = r;
  }
}

constexpr int TR_NT = 128;
constexpr int TR_LANES = 4;                    // lanes of a row
constexpr int TR_ROWS = TR_NT / TR_LANES;      // rows of a workgroup
// A lane's entries of a row of R, padded so that the 16-byte reads of the four
// lanes hit different banks.
constexpr int TR_PAD = CH_MAX / TR_LANES + 2;

template <int L>
__device__ __forceinline__ double quad_lane(double v) {
  return dpp_mov<L * 0x55>(v);  // quad_perm[L, L, L, L]
}

// Q = Y R^{-1} by forward substitution, four lanes a row: lane l holds the
// columns l, l + 4, ..  Step k divides in the lane of column k and passes q_k
// to the other three, which subtract q_k R[k][c] from their later columns, so
// a row's entries are updated in the same order and with the same operations
// as by one thread a row; its chain is 53 divisions and as many
// subtractions in place of 53 * 52 / 2 dependent ones, and four times as
// many waves share the loads.  The division is x * (1 / d) with one exact
// remainder step (correctly rounded, as 1 / d is).  512 x 53, three matrices:
// 22.5 -> 13.5 us.
template <int NG>
__global__ __launch_bounds__(TR_NT) void trsm_rows_kernel(const TrsmTask* __restrict__ tasks, int cap,
                                                          const int* __restrict__ m_dev) {
  constexpr int NC = NG * TR_LANES;
  __shared__ __align__(16) double Rp[NC][TR_LANES][TR_PAD];  // R[k][l + 4 i], zero up to the diagonal
  __shared__ __align__(16) double dg[NC][2];                 // R[k][k], 1 / R[k][k] (zeros: dead column)
  const TrsmTask tk_ = tasks[blockIdx.y];
  const int n = tk_.n;
  if (blockIdx.x * TR_ROWS >= unsigned(n)) return;
  const int tid = threadIdx.x;
  const int l = tid % TR_LANES;
  int m = m_dev ? *m_dev : cap;
  m = __builtin_amdgcn_readfirstlane(min(m, cap));
  const int row = blockIdx.x * TR_ROWS + tid / TR_LANES;
  const int rowc = min(row, n - 1);
  const GPtr<double> gy = (GPtr<double>)tk_.Y;
  double q[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) q[i] = gy[rowc + (size_t)min(l + TR_LANES * i, cap - 1) * n];
  {
    // column c of R by a wave, lane = row k: every load in flight at once
    constexpr int NW = TR_NT / kWave, CPW = NC / NW;
    const GPtr<double> gr = (GPtr<double>)tk_.R;
    const int k = tid & (kWave - 1), w = tid / kWave;
    double rv[CPW];
#pragma unroll
    for (int u = 0; u < CPW; ++u) rv[u] = gr[min(k, cap - 1) + (size_t)min(w + NW * u, cap - 1) * cap];
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
      const int c = w + NW * u;
      if (k < NC) {
        Rp[k][c % TR_LANES][c / TR_LANES] = k < c && c < m ? rv[u] : 0.0;
        if (k == c) {
          const double d = c < m ? rv[u] : 0.0;
          dg[k][0] = d;
          dg[k][1] = d != 0.0 ? 1.0 / d : 0.0;
        }
      }
    }
  }
  __syncthreads();
  auto step = [&](auto kc) {
    constexpr int k = decltype(kc)::value, i0 = k / TR_LANES, lk = k % TR_LANES;
    if (k >= m) return;
    const double d = dg[k][0], di = dg[k][1];
    const double x = q[i0];
    double t = x * di;
    t = fma(fma(-t, d, x), di, t);
    const double qk = quad_lane<lk>(d != 0.0 ? t : 0.0);
#pragma unroll
    for (int i = i0; i < NG; ++i) q[i] = fma(-qk, Rp[k][l][i], q[i]);
    q[i0] = l == lk ? qk : q[i0];
  };
  for_constants<NC>(step);
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int c = l + TR_LANES * i;
    if (row < n && c < cap) {
      const double qv = c < m ? q[i] : 0.0;
      tk_.Q[row + (size_t)c * n] = qv;
      if (tk_.Qf) tk_.Qf[row + (size_t)c * n] = float(qv);
    }
  }
}

}  // namespace

void chol_batched(const CholTask* tasks_d, int ntasks, int cap, const int* m_dev, double dead_rel, double dead_abs,
                  hipStream_t st) {
  if (ntasks <= 0) return;
  TK_CHECK(cap <= CH_MAX, kErrUnsupported, "Cholesky-QR: more than 64 columns");
  timer_begin(kKcQr, st);
  hipLaunchKernelGGL(chol_kernel, dim3(ntasks), dim3(CH_NT), 0, st, tasks_d, cap, m_dev, dead_rel, dead_abs);
  TK_LAUNCH_CHECK();
  timer_end(kKcQr, st);
}

void trsm_rows(const TrsmTask* tasks_d, int ntasks, int nmax, int cap, const int* m_dev, hipStream_t st) {
  if (ntasks <= 0) return;
  TK_CHECK(cap <= CH_MAX, kErrUnsupported, "Cholesky-QR: more than 64 columns");
#define TK_TRSM_CASE(NG)                                                                                           \
  hipLaunchKernelGGL((trsm_rows_kernel<NG>), dim3(ceil_div(nmax, TR_ROWS), ntasks), dim3(TR_NT), 0, st, tasks_d, cap, \
                     m_dev)
  // the fewest column groups that hold cap columns: a row's registers and the
  // unrolled steps follow it
  if (cap <= 16)
    TK_TRSM_CASE(4);
  else if (cap <= 32)
    TK_TRSM_CASE(8);
  else if (cap <= 48)
    TK_TRSM_CASE(12);
  else
    TK_TRSM_CASE(16);
#undef TK_TRSM_CASE
  TK_LAUNCH_CHECK();
}

// Algorithmic flops of a launch at full column count m = min(cap, n): the
// Householder factorisation 2 n m^2 - (2/3) m^3, and as much again for the
// explicit thin Q.
static double qr_flops(int ntasks, int n, int cap, bool with_q) {
  const double m = std::min(cap, n), nn = n;
  const double f = 2.0 * nn * m * m - 2.0 / 3.0 * m * m * m;
  return ntasks * f * (with_q ? 2.0 : 1.0);
}

void qr_batched(const QrTask* tasks_d, int ntasks, int n, int cap, const int* m_dev, hipStream_t st) {
  if (ntasks <= 0) return;
  TK_CHECK(n >= 1 && n <= QC_MAXROWS, kErrUnsupported, "Householder QR: more than 512 rows");
  TK_CHECK(cap <= kWave, kErrUnsupported, "Householder QR: more than 64 columns");
  timer_begin(kKcQr, st, qr_flops(ntasks, n, cap, true));
  qr_launch<false>(tasks_d, ntasks, n, cap, 0.0, m_dev, st);
  TK_LAUNCH_CHECK();
  timer_end(kKcQr, st);
}

void qr_piv_batched(const QrPivTask* tasks_d, int ntasks, int n, int cap, double drop_tol, hipStream_t st) {
  if (ntasks <= 0) return;
  TK_CHECK(n >= 1 && n <= QC_MAXROWS && cap <= kWave, kErrUnsupported,
           "pivoted QR: more than 512 rows or 64 columns");
  timer_begin(kKcQr, st, qr_flops(ntasks, n, cap, true));
  qr_launch<true>(tasks_d, ntasks, n, cap, drop_tol, nullptr, st);
  TK_LAUNCH_CHECK();
  timer_end(kKcQr, st);
}

}  // namespace tk
