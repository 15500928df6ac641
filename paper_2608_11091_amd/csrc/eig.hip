// Small symmetric eigensolvers, one workgroup per matrix.
//
//  * Eigenvalues only (N <= 160): Householder reduction to tridiagonal form
//    with the matrix distributed over the registers of 16 waves, then every
//    eigenvalue by multisection on Sturm counts.  Used by the RoundSum
//    effective-rank rule, which needs the spectrum but no vectors.
//  * Eigenvalues only (160 < N <= 512): the same reduction with the matrix in
//    global memory (it stays in the L2 of the workgroup's XCD), reduced in
//    place; each step streams the trailing block once, applying the previous
//    step's rank-2 update and forming the next product A v in the same pass.
//  * Eigenvalues and vectors of positive semidefinite matrices (N <= 64):
//    Cholesky factor and one-sided cyclic Jacobi on its columns, which stay in
//    registers.  The relative rotation criterion resolves the small
//    eigenvalues of graded matrices to high relative accuracy.
// Results are sorted in descending order; an optional rank rule (RoundSum
// effective rank / ST-HOSVD truncation) runs on the sorted spectrum.
#include <cfloat>

#include "chol.hpp"
#include "kernels.hpp"
#include "rotation.hpp"

namespace tk {

namespace {

constexpr int VAL_NMAX = kEigRegMax;
constexpr int VEC_NMAX = 64;
constexpr int GM_NMAX = 512;

template <typename T> struct Vec4;
template <> struct Vec4<float> { using type = float __attribute__((ext_vector_type(4))); };
template <> struct Vec4<double> { using type = double __attribute__((ext_vector_type(4))); };

template <typename T> struct Lim;
template <> struct Lim<double> {
  static __device__ constexpr double eps() { return DBL_EPSILON; }
  static __device__ constexpr double stop() { return 1.490116119384766e-08; }  // sqrt(eps)
  static __device__ constexpr double tiny() { return 1e-300; }
  static __device__ constexpr double pivot_tiny() { return 1e-300; }  // the least pivot
};
template <> struct Lim<float> {
  static __device__ constexpr float eps() { return FLT_EPSILON; }
  static __device__ constexpr float stop() { return 3.4526698e-04f; }  // sqrt(eps)
  static __device__ constexpr float tiny() { return 1e-37f; }
  static __device__ constexpr float pivot_tiny() { return 1e-36f; }
};

// A task does nothing when its pair flag or any rank certificate is set.
template <typename T>
__device__ __forceinline__ bool task_skipped(const EigTask<T>& t) {
  if (t.skip != nullptr && *t.skip != 0) return true;
  bool c = false;
  for (int i = 0; i < t.ncert; ++i) c |= t.cert[i] != 0;
  return c;
}

// Rank rules on a descending spectrum lam_desc(0) >= lam_desc(1) >= ..; returns
// the rank.
template <typename T, typename Lam>
__device__ int apply_rule(const EigRule& ru, Lam lam_desc, int N) {
  int r = 0;
  if (ru.kind == 1) {
    const double l0 = N > 0 ? double(lam_desc(0)) : 0.0;
    if (N > 0 && l0 > 0.0) {
      double total = 0.0;
      for (int i = 0; i < N; ++i) {
        const double li = double(lam_desc(i));
        total += li > ru.delta * l0 ? li : 0.0;
      }
      const double tau = *ru.tau;
      const double thr = tau * tau * total;
      double tail = 0.0;
      r = N;
      for (int i = N - 1; i >= 0; --i) {
        const double li = double(lam_desc(i));
        tail += li > ru.delta * l0 ? li : 0.0;
        if (tail <= thr) r = i;
        else break;
      }
    }
  } else if (ru.kind == 2) {
    const double total = *ru.total;
    if (ru.force && *ru.force >= 0) {
      r = *ru.force < N ? *ru.force : N;
    } else if (total <= *ru.zthr) {
      r = 1;
    } else {
      const double eps = *ru.eps;
      const double thr = eps * eps * total / ru.d;
      double tail = 0.0;
      r = N;
      for (int i = N - 1; i >= 0; --i) {
        const double li = double(lam_desc(i));
        tail += li > 0.0 ? li : 0.0;
        if (tail <= thr) r = i;
        else break;
      }
      if (r < 1) r = 1;
      if (r > ru.cap) r = ru.cap;
    }
  }
  return r;
}

// ------------------------------------------------------------ eigenvalues only

// Number of eigenvalues of the tridiagonal (d, e) below x, from the signs of
// the LDL^T pivots of T - x I (e2 = squared off-diagonal).  FP32 takes the
// hardware reciprocal: a Sturm count tolerates ulp-level relative errors in
// each pivot (the computed count is exact for a nearby matrix).
__device__ __forceinline__ float sturm_div(float a, float q) { return a * __builtin_amdgcn_rcpf(q); }
__device__ __forceinline__ double sturm_div(double a, double q) { return a / q; }
template <typename T>
__device__ int sturm_count(const T* d, const T* e2, int n, T x, T pivmin) {
  int c = 0;
  T q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  c += q < T(0);
  for (int k = 1; k < n; ++k) {
    q = d[k] - x - sturm_div(e2[k - 1], q);
    if (fabs(q) < pivmin) q = -pivmin;
    c += q < T(0);
  }
  return c;
}

// Eigenvalues of the symmetric tridiagonal (dd, ee) (ee[k] couples k, k+1),
// both in LDS, by multisection on Sturm counts: G lanes per eigenvalue test G
// interior points of the current interval at once.  Writes them descending to
// `lam` (LDS) and the task's outputs, then applies the task's rank rule.
// Called by all `nthreads` threads of the block; ee is squared in place.
template <typename T>
__device__ void tridiag_spectrum(const EigTask<T>& tk_, T* dd, T* ee, T* lam, T* sc, int N, int tid, int nthreads) {
  if (tid == 0) {
    T gl = dd[0], gu = dd[0], emax2 = T(0);
    for (int k = 0; k < N; ++k) {
      const T r = (k > 0 ? fabs(ee[k - 1]) : T(0)) + (k + 1 < N ? fabs(ee[k]) : T(0));
      gl = fmin(gl, dd[k] - r);
      gu = fmax(gu, dd[k] + r);
    }
    for (int k = 0; k + 1 < N; ++k) emax2 = fmax(emax2, ee[k] * ee[k]);
    sc[1] = gl;
    sc[2] = gu;
    sc[3] = emax2;
  }
  __syncthreads();
  const T gl = sc[1], gu = sc[2], emax2 = sc[3];
  for (int k = tid; k + 1 < N; k += nthreads) ee[k] = ee[k] * ee[k];
  __syncthreads();
  const T bnorm = fmax(fabs(gl), fabs(gu));
  const T pivmin = fmax(Lim<T>::tiny(), emax2 * Lim<T>::tiny() * T(1e10));
  const T tolx = T(2) * Lim<T>::eps() * bnorm;
  // Rank rule with a cap (kind 1, cap1 > 0): only min(r~, cap1) is needed,
  // and one Sturm count settles the common case.  If at least cap1
  // eigenvalues lie at or above x = max(tau^2 tot, delta (gu + tolx)) + 2 tolx,
  // with tot = trace + N (max(0, -gl) + tolx) bounding the rule's total (the
  // positive eigenvalues, as the multisection would compute them), then the
  // cap1-th largest counts as nonzero and alone exceeds tau^2 total, so the
  // tail from it on does too and r~ >= cap1.
  if (tk_.rule.kind == 1 && tk_.rule.cap1 > 0 && tk_.rule.cap1 <= N) {
    if (tid == 0) {
      double tr = 0.0;
      for (int k = 0; k < N; ++k) tr += double(dd[k]);
      const double tau = *tk_.rule.tau;
      const double tx = double(tolx);
      const double tot = tr + double(N) * (fmax(0.0, -double(gl)) + tx);
      const double x = fmax(tau * tau * tot, tk_.rule.delta * (double(gu) + tx)) + 2.0 * tx;
      const int below = sturm_count<T>(dd, ee, N, T(x), pivmin);
      sc[0] = (N - below >= tk_.rule.cap1) ? T(1) : T(0);
    }
    __syncthreads();
    if (sc[0] != T(0)) {
      if (tid == 0) *tk_.rule.rank_out = tk_.rule.cap1;
      return;  // uniform: every thread read the same flag after the barrier
    }
  }
  // FP64, and a tail threshold below the zero clamp whatever the spectrum
  // (tau^2 N < delta: the total is at most N lambda_1, so every eigenvalue
  // above delta lambda_1 exceeds tau^2 total by itself): r~ is the number of
  // eigenvalues above delta lambda_1, so only the largest one is located (256
  // points a round), as far as it takes the counts at delta times both ends of
  // its interval to agree: four rounds, but for an eigenvalue that lies between.
  // (Not in FP32, where the clamp lies below the Gram's rounding and the
  // count follows the noise of the eigenvalues as computed.)
  if constexpr (sizeof(T) == 8) {
    const double tau = tk_.rule.kind == 1 ? *tk_.rule.tau : 1.0;
    if (tk_.rule.kind == 1 && tk_.rule.cap1 > 0 && tau * tau * N * 2.0 < tk_.rule.delta) {
      T lo = gl - tolx, hi = gu + tolx;
      int* const first = reinterpret_cast<int*>(lam);  // scratch: first point above lambda_1, by wave
      for (int it = 0;; ++it) {
        if (it >= 4) {
          if (tid < kWave) {  // lane 0: the lower end, the others: the upper one
            const int c = sturm_count(dd, ee, N, T(tk_.rule.delta) * (tid == 0 ? lo : hi), pivmin);
            if (tid < 2) first[tid] = c;
          }
          __syncthreads();
          const bool done = first[0] == first[1] || !(hi - lo > tolx) || it == 16;
          __syncthreads();
          if (done) break;  // uniform
        }
        if (tid < 256) {
          const T mid = lo + (hi - lo) * (T(tid + 1) / T(257));
          const unsigned long long up = __ballot(sturm_count(dd, ee, N, mid, pivmin) == N);
          if ((tid & (kWave - 1)) == 0) first[tid / kWave] = up ? (tid & ~(kWave - 1)) + __builtin_ctzll(up) : 256;
        }
        __syncthreads();
        const int f = min(min(first[0], first[1]), min(first[2], first[3]));
        const T span = hi - lo;
        hi = f < 256 ? lo + span * (T(f + 1) / T(257)) : hi;
        lo = f > 0 ? lo + span * (T(f) / T(257)) : lo;
        __syncthreads();
      }
      if (tid == 0) {
        const int below = first[0] == first[1]
                              ? first[1]
                              : sturm_count(dd, ee, N, T(tk_.rule.delta) * (T(0.5) * (lo + hi)), pivmin);
        *tk_.rule.rank_out = hi > T(0) ? N - below : 0;
      }
      return;  // uniform
    }
  }
  // G = lanes per eigenvalue: the largest power of two <= min(16, nthreads / N)
  int G = 1;
  while (G < 16 && 2 * G * N <= nthreads) G *= 2;
  const int g = tid % G;
  const int gshift = (tid & (kWave - 1)) - g;  // first lane of the group within the wave
  const unsigned long long gmask = (G == 64 ? ~0ull : ((1ull << G) - 1ull));
  for (int i = tid / G; i < N; i += nthreads / G) {
    T lo = gl - tolx, hi = gu + tolx;
    for (int it = 0; it < 200 && hi - lo > tolx; ++it) {
      // interior points lo + (hi - lo) (q + 1) / (G + 1), q < G; counts are
      // monotone in q, so the new interval is (point f-1, point f] with f
      // the first point above eigenvalue i (every lane recomputes them)
      const T span = hi - lo;
      const T mid = lo + span * T(g + 1) / T(G + 1);
      const int above = (mid > lo && mid < hi) ? (sturm_count(dd, ee, N, mid, pivmin) > i) : (mid >= hi);
      const unsigned long long bits = (__ballot(above) >> gshift) & gmask;
      const int f = bits ? __builtin_ctzll(bits) : G;
      const T nhi = f < G ? lo + span * T(f + 1) / T(G + 1) : hi;
      const T nlo = f > 0 ? lo + span * T(f) / T(G + 1) : lo;
      if (!(nhi < hi || nlo > lo)) break;
      lo = fmax(lo, nlo);
      hi = fmin(hi, nhi);
    }
    lam[N - 1 - i] = T(0.5) * (lo + hi);
  }
  __syncthreads();
  if (tk_.lam)
    for (int i = tid; i < N; i += nthreads) tk_.lam[i] = lam[i];
  if (tid == 0 && tk_.rule.kind != 0) *tk_.rule.rank_out = apply_rule<T>(tk_.rule, [&](int i) { return lam[i]; }, N);
}

// Householder tridiagonalisation with the matrix in registers: lane l of
// wave w of W holds the entries (l + 64 a, w + W b), so the rank-2
// update of a step touches only registers and LDS carries vectors and partial
// sums, never the matrix.  Step j: the wave holding column j forms v (the
// Householder vector of the part below the diagonal) and tau; every thread
// forms its partial products of A_sub v and of v^T A_sub v, which are summed
// across the waves through LDS into p = tau A_sub v and
// w = p - (tau^2 / 2)(v^T A_sub v) v; every thread applies
// A_sub -= v w^T + w v^T to its entries.  Vectors alternate between two LDS
// buffers with the step parity.  Then the spectrum as above.
// Bound by latency, one workgroup per matrix: a serial chain of N steps with
// three barriers each.  The body is compiled for three orders (rows and
// columns a thread holds; the order is a device value), as the registers of
// order 160 for every matrix made the FP64 form spill at each of them.  With
// the count in place of the spectrum (below) and the narrower Gram side, the
// FP64 launches of a preconditioned training step at n = 128 went from 1122 to
// 218 us on average, those of twelve solver iterations at n = 512 from 295 to
// 106 us.
constexpr int TRG_NT = 1024;            // 16 waves
constexpr int TRG_NW = TRG_NT / kWave;

template <typename T>
struct TrgShared {
  T vb[2][VAL_NMAX], wb[2][VAL_NMAX];
  T pp[TRG_NW][VAL_NMAX];
  T qs[TRG_NW];
  T tau_s[2];
  T dd[VAL_NMAX], ee[VAL_NMAX], lam[VAL_NMAX];
  T sc[4];
};

// N <= min(64 RR, 16 RC)
template <typename T, int RR, int RC>
__device__ __forceinline__ void tridiag_reg(const EigTask<T>& tk_, TrgShared<T>& sh, int N) {
  auto &vb = sh.vb, &wb = sh.wb;
  auto& pp = sh.pp;
  auto& qs = sh.qs;
  auto& tau_s = sh.tau_s;
  auto &dd = sh.dd, &ee = sh.ee;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int e = tid; e < 2 * VAL_NMAX; e += TRG_NT) {
    vb[e / VAL_NMAX][e % VAL_NMAX] = T(0);
    wb[e / VAL_NMAX][e % VAL_NMAX] = T(0);
  }
  T a[RR][RC];
#pragma unroll
  for (int i = 0; i < RR; ++i)
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const int r = lane + kWave * i, c = wave + TRG_NW * k;
      T v = T(0);
      if (r < N && c < N) v = (r >= c) ? tk_.A[r + (size_t)c * tk_.lda] : tk_.A[c + (size_t)r * tk_.lda];
      a[i][k] = v;
    }
  __syncthreads();  // the first vector goes into what other waves clear
  // Householder vector of column jj from this wave's registers (called by the
  // wave holding column jj only; jj + 2 < N)
  auto householder = [&](int jj) {
    const int buf = jj & 1;
    const int r0 = jj + 1;
    const int kb = jj / TRG_NW;  // uniform
    T x[RR];
    T s2 = T(0);
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      T v = T(0);
#pragma unroll
      for (int k = 0; k < RC; ++k)
        if (k == kb) v = a[i][k];
      x[i] = v;
      const int r = lane + kWave * i;
      if (r > r0 && r < N) s2 += v * v;
    }
    s2 = wave_sum(s2);
    T xa = T(0);
#pragma unroll
    for (int i = 0; i < RR; ++i)
      if (i == r0 / kWave) xa = x[i];
    const T alpha = rdlane(xa, r0 & (kWave - 1));
    T beta, tau, scal;
    if (s2 == T(0)) {
      beta = alpha;
      tau = T(0);
      scal = T(0);
    } else {
      beta = -copysign(sqrt(alpha * alpha + s2), alpha);
      tau = (beta - alpha) / beta;
      scal = T(1) / (alpha - beta);
    }
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      const int r = lane + kWave * i;
      if (r >= r0 && r < N) vb[buf][r] = r == r0 ? T(1) : x[i] * scal;
      if (r == jj) dd[jj] = x[i];
    }
    if (lane == 0) {
      tau_s[buf] = tau;
      ee[jj] = beta;
    }
  };
  for (int j = 0; j + 2 < N; ++j) {
    const int buf = j & 1;
    const int r0 = j + 1;
    if (wave == (j & (TRG_NW - 1))) householder(j);
    __syncthreads();
    const T tau = tau_s[buf];
    if (tau == T(0)) continue;  // the same value in every thread: nothing to apply
    // unconditional loads (in-bounds indices; the buffers hold finite values)
    // times a 0/1 mask, so that all loads issue before a single wait
    T vr[RR], vc[RC];
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      const int r = lane + kWave * i;
      vr[i] = vb[buf][min(r, VAL_NMAX - 1)] * T(r >= r0 && r < N);
    }
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const int c = wave + TRG_NW * k;
      vc[k] = vb[buf][c] * T(c >= r0 && c < N);
    }
    // ---- partial products over this wave's columns
    T q = T(0);
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      T acc = T(0);
#pragma unroll
      for (int k = 0; k < RC; ++k) acc += a[i][k] * vc[k];
      q += vr[i] * acc;
      const int r = lane + kWave * i;
      if (r < N) pp[wave][r] = acc;
    }
    q = wave_sum(q);
    if (lane == 0) qs[wave] = q;
    __syncthreads();
    if (tid >= r0 && tid < N) {
      T sacc = T(0), vav = T(0);
#pragma unroll
      for (int w = 0; w < TRG_NW; ++w) {
        sacc += pp[w][tid];
        vav += qs[w];
      }
      const T K = T(0.5) * tau * tau * vav;
      wb[buf][tid] = tau * sacc - K * vb[buf][tid];
    }
    __syncthreads();
    // ---- rank-2 update of this thread's entries
    T wr[RR], wc[RC];
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      const int r = lane + kWave * i;
      wr[i] = wb[buf][min(r, VAL_NMAX - 1)] * T(r >= r0 && r < N);
    }
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const int c = wave + TRG_NW * k;
      wc[k] = wb[buf][c] * T(c >= r0 && c < N);
    }
#pragma unroll
    for (int i = 0; i < RR; ++i)
#pragma unroll
      for (int k = 0; k < RC; ++k) a[i][k] -= vr[i] * wc[k] + wr[i] * vc[k];
    // no barrier here: the next step's Householder vector comes from its
    // wave's own registers and goes to the other buffer, and every shared
    // array this step reads is written again only after the next step's
    // first barrier (pp, qs) or two steps on (vb, wb, tau_s by parity)
  }
  // last 2 x 2 block: diagonal entries and the coupling, from their holders
#pragma unroll
  for (int i = 0; i < RR; ++i)
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const int r = lane + kWave * i, c = wave + TRG_NW * k;
      if (N >= 2 && r == N - 2 && c == N - 2) dd[N - 2] = a[i][k];
      if (N >= 2 && r == N - 1 && c == N - 2) ee[N - 2] = a[i][k];
      if (r == N - 1 && c == N - 1) dd[N - 1] = a[i][k];
    }
  __syncthreads();
}

template <typename T>
__global__ __launch_bounds__(TRG_NT) void tridiag_reg_kernel(const EigTask<T>* __restrict__ tasks, int NL) {
  const EigTask<T> tk_ = tasks[blockIdx.x];
  if (task_skipped(tk_)) return;
  int N = NL;
  if (tk_.ndyn != nullptr) {
    const int nd = *tk_.ndyn;
    if (nd < 0 || nd > NL) {
      if (threadIdx.x == 0 && tk_.rule.rank_out) *tk_.rule.rank_out = -1;
      return;
    }
    N = nd;
  }
  if (N == 0) {
    if (threadIdx.x == 0 && tk_.rule.rank_out) *tk_.rule.rank_out = 0;
    return;
  }
  __shared__ TrgShared<T> sh;
  if (N <= 64)
    tridiag_reg<T, 1, 4>(tk_, sh, N);
  else if (N <= 112)
    tridiag_reg<T, 2, 7>(tk_, sh, N);
  else
    tridiag_reg<T, 3, 10>(tk_, sh, N);
  tridiag_spectrum<T>(tk_, sh.dd, sh.ee, sh.lam, sh.sc, N, int(threadIdx.x), TRG_NT);
}

// Householder tridiagonalisation of an N x N symmetric matrix (160 < N <= 512)
// held in global memory, column-major with leading dimension lda; only the
// lower triangle of the input is read and the matrix is overwritten.  One
// workgroup of 16 waves.  The lower triangle is first mirrored into the upper
// one through LDS tiles, so that the reduction can keep full storage and form
// A v as row sums (each lane owns rows, no cross-lane sums per column).
// Step j (sub-block S = rows/columns j+1..N-1, Householder vector v with
// v_{j+1} = 1, tau, and the pending update (vp, wp) of step j-1):
//   1. column j of the updated matrix, x_i = a_ij - vp_i wp_j - wp_i vp_j;
//      the diagonal entry and ||x_{j+2..}||^2 give v, tau and beta;
//   2. one pass over S: a <- a - vp wp^T - wp vp^T (stored back), and every
//      lane accumulates its rows of S v; the same pass accumulates v^T S v;
//   3. w = tau S v - (tau^2 / 2)(v^T S v) v becomes the pending update.
// The final 2 x 2 block takes the last pending update; then the spectrum by
// multisection as above.
template <typename T>
__global__ __launch_bounds__(1024) void tridiag_gm_kernel(const EigTask<T>* __restrict__ tasks, int NL) {
  constexpr int NT = 1024;
  constexpr int NW = NT / kWave;          // 16 waves
  constexpr int RCH = GM_NMAX / kWave;    // row chunks of 64
  const EigTask<T> tk_ = tasks[blockIdx.x];
  if (task_skipped(tk_)) return;
  int N = NL;
  if (tk_.ndyn != nullptr) {
    const int nd = *tk_.ndyn;
    if (nd < 0 || nd > NL) {
      if (threadIdx.x == 0 && tk_.rule.rank_out) *tk_.rule.rank_out = -1;
      return;
    }
    N = nd;
  }
  if (N == 0) {
    if (threadIdx.x == 0 && tk_.rule.rank_out) *tk_.rule.rank_out = 0;
    return;
  }
  T* A = const_cast<T*>(tk_.A);
  const size_t lda = size_t(tk_.lda);
  using T4 = typename Vec4<T>::type;
  T* const W = A;          // the trailing-block pass reads columns as 16-byte vectors
  const size_t ldw = lda;  // (lda is a multiple of 4 and A 16-byte aligned: checked by the launcher)
  __shared__ T xb[GM_NMAX], vp[GM_NMAX], wp[GM_NMAX];
  __shared__ T rowp[NW][GM_NMAX];  // per-wave row sums; also the mirror tiles
  __shared__ T part[NW], qpart[NW];
  __shared__ T dd[GM_NMAX], ee[GM_NMAX], lam[GM_NMAX];
  __shared__ T sc[4];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int i = tid; i < GM_NMAX; i += NT) {
    vp[i] = T(0);
    wp[i] = T(0);
  }
  // ---- mirror the lower triangle into the upper one, 64 x 64 tiles through LDS
  {
    T* tile = &rowp[0][0];  // 64 x 65 staging (fits in rowp)
    const int nt = (N + kWave - 1) / kWave;
    for (int I = 0; I < nt; ++I)
      for (int J = 0; J <= I; ++J) {
        // load tile (I, J): column c of the tile by the threads with c % 16 == wave
        for (int c = wave; c < kWave; c += NW) {
          const int r = I * kWave + lane, col = J * kWave + c;
          tile[c * (kWave + 1) + lane] = (r < N && col < N) ? A[r + size_t(col) * lda] : T(0);
        }
        __syncthreads();
        // store its transpose into tile (J, I), upper-triangle entries only
        for (int c = wave; c < kWave; c += NW) {
          const int r = J * kWave + lane, col = I * kWave + c;  // destination (r, col), r < col
          if (r < N && col < N && r < col) A[r + size_t(col) * lda] = tile[lane * (kWave + 1) + c];
        }
        __syncthreads();
      }
  }
  for (int j = 0; j + 2 < N; ++j) {
    // ---- 1. column j after the pending update, ||x_{j+2..N-1}||^2
    T s2p = T(0);
    if (tid >= j && tid < N) {
      const T x = A[tid + size_t(j) * lda] - (vp[tid] * wp[j] + wp[tid] * vp[j]);
      xb[tid] = x;
      if (tid == j) dd[j] = x;
      if (tid >= j + 2) s2p = x * x;
    }
    s2p = wave_sum(s2p);
    if (lane == 0) part[wave] = s2p;
    __syncthreads();
    T s2 = T(0);
#pragma unroll
    for (int w = 0; w < NW; ++w) s2 += part[w];
    const T alpha = xb[j + 1];
    T beta, tau, scal;
    if (s2 == T(0)) {
      beta = alpha;
      tau = T(0);
      scal = T(0);
    } else {
      beta = -copysign(sqrt(alpha * alpha + s2), alpha);
      tau = (beta - alpha) / beta;
      scal = T(1) / (alpha - beta);
    }
    if (tid == 0) ee[j] = beta;
    const T vmask = tau != T(0) ? T(1) : T(0);
    auto vval = [&](int i) -> T {  // Householder vector entry (0 outside j+1..N-1)
      return i == j + 1 ? vmask : (i > j + 1 && i < N ? xb[i] * scal : T(0));
    };
    // ---- 2. pass over the trailing block: lane l owns rows 4l + 256u .. +3
    //         (u < 2), 16-byte accesses; several columns per wave in flight
    const int r0 = j + 1;
    T4 vpr[2], wpr[2], acc[2];
    bool live[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int rb = 4 * lane + 256 * u;
      live[u] = rb < N && rb + 3 >= r0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = rb + e;
        const bool ok = i >= r0 && i < N;
        vpr[u][e] = ok ? vp[i] : T(0);
        wpr[u][e] = ok ? wp[i] : T(0);
        acc[u][e] = T(0);
      }
    }
    constexpr int CU = sizeof(T) == 4 ? 4 : 2;  // columns in flight per wave (FP64: register budget)
    for (int c0 = r0 + wave; c0 < N; c0 += CU * NW) {
      T4 a[CU][2];
      T vpc[CU], wpc[CU], vc[CU];
#pragma unroll
      for (int m = 0; m < CU; ++m) {
        const int c = c0 + m * NW;
        const bool cok = c < N;  // uniform across the wave
        vpc[m] = cok ? vp[c] : T(0);
        wpc[m] = cok ? wp[c] : T(0);
        vc[m] = cok ? vval(c) : T(0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const T4* src = reinterpret_cast<const T4*>(W + size_t(cok ? c : r0) * ldw + 4 * lane + 256 * u);
          a[m][u] = (cok && live[u]) ? *src : T4{};
        }
      }
#pragma unroll
      for (int m = 0; m < CU; ++m) {
        const int c = c0 + m * NW;
        if (c >= N) continue;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (!live[u]) continue;
          const int rb = 4 * lane + 256 * u;
          T4 v = a[m][u] - (vpr[u] * wpc[m] + wpr[u] * vpc[m]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool ok = rb + e >= r0 && rb + e < N;
            v[e] = ok ? v[e] : a[m][u][e];
            acc[u][e] += ok ? v[e] * vc[m] : T(0);
          }
          *reinterpret_cast<T4*>(W + size_t(c) * ldw + rb) = v;
        }
      }
    }
    T q = T(0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * lane + 256 * u + e;
        const bool ok = i >= r0 && i < N;
        q += ok ? vval(i) * acc[u][e] : T(0);
        if (ok) rowp[wave][i] = acc[u][e];
      }
    q = wave_sum(q);
    if (lane == 0) qpart[wave] = q;
    __syncthreads();
    // ---- 3. the new pending update
    if (tid >= r0 && tid < N) {
      T sv = T(0), vav = T(0);
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        sv += rowp[w][tid];
        vav += qpart[w];
      }
      const T vi = vval(tid);
      const T K = T(0.5) * tau * tau * vav;
      vp[tid] = vi;
      wp[tid] = tau * sv - K * vi;
    }
    __syncthreads();
  }
  // last 2 x 2 block (or the single entry) after the last pending update
  if (tid == 0) {
    if (N >= 2) {
      const int a = N - 2, b = N - 1;
      dd[a] = A[a + size_t(a) * lda] - T(2) * vp[a] * wp[a];
      ee[a] = A[b + size_t(a) * lda] - (vp[b] * wp[a] + wp[b] * vp[a]);
      dd[b] = A[b + size_t(b) * lda] - T(2) * vp[b] * wp[b];
    } else {
      dd[0] = A[0];
    }
  }
  __syncthreads();
  tridiag_spectrum<T>(tk_, dd, ee, lam, sc, N, tid, NT);
}

// ------------------------------------------------------------ eigenvalues + vectors

// Sum over the 8 lanes of a column group; every lane gets the same value.
template <typename T>
__device__ __forceinline__ T group8_sum(T v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  return v;
}

// Whether the columns with dot product d and squared norms nx, ny are to be
// rotated against each other (|d| > tol ||x|| ||y||).
__device__ __forceinline__ bool above_tol(double d, double nx, double ny, double tol) {
  return d * d > tol * tol * nx * ny;
}
__device__ __forceinline__ bool above_tol(float d, float nx, float ny, float tol) {
  // norms one by one: their product underflows on strongly graded spectra
  const float ad = fabsf(d);
  return ad > Lim<float>::tiny() && ad > tol * (__builtin_amdgcn_sqrtf(nx) * __builtin_amdgcn_sqrtf(ny));
}

// Symmetric positive semidefinite eigensolver with vectors, one workgroup per
// matrix of order N <= 64: pivoted Cholesky factor A = L L^T (rows in place),
// then one-sided Jacobi on the columns of L (scaled by a power of two, see
// jac_tan).  Rotations from the right make the columns orthogonal, L W = X with
// X^T X diagonal, so A = X X^T: the eigenvalues are the squared
// column norms and the eigenvectors the normalised columns; no eigenvector
// block is carried along.  Both steps keep the small eigenvalues of a graded
// matrix D H D to the relative accuracy that the conditioning of H allows, as
// the Cholesky factor is formed entry by entry relative to its diagonal and a
// rotation is taken whenever |x_p . x_q| > eps ||x_p|| ||x_q||.  A pivot at
// or below its rounding level N eps a_kk is raised to it and its column of L
// cut below the diagonal (what stands there is rounding noise that a division
// by such a pivot would amplify), which leaves L regular and the eigenvectors
// a full orthonormal set whatever the rank of A.
//
// Why this shape: the solver is one dependent chain of rounds on one CU, so
// the time of a round is what counts.  The two-sided form it replaces kept A
// and V in LDS and moved about 4 matrices' worth of LDS traffic a round over
// two barriers of 16 waves (1.5 us a round in FP64, 0.8 us in FP32).  Here
// lane l of group g (8 lanes) holds rows l, l + 8, .. of the two columns of
// pair g in registers, one wave per SIMD; the dot product is RPL FMAs and
// three DPP steps, and only one column of every pair moves between rounds.
// The rounds follow the odd-even transposition ordering: columns sit at
// positions 0 .. NP - 1, odd steps rotate (2g, 2g + 1), even steps
// (2g + 1, 2g + 2), and both swap the two columns, so every pair meets once in
// NP steps.  Group g owns position 2g + 1; before an even step every group
// publishes the column at position 2g (buffer 1) and takes its right
// neighbour's, after it hands the one at 2g + 2 on (buffer 2).  Position 0
// waits in buffer 1 during even steps.  Each buffer is written again only
// after a barrier that follows its readers, so a step needs one barrier.
// The squared norms travel with the columns, updated by the rotation
// (n_p - t d, n_q + t d) and computed afresh at the start of every sweep.
//
// Bound: the dependent chain of one wave per SIMD (about 6 cycles an
// instruction): a rotation step (dot and DPP reduction, the angle's
// reciprocals and square roots, the rotation, LDS hand-over and barrier) takes
// 930 cycles in FP64 and 750 in FP32, a pivoted Cholesky step 1000 and 800, one
// on panels 500 and 400.  Measured in RoundSums (the two-sided form's average
// over both passes in brackets): three rank-48 blocks at n = 512, order 53, first
// pass (three Grams a launch) 189 us, second (one Gram) 74.5 us in FP64 (243);
// two such blocks in FP32 134 and 47 us (128); twelve solver iterations of that
// size 152 and 55 us (181); three rank-10 blocks, order 15, 33 and 20 us (54).
// A second-pass Gram that is diagonal to rounding takes 36 us at order 53.
template <typename T, int RPL, bool PIV>
__global__ __launch_bounds__(1024) void jacobi_osj_kernel(const EigTask<T>* __restrict__ tasks, int N) {
  constexpr int NT = 1024;
  constexpr int JW = 4;                               // waves of the factorisation and the rotations
  constexpr int NM = 8 * RPL;                         // row capacity (N <= NM)
  constexpr int LDX = (RPL & 1) ? NM : NM + 8;        // an odd multiple of 8: groups in distinct LDS banks
  constexpr int LDG = VEC_NMAX + 1;
  constexpr int NB = 2 * RPL;                         // Cholesky columns per wave
  __shared__ T G[VEC_NMAX * LDG];                     // the matrix: G[c * LDG + r], lower triangle
  __shared__ T X0[VEC_NMAX * LDX];                    // columns of L
  __shared__ T buf[2][VEC_NMAX / 2][LDX];             // columns on the move
  __shared__ T nbuf[2][VEC_NMAX / 2];                 // their squared norms
  __shared__ __align__(16) T colk[2][kWave];          // pivot column, by step parity
  __shared__ T lam_s[VEC_NMAX], lam_d[VEC_NMAX];
  __shared__ int bigflag[3];
  const EigTask<T> tk_ = tasks[blockIdx.x];
  if (task_skipped(tk_)) return;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int NP = N + (N & 1);
  const int H = NP / 2;
  // ---- load: the lower triangle, contiguous along its columns (column c
  // starts at entry c N - c (c - 1) / 2 of the packed triangle)
  for (int e = tid; e < N * (N + 1) / 2; e += NT) {
    const float h = float(N) + 0.5f;
    int c = int(h - __builtin_amdgcn_sqrtf(h * h - 2.0f * float(e)));
    while (c > 0 && c * N - c * (c - 1) / 2 > e) --c;
    while ((c + 1) * N - (c + 1) * c / 2 <= e) ++c;
    const int r = c + e - (c * N - c * (c - 1) / 2);
    const size_t at = r + (size_t)c * tk_.lda;
    T a = T(0);
    if (tk_.part) {  // the matrix's split-K partials, summed in split order
      // (sixteen loads in flight at a time; the additions keep their order)
      const GPtr<T> pp = (GPtr<T>)(tk_.part + at);
      for (int sp = 0; sp < tk_.splits; sp += 16) {
        T v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = pp[min(sp + u, tk_.splits - 1) * tk_.pstride];
#pragma unroll
        for (int u = 0; u < 16; ++u) a += sp + u < tk_.splits ? v[u] : T(0);
      }
    } else {
      a = ((GPtr<T>)tk_.A)[at];
    }
    G[c * LDG + r] = a;
  }
  for (int e = tid; e < NP * LDX; e += NT) X0[e] = T(0);
  if (tid < 3) bigflag[tid] = 0;
  __syncthreads();
  if (wave >= (PIV ? JW : kCholWaves)) return;  // a barrier waits for the waves that are left

  // ---- scale by a power of two so that the trace is in [1/2, 1)
  T tr = T(0);
  {
    const T dg = lane < N ? G[lane * LDG + lane] : T(0);
    tr = wave_sum(dg);
  }
  int ex = 0;
  if (tr > T(0) && tr < T(INFINITY)) (void)frexp(tr, &ex);
  // (applied to an entry as an exponent: the factor itself would overflow for a
  // trace below 2^-128 in FP32, 2^-1024 in FP64, or in the last binade)
  auto down = [&](T x) { return ldexp(x, -ex); };

  // ---- Cholesky.  A matrix of any rank in any order takes the largest remaining
  // diagonal as pivot (PIV), without which a rank-deficient one amplifies
  // rounding; one whose rows are sorted (the second pass of ST-HOSVD, sorted by
  // the first) keeps their order and runs on panels (chol_rows).  A remaining
  // diagonal at or below the rounding of its own start (N eps a_kk) is cut:
  // that pivot is the floor and the rest of its column zero.  So is one below
  // the least pivot, whose root the hardware does not form in FP32 (a denormal
  // gives infinity, and NaN after the correction).  A NaN pivot stays.
  auto cut = [](T pv, T fl) { return pv <= fl || pv < Lim<T>::pivot_tiny(); };
  if constexpr (!PIV) {
    __shared__ CholShared<T> chs;
    T a[kCholRows];
#pragma unroll
    for (int r = 0; r < kCholRows; ++r) {
      const int i = wave + kCholPanel * r;
      a[r] = i < N && lane >= i && lane < N ? down(G[i * LDG + lane]) : T(0);
    }
    const T floor_l = lane < N ? down(G[lane * LDG + lane]) * (T(N) * Lim<T>::eps()) : T(0);
    chol_rows(
        a, N, lane, wave, chs,
        [&](int k, T pv, T row, T& f) {
          f = cut(pv, rdlane(floor_l, k)) ? T(0) : row / pv;
          return true;
        },
        [&](int k, T row) {
          const T pv = rdlane(row, k), fl = rdlane(floor_l, k);
          const bool dead = cut(pv, fl);
          const T d = dead ? fmax(fl, Lim<T>::pivot_tiny()) : pv;
          const T r = rsq_full(d);
          const T x = dead ? T(0) : row * r;
          if (lane < NM) X0[k * LDX + lane] = lane == k ? d * r : lane > k && lane < N ? x : T(0);
        });
    if (wave >= JW) return;
  }
  // Pivoted (PIV): lane = row, wave w holds the columns w NB .. w NB + NB - 1 of the
  // remaining symmetric matrix in registers and every wave the remaining
  // diagonal.  The pivot column goes through LDS, one barrier a step; its
  // entries for a wave's columns are read across lanes (as LDS broadcasts
  // they took longer than the whole update).  Pivots are compared to 17 bits,
  // ties to the lowest row; all waves derive the same p.
  if constexpr (PIV) {
    typedef T Cols __attribute__((ext_vector_type(16)));
    static_assert(NB <= 16, "a wave's columns fit the vector");
    Cols a;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int j = wave * NB + b;
      const bool in = lane < N && j < N;
      const int hi = in ? (j > lane ? j : lane) : 0, lo = in ? (j > lane ? lane : j) : 0;
      const T v = G[lo * LDG + hi];
      a[b] = in ? down(v) : T(0);
    }
    T dg = lane < N ? down(G[lane * LDG + lane]) : T(0);
    const T floor_l = dg * (T(N) * Lim<T>::eps());
    bool alive = lane < N;
    // every lane prepares its own row as the next pivot: l_pp in dl, 1 / l_pp in
    // ri (zero where the rest of the column is cut)
    T dl = T(0), ri = T(0);
    auto prepare = [&]() {
      const bool dead = cut(dg, floor_l);
      const T pv = dead ? fmax(floor_l, Lim<T>::pivot_tiny()) : dg;
      const T r = rsq_full(pv);
      dl = pv * r;
      ri = dead ? T(0) : r;
    };
    int p = 0;
    auto choose = [&](int k) {  // the pivot of step k, its column published to the step's buffer
      const unsigned bits = __float_as_uint(fmaxf(float(dg), 0.0f));
      p = 63 - int(wave_umax(alive ? 0x80000000u | (bits & ~63u) | unsigned(63 - lane) : 0u) & 63u);
      const int b = p - wave * NB;
      if (b >= 0 && b < NB) colk[k & 1][lane] = a[b];
    };
    prepare();
    choose(0);
    for (int k = 0; k < N; ++k) {
      const T rp = rdlane(ri, p);
      const bool own = lane == p;
      alive = alive && !own;
      const T rc = alive ? rp : T(0);  // row of L below the pivot: c rc
      __syncthreads();
      const T c = colk[k & 1][lane];
      T cj[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) cj[b] = rdlane(c, wave * NB + b);
      // all reads before the first update: a read right before its use stalls
      __builtin_amdgcn_sched_barrier(0);
      const T x = c * rc;
      const T f = x * rp;
      const T lk = own ? dl : x;
      dg = fma(-x, x, dg);
#pragma unroll
      for (int b = 0; b < NB; ++b) a[b] = fma(-f, cj[b], a[b]);
      prepare();
      if (k + 1 < N) choose(k + 1);
      if (wave == (k & (JW - 1)) && lane < NM) X0[k * LDX + lane] = lk;
    }
  }
  __syncthreads();

  // ---- one-sided Jacobi
  const int g = tid >> 3, l = tid & 7;
  const bool act = g < H;
  const bool last = g == H - 1;
  const bool pair = g < H - 1;
  // the last group idles in even steps: its column A becomes the one at its
  // position (the exchange that B needs comes with the rotation)
  const T c_off = last ? T(0) : T(1), s_off = last ? T(1) : T(0);
  const int gn = pair ? g + 1 : 0, gs = act ? g : 0, g0 = g == 0 ? 0 : 1;
  T A[RPL], B[RPL];
  T nA = T(0), nB = T(0);
#pragma unroll
  for (int i = 0; i < RPL; ++i) {
    A[i] = act ? ldexp(X0[(2 * g) * LDX + l + 8 * i], kJacExp<T> / 2) : T(0);
    B[i] = act ? ldexp(X0[(2 * g + 1) * LDX + l + 8 * i], kJacExp<T> / 2) : T(0);
  }
  bool big = false;
  // rotates (x, y) to orthogonal columns; where nothing is to be done applies
  // (co, so): the identity, or the exchange (x, y) <- (-y, x)
  auto rotate = [&](T (&x)[RPL], T (&y)[RPL], T& nx, T& ny, bool on, T co, T so) {
    T d0 = x[0] * y[0], d1 = T(0);
#pragma unroll
    for (int i = 2; i < RPL; i += 2) d0 = fma(x[i], y[i], d0);
#pragma unroll
    for (int i = 1; i < RPL; i += 2) d1 = i == 1 ? x[i] * y[i] : fma(x[i], y[i], d1);
    const T d = group8_sum(d0 + d1);
    const bool flag = on && above_tol(d, nx, ny, Lim<T>::eps());
    big |= flag && above_tol(d, nx, ny, Lim<T>::stop());
    const T t = flag ? jac_tan(d, nx, ny) : T(0);
    const T cr = rsq_full(fma(t, t, T(1)));
    const T c = flag ? cr : co;
    const T s = flag ? t * cr : so;
    nx = fma(-t, d, nx);
    ny = fma(t, d, ny);
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const T xi = x[i], yi = y[i];
      x[i] = fma(-s, yi, c * xi);
      y[i] = fma(s, xi, c * yi);
    }
  };
  auto norm2 = [&](const T (&x)[RPL]) {
    T d0 = T(0), d1 = T(0);
#pragma unroll
    for (int i = 0; i < RPL; i += 2) d0 = fma(x[i], x[i], d0);
#pragma unroll
    for (int i = 1; i < RPL; i += 2) d1 = fma(x[i], x[i], d1);
    return group8_sum(d0 + d1);
  };
  for (int sweep = 0; sweep < 40; ++sweep) {
    big = false;
    if (tid == 0) bigflag[(sweep + 1) % 3] = 0;
    nA = norm2(A);
    nB = norm2(B);
    for (int ds = 0; ds < H; ++ds) {
      rotate(A, B, nA, nB, act, T(1), T(0));
      // swapped: B sits at position 2g, A at 2g + 1
      if (act) {
#pragma unroll
        for (int i = 0; i < RPL; ++i) buf[0][g][l + 8 * i] = B[i];
        if (l == 0) nbuf[0][g] = nB;
      }
      __syncthreads();
      // (a group without a right neighbour reads some column and leaves it alone)
#pragma unroll
      for (int i = 0; i < RPL; ++i) B[i] = buf[0][gn][l + 8 * i];
      nB = nbuf[0][gn];
      rotate(A, B, nA, nB, pair, c_off, s_off);
      // swapped: B sits at position 2g + 1, A at 2g + 2 (the last group keeps A)
      if (pair) {
#pragma unroll
        for (int i = 0; i < RPL; ++i) buf[1][g + 1][l + 8 * i] = A[i];
        if (l == 0) nbuf[1][g + 1] = nA;
      }
      nB = last ? nA : nB;
      if (ds == H - 1) {
        const bool wb = __any(big);
        if (lane == 0 && wb) bigflag[sweep % 3] = 1;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RPL; ++i) A[i] = buf[g0][gs][l + 8 * i];
      nA = nbuf[g0][gs];
    }
    // Read after the sweep's last barrier: the same values in every thread.
    // Stop after a sweep whose rotations all had scaled products
    // |x_p . x_q| / (||x_p|| ||x_q||) at or below sqrt(eps): cyclic Jacobi
    // converges quadratically, so another sweep would only confirm.
    if (bigflag[sweep % 3] == 0) break;
  }

  // ---- eigenvalues, sorted descending (stable by position), rank rule, output
  nA = norm2(A);
  nB = norm2(B);
  if (act && l == 0) {
    lam_s[2 * g] = nA;
    lam_s[2 * g + 1] = nB;
  }
  __syncthreads();
  // the padding column of an odd order has norm zero, below every other one
  int posA = 0, posB = 0;
  if (act) {
    // each of the 8 lanes counts every eighth column
    for (int j = l; j < NP; j += 8) {
      const T lj = lam_s[j];
      posA += (lj > nA) || (lj == nA && j < 2 * g);
      posB += (lj > nB) || (lj == nB && j < 2 * g + 1);
    }
    for (int m = 1; m < 8; m *= 2) {
      posA += __shfl_xor(posA, m, 8);
      posB += __shfl_xor(posB, m, 8);
    }
    if (l == 0) {
      lam_d[posA] = ldexp(nA, ex - kJacExp<T>);
      lam_d[posB] = ldexp(nB, ex - kJacExp<T>);
    }
  }
  __syncthreads();
  const EigRule& ru = tk_.rule;
  // every wave applies the rule to the spectrum in its lanes
  const T lam_l = lane < N ? lam_d[lane] : T(0);
  int rkeep = N;
  if (ru.kind != 0) {
    const int r = apply_rule<T>(ru, [&](int i) { return rdlane(lam_l, i); }, N);
    if (tid == 0) *ru.rank_out = r;
    if (ru.kind == 2) rkeep = r;
  }
  if (tk_.lam && wave == 0 && lane < N) tk_.lam[lane] = lam_l;
  if (tk_.V && act) {
    const T ia = rsq_full(nA), ib = rsq_full(nB);
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const int r = l + 8 * i;
      if (r < N) {
        if (posA < N) tk_.V[r + (size_t)posA * N] = posA < rkeep ? A[i] * ia : T(0);
        if (posB < N) tk_.V[r + (size_t)posB * N] = posB < rkeep ? B[i] * ib : T(0);
      }
    }
  }
}

// Rank certificate of the effective-rank rule, one workgroup per mode (the
// statement is next to its declaration): the Cholesky factorisation of
// H - theta I (chol_rows), which stops at the first failed pivot.
constexpr int CERT_NT = kCholWaves * kWave;
constexpr int CERT_MAX = 64;

// certificates tried and passed since the library was loaded (per device)
__device__ unsigned long long g_cert_count[2];

template <typename T>
__global__ __launch_bounds__(CERT_NT) void rank_cert_kernel(const T* __restrict__ H, const double* __restrict__ w,
                                                            const double* __restrict__ fro, int nb_act,
                                                            const double* __restrict__ tau_dev, CertParams cp,
                                                            int* __restrict__ cert, int* __restrict__ rt) {
  __shared__ CholShared<double> chs;
  __shared__ double red[kCholWaves];
  const int k = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int m = cp.cap;
  const int nb = min(cp.nb, nb_act);
  double part = 0.0;
  for (int b = tid; b < nb; b += CERT_NT) part += w[b] * w[b] * fro[(size_t)k * cp.nb + b];
  const double tr = block_sum(part, red);
  const double tau = *tau_dev;
  const double theta = (4.0 * fmax(cp.delta, tau * tau) + cp.rnd[k]) * tr;
  const T* Hk = H + (size_t)k * m * m;
  // row i from column i of the symmetric H: contiguous over the lanes
  double a[kCholRows];
#pragma unroll
  for (int r = 0; r < kCholRows; ++r) {
    const int i = wave + kCholPanel * r;
    a[r] = double(((GPtr<T>)Hk)[min(lane, m - 1) + (size_t)min(i, m - 1) * m]) - (i == lane ? theta : 0.0);
  }
  bool ok = tr > 0.0 && tr < INFINITY;  // the same in every thread
  if (ok)
    ok = chol_rows(
        a, m, lane, wave, chs,
        [](int, double pv, double row, double& f) {
          f = row / pv;
          return pv > 0.0 && pv < INFINITY;
        },
        [](int, double) {});
  if (tid == 0) {
    cert[k] = ok ? 1 : 0;
    if (ok)
      for (int i = 0; i < cp.d; ++i) rt[i] = cp.cap;
    atomicAdd(&g_cert_count[0], 1ull);
    if (ok) atomicAdd(&g_cert_count[1], 1ull);
  }
}

}  // namespace

template <typename T>
void jacobi_eig(const EigTask<T>* tasks_d, int ntasks, int N, bool want_v, hipStream_t st, int in_splits,
                bool sorted) {
  if (ntasks <= 0 || N <= 0) return;
  // algorithmic work of a symmetric eigendecomposition of order N: 9 N^3 with
  // eigenvectors (symmetric QR algorithm count), (4/3) N^3 for the tridiagonal
  // reduction behind the eigenvalues-only path.  Bytes: the lower triangle of
  // every input slab (the matrix, or each split-K partial that the load sums),
  // plus the eigenvalues and, with vectors, the N x N eigenvectors.
  const int kc = want_v ? kKcJacobi : kKcEigVals;
  const double nn = double(N);
  const double in_b = (want_v ? double(in_splits) * nn * (nn + 1.0) / 2.0 : nn * nn);
  timer_begin(kc, st, double(ntasks) * (want_v ? 9.0 : 4.0 / 3.0) * nn * nn * nn,
              double(ntasks) * sizeof(T) * (in_b + (want_v ? nn * nn : 0.0) + nn));
  if (want_v) {
    TK_CHECK(N <= VEC_NMAX, kErrUnsupported, "symmetric eigensolver: eigenvectors above size 64");
    // rows per lane: the least that covers the order
    switch (ceil_div(N, 8)) {
#define TK_OSJ_CASE(R)                                                                                      \
  case R:                                                                                                   \
    if (sorted)                                                                                             \
      hipLaunchKernelGGL((jacobi_osj_kernel<T, R, false>), dim3(ntasks), dim3(1024), 0, st, tasks_d, N);    \
    else                                                                                                    \
      hipLaunchKernelGGL((jacobi_osj_kernel<T, R, true>), dim3(ntasks), dim3(1024), 0, st, tasks_d, N);     \
    break;
      TK_OSJ_CASE(1)
      TK_OSJ_CASE(2)
      TK_OSJ_CASE(3)
      TK_OSJ_CASE(4)
      TK_OSJ_CASE(5)
      TK_OSJ_CASE(6)
      TK_OSJ_CASE(7)
      TK_OSJ_CASE(8)
#undef TK_OSJ_CASE
    }
  } else {
    TK_CHECK(N <= GM_NMAX, kErrUnsupported, "symmetric eigensolver: matrix larger than 512");
    if (N <= VAL_NMAX)
      hipLaunchKernelGGL((tridiag_reg_kernel<T>), dim3(ntasks), dim3(TRG_NT), 0, st, tasks_d, N);
    else
      hipLaunchKernelGGL((tridiag_gm_kernel<T>), dim3(ntasks), dim3(1024), 0, st, tasks_d, N);
    // (the planner gives the order-512 path matrices with a leading dimension
    // that is a multiple of 4, in 256-byte aligned workspace blocks)
  }
  TK_LAUNCH_CHECK();
  timer_end(kc, st);
}

template <typename T>
void rank_certificate(const T* H, const double* w, const double* fro, int nb_active, const double* tau,
                      const CertParams& cp, int* cert, int* rt, hipStream_t st) {
  TK_CHECK(cp.cap >= 1 && cp.cap <= CERT_MAX && cp.d >= 1 && cp.d <= kMaxD && cp.nb >= 1 && nb_active >= 0,
           kErrUnsupported, "rank certificate: sizes out of range");
  timer_begin(kKcEigVals, st);
  hipLaunchKernelGGL((rank_cert_kernel<T>), dim3(cp.d), dim3(CERT_NT), 0, st, H, w, fro, nb_active, tau, cp, cert,
                     rt);
  TK_LAUNCH_CHECK();
  timer_end(kKcEigVals, st);
}

void rank_cert_counts(int64_t* tried, int64_t* passed) {
  unsigned long long h[2] = {0, 0};
  TK_HIP(hipMemcpyFromSymbol(h, HIP_SYMBOL(g_cert_count), sizeof(h), 0, hipMemcpyDeviceToHost));
  *tried = int64_t(h[0]);
  *passed = int64_t(h[1]);
}

template void rank_certificate<double>(const double*, const double*, const double*, int, const double*,
                                       const CertParams&, int*, int*, hipStream_t);
template void rank_certificate<float>(const float*, const double*, const double*, int, const double*,
                                      const CertParams&, int*, int*, hipStream_t);

template void jacobi_eig<double>(const EigTask<double>*, int, int, bool, hipStream_t, int, bool);
template void jacobi_eig<float>(const EigTask<float>*, int, int, bool, hipStream_t, int, bool);

}  // namespace tk
